// pcg_sums.h -- the order in which a PCG solve's sums over a scene are formed,
// shared by the resident form (k_pcg_team.hip) and the launched form
// (k_solver.hip), so a solve gives the same bits in either.
//
// A scene is cut into team_T chunks: chunk c holds team_nt / 2 consecutive
// matrix rows, team_nt / 256 consecutive update units, and the contact rows
// whose first incidence entry lies in its 1/T of the entries (contact rows
// cluster in a few slices of the matrix; by entries they spread evenly). A
// chunk's partials are added in order, then one wavefront adds the chunks (lane l takes l, l + 64, ...) and its fixed tree
// ends the sum.
#pragma once
#include <type_traits>

#include "device_util.h"
#include "ipc_internal.h"

namespace ipcg {

// y += A v for one 3x3 block, a chain of fused multiply-adds (one rounding a
// term; half the instructions of separate products and sums, which set the
// SpMV's time once its values are in registers)
template <class R>
__device__ __forceinline__ void block_fma(const R (&A)[9], R v0, R v1, R v2, R &y0, R &y1, R &y2)
{
    auto f = [](R a, R b, R c) {
        if constexpr (sizeof(R) == 8)
            return __builtin_fma(a, b, c);
        else
            return __builtin_fmaf(a, b, c);
    };
    y0 = f(A[2], v2, f(A[1], v1, f(A[0], v0, y0)));
    y1 = f(A[5], v2, f(A[4], v1, f(A[3], v0, y1)));
    y2 = f(A[8], v2, f(A[7], v1, f(A[6], v0, y2)));
}

// d.q of 32 rows (a lane pair per row, the odd lanes zero) and of a block of
// 64: the halves added
__device__ __forceinline__ double half_wave_sum(double v)
{
    return lane_add<1>(lane_add<2>(lane_add<4>(lane_add<8>(lane_add<16>(v)))));
}

__device__ __forceinline__ double chunk_rz(const SceneDev &S, const double *slot, int c)
{
    const int U = S.team_nt / kBlock;
    double t = 0.0;
    for (int u = c * U; u < min((c + 1) * U, S.pcg_nvp); ++u) t += glob(slot)[u];
    return t;
}

__device__ __forceinline__ double chunk_dq(const SceneDev &S, bool contact, int c)
{
    const int RB = S.team_nt / (2 * kRowsPerBlock);
    double a = 0.0;
    for (int k = c * RB; k < min((c + 1) * RB, S.nb_rows); ++k) a += glob(S.pcg_part)[k];
    return contact ? a + glob(S.pcg_cpart)[c] : a;
}

// Contact rows of chunk c in ascending order, by a whole block of NT threads:
// list gets up to CAP of them from the skip-th on; returns the number left
// from there. cnt: LDS, one per wavefront.
struct CRow {
    int32_t row, base, n;  // vertex, first block (3 c_ptr[row]), blocks
};
template <int NT, int CAP>
__device__ __forceinline__ int chunk_contact_rows(const SceneDev &S, int c, int skip, CRow *list, int *cnt)
{
    const int tid = (int)threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int64_t E = glob(S.c_ptr)[S.n];
    const int t0 = (int)(E * c / S.team_T), t1 = (int)(E * (c + 1) / S.team_T);
    int n = -skip;
    for (int base = t0; base < t1; base += NT) {
        const int t = base + tid, v = t < t1 ? glob(S.c_row)[t] : -1;
        const bool head = v >= 0 && glob(S.c_ptr)[v] == t;
        const unsigned long long bal = __ballot(head);
        if (lane == 0) cnt[wave] = __popcll(bal);
        __syncthreads();
        int at = n;
        for (int k = 0; k < NT / kWave; ++k) {
            if (k < wave) at += cnt[k];
            n += cnt[k];
        }
        at += __popcll(bal & ((1ull << lane) - 1));
        if (head && at >= 0 && at < CAP) list[at] = CRow{v, 3 * t, glob(S.c_n)[v]};
        __syncthreads();
    }
    return n;
}

// Contact part of q for the listed rows, sum over a row's blocks j of
// C_j d(col_j), by a block of NT threads: a team of W lanes a row (kRowTeam,
// or a wavefront for rows of more than kRowLong blocks: a coarse indenter's
// vertex has hundreds), lane u adding blocks u, u + W, ... in order, then an
// xor tree. cv, cc: the blocks' values and columns; dir(v, d): the direction
// at a vertex; put(row, sums) on one lane of each row, the row's d . sums in
// dot[]. A lane's next column is read ahead of the current one's direction;
// col0: the first one of the first row it shares (contact_first), which a
// solve that keeps its rows reads once.
__device__ __forceinline__ int contact_first(gptr<const int32_t> cc, const CRow *list, int n, int tid)
{
    const int h = tid / kRowTeam, u = tid % kRowTeam;
    return h < n && u < list[h].n ? cc[list[h].base + u] : 0;
}
template <int NT, class R, class D, class P>
__device__ __forceinline__ void contact_rows(gptr<const R> cv, gptr<const int32_t> cc, const CRow *list, int n, int tid,
                                             int col0, D dir, P put, double *dot)
{
    auto pass = [&](auto team, bool longer) {  // a team of lanes per row
        constexpr int W = decltype(team)::value;
        const int u = tid % W;
        for (int h = tid / W; h < n; h += NT / W) {
            const CRow cr = list[h];
            if ((cr.n > kRowLong) != longer) continue;
            int col = !longer && h == tid / W ? col0 : (u < cr.n ? cc[cr.base + u] : 0);
            R own[3];
            dir(cr.row, own);
            double acc[3] = {0.0, 0.0, 0.0};
            for (int j = u; j < cr.n; j += W) {
                const auto from = cv + 9 * ((int64_t)cr.base + j);
                R A[9], d[3], y0 = R(0), y1 = R(0), y2 = R(0);
#pragma unroll
                for (int e = 0; e < 9; ++e) A[e] = from[e];
                dir(col, d);
                if (j + W < cr.n) col = cc[cr.base + j + W];
                block_fma(A, d[0], d[1], d[2], y0, y1, y2);
                acc[0] += (double)y0;
                acc[1] += (double)y1;
                acc[2] += (double)y2;
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                if constexpr (W == kWave) acc[c] = lane_add<16>(lane_add<32>(acc[c]));
                acc[c] = lane_add<1>(lane_add<2>(lane_add<4>(lane_add<8>(acc[c]))));
            }
            if (u == 0) {
                const R q[3] = {(R)acc[0], (R)acc[1], (R)acc[2]};
                put(cr.row, q);
                dot[h] = (double)own[0] * (double)q[0] + (double)own[1] * (double)q[1] + (double)own[2] * (double)q[2];
            }
        }
    };
    pass(std::integral_constant<int, kRowTeam>{}, false);
    pass(std::integral_constant<int, kWave>{}, true);
}
// and a lane's part of the dots' sum (rows lane, lane + 64, ... in order; one
// wavefront's parts are then added by its tree)
__device__ __forceinline__ void contact_dots(const double *dot, int n, double &t)
{
    for (int h = (int)(threadIdx.x & (kWave - 1)); h < n; h += kWave) t += dot[h];
}

// Coarse part of the multilevel preconditioner for one group, by the kBlock
// threads of its unit (t: thread of the unit). Between block barriers:
//   1. mas_restrict(level 0), all threads: each aggregate's sum of its
//      members' residuals rm, four lanes per aggregate and component (lane k
//      takes members k, k + 4, ... in order);
//   2. mas_restrict(coarser levels), one wavefront: the children's sums;
//   3. mas_correct, all threads: e = E^-1 r_agg per aggregate replaces rm;
//      returns the thread's sum of r_agg . e.
// base, na: the level's first aggregate in ra and their number; range(i, a):
// first and end of aggregate a's members (rows of rm) or children (of ra),
// packed in 16 bits each, for item i (the t / 4-th and on); inv(q, k): entry k of
// aggregate q's inverse.
template <class V, class RANGE>
__device__ __forceinline__ void mas_restrict(int base, int na, const V (*from)[3], double (*ra)[3], int t, int nt,
                                             RANGE range)
{
    const int sub = t % 4;
    for (int i = t / 4; i < 3 * na; i += nt / 4) {
        const int a = i / 3, c = i - 3 * a;
        const uint32_t rg = range(i, a);
        const int j0 = (int)(rg & 0xffffu) + sub, j1 = (int)(rg >> 16);
        double acc = 0.0;
        for (int j = j0; j < j1; j += 16) {  // four reads in flight
            V v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = from[min(j + 4 * k, j1 - 1)][c];
#pragma unroll
            for (int k = 0; k < 4; ++k) acc += j + 4 * k < j1 ? (double)v[k] : 0.0;
        }
        acc += quad_other<0xb1>(acc);  // lane ^ 1
        acc += quad_other<0x4e>(acc);  // lane ^ 2
        if (sub == 0) ra[base + a][c] = acc;
    }
}
template <class R, class INV>
__device__ __forceinline__ double mas_correct(int total, R (*rm)[3], const double (*ra)[3], int t, INV inv)
{
    double rz = 0.0;
    for (int i = t; i < 3 * total; i += kBlock) {
        const int q = i / 3, c = i - 3 * q;
        const R e = inv(q, 3 * c) * (R)ra[q][0] + inv(q, 3 * c + 1) * (R)ra[q][1] + inv(q, 3 * c + 2) * (R)ra[q][2];
        rm[q][c] = e;
        rz += ra[q][c] * (double)e;
    }
    return rz;
}
// orders a wavefront's LDS writes before its other lanes' reads
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// the sums over all chunks, by one wavefront (every lane gets them)
__device__ __forceinline__ double sum_rz(const SceneDev &S, const double *slot)
{
    double acc = 0.0;
    for (int c = (int)(threadIdx.x & (kWave - 1)); c < S.team_T; c += kWave) acc += chunk_rz(S, slot, c);
    return wave_sum(acc);
}
__device__ __forceinline__ double sum_dq(const SceneDev &S, bool contact)
{
    double acc = 0.0;
    for (int c = (int)(threadIdx.x & (kWave - 1)); c < S.team_T; c += kWave) acc += chunk_dq(S, contact, c);
    return wave_sum(acc);
}

// Scenes without a resident form (65,000 to 131,000 rows and more) have a
// thousand partials and more: one flat sum in two parts, the loads of a
// thread's first U partials issued ahead of other dependent loads. In the
// chunks' order such a scene's iteration took 6 to 11 % longer (128,000
// vertices FP64, 158,000 mixed).
template <int U>
__device__ __forceinline__ void flat_load(const double *part, int n, int t, int stride, double (&a)[U])
{
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = t + u * stride < n ? glob(part)[t + u * stride] : 0.0;
}
template <int U>
__device__ __forceinline__ double flat_sum(const double *part, int n, int t, int stride, const double (&a)[U])
{
    double acc = 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) acc += a[u];
    for (int base = t + U * stride; base < n; base += 4 * stride) {
        double b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) b[u] = base + u * stride < n ? glob(part)[base + u * stride] : 0.0;
#pragma unroll
        for (int u = 0; u < 4; ++u) acc += b[u];
    }
    return acc;
}

}  // namespace ipcg
