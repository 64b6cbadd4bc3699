// pcg_sums.h -- the order in which a PCG solve's sums over a scene are formed,
// shared by the resident form (k_pcg_team.hip) and the launched form
// (k_solver.hip), so a solve gives the same bits in either. (A scene that one
// workgroup holds has an order and a kernel of its own, k_pcg_solo.hip.)
//
// A scene is cut into team_T chunks: chunk c holds team_rows consecutive
// matrix rows, team_units consecutive update units, and the contact rows
// whose first incidence entry lies in its 1/T of the entries (contact rows
// cluster in a few slices of the matrix; by entries they spread evenly). A
// chunk's partials are added in order, then one wavefront adds the chunks (lane
// l takes l, l + 64, ...) and its fixed tree ends the sum.
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
    const int U = S.team_units;
    double t = 0.0;
    for (int u = c * U; u < min((c + 1) * U, S.pcg_nvp); ++u) t += glob(slot)[u];
    return t;
}

__device__ __forceinline__ double chunk_dq(const SceneDev &S, bool contact, int c)
{
    const int RB = S.team_rows / kRowsPerBlock;
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
// C_j d(col_j): kRowTeam blocks at a time (an item) summed by the xor tree of
// kRowTeam lanes, then the row's items in order.
//
// The merged blocks, their products and the sums are FP64 in either precision:
// a merged block is a sum over pairs, and rounded to FP32 it would lose what
// the pairs' separate products keep.
//
// contact_rows: rows h0, h0 + 1, ... by a block of NT threads, a team of
// kRowTeam lanes each, or a wavefront (four items at a time) for rows of more
// than kRowLong blocks: a coarse indenter's vertex has hundreds. cv, cc: the
// blocks' values and columns; dir.start(v) reads what dir.end(v, raw, d) turns into the direction
// at a vertex; put(row,
// sums) on one lane of each row, the row's d . sums in dot[].
template <class R>
__device__ __forceinline__ void contact_item(bool has, const double (&A)[9], const R (&d)[3], double (&t)[3])
{
    double y0 = 0.0, y1 = 0.0, y2 = 0.0;
    block_fma(A, (double)d[0], (double)d[1], (double)d[2], y0, y1, y2);
    t[0] = has ? y0 : 0.0;
    t[1] = has ? y1 : 0.0;
    t[2] = has ? y2 : 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) t[c] = lane_add<1>(lane_add<2>(lane_add<4>(lane_add<8>(t[c]))));
}
template <class R>
__device__ __forceinline__ double contact_dot(const R (&own)[3], const double (&q)[3])
{
    return (double)own[0] * q[0] + (double)own[1] * q[1] + (double)own[2] * q[2];
}
template <int NT, class R, class D, class P>
__device__ __forceinline__ void contact_rows(gptr<const double> cv, gptr<const int32_t> cc, const CRow *list, int h0, int n,
                                             int tid, D &dir, P put, double *dot)
{
    static_assert(kRowTeam == 16, "the items' tree");
    auto pass = [&](auto team, bool longer) {  // a team of lanes per row
        constexpr int W = decltype(team)::value;
        const int u = tid % W;
        for (int h = h0 + tid / W; h < n; h += NT / W) {
            const CRow cr = list[h];
            if ((cr.n > kRowLong) != longer) continue;
            int col = u < cr.n ? cc[cr.base + u] : cr.row;
            auto ro = dir.start(cr.row);
            R own[3];
            double acc[3] = {0.0, 0.0, 0.0};
            for (int j = u; j - u < cr.n; j += W) {
                const bool has = j < cr.n;
                const auto at = cv + 9 * ((int64_t)cr.base + (has ? j : 0));
                R d[3];
                double A[9], t[3];
#pragma unroll
                for (int e = 0; e < 9; ++e) A[e] = at[e];
                auto rc = dir.start(col);
                const int c0 = col;
                if (j + W < cr.n) col = cc[cr.base + j + W];
                dir.end(c0, rc, d);
                contact_item<R>(has, A, d, t);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    if constexpr (W == kWave) {  // the items that exist, in order
#pragma unroll
                        for (int i = 0; i < W / kRowTeam; ++i) {
                            const double v = __shfl(t[c], kRowTeam * i, kWave);
                            acc[c] = j - u + kRowTeam * i < cr.n ? acc[c] + v : acc[c];
                        }
                    } else {
                        acc[c] += t[c];
                    }
                }
            }
            if (u == 0) {
                dir.end(cr.row, ro, own);
                put(cr.row, acc);
                dot[h] = contact_dot(own, acc);
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
// threads of its unit (t: thread of the unit), between block barriers:
//   1. mas_restrict, all threads: each level-0 aggregate's sum of its members'
//      residuals rm, four lanes per aggregate and component;
//   2. mas_coarse: the first wavefront sums the level-1 aggregates and the
//      second the level-2 ones, both from level 0, and each forms e = E^-1
//      r_agg of its level; the other two form level 0's. e replaces rm;
//      returns the thread's sum of r_agg . e.
// A chain of LDS round trips bounds it, so the levels run beside each other:
// level by level over all threads it took 3,600 cycles of an iteration's
// 19,000 (1,442 vertices, FP64).
// na: aggregates per level, one level after the other in ra; range(l, a, first):
// first and end of level l's aggregate a, packed in 16 bits each (level 0: rows
// of rm, else level-0 aggregates; first: of the lane's first item); inv(q, k): entry k of aggregate q's inverse.
// The code is straight for the usual sizes (a group has 10 to 40 level-0
// aggregates of 8 to 27 members): a taken branch costs about as much as an LDS
// read, so later rounds stand behind conditions that are uniform.
//
// Lanes that share a sum, as a shift: of level 0, 1 and 2.
constexpr int kMasShare[kMasLevels] = {2, 2, 3};
template <int L, class V, class RANGE>
__device__ __forceinline__ void mas_sums(int na, const V (*from)[3], double (*to)[3], int t, int nt, RANGE range)
{
    constexpr int SH = kMasShare[L], W = 1 << SH;
    const int sub = t & (W - 1), step = nt >> SH;
    int i = t >> SH, base = 0;
#pragma clang loop unroll(disable)
    do {
        if (i < 3 * na) {
            const int a = i / 3, c = i - 3 * a;
            const uint32_t rg = range(L, a, base == 0);
            int j = (int)(rg & 0xffffu) + sub;
            const int j1 = (int)(rg >> 16);
            double acc = 0.0;
            auto four = [&]() {  // four reads in flight
                V v[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) v[k] = from[min(j + W * k, j1 - 1)][c];
#pragma unroll
                for (int k = 0; k < 4; ++k) acc += j + W * k < j1 ? (double)v[k] : 0.0;
            };
            four();
            if (__any(j + 4 * W < j1)) {
#pragma clang loop unroll(disable)
                for (j += 4 * W; __any(j < j1); j += 4 * W) four();
            }
            acc += quad_other<0xb1>(acc);                         // lane ^ 1
            acc += quad_other<0x4e>(acc);                         // lane ^ 2
            if constexpr (SH > 2) acc += quad_other<0x141>(acc);  // the half row mirrored: the other quad of eight lanes
            if (sub == 0) to[a][c] = acc;
        }
        i += step;
        base += step;
    } while (base < 3 * na);
}
template <class R, class RANGE>
__device__ __forceinline__ void mas_restrict(int na0, const R (*rm)[3], double (*ra)[3], int t, RANGE range)
{
    mas_sums<0>(na0, rm, ra, t, kBlock, range);
}
template <class R, class RANGE, class INV>
__device__ __forceinline__ double mas_coarse(int nl, int na0, int na1, int na2, R (*rm)[3], double (*ra)[3], int t,
                                             RANGE range, INV inv)
{
    const int lane = t % kWave, wave = __builtin_amdgcn_readfirstlane(t / kWave);
    double rz = 0.0;
    auto solve = [&](int q0, int na, int first, int step) {
        int i = first, base = 0;
#pragma clang loop unroll(disable)
        do {
            if (i < 3 * na) {
                const int a = i / 3, c = i - 3 * a, q = q0 + a;
                const R i0 = inv(q, 3 * c), i1 = inv(q, 3 * c + 1), i2 = inv(q, 3 * c + 2);
                const double r0 = ra[q][0], r1 = ra[q][1], r2 = ra[q][2];
                const R e = i0 * (R)r0 + i1 * (R)r1 + i2 * (R)r2;
                rm[q][c] = e;
                rz += (c == 0 ? r0 : c == 1 ? r1 : r2) * (double)e;
            }
            i += step;
            base += step;
        } while (base < 3 * na);
    };
    if (wave == 0) {
        if (nl > 1) {
            mas_sums<1>(na1, ra, ra + na0, lane, kWave, range);
            wave_lds_fence();
            solve(na0, na1, lane, kWave);
        }
    } else if (wave == 1) {
        if (nl > 2) {
            mas_sums<2>(na2, ra, ra + na0 + na1, lane, kWave, range);
            wave_lds_fence();
            solve(na0 + na1, na2, lane, kWave);
        }
    } else {
        solve(0, na0, t - 2 * kWave, 2 * kWave);
    }
    return rz;
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
