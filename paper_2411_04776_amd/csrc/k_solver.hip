// k_solver.hip -- the launched form of PCG, vector kernels and segmented scans,
// all over a list of scenes (one launch per phase for every scene in the list).
//
// PCG solves H p = -g from p = 0 and stops when the preconditioned residual
// r^T M^-1 r reaches pcg_tol^2 times its initial value. A scene whose
// workgroups fit the chip is solved in one launch (k_pcg_team.hip; k_pcg_solo.hip
// for the smallest). The form here is for the others, and for a solve whose
// team did not form. Each iteration is two kernels with every scalar kept on
// the device:
//   A(it): every wavefront of a scene reduces that scene's r.z partials of
//          the previous iteration in a fixed order (all agree bit for bit;
//          no block barrier before the real work) and decides the stop;
//          block 0 keeps r.z for the next launches; a row block then forms d = z + beta
//          d_prev for its rows and for the columns it gathers, applies the
//          elastic BELL matrix and the merged contact blocks, and writes its
//          d.q partial;
//   B(it): every wavefront reduces the scene's d.q partials, alpha = rz / dq,
//          then p += alpha d, r -= alpha q, z = M^-1 r and the r.z partials.
// The host launches chunks of iterations and reads the per-scene done flags
// once per chunk; finished scenes turn the remaining launches into no-ops.
#include <algorithm>

#include "device_util.h"
#include "ipc_internal.h"
#include "pcg_sums.h"

namespace ipcg {

template <class R>
__device__ __forceinline__ R *as(void *p)
{
    return reinterpret_cast<R *>(p);
}

// partial-sum layout in pcg_part: [d.q of the row blocks: nb_rows][r.z slot 0][r.z slot 1], an
// r.z slot holding the pcg_nvp update-block partials
__device__ __forceinline__ double *rz_slot(const SceneDev &S, int it)
{
    return S.pcg_part + S.nb_rows + (size_t)(it & 1) * (size_t)S.pcg_nvp;
}

// Partial product of one BELL row: stream `part` of the row's kSpmvStreams
// takes slots part, part + kSpmvStreams, ... The vector applied is
// z + beta d_prev (formed at the gathered column) when beta_on, else z.
template <class R>
__device__ __forceinline__ void bell_row_part(const SceneDev &S, int row, int part, const R *__restrict__ z,
                                              const R *__restrict__ dold, R beta, bool beta_on, double y[3])
{
    int sl = row / kSlice, lane = row % kSlice;
    int s0 = S.slice_ptr[sl], s1 = S.slice_ptr[sl + 1];
    const R *__restrict__ bval = as<R>(S.bval);
    const int32_t *__restrict__ bcol = S.bcol;
    R y0 = R(0), y1 = R(0), y2 = R(0);
#pragma unroll 2
    for (int slot = s0 + part; slot < s1; slot += kSpmvStreams) {
        int col = bcol[(int64_t)slot * kSlice + lane];
        if (col >= 0) {
            const R *from = bval + (int64_t)slot * 9 * kSlice + lane;
            R A[9];
#pragma unroll
            for (int e = 0; e < 9; ++e) A[e] = from[e * kSlice];
            R v0 = z[3 * col], v1 = z[3 * col + 1], v2 = z[3 * col + 2];
            if (beta_on) {
                v0 += beta * dold[3 * col];
                v1 += beta * dold[3 * col + 1];
                v2 += beta * dold[3 * col + 2];
            }
            block_fma(A, v0, v1, v2, y0, y1, y2);
        }
    }
    y[0] = y0;
    y[1] = y1;
    y[2] = y2;
}

// The same row with both vectors applied: yz = A z and yd = A d_prev (when
// two), so that nothing here waits for beta.
template <class R>
__device__ __forceinline__ void bell_row_part2(const SceneDev &S, int row, int part, const R *__restrict__ z,
                                               const R *__restrict__ dold, bool two, double yz[3], double yd[3])
{
    int sl = row / kSlice, lane = row % kSlice;
    int s0 = S.slice_ptr[sl], s1 = S.slice_ptr[sl + 1];
    const R *__restrict__ bval = as<R>(S.bval);
    const int32_t *__restrict__ bcol = S.bcol;
    R a0 = R(0), a1 = R(0), a2 = R(0), b0 = R(0), b1 = R(0), b2 = R(0);
#pragma unroll 2
    for (int slot = s0 + part; slot < s1; slot += kSpmvStreams) {
        int col = bcol[(int64_t)slot * kSlice + lane];
        if (col >= 0) {
            const R *A = bval + (int64_t)slot * 9 * kSlice + lane;
            R m[9];
#pragma unroll
            for (int k = 0; k < 9; ++k) m[k] = A[k * kSlice];
            R v0 = z[3 * col], v1 = z[3 * col + 1], v2 = z[3 * col + 2];
            block_fma(m, v0, v1, v2, a0, a1, a2);
            if (two) {
                R w0 = dold[3 * col], w1 = dold[3 * col + 1], w2 = dold[3 * col + 2];
                block_fma(m, w0, w1, w2, b0, b1, b2);
            }
        }
    }
    yz[0] = a0;
    yz[1] = a1;
    yz[2] = a2;
    yd[0] = b0;
    yd[1] = b1;
    yd[2] = b2;
}

// Both slot streams of one row by one thread, interleaved (two independent
// chains of loads in flight); each stream accumulates its slots in the same
// order and with the same expressions as bell_row_part2, so the partial sums
// are bit-identical to the two-lane form. Used for large lists, whose matrix
// exceeds the caches: its values are streamed with non-temporal loads so the
// gathered vectors keep the cache.
template <class R>
__device__ __forceinline__ void bell_row_both(const SceneDev &S, int row, const R *__restrict__ z,
                                              const R *__restrict__ dold, bool two, double yz[2][3], double yd[2][3])
{
    int sl = row / kSlice, lane = row % kSlice;
    int s0 = S.slice_ptr[sl], s1 = S.slice_ptr[sl + 1];
    const R *__restrict__ bval = as<R>(S.bval);
    const int32_t *__restrict__ bcol = S.bcol;
    R a[2][3] = {{R(0), R(0), R(0)}, {R(0), R(0), R(0)}}, c[2][3] = {{R(0), R(0), R(0)}, {R(0), R(0), R(0)}};
#pragma unroll 2
    for (int slot = s0; slot < s1; slot += 2) {
        int col[2];
        col[0] = bcol[(int64_t)slot * kSlice + lane];
        col[1] = slot + 1 < s1 ? bcol[(int64_t)(slot + 1) * kSlice + lane] : -1;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (col[k] < 0) continue;
            const R *A = bval + (int64_t)(slot + k) * 9 * kSlice + lane;
            R m[9];
#pragma unroll
            for (int e = 0; e < 9; ++e) m[e] = __builtin_nontemporal_load(A + e * kSlice);  // read once per launch
            R v0 = z[3 * col[k]], v1 = z[3 * col[k] + 1], v2 = z[3 * col[k] + 2];
            block_fma(m, v0, v1, v2, a[k][0], a[k][1], a[k][2]);
            if (two) {
                R w0 = dold[3 * col[k]], w1 = dold[3 * col[k] + 1], w2 = dold[3 * col[k] + 2];
                block_fma(m, w0, w1, w2, c[k][0], c[k][1], c[k][2]);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            yz[k][e] = a[k][e];
            yd[k][e] = c[k][e];
        }
}

// PCG A(it): every wavefront reduces the r.z partials, decides the stop and
// forms beta; a row block forms its rows' d = z + beta d_prev and q = K_el d,
// a chunk block the contact part of q for its chunk's contact rows; both
// write a d.q partial. A scene that also fits the
// resident form applies the matrix to d, as that form does; a larger one
// applies it to z and to d_prev before beta is known.
// LPR lanes per row (1: a thread runs both slot streams, for coalesced rows in
// large lists; 2: a lane per stream, for latency): the arithmetic is the same
// (streams added in order, each 32 rows' d.q summed by one fixed tree, the
// halves of a block added), so a scene gets the same bits in either form.
constexpr int kPassRows = 256;  // contact rows of a chunk handled at a time (a multiple of the wavefront)
template <class R, int LPR>
__global__ void __launch_bounds__(kRowsPerBlock * LPR) k_pcg_A(Launch L, int it, int early)
{
    constexpr int NP = kSpmvStreams / LPR;  // streams per thread
    __shared__ double sdq[2], cdot[kPassRows];
    __shared__ CRow clist[kPassRows];
    __shared__ int ccnt[kRowsPerBlock * LPR / kWave];
    int lb, s = scene_of_block(L, lb);
    const SceneDev &S = *L.sc[s];
    // launches past the expected count of this scene's solve: a finished solve costs nothing
    if ((early || it > L.out[s].pcg_early) && S.pcg->done) return;
    const R *z = as<R>(S.z);
    const R *dold = as<R>((it & 1) ? S.dB : S.dA);
    const bool bon = it > 1, on_d = S.team_fit != 0;
    const int t = (int)threadIdx.x, rloc = t / LPR, part0 = t % LPR;
    const int row = lb * kRowsPerBlock + rloc;
    const bool live = lb < S.nb_rows && row < S.n;
    double yz[NP][3], yd[NP][3];
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
        for (int c = 0; c < 3; ++c) yz[q][c] = yd[q][c] = 0.0;
    const int lane = t & (kWave - 1);
    double rzp[2];
    if (!on_d) flat_load<2>(rz_slot(S, it - 1), S.pcg_nvp, lane, kWave, rzp);
    if (live && !on_d) {
        if constexpr (NP == 2)
            bell_row_both<R>(S, row, z, dold, bon, yz, yd);
        else
            bell_row_part2<R>(S, row, part0, z, dold, bon, yz[0], yd[0]);
    }
    if (S.pcg->done) return;
    double beta = 0.0;
    const double rz_cur = on_d ? sum_rz(S, rz_slot(S, it - 1))
                               : wave_sum(flat_sum<2>(rz_slot(S, it - 1), S.pcg_nvp, lane, kWave, rzp));
    if (it == 1) {
        if (!(rz_cur > 0.0)) {
            if (lb == 0 && t == 0) {
                S.pcg->done = 1;
                S.pcg->iters = 0;
                L.out[s].pcg_done = 1;
                L.out[s].pcg_iters = 0;
            }
            return;
        }
        if (lb == 0 && t == 0) {
            S.pcg->stop = S.pcg_tol2 * rz_cur;
            S.pcg->rzv[1] = rz_cur;
        }
    } else {
        bool conv = rz_cur <= S.pcg->stop;
        if (conv || it > S.pcg_maxit) {  // converged, or the scene's iteration cap is spent
            if (lb == 0 && t == 0) {
                S.pcg->done = 1;
                S.pcg->iters = it - 1;
                L.out[s].pcg_done = conv ? 1 : 2;
                L.out[s].pcg_iters = it - 1;
                L.out[s].pcg_early = max(8, ((it - 1) * 7) / 8);  // for the next solve
            }
            return;
        }
        // r.z of iteration it - 2, kept by block 0 of the previous launch
        double rz_prev = S.pcg->rzv[(it - 1) & 1];
        beta = rz_cur / rz_prev;
        if (lb == 0 && t == 0) S.pcg->rzv[it & 1] = rz_cur;
    }
    const R rb = (R)beta;
    if (lb >= S.nb_rows) {  // the chunk's contact rows
        constexpr int NT = kRowsPerBlock * LPR;
        const int c = lb - S.nb_rows;
        struct Dir {  // d = z + beta d_prev
            const R *z, *dold;
            R rb;
            bool bon;
            struct Raw {
                R z[3], d[3];
            };
            __device__ __forceinline__ Raw start(int v) const
            {
                Raw x;
                for (int k = 0; k < 3; ++k) {
                    x.z[k] = glob(z)[3 * (int64_t)v + k];
                    x.d[k] = bon ? glob(dold)[3 * (int64_t)v + k] : R(0);
                }
                return x;
            }
            __device__ __forceinline__ void end(int, const Raw &x, R (&d)[3]) const
            {
                for (int k = 0; k < 3; ++k) d[k] = bon ? x.z[k] + rb * x.d[k] : x.z[k];
            }
        } dir{z, dold, rb, bon};
        auto put = [&](int v, const double (&y)[3]) {
            for (int k = 0; k < 3; ++k) S.c_q[4 * (int64_t)v + k] = y[k];
        };
        double t_dq = 0.0;
        for (int skip = 0;; skip += kPassRows) {
            const int n = chunk_contact_rows<NT, kPassRows>(S, c, skip, clist, ccnt), m = min(n, kPassRows);
            const auto cc = glob((const int32_t *)S.c_col);
            contact_rows<NT, R>(glob((const double *)S.c_val), cc, clist, 0, m, t, dir, put, cdot);
            __syncthreads();
            contact_dots(cdot, m, t_dq);
            if (n <= kPassRows) break;
            __syncthreads();
        }
        t_dq = wave_sum(t_dq);
        if (t == 0) S.pcg_cpart[c] = t_dq;
        return;
    }
    double dq = 0.0;
    R *dnew = as<R>((it & 1) ? S.dA : S.dB);
    R *q = as<R>(S.q);
    if (live && on_d) {
#pragma unroll
        for (int k = 0; k < NP; ++k) bell_row_part<R>(S, row, part0 + k, z, dold, rb, bon, yz[k]);
    }
    double y[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        y[c] = yz[0][c] + beta * yd[0][c];
#pragma unroll
        for (int k = 1; k < NP; ++k) y[c] += yz[k][c] + beta * yd[k][c];
        if (LPR == 2) y[c] += __shfl_xor(y[c], 1, kWave);
    }
    if (live && part0 == 0) {
        for (int c = 0; c < 3; ++c) {
            R dv = bon ? z[3 * row + c] + rb * dold[3 * row + c] : z[3 * row + c];
            R qv = (R)y[c];
            dnew[3 * row + c] = dv;
            q[3 * row + c] = qv;
            dq += (double)dv * (double)qv;
        }
    }
    if (LPR == 2) {
        dq = wave_sum(dq);  // 32 rows
        if (t % kWave == 0) sdq[t / kWave] = dq;
        __syncthreads();
        if (t == 0) S.pcg_part[lb] = sdq[0] + sdq[1];
    } else {
        dq = half_wave_sum(dq);
        dq += __shfl(dq, 32, kWave);
        if (t == 0) S.pcg_part[lb] = dq;
    }
}

// one vertex's state for the update, loaded before alpha is known (q: both
// its elastic and its contact part)
template <class R>
struct VertexPcg {
    R q[3], d[3], p[3], r[3], M[9];
};

template <class R>
__device__ __forceinline__ void pcg_vertex_load(const SceneDev &S, int i, const R *dcur, VertexPcg<R> &v)
{
    const auto q = glob(as<R>(S.q)), Mi = glob(as<R>(S.Minv)), sol = glob(as<R>(S.sol)), r = glob(as<R>(S.r));
    const auto dc = glob(dcur);
    for (int c = 0; c < 3; ++c) {
        v.q[c] = q[3 * i + c];
        v.d[c] = dc[3 * i + c];
        v.p[c] = sol[3 * i + c];
        v.r[c] = r[3 * i + c];
    }
    if (glob(S.c_ptr)[i + 1] > glob(S.c_ptr)[i])
        for (int c = 0; c < 3; ++c) v.q[c] = (R)((double)v.q[c] + glob(S.c_q)[4 * (int64_t)i + c]);
    for (int k = 0; k < 9; ++k) v.M[k] = Mi[9 * i + k];
}

// p += alpha d, r -= alpha q, z = M^-1 r; returns r.z
template <class R>
__device__ __forceinline__ double pcg_vertex_update(const SceneDev &S, int i, R alpha, const VertexPcg<R> &v)
{
    const auto sol = glob(as<R>(S.sol)), r = glob(as<R>(S.r)), z = glob(as<R>(S.z));
    R ri[3];
    for (int c = 0; c < 3; ++c) {
        sol[3 * i + c] = v.p[c] + alpha * v.d[c];
        ri[c] = v.r[c] - alpha * v.q[c];
        r[3 * i + c] = ri[c];
    }
    double rz = 0.0;
    for (int a = 0; a < 3; ++a) {
        R za = v.M[3 * a] * ri[0] + v.M[3 * a + 1] * ri[1] + v.M[3 * a + 2] * ri[2];
        z[3 * i + a] = za;
        rz += (double)ri[a] * (double)za;
    }
    return rz;
}

// ---- multilevel additive preconditioner ----------------------------------
// z = D^-1 r + sum over levels l of P_l E_l^-1 P_l^T r: D the 3x3 diagonal
// blocks, P_l the piecewise-constant injection of the level-l aggregates of
// free gel vertices, E_l = P_l^T A P_l (the assembled block matrix summed over
// each aggregate: the aggregate translating as a whole). Symmetric positive
// definite, so PCG keeps its guarantees. Aggregates nest and a group of
// top-level aggregates is one block, so restriction, the coarse solves and
// prolongation of a group happen in LDS with no grid-wide dependency; every
// sum runs in a fixed order.

// k_mas_diag: each aggregate's own entries (those first shared at its level):
// a wavefront per level-0 aggregate, a block per coarser aggregate
template <class R>
__global__ void __launch_bounds__(kBlock) k_mas_diag(Launch L)
{
    int lb, s = scene_of_block(L, lb);
    const SceneDev &S = *L.sc[s];
    int g, t0, dt;
    bool per_block = lb >= S.mas_nd0;
    if (!per_block) {
        g = lb * (kBlock / kWave) + (int)threadIdx.x / kWave;
        t0 = (int)threadIdx.x % kWave;
        dt = kWave;
        if (g >= S.mas_n[0]) return;  // whole wavefronts leave
    } else {
        g = S.mas_n[0] + (lb - S.mas_nd0);
        t0 = (int)threadIdx.x;
        dt = (int)blockDim.x;
    }
    const R *bval = as<R>(S.bval);
    double A[9];
#pragma unroll
    for (int c = 0; c < 9; ++c) A[c] = 0.0;
    for (int t = S.mas_dptr[g] + t0; t < S.mas_dptr[g + 1]; t += dt) {
        int64_t e = S.mas_dsrc[t];
        int64_t slot = e / kSlice, lane = e % kSlice;
#pragma unroll
        for (int c = 0; c < 9; ++c) A[c] += (double)bval[(slot * 9 + c) * kSlice + lane];
    }
    if (per_block)
        block_sum_vec<9>(A);
    else
#pragma unroll
        for (int c = 0; c < 9; ++c) A[c] = wave_sum(A[c]);
    if (t0 == 0)
#pragma unroll
        for (int c = 0; c < 9; ++c) S.mas_ex[9 * (int64_t)g + c] = A[c];
}

// group's level-l aggregate range [a0, a1) (level-local ids); l = -1: members
__device__ __forceinline__ void mas_group_range(const SceneDev &S, int grp, int l, int &a0, int &a1)
{
    const auto row = glob(S.mas_gofs) + (size_t)(l + 1) * (S.mas_ng + 1);
    a0 = row[grp];
    a1 = row[grp + 1];
}

// k_mas_invert: per group, level by level, E(g) = own entries + the children's
// blocks (in child order), then its inverse
template <class R>
__global__ void __launch_bounds__(kBlock) k_mas_invert(Launch L)
{
    int grp, s = scene_of_block(L, grp);
    const SceneDev &S = *L.sc[s];
    R *Di = as<R>(S.mas_dinv);
    for (int l = 0; l < S.mas_levels; ++l) {
        int a0, a1;
        mas_group_range(S, grp, l, a0, a1);
        for (int a = a0 + (int)threadIdx.x; a < a1; a += blockDim.x) {
            int64_t g = S.mas_off[l] + a;
            double E[9];
#pragma unroll
            for (int c = 0; c < 9; ++c) E[c] = S.mas_ex[9 * g + c];
            if (l > 0)
                for (int ch = S.mas_mb[g]; ch < S.mas_me[g]; ++ch) {
                    int64_t gc = S.mas_off[l - 1] + ch;
#pragma unroll
                    for (int c = 0; c < 9; ++c) E[c] += S.mas_ex[9 * gc + c];
                }
            if (l + 1 < S.mas_levels)  // the parent level reads the whole block
#pragma unroll
                for (int c = 0; c < 9; ++c) S.mas_ex[9 * g + c] = E[c];
            double Inv[9];
            inverse3(E, Inv);
#pragma unroll
            for (int c = 0; c < 9; ++c) Di[9 * g + c] = (R)Inv[c];
        }
        __syncthreads();  // the next level reads these blocks
    }
}

// ---- PCG B(it) --------------------------------------------------------------
// Blocks of a scene: [preconditioner groups | vertex blocks]. With the
// multilevel preconditioner the vertex blocks cover
// the vertices outside the aggregates; without it, every vertex. Every block
// loads its vertices' data and contact sums first, then alpha from the d.q
// partials, then p += alpha d, r -= alpha q, z = D^-1 r (plus, in a group,
// the aggregate corrections) and its r.z partial. B(0) starts the solve
// from p = 0, r = -g instead.

// alpha = r.z / d.q of iteration it, d.q from the A launch's partials; every
// wavefront forms the same value
// in a scene without a resident form the whole block sums them, its first
// loads (pcg_alpha_load) issued before the vertices' data
template <class R>
__device__ __forceinline__ R pcg_alpha(const SceneDev &S, bool contact, int it, const double (&a)[4])
{
    double dq;
    if (S.team_fit) {
        dq = sum_dq(S, contact);
    } else {
        const int t = (int)threadIdx.x;
        dq = flat_sum<4>(S.pcg_part, S.nb_rows, t, kBlock, a);
        if (contact)
            for (int c = t; c < S.team_T; c += kBlock) dq += glob(S.pcg_cpart)[c];
        dq = block_sum_all(dq);
    }
    return (R)(glob(S.pcg)->rzv[it & 1] / dq);
}
__device__ __forceinline__ void pcg_alpha_load(const SceneDev &S, double (&a)[4])
{
    if (!S.team_fit) flat_load<4>(S.pcg_part, S.nb_rows, (int)threadIdx.x, kBlock, a);
}

// start of the solve for vertex i: r = -g, p = 0, z = D^-1 r; returns r.z
template <class R>
__device__ __forceinline__ double pcg_vertex_start(const SceneDev &S, int i, R zo[3], R ri[3])
{
    R *r = as<R>(S.r), *sol = as<R>(S.sol);
    const R *g = as<R>(S.grad), *Mi = as<R>(S.Minv);
    for (int c = 0; c < 3; ++c) ri[c] = -g[3 * i + c];
    double rz = 0.0;
    for (int a = 0; a < 3; ++a) {
        zo[a] = Mi[9 * i + 3 * a] * ri[0] + Mi[9 * i + 3 * a + 1] * ri[1] + Mi[9 * i + 3 * a + 2] * ri[2];
        rz += (double)ri[a] * (double)zo[a];
    }
    for (int c = 0; c < 3; ++c) {
        r[3 * i + c] = ri[c];
        sol[3 * i + c] = R(0);
    }
    return rz;
}

// LDS of an update block: the group's members' r, then the corrections, the
// aggregate sums, and the group's level ranges (block-uniform)
template <class R>
struct BShared {
    R rm[kMasCapM][3];
    double ra[kMasCapA][3];
    int32_t lv[kMasLevels][2];  // LDS base and number of the level's aggregates
    int32_t first[kMasLevels];  // and the first one's id in its level
};

template <class R>
__device__ void pcg_B_vertices(const Launch &L, const SceneDev &S, int s, int vb, int it, int lb, BShared<R> &sh)
{
    int k = vb * blockDim.x + threadIdx.x;
    int i = S.mas_levels > 0 ? (k < S.mas_nother ? S.mas_other[k] : -1) : (k < S.n ? k : -1);
    double rz = 0.0;
    if (it == 0) {
        if (i >= 0) {
            R zo[3], ri[3];
            rz = pcg_vertex_start<R>(S, i, zo, ri);
            R *z = as<R>(S.z);
            for (int c = 0; c < 3; ++c) z[3 * i + c] = zo[c];
        }
    } else {
        const R *dcur = as<R>((it & 1) ? S.dA : S.dB);
        const int done = glob(S.pcg)->done;
        const bool own = i >= 0;
        double dqa[4];
        pcg_alpha_load(S, dqa);
        VertexPcg<R> v;
        if (own) pcg_vertex_load<R>(S, i, dcur, v);
        if (done) return;
        const R alpha = pcg_alpha<R>(S, L.out[s].n_crow > 0, it, dqa);
        if (own) rz = pcg_vertex_update<R>(S, i, alpha, v);
    }
    rz = block_sum_all(rz);
    if (threadIdx.x == 0) glob(rz_slot(S, it))[lb] = rz;
}

// a[l] of a per-level register array at a run-time level: selects, so the
// array stays in registers (dynamic indexing would move it to scratch)
__device__ __forceinline__ int lvl(const int (&a)[kMasLevels], int l)
{
    static_assert(kMasLevels == 3, "lvl selects among three levels");
    return l == 0 ? a[0] : (l == 1 ? a[1] : a[2]);
}

static_assert(kMasCapA <= kMasCapM, "corrections reuse the members' LDS rows");
static_assert(kMasCapM % kBlock == 0, "members per thread");
constexpr int kMasSlots = kMasCapM / kBlock;  // members per thread of a group block

// One group: the members' update, then restriction of the new r to every
// aggregate (members, then children, in order), e = E^-1 r_agg per aggregate,
// and z = D^-1 r + the corrections of the member's aggregates. The r.z
// partial is r.D^-1 r + sum over the group's aggregates of r_agg.e. The
// members' index data is loaded at the start, beside their vertex data; the
// aggregates' member ranges and inverses where they are used.
template <class R>
__device__ void pcg_B_group(const Launch &L, const SceneDev &S, int s, int grp, int it, BShared<R> &sh)
{
    const int nl = S.mas_levels;
    const int tid = (int)threadIdx.x;
    int k0, k1;
    mas_group_range(S, grp, -1, k0, k1);
    // level ranges and LDS bases (each aggregate's member range is read in
    // the level loop: loaded up front, the ranges held enough registers to
    // cost a wavefront per SIMD)
    int ga0[kMasLevels], ga1[kMasLevels], gbase[kMasLevels];
    const R *Di = as<R>(S.mas_dinv);
    {
        int bsum = 0;
#pragma unroll
        for (int l = 0; l < kMasLevels; ++l) {
            int a0 = 0, a1 = 0;
            if (l < nl) mas_group_range(S, grp, l, a0, a1);
            ga0[l] = a0;
            ga1[l] = a1;
            gbase[l] = bsum;
            bsum += a1 - a0;
        }
    }
    if (tid < kMasLevels) {  // read back block-uniform
        sh.lv[tid][0] = lvl(gbase, tid);
        sh.lv[tid][1] = lvl(ga1, tid) - lvl(ga0, tid);
        sh.first[tid] = lvl(ga0, tid);
    }
    int vid[kMasSlots], loc[kMasSlots][kMasLevels];
    R zo[kMasSlots][3];
    double rz = 0.0;
#pragma unroll
    for (int j = 0; j < kMasSlots; ++j) {
        int k = k0 + tid + j * kBlock;
        vid[j] = k < k1 ? glob(S.mas_mem)[k] : -1;
#pragma unroll
        for (int l = 0; l < kMasLevels; ++l)
            loc[j][l] = (vid[j] >= 0 && l < nl) ? gbase[l] + glob(S.mas_manc)[(int64_t)l * S.mas_nf + k] - ga0[l] : 0;
    }
    if (it == 0) {
#pragma unroll
        for (int j = 0; j < kMasSlots; ++j)
            if (vid[j] >= 0) {
                R ri[3];
                rz += pcg_vertex_start<R>(S, vid[j], zo[j], ri);
                for (int c = 0; c < 3; ++c) sh.rm[tid + j * kBlock][c] = ri[c];
            }
    } else {
        const int done = glob(S.pcg)->done;
        const R *dcur = as<R>((it & 1) ? S.dA : S.dB);
        double dqa[4];
        pcg_alpha_load(S, dqa);
        VertexPcg<R> v[kMasSlots];
#pragma unroll
        for (int j = 0; j < kMasSlots; ++j)
            if (vid[j] >= 0) pcg_vertex_load<R>(S, vid[j], dcur, v[j]);
        if (done) return;
        const R alpha = pcg_alpha<R>(S, L.out[s].n_crow > 0, it, dqa);
        const auto sol = glob(as<R>(S.sol)), r = glob(as<R>(S.r));
#pragma unroll
        for (int j = 0; j < kMasSlots; ++j) {
            if (vid[j] < 0) continue;
            int i = vid[j], pos = tid + j * kBlock;
            R ri[3];
            for (int c = 0; c < 3; ++c) {
                sol[3 * i + c] = v[j].p[c] + alpha * v[j].d[c];
                ri[c] = v[j].r[c] - alpha * v[j].q[c];
                r[3 * i + c] = ri[c];
            }
            for (int a = 0; a < 3; ++a) {
                zo[j][a] = v[j].M[3 * a] * ri[0] + v[j].M[3 * a + 1] * ri[1] + v[j].M[3 * a + 2] * ri[2];
                rz += (double)ri[a] * (double)zo[j][a];
            }
            for (int c = 0; c < 3; ++c) sh.rm[pos][c] = ri[c];
        }
    }
    __syncthreads();
    const int na0 = sh.lv[0][1], na1 = nl > 1 ? sh.lv[1][1] : 0, na2 = nl > 2 ? sh.lv[2][1] : 0;
    auto range = [&](int l, int a, bool) {
        const auto mb = glob(S.mas_mb), me = glob(S.mas_me);
        const int64_t g = (int64_t)S.mas_off[l] + sh.first[l] + a;
        int b = mb[g], e = me[g], off = l == 0 ? k0 : sh.first[0];
        if (l == 2) {  // children of level 1: the first one's first child and the last one's end
            b = mb[S.mas_off[1] + b];
            e = me[S.mas_off[1] + e - 1];
        }
        return (uint32_t)(b - off) | (uint32_t)(e - off) << 16;
    };
    mas_restrict<R>(na0, sh.rm, sh.ra, tid, range);
    __syncthreads();
    rz += mas_coarse<R>(nl, na0, na1, na2, sh.rm, sh.ra, tid, range, [&](int q, int k) {
        const int l = q >= na0 + na1 ? 2 : (q >= na0 ? 1 : 0);
        return glob(Di)[9 * ((int64_t)S.mas_off[l] + sh.first[l] + q - sh.lv[l][0]) + k];
    });
    __syncthreads();
    // prolongation: z = D^-1 r + the corrections of the member's aggregates
    const auto z = glob(as<R>(S.z));
#pragma unroll
    for (int j = 0; j < kMasSlots; ++j) {
        if (vid[j] < 0) continue;
        double zi[3] = {(double)zo[j][0], (double)zo[j][1], (double)zo[j][2]};
#pragma unroll
        for (int l = 0; l < kMasLevels; ++l) {
            if (l >= nl) break;
#pragma unroll
            for (int c = 0; c < 3; ++c) zi[c] += (double)sh.rm[loc[j][l]][c];
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) z[3 * vid[j] + c] = (R)zi[c];
    }
    rz = block_sum_all(rz);
    if (tid == 0) glob(rz_slot(S, it))[grp] = rz;
}

template <class R>
__global__ void __launch_bounds__(kBlock) k_pcg_B(Launch L, int it, int early)
{
    int lb, s = scene_of_block(L, lb);
    const SceneDev &S = *L.sc[s];
    if ((early || it > L.out[s].pcg_early) && it > 0 && S.pcg->done) return;
    if (it == 0 && lb == 0 && threadIdx.x == 0) {  // a new solve
        S.pcg->done = 0;
        S.pcg->iters = 0;
        S.pcg->stop = 0.0;
        L.out[s].pcg_done = 0;
        L.out[s].pcg_iters = 0;
    }
    __shared__ BShared<R> sh;
    const int ngrp = S.mas_levels > 0 ? S.mas_ng : 0;
    if (lb < ngrp)
        pcg_B_group<R>(L, S, s, lb, it, sh);
    else
        pcg_B_vertices<R>(L, S, s, lb - ngrp, it, lb, sh);
}

// y = H v for the test hook (v in S.dB, y in S.q): a thread per row, both slot
// streams, then the row's contact blocks
template <class R>
__global__ void __launch_bounds__(kBlock) k_spmv_rows(Launch L)
{
    int lb, s = scene_of_block(L, lb);
    const SceneDev &S = *L.sc[s];
    const R *v = as<R>(S.dB);
    R *y = as<R>(S.q);
    int row = lb * kRowsPerBlock + (int)threadIdx.x;
    if (row >= S.n) return;
    double o[3] = {0.0, 0.0, 0.0}, o1[3];
    bell_row_part<R>(S, row, 0, v, nullptr, R(0), false, o);
    bell_row_part<R>(S, row, 1, v, nullptr, R(0), false, o1);
    for (int c = 0; c < 3; ++c) o[c] += o1[c];
    if (S.c_ptr[row + 1] > S.c_ptr[row]) {
        const int64_t base = 3 * (int64_t)S.c_ptr[row];
        for (int j = 0; j < S.c_n[row]; ++j) {
            const double *h = S.c_val + 9 * (base + j);
            const R *d = v + 3 * (int64_t)S.c_col[base + j];
            for (int i = 0; i < 3; ++i) o[i] += h[3 * i] * (double)d[0] + h[3 * i + 1] * (double)d[1] + h[3 * i + 2] * (double)d[2];
        }
    }
    for (int c = 0; c < 3; ++c) y[3 * row + c] = (R)o[c];
}

// ---- per-vertex kernels ------------------------------------------------------

template <class R>
__global__ void k_pinf(Launch L)
{
    int lb, s = scene_of_block(L, lb);
    const SceneDev &S = *L.sc[s];
    const R *p = as<R>(S.sol);
    int i = lb * blockDim.x + threadIdx.x;
    double v = 0.0;
    if (i < S.n && !S.fixed[i])
        v = fmax(fabs((double)p[3 * i]), fmax(fabs((double)p[3 * i + 1]), fabs((double)p[3 * i + 2])));
    v = block_max_all(v);
    if (threadIdx.x == 0) S.red[lb] = v;
}

// one block per scene: max over the producer's per-block partials
__global__ void k_final_pinf(Launch one, Launch prod)
{
    int lb, s = scene_of_block(one, lb);
    const SceneDev &S = *one.sc[s];
    int nb = blocks_of(prod, s);
    double v = 0.0;
    for (int i = threadIdx.x; i < nb; i += blockDim.x) v = fmax(v, S.red[i]);
    v = block_max_all(v);
    if (threadIdx.x == 0) one.out[s].pinf = v;
}

// x_trial = x + alpha p (one rounding per component, as the line search
// defines it); alpha per scene
template <class R>
__global__ void k_trial(Launch L, const double *__restrict__ alpha)
{
    int lb, s = scene_of_block(L, lb);
    const SceneDev &S = *L.sc[s];
    const R *p = as<R>(S.sol);
    int i = lb * blockDim.x + threadIdx.x;
    if (i >= S.n) return;
    double a = alpha[s];
    for (int c = 0; c < 3; ++c) S.xtrial[3 * i + c] = __dadd_rn(S.x[3 * i + c], __dmul_rn(a, (double)p[3 * i + c]));
}

__global__ void k_accept(Launch L)
{
    int lb, s = scene_of_block(L, lb);
    const SceneDev &S = *L.sc[s];
    int i = lb * blockDim.x + threadIdx.x;
    if (i >= S.n) return;
    for (int c = 0; c < 3; ++c) S.x[3 * i + c] = S.xtrial[3 * i + c];
}

// scene views put in place: block j copies view j of the staged block into
// the slot its pointer names, in 8-byte words
static_assert(sizeof(SceneDev) % 8 == 0, "views are copied in 8-byte words");
constexpr int kViewWords = (int)(sizeof(SceneDev) / 8);
__global__ void __launch_bounds__(kBlock) k_put_views(int n, const uint64_t *__restrict__ src)
{
    const int j = (int)blockIdx.x;
    uint64_t *dst = reinterpret_cast<uint64_t *>(src[j]);
    const uint64_t *from = src + view_head_bytes(n) / 8 + (int64_t)j * kViewWords;
    for (int w = (int)threadIdx.x; w < kViewWords; w += (int)blockDim.x) dst[w] = from[w];
}

// step start: keep x^t, inertial predictor for free gel vertices, indenter
// targets from the scene's pose, attached gel vertices' targets from the case
// pose
__global__ void k_begin_step(Launch L)
{
    int lb, s = scene_of_block(L, lb);
    const SceneDev &S = *L.sc[s];
    int i = lb * blockDim.x + threadIdx.x;
    if (i >= S.n) return;
    double h = S.h;
    for (int c = 0; c < 3; ++c) S.xt[3 * i + c] = S.x[3 * i + c];
    if (i < S.n_gel) {
        for (int c = 0; c < 3; ++c) {
            double xv = S.x[3 * i + c];
            S.xtilde[3 * i + c] = S.fixed[i] ? xv : xv + h * S.v[3 * i + c] + h * h * S.grav[c];
            S.yhat[3 * i + c] = xv;
        }
        if (S.attached && S.attached[i]) {  // the case pose applied to the rest position
            const double *X = S.X0 + 3 * i, *P = S.case_pose;
            for (int c = 0; c < 3; ++c)
                S.yhat[3 * i + c] = P[c * 4 + 0] * X[0] + P[c * 4 + 1] * X[1] + P[c * 4 + 2] * X[2] + P[c * 4 + 3];
        }
    } else {
        const double *y = S.Yloc + 3 * (i - S.n_gel);
        const double *P = S.pose;
        for (int c = 0; c < 3; ++c) {
            S.yhat[3 * i + c] = P[c * 4 + 0] * y[0] + P[c * 4 + 1] * y[1] + P[c * 4 + 2] * y[2] + P[c * 4 + 3];
            S.xtilde[3 * i + c] = S.x[3 * i + c];
            if (S.target_al) S.al_lam[3 * i + c] = 0.0;
        }
    }
}

// augmented-Lagrangian targets: lambda_j -= k_t (y_j - yhat_j) for the
// indenter vertices of the scenes in the launch
__global__ void k_al_update(Launch L)
{
    int lb, s = scene_of_block(L, lb);
    const SceneDev &S = *L.sc[s];
    int i = S.n_gel + lb * blockDim.x + threadIdx.x;
    if (i >= S.n) return;
    for (int c = 0; c < 3; ++c) S.al_lam[3 * i + c] -= S.k_target * (S.x[3 * i + c] - S.yhat[3 * i + c]);
}

__global__ void k_end_step(Launch L)
{
    int lb, s = scene_of_block(L, lb);
    const SceneDev &S = *L.sc[s];
    int i = lb * blockDim.x + threadIdx.x;
    if (i >= S.n) return;
    double inv_h = 1.0 / S.h;
    for (int c = 0; c < 3; ++c) S.v[3 * i + c] = (S.x[3 * i + c] - S.xt[3 * i + c]) * inv_h;
}

// max target lag over indenter vertices and per-block sums of gel positions
__global__ void k_lag_mean(Launch L)
{
    int lb, s = scene_of_block(L, lb);
    const SceneDev &S = *L.sc[s];
    int i = lb * blockDim.x + threadIdx.x;
    double lag = 0.0, m[3] = {0.0, 0.0, 0.0};
    if (i < S.n) {
        if (i >= S.n_gel) {
            double d0 = S.x[3 * i] - S.yhat[3 * i], d1 = S.x[3 * i + 1] - S.yhat[3 * i + 1],
                   d2 = S.x[3 * i + 2] - S.yhat[3 * i + 2];
            lag = sqrt(d0 * d0 + d1 * d1 + d2 * d2);
        } else {
            for (int c = 0; c < 3; ++c) m[c] = S.x[3 * i + c];
        }
    }
    lag = block_max_all(lag);
    for (int c = 0; c < 3; ++c) m[c] = block_sum_all(m[c]);
    if (threadIdx.x == 0) {
        S.red[4 * lb] = lag;
        for (int c = 0; c < 3; ++c) S.red[4 * lb + 1 + c] = m[c];
    }
}

__global__ void k_final_lag_mean(Launch one, Launch prod)
{
    int lb, s = scene_of_block(one, lb);
    const SceneDev &S = *one.sc[s];
    int nb = blocks_of(prod, s);
    double lag = 0.0, m[3] = {0.0, 0.0, 0.0};
    for (int i = threadIdx.x; i < nb; i += blockDim.x) {
        lag = fmax(lag, S.red[4 * i]);
        for (int c = 0; c < 3; ++c) m[c] += S.red[4 * i + 1 + c];
    }
    lag = block_max_all(lag);
    for (int c = 0; c < 3; ++c) m[c] = block_sum_all(m[c]);
    if (threadIdx.x == 0) {
        one.out[s].lag = lag;
        for (int c = 0; c < 3; ++c) one.out[s].obj[c] = m[c] / (double)S.n_gel;
    }
}

__global__ void k_gather_surface(int ns, const int32_t *__restrict__ ids, const double *__restrict__ x,
                                 double *__restrict__ out)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ns) return;
    int v = ids[i];
    out[3 * i] = x[3 * v];
    out[3 * i + 1] = x[3 * v + 1];
    out[3 * i + 2] = x[3 * v + 2];
}

// ---- segmented exclusive scan of per-scene int32 arrays ------------------------
// An array of up to kScanOne values takes one block and one launch (k_scan_one:
// 32 consecutive values a thread). A longer one is cut into tiles of kScanTile
// values (its own block range); per-tile sums are scanned by one block per
// scene; then each tile writes its exclusive prefix. out[len] and the scene's
// read-back slot get the total. Counts that a second pass counts again (hash
// buckets, contact entries) are cleared once they are read. A Newton iteration
// of a small gel made 18 launches of 2 to 3 us for its scans and 2 to clear,
// now 5.

struct ScanSel {
    const int32_t *in;
    int32_t *out;
    int64_t len;
};

__device__ __forceinline__ ScanSel scan_sel(const SceneDev &S, const SceneOut &O, int which)
{
    switch (which) {
    case kScanTri: return {S.ht_count[0], S.ht_start[0], (int64_t)1 << S.ht_bits[0]};
    case kScanEdge: return {S.ht_count[1], S.ht_start[1], (int64_t)1 << S.ht_bits[1]};
    case kScanQuery: return {S.q_count, S.q_off, (int64_t)S.n_pts + S.n_edges};
    case kScanContact: return {S.c_cnt, S.c_ptr, (int64_t)S.n};
    case kScanSwFilter: return {S.sw_flag, S.sw_off, S.n_sw_prev};
    default: return {S.act_flag, S.act_off, (int64_t)O.n_cand};
    }
}

template <int NT = kBlock>
__device__ int block_exclusive_scan(int v, int *total)
{
    __shared__ int sh[NT / 64];
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        int t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    if (lane == 63) sh[w] = incl;
    __syncthreads();
    int woff = 0, tot = 0;
    for (int k = 0; k < NT / 64; ++k) {
        if (k < w) woff += sh[k];
        tot += sh[k];
    }
    __syncthreads();
    *total = tot;
    return woff + incl - v;
}

constexpr int kScanItems = kScanTile / kBlock;

__global__ void __launch_bounds__(kBlock) k_scan_tiles(Launch L, int which)
{
    int lb, s = scene_of_block(L, lb);
    const SceneDev &S = *L.sc[s];
    ScanSel sel = scan_sel(S, L.out[s], which);
    int64_t base = (int64_t)lb * kScanTile + threadIdx.x * kScanItems;
    int sum = 0;
    for (int k = 0; k < kScanItems; ++k)
        if (base + k < sel.len) sum += sel.in[base + k];
    int tot;
    block_exclusive_scan(sum, &tot);
    if (threadIdx.x == 0) S.scan_tmp[lb] = tot;
}

__device__ __forceinline__ void scan_total(const SceneDev &S, SceneOut &O, int which, int query_sw, int total)
{
    const ScanSel sel = scan_sel(S, O, which);
    sel.out[sel.len] = total;
    if (which == kScanTri) O.ent_tri = total;
    if (which == kScanEdge) O.ent_edge = total;
    if (which == kScanQuery) {
        if (query_sw)
            O.n_sw = total;
        else
            O.n_cand = total;
    }
    if (which == kScanActive) O.n_act = total;
    if (which == kScanSwFilter) O.n_cand = total;
}

// counts that the next pass counts again
__device__ __forceinline__ bool scan_clears(int which)
{
    return which == kScanTri || which == kScanEdge || which == kScanContact;
}

constexpr int kScanWide = 1024;  // threads of k_scan_one
constexpr int kScanRun = kScanOne / kScanWide / 4;  // its four-value reads a thread
// Block lb of a scene scans array which + lb.
__global__ void __launch_bounds__(kScanWide) k_scan_one(Launch L, int which, int query_sw)
{
    int lb, s = scene_of_block(L, lb);
    const SceneDev &S = *L.sc[s];
    which += lb;
    const ScanSel sel = scan_sel(S, L.out[s], which);
    const int len = (int)min(sel.len, (int64_t)kScanOne);
    typedef int Int4 __attribute__((ext_vector_type(4)));
    const int run = (len + 4 * kScanWide - 1) / (4 * kScanWide), first = 4 * run * (int)threadIdx.x;
    const auto in = glob(const_cast<int32_t *>(sel.in));
    const auto out = glob(sel.out);
    Int4 v[kScanRun];
    int sum = 0;
#pragma unroll
    for (int k = 0; k < kScanRun; ++k) {
        const int i = first + 4 * k;
        v[k] = Int4{0, 0, 0, 0};
        if (k < run && i + 4 <= len)
            v[k] = *(gptr<const Int4>)(in + i);
        else if (k < run)
            for (int c = 0; c < 4; ++c)
                if (i + c < len) v[k][c] = in[i + c];
        sum += v[k][0] + v[k][1] + v[k][2] + v[k][3];
    }
    int tot;
    int ex = block_exclusive_scan<kScanWide>(sum, &tot);
    const bool clear = scan_clears(which);
#pragma unroll
    for (int k = 0; k < kScanRun; ++k) {
        const int i = first + 4 * k;
        Int4 o;
        for (int c = 0; c < 4; ++c) {
            o[c] = ex;
            ex += v[k][c];
        }
        if (k < run && i + 4 <= len) {
            *(gptr<Int4>)(out + i) = o;
            if (clear) *(gptr<Int4>)(in + i) = Int4{0, 0, 0, 0};
        } else if (k < run) {
            for (int c = 0; c < 4; ++c)
                if (i + c < len) {
                    out[i + c] = o[c];
                    if (clear) in[i + c] = 0;
                }
        }
    }
    if (threadIdx.x == 0) scan_total(S, L.out[s], which, query_sw, tot);
}

__global__ void __launch_bounds__(kBlock) k_scan_top(Launch one, Launch tiles, int which, int query_sw)
{
    int lb, s = scene_of_block(one, lb);
    const SceneDev &S = *one.sc[s];
    int nt = blocks_of(tiles, s);
    int carry = 0;
    for (int base = 0; base < nt; base += kBlock) {
        int i = base + threadIdx.x;
        int v = i < nt ? S.scan_tmp[i] : 0;
        int tot;
        int ex = block_exclusive_scan(v, &tot);
        if (i < nt) S.scan_tmp[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) scan_total(S, one.out[s], which, query_sw, carry);
}

__global__ void __launch_bounds__(kBlock) k_scan_apply(Launch L, int which)
{
    int lb, s = scene_of_block(L, lb);
    const SceneDev &S = *L.sc[s];
    ScanSel sel = scan_sel(S, L.out[s], which);
    int64_t base = (int64_t)lb * kScanTile + threadIdx.x * kScanItems;
    int vals[kScanItems];
    int sum = 0;
    for (int k = 0; k < kScanItems; ++k) {
        vals[k] = (base + k < sel.len) ? sel.in[base + k] : 0;
        sum += vals[k];
    }
    int tot;
    int ex = block_exclusive_scan(sum, &tot) + S.scan_tmp[lb];
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < sel.len) {
            sel.out[base + k] = ex;
            if (scan_clears(which)) const_cast<int32_t *>(sel.in)[base + k] = 0;
        }
        ex += vals[k];
    }
}

// ---- launchers ----------------------------------------------------------------

static bool mixed(const Batch &b) { return b.sc[0]->prm.precision == IPC_MIXED; }

static void long_scan(Batch &b, ScanWhich which, PhaseKind tiles, const std::vector<int64_t> &len, int query_sw)
{
    size_t ns = b.sc.size();
    std::vector<int32_t> nt(ns), one(ns);
    for (size_t i = 0; i < ns; ++i) {
        nt[i] = len[i] < 0 ? 0 : std::max<int32_t>(1, (int32_t)((len[i] + kScanTile - 1) / kScanTile));
        one[i] = len[i] < 0 ? 0 : 1;
    }
    b.set_phase(tiles, nt);
    b.set_phase(kPhOne, one);
    IPC_LAUNCH(b, k_scan_tiles, tiles, kBlock, (int)which);
    IPC_LAUNCH(b, k_scan_top, kPhOne, kBlock, b.launch(tiles), (int)which, query_sw);
    IPC_LAUNCH(b, k_scan_apply, tiles, kBlock, (int)which);
}

void segmented_scan(Batch &b, ScanWhich which, PhaseKind tiles, std::vector<int64_t> len, int query_sw)
{
    const PhaseKind ph = (PhaseKind)(kPhScan0 + which);
    std::vector<int32_t> small(len.size(), 0);
    bool rest = false;
    for (size_t i = 0; i < len.size(); ++i) {
        small[i] = len[i] >= 0 && len[i] <= kScanOne;
        if (small[i]) len[i] = -1;
        rest |= len[i] >= 0;
    }
    b.set_phase(ph, small);
    IPC_LAUNCH(b, k_scan_one, ph, kScanWide, (int)which, query_sw);
    if (rest) long_scan(b, which, tiles, len, query_sw);
}

// both hash tables' bucket counts
void segmented_scan_tables(Batch &b, std::vector<int64_t> lt, std::vector<int64_t> le)
{
    std::vector<int32_t> small(lt.size(), 0);
    bool rest = false;
    for (size_t i = 0; i < lt.size(); ++i) {
        small[i] = lt[i] >= 0 && std::max(lt[i], le[i]) <= kScanOne ? 2 : 0;
        if (small[i]) lt[i] = le[i] = -1;
        rest |= lt[i] >= 0;
    }
    static_assert(kScanEdge == kScanTri + 1, "block 1 of a scene scans the edges' counts");
    b.set_phase(kPhScan0, small);
    IPC_LAUNCH(b, k_scan_one, kPhScan0, kScanWide, (int)kScanTri, 0);
    if (!rest) return;
    long_scan(b, kScanTri, kPhTilesT, lt, 0);
    long_scan(b, kScanEdge, kPhTilesE, le, 0);
}

void launch_begin_step(Batch &b) { IPC_LAUNCH(b, k_begin_step, kPhVert, kBlock); }
void launch_end_step(Batch &b) { IPC_LAUNCH(b, k_end_step, kPhVert, kBlock); }

void launch_al_update(Batch &b, const std::vector<uint8_t> &on)
{
    std::vector<int32_t> nb(b.sc.size(), 0);
    for (size_t i = 0; i < b.sc.size(); ++i)
        if (on[i]) nb[i] = nblocks(std::max(b.sc[i]->h.n_ind, 1));
    b.set_phase(kPhOne, nb);
    IPC_LAUNCH(b, k_al_update, kPhOne, kBlock);
}

void launch_trial(Batch &b)
{
    if (mixed(b))
        IPC_LAUNCH(b, k_trial<float>, kPhVert, kBlock, (const double *)b.d_alpha);
    else
        IPC_LAUNCH(b, k_trial<double>, kPhVert, kBlock, (const double *)b.d_alpha);
}

void launch_accept(Batch &b) { IPC_LAUNCH(b, k_accept, kPhVert, kBlock); }

void launch_put_views(hipStream_t strm, int n, const void *d_src)
{
    if (n > 0)
        hipLaunchKernelGGL(k_put_views, dim3(n), dim3(kBlock), 0, strm, n, static_cast<const uint64_t *>(d_src));
}

static void one_per_active(Batch &b, PhaseKind prod)
{
    std::vector<int32_t> one(b.sc.size());
    for (size_t i = 0; i < b.sc.size(); ++i) one[i] = b.h_off[prod][i + 1] > b.h_off[prod][i] ? 1 : 0;
    b.set_phase(kPhOne, one);
}

void run_lag_and_mean(Batch &b)
{
    IPC_LAUNCH(b, k_lag_mean, kPhVert, kBlock);
    one_per_active(b, kPhVert);
    IPC_LAUNCH(b, k_final_lag_mean, kPhOne, kBlock, b.launch(kPhVert));
}

void launch_gather_surface(Scene &s, double *dst, hipStream_t strm)
{
    int ns = (int)s.h_surf_verts.size();
    hipLaunchKernelGGL(k_gather_surface, dim3(nblocks(ns)), dim3(kBlock), 0, strm, ns, s.h.surf_verts, s.h.x, dst);
}

void run_pinf(Batch &b)
{
    if (mixed(b))
        IPC_LAUNCH(b, k_pinf<float>, kPhVert, kBlock);
    else
        IPC_LAUNCH(b, k_pinf<double>, kPhVert, kBlock);
    one_per_active(b, kPhVert);
    IPC_LAUNCH(b, k_final_pinf, kPhOne, kBlock, b.launch(kPhVert));
}

void launch_mas_diag(Batch &b)
{
    if (mixed(b)) {
        IPC_LAUNCH(b, k_mas_diag<float>, kPhMas, kBlock);
        IPC_LAUNCH(b, k_mas_invert<float>, kPhMasG, kBlock);
    } else {
        IPC_LAUNCH(b, k_mas_diag<double>, kPhMas, kBlock);
        IPC_LAUNCH(b, k_mas_invert<double>, kPhMasG, kBlock);
    }
}

void launch_hess_apply(Batch &b)
{
    if (mixed(b))
        IPC_LAUNCH(b, k_spmv_rows<float>, kPhSlice, kRowsPerBlock);
    else
        IPC_LAUNCH(b, k_spmv_rows<double>, kPhSlice, kRowsPerBlock);
}

// PCG for every scene with blocks in the kPhVert map (the active-pair counts
// come from the last read-back of the narrow phase): the scenes that one
// workgroup holds or whose team fits in one resident launch each, the others
// (and a team that did not form) iteration by iteration.
static void run_pcg_launched(Batch &b, const std::vector<uint8_t> &on, std::vector<int> &iters, std::vector<int> &hit_cap);

// algorithmic bytes of one scene in one A launch: every stored 3x3 block
// (values and column) once, the merged contact blocks among them; per vertex
// the z and d gathers, the d and q writes and its row pointer
static double pcg_bytes_a(const Scene &s, const SceneOut &o)
{
    const double rs = s.prm.precision == IPC_MIXED ? 4.0 : 8.0;
    return (9 * rs + 4) * (double)s.nnzb + (9 * 8 + 4) * (double)o.n_cblk + (12 * rs + 4) * (double)s.h.n;
}
// and of one B launch: per vertex q, d, p, r and the 3x3 inverse read and
// p, r, z written (30 reals); per preconditioner member its vertex id and
// three level ids; the SpMV blocks' d.q partials
static double pcg_bytes_b(const Scene &s, const SceneOut &o)
{
    const double rs = s.prm.precision == IPC_MIXED ? 4.0 : 8.0;
    return 30 * rs * (double)s.h.n + 16.0 * (s.h.mas_levels > 0 ? (double)s.h.mas_nf : 0.0) + 8.0 * (double)s.h.nb_rows;
}

void run_pcg(Batch &b, std::vector<int> &iters, std::vector<int> &hit_cap)
{
    const size_t ns = b.sc.size();
    std::vector<uint8_t> team(ns, 0), solo(ns, 0), rest(ns, 0);
    bool any_team = false, any_rest = false;
    for (size_t i = 0; i < ns; ++i) {
        if (b.h_off[kPhVert][i + 1] == b.h_off[kPhVert][i]) continue;
        const SceneDev &h = b.sc[i]->h;
        const bool one = solo_layout(h);  // such a scene has no other form
        bool t = one || (h.team_fit && b.sc[i]->tune.team && chunk_rows_bound(*b.sc[i], b.h_out[i]) <= kChunkRows);
        // a team that was given up competes for its CUs with other work (another
        // stream's team): each try holds CUs while it waits, so it waits longer
        // between tries
        if (t && !one && b.sc[i]->team_rest > 0) {
            b.sc[i]->team_rest--;
            t = false;
        }
        (one ? solo : t ? team : rest)[i] = 1;
        (t ? any_team : any_rest) = true;
    }
    iters.assign(ns, 0);
    hit_cap.assign(ns, 0);
    if (any_team) {
        hipEvent_t ev[2];
        if (b.prof()) b.prof_begin(kProfPcgA, ev);
        launch_pcg_team(b, team);
        launch_pcg_solo(b, solo);
        const size_t timed = b.ev_pending.size();
        if (b.prof()) b.prof_end(kProfPcgA, ev);
        b.read_out();
        double bytes = 0.0, peak = 0.0;
        for (size_t i = 0; i < ns; ++i) {
            if (!team[i] && !solo[i]) continue;
            const SceneOut &o = b.h_out[i];
            if (!o.pcg_done || o.pcg_fail) {
                b.sc[i]->pcg_given_up++;
                b.sc[i]->team_fails = std::min(b.sc[i]->team_fails + 1, 5);
                b.sc[i]->team_rest = (1 << b.sc[i]->team_fails) - 1;
                rest[i] = 1;
                any_rest = true;
                continue;
            }
            b.sc[i]->pcg_resident++;
            b.sc[i]->team_fails = 0;
            iters[i] = o.pcg_iters;
            hit_cap[i] = o.pcg_done != 1;
            b.sc[i]->last_pcg_iters = o.pcg_iters;
            if (b.prof()) {
                bytes += (pcg_bytes_a(*b.sc[i], o) + pcg_bytes_b(*b.sc[i], o)) * o.pcg_iters;
                peak += pcg_bytes_a(*b.sc[i], o);
            }
        }
        if (b.prof()) {
            b.ev_pending[timed].bytes = bytes;
            b.ev_pending[timed].big = peak >= kProfBigBytes;
            b.prof_totals(kProfPcgA, 1, bytes);
            b.prof_collect();
        }
    }
    if (any_rest) run_pcg_launched(b, rest, iters, hit_cap);
}

static void run_pcg_launched(Batch &b, const std::vector<uint8_t> &on, std::vector<int> &iters, std::vector<int> &hit_cap)
{
    size_t ns = b.sc.size();
    bool mx = mixed(b);
    std::vector<int32_t> nab(ns, 0), nbb(ns, 0);
    for (size_t i = 0; i < ns; ++i) {
        if (!on[i]) continue;
        nab[i] = b.sc[i]->h.nb_rows + (pair_count(*b.sc[i], b.h_out[i]) > 0 ? b.sc[i]->h.team_T : 0);
        nbb[i] = b.sc[i]->h.pcg_nvp;
    }
    b.set_phase(kPhPcgA, nab);
    b.set_phase(kPhPcgB, nbb);
    if (mx)
        IPC_LAUNCH(b, k_pcg_B<float>, kPhPcgB, kBlock, 0, 0);
    else
        IPC_LAUNCH(b, k_pcg_B<double>, kPhPcgB, kBlock, 0, 0);
    int maxit = 0, last = 0;
    for (size_t i = 0; i < ns; ++i) {
        if (!on[i]) continue;
        const Scene &s = *b.sc[i];
        maxit = std::max(maxit, s.h.pcg_maxit);
        last = std::max(last, s.last_pcg_iters);
    }
    std::vector<double> scene_bytes(ns, 0.0), scene_bytes_b(ns, 0.0);
    for (size_t i = 0; i < ns; ++i) {
        if (!on[i]) continue;
        scene_bytes[i] = pcg_bytes_a(*b.sc[i], b.h_out[i]);
        scene_bytes_b[i] = pcg_bytes_b(*b.sc[i], b.h_out[i]);
    }
    // Timed A launches of a chunk get their bytes once the chunk's flags are
    // back: a scene counts in the launch of iteration it when its solve was
    // still running there (not finished, or finished with more than it - 1
    // iterations); finished solves exit before their first load.
    std::vector<std::pair<size_t, int>> timed_a, timed_b;  // (pending event index, it)
    auto launch_bytes = [&](const std::vector<double> &sb, int it_) {
        double v = 0.0;
        for (size_t i = 0; i < ns; ++i) {
            if (!on[i] || sb[i] == 0.0) continue;
            if (!b.h_out[i].pcg_done || it_ <= b.h_out[i].pcg_iters) v += sb[i];
        }
        return v;
    };
    auto settle = [&](std::vector<std::pair<size_t, int>> &timed, const std::vector<double> &sb) {
        for (auto &ta : timed) {
            b.ev_pending[ta.first].bytes = launch_bytes(sb, ta.second);
            // an iteration above the Infinity Cache: its SpMV launch's bytes decide
            b.ev_pending[ta.first].big = launch_bytes(scene_bytes, ta.second) >= kProfBigBytes;
        }
        timed.clear();
    };
    auto settle_bytes = [&]() {
        settle(timed_a, scene_bytes);
        settle(timed_b, scene_bytes_b);
    };
    // large lists are bandwidth-bound: a thread per row reads the slices fully coalesced
    // (lanes per row and chunk lengths from the tuning of the list's largest scene)
    int64_t rows_total = 0;
    const Scene *big = nullptr;
    for (size_t i = 0; i < ns; ++i)
        if (nab[i] > 0) {
            rows_total += b.sc[i]->h.n;
            if (!big || b.sc[i]->h.n > big->h.n) big = b.sc[i];
        }
    const Tuning tn = big ? big->tune : Tuning{};
    const bool one_lane = rows_total >= tn.spmv_one_lane_rows;
    int it = 1;
    // Chunk lengths: a quantile (tuned) of the running scenes' expected
    // remaining iterations (their previous solve's count minus the launches
    // done) times a fraction, at least 8. A short chunk costs a read-back; a
    // long one keeps finished scenes' blocks in the launches (they exit at
    // once, but still take dispatch slots). One scene: the fraction of its own
    // previous count.
    auto next_chunk = [&](double frac) {
        std::vector<int> rem;
        for (size_t i = 0; i < ns; ++i)
            if (nab[i] > 0 && !(it > 1 && b.h_out[i].pcg_done)) rem.push_back(std::max(0, b.sc[i]->last_pcg_iters - (it - 1)));
        if (rem.empty()) return 8;
        std::sort(rem.begin(), rem.end());
        size_t k = (size_t)(tn.pcg_list_quantile * (double)(rem.size() - 1) + 0.5);
        return std::max(8, (int)(frac * rem[std::min(k, rem.size() - 1)]));
    };
    int chunk = last > 16 ? next_chunk(tn.pcg_first_chunk) : 8;
    int early = 0;
    // every launch of a chunk, with the algorithmic bytes of the scenes whose
    // solve was running there (when profiling)
    auto account_chunk = [&](int it0, int it1) {
        if (!b.prof()) return;
        double ba = 0.0, bb = 0.0;
        for (int j = it0; j < it1; ++j)
            for (size_t i = 0; i < ns; ++i) {
                if (!on[i] || nab[i] == 0) continue;
                if (!b.h_out[i].pcg_done || j <= b.h_out[i].pcg_iters) {
                    ba += scene_bytes[i];
                    bb += scene_bytes_b[i];
                }
            }
        b.prof_totals(kProfPcgA, it1 - it0, ba);
        b.prof_totals(kProfPcgB, it1 - it0, bb);
    };
    hipEvent_t ev[2];
    // launch it = maxit + 1 too: its A kernel records the cap of the scenes
    // that did not converge
    while (it <= maxit + 1) {
        int c = std::min(chunk, maxit + 2 - it);
        const int it_chunk = it;
        for (int j = 0; j < c; ++j, ++it) {
            // time one launch in sixteen when profiling: iterations 2, 18, 34, ...
            // of the first chunk (the first iteration applies the matrix to one
            // vector only; later chunks may skip finished scenes early)
            bool timed = b.prof() && (it & 15) == 2 && !early;
            if (timed) b.prof_begin(kProfPcgA, ev);
            if (timed) timed_a.push_back({b.ev_pending.size(), it});
            if (one_lane) {
                if (mx)
                    IPC_LAUNCH(b, (k_pcg_A<float, 1>), kPhPcgA, kRowsPerBlock, it, early);
                else
                    IPC_LAUNCH(b, (k_pcg_A<double, 1>), kPhPcgA, kRowsPerBlock, it, early);
            } else {
                if (mx)
                    IPC_LAUNCH(b, (k_pcg_A<float, 2>), kPhPcgA, 2 * kRowsPerBlock, it, early);
                else
                    IPC_LAUNCH(b, (k_pcg_A<double, 2>), kPhPcgA, 2 * kRowsPerBlock, it, early);
            }
            if (timed) b.prof_end(kProfPcgA, ev, 0.0);
            if (timed) b.prof_begin(kProfPcgB, ev);
            if (timed) timed_b.push_back({b.ev_pending.size(), it});
            if (mx)
                IPC_LAUNCH(b, k_pcg_B<float>, kPhPcgB, kBlock, it, early);
            else
                IPC_LAUNCH(b, k_pcg_B<double>, kPhPcgB, kBlock, it, early);
            if (timed) b.prof_end(kProfPcgB, ev);
        }
        run_pinf(b);  // |p|_inf of the scenes done so far comes back with their flags
        b.read_out();
        settle_bytes();
        account_chunk(it_chunk, it);
        b.prof_collect();
        bool all = true;
        for (size_t i = 0; i < ns; ++i)
            if (on[i] && !b.h_out[i].pcg_done) all = false;
        if (all) break;
        chunk = next_chunk(tn.pcg_later_chunk);
        early = 1;
        // scenes that finished leave the remaining launches of the list
        bool shrink = false;
        for (size_t i = 0; i < ns; ++i)
            if (nab[i] > 0 && b.h_out[i].pcg_done) {
                nab[i] = nbb[i] = 0;
                shrink = true;
            }
        if (shrink) {
            b.set_phase(kPhPcgA, nab);
            b.set_phase(kPhPcgB, nbb);
        }
    }
    for (size_t i = 0; i < ns; ++i) {
        if (!on[i]) continue;
        iters[i] = b.h_out[i].pcg_done ? b.h_out[i].pcg_iters : b.sc[i]->h.pcg_maxit;
        hit_cap[i] = b.h_out[i].pcg_done != 1;
        b.sc[i]->last_pcg_iters = iters[i];
        b.sc[i]->pcg_launched++;
    }
}

}  // namespace ipcg
