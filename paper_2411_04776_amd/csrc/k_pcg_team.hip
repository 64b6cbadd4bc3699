// k_pcg_team.hip -- the whole PCG solve of a scene in one launch.
//
// A solve is a chain of iterations whose two parts (SpMV, update) each need
// one sum over the whole scene. Launched one by one (k_solver.hip) an
// iteration of a 1,000 to 20,000 vertex gel takes 21-26 us, of which its
// bytes need well under one: two kernel boundaries of 2.5 us and about
// twenty dependent loads of 0.5-0.8 us. Here a scene's workgroups (its team)
// stay resident for the solve: matrix rows in registers, the direction in
// LDS, the update's vectors in registers, and per iteration only what other
// workgroups need passes through memory: z, q, the contact rows' part of q,
// and one tagged partial per workgroup and sum. What bounds it is the
// exchange: two sums of 1.0-1.4 us (8 workgroups) to 3.1 us (256), each
// followed by a read of other workgroups' values.
//
// Split (team_nt threads a workgroup, T workgroups): two threads per matrix
// row, so team_nt / 2 consecutive rows, each half row's up to kTeamSlots
// blocks in registers; the directions of those rows' columns in LDS (grid
// rows share most columns: each is loaded once, not once per block);
// team_nt / 256 update units (a preconditioner group or 256 other vertices),
// a vertex per thread; and the chunk's contact rows, a team of 16 threads
// (or a wavefront) each.
//
// Measured (us per iteration, launched form before -> this): 90 vertices FP64
// 21 -> 6.5; 1,280 FP64 24 -> 9.1; 16,000 FP64 26 -> 12.3; 9,500 mixed 29 ->
// 14.1; 128,000 mixed 59 -> 36.7.
//
// Exchange. Values that cross workgroups are written and read with relaxed
// agent-scope accesses (they pass the non-coherent caches), so no cache is
// flushed. A sum's partials travel as two 8-byte words that each hold half
// of the double and a 32-bit iteration tag, so a reader polls the data
// itself; a member's data stores are waited for before its partial is
// published, so whoever has the partial of iteration it may read the
// member's values of iteration it. A slot is overwritten only after every
// member has read it (its next value depends on all members' answers).
//
// Waiting. A workgroup first adds itself to the scene's join word; the team
// runs only once all T have arrived, all of them resident from then on, so
// every later wait ends. While the team forms, a member that has waited
// team_spin polls sets the abort flag, unless the team became complete;
// later arrivals see the flag and leave. The host then runs that solve with
// the launched form, which forms the same sums in the same order and gives
// the same bits. Later waits are bounded too (kTeamPoll) and end the same way.
#include "device_util.h"
#include "ipc_internal.h"
#include "pcg_sums.h"

namespace ipcg {

template <class R>
__device__ __forceinline__ R *as(void *p)
{
    return reinterpret_cast<R *>(p);
}

using u64 = unsigned long long;
constexpr int kTeamPoll = 1 << 20;  // polls of a wait inside a running team (~0.5 s)

// values exchanged between workgroups: agent scope; a team of one reads its
// own workgroup's values, for which workgroup scope is enough
template <bool SOLO, class T>
__device__ __forceinline__ T xload(gptr<T> p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, SOLO ? __HIP_MEMORY_SCOPE_WORKGROUP : __HIP_MEMORY_SCOPE_AGENT);
}
template <bool SOLO, class T>
__device__ __forceinline__ void xstore(gptr<T> p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, SOLO ? __HIP_MEMORY_SCOPE_WORKGROUP : __HIP_MEMORY_SCOPE_AGENT);
}
// A vertex vector of the exchange: four values per vertex (the last unused),
// read and written whole with the agent-scope bit (sc1) of the buffer
// instructions: one instruction a vertex in FP32, two in FP64.
template <class R, bool SOLO>
struct XVec {
    static constexpr int kAux = SOLO ? 0 : 16;
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ XVec(void *p, int n)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(p, 0, (int)(4u * (uint32_t)n * (uint32_t)sizeof(R)), 0x27000))
    {
    }
    __device__ __forceinline__ void load(int v, R (&o)[3]) const
    {
        if constexpr (sizeof(R) == 4) {
            const auto a = __builtin_amdgcn_raw_buffer_load_b128(rsrc, 16 * v, 0, kAux);
            for (int c = 0; c < 3; ++c) o[c] = __uint_as_float(a[c]);
        } else {
            const auto a = __builtin_amdgcn_raw_buffer_load_b128(rsrc, 32 * v, 0, kAux);
            const auto b = __builtin_amdgcn_raw_buffer_load_b64(rsrc, 32 * v + 16, 0, kAux);
            o[0] = __hiloint2double((int)a[1], (int)a[0]);
            o[1] = __hiloint2double((int)a[3], (int)a[2]);
            o[2] = __hiloint2double((int)b[1], (int)b[0]);
        }
    }
    __device__ __forceinline__ void store(int v, const R (&o)[3]) const
    {
        typedef uint32_t U4 __attribute__((ext_vector_type(4)));
        typedef uint32_t U2 __attribute__((ext_vector_type(2)));
        if constexpr (sizeof(R) == 4) {
            const U4 a = {__float_as_uint(o[0]), __float_as_uint(o[1]), __float_as_uint(o[2]), 0u};
            __builtin_amdgcn_raw_buffer_store_b128(a, rsrc, 16 * v, 0, kAux);
        } else {
            uint64_t x[3];
            for (int c = 0; c < 3; ++c) x[c] = (uint64_t)__double_as_longlong(o[c]);
            const U4 a = {(uint32_t)x[0], (uint32_t)(x[0] >> 32), (uint32_t)x[1], (uint32_t)(x[1] >> 32)};
            const U2 b = {(uint32_t)x[2], (uint32_t)(x[2] >> 32)};
            __builtin_amdgcn_raw_buffer_store_b128(a, rsrc, 32 * v, 0, kAux);
            __builtin_amdgcn_raw_buffer_store_b64(b, rsrc, 32 * v + 16, 0, kAux);
        }
    }
};

// Element i of an array: a uniform base and a 32-bit byte offset, which one
// load or store instruction takes as they are (the arrays reached so, of nine
// values a vertex or the matrix's, are below 4 GiB: a scene that fits has at
// most 131,072 rows).
template <class T>
__device__ __forceinline__ gptr<T> at(T *base, uint32_t i)
{
    return (gptr<T>)((gptr<char>)glob(base) + (uint32_t)(i * (uint32_t)sizeof(T)));
}

// the calling wavefront's stores so far have reached the other workgroups
__device__ __forceinline__ void stores_arrived() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Workgroups are narrow (256 threads in FP64, 512 in FP32) or, for scenes
// whose team would be too large, twice that. Matrix slots of a half row: RS
// in registers, LS in LDS, the rest (MS) read again in each iteration, issued
// ahead of the barrier before their use. A narrow thread keeps all eight (144
// of 512 registers in FP64, 72 of 256 in FP32); a wide one has half the
// registers, and with all eight the loop spilled (FP64 SpMV 12,400 cycles an
// iteration, FP32 39,000).
template <class R>
constexpr int kTeamNarrow = sizeof(R) == 8 ? 256 : 512;
template <class R, int NT>
struct TeamSplit {
    static constexpr bool kWide = NT > kTeamNarrow<R>;
    static constexpr int RS = kWide ? 4 : 8, LS = kWide ? 2 : 0, MS = kTeamSlots - RS - LS;
};
int team_narrow(size_t real) { return real == 8 ? kTeamNarrow<double> : kTeamNarrow<float>; }
inline int team_lds_slots(int nt, size_t real) { return nt > team_narrow(real) ? 2 : 0; }

// A value the optimiser cannot trace back: addresses made from it are formed
// where they are used. Hoisted out of the iteration loop they would take the
// registers of the matrix rows (64 of them for the polled slots and the
// re-read matrix values alone).
template <class T>
__device__ __forceinline__ T here(T v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// LDS of one update unit: rm[256][3] members' residuals, then corrections (R);
// ra[A][3] aggregate sums (double); inverses A * 9 (R); member ranges A (two
// 16-bit positions); per level the number of the group's aggregates
__host__ __device__ inline size_t up8(size_t b) { return (b + 7) / 8 * 8; }
__host__ __device__ inline size_t team_unit_bytes(int A, size_t real)
{
    return 3 * kMasCapM * real + 24 * (size_t)A + up8(9 * (size_t)A * real) + up8(4 * (size_t)A) + 16;
}
size_t team_lds_bytes(int nt, int H, int A, size_t real)
{
    return up8(3 * (size_t)H * real) + (size_t)(nt / kBlock) * team_unit_bytes(A, real) +
           (size_t)team_lds_slots(nt, real) * 9 * nt * real + (8 + sizeof(CRow)) * (size_t)kChunkRows;
}

// Publish chunk w's partial, tagged (tags of a solve start at 1; slots are
// cleared before the team forms).
__device__ __forceinline__ void put_partial(u64 *ll, int w, double v, uint32_t tag)
{
    const u64 b = (u64)__double_as_longlong(v);
    xstore<false>(at(ll, 2 * w), (b & 0xffffffff00000000ull) | tag);
    xstore<false>(at(ll, 2 * w + 1), (b << 32) | tag);
}

// Sum of all T partials of `tag`, by one wavefront: lane l adds chunks l,
// l + 64, ... in order, then the fixed tree. False if a wait ran out. PER:
// slots a lane polls (lanes past T look at the last chunk and add nothing).
template <int PER>
__device__ __forceinline__ bool sum_partials(u64 *ll, int T, uint32_t tag, double &tot)
{
    const int lane = (int)threadIdx.x & (kWave - 1);
    u64 a[PER], b[PER];
    bool ok = false;
    for (int n = 0; n < kTeamPoll && !ok; ++n) {
        ok = true;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const uint32_t m = here(2u * (uint32_t)min(lane + u * kWave, T - 1));
            const auto slot = at(ll, m);
            a[u] = xload<false>(slot);
            b[u] = xload<false>(slot + 1);
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) ok &= ((uint32_t)a[u] == tag) & ((uint32_t)b[u] == tag);
    }
    double acc = 0.0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const double v = __longlong_as_double((long long)((a[u] & 0xffffffff00000000ull) | (b[u] >> 32)));
        acc += lane + u * kWave < T ? v : 0.0;
    }
    tot = wave_sum(acc);
    return !__any(!ok);
}

// The team forms: true once all T members are resident, false if it was
// given up (by this member or another).
__device__ __forceinline__ bool team_join(PcgState *P, int T, int spin)
{
    uint32_t *w = &P->join;
    uint32_t v = __hip_atomic_fetch_add(w, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (v & kTeamAbort) return false;
    for (int n = 0;; ++n) {
        v = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (v & kTeamAbort) return false;
        if (v == (uint32_t)T) return true;
        if (n >= spin) {
            // give up only from an incomplete count: the exchange fails if a
            // member arrived meanwhile, and the loop looks again
            if (__hip_atomic_compare_exchange_strong(w, &v, v | kTeamAbort, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT))
                return false;
        }
        __builtin_amdgcn_s_sleep(4);
    }
}

template <class R, int NT, bool SOLO>
__global__ void __launch_bounds__(NT) k_pcg_team(Launch L)
{
    constexpr int U = NT / kBlock, NW = NT / kWave, RPW = NT / 2;
    constexpr int RS = TeamSplit<R, NT>::RS, LS = TeamSplit<R, NT>::LS, MS = TeamSplit<R, NT>::MS;
    extern __shared__ double team_lds[];
    __shared__ double s_dq[NW], s_rz[NW], s_tot;
    __shared__ int s_ok, s_cnt[NW];
    // the launch's own block order (no XCD remap): consecutive workgroups go
    // to different XCDs, so a team of 256 finds a CU for each member
    int s, w;
    {
        int lo = 0, hi = L.ns;
        while (hi - lo > 1) {
            int mid = (lo + hi) >> 1;
            if (L.blk_off[mid] <= (int)blockIdx.x) lo = mid; else hi = mid;
        }
        s = lo;
        w = (int)blockIdx.x - L.blk_off[lo];
    }
    const SceneDev &S = *L.sc[s];
    const int T = SOLO ? 1 : S.team_T;
    int tid = (int)threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    // what the loop needs of the view, read here: after the kernel's first
    // store the compiler would read it by vector loads, a memory round trip each
    u64 *const ll_dq = S.team_ll, *const ll_rz = S.team_ll + 2 * (size_t)T;
    const XVec<R, SOLO> Z(S.team_z, S.n), Q(S.team_q, S.n), C(S.c_q, S.n);
    R *const Mi = as<R>(S.Minv), *const Bv = as<R>(S.bval), *const DA = as<R>(S.dA), *const DB = as<R>(S.dB);
    uint16_t *const Lc = S.team_lcol;
    int32_t *const Hl = S.team_hlist;
    const auto Cv = glob((const R *)as<R>(S.c_val));
    const auto Cc = glob((const int32_t *)S.c_col);
    const int n = S.n, maxit = S.pcg_maxit;
    const double tol2 = S.pcg_tol2;

    // ---- LDS
    const int H = S.team_H, A = S.team_A;
    R *const hd = reinterpret_cast<R *>(team_lds);  // directions of the chunk's columns: hd[c * H + i]
    char *const base_u = reinterpret_cast<char *>(team_lds) + up8(3 * (size_t)H * sizeof(R));
    char *const ubase = base_u + (size_t)(tid / kBlock) * team_unit_bytes(A, sizeof(R));
    R(*const rm)[3] = reinterpret_cast<R(*)[3]>(ubase);
    double(*const ra)[3] = reinterpret_cast<double(*)[3]>(ubase + 3 * kMasCapM * sizeof(R));
    R *const Dl = reinterpret_cast<R *>(ra + A);
    uint32_t *const rng = reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(Dl) + up8(9 * (size_t)A * sizeof(R)));
    int *const lv = reinterpret_cast<int *>(reinterpret_cast<char *>(rng) + up8(4 * (size_t)A));
    R *const ml = reinterpret_cast<R *>(base_u + (size_t)U * team_unit_bytes(A, sizeof(R)));  // ml[(k * 9 + e) * NT + tid]
    double *const cdot = reinterpret_cast<double *>(ml + (size_t)LS * 9 * NT);  // contact rows: their d.q
    CRow *const clist = reinterpret_cast<CRow *>(cdot + kChunkRows);             // and places

    // ---- this thread's half matrix row
    const int part = tid & 1, row = w * RPW + tid / 2;
    const bool live = row < n;
    R m[RS > 0 ? RS : 1][9];
    uint32_t lc[kTeamSlots / 2];  // two 16-bit column indices each
    int s0 = 0, s1 = 0;
    const int ln = live ? row % kSlice : 0;
    if (live) {
        s0 = glob(S.slice_ptr)[row / kSlice];
        s1 = glob(S.slice_ptr)[row / kSlice + 1];
    }
    {
        const auto bv = glob(Bv);
        const auto lcol = glob(Lc);
#pragma unroll
        for (int k = 0; k < kTeamSlots; ++k) {
            // absent slots and rows: slot 0's place is read, zeros are kept
            const bool has = s0 + part + 2 * k < s1;
            const int64_t slot = has ? s0 + part + 2 * k : s0;
            const uint32_t c = has ? (uint32_t)lcol[slot * kSlice + ln] : 0u;
            lc[k / 2] = (k & 1) ? lc[k / 2] | (c << 16) : c;
            if (k < RS + LS)
#pragma unroll
                for (int e = 0; e < 9; ++e) {
                    R v = bv[(slot * 9 + e) * kSlice + ln];
                    v = has ? v : R(0);
                    if (k < RS)
                        m[k < RS ? k : 0][e] = v;
                    else
                        ml[((k - RS) * 9 + e) * NT + tid] = v;
                }
        }
    }
    // ---- this thread's columns of the chunk's list
    const int h0 = glob(S.team_hptr)[w], nh = glob(S.team_hptr)[w + 1] - h0;
    int hv[kTeamHalo];
#pragma unroll
    for (int j = 0; j < kTeamHalo; ++j) hv[j] = tid + j * NT < nh ? glob(S.team_hlist)[h0 + tid + j * NT] : 0;
    for (int i = tid; i < 3 * H; i += NT) hd[i] = R(0);

    // ---- this thread's vertex of its update unit
    const int nl = S.mas_levels, ngrp = nl > 0 ? S.mas_ng : 0;
    const int unit = w * U + wave / (kBlock / kWave);
    int tu = tid % kBlock;
    const bool grp = unit < ngrp;
    int vid = -1;
    uint32_t loc = 0;  // the vertex's aggregate at each level, 8 bits each
    static_assert(kMasCapA <= 256 && kMasLevels <= 4, "8-bit positions of a group's aggregates");
    if (grp) {
        const auto go = glob(S.mas_gofs);
        const size_t G1 = (size_t)S.mas_ng + 1;
        const int k0 = go[unit], k1 = go[unit + 1], k = k0 + tu;
        if (k < k1) vid = glob(S.mas_mem)[k];
        int base = 0, pbase = 0, pa0 = 0;
#pragma unroll
        for (int l = 0; l < kMasLevels; ++l) {
            if (l >= nl) break;
            const int a0 = go[(l + 1) * G1 + unit], a1 = go[(l + 1) * G1 + unit + 1];
            if (vid >= 0) loc |= (uint32_t)(base + glob(S.mas_manc)[(int64_t)l * S.mas_nf + k] - a0) << (8 * l);
            for (int a = a0 + tu; a < a1; a += kBlock) {
                const int64_t g = (int64_t)S.mas_off[l] + a;
                // children as positions in LDS: members, or the level below
                const int off = l == 0 ? -k0 : pbase - pa0;
                rng[base + a - a0] = (uint32_t)(glob(S.mas_mb)[g] + off) | (uint32_t)(glob(S.mas_me)[g] + off) << 16;
                for (int c = 0; c < 9; ++c) Dl[9 * (base + a - a0) + c] = glob(as<R>(S.mas_dinv))[9 * g + c];
            }
            if (tu == 0) lv[l] = a1 - a0;
            pbase = base;
            pa0 = a0;
            base += a1 - a0;
        }
    } else if (unit < S.pcg_nvp) {
        const int k = (unit - ngrp) * kBlock + tu;
        vid = nl > 0 ? (k < S.mas_nother ? glob(S.mas_other)[k] : -1) : (k < S.n ? k : -1);
    }
    // contact rows: the chunk's share of the work; whether this thread's row
    // is one (its direction is read as a column) and its vertex (q has two parts)
    const bool contact = L.out[s].n_crow > 0;
    bool touched = false, vtouched = false;
    int ncrow = 0, col0 = 0;
    if (contact) {
        touched = live && part == 0 && glob(S.c_ptr)[row + 1] > glob(S.c_ptr)[row];
        vtouched = vid >= 0 && glob(S.c_ptr)[vid + 1] > glob(S.c_ptr)[vid];
        ncrow = chunk_contact_rows<NT, kChunkRows>(S, w, 0, clist, s_cnt);
        col0 = contact_first(Cc, clist, ncrow, tid);
    }

    // ---- the team forms (slots cleared first)
    if constexpr (!SOLO) {
        if (tid == 0) {
            for (int k = 0; k < 2; ++k) {
                xstore<false>(at(ll_dq, 2 * w + k), (u64)0);
                xstore<false>(at(ll_rz, 2 * w + k), (u64)0);
            }
            stores_arrived();
            s_ok = team_join(S.pcg, T, S.team_spin) ? 1 : 0;
            if (!s_ok) xstore<false>(glob(&L.out[s].pcg_fail), (int32_t)1);
        }
        __syncthreads();
        if (!s_ok) return;  // the whole workgroup
    }
    __syncthreads();

    // the unit's aggregates per level, and the ranges of this thread's items
    static_assert(kMasLevels == 3, "three levels' ranges");
    int na0 = 0, na1 = 0, na2 = 0;
    uint32_t rg0 = 0, rg1 = 0, rg2 = 0;
    if (grp) {
        na0 = __builtin_amdgcn_readfirstlane(lv[0]);
        na1 = nl > 1 ? __builtin_amdgcn_readfirstlane(lv[1]) : 0;
        na2 = nl > 2 ? __builtin_amdgcn_readfirstlane(lv[2]) : 0;
        if (tu < 12 * na0) rg0 = rng[tu / 12];
        if (tu < 12 * na1) rg1 = rng[na0 + tu / 12];
        if (tu < 12 * na2) rg2 = rng[na0 + na1 + tu / 12];
    }

    R p[3], r[3], z[3], d[3], M[9];
#pragma unroll
    for (int c = 0; c < 3; ++c) p[c] = r[c] = z[c] = d[c] = R(0);
    auto load_inverse = [&]() {
        if (vid >= 0)
#pragma unroll
            for (int c = 0; c < 9; ++c) M[c] = at(Mi, 9u * (uint32_t)vid)[c];
    };

    // z = M^-1 r for the unit's vertices, published; this chunk's r.z partial
    // with tag `tag`. Ends with the partial on its way.
    auto precondition = [&](uint32_t tag) {
        double rz = 0.0;
        R zo[3] = {R(0), R(0), R(0)};
        if (vid >= 0) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                zo[a] = M[3 * a] * r[0] + M[3 * a + 1] * r[1] + M[3 * a + 2] * r[2];
                rz += (double)r[a] * (double)zo[a];
            }
            if (grp)
#pragma unroll
                for (int c = 0; c < 3; ++c) rm[tu][c] = r[c];
        }
        if (nl > 0) {
            __syncthreads();
            if (grp) mas_restrict(0, na0, rm, ra, tu, kBlock, [&](int i, int a) { return i < kBlock / 4 ? rg0 : rng[a]; });
            __syncthreads();
            if (grp && tu < kWave) {
                if (nl > 1) {
                    mas_restrict(na0, na1, ra, ra, tu, kWave, [&](int i, int a) { return i < kWave / 4 ? rg1 : rng[na0 + a]; });
                    wave_lds_fence();
                }
                if (nl > 2)
                    mas_restrict(na0 + na1, na2, ra, ra, tu, kWave,
                                 [&](int i, int a) { return i < kWave / 4 ? rg2 : rng[na0 + na1 + a]; });
            }
            __syncthreads();
            if (grp) rz += mas_correct<R>(na0 + na1 + na2, rm, ra, tu, [&](int q, int k) { return Dl[9 * q + k]; });
            __syncthreads();
        }
        if (vid >= 0) {
            double zi[3] = {(double)zo[0], (double)zo[1], (double)zo[2]};
            if (grp)
#pragma unroll
                for (int l = 0; l < kMasLevels; ++l) {
                    if (l >= nl) break;
#pragma unroll
                    for (int c = 0; c < 3; ++c) zi[c] += (double)rm[(loc >> (8 * l)) & 0xffu][c];
                }
#pragma unroll
            for (int c = 0; c < 3; ++c) z[c] = (R)zi[c];
            Z.store(vid, z);
        }
        rz = wave_sum(rz);
        if (lane == 0) s_rz[wave] = rz;
        stores_arrived();
        __syncthreads();
        if (tid == 0) {
            double t = 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u) t += (s_rz[4 * u] + s_rz[4 * u + 2]) + (s_rz[4 * u + 1] + s_rz[4 * u + 3]);
            if constexpr (SOLO)
                s_tot = 0.0 + t;
            else
                put_partial(ll_rz, w, t, tag);
        }
    };
    // the sum over all chunks, for every thread; false if a wait ran out
    auto total = [&](u64 *ll, uint32_t tag, double &t) {
        if constexpr (!SOLO) {
            if (wave == 0) {
                double v;
                const bool ok = T <= kWave ? sum_partials<1>(ll, T, tag, v) : sum_partials<kTeamMax / kWave>(ll, T, tag, v);
                if (lane == 0) {
                    s_tot = v;
                    s_ok = ok ? 1 : 0;
                }
            }
        }
        __syncthreads();
        t = wave_first(s_tot);
        return SOLO || s_ok != 0;
    };

    // ---- start: p = 0, r = -g
    if (vid >= 0) {
        const auto g = glob(as<R>(S.grad));
#pragma unroll
        for (int c = 0; c < 3; ++c) r[c] = -g[3 * (int64_t)vid + c];
    }
    load_inverse();
    precondition(1u);

    double stop = 0.0, rz_prev = 0.0;
    int done = 0, iters = 0;
    for (int it = 1;; ++it) {
#pragma unroll
        for (int k = 0; k < kTeamSlots / 2; ++k) lc[k] = here(lc[k]);
#pragma unroll
        for (int j = 0; j < kTeamHalo; ++j) hv[j] = here(hv[j]);
        vid = here(vid);
        loc = here(loc);
        col0 = here(col0);
        tid = here(tid);
        tu = here(tu);
        lane = here(lane);
        double rz;
        if (!total(ll_rz, (uint32_t)it, rz)) break;
        const bool bon = it > 1;
        double beta = 0.0;
        if (!bon) {
            if (!(rz > 0.0)) {
                done = 1;
                break;
            }
            stop = tol2 * rz;
        } else {
            const bool conv = rz <= stop;
            if (conv || it > maxit) {
                done = conv ? 1 : 2;
                iters = it - 1;
                break;
            }
            beta = rz / rz_prev;
        }
        rz_prev = rz;
        const R rb = (R)beta;
        R *const dnew = (it & 1) ? DA : DB, *const dold = (it & 1) ? DB : DA;
        // the direction d = z + beta d_prev (beta and d_prev 0 at first) at the
        // chunk's columns and the unit's vertex; the contact rows' blocks, their
        // columns' directions from memory, while the columns' z are on their way
        {
            R zh[kTeamHalo][3];
            auto load_columns = [&]() {
#pragma unroll
                for (int j = 0; j < kTeamHalo; ++j)
                    if (j * NT < nh) Z.load(hv[j], zh[j]);  // uniform; ids past the list read vertex 0
            };
            constexpr bool kWide = TeamSplit<R, NT>::kWide;
            if constexpr (!kWide) load_columns();  // in flight beside the contact rows' loads, registers permitting
#pragma unroll
            for (int c = 0; c < 3; ++c) d[c] = z[c] + rb * d[c];
            if (ncrow > 0) {
                auto dir = [&](int v, R (&o)[3]) {  // no branch: all loads of a row are in flight together
                    Z.load(v, o);
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const R dp = xload<SOLO>(at(dold, 3u * (uint32_t)v) + c);
                        o[c] = o[c] + rb * (bon ? dp : R(0));
                    }
                };
                contact_rows<NT, R>(Cv, Cc, clist, ncrow, tid, col0, dir, [&](int v, const R (&y)[3]) { C.store(v, y); }, cdot);
            }
            if constexpr (kWide) load_columns();
#pragma unroll
            for (int j = 0; j < kTeamHalo; ++j)
                if (tid + j * NT < nh) {
                    R *const h = hd + tid + j * NT;
                    const R o0 = h[0], o1 = h[H], o2 = h[2 * H];
                    h[0] = zh[j][0] + rb * o0;
                    h[H] = zh[j][1] + rb * o1;
                    h[2 * H] = zh[j][2] + rb * o2;
                }
            for (int i = tid + kTeamHalo * NT; i < nh; i += NT) {
                R zv[3];
                Z.load(glob(Hl)[h0 + i], zv);
                for (int c = 0; c < 3; ++c) hd[c * H + i] = zv[c] + rb * hd[c * H + i];
            }
        }
        R ms[MS > 0 ? MS : 1][9];
        if constexpr (MS > 0) {
#pragma unroll
            for (int k = 0; k < MS; ++k) {
                const int sl = s0 + part + 2 * (RS + LS + k);
                const auto from = at(Bv, here((uint32_t)(sl < s1 ? sl : s0) * (9u * kSlice) + (uint32_t)ln));
#pragma unroll
                for (int e = 0; e < 9; ++e) ms[k][e] = from[e * kSlice];
            }
        }
        __syncthreads();
        // q = K d for the chunk's rows
        double dq = 0.0;
        {
            R y0 = R(0), y1 = R(0), y2 = R(0);
#pragma unroll
            for (int k = 0; k < kTeamSlots; ++k) {
                const int c = (int)((k & 1) ? lc[k / 2] >> 16 : lc[k / 2] & 0xffffu);
                const R v0 = hd[c], v1 = hd[H + c], v2 = hd[2 * H + c];
                R a[9];
#pragma unroll
                for (int e = 0; e < 9; ++e) {
                    if (k < RS)
                        a[e] = m[k < RS ? k : 0][e];
                    else if (k < RS + LS)
                        a[e] = ml[((k - RS) * 9 + e) * NT + tid];
                    else
                        a[e] = s0 + part + 2 * k < s1 ? ms[k < RS + LS ? 0 : k - RS - LS][e] : R(0);
                }
                block_fma(a, v0, v1, v2, y0, y1, y2);
            }
            for (int slot = s0 + part + 2 * kTeamSlots; slot < s1; slot += 2) {  // longer rows: the rest from memory
                const int c = glob(Lc)[(int64_t)slot * kSlice + ln];
                const auto B = glob(Bv) + (int64_t)slot * 9 * kSlice + ln;
                const R v0 = hd[c], v1 = hd[H + c], v2 = hd[2 * H + c];
                R a[9];
#pragma unroll
                for (int e = 0; e < 9; ++e) a[e] = B[e * kSlice];
                block_fma(a, v0, v1, v2, y0, y1, y2);
            }
            double y[3] = {(double)y0, (double)y1, (double)y2};
#pragma unroll
            for (int c = 0; c < 3; ++c) y[c] += quad_other<0xb1>(y[c]);
            if (live && part == 0) {
                const int own = (int)(lc[0] & 0xffffu);  // slot 0 is the diagonal
                R qv[3], dv[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    qv[c] = (R)y[c];
                    dv[c] = hd[c * H + own];
                    dq += (double)dv[c] * (double)qv[c];
                }
                Q.store(row, qv);
                if (touched)  // contact columns read it in the next iteration
#pragma unroll
                    for (int c = 0; c < 3; ++c) xstore<SOLO>(at(dnew, 3u * (uint32_t)row) + c, dv[c]);
            }
        }
        dq = wave_sum(dq);
        if (lane == 0) s_dq[wave] = dq;
        stores_arrived();  // q and the contact rows' directions
        __syncthreads();
        double cd = 0.0;
        if (contact && wave == 0) {
            contact_dots(cdot, ncrow, cd);
            cd = wave_sum(cd);
        }
        if (tid == 0) {
            double a = 0.0;
#pragma unroll
            for (int k = 0; k < NW; k += 2) a += s_dq[k] + s_dq[k + 1];
            if (contact) a = a + cd;
            if constexpr (SOLO)
                s_tot = 0.0 + a;
            else
                put_partial(ll_dq, w, a, (uint32_t)it);
        }
        double dqt;
        if (!total(ll_dq, (uint32_t)it, dqt)) break;
        // p += alpha d, r -= alpha q
        const R alpha = (R)(rz / dqt);
        load_inverse();
        if (vid >= 0) {
            R qv[3];
            Q.load(vid, qv);
            if (vtouched) {
                R qc[3];
                C.load(vid, qc);
#pragma unroll
                for (int c = 0; c < 3; ++c) qv[c] += qc[c];
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                p[c] = p[c] + alpha * d[c];
                r[c] = r[c] - alpha * qv[c];
            }
        }
        precondition((uint32_t)it + 1u);
    }
    if (!done) {  // a wait ran out (uniform over the workgroup)
        if (tid == 0) xstore<false>(glob(&L.out[s].pcg_fail), (int32_t)1);
        return;
    }
    // ---- the solution and its largest component over free vertices
    double pm = 0.0;
    if (vid >= 0) {
#pragma unroll
        for (int c = 0; c < 3; ++c) as<R>(S.sol)[3 * (int64_t)vid + c] = p[c];
        if (!S.fixed[vid]) pm = fmax(fabs((double)p[0]), fmax(fabs((double)p[1]), fabs((double)p[2])));
    }
    pm = wave_max(pm);
    if (lane == 0 && pm > 0.0)  // non-negative doubles order like their bits
        atomicMax(reinterpret_cast<u64 *>(&L.out[s].pinf), (u64)__double_as_longlong(pm));
    if (w == 0 && tid == 0) {
        S.pcg->done = 1;
        S.pcg->iters = iters;
        L.out[s].pcg_done = done;
        L.out[s].pcg_iters = iters;
    }
}

// ---- host ------------------------------------------------------------------

// narrow workgroups (0), wide ones (1); + 2: a team of one
static int team_variant(const SceneDev &h, size_t real)
{
    return (h.team_nt > team_narrow(real) ? 1 : 0) + (h.team_T == 1 ? 2 : 0);
}

template <class R>
static void launch_variant(Batch &b, int variant, size_t lds)
{
    constexpr int N = kTeamNarrow<R>;
    const PhaseKind ph = (PhaseKind)(kPhTeam0 + variant);
    const int nb = b.blocks(ph);
    if (nb == 0) return;
    b.flush_phases();
    const Launch l = b.launch(ph);
    switch (variant) {
    case 0: hipLaunchKernelGGL((k_pcg_team<R, N, false>), dim3(nb), dim3(N), lds, b.stream, l); break;
    case 1: hipLaunchKernelGGL((k_pcg_team<R, 2 * N, false>), dim3(nb), dim3(2 * N), lds, b.stream, l); break;
    case 2: hipLaunchKernelGGL((k_pcg_team<R, N, true>), dim3(nb), dim3(N), lds, b.stream, l); break;
    default: hipLaunchKernelGGL((k_pcg_team<R, 2 * N, true>), dim3(nb), dim3(2 * N), lds, b.stream, l); break;
    }
    IPC_HIP(hipGetLastError());
}

void launch_pcg_team(Batch &b, const std::vector<uint8_t> &on)
{
    const size_t ns = b.sc.size();
    const bool mx = b.sc[0]->prm.precision == IPC_MIXED;
    const size_t rs = mx ? sizeof(float) : sizeof(double);
    for (int v = 0; v < 4; ++v) {
        std::vector<int32_t> nb(ns, 0);
        size_t lds = 0;
        for (size_t i = 0; i < ns; ++i) {
            const SceneDev &h = b.sc[i]->h;
            if (!on[i] || team_variant(h, rs) != v) continue;
            nb[i] = h.team_T;
            lds = std::max(lds, team_lds_bytes(h.team_nt, h.team_H, h.team_A, rs));
        }
        b.set_phase((PhaseKind)(kPhTeam0 + v), nb);
        if (mx)
            launch_variant<float>(b, v, lds);
        else
            launch_variant<double>(b, v, lds);
    }
}

template <class R>
static void raise_lds()
{
    constexpr int N = kTeamNarrow<R>;
    for (const void *f : {(const void *)k_pcg_team<R, N, true>, (const void *)k_pcg_team<R, N, false>,
                          (const void *)k_pcg_team<R, 2 * N, true>, (const void *)k_pcg_team<R, 2 * N, false>})
        IPC_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kTeamLds - 1024));
}

void team_prepare_device()
{
    raise_lds<float>();
    raise_lds<double>();
}

}  // namespace ipcg
