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
// Split (T workgroups): team_rows consecutive matrix rows each, a thread or
// two per row with its blocks in registers (one thread a row: four of them in
// LDS); the directions of those rows' columns in LDS (grid rows share most
// columns: each is loaded once, not once per block); team_units update units (a
// preconditioner group or 256 other vertices), a vertex per thread and unit;
// and the chunk's contact rows, 16 lanes for 16 blocks, held in registers too
// as far as the lanes go. Wide workgroups (one thread a row, two units a
// thread) of 1,024 threads with half a row each had half the registers and
// spilled: 36.7 us an iteration at 130,600 vertices, not 25.3.
//
// Measured (us per iteration, launched form before -> this): 1,442 vertices
// FP64 24 -> 8.5; 16,800 FP64 26 -> 10.4; 10,100 mixed 29 -> 12.3; 130,600
// mixed 59 -> 25.3. A scene that one workgroup holds has a kernel of its own
// (k_pcg_solo.hip).
//
// Exchange. Values that cross workgroups are written and read with
// agent-scope accesses (they pass the non-coherent caches), so no cache is
// flushed. Every 8-byte word carries its iteration's tag beside the data, so a
// reader takes the data as soon as it is there and a writer waits for no
// store: 700 of 19,000 cycles an iteration (1,442 vertices, FP64) in place of
// 1,400 for untagged data with a wait before each partial. A sum's partial is
// one 16-byte slot, polled by one wavefront per workgroup (read as two 8-byte
// words, 16,800 vertices took 12.1 us an iteration, not 11.1). Reading the
// columns while the sum is still on its way, in all wavefronts, was slower
// (12.9 us: the polls get in the way of the partials).
//
// A slot is overwritten only after every member has read it: its next value
// depends on a sum that depends on all members' uses of the last one.
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

// values exchanged between workgroups: agent scope
template <class T>
__device__ __forceinline__ T xload(gptr<T> p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ void xstore(gptr<T> p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Element i of an array: a uniform base and a 32-bit byte offset, which one
// load or store instruction takes as they are (the arrays reached so, of nine
// values a vertex or the matrix's, are below 4 GiB: a scene that fits has at
// most 131,072 rows).
template <class T>
__device__ __forceinline__ gptr<T> at(T *base, uint32_t i)
{
    return (gptr<T>)((gptr<char>)glob(base) + (uint32_t)(i * (uint32_t)sizeof(T)));
}

// A vertex vector of the exchange: the space of four values per vertex, as
// 8-byte words that each carry 16 bits of the iteration's tag beside their
// share of the three values (two words in FP32, four in FP64). A reader needs
// no word from the writer that the data is there: it reads until the tags are
// the iteration's.
template <class R>
struct XVec {
    static constexpr int W = sizeof(R) == 4 ? 2 : 4, kAgent = 16;
    __amdgpu_buffer_rsrc_t rsrc;
    struct Raw {
        u64 w[W];
    };
    __device__ __forceinline__ XVec(void *p, int n)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(p, 0, (int)(8u * W * (uint32_t)n), 0x27000))
    {
    }
    __device__ __forceinline__ void load(int v, Raw &o) const
    {
#pragma unroll
        for (int k = 0; k < W; k += 2) {
            const auto a = __builtin_amdgcn_raw_buffer_load_b128(rsrc, 8 * W * v + 8 * k, 0, kAgent);
            o.w[k] = (u64)a[1] << 32 | a[0];
            o.w[k + 1] = (u64)a[3] << 32 | a[2];
        }
    }
    static __device__ __forceinline__ bool is(const Raw &o, uint32_t tag)
    {
        uint32_t x = 0;
#pragma unroll
        for (int k = 0; k < W; ++k) x |= ((uint32_t)(o.w[k] >> 32) ^ tag) & 0xffffu;
        return x == 0;
    }
    static __device__ __forceinline__ void get(const Raw &o, R (&d)[3])
    {
        uint32_t lo[W], hi[W];
#pragma unroll
        for (int k = 0; k < W; ++k) {
            lo[k] = (uint32_t)o.w[k];
            hi[k] = (uint32_t)(o.w[k] >> 32);
        }
        if constexpr (W == 2) {
            d[0] = __uint_as_float(lo[0]);
            d[1] = __uint_as_float((hi[0] & 0xffff0000u) | (hi[1] >> 16));
            d[2] = __uint_as_float(lo[1]);
        } else {
            d[0] = __hiloint2double((int)((hi[0] & 0xffff0000u) | (lo[3] >> 16)), (int)lo[0]);
            d[1] = __hiloint2double((int)((hi[1] & 0xffff0000u) | (lo[3] & 0xffffu)), (int)lo[1]);
            d[2] = __hiloint2double((int)((hi[2] & 0xffff0000u) | (hi[3] >> 16)), (int)lo[2]);
        }
    }
    __device__ __forceinline__ void store(int v, const R (&d)[3], uint32_t tag) const
    {
        u64 o[W];
        tag &= 0xffffu;
        auto word = [](uint32_t hi, uint32_t lo) { return (u64)hi << 32 | lo; };
        if constexpr (W == 2) {
            const uint32_t y = __float_as_uint(d[1]);
            o[0] = word((y & 0xffff0000u) | tag, __float_as_uint(d[0]));
            o[1] = word((y << 16) | tag, __float_as_uint(d[2]));
        } else {
            uint32_t hi[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const u64 x = (u64)__double_as_longlong(d[c]);
                hi[c] = (uint32_t)(x >> 32);
                o[c] = word((hi[c] & 0xffff0000u) | tag, (uint32_t)x);
            }
            o[3] = word((hi[2] << 16) | tag, (hi[0] << 16) | (hi[1] & 0xffffu));
        }
#pragma unroll
        for (int k = 0; k < W; k += 2) put(v, k, o[k], o[k + 1]);
    }
    __device__ __forceinline__ void put(int v, int k, u64 a, u64 b) const
    {
        typedef uint32_t U4 __attribute__((ext_vector_type(4)));
        const U4 x = {(uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32)};
        __builtin_amdgcn_raw_buffer_store_b128(x, rsrc, 8 * W * v + 8 * k, 0, kAgent);
    }
    // the value of iteration `tag`, read until it is there; false if the wait ran out
    __device__ __forceinline__ bool wait(int v, uint32_t tag, R (&d)[3]) const
    {
        Raw o;
        load(v, o);
        for (int n = 0; !is(o, tag) && n < kTeamPoll; ++n) load(v, o);
        get(o, d);
        return is(o, tag);
    }
    __device__ __forceinline__ void clear(int v) const
    {
#pragma unroll
        for (int k = 0; k < W; k += 2) put(v, k, 0, 0);
    }
};

// the calling wavefront's stores so far have reached the other workgroups
__device__ __forceinline__ void stores_arrived() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The layouts of a workgroup (256 threads in FP64, 512 in FP32: 512 and 256
// registers a thread): threads per matrix row (RT) and update units per 256
// threads (V). Two threads a row hold eight blocks each (144 of 512 registers
// in FP64, 72 of 256 in FP32), one thread a row eleven (198 and 99) and four
// in LDS, with its vertices' solution in memory; a longer row's other blocks are read again in each iteration. The
// compact layout (FP32, 256 threads) has the narrow one's chunks, a thread a
// row: two of its workgroups share a CU, for launches with more workgroups
// than CUs, where the waits of one are the time of the other. Entries 2 and 3
// give the rows and units of the one-workgroup layouts (k_pcg_solo.hip).
constexpr int kTeamRT[5] = {2, 1, 2, 1, 1}, kTeamV[5] = {1, 2, 2, 2, 2};
constexpr int team_lds_slots(int variant) { return kTeamRT[variant] == 2 ? 0 : variant == kTeamCompact ? 5 : 4; }
int team_contact_rows(int variant) { return variant == kTeamCompact ? kCompactRows : kChunkRows; }
constexpr int team_threads(int variant, size_t real) { return real == 8 ? 256 : variant == kTeamCompact ? 256 : 512; }
constexpr int team_columns(int variant) { return variant == kTeamCompact ? 5 : 4; }  // column ids a thread keeps in registers
int team_rows(int variant, size_t real) { return team_threads(variant, real) / kTeamRT[variant]; }
int team_units(int variant, size_t real) { return team_threads(variant, real) / kBlock * kTeamV[variant]; }

// LDS of one update unit: rm[256][3] members' residuals, then corrections (R);
// ra[A][3] aggregate sums (double); inverses A * 9 (R); member ranges A (two
// 16-bit positions); per level the number of the group's aggregates
__host__ __device__ inline size_t up8(size_t b) { return (b + 7) / 8 * 8; }
__host__ __device__ inline size_t team_unit_bytes(int A, size_t real)
{
    return 3 * kMasCapM * real + 24 * (size_t)A + up8(9 * (size_t)A * real) + up8(4 * (size_t)A) + 16;
}
size_t team_lds_bytes(int variant, int H, int A, size_t real)
{
    return up8(3 * (size_t)H * real) + (size_t)team_units(variant, real) * team_unit_bytes(A, real) +
           (size_t)team_lds_slots(variant) * 9 * team_threads(variant, real) * real +
           (8 + sizeof(CRow)) * (size_t)team_contact_rows(variant);
}

// The chunks' partials of one sum, 16 bytes each: two 8-byte words that each
// hold half of the double and the tag (tags of a solve start at 1; slots are
// cleared before the team forms).
struct Partials {
    static constexpr int kAgent = 16;
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ Partials(u64 *p, int T) : rsrc(__builtin_amdgcn_make_buffer_rsrc(p, 0, 16 * T, 0x27000)) {}
    __device__ __forceinline__ void put(int w, double v, uint32_t tag) const
    {
        typedef uint32_t U4 __attribute__((ext_vector_type(4)));
        const u64 b = (u64)__double_as_longlong(v);
        const U4 x = {tag, (uint32_t)(b >> 32), tag, (uint32_t)b};
        __builtin_amdgcn_raw_buffer_store_b128(x, rsrc, 16 * w, 0, kAgent);
    }
    // Sum of all T of `tag`, by one wavefront: lane l adds chunks l, l + 64, ...
    // in order, then the fixed tree. False if a wait ran out. PER: slots a lane
    // polls (lanes past T look at the last chunk and add nothing).
    template <int PER>
    __device__ __forceinline__ bool sum(int T, uint32_t tag, double &tot) const
    {
        const int lane = (int)threadIdx.x & (kWave - 1);
        double v[PER];
        bool ok = false;
        for (int n = 0; n < kTeamPoll && !ok; ++n) {
            ok = true;
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const auto x = __builtin_amdgcn_raw_buffer_load_b128(rsrc, here(16 * min(lane + u * kWave, T - 1)), 0, kAgent);
                v[u] = __hiloint2double((int)x[1], (int)x[3]);
                ok &= (x[0] == tag) & (x[2] == tag);
            }
        }
        double acc = 0.0;
#pragma unroll
        for (int u = 0; u < PER; ++u) acc += lane + u * kWave < T ? v[u] : 0.0;
        tot = wave_sum(acc);
        return !__any(!ok);
    }
};

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

template <class R, int VARIANT>
__global__ void __launch_bounds__(team_threads(VARIANT, sizeof(R)), VARIANT == kTeamCompact ? 2 : 1) k_pcg_team(Launch L)
{
    constexpr int NT = team_threads(VARIANT, sizeof(R)), NW = NT / kWave, G = NT / kBlock;  // G: threads' groups of 256
    constexpr int RT = kTeamRT[VARIANT], V = kTeamV[VARIANT], U = V * G, RPW = NT / RT;
    constexpr int HALO = team_columns(VARIANT), ROWS = VARIANT == kTeamCompact ? kCompactRows : kChunkRows;
    constexpr bool PMEM = RT == 1;  // p in memory: registers are short
    constexpr bool HOLD = RT == 2;  // contact blocks in registers
    constexpr int NS = RT == 2 ? kTeamSlots : 2 * kTeamSlots - 1;  // blocks on the chip,
    constexpr int RS = NS - team_lds_slots(VARIANT);               // the first RS of them in registers
    extern __shared__ double team_lds[];
    __shared__ double s_dq[NW], s_rz[V * NW], s_tot;
    __shared__ int s_ok, s_cnt[NW], s_at[NT / kRowTeam + 1];
    __shared__ double s_item[NT / kRowTeam][3];
    __shared__ R s_own[NT / kRowTeam][3];
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
    const int T = S.team_T;
    int tid = (int)threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    // what the loop needs of the view, read here: after the kernel's first
    // store the compiler would read it by vector loads, a memory round trip each
    const Partials P_dq(S.team_ll, T), P_rz(S.team_ll + 2 * (size_t)T, T);
    const XVec<R> Z(S.team_z, S.n), Q(S.team_q, S.n), DA(S.team_dA, S.n), DB(S.team_dB, S.n);
    const XVec<double> C(S.c_q, S.n);
    R *const Mi = as<R>(S.Minv), *const Bv = as<R>(S.bval), *const Sol = as<R>(S.sol);
    uint16_t *const Lc = S.team_lcol;
    int32_t *const Hl = S.team_hlist;
    const auto Cv = glob((const double *)S.c_val);
    const auto Cc = glob((const int32_t *)S.c_col);
    const int n = S.n, maxit = S.pcg_maxit;
    const double tol2 = S.pcg_tol2;

    // ---- LDS
    const int H = S.team_H, A = S.team_A;
    R *const hd = reinterpret_cast<R *>(team_lds);  // directions of the chunk's columns: hd[c * H + i]
    char *const base_u = reinterpret_cast<char *>(team_lds) + up8(3 * (size_t)H * sizeof(R));
    const size_t ub = team_unit_bytes(A, sizeof(R));
    struct Unit {
        R (*rm)[3];
        double (*ra)[3];
        R *Dl;
        uint32_t *rng;
        int *lv;
    };
    auto unit_at = [&](int u) {  // of the workgroup's units
        char *const b = base_u + (size_t)u * ub;
        Unit x;
        x.rm = reinterpret_cast<R(*)[3]>(b);
        x.ra = reinterpret_cast<double(*)[3]>(b + 3 * kMasCapM * sizeof(R));
        x.Dl = reinterpret_cast<R *>(x.ra + A);
        x.rng = reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(x.Dl) + up8(9 * (size_t)A * sizeof(R)));
        x.lv = reinterpret_cast<int *>(reinterpret_cast<char *>(x.rng) + up8(4 * (size_t)A));
        return x;
    };
    double *const cdot = reinterpret_cast<double *>(base_u + (size_t)U * ub);  // contact rows: their d.q
    CRow *const clist = reinterpret_cast<CRow *>(cdot + ROWS);           // and places
    R *const ml = reinterpret_cast<R *>(clist + ROWS);  // matrix blocks: ml[(k * 9 + e) * NT + tid]
    static_assert(sizeof(CRow) * ROWS % 8 == 0, "the arrays after the list are 8-byte aligned");

    // ---- this thread's matrix row or half row (slot k of the thread: part + RT * k of the row)
    const int part = RT == 2 ? tid & 1 : 0, row = w * RPW + tid / RT;
    const bool live = row < n;
    R m[RS][9];
    uint32_t lc[(NS + 1) / 2];  // two 16-bit column indices each
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
        for (int k = 0; k < NS; ++k) {
            // absent slots and rows: slot 0's place is read, zeros are kept
            const bool has = s0 + part + RT * k < s1;
            const int64_t slot = has ? s0 + part + RT * k : s0;
            const uint32_t c = has ? (uint32_t)lcol[slot * kSlice + ln] : 0u;
            lc[k / 2] = (k & 1) ? lc[k / 2] | (c << 16) : c;
#pragma unroll
            for (int e = 0; e < 9; ++e) {
                const R v = bv[(slot * 9 + e) * kSlice + ln];
                if (k < RS)
                    m[k < RS ? k : 0][e] = has ? v : R(0);
                else
                    ml[((k - RS) * 9 + e) * NT + tid] = has ? v : R(0);
            }
        }
    }
    // ---- this thread's columns of the chunk's list
    const int h0 = glob(S.team_hptr)[w], nh = glob(S.team_hptr)[w + 1] - h0;
    int hv[HALO];
#pragma unroll
    for (int j = 0; j < HALO; ++j) hv[j] = tid + j * NT < nh ? glob(Hl)[h0 + tid + j * NT] : 0;
    for (int i = tid; i < 3 * H; i += NT) hd[i] = R(0);

    // ---- this thread's vertices, one of each of its update units
    const int nl = S.mas_levels, ngrp = nl > 0 ? S.mas_ng : 0;
    int tu = tid % kBlock;
    const int ug = wave / (kBlock / kWave);  // its units: ug, ug + G, ... of the workgroup's
    int vid[V];
    uint32_t loc[V];  // the vertex's aggregate at each level, 8 bits each
    bool grp[V];
    static_assert(kMasCapA <= 256 && kMasLevels <= 4, "8-bit positions of a group's aggregates");
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int unit = w * U + v * G + ug;
        const Unit x = unit_at(v * G + ug);
        grp[v] = unit < ngrp;
        vid[v] = -1;
        loc[v] = 0;
        if (grp[v]) {
            const auto go = glob(S.mas_gofs);
            const size_t G1 = (size_t)S.mas_ng + 1;
            const int k0 = go[unit], k1 = go[unit + 1], k = k0 + tu;
            if (k < k1) vid[v] = glob(S.mas_mem)[k];
            const auto mb = glob(S.mas_mb), me = glob(S.mas_me);
            int base = 0, f0 = 0;
#pragma unroll
            for (int l = 0; l < kMasLevels; ++l) {
                if (l >= nl) break;
                const int a0 = go[(l + 1) * G1 + unit], a1 = go[(l + 1) * G1 + unit + 1];
                if (l == 0) f0 = a0;
                if (vid[v] >= 0) loc[v] |= (uint32_t)(base + glob(S.mas_manc)[(int64_t)l * S.mas_nf + k] - a0) << (8 * l);
                for (int a = a0 + tu; a < a1; a += kBlock) {
                    const int64_t g = (int64_t)S.mas_off[l] + a;
                    // its members' rows, or its level-0 aggregates
                    int b = mb[g], e = me[g];
                    const int off = l == 0 ? k0 : f0;
                    if (l == 2) {
                        b = mb[S.mas_off[1] + b];
                        e = me[S.mas_off[1] + e - 1];
                    }
                    x.rng[base + a - a0] = (uint32_t)(b - off) | (uint32_t)(e - off) << 16;
                    for (int c = 0; c < 9; ++c) x.Dl[9 * (base + a - a0) + c] = glob(as<R>(S.mas_dinv))[9 * g + c];
                }
                if (tu == 0) x.lv[l] = a1 - a0;
                base += a1 - a0;
            }
        } else if (unit < S.pcg_nvp) {
            const int k = (unit - ngrp) * kBlock + tu;
            vid[v] = nl > 0 ? (k < S.mas_nother ? glob(S.mas_other)[k] : -1) : (k < S.n ? k : -1);
        }
    }
    // contact rows: the chunk's share of the work; whether this thread's row
    // is one (its direction is published) and its vertex (q has two parts).
    // The items (kRowTeam blocks of a row) of the first hrows rows, as many as
    // there are teams of lanes, stay in registers, with the directions at
    // their columns and at their rows.
    const bool contact = L.out[s].n_crow > 0;
    bool touched = false, vtouched[V];
    int ncrow = 0, hrows = 0;
    double cA[9];
    R cd[3], cown[3];
    int ccol = 0, crow = 0;
    bool chas = false, cteam = false;  // the lane holds a block, an item
#pragma unroll
    for (int v = 0; v < V; ++v) vtouched[v] = false;
#pragma unroll
    for (int c = 0; c < 3; ++c) cd[c] = cown[c] = R(0);
#pragma unroll
    for (int c = 0; c < 9; ++c) cA[c] = 0.0;
    if (tid == 0) {
        s_ok = 1;
    }
    if (contact) {
        touched = live && part == 0 && glob(S.c_ptr)[row + 1] > glob(S.c_ptr)[row];
#pragma unroll
        for (int v = 0; v < V; ++v) vtouched[v] = vid[v] >= 0 && glob(S.c_ptr)[vid[v] + 1] > glob(S.c_ptr)[vid[v]];
        ncrow = chunk_contact_rows<NT, ROWS>(S, w, 0, clist, s_cnt);
        if constexpr (HOLD) {
            const int item = tid / kRowTeam, u = tid % kRowTeam;
            int at = 0, h = 0;
            for (; h < ncrow; ++h) {  // rows of items [at, at + k)
                // a row whose partners are all fixed has no block: an item of
                // none, so that its direction and its zero product are there
                // and there are never more rows than items
                const int k = max((clist[h].n + kRowTeam - 1) / kRowTeam, 1);
                if (at + k > NT / kRowTeam) break;
                if (tid == 0) s_at[h] = at;
                if (item >= at && item < at + k) {
                    cteam = true;
                    crow = clist[h].row;
                    const int j = (item - at) * kRowTeam + u;
                    chas = j < clist[h].n;
                    const int b = clist[h].base + (chas ? j : 0);
                    ccol = chas ? Cc[b] : crow;
#pragma unroll
                    for (int e = 0; e < 9; ++e) cA[e] = chas ? Cv[9 * (int64_t)b + e] : 0.0;
                }
                at += k;
            }
            hrows = h;
            if (tid == 0) s_at[h] = at;
        }
    }
    // the workgroup's part of the exchanged vectors: no tag of an earlier solve
    for (int i = tid; i < RPW; i += NT)
        if (w * RPW + i < n) {
            const int v = w * RPW + i;
            Z.clear(v);
            Q.clear(v);
            C.clear(v);
            DA.clear(v);
            DB.clear(v);
        }
    if (tid == 0) {
        P_dq.put(w, 0.0, 0u);
        P_rz.put(w, 0.0, 0u);
    }
    stores_arrived();
    __syncthreads();
    // ---- the team forms
    if (tid == 0) {
        if (!team_join(S.pcg, T, S.team_spin)) {
            s_ok = 0;
            xstore(glob(&L.out[s].pcg_fail), (int32_t)1);
        }
    }
    __syncthreads();
    if (!s_ok) return;  // the whole workgroup

    // the units' aggregates per level, and the ranges of this thread's items
    static_assert(kMasLevels == 3, "three levels' ranges");
    int na0[V], na1[V], na2[V];
    uint32_t rg0[V], rgc[V];  // level 0; level 1 or 2 in the wavefronts that sum those
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const Unit x = unit_at(v * G + ug);
        na0[v] = na1[v] = na2[v] = 0;
        rg0[v] = rgc[v] = 0;
        if (grp[v]) {
            na0[v] = __builtin_amdgcn_readfirstlane(x.lv[0]);
            na1[v] = nl > 1 ? __builtin_amdgcn_readfirstlane(x.lv[1]) : 0;
            na2[v] = nl > 2 ? __builtin_amdgcn_readfirstlane(x.lv[2]) : 0;
            const int i0 = tu >> kMasShare[0], i1 = lane >> kMasShare[1], i2 = lane >> kMasShare[2];
            if (i0 < 3 * na0[v]) rg0[v] = x.rng[i0 / 3];
            if (tu / kWave == 0 && i1 < 3 * na1[v]) rgc[v] = x.rng[na0[v] + i1 / 3];
            if (tu / kWave == 1 && i2 < 3 * na2[v]) rgc[v] = x.rng[na0[v] + na1[v] + i2 / 3];
        }
    }

    R p[V][3], r[V][3], z[V][3], d[V][3], M[V][9];
#pragma unroll
    for (int v = 0; v < V; ++v)
#pragma unroll
        for (int c = 0; c < 3; ++c) p[v][c] = r[v][c] = z[v][c] = d[v][c] = R(0);
    auto load_inverse = [&]() {
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (vid[v] >= 0)
#pragma unroll
                for (int c = 0; c < 9; ++c) M[v][c] = at(Mi, 9u * (uint32_t)vid[v])[c];
    };

    // z = M^-1 r for the units' vertices, published; this chunk's r.z partial
    // with tag `tag`. Ends with the partial on its way.
    auto precondition = [&](uint32_t tag) {
        double rz[V];
        R zo[V][3];
#pragma unroll
        for (int v = 0; v < V; ++v) {
            rz[v] = 0.0;
#pragma unroll
            for (int c = 0; c < 3; ++c) zo[v][c] = R(0);
            if (vid[v] >= 0) {
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    zo[v][a] = M[v][3 * a] * r[v][0] + M[v][3 * a + 1] * r[v][1] + M[v][3 * a + 2] * r[v][2];
                    rz[v] += (double)r[v][a] * (double)zo[v][a];
                }
                if (grp[v])
#pragma unroll
                    for (int c = 0; c < 3; ++c) unit_at(v * G + ug).rm[tu][c] = r[v][c];
            }
        }
        if (nl > 0) {
            __syncthreads();
#pragma unroll
            for (int v = 0; v < V; ++v)
                if (grp[v]) {
                    const Unit x = unit_at(v * G + ug);
                    mas_restrict<R>(na0[v], x.rm, x.ra, tu,
                                    [q = rg0[v], rng = x.rng](int, int a, bool first) { return !PMEM && first ? q : rng[a]; });
                }
            __syncthreads();
#pragma unroll
            for (int v = 0; v < V; ++v)
                if (grp[v]) {
                    const Unit x = unit_at(v * G + ug);
                    rz[v] += mas_coarse<R>(
                        nl, na0[v], na1[v], na2[v], x.rm, x.ra, tu,
                        [q = rgc[v], rng = x.rng + na0[v], n1 = na1[v]](int l, int a, bool first) {
                            return !PMEM && first ? q : rng[(l == 2 ? n1 : 0) + a];
                        },
                        [&](int q, int k) { return x.Dl[9 * q + k]; });
                }
            __syncthreads();
        }
#pragma unroll
        for (int v = 0; v < V; ++v) {
            if (vid[v] >= 0) {
                double zi[3] = {(double)zo[v][0], (double)zo[v][1], (double)zo[v][2]};
                if (grp[v])
#pragma unroll
                    for (int l = 0; l < kMasLevels; ++l) {
                        if (l >= nl) break;
#pragma unroll
                        for (int c = 0; c < 3; ++c) zi[c] += (double)unit_at(v * G + ug).rm[(loc[v] >> (8 * l)) & 0xffu][c];
                    }
#pragma unroll
                for (int c = 0; c < 3; ++c) z[v][c] = (R)zi[c];
                Z.store(vid[v], z[v], tag);
            }
            rz[v] = wave_sum(rz[v]);
            if (lane == 0) s_rz[v * NW + wave] = rz[v];
        }
        __syncthreads();
        if (tid == 0) {
            double t = 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u) t += (s_rz[4 * u] + s_rz[4 * u + 2]) + (s_rz[4 * u + 1] + s_rz[4 * u + 3]);
            if (s_ok) P_rz.put(w, t, tag);
        }
    };
    // the sum over all chunks, for every thread; false if a wait ran out
    auto total = [&](const Partials &P, uint32_t tag, double &t) {
        if (wave == 0) {
            bool ok;
            double v;
            switch ((T + kWave - 1) / kWave) {
            case 1: ok = P.sum<1>(T, tag, v); break;
            case 2: ok = P.sum<2>(T, tag, v); break;
            case 3: ok = P.sum<3>(T, tag, v); break;
            default: ok = P.sum<kTeamMax / kWave>(T, tag, v);
            }
            if (lane == 0) {
                s_tot = v;
                if (!ok) s_ok = 0;
            }
        }
        __syncthreads();
        t = wave_first(s_tot);
        return s_ok != 0;
    };

    // ---- start: p = 0, r = -g
    const auto g = glob(as<R>(S.grad));
#pragma unroll
    for (int v = 0; v < V; ++v)
        if (vid[v] >= 0)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                r[v][c] = -g[3 * (int64_t)vid[v] + c];
                if constexpr (PMEM) at(Sol, 3u * (uint32_t)vid[v])[c] = R(0);
            }
    load_inverse();
    precondition(1u);

    double stop = 0.0, rz_prev = 0.0;
    int done = 0, iters = 0;
    for (int it = 1;; ++it) {
#pragma unroll
        for (int k = 0; k < (NS + 1) / 2; ++k) lc[k] = here(lc[k]);
#pragma unroll
        for (int j = 0; j < HALO; ++j) hv[j] = here(hv[j]);
#pragma unroll
        for (int v = 0; v < V; ++v) {
            vid[v] = here(vid[v]);
            loc[v] = here(loc[v]);
        }
        ccol = here(ccol);
        crow = here(crow);
        tid = here(tid);
        tu = here(tu);
        lane = here(lane);
        const uint32_t tag = (uint32_t)it & 0xffffu;
        // z at the chunk's columns (and at the held contact block's)
        typename XVec<R>::Raw zr[HALO], zc, zo;
        auto columns = [&]() {
#pragma unroll
            for (int j = 0; j < HALO; ++j)
                if (j * NT < nh) Z.load(hv[j], zr[j]);  // uniform; ids past the list read vertex 0
            if (HOLD && cteam) {
                Z.load(ccol, zc);
                Z.load(crow, zo);
            }
            for (int k = 0;; ++k) {  // each until it is this iteration's
                bool ok = true;
#pragma unroll
                for (int j = 0; j < HALO; ++j)
                    if (j * NT < nh && !XVec<R>::is(zr[j], tag)) {
                        Z.load(hv[j], zr[j]);
                        ok = false;
                    }
                if (HOLD && cteam && !(XVec<R>::is(zc, tag) && XVec<R>::is(zo, tag))) {
                    Z.load(ccol, zc);
                    Z.load(crow, zo);
                    ok = false;
                }
                if (ok) return true;
                if (k == kTeamPoll) return false;
            }
        };
        double rz;
        if (!total(P_rz, (uint32_t)it, rz)) break;
        bool ok = columns();
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
        // the direction d = z + beta d_prev (beta and d_prev 0 at first) at the
        // chunk's columns and the units' vertices
        auto advance = [&](int i, const R (&zv)[3]) {
            R *const h = hd + i;
            const R o0 = h[0], o1 = h[H], o2 = h[2 * H];
            h[0] = zv[0] + rb * o0;
            h[H] = zv[1] + rb * o1;
            h[2 * H] = zv[2] + rb * o2;
        };
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int c = 0; c < 3; ++c) d[v][c] = z[v][c] + rb * d[v][c];
#pragma unroll
        for (int j = 0; j < HALO; ++j)
            if (tid + j * NT < nh) {
                R zv[3];
                XVec<R>::get(zr[j], zv);
                advance(tid + j * NT, zv);
            }
        for (int i = tid + HALO * NT; i < nh; i += NT) {
            R zv[3];
            ok &= Z.wait(glob(Hl)[h0 + i], tag, zv);
            advance(i, zv);
        }
        // contact rows: the held items, and the rows that are not held as the
        // launched form does, with directions from memory
        auto put_c = [&](int v, const double (&y)[3]) { C.store(v, y, tag); };
        auto items = [&]() {
            R zv[3];
            XVec<R>::get(zc, zv);
#pragma unroll
            for (int c = 0; c < 3; ++c) cd[c] = zv[c] + rb * cd[c];
            XVec<R>::get(zo, zv);
#pragma unroll
            for (int c = 0; c < 3; ++c) cown[c] = zv[c] + rb * cown[c];
            double t[3];
            contact_item<R>(chas, cA, cd, t);
            const int i = tid / kRowTeam;
            if (tid % kRowTeam == 0)
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    s_item[i][c] = t[c];
                    s_own[i][c] = cown[c];
                }
        };
        auto others = [&]() {
            struct Dir {
                XVec<R> Z, D;
                uint32_t tag;
                R rb;
                bool bon, ok;
                struct Raw {
                    typename XVec<R>::Raw z, d;
                };
                __device__ __forceinline__ Raw start(int v) const
                {
                    Raw x;
                    Z.load(v, x.z);
                    D.load(v, x.d);
                    return x;
                }
                __device__ __forceinline__ void end(int v, Raw &x, R (&o)[3])
                {
                    const uint32_t before = (tag - 1) & 0xffffu;
                    R dp[3] = {R(0), R(0), R(0)};
                    for (int n = 0; !(XVec<R>::is(x.z, tag) && (!bon || XVec<R>::is(x.d, before))); ++n) {
                        if (n == kTeamPoll) {
                            ok = false;
                            break;
                        }
                        x = start(v);
                    }
                    XVec<R>::get(x.z, o);
                    if (bon) XVec<R>::get(x.d, dp);
                    for (int c = 0; c < 3; ++c) o[c] = o[c] + rb * dp[c];
                }
            } dir{Z, (it & 1) ? DB : DA, tag, rb, bon, true};
            contact_rows<NT, R>(Cv, Cc, clist, hrows, ncrow, tid, dir, put_c, cdot);
            ok &= dir.ok;
        };
        // the rows' sums over their items, and the wavefront's part of d . q
        auto finish = [&]() {
            double t = 0.0;
            for (int h = lane; h < ncrow; h += kWave) {
                if (h >= hrows) {
                    t += cdot[h];
                    continue;
                }
                double a[3] = {0.0, 0.0, 0.0};
                const int i0 = s_at[h], i1 = s_at[h + 1];
                for (int i = i0; i < i1; ++i)
#pragma unroll
                    for (int c = 0; c < 3; ++c) a[c] += s_item[i][c];
                const R o[3] = {s_own[i0][0], s_own[i0][1], s_own[i0][2]};
                put_c(clist[h].row, a);
                t += contact_dot(o, a);
            }
            return t;
        };
        double cdq = 0.0;
        if (ncrow > 0) {
            if (HOLD && hrows > 0 && cteam) items();
            if (hrows < ncrow) others();
        }
        __syncthreads();
        // q = K d for the chunk's rows: even and odd slots in a sum each
        double dq = 0.0;
        {
            R y[2][3];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int c = 0; c < 3; ++c) y[h][c] = R(0);
#pragma unroll
            for (int k = 0; k < NS; ++k) {
                const int c = (int)((k & 1) ? lc[k / 2] >> 16 : lc[k / 2] & 0xffffu);
                R(&a)[3] = y[RT == 2 ? 0 : k % 2];
                if (k < RS) {
                    block_fma(m[k < RS ? k : 0], hd[c], hd[H + c], hd[2 * H + c], a[0], a[1], a[2]);
                } else {
                    R b[9];
#pragma unroll
                    for (int e = 0; e < 9; ++e) b[e] = ml[((k - RS) * 9 + e) * NT + tid];
                    block_fma(b, hd[c], hd[H + c], hd[2 * H + c], a[0], a[1], a[2]);
                }
            }
            for (int slot = s0 + part + RT * NS; slot < s1; slot += RT) {  // longer rows: the rest from memory
                const int c = glob(Lc)[(int64_t)slot * kSlice + ln];
                const auto B = glob(Bv) + (int64_t)slot * 9 * kSlice + ln;
                R a[9];
#pragma unroll
                for (int e = 0; e < 9; ++e) a[e] = B[e * kSlice];
                const bool odd = RT == 1 && ((slot - s0) & 1);
                R t[3];
#pragma unroll
                for (int e = 0; e < 3; ++e) t[e] = odd ? y[1][e] : y[0][e];
                block_fma(a, hd[c], hd[H + c], hd[2 * H + c], t[0], t[1], t[2]);
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    if (odd)
                        y[1][e] = t[e];
                    else
                        y[0][e] = t[e];
                }
            }
            double q[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                q[c] = (double)y[0][c];
                q[c] += RT == 2 ? quad_other<0xb1>(q[c]) : (double)y[1][c];
            }
            if (live && part == 0) {
                const int own = (int)(lc[0] & 0xffffu);  // slot 0 is the diagonal
                R qv[3], dv[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    qv[c] = (R)q[c];
                    dv[c] = hd[c * H + own];
                    dq += (double)dv[c] * (double)qv[c];
                }
                Q.store(row, qv, tag);
                if (touched) ((it & 1) ? DA : DB).store(row, dv, tag);  // for contact blocks that are not held
            }
        }
        // per 64 rows: the two halves' sums added
        if (contact && wave == 0) cdq = wave_sum(finish());
        dq = RT == 2 ? wave_sum(dq) : half_wave_sum(dq);
        if (RT == 1) dq += __shfl(dq, 32, kWave);
        if (lane == 0) s_dq[wave] = dq;
        if (!ok) s_ok = 0;
        __syncthreads();
        if (s_ok == 0) break;
        if (tid == 0) {
            double a = 0.0;
#pragma unroll
            for (int k = 0; k < NW; k += RT) a += RT == 2 ? s_dq[k] + s_dq[k + RT - 1] : s_dq[k];
            if (contact) a = a + cdq;
            P_dq.put(w, a, (uint32_t)it);
        }
        // q at the units' vertices and its contact part where there is one (in
        // the FP32 layouts with two vertices a thread one after the other: both
        // held too many registers)
        constexpr bool SPLIT = V > 1 && sizeof(R) == 4;
        typename XVec<R>::Raw qr[V];
        XVec<double>::Raw cr[V];
        auto fetch_both = [&]() {
#pragma unroll
            for (int v = 0; v < V; ++v) {
                if (vid[v] >= 0) Q.load(vid[v], qr[v]);
                if (vtouched[v]) C.load(vid[v], cr[v]);
            }
            for (int k = 0;; ++k) {
                bool all = true;
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    if (vid[v] >= 0 && !XVec<R>::is(qr[v], tag)) {
                        Q.load(vid[v], qr[v]);
                        all = false;
                    }
                    if (vtouched[v] && !XVec<double>::is(cr[v], tag)) {
                        C.load(vid[v], cr[v]);
                        all = false;
                    }
                }
                if (all) return true;
                if (k == kTeamPoll) return false;
            }
        };
        auto with_contact = [&](const XVec<double>::Raw &x, R (&q)[3]) {
            double qc[3];
            XVec<double>::get(x, qc);
#pragma unroll
            for (int c = 0; c < 3; ++c) q[c] = (R)((double)q[c] + qc[c]);
        };
        if constexpr (RT == 2) load_inverse();
        double dqt;
        if (!total(P_dq, (uint32_t)it, dqt)) break;
        if constexpr (RT == 1) load_inverse();  // not earlier: registers are short
        // a wait that ran out is seen before the next partial is published
        R qs[V][3];
        if constexpr (SPLIT) {
            auto fetch = [&](const auto &X, const bool (&on)[V], auto &x) {
#pragma unroll
                for (int v = 0; v < V; ++v)
                    if (on[v]) X.load(vid[v], x[v]);
                for (int k = 0;; ++k) {
                    bool all = true;
#pragma unroll
                    for (int v = 0; v < V; ++v)
                        if (on[v] && !X.is(x[v], tag)) {
                            X.load(vid[v], x[v]);
                            all = false;
                        }
                    if (all) return true;
                    if (k == kTeamPoll) return false;
                }
            };
            auto one_by_one = [&]() {
                typename XVec<R>::Raw xq[V];
                XVec<double>::Raw xc[V];
                bool on[V];
#pragma unroll
                for (int v = 0; v < V; ++v) on[v] = vid[v] >= 0;
                bool all = fetch(Q, on, xq);
#pragma unroll
                for (int v = 0; v < V; ++v)
                    if (on[v]) XVec<R>::get(xq[v], qs[v]);
                if (contact) {
                    all &= fetch(C, vtouched, xc);
#pragma unroll
                    for (int v = 0; v < V; ++v)
                        if (vtouched[v]) with_contact(xc[v], qs[v]);
                }
                return all;
            };
            if (!one_by_one()) s_ok = 0;
        } else if (!fetch_both()) {
            s_ok = 0;
        }
        // p += alpha d, r -= alpha q
        const R alpha = (R)(rz / dqt);
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (vid[v] >= 0) {
                R(&qv)[3] = qs[v];
                if constexpr (!SPLIT) {
                    XVec<R>::get(qr[v], qv);
                    if (vtouched[v]) with_contact(cr[v], qv);
                }
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    if constexpr (PMEM) {
                        const auto to = at(Sol, 3u * (uint32_t)vid[v]) + c;
                        *to = *to + alpha * d[v][c];
                    } else {
                        p[v][c] = p[v][c] + alpha * d[v][c];
                    }
                    r[v][c] = r[v][c] - alpha * qv[c];
                }
            }
        precondition((uint32_t)it + 1u);
    }
    if (!done) {  // a wait ran out (uniform over the workgroup)
        if (tid == 0) xstore(glob(&L.out[s].pcg_fail), (int32_t)1);
        return;
    }
    // ---- the solution and its largest component over free vertices
    double pm = 0.0;
#pragma unroll
    for (int v = 0; v < V; ++v)
        if (vid[v] >= 0) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                if constexpr (PMEM)
                    p[v][c] = at(Sol, 3u * (uint32_t)vid[v])[c];
                else
                    at(Sol, 3u * (uint32_t)vid[v])[c] = p[v][c];
            }
            if (!S.fixed[vid[v]])
                pm = fmax(pm, fmax(fabs((double)p[v][0]), fmax(fabs((double)p[v][1]), fabs((double)p[v][2]))));
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

static PhaseKind team_phase(int variant) { return variant == 0 ? kPhTeam0 : variant == 1 ? kPhTeam1 : kPhTeam2; }

template <class R>
static void launch_variant(Batch &b, int variant, size_t lds)
{
    const int N = team_threads(variant, sizeof(R));
    const PhaseKind ph = team_phase(variant);
    const int nb = b.blocks(ph);
    if (nb == 0) return;
    b.flush_phases();
    const Launch l = b.launch(ph);
    switch (variant) {
    case 0: hipLaunchKernelGGL((k_pcg_team<R, 0>), dim3(nb), dim3(N), lds, b.stream, l); break;
    case 1: hipLaunchKernelGGL((k_pcg_team<R, 1>), dim3(nb), dim3(N), lds, b.stream, l); break;
    default:
        if constexpr (sizeof(R) == 4) hipLaunchKernelGGL((k_pcg_team<R, kTeamCompact>), dim3(nb), dim3(N), lds, b.stream, l);
    }
    IPC_HIP(hipGetLastError());
}

void launch_pcg_team(Batch &b, const std::vector<uint8_t> &on)
{
    const size_t ns = b.sc.size();
    const bool mx = b.sc[0]->prm.precision == IPC_MIXED;
    const size_t rs = mx ? sizeof(float) : sizeof(double);
    // narrow teams that fill the CUs more than once: two workgroups a CU (a list
    // of 128 gels 84.8 -> 77.0 ms: 5.2 -> 4.0 ms a launch of 2,000 workgroups)
    int64_t narrow = 0;
    for (size_t i = 0; i < ns; ++i)
        if (on[i] && b.sc[i]->h.team_variant == 0) narrow += b.sc[i]->h.team_T;
    auto variant = [&](size_t i) {
        const SceneDev &h = b.sc[i]->h;
        const bool compact = mx && h.team_variant == 0 && narrow > kTeamMax &&
                             chunk_rows_bound(*b.sc[i], b.h_out[i]) <= kCompactRows &&
                             team_lds_bytes(kTeamCompact, h.team_H, h.team_A, rs) <= kTeamDyn / 2;
        return compact ? kTeamCompact : h.team_variant;
    };
    for (int v : {0, 1, kTeamCompact}) {
        std::vector<int32_t> nb(ns, 0);
        size_t lds = 0;
        for (size_t i = 0; i < ns; ++i) {
            const SceneDev &h = b.sc[i]->h;
            if (!on[i] || variant(i) != v) continue;
            b.sc[i]->pcg_compact += v == kTeamCompact;
            nb[i] = h.team_T;
            lds = std::max(lds, team_lds_bytes(v, h.team_H, h.team_A, rs));
        }
        b.set_phase(team_phase(v), nb);
        if (mx)
            launch_variant<float>(b, v, lds);
        else
            launch_variant<double>(b, v, lds);
    }
}

template <class R>
static void raise_lds()
{
    for (const void *f : {(const void *)k_pcg_team<R, 0>, (const void *)k_pcg_team<R, 1>})
        IPC_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kTeamDyn));
    if constexpr (sizeof(R) == 4)
        IPC_HIP(hipFuncSetAttribute((const void *)k_pcg_team<R, kTeamCompact>, hipFuncAttributeMaxDynamicSharedMemorySize, kTeamDyn));
}

void team_prepare_device()
{
    raise_lds<float>();
    raise_lds<double>();
}

}  // namespace ipcg
