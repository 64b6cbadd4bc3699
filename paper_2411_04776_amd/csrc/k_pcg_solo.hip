// k_pcg_solo.hip -- the whole PCG solve of a scene that one workgroup holds
// (up to 256 vertices in FP64, 512 in FP32), in one launch.
//
// Such a scene's iteration is a chain of a few dozen values through LDS; what
// bounds it is the chain's length, eight or so block barriers of some hundred
// cycles each. Matrix rows (a thread or two per row) and the update's vectors
// are in registers, z, the directions, q and the contact pairs' products in
// LDS; nothing leaves the CU until the solution is written. 90 vertices FP64:
// 21 us an iteration as launches of k_solver.hip, 6.7 here (252 vertices 21 and 7.7,
// 366 vertices mixed 24 and 9.7).
//
// Order of sums. A few dozen vertices make scenes whose outcome turns on the
// last bit (an indenter's vertex exactly over an edge of the gel's grid: the
// closest feature is a tie), so this form keeps the order in which launches of
// one step after the other add: K z and K d_prev apart, then beta; contact
// products pair by pair, a row's by eight lanes in turn and a tree, or, for a
// vertex outside the aggregates with more than kHeavyRow entries, by 256 lanes
// and a partial of r.z of its own; an aggregate's members one after the other,
// its level after the one below. No contact row is merged here: pairs are few,
// and their products cost less than the longer sums would move.
#include <type_traits>

#include "device_util.h"
#include "ipc_internal.h"

namespace ipcg {

template <class R>
__device__ __forceinline__ R *as(void *p)
{
    return reinterpret_cast<R *>(p);
}

constexpr int kSoloPairs = 512;  // contact pairs whose products are kept in LDS (the others': in c_val's space)
constexpr int kSoloTeam = 8;     // lanes that share a contact row's entries
constexpr int kSoloHeld = 3;     // of which a lane keeps the places of its first ones
// threads of a workgroup (FP64: 512 registers a thread for up to 128 vertices,
// 256 for up to 256; a thread a row in the largest FP32 layout, whose two
// threads a row would leave 128 registers each) and its update units
constexpr int solo_threads(size_t real, bool pair) { return real == 8 && pair ? 256 : 512; }
constexpr int solo_row_threads(size_t real, bool pair) { return real == 8 || pair ? 2 : 1; }
__host__ __device__ constexpr int solo_units(size_t real) { return real == 8 ? 2 : 4; }

struct SoloRow {
    int32_t row, e0, ne;  // vertex, first entry, entries (negative: summed by 256 lanes)
};

// A workgroup's LDS, in the order of the fields.
template <class R>
struct SoloLds {
    double *cq;            // contact part of q: cq[c * n + v]
    double *sdq;           // d.q of each row
    double *hp;            // r.z of the vertices with a partial of their own
    double *ppart;         // d.q of blocks of 64 pairs
    double (*ra)[3];       // the units' aggregate sums, A each
    R (*rm)[3];            // members' residuals, then corrections, kMasCapM a unit
    R *Dl;                 // aggregates' inverses, 9 A a unit
    R *z, *d, *q, *p;      // [c * n + v] each; d: of even iterations, then of odd ones
    R *Mi;                 // diagonal blocks' inverses: Mi[e * n + v]
    R *Y;                  // pair products, 12 a pair
    uint32_t *rng;         // aggregates' ranges (two 16-bit positions), A a unit
    SoloRow *rows;         // contact rows
    uint32_t *na;          // aggregates of a unit's levels, 9 bits each
    int32_t *ent;          // incidence entries
    uint16_t *pv;          // pairs' vertices, 4 each
    size_t bytes;
    __host__ __device__ SoloLds(char *base, int n, int A, int pairs)
    {
        constexpr int U = solo_units(sizeof(R));
        size_t at = 0;
        auto take = [&](auto *&p, size_t count) {
            p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(base + at);
            at += (count * sizeof(*p) + 7) / 8 * 8;
        };
        take(cq, 3 * (size_t)n);
        take(sdq, n);
        take(hp, n);
        take(ppart, kBlock);
        take(ra, (size_t)U * A);
        take(rm, (size_t)U * kMasCapM);
        take(Dl, 9 * (size_t)U * A);
        take(z, 3 * (size_t)n);
        take(d, 6 * (size_t)n);
        take(q, 3 * (size_t)n);
        take(p, 3 * (size_t)n);
        take(Mi, 9 * (size_t)n);
        take(Y, 12 * (size_t)pairs);
        take(rng, (size_t)U * A);
        take(rows, n);
        take(na, U);
        take(ent, 4 * (size_t)pairs);
        take(pv, 4 * (size_t)pairs);
        bytes = at;
    }
};

// the value N lanes further on in the same 16 (DPP row shift; zero past its end)
template <int N>
__device__ __forceinline__ double lane_on(double v)
{
    const uint64_t x = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)x, 0x100 + N, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(x >> 32), 0x100 + N, 0xf, 0xf, true);
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// The sum of the first 2 S lanes' values, by the distances S, ..., 1 of
// wave_sum's tree, on the first lane.
template <int S>
__device__ __forceinline__ double first_sum(double v)
{
    if constexpr (S > 4) v += lane_on<8>(v);
    if constexpr (S > 2) v += lane_on<4>(v);
    if constexpr (S > 1) v += lane_on<2>(v);
    if constexpr (S > 0) v += lane_on<1>(v);
    return v;
}

// PAIR: the layout for half the vertices (solo_threads). pairs: room for pair
// products in LDS.
//
// The update's positions (256 a unit, as a block each would hold them) are
// spread over the wavefronts, 64 at a time: a unit of 50 vertices takes one
// wavefront, not four.
template <class R, bool PAIR>
__global__ void __launch_bounds__(solo_threads(sizeof(R), PAIR), 1) k_pcg_solo(Launch L, int pairs)
{
    constexpr int NT = solo_threads(sizeof(R), PAIR), NW = NT / kWave, RT = solo_row_threads(sizeof(R), PAIR);
    constexpr int NP = kSpmvStreams / RT, NROW = NT / RT, U = solo_units(sizeof(R)), V = (NROW + 63 * U) / kWave > NW ? 2 : 1;
    static_assert((NROW + 63 * U) / kWave <= V * NW, "every position has a thread");
    static_assert(kSpmvStreams == 2, "a row's two streams");
    constexpr int NS = RT == 2 ? kTeamSlots : 2 * kTeamSlots - 1;  // blocks of a thread in registers
    constexpr int WU = kBlock / kWave;                             // wavefronts of a unit's positions
    extern __shared__ double solo_lds[];
    __shared__ double s_rz[U * WU], s_part[NROW / kRowsPerBlock];
    __shared__ uint64_t s_heavy[NW];
    __shared__ int s_cnt[NW];
    int lb;
    const int s = scene_of_block(L, lb);
    const SceneDev &S = *L.sc[s];
    int tid = (int)threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    // what the loop needs of the view, read here: after the kernel's first
    // store the compiler would read it by vector loads, a memory round trip
    // each; in scalar registers: a dozen LDS addresses are made from them
    auto uniform = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
    const int n = uniform(S.n), A = uniform(S.team_A), maxit = uniform(S.pcg_maxit), nl = uniform(S.mas_levels);
    const int nvp = uniform(S.pcg_nvp), nbr = uniform(S.nb_rows), ngrp = nl > 0 ? uniform(S.mas_ng) : 0;
    const double tol2 = S.pcg_tol2;
    const SoloLds<R> m(reinterpret_cast<char *>(solo_lds), n, A, pairs);
    const int npair = uniform(L.out[s].n_pair), nrow = uniform(L.out[s].n_crow);
    const bool inside = npair <= pairs;  // every pair's data is in LDS
    const int64_t cap = S.act_cap;
    const auto cl = glob((const int32_t *)S.c_list), av = glob((const int32_t *)S.act_v);
    const auto H = glob((const R *)as<R>(S.act_H));
    const auto Yg = glob(reinterpret_cast<R *>(S.c_val));  // products past the LDS: this solve reads no merged block

    // ---- this thread's matrix row, or its stream of one (slot k of the thread: part + RT * k)
    const int part = RT == 2 ? tid & 1 : 0;
    int row = tid / RT;
    const bool live = row < n;
    R K[NS][9];
    uint32_t lc[(NS + 1) / 2];  // two 16-bit columns each
    int s0 = 0, s1 = 0;
    const int ln = row % kSlice;
    if (live) {
        s0 = glob(S.slice_ptr)[row / kSlice];
        s1 = glob(S.slice_ptr)[row / kSlice + 1];
    }
    const auto bval = glob((const R *)as<R>(S.bval));
    const auto bcol = glob((const int32_t *)S.bcol);
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        // absent slots and rows: slot s0's place is read, zeros are kept
        const bool in = s0 + part + RT * k < s1;
        const int64_t slot = in ? s0 + part + RT * k : s0;
        const int col = in ? bcol[slot * kSlice + ln] : -1;
        const uint32_t c = (uint32_t)(col >= 0 ? col : min(row, n - 1));
        lc[k / 2] = (k & 1) ? lc[k / 2] | (c << 16) : c;
#pragma unroll
        for (int e = 0; e < 9; ++e) {
            const R v = bval[(slot * 9 + e) * kSlice + ln];
            K[k][e] = col >= 0 ? v : R(0);
        }
    }

    // ---- the units' aggregates, and this wavefront's positions: 64 of a unit, V times
    int unit[V], pos[V], vid[V];
    uint32_t loc[V];  // the vertex's aggregate at each level, 8 bits each
    static_assert(kMasCapA <= 256 && kMasLevels == 3, "8-bit positions of a group's aggregates, three levels");
    {
        const auto go = glob(S.mas_gofs), mb = glob(S.mas_mb), me = glob(S.mas_me);
        const size_t G1 = (size_t)S.mas_ng + 1;
#pragma unroll
        for (int v = 0; v < V; ++v) {
            unit[v] = vid[v] = -1;
            pos[v] = 0;
            loc[v] = 0;
        }
        for (int i = tid; i < U * WU; i += NT) s_rz[i] = 0.0;
        int w0 = 0;  // wavefronts of positions of the units before
        for (int u = 0; u < nvp; ++u) {
            const bool g = u < ngrp;
            const int k0 = g ? go[u] : (u - ngrp) * kBlock;
            const int cnt = g ? go[u + 1] - k0 : min((nl > 0 ? S.mas_nother : n) - k0, kBlock);
            const int nw = uniform((cnt + kWave - 1) / kWave);
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const int j = wave + v * NW - w0;
                if (j < 0 || j >= nw) continue;
                unit[v] = u;
                pos[v] = j * kWave + lane;
                if (pos[v] < cnt) {
                    const int k = k0 + pos[v];
                    vid[v] = g ? glob(S.mas_mem)[k] : nl > 0 ? glob(S.mas_other)[k] : k;
                }
            }
            w0 += nw;
            if (!g) continue;
            int base = 0, off = k0;
            uint32_t na = 0;
            for (int l = 0; l < nl; ++l) {
                const int a0 = go[(l + 1) * G1 + u], a1 = go[(l + 1) * G1 + u + 1];
#pragma unroll
                for (int v = 0; v < V; ++v)
                    if (unit[v] == u && vid[v] >= 0)
                        loc[v] |= (uint32_t)(base + glob(S.mas_manc)[(int64_t)l * S.mas_nf + k0 + pos[v]] - a0) << (8 * l);
                for (int a = a0 + tid; a < a1; a += NT) {  // its members, or its aggregates of the level below
                    const int64_t gid = (int64_t)S.mas_off[l] + a;
                    const int q = u * A + base + a - a0;
                    m.rng[q] = (uint32_t)(mb[gid] - off) | (uint32_t)(me[gid] - off) << 16;
                    for (int c = 0; c < 9; ++c) m.Dl[9 * q + c] = glob(as<R>(S.mas_dinv))[9 * gid + c];
                }
                na |= (uint32_t)(a1 - a0) << (9 * l);
                base += a1 - a0;
                off = a0;
            }
            if (tid == 0) m.na[u] = na;
        }
    }

    // ---- contact rows (in any order: each is summed by itself), and which
    // vertices have a partial of their own
    for (int i = tid; i < 3 * n; i += NT) {
        m.cq[i] = 0.0;
        m.p[i] = m.d[i] = m.d[3 * n + i] = R(0);
    }
    for (int i = tid; i < 9 * n; i += NT) m.Mi[(i % 9) * n + i / 9] = glob(as<R>(S.Minv))[i];
    for (int i = tid; i < n; i += NT) m.hp[i] = 0.0;
    {
        int ne = 0, e0 = 0;
        if (tid < n && npair > 0) {  // a thread per row: the scene has no more rows than threads
            e0 = glob(S.c_ptr)[tid];
            ne = glob(S.c_ptr)[tid + 1] - e0;
        }
        const unsigned long long b = __ballot(ne > 0), h = __ballot(ne > kHeavyRow);
        if (lane == 0) {
            s_cnt[wave] = __popcll(b);
            s_heavy[wave] = h;
        }
        __syncthreads();
        int at = __popcll(b & ((1ull << lane) - 1));
        for (int w = 0; w < wave; ++w) at += s_cnt[w];
        if (ne > 0) {
            const bool member = nl > 0 && glob(S.mas_vpos)[tid] >= 0;
            m.rows[at] = SoloRow{tid, e0, ne > kHeavyRow && !member ? -ne : ne};
        }
        const int entries = npair > 0 ? glob(S.c_ptr)[n] : 0;
        for (int t = tid; t < min(entries, 4 * pairs); t += NT) m.ent[t] = cl[t];
        for (int t = tid; t < 4 * min(npair, pairs); t += NT) m.pv[t] = (uint16_t)av[(int64_t)(t & 3) * cap + (t >> 2)];
    }
    int nheavy = 0, own[V];  // own: place of the vertex's own partial, or -1
    for (int w = 0; w < NW; ++w) nheavy += __popcll(s_heavy[w]);
    nheavy = uniform(nheavy);
#pragma unroll
    for (int v = 0; v < V; ++v) {
        own[v] = -1;
        if (vid[v] < 0 || unit[v] < ngrp || !(s_heavy[vid[v] / kWave] >> (vid[v] % kWave) & 1)) continue;
        int r = __popcll(s_heavy[vid[v] / kWave] & ((1ull << (vid[v] % kWave)) - 1));
        for (int w = 0; w < vid[v] / kWave; ++w) r += __popcll(s_heavy[w]);
        own[v] = r;
    }
    __syncthreads();
    // (in: every pair's data is in LDS)
    auto entry = [&](auto in, int t) {
        const int src = in || t < 4 * pairs ? m.ent[t] : cl[t];
        return 12 * (src >> 2) + 3 * (src & 3);  // its product's first component
    };
    auto vertex = [&](auto in, int p, int a) { return in || p < pairs ? (int)m.pv[4 * p + a] : av[(int64_t)a * cap + p]; };
    auto product = [&](auto in, int e) { return in || e < 12 * pairs ? m.Y[e] : Yg[e]; };
    using In = std::true_type;
    using Out = std::false_type;
    // kept in registers where there are enough: this thread's first pair row
    // with its vertices, the vertices of this lane's first pair of the d.q sums,
    // the places of its first entries of its team's first row, and of the first
    // level sums' ranges
    constexpr bool HOLD = PAIR;
    auto pair_row = [&](auto in, int x, R (&b)[9], int (&w)[3]) {  // row x % 12 of pair x / 12: its other vertices' blocks
        const int pr = x / 12, slot = (x - 12 * pr) / 3;
#pragma unroll
        for (int k = 0; k < 9; ++k) b[k] = H[12 * (int64_t)x + 3 * (k / 3 + (k / 3 >= slot ? 1 : 0)) + k % 3];
#pragma unroll
        for (int o = 0; o < 3; ++o) w[o] = vertex(in, pr, o + (o >= slot ? 1 : 0));
    };
    // pair rows go to the wavefronts that have no matrix row, where that is two
    // rounds or less, else to all, the last threads first
    const int idle = NT - (n * RT + kWave - 1) / kWave * kWave;
    const int PT = 12 * npair <= 2 * idle ? idle : NT;
    R hb[9];
    int hw[3] = {0, 0, 0};
    if (HOLD && inside && NT - 1 - tid < min(PT, 12 * npair)) pair_row(In{}, NT - 1 - tid, hb, hw);
    const int pb0 = NW - 1 - wave;  // blocks of 64 pairs: the last wavefronts' first
    int dv[4] = {0, 0, 0, 0};
    if (HOLD && inside && pb0 * kWave + lane < npair)
#pragma unroll
        for (int a = 0; a < 4; ++a) dv[a] = vertex(In{}, pb0 * kWave + lane, a);
    SoloRow hrow{0, 0, 0};
    int eo[kSoloHeld];
    const bool held = HOLD && inside && tid / kSoloTeam < nrow;
    if (held) hrow = m.rows[tid / kSoloTeam];
#pragma unroll
    for (int k = 0; k < kSoloHeld; ++k) {
        const int t = tid % kSoloTeam + kSoloTeam * k;
        eo[k] = held && t < hrow.ne ? entry(In{}, hrow.e0 + t) : -1;
    }
    uint32_t naU[U], naV[V], rg[kMasLevels];
#pragma unroll
    for (int u = 0; u < U; ++u) naU[u] = (uint32_t)uniform(u < ngrp ? (int)m.na[u] : 0);
#pragma unroll
    for (int v = 0; v < V; ++v) {
        unit[v] = uniform(unit[v]);
        naV[v] = (uint32_t)uniform(unit[v] >= 0 && unit[v] < ngrp ? (int)m.na[unit[v]] : 0);
    }
    auto level_n = [](uint32_t na, int l) { return (int)(na >> (9 * l) & 511u); };
    auto level_base = [&](uint32_t na, int l) { return (l > 0 ? level_n(na, 0) : 0) + (l > 1 ? level_n(na, 1) : 0) + (l > 2 ? level_n(na, 2) : 0); };
    // a level's sums: component c of aggregate a is item 3 a + c, the first
    // items the last threads' (the first ones form the level below's corrections)
#pragma unroll
    for (int l = 0; l < kMasLevels; ++l) {
        const int i = NT - 1 - tid;
        rg[l] = HOLD && i < 3 * level_n(naU[0], l) ? m.rng[level_base(naU[0], l) + i / 3] : 0u;
    }

    R r[V][3], zo[V][3];
    double rz[V];
#pragma unroll
    for (int v = 0; v < V; ++v)
        if (vid[v] >= 0)
#pragma unroll
            for (int c = 0; c < 3; ++c) r[v][c] = -glob(as<R>(S.grad))[3 * vid[v] + c];

    // z = M^-1 r for the units' vertices and the parts of r.z; ends before the
    // barrier after which they are there. first: the start, without own partials
    auto precondition = [&](bool first) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
            rz[v] = 0.0;
            if (unit[v] < 0 || vid[v] < 0) continue;
            R M[9];
#pragma unroll
            for (int e = 0; e < 9; ++e) M[e] = m.Mi[e * n + vid[v]];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                zo[v][a] = M[3 * a] * r[v][0] + M[3 * a + 1] * r[v][1] + M[3 * a + 2] * r[v][2];
                rz[v] += (double)r[v][a] * (double)zo[v][a];
            }
            if (unit[v] < ngrp)
#pragma unroll
                for (int a = 0; a < 3; ++a) m.rm[unit[v] * kMasCapM + pos[v]][a] = r[v][a];
            if (own[v] >= 0 && !first) {
                m.hp[own[v]] = rz[v];
                rz[v] = 0.0;
            }
        }
        if (nl > 0) {
            __syncthreads();
#pragma unroll
            for (int l = 0; l <= kMasLevels; ++l) {
                if (l > nl) break;
                if (l > 0)  // the corrections of the level below
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        if (unit[v] < 0 || unit[v] >= ngrp || pos[v] >= level_n(naV[v], l - 1)) continue;
                        const int a = level_base(naV[v], l - 1) + pos[v];
                        const R *D = m.Dl + 9 * (unit[v] * A + a);
                        const double *x = m.ra[unit[v] * A + a];
                        R(&to)[3] = m.rm[unit[v] * kMasCapM + a];
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            const R e = D[3 * c] * (R)x[0] + D[3 * c + 1] * (R)x[1] + D[3 * c + 2] * (R)x[2];
                            to[c] = e;
                            rz[v] += x[c] * (double)e;
                        }
                    }
                if (l < nl)
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        if (u >= ngrp) break;
                        const int na = level_n(naU[u], l), below = l > 0 ? level_base(naU[u], l - 1) : 0;
                        const auto rm = m.rm + u * kMasCapM;
                        const auto ra = m.ra + u * A;
                        for (int i = NT - 1 - tid; i < 3 * na; i += NT) {
                            const int a = level_base(naU[u], l) + i / 3, c = i % 3;
                            const uint32_t g = HOLD && u == 0 && i < NT ? rg[l < kMasLevels ? l : 0] : m.rng[u * A + a];
                            const int j1 = (int)(g >> 16);
                            constexpr int W = 8;  // reads in flight
                            int j = (int)(g & 0xffffu);
                            double acc = 0.0;
                            auto some = [&](auto all) {  // past the end: other values of the LDS, not added
                                double x[W];
#pragma unroll
                                for (int k = 0; k < W; ++k) x[k] = l == 0 ? (double)rm[j + k][c] : ra[below + j + k][c];
#pragma unroll
                                for (int k = 0; k < W; ++k) acc += all || j + k < j1 ? x[k] : -0.0;
                            };
                            for (; j + W <= j1; j += W) some(In{});
                            some(Out{});
                            ra[a][c] = acc;
                        }
                    }
                __syncthreads();
            }
        }
#pragma unroll
        for (int v = 0; v < V; ++v) {
            if (unit[v] < 0) continue;
            if (vid[v] >= 0) {
                double zi[3] = {(double)zo[v][0], (double)zo[v][1], (double)zo[v][2]};
                if (unit[v] < ngrp)
#pragma unroll
                    for (int l = 0; l < kMasLevels; ++l) {
                        if (l >= nl) break;
#pragma unroll
                        for (int c = 0; c < 3; ++c) zi[c] += (double)m.rm[unit[v] * kMasCapM + (int)((loc[v] >> (8 * l)) & 0xffu)][c];
                    }
#pragma unroll
                for (int c = 0; c < 3; ++c) m.z[c * n + vid[v]] = (R)zi[c];
            }
            rz[v] = wave_sum(rz[v]);
            if (lane == 0) s_rz[unit[v] * WU + pos[v] / kWave] = rz[v];
        }
    };
    precondition(true);
    __syncthreads();

    double stop = 0.0, rz_prev = 0.0;
    int done = 0, iters = 0;
    for (int it = 1;; ++it) {
#pragma unroll
        for (int k = 0; k < (NS + 1) / 2; ++k) lc[k] = here(lc[k]);
#pragma unroll
        for (int v = 0; v < V; ++v) {
            vid[v] = here(vid[v]);
            loc[v] = here(loc[v]);
            pos[v] = here(pos[v]);
        }
#pragma unroll
        for (int k = 0; k < kSoloHeld; ++k) eo[k] = here(eo[k]);
#pragma unroll
        for (int k = 0; k < 4; ++k) dv[k] = here(dv[k]);
#pragma unroll
        for (int k = 0; k < 3; ++k) hw[k] = here(hw[k]);
        tid = here(tid);
        lane = here(lane);
        row = here(row);
        const bool bon = it > 1;
        R *const dn = m.d + (it & 1) * 3 * n, *const dp = m.d + ((it & 1) ^ 1) * 3 * n;
        // K z and K d_prev, a stream's slots one after the other
        R yz[NP][3], yd[NP][3];
#pragma unroll
        for (int h = 0; h < NP; ++h)
#pragma unroll
            for (int c = 0; c < 3; ++c) yz[h][c] = yd[h][c] = R(0);
        auto apply = [&](const R (&a)[9], int c, R (&o)[3], R (&w)[3]) {
            const R z0 = m.z[c], z1 = m.z[n + c], z2 = m.z[2 * n + c];
            const R d0 = dp[c], d1 = dp[n + c], d2 = dp[2 * n + c];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                o[i] += a[3 * i] * z0 + a[3 * i + 1] * z1 + a[3 * i + 2] * z2;
                w[i] += a[3 * i] * d0 + a[3 * i + 1] * d1 + a[3 * i + 2] * d2;
            }
        };
        if (wave * (kWave / RT) < n)
#pragma unroll
            for (int k = 0; k < NS; ++k)
                apply(K[k], (int)((k & 1) ? lc[k / 2] >> 16 : lc[k / 2] & 0xffffu), yz[k % NP], yd[k % NP]);
        for (int q = s0 + part + RT * NS; q < s1; q += RT) {  // longer rows: the rest from memory
            const int c = bcol[(int64_t)q * kSlice + ln];
            if (c < 0) continue;
            R a[9];
#pragma unroll
            for (int e = 0; e < 9; ++e) a[e] = bval[((int64_t)q * 9 + e) * kSlice + ln];
            if (NP == 1 || !((q - s0) & 1))
                apply(a, c, yz[0], yd[0]);
            else
                apply(a, c, yz[NP - 1], yd[NP - 1]);
        }
        // r.z, the same in every wavefront: the units' parts, then the own ones
        double acc = 0.0;
        for (int u = lane; u < nvp + nheavy; u += kWave)
            acc += u < nvp ? (s_rz[4 * u] + s_rz[4 * u + 2]) + (s_rz[4 * u + 1] + s_rz[4 * u + 3]) : m.hp[u - nvp];
        static_assert(WU == 4, "a unit's four wavefronts");
        const double rzt = wave_first(nvp + nheavy <= 16 ? first_sum<8>(acc) : wave_sum(acc));
        double beta = 0.0;
        if (!bon) {
            if (!(rzt > 0.0)) {
                done = 1;
                break;
            }
            stop = tol2 * rzt;
        } else {
            const bool conv = rzt <= stop;
            if (conv || it > maxit) {
                done = conv ? 1 : 2;
                iters = it - 1;
                break;
            }
            beta = rzt / rz_prev;
        }
        rz_prev = rzt;
        const R rb = (R)beta;
        auto direction = [&](int v, int c) { return m.z[c * n + v] + rb * dp[c * n + v]; };  // at first 0 and 0: z
        // d, q = K_el d and d.q of the rows
        {
            double y[3], dq = 0.0;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                y[c] = (double)yz[0][c] + beta * (double)yd[0][c];
                if constexpr (RT == 2)
                    y[c] += quad_other<0xb1>(y[c]);
                else
                    y[c] += (double)yz[NP - 1][c] + beta * (double)yd[NP - 1][c];
            }
            if (live && part == 0) {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const R dv = direction(row, c), qv = (R)y[c];
                    dn[c * n + row] = dv;
                    m.q[c * n + row] = qv;
                    dq += (double)dv * (double)qv;
                }
                m.sdq[row] = dq;
            }
        }
        // y_a = sum over b != a of H_ab d_b: a thread per pair, slot a and component
        auto pair_products = [&](auto in) {
            auto put = [&](int x, const R (&b)[9], const int (&w)[3]) {
                double y = 0.0;
#pragma unroll
                for (int o = 0; o < 3; ++o)
                    y += (double)(b[3 * o] * direction(w[o], 0) + b[3 * o + 1] * direction(w[o], 1) + b[3 * o + 2] * direction(w[o], 2));
                if (in || x < 12 * pairs)
                    m.Y[x] = (R)y;
                else
                    Yg[x] = (R)y;
            };
            int x = NT - 1 - tid < PT ? NT - 1 - tid : 12 * npair;
            if constexpr (HOLD && in) {
                if (x < 12 * npair) put(x, hb, hw);
                x += PT;
            }
            for (; x < 12 * npair; x += PT) {
                R b[9];
                int w[3];
                pair_row(in, x, b, w);
                put(x, b, w);
            }
        };
        if (inside)
            pair_products(In{});
        else
            pair_products(Out{});
        __syncthreads();
        // d.q of 64 rows and of 64 pairs at a time, and the rows' sums over their pairs
        for (int b = wave; b < nbr; b += NW) {
            const int i = b * kRowsPerBlock + lane;
            const double t = wave_sum(i < n ? m.sdq[i] : 0.0);
            if (lane == 0) s_part[b] = t;
        }
        auto pair_sums = [&](auto in) {
            for (int b = pb0; b * kWave < npair; b += NW) {
                const int pr = min(b * kWave + lane, npair - 1);
                double dy = 0.0;
#pragma unroll
                for (int h = 0; h < 2; ++h) {  // two slots' reads at a time
                    double x[6], y[6];
#pragma unroll
                    for (int e = 0; e < 6; ++e) {
                        const int a = 2 * h + e / 3, v = HOLD && in && b == pb0 ? dv[a] : vertex(in, pr, a);
                        x[e] = (double)dn[(e % 3) * n + v];
                        y[e] = (double)product(in, 12 * pr + 6 * h + e);
                    }
#pragma unroll
                    for (int e = 0; e < 6; ++e) dy += x[e] * y[e];
                }
                dy = wave_sum(b * kWave + lane < npair ? dy : 0.0);
                if (lane == 0) m.ppart[b % kBlock] = b < kBlock ? dy : m.ppart[b % kBlock] + dy;
            }
        };
        auto team_sum = [&](auto in, const SoloRow &w, double (&a)[3], int t) {  // from the lane's entry t on
            for (; t < w.ne; t += kSoloTeam) {
                const int e = entry(in, w.e0 + t);
#pragma unroll
                for (int c = 0; c < 3; ++c) a[c] += (double)product(in, e + c);
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                a[c] += lane_on<4>(a[c]);
                a[c] += lane_on<2>(a[c]);
                a[c] += lane_on<1>(a[c]);
                if (tid % kSoloTeam == 0 && w.ne > 0) m.cq[c * n + w.row] = a[c];
            }
        };
        auto row_sums = [&](auto in, int h) {  // rows h, h + teams, ...; then the rows of 256 lanes
            for (; h < nrow; h += NT / kSoloTeam) {
                double a[3] = {0.0, 0.0, 0.0};
                team_sum(in, m.rows[h], a, tid % kSoloTeam);
            }
            if (nheavy > 0)
                for (h = wave; h < nrow; h += NW) {
                    const SoloRow w = m.rows[h];
                    if (w.ne > 0) continue;
                    double tot[3] = {0.0, 0.0, 0.0};
                    for (int k = 0; k < kBlock / kWave; ++k) {
                        double a[3] = {0.0, 0.0, 0.0};
                        for (int t = k * kWave + lane; t < -w.ne; t += kBlock) {
                            const int e = entry(in, w.e0 + t);
#pragma unroll
                            for (int c = 0; c < 3; ++c) a[c] += (double)product(in, e + c);
                        }
#pragma unroll
                        for (int c = 0; c < 3; ++c) tot[c] += wave_sum(a[c]);
                    }
                    if (lane < 3) m.cq[lane * n + w.row] = lane == 0 ? tot[0] : lane == 1 ? tot[1] : tot[2];
                }
        };
        if (inside) {
            if (held) {
                R x[kSoloHeld][3];
                double a[3] = {0.0, 0.0, 0.0};
#pragma unroll
                for (int k = 0; k < kSoloHeld; ++k)
#pragma unroll
                    for (int c = 0; c < 3; ++c) x[k][c] = eo[k] >= 0 ? m.Y[eo[k] + c] : R(-0.0);  // adds nothing
#pragma unroll
                for (int k = 0; k < kSoloHeld; ++k)
#pragma unroll
                    for (int c = 0; c < 3; ++c) a[c] += (double)x[k][c];
                team_sum(In{}, hrow, a, tid % kSoloTeam + kSoloTeam * kSoloHeld);
            }
            pair_sums(In{});
            row_sums(In{}, tid / kSoloTeam + (HOLD ? NT / kSoloTeam : 0));
        } else {
            pair_sums(Out{});
            row_sums(Out{}, tid / kSoloTeam);
        }
        __syncthreads();
        // alpha = r.z / d.q, the same in every wavefront
        const int nbp = (npair + kWave - 1) / kWave;
        const double dqr = wave_first(first_sum<NROW / kRowsPerBlock / 2>(lane < nbr ? s_part[lane] : 0.0));
        double dqp = 0.0;
        if (nbp <= 16)
            dqp += wave_first(first_sum<8>(lane < nbp ? m.ppart[lane] : 0.0));
        else
            for (int k = 0; k < WU; ++k)
                if (k * kWave < nbp) dqp += wave_sum(k * kWave + lane < nbp ? m.ppart[k * kWave + lane] : 0.0);
        const R alpha = (R)(rzt / (dqr + dqp));
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (unit[v] >= 0 && vid[v] >= 0)
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const int i = c * n + vid[v];
                    const R qv = (R)((double)m.q[i] + m.cq[i]);
                    m.p[i] = m.p[i] + alpha * dn[i];
                    r[v][c] = r[v][c] - alpha * qv;
                }
        precondition(false);
        __syncthreads();
    }
    // ---- the solution and its largest component over free vertices
    double pm = 0.0;
#pragma unroll
    for (int v = 0; v < V; ++v)
        if (vid[v] >= 0) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const R x = m.p[c * n + vid[v]];
                glob(as<R>(S.sol))[3 * vid[v] + c] = x;
                if (!S.fixed[vid[v]]) pm = fmax(pm, fabs((double)x));
            }
        }
    pm = wave_max(pm);
    if (lane == 0 && pm > 0.0)  // non-negative doubles order like their bits
        atomicMax(reinterpret_cast<unsigned long long *>(&L.out[s].pinf), (unsigned long long)__double_as_longlong(pm));
    if (tid == 0) {
        S.pcg->done = 1;
        S.pcg->iters = iters;
        L.out[s].pcg_done = done;
        L.out[s].pcg_iters = iters;
    }
}

// ---- host ------------------------------------------------------------------

// the scenes with on[i] whose rows have two threads each (PAIR), or one
template <class R, bool PAIR>
static void launch_rows(Batch &b, const std::vector<uint8_t> &on)
{
    const PhaseKind ph = PAIR ? kPhSolo0 : kPhSolo1;
    const size_t ns = b.sc.size();
    std::vector<int32_t> nb(ns, 0);
    int64_t pairs = 1;
    size_t none = 0, lds = 0;
    for (size_t i = 0; i < ns; ++i)
        if (on[i] && b.sc[i]->h.team_variant == (PAIR ? kTeamSoloPair : kTeamSolo)) {
            nb[i] = 1;
            pairs = std::max(pairs, pair_count(*b.sc[i], b.h_out[i]));
            none = std::max(none, SoloLds<R>(nullptr, b.sc[i]->h.n, b.sc[i]->h.team_A, 0).bytes);
        }
    b.set_phase(ph, nb);
    if (b.blocks(ph) == 0) return;
    // room for the pairs of the list's fullest scene, as far as the LDS goes
    constexpr int64_t per_pair = 12 * sizeof(R) + 4 * sizeof(int32_t) + 4 * sizeof(uint16_t);
    pairs = std::min({pairs, (int64_t)kSoloPairs, ((int64_t)kTeamDyn - (int64_t)none) / per_pair});
    for (size_t i = 0; i < ns; ++i)
        if (nb[i]) lds = std::max(lds, SoloLds<R>(nullptr, b.sc[i]->h.n, b.sc[i]->h.team_A, (int)pairs).bytes);
    b.flush_phases();
    hipLaunchKernelGGL((k_pcg_solo<R, PAIR>), dim3(b.blocks(ph)), dim3(solo_threads(sizeof(R), PAIR)), lds, b.stream,
                       b.launch(ph), (int)pairs);
    IPC_HIP(hipGetLastError());
}

void launch_pcg_solo(Batch &b, const std::vector<uint8_t> &on)
{
    if (b.sc[0]->prm.precision == IPC_MIXED) {
        launch_rows<float, true>(b, on);
        launch_rows<float, false>(b, on);
    } else {
        launch_rows<double, true>(b, on);
        launch_rows<double, false>(b, on);
    }
}

void solo_prepare_device()
{
    for (const void *f : {(const void *)k_pcg_solo<double, true>, (const void *)k_pcg_solo<double, false>,
                          (const void *)k_pcg_solo<float, true>, (const void *)k_pcg_solo<float, false>})
        IPC_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kTeamDyn));
}

}  // namespace ipcg
