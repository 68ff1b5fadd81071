// hx_maxflow.hip -- maximum flow of every candidate's network (Sec. 3.3) on gfx950.
//
// The paper solves each network with preflow-push.  Here a segment of SEG lanes owns one
// candidate and runs a synchronous push-relabel with the candidate's whole residual graph
// in LDS, one lane per node.  Small networks (SEG <= 64, e.g. <= 16 replicas per side) pack
// 64/SEG candidates into one wavefront, so a wave's rounds serve several candidates at
// once; larger networks (per-GPU nodes) take a workgroup of SEG = 128 or 256 lanes each.
//
// Network.  In the Sec. 3.3 network every replica is an in -> out chain with one edge in
// and the KV edges out (prefill) or the KV edges in and one edge out (decode), so the
// chains contract without changing any s-t cut: prefill node p gets a_p = min(src, p_cap)
// from the source, decode node d sends b_d = min(d_cap, sink) to the sink, and c_pd are the
// KV edges.  The contracted graph is bipartite: s -> P -> D -> t.
//
// Algorithm (Goldberg-Tarjan push-relabel, in synchronous rounds; the packed plans' form -- the workgroup
// plans run on bit words, push_relabel_bits).  The source sits at
// height V = P + D + 2, the sink at 0.  A round has two phases separated by barriers:
//   P-phase: each active prefill node pushes along its admissible arcs (to decode nodes one
//            level lower, then back to the source), then relabels if excess remains;
//   D-phase: each active decode node pushes to the sink and back along its reverse KV arcs,
//            then relabels if excess remains.
// Within a phase the active nodes lie on one side of the bipartition, so their pushes touch
// disjoint arcs and their relabels read only the other side's heights, which that phase never
// changes: the phase equals some sequential order of the same push/relabel operations, and
// the usual termination and optimality arguments apply.  Excess arriving at the other side
// is added with LDS atomics.  Exact heights (BFS distances to the sink, else V + distance to
// the source) are recomputed every few rounds by label-correcting sweeps (global relabel).
// A candidate is done when none of its nodes has excess: the preflow is then a maximum flow.
//
// Shortcuts.  Nodes that can carry nothing (a = 0 or b = 0) leave most networks trivial.
// Single-wavefront plans: if one side has a single node that can, the network is a star and
// its maximum flow has a closed form (with a flow that fills the star's arcs in node order).
// Every plan: if every KV arc can carry min(a_i, b_j), the maximum flow is min(sum a, sum b)
// with the north-west-corner flow (below).  Single-wavefront plans, value only: if the
// smaller side has m <= kEnumMax nodes that can carry flow, the minimum cut is taken over the
// 2^m ways to split that side.  Push-relabel runs for the rest; every path gives the unique
// maximum-flow value.
//
// Outputs: the flow value, the flow on every KV edge, and the canonical minimum cut (nodes of
// the uncontracted network reachable from the source in the residual graph).
#include <limits.h>

#include "hx_internal.h"

namespace hx {
namespace {

constexpr int kGlobalRelabelEvery = 2;  // rounds between exact relabels
// Largest smaller side whose 2^m minimum-cut subsets are enumerated when only the flow value
// is wanted (64 subsets over a candidate's lanes).
constexpr int kEnumMax = 6;
constexpr int kPackedLanes = 64;  // workgroup size for packed segments: one wavefront

struct MfLayout {
    int32_t* cap;   // [P][Ds] KV capacities, row stride Ds = D | 1 (odd: no bank conflicts)
    int32_t* fl;    // [P][Ds] KV flows
    int32_t* a;     // [P] source -> p capacity
    int32_t* fs;    // [P] source -> p flow
    int32_t* ep;    // [P] excess
    int32_t* hp;    // [P] height
    int32_t* b;     // [D] d -> sink capacity
    int32_t* ft;    // [D] d -> sink flow
    int32_t* ed;    // [D] excess
    int32_t* hd;    // [D] height
    int32_t* misc;  // [4] scalars
};

__host__ __device__ inline size_t mf_words(int max_p, int max_d, int max_pd) {
    return 2 * ((size_t)max_pd + max_p) + 4 * (size_t)max_p + 4 * (size_t)max_d + 4;
}

__device__ inline MfLayout carve(int32_t* sm, int max_p, int max_d, int max_pd, bool heights) {
    MfLayout L;
    const int arc = max_pd + max_p;  // P*(D|1) <= P*D + P
    L.cap = sm;
    L.fl = L.cap + arc;
    L.a = L.fl + arc;
    L.fs = heights ? L.a + max_p : L.a;
    L.ep = L.fs + max_p;
    L.hp = L.ep + max_p;
    L.b = heights ? L.hp + max_p : L.hp;
    L.ft = L.b + max_d;
    L.ed = L.ft + max_d;
    L.hd = L.ed + max_d;
    L.misc = heights ? L.hd + max_d : L.hd;
    return L;
}
// Plans whose every network runs on bit words (workgroup plans of at most 256 rows a side) need no
// heights, and the source flows can take the place of the source capacities (they start equal, and
// whoever changes the flows has read the capacities): four networks of 128 GPUs then share a CU, not three.
__host__ __device__ inline bool mf_heights(int seg, int max_p, int max_d) {
    return seg <= 64 || max_p > seg || max_d > seg;
}

// (The functions of a tile that take the layout are inlined by force: left as calls in the 256-lane kernels,
// they gave every wavefront a stack in scratch memory, and launches whose networks the passes before had
// settled took 94 us instead of 55 at 100 x 70 nodes x 512.)
//
// Exact heights by label-correcting sweeps: hd = 1 where d -> t has residual, hp = V + 1 where
// p -> s has residual (reverse of a used source edge), then relax along residual arcs.  Every
// lane of the workgroup calls it (barriers inside); lane l of a segment owns node l, l+SEG, ...
template <int SEG>
__device__ __forceinline__ void global_relabel(const MfLayout& L, int l, int P, int D, int Ds, int V, int INF) {
    for (int i = l; i < P; i += SEG) L.hp[i] = L.fs[i] > 0 ? V + 1 : INF;
    for (int j = l; j < D; j += SEG) L.hd[j] = L.b[j] - L.ft[j] > 0 ? 1 : INF;
    __syncthreads();
    for (;;) {
        bool changed = false;
        for (int i = l; i < P; i += SEG) {
            int h = L.hp[i];
            const int32_t* c = L.cap + i * Ds;
            const int32_t* f = L.fl + i * Ds;
            for (int d = 0; d < D; ++d)
                if (c[d] - f[d] > 0 && L.hd[d] + 1 < h) h = L.hd[d] + 1;
            if (h < L.hp[i]) {
                L.hp[i] = h;
                changed = true;
            }
        }
        __syncthreads();
        for (int j = l; j < D; j += SEG) {
            int h = L.hd[j];
            for (int q = 0; q < P; ++q)
                if (L.fl[q * Ds + j] > 0 && L.hp[q] + 1 < h) h = L.hp[q] + 1;
            if (h < L.hd[j]) {
                L.hd[j] = h;
                changed = true;
            }
        }
        if (!__syncthreads_or(changed)) break;
    }
}

// Push-relabel of the workgroup plans, by one wavefront of the workgroup: lane l owns prefill and
// decode nodes l, l + 64, ... (up to SEG a side), with the residual arcs as bit words: room[i] the
// decode nodes that prefill i can still push to, used[j] the prefill nodes that decode j holds flow of.
// Exact distances to the sink are formed anew in every round, a level at a time: a node joins the
// level when its words meet the last level's (a ballot per 64 nodes), and the bits that met are its
// admissible arcs.  A phase then walks those arcs alone, four at a time so that their LDS reads
// overlap.  Excess that cannot reach the sink stays where it is and is taken back at the end: a decode
// node returns it over its used arcs and a prefill node to the source, which leaves a maximum flow of
// the same value (when only the value is asked for, it is left).
// What bounds it: the latency of the dependent LDS accesses along a node's arcs; one wavefront needs
// no barrier, and the networks in flight are bound by their LDS (four per CU at 128 GPUs).  4,096
// networks of 16 to 64 nodes a side 1,836 -> 350 us, against a lane per node that scanned its whole row in
// every push and every sweep of a global relabel, with barriers between the phases (two wavefronts and
// barriers on bit words: 492).
template <int SEG>
struct MfBits {
    static constexpr int kM = SEG / 64;
    uint64_t room[SEG][kM], used[SEG][kM];
};

__device__ __forceinline__ void mf_wave_sync() {
    __builtin_amdgcn_s_waitcnt(0xC07F);  // LDS atomics landed (lgkmcnt(0))
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The bit words of the flow in L (flows: it is not all zero), by every lane l of the workgroup (followed by
// a barrier).  Eight LDS reads at a time, the last repeated past the end: one after another they made the
// flows and cuts of 1,024 networks of 100 x 27 nodes without flow 38 us instead of 35.
template <int SEG>
__device__ __forceinline__ void residual_bits(MfBits<SEG>& S, const MfLayout& L, int l, int P, int D, int Ds,
                                              bool flows) {
    constexpr int kM = MfBits<SEG>::kM;
    auto word = [](int n, auto bit) {  // bits 0 .. n - 1
        uint64_t m = 0;
        for (int x0 = 0; x0 < n; x0 += 8)
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int x = x0 + k < n ? x0 + k : n - 1;
                m |= (uint64_t)bit(x) << x;
            }
        return m;
    };
#pragma unroll
    for (int w = 0; w < kM; ++w) {
        if (l < P) {
            const int32_t *c = L.cap + l * Ds + 64 * w, *fl = L.fl + l * Ds + 64 * w;
            const int n = D - 64 * w < 64 ? D - 64 * w : 64;
            S.room[l][w] = flows ? word(n, [&](int x) { return c[x] - fl[x] > 0; })
                                 : word(n, [&](int x) { return c[x] > 0; });
        }
        if (l < D) {
            const int32_t* fl = L.fl + 64 * w * Ds + l;
            const int n = P - 64 * w < 64 ? P - 64 * w : 64;
            S.used[l][w] = flows ? word(n, [&](int x) { return fl[x * Ds] > 0; }) : 0;
        }
    }
}

// Decode node j returns up to e of its excess over the arcs of word w in m; returns the rest.
template <int SEG, bool kStats>
__device__ __forceinline__ int32_t push_back(MfBits<SEG>& S, const MfLayout& L, int j, int w, uint64_t m, int32_t e,
                                             int Ds, unsigned long long& pushes) {
    while (m && e > 0) {
        int x[4], n = 0;
        int32_t f0[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            x[k] = m ? __builtin_ctzll(m) : (k ? x[k - 1] : 0);
            n += m != 0;
            m &= m - 1;  // 0 stays 0
            f0[k] = L.fl[(64 * w + x[k]) * Ds + j];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int32_t amt = k < n ? (f0[k] < e ? f0[k] : e) : 0;
            if (amt > 0) {
                const int i = 64 * w + x[k];
                L.fl[i * Ds + j] = f0[k] - amt;
                e -= amt;
                atomicAdd(&L.ep[i], amt);
                atomicOr((unsigned long long*)&S.room[i][j >> 6], 1ull << (j & 63));
                if (amt == f0[k]) atomicAnd((unsigned long long*)&S.used[j][w], ~(1ull << x[k]));
                if (kStats) ++pushes;
            }
        }
    }
    return e;
}

// Returns whether active excess is left (the round budget ran out).  One wavefront; S holds the bit
// words of L's flow.
template <int SEG, bool kStats>
__device__ __forceinline__ bool push_relabel_bits(MfBits<SEG>& S, const MfLayout& L, int l, int P, int D, int Ds,
                                                  int32_t round_budget, bool settle, unsigned long long* stats) {
    constexpr int kM = MfBits<SEG>::kM;
    unsigned long long pushes = 0, relabels = 0;
    int32_t b[kM], ft[kM];
    int old_p[kM] = {}, old_d[kM] = {};  // kStats: the last distances
#pragma unroll
    for (int s = 0; s < kM; ++s) {
        b[s] = l + 64 * s < D ? L.b[l + 64 * s] : 0;
        ft[s] = 0;
    }
    bool left = false;
    for (int round = 0;; ++round) {
        // distances and admissible arcs
        int dp[kM], dd[kM];  // 0: does not reach the sink
        uint64_t ap[kM][kM], ad[kM][kM], front[kM];
        int32_t ep[kM], ed[kM];
#pragma unroll
        for (int s = 0; s < kM; ++s) {
            const int v = l + 64 * s;
            ep[s] = v < P ? L.ep[v] : 0;
            ed[s] = v < D ? L.ed[v] : 0;
            dp[s] = 0;
            dd[s] = v < D && b[s] - ft[s] > 0 ? 1 : 0;
#pragma unroll
            for (int w = 0; w < kM; ++w) ap[s][w] = ad[s][w] = 0;
            front[s] = __ballot(dd[s] == 1);
        }
        for (int lv = 1;; lv += 2) {
            uint64_t any = 0, fp[kM];
#pragma unroll
            for (int s = 0; s < kM; ++s) {
                const int v = l + 64 * s;
                bool hit = false;
                if (v < P && dp[s] == 0) {
#pragma unroll
                    for (int w = 0; w < kM; ++w) {
                        ap[s][w] = S.room[v][w] & front[w];
                        hit |= ap[s][w] != 0;
                    }
                    if (hit) dp[s] = lv + 1;
                }
                fp[s] = __ballot(hit);
                any |= fp[s];
            }
            if (!any) break;
            any = 0;
#pragma unroll
            for (int s = 0; s < kM; ++s) {
                const int v = l + 64 * s;
                bool hit = false;
                if (v < D && dd[s] == 0) {
#pragma unroll
                    for (int w = 0; w < kM; ++w) {
                        ad[s][w] = S.used[v][w] & fp[w];
                        hit |= ad[s][w] != 0;
                    }
                    if (hit) dd[s] = lv + 2;
                }
                front[s] = __ballot(hit);
                any |= front[s];
            }
            if (!any) break;
        }
        bool active = false;
#pragma unroll
        for (int s = 0; s < kM; ++s) {
            active |= (ep[s] > 0 && dp[s] > 0) || (ed[s] > 0 && dd[s] > 0);
            if (kStats) {
                relabels += (dp[s] != old_p[s] && round > 0) + (dd[s] != old_d[s] && round > 0);
                old_p[s] = dp[s];
                old_d[s] = dd[s];
            }
        }
        if (!__any(active)) break;
        if (round == round_budget) {
            left = true;
            break;
        }
        if (kStats && l == 0) {
            atomicAdd(&stats[HX_MF_ROUNDS], 1ull);
            atomicAdd(&stats[HX_MF_GLOBAL_RELABELS], 1ull);
        }
        // prefill nodes push one level down
#pragma unroll
        for (int s = 0; s < kM; ++s) {
            if (!(ep[s] > 0 && dp[s] > 0)) continue;
            const int v = l + 64 * s;
            const int32_t* c = L.cap + v * Ds;
            int32_t* fr = L.fl + v * Ds;
            int32_t e = ep[s];
#pragma unroll
            for (int w = 0; w < kM; ++w) {
                uint64_t full = 0, m = ap[s][w];
                while (m && e > 0) {
                    int x[4], n = 0;
                    int32_t f0[4], r0[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        x[k] = m ? __builtin_ctzll(m) : (k ? x[k - 1] : 0);
                        n += m != 0;
                        m &= m - 1;
                        f0[k] = fr[64 * w + x[k]];
                        r0[k] = c[64 * w + x[k]];
                    }
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int32_t rest = r0[k] - f0[k], amt = k < n ? (rest < e ? rest : e) : 0;
                        if (amt > 0) {
                            const int j = 64 * w + x[k];
                            fr[j] = f0[k] + amt;
                            e -= amt;
                            atomicAdd(&L.ed[j], amt);
                            atomicOr((unsigned long long*)&S.used[j][v >> 6], 1ull << (v & 63));
                            if (amt == rest) full |= 1ull << x[k];
                            if (kStats) ++pushes;
                        }
                    }
                }
                if (full) S.room[v][w] &= ~full;
            }
            L.ep[v] = e;
        }
        mf_wave_sync();
        // decode nodes push to the sink, or back to prefill nodes one level down
#pragma unroll
        for (int s = 0; s < kM; ++s) {
            const int v = l + 64 * s;
            int32_t e = v < D ? L.ed[v] : 0;
            if (!(e > 0 && dd[s] > 0)) continue;
            if (dd[s] == 1) {
                const int32_t rest = b[s] - ft[s], amt = rest < e ? rest : e;
                ft[s] += amt;
                e -= amt;
                if (kStats) ++pushes;
            } else {
#pragma unroll
                for (int w = 0; w < kM; ++w)
                    e = push_back<SEG, kStats>(S, L, v, w, ad[s][w], e, Ds, pushes);
            }
            L.ed[v] = e;
        }
        mf_wave_sync();
    }
    if (settle && !left) {
        // excess that cannot reach the sink goes back: decode to prefill, then prefill to the source
#pragma unroll
        for (int s = 0; s < kM; ++s) {
            const int v = l + 64 * s;
            int32_t e = v < D ? L.ed[v] : 0;
            if (e <= 0) continue;
            for (int w = 0; w < kM; ++w) e = push_back<SEG, kStats>(S, L, v, w, S.used[v][w], e, Ds, pushes);
            L.ed[v] = 0;
        }
        mf_wave_sync();
#pragma unroll
        for (int s = 0; s < kM; ++s) {
            const int v = l + 64 * s;
            const int32_t e = v < P ? L.ep[v] : 0;
            if (e <= 0) continue;
            L.fs[v] -= e;
            L.ep[v] = 0;
            if (kStats) ++pushes;
        }
    }
#pragma unroll
    for (int s = 0; s < kM; ++s)
        if (l + 64 * s < D) L.ft[l + 64 * s] = ft[s];
    if (kStats) {
        if (pushes) atomicAdd(&stats[HX_MF_PUSHES], pushes);
        if (relabels) atomicAdd(&stats[HX_MF_RELABELS], relabels);
    }
    return left;
}

// The canonical minimum cut of the flow in L, by one wavefront on the residual bit words: the same
// reachability as maxflow_tile's sweeps, a level at a time.  A reached prefill out-node offers its word
// of decode in-nodes with room, a reached decode in-node its word of prefill nodes it holds flow of;
// the in- and out-node of a chain follow from its flow.
template <int SEG>
__device__ __forceinline__ void cut_bits(const MfBits<SEG>& S, const MfLayout& L, const FlowNet& f, uint8_t* cut, int n,
                                         int l, int P, int D) {
    constexpr int kM = MfBits<SEG>::kM;
    const int64_t N = f.N;
    bool pin[kM], pout[kM], din[kM], fresh[kM];
    int32_t fs[kM];
#pragma unroll
    for (int s = 0; s < kM; ++s) {
        const int v = l + 64 * s;
        const int64_t o = (int64_t)v * N + n;
        fs[s] = v < P ? L.fs[v] : 0;
        pin[s] = v < P && f.src_cap[o] - fs[s] > 0;
        pout[s] = fresh[s] = pin[s] && f.p_cap[o] - fs[s] > 0;
        din[s] = false;
    }
    // the OR over the fresh nodes' words, in every lane
    auto offered = [&](const uint64_t (*words)[kM], uint64_t (&out)[kM]) {
#pragma unroll
        for (int w = 0; w < kM; ++w) {
            uint64_t m = 0;
#pragma unroll
            for (int s = 0; s < kM; ++s)
                if (fresh[s]) m |= words[l + 64 * s][w];
            for (int off = 32; off > 0; off >>= 1) m |= __shfl_xor((unsigned long long)m, off, 64);
            out[w] = m;
        }
    };
    for (;;) {
        uint64_t m[kM];
        offered(S.room, m);
        bool any = false;
#pragma unroll
        for (int s = 0; s < kM; ++s) {
            fresh[s] = l + 64 * s < D && !din[s] && ((m[s] >> l) & 1);
            din[s] |= fresh[s];
            any |= fresh[s];
        }
        if (!__any(any)) break;
        offered(S.used, m);
        any = false;
#pragma unroll
        for (int s = 0; s < kM; ++s) {
            fresh[s] = l + 64 * s < P && !pout[s] && ((m[s] >> l) & 1);
            pout[s] |= fresh[s];
            any |= fresh[s];
        }
        if (!__any(any)) break;
    }
#pragma unroll
    for (int s = 0; s < kM; ++s) {
        const int v = l + 64 * s;
        const int64_t o = (int64_t)v * N + n;
        pin[s] |= pout[s] && fs[s] > 0;
        if (v < P) cut[o] = (uint8_t)((pin[s] ? 1 : 0) | (pout[s] ? 2 : 0));
        if (v < D)
            cut[(int64_t)f.max_p * N + o] = (uint8_t)((din[s] ? 1 : 0) | (din[s] && f.d_cap[o] - L.ft[v] > 0 ? 2 : 0));
    }
}

// Dominant KV arcs.  When c_ij >= min(a_i, b_j) on every KV arc, no cut is below
// U = min(sum a, sum b): a cut keeping prefill set A on the source side costs
// sum_{i not in A} a_i + sum_j min(b_j, sum_{i in A} c_ij) >= sum_{i not in A} a_i +
// sum_j min(b_j, S) with S = sum_{i in A} a_i (each term: some a_i >= b_j gives b_j, else
// c_ij >= a_i for all of A), which is >= sum b when S >= every b_j and >= sum a otherwise.
// The maximum flow is then U, and the north-west-corner fill is one: with prefix sums A_i of a
// and B_j of b clamped to U, arc (i, j) carries the overlap of [A_{i-1}, A_i) and
// [B_{j-1}, B_j), at most min(a_i, b_j) <= c_ij; node i sends A_i - A_{i-1}, node j receives
// B_j - B_{j-1}.
__device__ __forceinline__ int32_t nw_overlap(int32_t ae, int32_t ai, int32_t be, int32_t bi) {
    const int32_t hi = ai < bi ? ai : bi, lo = ae > be ? ae : be;
    return hi > lo ? hi - lo : 0;
}

// Value-only pre-pass of the workgroup plans.  Those plans give a workgroup one candidate,
// whose KV rows then sit in as many cache lines as it has arcs; here lanes run over candidates
// (candidate-fastest, so every row load coalesces across the wavefront) in two kernels:
//   bound_kernel  one lane per candidate: writes min(sum a, sum b) as the candidate's flow
//                 value, 0 when no source-side or no sink-side node can carry flow, and -1 for
//                 networks with negative capacities or counts outside the plan;
//   dom_kernel    the dominant-KV condition c_ij >= min(a_i, b_j) on every arc, the arcs of a
//                 candidate split over kDomParts wavefronts (a long serial walk per candidate
//                 would leave the kernel waiting on one memory round per few arcs): an arc
//                 that fails it sets the flow value to -1.  It only ever writes -1, so the
//                 order of its writes does not matter.  c_ij >= a_i already implies the
//                 condition, so b_j is loaded only for arcs below a_i.
// maxflow_kernel then solves only the candidates left at -1.
constexpr int kBoundBlock = 256;
constexpr int kDomParts = 32;
constexpr int kDomUnroll = 8;

__device__ __forceinline__ bool plan_ok(const FlowNet& f, int P, int D) {
    return P >= 0 && D >= 0 && P <= f.max_p && D <= f.max_d && P * D <= f.max_pd;
}

__global__ void __launch_bounds__(kBoundBlock) bound_kernel(FlowNet f, int32_t* flow_value) {
    const int n = blockIdx.x * kBoundBlock + threadIdx.x;
    if (n >= f.N) return;
    const int64_t N = f.N;
    const int P = f.n_p[n], D = f.n_d[n];
    int32_t out = -1;
    if (plan_ok(f, P, D)) {
        long long sa = 0, sb = 0;
        bool neg = false, any_a = false, any_b = false;
        for (int i = 0; i < P; ++i) {
            const int32_t s = f.src_cap[(int64_t)i * N + n], c = f.p_cap[(int64_t)i * N + n];
            const int32_t a = s < c ? s : c;
            sa += a;
            neg |= a < 0;
            any_a |= a > 0;
        }
        for (int j = 0; j < D; ++j) {
            const int32_t c = f.d_cap[(int64_t)j * N + n], t = f.sink_cap[(int64_t)j * N + n];
            const int32_t b = c < t ? c : t;
            sb += b;
            neg |= b < 0;
            any_b |= b > 0;
        }
        if (!neg) out = (!any_a || !any_b) ? 0 : (int32_t)(sa < sb ? sa : sb);
    }
    flow_value[n] = out;
}

// Wavefront (part k, candidate chunk): arcs e in [k R, (k + 1) R) of each lane's candidate,
// R = ceil(max_pd / kDomParts), in ascending e (prefill node i = e / D, decode node j = e mod D).
__global__ void __launch_bounds__(64) dom_kernel(FlowNet f, int32_t* flow_value) {
    const int64_t N = f.N;
    // part-major: consecutive wavefronts take neighbouring candidate chunks of the same rows
    const int chunks = (int)((N + 63) / 64);
    const int part = blockIdx.x / chunks;
    const int64_t n = (int64_t)(blockIdx.x - part * chunks) * 64 + threadIdx.x;
    if (n >= N) return;
    if (flow_value[n] <= 0) return;  // -1: left to maxflow_kernel; 0: no flow either way
    const int P = f.n_p[n], D = f.n_d[n];
    const int R = (f.max_pd + kDomParts - 1) / kDomParts;
    const int E = P * D;
    const int lo = part * R, hi = lo + R < E ? lo + R : E;
    if (lo >= hi) return;
    auto a_of = [&](int i) {
        const int32_t s = f.src_cap[(int64_t)i * N + n], c = f.p_cap[(int64_t)i * N + n];
        return s < c ? s : c;
    };
    auto b_of = [&](int j) {
        const int32_t c = f.d_cap[(int64_t)j * N + n], t = f.sink_cap[(int64_t)j * N + n];
        return c < t ? c : t;
    };
    int i = lo / D, j = lo - i * D;
    int32_t ai = a_of(i);
    bool dom = true;
    for (int e0 = lo; e0 < hi && dom; e0 += kDomUnroll) {
        int32_t c[kDomUnroll];
#pragma unroll
        for (int x = 0; x < kDomUnroll; ++x) c[x] = e0 + x < hi ? f.kv_cap[(int64_t)(e0 + x) * N + n] : INT_MAX;
#pragma unroll
        for (int x = 0; x < kDomUnroll; ++x) {
            if (e0 + x < hi) {
                if (c[x] < ai) {
                    const int32_t bj = b_of(j);
                    dom = dom && c[x] >= (ai < bj ? ai : bj);
                }
                if (++j == D) {
                    j = 0;
                    if (++i < P && e0 + x + 1 < hi) ai = a_of(i);
                }
            }
        }
    }
    if (!dom) flow_value[n] = -1;
}

// SEG lanes per candidate; the workgroup holds max(64, SEG) lanes, i.e. 64/SEG candidates
// when SEG <= 64.  Workgroups are ordered XCD-aware: the hardware deals consecutive
// workgroups to the 8 XCDs in turn, so workgroup w takes tile (w mod 8) * chunk + w / 8 and
// each XCD walks a contiguous candidate range, sharing the L2 lines of the candidate-fastest
// input arrays.
// kStats: the diagnostic instantiation behind hx_maxflow_stats, which also counts into stats
// (HX_MF_STATS words, see hx.h) which path each candidate took and the push-relabel work; the
// production instantiation compiles none of it.
// The work of one tile (64/SEG candidates of a packed plan, or one candidate of a workgroup
// plan); every lane of the workgroup calls it with the same tile.
// kArg: fold the best of each wavefront's candidates (lane 0 of a segment holds its candidate's
// key, argmax_key) into the kArg slots of arg.  list: the tile's candidates are the tile-th kPer of the listed ones.
template <int SEG, bool kStats, int kArg = 0>
__device__ __forceinline__ void maxflow_tile(const FlowNet& f, int32_t* flow_value, int32_t* kv_flow, uint8_t* cut,
                                             int32_t round_budget, unsigned long long* stats, int tile,
                                             unsigned long long* arg = nullptr, const int32_t* list = nullptr,
                                             int listed = 0) {
    constexpr int kLanes = SEG < 64 ? kPackedLanes : SEG;
    constexpr int kPer = kLanes / SEG;
    const int N = f.N;
    const int tiles = (N + kPer - 1) / kPer;
    const int seg = threadIdx.x / SEG, l = threadIdx.x % SEG;
    const int at = tile * kPer + seg;
    const int n = list ? list[at < listed ? at : 0] : at;

    extern __shared__ int32_t smem[];
    const MfLayout L = carve(smem + seg * mf_words(f.max_p, f.max_d, f.max_pd), f.max_p, f.max_d, f.max_pd,
                             mf_heights(SEG, f.max_p, f.max_d));
    bool valid = list ? at < listed : tile < tiles && n < N;
    // value-only workgroup plans: bound_kernel has already written the candidates it could
    // (one candidate per workgroup, so the exit is uniform)
    if (SEG > 64 && kv_flow == nullptr && cut == nullptr && valid) {
        const int32_t pre = flow_value[n];
        if (pre >= 0) {
            if (kStats && l == 0) atomicAdd(&stats[HX_MF_PREPASS], 1ull);
            if constexpr (kArg > 0) fold_argmax<kArg>(l == 0 ? argmax_key(pre, n) : 0ull, arg);
            return;
        }
    }
    // kArg: a candidate in range that the checks below reject (HX_EINVAL) ends with valid false
    const bool in_range = valid;

    // Packed segments (SEG <= 64) own at most one node row per side and SEG/4 KV rows per
    // lane, so every global load is issued at once, before the counts that say which rows
    // are used have arrived: one memory round trip instead of three.  Unused rows are read
    // from the caller's [max][N] arrays and ignored.
    constexpr int kKvRows = SEG <= 64 ? (SEG / 4 > 0 ? SEG / 4 : 1) : 1;
    int32_t src0 = 0, pc0 = 0, dc0 = 0, sk0 = 0;
    int32_t kvr[kKvRows];
    int P = 0, D = 0;
    if (valid) {
        P = f.n_p[n];
        D = f.n_d[n];
        if (SEG <= 64) {
            if (l < f.max_p) {
                src0 = f.src_cap[(int64_t)l * N + n];
                pc0 = f.p_cap[(int64_t)l * N + n];
            }
            if (l < f.max_d) {
                dc0 = f.d_cap[(int64_t)l * N + n];
                sk0 = f.sink_cap[(int64_t)l * N + n];
            }
#pragma unroll
            for (int r = 0; r < kKvRows; ++r) {
                const int e = l + r * SEG;
                kvr[r] = e < f.max_pd ? f.kv_cap[(int64_t)e * N + n] : 0;
            }
        }
        // A network larger than the plan it was built for is rejected before any LDS or array
        // index is formed from it.
        if (P < 0 || D < 0 || P > f.max_p || D > f.max_d || P * D > f.max_pd ||
            (SEG <= 64 && (P > SEG || D > SEG || P * D > kKvRows * SEG))) {
            if (l == 0) flow_value[n] = HX_EINVAL;
            valid = false;
        }
    }
    if (!valid) P = D = 0;
    const int Ds = D | 1;

    // Node capacities first: a candidate whose source side or sink side carries nothing has
    // flow 0 and never needs its KV capacities (the cut sweep still sees zero flows).
    if (l == 0) {
        L.misc[0] = 0;
        L.misc[1] = 0;
        L.misc[2] = 0;
        L.misc[3] = 0;
    }
    __syncthreads();
    for (int i = l; i < P; i += SEG) {
        const int32_t s = SEG <= 64 ? src0 : f.src_cap[(int64_t)i * N + n];
        const int32_t c = SEG <= 64 ? pc0 : f.p_cap[(int64_t)i * N + n];
        const int32_t a = s < c ? s : c;
        L.a[i] = a;
        if (a > 0) L.misc[2] = 1;
    }
    for (int j = l; j < D; j += SEG) {
        const int32_t c = SEG <= 64 ? dc0 : f.d_cap[(int64_t)j * N + n];
        const int32_t t = SEG <= 64 ? sk0 : f.sink_cap[(int64_t)j * N + n];
        const int32_t b = c < t ? c : t;
        L.b[j] = b;
        L.ft[j] = 0;
        L.ed[j] = 0;
        if (b > 0) L.misc[3] = 1;
    }
    __syncthreads();
    const bool has_flow = P > 0 && D > 0 && L.misc[2] && L.misc[3];
    int path = has_flow ? HX_MF_PUSH_RELABEL : HX_MF_NO_FLOW;  // kStats: the path this candidate takes
    for (int i = l; i < P; i += SEG) {
        const int32_t a = has_flow ? L.a[i] : 0;
        L.fs[i] = a;  // saturate every source edge
        L.ep[i] = a;
    }
    bool thin = false;  // some KV arc below min(a_i, b_j)
    if (SEG <= 64) {
#pragma unroll
        for (int r = 0; r < kKvRows; ++r) {
            const int e = l + r * SEG;
            if (e < P * D) {
                const int i = e / D, d = e - i * D;
                L.cap[i * Ds + d] = kvr[r];
                L.fl[i * Ds + d] = 0;
            }
        }
    } else if (has_flow || kv_flow != nullptr || cut != nullptr) {
        // four rows' loads in flight per lane (rows past the last read it again and are dropped); the
        // dominance test on the way.  (More of them pull the lines that neighbouring candidates share out of
        // the L2: 4,096 networks of 64 x 64 nodes with their flows, 174 us without flow and 192 dominant with
        // four, 190 and 202 with eight, 206 and 205 with sixteen, 172 and 231 before the test was joined to the
        // loads.)
        constexpr int kBatch = 4;
        const int E = P * D;
        for (int e0 = l; e0 < E; e0 += kBatch * SEG) {
            int32_t v[kBatch];
#pragma unroll
            for (int x = 0; x < kBatch; ++x) v[x] = f.kv_cap[(int64_t)(e0 + x * SEG < E ? e0 + x * SEG : E - 1) * N + n];
#pragma unroll
            for (int x = 0; x < kBatch; ++x) {
                const int e = e0 + x * SEG;
                if (e < E) {
                    const int i = e / D, d = e - i * D;
                    L.cap[i * Ds + d] = v[x];
                    L.fl[i * Ds + d] = 0;
                    thin |= v[x] < (L.a[i] < L.b[d] ? L.a[i] : L.b[d]);
                }
            }
        }
    }
    __syncthreads();

    // One side with a single node that can carry flow (a > 0 on the prefill side, b > 0 on
    // the decode side) makes the network a star: with prefill node i alone the maximum flow
    // is min(a_i, sum_j min(c_ij, b_j)), with decode node j alone min(b_j, sum_i min(a_i,
    // c_ij)).  Such a candidate takes that value and a flow that fills the star's arcs in
    // node order (a prefix sum over the candidate's lanes), and skips push-relabel; the cut
    // sweep below works from any maximum flow.  Only the single-wavefront plans do this.
    // The shuffles below stay inside a candidate's lanes, whose branches agree.
    int32_t cut_value = -1;  // the flow value when a minimum cut was taken directly
    if (SEG <= 64) {
        const uint64_t segmask = SEG == 64 ? ~0ull : ((1ull << SEG) - 1);
        const int sh = (seg * SEG) & 63;
        const uint64_t ba = (__ballot(l < P && L.a[l] > 0) >> sh) & segmask;
        const uint64_t bb = (__ballot(l < D && L.b[l] > 0) >> sh) & segmask;
        const bool one_p = __popcll(ba) == 1, one_d = __popcll(bb) == 1;
#pragma unroll
        for (int r = 0; r < kKvRows; ++r) {
            const int e = l + r * SEG;
            if (e < P * D) {
                const int i = e / D, d = e - i * D;
                const int32_t m = L.a[i] < L.b[d] ? L.a[i] : L.b[d];
                thin |= L.cap[i * Ds + d] < m;
            }
        }
        const bool dominant = ((__ballot(thin) >> sh) & segmask) == 0;
        if (has_flow && (one_p || one_d)) {
            path = HX_MF_STAR;
            const int is = __ffsll((unsigned long long)ba) - 1, js = __ffsll((unsigned long long)bb) - 1;
            int32_t v = 0;
            if (one_p) {
                if (l < D && L.b[l] > 0) {
                    const int32_t c = L.cap[is * Ds + l];
                    v = c < L.b[l] ? c : L.b[l];
                }
            } else if (l < P && L.a[l] > 0) {
                const int32_t c = L.cap[l * Ds + js];
                v = c < L.a[l] ? c : L.a[l];
            }
            int32_t incl = v;
#pragma unroll
            for (int off = 1; off < SEG; off <<= 1) {
                const int32_t u = __shfl_up(incl, off, SEG);
                if (l >= off) incl += u;
            }
            const int32_t total = __shfl(incl, SEG - 1, SEG);
            const int32_t side = one_p ? L.a[is] : L.b[js];
            const int32_t F = total < side ? total : side;
            const int32_t room = F - (incl - v);
            const int32_t fv = room <= 0 ? 0 : (room < v ? room : v);
            if (one_p) {
                if (l < D) {
                    L.fl[is * Ds + l] = fv;
                    L.ft[l] = fv;
                }
                if (l == is) L.fs[is] = F;
            } else {
                if (l < P) {
                    L.fl[l * Ds + js] = fv;
                    L.fs[l] = fv;
                }
                if (l == js) L.ft[js] = F;
            }
            if (l < P) L.ep[l] = 0;
        } else if (has_flow && dominant) {
            path = HX_MF_DOMINANT;
            // lane l holds prefill node l and decode node l (packed plans: P, D <= SEG); the
            // sums stay below 64 * 2^24 < 2^31
            const int32_t av = l < P ? L.a[l] : 0, bv = l < D ? L.b[l] : 0;
            int32_t ia = av, ib = bv;
#pragma unroll
            for (int off = 1; off < SEG; off <<= 1) {
                const int32_t ua = __shfl_up(ia, off, SEG), ub = __shfl_up(ib, off, SEG);
                if (l >= off) {
                    ia += ua;
                    ib += ub;
                }
            }
            const int32_t ta = __shfl(ia, SEG - 1, SEG), tb = __shfl(ib, SEG - 1, SEG);
            const int32_t U = ta < tb ? ta : tb;
            const int32_t ai = ia < U ? ia : U, ae = ia - av < U ? ia - av : U;
            const int32_t bi = ib < U ? ib : U, be = ib - bv < U ? ib - bv : U;
            if (l < P) {
                L.fs[l] = ai - ae;
                L.ep[l] = 0;
            }
            if (l < D) L.ft[l] = bi - be;
#pragma unroll
            for (int r = 0; r < kKvRows; ++r) {
                const int e = l + r * SEG;
                const bool in = e < P * D;
                const int i = in ? e / D : 0, d = in ? e - i * D : 0;
                const int32_t Ai = __shfl(ai, i, SEG), Ae = __shfl(ae, i, SEG);
                const int32_t Bj = __shfl(bi, d, SEG), Be = __shfl(be, d, SEG);
                if (in) L.fl[i * Ds + d] = nw_overlap(Ae, Ai, Be, Bj);
            }
        } else if (has_flow && kv_flow == nullptr && cut == nullptr) {
            // Only the value is wanted: with m = min(P', D') <= kEnumMax nodes that can carry
            // flow on the smaller side, take the minimum cut directly.  Fixing which of those
            // nodes stay on the source side (a subset A of the prefill side, say) leaves every
            // other node one cheapest choice: cut = sum_{i not in A} a_i + sum_j min(b_j,
            // sum_{i in A} c_ij); the maximum flow is the minimum over the 2^m subsets, which
            // the candidate's lanes share.
            const int pe = __popcll(ba), de = __popcll(bb);
            const int m = pe <= de ? pe : de;
            if (m <= kEnumMax) {
                const bool byp = pe <= de;
                const uint64_t side = byp ? ba : bb, other = byp ? bb : ba;
                int32_t best = 0x7fffffff;
                for (int sub = l; sub < (1 << m); sub += SEG) {
                    int32_t cost = 0;
                    uint64_t rest = side;
                    for (int k = 0; rest; ++k, rest &= rest - 1)
                        if (!((sub >> k) & 1)) {
                            const int u = __ffsll((unsigned long long)rest) - 1;
                            cost += byp ? L.a[u] : L.b[u];
                        }
                    for (uint64_t ow = other; ow; ow &= ow - 1) {
                        const int w = __ffsll((unsigned long long)ow) - 1;
                        int32_t arcs = 0;
                        uint64_t in = side;
                        for (int k = 0; in; ++k, in &= in - 1)
                            if ((sub >> k) & 1) {
                                const int u = __ffsll((unsigned long long)in) - 1;
                                arcs += byp ? L.cap[u * Ds + w] : L.cap[w * Ds + u];
                            }
                        const int32_t cw = byp ? L.b[w] : L.a[w];
                        cost += cw < arcs ? cw : arcs;
                    }
                    best = cost < best ? cost : best;
                }
#pragma unroll
                for (int off = SEG / 2; off > 0; off >>= 1) {
                    const int32_t o2 = __shfl_xor(best, off, SEG);
                    best = o2 < best ? o2 : best;
                }
                cut_value = best;
                path = HX_MF_MIN_CUT;
                if (l < P) L.ep[l] = 0;
            }
        }
        __syncthreads();
    } else {
        // Workgroup plans (one candidate per workgroup, so every branch here is uniform).
        __shared__ long long wave_sum[SEG > 64 ? SEG / 64 : 1];
        if (!__syncthreads_or(thin) && has_flow) {
            path = HX_MF_DOMINANT;
            // block scan: lane l owns a contiguous run of nodes on each side; clamped inclusive
            // prefix sums go to ep (prefill) and ed (decode), then become the flows
            const int cp = (P + SEG - 1) / SEG, cd = (D + SEG - 1) / SEG;
            const int p0 = l * cp < P ? l * cp : P, p1 = p0 + cp < P ? p0 + cp : P;
            const int d0 = l * cd < D ? l * cd : D, d1 = d0 + cd < D ? d0 + cd : D;
            long long sa = 0, sb = 0;
            for (int i = p0; i < p1; ++i) sa += L.a[i];
            for (int j = d0; j < d1; ++j) sb += L.b[j];
            long long tot[2], excl[2];
            const long long v2[2] = {sa, sb};
            for (int k = 0; k < 2; ++k) {
                long long incl = v2[k];
                for (int off = 1; off < 64; off <<= 1) {
                    const long long u = __shfl_up(incl, off, 64);
                    if ((l & 63) >= off) incl += u;
                }
                if ((l & 63) == 63) wave_sum[l >> 6] = incl;
                __syncthreads();
                long long before = 0, all = 0;
                for (int w = 0; w < SEG / 64; ++w) {
                    if (w < (l >> 6)) before += wave_sum[w];
                    all += wave_sum[w];
                }
                __syncthreads();
                excl[k] = before + incl - v2[k];
                tot[k] = all;
            }
            const long long U = tot[0] < tot[1] ? tot[0] : tot[1];  // < 2^31: min(P, D) <= 127
            long long run = excl[0];
            for (int i = p0; i < p1; ++i) {
                run += L.a[i];
                L.ep[i] = (int32_t)(run < U ? run : U);
            }
            run = excl[1];
            for (int j = d0; j < d1; ++j) {
                run += L.b[j];
                L.ed[j] = (int32_t)(run < U ? run : U);
            }
            __syncthreads();
            for (int e = l; e < P * D; e += SEG) {
                const int i = e / D, d = e - i * D;
                L.fl[i * Ds + d] = nw_overlap(i > 0 ? L.ep[i - 1] : 0, L.ep[i], d > 0 ? L.ed[d - 1] : 0, L.ed[d]);
            }
            for (int i = l; i < P; i += SEG) L.fs[i] = L.ep[i] - (i > 0 ? L.ep[i - 1] : 0);
            for (int j = l; j < D; j += SEG) L.ft[j] = L.ed[j] - (j > 0 ? L.ed[j - 1] : 0);
            __syncthreads();
            for (int i = l; i < P; i += SEG) L.ep[i] = 0;
            for (int j = l; j < D; j += SEG) L.ed[j] = 0;
        }
        __syncthreads();
    }

    const int V = P + D + 2;
    const int INF = 2 * V + 2;
    bool active = false, left = false;  // left: out of rounds (push_relabel_bits)
    for (int i = l; i < P; i += SEG) active |= L.ep[i] > 0;
    unsigned long long pushes = 0, relabels = 0;  // kStats
    if (kStats && valid && l == 0) atomicAdd(&stats[path], 1ull);
    __shared__ MfBits<(SEG > 64 ? SEG : 64)> B;  // (workgroup plans)
    if constexpr (SEG > 64) {
        // (more than SEG nodes a side, which only arrays wider than 256 rows hold, stay with the loop below; the
        // 128-lane plan's arrays hold at most 128 a side, so it has neither the loop nor the heights it needs)
        if (path == HX_MF_PUSH_RELABEL && (SEG == 128 || (P <= SEG && D <= SEG))) {  // uniform: one candidate a workgroup
            residual_bits<SEG>(B, L, l, P, D, Ds, false);
            __syncthreads();
            if (threadIdx.x < 64)
                left = push_relabel_bits<SEG, kStats>(B, L, l, P, D, Ds, round_budget,
                                                      kv_flow != nullptr || cut != nullptr, stats);
            __syncthreads();
            active = false;
        }
    }
    for (int round = 0; SEG != 128 && __syncthreads_or(active) && round < round_budget; ++round) {
        if (kStats && threadIdx.x == 0) {
            atomicAdd(&stats[HX_MF_ROUNDS], 1ull);
            if (round % kGlobalRelabelEvery == 0) atomicAdd(&stats[HX_MF_GLOBAL_RELABELS], 1ull);
        }
        if (round % kGlobalRelabelEvery == 0) {
            global_relabel<SEG>(L, l, P, D, Ds, V, INF);
            __syncthreads();
        }
        // P-phase: push along admissible arcs and, in the same pass, track the lowest height
        // across arcs still holding residual capacity, for the relabel if excess remains.
        for (int i = l; i < P; i += SEG) {
            int e = L.ep[i];
            if (e <= 0) continue;
            const int h = L.hp[i];
            const int32_t* c = L.cap + i * Ds;
            int32_t* fr = L.fl + i * Ds;
            int mh = INF;
            for (int d = 0; d < D && e > 0; ++d) {
                int r = c[d] - fr[d];
                if (r <= 0) continue;
                const int hd = L.hd[d];
                if (h == hd + 1) {
                    const int amt = r < e ? r : e;
                    fr[d] += amt;
                    e -= amt;
                    r -= amt;
                    atomicAdd(&L.ed[d], amt);
                    if (kStats) ++pushes;
                }
                if (r > 0 && hd < mh) mh = hd;
            }
            if (e > 0 && h == V + 1) {
                const int amt = L.fs[i] < e ? L.fs[i] : e;
                L.fs[i] -= amt;
                e -= amt;
                if (kStats && amt > 0) ++pushes;
            }
            if (e > 0) {
                if (L.fs[i] > 0 && V < mh) mh = V;
                L.hp[i] = mh + 1 < INF ? mh + 1 : INF;
                if (kStats) ++relabels;
            }
            L.ep[i] = e;
        }
        __syncthreads();
        // D-phase: push to the sink, then back along used KV arcs, tracking the lowest height
        // across arcs left with residual capacity for the relabel.
        for (int j = l; j < D; j += SEG) {
            int e = L.ed[j];
            if (e <= 0) continue;
            const int h = L.hd[j];
            if (h == 1) {
                const int r = L.b[j] - L.ft[j];
                const int amt = r < e ? r : e;
                if (amt > 0) {
                    L.ft[j] += amt;
                    e -= amt;
                    if (kStats) ++pushes;
                }
            }
            int mh = INF;
            for (int q = 0; q < P && e > 0; ++q) {
                int fq = L.fl[q * Ds + j];
                if (fq <= 0) continue;
                const int hq = L.hp[q];
                if (h == hq + 1) {
                    const int amt = fq < e ? fq : e;
                    fq -= amt;
                    L.fl[q * Ds + j] = fq;
                    e -= amt;
                    atomicAdd(&L.ep[q], amt);
                    if (kStats) ++pushes;
                }
                if (fq > 0 && hq < mh) mh = hq;
            }
            if (e > 0) {
                if (L.b[j] - L.ft[j] > 0) mh = 0;
                L.hd[j] = mh + 1 < INF ? mh + 1 : INF;
                if (kStats) ++relabels;
            }
            L.ed[j] = e;
        }
        __syncthreads();
        active = false;
        for (int i = l; i < P; i += SEG) active |= L.ep[i] > 0;
        for (int j = l; j < D; j += SEG) active |= L.ed[j] > 0;
    }
    if (kStats) {
        if (pushes) atomicAdd(&stats[HX_MF_PUSHES], pushes);
        if (relabels) atomicAdd(&stats[HX_MF_RELABELS], relabels);
    }
    // Flow value = total flow into the sink; a candidate still holding excess ran out of rounds.
    for (int j = l; j < D; j += SEG)
        if (L.ft[j] > 0) atomicAdd(&L.misc[0], L.ft[j]);
    if (active || left) L.misc[1] = 1;
    __syncthreads();
    const int32_t value = cut_value >= 0 ? cut_value : (L.misc[1] ? HX_ENOCONV : L.misc[0]);
    if (valid && l == 0) flow_value[n] = value;
    if constexpr (kArg > 0) fold_argmax<kArg>(l == 0 && in_range ? argmax_key(valid ? value : HX_EINVAL, n) : 0ull, arg);
    if (valid && kv_flow)
        for (int e = l; e < P * D; e += SEG) {
            const int i = e / D, d = e - i * D;
            kv_flow[(int64_t)e * N + n] = L.fl[i * Ds + d];
        }
    if (!cut) return;  // uniform across the workgroup

    if constexpr (SEG > 64) {
        if (SEG == 128 || (P <= SEG && D <= SEG)) {
            if (path != HX_MF_PUSH_RELABEL) {  // uniform
                residual_bits<SEG>(B, L, l, P, D, Ds, path != HX_MF_NO_FLOW);
                __syncthreads();
            }
            if (threadIdx.x < 64) cut_bits<SEG>(B, L, f, cut, n, l, P, D);
            return;
        }
    }
    // Canonical minimum cut: reachability from s in the residual graph of the uncontracted
    // network, by sweeps until nothing changes.  Reuses a/ep (prefill in/out flags) and
    // b/ed (decode in/out flags); source/node/sink capacities are reloaded.
    int32_t* rin = L.ep;
    int32_t* rout = L.a;
    int32_t* din = L.ed;
    int32_t* dout = L.b;
    __syncthreads();
    for (int i = l; i < P; i += SEG) {
        rin[i] = f.src_cap[(int64_t)i * N + n] - L.fs[i] > 0;
        rout[i] = 0;
    }
    for (int j = l; j < D; j += SEG) {
        din[j] = 0;
        dout[j] = 0;
    }
    __syncthreads();
    for (;;) {
        bool changed = false;
        // prefill replica: phi_out is reached from a reached delta_in over a used KV edge (its
        // reverse arc), and in <-> out inside the chain along whichever arcs have residual.
        for (int i = l; i < P; i += SEG) {
            const int32_t fsi = L.fs[i];
            const int32_t pres = f.p_cap[(int64_t)i * N + n] - fsi;
            int in = rin[i], out = rout[i];
            for (int d = 0; d < D && !out; ++d) out = din[d] && L.fl[i * Ds + d] > 0;
            for (int k = 0; k < 2; ++k) {
                in |= out && fsi > 0;
                out |= in && pres > 0;
            }
            if (in != rin[i] || out != rout[i]) {
                rin[i] = in;
                rout[i] = out;
                changed = true;
            }
        }
        __syncthreads();
        // decode replica: delta_in is reached from a reached phi_out over a KV edge with
        // residual capacity, then in <-> out inside the chain.
        for (int j = l; j < D; j += SEG) {
            const int32_t ftj = L.ft[j];
            const int32_t dres = f.d_cap[(int64_t)j * N + n] - ftj;
            int in = din[j], out = dout[j];
            for (int q = 0; q < P && !in; ++q) in = rout[q] && L.cap[q * Ds + j] - L.fl[q * Ds + j] > 0;
            for (int k = 0; k < 2; ++k) {
                out |= in && dres > 0;
                in |= out && ftj > 0;
            }
            if (in != din[j] || out != dout[j]) {
                din[j] = in;
                dout[j] = out;
                changed = true;
            }
        }
        if (!__syncthreads_or(changed)) break;
    }
    if (!valid) return;
    for (int i = l; i < P; i += SEG) cut[(int64_t)i * N + n] = (uint8_t)(rin[i] | (rout[i] << 1));
    for (int j = l; j < D; j += SEG) cut[(int64_t)(f.max_p + j) * N + n] = (uint8_t)(din[j] | (dout[j] << 1));
}

// kArg (hx_score_batch): each wavefront also takes the best of its candidates' flow values
// (highest value, lowest index) and folds it into slot blockIdx mod kArgSlots of arg, as the key
// argmax_key, with a 64-bit atomic max; the slots must be zero at launch, and best_final_kernel
// reduces them.
template <int SEG, bool kStats, bool kArg = false>
__global__ void __launch_bounds__(SEG < 64 ? kPackedLanes : SEG, SEG <= 64 ? 8 : 1)
    maxflow_kernel(FlowNet f, int32_t* flow_value, int32_t* kv_flow, uint8_t* cut, int32_t round_budget,
                   unsigned long long* stats, unsigned long long* arg) {
    constexpr int kPer = (SEG < 64 ? kPackedLanes : SEG) / SEG;
    const int tiles = (f.N + kPer - 1) / kPer;
    const int chunk = (tiles + 7) / 8;
    const int tile = (int)(blockIdx.x & 7) * chunk + (int)(blockIdx.x >> 3);
    maxflow_tile<SEG, kStats, kArg ? kArgSlots : 0>(f, flow_value, kv_flow, cut, round_budget, stats, tile, arg);
}

// Value only, workgroup plans: the candidates listed (list[0 .. *count), written by the kernel that
// settled the others), a workgroup taking every gridDim.x-th entry.
template <int SEG>
__global__ void __launch_bounds__(SEG) maxflow_list_kernel(FlowNet f, int32_t* flow_value, int32_t round_budget,
                                                           const int32_t* list, const int32_t* count) {
    const int c = *count;
    for (int idx = blockIdx.x; idx < c; idx += gridDim.x) {
        maxflow_tile<SEG, false>(f, flow_value, nullptr, nullptr, round_budget, nullptr, idx, nullptr, list, c);
        __syncthreads();  // the next candidate reuses the LDS
    }
}

// The last kernel of hx_score_batch on replica networks: solves the candidates that net_kernel
// listed (usually none), folding their values into the argmax slots, and reduces the slots.  With
// nothing listed the first workgroup reduces them at once; otherwise the last workgroup to finish
// (tickets) does.
//
// The tiles of the list are dealt as maxflow_kernel's are, a contiguous eighth to the workgroups of each
// XCD, and only the workgroups that have one take a ticket: workgroup y of XCD x ticket 2 x + (y mod 2), and
// the last of each of these the last ticket.  The last workgroup reads nothing of the others' but what they
// wrote with device-scope atomics, so each waits until its own are done and needs no release fence, which
// would write back its XCD's L2.  The loop hides the network's dimensions from the compiler, which would
// otherwise keep what it derives from them in registers across tiles (28 to 42 spilled).
// What bounds it: the latency of a tile's dependent loads and LDS accesses, so up to 24 wavefronts a CU
// (kFinishGrid; LDS 4 to 7 KB each), which cost a call with nothing listed no measurable time.
// hx_score_batch with separate node, KV and max-flow kernels / with this kernel on 1,024 workgroups that
// all took one ticket behind fences / now, 65,536 candidates: 5 networks listed of 4,096 (32 GPUs) 89 / 108 /
// 73 us, 65,536 listed of 8 slots 182 / 261 / 183, 23,928 of 16 slots 119 / 171 / 98, 30,483 of 32 slots
// 181 / 367 / 169, 64,102 of 16 slots that take push-relabel 657 / 1,408 / 732 (33 us of it the network kernel's
// walks): there a network's latency is what counts, and 32 wavefronts a CU had one each.
constexpr int kFinishGrid = 6144;
constexpr int kFinishParts = kNetTickets / 8;  // tickets of an XCD

// Workgroups of XCD x that have a tile (rows: workgroups of an XCD).
__device__ __forceinline__ int finish_workers(int x, int tiles, int chunk, int rows) {
    const int left = tiles - x * chunk, t = left < chunk ? left : chunk;
    return t < 0 ? 0 : (t < rows ? t : rows);
}

template <int SEG>
__global__ void __launch_bounds__(kPackedLanes, 6)
    finish_kernel(FlowNet f, int32_t* flow_value, int32_t round_budget, const int32_t* list, unsigned long long* area,
                  int32_t* best) {
    static_assert(SEG <= 64, "packed plans");
    constexpr int kPer = kPackedLanes / SEG;
    const int c = *net_list_count(area);
    if (c > 0) {
        __shared__ int32_t last;
        const int tiles = (c + kPer - 1) / kPer, chunk = (tiles + 7) / 8, rows = (int)(gridDim.x >> 3);
        const int x = (int)(blockIdx.x & 7), y = (int)(blockIdx.x >> 3);
        const int mine = finish_workers(x, tiles, chunk, rows);
        if (y >= mine) return;  // uniform
        for (int i = y; i < chunk && x * chunk + i < tiles; i += rows) {
            FlowNet g = f;
            asm volatile("" : "+s"(g.N), "+s"(g.max_p), "+s"(g.max_d), "+s"(g.max_pd));
            maxflow_tile<SEG, false, kNetSlots>(g, flow_value, nullptr, nullptr, round_budget, nullptr, x * chunk + i,
                                                area, list, c);
            __syncthreads();  // the next candidates reuse the LDS
        }
        if (threadIdx.x == 0) {
            int32_t* ticket = net_list_count(area) + 1;
            const int q = y % kFinishParts, of = (mine - q + kFinishParts - 1) / kFinishParts;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's atomics are done
            last = 0;
            if (atomicAdd(net_list_count(area) + 2 * kNetLine * (1 + kFinishParts * x + q), 1) == of - 1) {
                int parts = 0;  // tickets that some workgroup takes
                for (int k = 0; k < 8; ++k) {
                    const int w = finish_workers(k, tiles, chunk, rows);
                    parts += w < kFinishParts ? w : kFinishParts;
                }
                last = atomicAdd(ticket, 1) == parts - 1;
            }
        }
        __syncthreads();
        if (!last) return;  // uniform
    } else if (blockIdx.x != 0) {
        return;
    }
    unsigned long long key = 0;
#pragma unroll
    for (int i = 0; i < kNetSlots / kPackedLanes; ++i) {
        const unsigned long long v = __hip_atomic_load(&area[i * kPackedLanes + threadIdx.x], __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT);
        key = v > key ? v : key;
    }
    for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long o = __shfl_xor(key, off, 64);
        key = o > key ? o : key;
    }
    if (threadIdx.x == 0) {
        best[0] = (int32_t)(0xFFFFFFFFu - (uint32_t)key);
        best[1] = (int32_t)((uint32_t)(key >> 32) ^ 0x80000000u);
    }
}

constexpr size_t kMaxLds = 64 * 1024;

// Lanes per candidate: the smallest power of two (at least 8) with one lane per node of the
// widest side and SEG/4 KV rows per lane covering max_pd (SEG^2/4 >= max_pd); beyond 256
// lanes a lane owns several nodes.
int segment_lanes(int max_p, int max_d, int max_pd) {
    const int widest = max_p > max_d ? max_p : max_d;
    int s = 8;
    while (s < 256 && (s < widest || (int64_t)s * s / 4 < max_pd)) s *= 2;
    return s;
}

__global__ void clear_stats_kernel(unsigned long long* stats) {
    if (threadIdx.x < HX_MF_STATS) stats[threadIdx.x] = 0;
}

// Dynamic LDS of a launch: per candidates of a workgroup.
size_t mf_launch_lds(int seg, int per, const FlowNet& f) {
    const size_t words = mf_words(f.max_p, f.max_d, f.max_pd);
    const size_t spare = mf_heights(seg, f.max_p, f.max_d) ? 0 : 2 * (size_t)f.max_p + f.max_d;  // hp, hd and fs
    return per * (words - spare) * sizeof(int32_t);
}

template <int SEG>
hipError_t launch_seg(const FlowNet& f, int32_t* fv, int32_t* kv, uint8_t* cut, int32_t budget,
                      unsigned long long* stats, unsigned long long* arg, hipStream_t s) {
    constexpr int kLanes = SEG < 64 ? kPackedLanes : SEG;
    constexpr int kPer = kLanes / SEG;
    const size_t lds = mf_launch_lds(SEG, kPer, f);
    const int tiles = (f.N + kPer - 1) / kPer;
    const int blocks = 8 * ((tiles + 7) / 8);
    prof_mark(kKMaxflow, false, s);
    if (SEG > 64 && kv == nullptr && cut == nullptr) {
        hipLaunchKernelGGL(bound_kernel, dim3((f.N + kBoundBlock - 1) / kBoundBlock), dim3(kBoundBlock), 0, s, f, fv);
        const int chunks = (f.N + 63) / 64;
        hipLaunchKernelGGL(dom_kernel, dim3(chunks * kDomParts), dim3(64), 0, s, f, fv);
    }
    if (stats) {
        hipLaunchKernelGGL(clear_stats_kernel, dim3(1), dim3(64), 0, s, stats);
        hipLaunchKernelGGL((maxflow_kernel<SEG, true>), dim3(blocks), dim3(kLanes), lds, s, f, fv, kv, cut, budget,
                           stats, nullptr);
    } else if (arg) {
        hipLaunchKernelGGL((maxflow_kernel<SEG, false, true>), dim3(blocks), dim3(kLanes), lds, s, f, fv, kv, cut,
                           budget, nullptr, arg);
    } else {
        hipLaunchKernelGGL((maxflow_kernel<SEG, false>), dim3(blocks), dim3(kLanes), lds, s, f, fv, kv, cut, budget,
                           nullptr, nullptr);
    }
    prof_mark(kKMaxflow, true, s);
    return hipGetLastError();
}

}  // namespace

size_t maxflow_lds_bytes(int32_t max_p, int32_t max_d, int32_t max_pd) {
    const int seg = segment_lanes(max_p, max_d, max_pd);
    const int per = seg < 64 ? kPackedLanes / seg : 1;
    const size_t bytes = per * mf_words(max_p, max_d, max_pd) * sizeof(int32_t);
    return bytes <= kMaxLds ? bytes : 0;
}

bool maxflow_workgroup_plan(int32_t max_p, int32_t max_d, int32_t max_pd) {
    return segment_lanes(max_p, max_d, max_pd) > 64;
}

hipError_t launch_maxflow_listed(const FlowNet& f, int32_t* flow_value, int32_t round_budget, const int32_t* list,
                                 const int32_t* count, hipStream_t s) {
    const int seg = segment_lanes(f.max_p, f.max_d, f.max_pd);
    const size_t lds = mf_launch_lds(seg, 1, f);
    const int blocks = f.N < 2048 ? f.N : 2048;  // eight workgroups per CU at most
    prof_mark(kKMaxflow, false, s);
    if (seg == 128)
        hipLaunchKernelGGL(maxflow_list_kernel<128>, dim3(blocks), dim3(128), lds, s, f, flow_value, round_budget, list,
                           count);
    else
        hipLaunchKernelGGL(maxflow_list_kernel<256>, dim3(blocks), dim3(256), lds, s, f, flow_value, round_budget, list,
                           count);
    prof_mark(kKMaxflow, true, s);
    return hipGetLastError();
}

hipError_t launch_finish(const Problem& p, const FlowNet& f, int32_t* flow_value, int32_t round_budget,
                         unsigned long long* area, const int32_t* list, int32_t* best, hipStream_t s) {
    // the networks have at most Kmax nodes in all, whatever room the caller's arrays have
    FlowNet t = f;
    t.max_p = t.max_d = p.Kmax;
    t.max_pd = (p.Kmax / 2) * ((p.Kmax + 1) / 2);
    if (t.max_pd < 1) t.max_pd = 1;
    const int seg = segment_lanes(t.max_p, t.max_d, t.max_pd);  // at most 32 (Kmax <= 32)
    const int per = kPackedLanes / seg;
    const size_t lds = per * mf_words(t.max_p, t.max_d, t.max_pd) * sizeof(int32_t);
    const int tiles = (f.N + per - 1) / per;
    const dim3 grid(8 * (((tiles < kFinishGrid ? tiles : kFinishGrid) + 7) / 8));
    prof_mark(kKMaxflow, false, s);
    if (seg == 8)
        hipLaunchKernelGGL(finish_kernel<8>, grid, dim3(kPackedLanes), lds, s, t, flow_value, round_budget, list, area,
                           best);
    else if (seg == 16)
        hipLaunchKernelGGL(finish_kernel<16>, grid, dim3(kPackedLanes), lds, s, t, flow_value, round_budget, list, area,
                           best);
    else
        hipLaunchKernelGGL(finish_kernel<32>, grid, dim3(kPackedLanes), lds, s, t, flow_value, round_budget, list, area,
                           best);
    prof_mark(kKMaxflow, true, s);
    return hipGetLastError();
}

hipError_t launch_maxflow(const FlowNet& f, int32_t* flow_value, int32_t* kv_flow, uint8_t* cut, int32_t round_budget,
                          unsigned long long* stats, hipStream_t s, unsigned long long* arg) {
    switch (segment_lanes(f.max_p, f.max_d, f.max_pd)) {
        case 8: return launch_seg<8>(f, flow_value, kv_flow, cut, round_budget, stats, arg, s);
        case 16: return launch_seg<16>(f, flow_value, kv_flow, cut, round_budget, stats, arg, s);
        case 32: return launch_seg<32>(f, flow_value, kv_flow, cut, round_budget, stats, arg, s);
        case 64: return launch_seg<64>(f, flow_value, kv_flow, cut, round_budget, stats, arg, s);
        case 128: return launch_seg<128>(f, flow_value, kv_flow, cut, round_budget, stats, arg, s);
        default: return launch_seg<256>(f, flow_value, kv_flow, cut, round_budget, stats, arg, s);
    }
}

}  // namespace hx
