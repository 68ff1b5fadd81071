// hx_refine.hip -- max-flow guided refinement (Sec. 3.4) on gfx950.
//
// The refinement step compares every edge's flow with its capacity and moves GPUs between
// groups to relieve bottleneck edges with underutilized ones.  A maximum flow assignment is
// not unique, so the classes are the flow-independent ones (identical for every maximum flow):
//   bottleneck     raising the capacity by one raises the maximum flow: in the residual graph
//                  of a maximum flow, s reaches the edge's tail and its head reaches t;
//   underutilized  capacity >= 1 and lowering it by one keeps the maximum flow: the edge has
//                  spare capacity, or its tail reaches its head in the residual graph.
//
//   classes_kernel  one workgroup per candidate: the residual graph of the flow given by
//                   kv_flow (node flows follow by conservation), contracted to the replicas' KV
//                   sides, its transitive closure as bitset rows in LDS (64 pivots at a time), then
//                   the class of every edge;
//   moves_kernel    one workgroup per (parent, 256 children): the parent's donor GPUs,
//                   receiver groups and flip-eligible groups, listed in ascending id in LDS;
//                   then a lane per child applies one MOVE, SWAP or FLIP chosen by its draw;
//   gather_kernel   copies chosen columns of a batch (the best child) into another batch.
// All three are graph and byte work, not dense contractions: no MFMA.
#include "hx_internal.h"

namespace hx {
namespace {

__device__ __forceinline__ void drain_barrier() {
    // LDS atomics with unused results must have landed before the workgroup reads their
    // targets: wait for this wave's LDS operations (lgkmcnt(0)), then the barrier.
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __syncthreads();
}

struct ClsArgs {
    FlowNet f;
    const int32_t* flow_value;
    const int32_t* kv_flow;
    uint8_t* node_cls;
    uint8_t* kv_cls;
};

// The closure runs on the contracted residual graph: a replica's coordinator-side vertex (prefill in,
// decode out) has one neighbour on either side, so reachability through it follows from the node
// flows, and the vertices kept are din(j) = j, pout(i) = D + i, s = P + D and t = s + 1 (at most 257)
// with
//   pout(i) -> din(j) when the KV edge has room, din(j) -> pout(i) when it carries flow;
//   s -> pout(i) when source and node edge have room, pout(i) -> s when prefill i carries flow;
//   din(j) -> t when node and sink edge have room, t -> din(j) when decode j carries flow.
// A wavefront per network takes at most 64 nodes (kBlock 64), a workgroup of four 255.
template <int kBlock>
struct ClsShape {
    static constexpr int kNodes = kBlock == 64 ? 64 : kClsMaxV / 2 - 1;
    static constexpr int kRows = kNodes + 2;
    static constexpr int kWords = (kRows + 63) / 64;  // bitset words per row
    static constexpr int kStride = kWords | 1;        // odd, so that the rows of a wavefront's lanes spread over the banks
};

__device__ __forceinline__ uint64_t lane_word(uint64_t v, int k) {
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), k) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)v, k);
}

// acc | OR over the set bits k < nk of m of v's value in lane k (m: this lane's mask; nk a multiple
// of 8 at most 64).
__device__ __forceinline__ uint64_t or_lanes(uint64_t acc, uint64_t m, uint64_t v, int nk) {
    for (int k0 = 0; k0 < nk; k0 += 8)
#pragma unroll
        for (int x = 0; x < 8; ++x) acc |= (0 - ((m >> (k0 + x)) & 1)) & lane_word(v, k0 + x);
    return acc;
}

// Transitive closure of V rows of kW words (row stride kS), 64 pivots at a time: the pivots'
// own 64 x 64 block is closed in registers (a lane per row, Warshall's order, no barrier: every
// wavefront forms it itself), the pivot rows take the rows that this block reaches, then every other
// row takes the pivot rows its word of the block names.  Three barriers per 64 vertices where one
// pivot at a time takes 64.
template <int kW, int kS, int kBlock>
__device__ void closure(uint64_t* reach, int V) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int kb = 0; kb < kW; ++kb) {
        const int nk = V - 64 * kb < 64 ? V - 64 * kb : 64, nk8 = (nk + 7) & ~7;
        uint64_t* prow = reach + (64 * kb + lane) * kS;
        uint64_t d = lane < nk ? prow[kb] : 0;
        if (kW > 1) __syncthreads();  // every wavefront has the block
        for (int k0 = 0; k0 < nk8; k0 += 8)
#pragma unroll
            for (int x = 0; x < 8; ++x) d |= (0 - ((d >> (k0 + x)) & 1)) & lane_word(d, k0 + x);
        for (int w = wave; w < kW; w += kBlock / 64) {
            if (w == kb) {
                if (lane < nk) prow[w] = d;
                continue;
            }
            const uint64_t v = lane < nk ? prow[w] : 0;
            const uint64_t acc = or_lanes(v, d, v, nk8);
            if (lane < nk) prow[w] = acc;
        }
        __syncthreads();
        if (kW == 1) return;
        for (int u = tid; u < V; u += kBlock) {
            if ((u >> 6) == kb) continue;
            uint64_t* ru = reach + u * kS;
            const uint64_t m = ru[kb];
            uint64_t acc[kW];
#pragma unroll
            for (int w = 0; w < kW; ++w) acc[w] = ru[w];
            for (int k = 0; k < nk; ++k) {
                const uint64_t on = 0 - ((m >> k) & 1);
                const uint64_t* rk = reach + (64 * kb + k) * kS;
#pragma unroll
                for (int w = 0; w < kW; ++w) acc[w] |= rk[w] & on;
            }
#pragma unroll
            for (int w = 0; w < kW; ++w) ru[w] = acc[w];
        }
        __syncthreads();
    }
}

// What bounds it: the closure's instructions, and the loads of the KV rows (one 4-byte word of a
// cache line each; the XCD-aware order lets neighbouring candidates share the lines in one L2).  Each
// KV row is read once: a wavefront per prefill node turns it into bit words with ballots.  Measured
// against a closure of all 2 + 2 (P + D) vertices by one pivot per barrier that read the KV rows seven
// times: one network of 128 GPUs 181 -> 34 us, 8,192 networks of 64 GPUs' replicas 200 -> 28 us, 4,096 of
// 16 to 64 nodes a side 855 -> 130 us.
template <int kBlock>
__global__ void __launch_bounds__(kBlock) classes_kernel(ClsArgs a) {
    using Sh = ClsShape<kBlock>;
    constexpr int kS = Sh::kStride;
    __shared__ uint64_t reach[Sh::kRows * kS];                      // row u: the vertices u reaches
    __shared__ uint64_t some[Sh::kNodes][(Sh::kNodes + 63) / 64];  // prefill i: its KV edges of capacity >= 1
    __shared__ int32_t pf[Sh::kNodes], df[Sh::kNodes];
    const FlowNet& f = a.f;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t N = f.N;
    const int chunk = (int)((N + 7) / 8);
    const int n = (int)(blockIdx.x & 7) * chunk + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= chunk || n >= N) return;  // uniform
    const int P = f.n_p[n], D = f.n_d[n];
    // a network that does not fit its arrays or the closure's LDS rows, or whose max-flow
    // failed, gets no classes
    if (P < 0 || D < 0 || P > f.max_p || D > f.max_d || P * D > f.max_pd || P + D > Sh::kNodes ||
        a.flow_value[n] < 0) {
        for (int r = tid; r < f.max_p + f.max_d; r += kBlock) a.node_cls[(int64_t)r * N + n] = 0;
        return;
    }
    const int V = P + D + 2, W = (V + 63) >> 6, vs = P + D, vt = vs + 1;
    for (int e = tid; e < V * kS; e += kBlock) reach[e] = 0;
    for (int j = tid; j < D; j += kBlock) df[j] = 0;
    __syncthreads();
    // a wavefront per prefill node: its KV row's bit words, its flow (the row's sum), and the decode
    // nodes' flows and reverse arcs
    for (int i = wave; i < P; i += kBlock / 64) {
        uint64_t* row = reach + (D + i) * kS;
        int32_t sum = 0;
        for (int j0 = 0; j0 < D; j0 += 64) {
            const int j = j0 + lane;
            const int64_t o = (int64_t)(i * D + (j < D ? j : D - 1)) * N + n;
            const int32_t fl = j < D ? a.kv_flow[o] : 0, c = j < D ? f.kv_cap[o] : 0;
            const uint64_t room = __ballot(fl < c), any = __ballot(c >= 1);
            if (lane == 0) {
                row[j0 >> 6] |= room;
                some[i][j0 >> 6] = any;
            }
            sum += fl;
            if (fl != 0) atomicAdd(&df[j], fl);
            if (fl > 0)
                atomicOr((unsigned long long*)&reach[j * kS + ((D + i) >> 6)], 1ull << ((D + i) & 63));
        }
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
        if (lane == 0) pf[i] = sum;
    }
    drain_barrier();
    // the arcs at s and t, and every vertex reaching itself
    auto set = [&](int u, int v) {
        atomicOr((unsigned long long*)&reach[u * kS + (v >> 6)], 1ull << (v & 63));
    };
    for (int u = tid; u < V; u += kBlock) set(u, u);
    for (int i = tid; i < P; i += kBlock) {
        const int64_t o = (int64_t)i * N + n;
        if (pf[i] < f.src_cap[o] && pf[i] < f.p_cap[o]) set(vs, D + i);
        if (pf[i] > 0) set(D + i, vs);
    }
    for (int j = tid; j < D; j += kBlock) {
        const int64_t o = (int64_t)j * N + n;
        if (df[j] < f.d_cap[o] && df[j] < f.sink_cap[o]) set(j, vt);
        if (df[j] > 0) set(vt, j);
    }
    drain_barrier();
    if (W == 1) closure<1, kS, kBlock>(reach, V);
    else if (W == 2) closure<2, kS, kBlock>(reach, V);
    else if constexpr (Sh::kWords > 2) {
        if (W == 3) closure<3, kS, kBlock>(reach, V);
        else closure<Sh::kWords, kS, kBlock>(reach, V);
    }

    auto reaches = [](int u, int v) { return (int)((reach[u * kS + (v >> 6)] >> (v & 63)) & 1ull); };
    // bit 0: bottleneck (s reaches the tail, the head reaches t); bit 1: underutilized (capacity c >= 1
    // and room left, or the tail reaches the head otherwise: `around`, asked of saturated edges)
    auto cls = [](int tail, int head, int32_t fl, int32_t c, int around) {
        return (tail & head) | (c >= 1 && (fl < c || around) ? 2 : 0);
    };
    const int st = reaches(vs, vt);
    bool any_p = false, any_d = false;  // some pout that s reaches, some din that reaches t
    for (int w = 0; w < W; ++w) {
        const int lo = 64 * w;
        const uint64_t dins = D - lo >= 64 ? ~0ull : (D > lo ? (1ull << (D - lo)) - 1 : 0);
        const uint64_t core = vs - lo >= 64 ? ~0ull : (vs > lo ? (1ull << (vs - lo)) - 1 : 0);
        any_p |= (reach[vs * kS + w] & core & ~dins) != 0;
    }
    for (int j0 = 0; j0 < D; j0 += 64) any_d |= __any(j0 + lane < D && reaches(j0 + lane < D ? j0 + lane : 0, vt)) != 0;
    for (int i = tid; i < P; i += kBlock) {
        const int64_t o = (int64_t)i * N + n;
        const int32_t fl = pf[i], cp = f.p_cap[o], cs = f.src_cap[o];
        const int s_out = reaches(vs, D + i), out_t = reaches(D + i, vt);
        const int s_in = (fl < cs) | (s_out & (fl > 0));                    // s reaches the in-node
        const int in_t = ((fl < cp) & out_t) | ((fl > 0) & st);             // the in-node reaches t
        const int k = cls(s_in, out_t, fl, cp, s_out) | (cls(1, in_t, fl, cs, s_out) << 2);
        a.node_cls[o] = (uint8_t)(k | ((s_out && any_d ? 1 : 0) << 4));
    }
    for (int j = tid; j < D; j += kBlock) {
        const int64_t o = (int64_t)j * N + n;
        const int32_t fl = df[j], cd = f.d_cap[o], ct = f.sink_cap[o];
        const int s_in = reaches(vs, j), in_t = reaches(j, vt);
        const int out_t = (fl < ct) | (in_t & (fl > 0));                    // the out-node reaches t
        const int s_out = ((fl < cd) & s_in) | ((fl > 0) & st);             // s reaches the out-node
        const int k = cls(s_in, out_t, fl, cd, in_t) | (cls(s_out, 1, fl, ct, in_t) << 2);
        a.node_cls[(int64_t)(f.max_p + j) * N + n] = (uint8_t)(k | ((in_t && any_p ? 1 : 0) << 4));
    }
    // a KV edge with room is an arc of the closure, so its second bit is capacity and reachability
    for (int i = wave; i < P; i += kBlock / 64) {
        const int s_out = reaches(vs, D + i);
        for (int j = lane; j < D; j += 64) {
            const int c1 = (int)((some[i][j >> 6] >> (j & 63)) & 1);
            a.kv_cls[(int64_t)(i * D + j) * N + n] =
                (uint8_t)((s_out & reaches(j, vt)) | ((c1 & reaches(D + i, j)) << 1));
        }
    }
}

// ------------------------------------------------------------------ guided moves

constexpr int kMoveBlock = 256;  // >= HX_MAX_GPUS + 1 and HX_MAX_GROUPS + 1: a lane per GPU / group

struct MoveArgs {
    int32_t G, K, gran, M, n_child, max_p, max_d;
    const uint8_t *p_assign, *p_role;            // [G][M], [K][M]
    const int32_t *n_p, *n_d, *p_slot, *d_slot;  // the parents' network
    const uint8_t* node_cls;                     // [max_p + max_d][M]
    const uint64_t* rnd;                         // [n_child]
    uint8_t *c_assign, *c_role;                  // [G][n_child], [K][n_child]
    int32_t* move;                               // [n_child]
};

// Index into m candidates from a b-bit draw u: floor(u m / 2^b).
__device__ __forceinline__ int pick(uint64_t u, int m, int bits) { return (int)((u * (uint64_t)m) >> bits); }

// Block-wide compaction of lane flags into an ascending list of lane ids; returns the count.
__device__ int compact(bool flag, uint8_t* list, int32_t* wave_cnt) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t b = __ballot(flag);
    if (lane == 0) wave_cnt[wave] = __popcll(b);
    __syncthreads();
    int off = 0, total = 0;
    for (int w = 0; w < kMoveBlock / 64; ++w) {
        if (w < wave) off += wave_cnt[w];
        total += wave_cnt[w];
    }
    if (flag) list[off + __popcll(b & ((1ull << lane) - 1))] = (uint8_t)tid;
    __syncthreads();  // wave_cnt is reused by the next compaction
    return total;
}

__global__ void __launch_bounds__(kMoveBlock) moves_kernel(MoveArgs a) {
    __shared__ uint8_t pa[256], pr[256];
    __shared__ int16_t grp[256];
    __shared__ int32_t node_p[256], node_d[256];  // slot key -> node index (largest on repeats)
    __shared__ int32_t members[256], donors_in[256];
    __shared__ uint8_t donor[256], recv[256];
    __shared__ int32_t recv_role[2];
    __shared__ uint8_t recv_list[256], donor_list[256], rgpu_list[256], flip_list[256];
    __shared__ int32_t wave_cnt[kMoveBlock / 64];
    const int m = blockIdx.y, tid = threadIdx.x;
    const int G = a.G, K = a.K, M = a.M;
    if (tid < G) pa[tid] = a.p_assign[(int64_t)tid * M + m];
    if (tid < K) pr[tid] = a.p_role[(int64_t)tid * M + m];
    members[tid] = 0;
    donors_in[tid] = 0;
    recv[tid] = 0;
    node_p[tid] = -1;
    node_d[tid] = -1;
    if (tid < 2) recv_role[tid] = 0;
    int P = a.n_p[m], D = a.n_d[m];
    if (P < 0 || D < 0 || P > a.max_p || D > a.max_d) P = D = 0;  // no usable network
    __syncthreads();
    // groups and flow-node lookup
    int g_grp = -1;
    if (tid < G) {
        const int as = pa[tid];
        const int r = as < K ? pr[as] : HX_UNUSED;
        g_grp = (as < K && (r == HX_PREFILL || r == HX_DECODE)) ? as : -1;
        grp[tid] = (int16_t)g_grp;
        if (g_grp >= 0) atomicAdd(&members[g_grp], 1);
    }
    for (int i = tid; i < P; i += kMoveBlock) {
        const int key = a.p_slot[(int64_t)i * M + m];
        if (key >= 0 && key < 256) atomicMax(&node_p[key], i);
    }
    for (int j = tid; j < D; j += kMoveBlock) {
        const int key = a.d_slot[(int64_t)j * M + m];
        if (key >= 0 && key < 256) atomicMax(&node_d[key], j);
    }
    drain_barrier();
    // donors (unused, or an underutilized node edge) and receivers (a bottleneck node or KV
    // edge at a member's node)
    bool is_donor = false;
    if (tid < G) {
        is_donor = g_grp < 0;
        if (g_grp >= 0) {
            const int key = a.gran == 0 ? g_grp : tid;
            const int role = pr[g_grp];
            const int row = role == HX_PREFILL ? node_p[key] : (node_d[key] >= 0 ? a.max_p + node_d[key] : -1);
            if (row >= 0) {
                const uint8_t nc = a.node_cls[(int64_t)row * M + m];
                if (nc & 2) is_donor = true;
                if (nc & 17) {
                    recv[g_grp] = 1;
                    recv_role[role] = 1;
                }
            }
            if (is_donor) atomicAdd(&donors_in[g_grp], 1);
        }
        donor[tid] = is_donor;
    }
    drain_barrier();
    bool flip = false;
    if (tid < K && members[tid] > 0 && !recv[tid] && donors_in[tid] == members[tid])
        flip = recv_role[1 - pr[tid]] != 0;
    const int n_recv = compact(tid < K && recv[tid], recv_list, wave_cnt);
    const int n_flip = compact(flip, flip_list, wave_cnt);
    const int n_donor = compact(is_donor, donor_list, wave_cnt);
    const int n_rgpu = compact(tid < G && g_grp >= 0 && recv[g_grp], rgpu_list, wave_cnt);

    // one child per lane: children m, m + M, m + 2M, ... descend from parent m
    const int64_t t = (int64_t)blockIdx.x * kMoveBlock + tid;
    const int64_t c = m + t * M;
    if (c >= a.n_child) return;
    const int64_t Nc = a.n_child;
    int code = 0, g1 = -1, g2 = -1, v1 = 0, v2 = 0, fk = -1;
    if (c >= M) {
        const uint64_t r = a.rnd[c];
        const uint64_t u0 = r & 0xFFFFull, u1 = (r >> 16) & 0xFFFFFFull, u2 = r >> 40;
        const int t0 = pick(u0, 3, 16);
        for (int at = 0; at < 3 && code == 0; ++at) {
            const int ty = (t0 + at) % 3;
            if (ty == 0 && n_recv > 0) {
                const int k = recv_list[pick(u1, n_recv, 24)];
                const int na = n_donor - donors_in[k];
                if (na == 0) continue;
                int want = pick(u2, na, 24), g = -1;
                for (int x = 0; x < n_donor; ++x) {
                    const int d = donor_list[x];
                    if (grp[d] == k) continue;
                    if (want-- == 0) { g = d; break; }
                }
                g1 = g;
                v1 = k;
                code = 1 | (g << 8) | (k << 16);
            } else if (ty == 1 && n_rgpu > 0) {
                const int g = rgpu_list[pick(u1, n_rgpu, 24)];
                const int kg = grp[g];
                const int na = n_donor - donors_in[kg];
                if (na == 0) continue;
                int want = pick(u2, na, 24), h = -1;
                for (int x = 0; x < n_donor; ++x) {
                    const int d = donor_list[x];
                    if (grp[d] == kg) continue;
                    if (want-- == 0) { h = d; break; }
                }
                g1 = g;
                v1 = pa[h];
                g2 = h;
                v2 = pa[g];
                code = 2 | (g << 8) | (h << 16);
            } else if (ty == 2 && n_flip > 0) {
                fk = flip_list[pick(u1, n_flip, 24)];
                code = 3 | (fk << 8);
            }
        }
    }
    for (int g = 0; g < G; ++g)
        a.c_assign[(int64_t)g * Nc + c] = g == g1 ? (uint8_t)v1 : (g == g2 ? (uint8_t)v2 : pa[g]);
    for (int k = 0; k < K; ++k) a.c_role[(int64_t)k * Nc + c] = k == fk ? (uint8_t)(1 - pr[k]) : pr[k];
    a.move[c] = code;
}

// ------------------------------------------------------------------ gather

__global__ void gather_kernel(int G, int K, int Ns, const uint8_t* sa, const uint8_t* sr, const int32_t* index,
                              int count, uint8_t* da, uint8_t* dr) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)(G + K) * count) return;
    const int row = (int)(e / count), m = (int)(e - (int64_t)row * count);
    const int idx = index[m];
    const bool ok = idx >= 0 && idx < Ns;
    if (row < G) da[(int64_t)row * count + m] = ok ? sa[(int64_t)row * Ns + idx] : (uint8_t)HX_UNUSED;
    else dr[(int64_t)(row - G) * count + m] = ok ? sr[(int64_t)(row - G) * Ns + idx] : (uint8_t)HX_UNUSED;
}

}  // namespace

hipError_t launch_classes(const FlowNet& f, const int32_t* flow_value, const int32_t* kv_flow, uint8_t* node_cls,
                          uint8_t* kv_cls, hipStream_t s) {
    prof_mark(kKClasses, false, s);
    const ClsArgs a{f, flow_value, kv_flow, node_cls, kv_cls};
    const dim3 grid(8 * (unsigned)(((int64_t)f.N + 7) / 8));  // XCD-aware order
    // one wavefront per network where the arrays hold at most 64 nodes in all: at most two bit words a
    // row, and several networks per CU
    if (f.max_p + f.max_d <= 64)
        hipLaunchKernelGGL(classes_kernel<64>, grid, dim3(64), 0, s, a);
    else
        hipLaunchKernelGGL(classes_kernel<256>, grid, dim3(256), 0, s, a);
    prof_mark(kKClasses, true, s);
    return hipGetLastError();
}

hipError_t launch_moves(int32_t G, int32_t K, int32_t gran, int32_t M, const uint8_t* p_assign,
                        const uint8_t* p_role, const FlowNet& pn, const uint8_t* node_cls, int32_t n_child,
                        const uint64_t* rnd, uint8_t* c_assign, uint8_t* c_role, int32_t* move, hipStream_t s) {
    const int64_t per = ((int64_t)n_child + M - 1) / M;  // children of parent 0, the most
    const dim3 grid((unsigned)((per + kMoveBlock - 1) / kMoveBlock), (unsigned)M);
    MoveArgs a{G, K, gran, M, n_child, pn.max_p, pn.max_d, p_assign, p_role, pn.n_p, pn.n_d, pn.p_slot, pn.d_slot,
               node_cls, rnd, c_assign, c_role, move};
    prof_mark(kKMoves, false, s);
    hipLaunchKernelGGL(moves_kernel, grid, dim3(kMoveBlock), 0, s, a);
    prof_mark(kKMoves, true, s);
    return hipGetLastError();
}

hipError_t launch_gather(int32_t G, int32_t K, int32_t Ns, const uint8_t* sa, const uint8_t* sr, const int32_t* index,
                         int32_t count, uint8_t* da, uint8_t* dr, hipStream_t s) {
    const int64_t cells = (int64_t)(G + K) * count;
    prof_mark(kKGather, false, s);
    hipLaunchKernelGGL(gather_kernel, dim3((unsigned)((cells + 255) / 256)), dim3(256), 0, s, G, K, Ns, sa, sr, index,
                       count, da, dr);
    prof_mark(kKGather, true, s);
    return hipGetLastError();
}

}  // namespace hx
