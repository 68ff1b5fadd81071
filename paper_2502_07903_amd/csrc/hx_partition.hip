// hx_partition.hip -- the graph-partition phase of Sec. 3.2 as a candidate generator, on gfx950.
//
// The device graph has the GPUs as nodes, weighted by memory, and the links as edges, weighted by
// bandwidth.  Edge weights are whole MB/s of the symmetrised bandwidth (clamped to 2^47, which
// keeps every cut of a graph of up to 255 GPUs below 2^62), so every cut, gain and coarsened
// weight is an exact 64-bit integer sum and does not depend on the order of the additions; only
// the spectral step is floating point, and it sums in ascending index order.
//
//   graph_kernel      one lane per GPU pair: w = floor(((beta_de + beta_ed) * 0.5) / 1e6);
//   spectral_kernel   one workgroup: power iteration on (cap I - Lap) for the Fiedler direction,
//                     a lane per row (ascending products), the mean and the squared norm summed in
//                     ascending order (the order depends only on the cluster, so a search computes
//                     it once); the GPUs ranked by (x, id);
//   partition_gain_kernel, partition_kernel  a candidate each: (i) the rotated spectral order cut into K
//                     memory-balanced groups, then Kernighan-Lin passes: every pair of GPUs has its
//                     swap's gain, kept up to date in registers (or, past the exact ranges of
//                     binary64, formed anew from per-GPU group sums), a maximum over them picks the
//                     largest reduction (negative ones too; lowest pair on ties), the swap is made
//                     tentatively and its two GPUs locked; the pass keeps its best prefix and undoes
//                     the rest; (ii) groups coarsened into super nodes (LDS
//                     atomics) and split into prefill and decode by single flips that raise the
//                     cut; (iii) the projection written as the candidate's assign and role columns.
// Graph and integer work: no MFMA.
#include "hx_internal.h"

namespace hx {
namespace {

constexpr int kPgBlock = 256;   // >= HX_MAX_GPUS + 1: a lane per GPU
constexpr int kPgMaxK = 32;     // groups of one candidate
constexpr double kPgWeightMax = 140737488355328.0;  // 2^47 MB/s
constexpr int kKlPasses = 64;   // Kernighan-Lin passes at most

__global__ void graph_kernel(int G, const double* beta, int64_t* w) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)G * G) return;
    const int d = (int)(i / G), e = (int)(i - (int64_t)d * G);
    double v = 0.0;
    if (d != e) {
        v = floor(((beta[(int64_t)d * G + e] + beta[(int64_t)e * G + d]) * 0.5) / 1.0e6);
        if (!(v >= 0.0)) v = 0.0;
        if (v > kPgWeightMax) v = kPgWeightMax;
    }
    w[i] = (int64_t)v;
}

// s + element 0 + element 1 + ... + element 15 of v, in that order, where lane l of every row of
// sixteen lanes holds element l: row_newbcast hands element k to every lane as the operand of
// fma(element, 1.0, s), the one binary64 form that takes it, which rounds as s + element does.
// 6.3 cycles an element, the latency of the addition; the s_nop covers a VALU write of v just before.
__device__ __forceinline__ double add16(double s, double v) {
    asm("s_nop 1\n"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:0 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:1 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:2 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:4 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:5 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:6 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:7 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:8 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:9 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:10 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:11 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:12 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:13 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:14 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f64_dpp %0, %1, %2 row_newbcast:15 row_mask:0xf bank_mask:0xf\n"
        : "+v"(s)
        : "v"(v), "v"(1.0));
    return s;
}
// v[0] + v[1] + ... + v[G - 1] from 0.0, v in LDS with zeros up to 16 kB >= G (adding +0.0 to a sum
// that started at +0.0 changes no bit).  Every lane forms the same sum, so nothing has to be
// broadcast back; one LDS read per sixteen elements.
template <int kB>
__device__ __forceinline__ double sum_in_order(const double* v) {
    double c[kB];
#pragma unroll
    for (int i = 0; i < kB; ++i) c[i] = v[16 * i + (threadIdx.x & 15)];
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < kB; ++i) s = add16(s, c[i]);
    return s;
}

// A lane per GPU row, 16 kB >= G; kRegs: the row stays in registers (up to 128 GPUs), otherwise it is
// read from memory in every iteration.  An iteration is three chains of G dependent additions, whose
// order is part of the result: the row's product, the mean and the squared norm.  The row stays in
// registers as binary64 and every lane forms both sums itself, which leaves the chains, two divisions
// and a square root (110 to 150 cycles each) and three barriers (a wait when one wavefront holds the
// cluster).  kB is a template parameter because the loops over it then have no branches: with the
// chunks tested against G, 1,000 iterations at 32 GPUs took 665 us against 784.  Before, the row was
// read from memory in every iteration and one lane formed the sums: 2.0 ms at 32 GPUs, 6.6 at 100
// (now 1.76).
template <int kB, bool kRegs>
__global__ void __launch_bounds__((kB + 3) / 4 * 64) spectral_kernel(int G, const int64_t* w, int iters, int32_t* order,
                                                                     double* fiedler) {
    constexpr int kBlock = (kB + 3) / 4 * 64, kLen = 16 * kB;
    __shared__ __attribute__((aligned(16))) double x[kLen], y[kLen], sq[kLen];
    __shared__ double deg[kLen];
    const int d = threadIdx.x;
    double row[kRegs ? kLen : 1];
    for (int e = d; e < kLen; e += kBlock) x[e] = y[e] = sq[e] = 0.0;
    __syncthreads();
    double dg = 0.0, xd = 0.0;
    if (d < G) {
        long long s = 0;
        for (int e = 0; e < G; ++e) s += w[(int64_t)e * G + d];  // column = row: w is symmetric
        dg = (double)s;
        deg[d] = dg;
        xd = (double)d - (double)(G - 1) * 0.5;
        x[d] = xd;
    }
    if (kRegs) {
        const int dc = d < G ? d : G - 1;
#pragma unroll
        for (int e = 0; e < kLen; ++e) row[e] = (double)w[(int64_t)(e < G ? e : G - 1) * G + dc];
    }
    __syncthreads();
    double cap = 0.0;
    for (int e = 0; e < G; ++e)
        if (2.0 * deg[e] > cap) cap = 2.0 * deg[e];
    const double Gd = (double)G;
    for (int it = 0; it < iters; ++it) {
        double s = 0.0;
        if (kRegs) {
            // x is 0 past G, where the row repeats its last entry
#pragma unroll
            for (int e0 = 0; e0 < kLen; e0 += 16) {
                double2 c[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) c[i] = reinterpret_cast<const double2*>(x + e0)[i];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    s = s + row[e0 + 2 * i] * c[i].x;
                    s = s + row[e0 + 2 * i + 1] * c[i].y;
                }
            }
        } else {
            // kC weights in flight while the chunk before is summed; lanes past G read the last column, rows
            // past G the last row, where x is 0 as above.  1,000 iterations at 129, 160, 200, 255 GPUs: 7.8, 9.4,
            // 11.7, 15.4 ms with one lane forming the sums, 10.7, 12.5, 16.6, 20.7 with eight weights loaded, then
            // summed, 6.2, 6.7, 8.2, 9.6 now (32 or 64 weights: 10.9 and 12.9 at 255).
            constexpr int kC = 16;
            const int dc = d < G ? d : G - 1;
            int64_t next[kC];
            auto load = [&](int e0) {
#pragma unroll
                for (int i = 0; i < kC; ++i) next[i] = w[(int64_t)(e0 + i < G ? e0 + i : G - 1) * G + dc];
            };
            load(0);
            for (int e0 = 0; e0 < G; e0 += kC) {
                int64_t v[kC];
#pragma unroll
                for (int i = 0; i < kC; ++i) v[i] = next[i];
                if (e0 + kC < G) load(e0 + kC);
#pragma unroll
                for (int i = 0; i < kC; ++i) s = s + (double)v[i] * x[e0 + i];
            }
        }
        const double yv = (cap - dg) * xd + s;
        if (d < G) y[d] = yv;
        __syncthreads();
        const double yd = yv - sum_in_order<kB>(y) / Gd;
        if (d < G) sq[d] = yd * yd;
        __syncthreads();
        const double nrm = sqrt(sum_in_order<kB>(sq));
        if (!(nrm > 0.0)) break;  // uniform: every lane formed the same value
        xd = yd / nrm;
        if (d < G) x[d] = xd;
        __syncthreads();
    }
    if (d < G) {
        int rank = 0;
        for (int e = 0; e < G; ++e) rank += (x[e] < x[d] || (x[e] == x[d] && e < d)) ? 1 : 0;
        order[rank] = d;
        if (fiedler) fiedler[d] = x[d];
    }
}

// The instantiation for G GPUs.
template <int kB>
void launch_spectral_b(int b, int G, const int64_t* w, int iters, int32_t* order, double* fiedler, hipStream_t s) {
    if constexpr (kB > 16) {
        return;
    } else {
        if (b != kB) return launch_spectral_b<(kB < 8 ? kB + 1 : kB + 8)>(b, G, w, iters, order, fiedler, s);
        hipLaunchKernelGGL((spectral_kernel<kB, (kB <= 8)>), dim3(1), dim3((kB + 3) / 4 * 64), 0, s, G, w, iters, order,
                           fiedler);
    }
}

__device__ __forceinline__ void drain_barrier() {
    __builtin_amdgcn_s_waitcnt(0xC07F);  // this wave's LDS operations done (lgkmcnt(0))
    __syncthreads();
}

// (gain, pair) ordered by larger gain, then lower pair index; pair kNoPair = none.
constexpr int kNoPair = 0x7fffffff;
__device__ __forceinline__ bool better(long long g, int p, long long g2, int p2) {
    return p != kNoPair && (p2 == kNoPair || g > g2 || (g == g2 && p < p2));
}

// Workgroup best (gain, pair): every lane receives it.
__device__ void block_best(long long& g, int& p, long long* redg, int* redp) {
    for (int s = 32; s > 0; s >>= 1) {
        const long long og = __shfl_xor(g, s, 64);
        const int op = __shfl_xor(p, s, 64);
        if (better(og, op, g, p)) {
            g = og;
            p = op;
        }
    }
    if ((threadIdx.x & 63) == 0) {
        redg[threadIdx.x >> 6] = g;
        redp[threadIdx.x >> 6] = p;
    }
    __syncthreads();
    g = redg[0];
    p = redp[0];
    for (int k = 1; k < kPgBlock / 64; ++k)
        if (better(redg[k], redp[k], g, p)) {
            g = redg[k];
            p = redp[k];
        }
    __syncthreads();
}

struct PgArgs {
    int G, Kmax, N, L;
    double H, Hkv, B, s_in, s_out;
    const int64_t* w;        // [G][G]
    const int32_t* order;    // [G] spectral order
    const int32_t* gpu_type;
    const double* mem;       // [T] memory limits
    int T;
    const uint64_t* rnd;     // [N]
    uint8_t *assign, *role;  // [G][N], [Kmax][N]
};

// Exchange GPUs u and v (different groups): the per-GPU group sums follow (a lane per GPU), then
// lane 0 moves the two GPUs and the groups' memory.  The same call undoes it.
__device__ void pg_exchange(const PgArgs& a, int u, int v, int* grp, long long* gval, long long* gmem,
                            const long long* memv) {
    const int G = a.G, tid = threadIdx.x;
    const int A = grp[u], B = grp[v];
    if (tid < G) {
        const long long wxu = a.w[(int64_t)u * G + tid], wxv = a.w[(int64_t)v * G + tid];
        gval[tid * kPgMaxK + A] += wxv - wxu;
        gval[tid * kPgMaxK + B] += wxu - wxv;
    }
    __syncthreads();
    if (tid == 0) {
        gmem[A] += memv[v] - memv[u];
        gmem[B] += memv[u] - memv[v];
        grp[u] = B;
        grp[v] = A;
    }
    __syncthreads();
}

// Dynamic LDS of partition_kernel: gval[u][k], the sum of w(u, x) over the GPUs x of group k.
__host__ __device__ inline size_t pg_lds_bytes(int G) { return (size_t)G * kPgMaxK * sizeof(long long); }

// ------------------------------------------------------------------ partition, incremental gains
//
// The same search with every pair's gain kept in a register.  Swapping u (group A) with v (group B)
// moves w(x, v) - w(x, u) =: d_x from x's sum over B to its sum over A, so with s = +1 in A, -1 in B
// and 0 elsewhere the gain of a pair (x, y) changes by (d_x - d_y)(s_y - s_x): three binary64
// operations per pair where rescanning it reads four group sums, two groups, their memories and a
// weight.  Likewise with h_x = the memory of x's group without x, the swap (x, y) does not widen the
// memory gap when (m_y - m_x)(h_x - h_y) <= 0, and h follows the swaps by h_x += s_x (m_v - m_u).
//
// A pair's key is 2^16 gain + (2^16 - 1 - pair) as a binary64 integer, so that one maximum picks the
// largest gain and, on ties, the lowest pair.  All values are whole numbers held exactly, which needs
// a row of weights below 2^29 MB/s and memories below 2^52 in all: graphs past these (links of 16 TB/s
// at 32 GPUs, 2 TB/s at 255) are left to partition_kernel, which holds them as 64-bit integers.
//
// The pairs are laid out as (a, a + s mod G), s = 1 .. G/2: lane a of a set of P lanes holds node a's
// state, and the NT / P sets take every (NT / P)-th shift s.  A node's partner is then at a constant
// LDS offset (node records are stored twice, at x and x + G).  Up to 64 GPUs a wavefront has a
// candidate to itself and needs no barrier; above, NT lanes share one.
//
// What bounds it: instruction issue, about 14 instructions a pair and step, and the latency of a step's
// reduction.  Measured against partition_kernel: 32 GPUs x 16,384 candidates 1,710 -> 363 us, 100 GPUs x
// 1,000 7.4 -> 2.2 ms (2.3 with the weights read from memory; 3.2 and 3.9 with registers bounded to 168
// and 128 for three and four wavefronts per SIMD, which spills; 2.5 with 512 lanes a candidate).
template <int P>
struct PgShape {
    static constexpr int kNT = P <= 64 ? 64 : (P == 128 ? 256 : 1024);  // lanes of a candidate
    static constexpr int kPer = P <= 64 ? 4 : 1;                        // candidates of a workgroup
    static constexpr int kSub = kNT / P;                                // sets of P lanes
    static constexpr int kSlots = P / 2 / kSub;                         // shifts of a lane, at most
    static constexpr int kBlock = kNT * kPer;
};

struct __attribute__((aligned(16))) PgNode {
    double h, d;  // group memory without the node (NaN: locked); 2^16 d_x of the last swap
};
struct __attribute__((aligned(8))) PgSide {
    int grp;
    float s;  // s_x of the last swap
};

// Dynamic LDS of one candidate: node records and sides (twice G), groups and memories, sums of
// weights by group (int32 [G][ld]), which the coarse weights (int64 [K][K]) later overwrite, and
// scalars.
__host__ __device__ inline size_t pg_fast_sums(int G, int K) {
    const size_t a = sizeof(int32_t) * (size_t)G * (K | 1), b = sizeof(long long) * (size_t)K * K;
    return ((a > b ? a : b) + 15) & ~(size_t)15;
}
__host__ __device__ inline size_t pg_fast_lds(int G, int K) {
    return 2 * (size_t)G * (sizeof(PgNode) + sizeof(PgSide)) + (((size_t)G * (sizeof(double) + sizeof(int))) + 15) / 16 * 16 +
           pg_fast_sums(G, K) + sizeof(long long) * kPgMaxK + 3 * sizeof(int) * kPgMaxK + 256;
}

// The largest x of a wavefront's lanes, by row shifts and row broadcasts (no LDS).
template <int kCtrl, int kRows>
__device__ __forceinline__ double dpp_max_step(double x) {
    const int lo = __double2loint(x), hi = __double2hiint(x);
    const double y = __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, kCtrl, kRows, 0xf, false),
                                      __builtin_amdgcn_update_dpp(lo, lo, kCtrl, kRows, 0xf, false));
    return y > x ? y : x;
}
__device__ __forceinline__ double wave_max(double x) {
    x = dpp_max_step<0x111, 0xf>(x);  // row_shr:1, 2, 4, 8: lane 15 of each row holds the row's
    x = dpp_max_step<0x112, 0xf>(x);
    x = dpp_max_step<0x114, 0xf>(x);
    x = dpp_max_step<0x118, 0xf>(x);
    x = dpp_max_step<0x142, 0xa>(x);  // row_bcast15: rows 1 and 3
    x = dpp_max_step<0x143, 0xc>(x);  // row_bcast31: rows 2 and 3
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 63),
                            __builtin_amdgcn_readlane(__double2loint(x), 63));
}

// Orders a candidate's LDS accesses: a barrier when several wavefronts share it.
template <int P>
__device__ __forceinline__ void pg_sync() {
    __builtin_amdgcn_s_waitcnt(0xC07F);  // LDS atomics landed (lgkmcnt(0))
    if (PgShape<P>::kPer == 1) {
        __syncthreads();
    } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// Workgroups of a grid row: HIP takes less than 2^32 threads in a dimension, which 2^22 workgroups of 1,024
// lanes would reach (partition_kernel alone took 2^24 candidates).
constexpr int64_t kPgGridX = 1 << 21;

constexpr double kPgNone = -4611686018427387904.0;  // -2^62: below every key

// kLdsW: the weights staged in LDS as 32-bit integers.
template <int P, bool kLdsW>
__global__ void __launch_bounds__(PgShape<P>::kBlock) partition_gain_kernel(PgArgs a, int Kh) {
    using Sh = PgShape<P>;
    constexpr int kNT = Sh::kNT, kSub = Sh::kSub, kSlots = Sh::kSlots;
    extern __shared__ __attribute__((aligned(16))) unsigned char pg_sm[];
    __shared__ double red[16];
    const int G = a.G, tid = threadIdx.x % kNT, cand = threadIdx.x / kNT;
    const int x = tid % P, sub = tid / P, lane = threadIdx.x & 63;
    const int64_t N = a.N;
    const int64_t n = ((int64_t)blockIdx.y * kPgGridX + blockIdx.x) * Sh::kPer + cand;
    int32_t* wl = reinterpret_cast<int32_t*>(pg_sm);  // kLdsW: [G][G]
    const size_t wbytes = kLdsW ? (sizeof(int32_t) * (size_t)G * G + 15) & ~(size_t)15 : 0;
    unsigned char* base = pg_sm + wbytes + cand * pg_fast_lds(G, Kh);
    PgNode* node = reinterpret_cast<PgNode*>(base);           // [2 G]
    PgSide* side2 = reinterpret_cast<PgSide*>(node + 2 * G);  // [2 G]
    double* memd = reinterpret_cast<double*>(side2 + 2 * G);  // [G]
    int* grp = reinterpret_cast<int*>(memd + G);              // [G]
    unsigned char* sums = base + 2 * (size_t)G * (sizeof(PgNode) + sizeof(PgSide)) +
                          ((size_t)G * (sizeof(double) + sizeof(int)) + 15) / 16 * 16;
    int32_t* gval = reinterpret_cast<int32_t*>(sums);  // [G][ld]
    long long* sw = reinterpret_cast<long long*>(sums);  // [Kh][Kh]
    long long* gmem = reinterpret_cast<long long*>(sums + pg_fast_sums(G, Kh));  // [32]
    int* first = reinterpret_cast<int*>(gmem + kPgMaxK);
    int* newid = first + kPgMaxK;
    int* side = newid + kPgMaxK;
    const int ld = Kh | 1;

    // the graph within the exact ranges?  (every workgroup finds the same answer)
    const long long wlimit = (1ll << 29) / (G + 1);  // sums of a row below 2^29, gains below 2^31
    bool bad = false;
    for (int e = threadIdx.x; e < G * G; e += Sh::kBlock) {
        const long long v = a.w[e];
        bad |= v >= wlimit;
        if (kLdsW) wl[e] = (int32_t)v;
    }
    double mx = 0.0;
    if (x < G) {
        const int t = a.gpu_type[x];
        mx = (t >= 0 && t < a.T) ? a.mem[t] : 0.0;
        bad |= !(mx >= 0.0 && mx < 17592186044416.0);  // 2^44: 255 of them stay below 2^52
        mx = floor(mx);
        if (sub == 0) memd[x] = mx;
    }
    bad = __syncthreads_or(bad) != 0;
    // a candidate left to partition_kernel is marked in its assignment: GPU 0 unused (its group is 0 in
    // every partition)
    if (bad && n < N && tid == 0) a.assign[n] = HX_UNUSED;
    if (bad || n >= N) return;  // wavefronts of their own candidates, or the whole workgroup
    auto weight = [&](int u, int v) -> int32_t {
        return kLdsW ? wl[u * G + v] : (int32_t)a.w[(int64_t)u * G + v];
    };

    const uint64_t r = a.rnd[n];
    // K: floor(total memory / replica memory), the replica holding the weights and the KV caches of 32
    // requests (Appendix A), shifted by the draw
    double mtot = 0.0;
    for (int e = 0; e < G; ++e) mtot = mtot + memd[e];
    long long total = (long long)mtot;
    const double Ld = (double)a.L;
    const double rep = 12.0 * a.H * a.H * a.B * Ld + 32.0 * (2.0 * (a.s_in + a.s_out) * a.Hkv * a.B * Ld);
    int K = (int)floor(mtot / rep) + (int)((r & 7) % 5) - 2;
    if (K > Kh) K = Kh;
    if (K < 2) K = 2;
    const int rot = (int)(((r >> 3) & 0xFF) % (uint64_t)G);
    if (total <= 0) total = 1;  // memories all zero: every GPU lands in group 0
    // step (i): the rotated spectral order cut by memory midpoints into K groups
    int dd = -1;
    double cum = 0.0;
    if (x < G) dd = a.order[(x + rot) % G];
    if (sub == 0 && x < G) {
        grp[x] = 0;
        gval[x] = dd;  // staged for the prefix sums
    }
    pg_sync<P>();
    for (int i = 0; i < G; ++i) {
        const int e = gval[i];
        const double m = e >= 0 && e < G ? memd[e] : 0.0;
        cum = cum + (i < x ? m : 0.0);
    }
    if (sub == 0 && x < G && dd >= 0 && dd < G) {
        const long long k = ((long long)K * (2 * (long long)cum + (long long)memd[dd])) / (2 * total);
        grp[dd] = (int)(k < K - 1 ? k : K - 1);
    }
    pg_sync<P>();
    int gx = x < G ? grp[x] : -1;

    double key[kSlots];
    float dm[kSlots];  // sign of m_y - m_x; NaN: no such pair
    // (lanes past G read lane 0's partners: at most G - 1 + G / 2 + kSub < 2 G)
    const PgNode* py = node + (x < G ? x : 0) + 1 + sub;
    const PgSide* ps = side2 + (x < G ? x : 0) + 1 + sub;
#pragma unroll
    for (int j = 0; j < kSlots; ++j) {
        const int s = 1 + sub + kSub * j;
        dm[j] = __builtin_nanf("");
        if (2 * s <= G && x < G && !(2 * s == G && x >= s)) {
            const int y = x + s < G ? x + s : x + s - G;
            const double d = memd[y] - mx;
            dm[j] = d > 0.0 ? 1.0f : (d < 0.0 ? -1.0f : 0.0f);
        }
    }
    for (int pass = 0; pass < kKlPasses; ++pass) {
        // sums of weights by group, and the groups' memories
        for (int e = tid; e < G * ld; e += kNT) gval[e] = 0;
        if (tid < kPgMaxK) gmem[tid] = 0;
        pg_sync<P>();
        if (x < G) {
            for (int e = sub; e < G; e += kSub) atomicAdd(&gval[x * ld + grp[e]], weight(e, x));
            if (sub == 0) atomicAdd((unsigned long long*)&gmem[gx], (unsigned long long)(long long)mx);
        }
        pg_sync<P>();
        double hx = 0.0;
        const int g0 = gx;
        if (x < G) {
            hx = (double)gmem[gx] - mx;
            if (sub == 0) {
                node[x] = node[x + G] = PgNode{hx, 0.0};
                side2[x] = side2[x + G] = PgSide{gx, 0.0f};
            }
        }
        pg_sync<P>();
        // the pass's opening gains.  (xo and Go hide x and G from the compiler, which would otherwise
        // keep every shift's partner, weight and pair in registers across passes, and its bounds in
        // scalar registers: 81 spilled registers at 64 GPUs.)
        int xo = x, Go = G;
        asm volatile("" : "+v"(xo));
        asm volatile("" : "+s"(Go));
#pragma unroll
        for (int j = 0; j < kSlots; ++j) {
            const int s = 1 + sub + kSub * j;
            key[j] = 0.0;
            if (2 * (1 + kSub * j) > Go) break;  // uniform: no lane has this shift
            if (2 * s <= Go && xo < Go && !(2 * s == Go && xo >= s)) {
                const int y = xo + s < Go ? xo + s : xo + s - Go;
                const int gy = grp[y];
                const int gain = (gval[xo * ld + gy] - gval[xo * ld + gx]) + (gval[y * ld + gx] - gval[y * ld + gy]) -
                                 2 * weight(xo, y);
                const int pair = xo < y ? xo * Go + y : y * Go + xo;
                key[j] = (double)gain * 65536.0 + (double)(65535 - pair);
            }
        }
        int n_swaps = 0, kbest = 0, moved = 1 << 30;
        long long run = 0, bestsum = 0;
        double dx = 0.0;
        float sx = 0.0f;
        for (;;) {
            double best = kPgNone;
            asm volatile("" : "+s"(Go));
#pragma unroll
            for (int j = 0; j < kSlots; ++j) {
                if (2 * (1 + kSub * j) > Go) break;  // uniform: no lane has this shift
                if (j % 4 == 0) __builtin_amdgcn_sched_barrier(0);
                const PgNode q = py[kSub * j];
                const PgSide z = ps[kSub * j];
                key[j] = __builtin_fma(dx - q.d, (double)(z.s - sx), key[j]);
                const bool ok = dm[j] * (float)(hx - q.h) <= 0.0f && z.grp != gx;
                const double k = ok ? key[j] : kPgNone;
                best = k > best ? k : best;
            }
            best = wave_max(best);
            if (Sh::kPer == 1) {
                if (lane == 0) red[threadIdx.x >> 6] = best;
                __syncthreads();
#pragma unroll
                for (int i = 0; i < kNT / 64; ++i) best = red[i] > best ? red[i] : best;
            }
            if (best == kPgNone) break;  // uniform: no admissible pair left
            const long long kk = (long long)best;
            const int pair = 65535 - (int)(kk & 65535);
            const int u = pair / G, v = pair - u * G;
            ++n_swaps;
            run += kk >> 16;
            if (run > bestsum) {
                bestsum = run;
                kbest = n_swaps;
            }
            const int A = side2[u].grp, B = side2[v].grp;
            const double dmem = memd[v] - memd[u];
            pg_sync<P>();  // every wavefront has read the two groups
            if (x < G) {
                dx = 65536.0 * (double)(weight(v, x) - weight(u, x));
                sx = gx == A ? 1.0f : (gx == B ? -1.0f : 0.0f);
                hx = hx + (double)sx * dmem;
                if (x == u || x == v) {
                    hx = __builtin_nan("");  // locked: no comparison with it holds
                    gx = x == u ? B : A;
                    moved = n_swaps;
                }
                if (sub == 0) {
                    node[x] = node[x + G] = PgNode{hx, dx};
                    side2[x] = side2[x + G] = PgSide{gx, sx};
                }
            }
            pg_sync<P>();
        }
        // the swaps past the best prefix are undone: a GPU moves at most once in a pass
        if (moved > kbest) gx = g0;
        if (sub == 0 && x < G) grp[x] = gx;
        pg_sync<P>();
        if (kbest == 0) break;  // uniform
    }
    // groups numbered by smallest member
    if (tid < kPgMaxK) first[tid] = 1 << 30;
    pg_sync<P>();
    if (sub == 0 && x < G) atomicMin(&first[gx], x);
    pg_sync<P>();
    if (tid < kPgMaxK) {
        int id = 0;
        for (int k = 0; k < kPgMaxK; ++k) id += first[k] < first[tid] ? 1 : 0;
        newid[tid] = id;
    }
    for (int e = tid; e < Kh * Kh; e += kNT) sw[e] = 0;
    int used = 0;
    for (int k = 0; k < kPgMaxK; ++k) used += first[k] < (1 << 30) ? 1 : 0;
    pg_sync<P>();
    if (x < G) {
        gx = newid[gx];
        if (sub == 0) grp[x] = gx;
    }
    pg_sync<P>();
    // step (ii): coarsened weights and the max-cut split
    if (x < G)
        for (int e = sub; e < G; e += kSub) {
            const int ge = grp[e];
            if (ge != gx) atomicAdd((unsigned long long*)&sw[gx * Kh + ge], (unsigned long long)weight(e, x));
        }
    if (tid < kPgMaxK) side[tid] = tid < used ? (int)((r >> (11 + tid)) & 1) : 0;
    pg_sync<P>();
    if (tid < 64) {  // one wavefront: a lane per super node
        uint64_t ones = __ballot(lane < used && side[lane & (kPgMaxK - 1)] != 0);
        if (ones == 0 || ones == ((1ull << used) - 1)) ones ^= 1ull << (used - 1);
        for (int step = 0; step < used * used; ++step) {
            const int n1 = __popcll(ones);
            const bool one = (ones >> lane) & 1;
            long long gain = 0;
            if (lane < used && !(one && n1 == 1) && !(!one && n1 == used - 1))
                for (int l = 0; l < used; ++l) {
                    const long long v = l == lane ? 0 : sw[lane * Kh + l];
                    gain += (((ones >> l) & 1) != 0) == one ? v : -v;
                }
            // largest gain, then lowest super node; gains are below 2^47 in all
            const double bk = wave_max(gain > 0 ? (double)(gain * 64 + (63 - lane)) : 0.0);
            if (!(bk > 0.0)) break;  // uniform
            ones ^= 1ull << (63 - (int)((long long)bk & 63));
        }
        for (int k = lane; k < a.Kmax; k += 64)
            a.role[(int64_t)k * N + n] =
                k < used ? (uint8_t)((ones >> k) & 1 ? HX_DECODE : HX_PREFILL) : (uint8_t)HX_UNUSED;
    }
    // step (iii): the projection
    if (sub == 0 && x < G) a.assign[(int64_t)x * N + n] = (uint8_t)gx;
}

// Candidate n of any graph, in 64-bit integers, by a workgroup (lane tid).
__device__ __forceinline__ void partition_one(const PgArgs& a, int G, int tid, int n) {
    extern __shared__ __attribute__((aligned(16))) unsigned char pg_sm[];
    long long* gval = reinterpret_cast<long long*>(pg_sm);  // [G][kPgMaxK]
    __shared__ long long memv[kPgBlock];
    __shared__ int grp[kPgBlock];
    __shared__ int locked[kPgBlock];
    __shared__ int su[kPgBlock / 2], sv[kPgBlock / 2];  // a pass's tentative swaps
    __shared__ long long gmem[kPgMaxK];
    __shared__ long long red[kPgBlock / 64];
    __shared__ int redp[kPgBlock / 64];
    __shared__ int first[kPgMaxK], newid[kPgMaxK], side[kPgMaxK];
    __shared__ long long sw[kPgMaxK * kPgMaxK];
    __shared__ long long cum[kPgBlock];
    const int64_t N = a.N;
    const uint64_t r = a.rnd[n];
    if (tid < G) {
        const int t = a.gpu_type[tid];
        memv[tid] = (t >= 0 && t < a.T) ? (long long)a.mem[t] : 0;
        grp[tid] = 0;
    }
    __syncthreads();
    // K: floor(total memory / replica memory), the replica holding the weights and the KV
    // caches of 32 requests (Appendix A), shifted by the draw
    long long total = 0;
    double mtot = 0.0;
    for (int e = 0; e < G; ++e) {
        total += memv[e];
        mtot = mtot + (double)memv[e];
    }
    const double Ld = (double)a.L;
    const double rep = 12.0 * a.H * a.H * a.B * Ld + 32.0 * (2.0 * (a.s_in + a.s_out) * a.Hkv * a.B * Ld);
    int kmax = a.Kmax < G ? a.Kmax : G;
    if (kmax > kPgMaxK) kmax = kPgMaxK;
    int K = (int)floor(mtot / rep) + (int)((r & 7) % 5) - 2;
    if (K > kmax) K = kmax;
    if (K < 2) K = 2;
    const int rot = (int)(((r >> 3) & 0xFF) % (uint64_t)G);
    if (total <= 0) total = 1;  // memories all zero: every GPU lands in group 0
    // step (i): the rotated spectral order cut by memory midpoints into K groups
    if (tid == 0) {
        long long run = 0;
        for (int i = 0; i < G; ++i) {
            const int dd = a.order[(i + rot) % G];
            const bool ok = dd >= 0 && dd < G;
            cum[i] = run;
            run += ok ? memv[dd] : 0;
        }
    }
    __syncthreads();
    if (tid < G) {
        const int dd = a.order[(tid + rot) % G];
        if (dd >= 0 && dd < G) {
            const long long k = ((long long)K * (2 * cum[tid] + memv[dd])) / (2 * total);
            grp[dd] = (int)(k < K - 1 ? k : K - 1);
        }
    }
    if (tid < kPgMaxK) gmem[tid] = 0;
    __syncthreads();
    if (tid < G) atomicAdd((unsigned long long*)&gmem[grp[tid]], (unsigned long long)memv[tid]);
    if (tid < G) {
        long long* row = gval + tid * kPgMaxK;
        for (int k = 0; k < kPgMaxK; ++k) row[k] = 0;
        for (int x = 0; x < G; ++x) row[grp[x]] += a.w[(int64_t)x * G + tid];
    }
    drain_barrier();
    // Kernighan-Lin passes: tentative best swaps on unlocked GPUs (negative gains too), then the
    // pass's best prefix is kept and the rest undone; passes repeat while one lowers the cut
    const int pairs = G * G;
    for (int pass = 0; pass < kKlPasses; ++pass) {
        if (tid < G) locked[tid] = 0;
        __syncthreads();
        int n_swaps = 0, kbest = 0;
        long long run = 0, bestsum = 0;
        for (;;) {
            long long bg = 0;
            int bp = kNoPair;
            for (int p = tid; p < pairs; p += kPgBlock) {
                const int u = p / G, v = p - u * G;
                if (v <= u || locked[u] || locked[v]) continue;
                const int A = grp[u], B = grp[v];
                if (A == B) continue;
                const long long d0 = gmem[A] - gmem[B];
                const long long d1 = (gmem[A] - memv[u] + memv[v]) - (gmem[B] - memv[v] + memv[u]);
                if ((d1 < 0 ? -d1 : d1) > (d0 < 0 ? -d0 : d0)) continue;
                const long long wuv = a.w[(int64_t)u * G + v];
                const long long gain = (gval[u * kPgMaxK + B] - gval[u * kPgMaxK + A] - wuv) +
                                       (gval[v * kPgMaxK + A] - gval[v * kPgMaxK + B] - wuv);
                if (better(gain, p, bg, bp)) {
                    bg = gain;
                    bp = p;
                }
            }
            block_best(bg, bp, red, redp);
            if (bp == kNoPair) break;  // uniform: no admissible pair left
            const int u = bp / G, v = bp - u * G;
            pg_exchange(a, u, v, grp, gval, gmem, memv);
            if (tid == 0) {
                locked[u] = locked[v] = 1;
                su[n_swaps] = u;
                sv[n_swaps] = v;
            }
            __syncthreads();
            ++n_swaps;
            run += bg;
            if (run > bestsum) {
                bestsum = run;
                kbest = n_swaps;
            }
        }
        // undo the swaps past the best prefix, last first
        for (int i = n_swaps - 1; i >= kbest; --i) pg_exchange(a, su[i], sv[i], grp, gval, gmem, memv);
        if (kbest == 0) break;  // uniform
    }
    // groups numbered by smallest member
    if (tid < kPgMaxK) first[tid] = 1 << 30;
    __syncthreads();
    if (tid < G) atomicMin(&first[grp[tid]], tid);
    drain_barrier();
    if (tid < kPgMaxK) {
        int id = 0;
        for (int k = 0; k < kPgMaxK; ++k) id += first[k] < first[tid] ? 1 : 0;
        newid[tid] = id;
    }
    __syncthreads();
    int used = 0;
    for (int k = 0; k < kPgMaxK; ++k) used += first[k] < (1 << 30) ? 1 : 0;
    if (tid < G) grp[tid] = newid[grp[tid]];
    for (int i = tid; i < kPgMaxK * kPgMaxK; i += kPgBlock) sw[i] = 0;
    __syncthreads();
    // step (ii): coarsened weights and the max-cut split
    for (int p = tid; p < pairs; p += kPgBlock) {
        const int dd = p / G, e = p - dd * G;
        const int gd = grp[dd], ge = grp[e];
        if (gd != ge) atomicAdd((unsigned long long*)&sw[gd * kPgMaxK + ge], (unsigned long long)a.w[p]);
    }
    if (tid < kPgMaxK) side[tid] = tid < used ? (int)((r >> (11 + tid)) & 1) : 0;
    drain_barrier();
    int n1 = 0;
    for (int k = 0; k < used; ++k) n1 += side[k];
    __syncthreads();
    if (n1 == 0 || n1 == used) {
        if (tid == 0) side[used - 1] ^= 1;
        n1 += (n1 == 0) ? 1 : -1;
    }
    __syncthreads();
    for (int step = 0; step < used * used; ++step) {
        long long bg = 0;
        int bk = kNoPair;
        if (tid < used) {
            const bool blocked = (side[tid] && n1 == 1) || (!side[tid] && n1 == used - 1);
            if (!blocked) {
                long long gain = 0;
                for (int l = 0; l < used; ++l) {
                    if (l == tid) continue;
                    const long long s = sw[tid * kPgMaxK + l];
                    gain += side[l] == side[tid] ? s : -s;
                }
                if (gain > 0) {  // largest gain, then lowest super node
                    bg = gain;
                    bk = tid;
                }
            }
        }
        block_best(bg, bk, red, redp);
        if (bk == kNoPair) break;  // uniform
        const int k = bk;
        n1 += side[k] ? -1 : 1;
        __syncthreads();
        if (tid == 0) side[k] ^= 1;
        __syncthreads();
    }
    // step (iii): the projection
    if (tid < G) a.assign[(int64_t)tid * N + n] = (uint8_t)grp[tid];
    for (int k = tid; k < a.Kmax; k += kPgBlock)
        a.role[(int64_t)k * N + n] = k < used ? (uint8_t)(side[k] ? HX_DECODE : HX_PREFILL) : (uint8_t)HX_UNUSED;
}

// The candidates that partition_gain_kernel left marked (all or none), a workgroup every gridDim.x-th one.
// kPgGrid workgroups are several times what the chip holds at once (24 KB of LDS each at 32 GPUs), so that
// those that end early are replaced, and few enough to cost a call with none marked 3 us at most (a
// workgroup per candidate: 20 us at 8 GPUs x 100,000).  G and the lane are hidden from the compiler, which
// would otherwise keep what it derives from them in registers across candidates (93 instead of 72).
// Calls past the ranges with this kernel alone, a workgroup per candidate / with 512 workgroups / now:
// 16 GPUs x 16,384 406 / 1,058 / 432 us (18 of them the gain kernel's), 32 x 16,384 1,770 / 4,409 / 1,784,
// 64 x 2,048 2,250 / 3,740 / 2,200, 100 x 1,000 7.2 / 8.8 / 7.2 ms, 255 x 600 117 / 153 / 118 ms; with
// 4,096 workgroups 489 us and 2,020 us at the first two.
constexpr int kPgGrid = 16384;
__global__ void __launch_bounds__(kPgBlock) partition_kernel(PgArgs a) {
    for (int64_t n = blockIdx.x; n < a.N; n += gridDim.x) {
        if (a.assign[n] != HX_UNUSED) return;  // uniform
        int G = a.G, tid = threadIdx.x;
        asm volatile("" : "+s"(G), "+v"(tid));
        partition_one(a, G, tid, (int)n);
        __syncthreads();  // the next candidate reuses the LDS
    }
}

}  // namespace

hipError_t launch_spectral(int32_t G, const double* beta, int64_t* w, int32_t iters, int32_t* order, double* fiedler,
                           hipStream_t s) {
    const int64_t cells = (int64_t)G * G;
    hipLaunchKernelGGL(graph_kernel, dim3((unsigned)((cells + 255) / 256)), dim3(256), 0, s, G, beta, w);
    prof_mark(kKSpectral, false, s);
    const int b = (G + 15) / 16;
    launch_spectral_b<1>(b <= 8 ? b : 16, G, w, iters, order, fiedler, s);
    prof_mark(kKSpectral, true, s);
    return hipGetLastError();
}

template <int P, bool kLdsW>
static hipError_t launch_gain(const PgArgs& a, int Kh, hipStream_t s) {
    using Sh = PgShape<P>;
    const size_t lds = (kLdsW ? (sizeof(int32_t) * (size_t)a.G * a.G + 15) & ~(size_t)15 : 0) +
                       Sh::kPer * pg_fast_lds(a.G, Kh);
    if (lds > 32 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&partition_gain_kernel<P, kLdsW>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    const int64_t wgs = ((int64_t)a.N + Sh::kPer - 1) / Sh::kPer;
    const dim3 grid((unsigned)(wgs < kPgGridX ? wgs : kPgGridX), (unsigned)((wgs + kPgGridX - 1) / kPgGridX));
    hipLaunchKernelGGL((partition_gain_kernel<P, kLdsW>), grid, dim3(Sh::kBlock), lds, s, a, Kh);
    return hipGetLastError();
}

hipError_t launch_partition(const Problem& p, int64_t* w, const int32_t* order, const uint64_t* rnd, uint8_t* assign,
                            uint8_t* role, hipStream_t s) {
    const int64_t cells = (int64_t)p.G * p.G;
    hipLaunchKernelGGL(graph_kernel, dim3((unsigned)((cells + 255) / 256)), dim3(256), 0, s, p.G, p.beta, w);
    PgArgs a{p.G, p.Kmax, p.N, p.L, p.H, p.Hkv, p.B, p.s_in, p.s_out, w, order, p.gpu_type, p.mem, p.T, rnd,
             assign, role};
    int Kh = p.Kmax < p.G ? p.Kmax : p.G;
    if (Kh > kPgMaxK) Kh = kPgMaxK;
    if (Kh < 2) Kh = 2;
    prof_mark(kKPartition, false, s);
    hipError_t e;
    if (p.G <= 32) e = launch_gain<32, true>(a, Kh, s);
    else if (p.G <= 64) e = launch_gain<64, true>(a, Kh, s);
    // above 104 GPUs the staged weights would leave a CU one workgroup (more than 80 KB of LDS)
    else if (p.G <= 104) e = launch_gain<128, true>(a, Kh, s);
    else if (p.G <= 128) e = launch_gain<128, false>(a, Kh, s);
    else e = launch_gain<256, false>(a, Kh, s);
    if (e != hipSuccess) return e;
    // gval of 255 GPUs (65,280 bytes) takes the workgroup past 64 KB of LDS, which gfx950 allows
    // (160 KB per workgroup) once the kernel's dynamic limit is raised
    const size_t lds = pg_lds_bytes(p.G);
    if (lds > 32 * 1024) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(partition_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(partition_kernel, dim3((unsigned)(p.N < kPgGrid ? p.N : kPgGrid)), dim3(kPgBlock), lds, s, a);
    prof_mark(kKPartition, true, s);
    return hipGetLastError();
}

}  // namespace hx
