// Gradients of stages a3 and a4 for a fixed index set I_sparse (Eq. 7, Eq. 8, Eq. 12;
// retraining a prob-sparse model from a trained dense one, Sec. 4.2).  The selection is
// a hard choice, so nothing flows through stages a1 and a2.  Per head, with G the
// upstream gradient of `out`, p_ij the softmax weights of the kept queries and
// scale = 1/sqrt(d):
//   c_ij = G_i . v_j           D_i = sum_j p_ij c_ij          g_ij = scale * p_ij (c_ij - D_i)
//   dQ_i = sum_j g_ij k_j      dK_j = sum_i g_ij q_i          dV_j = sum_i p_ij G_i   (+ the fill's share)
// The weights are recomputed from Q and K (the forward keeps no statistics):
//   bwd_stats_kernel   partial (max, sum, weighted sum of c) per kept query and key split
// and then one of two forms (make_bwd_plan): fused,
//   bwd_main_kernel    combines them, then dK, dV, the fill's gradient, zero rows, and dQ (per key split)
//   bwd_dq_reduce_kernel  adds the key splits of dQ in split order
// or, where those partial sums of dQ would take too much memory,
//   bwd_dq_kernel      combines them, then dQ of 16 kept queries over all keys
//   bwd_main_kernel    (kKeysOnly) dK, dV, the fill's gradient, zero rows
// All five contractions run on the matrix cores (v_mfma_f64_16x16x4f64 on exactly widened inputs):
//   lane (c, g) = (lane % 16, lane / 16)
//   A[i][k]: i = c, k = g      B[k][j]: k = g, j = c      D[i][j]: i = 4r + g, j = c  (r = 0..3)
// These are the kernels of float32 tensors, whose gradients are computed in float64 (bfloat16 tensors: psa_backward_bf16.hip,
// and the plan below bounds the scratch of both).  Every sum has a fixed order, so results do not depend on scheduling.
//
// What bounds it: the matrix pipe.  A float64 MFMA takes 65 cycles of its SIMD, and the SIMD issues no vector
// instruction meanwhile (micro-benchmark: the times of both add up, whatever waves they come from), so a vector
// instruction costs its own 3 to 5 cycles on top.  The kernels therefore
//   * form the scores s and c twice, not three times: one kernel computes dQ with dK and dV, so a tile of 16
//     queries x 16 keys costs 32 (statistics) + 80 MFMAs; recomputing them once more for dQ alone made it 144;
//   * widen every operand once: a wave keeps the 16 key rows it owns as float64 in registers and finds the
//     group's query rows as float64 in LDS, where the work-group has put them once;
//   * run two work-groups of 4 waves (one per SIMD) on a CU, so that one fills the matrix pipe while the other
//     stages rows, waits at a barrier or stores (or, for full batches, one of 8 waves, which has half the partial sums of
//     dQ), and cut the key axis so that their number fills whole rounds of the CUs;
//   * keep a head's work-groups on one XCD where the heads divide evenly: each L2 fetches the rows of its own heads, not
//     the kept rows of Q and G of all (the first product of a work-group waits for 11 us, not for 14.5).
// Measured (whole call): B=16 H=4 L=512, 256 kept queries 225 -> 147 us, the last point 4 and the 8 waves 15 of them; B=8 H=8 L=300, 120 kept
// 102.2 -> 97.5 by the last point, B=24 H=8 L=200, 100 kept 133.2 -> 129.2 us.
#include <type_traits>

#include "psa_backward_common.h"

namespace psa {

constexpr int kBwdThreads = 256;     // 4 waves, one per SIMD; two work-groups share a CU
constexpr int kBwdWaves = kBwdThreads / 64;
constexpr int kBwdKeys = 64;         // keys per block of the statistics kernel: 16 per wave
constexpr int kBwdQ = 16;            // kept queries per tile
// LDS row strides, chosen so that every access pattern below spreads evenly over the 64 banks
constexpr int kBwdQRow = kD + 2;             // doubles between staged query rows
constexpr int kBwdKRow = kD + 4;             // floats between staged key rows
constexpr int kBwdStatGroup = 64;    // kept queries staged in LDS at a time by the statistics kernel (4 tiles) ...
constexpr int kBwdStatTiles = kBwdStatGroup / kBwdQ;
constexpr int kBwdStatsLds = 2 * kBwdStatGroup * kBwdQRow * 8;                   // 67584
constexpr int kBwdGroup = 32;        // ... and by the gradient kernel (2 tiles)
constexpr int kBwdTiles = kBwdGroup / kBwdQ;
constexpr int kBwdChunk = 2048;      // rows per bit mask of the fill's column sums
constexpr int kBwdMaxSplit = 64;     // key splits (their partial results are added up by one thread each)
constexpr size_t kBwdPartBytes = (size_t)256 << 20;   // partial sums of dQ that a call may always have (see make_bwd_plan)
constexpr int kBwdKeepStats = 768;   // most kept queries whose statistics the gradient kernel keeps in LDS (two work-groups per CU)
typedef double bwd_x4 __attribute__((ext_vector_type(4)));
typedef double bwd_x2 __attribute__((ext_vector_type(2)));

// How the 4 (KS = 8: 8) waves of the gradient kernel's work-group share its keys and the two tiles of a group: KS waves of 16
// keys each; with KS = 2 two waves have the same keys and one query tile each.
template <int KS> struct BwdShare {
    static constexpr int kWaves = KS > kBwdWaves ? KS : kBwdWaves;       // 8 (KS = 8), else 4
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int kSlots = kWaves / KS;                           // 1, 2
    static constexpr int kKeys = 16 * KS;                                // keys per block: 128, 64, 32
    static constexpr int kPerSlot = kBwdTiles / kSlots;                  // tiles a wave takes of a group: 2, 1
    static constexpr int kGRow = kKeys + 2;                              // doubles between the rows (queries) of a g tile
    static constexpr int kFixed = 2 * kBwdGroup * kBwdQRow * 8 + kBwdGroup * kGRow * 8 + kKeys * kBwdKRow * 4;   // 101888, 68096, 51200
    static constexpr int kLds = kFixed + kBwdKeepStats * 16;             // the most: u_pad statistics of 16 bytes
};

// N contiguous elements (N = 4, 8 or 16) as they lie in memory, widened where they are used (so that a request
// stays a request until then), and a 4-element store
template <int N> struct BwdRow {
    float4 x[N / 4];
    __device__ __forceinline__ void load(const float* p) {
#pragma unroll
        for (int k = 0; k < N / 4; ++k) x[k] = reinterpret_cast<const float4*>(p)[k];
    }
    __device__ __forceinline__ float at(int e) const {
        const float4 v = x[e >> 2];
        return (e & 3) == 0 ? v.x : (e & 3) == 1 ? v.y : (e & 3) == 2 ? v.z : v.w;
    }
};
__device__ __forceinline__ void bwd_store4(float* p, const float (&v)[4]) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}

// 16 bytes of a row: the values, or zeros
__device__ __forceinline__ void bwd_store16(float* p, const float (&v)[4], bool keep) {
    *reinterpret_cast<float4*>(p) = keep ? make_float4(v[0], v[1], v[2], v[3]) : make_float4(0.f, 0.f, 0.f, 0.f);
}

constexpr double kBwdScaleLog2e = 0.125 * 1.4426950408889634074;     // scores to base-2 exponents

// What bwd_main_kernel does beside dK and dV:
//   kFused      dQ as well; the statistics of all kept queries (up to kBwdKeepStats) are put together in LDS once
//   kFusedOne   the same with one block a split (KS = 8)
//   kFusedMany  the same with more kept queries: the statistics of a group are put together anew for every block
//   kKeysOnly   nothing: bwd_dq_kernel has computed dQ and left the statistics in memory
enum BwdForm { kFused, kFusedMany, kKeysOnly, kFusedOne };

struct BwdParams {
    const void* Q; const void* K; const void* V; const void* G;
    const int* lengths; const int* sel; const int* u;
    void* dQ; void* dK; void* dV;
    double* stats_part;    // [BH][S1][u_pad][3]  (max, sum, weighted c) per kept query and key split, base 2
    double* gsum_part;     // [BH][S1][64]        column sums of G over the valid rows outside I_sparse, per key split
    double* dq_part;       // [BH][S2][u_pad][64], or nullptr: dQ rows are written directly (KS = 8: two slots a split, below)
    double* stats;         // [BH][u_pad][2]       (log2 sum exp, -D/8) per kept query, kKeysOnly form; else nullptr
    int H, L, u_stride, u_pad, n_group, S1, blocks1, S2, blocks2, fill;
    int head_shift;        // 3: eight heads on the fastest axis of the grid, so that a head's work-groups share one XCD's L2; else 0
};
__device__ __forceinline__ int bwd_head(const BwdParams& P, int y) { return (y << P.head_shift) + (int)(blockIdx.x & ((1u << P.head_shift) - 1u)); }
__device__ __forceinline__ int bwd_index(const BwdParams& P) { return (int)(blockIdx.x >> P.head_shift); }

// Kept queries q0 .. q0 + ROWS - 1 of the head: their rows of Q and of G as float64 in LDS (zeros for an absent
// entry), 8 or 16 threads per row.  `find` looks the rows up in the list, `request` asks for them, `put` writes them to
// LDS (the caller's barrier makes them visible); a caller may have other work between the three.
template <int ROWS, int NT>
struct QueryStage {
    static constexpr int kPer = NT > ROWS * 8 ? 16 : 8;      // threads per row
    static constexpr int kPasses = ROWS * kPer / NT, kElems = kD / kPer;
    static_assert(kPasses * NT == ROWS * kPer, "whole passes");
    int qi[kPasses];                          // list entries as they lie in memory, rows (or -1) from `request` on
    BwdRow<kElems> a[kPasses], b[kPasses];
    static __device__ __forceinline__ int row_of(int k) { return k * (NT / kPer) + (int)threadIdx.x / kPer; }
    __device__ __forceinline__ void find(const BwdParams& P, int head, int q0) {
#pragma unroll
        for (int k = 0; k < kPasses; ++k) {
            const int t = q0 + row_of(k);
            qi[k] = P.sel[(size_t)head * P.u_stride + (t < P.u_stride ? t : P.u_stride - 1)];
        }
    }
    __device__ __forceinline__ void request(const float* Qh, const float* Gh, int q0, int n, int ub) {
        const int part = threadIdx.x % kPer;
#pragma unroll
        for (int k = 0; k < kPasses; ++k) {
            if (q0 + row_of(k) >= ub || qi[k] < 0 || qi[k] >= n) qi[k] = -1;
            a[k].load(Qh + (size_t)(qi[k] >= 0 ? qi[k] : 0) * kD + kElems * part);
            b[k].load(Gh + (size_t)(qi[k] >= 0 ? qi[k] : 0) * kD + kElems * part);
        }
    }
    __device__ __forceinline__ void put(double* sQ, double* sG) const {
        const int part = threadIdx.x % kPer;
#pragma unroll
        for (int k = 0; k < kPasses; ++k) {
            bwd_x2* dq = reinterpret_cast<bwd_x2*>(sQ + row_of(k) * kBwdQRow + kElems * part);
            bwd_x2* dg = reinterpret_cast<bwd_x2*>(sG + row_of(k) * kBwdQRow + kElems * part);
#pragma unroll
            for (int e = 0; e < kElems / 2; ++e) {
                dq[e] = qi[k] >= 0 ? bwd_x2{(double)a[k].at(2 * e), (double)a[k].at(2 * e + 1)} : bwd_x2{0.0, 0.0};
                dg[e] = qi[k] >= 0 ? bwd_x2{(double)b[k].at(2 * e), (double)b[k].at(2 * e + 1)} : bwd_x2{0.0, 0.0};
            }
        }
    }
};

// Widens a wave's key rows into registers, once: the compiler would rather repeat the conversion at every use.
__device__ __forceinline__ void widen16(const BwdRow<16>& x, double (&d)[16])
{
#pragma unroll
    for (int t = 0; t < 16; ++t) { d[t] = (double)x.at(t); asm volatile("" : "+v"(d[t])); }
}

// The two score products of a tile's 16 staged queries against the wave's 16 keys, two independent MFMA chains.
// Lane group g takes elements 16 g .. 16 g + 15 of its row on both sides (the contraction order is free).
// QUERY_ROWS: queries on the rows of the result (lane: queries 4r + g against key c), else keys on the rows.
// The staged operands of 4 elements are read while the products of the 4 before them run.
template <bool QUERY_ROWS>
__device__ __forceinline__ void score_products(const double* sQ, const double* sG, int tile, int c, int g,
                                               const double (&kd)[16], const double (&vd)[16], bwd_x4& s, bwd_x4& cc)
{
    s = bwd_x4{0.0, 0.0, 0.0, 0.0};
    cc = bwd_x4{0.0, 0.0, 0.0, 0.0};
    const bwd_x2* qr = reinterpret_cast<const bwd_x2*>(sQ + (16 * tile + c) * kBwdQRow + 16 * g);
    const bwd_x2* gr = reinterpret_cast<const bwd_x2*>(sG + (16 * tile + c) * kBwdQRow + 16 * g);
    bwd_x2 q2[2][2], g2[2][2];
    q2[0][0] = qr[0]; q2[0][1] = qr[1]; g2[0][0] = gr[0]; g2[0][1] = gr[1];
#pragma unroll
    for (int st = 0; st < 4; ++st) {
        const int cur = st & 1;
        if (st < 3) {
            q2[cur ^ 1][0] = qr[2 * st + 2]; q2[cur ^ 1][1] = qr[2 * st + 3];
            g2[cur ^ 1][0] = gr[2 * st + 2]; g2[cur ^ 1][1] = gr[2 * st + 3];
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double qv = q2[cur][e >> 1][e & 1], gv = g2[cur][e >> 1][e & 1];
            if (QUERY_ROWS) {
                s = __builtin_amdgcn_mfma_f64_16x16x4f64(qv, kd[4 * st + e], s, 0, 0, 0);
                cc = __builtin_amdgcn_mfma_f64_16x16x4f64(gv, vd[4 * st + e], cc, 0, 0, 0);
            } else {
                s = __builtin_amdgcn_mfma_f64_16x16x4f64(kd[4 * st + e], qv, s, 0, 0, 0);
                cc = __builtin_amdgcn_mfma_f64_16x16x4f64(vd[4 * st + e], gv, cc, 0, 0, 0);
            }
        }
    }
}

__device__ __forceinline__ int opaque(int x) { asm volatile("" : "+v"(x)); return x; }

// a maximum over no key: far below any score, and finite, so that differences of such values stay numbers
constexpr double kBwdNoMax = -1e300;

// ---- partial softmax statistics per kept query and key split; column sums of G over the rows the mean fill serves.
// grid (key splits, groups of 64 kept queries, heads), eight heads (or one) on the first axis
__global__ __launch_bounds__(kBwdThreads, 2)
void bwd_stats_kernel(const BwdParams P)
{
    extern __shared__ __attribute__((aligned(16))) double bwd_smem[];
    __shared__ unsigned s_bits[kBwdChunk / 32];
    double* sQ = bwd_smem;
    double* sG = bwd_smem + kBwdStatGroup * kBwdQRow;
    const int split = bwd_index(P), group = blockIdx.y, head = bwd_head(P, blockIdx.z);
    const int b = head / P.H, L = P.L;
    const int n = valid_len(P.lengths, b, L);
    const int ub = kept_count(P, b, n);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = lane & 15, g = lane >> 4;
    const float* Qh = static_cast<const float*>(P.Q) + (size_t)head * L * kD;
    const float* Kh = static_cast<const float*>(P.K) + (size_t)head * L * kD;
    const float* Vh = static_cast<const float*>(P.V) + (size_t)head * L * kD;
    const float* Gh = static_cast<const float*>(P.G) + (size_t)head * L * kD;
    const int k_first = split * P.blocks1 * kBwdKeys;
    int k_end = k_first + P.blocks1 * kBwdKeys;
    k_end = k_end < n ? k_end : n;
    const bool sums = group == 0 && P.fill == PSA_FILL_MEAN;         // work-group-uniform: this one sums G
    const int q0 = group * kBwdStatGroup;
    int n_t = (ub - q0 + kBwdQ - 1) / kBwdQ;                         // tiles of kept queries: 0 .. 4
    n_t = n_t < 0 ? 0 : (n_t < kBwdStatTiles ? n_t : kBwdStatTiles);
    if (n_t == 0 && !sums) return;

    // the wave's 16 key rows (lane: 16 elements of row c) and, for the column sums, the same 16 rows of G (lane:
    // elements 4c .. 4c + 3 of rows 4 i + g); the next block's are requested before the current one is worked on
    // (on a clamped row: harmless past the end)
    BwdRow<16> kn, vn;
    BwdRow<4> gn[4];
    auto request = [&](int j0) {
        if (n_t > 0) {
            const int row = j0 + c < n ? j0 + c : n - 1;
            kn.load(Kh + (size_t)row * kD + 16 * g);
            vn.load(Vh + (size_t)row * kD + 16 * g);
        }
        if (sums) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = j0 + 4 * i + g < n ? j0 + 4 * i + g : n - 1;
                gn[i].load(Gh + (size_t)row * kD + 4 * c);
            }
        }
    };
    if (k_first < k_end) request(k_first + 16 * wave);               // (n > 0)
    if (n_t > 0) {
        QueryStage<kBwdStatGroup, kBwdThreads> qs;
        qs.find(P, head, q0);
        qs.request(Qh, Gh, q0, n, ub);
        qs.put(sQ, sG);
    }
    __syncthreads();

    // this lane: query c of every tile, keys 4r + g of the wave's 16
    double m[kBwdStatTiles], l[kBwdStatTiles], dacc[kBwdStatTiles], tot[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int tt = 0; tt < kBwdStatTiles; ++tt) { m[tt] = kBwdNoMax; l[tt] = 0.0; dacc[tt] = 0.0; }
#pragma unroll 1
    for (int blk0 = k_first; blk0 < k_end; blk0 += kBwdKeys) {       // work-group-uniform
        const int j0 = blk0 + 16 * wave;
        if (sums && (blk0 - k_first) % kBwdChunk == 0) {
            // mark the kept rows of the next 2048: they take no part in the column sums
            __syncthreads();
            if (tid < kBwdChunk / 32) s_bits[tid] = 0u;
            __syncthreads();
            for (int t = tid; t < ub; t += kBwdThreads) {
                const int i = P.sel[(size_t)head * P.u_stride + t] - blk0;
                if (i >= 0 && i < kBwdChunk) atomicOr(&s_bits[i >> 5], 1u << (i & 31));
            }
            __syncthreads();
        }
        if (j0 >= k_end) continue;                                   // wave-uniform
        double kd[16], vd[16];
        if (n_t > 0) { widen16(kn, kd); widen16(vn, vd); }
        if (sums) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int rr = (j0 - k_first) % kBwdChunk + 4 * i + g;
                const bool use = j0 + 4 * i + g < k_end && !((s_bits[rr >> 5] >> (rr & 31)) & 1u);
#pragma unroll
                for (int e = 0; e < 4; ++e) tot[e] += (double)(use ? gn[i].at(e) : 0.f);
            }
        }
        if (j0 + kBwdKeys < k_end) request(j0 + kBwdKeys);
#pragma unroll
        for (int tt = 0; tt < kBwdStatTiles; ++tt) {
            if (tt < n_t) {                                          // work-group-uniform
                bwd_x4 s, cc;
                score_products<false>(sQ, sG, tt, c, g, kd, vd, s, cc);
                double sc[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) sc[r] = s[r] * kBwdScaleLog2e;
                if (j0 + 16 > k_end) {                               // wave-uniform: the last keys
#pragma unroll
                    for (int r = 0; r < 4; ++r) sc[r] = j0 + 4 * r + g < k_end ? sc[r] : -INFINITY;
                }
                const double mn = fmax(fmax(fmax(sc[0], sc[1]), fmax(sc[2], sc[3])), m[tt]);
                const double a = exp2_f64(m[tt] - mn);               // (0 for the first key)
                double w[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) w[r] = exp2_f64(sc[r] - mn);
                l[tt] = fma(l[tt], a, (w[0] + w[1]) + (w[2] + w[3]));
                dacc[tt] *= a;
#pragma unroll
                for (int r = 0; r < 4; ++r) dacc[tt] = fma(w[r], cc[r], dacc[tt]);
                m[tt] = mn;
            }
        }
    }
    __syncthreads();                                                 // the query rows have been read
    if (sums) {
        double (*s_gs)[kD] = reinterpret_cast<double (*)[kD]>(bwd_smem + kBwdWaves * kBwdStatGroup * 3);     // [4 * waves][64], behind s_part
#pragma unroll
        for (int e = 0; e < 4; ++e) s_gs[wave * 4 + g][4 * c + e] = tot[e];
        __syncthreads();
        if (tid < kD) {
            double t = 0.0;
#pragma unroll
            for (int k = 0; k < 4 * kBwdWaves; ++k) t += s_gs[k][tid];   // fixed order
            P.gsum_part[((size_t)head * P.S1 + split) * kD + tid] = t;
        }
    }
    if (n_t == 0) return;
    // fold the four lane groups (the same query, different keys), then the waves, in fixed order
    double (*s_part)[kBwdStatGroup][3] = reinterpret_cast<double (*)[kBwdStatGroup][3]>(bwd_smem);    // [wave][query][m, l, d]
#pragma unroll
    for (int tt = 0; tt < kBwdStatTiles; ++tt) {
        double mw = fmax(m[tt], __shfl_xor(m[tt], 16, 64));
        mw = fmax(mw, __shfl_xor(mw, 32, 64));
        const double a = exp2_f64(m[tt] - mw);
        double lw = l[tt] * a, dw = dacc[tt] * a;
        lw += __shfl_xor(lw, 16, 64); dw += __shfl_xor(dw, 16, 64);
        lw += __shfl_xor(lw, 32, 64); dw += __shfl_xor(dw, 32, 64);
        if (g == 0) { s_part[wave][16 * tt + c][0] = mw; s_part[wave][16 * tt + c][1] = lw; s_part[wave][16 * tt + c][2] = dw; }
    }
    __syncthreads();
    if (tid < n_t * kBwdQ) {                                         // (at most 64)
        double mx = kBwdNoMax;
#pragma unroll
        for (int w = 0; w < kBwdWaves; ++w) mx = fmax(mx, s_part[w][tid][0]);
        double lt = 0.0, dt = 0.0;
#pragma unroll
        for (int w = 0; w < kBwdWaves; ++w) {
            const double a = exp2_f64(s_part[w][tid][0] - mx);
            lt = fma(a, s_part[w][tid][1], lt); dt = fma(a, s_part[w][tid][2], dt);
        }
        double* sp = P.stats_part + (((size_t)head * P.S1 + split) * P.u_pad + q0 + tid) * 3;
        sp[0] = mx; sp[1] = lt; sp[2] = dt;
    }
}

// the key splits' statistics of kept query t together: log2 of the sum of exponentials, and D
__device__ __forceinline__ void combine_stats(const BwdParams& P, int head, int t, double& lse, double& D)
{
    const double* sp = P.stats_part + ((size_t)head * P.S1 * P.u_pad + t) * 3;
    const size_t step = (size_t)P.u_pad * 3;
    double mx = kBwdNoMax, lt = 0.0, dt = 0.0;
    for (int s0 = 0; s0 < P.S1; s0 += 4) {                           // split order, 4 in flight
        double ms[4], ls[4], ds[4], mn = mx;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double* q = sp + (size_t)(s0 + k < P.S1 ? s0 + k : P.S1 - 1) * step;
            ms[k] = q[0]; ls[k] = q[1]; ds[k] = q[2];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) mn = fmax(mn, ms[k]);
        const double a0 = exp2_f64(mx - mn);
        lt *= a0; dt *= a0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double a = s0 + k < P.S1 ? exp2_f64(ms[k] - mn) : 0.0;
            lt = fma(a, ls[k], lt); dt = fma(a, ds[k], dt);
        }
        mx = mn;
    }
    lse = mx + log2(lt);                                             // (lt > 0: a kept query has at least one valid key)
    D = dt / lt;
}

// (log2 sum exp, -D/8) of kept query t of the head; an absent entry of the list has no weight on any key
__device__ __forceinline__ bwd_x2 stat_of(const BwdParams& P, int head, int t, int n, int ub)
{
    double lse = INFINITY, D = 0.0;
    if (kept_row(P, head, t, n, ub) >= 0) combine_stats(P, head, t, lse, D);
    return bwd_x2{lse, -0.125 * D};
}

// ---- dQ of a tile of 16 kept queries over all keys of the head, and their statistics for the kKeysOnly form of
// bwd_main_kernel.  Scores are formed transposed (keys on the rows), so that a lane's four g values belong to query c
// and are, unchanged, the B operand of the product that contracts over keys.  Wave w takes the 16 keys 16 w .. + 15 of
// every 64; the waves' shares of dQ are added in wave order at the end, so nothing goes through memory.  The price is
// the two score products, formed a third time (48 MFMAs for a tile of 16 queries x 16 keys instead of 16).
// grid (tiles of 16 kept queries, heads), heads as above
__global__ __launch_bounds__(kBwdThreads, 2)
void bwd_dq_kernel(const BwdParams P)
{
    __shared__ bwd_x2 s_stat[kBwdQ];
    __shared__ double s_acc[kBwdWaves][16][64];                      // the waves' accumulators, register by register
    const int q0 = bwd_index(P) * kBwdQ, head = bwd_head(P, blockIdx.y);
    const int b = head / P.H, L = P.L;
    const int n = valid_len(P.lengths, b, L);
    const int ub = kept_count(P, b, n);
    if (q0 >= ub) return;                                            // work-group-uniform (n > 0 behind this)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = lane & 15, g = lane >> 4;
    const float* Qh = static_cast<const float*>(P.Q) + (size_t)head * L * kD;
    const float* Kh = static_cast<const float*>(P.K) + (size_t)head * L * kD;
    const float* Vh = static_cast<const float*>(P.V) + (size_t)head * L * kD;
    const float* Gh = static_cast<const float*>(P.G) + (size_t)head * L * kD;

    // operands of 16 keys: the lane's key row for the score products (16 elements of key c), and for the product that
    // contracts over keys elements 4c .. 4c + 3 of keys 4r + g; the next keys' are requested before these are worked
    // on (on a clamped row: harmless past the end)
    BwdRow<16> kn, vn;
    BwdRow<4> k4n[4];
    auto request = [&](int j0) {
        const int row = j0 + c < n ? j0 + c : n - 1;
        kn.load(Kh + (size_t)row * kD + 16 * g);
        vn.load(Vh + (size_t)row * kD + 16 * g);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int key = j0 + 4 * r + g < n ? j0 + 4 * r + g : n - 1;
            k4n[r].load(Kh + (size_t)key * kD + 4 * c);
        }
    };
    request(16 * wave);
    const int qi = kept_row(P, head, q0 + c, n, ub);
    double qd[16], gd[16];                                           // B operands of the score products: query c (zeros for an absent entry)
    {
        BwdRow<16> qf, gf;
        qf.load(Qh + (size_t)(qi >= 0 ? qi : 0) * kD + 16 * g);
        gf.load(Gh + (size_t)(qi >= 0 ? qi : 0) * kD + 16 * g);
#pragma unroll
        for (int t = 0; t < 16; ++t) { qd[t] = qi >= 0 ? (double)qf.at(t) : 0.0; gd[t] = qi >= 0 ? (double)gf.at(t) : 0.0; }
    }
    if (tid < kBwdQ) {
        const bwd_x2 sd = stat_of(P, head, q0 + tid, n, ub);
        s_stat[tid] = sd;
        reinterpret_cast<bwd_x2*>(P.stats)[(size_t)head * P.u_pad + q0 + tid] = sd;
    }
    __syncthreads();
    const bwd_x2 sd = s_stat[c];
    bwd_x4 acc[4];                                                   // dQ^T of this wave's keys: acc[dt][r] is element 4 (4r + g) + dt of query c
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) acc[dt] = bwd_x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int j0 = 16 * wave; j0 < n; j0 += 16 * kBwdWaves) {         // wave-uniform
        BwdRow<16> kf = kn, vf = vn;
        BwdRow<4> k4[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) k4[r] = k4n[r];
        if (j0 + 16 * kBwdWaves < n) request(j0 + 16 * kBwdWaves);
        bwd_x4 s = bwd_x4{0.0, 0.0, 0.0, 0.0}, cc = bwd_x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            s = __builtin_amdgcn_mfma_f64_16x16x4f64((double)kf.at(t), qd[t], s, 0, 0, 0);
            cc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)vf.at(t), gd[t], cc, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool ok = j0 + 4 * r + g < n;
            const double p = ok ? exp2_f64(fma(s[r], kBwdScaleLog2e, -sd[0])) : 0.0;
            const double gv = ok ? p * fma(cc[r], 0.125, sd[1]) : 0.0;       // g_ij of query c and key 4r + g
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) acc[dt] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)k4[r].at(dt), gv, acc[dt], 0, 0, 0);
        }
    }
    // the four waves' shares in wave order: thread (wave w, lane) adds up register r = w of every accumulator, which
    // gives it the four elements 16 w + 4 g .. + 3 of query c
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 4; ++r) s_acc[wave][4 * dt + r][lane] = acc[dt][r];
    __syncthreads();
    float v[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < kBwdWaves; ++w) t += s_acc[w][4 * dt + wave][lane];
        v[dt] = (float)t;
    }
    if (qi >= 0) bwd_store4(static_cast<float*>(P.dQ) + ((size_t)head * L + qi) * kD + 16 * wave + 4 * g, v);
}

// ---- dK and dV of blocks of 16 KS keys over all kept queries of the head, and dQ over those keys.
// Wave w takes keys 16 (w % KS) .. + 15 of the block and, of the two query tiles of a group, both (KS = 4, 8) or tile
// w / 2 (KS = 2).  Scores are formed upright (queries on the rows), so that a lane's four p and g values are,
// unchanged, the B operand of the products that contract over queries (dK, dV).  For dQ, which contracts over keys,
// the waves put their g values into LDS; wave w then takes, over all keys of the block, elements 16 (w % 4) .. + 15 of
// both tiles, or of 8 waves of tile w / 4, so that nothing has to be added up across waves.
// grid (key splits, heads), heads as above, blocks2 key blocks per work-group, which adds to the dQ it wrote for the block before.
template <int KS, BwdForm FORM>
__global__ __launch_bounds__(BwdShare<KS>::kThreads, 2)
void bwd_main_kernel(const BwdParams P)
{
    using SH = BwdShare<KS>;
    constexpr bool kKeep = FORM == kFused || FORM == kFusedOne;
    const int blocks2 = FORM == kFusedOne ? 1 : P.blocks2;
    constexpr int GR = SH::kGRow, NT = SH::kThreads;
    constexpr int DT = kBwdTiles * kBwdWaves / SH::kWaves;           // query tiles of a group whose dQ a wave forms: 2, or 1 of 8 waves
    extern __shared__ __attribute__((aligned(16))) double bwd_smem[];
    __shared__ double s_gm[kD];
    __shared__ unsigned s_bits[kBwdChunk / 32];                      // the kept ones among 2048 rows
    double* sQ = bwd_smem;
    double* sG = sQ + kBwdGroup * kBwdQRow;
    double* sg = sG + kBwdGroup * kBwdQRow;                          // [2 tiles][16 queries][GR]
    float* sK = reinterpret_cast<float*>(sg + kBwdGroup * GR);       // [keys][kBwdKRow]
    bwd_x2* s_stat = reinterpret_cast<bwd_x2*>(sK + SH::kKeys * kBwdKRow);       // [queries] (log2 sum exp, -D/8)
    const int split = bwd_index(P), head = bwd_head(P, blockIdx.y);
    const int b = head / P.H, L = P.L;
    const int n = valid_len(P.lengths, b, L);
    const int ub = kept_count(P, b, n);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ks = wave % KS, slot = wave / KS;
    const int we = wave & 3, wt = wave >> 2;                         // of dQ: elements 16 we .. + 15 of tiles wt .. wt + DT - 1
    const float* Qh = static_cast<const float*>(P.Q) + (size_t)head * L * kD;
    const float* Kh = static_cast<const float*>(P.K) + (size_t)head * L * kD;
    const float* Vh = static_cast<const float*>(P.V) + (size_t)head * L * kD;
    const float* Gh = static_cast<const float*>(P.G) + (size_t)head * L * kD;

    // the key rows of a block: requested ahead (clamped: harmless if none is valid)
    const int r_first = split * blocks2 * SH::kKeys;
    BwdRow<16> kn, vn;
    auto request = [&](int r0) {
        const int lo = opaque(lane), j = r0 + 16 * ks + (lo & 15), row = j < n ? j : (n > 0 ? n - 1 : 0);
        kn.load(Kh + (size_t)row * kD + 16 * (lo >> 4));
        vn.load(Vh + (size_t)row * kD + 16 * (lo >> 4));
    };
    if (r_first < n) {
        // the mean fill's share of dV: every valid v_j receives 1/n of each filled row's gradient
        if (tid < kD) {
            double t = 0.0;
            if (P.fill == PSA_FILL_MEAN) {
                const double* gs = P.gsum_part + (size_t)head * P.S1 * kD + tid;
#pragma unroll 8
                for (int s = 0; s < P.S1; ++s) t += gs[(size_t)s * kD];      // split order
            }
            s_gm[tid] = t / (double)n;
        }
        if (kKeep) for (int t = tid; t < P.u_pad; t += NT) s_stat[t] = stat_of(P, head, t, n, ub);
        request(r_first);
    }

    if (FORM != kKeysOnly && r_first >= n && P.dq_part) {                                 // no valid key here: zeros
        for (int t = tid >> 4; t < ub; t += NT / 16) {
            bwd_x2* dp = reinterpret_cast<bwd_x2*>(P.dq_part + (((size_t)head * P.S2 + split) * P.u_pad + t) * kD + 4 * (tid & 15));
            dp[0] = dp[1] = bwd_x2{0.0, 0.0};
        }
    }
    QueryStage<kBwdGroup, NT> qs;
    if (r_first < n) { qs.find(P, head, 0); qs.request(Qh, Gh, 0, n, ub); qs.put(sQ, sG); }

    // (Barriers order LDS only: the stores of a block and the loads of the next need not be waited for.  Positions
    // within a tile are derived anew from an opaque lane number where they are used: hoisted out of the loops they
    // would cost registers, and a spilled register is worse than its few instructions, since reading it back waits
    // for the stores before it.)
#pragma unroll 1
    for (int blk = 0; blk < blocks2; ++blk) {
        const int r0 = r_first + blk * SH::kKeys;
        if (r0 >= L) break;                                          // work-group-uniform
        if ((blk * SH::kKeys) % kBwdChunk == 0) {
            // mark the kept rows among the next 2048
            if (tid < kBwdChunk / 32) s_bits[tid] = 0u;
            lds_barrier();
            for (int t = tid; t < ub; t += NT) {
                const int i = P.sel[(size_t)head * P.u_stride + t] - r0;
                if (i >= 0 && i < kBwdChunk && r0 + i < n) atomicOr(&s_bits[i >> 5], 1u << (i & 31));
            }
        }
        // dK^T, dV^T of this wave's 16 keys: acc[dt][r] is element 4 (4r + g) + dt of key c
        bwd_x4 dk[4], dv[4];
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) { dk[dt] = bwd_x4{0.0, 0.0, 0.0, 0.0}; dv[dt] = bwd_x4{0.0, 0.0, 0.0, 0.0}; }
        if (r0 < n && ub > 0) {                                      // work-group-uniform
            const bool wave_live = r0 + 16 * ks < n;                 // wave-uniform: some key of the wave is valid
            const bool more = blk + 1 < blocks2 && r0 + SH::kKeys < n;     // another block with a valid key follows
            // B operands of the score products: this lane's key row.  A row beyond n stands for the last valid one:
            // what comes of it is not stored, and for dQ the staged row is zero.
            double kd[16], vd[16];
            if (FORM != kKeysOnly && slot == 0) {                    // the block's keys as float for the dQ product
                const int lo = opaque(lane), c = lo & 15, g = lo >> 4;
                float4* kr = reinterpret_cast<float4*>(sK + (16 * ks + c) * kBwdKRow + 16 * g);
                const bool ok = r0 + 16 * ks + c < n;
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    kr[k] = ok ? make_float4(kn.at(4 * k), kn.at(4 * k + 1), kn.at(4 * k + 2), kn.at(4 * k + 3)) : make_float4(0.f, 0.f, 0.f, 0.f);
            }
            widen16(kn, kd);
            widen16(vn, vd);

            bwd_x2 old[DT][2];                                // what this very lane wrote of dQ for the block before
            int q_next = 0;
            bool stage_next = false;
            // this wave's share of dQ, elements 16 we .. + 15 of tiles wt .. of group q0 (the A operand's rows are taken
            // in such an order that a lane's four values are elements e_own .. e_own + 3 of query c); two MFMA chains,
            // 16 keys at a time, the next 16 keys' operands read while these products run
            auto finish_group = [&](int q0) {
                if (FORM == kKeysOnly) {
                    if (stage_next) qs.put(sQ, sG);
                    return;
                }
                const int lo = opaque(lane), c = lo & 15, g = lo >> 4;
                const double* gr = sg + (16 * wt + c) * GR + g;
                const float* kr = sK + g * kBwdKRow + 16 * we + 4 * (c & 3) + (c >> 2);
                bwd_x4 dq[DT], dq2 = {0.0, 0.0, 0.0, 0.0};           // dq2: the block's second 64 keys (KS = 8)
                // KS = 8: what this very lane wrote for the block before, and, in the last block, for the split's first half
                // (requested here, under the products: kept from before the barrier they are spilled)
                bwd_x2 first[2];
                if (KS == 8 && blk > 0) {
                    const int t = (q0 + 16 * wt < ub ? q0 + 16 * wt : q0) + c;
                    const double* dp = P.dq_part + (((size_t)head * P.S2 + 2 * split) * P.u_pad + t) * kD + 16 * we + 4 * g;
                    const bwd_x2* op = reinterpret_cast<const bwd_x2*>(2 * blk > blocks2 ? dp + (size_t)P.u_pad * kD : dp);
                    old[0][0] = op[0]; old[0][1] = op[1];
                    if (!more && 2 * blk >= blocks2) { first[0] = reinterpret_cast<const bwd_x2*>(dp)[0]; first[1] = reinterpret_cast<const bwd_x2*>(dp)[1]; }
                }
#pragma unroll
                for (int i = 0; i < DT; ++i) dq[i] = bwd_x4{0.0, 0.0, 0.0, 0.0};
                auto product = [&](auto tiles) {
                    constexpr int NQ = decltype(tiles)::value;
                    float ka[2][4];
                    double gb[2][NQ][4];
                    auto fetch = [&](int kq) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            ka[kq & 1][r] = kr[(16 * kq + 4 * r) * kBwdKRow];
#pragma unroll
                            for (int i = 0; i < NQ; ++i) gb[kq & 1][i][r] = gr[16 * i * GR + 16 * kq + 4 * r];
                        }
                    };
                    fetch(0);
#pragma unroll
                    for (int kq = 0; kq < KS; ++kq) {                // keys in order
                        if (kq + 1 < KS) fetch(kq + 1);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const double kv = (double)ka[kq & 1][r];
#pragma unroll
                            for (int i = 0; i < NQ; ++i) {
                                bwd_x4& sum = kq < 4 ? dq[i] : dq2;
                                sum = __builtin_amdgcn_mfma_f64_16x16x4f64(kv, gb[kq & 1][i][r], sum, 0, 0, 0);
                            }
                        }
                    }
                };
                if constexpr (DT == 2) {
                    if (q0 + 16 < ub) product(std::integral_constant<int, 2>{});
                    else              product(std::integral_constant<int, 1>{});
                } else if (q0 + 16 * wt < ub) {                      // wave-uniform
                    product(std::integral_constant<int, 1>{});
                }
                if (stage_next) qs.put(sQ, sG);                      // (their readers are behind the barrier before this)
                const int e_own = 16 * we + 4 * g;
#pragma unroll
                for (int i = 0; i < DT; ++i) {
                    const int t = q0 + 16 * (wt + i);
                    if (t >= ub) continue;                           // wave-uniform
                    if constexpr (KS == 8) {
                        // The sums of the 4-wave form in its order, so that a call gives the same bits with lengths that are all L
                        // and without: a block is two of its blocks, a split two of its splits (`half` of its blocks each), which
                        // meet in the last block.
                        const int half = blocks2, u = 2 * blk;     // the block's first 64 keys are number u of the split's
                        const bwd_x4 before = bwd_x4{old[i][0][0], old[i][0][1], old[i][1][0], old[i][1][1]};
                        if (blk > 0 && u != half) dq[i] += before;
                        double* const slot = P.dq_part + (((size_t)head * P.S2 + 2 * split) * P.u_pad + t + c) * kD + e_own;
                        auto store = [](double* p, const bwd_x4& v) {
                            reinterpret_cast<bwd_x2*>(p)[0] = bwd_x2{v[0], v[1]};
                            reinterpret_cast<bwd_x2*>(p)[1] = bwd_x2{v[2], v[3]};
                        };
                        if (u + 1 == half && more) {                // the halves meet within the block
                            store(slot, dq[i]);
                            store(slot + (size_t)P.u_pad * kD, dq2);
                            continue;
                        }
                        dq[i] += dq2;
                        if (u >= half && !more) dq[i] += bwd_x4{first[0][0], first[0][1], first[1][0], first[1][1]};
                        if (P.dq_part != nullptr) { store(u >= half && more ? slot + (size_t)P.u_pad * kD : slot, dq[i]); continue; }
                        dq[i] += bwd_x4{0.0, 0.0, 0.0, 0.0};         // (the reduction's sums start from +0)
                    }
                    if (P.dq_part == nullptr) {                      // the only block of the head
                        const int qi = kept_row(P, head, t + c, n, ub);
                        const float v[4] = {(float)dq[i][0], (float)dq[i][1], (float)dq[i][2], (float)dq[i][3]};
                        if (qi >= 0) bwd_store4(static_cast<float*>(P.dQ) + ((size_t)head * L + qi) * kD + e_own, v);
                    } else {
                        if (blk > 0) dq[i] += bwd_x4{old[i][0][0], old[i][0][1], old[i][1][0], old[i][1][1]};
                        bwd_x2* dp = reinterpret_cast<bwd_x2*>(P.dq_part + (((size_t)head * P.S2 + split) * P.u_pad + t + c) * kD + e_own);
                        dp[0] = bwd_x2{dq[i][0], dq[i][1]};
                        dp[1] = bwd_x2{dq[i][2], dq[i][3]};
                    }
                }
            };
            int q0 = 0;
#pragma unroll 1
            for (;; q0 += kBwdGroup) {                               // work-group-uniform
                // the list entries of what comes after this group: the next group, or the first for the next block
                q_next = q0 + kBwdGroup < ub ? q0 + kBwdGroup : 0;
                stage_next = ub > kBwdGroup && (q_next > 0 || more); // work-group-uniform
                if (stage_next) qs.find(P, head, q_next);
                const bwd_x2* stat = s_stat + (kKeep ? q0 : 0);
                if (FORM == kFusedMany && tid < kBwdGroup) s_stat[tid] = stat_of(P, head, q0 + tid, n, ub);
                if (FORM == kKeysOnly && tid < kBwdGroup && q0 + (tid & ~(kBwdQ - 1)) < ub)      // (bwd_dq_kernel wrote whole tiles)
                    s_stat[tid] = reinterpret_cast<const bwd_x2*>(P.stats)[(size_t)head * P.u_pad + q0 + tid];
                lds_barrier();
                {
                    const int lo = opaque(lane), c = lo & 15, g = lo >> 4;
#pragma unroll 1
                    for (int i = 0; i < SH::kPerSlot; ++i) {         // query tiles in order
                        const int tt = slot + i;
                        if (q0 + 16 * tt >= ub) break;               // wave-uniform
                        double* g_out = sg + (16 * tt + g) * GR + 16 * ks + c;
                        if (!wave_live) {                            // (these keys take no part in dQ)
                            if (FORM != kKeysOnly) {
#pragma unroll
                                for (int r = 0; r < 4; ++r) g_out[4 * r * GR] = 0.0;
                            }
                            continue;
                        }
                        bwd_x4 s, cc;
                        score_products<true>(sQ, sG, tt, c, g, kd, vd, s, cc);       // [r]: staged query 16 tt + 4r + g against key c
                        // A operands of the products that contract over the queries: elements 4c .. 4c + 3 of row
                        // 16 tt + 4r + g, the next row's read while this one's products run
                        const double* qr = sQ + (16 * tt + g) * kBwdQRow + 4 * c;
                        const double* gr = sG + (16 * tt + g) * kBwdQRow + 4 * c;
                        bwd_x2 qa[2][2], ga[2][2];
                        auto fetch = [&](int r) {
                            const bwd_x2* x = reinterpret_cast<const bwd_x2*>(qr + 4 * r * kBwdQRow);
                            const bwd_x2* y = reinterpret_cast<const bwd_x2*>(gr + 4 * r * kBwdQRow);
                            qa[r & 1][0] = x[0]; qa[r & 1][1] = x[1]; ga[r & 1][0] = y[0]; ga[r & 1][1] = y[1];
                        };
                        fetch(0);
                        double p[4], gv[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const bwd_x2 sd = stat[16 * tt + 4 * r + g];
                            p[r] = exp2_f64(fma(s[r], kBwdScaleLog2e, -sd[0]));
                            gv[r] = fma(cc[r], 0.125, sd[1]);
                        }
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            gv[r] *= p[r];
                            if (FORM != kKeysOnly) g_out[4 * r * GR] = gv[r];
                        }
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            if (r < 3) { fetch(r + 1); __builtin_amdgcn_sched_barrier(0); }
#pragma unroll
                            for (int dt = 0; dt < 4; ++dt) {
                                dk[dt] = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[r & 1][dt >> 1][dt & 1], gv[r], dk[dt], 0, 0, 0);
                                dv[dt] = __builtin_amdgcn_mfma_f64_16x16x4f64(ga[r & 1][dt >> 1][dt & 1], p[r], dv[dt], 0, 0, 0);
                            }
                        }
                    }
                }
                // under this group's dQ travel: what was written of it for the block before, and the rows of what
                // comes next
                if (FORM != kKeysOnly && KS < 8 && blk > 0) {
                    const int lo = opaque(lane), e_own = 16 * we + 4 * (lo >> 4);
#pragma unroll
                    for (int i = 0; i < DT; ++i) {
                        const int t = (q0 + 16 * (wt + i) < ub ? q0 + 16 * (wt + i) : q0) + (lo & 15);
                        const bwd_x2* dp = reinterpret_cast<const bwd_x2*>(P.dq_part + (((size_t)head * P.S2 + split) * P.u_pad + t) * kD + e_own);
                        old[i][0] = dp[0]; old[i][1] = dp[1];
                    }
                }
                if (stage_next) qs.request(Qh, Gh, q_next, n, ub);
                if (q0 + kBwdGroup >= ub) break;
                lds_barrier();
                finish_group(q0);
            }
            // the last group: the next block's key rows travel too, now that the registers of this one's are free
            if (more) request(r0 + SH::kKeys);
            lds_barrier();
            finish_group(q0);
        }
        lds_barrier();                                               // s_bits; every wave is done with this block's LDS
        if constexpr (SH::kSlots == 2) {
            // the two slots' shares of dK and dV together, through the g tiles' LDS
            const int lo = opaque(lane);
            double* at = sg + (size_t)ks * 8 * 64 + lo;
#pragma unroll
            for (int part = 0; part < 4; ++part) {
                bwd_x4 (&x)[4] = part < 2 ? dk : dv;
                if (part > 0) lds_barrier();
                if (slot == 1) {
#pragma unroll
                    for (int d2 = 0; d2 < 2; ++d2)
#pragma unroll
                        for (int r = 0; r < 4; ++r) at[(4 * d2 + r) * 64] = x[2 * (part & 1) + d2][r];
                }
                lds_barrier();
                if (slot == 0) {
#pragma unroll
                    for (int d2 = 0; d2 < 2; ++d2)
#pragma unroll
                        for (int r = 0; r < 4; ++r) x[2 * (part & 1) + d2][r] += at[(4 * d2 + r) * 64];
                }
            }
        }
        // Rows of dK and dV (and the rows of dQ outside I_sparse, which no gradient reaches).  A lane holds 4-element
        // pieces of one row; they go through the g tiles' LDS, 16 rows of 64 floats per wave (pieces of 16 bytes
        // swapped by row, for the banks), so that a store instruction writes whole rows, 16 bytes per lane.
        if (slot == 0) {
            constexpr int EPV = 4, LPR = kD / EPV, RPI = 64 / LPR;      // elements per lane, lanes per row, rows per instruction
            const int lo = opaque(lane), c = lo & 15, g = lo >> 4;
            float* stage = reinterpret_cast<float*>(sg) + (size_t)ks * 16 * kD;
            const int row_l = lo / LPR, e_l = (lo % LPR) * EPV;
            const int j0 = r0 + 16 * ks, bit0 = (j0 - r_first) % kBwdChunk;          // (a multiple of 16)
            const unsigned bits = (s_bits[bit0 >> 5] >> (bit0 & 31)) & 0xFFFFu;      // kept rows among these 16 (none at or beyond n)
            // the value fill hands v_j the gradient of its own row
            const bool use_own = P.fill != PSA_FILL_MEAN && j0 + c < n && !((bits >> c) & 1u);
            BwdRow<4> own[4];
            if (use_own) {
#pragma unroll
                for (int r = 0; r < 4; ++r) own[r].load(Gh + (size_t)(j0 + c) * kD + 16 * r + 4 * g);
            }
            auto piece = [&](int row, int p4) -> float4* { return reinterpret_cast<float4*>(stage + row * kD + 4 * (p4 ^ row)); };
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const bwd_x4 (&x)[4] = half == 0 ? dk : dv;
                wave_lds_sync();                                     // the first tensor has been read
#pragma unroll
                for (int r = 0; r < 4; ++r) {                        // elements 4 (4r + g) .. + 3 of key c
                    double v[4];
#pragma unroll
                    for (int dt = 0; dt < 4; ++dt) {
                        v[dt] = x[dt][r];
                        if (half == 1 && P.fill == PSA_FILL_MEAN) v[dt] += s_gm[16 * r + 4 * g + dt];
                        if (half == 1 && use_own) v[dt] += (double)own[r].at(dt);
                    }
                    *piece(c, 4 * r + g) = make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
                }
                wave_lds_sync();
                float* base = static_cast<float*>(half == 0 ? P.dK : P.dV) + ((size_t)head * L + j0) * kD + e_l;
                float* base_q = static_cast<float*>(P.dQ) + ((size_t)head * L + j0) * kD + e_l;
#pragma unroll
                for (int it = 0; it < 16 / RPI; ++it) {
                    const int row = it * RPI + row_l;
                    const bool valid = j0 + row < n;
                    float v[EPV];
#pragma unroll
                    for (int q = 0; q < EPV / 4; ++q) {
                        const float4 f = *piece(row, e_l / 4 + q);
                        v[4 * q] = f.x; v[4 * q + 1] = f.y; v[4 * q + 2] = f.z; v[4 * q + 3] = f.w;
                    }
                    if (j0 + row < L) {
                        bwd_store16(base + (size_t)row * kD, v, valid);
                        if (half == 0 && !((bits >> row) & 1u)) bwd_store16(base_q + (size_t)row * kD, v, false);
                    }
                }
            }
        }
        lds_barrier();                                               // the next block's LDS
    }
}

// adds the key splits of dQ in split order, two and two first (a split of the 8-wave form is the sum of two; PAIRS: the sums are
// still to be formed); 16 threads per kept query, 4 elements each
template <bool PAIRS>
__global__ __launch_bounds__(256)
void bwd_dq_reduce_kernel(const BwdParams P)
{
    const int head = bwd_head(P, blockIdx.y);
    const int n = valid_len(P.lengths, head / P.H, P.L);
    const int ub = kept_count(P, head / P.H, n);
    const int t = bwd_index(P) * 16 + (threadIdx.x >> 4), e0 = 4 * (threadIdx.x & 15);
    const int qi = kept_row(P, head, t, n, ub);
    if (qi < 0) return;
    const double* dp = P.dq_part + ((size_t)head * P.S2 * P.u_pad + t) * kD + e0;
    const size_t step = (size_t)P.u_pad * kD;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    constexpr int kBatch = PAIRS ? 2 : 4;
#pragma unroll kBatch
    for (int s = 0; s < P.S2; s += 2) {
        bwd_x2 x = *reinterpret_cast<const bwd_x2*>(dp + s * step), y = *reinterpret_cast<const bwd_x2*>(dp + s * step + 2);
        if (PAIRS) {
            const bool one = s + 1 == P.S2;
            const double* second = dp + (one ? s : s + 1) * step;
            const bwd_x2 x2 = *reinterpret_cast<const bwd_x2*>(second), y2 = *reinterpret_cast<const bwd_x2*>(second + 2);
            x += one ? bwd_x2{0.0, 0.0} : x2;
            y += one ? bwd_x2{0.0, 0.0} : y2;
        }
        acc[0] += x[0]; acc[1] += x[1]; acc[2] += y[0]; acc[3] += y[1];
    }
    const float v[4] = {(float)acc[0], (float)acc[1], (float)acc[2], (float)acc[3]};
    bwd_store4(static_cast<float*>(P.dQ) + ((size_t)head * P.L + qi) * kD + e0, v);
}

static hipError_t raise_bwd_limits()
{
    constexpr int N = 8;
    static std::atomic<uint64_t> raised[N];            // per kernel: devices already served
    const void* fn[N] = {(const void*)bwd_stats_kernel, (const void*)bwd_main_kernel<4, kFused>,
                         (const void*)bwd_main_kernel<2, kFused>, (const void*)bwd_main_kernel<4, kFusedMany>,
                         (const void*)bwd_main_kernel<4, kKeysOnly>, (const void*)bwd_main_kernel<2, kKeysOnly>,
                         (const void*)bwd_main_kernel<8, kFused>, (const void*)bwd_main_kernel<8, kFusedOne>};
    const int lds[N] = {kBwdStatsLds, BwdShare<4>::kLds, BwdShare<2>::kLds, BwdShare<4>::kLds, BwdShare<4>::kLds, BwdShare<2>::kLds, BwdShare<8>::kLds, BwdShare<8>::kLds};
    for (int k = 0; k < N; ++k) { const hipError_t e = ensure_lds_limit(fn[k], lds[k], raised[k]); if (e != hipSuccess) return e; }
    return hipSuccess;
}
hipError_t init_backward() { return raise_bwd_limits(); }

static hipError_t launch_bwd(const BwdParams& P, int BH, int ks, int splits, hipStream_t stream)
{
    const hipError_t e = raise_bwd_limits();
    if (e != hipSuccess) return e;
    auto dealt = [&](int x) { return (unsigned)x << P.head_shift; };
    const unsigned heads = (unsigned)BH >> P.head_shift;
    const dim3 grid(dealt(splits), heads), block(kBwdThreads);
    hipLaunchKernelGGL(bwd_stats_kernel, dim3(dealt(P.S1), P.n_group, heads), block, kBwdStatsLds, stream, P);
    if (P.stats) {
        hipLaunchKernelGGL(bwd_dq_kernel, dim3(dealt(P.u_pad / kBwdQ), heads), block, 0, stream, P);
        if (ks == 4) hipLaunchKernelGGL((bwd_main_kernel<4, kKeysOnly>), grid, block, BwdShare<4>::kFixed + kBwdGroup * 16, stream, P);
        else         hipLaunchKernelGGL((bwd_main_kernel<2, kKeysOnly>), grid, block, BwdShare<2>::kFixed + kBwdGroup * 16, stream, P);
    } else if (P.u_pad > kBwdKeepStats)
        hipLaunchKernelGGL((bwd_main_kernel<4, kFusedMany>), grid, block, BwdShare<4>::kFixed + kBwdGroup * 16, stream, P);
    else if (ks == 8 && P.blocks2 == 1)
        hipLaunchKernelGGL((bwd_main_kernel<8, kFusedOne>), grid, dim3(BwdShare<8>::kThreads), BwdShare<8>::kFixed + P.u_pad * 16, stream, P);
    else if (ks == 8)
        hipLaunchKernelGGL((bwd_main_kernel<8, kFused>), grid, dim3(BwdShare<8>::kThreads), BwdShare<8>::kFixed + P.u_pad * 16, stream, P);
    else if (ks == 4)
        hipLaunchKernelGGL((bwd_main_kernel<4, kFused>), grid, block, BwdShare<4>::kFixed + P.u_pad * 16, stream, P);
    else
        hipLaunchKernelGGL((bwd_main_kernel<2, kFused>), grid, block, BwdShare<2>::kFixed + P.u_pad * 16, stream, P);
    const dim3 grid_r(dealt(P.u_pad / kBwdQ), heads);
    if (P.dq_part && ks == 8) hipLaunchKernelGGL((bwd_dq_reduce_kernel<false>), grid_r, dim3(256), 0, stream, P);
    else if (P.dq_part)       hipLaunchKernelGGL((bwd_dq_reduce_kernel<true>), grid_r, dim3(256), 0, stream, P);
    return hipGetLastError();
}

// Time of `wgs` equal work-groups, two per CU in rounds of 512, in times of one round (a CU with one work-group takes
// 0.6 of the time of one with two).
static double bwd_rounds(int64_t wgs)
{
    const int64_t half = (wgs + 255) / 256;
    return (double)(half / 2) + (half & 1 ? 0.6 : 0.0);
}
// Key blocks per work-group for `rows` (head, query group) pairs of `n_blocks` blocks: the number that takes the
// least time, each work-group paying `fixed` (staging, first loads; in units of a block's work) beside its blocks.  At
// most `max_split` splits.
static int blocks_per_split(int64_t rows, int n_blocks, int64_t max_split, double fixed, double* cost_out)
{
    int best = n_blocks;
    double best_cost = 1e300;
    for (int r = 1; r <= 8; ++r) {                              // half rounds of the CUs aimed at
        int64_t S = 256 * r / rows;
        S = S < 1 ? 1 : (S > max_split ? max_split : (S > n_blocks ? n_blocks : S));
        const int per = (int)((n_blocks + S - 1) / S);
        const double cost = bwd_rounds(rows * ((n_blocks + per - 1) / per)) * (per + fixed);
        if (cost < best_cost) { best_cost = cost; best = per; }
    }
    *cost_out = best_cost;
    return best;
}

// Plan of the backward: query groups, key splits and the carving of its workspace (host arithmetic).
BwdPlan make_bwd_plan(const psa_shape_t& s, int u_stride)
{
    BwdPlan p;
    const int64_t BH = (int64_t)s.B * s.H;
    p.n_group = (u_stride + kBwdStatGroup - 1) / kBwdStatGroup;
    p.u_pad = (u_stride + kBwdQ - 1) / kBwdQ * kBwdQ;
    const int tiles = p.u_pad / kBwdQ;
    double cost;
    const int n_blocks = (s.L_K + kBwdKeys - 1) / kBwdKeys;
    p.blocks1 = blocks_per_split(BH * p.n_group, n_blocks, kBwdMaxSplit, 4.0 / (tiles < 4 ? tiles : 4), &cost);
    p.S1 = (n_blocks + p.blocks1 - 1) / p.blocks1;
    // The gradient kernel: blocks of 64 keys, or of 32 with the waves sharing out the query tiles as well where
    // there are too few heads and keys to give every CU work of the larger kind.  In units of one query tile on 4
    // waves (80 MFMAs, 2.2 us); beside its tiles a work-group pays about two such units, and the smaller blocks a
    // little more for adding up the slots' shares and for more splits of dQ.
    // Fused form: the float64 partial sums of dQ, one set per key split, stay within a quarter of the memory that the
    // call's own seven tensors take, or 256 MiB where that is more (without a bound one sequence of 16384 frames with
    // half of its queries kept asked for 2.1 GB beside tensors of 17 MB).  They are written for every key block, read
    // for every one after a work-group's first, and read by the reduce kernel: a unit for 50 MB.
    const size_t split_bytes = (size_t)BH * p.u_pad * kD * sizeof(double);
    const size_t tensors = (size_t)BH * s.L_K * kD * (s.dtype == PSA_F32 ? 4 : 2) * 7;       // Q, K, V, dOut, dQ, dK, dV
    const size_t fit = (tensors / 4 > kBwdPartBytes ? tensors / 4 : kBwdPartBytes) / split_bytes;
    const int max_split = fit < (size_t)kBwdMaxSplit ? (int)fit : kBwdMaxSplit;
    double best = 1e300;
    for (int ks = 4; ks >= (p.u_pad > kBwdKeepStats ? 4 : 2) && max_split > 0; ks >>= 1) {
        const int slots = kBwdWaves / ks, nb = (s.L_K + 16 * ks - 1) / (16 * ks);
        const double per_block = (double)((tiles + slots - 1) / slots) + (slots > 1 ? 0.5 : 0.0);
        const int per = blocks_per_split(BH, nb, max_split, 2.0 / per_block, &cost);
        if (cost * per_block < best * 0.95) {
            best = cost * per_block;
            p.ks = ks; p.blocks2 = per; p.S2 = (nb + per - 1) / per;
        }
    }
    p.keys_only = 0;
    if (best < 1e300) {
        const int nb = (s.L_K + 16 * p.ks - 1) / (16 * p.ks);
        best = best * (p.u_pad > kBwdKeepStats ? 1.09 : 1.0) + (double)split_bytes * (2 * nb) / 50e6;
    }
    // The form without partial sums: 0.8 of the products in bwd_main_kernel, one block a work-group, and 0.6 of them in
    // bwd_dq_kernel (a work-group for each query tile, all keys).  It is taken where it is estimated to be faster: where the
    // bound on the partial sums leaves too few key splits, or where few heads with many kept queries do not fill the
    // CUs with blocks of 64 keys.  Measured (whole call), fused against this form: B=16 H=4 L=512, 256 kept 168 | 203
    // us; B=8 H=8 L=2048, 1024 kept 2381 | 2672; B=4 H=4 L=1600, 800 kept 483 | 551; B=1 H=4 L=2000, 1000 kept 338 | 209;
    // B=1 H=8 L=4096, 2048 kept 1412 (in the 32 splits that fit) | 1355; L=16384, 8192 kept 76500 (8 splits) | 20970.
    const double dq = bwd_rounds(BH * tiles) * (0.6 * n_blocks + 1.0) + 1.5;
    for (int ks = 4; ks >= 2; ks >>= 1) {
        const int slots = kBwdWaves / ks, nb = (s.L_K + 16 * ks - 1) / (16 * ks);
        const double per_block = (double)((tiles + slots - 1) / slots) + (slots > 1 ? 0.5 : 0.0);
        const double c = bwd_rounds(BH * nb) * (0.8 * per_block + 1.0) + dq;
        if (c < best * (p.keys_only ? 0.95 : 1.0)) {
            best = c;
            p.keys_only = 1; p.ks = ks; p.blocks2 = 1; p.S2 = nb;
        }
    }
    // Fused form, blocks of 128 keys on work-groups of 8 waves, one to a CU, instead of two of 4 waves: half the partial sums of dQ to
    // write and to add up, the group's query rows staged once instead of twice.  Where they take no more rounds (a CU with one
    // of the smaller work-groups is faster than one with two; these come whole), and only for calls without lengths, which
    // alone are known to be full batches: with lengths the smaller ones spread better.  Whole call: B=16 H=4 L=512, 256 kept
    // 162.9 -> 150.4 us, and 147 where one block a split is compiled on its own (no registers spilled); B=16 H=8 L=256, 128 kept
    // 93.7 -> 86.5, 84; B=8 H=8 L=1024, 512 kept 571.6 -> 533.0; B=32 H=4 L=512, 205 kept 263.5 -> 249.2; two rounds for one and a half, B=24 H=8 L=200, 100 kept 129.6 -> 136.6; lengths of 64 .. 512 at B=8 H=8
    // L=512, 256 kept 132.2 -> 139.7, of 50 .. 400 at B=16 H=8 L=400, 200 kept 194.7 -> 209.3.
    p.wide_S2 = 0;
    if (!p.keys_only && p.ks == 4 && p.u_pad <= kBwdKeepStats && p.S2 > 1) {
        const int nb = (s.L_K + BwdShare<8>::kKeys - 1) / BwdShare<8>::kKeys, S = (nb + p.blocks2 - 1) / p.blocks2;
        const int64_t wgs = BH * S;
        if (wgs >= 256 && (double)((wgs + 255) / 256) <= bwd_rounds(BH * p.S2)) p.wide_S2 = S;
    }
    // dQ goes straight to memory where one block holds all keys of a head
    p.parts = !p.keys_only && (p.S2 > 1 || p.blocks2 > 1);
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    size_t off = 0;
    p.off_stats_part = off; off += al((size_t)BH * p.S1 * p.u_pad * 3 * sizeof(double));
    p.off_gsum = off;       off += al((size_t)BH * p.S1 * kD * sizeof(double));
    p.off_stats = off;      off += p.keys_only ? al((size_t)BH * p.u_pad * 2 * sizeof(double)) : 0;
    p.off_dq_part = off;    off += p.parts ? al((size_t)BH * p.S2 * p.u_pad * kD * sizeof(double)) : 0;
    p.total = off;
    return p;
}

hipError_t launch_backward(const psa_shape_t& s, const BwdPlan& bp, const void* Q, const void* K, const void* V,
                           const int* lengths, const int* sel, const int* u, int u_stride, int fill, const void* G,
                           void* dQ, void* dK, void* dV, void* workspace, hipStream_t stream)
{
    if (s.dtype != PSA_F32)
        return launch_backward_bf16(s, make_bwd16_plan(s, u_stride, bp.total), Q, K, V, lengths, sel, u, u_stride, fill, G, dQ, dK, dV, workspace, stream);
    unsigned char* w = static_cast<unsigned char*>(workspace);
    BwdParams P;
    P.Q = Q; P.K = K; P.V = V; P.G = G; P.lengths = lengths; P.sel = sel; P.u = u;
    P.dQ = dQ; P.dK = dK; P.dV = dV;
    P.stats_part = reinterpret_cast<double*>(w + bp.off_stats_part);
    P.gsum_part = reinterpret_cast<double*>(w + bp.off_gsum);
    const bool wide = bp.wide_S2 > 0 && lengths == nullptr;          // (fewer key splits than the scratch has room for)
    const bool parts = wide ? bp.wide_S2 > 1 || bp.blocks2 > 1 : bp.parts;
    P.dq_part = parts ? reinterpret_cast<double*>(w + bp.off_dq_part) : nullptr;
    P.stats = bp.keys_only ? reinterpret_cast<double*>(w + bp.off_stats) : nullptr;
    P.H = s.H; P.L = s.L_K; P.u_stride = u_stride; P.u_pad = bp.u_pad; P.n_group = bp.n_group;
    P.S1 = bp.S1; P.blocks1 = bp.blocks1; P.S2 = bp.S2; P.blocks2 = bp.blocks2;
    P.fill = fill; P.head_shift = (s.B * s.H) % 8 == 0 ? 3 : 0;
    return launch_bwd(P, s.B * s.H, wide ? 8 : bp.ks, wide ? bp.wide_S2 : bp.S2, stream);
}

}  // namespace psa
