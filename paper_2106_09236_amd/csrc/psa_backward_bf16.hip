// Gradients of stages a3 and a4 for bfloat16 tensors (what they are: psa_backward.hip), on the bfloat16 matrix cores.
//   bwd16_stats_kernel    softmax statistics per kept query and key split; column sums of dOut over the filled rows
//   bwd16_main_kernel     work-groups of two kinds: some take 32 kept queries and walk keys (dQ), the others take 128 keys and
//                         walk the kept queries (dK, dV, the fill's share, zero rows)
//   bwd16_reduce_kernel   adds the partial sums of dQ, where the keys of a head were split among work-groups
//
// Arithmetic: float32 throughout.  Products of two bfloat16 values are exact in the MFMA's float32 accumulator; a float32
// operand (the weights p and what multiplies them) enters as three bfloat16 planes cut from its 24 significant bits, whose sum
// is the value itself.  What made float32 unusable for these gradients (errors of 4 times the gradient's size where attention
// is sharply peaked) is the difference c_ij - D_i, c_ij = G_i . v_j, of nearly equal numbers: a softmax row with p = 1 - e on one key
// has gradients of size e.  They depend on differences of c within the row only, so c is taken relative to a reference c*_i,
// its value at the row's heaviest key, or the mean so far:
//   c'_ij = c_ij - c*_i     w_i = sum_j e_ij c'_ij     D'_i = w_i / l_i     g_ij = p_ij (c'_ij - D'_i) / sqrt(d)
// A key that holds nearly all the weight then contributes next to nothing to w, every other term carries its small weight,
// and no two large terms are left to cancel: the errors are those of float32, relative to each term.  dQ has to wait for D'
// for the same reason: sum e c' k - D' sum e k, which needs one pass less, cancels what the keys have in common and
// measured 5 times the error of sum g k.
//
// Relative error (2-norm) against float64: 1.6e-3 .. 1.7e-3 for each gradient, that of the last rounding to bfloat16 and the same as
// with float64 throughout, on 24 shapes of normal, peaked and mixed inputs (B=1..58, L=40..2892, both rules for u).
//
// What bounds it: B=8 H=8 L=2048, 39 kept queries: statistics 17 us (51 MB read, in about 10 us; the rest is the start, the column
// sums' exchange and the merge of the streams), main kernel 27 us (34 MB read twice, 50 MB written; chains of loads, score
// products, weights, products of two waves a SIMD).  Whole call 138 us in float64 on the float64 matrix pipe -> 42 us; 1024 kept
// 2389 -> 403 us; B=1 H=8 L=16384, 49 kept 181 -> 49 us; B=1 H=4 L=128, 25 kept 21.6 -> 14.3 us.  Measured on the main kernel and
// not kept: dK and dV from waves of their own, four to a SIMD (47 us); two key splits for dQ and their sum 29 + 4 us; work-groups
// of one block of keys 31 us, dQ's work-groups last 33 us.
//
// A plane of a weight that is zero times an infinite dOut or K is NaN: with infinities in the inputs gradients that were
// infinite are NaN.
//
// MFMA lanes: psa_tile.h.  Scores are formed with the kept queries on the columns where queries are walked over keys, with
// the keys on the columns in the other kind; either way the accumulator registers are, unchanged, the B operand of the
// products that follow.
#include "psa_backward_common.h"
#include "psa_tile.h"

namespace psa {

constexpr int kB16Threads = 512, kB16Waves = kB16Threads / 64;   // statistics: 8 waves
constexpr int kM16Threads = 256, kM16Waves = kM16Threads / 64;   // main kernel: 4 waves of up to 256 registers, two work-groups per CU
constexpr int kM16Keys = 32 * kM16Waves;                         // keys per block
constexpr int kM16Group = 64;                                    // kept queries staged in LDS at a time
constexpr int kRowF = kD + 4;                                    // floats between staged float rows
constexpr int kBitRows = 2048;                                   // rows per bit mask of kept rows

// Softmax statistics of one kept query over some keys, relative to maximum m (base 2) and reference c*.  l and w are float64
// between tiles and from there on: an error of D' is an error of the sum of a query's g, which multiplies what its keys
// have in common (mixtures of 32 centres, 16384 keys: float32 sums 5 times the error of dQ there).
struct Stat16 { float m, c; double l, w; };
__device__ __forceinline__ float stat_factor(float m, float M) { return m == -INFINITY ? 0.f : fast_exp2(m - M); }
__device__ __forceinline__ Stat16 stat_merge(const Stat16& a, const Stat16& b)
{
    Stat16 t;
    t.m = fmaxf(a.m, b.m);
    t.c = a.m >= b.m ? a.c : b.c;
    const double fa = stat_factor(a.m, t.m), fb = stat_factor(b.m, t.m);
    t.l = fa * a.l + fb * b.l;
    t.w = fa * fma((double)a.c - (double)t.c, a.l, a.w) + fb * fma((double)b.c - (double)t.c, b.l, b.w);
    return t;
}

struct Bwd16Params {
    const bf16_t* Q; const bf16_t* K; const bf16_t* V; const bf16_t* G;
    const int* lengths; const int* sel; const int* u;
    bf16_t* dQ; bf16_t* dK; bf16_t* dV;
    Stat16* stat;          // [BH][S1][u_stride]  per kept query and key split
    double* gsum_part;     // [BH][S1 n_group][64]  column sums of G over valid rows outside I_sparse
    float* dq_part;        // [BH][SQ][u_stride][64]  dQ of the key splits (SQ > 1)
    int H, L, BH, u_stride, n_group, S1, tiles1, SQ, tilesq, S2, blocks2, fill, n_dq;    // n_dq: work-groups that compute dQ
};

// Eight float32 values of a lane (MFMA k slots 8h .. 8h + 7) as three bfloat16 planes whose sum they are: the upper 16
// bits of the value, of what is left, and of what is left then (8 significant bits each; truncation, so all exact).  What is
// left comes from one v_dot2_f32_bf16, the pair of planes times (-1, 0) or (0, -1), where a mask and a difference are two.
__device__ __forceinline__ void planes3(const float (&x)[8], uint4 (&pl)[3])
{
    // in scalar registers: as a literal the compiler encodes (-1, 0) as the inline constant -1.0, which the instruction
    // reads as another pair
    uint32_t minus_lo = 0x0000BF80u, minus_hi = 0xBF800000u;
    asm("" : "+s"(minus_lo), "+s"(minus_hi));
    uint32_t w[3][4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float a = x[2 * e], b = x[2 * e + 1];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            w[k][e] = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
            if (k < 2) {
                const bf16x2 top = __builtin_bit_cast(bf16x2, w[k][e]);
                a = __builtin_amdgcn_fdot2_f32_bf16(top, __builtin_bit_cast(bf16x2, minus_lo), a, false);
                b = __builtin_amdgcn_fdot2_f32_bf16(top, __builtin_bit_cast(bf16x2, minus_hi), b, false);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) pl[k] = make_uint4(w[k][0], w[k][1], w[k][2], w[k][3]);
}
__device__ __forceinline__ floatx16 mfma16(const uint4& a, const uint4& b, const floatx16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ floatx16 zero16() {
    floatx16 z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.f;
    return z;
}
// Transposed operand of 32 staged rows (stride kB16Stride): row slots of step st, column 32 dt + c (psa_tile.h, load_v_operand)
__device__ __forceinline__ uint4 transposed(const uint16_t* s, int st, int dt, int c, int h)
{
    typedef short shortx4 __attribute__((ext_vector_type(4)));
    const int s16 = c & 15;
    const uint16_t* p = s + (16 * st + 4 * h + (s16 >> 2)) * kB16Stride + 32 * dt + (c & 16) + 4 * (s16 & 3);
    const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)(p)));
    const uint2 hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (shortx4 __attribute__((address_space(3)))*)(p + 8 * kB16Stride)));
    return make_uint4(lo.x, lo.y, hi.x, hi.y);
}
// this lane's 64 bytes (elements 32h .. 32h + 31) of a row of a head: zeros at or beyond the length, and for row < 0
__device__ __forceinline__ void load_half_row(uint4 (&x)[4], __amdgpu_buffer_rsrc_t rows, int row, int h)
{
    const int ofs = row < 0 ? -64 : row * 128 + 64 * h;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) x[kk] = buffer_load16<uint4>(rows, ofs + (row < 0 ? 0 : 16 * kk));
}

// A tile of 32 rows from `first` on as it lies in memory, eight lanes a row (whole lines: as MFMA operands straight from memory,
// 16 bytes of 64 rows in an instruction, the loads alone took 14 us of a work-group that walks 64 tiles), zeros beyond the
// length; `want` false: zeros.  The request is made either way, since one in a branch of its own makes every later wait of the
// loop count as if it had not been made.
constexpr int kNoRows = 1 << 23;                                     // beyond any head (L <= 2^22)
__device__ __forceinline__ void load_rows(uint4 (&x)[4], __amdgpu_buffer_rsrc_t rows, bool want, int first, int lane)
{
    const int ofs = (want ? first + (lane >> 3) : kNoRows) * 128 + 16 * (lane & 7);
#pragma unroll
    for (int it = 0; it < 4; ++it) x[it] = buffer_load16<uint4>(rows, ofs + 1024 * it);
}
// ... into a wave's LDS tile, and from there as an MFMA operand: elements 32h .. 32h + 31 of row c
__device__ __forceinline__ void put_rows(const uint4 (&x)[4], uint16_t* s, int lane)
{
#pragma unroll
    for (int it = 0; it < 4; ++it) *reinterpret_cast<uint4*>(s + (8 * it + (lane >> 3)) * kB16Stride + 8 * (lane & 7)) = x[it];
}
__device__ __forceinline__ void get_operand(uint4 (&x)[4], const uint16_t* s, int c, int h)
{
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) x[kk] = *reinterpret_cast<const uint4*>(s + c * kB16Stride + 32 * h + 8 * kk);
}
// both in turn through the same LDS tile
__device__ __forceinline__ void to_operands(const uint4 (&kx)[4], const uint4 (&vx)[4], uint16_t* s, uint4 (&ka)[4], uint4 (&va)[4], int lane)
{
    wave_lds_sync();
    put_rows(kx, s, lane);
    wave_lds_sync();
    get_operand(ka, s, lane & 31, lane >> 5);
    wave_lds_sync();
    put_rows(vx, s, lane);
    wave_lds_sync();
    get_operand(va, s, lane & 31, lane >> 5);
}

// (head, index within the head) of work-group `id`: all work-groups of a head on one XCD where the heads divide evenly
__device__ __forceinline__ void head_of(int id, int BH, int per_head, int& head, int& x)
{
    if (BH % 8 == 0) { const int slot = id >> 3; head = slot / per_head * 8 + (id & 7); x = slot % per_head; }
    else             { head = id / per_head; x = id % per_head; }
}

// ---- statistics.  A work-group takes up to 64 kept queries (rows of Q and G in LDS) over the keys of one split; each of its
// waves takes a key stream of its own (32 keys a step: rows of K and V in registers, read once for both query tiles), and the
// streams are merged through LDS at the end.
__global__ __launch_bounds__(kB16Threads)
void bwd16_stats_kernel(const Bwd16Params P)
{
    __shared__ __attribute__((aligned(16))) uint16_t sQ[kM16Group * kB16Stride], sG[kM16Group * kB16Stride];
    __shared__ __attribute__((aligned(16))) uint16_t s_tiles[kB16Waves][32 * kB16Stride];    // a tile for each wave, its statistics in the end
    __shared__ double s_gs[kB16Waves][kD];
    __shared__ unsigned s_bits[kBitRows / 32];
    int head, x;
    head_of(blockIdx.x, P.BH, P.S1 * P.n_group, head, x);
    const int split = x / P.n_group, group = x % P.n_group;
    const int b = head / P.H, L = P.L;
    const int n = valid_len(P.lengths, b, L);
    const int ub = kept_count(P, b, n);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), c = lane & 31, h = lane >> 5;
    const int q0 = group * kM16Group;
    const size_t base = (size_t)head * L * kD;
    const __amdgpu_buffer_rsrc_t Kr = head_rows<128>(P.K + base, n), Vr = head_rows<128>(P.V + base, n), Gr = head_rows<128>(P.G + base, n);
    const int t_first = split * P.tiles1, t_all = (n + 31) >> 5;
    const int t_end = t_first + P.tiles1 < t_all ? t_first + P.tiles1 : t_all;
    const bool any = q0 < ub;                                        // work-group-uniform: some kept query is here
    const bool sums = P.fill == PSA_FILL_MEAN;

    // everything that is needed first, in the order in which it is: list entries, rows of Q and G (8 threads a row), key rows
    int t = t_first + wave;
    uint4 kx[4], vx[4], xq, xg;
    if (any) {
        const int row = kept_row(P, head, q0 + (tid >> 3), n, ub);
        const int ofs = row < 0 ? -16 : row * 128 + 16 * (tid & 7);
        xq = buffer_load16<uint4>(head_rows<128>(P.Q + base, n), ofs);
        xg = buffer_load16<uint4>(Gr, ofs);
        load_rows(kx, Kr, t < t_end, 32 * t, lane);
        load_rows(vx, Vr, t < t_end, 32 * t, lane);
    }
    // the rows of G whose columns this work-group adds up: its share of the split's (they are dealt to the groups)
    constexpr int RPP = kB16Threads / 8, NB = 2;                     // rows per pass, passes per batch
    static_assert(kBitRows % (NB * RPP) == 0, "a batch lies in one bit mask");
    const int share = ((P.tiles1 + P.n_group - 1) / P.n_group) * 32;
    const int r_first = t_first * 32 + group * share;
    int r_end = (t_first + P.tiles1) * 32;
    r_end = r_end < r_first + share ? r_end : r_first + share;
    r_end = sums ? (r_end < n ? r_end : n) : r_first;
    uint4 g[NB];
    auto request = [&](int r0) {
#pragma unroll
        for (int k = 0; k < NB; ++k) g[k] = buffer_load16<uint4>(Gr, (r0 + k * RPP + (tid >> 3)) * 128 + 16 * (tid & 7));
    };
    if (r_first < r_end) request(r_first);
    if (any) {
        *reinterpret_cast<uint4*>(sQ + (tid >> 3) * kB16Stride + 8 * (tid & 7)) = xq;
        *reinterpret_cast<uint4*>(sG + (tid >> 3) * kB16Stride + 8 * (tid & 7)) = xg;
        lds_barrier();
    }

    Stat16 st[2] = {{-INFINITY, 0.f, 0.0, 0.0}, {-INFINITY, 0.f, 0.0, 0.0}};     // (l and w of this lane's keys)
    auto tile_step = [&](int step) {
        const int j0 = 32 * t;
        uint4 ka[4], va[4];
        to_operands(kx, vx, s_tiles[wave], ka, va, lane);
        load_rows(kx, Kr, t + kB16Waves < t_end, j0 + 32 * kB16Waves, lane);
        load_rows(vx, Vr, t + kB16Waves < t_end, j0 + 32 * kB16Waves, lane);
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
            if (q0 + 32 * qt >= ub) break;                           // work-group-uniform
            floatx16 s = zero16(), cc = zero16();
            const int at = (32 * qt + c) * kB16Stride + 32 * h;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) s = mfma16(ka[kk], *reinterpret_cast<const uint4*>(sQ + at + 8 * kk), s);
            __builtin_amdgcn_sched_barrier(0);                       // (or all operands are read ahead, and registers spilled)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) cc = mfma16(va[kk], *reinterpret_cast<const uint4*>(sG + at + 8 * kk), cc);
            if (j0 + 32 > n) {                                       // wave-uniform: the item's last keys
#pragma unroll
                for (int r = 0; r < 16; ++r) s[r] = j0 + 8 * (r >> 2) + 4 * h + (r & 3) < n ? s[r] : -INFINITY;
            }
            Stat16& y = st[qt];
            float tmax = s[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) tmax = fmaxf(tmax, s[r]);
            const float tm = max_xor32(tmax) * kScaleLog2e;
            const bool centre = (step & (step - 1)) == 0;            // wave-uniform
            if (centre || __ballot(tm > y.m + kLagLog2) != 0ull) {
                // some query's scores have grown: its maximum and reference move to this tile's heaviest key; the others'
                // references move to the mean of c so far
                float cr = cc[0];
#pragma unroll
                for (int r = 1; r < 16; ++r) cr = s[r] == tmax ? cc[r] : cr;
                const float t_o = __shfl_xor(tmax, 32, 64), c_o = __shfl_xor(cr, 32, 64);
                cr = tmax > t_o || (tmax == t_o && h == 0) ? cr : c_o;
                const bool grow = tm > y.m + kLagLog2;
                const float lt = (float)(y.l + __shfl_xor(y.l, 32, 64)), wt = (float)(y.w + __shfl_xor(y.w, 32, 64));
                const float mean = lt > 0.f ? y.c + wt / lt : y.c;
                const float m_new = grow ? tm : y.m, c_new = grow ? cr : mean;
                const double a = grow ? stat_factor(y.m, m_new) : 1.f;
                y.w = a * fma((double)y.c - (double)c_new, y.l, y.w);
                y.l *= a;
                y.m = m_new; y.c = c_new;
            }
            float lt = 0.f, wt = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float e = fast_exp2(fmaf(s[r], kScaleLog2e, -y.m));
                lt += e;
                wt = fmaf(e, cc[r] - y.c, wt);
            }
            y.l += (double)lt;
            y.w += (double)wt;
        }
    };
    // the first step before the column sums, whose rows arrive behind the first key rows (and the next under the sums)
    const bool first = any && t < t_end;                             // wave-uniform
    if (first) { tile_step(0); t += kB16Waves; }

    if (sums) {
        double acc[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = 0.0;
#pragma unroll 1
        for (int r0 = r_first; r0 < r_end; r0 += NB * RPP) {         // work-group-uniform
            const int bit0 = (r0 - r_first) % kBitRows;
            if (bit0 == 0) {
                // mark the kept rows among the next 2048: they take no part in the column sums
                lds_barrier();
                if (tid < kBitRows / 32) s_bits[tid] = 0u;
                lds_barrier();
                for (int k = tid; k < ub; k += kB16Threads) {
                    const int i = P.sel[(size_t)head * P.u_stride + k] - r0;
                    if (i >= 0 && i < kBitRows) atomicOr(&s_bits[i >> 5], 1u << (i & 31));
                }
                lds_barrier();
            }
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const int r = k * RPP + (tid >> 3), bit = bit0 + r;
                const bool use = r0 + r < r_end && !((s_bits[bit >> 5] >> (bit & 31)) & 1u);
                const uint32_t v[4] = {g[k].x, g[k].y, g[k].z, g[k].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    acc[2 * e] += (double)(use ? bf16_lo(v[e]) : 0.f);
                    acc[2 * e + 1] += (double)(use ? bf16_hi(v[e]) : 0.f);
                }
            }
            if (r0 + NB * RPP < r_end) request(r0 + NB * RPP);
        }
        // over the 8 lanes that hold the same columns, halving the columns of a lane at each exchange
#pragma unroll
        for (int half = 4; half > 0; half >>= 1) {
            const bool upper = lane & (8 * half);
#pragma unroll
            for (int e = 0; e < half; ++e) {
                const double send = upper ? acc[e] : acc[e + half];
                acc[e] = (upper ? acc[e + half] : acc[e]) + __shfl_xor(send, 8 * half, 64);
            }
        }
        s_gs[wave][8 * (lane & 7) + (lane >> 3)] = acc[0];
        lds_barrier();
        if (tid < kD) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < kB16Waves; ++w) s += s_gs[w][tid];    // fixed order
            P.gsum_part[((size_t)head * P.S1 * P.n_group + x) * kD + tid] = s;
        }
    }
    if (!any) return;

#pragma unroll 1
    for (int step = 1; t < t_end; t += kB16Waves, ++step) tile_step(step);       // wave-uniform
    // the key streams together, in wave order
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
        st[qt].l += __shfl_xor(st[qt].l, 32, 64);
        st[qt].w += __shfl_xor(st[qt].w, 32, 64);
        if (h == 0) reinterpret_cast<Stat16*>(s_tiles[wave])[32 * qt + c] = st[qt];
    }
    lds_barrier();
    if (tid < kM16Group && q0 + tid < ub) {
        Stat16 tot = reinterpret_cast<const Stat16*>(s_tiles[0])[tid];
#pragma unroll
        for (int k = 1; k < kB16Waves; ++k) tot = stat_merge(tot, reinterpret_cast<const Stat16*>(s_tiles[k])[tid]);
        P.stat[((size_t)head * P.S1 + split) * P.u_stride + q0 + tid] = tot;
    }
}

// The key splits' statistics of kept query t together, by 4 adjacent threads (`sub` 0 .. 3), which all get (log2 sum exp, and
// c* + D' as the sum of two floats, since its own last bit would count); an absent entry has no weight on any key.
__device__ __forceinline__ float4 stat_of(const Bwd16Params& P, int head, int t, int row, int sub)
{
    if (row < 0) return make_float4(INFINITY, 0.f, 0.f, 0.f);
    const Stat16* sp = P.stat + (size_t)head * P.S1 * P.u_stride + t;
    Stat16 st{-INFINITY, 0.f, 0.0, 0.0};
#pragma unroll 4
    for (int s = sub; s < P.S1; s += 4) st = stat_merge(st, sp[(size_t)s * P.u_stride]);
#pragma unroll
    for (int off = 1; off < 4; off <<= 1) {                          // (both threads of a pair merge the same two in the same order)
        const Stat16 o{__shfl_xor(st.m, off, 64), __shfl_xor(st.c, off, 64), __shfl_xor(st.l, off, 64), __shfl_xor(st.w, off, 64)};
        st = (sub & off) ? stat_merge(o, st) : stat_merge(st, o);
    }
    const double ref = (double)st.c + st.w / st.l;
    return make_float4(st.m + log2f((float)st.l), (float)ref, (float)(ref - (double)(float)ref), 0.f);
}

// ---- dQ of 32 kept queries over the keys of one split: four key streams, added up in wave order through LDS
__device__ __forceinline__ void bwd16_queries(const Bwd16Params& P, uint16_t* s_rows, float* s_out, float4* s_stat)
{
    const int tiles_q = (P.u_stride + 31) >> 5;
    int head, x;
    head_of(blockIdx.x, P.BH, tiles_q * P.SQ, head, x);
    const int split = x / tiles_q, q0 = 32 * (x % tiles_q);
    const int n = valid_len(P.lengths, head / P.H, P.L);
    const int ub = kept_count(P, head / P.H, n);
    if (q0 >= ub) return;                                            // work-group-uniform
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), c = lane & 31, h = lane >> 5;
    const size_t base = (size_t)head * P.L * kD;
    const __amdgpu_buffer_rsrc_t Kr = head_rows<128>(P.K + base, n), Vr = head_rows<128>(P.V + base, n);
    const int t_all = (n + 31) >> 5;
    int t = split * P.tilesq + wave;
    const int t_end = (split + 1) * P.tilesq < t_all ? (split + 1) * P.tilesq : t_all;
    uint4 kx[4], vx[4], qreg[4], greg[4];
    load_rows(kx, Kr, t < t_end, 32 * t, lane);
    load_rows(vx, Vr, t < t_end, 32 * t, lane);
    {
        const int row = kept_row(P, head, q0 + c, n, ub);
        load_half_row(qreg, head_rows<128>(P.Q + base, n), row, h);
        load_half_row(greg, head_rows<128>(P.G + base, n), row, h);
    }
    if (tid < 128) {
        const int k = q0 + (tid >> 2);
        const float4 y = stat_of(P, head, k, kept_row(P, head, k, n, ub), tid & 3);
        if ((tid & 3) == 0) s_stat[tid >> 2] = y;
    }
    lds_barrier();
    const float4 sy = s_stat[c];
    // element 32 dt + 8 (r / 4) + 4h + r % 4 of query c
    floatx16 A[2] = {zero16(), zero16()};
    uint16_t* sK = s_rows + wave * 32 * kB16Stride;
    uint16_t* sV = reinterpret_cast<uint16_t*>(s_out) + wave * 32 * kB16Stride;
#pragma unroll 1
    for (; t < t_end; t += kM16Waves) {                              // wave-uniform
        const int j0 = 32 * t;
        wave_lds_sync();                                             // the tiles before have been read
        put_rows(kx, sK, lane);
        put_rows(vx, sV, lane);
        load_rows(kx, Kr, t + kM16Waves < t_end, j0 + kM16Keys, lane);
        load_rows(vx, Vr, t + kM16Waves < t_end, j0 + kM16Keys, lane);
        wave_lds_sync();
        uint4 ka[4], va[4];
        get_operand(ka, sK, c, h);
        get_operand(va, sV, c, h);
        floatx16 s = zero16(), cc = zero16();
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) { s = mfma16(ka[kk], qreg[kk], s); cc = mfma16(va[kk], greg[kk], cc); }
        if (j0 + 32 > n) {                                           // wave-uniform: the item's last keys
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = j0 + 8 * (r >> 2) + 4 * h + (r & 3) < n ? s[r] : -INFINITY;
        }
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2) {
            uint4 pg[3];
            float g8[8];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                g8[e] = fast_exp2(fmaf(s[8 * k2 + e], kScaleLog2e, -sy.x)) * ((cc[8 * k2 + e] - sy.y) - sy.z);
            planes3(g8, pg);
#pragma unroll
            for (int dt = 0; dt < 2; ++dt) {
                const uint4 kt = transposed(sK, k2, dt, c, h);
#pragma unroll
                for (int k = 0; k < 3; ++k) A[dt] = mfma16(kt, pg[k], A[dt]);
            }
        }
    }
    lds_barrier();                                                   // every wave's V tile has been read
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<float4*>(s_out + (wave * 32 + c) * kRowF + 32 * dt + 8 * q + 4 * h) =
                make_float4(A[dt][4 * q], A[dt][4 * q + 1], A[dt][4 * q + 2], A[dt][4 * q + 3]);
    lds_barrier();
    const int e0 = 8 * (tid & 7), k = q0 + (tid >> 3);               // 8 threads a query
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = 0.f;
#pragma unroll
    for (int w = 0; w < kM16Waves; ++w) {
        const float* p = s_out + (w * 32 + (tid >> 3)) * kRowF + e0;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += p[e];
    }
    if (k >= ub) return;
    if (P.SQ > 1) {
        float4* dst = reinterpret_cast<float4*>(P.dq_part + (((size_t)head * P.SQ + split) * P.u_stride + k) * kD + e0);
        dst[0] = make_float4(v[0], v[1], v[2], v[3]);
        dst[1] = make_float4(v[4], v[5], v[6], v[7]);
    } else {
        const int row = kept_row(P, head, k, n, ub);
        if (row >= 0)
            *reinterpret_cast<uint4*>(P.dQ + base + (size_t)row * kD + e0) =
                make_uint4(cvt_pk_bf16(0.125f * v[0], 0.125f * v[1]), cvt_pk_bf16(0.125f * v[2], 0.125f * v[3]),
                           cvt_pk_bf16(0.125f * v[4], 0.125f * v[5]), cvt_pk_bf16(0.125f * v[6], 0.125f * v[7]));
    }
}

// ---- dK, dV and the rest.  A work-group takes blocks2 blocks of 128 keys, 32 to a wave; the kept queries pass through LDS
// in groups of 64 (once for all blocks where there is one group).
__device__ __forceinline__ void bwd16_keys(const Bwd16Params& P, uint16_t* s_rows, float* s_outs, float* s_lse, float* s_ref, float* s_gm, unsigned* s_bits)
{
    uint16_t* sQ = s_rows;
    uint16_t* sG = s_rows + kM16Group * kB16Stride;
    int head, x;
    head_of(blockIdx.x - P.n_dq, P.BH, P.S2, head, x);
    const int b = head / P.H, L = P.L;
    const int n = valid_len(P.lengths, b, L);
    const int ub = kept_count(P, b, n);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), c = lane & 31, h = lane >> 5;
    const size_t base = (size_t)head * L * kD;
    const __amdgpu_buffer_rsrc_t Kr = head_rows<128>(P.K + base, n), Vr = head_rows<128>(P.V + base, n);
    const __amdgpu_buffer_rsrc_t Qr = head_rows<128>(P.Q + base, n), Gr = head_rows<128>(P.G + base, n);
    const int r_first = x * P.blocks2 * kM16Keys;

    // kept queries q0 .. q0 + 63: their rows of Q and G (4 threads a row, 32 bytes each) and their statistics (the key splits' by 4 threads)
    uint4 rq[2], rg[2];
    float4 st4;
    auto request = [&](int q0) {
        const int row = kept_row(P, head, q0 + (tid >> 2), n, ub);
        const int ofs = row < 0 ? -32 : row * 128 + 32 * (tid & 3);
#pragma unroll
        for (int k = 0; k < 2; ++k) { rq[k] = buffer_load16<uint4>(Qr, ofs + (row < 0 ? 0 : 16 * k)); rg[k] = buffer_load16<uint4>(Gr, ofs + (row < 0 ? 0 : 16 * k)); }
        st4 = stat_of(P, head, q0 + (tid >> 2), row, tid & 3);
    };
    auto put = [&]() {
        const int row = tid >> 2, part = tid & 3;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            *reinterpret_cast<uint4*>(sQ + row * kB16Stride + 16 * part + 8 * k) = rq[k];
            *reinterpret_cast<uint4*>(sG + row * kB16Stride + 16 * part + 8 * k) = rg[k];
        }
        if (part == 0) { s_lse[row] = st4.x; s_ref[row] = st4.y; s_ref[kM16Group + row] = st4.z; }
    };
    const bool any = ub > 0 && r_first < n;                          // work-group-uniform
    if (any) request(0);
    uint4 ka[4], va[4];
    float* so = s_outs + wave * 32 * kRowF;
    uint4 kn[4], vn[4];
    load_rows(kn, Kr, true, r_first + 32 * wave, lane);
    load_rows(vn, Vr, true, r_first + 32 * wave, lane);
    if (tid < kD) {
        // the mean fill's share of dV: every valid v_j receives 1/n of each filled row's gradient
        double s = 0.0;
        if (P.fill == PSA_FILL_MEAN && n > 0) {
            const int parts = P.S1 * P.n_group;
            const double* gs = P.gsum_part + (size_t)head * parts * kD + tid;
#pragma unroll 8
            for (int k = 0; k < parts; ++k) s += gs[(size_t)k * kD];  // fixed order
            s /= (double)n;
        }
        s_gm[tid] = (float)s;
    }
    if (any) put();
    to_operands(kn, vn, reinterpret_cast<uint16_t*>(so), ka, va, lane);
    const bool one_group = ub <= kM16Group;

#pragma unroll 1
    for (int blk = 0; blk < P.blocks2; ++blk) {
        const int r0 = r_first + blk * kM16Keys, j0 = r0 + 32 * wave;
        if (r0 >= L) break;                                          // work-group-uniform
        if ((blk * kM16Keys) % kBitRows == 0) {
            // mark the kept rows among the next 2048 (the barrier also covers what was staged)
            lds_barrier();
            if (tid < kBitRows / 32) s_bits[tid] = 0u;
            lds_barrier();
            for (int k = tid; k < ub; k += kM16Threads) {
                const int i = P.sel[(size_t)head * P.u_stride + k] - r0;
                if (i >= 0 && i < kBitRows && r0 + i < n) atomicOr(&s_bits[i >> 5], 1u << (i & 31));
            }
            lds_barrier();
        }
        // element 32 dt + 8 (r / 4) + 4h + r % 4 of key j0 + c
        load_rows(kn, Kr, blk + 1 < P.blocks2, j0 + kM16Keys, lane);
        load_rows(vn, Vr, blk + 1 < P.blocks2, j0 + kM16Keys, lane);
        floatx16 dk[2] = {zero16(), zero16()}, dv[2] = {zero16(), zero16()};
        if (r0 < n) {                                                // work-group-uniform
#pragma unroll 1
            for (int q0 = 0; q0 < ub; q0 += kM16Group) {              // work-group-uniform
                const bool more = !one_group && (q0 + kM16Group < ub || (blk + 1 < P.blocks2 && r0 + kM16Keys < n));
                if (more) request(q0 + kM16Group < ub ? q0 + kM16Group : 0);
                if (j0 < n) {                                        // wave-uniform: some key of the wave is valid
#pragma unroll 1
                    for (int tt = 0; tt < 2; ++tt) {
                        if (q0 + 32 * tt >= ub) break;               // wave-uniform
                        const uint16_t* tq = sQ + 32 * tt * kB16Stride;
                        const uint16_t* tg = sG + 32 * tt * kB16Stride;
                        floatx16 s = zero16(), cc = zero16();
#pragma unroll
                        for (int kk = 0; kk < 4; ++kk) {
                            s = mfma16(*reinterpret_cast<const uint4*>(tq + c * kB16Stride + 32 * h + 8 * kk), ka[kk], s);
                            cc = mfma16(*reinterpret_cast<const uint4*>(tg + c * kB16Stride + 32 * h + 8 * kk), va[kk], cc);
                        }
                        // the tile's queries 16 k2 .. + 15, which are rows 8 k2 .. + 7 of the accumulators
                        auto half_tile = [&](int k2) {
                            float e8[8], g8[8];
#pragma unroll
                            for (int q = 0; q < 2; ++q) {            // queries 32 tt + 16 k2 + 8q + 4h + e against key c
                                const int at = 32 * tt + 16 * k2 + 8 * q + 4 * h;
                                const float4 l4 = *reinterpret_cast<const float4*>(s_lse + at), c4 = *reinterpret_cast<const float4*>(s_ref + at),
                                             r4 = *reinterpret_cast<const float4*>(s_ref + kM16Group + at);
                                const float le[4] = {l4.x, l4.y, l4.z, l4.w}, ce[4] = {c4.x, c4.y, c4.z, c4.w}, re[4] = {r4.x, r4.y, r4.z, r4.w};
#pragma unroll
                                for (int e = 0; e < 4; ++e) {
                                    e8[4 * q + e] = fast_exp2(fmaf(s[8 * k2 + 4 * q + e], kScaleLog2e, -le[e]));
                                    g8[4 * q + e] = e8[4 * q + e] * ((cc[8 * k2 + 4 * q + e] - ce[e]) - re[e]);
                                }
                            }
                            uint4 pp[3], pg[3];
                            planes3(e8, pp);
                            planes3(g8, pg);
#pragma unroll
                            for (int dt = 0; dt < 2; ++dt) {
                                const uint4 gt = transposed(tg, k2, dt, c, h), qx = transposed(tq, k2, dt, c, h);
#pragma unroll
                                for (int k = 0; k < 3; ++k) { dv[dt] = mfma16(gt, pp[k], dv[dt]); dk[dt] = mfma16(qx, pg[k], dk[dt]); }
                            }
                        };
                        half_tile(0);
                        if (q0 + 32 * tt + 16 < ub) half_tile(1);    // wave-uniform
                    }
                }
                if (!one_group) {
                    lds_barrier();                                   // every wave is done with the staged queries
                    if (more) put();
                    lds_barrier();
                }
            }
        }
        // Rows of dK and dV, and zero rows of dQ outside I_sparse: through LDS, so that a store instruction writes whole rows
        // The next block's key rows have had this block's time to arrive; waiting for them here and not where they are used,
        // behind the stores, keeps the next block from waiting for those
        __builtin_amdgcn_s_waitcnt(0x0F70);                          // vmcnt(0)
        to_operands(kn, vn, reinterpret_cast<uint16_t*>(so), ka, va, lane);
        const int bit0 = (j0 - r_first) % kBitRows;                  // (a multiple of 32)
        const unsigned bits = s_bits[bit0 >> 5];                     // kept rows among the wave's 32 (none at or beyond n)
        const int e0 = 8 * (lane & 7);
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            wave_lds_sync();                                         // the rows before have been read
#pragma unroll
            for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const floatx16& y = half == 0 ? dk[dt] : dv[dt];
                    const float sc = half == 0 ? 0.125f : 1.f;
                    *reinterpret_cast<float4*>(so + c * kRowF + 32 * dt + 8 * q + 4 * h) =
                        make_float4(sc * y[4 * q], sc * y[4 * q + 1], sc * y[4 * q + 2], sc * y[4 * q + 3]);
                }
            wave_lds_sync();
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int row = 8 * it + (lane >> 3), j = j0 + row;
                const float4 lo = *reinterpret_cast<const float4*>(so + row * kRowF + e0), hi = *reinterpret_cast<const float4*>(so + row * kRowF + e0 + 4);
                float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
                const bool kept = (bits >> row) & 1u;
                if (half == 1 && P.fill == PSA_FILL_MEAN) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] += s_gm[e0 + e];
                }
                if (half == 1 && P.fill != PSA_FILL_MEAN && !kept) { // the value fill hands v_j the gradient of its own row
                    const uint4 g = buffer_load16<uint4>(Gr, j * 128 + 2 * e0);
                    const uint32_t w[4] = {g.x, g.y, g.z, g.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) { v[2 * e] += bf16_lo(w[e]); v[2 * e + 1] += bf16_hi(w[e]); }
                }
                if (j < L) {
                    const uint4 z = make_uint4(0u, 0u, 0u, 0u);
                    const uint4 o = j < n ? make_uint4(cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]), cvt_pk_bf16(v[4], v[5]), cvt_pk_bf16(v[6], v[7])) : z;
                    *reinterpret_cast<uint4*>((half == 0 ? P.dK : P.dV) + base + (size_t)j * kD + e0) = o;
                    if (half == 0 && !kept) *reinterpret_cast<uint4*>(P.dQ + base + (size_t)j * kD + e0) = z;
                }
            }
        }
    }
}

__global__ __launch_bounds__(kM16Threads, 2)
void bwd16_main_kernel(const Bwd16Params P)
{
    __shared__ __attribute__((aligned(16))) uint16_t s_rows[2 * kM16Group * kB16Stride];     // staged rows of Q and G, or the waves' K tiles
    __shared__ __attribute__((aligned(16))) float s_out[kM16Waves * 32 * kRowF];
    __shared__ float4 s_stat[kM16Group];                             // dQ: (log2 sum exp, c* + D' in two floats); keys: three arrays of floats
    __shared__ float s_gm[kD];
    __shared__ unsigned s_bits[kBitRows / 32];
    static_assert(kM16Waves * 32 <= 2 * kM16Group, "the waves' K tiles");
    if ((int)blockIdx.x < P.n_dq) bwd16_queries(P, s_rows, s_out, s_stat);                   // (the longer ones first)
    else                          bwd16_keys(P, s_rows, s_out, reinterpret_cast<float*>(s_stat), reinterpret_cast<float*>(s_stat) + kM16Group, s_gm, s_bits);
}

// ---- the key splits of dQ, in split order; 8 threads a query
__global__ __launch_bounds__(256)
void bwd16_reduce_kernel(const Bwd16Params P)
{
    const int per_head = (P.u_stride + 31) >> 5, head = blockIdx.x / per_head;
    const int n = valid_len(P.lengths, head / P.H, P.L);
    const int ub = kept_count(P, head / P.H, n);
    const int k = 32 * (blockIdx.x % per_head) + ((int)threadIdx.x >> 3), e0 = 8 * (threadIdx.x & 7);
    const int row = kept_row(P, head, k, n, ub);
    if (row < 0) return;
    const float* p = P.dq_part + ((size_t)head * P.SQ * P.u_stride + k) * kD + e0;
    const size_t step = (size_t)P.u_stride * kD;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = 0.f;
#pragma unroll 8
    for (int s = 0; s < P.SQ; ++s) {
        const float4 a = *reinterpret_cast<const float4*>(p + s * step), b = *reinterpret_cast<const float4*>(p + s * step + 4);
        v[0] += a.x; v[1] += a.y; v[2] += a.z; v[3] += a.w; v[4] += b.x; v[5] += b.y; v[6] += b.z; v[7] += b.w;
    }
    *reinterpret_cast<uint4*>(P.dQ + ((size_t)head * P.L + row) * kD + e0) =
        make_uint4(cvt_pk_bf16(0.125f * v[0], 0.125f * v[1]), cvt_pk_bf16(0.125f * v[2], 0.125f * v[3]),
                   cvt_pk_bf16(0.125f * v[4], 0.125f * v[5]), cvt_pk_bf16(0.125f * v[6], 0.125f * v[7]));
}

// Key splits and blocks per work-group, and where the scratch lies, within `room` bytes (what make_bwd_plan has given such
// calls since before these kernels: they need less).
Bwd16Plan make_bwd16_plan(const psa_shape_t& s, int u_stride, size_t room)
{
    Bwd16Plan p;
    const int64_t BH = (int64_t)s.B * s.H;
    p.n_group = (u_stride + kM16Group - 1) / kM16Group;
    const int tiles = (s.L_K + 31) / 32, tiles_q = (u_stride + 31) / 32;
    auto clamp = [](int64_t x, int64_t most) { x = x > most ? most : x; return x > 64 ? 64 : (x < 1 ? 1 : x); };
    // statistics: one work-group per CU, every key stream with a tile of its own
    int64_t S1 = clamp(256 / (BH * p.n_group), tiles / kB16Waves);
    // dQ: a quarter of the main kernel's places (two work-groups per CU), every key stream with two tiles; one split needs no
    // partial sums and no third launch
    int64_t SQ = clamp(128 / (BH * tiles_q), tiles / (2 * kM16Waves));
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    for (;;) {
        p.tiles1 = (int)((tiles + S1 - 1) / S1); p.S1 = (tiles + p.tiles1 - 1) / p.tiles1;
        p.tilesq = (int)((tiles + SQ - 1) / SQ); p.SQ = (tiles + p.tilesq - 1) / p.tilesq;
        size_t off = 0;
        p.off_stat = off; off += al((size_t)BH * p.S1 * u_stride * sizeof(Stat16));
        p.off_gsum = off; off += al((size_t)BH * p.S1 * p.n_group * kD * sizeof(double));
        p.off_dq = off;   off += p.SQ > 1 ? al((size_t)BH * p.SQ * u_stride * kD * sizeof(float)) : 0;
        p.total = off;
        if (off <= room || (S1 == 1 && SQ == 1)) break;
        if (SQ > 1) --SQ; else --S1;
    }
    p.n_dq = (int)(BH * tiles_q * p.SQ);
    const int nb = (s.L_K + kM16Keys - 1) / kM16Keys;
    const int64_t room_keys = 512 - (p.n_dq < 256 ? p.n_dq : 256);   // two work-groups per CU: one round with those for dQ
    const int64_t per = (BH * nb + room_keys - 1) / room_keys;
    p.blocks2 = (int)(per < 1 ? 1 : (per > nb ? nb : per));
    p.S2 = (nb + p.blocks2 - 1) / p.blocks2;
    return p;
}

hipError_t launch_backward_bf16(const psa_shape_t& s, const Bwd16Plan& bp, const void* Q, const void* K, const void* V,
                                const int* lengths, const int* sel, const int* u, int u_stride, int fill, const void* G,
                                void* dQ, void* dK, void* dV, void* workspace, hipStream_t stream)
{
    unsigned char* w = static_cast<unsigned char*>(workspace);
    Bwd16Params P;
    P.Q = static_cast<const bf16_t*>(Q); P.K = static_cast<const bf16_t*>(K);
    P.V = static_cast<const bf16_t*>(V); P.G = static_cast<const bf16_t*>(G);
    P.lengths = lengths; P.sel = sel; P.u = u;
    P.dQ = static_cast<bf16_t*>(dQ); P.dK = static_cast<bf16_t*>(dK); P.dV = static_cast<bf16_t*>(dV);
    P.stat = reinterpret_cast<Stat16*>(w + bp.off_stat);
    P.gsum_part = reinterpret_cast<double*>(w + bp.off_gsum);
    P.dq_part = reinterpret_cast<float*>(w + bp.off_dq);
    P.H = s.H; P.L = s.L_K; P.BH = s.B * s.H; P.u_stride = u_stride; P.n_group = bp.n_group;
    P.S1 = bp.S1; P.tiles1 = bp.tiles1; P.SQ = bp.SQ; P.tilesq = bp.tilesq; P.S2 = bp.S2; P.blocks2 = bp.blocks2;
    P.fill = fill; P.n_dq = bp.n_dq;
    const dim3 grid1(P.BH * P.S1 * P.n_group);
    hipLaunchKernelGGL(bwd16_stats_kernel, grid1, dim3(kB16Threads), 0, stream, P);
    hipLaunchKernelGGL(bwd16_main_kernel, dim3(P.n_dq + P.BH * P.S2), dim3(kM16Threads), 0, stream, P);
    if (P.SQ > 1) hipLaunchKernelGGL(bwd16_reduce_kernel, dim3(P.BH * ((u_stride + 31) / 32)), dim3(256), 0, stream, P);
    return hipGetLastError();
}

}  // namespace psa
