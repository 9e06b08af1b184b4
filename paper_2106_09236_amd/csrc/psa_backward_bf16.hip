// Gradients of stages a3 and a4 for bfloat16 tensors (what they are: psa_backward.hip), on the bfloat16 matrix cores.
//   bwd16_stats_kernel    softmax statistics per kept query and key split; column sums of dOut over the filled rows
//   bwd16_main_kernel     work-groups of two kinds: some take 32 kept queries and walk keys (dQ), the others take 128 keys and
//                         walk the kept queries (dK, dV, the fill's share, zero rows)
//   bwd16_reduce_kernel   adds the partial sums of dQ, where the keys of a head were split among work-groups
//
// Arithmetic: float32, for heads that it carries (below).  Products of two bfloat16 values are exact in the MFMA's float32 accumulator; a float32
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
// Heads that float32 does not carry (scores beyond 2^10, rows of K or V with much more in common than they differ, infinities, extreme
// scales; needs_float64) are found by the statistics kernel as it goes, at no measurable cost, and computed in float64 by branches of
// the same two kernels.  With all heads like that: B=8 H=8 L=2048, 39 kept 226 us; B=16 H=4 L=512, 256 kept 210; B=1 H=8 L=16384,
// 49 kept 266 (138, 162 and 181 by the float64 kernels of float32 tensors, made for bfloat16).
//
// MFMA lanes: psa_tile.h.  Scores are formed with the kept queries on the columns where queries are walked over keys, with
// the keys on the columns in the other kind; either way the accumulator registers are, unchanged, the B operand of the
// products that follow.
#include <type_traits>

#include "psa_backward_common.h"
#include "psa_tile.h"

namespace psa {

constexpr int kB16Threads = 512, kB16Waves = kB16Threads / 64;   // statistics: 8 waves
constexpr int kM16Threads = 256, kM16Waves = kM16Threads / 64;   // main kernel: 4 waves of up to 256 registers, two work-groups per CU
constexpr int kM16Keys = 32 * kM16Waves;                         // keys per block
constexpr int kM16Group = 64;                                    // kept queries staged in LDS at a time
constexpr int kRowF = kD + 4;                                    // floats between staged float rows
constexpr int kBitRows = 2048;                                   // rows per bit mask of kept rows

// Softmax statistics of one kept query over some keys while a wave walks them, relative to maximum m (base 2) and reference c*.
// l and w are float64 between tiles and from there on: an error of D' is an error of the sum of a query's g, which multiplies what
// its keys have in common (mixtures of 32 centres, 16384 keys: float32 sums 5 times the error of dQ there).
struct Run16 { float m, c; double l, w; };
// ... and as they are kept: relative to maximum m, l = sum e, w = sum e c (float64 needs no reference); in memory l is negative where
// the work-group asks for float64 (below)
struct Stat16 { double m, l, w; };
constexpr double kNoMax16 = -1e300;                                  // the maximum over no key: finite, so that differences stay numbers
// (EXACT: a maximum of float64 scores; else it is a float32 number, or none)
template <bool EXACT>
__device__ __forceinline__ double stat_factor(double m, double M) { return EXACT ? exp2_f64(m - M) : (double)fast_exp2((float)(m - M)); }
template <bool EXACT>
__device__ __forceinline__ Stat16 stat_merge(const Stat16& a, const Stat16& b)
{
    Stat16 t;
    t.m = fmax(a.m, b.m);
    const double fa = stat_factor<EXACT>(a.m, t.m), fb = stat_factor<EXACT>(b.m, t.m);
    t.l = fa * a.l + fb * b.l;
    t.w = fa * a.w + fb * b.w;
    return t;
}

struct Bwd16Params {
    const bf16_t* Q; const bf16_t* K; const bf16_t* V; const bf16_t* G;
    const int* lengths; const int* sel; const int* u;
    bf16_t* dQ; bf16_t* dK; bf16_t* dV;
    Stat16* stat;          // [BH][S1][u_stride]  per kept query and key split
    double* gsum_part;     // [BH][S1 n_group][64]  column sums of G over valid rows outside I_sparse
    double* dq_part;       // [BH][SQ][u_stride][64]  dQ of the key splits (SQ > 1)
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

// ---- Heads that float32 does not carry.  A float32 score's error grows with the score (of 1e5: 1 % of the weight), that of c with
// what the rows of V have in common beside their differences, that of dQ with the same in K; a zero plane of a weight times an
// infinite dOut is NaN.  So a work-group of the statistics kernel keeps the largest squared norms of the rows it reads and, of its
// waves' first tiles, the widest range of a query's scores and of its c over four keys (Seen16).  What fails needs_float64 is computed in
// float64 by the functions named exact_... on the float64 matrix cores, in the same launches: the statistics by the work-group itself, the
// gradients for the whole head.  Measured of this look: comparisons of whole rows with a tile's first, and maxima over all lanes of every
// wave at the end, cost 0.8 to 1.4 us of a call; four keys of a lane, and maxima kept by lane in LDS and put together by one wave each
// while another merges the streams, are within the noise (B=1 H=4 L=128 14.3 -> 14.2 us, B=8 H=8 L=2048 40.3 -> 40.3).
struct Seen16 { unsigned q2, g2, k2, v2, s_range, c_range; };        // bits of floats that are not negative, which order like the values (NaN the largest)
constexpr float kMaxNorm2 = 1.2089258e24f;                           // 2^80: no product or sum of the gradients nears the end of float32
constexpr float kMaxScore2 = 1048576.f / (kScaleLog2e * kScaleLog2e);          // |q|^2 |k|^2 of scores up to 2^10, base 2: an error of a weight of 2^-13,
                                                                     // a sixteenth of the last rounding
constexpr float kMinProduct2 = 7.5231638e-37f;                       // 2^-120, of |G|^2 |V|^2 that is not 0: all planes of g lie above the smallest normal number
constexpr float kRangeC = 1.f / 512, kRangeS = 1.f / 256;            // range / product of the norms, 0.1 and more for unrelated rows; the range of c (of the
                                                                     // scores) is at most |G| (|Q|) times the largest distance of two rows of V (K)
__device__ __forceinline__ bool needs_float64(const Seen16& y, bool& same_v, bool& same_k)
{
    const float q2 = __uint_as_float(y.q2), g2 = __uint_as_float(y.g2), k2 = __uint_as_float(y.k2), v2 = __uint_as_float(y.v2),
                s = __uint_as_float(y.s_range), c = __uint_as_float(y.c_range);
    if (!(q2 <= kMaxNorm2 && g2 <= kMaxNorm2 && k2 <= kMaxNorm2 && v2 <= kMaxNorm2 && q2 * k2 <= kMaxScore2)) return true;
    same_v = c == 0.f && v2 > 0.f && g2 > 0.f;                       // no range: fine where all rows are the same, which is to be seen
    same_k = s == 0.f && k2 > 0.f && q2 > 0.f;
    return (g2 * v2 > 0.f && g2 * v2 < kMinProduct2) || (c > 0.f && c < kRangeC * __builtin_amdgcn_sqrtf(g2) * __builtin_amdgcn_sqrtf(v2)) ||
           (s > 0.f && s < kRangeS * __builtin_amdgcn_sqrtf(q2) * __builtin_amdgcn_sqrtf(k2));
}
// squared norm of half a row, on four independent chains
__device__ __forceinline__ float dot_half(const uint4 (&a)[4])
{
    float t[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) t[k] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a[k].x), __builtin_bit_cast(bf16x2, a[k].x), 0.f, false);
#pragma unroll
    for (int k = 0; k < 4; ++k) t[k] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a[k].y), __builtin_bit_cast(bf16x2, a[k].y), t[k], false);
#pragma unroll
    for (int k = 0; k < 4; ++k) t[k] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a[k].z), __builtin_bit_cast(bf16x2, a[k].z), t[k], false);
#pragma unroll
    for (int k = 0; k < 4; ++k) t[k] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a[k].w), __builtin_bit_cast(bf16x2, a[k].w), t[k], false);
    return (t[0] + t[1]) + (t[2] + t[3]);
}
__device__ __forceinline__ float dot_eighth(const uint4& a)
{
    float t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a.x), __builtin_bit_cast(bf16x2, a.x), 0.f, false);
    t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a.y), __builtin_bit_cast(bf16x2, a.y), t, false);
    t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a.z), __builtin_bit_cast(bf16x2, a.z), t, false);
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a.w), __builtin_bit_cast(bf16x2, a.w), t, false);
}
__device__ __forceinline__ unsigned umax(unsigned a, unsigned b) { return a > b ? a : b; }
// maximum over the wave, in every lane
__device__ __forceinline__ unsigned wave_umax(unsigned x)
{
    x = umax(x, __float_as_uint(dpp_mov<0xB1>(__uint_as_float(x))));
    x = umax(x, __float_as_uint(dpp_mov<0x4E>(__uint_as_float(x))));
    x = umax(x, __float_as_uint(dpp_mov<0x141>(__uint_as_float(x))));
    x = umax(x, __float_as_uint(dpp_mov<0x140>(__uint_as_float(x))));
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = umax(r[0], r[1]);
    const auto q = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return umax(q[0], q[1]);
}
// Does any of rows first .. end - 1 differ from row `first`?  Asked of the threads of a work-group, 8 a row; this thread's answer.
__device__ __forceinline__ bool rows_differ(__amdgpu_buffer_rsrc_t rows, int first, int end)
{
    const int part = 16 * ((int)threadIdx.x & 7);
    const uint4 a = buffer_load16<uint4>(rows, first * 128 + part);
    uint32_t bits = 0;
    for (int r = first + ((int)threadIdx.x >> 3); r < end; r += kB16Threads / 8) {
        const uint4 x = buffer_load16<uint4>(rows, r * 128 + part);
        bits |= (x.x ^ a.x) | (x.y ^ a.y) | (x.z ^ a.z) | (x.w ^ a.w);
    }
    return bits != 0u;
}
// float64 products: v_mfma_f64_16x16x4f64, lane (c, g) = (lane % 16, lane / 16): A[i][k]: i = c, k = g   B[k][j]: k = g, j = c
// D[i][j]: i = 4r + g, j = c.  A score product takes elements 16 g .. 16 g + 15 of a row on both sides.
__device__ __forceinline__ doublex4 mfma64(double a, double b, const doublex4& c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
__device__ __forceinline__ void widen8(const uint4& a, double* d)
{
    const uint32_t x[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) { d[2 * k] = (double)bf16_lo(x[k]); d[2 * k + 1] = (double)bf16_hi(x[k]); }
}
__device__ __forceinline__ void widen16(const uint4 (&a)[2], double (&d)[16]) { widen8(a[0], d); widen8(a[1], d + 8); }
__device__ __forceinline__ void load16(uint4 (&x)[2], __amdgpu_buffer_rsrc_t rows, int row, int g)
{
    const int ofs = row < 0 ? -32 : row * 128 + 32 * g;
#pragma unroll
    for (int k = 0; k < 2; ++k) x[k] = buffer_load16<uint4>(rows, ofs + (row < 0 ? 0 : 16 * k));
}
__device__ __forceinline__ void read16(const uint16_t* row, int g, double (&d)[16])
{
    const uint4 x[2] = {*reinterpret_cast<const uint4*>(row + 16 * g), *reinterpret_cast<const uint4*>(row + 16 * g + 8)};
    widen16(x, d);
}
// four elements (8 bytes)
__device__ __forceinline__ void widen4(const uint2& x, double (&d)[4]) {
    d[0] = (double)bf16_lo(x.x); d[1] = (double)bf16_hi(x.x); d[2] = (double)bf16_lo(x.y); d[3] = (double)bf16_hi(x.y);
}
__device__ __forceinline__ uint2 round4(const doublex4& v) {
    return make_uint2(cvt_pk_bf16((float)v[0], (float)v[1]), cvt_pk_bf16((float)v[2], (float)v[3]));
}
__device__ __forceinline__ uint4 round8(const double (&v)[8]) {
    return make_uint4(cvt_pk_bf16((float)v[0], (float)v[1]), cvt_pk_bf16((float)v[2], (float)v[3]),
                      cvt_pk_bf16((float)v[4], (float)v[5]), cvt_pk_bf16((float)v[6], (float)v[7]));
}
// Does any work-group of the statistics ask for float64 in this head?  Wave-uniform, and the same in every wave.  `asked`: the sign of
// what the first 64 of them left, requested ahead.
__device__ __forceinline__ int asked_by(const Bwd16Params& P, int head, int groups, int k)
{
    const Stat16* st = P.stat + ((size_t)head * P.S1 + k / groups) * P.u_stride + k % groups * kM16Group;      // its first query's
    return reinterpret_cast<const int*>(&st->l)[1];
}
__device__ __forceinline__ int first_asked(const Bwd16Params& P, int head, int ub, int lane)
{
    const int groups = ub > 0 ? (ub + kM16Group - 1) / kM16Group : 1;
    return asked_by(P, head, groups, lane < P.S1 * groups ? lane : 0);
}
__device__ __forceinline__ bool head_exact(const Bwd16Params& P, int head, int ub, int lane, int asked)
{
    const int groups = (ub + kM16Group - 1) / kM16Group;
    for (int k = lane + 64; k < P.S1 * groups; k += 64) asked |= asked_by(P, head, groups, k);
    return __ballot(asked < 0) != 0ull;
}
// Statistics of the 64 staged queries over every eighth tile of 16 keys from j0 on, to out[query]: keys on the rows of the score products
__device__ __forceinline__ void exact_stats(const uint16_t* sQ, const uint16_t* sG, __amdgpu_buffer_rsrc_t Kr, __amdgpu_buffer_rsrc_t Vr, int j0,
                                            int j_end, int n_q, int lane, Stat16* out)
{
    const int c = lane & 15, g = lane >> 4;
    Stat16 st[4];
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) st[tt] = Stat16{kNoMax16, 0.0, 0.0};
#pragma unroll 1
    for (; j0 < j_end; j0 += 16 * kB16Waves) {                       // wave-uniform
        uint4 kx[2], vx[2];
        double kd[16], vd[16];
        load16(kx, Kr, j0 + c, g);
        load16(vx, Vr, j0 + c, g);
        widen16(kx, kd);
        widen16(vx, vd);
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            if (16 * tt >= n_q) break;                               // work-group-uniform
            double qd[16], gd[16];
            read16(sQ + (16 * tt + c) * kB16Stride, g, qd);
            read16(sG + (16 * tt + c) * kB16Stride, g, gd);
            doublex4 s = {0.0, 0.0, 0.0, 0.0}, cc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int e = 0; e < 16; ++e) { s = mfma64(kd[e], qd[e], s); cc = mfma64(vd[e], gd[e], cc); }
            Stat16& y = st[tt];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (j0 + 4 * r + g < j_end) {
                    const double x = s[r] * kScaleLog2eD, m = fmax(y.m, x), a = exp2_f64(y.m - m), e = exp2_f64(x - m);
                    y.l = fma(y.l, a, e);
                    y.w = fma(y.w, a, e * cc[r]);
                    y.m = m;
                }
            }
        }
    }
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) {
#pragma unroll
        for (int off = 16; off < 64; off <<= 1) {                    // (both lanes of a pair merge the same two in the same order)
            const Stat16 o{__shfl_xor(st[tt].m, off, 64), __shfl_xor(st[tt].l, off, 64), __shfl_xor(st[tt].w, off, 64)};
            st[tt] = (lane & off) ? stat_merge<true>(o, st[tt]) : stat_merge<true>(st[tt], o);
        }
        if (g == 0) out[16 * tt + c] = st[tt];
    }
}

// (head, index within the head) of work-group `id`: all work-groups of a head on one XCD where the heads divide evenly
__device__ __forceinline__ void head_of(int id, int BH, int per_head, int& head, int& x)
{
    if (BH % 8 == 0) { const int slot = id >> 3; head = slot / per_head * 8 + (id & 7); x = slot % per_head; }
    else             { head = id / per_head; x = id % per_head; }
}

// the waves' statistics of staged query k together, in wave order
template <bool EXACT>
__device__ __forceinline__ Stat16 merged_streams(const uint16_t (*s_tiles)[32 * kB16Stride], int k)
{
    Stat16 x[kB16Waves], t{kNoMax16, 0.0, 0.0};
#pragma unroll
    for (int w = 0; w < kB16Waves; ++w) { x[w] = reinterpret_cast<const Stat16*>(s_tiles[w])[k]; t.m = fmax(t.m, x[w].m); }
#pragma unroll
    for (int w = 0; w < kB16Waves; ++w) {
        const double f = stat_factor<EXACT>(x[w].m, t.m);
        t.l = fma(f, x[w].l, t.l);
        t.w = fma(f, x[w].w, t.w);
    }
    return t;
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
    __shared__ unsigned s_seen[6][64];                               // maxima over the waves, by lane; then over the lanes in column 0
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
    Seen16 seen = {0u, 0u, 0u, 0u, 0u, 0u};                          // (of this lane's rows)
    if (tid < 6 * 64) s_seen[0][tid] = 0u;
    if (any) {
        *reinterpret_cast<uint4*>(sQ + (tid >> 3) * kB16Stride + 8 * (tid & 7)) = xq;
        *reinterpret_cast<uint4*>(sG + (tid >> 3) * kB16Stride + 8 * (tid & 7)) = xg;
        lds_barrier();
        seen.q2 = __float_as_uint(dot_eighth(xq));                   // (an eighth of the row: summed at the end)
        seen.g2 = __float_as_uint(dot_eighth(xg));
    }

    Run16 st[2] = {{-INFINITY, 0.f, 0.0, 0.0}, {-INFINITY, 0.f, 0.0, 0.0}};      // (l and w of this lane's keys)
    auto tile_step = [&](auto first_step, int step) {
        const int j0 = 32 * t;
        uint4 ka[4], va[4];
        to_operands(kx, vx, s_tiles[wave], ka, va, lane);
        seen.k2 = umax(seen.k2, __float_as_uint(dot_half(ka)));      // (half of the row; rows beyond the item are zeros)
        seen.v2 = umax(seen.v2, __float_as_uint(dot_half(va)));
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
            Run16& y = st[qt];
            float tmax = s[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) tmax = fmaxf(tmax, s[r]);
            if (decltype(first_step)::value) {
                // ranges over four of this lane's keys, all of one query
                float s_lo = s[0], s_hi = s[0], c_lo = cc[0], c_hi = cc[0];
#pragma unroll
                for (int r = 1; r < 4; ++r) {
                    const bool ok = j0 + 4 * h + r < n;              // (key r = 0 may be masked as well: then all are)
                    s_lo = fminf(s_lo, ok ? s[r] : s[0]); s_hi = fmaxf(s_hi, ok ? s[r] : s[0]);
                    c_lo = fminf(c_lo, ok ? cc[r] : cc[0]); c_hi = fmaxf(c_hi, ok ? cc[r] : cc[0]);
                }
                seen.s_range = umax(seen.s_range, __float_as_uint(j0 + 4 * h < n ? fmaxf(s_hi - s_lo, 0.f) : 0.f));
                seen.c_range = umax(seen.c_range, __float_as_uint(j0 + 4 * h < n ? fmaxf(c_hi - c_lo, 0.f) : 0.f));
            }
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
                const double a = grow ? (y.m == -INFINITY ? 0.f : fast_exp2(y.m - m_new)) : 1.f;
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
    if (first) { tile_step(std::true_type{}, 0); t += kB16Waves; }

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
    for (int step = 1; t < t_end; t += kB16Waves, ++step) tile_step(std::false_type{}, step);        // wave-uniform
    // the key streams together, in wave order
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
        Run16& y = st[qt];
        y.l += __shfl_xor(y.l, 32, 64);
        y.w += __shfl_xor(y.w, 32, 64);
        if (h == 0) reinterpret_cast<Stat16*>(s_tiles[wave])[32 * qt + c] = Stat16{y.m == -INFINITY ? kNoMax16 : (double)y.m, y.l, fma((double)y.c, y.l, y.w)};
    }
    {
        // (NaN, which a maximum of floats would drop, is the largest of the bits)
        const unsigned most[6] = {__float_as_uint(group_sum8(__uint_as_float(seen.q2))), __float_as_uint(group_sum8(__uint_as_float(seen.g2))),
                                  seen.k2, seen.v2, seen.s_range, seen.c_range};
#pragma unroll
        for (int k = 0; k < 6; ++k) atomicMax(&s_seen[k][lane], most[k]);
    }
    lds_barrier();
    // one wave puts the key streams together while others find the maxima
    Stat16* const stat = P.stat + ((size_t)head * P.S1 + split) * P.u_stride + q0;
    if (wave < 6) {
        const unsigned most = wave_umax(s_seen[wave][lane]);
        if (lane == 0) s_seen[wave][0] = most;
    } else if (wave == 7 && q0 + lane < ub) {
        stat[lane] = merged_streams<false>(s_tiles, lane);
    }
    lds_barrier();
    seen = {s_seen[0][0], s_seen[1][0], s_seen[2][0], s_seen[3][0], s_seen[4][0], s_seen[5][0]};
    seen.k2 = __float_as_uint(2.f * __uint_as_float(seen.k2));       // (a row has two halves)
    seen.v2 = __float_as_uint(2.f * __uint_as_float(seen.v2));
    bool same_v = false, same_k = false;
    bool f64 = needs_float64(seen, same_v, same_k);                  // work-group-uniform
    const int j_first = 32 * t_first, j_end = 32 * t_end < n ? 32 * t_end : n;
    if (!f64 && (same_v || same_k))                                  // work-group-uniform
        f64 = __syncthreads_or((same_v && rows_differ(Vr, j_first, j_end)) || (same_k && rows_differ(Kr, j_first, j_end))) != 0;
    if (!f64) return;
    exact_stats(sQ, sG, Kr, Vr, j_first + 16 * wave, j_end, ub - q0, lane, reinterpret_cast<Stat16*>(s_tiles[wave]));
    lds_barrier();
    if (wave == 7 && q0 + lane < ub) {                               // (the same threads as before)
        Stat16 tot = merged_streams<true>(s_tiles, lane);
        tot.l = copysign(tot.l, -1.0);
        stat[lane] = tot;
    }
}

// The key splits' statistics of kept query t together, by 4 adjacent threads (`sub` 0 .. 3), which all get them
template <bool EXACT>
__device__ __forceinline__ Stat16 merged_stat(const Bwd16Params& P, int head, int t, int sub)
{
    const Stat16* sp = P.stat + (size_t)head * P.S1 * P.u_stride + t;
    Stat16 st{kNoMax16, 0.0, 0.0};
#pragma unroll 4
    for (int s = sub; s < P.S1; s += 4) {
        Stat16 x = sp[(size_t)s * P.u_stride];
        x.l = fabs(x.l);
        st = stat_merge<EXACT>(st, x);
    }
#pragma unroll
    for (int off = 1; off < 4; off <<= 1) {                          // (both threads of a pair merge the same two in the same order)
        const Stat16 o{__shfl_xor(st.m, off, 64), __shfl_xor(st.l, off, 64), __shfl_xor(st.w, off, 64)};
        st = (sub & off) ? stat_merge<EXACT>(o, st) : stat_merge<EXACT>(st, o);
    }
    return st;
}
// (log2 sum exp, and D as the sum of two floats, since its own last bit would count); an absent entry has no weight on any key
__device__ __forceinline__ float4 stat_of(const Bwd16Params& P, int head, int t, int row, int sub)
{
    if (row < 0) return make_float4(INFINITY, 0.f, 0.f, 0.f);
    const Stat16 st = merged_stat<false>(P, head, t, sub);
    const double ref = st.w / st.l;
    return make_float4((float)st.m + log2f((float)st.l), (float)ref, (float)(ref - (double)(float)ref), 0.f);
}
// (log2 sum exp, D) in float64
__device__ __forceinline__ double2 exact_stat_of(const Bwd16Params& P, int head, int t, int row, int sub)
{
    if (row < 0) return make_double2(INFINITY, 0.0);
    const Stat16 st = merged_stat<true>(P, head, t, sub);
    return make_double2(st.m + log2(st.l), st.w / st.l);
}

// dQ of kept queries q0 .. q0 + 31 over keys j_first .. j_end - 1 in float64: two waves take the same 16 queries and every other tile of
// 16 keys.  Keys on the rows of the score products, so that a lane's four g are the B operand of the product over keys.
__device__ __forceinline__ void exact_queries(const Bwd16Params& P, int head, int split, int q0, int n, int ub, size_t base, int j_first, int j_end,
                                              __amdgpu_buffer_rsrc_t Kr, __amdgpu_buffer_rsrc_t Vr, double2* s_stat, double* s_acc)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), c = lane & 15, g = lane >> 4;
    const int qt = 16 * (wave & 1), stream = wave >> 1;
    double qd[16], gd[16];
    {
        const int row = kept_row(P, head, q0 + qt + c, n, ub);
        uint4 x[2], y[2];
        load16(x, head_rows<128>(P.Q + base, n), row, g);
        load16(y, head_rows<128>(P.G + base, n), row, g);
        widen16(x, qd);
        widen16(y, gd);
    }
    if (tid < 128) {
        const int k = q0 + (tid >> 2);
        const double2 y = exact_stat_of(P, head, k, kept_row(P, head, k, n, ub), tid & 3);
        if ((tid & 3) == 0) s_stat[tid >> 2] = y;
    }
    lds_barrier();
    const double2 st = s_stat[qt + c];
    doublex4 acc[4];                                              // acc[dt][r]: element 4 (4r + g) + dt of query c
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) acc[dt] = doublex4{0.0, 0.0, 0.0, 0.0};
    uint4 kx[2], vx[2];
    uint2 k4[4];                                                     // elements 4c .. 4c + 3 of keys 4r + g
    auto request = [&](int j0) {
        load16(kx, Kr, j0 + c, g);
        load16(vx, Vr, j0 + c, g);
#pragma unroll
        for (int r = 0; r < 4; ++r) k4[r] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(Kr, (j0 + 4 * r + g) * 128 + 8 * c, 0, 0));
    };
    request(j_first + 16 * stream);                                  // (rows beyond the item are zeros)
#pragma unroll 1
    for (int j0 = j_first + 16 * stream; j0 < j_end; j0 += 32) {     // wave-uniform
        double kd[16], vd[16], ka[4][4];
        widen16(kx, kd);
        widen16(vx, vd);
#pragma unroll
        for (int r = 0; r < 4; ++r) widen4(k4[r], ka[r]);
        request(j0 + 32);
        doublex4 s = {0.0, 0.0, 0.0, 0.0}, cc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < 16; ++e) { s = mfma64(kd[e], qd[e], s); cc = mfma64(vd[e], gd[e], cc); }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const double p = exp2_f64(fma(s[r], kScaleLog2eD, -st.x)), gv = j0 + 4 * r + g < j_end ? p * (cc[r] - st.y) : 0.0;
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) acc[dt] = mfma64(ka[r][dt], gv, acc[dt]);
        }
    }
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 4; ++r) s_acc[(32 * stream + qt + c) * kD + 16 * r + 4 * g + dt] = acc[dt][r];
    lds_barrier();
    const int e0 = 8 * (tid & 7), k = q0 + (tid >> 3);               // 8 threads a query
    double v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = s_acc[(tid >> 3) * kD + e0 + e] + s_acc[(32 + (tid >> 3)) * kD + e0 + e];
    if (k >= ub) return;
    if (P.SQ > 1) {
        double* const dst = P.dq_part + (((size_t)head * P.SQ + split) * P.u_stride + k) * kD + e0;
#pragma unroll
        for (int e = 0; e < 8; e += 2) *reinterpret_cast<double2*>(dst + e) = make_double2(v[e], v[e + 1]);
    } else {
        const int row = kept_row(P, head, k, n, ub);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] *= 0.125;
        if (row >= 0) *reinterpret_cast<uint4*>(P.dQ + base + (size_t)row * kD + e0) = round8(v);
    }
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
    // (the list entries arrive with the answer, and what follows from both behind the branch: requested before it, the rows
    // would be spilled around the float64 code)
    const int asked = first_asked(P, head, ub, lane), row = kept_row(P, head, q0 + c, n, ub);
    if (head_exact(P, head, ub, lane, asked)) {                          // work-group-uniform
        exact_queries(P, head, split, q0, n, ub, base, 32 * split * P.tilesq, 32 * t_end < n ? 32 * t_end : n, Kr, Vr, reinterpret_cast<double2*>(s_stat),
                      reinterpret_cast<double*>(s_out));
        return;
    }
    load_half_row(qreg, head_rows<128>(P.Q + base, n), row, h);
    load_half_row(greg, head_rows<128>(P.G + base, n), row, h);
    load_rows(kx, Kr, t < t_end, 32 * t, lane);
    load_rows(vx, Vr, t < t_end, 32 * t, lane);
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
        double* const dst = P.dq_part + (((size_t)head * P.SQ + split) * P.u_stride + k) * kD + e0;
#pragma unroll
        for (int e = 0; e < 8; e += 2) *reinterpret_cast<double2*>(dst + e) = make_double2((double)v[e], (double)v[e + 1]);
    } else {
        const int row = kept_row(P, head, k, n, ub);
        if (row >= 0)
            *reinterpret_cast<uint4*>(P.dQ + base + (size_t)row * kD + e0) =
                make_uint4(cvt_pk_bf16(0.125f * v[0], 0.125f * v[1]), cvt_pk_bf16(0.125f * v[2], 0.125f * v[3]),
                           cvt_pk_bf16(0.125f * v[4], 0.125f * v[5]), cvt_pk_bf16(0.125f * v[6], 0.125f * v[7]));
    }
}

// the mean fill's share of element e of dV: every valid v_j receives 1/n of each filled row's gradient
__device__ __forceinline__ double fill_share(const Bwd16Params& P, int head, int n, int e)
{
    double s = 0.0;
    if (P.fill != PSA_FILL_MEAN || n <= 0) return s;
    const int parts = P.S1 * P.n_group;
    const double* gs = P.gsum_part + (size_t)head * parts * kD + e;
#pragma unroll 8
    for (int k = 0; k < parts; ++k) s += gs[(size_t)k * kD];          // fixed order
    return s / (double)n;
}
// marks the kept rows among r0 .. r0 + 2047 (every wave is done with the marks before, and sees these)
__device__ __forceinline__ void mark_kept_rows(const Bwd16Params& P, int head, int r0, int n, int ub, unsigned* s_bits)
{
    const int tid = threadIdx.x;
    lds_barrier();
    if (tid < kBitRows / 32) s_bits[tid] = 0u;
    lds_barrier();
    for (int k = tid; k < ub; k += kM16Threads) {
        const int i = P.sel[(size_t)head * P.u_stride + k] - r0;
        if (i >= 0 && i < kBitRows && r0 + i < n) atomicOr(&s_bits[i >> 5], 1u << (i & 31));
    }
    lds_barrier();
}

// dK, dV and zero rows of dQ for keys r_first .. r_end - 1 in float64, 16 keys to a wave at a time.  Queries on the rows of the score
// products, so that a lane's four p and g are the B operands of the products over queries.
__device__ __forceinline__ void exact_keys(const Bwd16Params& P, int head, int n, int ub, size_t base, int r_first, int r_end, __amdgpu_buffer_rsrc_t Kr,
                                           __amdgpu_buffer_rsrc_t Vr, __amdgpu_buffer_rsrc_t Qr, __amdgpu_buffer_rsrc_t Gr, uint16_t* s_rows,
                                           double2* s_stat, double* s_share, unsigned* s_bits)
{
    static_assert(kM16Threads == 4 * kM16Group && kBitRows % (16 * kM16Waves) == 0, "four threads stage a row; a step lies in one bit mask");
    uint16_t* const sQ = s_rows;
    uint16_t* const sG = s_rows + kM16Group * kB16Stride;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), c = lane & 15, g = lane >> 4;
    if (tid < kD) s_share[tid] = fill_share(P, head, n, tid);
#pragma unroll 1
    for (int r0 = r_first; r0 < r_end; r0 += 16 * kM16Waves) {       // work-group-uniform
        if ((r0 - r_first) % kBitRows == 0) mark_kept_rows(P, head, r0, n, ub, s_bits);
        const int j0 = r0 + 16 * wave, j = j0 + c;
        double kd[16], vd[16];
        {
            uint4 kx[2], vx[2];
            load16(kx, Kr, j, g);
            load16(vx, Vr, j, g);
            widen16(kx, kd);
            widen16(vx, vd);
        }
        doublex4 dk[4], dv[4];                                    // [dt][r]: element 4 (4r + g) + dt of key c
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) { dk[dt] = doublex4{0.0, 0.0, 0.0, 0.0}; dv[dt] = doublex4{0.0, 0.0, 0.0, 0.0}; }
#pragma unroll 1
        for (int q0 = 0; q0 < ub && r0 < n; q0 += kM16Group) {       // work-group-uniform
            lds_barrier();                                           // what was staged before has been read
            {
                const int k = tid >> 2, part = tid & 3, row = kept_row(P, head, q0 + k, n, ub), at = row < 0 ? -32 : row * 128 + 32 * part;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    *reinterpret_cast<uint4*>(sQ + k * kB16Stride + 16 * part + 8 * i) = buffer_load16<uint4>(Qr, at + (row < 0 ? 0 : 16 * i));
                    *reinterpret_cast<uint4*>(sG + k * kB16Stride + 16 * part + 8 * i) = buffer_load16<uint4>(Gr, at + (row < 0 ? 0 : 16 * i));
                }
                const double2 st = exact_stat_of(P, head, q0 + k, row, part);
                if (part == 0) s_stat[k] = st;
            }
            lds_barrier();
            if (j0 >= n) continue;                                   // wave-uniform
#pragma unroll 1
            for (int tt = 0; tt < 4; ++tt) {
                if (q0 + 16 * tt >= ub) break;                       // work-group-uniform
                double qd[16], gd[16];
                read16(sQ + (16 * tt + c) * kB16Stride, g, qd);
                read16(sG + (16 * tt + c) * kB16Stride, g, gd);
                doublex4 s = {0.0, 0.0, 0.0, 0.0}, cc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int e = 0; e < 16; ++e) { s = mfma64(qd[e], kd[e], s); cc = mfma64(gd[e], vd[e], cc); }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int k = 16 * tt + 4 * r + g;
                    const double2 st = s_stat[k];
                    const double p = exp2_f64(fma(s[r], kScaleLog2eD, -st.x)), gv = st.x == INFINITY ? 0.0 : p * (cc[r] - st.y);
                    double qa[4], ga[4];                             // elements 4c .. 4c + 3 of query 4r + g
                    widen4(*reinterpret_cast<const uint2*>(sQ + k * kB16Stride + 4 * c), qa);
                    widen4(*reinterpret_cast<const uint2*>(sG + k * kB16Stride + 4 * c), ga);
#pragma unroll
                    for (int dt = 0; dt < 4; ++dt) { dk[dt] = mfma64(qa[dt], gv, dk[dt]); dv[dt] = mfma64(ga[dt], p, dv[dt]); }
                }
            }
        }
        if (j >= P.L) continue;
        const int bit = (j - r_first) % kBitRows;
        const bool kept = (s_bits[bit >> 5] >> (bit & 31)) & 1u;
        double a[4][4], b[4][4];                                     // [r][dt]: elements 16r + 4g + dt
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) { a[r][dt] = 0.125 * dk[dt][r]; b[r][dt] = dv[dt][r] + s_share[16 * r + 4 * g + dt]; }      // (0 under the value fill)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int e0 = 16 * r + 4 * g;
            if (P.fill != PSA_FILL_MEAN && !kept) {                  // the value fill hands v_j the gradient of its own row
                double own[4];
                widen4(__builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(Gr, j * 128 + 2 * e0, 0, 0)), own);
#pragma unroll
                for (int dt = 0; dt < 4; ++dt) b[r][dt] += own[dt];
            }
            const uint2 z = make_uint2(0u, 0u);
            const size_t at = base + (size_t)j * kD + e0;
            *reinterpret_cast<uint2*>(P.dK + at) = j < n ? round4(doublex4{a[r][0], a[r][1], a[r][2], a[r][3]}) : z;
            *reinterpret_cast<uint2*>(P.dV + at) = j < n ? round4(doublex4{b[r][0], b[r][1], b[r][2], b[r][3]}) : z;
            if (!kept) *reinterpret_cast<uint2*>(P.dQ + at) = z;
        }
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
    const bool any = ub > 0 && r_first < n;                          // work-group-uniform
    const int asked = first_asked(P, head, ub, lane), row0 = kept_row(P, head, tid >> 2, n, ub);
    if (any && head_exact(P, head, ub, lane, asked)) {                   // work-group-uniform
        const int r_end = r_first + P.blocks2 * kM16Keys;
        exact_keys(P, head, n, ub, base, r_first, r_end < L ? r_end : L, Kr, Vr, Qr, Gr, s_rows, reinterpret_cast<double2*>(s_lse),
                   reinterpret_cast<double*>(s_outs), s_bits);
        return;
    }

    // kept queries q0 .. q0 + 63: their rows of Q and G (4 threads a row, 32 bytes each) and their statistics (the key splits' by 4 threads)
    uint4 rq[2], rg[2];
    float4 st4;
    auto request = [&](int q0, int row) {
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
    if (any) request(0, row0);
    uint4 ka[4], va[4];
    float* so = s_outs + wave * 32 * kRowF;
    uint4 kn[4], vn[4];
    load_rows(kn, Kr, true, r_first + 32 * wave, lane);
    load_rows(vn, Vr, true, r_first + 32 * wave, lane);
    if (tid < kD) s_gm[tid] = (float)fill_share(P, head, n, tid);
    if (any) put();
    to_operands(kn, vn, reinterpret_cast<uint16_t*>(so), ka, va, lane);
    const bool one_group = ub <= kM16Group;

#pragma unroll 1
    for (int blk = 0; blk < P.blocks2; ++blk) {
        const int r0 = r_first + blk * kM16Keys, j0 = r0 + 32 * wave;
        if (r0 >= L) break;                                          // work-group-uniform
        if ((blk * kM16Keys) % kBitRows == 0) mark_kept_rows(P, head, r0, n, ub, s_bits);     // (its barriers cover what was staged as well)
        // element 32 dt + 8 (r / 4) + 4h + r % 4 of key j0 + c
        load_rows(kn, Kr, blk + 1 < P.blocks2, j0 + kM16Keys, lane);
        load_rows(vn, Vr, blk + 1 < P.blocks2, j0 + kM16Keys, lane);
        floatx16 dk[2] = {zero16(), zero16()}, dv[2] = {zero16(), zero16()};
        if (r0 < n) {                                                // work-group-uniform
#pragma unroll 1
            for (int q0 = 0; q0 < ub; q0 += kM16Group) {              // work-group-uniform
                const bool more = !one_group && (q0 + kM16Group < ub || (blk + 1 < P.blocks2 && r0 + kM16Keys < n));
                if (more) {
                    const int q_next = q0 + kM16Group < ub ? q0 + kM16Group : 0;
                    request(q_next, kept_row(P, head, q_next + (tid >> 2), n, ub));
                }
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
    const double* p = P.dq_part + ((size_t)head * P.SQ * P.u_stride + k) * kD + e0;
    const size_t step = (size_t)P.u_stride * kD;
    double v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = 0.0;
#pragma unroll 8
    for (int s = 0; s < P.SQ; ++s) {
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            const double2 x = *reinterpret_cast<const double2*>(p + s * step + e);
            v[e] += x.x; v[e + 1] += x.y;
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] *= 0.125;
    *reinterpret_cast<uint4*>(P.dQ + ((size_t)head * P.L + row) * kD + e0) = round8(v);
}

// Key splits and blocks per work-group, and where the scratch lies: within `room` bytes (what make_bwd_plan has given such calls since
// before these kernels).
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
        p.off_dq = off;   off += p.SQ > 1 ? al((size_t)BH * p.SQ * u_stride * kD * sizeof(double)) : 0;
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
    P.dq_part = reinterpret_cast<double*>(w + bp.off_dq);
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
