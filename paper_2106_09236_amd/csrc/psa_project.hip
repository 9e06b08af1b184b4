// The projections around the attention path (Sec. 3.1: Q = X W_q, K = X W_k,
// V = X W_v; Sec. 2.2, Eq. 5: the multi-head self-attention module; Sec. 4.2: 4
// heads of 64 dimensions): one GEMM kernel, C[m][n] = sum_k A[m][k] W[n][k] + bias[n],
// with the head split of the projected tensors folded into its addressing, so
// that Q, K, V are produced directly as [B, H, L, 64] and the output matrix reads
// the attention result in that layout: no transposes in memory.
//
// Both operands have the contraction index contiguous (W is stored [d_out, d_in]),
// which is the layout the MFMA operands want.  A work-group of 4 waves computes a
// 128 x 128 tile of C, each wave a 64 x 64 quarter as 2 x 2 MFMA tiles of 32 x 32
// (128 x 64 with 2 x 1 MFMA tiles per wave, or 64 x 64, for shapes that would
// otherwise leave compute units without work).  The products are taken as C^T = W A^T (rows of W on
// the MFMA row axis), so that a lane ends up with one row of C and runs of four
// consecutive columns:
//   v_mfma_f32_32x32x16_bf16, lane (c, h) = (lane % 32, lane / 32):
//   A[i = c][k = 8h + e], B[k = 8h + e][j = c], D[i = 8(r/4) + 4h + r%4][j = c]
// The contraction runs in chunks (64 bfloat16 / 32 float32 elements) through LDS,
// the next chunk's global loads in flight during the current chunk's products.
// bfloat16 tensors: project_kernel.  float32 tensors: project_split_kernel, which
// runs on the same bfloat16 MFMA with every operand split into three bfloat16 parts.
#include <type_traits>

#include "psa_device.h"
#include "psa_internal.h"
#include "psa_trace.h"

namespace psa {

struct ProjectParams {
    const void* A;                            // [M, Kd] rows, or [B, H, L, 64] when a_heads
    const void* W[3];                         // [N, Kd] each
    const void* bias[3];                      // [N] or nullptr
    void* C[3];                               // [M, N] rows, or [B, H, L, 64] when c_heads
    int M, N, Kd, L, H, a_heads, c_heads, n_mat;
};

constexpr int kProjChunk = 64;                // bfloat16 contraction elements per step through LDS
constexpr int kProjStride = 72;               // bfloat16 per LDS row (64 + 8 pad)

// A wave computes WM x WN MFMA tiles (rows x columns of C); the four waves of a work-group
// form a 2 x 2 grid, so the work-group's tile of C is 64 WM x 64 WN.
template <int WM, int WN>
struct ProjLayout {
    static constexpr int kTM = 64 * WM, kTN = 64 * WN;                     // tile rows, tile columns
    static constexpr int kOperandElems = (kTM + kTN) * kProjStride;        // A tile, then W tile
    static constexpr int kEpiStride = kTN + 8;                             // staged output row, elements
    static constexpr int kEpiRows = 32 * WM;                               // rows per epilogue pass: one row of waves
    static_assert(kEpiRows * kEpiStride <= kOperandElems, "the staging tile fits in the operand tiles");
};

// Few rows (64 x 64 tiles, all work-groups there at once): a tile's chunks come one after the other, each waiting for rows that were
// asked for one chunk ahead, which is less than their way takes.  PF > 1: they are asked for PF chunks ahead, past barriers that leave loads in
// flight.  Whole module, 1 -> 2: B=1 H=4 L=333 25.1 -> 24.8 us, B=1 H=8 L=333 29.0 -> 28.2, B=4 H=8 L=400 34.1 -> 33.2, B=1 H=4 L=40
// 18.5 | 18.5; 3 ahead (124 registers) the same with d_model = 512 and 0.2 more with 256.  For float32 tensors, whose chunks are bound by
// the splitting, 37.2 (2) and 38.0 (3) against 36.8 us at B=1 H=4 L=333.
constexpr int kProjAhead = 2;
template <bool LDS_ONLY> __device__ __forceinline__ void group_barrier() { if constexpr (LDS_ONLY) lds_barrier(); else __syncthreads(); }
// One chunk of a thread's rows of A and of the tile's rows of W by way of buffers, which are empty for a chunk past the end: such
// loads go nowhere, and the number of loads in flight does not depend on the chunk.  (A tensor with few rows has less than 2^31 bytes: the
// launch has at most 1024 tiles of 64 x 64, and W's buffer is the tile's 64 rows.)
template <int NA, int NW, typename Vec, typename T>
__device__ __forceinline__ void fetch_rows(Vec (&ra)[NA], Vec (&rw)[NW], const T* A, const T* Wt, const T* const (&a_ptr)[NA], const T* const (&w_ptr)[NW],
                                           int ka, int k0, bool there, int M, int Kd)
{
    const __amdgpu_buffer_rsrc_t ar = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(A), 0, there ? M * Kd * (int)sizeof(T) : 0, 0x00020000);
    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(Wt), 0, there ? 64 * Kd * (int)sizeof(T) : 0, 0x00020000);
#pragma unroll
    for (int j = 0; j < NA; ++j)
        ra[j] = __builtin_bit_cast(Vec, __builtin_amdgcn_raw_buffer_load_b128(ar, (int)((a_ptr[j] - A) + ka) * (int)sizeof(T), 0, 0));
#pragma unroll
    for (int j = 0; j < NW; ++j)
        rw[j] = __builtin_bit_cast(Vec, __builtin_amdgcn_raw_buffer_load_b128(wr, (int)((w_ptr[j] - Wt) + k0) * (int)sizeof(T), 0, 0));
}

// (Calls with many rows go to project_stream_kernel below.)
// What bounds it (in-kernel time stamps and probes at B*L = 16384, d_model = 512, bfloat16): not
// the contraction loop.  A loop with this mix of LDS reads, LDS writes, loads and one barrier per
// 32 MFMAs sustains 1.6 PFLOP/s when it runs for thousands of chunks; with d_model = 256..512 a
// tile has only 4..8 chunks, and the first loads of a work-group and its output stores take as
// long as its products (stores alone: 10 of 51 us).  Wave tiles of 4 x 2 MFMA tiles, and a
// variant feeding the rows of A straight from memory into operand registers (W alone in LDS),
// both ended at the same time as this kernel, as did two register sets with two LDS stages; two
// tiles per work-group with the second tile's first loads issued before the first tile's
// epilogue were slower (the registers those loads hold cost the third work-group per compute
// unit).  So the simple form is kept, with up to three work-groups per compute unit to overlap
// the phases.
template <int WM, int WN, int PF>
__global__ __launch_bounds__(256, PF > 1 ? 4 : 2)
void project_kernel(const ProjectParams P)
{
    using T = bf16_t;
    using LY = ProjLayout<WM, WN>;
    typedef unsigned int Vec __attribute__((ext_vector_type(4)));         // (native vectors: arrays of them stay in registers)
    constexpr int S = kProjStride, CH = kProjChunk;
    constexpr int TM = LY::kTM, TN = LY::kTN;
    constexpr int VPR = CH * 2 / 16;                       // 16-byte vectors per tile row: 8
    constexpr int NA = TM / 32, NW = TN / 32;              // vectors per thread and chunk: rows of A, rows of W
    static_assert(256 / VPR == 32, "32 tile rows per pass of the work-group");
    __shared__ __attribute__((aligned(16))) T smem[LY::kOperandElems];
    __shared__ __attribute__((aligned(16))) float sBias[TN];
    T* const sA = smem;
    T* const sW = smem + TM * S;

    PSA_TS(0);
    PSA_TS_WALL(5);
    // Work-groups are dealt to the 8 XCDs (each with an L2 of its own) in turn by their linear id.
    // All tiles that share a block of rows of A (every column tile of every matrix) are given to ONE
    // XCD in consecutive slots, so that block of A comes from memory once and from that L2 afterwards.
    const int n_nt = (P.N + TN - 1) / TN, n_mt = (P.M + TM - 1) / TM;
    const int per_rows = n_nt * P.n_mat;
    const int slot = blockIdx.x >> 3;
    const int mt = (slot / per_rows) * 8 + (blockIdx.x & 7);
    if (mt >= n_mt) return;
    const int inner = slot % per_rows;
    const int which = inner / n_nt;
    const T* A = static_cast<const T*>(P.A);
    // (selected with conditionals: indexing the argument arrays by a run-time value would move them to scratch)
    const T* W = static_cast<const T*>(which == 0 ? P.W[0] : (which == 1 ? P.W[1] : P.W[2]));
    const T* bias = static_cast<const T*>(which == 0 ? P.bias[0] : (which == 1 ? P.bias[1] : P.bias[2]));
    T* C = static_cast<T*>(which == 0 ? P.C[0] : (which == 1 ? P.C[1] : P.C[2]));
    const int n0 = (inner % n_nt) * TN, m0 = mt * TM;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 31, h = lane >> 5;
    const int wm = wave >> 1, wn = wave & 1;
    const int n_kc = P.Kd / CH;

    // this thread's share of the tiles: vector `col` of rows row0 + 32 j
    const int row0 = tid / VPR, col = tid % VPR;
    const T* a_ptr[NA];
    const T* w_ptr[NW];
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        int m = m0 + row0 + 32 * j;
        m = m < P.M ? m : P.M - 1;                         // clamped: rows beyond M are never stored
        size_t off;
        if (P.a_heads) { const int b = m / P.L, l = m - b * P.L; off = ((size_t)b * P.H * P.L + l) * kD; }
        else off = (size_t)m * P.Kd;
        a_ptr[j] = A + off + col * 8;
    }
#pragma unroll
    for (int j = 0; j < NW; ++j) {
        const int nr = n0 + row0 + 32 * j;
        w_ptr[j] = W + (size_t)(nr < P.N ? nr : P.N - 1) * P.Kd + col * 8;   // clamped likewise
    }
    // contraction element k0 (a multiple of the chunk, so inside one head) of a row of A
    const size_t head_stride = (size_t)P.L * kD;

    Vec ra[PF][NA], rw[PF][NW];
    floatx16 acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    auto fetch = [&](int set, int kc) {
        const int k0 = kc * CH;
        const size_t ka = P.a_heads ? (size_t)(k0 >> 6) * head_stride + (k0 & 63) : (size_t)k0;
        if constexpr (PF == 1) {
#pragma unroll
            for (int j = 0; j < NA; ++j) ra[set][j] = *reinterpret_cast<const Vec*>(a_ptr[j] + ka);
#pragma unroll
            for (int j = 0; j < NW; ++j) rw[set][j] = *reinterpret_cast<const Vec*>(w_ptr[j] + k0);
        } else {
            fetch_rows<NA, NW>(ra[set], rw[set], A, W + (size_t)n0 * P.Kd, a_ptr, w_ptr, (int)ka, k0, kc < n_kc, P.M, P.Kd);
        }
    };

    // the tile's bias values go to LDS once (an unconditional, clamped load; W stands in for a missing bias)
    T bias_raw;
    {
        const int nb = n0 + (tid & (TN - 1));
        bias_raw = (bias ? bias : W)[nb < P.N ? nb : P.N - 1];
    }
    __builtin_amdgcn_sched_barrier(0);                    // (the bias first: it is waited for alone)
#pragma unroll
    for (int p = 0; p < PF; ++p) fetch(p, p);
    if (tid < TN) {
        sBias[tid] = (bias && n0 + tid < P.N) ? bf16_lo((uint32_t)bias_raw.x) : 0.f;
    }
    for (int first = 0; first < n_kc; first += PF) {
#pragma unroll
    for (int p = 0; p < PF; ++p) {
        const int kc = first + p;
        if (PF > 1 && kc >= n_kc) goto products_done;     // (out of both loops, so that the waits for loads stay exact)
        if (kc < 2) PSA_TS(1 + kc);
        group_barrier<(PF > 1)>();                        // the previous chunk's reads of LDS are done
        {
            T* sa = sA + row0 * S + col * 8;
            T* sw = sW + row0 * S + col * 8;
#pragma unroll
            for (int j = 0; j < NA; ++j) *reinterpret_cast<Vec*>(sa + 32 * j * S) = ra[p][j];
#pragma unroll
            for (int j = 0; j < NW; ++j) *reinterpret_cast<Vec*>(sw + 32 * j * S) = rw[p][j];
        }
        group_barrier<(PF > 1)>();
        if (PF > 1 || kc + 1 < n_kc) fetch(p, kc + PF);   // travels during the products
        __builtin_amdgcn_sched_barrier(0);                // (keeps the loads above them)
        const T* ar = sA + (wm * 32 * WM + c) * S;
        const T* wr = sW + (wn * 32 * WN + c) * S;
#pragma unroll
        for (int kk = 0; kk < CH / 16; ++kk) {
            bf16x8 a[WM], b[WN];
#pragma unroll
            for (int i = 0; i < WM; ++i)
                a[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(ar + i * 32 * S + kk * 16 + 8 * h));
#pragma unroll
            for (int j = 0; j < WN; ++j)
                b[j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(wr + j * 32 * S + kk * 16 + 8 * h));
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
        }
    }
    }
products_done:
    PSA_TS(3);

    // ---- epilogue.  The products were taken as C^T = W A^T (W rows on the MFMA row axis), so a
    // lane owns ONE row m of C and, per register quad, four consecutive columns n.  Bias is added
    // and the value rounded to the storage type in registers; the tile then goes through LDS
    // (reusing the operand tiles), one row of waves at a time, so that every store instruction
    // writes whole 128-byte lines, either row-major or into the head-split layout.
    constexpr int EPV = 8;                                // elements per 16-byte vector
    constexpr int ES = LY::kEpiStride;
    constexpr int VROW = TN / EPV;                        // vectors per staged row
    constexpr int RPP = 256 / VROW;                       // rows per pass of the work-group
    float4 bb[WN][4];                                     // this lane's bias values
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) bb[j][q] = *reinterpret_cast<const float4*>(sBias + wn * 32 * WN + j * 32 + 8 * q + 4 * h);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        __syncthreads();                                  // the operand tiles (or the previous pass) are no longer read
        if (wm == p) {
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int nt = wn * 32 * WN + j * 32 + 8 * q + 4 * h;    // first of four consecutive tile columns
                        const float v0 = acc[i][j][4 * q + 0] + bb[j][q].x, v1 = acc[i][j][4 * q + 1] + bb[j][q].y;
                        const float v2 = acc[i][j][4 * q + 2] + bb[j][q].z, v3 = acc[i][j][4 * q + 3] + bb[j][q].w;
                        T* dst = smem + (i * 32 + c) * ES + nt;
                        *reinterpret_cast<uint2*>(dst) = make_uint2(cvt_pk_bf16(v0, v1), cvt_pk_bf16(v2, v3));
                    }
        }
        __syncthreads();
        const int vec = tid % VROW;
        const int n = n0 + vec * EPV;                     // N is a multiple of 64: a vector is inside or outside
#pragma unroll
        for (int rp = 0; rp < LY::kEpiRows / RPP; ++rp) {
            const int row = rp * RPP + tid / VROW;
            const int m = m0 + p * LY::kEpiRows + row;
            const Vec v = *reinterpret_cast<const Vec*>(smem + row * ES + vec * EPV);
            if (m < P.M && n < P.N) {
                size_t off;
                if (P.c_heads) {
                    const int b = m / P.L, l = m - b * P.L;
                    off = (((size_t)b * P.H + (n >> 6)) * P.L + l) * kD + (n & 63);
                } else {
                    off = (size_t)m * P.N + n;
                }
                *reinterpret_cast<Vec*>(C + off) = v;
            }
        }
    }
    PSA_TS(4);
    PSA_TS_WALL(6);
}

// ---- bfloat16, many rows: 256 x 128 tiles of C, a resident work-group of 8 waves per compute unit that walks several of them.
// With tiles of 4..8 chunks the kernel above spends as long on a tile's first loads and its stores as on its products.  Here the
// chunks of all tiles of a work-group are one stream: loads run two chunks ahead, straight into LDS (no registers to hold),
// across the tiles' borders, and a tile's stores complete under the next tile's products.
// What bounds it: a wave's instructions, not its bytes.  With loads, operand reads and products all left out (a copy made to
// time the rest) a chunk still took 1100 of 2000 cycles at first: a taken branch costs a wave some 80 cycles, and with one
// barrier per chunk all waves pay it at the same time.  So the loop body has no branch (the choice of the next chunk's source is a
// select, loads past the end are asked of an empty buffer, waits are constants, a tile's first chunk has a body of its own), its loads
// stand between the products (asked for together they hold every wave up for 300 cycles), and the barrier stands before the last
// step's products, which cover the first reads behind it: 1430 cycles per chunk, of which the products take 1024.
// Measured at B*L = 16384, d_model = 512, Q, K and V: 49 thousand cycles instead of 62 (three tiles per work-group; 4.4 of
// them before the first product, 2.0 per tile's end), but at 1.85 GHz instead of 2.2, which the card falls to under more
// matrix work: 35.8 -> 30.9 us.
constexpr int kStreamTM = 256, kStreamTN = 128;
constexpr int kStreamThreads = 512;
constexpr int kStreamStages = 3;
constexpr int kStreamRowBytes = kProjChunk * 2;                            // 128: rows without padding, vectors swapped by row
constexpr int kStreamStageBytes = (kStreamTM + kStreamTN) * kStreamRowBytes;       // 49152
constexpr int kStreamMaxBias = 3840;                                       // bias values (floats) of all matrices
constexpr int kStreamGroups = 256;                                         // resident work-groups: one per compute unit
constexpr int kStreamEpiStride = 64 + 8;                                   // staged output row of a wave, elements
static_assert(8 * 32 * kStreamEpiStride * 2 <= kStreamStageBytes, "the waves' staging tiles fit in one stage");
static_assert(kStreamStages * kStreamStageBytes + kStreamTM * 4 + kStreamMaxBias * 4 <= 160 * 1024, "all of it fits in LDS");

// An operand's rows from `base` on as a raw buffer of `bytes` bytes (reads beyond them give zeros), the same in all lanes.
struct RowBuffer { unsigned lo, hi, bytes; };
__device__ __forceinline__ RowBuffer row_buffer(const void* base, unsigned bytes)
{
    const unsigned long long a = reinterpret_cast<unsigned long long>(base);
    return RowBuffer{(unsigned)a, (unsigned)(a >> 32) & 0xFFFFu, bytes};
}
// 16 bytes per lane from memory to LDS (lane l's at lds + 16 l), past the registers.  In assembly because the compiler, which
// cannot tell the stages apart, waits for ALL loads of this kind before any read of LDS; so the waits below count them.
// (M0 holds the LDS address: an operand, so that the compiler writes it and knows.)
__device__ __forceinline__ void load_to_lds(const RowBuffer& buf, unsigned lds, unsigned voffset, unsigned soffset)
{
#if defined(__HIP_DEVICE_COMPILE__)
    typedef unsigned int Rsrc __attribute__((ext_vector_type(4)));
    const Rsrc r = {buf.lo, buf.hi, buf.bytes, 0x00020000u};
    asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "{m0}"(lds), "v"(voffset), "s"(r), "s"(soffset) : "memory");
#endif
}

// A_HEADS: A is [B, H, L, 64], else rows; C_HEADS likewise.  Kd is at least 3 chunks.
template <bool A_HEADS, bool C_HEADS>
__global__ __launch_bounds__(kStreamThreads, 2)
void project_stream_kernel(const ProjectParams P)
{
    using T = bf16_t;
    typedef unsigned int Vec __attribute__((ext_vector_type(4)));
    constexpr int TM = kStreamTM, TN = kStreamTN, CH = kProjChunk;
    constexpr unsigned kBeyond = 0xF0000000u;              // an offset beyond any buffer here
    extern __shared__ __attribute__((aligned(16))) unsigned char stream_smem[];
    unsigned* const sRow = reinterpret_cast<unsigned*>(stream_smem + kStreamStages * kStreamStageBytes);     // the tile's rows in C
    float* const sBias = reinterpret_cast<float*>(sRow + TM);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, h = lane >> 5;
    const int wm = wave >> 1, wn = wave & 1;               // this wave's 64 x 64 part of the tile
    const int n_kc = P.Kd / CH;
    const int n_nt = (P.N + TN - 1) / TN, n_mt = (P.M + TM - 1) / TM;
    const int per_rows = n_nt * P.n_mat;
    // This work-group's tiles.  All column tiles of a block of rows go to ONE XCD (work-groups are dealt to the 8 XCDs in turn),
    // in consecutive slots of its work-groups, so that the block of A comes from memory once.
    const int xcd = blockIdx.x & 7, first = blockIdx.x >> 3, step = gridDim.x >> 3;
    const int slots = ((n_mt - xcd + 7) >> 3) * per_rows;   // of this XCD (n_mt - xcd + 7 >= 0)
    if (first >= slots) return;
    const int n_tiles = (slots - first + step - 1) / step;

    struct Tile { int m0, n0, which; };
    auto tile_of = [&](int k) {                            // k-th tile of this work-group
        const int slot = first + k * step, mi = slot / per_rows, inner = slot - mi * per_rows;
        const int which = inner / n_nt;
        return Tile{(mi * 8 + xcd) * TM, (inner - which * n_nt) * TN, which};
    };
    // row m of a [B, H, L, 64] tensor, from its row m0 on, in bytes (M is at most B * L: rows beyond are caught by the caller)
    auto head_row = [&](int m, int b0, int l0) {
        const int b = m / P.L, l = m - b * P.L;
        return ((unsigned)(b - b0) * (unsigned)P.H * (unsigned)P.L + (unsigned)(l - l0)) * (kD * 2u);
    };
    // ---- the loads, two chunks ahead.  An instruction of a wave fills 8 rows of a stage; lane l: vector l % 8 of row l / 8, which
    // holds the row's vector (l % 8) ^ (row / 2 % 8), so that 16 lanes reading one vector of 16 consecutive rows touch all 64 banks.
    const int srow = wave * 8 + (lane >> 3);               // + 64 per instruction
    const unsigned svec = (unsigned)(((lane & 7) ^ ((srow >> 1) & 7)) * 16);
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)stream_smem + (unsigned)wave * 1024u;
    unsigned va[4], vw[2], va_next[4];                     // (va changes from tile to tile where A is split into heads)
#pragma unroll
    for (int j = 0; j < 4; ++j) va[j] = (unsigned)(srow + 64 * j) * (unsigned)P.Kd * 2u + svec;
#pragma unroll
    for (int j = 0; j < 2; ++j) vw[j] = (unsigned)(srow + 64 * j) * (unsigned)P.Kd * 2u + svec;
    auto sources = [&](int k, RowBuffer& a, RowBuffer& w, unsigned (&v)[4]) {      // of the k-th tile; nothing beyond the last
        const bool live = k < n_tiles;
        const Tile t = tile_of(live ? k : 0);
        const T* A = static_cast<const T*>(P.A);
        if (A_HEADS) {
            const int b0 = t.m0 / P.L, l0 = t.m0 - b0 * P.L;
            a = row_buffer(A + ((size_t)b0 * P.H * P.L + l0) * kD, live ? 0x80000000u : 0u);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int m = t.m0 + srow + 64 * j;
                v[j] = m < P.M ? head_row(m, b0, l0) + svec : kBeyond;
            }
        } else {
            const int rows = P.M - t.m0 < TM ? P.M - t.m0 : TM;
            a = row_buffer(A + (size_t)t.m0 * P.Kd, live ? (unsigned)rows * (unsigned)P.Kd * 2u : 0u);
        }
        const T* W = static_cast<const T*>(t.which == 0 ? P.W[0] : (t.which == 1 ? P.W[1] : P.W[2]));
        const int cols = P.N - t.n0 < TN ? P.N - t.n0 : TN;
        w = row_buffer(W + (size_t)t.n0 * P.Kd, live ? (unsigned)cols * (unsigned)P.Kd * 2u : 0u);
    };
    const unsigned a_step = A_HEADS ? (unsigned)P.L * kD * 2u : (unsigned)kStreamRowBytes;     // from chunk to chunk of a row of A
    RowBuffer ra, rw, ra_next, rw_next;
    sources(0, ra, rw, va);
    int load_kc = 0;
    unsigned load_lds = lds0, sa = 0, sw = 0;
    auto request = [&](int part) {                         // a third of a chunk's loads
        if (part < 2) {
            load_to_lds(ra, load_lds + (2 * part) * 8192, va[2 * part], sa);
            load_to_lds(ra, load_lds + (2 * part + 1) * 8192, va[2 * part + 1], sa);
        } else {
            load_to_lds(rw, load_lds + TM * kStreamRowBytes, vw[0], sw);
            load_to_lds(rw, load_lds + TM * kStreamRowBytes + 8192, vw[1], sw);
        }
    };
    auto advance = [&]() {                                 // to the next chunk, without a branch
        load_lds = load_lds == lds0 + (kStreamStages - 1) * kStreamStageBytes ? lds0 : load_lds + kStreamStageBytes;
        const bool wrap = load_kc + 1 == n_kc;
        load_kc = wrap ? 0 : load_kc + 1;
        sa = wrap ? 0u : sa + a_step;
        sw = wrap ? 0u : sw + kStreamRowBytes;
        ra.lo = wrap ? ra_next.lo : ra.lo; ra.hi = wrap ? ra_next.hi : ra.hi; ra.bytes = wrap ? ra_next.bytes : ra.bytes;
        rw.lo = wrap ? rw_next.lo : rw.lo; rw.hi = wrap ? rw_next.hi : rw.hi; rw.bytes = wrap ? rw_next.bytes : rw.bytes;
        if (A_HEADS) {
#pragma unroll
            for (int j = 0; j < 4; ++j) va[j] = wrap ? va_next[j] : va[j];
        }
    };
    constexpr int kLoads = 6, kStores = 8;                 // vector memory instructions of a wave: per chunk, per tile

    ra_next = ra; rw_next = rw;
#pragma unroll
    for (int j = 0; j < 4; ++j) va_next[j] = va[j];
    for (int k = 0; k < 2; ++k) { request(0); request(1); request(2); advance(); }       // (within the tile: n_kc >= 3)
    // the bias values of all matrices, once: behind the first chunks' loads, the matrices' loads together (one that has no bias
    // reads its weights)
    for (int n = tid; n < P.N; n += kStreamThreads) {
        T raw[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) raw[k] = static_cast<const T*>(k < P.n_mat && P.bias[k] ? P.bias[k] : P.W[0])[n];
#pragma unroll
        for (int k = 0; k < 3; ++k) if (k < P.n_mat) sBias[k * P.N + n] = P.bias[k] ? bf16_lo((uint32_t)raw[k].x) : 0.f;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();

    floatx16 acc[2][2];
    bf16x8 a[2][2], b[2][2];
    const unsigned char* const smem_a = stream_smem + (wm * 64 + c) * kStreamRowBytes;
    const unsigned char* const smem_w = stream_smem + (TM + wn * 64 + c) * kStreamRowBytes;
    int stage = 0;                                         // byte offset of the chunk's stage
    auto operands = [&](int at, int kk) {
        const int vo = at + ((2 * kk + h) ^ ((c >> 1) & 7)) * 16;     // (32 more rows leave row / 2 % 8 as it is)
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            a[kk & 1][x] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(smem_a + x * 32 * kStreamRowBytes + vo));
            b[kk & 1][x] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(smem_w + x * 32 * kStreamRowBytes + vo));
        }
    };
    // One chunk, its first operands read already: four steps of products, a step's operands read before the step before it, and the
    // loads of the chunk after the next between them.  The barrier stands before the last step, whose products cover the read of
    // the next chunk's first operands: there the next chunk is in LDS, for every wave, and this one has been read by all.
    // FIRST of its tile: the stores of the tile before may still be in flight as well.
    auto chunk = [&](auto first_of_tile, int tile) {
        constexpr bool FIRST = decltype(first_of_tile)::value;
        const int next = stage == (kStreamStages - 1) * kStreamStageBytes ? 0 : stage + kStreamStageBytes;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            if (kk < 3) operands(stage, kk + 1);
            if (kk == 3) {
                if (FIRST) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(kLoads + kStores) : "memory");
                else       asm volatile("s_waitcnt vmcnt(%0)" :: "n"(kLoads) : "memory");
                lds_barrier();
                operands(next, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y) {
                    if (FIRST && kk == 0) {
                        floatx16 zero;
#pragma unroll
                        for (int r = 0; r < 16; ++r) zero[r] = 0.f;
                        acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[0][y], a[0][x], zero, 0, 0, 0);
                    } else {
                        acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[kk & 1][y], a[kk & 1][x], acc[x][y], 0, 0, 0);
                    }
                }
            __builtin_amdgcn_sched_barrier(0);
            if (kk < 3) request(kk);
            if (FIRST && kk == 1) sources(tile + 1, ra_next, rw_next, va_next);      // (wanted by the advance below at the earliest: n_kc >= 3)
        }
        advance();
        stage = next;
    };
    operands(0, 0);
#pragma unroll 1
    for (int tile = 0; tile < n_tiles; ++tile) {
        const Tile t = tile_of(tile);
        const int b0 = C_HEADS ? t.m0 / P.L : 0, l0 = t.m0 - b0 * P.L;
        chunk(std::true_type{}, tile);
        // (behind the first chunk's barrier: every wave is done with the tile before; read behind the next one's)
        if (tid < TM) {
            const int m = t.m0 + tid;
            sRow[tid] = m < P.M ? (C_HEADS ? head_row(m, b0, l0) : (unsigned)tid * (unsigned)P.N * 2u) : kBeyond;
        }
#pragma unroll 1
        for (int kc = 1; kc < n_kc; ++kc) chunk(std::false_type{}, tile);
        // ---- the tile is done: bias, rounding, and rows of 128 bytes through this wave's part of the stage read last
        T* C = static_cast<T*>(t.which == 0 ? P.C[0] : (t.which == 1 ? P.C[1] : P.C[2]));
        const size_t base = C_HEADS ? ((size_t)b0 * P.H * P.L + l0) * kD : (size_t)t.m0 * P.N;
        const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(C + base, 0, 0x7FFFFFFF, 0x00020000);
        const int n0 = t.n0 + wn * 64;                     // this wave's 64 columns: one head
        const bool live = n0 < P.N;
        const unsigned col = C_HEADS ? (unsigned)(n0 >> 6) * (unsigned)P.L * (kD * 2u) : (unsigned)n0 * 2u;
        const float* bp = sBias + t.which * P.N + (live ? n0 : 0) + 4 * h;
        float4 bb[2][4];
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int q = 0; q < 4; ++q) bb[y][q] = *reinterpret_cast<const float4*>(bp + y * 32 + 8 * q);
        unsigned ro[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) ro[k] = sRow[wm * 64 + k * 8 + (lane >> 3)];
        const int last = stage == 0 ? (kStreamStages - 1) * kStreamStageBytes : stage - kStreamStageBytes;
        T* out = reinterpret_cast<T*>(stream_smem + last) + wave * 32 * kStreamEpiStride;
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            if (x > 0) wave_lds_sync();
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float v0 = acc[x][y][4 * q + 0] + bb[y][q].x, v1 = acc[x][y][4 * q + 1] + bb[y][q].y;
                    const float v2 = acc[x][y][4 * q + 2] + bb[y][q].z, v3 = acc[x][y][4 * q + 3] + bb[y][q].w;
                    *reinterpret_cast<uint2*>(out + c * kStreamEpiStride + y * 32 + 8 * q + 4 * h) = make_uint2(cvt_pk_bf16(v0, v1), cvt_pk_bf16(v2, v3));
                }
            wave_lds_sync();
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const Vec v = *reinterpret_cast<const Vec*>(out + (it * 8 + (lane >> 3)) * kStreamEpiStride + (lane & 7) * 8);
                const unsigned off = live && ro[4 * x + it] != kBeyond ? ro[4 * x + it] + col + (lane & 7) * 16u : kBeyond;
                __builtin_amdgcn_raw_buffer_store_b128(v, rc, off, 0, 0);       // (always issued: the waits count on it)
            }
        }
        lds_barrier();                                     // every wave is done with the stage, which the next chunk requests anew
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // (loads asked of the empty buffer)
}

// float32 tensors on the bfloat16 matrix cores.  A float32 value is the exact sum of three
// bfloat16 values up to 2^-27 of its size (hi = bf16(x), mid = bf16(x - hi), lo = bf16(x - hi - mid);
// the differences are exact in float32), so a product a * w is, to 2^-25 relative, the sum of the six
// bfloat16 products hi*hi, hi*mid, mid*hi, mid*mid, hi*lo, lo*hi, each exact in the float32
// accumulator of the MFMA: the accuracy of a float32 MFMA contraction (same accumulator, same number
// of additions per term up to the factor 6) at 16/6 times its rate, since a bfloat16 MFMA covers 16
// contraction elements in half the cycles a float32 MFMA needs for 2.  The operands are split once,
// on their way from registers into LDS (three planes of bfloat16 per tile), so the split costs a few
// VALU instructions per loaded element.  The rest is project_kernel: 128 x (64 WN) tiles, 2 x WN
// MFMA tiles per wave, C^T = W A^T, chunks of 32 elements, the same epilogue.
template <int WM, int WN>
struct SplitLayout {
    static constexpr int kTM = 64 * WM, kTN = 64 * WN;
    static constexpr int kRow = 40;                                        // bfloat16 per LDS row: 32 + 8 pad (80 bytes)
    static constexpr int kPlane = (kTM + kTN) * kRow;                      // elements of one plane: A rows, then W rows
    static constexpr int kEpiStride = kTN + 4;                             // staged output row, floats
    static constexpr int kEpiRows = 32 * WM;                               // one row of waves per pass
    static_assert(kEpiRows * kEpiStride * 4 <= 3 * kPlane * 2, "the staging tile fits in the operand planes");
};

// KG = 2, for few rows: two groups of 4 waves take every other chunk, each with planes of its own, and their sums are added at the end.
// What bounds such a call is the chain of one work-group's chunks (split, LDS, reads, twelve dependent MFMAs: 0.5 us each),
// which the second group halves; four groups gained less (B=1 H=4 L=333: 39.9, 37.4, 38.2 us with one, two, four).  The
// sums are half as long, so their error is no larger.
template <int WM, int WN, int KG>
__global__ __launch_bounds__(256 * KG, 2)
void project_split_kernel(const ProjectParams P)
{
    using LY = SplitLayout<WM, WN>;
    typedef float Vec __attribute__((ext_vector_type(4)));
    constexpr int CH = 32, S = LY::kRow, TM = LY::kTM, TN = LY::kTN;
    constexpr int NA = TM / 32, NW = TN / 32;              // float4 vectors per thread and chunk: rows of A, rows of W
    __shared__ __attribute__((aligned(16))) uint16_t s_planes[KG][3 * LY::kPlane];
    __shared__ __attribute__((aligned(16))) float sBias[TN];

    PSA_TS(0);
    PSA_TS_WALL(5);
    // (the same dealing of tiles to XCDs as in project_kernel)
    const int n_nt = (P.N + TN - 1) / TN, n_mt = (P.M + TM - 1) / TM;
    const int per_rows = n_nt * P.n_mat;
    const int slot = blockIdx.x >> 3;
    const int mt = (slot / per_rows) * 8 + (blockIdx.x & 7);
    if (mt >= n_mt) return;
    const int inner = slot % per_rows;
    const int which = inner / n_nt;
    const float* A = static_cast<const float*>(P.A);
    const float* W = static_cast<const float*>(which == 0 ? P.W[0] : (which == 1 ? P.W[1] : P.W[2]));
    const float* bias = static_cast<const float*>(which == 0 ? P.bias[0] : (which == 1 ? P.bias[1] : P.bias[2]));
    float* C = static_cast<float*>(which == 0 ? P.C[0] : (which == 1 ? P.C[1] : P.C[2]));
    const int n0 = (inner % n_nt) * TN, m0 = mt * TM;
    const int kg = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);       // which chunks: kg, kg + KG, ...
    uint16_t* const smem = s_planes[kg];
    const int tid = threadIdx.x & 255, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 31, h = lane >> 5;
    const int wm = wave >> 1, wn = wave & 1;
    const int rounds = P.Kd / (CH * KG);                   // (Kd is a multiple of 64: as many for each group)
    static_assert(64 % (CH * KG) == 0, "whole rounds");

    // this thread's share of the tiles: float4 `col` of rows row0 + 32 j
    const int row0 = tid >> 3, col = tid & 7;
    const float* a_ptr[NA];
    const float* w_ptr[NW];
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        int m = m0 + row0 + 32 * j;
        m = m < P.M ? m : P.M - 1;                         // clamped: rows beyond M are never stored
        size_t off;
        if (P.a_heads) { const int b = m / P.L, l = m - b * P.L; off = ((size_t)b * P.H * P.L + l) * kD; }
        else off = (size_t)m * P.Kd;
        a_ptr[j] = A + off + col * 4;
    }
#pragma unroll
    for (int j = 0; j < NW; ++j) {
        const int nr = n0 + row0 + 32 * j;
        w_ptr[j] = W + (size_t)(nr < P.N ? nr : P.N - 1) * P.Kd + col * 4;                     // clamped likewise
    }
    const size_t head_stride = (size_t)P.L * kD;

    Vec ra[NA], rw[NW];
    floatx16 acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    auto fetch = [&](int round) {
        const int k0 = (KG * round + kg) * CH;
        const size_t ka = P.a_heads ? (size_t)(k0 >> 6) * head_stride + (k0 & 63) : (size_t)k0;
#pragma unroll
        for (int j = 0; j < NA; ++j) ra[j] = *reinterpret_cast<const Vec*>(a_ptr[j] + ka);
#pragma unroll
        for (int j = 0; j < NW; ++j) rw[j] = *reinterpret_cast<const Vec*>(w_ptr[j] + k0);
    };
    // four floats -> their hi, mid and lo bfloat16 parts, 8 bytes into each plane
    auto put_split = [&](uint16_t* dst, Vec x) {
        const uint32_t h0 = cvt_pk_bf16(x.x, x.y), h1 = cvt_pk_bf16(x.z, x.w);
        float r0 = x.x - bf16_lo(h0), r1 = x.y - bf16_hi(h0), r2 = x.z - bf16_lo(h1), r3 = x.w - bf16_hi(h1);
        const uint32_t m0_ = cvt_pk_bf16(r0, r1), m1_ = cvt_pk_bf16(r2, r3);
        r0 -= bf16_lo(m0_); r1 -= bf16_hi(m0_); r2 -= bf16_lo(m1_); r3 -= bf16_hi(m1_);
        const uint32_t l0 = cvt_pk_bf16(r0, r1), l1 = cvt_pk_bf16(r2, r3);
        *reinterpret_cast<uint2*>(dst) = make_uint2(h0, h1);
        *reinterpret_cast<uint2*>(dst + LY::kPlane) = make_uint2(m0_, m1_);
        *reinterpret_cast<uint2*>(dst + 2 * LY::kPlane) = make_uint2(l0, l1);
    };

    float bias_raw;
    {
        const int nb = n0 + (tid & (TN - 1));
        bias_raw = (bias ? bias : W)[nb < P.N ? nb : P.N - 1];    // unconditional, clamped; W stands in for a missing bias
    }
    fetch(0);
    if (kg == 0 && tid < TN) sBias[tid] = (bias && n0 + tid < P.N) ? bias_raw : 0.f;
    for (int round = 0; round < rounds; ++round) {
        if (round < 2) PSA_TS(1 + round);
        __syncthreads();                                  // the previous chunk's reads of LDS are done
        {
            uint16_t* sa = smem + row0 * S + col * 4;
            uint16_t* sw = smem + (TM + row0) * S + col * 4;
#pragma unroll
            for (int j = 0; j < NA; ++j) put_split(sa + 32 * j * S, ra[j]);
#pragma unroll
            for (int j = 0; j < NW; ++j) put_split(sw + 32 * j * S, rw[j]);
        }
        __syncthreads();
        if (round + 1 < rounds) fetch(round + 1);         // travels during the products
        __builtin_amdgcn_sched_barrier(0);                // (keeps the loads above them)
        const uint16_t* ar = smem + (wm * 32 * WM + c) * S + 8 * h;
        const uint16_t* wr = smem + (TM + wn * 32 * WN + c) * S + 8 * h;
#pragma unroll
        for (int kk = 0; kk < CH / 16; ++kk) {
            bf16x8 a[3][WM], b[3][WN];
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) {
#pragma unroll
                for (int i = 0; i < WM; ++i)
                    a[pl][i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(ar + pl * LY::kPlane + i * 32 * S + kk * 16));
#pragma unroll
                for (int j = 0; j < WN; ++j)
                    b[pl][j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(wr + pl * LY::kPlane + j * 32 * S + kk * 16));
            }
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j) {
                    // smallest terms first
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[2][j], a[0][i], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[0][j], a[2][i], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[1][j], a[1][i], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[1][j], a[0][i], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[0][j], a[1][i], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[0][j], a[0][i], acc[i][j], 0, 0, 0);
                }
        }
    }
    PSA_TS(3);
    if constexpr (KG > 1) {
        // the groups' shares of the tile together, in order of the groups: each through its own planes' LDS
        static_assert(WM == 1 && WN == 1 && 4 * 16 * 64 * 4 <= 3 * LY::kPlane * 2, "a group's sums fit in its planes");
        __syncthreads();
        float* const mine = reinterpret_cast<float*>(smem) + (wave * 16) * 64 + lane;
        if (kg > 0) {
#pragma unroll
            for (int r = 0; r < 16; ++r) mine[r * 64] = acc[0][0][r];
        }
        __syncthreads();
        if (kg == 0) {
#pragma unroll
            for (int k = 1; k < KG; ++k) {
                const float* other = reinterpret_cast<const float*>(s_planes[k]) + (wave * 16) * 64 + lane;
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[0][0][r] += other[r * 64];
            }
        }
    }

    // ---- epilogue (as in project_kernel): bias in registers, the tile through LDS one row of
    // waves at a time, stores of whole 128-byte lines
    constexpr int ES = LY::kEpiStride;
    constexpr int VROW = TN / 4;                          // float4 vectors per staged row
    constexpr int RPP = 256 / VROW;                       // rows per pass of the work-group
    float* const stage = reinterpret_cast<float*>(smem);
    float4 bb[WN][4];
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) bb[j][q] = *reinterpret_cast<const float4*>(sBias + wn * 32 * WN + j * 32 + 8 * q + 4 * h);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        __syncthreads();                                  // the operand planes (or the previous pass) are no longer read
        if (kg == 0 && wm == p) {
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int nt = wn * 32 * WN + j * 32 + 8 * q + 4 * h;    // first of four consecutive tile columns
                        *reinterpret_cast<float4*>(stage + (i * 32 + c) * ES + nt) =
                            make_float4(acc[i][j][4 * q + 0] + bb[j][q].x, acc[i][j][4 * q + 1] + bb[j][q].y,
                                        acc[i][j][4 * q + 2] + bb[j][q].z, acc[i][j][4 * q + 3] + bb[j][q].w);
                    }
        }
        __syncthreads();
        if (KG > 1 && kg > 0) continue;                   // wave-uniform
        const int vec = tid % VROW;
        const int n = n0 + vec * 4;                       // N is a multiple of 64: a vector is inside or outside
#pragma unroll
        for (int rp = 0; rp < LY::kEpiRows / RPP; ++rp) {
            const int row = rp * RPP + tid / VROW;
            const int m = m0 + p * LY::kEpiRows + row;
            const Vec v = *reinterpret_cast<const Vec*>(stage + row * ES + vec * 4);
            if (m < P.M && n < P.N) {
                size_t off;
                if (P.c_heads) {
                    const int b = m / P.L, l = m - b * P.L;
                    off = (((size_t)b * P.H + (n >> 6)) * P.L + l) * kD + (n & 63);
                } else {
                    off = (size_t)m * P.N + n;
                }
                *reinterpret_cast<Vec*>(C + off) = v;
            }
        }
    }
    PSA_TS(4);
    PSA_TS_WALL(6);
}

template <int WM, int WN, int KG = 1>
static hipError_t launch_project_split(const ProjectParams& P, hipStream_t stream)
{
    using LY = SplitLayout<WM, WN>;
    const int n_nt = (P.N + LY::kTN - 1) / LY::kTN, n_mt = (P.M + LY::kTM - 1) / LY::kTM;
    hipLaunchKernelGGL((project_split_kernel<WM, WN, KG>), dim3(8 * ((n_mt + 7) / 8) * n_nt * P.n_mat), dim3(256 * KG), 0, stream, P);
    return hipGetLastError();
}

template <int WM, int WN, int PF = 1>
static hipError_t launch_project_as(const ProjectParams& P, hipStream_t stream)
{
    using LY = ProjLayout<WM, WN>;
    const int n_nt = (P.N + LY::kTN - 1) / LY::kTN, n_mt = (P.M + LY::kTM - 1) / LY::kTM;
    hipLaunchKernelGGL((project_kernel<WM, WN, PF>), dim3(8 * ((n_mt + 7) / 8) * n_nt * P.n_mat), dim3(256), 0, stream, P);
    return hipGetLastError();
}

// Offsets from a tile's first row must fit a buffer descriptor's range: a tile of 256 rows spans at most 256 / L + 2 items.
static bool stream_fits(const ProjectParams& P)
{
    const long rows = 2l * P.L + 2 * kStreamTM;
    return rows * P.H * kD * 2 < (1l << 30) && (long)P.N * P.Kd * 2 < (1l << 30) && P.n_mat * P.N <= kStreamMaxBias && P.Kd >= 3 * kProjChunk;
}

// The resident work-groups take one tile each per round.  From two rounds on (what the first round's loads and the last one's stores
// cost is then shared) and where at least 7 of 8 tiles' worth of every round is needed:
//   rows x columns x matrices (d_model)   rounds  needed   128 x 128 tiles -> this kernel (whole module but for the last)
//   32768 x 512 x 3, x 1 (512)             6, 2     100%      213.4 -> 205.6 us
//   16384 x 512 x 3 (512)                   3       100%      107.8 -> 105.0 us
//   32768 x 256 x 3 (256)                   3       100%       91.8 ->  91.4 us
//   10101 x 512 x 3 (512)                   2        93%       88.0 ->  86.1 us
//   12000 x 512 x 3 (512)                   3        73%       97.9 ->  97.5 us
//   16384 x 256 x 3 (256)                   2        75%       47.4 ->  48.8 us
//   16384 x 512 x 1 (512)                   1       100%       14.9 ->  14.7 us
static bool stream_pays(const ProjectParams& P)
{
    const int n_nt = (P.N + kStreamTN - 1) / kStreamTN, n_mt = (P.M + kStreamTM - 1) / kStreamTM;
    const long slots = (long)((n_mt + 7) / 8) * n_nt * P.n_mat, per_xcd = kStreamGroups / 8;        // of the fullest XCD
    const long rounds = (slots + per_xcd - 1) / per_xcd;
    return rounds >= 2 && 8l * P.M * P.N * P.n_mat >= 7l * rounds * kStreamGroups * kStreamTM * kStreamTN;
}

template <bool A_HEADS, bool C_HEADS>
static hipError_t raise_stream_limit()
{
    static std::atomic<uint64_t> raised;
    return ensure_lds_limit((const void*)project_stream_kernel<A_HEADS, C_HEADS>,
                            kStreamStages * kStreamStageBytes + kStreamTM * 4 + kStreamMaxBias * (int)sizeof(float), raised);
}
hipError_t init_project()
{
    const hipError_t e = raise_stream_limit<false, true>();
    return e != hipSuccess ? e : raise_stream_limit<true, false>();
}

template <bool A_HEADS, bool C_HEADS>
static hipError_t launch_project_stream(const ProjectParams& P, hipStream_t stream)
{
    const hipError_t e = raise_stream_limit<A_HEADS, C_HEADS>();
    if (e != hipSuccess) return e;
    const int n_nt = (P.N + kStreamTN - 1) / kStreamTN, n_mt = (P.M + kStreamTM - 1) / kStreamTM;
    const int lds = kStreamStages * kStreamStageBytes + kStreamTM * 4 + P.n_mat * P.N * (int)sizeof(float);
    const long most = 8l * ((n_mt + 7) / 8) * n_nt * P.n_mat;
    hipLaunchKernelGGL((project_stream_kernel<A_HEADS, C_HEADS>), dim3((unsigned)(most < kStreamGroups ? most : kStreamGroups)), dim3(kStreamThreads), lds, stream, P);
    return hipGetLastError();
}

// Which kernel a launch takes: project_kernel and project_split_kernel by their tiles
enum ProjectRoute { kStream, kTiles22, kTiles21, kTiles11, kSplit22, kSplit21, kSplit11, kSplit11TwoGroups };
static ProjectRoute project_route(const ProjectParams& P, int dtype)
{
    // 128 x 128 tiles when they give every compute unit at least two work-groups, else 128 x 64
    const long wg128 = (long)((P.N + 127) / 128) * ((P.M + 127) / 128) * P.n_mat;
    if (dtype == PSA_F32) {
        // (128 x 64 tiles give 2 wg128 work-groups, 64 x 64 tiles 4 wg128)
        if (wg128 >= 512) return kSplit22;
        if (2 * wg128 >= 512) return kSplit21;
        // (two groups of waves while their work-groups, two to a compute unit, are there at once: whole module, B=1 H=4 L=333, 96
        // and 24 of them, 39.9 -> 37.4 us; B=1 H=8 L=333 52.1 -> 45.2; B=8 H=4 L=300, 456, 43.6 -> 42.1; B=8 H=8 L=300, 912, 75.6 -> 77.0)
        const long wg64 = (long)((P.N + 63) / 64) * ((P.M + 63) / 64) * P.n_mat;
        return wg64 <= 512 ? kSplit11TwoGroups : kSplit11;
    }
    if (stream_pays(P) && stream_fits(P)) return kStream;
    // Few rows: 64 x 64 tiles, four times as many work-groups with half of the loads and a quarter of the stores each, as long
    // as all are there at once (four to a compute unit).  Whole module, 128 x 64 -> 64 x 64: B=1 H=4 L=40 20.8 -> 19.2 us, B=1
    // H=8 L=333 33.6 -> 31.0, B=4 H=8 L=400 (624 of them for Q, K and V) 37.2 -> 34.8, B=3 H=8 L=2000 (752 for the output
    // matrix) 70.5 -> 69.2; B=24 H=8 L=500 (1504 for the output matrix) 78.3 -> 78.8.
    if (wg128 <= 256) return kTiles11;
    return wg128 >= 512 ? kTiles22 : kTiles21;
}

static hipError_t launch_project(const ProjectParams& P, int dtype, hipStream_t stream)
{
    switch (project_route(P, dtype)) {
        case kStream:  return P.a_heads ? launch_project_stream<true, false>(P, stream) : launch_project_stream<false, true>(P, stream);
        case kTiles22: return launch_project_as<2, 2>(P, stream);
        case kTiles21: return launch_project_as<2, 1>(P, stream);
        case kTiles11: return launch_project_as<1, 1, kProjAhead>(P, stream);
        case kSplit22: return launch_project_split<2, 2>(P, stream);
        case kSplit21: return launch_project_split<2, 1>(P, stream);
        case kSplit11: return launch_project_split<1, 1>(P, stream);
        default:       return launch_project_split<1, 1, 2>(P, stream);
    }
}

// the sizes of the launch for Q, K and V (three matrices) or for the output matrix (one)
static ProjectParams project_sizes(const psa_shape_t& s, int n_mat)
{
    ProjectParams P{};
    P.M = s.B * s.L_K; P.N = P.Kd = s.H * kD; P.L = s.L_K; P.H = s.H;
    P.n_mat = n_mat; P.a_heads = n_mat == 1; P.c_heads = n_mat != 1;
    return P;
}
const char* project_route_name(const psa_shape_t& s, int n_mat)
{
    static const char* const names[] = {"stream", "tiles_128x128", "tiles_128x64", "tiles_64x64", "tiles_128x128", "tiles_128x64", "tiles_64x64",
                                        "tiles_64x64_two_groups"};
    return names[project_route(project_sizes(s, n_mat), s.dtype)];
}

hipError_t launch_qkv_project(const psa_shape_t& s, const void* X, const psa_mhsa_weights_t& w,
                              void* Q, void* K, void* V, hipStream_t stream)
{
    ProjectParams P = project_sizes(s, 3);
    P.A = X;
    P.W[0] = w.Wq; P.W[1] = w.Wk; P.W[2] = w.Wv;
    P.bias[0] = w.bq; P.bias[1] = w.bk; P.bias[2] = w.bv;
    P.C[0] = Q; P.C[1] = K; P.C[2] = V;
    return launch_project(P, s.dtype, stream);
}

hipError_t launch_out_project(const psa_shape_t& s, const void* A, const psa_mhsa_weights_t& w, void* Y, hipStream_t stream)
{
    ProjectParams P = project_sizes(s, 1);
    P.A = A;
    P.W[0] = w.Wo;
    P.bias[0] = w.bo;
    P.C[0] = Y;
    return launch_project(P, s.dtype, stream);
}

}  // namespace psa
