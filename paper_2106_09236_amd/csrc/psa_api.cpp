// C ABI of libprobsparse.so: argument checks, launch plan, workspace carving and
// the stage pipeline.  All checks run before the first launch; nothing here
// allocates, frees or synchronises.
#include <stdio.h>
#include <math.h>
#include <string.h>

#include "psa_internal.h"

namespace psa {

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

static int check_shape(const psa_shape_t* s)
{
    if (!s) return PSA_ERR_NULL;
    if (s->dtype != PSA_F32 && s->dtype != PSA_BF16) return PSA_ERR_DTYPE;
    if (s->B < 1 || s->H < 1 || s->L_Q < 1 || s->L_K < 1 || s->U < 1) return PSA_ERR_SHAPE;
    if (s->D != kD) return PSA_ERR_SHAPE;
    if (s->L_Q != s->L_K) return PSA_ERR_SHAPE;           // self-attention only (Sec. 3.1)
    if ((int64_t)s->B * s->H > 65535) return PSA_ERR_SHAPE;   // heads ride on a 16-bit grid axis
    if (s->L_K > (1 << 22)) return PSA_ERR_SHAPE;
    if (s->U > (1 << 16)) return PSA_ERR_SHAPE;
    return PSA_OK;
}

static int u_max_of(URule r, int L)
{
    double x = r.rule == PSA_U_RATIO ? ceil(r.factor * (double)L) : ceil(r.factor * log((double)L));
    if (!(x >= 1.0)) x = 1.0;
    if (x > (double)L) x = (double)L;
    return (int)x;
}

static bool good_rule(URule r)
{
    return (r.rule == PSA_U_LOG || r.rule == PSA_U_RATIO) && r.factor > 0.0 && isfinite(r.factor);
}

// float32 tensors, heads in one key split: work-groups that share the output elements of a query group, as many (1, 2, 4) as
// the compute units hold (one each: LDS and registers).  Each forms all scores and 1/d of the second product, 32 + 32/d float64 MFMAs for
// a tile of 32 keys instead of 64, and there is nothing to hand over.  Whole call, 1 -> d work-groups: B=1 H=4 L=128 (8 -> 32 of
// them) 14.3 -> 13.3 us, B=1 H=4 L=333 24.1 -> 21.7, B=4 H=4 L=300 23.0 -> 20.3, B=8 H=4 L=200 (64 -> 256) 20.3 -> 18.6 us.
static int elem_split(int64_t wgs) { return 4 * wgs <= 256 ? 4 : 2 * wgs <= 256 ? 2 : 1; }

// Given sets, mean fill, short heads: each attend work-group (n_wg of a head) reads all of its head's V for the column sums it needs (out of
// its L2, where the head's other work-groups and its own products find V then) instead of a launch that does.  In microseconds: a
// CU takes in 105 KB, the launch costs 3.5 and reads V at 5 TB/s.  Whole call, launch -> own: B=16 H=4 L=512 float32, 32 kept
// 21.2 -> 17.7 us, B=1 H=4 L=128 10.5 -> 8.1, B=32 H=8 L=512 with 100 kept (4 work-groups a head) 118 -> 114, but B=64 H=8 L=400 with
// 200 kept (7) 349 | 354; bfloat16 B=32 H=4 L=512 15.8 -> 11.1, B=128 H=8 L=1024 135 -> 104, B=8 H=8 L=1024 with 512 kept 27.0 -> 22.7.
static bool sums_in_attend(const Plan& p, int n_wg)
{
    const size_t v_bytes = (size_t)p.L * (p.dtype == PSA_F32 ? 256 : 128);
    if (!p.given_indices || p.u_max > kSelLdsMax || v_bytes > kOwnSumBytes) return false;
    const float heads = (float)p.BH * (float)v_bytes;
    return heads * (float)n_wg / (256.f * 105e3f) + 0.5f <= 3.5f + heads / 5e6f;
}
// ... and what the launch that clears the tickets then costs, which a cut without hand-over does not need (B=16 H=4 L=512, 32 kept: one
// split 17.7 us, four splits 20.2).  Elsewhere the launch for the column sums clears them.  (With value fill nothing needs those
// sums, but a plan holds for both fills: a call whose heads are split still takes the launch for its tickets.)
constexpr float kTicketLaunch = 2.f;

// float32 tensors: queries per group and key splits of the key-split attend kernel, by the time of its rounds of
// work-groups (one per CU).  In microseconds, fitted to sweeps of both over 15 shapes: 5.5 to start a work-group and
// pick the selection, 2.3 for each tile step of a SIMD (64 float64 MFMAs), and for a split the hand-over of records:
// 3 and 1.5 for each trip of the last work-group's merge (32 queries x 4 splits), or the merge kernel.  Heads in one split whose
// elements four work-groups share take 0.75 of a step (by the MFMAs 0.63, which would keep B=2 H=4 L=800 in one split: 34.5 us
// against 31.0; B=1 H=4 L=500 in two splits 23.1, in one 21.9 us).  A last round
// of work-groups that is not full counts half: heads are often shorter than L.
// Against groups of 32 and 512 work-groups for every shape: B=24 H=4 L=750 ragged 87 -> 75 us, B=16 H=4 L=1000
// 83 -> 63, B=64 H=4 L=200 52 -> 36, B=1 H=4 L=333 26.0 -> 23.8 us.
static void split_f32(Plan* p, int n_tiles)
{
    float best = INFINITY;
    for (int ncg = 2; ncg >= 1; --ncg) {                      // (of equals the larger groups: they read K and V less often)
        const int nq = 16 * ncg, tiles_wg = 8 / ncg;
        const int n_qgroup = (p->u_max + nq - 1) / nq;
        const int64_t per_split = (int64_t)p->BH * n_qgroup;
        int max_split = (n_tiles + tiles_wg - 1) / tiles_wg;
        if (max_split > kMaxSplit) max_split = kMaxSplit;
        // 1 .. 8 splits, or as many as give each CU a work-group
        const int fill = per_split < 256 ? (int)(256 / per_split) : 1;
        for (int k = 1; k <= kTicketMaxSplit + 1; ++k) {
            int split = k <= kTicketMaxSplit ? k : fill;
            if (split > max_split) split = max_split;
            const int rounds = (n_tiles + split * tiles_wg - 1) / (split * tiles_wg);
            split = (n_tiles + rounds * tiles_wg - 1) / (rounds * tiles_wg);
            const int tiles = n_tiles < rounds * tiles_wg ? n_tiles : rounds * tiles_wg;
            const int steps = (tiles * ncg + 3) / 4;
            const float fills = (float)(per_split * split) / 256.f;
            const float part = split == 1 && elem_split(per_split) == 4 ? 0.75f : 1.f;      // of a tile step
            const float ticket = sums_in_attend(*p, n_qgroup * split) ? kTicketLaunch : 0.f;
            const float cost = (fills <= 1.f ? 1.f : 0.5f * (fills + ceilf(fills))) * (5.5f + 2.3f * part * (float)steps) +
                (split == 1 ? 0.f : split > kTicketMaxSplit ? 6.f : ticket + 3.f + 1.5f * (float)((p->u_max + 31) / 32 * ((split + 3) / 4)));
            if (cost < best) {
                best = cost;
                p->nq_group = nq; p->n_qgroup = n_qgroup; p->n_split = split; p->tiles_per_wave = rounds;
            }
            if (k >= max_split) break;
        }
    }
}

// Streaming measure kernel with `cpw` chunks per work-group: length of the sorted list each work-group hands on, or 0
// where a select kernel follows.  Lists only where the attend prologue can merge them (up to 8 per head; no select
// launch: 8.3 us at B=8 H=8 L=2048), the ranking at the end of a work-group is short (`most` queries at most: kListMax,
// or kListMaxF32 for float32; a microsecond), and the candidates are few: every attend work-group of the head merges
// them (with half of 2048 queries kept 134 us with lists against 123 us with the select kernel).
static int stream_list_len(const Plan& p, int cpw, int most)
{
    const int groups = (p.n_chunk + cpw - 1) / cpw, span = cpw * kMeasureQueries;
    const int len = p.u_max < span ? p.u_max : span;
    return p.U <= kPipeMaxSamples && groups <= 8 && span <= most && (int64_t)groups * len <= 512 ? len : 0;
}

// Streaming measure kernel, float32: consecutive chunks of a head that one of its persistent work-groups takes, by the
// chunks of the busiest CU when every item is full.  A float32 work-group (256-byte rows) reaches the rate of the CU's
// return path alone and only takes turns with a second one (B=16 H=4 L=1000: 30.2 us in 256 work-groups of 4 chunks, 33.5
// in 512 of 2).  A head's work-groups all run on one XCD, 32 CUs, the whole ones of all its heads first and the last,
// shorter ones behind them; those share a CU with one another where enough CUs are left for them, else with a whole one.
// In chunks: a quarter for each further work-group of a CU, 0.9 for the select kernel where no list fits.  Of cuts within 3 % the
// finer one: it loses less where items are shorter than L.
// Lengths are known on the device only, so calls with and without them take the same cut; one that counted on a fifth of
// padding took 54 us for the measure of a full B=24 H=4 L=750 where two work-groups per CU take 44 and this one 35.
// Whole call on full batches, two work-groups per CU | this rule: B=24 H=4 L=750 90 | 81 us, B=12 H=8 L=520 54 | 49, B=9 H=4
// L=1700 87 | 76, B=1 H=2 L=9000 79 | 71, B=36 H=4 L=800 113 | 121 (the most lost in 35 shapes; 4 % gained in the mean).
// Ragged batches of few items lose up to an eighth against the cut that counted on padding (B=5 H=4 L=3000 70 | 78 us).
// bfloat16 work-groups share a CU to advantage (B=8 H=8 L=2048 55.8 us in 512, 63.4 in 256).
static float stream_cost_f32(const Plan& p, int cpw)
{
    const int heads = (p.BH + 7) / 8, span = cpw * kMeasureQueries;      // heads of an XCD
    int whole = heads * (p.L / span), part = p.L % span ? heads : 0;     // its work-groups of cpw chunks, and shorter ones
    const float rest = (float)(p.L % span) / (float)kMeasureQueries;     // chunks of those
    float longest = (float)cpw;
    if (whole == 0) { whole = part; part = 0; longest = rest; }
    const int rounds = (whole + 31) / 32, left = 32 * rounds - whole;    // CUs that have one whole work-group less than others
    float cost = longest * (float)rounds + 0.25f * (float)(rounds - 1);
    if (part > left) {
        if (rounds == 1 && left >= 4 && part <= 2 * left) cost = fmaxf(longest, 2.f * rest + 0.25f);
        else cost += rest + 0.25f;
    }
    return cost + (stream_list_len(p, cpw, kListMaxF32) > 0 ? 0.f : 0.9f);
}
static int stream_cut_f32(const Plan& p)
{
    const int most = p.n_chunk < 16 ? p.n_chunk : 16;
    float best = INFINITY;
    for (int cpw = 1; cpw <= most; ++cpw) best = fminf(best, stream_cost_f32(p, cpw));
    int cpw = 1;
    while (cpw < most && stream_cost_f32(p, cpw) > 1.03f * best) ++cpw;
    return cpw;
}

// Streamed heads whose K fits LDS in two parts: passes of 128 queries that a work-group of the measure kernel which gathers from
// there takes, or 0 where the heads stay with the gather out of L2.  Its time hardly depends on the samples (8.4 us to start
// with K and the first indices, 4 for each pass, 2.3 for the ranking), that of a gather out of L2 does, so it takes calls with more
// than 28.  A CU holds one of its work-groups, which K has to be copied for, so they have to fill more than half of the chip.
// float32, two passes (whole call, L2 -> parts): B=16 H=4 L=750 with 34 samples 49.5 -> 44.0 us, with 24 45.3 -> 43.8, with 16 42.5 | 43.9; B=8
// H=4 L=640 (96 work-groups) 36.1 | 36.6, B=12 H=4 L=750 (144) 47.9 -> 43.7.  Of 168 calls of 44 to 192 heads of 513 to 1024 frames,
// full and ragged, it loses 2 to 3 % in three.
// bfloat16: the gather out of L2 works at one rate whatever the shape, but these work-groups come in rounds of an XCD's 32
// CUs, and a round that is not full costs what a full one does.
//   * Two passes where all work-groups run in one round, with at least 160 of them (192 for fewer than 28 heads, whose items are few: lengths
//     may leave little of them): B=10 H=4 L=1500 (35 samples) 40.1 -> 33.8 us, with lengths from an eighth up 38.2 -> 34.6; B=7 H=4 L=1281 (168) 37.9
//     -> 34.5 and 36.5 -> 34.0, but L=1100 (140) 36.7 -> 33.2 and 32.1 | 33.0; B=3 H=8 L=1600 (168) 38.3 -> 35.3 and 34.1 | 36.0.
//   * Else four passes, where the rounds (parts_rounds, a start counted like a pass) give enough samples of enough queries in their
//     time: 21 samples per lane of queries there, 24 beyond 1536 frames, where lengths leave whole work-groups out of
//     the last round.  Measured for 28 to 192 heads and 27 to 39 samples, full | ragged: B=24 H=4 L=1040 (21.3) 61.9 -> 55.5 | 59.6 -> 53.2,
//     B=48 H=4 L=1300 (22.8) 118.8 -> 107.6 | 101.4 -> 91.8, L=2048 B=16 H=4 (31.2) 54.8 -> 48.5 | 55.7 -> 47.9; and not: B=24 H=4 L=1300 (18.6)
//     66.0 | 70.2 and 64.0 -> 55.6, B=16 H=4 L=1300 with 31 (15.7) 42.0 | 45.4 and 43.6 | 45.5, L=2048 B=24 H=4 (23.4) 87.6 | 90.0 and 79.5 | 83.6.
//     Two passes in more than one round lose on most of these (L=2048 B=16 H=4 54.8 | 54.9 and 55.7 -> 53.7).
// Four passes wherever two made more than 32 whole work-groups of an XCD, for all calls with 129 work-groups or more, took B=9 H=8 L=2048 with 31
// samples from 70.1 to 83.0 us, B=14 H=8 L=1400 with 29 from 69.9 to 78.8.  168 calls of 24 to 256 heads of 1150 to 2048 frames, full and
// ragged, none of those above: 5 % gained in the mean, two lose 2 to 2.5 %.
// Lengths are known on the device only, so calls with and without them take the same form.
static int parts_rounds(const Plan& p, int passes)
{
    const int heads = (p.BH + 7) / 8, span = passes * 2 * kMeasureQueries, whole = heads * (p.L / span), rest = p.L % span;
    const int full = 1 + passes, part = 1 + (rest + 2 * kMeasureQueries - 1) / (2 * kMeasureQueries);
    // the whole work-groups of an XCD first, then the shorter ones of its heads, on the CUs as they come free
    const int rounds = whole / 32, more = whole % 32;
    int time = (rounds + (more > 0)) * full;
    if (rest == 0) return time;
    while (more * (time / full > rounds ? (time - (rounds + 1) * full) / part : 0) + (32 - more) * ((time - rounds * full) / part) < heads) ++time;
    return time;
}
static int part_passes(const Plan& p, size_t k_bytes)
{
    const int heads = (p.BH + 7) / 8, span = kPartChunks * kMeasureQueries, groups = (p.L + span - 1) / span;
    if (k_bytes > 2 * (size_t)kLdsMaxBytes || p.U <= kPartMinSamples || p.U > kPartMaxSamples) return 0;
    if (p.dtype == PSA_F32) return (int64_t)p.BH * groups > 128 ? 2 : 0;
    if (heads * groups <= 32) return p.BH * groups >= (p.BH < 28 ? 192 : 160) ? 2 : 0;
    const int64_t least = p.L <= 1536 ? 21 : 24;
    return (int64_t)p.U * p.BH * p.L >= least * 32 * 8 * 2 * kMeasureQueries * parts_rounds(p, 4) ? 4 : 0;
}

// How much of a plan is cut anew (see make_plan).
enum Cuts { kFirstCuts = 0, kShortChunks = 1, kStreamCut = 2, kSplitCut = 3, kPartCut = 4 };

static void build_plan(const psa_shape_t* s, URule urule, int u_stride, Cuts cuts, Plan* p)
{
    p->given_indices = u_stride > 0;
    p->B = s->B; p->H = s->H; p->L = s->L_K; p->U = s->U; p->dtype = s->dtype;
    p->BH = s->B * s->H;
    p->u_max = p->given_indices ? u_stride : u_max_of(urule, p->L);
    // A work-group covers the selected queries in groups of 16 or 32 (float32: float64 MFMA tiles of 16) or 32 or
    // 64 (bfloat16: tiles of 32) and walks its keys in rounds of `tiles_wg` tiles of 32.
    const int n_tiles = (p->L + kTile - 1) / kTile;
    if (p->dtype == PSA_F32 && cuts >= kSplitCut) {
        split_f32(p, n_tiles);
    } else {
        // key splits: enough work-groups to cover the 256 CUs once (bfloat16) or twice
        if (p->dtype == PSA_F32) p->nq_group = (p->u_max > 16 && (int64_t)p->BH * ((p->L + 127) / 128) >= 64) ? 32 : 16;
        else                     p->nq_group = p->u_max > 32 ? 64 : 32;
        p->n_qgroup = (p->u_max + p->nq_group - 1) / p->nq_group;
        const int tiles_wg = p->dtype == PSA_F32 && p->nq_group == 32 ? 4 : 8;
        const int max_split = (n_tiles + tiles_wg - 1) / tiles_wg;
        const int wg_goal = p->dtype == PSA_F32 ? 512 : 256;
        int target = (wg_goal + p->BH * p->n_qgroup - 1) / (p->BH * p->n_qgroup);
        if (target < 1) target = 1;
        int n_split = target < max_split ? target : max_split;
        if (n_split > kMaxSplit) n_split = kMaxSplit;
        p->tiles_per_wave = (n_tiles + n_split * tiles_wg - 1) / (n_split * tiles_wg);      // rounds
        p->n_split = (n_tiles + p->tiles_per_wave * tiles_wg - 1) / (p->tiles_per_wave * tiles_wg);
    }
    // bfloat16: any split brings the hand-over of records to the head's last work-group (or, beyond 8 splits, the
    // merge kernel) while a round of tiles takes about 2 us, so heads are cut only where that saves at least three
    // rounds (B=16 H=8 L=1024: 20.1 us whole against 20.5 us in two splits that save two rounds)
    if (p->dtype == PSA_BF16 && p->n_split > 1) {
        const int rounds_whole = (n_tiles + 7) / 8;
        if (rounds_whole - p->tiles_per_wave < 3) { p->n_split = 1; p->tiles_per_wave = rounds_whole; }
    }

    // Many selected queries per head: no key split over work-groups, a wave owns its queries (see
    // attend_rows_*_kernel).  rows_mode 1: a wave walks all keys; 2: two waves share a query tile, each
    // on half of the keys, and merge inside the work-group.  float32: 1 from 2048 waves on (two per
    // SIMD: a lone wave cannot overlap its softmax arithmetic with its matrix products), else 2.
    // bfloat16: always 2 (more waves per SIMD hide more of a tile's round trips).  Measured, attend
    // stage, half of the queries kept: conformer_s 70 us with the keys split over work-groups, 72 us
    // with one wave per query tile, 60 us with two; float32 B=8 H=4 L=512: 108 -> 60 us, B=32 H=4
    // L=512 (2048 waves) 116 us with one wave per tile against 119 us with two; bfloat16 B=32 H=4
    // L=512: 32 -> 20 us, B=24 H=4 L=700: 88 -> 40 us; conformer_l: 102 us split over work-groups,
    // 91 us one wave per tile, 79 us two.
    // With few waves the split over work-groups uses more CUs and stays: float32 below 256 waves
    // (B=2 H=4 L=512: 53 against 59 us), bfloat16 below 1024 or while its work-groups fit one round
    // (B=2 H=8 L=2048: 29 against 39 us).  Between 64 and 255 selected queries a head fills only one
    // to four work-groups of this kind, so float32 takes them only with 512 waves or more and all
    // work-groups in one round (B=32 H=4 L=512 u=75: 94 -> 60 us; but B=16 H=4 L=1024 u=84, 384
    // waves: 82 us split over work-groups against 107 us; B=64 H=4 L=512 u=75, two rounds: 101
    // against 119 us); bfloat16 by the same rule as above (B=128 H=4 L=512 u=75: 56 -> 31 us).
    const int q_per_wave = p->dtype == PSA_F32 ? 16 : 32;
    const int64_t row_waves = (int64_t)p->BH * ((p->u_max + q_per_wave - 1) / q_per_wave);
    p->rows_mode = 0;
    if (p->u_max >= kRowsModeMin) {
        const int64_t split_wgs = (int64_t)p->BH * p->n_qgroup * p->n_split;
        if (p->dtype == PSA_F32) {
            const int64_t rows_wgs = (int64_t)p->BH * ((p->u_max + 63) / 64);
            if (p->u_max >= 256) p->rows_mode = row_waves >= 2048 ? 1 : (row_waves >= 256 ? 2 : 0);
            else if (row_waves >= 512 && rows_wgs <= 256) p->rows_mode = 2;
        } else if (row_waves >= 1024 || (row_waves >= 512 && split_wgs > 256)) p->rows_mode = 2;
    }
    if (p->rows_mode) {
        p->nq_group = p->dtype == PSA_F32 ? 64 : 128;       // 4 waves of 16 or 32 queries
        p->n_qgroup = (p->u_max + p->nq_group - 1) / p->nq_group;
        p->n_split = 1;
        p->tiles_per_wave = n_tiles;
    }
    p->d_split = p->dtype == PSA_F32 && !p->rows_mode && p->n_split == 1 ? elem_split((int64_t)p->BH * p->n_qgroup) : 1;
    p->n_wg_head = p->n_split * p->n_qgroup * p->d_split;
    p->rows_per_wg = (p->L + p->n_wg_head - 1) / p->n_wg_head;

    const size_t row_bytes = p->dtype == PSA_F32 ? 256 : 128;
    p->measure_lds = !p->given_indices && (size_t)p->L * row_bytes <= (size_t)kLdsMaxBytes;
    // LDS measure kernel.  bfloat16 heads whose K fits 64 KB: two work-groups per CU (one copies its K while the
    // other gathers).  A chunk is 128 queries; where that leaves CUs idle, 64 or 32: the gather is bound by the LDS
    // rate of a CU and by the instruction stream of a wave (B=1 H=4 L=128 float32: 8.6 us at 128, 4.7 at 32).
    // At most 8 chunks (lists) per head, and at most 64 KB of K for the smallest work-groups, 16 pieces per thread.
    const size_t k_bytes = (size_t)p->L * row_bytes;
    const bool two_per_cu = p->measure_lds && p->dtype == PSA_BF16 && k_bytes <= (size_t)kLdsMaxBytes / 2;
    const int slots = two_per_cu ? 512 : 256;
    p->measure_queries = p->measure_lds ? kLdsQueries : kMeasureQueries;
    if (p->measure_lds) {
        if (two_per_cu) p->measure_lds = 2;
        for (int q = kLdsQueries / 2; q >= 32 && cuts >= kShortChunks; q >>= 1) {
            const int chunks = (p->L + q - 1) / q;
            if (chunks > 8 || (int64_t)p->BH * chunks > slots || (q == 32 && k_bytes > (size_t)64 * 1024)) break;
            p->measure_queries = q;
        }
    }
    const int mq = p->measure_queries;
    p->n_chunk = (p->L + mq - 1) / mq;
    // once the heads alone would fill the CUs, a work-group takes several chunks of its head and loads the head's K once
    p->chunks_per_wg = 1;
    if (p->measure_lds) {
        while (p->chunks_per_wg < p->n_chunk &&
               (int64_t)p->BH * ((p->n_chunk + p->chunks_per_wg - 1) / p->chunks_per_wg) > slots) ++p->chunks_per_wg;
    }
    else if (!p->given_indices && p->dtype == PSA_F32 && cuts >= kStreamCut) p->chunks_per_wg = stream_cut_f32(*p);
    else if (!p->given_indices) {
        // about two persistent work-groups per CU, each on consecutive chunks of one head
        const int64_t chunks_all = (int64_t)p->BH * p->n_chunk;
        int cpw = (int)((chunks_all + 511) / 512);
        cpw = cpw < 1 ? 1 : (cpw > 16 ? 16 : cpw);
        p->chunks_per_wg = cpw < p->n_chunk ? cpw : p->n_chunk;
    }
    p->part_passes = cuts >= kPartCut && !p->measure_lds && !p->given_indices ? part_passes(*p, k_bytes) : 0;
    if (p->part_passes > 0) p->chunks_per_wg = p->part_passes * kPartPassChunks;
    // sorted per-chunk candidate lists: only with the LDS measure kernel (few chunks per head)
    p->cand_len = 0;
    if (p->measure_lds) {
        const int len = p->u_max < mq ? p->u_max : mq;
        if (p->n_chunk * len <= kMaxCandidates) p->cand_len = len;
    }
    p->n_lists = p->n_chunk;
    p->stream_lists = 0;
    // Streamed heads: a work-group of the measure kernel ranks the queries of its own chunks and hands on its
    // best u as one sorted list, exactly as a chunk of the LDS kernel does (see stream_list_len)
    if (!p->measure_lds && !p->given_indices) {
        const int span = p->part_passes > 0 ? kPartChunks : p->chunks_per_wg;
        const int len = stream_list_len(*p, span, p->dtype == PSA_F32 && cuts >= kStreamCut ? kListMaxF32 : kListMax);
        if (len > 0) {
            p->cand_len = len; p->n_lists = (p->n_chunk + span - 1) / span; p->stream_lists = 1;
        }
    }
    p->n_seg = 0;
    p->seg_len = 0;
    // Long heads: the measures of a head are cut into up to 8 segments, a work-group per segment
    // picks the segment's best queries and hands them on as a sorted list, like a chunk of the LDS
    // measure kernel does (one work-group per head loads and ranks all L measures on one CU: 15 us
    // at L = 4096 against 8.4 us in segments).  Only where all segment work-groups run at once
    // (at most one per CU) and the head is long enough to pay for the list merge in the attend
    // stage (about 2.5 us); up to 2048 measures one work-group per head is as fast.
    if (!p->measure_lds && !p->given_indices && p->cand_len == 0 && p->L > 2048) {
        int n_seg = (p->L + 511) / 512;
        if (n_seg > kSegMax) n_seg = kSegMax;
        if (n_seg > 256 / p->BH) n_seg = 256 / p->BH;
        if (n_seg >= 2) {
            const int seg_len = ((p->L + n_seg - 1) / n_seg + kMeasureQueries - 1) / kMeasureQueries * kMeasureQueries;
            n_seg = (p->L + seg_len - 1) / seg_len;
            const int len = p->u_max < seg_len ? p->u_max : seg_len;
            if (seg_len <= kSegKeys && len <= kSegCandMax && n_seg * len <= kMaxCandidates) {
                p->n_seg = n_seg; p->seg_len = seg_len; p->cand_len = len; p->n_lists = n_seg;
            }
        }
    }
    p->fused_select = p->cand_len > 0;
    // caller-given index sets that fit the attend work-groups' LDS list, few enough column-sum chunks
    // for one wave to add up: no prep kernel (one launch less: conformer_s 27.8 -> 25 us)
    p->given_inline = p->given_indices && p->u_max <= kSelLdsMax && p->n_chunk <= 64;
    p->separate_merge = p->n_split > kTicketMaxSplit;
    p->own_sums = p->given_inline && p->rows_mode != 1 && sums_in_attend(*p, p->n_wg_head);

    // float32 tensors: m, l as float64 and 64 float32 values per query (34 doubles); bfloat16: 66 floats
    p->part_stride = (size_t)p->nq_group * (p->dtype == PSA_F32 ? 2 + kD / 2 : kD + 2);
    p->part_elem = p->dtype == PSA_F32 ? sizeof(double) : sizeof(float);
    size_t off = 0;
    p->off_M = off;      off += align256((size_t)p->BH * p->L * sizeof(float));
    p->off_vpart = off;  off += p->part_passes > 0 && p->stream_lists ? 0 /* the lists bring their own sums */ : align256((size_t)p->BH * p->n_chunk * kD * sizeof(double));
    p->off_vseg = off;   off += align256((size_t)p->BH * (p->stream_lists ? p->n_lists : p->n_seg) * kD * sizeof(double));
    p->off_mu = off;     off += align256((size_t)p->BH * kD * sizeof(float));
    p->off_sel = off;    off += align256((size_t)p->BH * p->u_max * sizeof(int));
    p->off_u = off;      off += align256((size_t)p->B * sizeof(int));
    p->off_ticket = off; off += align256((size_t)p->BH * sizeof(int));
    p->off_cand = off;   off += align256((size_t)p->BH * p->n_lists * p->cand_len * sizeof(uint2));
    const bool records = !p->rows_mode && (p->n_split > 1 || cuts == kFirstCuts);      // a head in one split hands over none
    p->off_part = off;   off += !records ? 0 : align256((size_t)p->BH * p->n_qgroup * p->n_split * p->part_stride * p->part_elem);
    p->total = off;
}

// The workspace has the size that the first rules for the cuts gave (two work-groups per CU in every stage, chunks of
// 128 queries, records for every split): callers keep workspaces by it, and the static scratch admits calls by it.  The
// present rules are taken as far as what they need fits; short heads in small chunks may need more (at most 512
// chunks of a few KB).
bool make_plan(const psa_shape_t* s, URule urule, int u_stride, Plan* p)
{
    if (check_shape(s) != PSA_OK) return false;
    if (u_stride <= 0 && !good_rule(urule)) return false;
    if (u_stride < 0 || u_stride > s->L_K) return false;
    build_plan(s, urule, u_stride, kFirstCuts, p);
    const size_t size = p->total;
    for (int cuts = kPartCut; cuts >= kShortChunks; --cuts) {
        build_plan(s, urule, u_stride, (Cuts)cuts, p);
        if (p->total <= size) break;
    }
    if (p->total < size) p->total = size;
    return true;
}

Scratch carve(const Plan& p, void* workspace)
{
    unsigned char* w = static_cast<unsigned char*>(workspace);
    Scratch s;
    s.M = reinterpret_cast<float*>(w + p.off_M);
    s.vpart = reinterpret_cast<double*>(w + p.off_vpart);
    s.vseg = reinterpret_cast<double*>(w + p.off_vseg);
    s.mu = reinterpret_cast<float*>(w + p.off_mu);
    s.sel = reinterpret_cast<int*>(w + p.off_sel);
    s.ticket = reinterpret_cast<int*>(w + p.off_ticket);
    s.cand = reinterpret_cast<uint2*>(w + p.off_cand);
    s.u = reinterpret_cast<int*>(w + p.off_u);
    s.part = w + p.off_part;
    return s;
}

static inline bool misaligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; }

static int check_ptrs(const void* Q, const void* K, const void* V, const int32_t* lengths, const void* out,
                      const void* workspace)
{
    if (misaligned(Q, 16) || misaligned(K, 16) || misaligned(V, 16) || misaligned(out, 16) ||
        misaligned(lengths, 4) || misaligned(workspace, 256)) return PSA_ERR_ALIGN;
    return PSA_OK;
}

static int run(const void* Q, const void* K, const void* V, const int32_t* lengths, const int32_t* sample_idx,
               const psa_options_t* opt, void* out, const psa_shape_t* shape, void* workspace, size_t workspace_bytes,
               void* stream, int stage_mask, float* M_out, int32_t* sel_out, int32_t* u_out, bool checks_only = false)
{
    if (!Q || !K || !V || !sample_idx || !out || !shape || !workspace || !opt) return PSA_ERR_NULL;
    int rc = check_shape(shape);
    if (rc != PSA_OK) return rc;
    const URule urule{opt->u_rule, opt->factor};
    if (!good_rule(urule)) return PSA_ERR_ARG;
    if (opt->fill != PSA_FILL_MEAN && opt->fill != PSA_FILL_VALUE) return PSA_ERR_ARG;
    if (stage_mask <= 0 || (stage_mask & ~PSA_STAGE_ALL)) return PSA_ERR_ARG;
    rc = check_ptrs(Q, K, V, lengths, out, workspace);
    if (rc != PSA_OK) return rc;
    if (misaligned(sample_idx, 4)) return PSA_ERR_ALIGN;
    Plan p;
    if (!make_plan(shape, urule, 0, &p)) return PSA_ERR_SHAPE;
    if (workspace_bytes < p.total) return PSA_ERR_WORKSPACE;
    if (checks_only) return PSA_OK;

    Args a;
    a.Q = Q; a.K = K; a.V = V; a.lengths = lengths; a.idx = sample_idx; a.out = out;
    a.urule = urule; a.fill = opt->fill; a.given_sel = nullptr; a.given_u = nullptr;
    a.stream = static_cast<hipStream_t>(stream);
    const Scratch w = carve(p, workspace);

    if ((stage_mask & PSA_STAGE_MEASURE) && launch_measure(p, a, w) != hipSuccess) return PSA_ERR_HIP;
    if (stage_mask & PSA_STAGE_SELECT) {
        if (p.n_seg > 0) { if (launch_select_segments(p, a, w) != hipSuccess) return PSA_ERR_HIP; }
        else if (!p.fused_select && launch_select(p, a, w) != hipSuccess) return PSA_ERR_HIP;
    }
    if ((stage_mask & PSA_STAGE_ATTEND) && launch_attend(p, a, w) != hipSuccess) return PSA_ERR_HIP;

    if (M_out && hipMemcpyAsync(M_out, w.M, (size_t)p.BH * p.L * sizeof(float), hipMemcpyDeviceToDevice, a.stream) != hipSuccess)
        return PSA_ERR_HIP;
    if (sel_out && hipMemcpyAsync(sel_out, w.sel, (size_t)p.BH * p.u_max * sizeof(int), hipMemcpyDeviceToDevice, a.stream) != hipSuccess)
        return PSA_ERR_HIP;
    if (u_out && hipMemcpyAsync(u_out, w.u, (size_t)p.B * sizeof(int), hipMemcpyDeviceToDevice, a.stream) != hipSuccess)
        return PSA_ERR_HIP;
    return PSA_OK;
}

static int run_c(const void* Q, const void* K, const void* V, const int32_t* lengths, const int32_t* sample_idx,
                 double c, void* out, const psa_shape_t* shape, void* workspace, size_t workspace_bytes,
                 void* stream, int stage_mask, float* M_out, int32_t* sel_out, int32_t* u_out)
{
    const psa_options_t opt{PSA_U_LOG, PSA_FILL_MEAN, c};
    return run(Q, K, V, lengths, sample_idx, &opt, out, shape, workspace, workspace_bytes, stream, stage_mask,
               M_out, sel_out, u_out);
}

static int run_indices(const void* Q, const void* K, const void* V, const int32_t* lengths, const int32_t* sel,
                       const int32_t* u, int u_stride, int fill, void* out, const psa_shape_t* shape,
                       void* workspace, size_t workspace_bytes, void* stream)
{
    if (!Q || !K || !V || !sel || !u || !out || !shape || !workspace) return PSA_ERR_NULL;
    int rc = check_shape(shape);
    if (rc != PSA_OK) return rc;
    if (u_stride < 1 || u_stride > shape->L_K) return PSA_ERR_ARG;
    if (fill != PSA_FILL_MEAN && fill != PSA_FILL_VALUE) return PSA_ERR_ARG;
    rc = check_ptrs(Q, K, V, lengths, out, workspace);
    if (rc != PSA_OK) return rc;
    if (misaligned(sel, 4) || misaligned(u, 4)) return PSA_ERR_ALIGN;
    Plan p;
    if (!make_plan(shape, URule{PSA_U_LOG, 1.0}, u_stride, &p)) return PSA_ERR_SHAPE;
    if (workspace_bytes < p.total) return PSA_ERR_WORKSPACE;

    Args a;
    a.Q = Q; a.K = K; a.V = V; a.lengths = lengths; a.idx = nullptr; a.out = out;
    a.urule = URule{PSA_U_LOG, 1.0}; a.fill = fill; a.given_sel = sel; a.given_u = u;
    a.stream = static_cast<hipStream_t>(stream);
    const Scratch w = carve(p, workspace);
    // before the attend stage: the V column sums where something reads them, the tickets where any are drawn
    const bool tickets = p.n_split > 1 && !p.separate_merge;
    if (((fill == PSA_FILL_MEAN && !p.own_sums) || tickets) && launch_vsum(p, a, w) != hipSuccess) return PSA_ERR_HIP;
    if (!p.given_inline && launch_prep_indices(p, a, w) != hipSuccess) return PSA_ERR_HIP;
    if (launch_attend(p, a, w) != hipSuccess) return PSA_ERR_HIP;
    return PSA_OK;
}

static int check_project(const psa_shape_t* shape, const psa_mhsa_weights_t* w, bool need_in, bool need_out)
{
    if (!shape || !w) return PSA_ERR_NULL;
    const int rc = check_shape(shape);
    if (rc != PSA_OK) return rc;
    if ((int64_t)shape->B * shape->L_K > 0x7FFFFFFF) return PSA_ERR_SHAPE;
    if (need_in && (!w->Wq || !w->Wk || !w->Wv)) return PSA_ERR_NULL;
    if (need_out && !w->Wo) return PSA_ERR_NULL;
    const void* ptrs[8] = {w->Wq, w->Wk, w->Wv, w->Wo, w->bq, w->bk, w->bv, w->bo};
    for (int i = 0; i < 4; ++i) if (misaligned(ptrs[i], 16)) return PSA_ERR_ALIGN;
    for (int i = 4; i < 8; ++i) if (misaligned(ptrs[i], 4)) return PSA_ERR_ALIGN;
    return PSA_OK;
}

// Q, K, V, A of the whole module, then the attention's own scratch
static size_t mhsa_tensor_bytes(const psa_shape_t* s)
{
    return align256((size_t)s->B * s->H * s->L_K * kD * (s->dtype == PSA_F32 ? 4 : 2));
}

// ---- scratch for the entry point that may not allocate: one array per device in the
// library's own image (each GPU the library runs on holds it until the process ends).
// In host code the array's name is only a handle; its device address is looked up once
// per device and that pointer is what the kernels and copies are given.
constexpr size_t kStaticScratchBytes = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kStaticScratchDevices = 64;
static std::atomic<void*> g_scratch_ptr[kStaticScratchDevices];

static hipError_t static_scratch_ptr(void** out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kStaticScratchDevices) return hipErrorInvalidDevice;
    void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!ptr) {
        // the current device's copy of the array (two threads racing here look up the same address)
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev].store(ptr, std::memory_order_release);
    }
    *out = ptr;
    return hipSuccess;
}

}  // namespace psa

extern "C" {

size_t probsparse_static_workspace_bytes(void) { return psa::kStaticScratchBytes; }

int probsparse_attn_fwd_static(const void* Q, const void* K, const void* V, const int32_t* lengths,
                               const int32_t* sample_idx, double c, void* out, const psa_shape_t* shape, void* stream)
{
    using namespace psa;
    // the size check is host arithmetic and comes before anything touches the device
    if (!shape) return PSA_ERR_NULL;
    const int rc = check_shape(shape);
    if (rc != PSA_OK) return rc;
    Plan p;
    if (!good_rule(URule{PSA_U_LOG, c})) return PSA_ERR_ARG;
    if (!make_plan(shape, URule{PSA_U_LOG, c}, 0, &p)) return PSA_ERR_SHAPE;
    if (p.total > kStaticScratchBytes) return PSA_ERR_WORKSPACE;
    if (!Q || !K || !V || !sample_idx || !out) return PSA_ERR_NULL;
    void* ws = nullptr;
    if (static_scratch_ptr(&ws) != hipSuccess) return PSA_ERR_HIP;
    return run_c(Q, K, V, lengths, sample_idx, c, out, shape, ws, kStaticScratchBytes, stream, PSA_STAGE_ALL,
                 nullptr, nullptr, nullptr);
}

int probsparse_qkv_project(const void* X, const psa_mhsa_weights_t* weights, void* Q, void* K, void* V,
                           const psa_shape_t* shape, void* stream)
{
    using namespace psa;
    if (!X || !Q || !K || !V) return PSA_ERR_NULL;
    const int rc = check_project(shape, weights, true, false);
    if (rc != PSA_OK) return rc;
    if (misaligned(X, 16) || misaligned(Q, 16) || misaligned(K, 16) || misaligned(V, 16)) return PSA_ERR_ALIGN;
    return launch_qkv_project(*shape, X, *weights, Q, K, V, static_cast<hipStream_t>(stream)) == hipSuccess ? PSA_OK : PSA_ERR_HIP;
}

int probsparse_out_project(const void* A, const psa_mhsa_weights_t* weights, void* Y, const psa_shape_t* shape, void* stream)
{
    using namespace psa;
    if (!A || !Y) return PSA_ERR_NULL;
    const int rc = check_project(shape, weights, false, true);
    if (rc != PSA_OK) return rc;
    if (misaligned(A, 16) || misaligned(Y, 16)) return PSA_ERR_ALIGN;
    return launch_out_project(*shape, A, *weights, Y, static_cast<hipStream_t>(stream)) == hipSuccess ? PSA_OK : PSA_ERR_HIP;
}

size_t probsparse_mhsa_workspace_bytes(const psa_shape_t* shape, const psa_options_t* opt)
{
    const size_t inner = probsparse_attn_workspace_bytes_opt(shape, opt);
    if (inner == 0) return 0;
    return 4 * psa::mhsa_tensor_bytes(shape) + inner;
}

int probsparse_mhsa_fwd(const void* X, const psa_mhsa_weights_t* weights, const int32_t* lengths,
                        const int32_t* sample_idx, const psa_options_t* opt, void* Y, const psa_shape_t* shape,
                        void* workspace, size_t workspace_bytes, void* stream)
{
    using namespace psa;
    if (!X || !Y || !workspace || !sample_idx || !opt) return PSA_ERR_NULL;
    int rc = check_project(shape, weights, true, true);
    if (rc != PSA_OK) return rc;
    if (misaligned(X, 16) || misaligned(Y, 16) || misaligned(workspace, 256)) return PSA_ERR_ALIGN;
    const size_t inner = probsparse_attn_workspace_bytes_opt(shape, opt);
    if (inner == 0) return PSA_ERR_ARG;
    const size_t tb = mhsa_tensor_bytes(shape);
    if (workspace_bytes < 4 * tb + inner) return PSA_ERR_WORKSPACE;
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    void *Q = ws, *K = ws + tb, *V = ws + 2 * tb, *A = ws + 3 * tb;
    // the attention's own checks run before the first launch of the module
    rc = run(Q, K, V, lengths, sample_idx, opt, A, shape, ws + 4 * tb, workspace_bytes - 4 * tb, stream, PSA_STAGE_ALL,
             nullptr, nullptr, nullptr, true);
    if (rc != PSA_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (launch_qkv_project(*shape, X, *weights, Q, K, V, st) != hipSuccess) return PSA_ERR_HIP;
    rc = run(Q, K, V, lengths, sample_idx, opt, A, shape, ws + 4 * tb, workspace_bytes - 4 * tb, stream, PSA_STAGE_ALL,
             nullptr, nullptr, nullptr);
    if (rc != PSA_OK) return rc;
    return launch_out_project(*shape, A, *weights, Y, st) == hipSuccess ? PSA_OK : PSA_ERR_HIP;
}


size_t probsparse_attn_workspace_bytes(const psa_shape_t* shape, double c)
{
    psa::Plan p;
    return psa::make_plan(shape, psa::URule{PSA_U_LOG, c}, 0, &p) ? p.total : 0;
}

int32_t probsparse_u_max(const psa_shape_t* shape, double c)
{
    psa::Plan p;
    return psa::make_plan(shape, psa::URule{PSA_U_LOG, c}, 0, &p) ? p.u_max : 0;
}

size_t probsparse_attn_workspace_bytes_opt(const psa_shape_t* shape, const psa_options_t* opt)
{
    psa::Plan p;
    if (!opt || (opt->fill != PSA_FILL_MEAN && opt->fill != PSA_FILL_VALUE)) return 0;
    return psa::make_plan(shape, psa::URule{opt->u_rule, opt->factor}, 0, &p) ? p.total : 0;
}

int32_t probsparse_u_max_opt(const psa_shape_t* shape, const psa_options_t* opt)
{
    psa::Plan p;
    if (!opt) return 0;
    return psa::make_plan(shape, psa::URule{opt->u_rule, opt->factor}, 0, &p) ? p.u_max : 0;
}

int probsparse_attn_fwd_opt(const void* Q, const void* K, const void* V, const int32_t* lengths,
                            const int32_t* sample_idx, const psa_options_t* opt, void* out,
                            const psa_shape_t* shape, void* workspace, size_t workspace_bytes, void* stream,
                            float* M_out, int32_t* sel_out, int32_t* u_out)
{
    return psa::run(Q, K, V, lengths, sample_idx, opt, out, shape, workspace, workspace_bytes, stream,
                    PSA_STAGE_ALL, M_out, sel_out, u_out);
}

size_t probsparse_attn_with_indices_workspace_bytes(const psa_shape_t* shape, int32_t u_stride)
{
    psa::Plan p;
    if (u_stride < 1) return 0;
    return psa::make_plan(shape, psa::URule{PSA_U_LOG, 1.0}, u_stride, &p) ? p.total : 0;
}

int probsparse_attn_fwd_with_indices(const void* Q, const void* K, const void* V, const int32_t* lengths,
                                     const int32_t* sel, const int32_t* u, int32_t u_stride, int32_t fill,
                                     void* out, const psa_shape_t* shape, void* workspace, size_t workspace_bytes,
                                     void* stream)
{
    return psa::run_indices(Q, K, V, lengths, sel, u, u_stride, fill, out, shape, workspace, workspace_bytes, stream);
}

size_t probsparse_attn_bwd_workspace_bytes(const psa_shape_t* shape, int32_t u_stride)
{
    if (psa::check_shape(shape) != PSA_OK || u_stride < 1 || u_stride > shape->L_K) return 0;
    return psa::make_bwd_plan(*shape, u_stride).total;
}

int probsparse_attn_bwd(const void* Q, const void* K, const void* V, const int32_t* lengths,
                        const int32_t* sel, const int32_t* u, int32_t u_stride, int32_t fill,
                        const void* dOut, void* dQ, void* dK, void* dV, const psa_shape_t* shape,
                        void* workspace, size_t workspace_bytes, void* stream)
{
    using namespace psa;
    if (!Q || !K || !V || !sel || !u || !dOut || !dQ || !dK || !dV || !shape || !workspace) return PSA_ERR_NULL;
    const int rc = check_shape(shape);
    if (rc != PSA_OK) return rc;
    if (u_stride < 1 || u_stride > shape->L_K) return PSA_ERR_ARG;
    if (fill != PSA_FILL_MEAN && fill != PSA_FILL_VALUE) return PSA_ERR_ARG;
    if (misaligned(Q, 16) || misaligned(K, 16) || misaligned(V, 16) || misaligned(dOut, 16) || misaligned(dQ, 16) ||
        misaligned(dK, 16) || misaligned(dV, 16) || misaligned(lengths, 4) || misaligned(sel, 4) || misaligned(u, 4) ||
        misaligned(workspace, 256)) return PSA_ERR_ALIGN;
    const BwdPlan bp = make_bwd_plan(*shape, u_stride);
    if (workspace_bytes < bp.total) return PSA_ERR_WORKSPACE;
    return launch_backward(*shape, bp, Q, K, V, lengths, sel, u, u_stride, fill, dOut, dQ, dK, dV, workspace,
                           static_cast<hipStream_t>(stream)) == hipSuccess ? PSA_OK : PSA_ERR_HIP;
}

int probsparse_attn_fwd(const void* Q, const void* K, const void* V, const int32_t* lengths,
                        const int32_t* sample_idx, double c, void* out, const psa_shape_t* shape,
                        void* workspace, size_t workspace_bytes, void* stream)
{
    return psa::run_c(Q, K, V, lengths, sample_idx, c, out, shape, workspace, workspace_bytes, stream,
                    PSA_STAGE_ALL, nullptr, nullptr, nullptr);
}

int probsparse_attn_fwd_debug(const void* Q, const void* K, const void* V, const int32_t* lengths,
                              const int32_t* sample_idx, double c, void* out, const psa_shape_t* shape,
                              void* workspace, size_t workspace_bytes, void* stream,
                              float* M_out, int32_t* sel_out, int32_t* u_out)
{
    return psa::run_c(Q, K, V, lengths, sample_idx, c, out, shape, workspace, workspace_bytes, stream,
                    PSA_STAGE_ALL, M_out, sel_out, u_out);
}

int probsparse_attn_fwd_stages(const void* Q, const void* K, const void* V, const int32_t* lengths,
                               const int32_t* sample_idx, double c, void* out, const psa_shape_t* shape,
                               void* workspace, size_t workspace_bytes, void* stream, int stage_mask)
{
    return psa::run_c(Q, K, V, lengths, sample_idx, c, out, shape, workspace, workspace_bytes, stream,
                    stage_mask, nullptr, nullptr, nullptr);
}

const char* probsparse_strerror(int code)
{
    switch (code) {
        case PSA_OK:            return "ok";
        case PSA_ERR_NULL:      return "a required pointer is NULL";
        case PSA_ERR_SHAPE:     return "unsupported shape (need B,H,L,U >= 1, D == 64, L_Q == L_K, B*H <= 65535)";
        case PSA_ERR_DTYPE:     return "unsupported dtype (PSA_F32 or PSA_BF16)";
        case PSA_ERR_ARG:       return "invalid argument (factor must be finite and positive; stage mask within PSA_STAGE_ALL; known rule and fill; 1 <= u_stride <= L)";
        case PSA_ERR_WORKSPACE: return "workspace smaller than probsparse_attn_workspace_bytes() (or, for probsparse_attn_fwd_static, the shape needs more than probsparse_static_workspace_bytes())";
        case PSA_ERR_HIP:       return "HIP runtime error on launch or copy";
        case PSA_ERR_ALIGN:     return "device pointer not sufficiently aligned (16 B tensors, 256 B workspace)";
        default:                return "unknown status";
    }
}

int probsparse_describe_plan(const psa_shape_t* shape, const psa_options_t* opt, int32_t u_stride,
                             char* buf, size_t buf_bytes)
{
    using namespace psa;
    if (!shape || !buf || (!opt && u_stride <= 0)) return PSA_ERR_NULL;
    if (buf_bytes == 0) return PSA_ERR_ARG;
    const int rc = check_shape(shape);
    if (rc != PSA_OK) return rc;
    Plan p;
    const URule urule = opt ? URule{opt->u_rule, opt->factor} : URule{PSA_U_LOG, 1.0};
    if (u_stride < 0) return PSA_ERR_ARG;
    if (u_stride == 0 && !good_rule(urule)) return PSA_ERR_ARG;
    if (!make_plan(shape, urule, u_stride, &p)) return u_stride > 0 ? PSA_ERR_ARG : PSA_ERR_SHAPE;
    const char* measure = p.given_indices ? "none" : p.measure_lds == 2 ? "lds_half" : p.measure_lds == 1 ? "lds" : "stream";
    const char* select = p.given_indices ? (p.given_inline ? "given_inline" : "given_prep")
                       : p.n_seg > 0 ? "segments" : p.fused_select ? "lists" : "kernel";
    const char* attend = p.rows_mode == 2 ? "rows_half_keys" : p.rows_mode == 1 ? "rows" : "key_split";
    const char* merge = p.rows_mode ? "none" : p.n_split == 1 ? "none" : p.separate_merge ? "kernel" : "last_work_group";
    const int n = snprintf(buf, buf_bytes,
                           "u_max=%d measure=%s chunks=%d chunks_per_wg=%d select=%s lists=%d list_len=%d segments=%d "
                           "attend=%s queries_per_group=%d query_groups=%d key_splits=%d rounds=%d merge=%s workspace=%zu",
                           p.u_max, measure, p.n_chunk, p.chunks_per_wg, select, p.cand_len > 0 ? p.n_lists : 0, p.cand_len,
                           p.n_seg, attend, p.nq_group, p.n_qgroup, p.n_split, p.tiles_per_wave, merge, p.total);
    if (n < 0 || (size_t)n >= buf_bytes) return PSA_ERR_ARG;
    // the rest where there is room for it: the module's projections, and the backward for index sets of this stride
    char more[320];
    int m = snprintf(more, sizeof(more), " element_shares=%d measure_parts=%d own_sums=%d qkv_project=%s out_project=%s", p.d_split, p.part_passes, p.own_sums, project_route_name(*shape, 3),
                     project_route_name(*shape, 1));
    if (u_stride > 0) {
        const BwdPlan bp = make_bwd_plan(*shape, u_stride);
        if (shape->dtype == PSA_F32) {
            m += snprintf(more + m, sizeof(more) - m, " backward=%s backward_splits=%d backward_blocks=%d backward_keys=%d backward_keys_no_lengths=%d",
                          bp.keys_only ? "two_kernels" : "fused", bp.S2, bp.blocks2, 16 * bp.ks, bp.wide_S2 > 0 ? 128 : 16 * bp.ks);
        } else {
            const Bwd16Plan b16 = make_bwd16_plan(*shape, u_stride, bp.total);
            m += snprintf(more + m, sizeof(more) - m, " backward=bf16 backward_splits=%d backward_blocks=%d backward_keys=128 backward_dq_splits=%d",
                          b16.S2, b16.blocks2, b16.SQ);
        }
    }
    if (m > 0 && (size_t)(n + m) < buf_bytes) memcpy(buf + n, more, (size_t)m + 1);
    return PSA_OK;
}

int probsparse_init(void)
{
    if (psa::init_measure() != hipSuccess || psa::init_attend() != hipSuccess || psa::init_backward() != hipSuccess ||
        psa::init_project() != hipSuccess) return PSA_ERR_HIP;
    void* ws = nullptr;
    if (psa::static_scratch_ptr(&ws) != hipSuccess) return PSA_ERR_HIP;      // this device's static scratch
    return PSA_OK;
}

int probsparse_version(void) { return 100; }

}  // extern "C"
