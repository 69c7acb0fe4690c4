// Integer rules that kernels and launchers share: who writes what, which index is read.  No device code and no HIP types, so
// that the same functions can be compiled and enumerated on the host (tests/test_kernel_rules.py).
#pragma once
#include <stddef.h>

#if defined(__HIPCC__)
#define SSD_HD __host__ __device__ __forceinline__
#else
#define SSD_HD inline
#endif

namespace ssdk {

// 16-row kernels, eight waves: the rows whose RMS scale wave `wave` writes.  Every row of the tile belongs to one wave.
template <typename F> SSD_HD void rows_of_wave(int wave, F&& f)
{
    for (int c = wave; c < 16; c += 8) f(c);
}

// Row of the embedding table that is read for token id `tok`, whatever the id holds: a caller's id, or the 0x7fffffff of a
// row of logits without a maximum.
SSD_HD size_t embed_row(int tok, int V) { return (size_t)(tok < 0 ? 0 : tok < V ? tok : V - 1); }

SSD_HD int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Weight rows per tile of the large-tile QKV launch: n_total rows (a multiple of 128), m_blocks blocks of 128 activation rows.
// What decides is the number of rounds that the blocks take on the CUs' slots -- one block per CU for 256- and 192-row
// tiles, two for 128-row ones -- after the cut along K that fills idle slots (up to four slices).  Time of a round, in
// those of 256-row tiles: 192-row ones 0.88 (whole launches of as many rounds, rotary epilogue and cache rows included, random
// data: 0.86 to 0.92), 128-row ones (two per slot) 1.2 to 1.6.  Measured, us: 7B, 512 rows: 256-row tiles 136.5, 192 121; 13B,
// 320 rows: 158, 138; 512 rows: 167, 256; width 4992, 512 rows: 192-row tiles 246, 128 217; 320 rows: 136, 203; width 3200, 384
// rows: 99.6, 87.1; 512 rows: 100.8, 141.
SSD_HD int qkv_tile_rows(int n_total, int m_blocks)
{
    int best = 128;
    double best_cost = 0.0;
    for (int t = 128; t <= 256; t += 64) {
        if (n_total % t) continue;
        const int slots = t == 128 ? 512 : 256, blocks = n_total / t * m_blocks;
        int ks = slots / blocks;
        ks = ks < 1 ? 1 : ks > 4 ? 4 : ks;
        const double cost = (double)ceil_div(blocks * ks, slots) / ks * (t == 128 ? 1.5 : t == 192 ? 0.88 : 1.0);
        if (t == 128 || cost <= best_cost) { best = t; best_cost = cost; }
    }
    return best;
}

// K slices of a large-tile launch of `blocks` blocks for `slots` of them at a time, `stripes` 64-wide stripes long: the least of an
// estimate of the launch and its finishing launch, in us.  A block costs 8 and 1.9 per stripe (128-row tiles, two to a CU: 2.85), the
// finishing launch 6 and its slices, of slice_bytes, at 4 TB/s.  More slices than fill the slots once pay where a last round would be
// nearly empty.  Measured, us, launch and finish, filling the slots at most once / so: 70B, 300 rows, gate/up 661 / 603, output and down
// projection 238 / 215 on average; 13B, 512 rows, keys and values 203 / 147.
SSD_HD int k_slices(int blocks, int slots, int stripes, double slice_bytes, int most)
{
    const double stripe = slots > 256 ? 2.85 : 1.9;
    int best = 1;
    double best_us = 0.0;
    for (int ks = 1; ks <= most && ks <= stripes; ks++) {
        const double us = ceil_div(blocks * ks, slots) * (8.0 + stripe * ceil_div(stripes, ks)) + (ks > 1 ? 6.0 + ks * slice_bytes / 4e6 : 0.0);
        if (ks == 1 || us < best_us) { best = ks; best_us = us; }
    }
    return best;
}

// ---- attention launch plan ---------------------------------------------------------------------------------------------
// Few query vectors per KV head (M x group size <= AW_MAXQ_TOTAL): the register-resident kernel over ranges of 64 positions
// and more -- a single CU pulls only a few tens of GB/s, so a head's cache is spread over many blocks even though that
// costs the fold of the partial results.  Many query vectors (prompt blocks, wide GQA groups): the LDS-staged kernel,
// which fetches K/V once for all of them.
constexpr int AT_CHUNK = 96;     // cache positions a block of the LDS-staged kernel owns (K and V of the chunk live in LDS together)
constexpr int GV_FOLD_MAX = 8;   // attention partials per head the output projection can fold itself
constexpr int AW_MAXQ_TOTAL = 4;
constexpr int AW_MAX_ROWS = 8;
constexpr int AW_RANGE_BYTES = 32 * 1024;   // K bytes of a range: one pass of the narrowest block shape (8 waves, 4 loads each)
constexpr int AW_MAX_RANGES = 16;

struct AttnShape { int G, Hkv, hd; bool kv_f32, w_f32; };   // query heads per KV head, KV heads, head size, element types
struct AttnPlan { bool wide; int n_splits; int chunk; bool defer_fold; };   // chunk: cache rows per range

// Plan for M rows of which the last one sees ctx positions.  force_splits, force_kernel: tuning hooks (0 = this rule).
inline AttnPlan attn_plan(const AttnShape& a, int ctx, int M, int force_splits, int force_kernel)
{
    AttnPlan pl;
    pl.defer_fold = false;
    const int Q = a.G * M;
    // More than 4 query vectors per KV head: the MFMA form of the LDS-staged kernel (12.9 us against 14.5 us at 5 rows,
    // 7B shape, 16-bit cache, fold included).  A model with fp32 WEIGHTS stays in fp32 arithmetic throughout: there a
    // few rows with 1, 2, 4 or 8 query heads per KV head run the register-resident kernel, one block per row and range
    // serving the row's group of heads (two blocks for a group of 8), re-reading a range's K/V from the cache.
    pl.wide = Q <= AW_MAXQ_TOTAL ||
              (a.kv_f32 && a.w_f32 && (a.G == 1 || a.G == 2 || a.G == 4 || a.G == 8) && M <= AW_MAX_ROWS);
    if (force_kernel == 1 || force_kernel == 3) pl.wide = false;
    if (!pl.wide) {
        pl.n_splits = ceil_div(ctx, AT_CHUNK);
        pl.chunk = AT_CHUNK;
        return pl;
    }
    // ranges of one pass of the narrowest block shape (128 positions of 16-bit 128-wide heads, 64 of fp32 ones) ..
    pl.chunk = AW_RANGE_BYTES / (a.hd * (a.kv_f32 ? 4 : 2));
    pl.n_splits = ceil_div(ctx, pl.chunk);
    // .. up to a limit: 16; for a single row what the output projection folds itself, up to 4 K positions (a longer range
    // costs the attention kernel about 1 us, a separate fold launch 5); for several query vectors per block, whose
    // registers leave one block per CU, what one round of blocks takes (two rows, 32 heads, about 550 positions: 7.9 us
    // with 7 ranges, as many as where the length comes from the position on the device; 12.7 with 9)
    int limit = AW_MAX_RANGES;
    if (M == 1 && ctx <= GV_FOLD_MAX * 512) limit = GV_FOLD_MAX;
    if (M > 1 && Q <= AW_MAXQ_TOTAL && 256 / a.Hkv < limit) limit = 256 / a.Hkv > 4 ? 256 / a.Hkv : 4;
    if (force_splits > 0) {
        pl.chunk = ceil_div(ctx, force_splits < ctx ? force_splits : ctx);
        pl.n_splits = ceil_div(ctx, pl.chunk);
    } else if (pl.n_splits > limit) {
        // Beyond it the ranges grow.  Their length is part of the launch, not computed from the position on the device
        // (that would put the load of the position in front of the first K and V loads), so a captured launch sequence
        // serves one length only.  Steps of 16 rows, one capture per 16 `limit` positions: a range's length is the time of its
        // block.  1024-wide, 24 layers, 1000 tokens from position 1024, ms with all captures / replays only: 712 / 708, with
        // four lengths per doubling 720 / 717, with the length computed on the device 742 / 740.
        pl.chunk = ceil_div(ceil_div(ctx, limit), 16) * 16;
        pl.n_splits = ceil_div(ctx, pl.chunk);
    }
    return pl;
}

// The same for a single row whose launch folds its partials itself (the last block of a head does): few KV heads leave most of the
// device idle with the eight ranges that the output projection folds, so a long context gets ranges of one pass, as many as
// give every CU a block, and longer ones beyond that.  Their number goes in steps of four (ranges behind the position are empty): one
// launch plan per four ranges.  Llama-3-8B widths (8 KV heads), us per layer beyond what 600 positions take, before / so: 16-bit cache, 2200
// positions 7.5 / 4, 3000 8 / 5.5, 4000 7.5 / 7, 6000 17.5 / 10, 9000 23.5 / 14.5; fp32 cache, 4000 13 / 8, 9000 26 / 15.5.
constexpr int AW_MANY_FROM = 12;   // one-pass ranges beyond which this plan is taken (up to there the eight ranges are one pass of a wider block)
constexpr int AW_MANY_MAX = 64;
inline AttnPlan attn_plan_many(const AttnShape& a, int ctx, int force_splits, int force_kernel)
{
    const AttnPlan pl = attn_plan(a, ctx, 1, force_splits, force_kernel);
    const int base = AW_RANGE_BYTES / (a.hd * (a.kv_f32 ? 4 : 2)), want = ceil_div(ctx, base);
    const int limit = 256 / a.Hkv < AW_MANY_MAX ? 256 / a.Hkv : AW_MANY_MAX;
    if (!pl.wide || force_splits > 0 || want <= AW_MANY_FROM || limit < 12) return pl;
    AttnPlan many = pl;
    many.n_splits = ceil_div(want, 4) * 4;
    many.chunk = base;
    if (many.n_splits > limit) {
        const int even = ceil_div(ceil_div(ctx, limit), 16) * 16;
        if (even > base) many.chunk = even;
        many.n_splits = ceil_div(ctx, many.chunk);
    }
    return many.n_splits > pl.n_splits ? many : pl;
}

// Context that the steps of a draft of up to k tokens behind n committed ones are planned for: the last step's, for all of
// them, so that a draft has one plan and not a mixture of two where it changes inside the draft (k = 4, positions 600 to 4086,
// 128-wide fp32 heads: 30 launch sequences instead of 117, each of which runs kernel by kernel once and is then captured).
SSD_HD int draft_plan_ctx(int n, int k) { return n + k - 1; }

// ---- whole single-row steps in one launch --------------------------------------------------------------------------------
// Narrow 16-bit and fp32 models: every launch of a decode layer moves a few MB, so the five launches cost their fixed time
// (about 5 us each) and not their bytes.  There one launch of resident blocks walks the layers, see step_kernel.
constexpr int ST_WAVES = 8;
constexpr int ST_GU = 2;                // gate / up pairs of a wave
constexpr int ST_CD = 2, ST_CF = 6;     // 16-byte loads per lane and row that a wave keeps of matrices with d or dq columns, with f columns
constexpr int ST_BLOCKS = 256;
constexpr int ST_WAIT_WORDS = 8;        // control words in front of the hand-over words: launch number, error flag

struct StepShape { int d, dq, dkv, f, V, hd, H, Hkv; int wt, kt; int L; };   // wt, kt: WeightType codes

// First of the n units (row pairs, rows) that block b of nb owns; it owns those up to the next block's first.
SSD_HD int step_begin(int n, int b, int nb) { return (int)((long)n * b / nb); }

// Blocks of the launch on a device with `cus` compute units, 0 where the launches per matrix are used.  A wave
// owns at most one row (pair) of every stage, two of gate / up, and holds their weights in registers (80 of 256), hence the limits
// on the widths; every block owns a row of the residual stream, so that a block that has seen
// the whole of it knows that every other block has finished what went before.
inline int step_blocks(const StepShape& s, int cus)
{
    const int ch = 64 * (s.wt == 0 ? 4 : 8);
    if (s.d > ST_CD * ch || s.dq > ST_CD * ch || s.f > ST_CF * ch) return 0;
    if (s.hd != 64 && s.hd != 128) return 0;
    if (s.dq % 64 || s.dkv % 64) return 0;
    if (s.kt != 0 && s.kt != s.wt) return 0;   // caches of the other 16-bit type
    int nb = cus < ST_BLOCKS ? cus : ST_BLOCKS;
    if (nb > s.d) nb = s.d;
    if (nb < 1) return 0;
    // Models of less width than the device has CUs: the LM head streams through d of them only.  A wave's row pairs beyond some 24 cost 0.4 us
    // each, a layer in one launch gains 8 to 9 (us per step, one launch / per matrix, 1 layer and 4: 64 x 32000 53 / 51 and 79 / 105,
    // 64 x 128256 96 / 62 and 124 / 116, 128 x 128256 69 / 62 and 96 / 117, 192 x 128256 60 / 62 and 89 / 117); 14 pairs per layer, since a
    // draft leaves layers out.
    if (nb < cus && s.V / 2 > nb * ST_WAVES * (24 + 14 * (s.L - 1))) return 0;
    if (ceil_div(s.d, nb) > ST_WAVES || ceil_div((s.dq + 2 * s.dkv) / 2, nb) > ST_WAVES || ceil_div(s.f, nb) > ST_GU * ST_WAVES) return 0;
    return nb;
}

// Hand-over words of a step: residual stream twice, q / k / v of the position, attention partials, FFN activations.
struct StepMail { size_t x, qkv, part, act, total; };
inline StepMail step_mail(const StepShape& s)
{
    StepMail m;
    size_t o = ST_WAIT_WORDS;
    m.x = o;    o += (size_t)2 * s.d;
    m.qkv = o;  o += (size_t)s.dq + 2 * s.dkv;
    m.part = o; o += (size_t)s.H * AW_MAX_RANGES * (s.hd + 2);
    m.act = o;  o += (size_t)s.f;
    m.total = o;
    return m;
}

// When a context tries one launch again behind one that gave up, which cost it the bound of a wait (50 ms; requests of these models
// take 2 to 20).  Not before the next reset; and where it fails again, because another process keeps the CUs or the stream may not
// use all of them, only behind 3, 7, .. 1023 more: a thousand requests lose at most ten waits instead of a thousand.  Sixteen
// sequences that went well make up for one give-up.
struct StepBackoff {
    int fails = 0;       // give-ups not made up for
    int skip = 0;        // resets until the next try
    int good = 0;        // sequences in a row that went well
    bool ran = false;    // a call of this sequence ended as one launch
    bool on() const { return skip == 0; }
    void gave_up()
    {
        if (fails < 10) fails++;
        skip = (1 << fails) - 1;
        good = 0;
    }
    void reset()
    {
        if (skip > 0) skip--;
        else if (ran && ++good == 16) { good = 0; if (fails > 0) fails--; }
        ran = false;
    }
};

// ---- whole verifications in one launch -----------------------------------------------------------------------------------
// The same for the k + 1 rows of a verification, see rows_step_kernel.
constexpr int RS_ROWS = 9;                     // rows that fit LDS beside each other (16-bit weights: 12 KB each) and the registers
// K bytes of a head that one block walks.  Measured up to there, one launch against a launch per matrix, us per verification, 2 and 9
// rows, 8 layers: 16-bit cache of 64-wide heads, 1000 positions 194 / 315 and 297 / 363; fp32 cache, 256 positions 182 / 294 and
// 275 / 330, of 128-wide heads, 128 positions (16 layers) 322 / 542 and 487 / 624.  It is no line where the two meet.
constexpr int RS_KEY_BYTES = 128 * 1024;

// Rows that the kernel for M rows computes.
SSD_HD int rows_step_rows(int M) { return M <= 3 ? 3 : M <= 5 ? 5 : RS_ROWS; }

// One block per head and row walks the whole context.  max_rows: rows of the widest kernel whose blocks are resident on the device.
inline bool rows_step_fits(const StepShape& s, int M, int ctx, int blocks, int max_rows)
{
    // Six to eight rows cost what nine do, and up to AT_CHUNK positions a launch per matrix has its cheapest attention (16-bit caches of
    // 64-wide heads: one range, no fold).  There the two are within 2 % of each other for bf16 weights, and a launch per matrix is ahead
    // where the FFN, whose activations are most of what is handed over, is wide for the model (us, 6 rows, 16 layers, one launch / per
    // matrix: 512 x 2560 413 / 411, 256 x 3072 409 / 398, 768 x 3072 463 / 452; but 1024 x 2816 466 / 492, 512 x 2048 394 / 395) and for
    // fp16 weights, whose conversion costs more (1024 x 2816 513 / 486, 768 x 2048 467 / 431, 512 x 1408 399 / 388).  Shapes outside its
    // tiling have no such attention to lose to (256 x 688, fp16: 384 / 503), nor have 128-wide heads (fp16 507 / 512, 8 rows 507 / 529).
    const bool tiled = s.d % 64 == 0 && s.dq % 64 == 0 && s.f % 64 == 0;
    if (M > 5 && M < RS_ROWS && ctx <= AT_CHUNK && s.wt != 0 && s.kt != 0 && s.hd == 64 && tiled && (s.wt == 2 || s.f >= 4 * s.d)) return false;
    return M >= 2 && M <= RS_ROWS && rows_step_rows(M) <= max_rows && ctx >= M && s.H * M <= blocks &&
           (long)ctx * s.hd * (s.kt == 0 ? 4 : 2) <= RS_KEY_BYTES;
}

// Hand-over words, RS_ROWS of each: residual rows twice, q / k / v, attention output, FFN activations.
struct RowsMail { size_t x, qkv, att, act, total; };
inline RowsMail rows_mail(const StepShape& s)
{
    RowsMail m;
    size_t o = 0;
    m.x = o;    o += (size_t)2 * RS_ROWS * s.d;
    m.qkv = o;  o += (size_t)RS_ROWS * (s.dq + 2 * s.dkv);
    m.att = o;  o += (size_t)RS_ROWS * s.dq;
    m.act = o;  o += (size_t)RS_ROWS * s.f;
    m.total = o;
    return m;
}

}  // namespace ssdk
