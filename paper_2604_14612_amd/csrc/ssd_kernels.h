// Internal launch interface between the host state machine (ssd_api.cpp) and the gfx950
// kernels (ssd_kernels.hip).  Plain pointers and sizes only; every launcher enqueues on the
// given stream and returns the HIP status of the launch.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ssdk {

enum WeightType { WT_F32 = 0, WT_BF16 = 1, WT_F16 = 2 };

// Launch options of one context: tuning hooks (0 = the library's own choice) and the one-shot request to time the
// next GEMV launch.  Owned by whoever owns the Dims that point to it; nothing here is process-global.
struct LaunchOpts {
    int gemv_block_cap = 0;     // > 0 overrides the block cap of the GEMV launches
    int gemv_resid_cfg = 0;     // residual projections: 100 R + 10 D + KS forces rows per group / steps in flight / K split
    int rows_depth = 0;         // > 0 forces the number of weight stripes a 16-row block keeps in flight
    int wide_depth = 0;         // the same for the 64-row blocks; large tiles: weight rows per tile
    int gemv_cfg = 0;           // single-row GEMVs other than the residual projections: 100 R + 10 D + KS of a work split (kernel_bench sweeps)
    int wide_ksplit = 0;        // 64-row blocks: 1 = never cut K, > 1 forces the number of K slices
    int attn_splits = 0;        // > 0 forces the number of ranges of the register-resident attention kernel (scratch must have been sized for it)
    int attn_kernel = 0;        // 0 heuristic, 1 LDS-staged kernel always, 3 the same in its plain (non-MFMA) form
    // When set, the next GEMV launch records its own begin / end timestamps into the two events (kernel time as a
    // profiler reports it, without the dispatch latency a pair of stream events around the launch would include)
    // and clears the request.
    hipEvent_t time_start = nullptr, time_stop = nullptr;
};

// Shape constants shared by all launches of one context.
struct Dims {
    int L, d, H, Hkv, hd, dq, dkv, f, V, max_seq;
    float eps;
    int wt;  // WeightType of the matrices; the hi/lo activation pairs of the multi-row path use the same element type
    int kt;  // WeightType code of the KV cache elements (independent of wt)
    LaunchOpts* opt = nullptr;  // may be null: library defaults, no timing
};

// Token ids of a row block: ids[r], in host-pinned memory (read once per row, over the bus) or on the device; row 0 takes
// first[0] instead when first is set (the pending token, which only the device knows).
struct Tokens { const int32_t* ids; const int32_t* first; };
// x[r][:] = embed[token r][:] widened to fp32 (ids clamped to the vocabulary).
// rope_row (may be null): hd floats, receives row *pos_dev + pos_off of the rotary table (what gemv_qkv takes).
hipError_t embed_rows(const Dims& D, const void* embed, Tokens tok, int M, float* x, hipStream_t s, const float* rope = nullptr,
                      const int* pos_dev = nullptr, int pos_off = 0, float* rope_row = nullptr);

// ---- single-row (draft / vanilla decode) path: weight-streaming GEMV kernels ----------------
// h = rmsnorm(x, gain); q,k,v = Wq h, Wk h, Wv h; rotary on q,k at position *pos_dev + pos_off, whose row of the
// table is rope_row (hd floats);
// q -> qbuf (fp32), k,v -> cache rows of this layer.
hipError_t gemv_qkv(const Dims& D, const void* wq, const void* wk, const void* wv, const float* gain,
                    const float* x, const float* rope_row, const int* pos_dev, int pos_off, float* qbuf,
                    void* kcache_l, void* vcache_l, hipStream_t s);
// x[n] += W[n][:] . in[:]   (N x K), optional tap copy of the updated x
hipError_t gemv_resid(const Dims& D, const void* w, int N, int K, const float* in, float* x, float* tap,
                      hipStream_t s);
// x += Wo . att (d x dq), att being the fold of the n_splits attention partials of a single row that
// attention() left in part when asked to defer the fold
hipError_t gemv_resid_attn(const Dims& D, const void* w, const float* part, int n_splits, float* x, float* tap,
                           hipStream_t s);
// act[n] = silu(Wg[n] . h) * (Wu[n] . h), h = rmsnorm(x, gain)
hipError_t gemv_swiglu(const Dims& D, const void* wg, const void* wu, const float* gain, const float* x,
                       float* act, hipStream_t s);
// logits[n] = Wlm[n] . rmsnorm(x, gain)
hipError_t gemv_lmhead(const Dims& D, const void* wlm, const float* gain, const float* x, float* logits,
                       hipStream_t s);

// The same with the end of a greedy step folded in: every block also leaves (max, sum of exp, arg-max) of its clamped
// logits in vstat (3 floats per block, GEMV_MAX_BLOCKS blocks at most) and a one-block kernel combines them into the greedy
// token (lowest index among equal maxima) and its soft-max probability, and prepares the next step.
struct StepOut {
    int32_t* tok_out;                            // device slot
    int32_t* tok_host; float* maxprob_host;      // host-pinned: the host reads them after synchronising, no copy is enqueued
    int* pos_dev; int32_t* tok0;   // decode: *pos_dev += 1, *tok0 = token (both null: left alone)
    int32_t* tok_log;              // decode, may be null (host-pinned): tok_log[*pos_dev before that] = token
    const void* embed; float* x_next;   // x_next set: x_next[0..d) = embedding row of the token
    const float* rope; const int* rope_pos; int rope_off; float* rope_row;   // rope_row set: rotary row *rope_pos + rope_off of the next step (the table's last one at most)
    unsigned* step_ctrl; unsigned step_hops; int32_t* step_err_host;   // of step_fused: its control words, the hand-overs of the step, set to 1 (host-pinned) where a wait gave up
};
constexpr int GEMV_MAX_BLOCKS = 1024;
hipError_t gemv_lmhead_argmax(const Dims& D, const void* wlm, const float* gain, const float* x, float* logits, float clamp,
                              float* vstat, const StepOut& out, hipStream_t s);

// ---- a whole single-row step in one launch (narrow models) ---------------------------------------------------
// Layers, LM head and the end of the step as gemv_lmhead_argmax leaves it, by resident blocks that hand the activations to
// each other through memory.  Blocks wait for each other: two such launches in flight on a device would each hold CUs that the other
// one needs.  A wait that takes longer than wait_ticks (blocks that are not resident, CUs held by others) ends the launch with
// *step_err_host = 1, nothing committed; scratch[1] (32-bit words) has to be cleared before the next launch then.  wait_ticks < 0
// (fp32, 64-wide heads): the last block leaves at once, so that the others wait in vain (tests of that path).
constexpr long STEP_TICKS_PER_US = 100;   // of wait_ticks (looked at every 64 polls, so no bound is below some 100 us)
struct StepWeights { const void* p[9]; };   // attention norm gain, wq, wk, wv, wo, MLP norm gain, wg, wu, wd of a layer (device table)
size_t step_scratch_bytes(const Dims& D);   // 0: shape not supported.  Cleared to zero before the first launch, weight table excepted
size_t step_table_offset(const Dims& D);    // bytes from the scratch's start to the weight table [L]
// Blocks of a launch on this device (0: not supported there) and the most rows of a verification whose blocks are all resident.
hipError_t step_device_blocks(const Dims& D, int device, int* blocks_out, int* max_rows_out);
bool step_plan_fits(const Dims& D, int ctx, int blocks);   // attention over ctx positions has enough blocks
struct StepLaunch {
    int blocks;
    void* scratch;
    long wait_ticks;
    const uint8_t* sub;         // host, may be null: two entries per layer, [2l] != 0 leaves out the attention sub-block, [2l+1] the MLP
    const void* lm_head; const float* final_norm;
    const float* x; const float* rope_row; const int* pos_dev; int pos_off;
    int plan_ctx;               // positions attention is planned for, at least those the row sees
    void* kv; size_t kv_layer;  // cache, bytes of K (or V) of one layer
    float* logits; float* vstat; float clamp;
};
hipError_t step_fused(const Dims& D, const StepLaunch& a, const StepOut& o, hipStream_t s);

// The M rows of a verification in one launch and their greedy tokens in a second one: x holds the embedding rows; K and V rows
// *pos_dev .. + M - 1, taps [M][L][2][d], logits [M][V] are written.  Blocks, scratch, waits and *err_host as above.
bool rows_step_fits(const Dims& D, int M, int ctx, int blocks, int max_rows);   // ctx: positions the last row sees
struct RowsStepLaunch {
    int blocks; void* scratch; long wait_ticks;
    int M, ctx;
    const void* lm_head; const float* final_norm;
    const float* x; const float* rope; const int* pos_dev;   // rope: the whole table
    void* kv; size_t kv_layer;
    float* logits; float* taps; float2* vmax; float clamp;   // vmax: [M][blocks]
    int32_t* tok_out; int32_t* tok_host; int32_t* err_host;
};
hipError_t rows_step_fused(const Dims& D, const RowsStepLaunch& a, hipStream_t s);

// ---- multi-row (verify / prefill / confidence) path ------------------------------------------
// out[r][:] = rmsnorm(in[r][:], gain) for r < M   (rows of length K)
hipError_t rmsnorm_rows(const float* in, const float* gain, int M, int K, float eps, float* out, hipStream_t s);
// Y[r][n] (op)= sum_k W[n][k] X[r][k], r < M <= 16, on MFMA tiles.
//   mode 0: store to y (ld = N_total), up to three stacked matrices (QKV) written side by side
//   mode 1: y += (residual add), optional tap copy (tap row stride tap_ld)
//   mode 2: y = silu(W0 x) * (W1 x)  (two matrices of n0 rows each)
struct RowsGemm {
    const void* w[3];
    int n[3];
    int K;
    const float* x;  // [M][K]
    float* y;        // [M][ldy]
    int ldy;
    float* tap;      // mode 1 only, may be null
    int tap_ld;
    int M;
    int mode;
};
hipError_t gemm_rows(const Dims& D, const RowsGemm& g, hipStream_t s);   // bf16 weights
// The same for fp32 / fp16 weights in fp32 arithmetic, with the RMSNorm of the input rows folded in (gain), and mode 3:
// QKV with rotary embedding and cache rows (q -> y [M][dq]).  Modes 0 and 1 take one matrix.
struct RowsPlain {
    const void* w[3];
    int n[3];
    int K;
    const float* x;
    const float* gain;   // null: rows as they are
    float* y; int ldy;
    float* tap; int tap_ld;
    int M;               // up to PLAIN_ROWS
    int mode;
    const float* rope; const int* pos_dev; int pos_off;
    void* kc; void* vc;
    int tap_only;        // > 0: only row tap_only - 1 writes its tap, into tap row 0
};
constexpr int PLAIN_ROWS = 64;
bool rows_plain_supported(const Dims& D);
hipError_t rows_plain(const Dims& D, const RowsPlain& g, hipStream_t s);
// Multi-row MFMA GEMM for bf16 / fp16 weights with K a multiple of 64.  Activations come pre-split into
// hi/lo arrays of the same 16-bit type [M][ldb] (rows_prep, embed_split, attention with out_hi/out_lo, the SwiGLU mode
// or a RESID projection with gain_out).
//   mode 0 store fp32, 1 residual add into y (+ tap), 2 SwiGLU of two matrices written as hi/lo to
//   oh/ol, 3 QKV: rotary on q and k at positions *pos_dev + pos_off + r, q -> y [M][dq] fp32,
//   k and v -> cache rows.  n[0] = 0 (rows_wide, rows_big: keys and values only) and n[1] = n[2] = 0 (rows_fused: queries only)
//   leave out the others.
// RMSNorm without a kernel: a mode-1 call with gain_out set also writes split(y * gain_out) to oh/ol
// [M][ldo] and the sums of y^2 over each 16-column tile to ssq_out [M][n/16]; a mode-0/2/3 call with
// ssq set treats bh/bl as such un-normalised rows and scales its results by
// rsqrt(sum(ssq[r][0..n_ssq)) / K + eps).
struct RowsFused {
    const void* w[3];
    int n[3];
    int K;
    const uint16_t* bh; const uint16_t* bl; int ldb;
    float* y; int ldy;
    uint16_t* oh; uint16_t* ol; int ldo;
    float* tap; int tap_ld;
    int M;
    int mode;
    const float* rope; const int* pos_dev; int pos_off;
    void* kc; void* vc;
    const float* ssq; int n_ssq;
    const float* gain_out; float* ssq_out;
    float* kpart; size_t kpart_floats;  // rows_wide / rows_big: scratch for a split along K (may be null: no split)
    int tap_only;                       // > 0: only row tap_only - 1 writes its tap, into tap row 0
    float2* vmax; float clamp;          // rows_fused mode 0, may be null: [M][n / 16] (maximum of a 16-column tile's clamped results, its lowest column)
};
bool rows_fused_supported(const Dims& D);
hipError_t rows_fused(const Dims& D, const RowsFused& f, hipStream_t s);
// y[r][n] = sum_k W[n][k] (bh + bl)[r][k] for up to 64 pre-split rows at once (the per-layer confidence rows
// against the LM head): W is streamed once for all of them.  bf16, N a multiple of 64, K a multiple of 128.
// The same GEMMs for any number of rows in one launch, on 128 x 128 tiles (prompts, the context window): weights
// cross the chip once for all rows.  16-bit weights; d, dq, dkv, V multiples of 128, f of 64, K of 64.
bool rows_big_supported(const Dims& D);
hipError_t rows_big(const Dims& D, const RowsFused& f, hipStream_t s);
bool rows_many_supported(const Dims& D, int N, int K);
hipError_t rows_many(const Dims& D, const void* w, int N, int K, const uint16_t* bh, const uint16_t* bl, int ldb, int M,
                     float* y, int ldy, hipStream_t s);
// The modes of rows_fused for up to 64 rows per pass (prompt blocks): 64-row weight tiles, n[] multiples of 64,
// K a multiple of 128; the sums of squares it reads / writes are per 64-column tile.
bool rows_wide_supported(const Dims& D);
hipError_t rows_wide(const Dims& D, const RowsFused& f, hipStream_t s);
// hi/lo bf16 split of M rows (row stride ldx) of length K into [M][K] arrays, RMS-normalised with
// gain first when gain != nullptr
hipError_t rows_prep(const Dims& D, const float* in, int ldx, const float* gain, int M, int K, float eps, uint16_t* hi,
                     uint16_t* lo, hipStream_t s);
// x[r] = embedding row of token r (16-bit weights, d a multiple of 64), hi/lo = split(x * gain) (no norm scale) and ssq[r][t] = sum of x[r][group t .. group (t+1))^2,
// group = 16 (rows_fused) or 64 (rows_wide, rows_big): the form in which a RESID projection with gain_out hands rows to
// its consumer
hipError_t embed_split(const Dims& D, const void* embed, Tokens tok, int M, const float* gain, float* x, uint16_t* hi,
                       uint16_t* lo, float* ssq, int group, hipStream_t s);
// rotary on q,k rows + cache write for the multi-row path. qkv: [M][dq + 2 dkv]; q is rotated in place.
hipError_t rope_kv_rows(const Dims& D, float* qkv, const float* rope, const int* pos_dev, int pos_off, int M,
                        void* kcache_l, void* vcache_l, hipStream_t s);

// ---- attention over the KV cache ---------------------------------------------------------------
// Row r (r < M) at position p_r = *pos_dev + pos_off + r attends cache positions 0..p_r.
// q: [M][ldq] fp32 (head h at offset h*hd); out: [M][dq] fp32, or, when out_hi != nullptr, the bf16
// hi/lo pair [M][dq] instead.  part: scratch for the split partials.
hipError_t attention(const Dims& D, const float* q, int ldq, const void* kcache_l, const void* vcache_l,
                     const int* pos_dev, int pos_off, int pos_host_hint, int M, float* part, float* out,
                     uint16_t* out_hi, uint16_t* out_lo, hipStream_t s, int* deferred_splits = nullptr, unsigned* arrive = nullptr);
// deferred_splits (single row only): when the positions are split over several blocks the fold is left to
// the consumer; *deferred_splits = the number of partials per head to pass to gemv_resid_attn, or 0 when
// out already holds the result.
// arrive (may be null): ATTN_COUNTERS words that are zero before the first launch and after every one; where the launch has several ranges
// and its kernel can, the last block of a head folds them and no second launch does.
constexpr int ATTN_COUNTERS = 1024;
size_t attention_scratch_floats(const Dims& D, int max_rows);
// launch shape attention() uses when the last of M rows sees ctx positions: the number of position ranges,
// negated and joined with their length, without and with arrive, for the register-resident kernel (two calls with equal values enqueue
// identical launches)
long attention_splits(const Dims& D, int ctx, int M);
int attention_ranges(const Dims& D, int ctx, int M);   // the number of position ranges itself

// ---- vocabulary reduction ------------------------------------------------------------------------
// Per row of logits [M][V]: arg-max (lowest index on ties), softmax max-probability and, when
// conf != nullptr, the entropy confidence of Eq. 1-4 (clamp applied first).  tok_out[r] and tok_host[r] (host-pinned)
// receive the arg-max when tok_out != nullptr.
hipError_t vocab_reduce(const float* logits, int M, int V, float clamp, float eps, int32_t* tok_out,
                        int32_t* tok_host, int32_t* argmax_out, float* maxprob_out, float* conf_out,
                        hipStream_t s);

// tok_out[r] = tok_host[r] (host-pinned) = lowest column of the largest clamped logit of row r, from the vmax records of a rows_fused LM-head launch
hipError_t argmax_tiles(const float2* vmax, int M, int n_tiles, int32_t* tok_out, int32_t* tok_host, hipStream_t s, unsigned* step_ctrl = nullptr,
                        unsigned step_hops = 0, int32_t* step_err_host = nullptr);
// Confidence, max-probability and arg-max of M rows as vocab_reduce gives them, cut along the vocabulary where the rows
// alone leave the chip idle; scratch (may be null: never cut) takes 24 bytes per row and slice.
hipError_t vocab_confidence(const float* logits, int M, int V, float clamp, float eps, int32_t* argmax_out, float* maxprob_out,
                            float* conf_out, void* scratch, size_t scratch_bytes, hipStream_t s);

// means[t] = mean over positions p < n_pos of v[p * n_taps + t] (context-window average of per-row confidences)
hipError_t window_mean(const float* v, int n_pos, int n_taps, float* means, hipStream_t s);

// ---- static scratch -----------------------------------------------------------------------------------
// A fixed-size device array inside the library image, for the one entry point that must not allocate.  Every
// device holds its own copy at its own address: static_scratch_for_device resolves it once per device (that device
// must be current) and returns the cached device pointer afterwards.  Contents persist from call to call.
size_t static_scratch_bytes();
hipError_t static_scratch_for_device(int device, void** ptr_out);

// ---- small state kernels ---------------------------------------------------------------------------
// tok0 = token, *pos_dev = pos
hipError_t set_state(int32_t* tok0, int32_t token, int* pos_dev, int pos, hipStream_t s);
// *pos_dev += delta;  tok0 = src[0] when src != nullptr
hipError_t advance_state(int* pos_dev, int delta, int32_t* tok0, const int32_t* src, hipStream_t s);
// NaN-fill cache positions >= *pos_dev of all layers
hipError_t kv_poison(const Dims& D, void* kv_all, const int* pos_dev, hipStream_t s);
// copy n floats
hipError_t copy_f32(const float* src, float* dst, size_t n, hipStream_t s);
// read-only streaming probe; *sink_dev receives a checksum so the loads cannot be dropped
hipError_t read_probe(const void* dev, size_t bytes, float* sink_dev, hipStream_t s);

}  // namespace ssdk
