// Internal launch interface between the C-ABI layer (api.hip) and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mf {

// Tokens per two waves of the bulk compression (one lane per token at d = 64, two
// lanes per token from d = 128 on), its smallest workgroup.
constexpr int compress_chunk_tokens(int T) { return T >= 2 ? 64 : 128; }
// Smallest chunk over the supported head sizes, for workspace sizing.
constexpr int kMinCompressChunk = 64;

struct CacheView {
  uint64_t* bitmaps;
  uint32_t* offsets;
  uint16_t* values;
  uint32_t* stream_len;
  int BH;            // streams = batch * kv-heads
  int T;             // tiles per token = d / 64
  int n_keep;        // kept channels per token
  int cap_tokens;    // token capacity per stream
  int64_t val_stride;
  int group_keep;    // per-channel caches: tokens kept per channel and group of 32; else -1
  // Host only, for launch_compress and launch_compress_channel: the tokens to
  // compress of each batch entry (entry_streams streams each, at most
  // kMaxPruneHeads entries); n_new is then the largest of them.
  int entry_streams = 0;
  const int32_t* entry_tokens = nullptr;
  int waves = 0;     // their waves per workgroup (0: compress_waves)
};

// Waves per workgroup of the bulk compression of n_new tokens in each of BH streams,
// i.e. its chunk. A chunk's base needs the totals of all chunks before it, and few
// streams have many chunks of each in flight that wait for one another, so they take
// wide chunks; short calls have no queue and take less LDS and fewer idle waves, and from
// 512 streams on two waves leave more workgroups a CU. us, in 2 / 4 / 8 / 16 waves (d =
// 128, 50%): 4 streams of 100 tokens 9.8 / 9.0 / 10.0 / 12.2, 8 of 2048 13.3 / 11.7 / 12.4
// / 14.7, 8 of 16K 50 / 34 / 24 / 21, 32 of 2048 21.9 / 16.2 / 14.7 / 16.8, 32 of 16K 109 /
// 75 / 62 / 68, 96 of 4096 56 / 43 / 42, 128 of 16K 217 / 180 / 185, 256 of 4096 97 / 93 /
// 98 / 120, 512 of 1024 48.7 / 50.6 / 52 / 66; d = 64, 256 of 4096 50 / 47 / 53 / 72; d = 256,
// 32 of 8192 79 / 63 / 70, 128 of 2048 59 / 55 / 69.
constexpr int64_t kManyStreams = 512;
constexpr int compress_waves(int T, int64_t BH, int64_t n_new) {
  if (BH >= kManyStreams) return 2;
  const int64_t tokens = compress_chunk_tokens(T) / 2, waves = BH * ((n_new + tokens - 1) / tokens);
  if (T == 4 || BH >= 128 || waves < 2048) return 4;
  return BH <= 16 && waves >= 4096 ? 16 : 8;
}
constexpr int widest_compress(int T) { return T == 4 ? 4 : 16; }
// The same for the scored and 2:4 selections, in 4 / 8 waves (d = 128): scored 8 streams of
// 16K 48 / 39, 32 of 16K 118 / 127, 128 of 4096 98 / 125, 512 of 1024 99 / 124 (102 in two); 2:4
// 8 of 16K 34 / 26, 32 of 16K 68.6 / 69.3, 128 of 4096 58 / 64, 512 of 1024 57 / 63 (54 in
// two). d = 256, scored, 32 of 2048 37 / 42.
constexpr int compress_waves_selected(int T, int64_t BH, int64_t n_new) {
  return compress_waves(T, BH, n_new) == 16 ? 8 : 4;
}

// A stream whose bulk compression gave up waiting in the look-back (see
// k_compress) has this stream_len; every later call skips it.
constexpr uint32_t kStreamPoisoned = 0xffffffffu;
// Look-back polls before a chunk gives up (never reached in practice: the
// chunks a chunk waits for are already running).
constexpr uint32_t kLookbackPolls = 1u << 20;

// Workspace of the bulk compression: a u32 status word at byte 0 (nonzero once a
// stream gave up; 16 bytes reserved), then u64 look-back flags [BH][n_chunks],
// u32 ticket counters [BH] and u32 counts of decided chunks [BH] (with the give-up
// mark). Cleared by each call.
struct CompressWs {
  uint32_t* status;
  uint64_t* flags;
  uint32_t* ticket;
  uint32_t* decided;
  int64_t words;  // 32-bit words to clear from ws
};
inline int64_t compress_ws_words(int64_t BH, int64_t n_chunks) { return 4 + 2 * BH * n_chunks + 2 * BH; }
inline CompressWs compress_ws(uint32_t* ws, int64_t BH, int64_t n_chunks) {
  CompressWs w;
  w.status = ws;
  w.flags = reinterpret_cast<uint64_t*>(ws + 4);
  w.ticket = reinterpret_cast<uint32_t*>(w.flags + BH * n_chunks);
  w.decided = w.ticket + BH;
  w.words = compress_ws_words(BH, n_chunks);
  return w;
}

inline size_t compress_ws_bytes(int T, int64_t BH, int64_t n_new, int waves) {
  const int64_t chunk = compress_chunk_tokens(T) / 2 * waves;
  return 4u * (size_t)compress_ws_words(BH, (n_new + chunk - 1) / chunk);
}

// Compress n_new tokens per stream (x: [BH][x_stride][64T] fp16, x_stride = n_new
// when 0) after tok0 tokens, with the workspace above; a chunk's look-back gives
// up after max_polls polls.
hipError_t launch_compress(const CacheView& c, const uint16_t* x, int n_new, int tok0, uint32_t* ws,
                           hipStream_t s, int64_t x_stride = 0, uint32_t max_polls = kLookbackPolls);
// Compress one token per stream (x: [BH][64T]) as token tok0.
hipError_t launch_append(const CacheView& c, const uint16_t* x, int tok0, hipStream_t s);
// launch_append of the keys and the values of one step in one launch (same shapes).
hipError_t launch_append_kv(const CacheView& kc, const CacheView& vc, const uint16_t* k, const uint16_t* v,
                            int tok0, hipStream_t s);

// Pruner variants of the same format (the magnitude top-k of k_compress is the
// default): per-head kept counts, 2:4 per token, output-aware key scores.
constexpr int kPruneMagnitude = 0, kPrune24 = 1, kPruneOutputAware = 2, kPruneChannel = 3,
              kPruneChannelOutputAware = 4;
constexpr int kMaxPruneHeads = 256;
struct PruneOpts {
  int mode = 0;
  int H = 1;                  // kv-heads: stream s is head s % H
  int per_head = 0;           // head_keep holds each head's kept count
  int per_entry = 0;          // head_keep holds the tokens to compress of each batch entry (H streams)
  const float* weights = nullptr;  // output-aware: fp32 [BH][x_stride][64T] channel weights
  int32_t head_keep[kMaxPruneHeads] = {};
};
// The bulk compression with a variant's selection (k_compress in its scored and
// 2:4 modes).
hipError_t launch_compress_variant(const CacheView& c, const uint16_t* x, int n_new, int tok0,
                                   uint32_t* ws, hipStream_t s, const PruneOpts& o);
hipError_t launch_append_variant(const CacheView& c, const uint16_t* x, int tok0, hipStream_t s,
                                 const PruneOpts& o);
// Per-channel pruning in groups of 32 tokens (n_new and tok0 multiples of 32):
// selection (bitmaps, one wave per stream and group) then k_compress in its
// preset mode. w: NULL (magnitude) or fp32 token weights [BH][n_new].
constexpr int kGroup = 32;
hipError_t launch_compress_channel(const CacheView& c, const uint16_t* x, int n_new, int tok0,
                                   uint32_t* ws, hipStream_t s, const float* w, int64_t x_stride = 0,
                                   uint32_t max_polls = kLookbackPolls);
// Output-aware weights: w[b][h][T][c] = sum over t = T .. min(T+L, Nq)-1, then over
// the G query heads of h, of |q[b][h*G+g][t][c]| (fp32, in that order).
hipError_t launch_query_lookahead(const uint16_t* q, int B, int Hq, int Hkv, int n_q, int T, int L,
                                  float* w, hipStream_t s);

// One window step per active batch entry (see mustafar_window_step): the ring
// slots k, v [BH][W][64T], device state len/head/n_comp [B], H streams per entry.
struct WindowView {
  uint16_t* k;
  uint16_t* v;
  int32_t* len;
  int32_t* head;
  int32_t* n_comp;
  int B, H, W;
  // Host only, for launch_window_fill: the first token and the tokens of entries
  // b .. b + fill_entries - 1 (at most kMaxPruneHeads); count is then the largest.
  int fill_entries = 0;
  const int32_t* fill_first = nullptr;
  const int32_t* fill_count = nullptr;
};
hipError_t launch_window_fill(const WindowView& w, int b, int d, const uint16_t* xk,
                              const uint16_t* xv, int64_t x_stride, int count, hipStream_t s);
// kacc: null for magnitude keys, else the window's output-aware key weights
// [BH][W][64T] fp32 (the leaving key is pruned with its slot's weights).
hipError_t launch_window_step(const CacheView& kc, const CacheView& vc, const WindowView& w,
                              const uint16_t* k_new, const uint16_t* v_new, const int32_t* active,
                              hipStream_t s, float* kacc = nullptr);
// kacc[bh][slot] += |q| of the G query heads of bh, for the newest 32 window tokens
// of every active entry (active: int32 [B] or null for all).
hipError_t launch_window_key_weights(const WindowView& w, const uint16_t* q, int G, int T,
                                     const int32_t* active, float* kacc, hipStream_t s);
// Grouped lifecycle step (see mustafar_window_step_grouped): kc per token, vc
// per channel; acc: fp32 [B][H][W] scores or NULL (magnitude).
hipError_t launch_window_step_grouped(const CacheView& kc, const CacheView& vc, const WindowView& w,
                                      const uint16_t* k_new, const uint16_t* v_new,
                                      const int32_t* active, float* acc, hipStream_t s);
// Scores of the window tokens younger than 32 steps: acc[b][h][slot] += sum over
// the G query heads of h of exp2(scale_log2 * q.k - lse2[b][hq]) (lse2: the
// log2-domain log-sum-exp the merge wrote), for the active entries (active:
// int32 [B] or null for all).
hipError_t launch_window_scores(const WindowView& w, const uint16_t* q, int G, int T,
                                float scale_log2, const float* lse2, const int32_t* active, float* acc,
                                hipStream_t s);

struct SparseSide {
  const uint64_t* bitmaps;
  const uint32_t* offsets;
  const uint16_t* values;
  const uint32_t* stream_len;  // a poisoned stream is read as empty
  int64_t val_stride;
  int cap_tokens;
  int n_keep;
  int group_keep = -1;  // per-channel caches (see CacheView)
};

struct AttnShape {
  int BHkv;       // streams
  int G;          // query heads per kv-head
  int T;          // tiles per token
  int n_s;        // compressed tokens per stream (0 for the dense kernel)
  int n_dense;    // dense tokens per stream (window, or the whole dense cache)
  int n_sparse_segs, sparse_seg_tokens;
  int n_dense_segs, dense_seg_tokens;
  float scale_log2;  // score scale times log2(e)
  // Per-batch-entry lengths (all null for uniform streams): compressed tokens
  // n_comp[b] <= n_s, and a ring window of n_dense slots holding len[b] tokens
  // from slot head[b] on. Hkv maps a stream to its batch entry.
  const int32_t* n_comp = nullptr;
  const int32_t* win_len = nullptr;
  const int32_t* win_head = nullptr;
  int Hkv = 1;
  // If set, the final merge also writes each query head's log-sum-exp of the
  // scores in the log2 domain, m + log2(l), to lse2 [BHq].
  float* lse2 = nullptr;
  // Compressed segments on the matrix-core kernel instead of the walks.
  bool mfma = false;
};

// Split-K merge in two levels when a single level would run on too few
// workgroups for its segments: the number of first-level parts of 32 segments, or
// 1 for a single-level merge. The workspace provides for two levels from 128
// segments on; the launch takes one up to 512 (8 streams of 128K tokens, 342 segments
// of 32 query heads: 56.4 us a call with one, 58.4 with two and the launch between).
constexpr int kMergeMostSingle = 512;
inline int merge_parts(int64_t n_seg, int64_t BHq, int most_single = 128) {
  return (n_seg > most_single && BHq < 256) ? (int)((n_seg + 31) / 32) : 1;
}

// Partial results of every segment into ws_ml [n_seg][BHq] (max, sum) and
// ws_o [n_seg][BHq][d], then the merge into out [BHq][d] fp16 (a two-level merge
// uses [parts][BHq] (max, sum) and [parts][BHq][d] after ws_o).
hipError_t launch_attention(const AttnShape& sh, const uint16_t* q, const SparseSide& K,
                            const SparseSide& V, const uint16_t* kd, const uint16_t* vd,
                            float* ws_ml, float* ws_o, uint16_t* out, hipStream_t s);

}  // namespace mf
