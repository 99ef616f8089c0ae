// Host-side internals of libsa.so: workspace layout and kernel launchers.
// The public entry points (sa_api.hip) validate every argument, then call
// these launchers, which only enqueue kernels on the given stream.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace sa {

// Tunables fixed at build time.
constexpr int kLseChunk = 1024;   // video keys per a->v log-sum-exp partial that the
                                  // workspace holds room for (fp32: the chunk of long
                                  // clips, shortened where room and size allow)
constexpr int kMaxKeyChunk = 1024;  // most video keys of an a->v workgroup, bf16 path
constexpr int kQSlab = 512;       // queries per 16-wave workgroup slab
constexpr int kV2aChunk = 512;    // video queries per v->a workgroup
constexpr int kMaxBlocks = 2048;  // largest supported n_b
constexpr int kMaxPairs = 65535;  // largest B*H (a grid dimension indexes (b, h))

constexpr size_t align_up(size_t x) { return (x + 255) & ~size_t(255); }

// Grid of n workgroups in x and z (y as given): a launch holds less than 2^32
// threads in one dimension.  Workgroup blockIdx.z * gridDim.x + blockIdx.x; the
// kernel leaves out those from n on.
constexpr long kGridX = 1 << 16;
inline dim3 wide_grid(long n, int y = 1) {
  return dim3(static_cast<unsigned>(n < kGridX ? n : kGridX), y,
              static_cast<unsigned>((n + kGridX - 1) / kGridX));
}

// Workspace of sa_cross_scores.  The bf16 path's parts; the fp32 path lays its
// own out within the same total.
struct CrossWs {
  size_t lse_part;   // float2 [B,H,nchunk,L_a]  (m, l) partials, bf16 path
  size_t lse_a;      // float  [B,H,L_a]         (counted; not used by the bf16 path)
  size_t colmass;    // float  [B,H,L_v]         per-head a->v column mass
  size_t lse_v;      // float  [B,H,L_v]         (counted; not used by the bf16 path)
  size_t v2a_part;   // float  [B,H,nchunk3,L_a] v->a column-mass partials
  size_t v2a_head;   // float  [B,H,L_a]         a->v log2-sum-exp, bf16 path
  size_t total;
};

inline CrossWs cross_ws_layout(int B, int H, int L_v, int L_a) {
  CrossWs w{};
  const size_t nchunk = (L_v + kLseChunk - 1) / kLseChunk;
  const size_t nchunk3 = (L_v + kV2aChunk - 1) / kV2aChunk;
  size_t off = 0;
  w.lse_part = off; off += align_up(sizeof(float) * 2 * B * H * nchunk * L_a);
  w.lse_a = off;    off += align_up(sizeof(float) * B * H * L_a);
  w.colmass = off;  off += align_up(sizeof(float) * B * H * L_v);
  w.lse_v = off;    off += align_up(sizeof(float) * B * H * L_v);
  w.v2a_part = off; off += align_up(sizeof(float) * B * H * nchunk3 * L_a);
  w.v2a_head = off; off += align_up(sizeof(float) * B * H * L_a);
  w.total = off;
  return w;
}

// Column count of the pooled block means and of the mask rows: 64 * E, with
// E the smallest of the instantiated widths {1, 2, 3, 4, 5, 6, 8, 10, 12,
// 16, 20, 24, 32} that covers n_b (n_b <= 2048).
inline int mask_e(int n_b) {
  constexpr int kWidths[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32};
  const int need = (n_b + 63) / 64;
  for (int e : kWidths)
    if (e >= need) return e;
  return 32;
}
inline int mask_n_pad(int n_b) { return 64 * mask_e(n_b); }

struct MaskWs {
  size_t qbar;   // double [B,H,d,n_pad]  pooled query means, block index innermost
  size_t kbar;   // double [B,H,d,n_pad]  pooled key means, block index innermost
  size_t total;
};

inline MaskWs mask_ws_layout(int B, int H, int n_b, int d) {
  MaskWs w{};
  const size_t n_pad = static_cast<size_t>(mask_n_pad(n_b));
  size_t off = 0;
  w.qbar = off; off += align_up(sizeof(double) * B * H * d * n_pad);
  w.kbar = off; off += align_up(sizeof(double) * B * H * d * n_pad);
  w.total = off;
  return w;
}

constexpr int kXcds = 8, kCusPerXcd = 32;  // MI355X

// bf16 sparse attention: workgroups that the chip holds at once, two of 4 waves
// (256 VGPRs a wave) a CU, or of 2 waves two (d = 128: 68 KB of LDS each) or
// four.
constexpr int attn_slots(int d, int block) {
  return kXcds * kCusPerXcd * (block == 64 && d == 64 ? 4 : 2);
}
// Whether rows go out one workgroup each, full rows of every pair first, without
// the schedule kernel and the claims of its lists (about 10 us in all, and 1.5 us a
// 128 pairs): rows that all run at once; pairs whose K and V take at most 256 KB,
// which gain nothing from one XCD's L2; and small calls, by the multiply-adds of
// their dense Q K^T.  Over some 4400 calls of 5 to 63 blocks a pair, densities of
// 0.1 to 0.5 and 0 to 10 % full rows this is 0.87 of the time of heaviest rows first
// by a ranking kernel (95 % of them at most 0.98, where the schedule took up to 1.5
// times as long below 2^33 multiply-adds and 1.1 up to 2^34); above 2^36 the
// schedule takes 0.82 of that time and this 0.97.
inline bool direct_rows(int P, int n_b, int d, int block) {
  const long long rows = static_cast<long long>(P) * n_b;
  return rows <= attn_slots(d, block) || n_b * block * d <= 65536 ||
         rows * n_b * block * block * d <= 1ll << 34;
}

// Whether the lists may be cut into one equal run per slot (the schedule kernel
// decides, from the lists' lengths): with more than four rows a slot, or lists
// of less than 64 blocks, whole rows were at least as fast at every density
// down to 10 %, and the calls are spared the cut and the merge's launch (4 to 6 us).
constexpr int kSplitRounds = 4;
inline bool split_rows(int P, int n_b, int d, int block) {
  return n_b >= 64 && static_cast<long long>(P) * n_b <= kSplitRounds * attn_slots(d, block);
}

struct AttnWs {
  size_t sched;   // int [B*H][n_b]  the XCDs' launch lists, one after the other
  size_t claim;   // int [8][64]  rows taken from each XCD's list (one per 256 bytes)
  size_t min;     // bytes without the parts below, which a call can do without
  size_t starts;  // int2 [slots + 2]  first list entry of each run; whether to use them
  size_t part;    // float [2 slots][block][d], then float2 [2 slots][block]
  size_t total;
};

constexpr size_t attn_starts_bytes(int d, int block) {
  return align_up(8 * (static_cast<size_t>(attn_slots(d, block)) + 2));
}
// `starts` and `part` of a call that may cut its lists.
constexpr size_t attn_split_bytes(int d, int block) {
  return attn_starts_bytes(d, block) +
         align_up(2 * static_cast<size_t>(attn_slots(d, block)) * block *
                  (static_cast<size_t>(d) * 4 + 8));
}

// The lists take half of what `min` has room for: that size is kept, since it
// also bounds what sa_sparse_attention_noalloc accepts.
inline AttnWs attn_ws_layout(int B, int H, int n_b, int d, int block) {
  AttnWs w{};
  size_t off = 0;
  w.sched = off; off += 2 * align_up(sizeof(int32_t) * B * H * n_b);
  w.claim = off; off += align_up(sizeof(int32_t) * 8 * 64);
  w.min = off;
  w.starts = w.part = w.total = off;
  if (split_rows(B * H, n_b, d, block)) {
    w.part = off + attn_starts_bytes(d, block);
    w.total = off + attn_split_bytes(d, block);
  }
  return w;
}

// ---- launchers (defined in the kernel sources) ----------------------------
constexpr int kMaxTokens = kMaxBlocks * 128;  // longest token sequence (L)
// Cache-reuse indicator: 9 fp32 partial sums per workgroup of the first pass
// ([9][workgroups]); 1024 video workgroups fill one round of 256 CUs x 4.
inline int cache_workgroups_video(size_t rows_v) {
  return static_cast<int>(rows_v < 1024 ? rows_v : 1024);
}
inline int cache_workgroups_audio(size_t rows_a) {
  return static_cast<int>(rows_a < 64 ? rows_a : 64);
}
inline size_t cache_ws_bytes(int B, int L_v, int L_a) {
  const size_t nwg = static_cast<size_t>(cache_workgroups_video(static_cast<size_t>(B) * L_v)) +
                     cache_workgroups_audio(static_cast<size_t>(B) * (L_a > 0 ? L_a : 0));
  return align_up(nwg * 9 * sizeof(float));
}
void launch_cache_indicator(const void* y_v, const void* y_v_hat, const uint8_t* prot_flag,
                            const void* y_a, const void* y_a_hat, const float* s_bar,
                            const float* s_hat, int B, int L_v, int L_a, int C, int dtype,
                            float lambda_p, float lambda_s, float tau, float eps,
                            float* out, char* ws, hipStream_t s);
void launch_saliency_ema(float* s_bar, const float* s, size_t n, float alpha,
                         hipStream_t st);
void launch_select_protected_tokens(const float* sal_tok, int B, int L, int k_tok,
                                    int32_t* tok_idx, uint8_t* tok_flag, hipStream_t st);
// Protected-token rows run in workgroups of kTokRowBlock gathered rows.  The
// keys of a row are cut into n_split runs so that the launch fills the 512
// workgroup slots of the chip (256 CUs, 2 attention workgroups each) in
// whole rounds: n_split minimises rounds/n_split * (1 + 0.02*n_split), where
// the second factor prices each workgroup's fixed cost (pipeline fill, the
// partial row, its share of the combine); 1 <= n_split <= 8, and every run
// keeps at least 4 key blocks.
constexpr int kTokRowBlock = 128;
inline int token_attn_splits(int P, int k_tok, int n_b) {
  const long units = static_cast<long>(P) * ceil_div(k_tok, kTokRowBlock);
  int smax = n_b / 4;
  smax = smax < 1 ? 1 : (smax > 8 ? 8 : smax);
  int best = 1;
  double best_cost = 0.0;
  for (int s = 1; s <= smax; ++s) {
    const double rounds = static_cast<double>((units * s + 511) / 512);
    const double cost = rounds / s * (1.0 + 0.02 * s);
    if (s == 1 || cost < best_cost - 1e-9) {
      best = s;
      best_cost = cost;
    }
  }
  return best;
}
// Partial rows [n_split][B*H][k_tok][d] f32, then (m, l) [n_split][B*H][k_tok]
// float2; none with one split.
inline size_t token_attn_ws_bytes(int B, int H, int L, int d, int k_tok) {
  const int ns = token_attn_splits(B * H, k_tok, ceil_div(L, kTokRowBlock));
  if (ns <= 1 || k_tok <= 0) return 0;
  return align_up(static_cast<size_t>(ns) * B * H * k_tok * (static_cast<size_t>(d) * 4 + 8));
}
void launch_protected_token_attention_bf16(const uint16_t* q, const uint16_t* k,
                                           const uint16_t* v, uint16_t* o, float* lse,
                                           int B, int H, int L, int d, float scale,
                                           const int32_t* tok_idx, int k_tok, char* ws,
                                           hipStream_t s);
// Dense cross-modal attention (queries [B,H,Lq,d], keys/values [B,H,Lk,d]);
// the workspace is token_attn_ws_bytes(B, H, Lk, d, Lq).
void launch_cross_attention_bf16(const uint16_t* q, const uint16_t* k, const uint16_t* v,
                                 uint16_t* o, float* lse, int B, int H, int Lq, int Lk, int d,
                                 float scale, char* ws, hipStream_t s);
void launch_protected_token_attention_f32(const float* q, const float* k, const float* v,
                                          float* o, float* lse, int B, int H, int L, int d,
                                          float scale, const int32_t* tok_idx, int k_tok,
                                          hipStream_t s);
void launch_cross_scores_bf16(const uint16_t* q_a, const uint16_t* k_v,
                              const uint16_t* q_v, const uint16_t* k_a, int B,
                              int H, int L_v, int L_a, int d, float scale,
                              int block, float* sal_v_tok, float* sal_v_blk,
                              float* sal_a_tok, int accumulate, double* qbar,
                              double* kbar, char* ws, hipStream_t s);
// Saliency from the row LSEs (natural log, [B,H,L_a] and [B,H,L_v]) of the
// two cross-attention forwards; the workspace is cross_ws_layout's.
void launch_cross_scores_from_lse_bf16(const uint16_t* q_a, const uint16_t* k_v,
                                       const uint16_t* q_v, const uint16_t* k_a,
                                       const float* lse_a, const float* lse_v, int B, int H,
                                       int L_v, int L_a, int d, float scale, int block,
                                       float* sal_v_tok, float* sal_v_blk, float* sal_a_tok,
                                       int accumulate, double* qbar, double* kbar, char* ws,
                                       hipStream_t s);
void launch_cross_scores_f32(const float* q_a, const float* k_v,
                             const float* q_v, const float* k_a, int B, int H,
                             int L_v, int L_a, int d, float scale, int block,
                             float* sal_v_tok, float* sal_v_blk,
                             float* sal_a_tok, int accumulate, char* ws,
                             hipStream_t s);
void launch_select_protected(const float* sal_blk, int B, int n_b, int k_prot,
                             int32_t* prot_idx, uint8_t* prot_flag,
                             hipStream_t s);
void launch_build_block_mask(const void* q_v, const void* k_v, int B, int H,
                             int L_v, int d, int dtype, float scale, int block,
                             int k_keep, const uint8_t* prot_flag,
                             int32_t* kv_idx, int32_t* kv_cnt, uint8_t* mask,
                             float* scores, char* ws, hipStream_t s);
// The pooling pass alone (K5): block means of q_v and k_v into qbar, kbar
// ([B,H,d,mask_n_pad(n_b)]).
void launch_block_pool(const void* q_v, const void* k_v, int B, int H, int L_v, int d,
                       int dtype, int block, double* qbar, double* kbar, hipStream_t s);
// The mask from given block means (K6 alone).
void launch_mask_from_means(const double* qbar, const double* kbar, int B, int H, int L_v,
                            int d, float scale, int block, int k_keep,
                            const uint8_t* prot_flag, int32_t* kv_idx, int32_t* kv_cnt,
                            uint8_t* mask, float* scores, hipStream_t s);
void launch_sparse_attention_bf16(const uint16_t* q, const uint16_t* k,
                                  const uint16_t* v, uint16_t* o, float* lse,
                                  int B, int H, int L, int d, float scale,
                                  int block, const int32_t* kv_idx,
                                  const int32_t* kv_cnt, char* ws,
                                  hipStream_t s);
// The same with the lists cut into one run per slot (split_rows): ws holds
// attn_ws_layout's total.
void launch_sparse_attention_split_bf16(const uint16_t* q, const uint16_t* k, const uint16_t* v,
                                        uint16_t* o, float* lse, int B, int H, int L, int d,
                                        float scale, int block, const int32_t* kv_idx,
                                        const int32_t* kv_cnt, char* ws, hipStream_t s);
void launch_sparse_attention_f32(const float* q, const float* k,
                                 const float* v, float* o, float* lse, int B,
                                 int H, int L, int d, float scale, int block,
                                 const int32_t* kv_idx, const int32_t* kv_cnt,
                                 char* ws, hipStream_t s);

}  // namespace sa
