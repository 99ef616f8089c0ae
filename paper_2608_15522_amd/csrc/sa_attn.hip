// Protected block-sparse flash attention (Sec. 4.2, Eq. (10) in the row
// form of Eq. (11); Eq. (5) when a list holds every key block).
//
// bf16 path (MFMA, gfx950)
// ------------------------
// One workgroup per query block (BLOCK rows, BLOCK/32 waves of 32 query rows
// each).  The workgroup walks its compacted key-block list; every key block
// is streamed as 64-key tiles of K and V into double-buffered LDS by
// global_load_lds_dwordx4 (planes of 32 d per key, 16-byte slots swizzled by
// row), so the copy of tile t+1 runs under the math of tile t without
// staging registers.  Each wave computes S^T = K Q^T with v_mfma_f32_32x32x16_bf16,
// so a lane owns one query column: the row max and row sum of the online
// softmax are lane-local, plus one exchange with the lane holding the other
// 16 keys of the same query.  P^T is packed to bf16 in registers and feeds
// O^T += V^T P^T directly as the B operand; the V^T operand is read from the
// key-major tile with ds_read_b64_tr_b16 (a transposing LDS read).  The row
// sum is taken on the same bf16 probabilities with v_dot2_f32_bf16 (the
// gather form adds the fp32 probabilities instead, for an lse exact to fp32
// rounding).  The scale is folded into exp2; the running output is rescaled
// only when a lane's max grows by more than 2^8.  Keys past L are -inf, rows
// past L are never written.
//
// Rows go through a launch schedule: each XCD takes every 8th (batch, head) pair,
// first the full rows of all its pairs (protected rows hold the full list), then
// the other rows one pair at a time, so that a pair's K/V blocks are shared through
// one XCD's L2 and the long full rows do not run alone at the end of the launch.
// Small calls and short pairs go out directly, one workgroup a row (direct_rows).
// Calls of few rows may cut the rows' lists into equal runs instead, and merge the
// rows that runs share.
//
// Gather form: dense rows gathered by index (protected tokens) or all rows
// of a query tensor of another length (cross-modal attention), every key
// kept; the keys of a row block may be split into runs whose partial rows
// token_combine_kernel merges.
//
// f32 path: fp32 matrix products (v_mfma_f32_16x16x4_f32) from operands held
// in registers, the keys of a 16-row block split over the workgroup's waves.
#include <float.h>

#include <algorithm>

#include "sa_device.h"
#include "sa_internal.h"

namespace sa {
namespace {

constexpr int kTile = 64;       // keys per LDS tile

// Launch schedule.  Workgroup w runs on XCD w % 8, which owns the pairs x,
// x+8, x+16, ... (b,h); entry i of XCD x's list (pair << 11 | query block) is
// one row of work.  The list holds first the full rows (lists of all n_b key
// blocks: the protected query blocks) of every pair the XCD owns, pair by
// pair, then the other rows pair by pair, each pair's rows in eight classes of
// list length, longest first, by index within a class.  A full row takes
// n_b / k_keep times as long as the others; started first, the full rows of
// the XCD's last pairs do not run alone at the end of the launch, while the
// other rows still go through one pair at a time, so that their K/V blocks are
// shared through the XCD's L2.
// One workgroup per XCD, one wave per pair at a time (ballot counts, two
// barriers in all).  Ranking every row exactly in a kernel of its own first
// and writing the lists in a second took 5 + 6 us at P = 24, n_b = 256; this
// one takes about 6.
constexpr int kLenClasses = 8;
__host__ __device__ constexpr int xcd_pairs(int P, int x) { return (P - x + kXcds - 1) / kXcds; }
// Pairs of the XCDs before x: their lists come first in `sched`.
__host__ __device__ constexpr int xcd_first(int P, int x) {
  const int q = P / kXcds, rem = P % kXcds;
  return x * q + (x < rem ? x : rem);
}

//
// Calls of few rows (split_rows) have one workgroup more, which lays the rows'
// lists end to end, pair by pair, and cuts them into one equal run per
// workgroup slot, so that a slot may begin and end inside a list: `starts` gets
// (row, list entry) of every run's first entry; run c ends where run c + 1
// starts, the last at row R, entry 0.  A row costs kRowCost entries besides its
// own (list, Q rows, pipeline fill, epilogue: about 15 k cycles against 5.7 k
// an entry of 128 keys at d 128), a run has at least kMinRun of them, and a cut
// within kSnap entries of a list's end moves to that end.  starts[slots + 1].x says
// whether the runs are to be used (RunRule).
constexpr int kRowCost = 2;
constexpr int kMinRun = 16;
constexpr int kSnap = 4;
// When runs are used, in list entries: claimed whole rows end with the longest one,
// which has its CU to itself by then (`alone` of an entry's usual time; 0.6 if no two
// rows share a CU at all), or, with more rows than slots, when the last round ends,
// of which `tail` of the empty part counts; runs end together, after `ratio` of their
// length (static, they wait for the slowest XCD) and the merge of what they share.
// Fitted for each form over 1200 to 1800 calls that may cut their lists (1 to 32
// pairs, 64 to 780 blocks, densities of 0.1 to 0.5, up to 10 % full rows), every one
// timed with runs and with whole rows: a call then takes 0.84, 0.80, 0.75 and 0.75 of
// the time of whole rows, heaviest first, on average (in the order below), 1.03, 1.03,
// 1.00 and 1.02 of it at the 95th percentile.  One rule for all forms, from figures at
// d 128 and block 128 alone, put one call in twenty to 1.08 times that time or more
// and one in a hundred to 1.4 times.
struct RunRule {
  float alone, tail, ratio, merge;
};
template <int D, int BLOCK>
constexpr RunRule run_rule() {
  if constexpr (D == 128 && BLOCK == 128) return {1.f, 0.8f, 1.1f, 24.f};
  if constexpr (D == 128 && BLOCK == 64) return {0.78f, 0.4f, 1.2f, 8.f};
  if constexpr (D == 64 && BLOCK == 128) return {1.f, 0.8f, 1.1f, 16.f};
  return {1.f, 0.8f, 1.2f, 16.f};
}
__device__ void cut_rows(const int32_t* __restrict__ kv_cnt, int2* __restrict__ starts, int slots,
                         int R, int n_b, RunRule rule) {
  __shared__ int wave_tot[1024 / 64], wave_max[1024 / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int K = ceil_div(R, 1024);  // rows per thread
  const int r0 = min(tid * K, R), r1 = min(r0 + K, R);
  auto row_cnt = [&](int r) { return min(max(kv_cnt[r], 0), n_b); };
  int own = 0, longest = 0;
  for (int r = r0; r < r1; ++r) {
    const int w = row_cnt(r) + kRowCost;
    own += w;
    longest = max(longest, w);
  }
  int incl = own;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(incl, o, 64);
    if (lane >= o) incl += u;
    longest = max(longest, __shfl_xor(longest, o, 64));
  }
  if (lane == 63) {
    wave_tot[wave] = incl;
    wave_max[wave] = longest;
  }
  __syncthreads();
  int before = incl - own, total = 0;
#pragma unroll
  for (int w = 0; w < 1024 / 64; ++w) {
    if (w < wave) before += wave_tot[w];
    total += wave_tot[w];
    longest = max(longest, wave_max[w]);
  }
  const int run = max(ceil_div(total, slots), kMinRun);
  if (tid == 0) {
    float whole = (R <= kXcds * kCusPerXcd ? 0.6f : rule.alone) * longest;
    if (R > slots)
      whole = fmaxf(whole, run + rule.tail * (ceil_div(R, slots) - static_cast<float>(R) / slots) *
                                     total / R);
    starts[slots + 1] = make_int2(whole > rule.ratio * run + rule.merge ? 1 : 0, 0);
  }
  for (int r = r0; r < r1; ++r) {
    const int cnt = row_cnt(r);
    // cuts c * run in [before, before + cnt + kRowCost)
    for (int c = ceil_div(before, run); c * run < before + cnt + kRowCost; ++c) {
      const int e = c * run - before - kRowCost;
      starts[c] = e < kSnap         ? make_int2(r, 0)
                  : cnt - e < kSnap ? make_int2(r + 1, 0)
                                    : make_int2(r, e);
    }
    before += cnt + kRowCost;
  }
  for (int c = ceil_div(total, run) + tid; c <= slots; c += 1024) starts[c] = make_int2(R, 0);
}

__global__ void __launch_bounds__(1024)
schedule_rows_kernel(const int32_t* __restrict__ kv_cnt, int32_t* __restrict__ sched,
                     int* __restrict__ claim, int P, int n_b, int2* __restrict__ starts, int slots,
                     RunRule rule) {
  __shared__ int full_before[kMaxPairs / kXcds + 2];  // full rows of the list's earlier pairs
  if (sched == nullptr || blockIdx.x == kXcds) {
    cut_rows(kv_cnt, starts, slots, P * n_b, n_b, rule);
    return;
  }
  const int x = blockIdx.x, np = xcd_pairs(P, x), tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  constexpr int NW = 1024 / 64;
  if (tid == 0) claim[64 * x] = 0;  // the attention kernel's row counter of XCD x
  const uint64_t lanes_below = (1ull << lane) - 1ull;
  for (int j = wave; j < np; j += NW) {
    const int32_t* cnt = kv_cnt + static_cast<size_t>(x + kXcds * j) * n_b;
    int nf = 0;
    for (int r0 = 0; r0 < n_b; r0 += 64)
      nf += __popcll(__ballot(r0 + lane < n_b && cnt[min(r0 + lane, n_b - 1)] >= n_b));
    if (lane == 0) full_before[j + 1] = nf;
  }
  __syncthreads();
  if (wave == 0) {  // prefix over the pairs, in pair order
    int acc = 0;
    for (int j0 = 0; j0 < np; j0 += 64) {
      int v = j0 + lane < np ? full_before[j0 + lane + 1] : 0;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(v, o, 64);
        if (lane >= o) v += u;
      }
      if (j0 + lane < np) full_before[j0 + lane + 1] = acc + v;
      acc += __shfl(v, 63, 64);
    }
    if (lane == 0) full_before[0] = 0;
  }
  __syncthreads();
  int32_t* out = sched + static_cast<size_t>(xcd_first(P, x)) * n_b;
  const int F = full_before[np];
  for (int j = wave; j < np; j += NW) {
    const int pair = x + kXcds * j;
    const int32_t* cnt = kv_cnt + static_cast<size_t>(pair) * n_b;
    // class of a row: -1 full, else 0 (longest) .. kLenClasses - 1
    auto row_class = [&](int r) {
      const int c = max(cnt[min(r, n_b - 1)], 0);
      return c >= n_b ? -1 : kLenClasses - 1 - c * kLenClasses / n_b;
    };
    int at[kLenClasses];  // next place of each class, first its number of rows
#pragma unroll
    for (int k = 0; k < kLenClasses; ++k) at[k] = 0;
    for (int r0 = 0; r0 < n_b; r0 += 64) {
      const int c = r0 + lane < n_b ? row_class(r0 + lane) : kLenClasses;
#pragma unroll
      for (int k = 0; k < kLenClasses; ++k) at[k] += __popcll(__ballot(c == k));
    }
    int full = full_before[j];
    int next = F + j * n_b - full;  // after the earlier pairs' other rows
#pragma unroll
    for (int k = 0; k < kLenClasses; ++k) {
      const int n = at[k];
      at[k] = next;
      next += n;
    }
    for (int r0 = 0; r0 < n_b; r0 += 64) {
      const int r = r0 + lane;
      const int c = r < n_b ? row_class(r) : kLenClasses;
      const uint64_t mf = __ballot(c == -1);
      int pos = full + __popcll(mf & lanes_below);
      full += __popcll(mf);
#pragma unroll
      for (int k = 0; k < kLenClasses; ++k) {
        const uint64_t m = __ballot(c == k);
        if (c == k) pos = at[k] + __popcll(m & lanes_below);
        at[k] += __popcll(m);
      }
      if (r < n_b) out[pos] = (pair << 11) | r;
    }
  }
}

// The rank-th query block of a pair in the order full lists (protected query
// blocks, n_b / k_keep times as long as the others), then the rest, by index;
// every wave finds it by ballots.
__device__ __forceinline__ int full_first_row(const int32_t* __restrict__ cnts, int n_b, int rank) {
  const int lane = threadIdx.x & 63;
  int nfull = 0;
  for (int i0 = 0; i0 < n_b; i0 += 64)
    nfull += __popcll(__ballot(i0 + lane < n_b && cnts[min(i0 + lane, n_b - 1)] >= n_b));
  const bool want_full = rank < nfull;
  int skip = want_full ? rank : rank - nfull;
  for (int i0 = 0; i0 < n_b; i0 += 64) {
    uint64_t m = __ballot(i0 + lane < n_b &&
                          (cnts[min(i0 + lane, n_b - 1)] >= n_b) == want_full);
    const int c64 = __popcll(m);
    if (skip < c64) {
      for (; skip > 0; --skip) m &= m - 1;
      return __builtin_amdgcn_readfirstlane(i0 + __ffsll(static_cast<unsigned long long>(m)) - 1);
    }
    skip -= c64;
  }
  return 0;
}

typedef __attribute__((address_space(3))) uint16_t lds_u16_t;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4_t;

// Rescale the running output only when some lane's max has grown by more
// than 2^8: the stale max keeps every probability below 256, exact after the
// final division by the row sum taken against the same max.
constexpr float kRescaleSlack = 8.0f;
constexpr float kSlackWeight = 1.f / 256.f;  // 2^-kRescaleSlack

template <bool B>
struct CopyFlag {
  static constexpr bool value = B;
};

// Max of x over the two lanes n and n+32 (robust to which half each output
// of the swap carries).
__device__ __forceinline__ float max_halves(float x) {
  const auto pr = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x),
                                                   false, false);
  return fmaxf(x, fmaxf(__uint_as_float(pr[0]), __uint_as_float(pr[1])));
}

// GATHER (dense rows): queries and outputs have Lq rows per pair, keys and
// values L.  Workgroup row j of pair (b,h) is query rows[b*n_rows + j], or j
// itself when rows is NULL (rows >= n_rows, or a query outside [0, Lq), are
// skipped); kv_idx, kv_cnt and order are not read.  This serves the dense
// rows of protected tokens (Eq. (11) first case, Lq == L) and cross-modal
// attention (Lq != L).  The key blocks are cut into n_split equal runs, one
// per workgroup: with n_split == 1 the workgroup keeps every key and writes
// O and lse to the query's own row; otherwise it writes its unnormalised O,
// running max m (log2 units) and row sum to `part` for token_combine_kernel.
// SPLIT: if the schedule says so, run c of `starts` per workgroup (otherwise
// whole rows by `sched` as above); a row that the run
// holds whole is written to O and lse, and of a row that it shares with other
// runs the part of the list that it holds goes to partial 2c (the run starts
// inside the list) or 2c + 1 (it starts at the list's start) for
// row_combine_kernel.
// LIST: persistent workgroups claim whole rows by `sched`, or, without one, one
// workgroup a row in index order; DIRECT: one workgroup a row, full rows first (a
// form of its own: in the persistent one its code costs 0.5 to 0.9 %).
enum class Rows { kList, kDirect, kGather, kSplit };
template <int D, int BLOCK, Rows ROWS>
__global__ void __launch_bounds__(BLOCK * 2) __attribute__((amdgpu_waves_per_eu(2, 2)))
sparse_attn_bf16_kernel(const uint16_t* __restrict__ q,
                        const uint16_t* __restrict__ k,
                        const uint16_t* __restrict__ v,
                        uint16_t* __restrict__ o, float* __restrict__ lse,
                        const int32_t* __restrict__ kv_idx,
                        const int32_t* __restrict__ kv_cnt,
                        const int32_t* __restrict__ sched, int* __restrict__ claim, int P,
                        int L, int n_b, float c, const int32_t* __restrict__ rows,
                        int n_rows, int H, int n_split, float* __restrict__ part, int Lq,
                        const int2* __restrict__ starts) {
  constexpr bool GATHER = ROWS == Rows::kGather;
  constexpr bool SPLIT = ROWS == Rows::kSplit;
  constexpr bool DIRECT = ROWS == Rows::kDirect;
  constexpr int NW = BLOCK / 32;             // waves per workgroup
  constexpr int TPB = BLOCK / kTile;         // tiles per key block
  constexpr int KC = D / 16;                 // k-steps of Q K^T
  constexpr int DT = D / 32;                 // 32-row d tiles of O^T (= planes)
  constexpr int SPANS = kTile * D * 2 / 1024;
  constexpr int NI = SPANS / NW;             // DMA instructions per wave per matrix
  constexpr int TILE_ELEMS = kTile * D;
  static_assert(SPANS % NW == 0, "tile spans must split over waves");

  __shared__ __attribute__((aligned(1024))) uint16_t Ks[2][TILE_ELEMS];
  __shared__ __attribute__((aligned(1024))) uint16_t Vs[2][TILE_ELEMS];
  __shared__ uint16_t tiles[GATHER ? 1 : kMaxBlocks * TPB];  // valid tiles, as key0 / 64
  __shared__ int ntiles_sh, nfull_sh, item_sh;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave_u = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, n = lane & 31;

  // Workgroup w runs on XCD w % 8.  Block lists with a launch schedule: the
  // workgroups are persistent, and those of XCD x take rows from x's launch
  // list (its pairs' full rows, then its pairs one at a time, so that a pair's
  // K/V blocks are shared through one L2) by an atomic counter per XCD; once
  // that list is used up they take rows from the other XCDs' lists, which
  // evens out XCDs that run at different speeds or own fewer pairs (an XCD
  // without a pair of its own starts at list x % P).  Each row is computed the
  // same way whichever workgroup takes it.  Otherwise there is one workgroup
  // per row (dense rows: XCD-major over pairs).
  const bool runs =
      SPLIT && __builtin_amdgcn_readfirstlane(starts[static_cast<int>(gridDim.x) + 1].x) != 0;
  const bool persistent = !GATHER && !DIRECT && !runs && sched != nullptr;
  const int xcd = P < kXcds ? (blockIdx.x & 7) % P : blockIdx.x & 7;
  int exhausted = 0;                   // lists found empty (thread 0)
  // SPLIT: consecutive runs on one XCD, so that a pair's K/V blocks are shared
  // through its L2
  int run = 0, split_row = 0, split_i = 0;
  int2 run_end = make_int2(0, 0);
  if (runs) {
    run = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    split_row = __builtin_amdgcn_readfirstlane(starts[run].x);
    split_i = __builtin_amdgcn_readfirstlane(starts[run].y);
    run_end.x = __builtin_amdgcn_readfirstlane(starts[run + 1].x);
    run_end.y = __builtin_amdgcn_readfirstlane(starts[run + 1].y);
  }
  for (int item_iter = 0;; ++item_iter) {
  const int n_qr = GATHER ? ceil_div(n_rows, BLOCK) : n_b;  // query blocks per pair
  const int n_q = GATHER ? n_qr * n_split : n_b;              // workgroups per pair
  int pair, rank = 0, r = 0;
  if (runs) {
    if (split_row > run_end.x || (split_row == run_end.x && split_i >= run_end.y)) break;
    pair = split_row / n_b;
    r = split_row - pair * n_b;
  } else if (persistent) {
    if (tid == 0) {
      int item = -1;
      for (int k = 0; k < 8 && item < 0; ++k) {
        const int xq = (xcd + k) & 7;
        if (exhausted & (1 << xq)) continue;
        const int rows_x = xcd_pairs(P, xq) * n_b;  // 0 for an XCD without pairs
        const int i = rows_x > 0 ? atomicAdd(claim + 64 * xq, 1) : 0;
        if (i < rows_x)
          item = xcd_first(P, xq) * n_b + i;
        else
          exhausted |= 1 << xq;
      }
      item_sh = item;
    }
    __syncthreads();
    const int item = __builtin_amdgcn_readfirstlane(item_sh);  // uniform: scalar addressing
    if (item < 0) break;
    const int e = __builtin_amdgcn_readfirstlane(sched[item]);
    pair = e >> 11;
    r = e & 2047;
  } else {
    if (item_iter > 0) break;
    if (GATHER && (P & 7) == 0) {
      const int i = blockIdx.x >> 3;
      pair = (blockIdx.x & 7) + 8 * (i / n_q);
      rank = i % n_q;
    } else {
      pair = blockIdx.x % P;
      rank = blockIdx.x / P;
      if (SPLIT && rank >= n_b) break;  // one workgroup per slot, fewer rows
      if constexpr (DIRECT || SPLIT) {
        // in index order two full rows may share a CU, or start last (1.2 times as
        // long); at most one row a CU, the order is the same to all
        if (DIRECT || P * n_b > kXcds * kCusPerXcd)
          rank = full_first_row(kv_cnt + static_cast<size_t>(pair) * n_b, n_b, rank);
      }
    }
  }
  const size_t row_base = static_cast<size_t>(pair) * n_b;
  int cnt, kb0 = 0, split = 0;
  bool partial = false;  // SPLIT: the run holds a part of the row's list
  const int32_t* idx = nullptr;
  if constexpr (GATHER) {
    // consecutive ranks share a key run and so its K/V tiles in L2
    split = rank / n_qr;
    r = rank - split * n_qr;
    kb0 = n_b * split / n_split;
    cnt = n_b * (split + 1) / n_split - kb0;
  } else {
    if (!persistent && !runs) r = rank;
    cnt = kv_cnt[row_base + r];
    cnt = cnt < 0 ? 0 : (cnt > n_b ? n_b : cnt);
    idx = kv_idx + (row_base + r) * n_b;
    if (runs) {  // entries [split_i, last) of the list
      const int last = split_row == run_end.x ? min(run_end.y, cnt) : cnt;
      partial = split_i > 0 || last < cnt;
      idx += split_i;
      cnt = last - split_i;
    }
  }

  // Compact the list into 64-key tiles (wave 0): entries outside [0, n_b)
  // are dropped, and so is the second half of a last block of <= 64 keys.
  // Full tiles keep the list order; the tile that reaches past L (at most
  // one per list entry of block n_b-1) is placed after all of them, so that
  // only the last iterations mask keys.  GATHER: the tiles of the run in order,
  // without a list; with that and the 16-byte stores of O the two cross-modal
  // forwards and the saliency at H24 L_v32760 L_a512 take 751 instead of 777
  // us (8 tiles a row there, so that what surrounds the loop weighs most).
  if (!GATHER && tid < 64) {
    int nfull = 0, npart = 0;
    const uint64_t below = (1ull << lane) - 1ull;
    for (int i0 = 0; i0 < cnt; i0 += 64) {
      const int i = i0 + lane;
      const int kb = i < cnt ? idx[i] : -1;
      const bool v0 = kb >= 0 && kb < n_b;
      const bool v1 = TPB == 2 && v0 && kb * BLOCK + kTile < L;
      const bool f0 = v0 && kb * BLOCK + kTile <= L;
      const bool f1 = v1 && kb * BLOCK + 2 * kTile <= L;  // implies f0
      const uint64_t b0 = __ballot(f0), b1 = __ballot(f1);
      const int pos = nfull + __popcll(b0 & below) + __popcll(b1 & below);
      if (f0) tiles[pos] = static_cast<uint16_t>(kb * TPB);
      if (f1) tiles[pos + 1] = static_cast<uint16_t>(kb * TPB + 1);
      nfull += __popcll(b0) + __popcll(b1);
      npart += __popcll(__ballot(v0 && !f0)) + __popcll(__ballot(v1 && !f1));
    }
    for (int j = lane; j < npart; j += 64)
      tiles[nfull + j] = static_cast<uint16_t>((L - 1) / kTile);
    if (lane == 0) {
      ntiles_sh = nfull + npart;
      nfull_sh = nfull;
    }
  }

  const int LQ = GATHER ? Lq : L;  // query and output rows per pair
  const uint16_t* qh = q + static_cast<size_t>(pair) * LQ * D;
  const char* kh = reinterpret_cast<const char*>(k + static_cast<size_t>(pair) * L * D);
  const char* vh = reinterpret_cast<const char*>(v + static_cast<size_t>(pair) * L * D);

  int qrow = r * BLOCK + (tid >> 6) * 32 + n;
  if constexpr (GATHER) {
    if (qrow >= n_rows)
      qrow = -1;
    else if (rows != nullptr)
      qrow = rows[static_cast<size_t>(pair / H) * n_rows + qrow];
    if (qrow >= LQ) qrow = -1;
  }
  const bool qvalid = GATHER ? qrow >= 0 : qrow < L;
  u32x4 qf[KC];
#pragma unroll
  for (int kc = 0; kc < KC; ++kc) {
    qf[kc] = qvalid ? ldg16(qh + static_cast<size_t>(qrow) * D + 16 * kc + 8 * g)
                    : u32x4{0u, 0u, 0u, 0u};
  }

  // DMA instruction i of wave w fills span w + NW*i of a tile: its lanes
  // cover key row 16*(span%4) + lane/4 of plane span/4, and lane l's source is
  // the logical 16-byte slot that the swizzle stores at physical slot l%4.
  int dma_row[NI];
  uint32_t dma_col[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int span = wave_u + NW * i;
    dma_row[i] = 16 * (span & 3) + (lane >> 2);
    dma_col[i] = static_cast<uint32_t>((span >> 2) * 64 +
                                       16 * ((lane & 3) ^ plane_swz(dma_row[i])));
  }

  // Lane-constant LDS byte offsets of the operand reads.
  //  K (A operand of S^T = K Q^T): row 32*st + n, slot 2*(kc&1) + g of plane kc/2.
  const int k_off0 = n * 64 + 16 * ((0 + g) ^ plane_swz(n));
  const int k_off1 = n * 64 + 16 * ((2 + g) ^ plane_swz(n));
  //  V (ds_read_b64_tr_b16): within each 16-lane group, source lane i points
  //  at V[kb + i/4][db + 4*(i%4) .. +3] so that lane i receives
  //  V[kb + 0..3][db + i]; rows 16*mm + 8*h + tr_key, d = 32*dt + tr_d.
  const int grp = lane >> 4, gi = lane & 15;
  const int tr_key = 4 * (grp >> 1) + (gi >> 2);
  const int tr_byte = 32 * (grp & 1) + 8 * (gi & 3);
  const int v_off0 = tr_key * 64 + 16 * ((tr_byte >> 4) ^ plane_swz(tr_key)) + (tr_byte & 15);
  const int v_off1 = (8 + tr_key) * 64 + 16 * ((tr_byte >> 4) ^ plane_swz(8 + tr_key)) +
                     (tr_byte & 15);

  if constexpr (!GATHER) __syncthreads();  // the tile list is visible
  const int run_keys = min((kb0 + cnt) * BLOCK, L) - kb0 * BLOCK;  // GATHER
  const int T = GATHER ? ceil_div(run_keys, kTile) : ntiles_sh;
  const int T_full = GATHER ? run_keys / kTile : nfull_sh;
  auto tile_key0 = [&](int t) {
    if constexpr (GATHER) return kb0 * BLOCK + t * kTile;
    return __builtin_amdgcn_readfirstlane(static_cast<int>(tiles[t]) * kTile);
  };
  // Source offsets of tile t's copy; rows past L (tail tile only) repeat
  // row L-1, whose values the -inf mask discards.
  auto prep = [&](const char* src, int t, uint32_t* off) {
    const int key0 = tile_key0(t);
    const int limit = min(kTile - 1, L - 1 - key0);
#pragma unroll
    for (int i = 0; i < NI; ++i)
      off[i] = static_cast<uint32_t>(min(dma_row[i], limit) * (D * 2)) + dma_col[i];
    return src + static_cast<size_t>(key0) * D * 2;
  };
  auto dma = [&](const char* base, const uint32_t* off, uint16_t* lds, int i) {
    const uint32_t lds_base = (uint32_t)(size_t)(lds_void_t*)lds;  // LDS byte address
    lds_dma16(base, off[i], __builtin_amdgcn_readfirstlane(lds_base + (wave_u + NW * i) * 1024));
  };
  auto issue = [&](const char* src, int t, uint16_t* lds) {
    uint32_t off[NI];
    const char* base = prep(src, t, off);
#pragma unroll
    for (int i = 0; i < NI; ++i) dma(base, off, lds, i);
  };
  // S^T of one tile: rows 0..31 in s0, 32..63 in s1.
  // The NI copy instructions of the next K tile are spread over the k-steps
  // (one every NW/2 steps) so that no wave stalls on a full memory queue in
  // front of its matrix instructions.
  auto qk = [&](auto with_copy, const uint16_t* Kt, f32x16& s0, f32x16& s1,
                const char* dbase, const uint32_t* doff, uint16_t* dlds) {
    const char* Kb = reinterpret_cast<const char*>(Kt);
    s0 = zero16();
    s1 = zero16();
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {
      const int off = (kc & 1) ? k_off1 : k_off0;
      const u32x4 a0 = *reinterpret_cast<const u32x4*>(Kb + (kc >> 1) * 4096 + off);
      const u32x4 a1 = *reinterpret_cast<const u32x4*>(Kb + (kc >> 1) * 4096 + 2048 + off);
      s0 = mfma32x32x16(a0, qf[kc], s0);
      s1 = mfma32x32x16(a1, qf[kc], s1);
      if constexpr (decltype(with_copy)::value) {
        if (kc % (KC / NI) == KC / NI - 1) dma(dbase, doff, dlds, kc / (KC / NI));
      }
    }
  };
  // Lane-local row max over the 64 keys of a tile.  Rows past L were copied
  // from row L-1 of the same tile, so they repeat a valid logit and leave
  // the max unchanged; their probabilities are zeroed when P is formed.
  auto tile_max = [&](const f32x16& s0, const f32x16& s1) {
    float mx = s0[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s0[i]);
#pragma unroll
    for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s1[i]);
    return mx;
  };

  f32x16 acc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) acc[dt] = zero16();
  // The running reference starts at the lowest finite value: against it a logit
  // of -inf weighs 0 from the first tile on, while -inf - -inf is a NaN that no
  // later tile repairs.  A list may begin with keys of -inf logits, and so may
  // any run or key split of a list that does not.
  float m = -FLT_MAX;
  float lsum = 0.f;
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const bf16x2_t ones = {static_cast<__bf16>(1.0f), static_cast<__bf16>(1.0f)};

  // Pipeline: K runs one tile ahead of V.  On entry to iteration t, K(t+1)
  // and V(t) are in LDS and S(t) is in registers.
  f32x16 sc0 = zero16(), sc1 = zero16(), sn_0, sn_1;
  float mx_cur = -INFINITY;
  if (T > 0) {
    issue(kh, 0, Ks[0]);
    issue(vh, 0, Vs[0]);
  }
  if (T > 1) issue(kh, 1, Ks[1]);
  wait_dma();
  __syncthreads();
  if (T > 0) {
    qk(CopyFlag<false>{}, Ks[0], sc0, sc1, nullptr, nullptr, nullptr);
    mx_cur = tile_max(sc0, sc1);
  }
  __syncthreads();  // every wave has read K(0) before iteration 0 refills its buffer
  // One iteration: the copies of K(t+2) and V(t+1) run under S(t+1) = QK^T
  // on the matrix cores, P(t) on the VALUs, and PV(t).  Past the end of the
  // list the last tile is copied again into the free buffer, which keeps the
  // iteration free of branches around the copies.  `tail` marks iterations
  // whose tile t reaches past L: only they zero P for rows past L.
  auto iteration = [&](int t, auto tail) {
    uint32_t koff[NI], voff[NI];
    const char* kbase = prep(kh, min(t + 2, T - 1), koff);
    const char* vbase = prep(vh, min(t + 1, T - 1), voff);
    const float mx = max_halves(mx_cur) * c;
    if (__any(mx > m + kRescaleSlack)) {
      const float m_new = fmaxf(m, mx);
      const float alpha = fast_exp2(m - m_new);
      m = m_new;
      lsum *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[dt][i] *= alpha;
    }
    // S(t+1) on the matrix cores (computed on stale data in the last
    // iteration and discarded) while the VALUs form P(t).
    f32x16 sn0, sn1;
    qk(CopyFlag<true>{}, Ks[(t + 1) & 1], sn0, sn1, kbase, koff, Ks[t & 1]);
    uint32_t pb0[8], pb1[8];
    if constexpr (decltype(tail)::value) {
      const int kv = L - tile_key0(t);  // valid rows of this tile
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float p0 = crow(2 * i, g) < kv ? fast_exp2(fmaf(sc0[2 * i], c, -m)) : 0.f;
        const float p1 = crow(2 * i + 1, g) < kv ? fast_exp2(fmaf(sc0[2 * i + 1], c, -m)) : 0.f;
        const float p2 = 32 + crow(2 * i, g) < kv ? fast_exp2(fmaf(sc1[2 * i], c, -m)) : 0.f;
        const float p3 =
            32 + crow(2 * i + 1, g) < kv ? fast_exp2(fmaf(sc1[2 * i + 1], c, -m)) : 0.f;
        pb0[i] = pack_bf16x2(p0, p1);
        pb1[i] = pack_bf16x2(p2, p3);
        if constexpr (GATHER) lsum += (p0 + p1) + (p2 + p3);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float p0 = fast_exp2(fmaf(sc0[2 * i], c, -m));
        const float p1 = fast_exp2(fmaf(sc0[2 * i + 1], c, -m));
        const float p2 = fast_exp2(fmaf(sc1[2 * i], c, -m));
        const float p3 = fast_exp2(fmaf(sc1[2 * i + 1], c, -m));
        pb0[i] = pack_bf16x2(p0, p1);
        pb1[i] = pack_bf16x2(p2, p3);
        if constexpr (GATHER) lsum += (p0 + p1) + (p2 + p3);
      }
    }
    // row sum: of the bf16 probabilities that the PV product uses, or (GATHER)
    // of the fp32 probabilities, so that lse is exact to fp32 rounding
    if constexpr (!GATHER) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        lsum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, pb0[i]), ones,
                                               lsum, false);
        lsum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, pb1[i]), ones,
                                               lsum, false);
      }
    }
    // O^T += V(t)^T P(t)^T while the row max of S(t+1) is taken.
    const lds_u16_t* Vb = (const lds_u16_t*)Vs[t & 1];
#pragma unroll
    for (int mm = 0; mm < 4; ++mm) {
      const uint32_t* pb = (mm < 2) ? pb0 : pb1;
      const int h = (mm & 1) * 4;
      const u32x4 b = {pb[h], pb[h + 1], pb[h + 2], pb[h + 3]};
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const lds_u16_t* base = Vb + (dt * 4096 + mm * 1024) / 2;
        const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_s16x4_t*)(base + v_off0 / 2)));
        const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_s16x4_t*)(base + v_off1 / 2)));
        const u32x4 a = {lo.x, lo.y, hi.x, hi.y};
        acc[dt] = mfma32x32x16(a, b, acc[dt]);
        const int j = mm * DT + dt;
        if (j % NW == NW - 1) dma(vbase, voff, Vs[(t + 1) & 1], j / NW);
      }
    }
    // max of S(t+1); in the last iteration it is not used
    mx_cur = tile_max(sn0, sn1);
    sc0 = sn0;
    sc1 = sn1;
    wait_dma();
    __syncthreads();
  };
  // Steady-state iteration: tiles t, t+1 and t+2 hold 64 keys each, with the
  // copy indices t+1 and t+2 clamped to the last tile (a list without a tail
  // tile runs every iteration here; past its end the last tile is copied
  // again into the free buffer, and S(t+1) of the last iteration is
  // discarded).  The issue order is fixed by scheduling barriers so that
  // every MFMA is followed by a share of the VALU work: in the QK^T phase
  // (S(t+1) into n0/n1) one bf16 pair of P(t) per MFMA; in the PV phase the
  // row sums of P(t), then the row max of S(t+1).  Operand reads run two
  // MFMAs ahead, and the NI copies of each matrix are spread over its phase.
  uint32_t dma_full[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) dma_full[i] = static_cast<uint32_t>(dma_row[i] * (D * 2)) + dma_col[i];
  auto main_iter = [&](int t, f32x16& c0, f32x16& c1, f32x16& n0, f32x16& n1) {
    const char* kbase = kh + static_cast<size_t>(tile_key0(min(t + 2, T - 1))) * D * 2;
    const char* vbase = vh + static_cast<size_t>(tile_key0(min(t + 1, T - 1))) * D * 2;
    const float mx = max_halves(mx_cur) * c;
    if (__any(mx > m + kRescaleSlack)) {
      const float m_new = fmaxf(m, mx);
      const float alpha = fast_exp2(m - m_new);
      m = m_new;
      lsum *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[dt][i] *= alpha;
    }
    const char* Kb = reinterpret_cast<const char*>(Ks[(t + 1) & 1]);
    const lds_u16_t* Vb = (const lds_u16_t*)Vs[t & 1];
    uint16_t* kdst = Ks[t & 1];
    uint16_t* vdst = Vs[(t + 1) & 1];
    auto kread = [&](int kc, u32x4* dst) {
      const int off = (kc & 1) ? k_off1 : k_off0;
      dst[0] = *reinterpret_cast<const u32x4*>(Kb + (kc >> 1) * 4096 + off);
      dst[1] = *reinterpret_cast<const u32x4*>(Kb + (kc >> 1) * 4096 + 2048 + off);
    };
    auto vread = [&](int j, u32x4& dst) {
      const lds_u16_t* base = Vb + ((j % DT) * 4096 + (j / DT) * 1024) / 2;
      const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (lds_s16x4_t*)(base + v_off0 / 2)));
      const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (lds_s16x4_t*)(base + v_off1 / 2)));
      dst = u32x4{lo.x, lo.y, hi.x, hi.y};
    };
    // ---- QK^T phase: S(t+1) on the matrix cores, P(t) on the VALUs.  The
    // wave issues at raised priority here, where most of its VALU work lies,
    // and at normal priority in the PV phase.
    __builtin_amdgcn_s_setprio(1);
    constexpr int NA = 2 * KC;          // MFMAs
    constexpr int PPA = 16 / NA;        // bf16 pairs of P per MFMA
    u32x4 ka[3][2];
    uint32_t pb[16];
    kread(0, ka[0]);
    kread(1, ka[1]);
    n0 = zero16();
    n1 = zero16();
    // P(t) is formed in three stages a step apart, so that no instruction
    // waits on the one just before it: in step st the FMAs of pair group
    // st+1, the exponentials of group st, and the bf16 packing of group st-1
    // (a group is the PPA pairs of one step; pair pk holds elements 2pk and
    // 2pk+1 of S(t), from c0 for pk < 8, else from c1).
    float fx[2][PPA][2], ex[2][PPA][2];
    auto stage_fma = [&](int grp) {
#pragma unroll
      for (int u = 0; u < PPA; ++u) {
        const int pk = grp * PPA + u;
        const f32x16& src = pk < 8 ? c0 : c1;
        const int e = 2 * (pk & 7);
        fx[grp & 1][u][0] = fmaf(src[e], c, -m);
        fx[grp & 1][u][1] = fmaf(src[e + 1], c, -m);
      }
    };
    auto stage_exp = [&](int grp) {
#pragma unroll
      for (int u = 0; u < PPA; ++u) {
        ex[grp & 1][u][0] = fast_exp2(fx[grp & 1][u][0]);
        ex[grp & 1][u][1] = fast_exp2(fx[grp & 1][u][1]);
        if constexpr (GATHER) lsum += ex[grp & 1][u][0] + ex[grp & 1][u][1];  // fp32 row sum
      }
    };
    auto stage_pack = [&](int grp) {
#pragma unroll
      for (int u = 0; u < PPA; ++u)
        pb[grp * PPA + u] = pack_bf16x2(ex[grp & 1][u][0], ex[grp & 1][u][1]);
    };
    stage_fma(0);
#pragma unroll
    for (int st = 0; st < NA; ++st) {
      const int kc = st >> 1;
      if ((st & 1) == 0 && kc + 2 < KC) kread(kc + 2, ka[(kc + 2) % 3]);
      if (st & 1)
        n1 = mfma32x32x16(ka[kc % 3][1], qf[kc], n1);
      else
        n0 = mfma32x32x16(ka[kc % 3][0], qf[kc], n0);
      if (st > 0) stage_pack(st - 1);
      stage_exp(st);
      if (st + 1 < NA) stage_fma(st + 1);
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        if (i * NA / NI == st) {
          const uint32_t la = (uint32_t)(size_t)(lds_void_t*)kdst;
          lds_dma16(kbase, dma_full[i],
                    __builtin_amdgcn_readfirstlane(la + (wave_u + NW * i) * 1024));
        }
        if (i * NA / NI + NA / (2 * NI) == st) {
          const uint32_t la = (uint32_t)(size_t)(lds_void_t*)vdst;
          lds_dma16(vbase, dma_full[i],
                    __builtin_amdgcn_readfirstlane(la + (wave_u + NW * i) * 1024));
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    stage_pack(NA - 1);
    // ---- PV phase: O^T += V(t)^T P(t)^T; row sums of P(t), row max of S(t+1)
    __builtin_amdgcn_s_setprio(0);
    constexpr int NB = 4 * DT;          // MFMAs
    constexpr int VB = 32 / NB;         // VALU ops per MFMA
    u32x4 va[3];
    vread(0, va[0]);
    vread(1, va[1]);
    float mxn = -INFINITY;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if (j + 2 < NB) vread(j + 2, va[(j + 2) % 3]);
      const int mm = j / DT, dt = j % DT;
      const int h = (mm & 1) * 4 + (mm < 2 ? 0 : 8);
      const u32x4 b = {pb[h], pb[h + 1], pb[h + 2], pb[h + 3]};
      acc[dt] = mfma32x32x16(va[j % 3], b, acc[dt]);
#pragma unroll
      for (int u = 0; u < VB; ++u) {
        const int w = j * VB + u;  // 0..15: row sums, 16..31: max pairs
        if (w < 16) {
          if constexpr (!GATHER)
            lsum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, pb[w]), ones,
                                                   lsum, false);
        } else {
          const int e = w - 16;  // pair e: elements 2e, 2e+1 of n0 (e < 8) or n1
          const f32x16& src = e < 8 ? n0 : n1;
          mxn = fmaxf(mxn, src[2 * (e & 7)]);
          mxn = fmaxf(mxn, src[2 * (e & 7) + 1]);
          asm volatile("" : "+v"(mxn));  // keeps this share of the max in its slot
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    mx_cur = mxn;
    __builtin_amdgcn_s_setprio(0);
    wait_dma();
    __syncthreads();
  };

  // With a tail tile (T_full < T), its copies (row clamp) and its masked P
  // take the generic iterations, from the one that first copies it.
  const int T_main = T_full == T ? T : (T_full > 2 ? T_full - 2 : 0);
  int t = 0;
  for (; t + 1 < T_main; t += 2) {
    main_iter(t, sc0, sc1, sn_0, sn_1);
    main_iter(t + 1, sn_0, sn_1, sc0, sc1);
  }
  if (t < T_main) {
    main_iter(t, sc0, sc1, sn_0, sn_1);
    sc0 = sn_0;
    sc1 = sn_1;
    ++t;
  }
  for (; t < T; ++t) iteration(t, CopyFlag<true>{});

  const float ltot = lsum + swap_halves(lsum);
  if constexpr (GATHER) {
    if (part != nullptr) {
      if (qvalid) {
        const size_t prow = static_cast<size_t>(split * P + pair) * n_rows +
                            (r * BLOCK + (tid >> 6) * 32 + n);
        float* orow = part + prow * D;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int rg = 0; rg < 4; ++rg) {
            const f32x4 val = {acc[dt][4 * rg], acc[dt][4 * rg + 1], acc[dt][4 * rg + 2],
                               acc[dt][4 * rg + 3]};
            *reinterpret_cast<f32x4*>(orow + 32 * dt + 8 * rg + 4 * g) = val;
          }
        if (g == 0) {
          float2* ml = reinterpret_cast<float2*>(
              part + static_cast<size_t>(n_split) * P * n_rows * D);
          ml[prow] = make_float2(m, ltot);
        }
      }
      return;
    }
  }
  if (runs) {
    const int id = 2 * run + (split_i > 0 ? 0 : 1);
    split_i = 0;
    ++split_row;
    if (partial) {
      const size_t prow = static_cast<size_t>(id) * BLOCK + (tid >> 6) * 32 + n;
      float* orow = part + prow * D;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
          const f32x4 val = {acc[dt][4 * rg], acc[dt][4 * rg + 1], acc[dt][4 * rg + 2],
                             acc[dt][4 * rg + 3]};
          *reinterpret_cast<f32x4*>(orow + 32 * dt + 8 * rg + 4 * g) = val;
        }
      if (g == 0)
        reinterpret_cast<float2*>(part + 2 * static_cast<size_t>(gridDim.x) * BLOCK * D)[prow] =
            make_float2(m, ltot);
      continue;
    }
  }
  const float inv = ltot > 0.f ? 1.f / ltot : 0.f;
  if (qvalid) {
    uint16_t* orow = o + (static_cast<size_t>(pair) * LQ + qrow) * D;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
      for (int rp = 0; rp < 2; ++rp) {
        // the lane's channels 16rp + 4g .. +3 and 16rp + 8 + 4g .. +3 of tile
        // dt; exchanged with the lane of the other half, 8 in a row: half as
        // many stores, 32 bytes a row each instead of 16
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          w[i] = pack_bf16x2(acc[dt][8 * rp + 2 * i] * inv, acc[dt][8 * rp + 2 * i + 1] * inv);
        const auto e0 = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
        const auto e1 = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
        stg16(orow + 32 * dt + 16 * rp + 8 * g, u32x4{e0[0], e1[0], e0[1], e1[1]});
      }
    }
    if (lse != nullptr && g == 0)
      lse[static_cast<size_t>(pair) * LQ + qrow] =
          ltot > 0.f ? (m + __log2f(ltot)) * kLn2 : -INFINITY;
  }
  }  // next row
}

// Merges the n_split partial rows of each gathered query (rows[b*n_rows + j],
// or j when rows is NULL; Lq output rows per pair): with M the largest
// running max, O = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s and
// lse = (M + log2 of the denominator) ln 2, the splits added in index order.
// One thread per 4 channels of a row.
template <int D>
__global__ void __launch_bounds__(256)
token_combine_kernel(const float* __restrict__ part, int n_split, int P, int Lq, int H,
                     const int32_t* __restrict__ rows, int n_rows, uint16_t* __restrict__ o,
                     float* __restrict__ lse) {
  constexpr int TPR = D / 4;
  const size_t gid = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
  const size_t pr = gid / TPR;  // pair * n_rows + j
  if (pr >= static_cast<size_t>(P) * n_rows) return;
  const int d4 = static_cast<int>(gid % TPR) * 4;
  const int pair = static_cast<int>(pr / n_rows), j = static_cast<int>(pr % n_rows);
  const int t = rows != nullptr ? rows[static_cast<size_t>(pair / H) * n_rows + j] : j;
  if (t < 0 || t >= Lq) return;
  const size_t stride = static_cast<size_t>(P) * n_rows;  // rows per split
  const float2* ml = reinterpret_cast<const float2*>(part + n_split * stride * D);
  float M = -INFINITY;
  for (int s = 0; s < n_split; ++s) {
    const float2 v = ml[s * stride + pr];
    if (v.y > 0.f) M = fmaxf(M, v.x);
  }
  float den = 0.f;
  f32x4 num = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < n_split; ++s) {
    const float2 v = ml[s * stride + pr];
    const float w = v.y > 0.f ? exp2f(v.x - M) : 0.f;
    const f32x4 x = *reinterpret_cast<const f32x4*>(part + (s * stride + pr) * D + d4);
    den = fmaf(w, v.y, den);
#pragma unroll
    for (int e = 0; e < 4; ++e) num[e] = fmaf(w, x[e], num[e]);
  }
  const float inv = den > 0.f ? 1.f / den : 0.f;
  const u32x2 val = {pack_bf16x2(num[0] * inv, num[1] * inv),
                     pack_bf16x2(num[2] * inv, num[3] * inv)};
  *reinterpret_cast<u32x2*>(o + (static_cast<size_t>(pair) * Lq + t) * D + d4) = val;
  if (lse != nullptr && d4 == 0)
    lse[static_cast<size_t>(pair) * Lq + t] = den > 0.f ? (M + __log2f(den)) * kLn2 : -INFINITY;
}

// The rows that several runs share: workgroup c merges the row whose first part
// run c holds (if there is one), in run order, as token_combine_kernel does.
constexpr int kRowCombThreads = 256;
template <int D, int BLOCK>
__global__ void __launch_bounds__(kRowCombThreads)
row_combine_kernel(const float* __restrict__ part, const int2* __restrict__ starts, int n_b, int L,
                   uint16_t* __restrict__ o, float* __restrict__ lse) {
  const int c = blockIdx.x, runs = gridDim.x;
  if (starts[runs + 1].x == 0) return;
  const int2 cut = starts[c + 1], from = starts[c];
  if (cut.y == 0 || (from.x == cut.x && from.y > 0)) return;  // no shared row begins in run c
  int n = 2;  // parts: run c's second partial, then the first ones of runs c + 1, ...
  while (c + n <= runs && starts[c + n].x == cut.x && starts[c + n].y > 0) ++n;
  const float2* ml =
      reinterpret_cast<const float2*>(part + 2 * static_cast<size_t>(runs) * BLOCK * D);
  const int pair = cut.x / n_b, row0 = (cut.x - pair * n_b) * BLOCK;
  constexpr int TPR = D / 4;
#pragma unroll 4
  for (int u = 0; u < BLOCK * TPR / kRowCombThreads; ++u) {
    const int t = u * kRowCombThreads + static_cast<int>(threadIdx.x);
    const int j = t / TPR, d4 = (t % TPR) * 4;
    if (row0 + j >= L) continue;
    auto prow = [&](int s) {
      return static_cast<size_t>(s == 0 ? 2 * c + 1 : 2 * (c + s)) * BLOCK + j;
    };
    float M = -INFINITY;
    for (int s = 0; s < n; ++s) {
      const float2 v = ml[prow(s)];
      if (v.y > 0.f) M = fmaxf(M, v.x);
    }
    float den = 0.f;
    f32x4 num = {0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < n; ++s) {
      const float2 v = ml[prow(s)];
      const float w = v.y > 0.f ? exp2f(v.x - M) : 0.f;
      const f32x4 x = ldg_f32x4(part + prow(s) * D + d4);
      den = fmaf(w, v.y, den);
#pragma unroll
      for (int e = 0; e < 4; ++e) num[e] = fmaf(w, x[e], num[e]);
    }
    const float inv = den > 0.f ? 1.f / den : 0.f;
    const u32x2 val = {pack_bf16x2(num[0] * inv, num[1] * inv),
                       pack_bf16x2(num[2] * inv, num[3] * inv)};
    const size_t orow = static_cast<size_t>(pair) * L + row0 + j;
    *reinterpret_cast<u32x2*>(o + orow * D + d4) = val;
    if (lse != nullptr && d4 == 0)
      lse[orow] = den > 0.f ? (M + __log2f(den)) * kLn2 : -INFINITY;
  }
}

// ---- fp32 path ------------------------------------------------------------
// One workgroup of kF32Waves waves per 16 query rows; the waves take the
// 16-key tiles of the row block's list in turn and merge their partial rows
// through LDS at the end.  fp32 calls are small (a few heads, a few thousand
// tokens), so the keys are split inside the workgroup and the rows are cut
// into the smallest matrix tile: that is what fills the chip.  All products
// run on the matrix cores in fp32 (v_mfma_f32_16x16x4_f32, 157 TFLOP/s):
//   S^T = K Q^T   lane (n, gk) = (l % 16, l / 16) holds Q[n] and K[n] at the
//                 channels 16i + 4gk + e, and the result leaves the lane with
//                 query n and keys 4gk .. 4gk+3;
//   O^T += V^T P^T with k slot gk of step r standing for key 4gk + r, which
//                 makes P's registers the B operand as they are, and row i of
//                 channel tile (dq, e) standing for channel 64dq + 4i + e, so
//                 that one 16-byte load of V feeds four channel tiles.
// Each wave copies its own K tiles through its own LDS buffers (RowTile16)
// and loads V into registers, both one tile ahead, so the loop has no
// barrier.  The row max is raised only when a score exceeds it by 2^8 (decided per
// wave), so the exchange of the max between the four lanes of a query is rare.
// At B1 H4 L4680 d128 (0.28 of the pairs kept) it takes 172 us, 83 TFLOP/s, the
// matrix cores busy 0.55 of it: few and uneven workgroups, the full rows' 293 tiles
// the longest chain, and every workgroup streams K and V for its own 16 rows (16 KB
// past L1 a tile, 18 bytes a cycle and CU); the
// one-thread-per-row form before it took 16.4 ms, this one with K loaded
// straight into the operand layout 192-264 us.
constexpr int kF32Waves = 4;
constexpr int kF32Rows = 16;  // query rows per workgroup
constexpr int kF32Keys = 16;  // keys per tile

// GATHER: as in the bf16 kernel, row j of pair (b,h) is token
// rows[b*n_rows + j] and every key is kept.
template <int D, bool GATHER>
__global__ void __launch_bounds__(64 * kF32Waves, 2)
sparse_attn_f32_kernel(const float* __restrict__ q, const float* __restrict__ k,
                       const float* __restrict__ v, float* __restrict__ o,
                       float* __restrict__ lse,
                       const int32_t* __restrict__ kv_idx,
                       const int32_t* __restrict__ kv_cnt, int L, int n_b,
                       int block, Log2Scale c, const int32_t* __restrict__ rows,
                       int n_rows, int H) {
  constexpr int KI = D / 16;  // 16-byte chunks of a lane's K or Q row
  constexpr int DQ = D / 64;  // 64-channel groups of O
  using KTile = RowTile16<D>;
  // the waves' K buffers; after the loop, their partial rows
  constexpr int kPartBytes = kF32Waves * kF32Rows * (D + 4) * 4;
  constexpr int kRingBytes = kF32Waves * 2 * KTile::kBytes;
  static_assert(kPartBytes <= kRingBytes, "the partial rows reuse the K buffers");
  __shared__ __attribute__((aligned(1024))) char ring[kRingBytes];
  float(*part)[kF32Rows][D + 4] = reinterpret_cast<float(*)[kF32Rows][D + 4]>(ring);
  __shared__ float part_m[kF32Waves][kF32Rows], part_l[kF32Waves][kF32Rows];
  __shared__ uint16_t list[GATHER ? 1 : kMaxBlocks];
  __shared__ int n_list;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, gk = lane >> 4;
  const int pair = blockIdx.x;
  const int tpb = GATHER ? 1 : block / kF32Keys;  // key tiles of a key block
  int row0 = blockIdx.y * kF32Rows;

  if constexpr (!GATHER) {
    // Row tiles of full lists start first: workgroup y of a pair takes row tile
    // y % per_block of the (y / per_block)-th block in that order.
    const int per_block = block / kF32Rows;
    const int r = full_first_row(kv_cnt + static_cast<size_t>(pair) * n_b, n_b,
                                 blockIdx.y / per_block);
    row0 = r * block + (blockIdx.y % per_block) * kF32Rows;
    if (row0 >= L) return;  // row tiles of the last block past the last token
    // the list's valid entries (wave 0), in list order
    if (tid < 64) {
      const size_t row_base = static_cast<size_t>(pair) * n_b + r;
      const int32_t* idx = kv_idx + row_base * n_b;
      int cnt = kv_cnt[row_base];
      cnt = cnt < 0 ? 0 : (cnt > n_b ? n_b : cnt);
      int at = 0;
      for (int i0 = 0; i0 < cnt; i0 += 64) {
        const int kb = i0 + lane < cnt ? idx[i0 + lane] : -1;
        const bool ok = kb >= 0 && kb < n_b;
        const uint64_t m = __ballot(ok);
        if (ok) list[at + __popcll(m & ((1ull << lane) - 1ull))] = static_cast<uint16_t>(kb);
        at += __popcll(m);
      }
      if (lane == 0) n_list = at;
    }
  }
  const float* kh = k + static_cast<size_t>(pair) * L * D;
  const float* vh = v + static_cast<size_t>(pair) * L * D;
  int qrow = row0 + n;
  bool qvalid = qrow < L;
  if constexpr (GATHER) {
    qvalid = qrow < n_rows;
    qrow = qvalid ? rows[static_cast<size_t>(pair / H) * n_rows + qrow] : -1;
    qvalid = qrow >= 0 && qrow < L;
  }
  const float* qh = q + static_cast<size_t>(pair) * L * D;
  f32x4 qf[KI];
#pragma unroll
  for (int i = 0; i < KI; ++i)
    qf[i] = qvalid ? ldg_f32x4(qh + static_cast<size_t>(qrow) * D + 16 * i + 4 * gk)
                   : f32x4{0.f, 0.f, 0.f, 0.f};
  __syncthreads();  // the list is visible
  const int T = GATHER ? ceil_div(L, kF32Keys) : n_list * tpb;
  // First key of tile t; tiles of the last block that start past L hold no
  // key (their loads read row L-1, their probabilities are zero).
  auto tile_key0 = [&](int t) {
    if constexpr (GATHER) return t * kF32Keys;
    const int b = t / tpb;
    return __builtin_amdgcn_readfirstlane(static_cast<int>(list[b])) * block +
           (t - b * tpb) * kF32Keys;
  };
  KTile kt;
  kt.init(ring + wave * 2 * KTile::kBytes, lane);
  struct Tile {
    f32x4 v[4][DQ];
    int key0;
  };
  auto load = [&](int t, int buf, Tile& x) {
    x.key0 = tile_key0(t);
    kt.copy(kh, x.key0, L, buf);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const float* vs = vh + static_cast<size_t>(min(x.key0 + 4 * gk + s, L - 1)) * D + 4 * n;
#pragma unroll
      for (int dq = 0; dq < DQ; ++dq) x.v[s][dq] = ldg_f32x4(vs + 64 * dq);
    }
  };
  f32x4 acc[DQ][4];
#pragma unroll
  for (int dq = 0; dq < DQ; ++dq)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[dq][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, lsum = 0.f;
  // One tile, its K in buffer buf: the loads of tile t + kF32Waves go out
  // first and land under this tile's products.
  auto step = [&](int t, int buf, Tile& x, Tile& nx) {
    wait_dma();
    __builtin_amdgcn_sched_barrier(0);
    f32x4 kf[KI];
    kt.read(buf, kf);
    load(min(t + kF32Waves, T - 1), buf ^ 1, nx);
    __builtin_amdgcn_sched_barrier(0);
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < KI; ++i)
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        s0 = mfma16x16x4_f32(kf[i][e], qf[i][e], s0);
        s1 = mfma16x16x4_f32(kf[i][e + 1], qf[i][e + 1], s1);
      }
    float s[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = s0[e] + s1[e];
    // rows past L repeat row L-1's logit (already in the max) or belong to a
    // tile without keys, which only raises the reference
    const float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])) * c.hi;
    if (__any(mx > m + kRescaleSlack)) {
      float m_new = fmaxf(m, mx);
      m_new = fmaxf(m_new, __shfl_xor(m_new, 16, 64));
      m_new = fmaxf(m_new, __shfl_xor(m_new, 32, 64));
      const float alpha = m == m_new ? 1.f : fast_exp2(m - m_new);  // 0 the first time
      m = m_new;
      lsum *= alpha;
#pragma unroll
      for (int dq = 0; dq < DQ; ++dq)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[dq][e] *= alpha;
    }
    const float mref = m == -INFINITY ? 0.f : m;  // only -inf scores so far: they weigh 0
    // the slack taken off exactly: weights of at most 1 keep P V within the range of V
    float p[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) p[e] = kSlackWeight * fast_exp2(log2_score(s[e], c, mref));
    if (x.key0 + kF32Keys > L) {  // rows past L weigh nothing, whatever row L-1 holds
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (x.key0 + 4 * gk + e >= L) {
          p[e] = 0.f;
#pragma unroll
          for (int dq = 0; dq < DQ; ++dq) x.v[e][dq] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    lsum += (p[0] + p[1]) + (p[2] + p[3]);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int dq = 0; dq < DQ; ++dq)
#pragma unroll
        for (int w = 0; w < 4; ++w)
          acc[dq][w] = mfma16x16x4_f32(x.v[e][dq][w], p[e], acc[dq][w]);
  };
  Tile ta, tb;
  if (wave < T) {
    load(wave, 0, ta);
    int t = wave;
    for (; t + kF32Waves < T; t += 2 * kF32Waves) {
      step(t, 0, ta, tb);
      step(t + kF32Waves, 1, tb, ta);
    }
    if (t < T) step(t, 0, ta, tb);
  }
  wait_dma();
  __syncthreads();  // every wave is past its last K read and copy: `part` may be written
  lsum += __shfl_xor(lsum, 16, 64);
  lsum += __shfl_xor(lsum, 32, 64);
  if (gk == 0) {
    part_m[wave][n] = m;
    part_l[wave][n] = lsum;
  }
  // acc[dq][e][s] is channel 64dq + 16gk + 4s + e of query n
#pragma unroll
  for (int dq = 0; dq < DQ; ++dq)
#pragma unroll
    for (int s = 0; s < 4; ++s)
      *reinterpret_cast<f32x4*>(&part[wave][n][64 * dq + 16 * gk + 4 * s]) =
          f32x4{acc[dq][0][s], acc[dq][1][s], acc[dq][2][s], acc[dq][3][s]};
  __syncthreads();
  // Merge the waves' rows in wave order; 4 channels of a row per thread.
  constexpr int TPR = D / 4;
  for (int u = tid; u < kF32Rows * TPR; u += 64 * kF32Waves) {
    const int j = u / TPR, d4 = (u % TPR) * 4;
    int orow = row0 + j;
    bool ok = orow < L;
    if constexpr (GATHER) {
      ok = orow < n_rows;
      orow = ok ? rows[static_cast<size_t>(pair / H) * n_rows + orow] : -1;
      ok = orow >= 0 && orow < L;
    }
    if (!ok) continue;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w) M = fmaxf(M, part_m[w][j]);
    float den = 0.f;
    f32x4 num = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w) {
      const float pm = part_m[w][j];  // -inf: no key seen, the row is zero
      const float f = pm == -INFINITY ? 0.f : exp2f(pm - M);
      const f32x4 x = *reinterpret_cast<const f32x4*>(&part[w][j][d4]);
      den = fmaf(f, part_l[w][j], den);
#pragma unroll
      for (int e = 0; e < 4; ++e) num[e] = fmaf(f, x[e], num[e]);
    }
    const float inv = den > 0.f ? 1.f / den : 0.f;
    const f32x4 val = {num[0] * inv, num[1] * inv, num[2] * inv, num[3] * inv};
    *reinterpret_cast<f32x4*>(o + (static_cast<size_t>(pair) * L + orow) * D + d4) = val;
    if (lse != nullptr && d4 == 0)
      lse[static_cast<size_t>(pair) * L + orow] =
          den > 0.f ? static_cast<float>(static_cast<double>(M) * 0.6931471805599453 +
                                         static_cast<double>(logf(den * (1.f / kSlackWeight))))
                : -INFINITY;
  }
}

}  // namespace

template <int D, int BLOCK>
static void sparse_attention_bf16(const uint16_t* q, const uint16_t* k, const uint16_t* v,
                                  uint16_t* o, float* lse, int B, int H, int L, float scale,
                                  const int32_t* kv_idx, const int32_t* kv_cnt, char* ws,
                                  bool split, hipStream_t s) {
  const int n_b = ceil_div(L, BLOCK), P = B * H;
  const AttnWs lay = attn_ws_layout(B, H, n_b, D, BLOCK);
  const float c = scale * kLog2e;
  const int slots = attn_slots(D, BLOCK);
  const int rows = P * n_b;
  // a call that may cut its lists has a workgroup per slot, so that only as many
  // rows go out directly
  const bool direct = split ? rows <= slots : direct_rows(P, n_b, D, BLOCK);
  int32_t* sched = direct ? nullptr : reinterpret_cast<int32_t*>(ws + lay.sched);
  int* claim = direct ? nullptr : reinterpret_cast<int*>(ws + lay.claim);
  if (split) {
    int2* starts = reinterpret_cast<int2*>(ws + lay.starts);
    float* part = reinterpret_cast<float*>(ws + lay.part);
    hipLaunchKernelGGL(schedule_rows_kernel, dim3(direct ? 1 : kXcds + 1), dim3(1024), 0, s, kv_cnt,
                       sched, claim, P, n_b, starts, slots, run_rule<D, BLOCK>());
    hipLaunchKernelGGL((sparse_attn_bf16_kernel<D, BLOCK, Rows::kSplit>), dim3(slots),
                       dim3(2 * BLOCK), 0, s, q, k, v, o, lse, kv_idx, kv_cnt, sched, claim, P, L,
                       n_b, c, nullptr, 0, H, 1, part, L, starts);
    hipLaunchKernelGGL((row_combine_kernel<D, BLOCK>), dim3(slots), dim3(kRowCombThreads), 0, s,
                       part, starts, n_b, L, o, lse);
    return;
  }
  if (direct && rows > kXcds * kCusPerXcd) {
    hipLaunchKernelGGL((sparse_attn_bf16_kernel<D, BLOCK, Rows::kDirect>), dim3(rows),
                       dim3(2 * BLOCK), 0, s, q, k, v, o, lse, kv_idx, kv_cnt, nullptr, nullptr, P,
                       L, n_b, c, nullptr, 0, H, 1, nullptr, L, nullptr);
    return;
  }
  if (!direct)
    hipLaunchKernelGGL(schedule_rows_kernel, dim3(kXcds), dim3(1024), 0, s, kv_cnt, sched, claim, P,
                       n_b, nullptr, 0, RunRule{});
  hipLaunchKernelGGL((sparse_attn_bf16_kernel<D, BLOCK, Rows::kList>), dim3(direct ? rows : slots),
                     dim3(2 * BLOCK), 0, s, q, k, v, o, lse, kv_idx, kv_cnt, sched, claim, P, L,
                     n_b, c, nullptr, 0, H, 1, nullptr, L, nullptr);
}

static void sparse_attention_bf16(const uint16_t* q, const uint16_t* k, const uint16_t* v,
                                  uint16_t* o, float* lse, int B, int H, int L, int d, float scale,
                                  int block, const int32_t* kv_idx, const int32_t* kv_cnt, char* ws,
                                  bool split, hipStream_t s) {
#define SA_ATTN(DV, BV)                                                                    \
  sparse_attention_bf16<DV, BV>(q, k, v, o, lse, B, H, L, scale, kv_idx, kv_cnt, ws, split, s)
  if (d == 128 && block == 128)
    SA_ATTN(128, 128);
  else if (d == 128)
    SA_ATTN(128, 64);
  else if (block == 128)
    SA_ATTN(64, 128);
  else
    SA_ATTN(64, 64);
#undef SA_ATTN
}

void launch_sparse_attention_bf16(const uint16_t* q, const uint16_t* k,
                                  const uint16_t* v, uint16_t* o, float* lse,
                                  int B, int H, int L, int d, float scale,
                                  int block, const int32_t* kv_idx,
                                  const int32_t* kv_cnt, char* ws,
                                  hipStream_t s) {
  sparse_attention_bf16(q, k, v, o, lse, B, H, L, d, scale, block, kv_idx, kv_cnt, ws, false, s);
}

void launch_sparse_attention_split_bf16(const uint16_t* q, const uint16_t* k, const uint16_t* v,
                                        uint16_t* o, float* lse, int B, int H, int L, int d,
                                        float scale, int block, const int32_t* kv_idx,
                                        const int32_t* kv_cnt, char* ws, hipStream_t s) {
  sparse_attention_bf16(q, k, v, o, lse, B, H, L, d, scale, block, kv_idx, kv_cnt, ws, true, s);
}

void launch_sparse_attention_f32(const float* q, const float* k,
                                 const float* v, float* o, float* lse, int B,
                                 int H, int L, int d, float scale, int block,
                                 const int32_t* kv_idx, const int32_t* kv_cnt,
                                 char* /*ws*/, hipStream_t s) {
  const int n_b = ceil_div(L, block);
  const dim3 grid(B * H, n_b * (block / kF32Rows));
  if (d == 128)
    hipLaunchKernelGGL((sparse_attn_f32_kernel<128, false>), grid, dim3(64 * kF32Waves), 0, s, q,
                       k, v, o, lse, kv_idx, kv_cnt, L, n_b, block, log2_scale(scale), nullptr, 0,
                       H);
  else
    hipLaunchKernelGGL((sparse_attn_f32_kernel<64, false>), grid, dim3(64 * kF32Waves), 0, s, q,
                       k, v, o, lse, kv_idx, kv_cnt, L, n_b, block, log2_scale(scale), nullptr, 0,
                       H);
}

// Dense rows gathered from Q ([B,H,Lq,d]; rows[b*n_rows + j], or j when rows
// is NULL) against every key of K/V ([B,H,Lk,d]), in blocks of 128 rows;
// with more than one key split the partials go to ws and
// token_combine_kernel writes O/lse.
void launch_gather_attention_bf16(const uint16_t* q, const uint16_t* k, const uint16_t* v,
                                  uint16_t* o, float* lse, int B, int H, int Lq, int Lk,
                                  int d, float scale, const int32_t* rows, int n_rows,
                                  char* ws, hipStream_t s) {
  const int n_b = ceil_div(Lk, kTokRowBlock);
  const int P = B * H;
  const float c = scale * kLog2e;
  const int ns = token_attn_splits(P, n_rows, n_b);
  float* part = ns > 1 ? reinterpret_cast<float*>(ws) : nullptr;
  const dim3 grid(P * ceil_div(n_rows, kTokRowBlock) * ns);
  if (d == 128)
    hipLaunchKernelGGL((sparse_attn_bf16_kernel<128, kTokRowBlock, Rows::kGather>), grid,
                       dim3(256), 0, s, q, k, v, o, lse, nullptr, nullptr, nullptr, nullptr, P, Lk,
                       n_b, c, rows, n_rows, H, ns, part, Lq, nullptr);
  else
    hipLaunchKernelGGL((sparse_attn_bf16_kernel<64, kTokRowBlock, Rows::kGather>), grid,
                       dim3(256), 0, s, q, k, v, o, lse, nullptr, nullptr, nullptr, nullptr, P, Lk,
                       n_b, c, rows, n_rows, H, ns, part, Lq, nullptr);
  if (ns > 1) {
    const size_t threads = static_cast<size_t>(P) * n_rows * (d / 4);
    const dim3 cgrid(static_cast<unsigned>((threads + 255) / 256));
    if (d == 128)
      hipLaunchKernelGGL(token_combine_kernel<128>, cgrid, dim3(256), 0, s, part, ns, P, Lq, H,
                         rows, n_rows, o, lse);
    else
      hipLaunchKernelGGL(token_combine_kernel<64>, cgrid, dim3(256), 0, s, part, ns, P, Lq, H,
                         rows, n_rows, o, lse);
  }
}

// Dense rows of the protected tokens (Eq. (11) first case), written over O
// and lse.
void launch_protected_token_attention_bf16(const uint16_t* q, const uint16_t* k,
                                           const uint16_t* v, uint16_t* o, float* lse,
                                           int B, int H, int L, int d, float scale,
                                           const int32_t* tok_idx, int k_tok, char* ws,
                                           hipStream_t s) {
  launch_gather_attention_bf16(q, k, v, o, lse, B, H, L, L, d, scale, tok_idx, k_tok, ws, s);
}

// Cross-modal attention: every query of Q [B,H,Lq,d] against K/V [B,H,Lk,d].
void launch_cross_attention_bf16(const uint16_t* q, const uint16_t* k, const uint16_t* v,
                                 uint16_t* o, float* lse, int B, int H, int Lq, int Lk, int d,
                                 float scale, char* ws, hipStream_t s) {
  launch_gather_attention_bf16(q, k, v, o, lse, B, H, Lq, Lk, d, scale, nullptr, Lq, ws, s);
}

void launch_protected_token_attention_f32(const float* q, const float* k, const float* v,
                                          float* o, float* lse, int B, int H, int L, int d,
                                          float scale, const int32_t* tok_idx, int k_tok,
                                          hipStream_t s) {
  const dim3 grid(B * H, ceil_div(k_tok, kF32Rows));
  if (d == 128)
    hipLaunchKernelGGL((sparse_attn_f32_kernel<128, true>), grid, dim3(64 * kF32Waves), 0, s, q,
                       k, v, o, lse, nullptr, nullptr, L, 0, 0, log2_scale(scale), tok_idx, k_tok,
                       H);
  else
    hipLaunchKernelGGL((sparse_attn_f32_kernel<64, true>), grid, dim3(64 * kF32Waves), 0, s, q,
                       k, v, o, lse, nullptr, nullptr, L, 0, 0, log2_scale(scale), tok_idx, k_tok,
                       H);
}

}  // namespace sa
