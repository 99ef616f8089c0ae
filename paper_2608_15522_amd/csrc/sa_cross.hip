// Cross-modal saliency (Sec. 4.1, Eq. (1)-(2) and the reverse v->a
// direction).
//
// a->v: s^v_i = 1/(H*L_a) * sum_h sum_j softmax_i(scale * q^a_j . k^v_i).
//   K1 a2v_lse_partial : per (key chunk, 512-query slab, b*h) one 8-wave
//                        workgroup holding the slab's audio queries (64 per
//                        wave) streams the chunk's video keys with
//                        S^T = K^v Q^a^T, so a lane owns an audio query and
//                        keeps a lane-local (max, sum); partials go to
//                        workspace.
//   K1b lse_combine    : fixed-order merge of the chunk partials (log2 units).
//   K2 a2v_colmass     : per (key chunk, h, b) the workgroup streams the
//                        chunk's video keys once per audio slab with
//                        S = Q^a K^v^T, so a lane owns a video key column and
//                        sums exp2(S*c - lse) over its query rows; the 16
//                        lane partials of a key are added in a fixed order.
// v->a: s^a_j = 1/(H*L_v) * sum_h sum_i softmax_j(scale * q^v_i . k^a_j).
//   K3 v2a_colmass     : per (512 video queries, b*h); pass 1 streams every
//                        audio key with S^T for each video query's
//                        log-sum-exp, pass 2 streams them again, 512 at a
//                        time, with S and sums the column mass of each key.
// Both: saliency_finalize, one launch of fixed-order sums: over heads, / (H*L_a)
// and per block for the video map; over video chunks and heads, / (H*L_v), for
// the audio map.
// From the forwards: with the row LSEs of the a->v and v->a cross-attention
// forwards (natural log, as the attention kernels write them), K1/K1b and
// pass 1 of K3 are skipped: K2 reads lse_a and K3 lse_v.
// All bf16 kernels share one key-stream engine (below).  No atomics: every
// output element has one writer, so results are reproducible.
// fp32 inputs run the same two passes on fp32 matrix products (fp32 path below).
#include <float.h>

#include <algorithm>

#include "sa_device.h"
#include "sa_internal.h"

namespace sa {
namespace {

template <int D>
__device__ __forceinline__ void load_qfrag(const uint16_t* base, int row, int nrows,
                                           int g, u32x4* qf) {
#pragma unroll
  for (int kc = 0; kc < D / 16; ++kc)
    qf[kc] = row < nrows ? ldg16(base + static_cast<size_t>(row) * D + 16 * kc + 8 * g)
                         : u32x4{0u, 0u, 0u, 0u};
}

// sum_{i < n} p[i * stride], added in index order; the loads are issued in
// batches of 8 so that they are in flight together.
__device__ __forceinline__ float sum_strided(const float* __restrict__ p, size_t stride,
                                             int n) {
  float acc = 0.f;
  int i = 0;
  for (; i + 8 <= n; i += 8) {
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = p[static_cast<size_t>(i + k) * stride];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc += v[k];
  }
  for (; i < n; ++i) acc += p[static_cast<size_t>(i) * stride];
  return acc;
}

// ---- bf16 key-stream engine (K1, K2, K3) -------------------------------------
// A workgroup of 8 waves holds 512 query rows in registers, 64 per wave as two
// 32-row MFMA blocks, and streams 64-key tiles of one key matrix through an
// LDS ring (plane layout of sa_device.h) in groups of two tiles: the copy of
// the next group is in flight while the current one is read.  A wave works in units of 32 keys
// (one half of a tile): the D/8 MFMAs of unit u+1 are interleaved with the
// exponentials of unit u, so that the matrix cores and the vector ALU of a
// SIMD work at the same time.
constexpr int kXW = 8;                 // waves per workgroup
constexpr int kXNT = kXW * 64;         // threads per workgroup
constexpr int kGroup = 2;              // tiles per barrier interval
constexpr int kRing = 2 * kGroup;      // stages of the LDS key ring
static_assert(kXW * 64 == kQSlab && kXW * 64 == kV2aChunk,
              "one workgroup holds one slab of 512 query rows");
constexpr int kColKeys = kMaxKeyChunk;  // video keys per K2 workgroup, at most
constexpr int kAWin = 512;             // audio keys per K3 column-mass window
// A log-sum-exp unit whose sum against the running max reaches 2^64 is
// redone against its own max (the running max is only raised then).
constexpr float kSumGuard = 18446744073709551616.0f;

template <int D>
struct KeyRing {
  static constexpr int TB = 128 * D;            // bytes per 64-key tile
  static constexpr int CPT = TB / (16 * kXNT);  // 16-byte copies per thread per tile
  static_assert(CPT >= 1 && CPT * 16 * kXNT == TB, "tile copy split");
  uint32_t lds;         // LDS byte address of stage 0
  uint32_t span[CPT];   // byte offset of this wave's 1 KB spans in a stage
  int row[CPT];         // tile row copied by this lane
  uint32_t col[CPT];    // byte offset of the lane's source slot within the row
  int rd[2];            // lane offsets of the operand reads (k-step even / odd)

  __device__ __forceinline__ void init(char* ring, int wave, int lane) {
    lds = (uint32_t)(size_t)(lds_void_t*)ring;
    const int n = lane & 31, g = lane >> 5;
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int sp = wave + kXW * i;  // span sp = plane sp/4, rows 16*(sp%4) ..
      span[i] = sp * 1024;
      row[i] = 16 * (sp & 3) + (lane >> 2);
      col[i] = static_cast<uint32_t>((sp >> 2) * 64 + 16 * ((lane & 3) ^ plane_swz(row[i])));
    }
    // operand row n (+32 for the second unit of a tile), slot 2*(kc&1) + g
    rd[0] = n * 64 + 16 * (g ^ plane_swz(n));
    rd[1] = n * 64 + 16 * ((2 + g) ^ plane_swz(n));
  }
  // Copy keys [key0, key0 + 64) of the [L][D] matrix at src into stage st;
  // rows past L repeat row L - 1.
  __device__ __forceinline__ void issue(const char* src, int key0, int L, int st) const {
    const char* base = src + static_cast<size_t>(key0) * (2 * D);
    const int limit = min(63, L - 1 - key0);
#pragma unroll
    for (int i = 0; i < CPT; ++i)
      lds_dma16(base, static_cast<uint32_t>(min(row[i], limit) * (2 * D)) + col[i],
                __builtin_amdgcn_readfirstlane(lds + st * TB + span[i]));
  }
};

// MFMAs of one unit: keys 32*kb .. 32*kb+31 of the tile at `tile` against both
// query blocks, into acc.  KEYS_A: acc[h] = K Q_h^T (a lane owns a query
// column, its 16 elements are keys crow(i, g)); otherwise acc[h] = Q_h K^T (a
// lane owns a key column, its elements are query rows 32h + crow(i, g)).
// work(s), s = 0 .. D/8-1, runs on the vector ALU before the s-th MFMA.
template <int D, bool KEYS_A, class W>
__device__ __forceinline__ void unit_mfma(const char* tile, const int (&rd)[2], int kb,
                                          const u32x4 (&qf)[2][D / 16], f32x16 (&acc)[2],
                                          W&& work) {
  constexpr int KC = D / 16;
  auto rdk = [&](int kc) {
    return *reinterpret_cast<const u32x4*>(tile + (kc >> 1) * 4096 + kb * 2048 + rd[kc & 1]);
  };
  u32x4 kf[KC];
  kf[0] = rdk(0);
  kf[1] = rdk(1);
#pragma unroll
  for (int kc = 0; kc < KC; ++kc) {
    if (kc + 2 < KC) kf[kc + 2] = rdk(kc + 2);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      work(2 * kc + h);
      const f32x16 c0 = kc == 0 ? zero16() : acc[h];
      acc[h] = KEYS_A ? mfma32x32x16(kf[kc], qf[h][kc], c0) : mfma32x32x16(qf[h][kc], kf[kc], c0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// Wait until at most n (0 <= n <= N, wave-uniform) vector-memory operations
// of this wave are outstanding.
template <int N>
__device__ __forceinline__ void wait_vm_le(int n) {
  if constexpr (N > 0) {
    if (n >= N) {
      wait_vm<N>();
      return;
    }
    wait_vm_le<N - 1>(n);
  } else {
    wait_vm<0>();
  }
}

// Streams tiles t = 0 .. T-1 (T >= 1) of keys key_begin + 64t of the [L][D]
// matrix at src; unit u = 2t + kb.  Tiles go through the ring in groups of
// kGroup (stage t % kRing): the copies of group j+1 are issued right after
// the barrier that opens group j, whose stages held group j-1, and are
// awaited at the barrier that opens group j+1, so one barrier serves
// 2*kGroup units of every wave.  acc.first(x) sees unit 0 once,
// acc.slot(x, s, u, last) is the share of the work on a finished unit placed
// beside the s-th MFMA of the next one, acc.fin(x, u, last) closes the unit;
// `last` marks the units of tile T-1.  Ends with a barrier (ring free).
template <int D, bool KEYS_A, class Acc>
__device__ __forceinline__ void stream_keys(const KeyRing<D>& ring, const char* ring_lds,
                                            const char* src, int key_begin, int L, int T,
                                            const u32x4 (&qf)[2][D / 16], Acc& acc) {
  constexpr int TB = KeyRing<D>::TB, CPT = KeyRing<D>::CPT, NS = D / 8;
  auto issue_group = [&](int grp) {
#pragma unroll
    for (int i = 0; i < kGroup; ++i) {
      const int t = grp * kGroup + i;
      if (t < T) ring.issue(src, key_begin + 64 * t, L, t % kRing);
    }
  };
  issue_group(0);
  issue_group(1);
  // group 0 has landed once at most the copies of group 1 are outstanding
  wait_vm_le<kGroup * CPT>(CPT * min(kGroup, max(0, T - kGroup)));
  __syncthreads();
  f32x16 a[2], b[2];
  unit_mfma<D, KEYS_A>(ring_lds, ring.rd, 0, qf, a, [](int) {});
  acc.first(a);
  for (int t = 0; t + 1 < T; ++t) {
    unit_mfma<D, KEYS_A>(ring_lds + (t % kRing) * TB, ring.rd, 1, qf, b,
                         [&](int s) { acc.slot(a, s, 2 * t, false); });
    acc.fin(a, 2 * t, false);
    if ((t + 1) % kGroup == 0) {
      wait_vm<0>();  // this wave's copies of the group that opens here
      __syncthreads();
      issue_group((t + 1) / kGroup + 1);
    }
    unit_mfma<D, KEYS_A>(ring_lds + ((t + 1) % kRing) * TB, ring.rd, 0, qf, a,
                         [&](int s) { acc.slot(b, s, 2 * t + 1, false); });
    acc.fin(b, 2 * t + 1, false);
  }
  unit_mfma<D, KEYS_A>(ring_lds + ((T - 1) % kRing) * TB, ring.rd, 1, qf, b,
                       [&](int s) { acc.slot(a, s, 2 * T - 2, true); });
  acc.fin(a, 2 * T - 2, true);
#pragma unroll
  for (int s = 0; s < NS; ++s) acc.slot(b, s, 2 * T - 1, true);
  acc.fin(b, 2 * T - 1, true);
  __syncthreads();
}

// Lane-local online log2-sum-exp over the keys of KEYS_A units, for the two
// query columns of the lane.  The running max m starts at the max of unit 0
// (the lowest finite value at least: against it units whose scores are all
// -inf, wherever a chunk begins, weigh 0 instead of -inf - -inf) and is raised
// only when a unit's sum against it reaches kSumGuard, so the per-score work is
// one FMA, one exp2 and one add.  Keys >= key_end (tail of the last tile) are
// masked to -inf.
template <int D>
struct LseAcc {
  static constexpr int VPS = 32 / (D / 8);  // scores per lane per slot
  float m[2], l[2], rs[2];
  float c;
  int key_begin, key_end, g;

  __device__ __forceinline__ float val(const f32x16 (&x)[2], int h, int i, int u,
                                       bool last) const {
    const float v = x[h][i];
    return (last && key_begin + 32 * u + crow(i, g) >= key_end) ? -INFINITY : v;
  }
  __device__ __forceinline__ void first(const f32x16 (&x)[2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float mx = x[h][0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mx = fmaxf(mx, x[h][i]);
      m[h] = fmaxf(mx * c, -FLT_MAX);
      l[h] = 0.f;
    }
  }
  __device__ __forceinline__ void slot(const f32x16 (&x)[2], int s, int u, bool last) {
#pragma unroll
    for (int j = 0; j < VPS; ++j) {
      const int v = s * VPS + j, h = v >> 4, i = v & 15;
      const float p = fast_exp2(fmaf(val(x, h, i, u, last), c, -m[h]));
      rs[h] = i == 0 ? p : rs[h] + p;
    }
    // keep this slot's share beside its MFMA (the compiler would otherwise
    // sink it towards the first use of the sum)
    asm volatile("" : "+v"(rs[(s * VPS) >> 4]));
  }
  __device__ __forceinline__ void fin(const f32x16 (&x)[2], int u, bool last) {
    if (!(rs[0] < kSumGuard) || !(rs[1] < kSumGuard)) redo(x, u, last);
    l[0] += rs[0];
    l[1] += rs[1];
  }
  // Rare path: raise the running max to the unit's max and redo its sum.
  __device__ __forceinline__ void redo(const f32x16 (&x)[2], int u, bool last) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (!(rs[h] < kSumGuard)) {
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, val(x, h, i, u, last));
        const float mn = fmaxf(m[h], mx * c);
        float r = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) r += fast_exp2(fmaf(val(x, h, i, u, last), c, -mn));
        l[h] *= fast_exp2(m[h] - mn);
        m[h] = mn;
        rs[h] = r;
      }
    }
  }
  // (max, sum) of query column h over the keys of both lane halves.
  __device__ __forceinline__ float2 merged(int h) const {
    const float m2 = swap_halves(m[h]), l2 = swap_halves(l[h]);
    const float mm = fmaxf(m[h], m2);
    float lt = 0.f;
    if (mm > -INFINITY) lt = l[h] * fast_exp2(m[h] - mm) + l2 * fast_exp2(m2 - mm);
    return make_float2(mm, lt);
  }
};

// Column mass of !KEYS_A units: the lane sums 2^(S*c - lse_row) over its 32
// query rows and adds it to its own LDS slot of the unit's key (one writer
// per slot, fixed order).  Rows without a query carry lse = +inf.
template <int D>
struct ColAcc {
  static constexpr int VPS = 32 / (D / 8);
  float lr[2][16];
  float cs;
  float c;
  float* red;  // this lane's slot row, offset by its key column n

  __device__ __forceinline__ void first(const f32x16 (&)[2]) {}
  __device__ __forceinline__ void slot(const f32x16 (&x)[2], int s, int, bool) {
#pragma unroll
    for (int j = 0; j < VPS; ++j) {
      const int v = s * VPS + j, h = v >> 4, i = v & 15;
      const float p = fast_exp2(fmaf(x[h][i], c, -lr[h][i]));
      cs = v == 0 ? p : cs + p;
    }
    asm volatile("" : "+v"(cs));
  }
  __device__ __forceinline__ void fin(const f32x16 (&)[2], int u, bool) { red[32 * u] += cs; }
};

// ---- block means fused into the streams (Sec. 4.2, Eq. (6)) ------------------
// The mean of Q^v and of K^v over each block of `block` tokens (the last block
// over its true length), written as [d][n_pad] per (b,h) like the mask call's
// own pooling.  A sum of at most 128 bf16 values (8 significant bits each) is
// exact in fp64 whenever their magnitudes lie within 2^44 of each other, so
// the means equal that pooling bit for bit whatever the order of the
// additions, and are divided once.

// 8 bf16 of a 16-byte chunk added to acc in fp64.
__device__ __forceinline__ void add_bf16x8(u32x4 v, double (&acc)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    acc[2 * i] += static_cast<double>(__uint_as_float(v[i] << 16));
    acc[2 * i + 1] += static_cast<double>(__uint_as_float(v[i] & 0xffff0000u));
  }
}

// x summed over the 16 lanes of its DPP row, the same total in every lane:
// lane pairs (quad_perm 1,0,3,2), then quads (2,3,0,1), then the two halves
// of each 8 lanes (half-row mirror) and of the row (row mirror).  Each step
// moves the two dwords of x with DPP and adds in fp64.
__device__ __forceinline__ double dpp_row_sum(double x) {
  auto step = [](double v, int ctrl) {
    const uint64_t u = static_cast<uint64_t>(__double_as_longlong(v));
    const int lo = static_cast<int>(u & 0xffffffffu), hi = static_cast<int>(u >> 32);
    int plo, phi;
    switch (ctrl) {  // the DPP control must be a constant
      case 0:
        plo = __builtin_amdgcn_mov_dpp(lo, 0xB1, 0xF, 0xF, false);
        phi = __builtin_amdgcn_mov_dpp(hi, 0xB1, 0xF, 0xF, false);
        break;
      case 1:
        plo = __builtin_amdgcn_mov_dpp(lo, 0x4E, 0xF, 0xF, false);
        phi = __builtin_amdgcn_mov_dpp(hi, 0x4E, 0xF, 0xF, false);
        break;
      case 2:
        plo = __builtin_amdgcn_mov_dpp(lo, 0x141, 0xF, 0xF, false);
        phi = __builtin_amdgcn_mov_dpp(hi, 0x141, 0xF, 0xF, false);
        break;
      default:
        plo = __builtin_amdgcn_mov_dpp(lo, 0x140, 0xF, 0xF, false);
        phi = __builtin_amdgcn_mov_dpp(hi, 0x140, 0xF, 0xF, false);
        break;
    }
    const uint64_t w = (static_cast<uint64_t>(static_cast<uint32_t>(phi)) << 32) |
                       static_cast<uint32_t>(plo);
    return v + __longlong_as_double(static_cast<long long>(w));
  };
  x = step(x, 0);
  x = step(x, 1);
  x = step(x, 2);
  return step(x, 3);
}

// Keys of a column-mass stream (K2), pooled from the LDS ring.  Lane l of
// wave w takes d quarter q = 4w + l/16 (d = 4q .. 4q+3) of key rows l % 16 and
// l % 16 + 16 of every 32-key unit, read while the unit's MFMAs run; at the
// end of a block the 16 lanes that share q (one DPP row) add their sums
// (dpp_row_sum), and the lane of row 0 writes the 4 means.  Waves from D/16
// on (at d = 64) take no part.
template <int D>
struct KeyPool {
  static constexpr int TB = KeyRing<D>::TB;
  double acc[4];
  u32x2 raw[2];
  const char* ring;    // LDS ring, stage 0
  int off;             // lane offset of its quarter of row l % 16 in a unit
  int key_begin, L, block, nunits, n_pad;
  bool on;             // wave-uniform: this wave pools
  double* dst;         // kbar + pair * D * n_pad

  __device__ __forceinline__ void init(const char* ring_lds, int wave, int lane, int key_begin_,
                                       int L_, int block_, int T, int n_pad_, double* dst_) {
    const int r = lane & 15;
    const int q = 4 * wave + (lane >> 4);  // = threadIdx.x / 16
    on = 4 * wave < D / 4;
    const int cc = q >> 1;  // 16-byte chunk; the plane swizzle of rows r, r + 16 and
                            // 32*kb + r is that of row r
    off = (cc >> 2) * 4096 + r * 64 + 16 * ((cc & 3) ^ plane_swz(r)) + 8 * (q & 1);
    ring = ring_lds;
    key_begin = key_begin_;
    L = L_;
    block = block_;
    nunits = 2 * T;
    n_pad = n_pad_;
    dst = dst_;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = 0.0;
  }
  // unit p = keys key_begin + 32p ..; tile p/2 sits in stage (p/2) % kRing
  __device__ __forceinline__ void load(int p) {
    if (on && p < nunits) {
      const char* base = ring + ((p >> 1) % kRing) * TB + (p & 1) * 2048 + off;
      raw[0] = *reinterpret_cast<const u32x2*>(base);
      raw[1] = *reinterpret_cast<const u32x2*>(base + 16 * 64);
    }
  }
  // Dword part (0..3) of the unit's two rows: 2 elements.
  __device__ __forceinline__ void add(int p, int part) {
    if (on && p < nunits) {
      const int j = part >> 1, i = part & 1;
      uint32_t v = raw[j][i];
      // rows past L repeat row L-1 in the ring: they add nothing
      if (key_begin + 32 * p + 32 > L && key_begin + 32 * p + (threadIdx.x & 15) + 16 * j >= L)
        v = 0u;
      acc[2 * i] += static_cast<double>(__uint_as_float(v << 16));
      acc[2 * i + 1] += static_cast<double>(__uint_as_float(v & 0xffff0000u));
    }
  }
  // After unit p: at the end of a block, sum over the 32 rows and write.
  __device__ __forceinline__ void close(int p) {
    const int upb = block >> 5;  // units per block
    if (!on || p >= nunits || (p % upb != upb - 1 && p != nunits - 1)) return;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = dpp_row_sum(acc[e]);
    const int c = (key_begin + 32 * p) / block;
    const int len = min(block, L - c * block);
    if ((threadIdx.x & 15) == 0) {
      const int q = threadIdx.x >> 4;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        dst[static_cast<size_t>(4 * q + e) * n_pad + c] = acc[e] / static_cast<double>(len);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = 0.0;
  }
};

// ColAcc with the keys' block means: unit p = u + 1 (whose MFMAs run beside
// the slots of unit u) is read a few slots in and added two elements at a
// time beside four of the later MFMAs; unit 0 is pooled in first().
template <int D>
struct ColPoolAcc : ColAcc<D> {
  KeyPool<D> pool;
  static constexpr int NS = D / 8;
  __device__ __forceinline__ void first(const f32x16 (&)[2]) {
    pool.load(0);
#pragma unroll
    for (int part = 0; part < 4; ++part) pool.add(0, part);
    pool.close(0);
  }
  __device__ __forceinline__ void slot(const f32x16 (&x)[2], int s, int u, bool last) {
    constexpr int GAP = NS / 8;  // slots between two parts
    if (s == NS / 4 - GAP) pool.load(u + 1);
    // the four dword parts beside four of the later MFMAs
    if (s >= NS / 4 && s < NS / 4 + 4 * GAP && (s - NS / 4) % GAP == 0)
      pool.add(u + 1, (s - NS / 4) / GAP);
    ColAcc<D>::slot(x, s, u, last);
  }
  __device__ __forceinline__ void fin(const f32x16 (&x)[2], int u, bool last) {
    ColAcc<D>::fin(x, u, last);
    pool.close(u + 1);
  }
};

// Query rows of a v->a workgroup (K3), pooled from a second load of the rows
// it has just loaded for its MFMAs (L2 hits).  Thread t takes block
// t / block of the kV2aChunk rows from row0, 16-byte chunk cc and every
// (block / CPR)-th row of that block (CPR rows); the partial sums go through
// `part` (32 KB of LDS, [thread][element]) and are added in a fixed order.
// Ends with a barrier, after which `part` may be reused.
template <int D>
__device__ __forceinline__ void pool_query_chunk(const uint16_t* __restrict__ src, int row0,
                                                 int L, int block, int n_pad,
                                                 double* __restrict__ dst, double* part) {
  constexpr int CPR = D / 8;
  const int t = threadIdx.x;
  const int bl = t / block, w = t % block;
  const int cc = w % CPR, rg = w / CPR;
  const int RG = block / CPR;  // row groups of a block
  const int rb = row0 + bl * block;
  double acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.0;
#pragma unroll
  for (int i0 = 0; i0 < CPR; i0 += 8) {
    u32x4 raw[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = rb + rg + RG * (i0 + i);
      raw[i] = r < L ? ldg16(src + static_cast<size_t>(r) * D + 8 * cc)
                     : u32x4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) add_bf16x8(raw[i], acc);
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) part[8 * t + e] = acc[e];
  __syncthreads();
  const int nbl = kV2aChunk / block;
  for (int o = t; o < nbl * D; o += kXNT) {
    const int b2 = o / D, dd = o % D;
    const int rs = row0 + b2 * block;
    if (rs >= L) continue;
    const int len = min(block, L - rs);
    const int base = b2 * block + dd / 8;  // thread of row group 0, chunk dd / 8
    double sum = 0.0;
    for (int g = 0; g < RG; ++g) sum += part[8 * (base + g * CPR) + (dd & 7)];
    dst[static_cast<size_t>(dd) * n_pad + rs / block] = sum / static_cast<double>(len);
  }
  __syncthreads();
}

// ---- K1 ---------------------------------------------------------------------
template <int D>
__global__ void __launch_bounds__(kXNT) __attribute__((amdgpu_waves_per_eu(2, 2)))
a2v_lse_partial_kernel(const uint16_t* __restrict__ q_a,
                       const uint16_t* __restrict__ k_v,
                       float2* __restrict__ part, int L_v, int L_a, int nchunk,
                       int chunk_keys, float c) {
  __shared__ __attribute__((aligned(1024))) char ring_lds[kRing * KeyRing<D>::TB];
  const int chunk = blockIdx.x, slab = blockIdx.y, pair = blockIdx.z;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 5, n = lane & 31;
  const int j0 = slab * kQSlab + wave * 64;  // first audio query row of the wave
  const int key_begin = chunk * chunk_keys;
  const int key_end = min(key_begin + chunk_keys, L_v);

  u32x4 qf[2][D / 16];
  const uint16_t* qh = q_a + static_cast<size_t>(pair) * L_a * D;
  load_qfrag<D>(qh, j0 + n, L_a, g, qf[0]);
  load_qfrag<D>(qh, j0 + 32 + n, L_a, g, qf[1]);
  KeyRing<D> ring;
  ring.init(ring_lds, wave, lane);
  LseAcc<D> acc;
  acc.c = c;
  acc.key_begin = key_begin;
  acc.key_end = key_end;
  acc.g = g;
  stream_keys<D, true>(ring, ring_lds,
                       reinterpret_cast<const char*>(k_v + static_cast<size_t>(pair) * L_v * D),
                       key_begin, L_v, ceil_div(key_end - key_begin, 64), qf, acc);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const float2 ml = acc.merged(h);
    const int j = j0 + 32 * h + n;
    if (g == 0 && j < L_a)
      part[(static_cast<size_t>(pair) * nchunk + chunk) * L_a + j] = ml;
  }
}

// lse2[t] = log2(sum over chunks of l * 2^m) for t = (pair, j): 16 threads a
// value merge the chunks ph, ph + 16, ... in order, then the 16 (max, sum)
// pairs are merged in order.  One thread a value took 9 us at 64 chunks of
// 1536 values (24 waves, two dependent passes over the chunks).
constexpr int kCombPhases = 16;
__global__ void __launch_bounds__(256)
lse_combine_kernel(const float2* __restrict__ part, float* __restrict__ lse2, int P,
                   int L_a, int nchunk) {
  __shared__ float2 red[kCombPhases][16];
  const int ph = threadIdx.x >> 4, jj = threadIdx.x & 15;
  const size_t n = static_cast<size_t>(P) * L_a;
  const size_t t = (static_cast<size_t>(blockIdx.z) * gridDim.x + blockIdx.x) * 16 + jj;
  // Every chunk counts, by its finite maximum (ph without a chunk: the lowest, and
  // a sum of 0): one whose sum is a NaN makes the value a NaN.
  float M = -FLT_MAX, S = 0.f;
  if (t < n) {
    const float2* p = part + t / L_a * nchunk * L_a + t % L_a;
    for (int c0 = ph; c0 < nchunk; c0 += 4 * kCombPhases) {
      float2 v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int c = c0 + k * kCombPhases;
        v[k] = c < nchunk ? p[static_cast<size_t>(c) * L_a] : make_float2(-FLT_MAX, 0.f);
      }
      float m = M;
#pragma unroll
      for (int k = 0; k < 4; ++k) m = fmaxf(m, v[k].x);
      float s = S * fast_exp2(M - m);
#pragma unroll
      for (int k = 0; k < 4; ++k) s += v[k].y * fast_exp2(v[k].x - m);
      M = m;
      S = s;
    }
  }
  red[ph][jj] = make_float2(M, S);
  __syncthreads();
  if (ph != 0 || t >= n) return;
#pragma unroll
  for (int k = 1; k < kCombPhases; ++k) M = fmaxf(M, red[k][jj].x);
  S = 0.f;
#pragma unroll
  for (int k = 0; k < kCombPhases; ++k) {
    const float2 v = red[k][jj];
    S += v.y * fast_exp2(v.x - M);
  }
  lse2[t] = M + __log2f(S);
}

// ---- K2 ---------------------------------------------------------------------
// a->v column mass: grid (ceil(L_v/chunk_keys), H, B); the workgroup streams its
// chunk_keys <= 1024 video keys once per slab of 512 audio queries (S = Q^a K^v^T, a lane
// owns a key column) and adds exp2(S*c - lse) into per-lane LDS slots; the 16
// slots of a key (8 waves x 2 lane halves) are then summed in a fixed order.
// Keys past L_v only reach their own columns, which are not written.  lse_mul
// turns the given LSEs into log2 units.
// POOL: the stream of the first slab also writes the block means of K^v
// (KeyPool) to kbar ([B,H,d,n_pad]).
template <int D, bool POOL>
__global__ void __launch_bounds__(kXNT) __attribute__((amdgpu_waves_per_eu(2, 2)))
a2v_colmass_kernel(const uint16_t* __restrict__ q_a,
                   const uint16_t* __restrict__ k_v,
                   const float* __restrict__ lse, float lse_mul, float* __restrict__ colmass,
                   int H, int L_v, int L_a, int chunk_keys, float c, double* __restrict__ kbar,
                   int block, int n_pad) {
  constexpr int RS = kColKeys + 32;  // slot row stride (the two lane halves use different banks)
  __shared__ __attribute__((aligned(1024))) char ring_lds[kRing * KeyRing<D>::TB];
  __shared__ float red[2 * kXW][RS];
  const int chunk = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 5, n = lane & 31;
  const int key_begin = chunk * chunk_keys;
  const int key_end = min(key_begin + chunk_keys, L_v);
  const size_t pair = static_cast<size_t>(b) * H + h;
  const uint16_t* qh = q_a + pair * L_a * D;
  const float* lh = lse + pair * L_a;
  const char* kh = reinterpret_cast<const char*>(k_v + pair * L_v * D);
  const int T = ceil_div(key_end - key_begin, 64);

  KeyRing<D> ring;
  ring.init(ring_lds, wave, lane);
  ColAcc<D> acc;
  acc.c = c;
  acc.red = &red[2 * wave + g][n];
#pragma unroll 4
  for (int k = 0; k < chunk_keys; k += 32) acc.red[k] = 0.f;  // the lane's own slots

  for (int slab = 0; slab * kQSlab < L_a; ++slab) {
    const int j0 = slab * kQSlab + wave * 64;
    u32x4 qf[2][D / 16];
    load_qfrag<D>(qh, j0 + n, L_a, g, qf[0]);
    load_qfrag<D>(qh, j0 + 32 + n, L_a, g, qf[1]);
    // unconditional loads at clamped rows, so that all 32 are in flight at once
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        acc.lr[hh][i] = lh[min(j0 + 32 * hh + crow(i, g), L_a - 1)];
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        acc.lr[hh][i] = j0 + 32 * hh + crow(i, g) < L_a ? acc.lr[hh][i] * lse_mul : INFINITY;
    if (POOL && slab == 0) {
      ColPoolAcc<D> pacc;
      static_cast<ColAcc<D>&>(pacc) = acc;
      pacc.pool.init(ring_lds, wave, lane, key_begin, L_v, block, T, n_pad,
                     kbar + pair * D * n_pad);
      stream_keys<D, false>(ring, ring_lds, kh, key_begin, L_v, T, qf, pacc);
    } else {
      stream_keys<D, false>(ring, ring_lds, kh, key_begin, L_v, T, qf, acc);
    }
  }
  for (int k = threadIdx.x; k < chunk_keys; k += kXNT) {
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < 2 * kXW; ++w) sum += red[w][k];
    if (key_begin + k < L_v) colmass[pair * L_v + key_begin + k] = sum;
  }
}

// ---- K3 ---------------------------------------------------------------------
// v->a column mass: grid (ceil(L_v/512), 1, P).  The workgroup holds 512
// video queries; pass 1 streams every audio key with S^T = K^a Q^v^T (a lane
// owns a video query) for its log2-sum-exp, pass 2 streams the audio keys
// again, one window of 512 at a time, with S = Q^v K^a^T and sums the column
// mass of each key over the 512 queries (per-lane LDS slots, fixed order).
// FROM_LSE: pass 1 is replaced by the natural-log LSE of each video query
// that a v->a cross-attention forward produced (lse_v [P][L_v]).
// qbar != NULL: the workgroup first writes the block means of its 512 video
// queries (pool_query_chunk) to qbar ([B,H,d,n_pad]).
template <int D, bool FROM_LSE>
__global__ void __launch_bounds__(kXNT) __attribute__((amdgpu_waves_per_eu(2, 2)))
v2a_colmass_kernel(const uint16_t* __restrict__ q_v,
                   const uint16_t* __restrict__ k_a, float* __restrict__ part,
                   int L_v, int L_a, int nchunk, float c, const float* __restrict__ lse_v,
                   double* __restrict__ qbar, int block, int n_pad) {
  constexpr int RS = kAWin + 32;
  __shared__ __attribute__((aligned(1024))) char ring_lds[kRing * KeyRing<D>::TB];
  __shared__ float red[2 * kXW][RS];
  __shared__ float lse_w[kXW][64];
  const int chunk = blockIdx.x, pair = blockIdx.z;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 5, n = lane & 31;
  const int i0 = chunk * kV2aChunk + wave * 64;  // first video query row of the wave
  const char* kah = reinterpret_cast<const char*>(k_a + static_cast<size_t>(pair) * L_a * D);

  u32x4 qf[2][D / 16];
  const uint16_t* qh = q_v + static_cast<size_t>(pair) * L_v * D;
  load_qfrag<D>(qh, i0 + n, L_v, g, qf[0]);
  load_qfrag<D>(qh, i0 + 32 + n, L_v, g, qf[1]);
  KeyRing<D> ring;
  ring.init(ring_lds, wave, lane);
  if (qbar != nullptr)  // the ring is free until the first stream
    pool_query_chunk<D>(qh, chunk * kV2aChunk, L_v, block, n_pad,
                        qbar + static_cast<size_t>(pair) * D * n_pad,
                        reinterpret_cast<double*>(ring_lds));

  if constexpr (FROM_LSE) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int row = i0 + 32 * h + n;
      if (g == 0)
        lse_w[wave][32 * h + n] =
            row < L_v ? lse_v[static_cast<size_t>(pair) * L_v + row] * kLog2e : INFINITY;
    }
  } else {
    // pass 1: log2-sum-exp of every video query over all audio keys
    LseAcc<D> acc;
    acc.c = c;
    acc.key_begin = 0;
    acc.key_end = L_a;
    acc.g = g;
    stream_keys<D, true>(ring, ring_lds, kah, 0, L_a, ceil_div(L_a, 64), qf, acc);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float2 ml = acc.merged(h);
      // rows past L_v get +inf: their probabilities are exactly 0
      if (g == 0) lse_w[wave][32 * h + n] = (i0 + 32 * h + n < L_v) ? ml.x + __log2f(ml.y) : INFINITY;
    }
  }
  __syncthreads();

  // pass 2: column mass of the audio keys, one window of 512 keys at a time
  ColAcc<D> acc;
  acc.c = c;
  acc.red = &red[2 * wave + g][n];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc.lr[h][i] = lse_w[wave][32 * h + crow(i, g)];
  for (int key_begin = 0; key_begin < L_a; key_begin += kAWin) {
    const int key_end = min(key_begin + kAWin, L_a);
    if (key_begin > 0) __syncthreads();  // the previous window's slots have been read
    for (int k = 0; k < kAWin; k += 32) acc.red[k] = 0.f;
    // ends with a barrier: every wave's slots are complete below
    stream_keys<D, false>(ring, ring_lds, kah, key_begin, L_a,
                          ceil_div(key_end - key_begin, 64), qf, acc);
    for (int k = threadIdx.x; k < key_end - key_begin; k += kXNT) {
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < 2 * kXW; ++w) sum += red[w][k];
      part[(static_cast<size_t>(pair) * nchunk + chunk) * L_a + key_begin + k] = sum;
    }
  }
}

// ---- finalize ---------------------------------------------------------------
// Both directions' sums in one launch of 1024-thread workgroups, batch item
// blockIdx.y, workgroup w of its n_b + n_aud.
//  w in [0, n_b): sal_v_tok and sal_v_blk of one video block from the column
//    masses [B][H][L_v]: thread (ph, t) adds the heads ph, ph + NP, ... of
//    token t in order (NP = 1024 / block phases), the phases are added in
//    order, then the tokens by a tree.
//  the rest: sal_a_tok of 16 audio tokens from v2a_part [B][nparts][L_a]:
//    64 phases a token, added in phase order.
constexpr int kFinThreads = 1024;
constexpr int kFinAud = 16;  // audio tokens per workgroup
__global__ void __launch_bounds__(kFinThreads)
saliency_finalize_kernel(const float* __restrict__ colmass, float* __restrict__ sal_v_tok,
                         float* __restrict__ sal_v_blk, int H, int L_v, int block, float inv_norm_v,
                         const float* __restrict__ v2a_part, float* __restrict__ sal_a_tok,
                         int nparts, int L_a, int n_aud, float inv_norm_a, int accumulate) {
  __shared__ float red[kFinThreads];
  const int tid = threadIdx.x, n_b = ceil_div(L_v, block);
  const int b = blockIdx.y, w = blockIdx.z * gridDim.x + blockIdx.x;
  if (w < n_b) {
    const int c = w;
    const int NP = kFinThreads / block, ph = tid / block, t = tid % block;
    const int i = c * block + t;
    float v = 0.f;
    if (i < L_v && ph < H)
      v = sum_strided(colmass + (static_cast<size_t>(b) * H + ph) * L_v + i,
                      static_cast<size_t>(NP) * L_v, (H - ph + NP - 1) / NP);
    red[tid] = v;
    __syncthreads();
    if (tid < block) {
      for (int p = 1; p < NP; ++p) v += red[p * block + tid];
      v *= inv_norm_v;
      if (i < L_v && sal_v_tok != nullptr) {
        float* dst = sal_v_tok + static_cast<size_t>(b) * L_v + i;
        *dst = accumulate ? *dst + v : v;
      }
      red[tid] = v;
    }
    __syncthreads();
    for (int s = block / 2; s > 0; s >>= 1) {
      if (tid < s) red[tid] += red[tid + s];
      __syncthreads();
    }
    if (tid == 0) {
      float* dst = sal_v_blk + static_cast<size_t>(b) * n_b + c;
      *dst = accumulate ? *dst + red[0] : red[0];
    }
    return;
  }
  if (w - n_b >= n_aud) return;
  const int j = (w - n_b) * kFinAud + tid % kFinAud;
  constexpr int NP = kFinThreads / kFinAud;
  const int ph = tid / kFinAud;
  float v = 0.f;
  if (j < L_a && ph < nparts)
    v = sum_strided(v2a_part + (static_cast<size_t>(b) * nparts + ph) * L_a + j,
                    static_cast<size_t>(NP) * L_a, (nparts - ph + NP - 1) / NP);
  red[tid] = v;
  __syncthreads();
  // 8 threads a token add 8 phases each, the first of them those 8 sums
  if (tid < 8 * kFinAud) {
    const int g = tid / kFinAud;
    v = 0.f;
    for (int p = 0; p < NP / 8; ++p) v += red[(g * (NP / 8) + p) * kFinAud + tid % kFinAud];
  }
  __syncthreads();
  red[tid] = v;
  __syncthreads();
  if (tid < kFinAud && j < L_a) {
    v = 0.f;
    for (int g = 0; g < 8; ++g) v += red[g * kFinAud + tid];
    v *= inv_norm_a;
    float* dst = sal_a_tok + static_cast<size_t>(b) * L_a + j;
    *dst = accumulate ? *dst + v : v;
  }
}

// sal_a_tok == NULL: the a->v direction only.
void launch_finalize(const float* colmass, float* sal_v_tok, float* sal_v_blk, int B, int H,
                     int L_v, int block, const float* v2a_part, float* sal_a_tok, int nchunk3,
                     int L_a, int accumulate, hipStream_t s) {
  const int n_v = ceil_div(L_v, block);
  const int n_a = sal_a_tok != nullptr ? ceil_div(L_a, kFinAud) : 0;
  hipLaunchKernelGGL(saliency_finalize_kernel, wide_grid(static_cast<long>(n_v) + n_a, B),
                     dim3(kFinThreads), 0, s, colmass, sal_v_tok, sal_v_blk, H, L_v, block,
                     1.0f / (static_cast<float>(H) * static_cast<float>(L_a)), v2a_part, sal_a_tok,
                     H * nchunk3, L_a, n_a,
                     1.0f / (static_cast<float>(H) * static_cast<float>(L_v)), accumulate);
}

// ---- fp32 path --------------------------------------------------------------
// Both passes form 16 x 16 score tiles with v_mfma_f32_16x16x4_f32, one
// operand held in registers, the other streamed through LDS, and take both
// directions in one launch (a.n_wg + v.n_wg workgroups a pair: the first a.n_wg
// workgroups of a pair serve a->v, the rest v->a), because either alone leaves
// most of the chip idle at the sizes fp32 is used at.
// Log-sum-exps: 16 queries a workgroup, whose waves share out the key tiles,
// each through LDS buffers of its own (RowTile16).  Column masses: 16 keys a
// wave, four waves sharing the query tiles through one LDS ring (RowRing16);
// launches of at most one workgroup a CU (SPLIT = 4) have 16 waves, four groups
// that hold the same keys and share out the query tiles.  At B1 H4 L_v4680
// L_a512 d128 the passes take 68 and 66 us; with rings private to a wave
// the second took 85, a merge of the key chunks in a launch of its own 5 more.
constexpr int kF32XWaves = 4;
constexpr int kF32XRows = 16 * kF32XWaves;  // keys per column-mass workgroup
constexpr int kF32XLse = 512;               // queries whose LSEs are in LDS at a time
constexpr int kF32XMerge = 16;              // most LSE partials of a query

// One direction's share of a launch.
struct F32Dir {
  const float* q;   // [P][Lq][D]
  const float* k;   // [P][Lk][D]
  float* lse2;      // log2-sum-exp over each key chunk [P][nlse][Lq]
  float* out;       // column mass [P][nchunk][Lk]
  int Lq, Lk;
  int nlse;         // key chunks of the LSE pass
  int lse_chunk;    // keys per chunk, a multiple of 16
  int nchunk;       // query chunks of the column-mass pass
  int chunk;        // queries per chunk
  int n_wg;         // workgroups per pair of the launch at hand
};

// LDS ring of 16-row tiles shared by a group of four waves: a tile's 1 KB spans are
// copied by the waves in turn; slots are swizzled as in RowTile16.
template <int D>
struct RowRing16 {
  static constexpr int kBytes = 16 * D * 4;
  static constexpr int kCopies = kBytes / 1024 / kF32XWaves;  // per wave and tile
  static constexpr int kStages = 3;
  const char* lds;
  uint32_t lds_addr;
  int row[kCopies];
  uint32_t col[kCopies];
  int rd;

  __device__ __forceinline__ void init(char* ring, int wave, int lane) {
    lds = ring;
    lds_addr = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(lds_void_t*)ring +
                                              static_cast<uint32_t>(wave * kCopies * 1024));
#pragma unroll
    for (int i = 0; i < kCopies; ++i) {
      const int chunk = 64 * (wave * kCopies + i) + lane;
      row[i] = chunk / (D / 4);
      col[i] = 16u * static_cast<uint32_t>((chunk % (D / 4)) ^ row[i]);
    }
    const int n = lane & 15, gk = lane >> 4;
    rd = n * D * 4 + 16 * (gk ^ n);
  }
  // Rows [row0, row0 + 16) of the [L][D] matrix src (row0 < L) to stage st;
  // rows past L repeat row L - 1.
  __device__ __forceinline__ void copy(const float* src, int row0, int L, int st) const {
    const char* base = reinterpret_cast<const char*>(src + static_cast<size_t>(row0) * D);
    const int limit = L - 1 - row0;
#pragma unroll
    for (int i = 0; i < kCopies; ++i)
      lds_dma16(base, static_cast<uint32_t>(min(row[i], limit) * (D * 4)) + col[i],
                __builtin_amdgcn_readfirstlane(lds_addr + st * kBytes + i * 1024));
  }
  // f(row, tile) for the tiles at rows r0, r0 + 16, ... < r1 <= L (none for r1
  // <= r0), in T steps, the same for every group of the workgroup.  A barrier
  // opens each tile; the copy of the second tile after it goes out right
  // behind, into the stage that every wave has read before that barrier.
  // Begins after a barrier of the caller's, where an earlier stream used the
  // ring, and ends without copies in flight.
  template <class F>
  __device__ __forceinline__ void stream(const float* src, int r0, int r1, int L, int T,
                                         F&& f) const {
    const int own = r1 > r0 ? ceil_div(r1 - r0, 16) : 0;
#pragma unroll
    for (int t = 0; t < kStages - 1; ++t)
      if (t < own) copy(src, r0 + 16 * t, L, t);
    int st = 0;
    for (int t = 0; t < T; ++t) {
      // tile t has landed once at most the copies of t + 1 are out
      if (t + 1 < own)
        wait_vm<kCopies>();
      else
        wait_vm<0>();
      __syncthreads();
      f32x4 x[D / 16];
      const char* tile = lds + st * kBytes;
      if (t < own) {
#pragma unroll
        for (int i = 0; i < D / 16; ++i)
          x[i] = *reinterpret_cast<const f32x4*>(tile + (rd ^ (64 * i)));
      }
      const int free_st = st == 0 ? kStages - 1 : st - 1;
      if (t + kStages - 1 < own) copy(src, r0 + 16 * (t + kStages - 1), L, free_st);
      __builtin_amdgcn_sched_barrier(0);
      if (t < own) f(r0 + 16 * t, x);
      st = st + 1 == kStages ? 0 : st + 1;
    }
  }
};

template <int D>
__device__ __forceinline__ void load_row_f32(const float* base, int row, int L, int gk,
                                             f32x4 (&dst)[D / 16]) {
  const float* src = base + static_cast<size_t>(min(row, L - 1)) * D + 4 * gk;
#pragma unroll
  for (int i = 0; i < D / 16; ++i) dst[i] = ldg_f32x4(src + 16 * i);
}

// A B^T of two 16-row operands: element e of lane (n, gk) is row 4gk + e of A
// against row n of B.
template <int D>
__device__ __forceinline__ f32x4 tile_f32(const f32x4 (&a)[D / 16], const f32x4 (&b)[D / 16]) {
  f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < D / 16; ++i)
#pragma unroll
    for (int e = 0; e < 4; e += 2) {
      s0 = mfma16x16x4_f32(a[i][e], b[i][e], s0);
      s1 = mfma16x16x4_f32(a[i][e + 1], b[i][e + 1], s1);
    }
  return s0 + s1;
}

// Merge of two (max, sum) pairs; a pair without keys is (-inf, 0).
__device__ __forceinline__ float2 merge_lse(float2 a, float2 b) {
  const float m = fmaxf(a.x, b.x);
  if (m == -INFINITY) return make_float2(m, a.y + b.y);
  return make_float2(m, a.y * exp2f(a.x - m) + b.y * exp2f(b.x - m));
}

// Log2-sum-exp of scale * Q K^T over a chunk of keys: one workgroup per 16
// query rows, its waves taking the chunk's 16-key tiles in turn (S^T = K Q^T,
// so a lane keeps a running (max, sum) of query n over its own keys).
template <int D>
__global__ void __launch_bounds__(64 * kF32XWaves)
row_lse2_f32_kernel(F32Dir a, F32Dir v, Log2Scale c) {
  __shared__ __attribute__((aligned(1024))) char ring[kF32XWaves * 2 * RowTile16<D>::kBytes];
  __shared__ float2 red[kF32XWaves][16];
  const int w = blockIdx.z * gridDim.x + blockIdx.x;
  if (w >= a.n_wg + v.n_wg) return;
  const bool second = w >= a.n_wg;
  const F32Dir& p = second ? v : a;
  const int wg = w - (second ? a.n_wg : 0);
  const int nt = ceil_div(p.Lq, 16);
  const int qt = wg % nt, ch = wg / nt, pair = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = lane & 15, gk = lane >> 4;
  const int Lq = p.Lq, Lk = p.Lk;
  const int k0 = ch * p.lse_chunk, k1 = min(k0 + p.lse_chunk, Lk);
  f32x4 qf[D / 16];
  const float* kh = p.k + static_cast<size_t>(pair) * Lk * D;
  float m = -INFINITY, l = 0.f;
  constexpr int kStep = 16 * kF32XWaves;
  RowTile16<D> tile;
  tile.init(ring + wave * 2 * RowTile16<D>::kBytes, lane);
  int buf = 0;
  tile.copy(kh, k0 + 16 * wave, Lk, 0);
  load_row_f32<D>(p.q + static_cast<size_t>(pair) * Lq * D, 16 * qt + n, Lq, gk, qf);
  for (int key = k0 + 16 * wave; key < k1; key += kStep) {
    wait_dma();
    __builtin_amdgcn_sched_barrier(0);
    f32x4 kf[D / 16];
    tile.read(buf, kf);
    buf ^= 1;
    if (key + kStep < k1) tile.copy(kh, key + kStep, Lk, buf);
    __builtin_amdgcn_sched_barrier(0);
    const f32x4 s = tile_f32<D>(kf, qf);
    const float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])) * c.hi;
    if (__any(mx > m + 8.f)) {
      const float m_new = fmaxf(m, mx);
      l *= m == m_new ? 1.f : fast_exp2(m - m_new);
      m = m_new;
    }
    const float mref = m == -INFINITY ? 0.f : m;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x = fast_exp2(log2_score(s[e], c, mref));
      l += key + 4 * gk + e < k1 ? x : 0.f;
    }
  }
  wait_dma();  // a wave without tiles still has its first copy in flight
  float2 ml = make_float2(m, l);
#pragma unroll
  for (int o = 16; o <= 32; o <<= 1)
    ml = merge_lse(ml, make_float2(__shfl_xor(ml.x, o, 64), __shfl_xor(ml.y, o, 64)));
  if (gk == 0) red[wave][n] = ml;
  __syncthreads();
  const int row = 16 * qt + static_cast<int>(threadIdx.x);
  if (threadIdx.x < 16 && row < Lq) {
    ml = red[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < kF32XWaves; ++w) ml = merge_lse(ml, red[w][threadIdx.x]);
    p.lse2[(static_cast<size_t>(pair) * p.nlse + ch) * Lq + row] = ml.x + log2f(ml.y);
  }
}

// Column mass over a chunk of queries: out[pair][chunk][key] = sum over the
// chunk's queries of 2^(c * q . k - lse2[q]).  A wave holds 16 keys (S = Q
// K^T: a lane sums key n over the queries 4gk .. 4gk+3 of every tile) and
// streams the chunk, kF32XLse queries at a time, whose LSEs are merged into
// LDS first; the 4 lanes of a key are added at the end.
template <int D, int SPLIT>
__global__ void __launch_bounds__(64 * kF32XWaves * SPLIT)
    __attribute__((amdgpu_waves_per_eu(SPLIT > 1 ? 4 : 5)))
colmass_f32_kernel(F32Dir a, F32Dir v, Log2Scale c) {
  constexpr int kRingBytes = RowRing16<D>::kStages * RowRing16<D>::kBytes;
  __shared__ __attribute__((aligned(1024))) char ring_lds[SPLIT * kRingBytes];
  __shared__ float red[SPLIT][kF32XRows];
  __shared__ __attribute__((aligned(16))) float lse_s[kF32XLse];
  const int w = blockIdx.z * gridDim.x + blockIdx.x;
  if (w >= a.n_wg + v.n_wg) return;
  const bool second = w >= a.n_wg;
  const F32Dir& p = second ? v : a;
  const int wg = w - (second ? a.n_wg : 0);
  const int Lq = p.Lq, Lk = p.Lk;
  const int nt = ceil_div(Lk, kF32XRows);
  const int kt = wg % nt, ch = wg / nt, pair = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = (threadIdx.x >> 6) % kF32XWaves;
  const int part =
      SPLIT > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / (64 * kF32XWaves)) : 0;
  const int n = lane & 15, gk = lane >> 4;
  const int key = kt * kF32XRows + 16 * wave + n;
  const int q0 = ch * p.chunk, q1 = min(q0 + p.chunk, Lq);
  f32x4 kf[D / 16];
  load_row_f32<D>(p.k + static_cast<size_t>(pair) * Lk * D, key, Lk, gk, kf);
  float sum = 0.f;
  RowRing16<D> ring;
  ring.init(ring_lds + part * kRingBytes, wave, lane);
  for (int w0 = q0; w0 < q1; w0 += kF32XLse) {
    const int w1 = min(w0 + kF32XLse, q1);
    if (w0 > q0) __syncthreads();  // the previous window has been read
    for (int i = threadIdx.x; i < kF32XLse; i += 64 * kF32XWaves * SPLIT) {
      float x = INFINITY;  // past the chunk: adds 0
      if (w0 + i < w1) {
        const float* src = p.lse2 + static_cast<size_t>(pair) * p.nlse * Lq + w0 + i;
        x = src[0];
        if (p.nlse > 1) {
          float y[kF32XMerge];
#pragma unroll
          for (int j = 0; j < kF32XMerge; ++j)
            y[j] = j < p.nlse ? src[static_cast<size_t>(j) * Lq] : -INFINITY;
#pragma unroll
          for (int j = 1; j < kF32XMerge; ++j) x = fmaxf(x, y[j]);
          float t = 0.f;
#pragma unroll
          for (int j = 0; j < kF32XMerge; ++j) t += exp2f(y[j] - x);
          x = x == -INFINITY ? x : x + log2f(t);
        }
      }
      lse_s[i] = x;
    }
    // the stream's first barrier makes them visible
    const int T = ceil_div(ceil_div(w1 - w0, 16), SPLIT);
    const int s0 = w0 + 16 * T * part;
    ring.stream(p.q + static_cast<size_t>(pair) * Lq * D, s0, min(s0 + 16 * T, w1), Lq, T,
                [&](int q, const f32x4 (&qf)[D / 16]) {
      const f32x4 lr = *reinterpret_cast<const f32x4*>(&lse_s[q - w0 + 4 * gk]);
      const f32x4 s = tile_f32<D>(qf, kf);
      float t[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) t[e] = fast_exp2(log2_score(s[e], c, lr[e]));
      sum += (t[0] + t[1]) + (t[2] + t[3]);
    });
  }
  sum += __shfl_xor(sum, 16, 64);
  sum += __shfl_xor(sum, 32, 64);
  if constexpr (SPLIT > 1) {
    if (gk == 0) red[part][16 * wave + n] = sum;
    __syncthreads();
    if (part > 0) return;
#pragma unroll
    for (int j = 1; j < SPLIT; ++j) sum += red[j][16 * wave + n];
  }
  if (gk == 0 && key < Lk) p.out[(static_cast<size_t>(pair) * p.nchunk + ch) * Lk + key] = sum;
}

// Video keys per K1 or K2 workgroup: the multiple of 128 (whole blocks) up to
// kMaxKeyChunk that takes least time by rounds of the 256 workgroups that run
// at once (one per CU), a round lasting as many tiles as the chunk has plus
// kFill for the query slab's load and the pipeline's fill; `max_chunks` bounds
// their number (the room for K1's partials).  1024 keys leave a call of few
// heads or short clips on part of the chip (96 workgroups at H3 L_v32760).
int key_chunk(int L_v, long per_chunk, long max_chunks) {
  constexpr int kFill = 3;
  int best = kMaxKeyChunk;
  long best_cost = 0;
  for (int ck = kMaxKeyChunk; ck >= 128; ck -= 128) {
    const long n = ceil_div(L_v, ck);
    if (n > max_chunks) break;
    const long cost = (n * per_chunk + 255) / 256 * (std::min(ck, L_v) / 64 + kFill);
    if (ck == kMaxKeyChunk || cost < best_cost) {
      best = ck;
      best_cost = cost;
    }
  }
  return best;
}

// K2, with the block means of K^v written to kbar when it is not NULL.
template <int D>
void launch_a2v_colmass(const uint16_t* q_a, const uint16_t* k_v, const float* lse, float lse_mul,
                        float* colmass, int B, int H, int L_v, int L_a, float c, double* kbar,
                        int block, hipStream_t s) {
  const int ck = key_chunk(L_v, static_cast<long>(B) * H, L_v);
  const dim3 grid(ceil_div(L_v, ck), H, B);
  const int n_pad = mask_n_pad(ceil_div(L_v, block));
  if (kbar != nullptr)
    hipLaunchKernelGGL((a2v_colmass_kernel<D, true>), grid, dim3(kXNT), 0, s, q_a, k_v, lse,
                       lse_mul, colmass, H, L_v, L_a, ck, c, kbar, block, n_pad);
  else
    hipLaunchKernelGGL((a2v_colmass_kernel<D, false>), grid, dim3(kXNT), 0, s, q_a, k_v, lse,
                       lse_mul, colmass, H, L_v, L_a, ck, c, kbar, block, n_pad);
}

// The two column-mass passes and the sums, from the a->v row LSEs (times
// lse_mul in log2 units) and, when lse_v is not NULL, the v->a ones (natural
// log); otherwise K3 forms its own.
template <int D>
void column_masses(const uint16_t* q_a, const uint16_t* k_v, const uint16_t* q_v,
                   const uint16_t* k_a, const float* lse_a, float lse_mul, const float* lse_v,
                   int B, int H, int L_v, int L_a, float c, int block, float* sal_v_tok,
                   float* sal_v_blk, float* sal_a_tok, int accumulate, double* qbar, double* kbar,
                   const CrossWs& lay, char* ws, hipStream_t s) {
  float* colmass = reinterpret_cast<float*>(ws + lay.colmass);
  float* v2a_part = reinterpret_cast<float*>(ws + lay.v2a_part);
  launch_a2v_colmass<D>(q_a, k_v, lse_a, lse_mul, colmass, B, H, L_v, L_a, c, kbar, block, s);
  const int nchunk3 = ceil_div(L_v, kV2aChunk);
  if (q_v != nullptr) {
    const dim3 grid(nchunk3, 1, B * H);
    const int n_pad = mask_n_pad(ceil_div(L_v, block));
    if (lse_v != nullptr)
      hipLaunchKernelGGL((v2a_colmass_kernel<D, true>), grid, dim3(kXNT), 0, s, q_v, k_a, v2a_part,
                         L_v, L_a, nchunk3, c, lse_v, qbar, block, n_pad);
    else
      hipLaunchKernelGGL((v2a_colmass_kernel<D, false>), grid, dim3(kXNT), 0, s, q_v, k_a,
                         v2a_part, L_v, L_a, nchunk3, c, nullptr, qbar, block, n_pad);
  }
  launch_finalize(colmass, sal_v_tok, sal_v_blk, B, H, L_v, block, v2a_part,
                  q_v != nullptr ? sal_a_tok : nullptr, nchunk3, L_a, accumulate, s);
}

template <int D>
void cross_bf16(const uint16_t* q_a, const uint16_t* k_v, const uint16_t* q_v,
                const uint16_t* k_a, int B, int H, int L_v, int L_a, float scale,
                int block, float* sal_v_tok, float* sal_v_blk, float* sal_a_tok,
                int accumulate, double* qbar, double* kbar, char* ws, hipStream_t s) {
  const CrossWs lay = cross_ws_layout(B, H, L_v, L_a);
  const float c = scale * kLog2e;
  const int P = B * H;
  const int nslab = ceil_div(L_a, kQSlab);
  // K1's partials may fill the workspace up to v2a_head: nothing in that part
  // is in use before lse_combine has read them, and its result goes to
  // v2a_head, which the bf16 path does not need otherwise.
  float2* lse_part = reinterpret_cast<float2*>(ws + lay.lse_part);
  float* lse_a = reinterpret_cast<float*>(ws + lay.v2a_head);
  const size_t nlse = static_cast<size_t>(P) * L_a;
  const long max_chunks =
      static_cast<long>((lay.v2a_head - lay.lse_part) / (sizeof(float2) * nlse));
  const int ck = key_chunk(L_v, static_cast<long>(nslab) * P, max_chunks);
  const int nchunk = ceil_div(L_v, ck);
  hipLaunchKernelGGL(a2v_lse_partial_kernel<D>, dim3(nchunk, nslab, P), dim3(kXNT), 0, s,
                     q_a, k_v, lse_part, L_v, L_a, nchunk, ck, c);
  hipLaunchKernelGGL(lse_combine_kernel, wide_grid((nlse + 15) / 16), dim3(256), 0, s, lse_part,
                     lse_a, P, L_a, nchunk);
  column_masses<D>(q_a, k_v, q_v, k_a, lse_a, 1.f, nullptr, B, H, L_v, L_a, c, block, sal_v_tok,
                   sal_v_blk, sal_a_tok, accumulate, qbar, kbar, lay, ws, s);
}

// The saliency of both directions from the row LSEs of the two cross-
// attention forwards: K2 and K3's column-mass pass only.
template <int D>
void cross_bf16_from_lse(const uint16_t* q_a, const uint16_t* k_v, const uint16_t* q_v,
                         const uint16_t* k_a, const float* lse_a, const float* lse_v, int B,
                         int H, int L_v, int L_a, float scale, int block, float* sal_v_tok,
                         float* sal_v_blk, float* sal_a_tok, int accumulate, double* qbar,
                         double* kbar, char* ws, hipStream_t s) {
  column_masses<D>(q_a, k_v, q_v, k_a, lse_a, kLog2e, lse_v, B, H, L_v, L_a, scale * kLog2e,
                   block, sal_v_tok, sal_v_blk, sal_a_tok, accumulate, qbar, kbar,
                   cross_ws_layout(B, H, L_v, L_a), ws, s);
}

template <int D>
void cross_f32(const float* q_a, const float* k_v, const float* q_v,
               const float* k_a, int B, int H, int L_v, int L_a, float scale,
               int block, float* sal_v_tok, float* sal_v_blk, float* sal_a_tok,
               int accumulate, char* ws, hipStream_t s) {
  const Log2Scale c = log2_scale(scale);
  const int P = B * H;
  const int nchunk3 = ceil_div(L_v, kV2aChunk);
  const size_t n_v = static_cast<size_t>(P) * L_v, n_a = static_cast<size_t>(P) * L_a;
  size_t off = 0;
  auto take = [&](size_t n) {
    float* p = reinterpret_cast<float*>(ws + off);
    off += align_up(sizeof(float) * n);
    return p;
  };
  float* colmass = take(n_v);
  float* lse_v = take(n_v);
  float* v2a_part = take(n_a * nchunk3);
  float* lse_a = take(0);
  // Video keys per a->v log-sum-exp workgroup: kLseChunk (a sixteenth of longer
  // clips), whose partials the workspace has room for, or down to 256 while the
  // launch has less than two workgroups a CU and the rest of the workspace holds
  // the partials, which the column-mass workgroups merge where they read them
  // (11.3 -> 5.5 us at B1 H2 L_v1024 L_a128 d64; at H8 L_v4680 L_a512 d128
  // chunks of 400 keys were 10 us slower than 1024).
  const bool rev = q_v != nullptr;
  const long room =
      static_cast<long>((cross_ws_layout(B, H, L_v, L_a).total - off) / (sizeof(float) * n_a));
  auto lse_wgs = [&](int chunk) {
    return static_cast<long>(P) * (static_cast<long>(ceil_div(L_a, 16)) * ceil_div(L_v, chunk) +
                                   (rev ? ceil_div(L_v, 16) : 0));
  };
  int lse_chunk = std::max(kLseChunk, ceil_div(ceil_div(L_v, kF32XMerge), 16) * 16);
  while (lse_chunk > 256 && lse_wgs(lse_chunk) < 2 * kXcds * kCusPerXcd &&
         ceil_div(L_v, lse_chunk / 2) <= std::min(room, static_cast<long>(kF32XMerge)))
    lse_chunk /= 2;
  const int nlse = ceil_div(L_v, lse_chunk);
  F32Dir a{q_a, k_v, lse_a, colmass, L_a, L_v, nlse, lse_chunk, 1, L_a, 0};
  F32Dir v{q_v, k_a, lse_v, v2a_part, L_v, L_a, 1, L_a, nchunk3, kV2aChunk, 0};
  a.n_wg = ceil_div(L_a, 16) * nlse;
  v.n_wg = rev ? ceil_div(L_v, 16) : 0;
  hipLaunchKernelGGL(row_lse2_f32_kernel<D>, wide_grid(static_cast<long>(a.n_wg) + v.n_wg, P),
                     dim3(64 * kF32XWaves), 0, s, a, v, c);
  // Column masses: a->v over all audio queries, v->a in chunks of 512 video
  // queries.
  a.n_wg = ceil_div(L_v, kF32XRows);
  v.n_wg = rev ? ceil_div(L_a, kF32XRows) * nchunk3 : 0;
  const long n_wg = static_cast<long>(a.n_wg) + v.n_wg;
  const dim3 grid = wide_grid(n_wg, P);
  if (n_wg * P <= kXcds * kCusPerXcd)
    hipLaunchKernelGGL((colmass_f32_kernel<D, 4>), grid, dim3(4 * 64 * kF32XWaves), 0, s, a, v, c);
  else
    hipLaunchKernelGGL((colmass_f32_kernel<D, 1>), grid, dim3(64 * kF32XWaves), 0, s, a, v, c);
  launch_finalize(colmass, sal_v_tok, sal_v_blk, B, H, L_v, block, v2a_part,
                  q_v != nullptr ? sal_a_tok : nullptr, nchunk3, L_a, accumulate, s);
}

}  // namespace

void launch_cross_scores_bf16(const uint16_t* q_a, const uint16_t* k_v,
                              const uint16_t* q_v, const uint16_t* k_a, int B,
                              int H, int L_v, int L_a, int d, float scale,
                              int block, float* sal_v_tok, float* sal_v_blk,
                              float* sal_a_tok, int accumulate, double* qbar,
                              double* kbar, char* ws, hipStream_t s) {
  if (d == 128)
    cross_bf16<128>(q_a, k_v, q_v, k_a, B, H, L_v, L_a, scale, block, sal_v_tok,
                    sal_v_blk, sal_a_tok, accumulate, qbar, kbar, ws, s);
  else
    cross_bf16<64>(q_a, k_v, q_v, k_a, B, H, L_v, L_a, scale, block, sal_v_tok,
                   sal_v_blk, sal_a_tok, accumulate, qbar, kbar, ws, s);
}

void launch_cross_scores_from_lse_bf16(const uint16_t* q_a, const uint16_t* k_v,
                                       const uint16_t* q_v, const uint16_t* k_a,
                                       const float* lse_a, const float* lse_v, int B, int H,
                                       int L_v, int L_a, int d, float scale, int block,
                                       float* sal_v_tok, float* sal_v_blk, float* sal_a_tok,
                                       int accumulate, double* qbar, double* kbar,
                                       char* ws, hipStream_t s) {
  if (d == 128)
    cross_bf16_from_lse<128>(q_a, k_v, q_v, k_a, lse_a, lse_v, B, H, L_v, L_a, scale, block,
                             sal_v_tok, sal_v_blk, sal_a_tok, accumulate, qbar, kbar, ws, s);
  else
    cross_bf16_from_lse<64>(q_a, k_v, q_v, k_a, lse_a, lse_v, B, H, L_v, L_a, scale, block,
                            sal_v_tok, sal_v_blk, sal_a_tok, accumulate, qbar, kbar, ws, s);
}

void launch_cross_scores_f32(const float* q_a, const float* k_v,
                             const float* q_v, const float* k_a, int B, int H,
                             int L_v, int L_a, int d, float scale, int block,
                             float* sal_v_tok, float* sal_v_blk,
                             float* sal_a_tok, int accumulate, char* ws,
                             hipStream_t s) {
  if (d == 128)
    cross_f32<128>(q_a, k_v, q_v, k_a, B, H, L_v, L_a, scale, block, sal_v_tok,
                   sal_v_blk, sal_a_tok, accumulate, ws, s);
  else
    cross_f32<64>(q_a, k_v, q_v, k_a, B, H, L_v, L_a, scale, block, sal_v_tok,
                  sal_v_blk, sal_a_tok, accumulate, ws, s);
}

}  // namespace sa
