// Token-granular protection (Sec. 4.1 Eq. (3)/(8) at token level) and the
// lagged saliency update (Eq. (4)).
//
// K8 saliency_ema: s_bar = alpha * s_bar + (1 - alpha) * s, elementwise fp32.
// K9 select_tokens: per batch item one workgroup (one wave up to L = 512,
//    else 1024 threads) finds the k_tok-th smallest value key T (saliency
//    descending) of the L tokens by a radix search: the bits that every key
//    shares are decided by one AND/OR reduction, then each step decides eight
//    bits from an LDS histogram of the prefix group's digits, until one key is
//    left in the group.  Tokens tied at T are taken in index order.  Each wave
//    owns a contiguous range of tokens (in registers up to L = 32768), read 64
//    consecutive tokens at a time, so ballot prefix counts and one scan of the
//    per-wave totals write the kept tokens in ascending order.
//    Bound by latency: one workgroup, a chain of barriers.  Two bits a step
//    (counts by wave sums, candidates copied to LDS) took 53 us at L =
//    32760, 17 at 2049 and 10 at 512 against 27, 8 and 8.
// The dense attention rows of the protected tokens are the gather variant of
// the attention kernel (sa_attn.hip).
#include "sa_device.h"
#include "sa_internal.h"

namespace sa {
namespace {

// ---- K8 ---------------------------------------------------------------------
__global__ void __launch_bounds__(256)
saliency_ema_kernel(float* __restrict__ s_bar, const float* __restrict__ s, size_t n,
                    float alpha) {
  const float beta = 1.0f - alpha;
  for (size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += static_cast<size_t>(gridDim.x) * blockDim.x)
    s_bar[i] = fmaf(alpha, s_bar[i], beta * s[i]);
}

// ---- K9 ---------------------------------------------------------------------
constexpr int kDigitBits = 8;  // bits decided per step

// Exclusive prefix over the NW waves of a per-wave value (given by every
// lane of the wave); ends with a barrier after the LDS slots are read.
template <int NW>
__device__ __forceinline__ int wave_exclusive_base(int v, int* wave_tot) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) wave_tot[wave] = v;
  __syncthreads();
  int base = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w)
    if (w < wave) base += wave_tot[w];
  __syncthreads();
  return base;
}

// The order key of a token is its value key: the fp32 saliency mapped to a
// monotone integer and inverted, so that a larger saliency is a smaller key.
// The k_tok-th smallest value key T is found first; tokens with a key below T
// are kept, and of the tokens whose key equals T the lowest indices fill the
// remaining places (larger saliency first, then lower index).
// NT threads (NW = NT/64 waves); wave w owns the tokens [w*S, (w+1)*S),
// S = ceil(L/NW); lane l holds tokens w*S + 64 j + l.  R > 0: the keys stay
// in registers (64 R >= S); R == 0: they are read from global memory on
// every pass.
template <int R, int NT>
__global__ void __launch_bounds__(NT)
select_tokens_kernel(const float* __restrict__ sal, int L, int k_tok,
                     int32_t* __restrict__ tok_idx, uint8_t* __restrict__ tok_flag) {
  constexpr int NW = NT / 64;
  constexpr int kDigits = 1 << kDigitBits;
  static_assert(kDigits == 4 * 64, "a lane of wave 0 scans four digits");
  __shared__ __attribute__((aligned(16))) uint32_t hist[kDigits];
  __shared__ int sel_sh[3];
  __shared__ uint32_t red_sh[NW][2];
  __shared__ int wave_tot[NW];
  const int b = blockIdx.x;
  const float* s = sal + static_cast<size_t>(b) * L;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int S = ceil_div(L, NW);
  const int w0 = min(wave * S, L), w1 = min(w0 + S, L);
  const int J = R > 0 ? R : ceil_div(S, 64);
  const uint64_t lanes_below = (1ull << lane) - 1ull;

  constexpr int RR = R > 0 ? R : 1;
  uint32_t vk[RR];
  if constexpr (R > 0) {
    // unconditional loads at a clamped index, so that all of them are in
    // flight at once
    float x[R];
#pragma unroll
    for (int j = 0; j < R; ++j) x[j] = s[min(w0 + 64 * j + lane, L - 1)];
#pragma unroll
    for (int j = 0; j < R; ++j) vk[j] = w0 + 64 * j + lane < w1 ? ~float_order_key(x[j]) : 0u;
  }
  // f(key, token, valid) for j = 0 .. J-1, the same j on every lane
  auto for_all = [&](auto f) {
    if constexpr (R > 0) {
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const int i = w0 + 64 * j + lane;
        f(vk[j], i, i < w1);
      }
    } else {
      for (int j0 = 0; j0 < J; j0 += 8) {  // eight loads in flight
        float x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = s[min(w0 + 64 * (j0 + u) + lane, L - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int i = w0 + 64 * (j0 + u) + lane;
          const bool ok = i < w1;
          f(ok ? ~float_order_key(x[u]) : 0u, i, ok);
        }
      }
    }
  };
  auto for_keys = [&](auto f) {
    for_all([&](uint32_t key, int, bool ok) {
      if (ok) f(key);
    });
  };

  auto first_lane = [](uint64_t m) { return __ffsll(static_cast<unsigned long long>(m)) - 1; };
  // Whether the wave's keys share their digits so much that adding them one by one
  // would serialise (the LDS takes a wave's adds to one address in turn): judged by
  // the first and the middle 64 of them, as runs of equal saliencies (a floor, zeros)
  // are what makes them so.  At 32760 tokens a constant map but for one token took
  // 136 us without this and 50 with it (two bits a step: 99), a floor under 90 % of
  // the tokens 125 and 51 (89), and a saliency map 26.7 and 27.1.  One wave's adds
  // (up to 512 tokens) are faster one by one (8 us against 11), and keys read again
  // from memory on every pass stay ahead of two bits a step without it (277 against
  // 300 at 65536).
  auto crowded = [&](auto counts, auto digit) {
    if constexpr (R > 0 && NW > 1) {
      int most = 0;
#pragma unroll
      for (int j = 0; j < R; j += R / 2) {
        const bool in = w0 + 64 * j + lane < w1 && counts(vk[j]);
        const uint64_t m = __ballot(in);
        if (m == 0) continue;
        const uint32_t d = digit(vk[j]);
        const uint32_t d0 = __builtin_amdgcn_readlane(d, first_lane(m));
        most = max(most, static_cast<int>(__popcll(__ballot(in && d == d0))));
      }
      return most >= 32;
    } else {
      return false;
    }
  };

  // Search for T, for 0 < k_tok < L.  `fixed` marks the decided bits of T,
  // `prefix` their values; `below` keys lie under the prefix group and
  // `size` keys share it.  k_tok == L keeps every token, k_tok == 0 none.
  uint32_t prefix = 0, fixed = 0;
  int below = 0, size = L;
  if (k_tok > 0 && k_tok < L) {
    // bits that every key shares are decided at once
    uint32_t a = 0xffffffffu, o = 0u;
    for_keys([&](uint32_t key) { a &= key; o |= key; });
    a = __reduce_and_sync(~0ull, a);
    o = __reduce_or_sync(~0ull, o);
    if (lane == 0) {
      red_sh[wave][0] = a;
      red_sh[wave][1] = o;
    }
    __syncthreads();
    a = 0xffffffffu;
    o = 0u;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      a &= red_sh[w][0];
      o |= red_sh[w][1];
    }
    const uint32_t diff = a ^ o;
    int hb = diff != 0u ? 31 - __clz(diff) : -1;  // highest undecided bit
    fixed = hb >= 0 ? ~static_cast<uint32_t>((2ull << hb) - 1ull) : 0xffffffffu;
    prefix = a & fixed;
    while (hb >= 0 && size > 1) {
      const int lo = max(hb - (kDigitBits - 1), 0);
      const uint32_t digit_mask = (2u << (hb - lo)) - 1u;
      for (int i = tid; i < kDigits; i += NT) hist[i] = 0u;
      __syncthreads();
      auto counts = [&](uint32_t key) { return (key & fixed) == prefix; };
      auto digit = [&](uint32_t key) { return (key >> lo) & digit_mask; };
      if (crowded(counts, digit)) {
        // one add for the keys that share the digit of the wave's first one
        for_all([&](uint32_t key, int, bool ok) {
          const bool in = ok && counts(key);
          const uint64_t m = __ballot(in);
          if (m == 0) return;
          const uint32_t d = digit(key);
          const uint32_t d0 = __builtin_amdgcn_readlane(d, first_lane(m));
          const uint64_t same = __ballot(in && d == d0);
          if (in && d != d0) atomicAdd(&hist[d], 1u);
          if (lane == 0) atomicAdd(&hist[d0], static_cast<uint32_t>(__popcll(same)));
        });
      } else {
        for_keys([&](uint32_t key) {
          if (counts(key)) atomicAdd(&hist[digit(key)], 1u);
        });
      }
      __syncthreads();
      if (wave == 0) {
        // the digit that holds the k_tok-th key, in the lane of its four
        const u32x4 h = *reinterpret_cast<const u32x4*>(&hist[4 * lane]);
        int incl = static_cast<int>(h[0] + h[1] + h[2] + h[3]);
        int at = below - incl;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int u = __shfl_up(incl, o, 64);
          if (lane >= o) incl += u;
        }
        at += incl;  // keys below the lane's digits
        if (at < k_tok && below + incl >= k_tok) {
          int j = 0;
#pragma unroll
          for (int e = 0; e < 3; ++e)
            if (j == e && at + static_cast<int>(h[e]) < k_tok) {
              at += static_cast<int>(h[e]);
              j = e + 1;
            }
          sel_sh[0] = 4 * lane + j;
          sel_sh[1] = at;
          sel_sh[2] = static_cast<int>(j == 0 ? h[0] : j == 1 ? h[1] : j == 2 ? h[2] : h[3]);
        }
      }
      __syncthreads();
      prefix |= static_cast<uint32_t>(sel_sh[0]) << lo;
      fixed |= digit_mask << lo;
      below = sel_sh[1];
      size = sel_sh[2];
      hb = lo - 1;
    }
  }
  // size > 1 here only if every bit is decided: `size` keys equal T, and the
  // k_tok - below lowest-index ones among them are kept
  const bool ties = k_tok > 0 && k_tok < L && size > 1;
  const int need = k_tok - below;
  auto is_tie = [&](uint32_t key, bool ok) { return ties && ok && key == prefix; };
  auto kept = [&](uint32_t key, bool ok, int tie_rank) {
    if (!ok || k_tok == 0) return false;
    if (k_tok == L) return true;
    if (!ties) return (key & fixed) <= prefix;
    return key < prefix || (key == prefix && tie_rank < need);
  };
  // tokens before this wave's range that tie at T, and that are kept
  int tie_wave = 0;
  if (ties) {  // uniform over the workgroup
    for_all([&](uint32_t key, int, bool ok) { tie_wave += __popcll(__ballot(is_tie(key, ok))); });
  }
  const int tie_base = ties ? wave_exclusive_base<NW>(tie_wave, wave_tot) : 0;
  int kept_wave = 0;
  {
    int tr = tie_base;
    for_all([&](uint32_t key, int, bool ok) {
      const uint64_t tb = __ballot(is_tie(key, ok));
      const bool on = kept(key, ok, tr + __popcll(tb & lanes_below));
      tr += __popcll(tb);
      kept_wave += __popcll(__ballot(on));
    });
  }
  int pos = wave_exclusive_base<NW>(kept_wave, wave_tot);
  int32_t* out = tok_idx != nullptr ? tok_idx + static_cast<size_t>(b) * k_tok : nullptr;
  uint8_t* flag = tok_flag != nullptr ? tok_flag + static_cast<size_t>(b) * L : nullptr;
  int tr = tie_base;
  for_all([&](uint32_t key, int i, bool ok) {
    const uint64_t tb = __ballot(is_tie(key, ok));
    const bool on = kept(key, ok, tr + __popcll(tb & lanes_below));
    tr += __popcll(tb);
    const uint64_t kb = __ballot(on);
    const int p = pos + __popcll(kb & lanes_below);
    pos += __popcll(kb);
    // exactly k_tok tokens are kept; the bound only keeps the writes inside
    // tok_idx whatever the input values are
    if (on && out != nullptr && p < k_tok) out[p] = i;
    if (ok && flag != nullptr) flag[i] = on ? 1 : 0;
  });
}

}  // namespace

void launch_saliency_ema(float* s_bar, const float* s, size_t n, float alpha, hipStream_t st) {
  const size_t blocks = n / 256 + 1 < 4096 ? n / 256 + 1 : 4096;
  hipLaunchKernelGGL(saliency_ema_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0,
                     st, s_bar, s, n, alpha);
}

void launch_select_protected_tokens(const float* sal_tok, int B, int L, int k_tok,
                                    int32_t* tok_idx, uint8_t* tok_flag, hipStream_t st) {
  const dim3 grid(B);
#define SA_SELECT(R, NT)                                                                 \
  hipLaunchKernelGGL((select_tokens_kernel<R, NT>), grid, dim3(NT), 0, st, sal_tok, L, k_tok, \
                     tok_idx, tok_flag)
  // One wave up to 512 tokens (no barrier costs anything there); from there on
  // 16 waves (8 us at 2049 tokens, one wave with 32 tokens a lane 15 at 2048).
  if (L <= 512) {
    SA_SELECT(8, 64);
  } else {  // tokens per lane ceil(ceil(L/16)/64)
    const int J = ceil_div(ceil_div(L, 16), 64);
    if (J <= 4)
      SA_SELECT(4, 1024);
    else if (J <= 16)
      SA_SELECT(16, 1024);
    else if (J <= 32)
      SA_SELECT(32, 1024);
    else
      SA_SELECT(0, 1024);
  }
#undef SA_SELECT
}

}  // namespace sa
