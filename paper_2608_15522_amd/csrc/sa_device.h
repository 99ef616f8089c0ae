// Device helpers shared by the gfx950 kernels of libsa.so.
//
// MFMA operand layout used throughout (v_mfma_f32_32x32x16_bf16, wave64):
//   A operand (32 x 16): lane l holds row (l % 32), 8 consecutive k values
//                        starting at 8 * (l / 32);
//   B operand (16 x 32): lane l holds column (l % 32), the same 8 k values;
//   C/D (32 x 32, 16 floats per lane): element r of lane l sits at
//       row crow(r, l / 32) = 8 * (r / 4) + 4 * (l / 32) + r % 4,
//       column l % 32.
// A and B are always filled symmetrically (the same k index for the same
// lane half and element), so a contraction is correct whatever order the
// hardware gives the k values inside a lane.
#pragma once

#include <float.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr int kWave = 64;

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

__device__ __forceinline__ constexpr int crow(int r, int g) {
  return 8 * (r >> 2) + 4 * g + (r & 3);
}

__device__ __forceinline__ f32x16 mfma32x32x16(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(
      __builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// fp32 products and sums: v_mfma_f32_16x16x4_f32.  A[i][k] sits in lane
// i + 16k, B[k][j] in lane j + 16k, and C/D[i][j] in lane j + 16(i / 4),
// element i % 4.  It runs at 64 flop per cycle and SIMD, twice the rate of
// scalar fp32 FMAs, with the same fp32 rounding of products and sums.
__device__ __forceinline__ f32x4 mfma16x16x4_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 ldg_f32x4(const float* p) {
  return *reinterpret_cast<const f32x4*>(p);
}

// scale * log2(e) as an fp32 pair: the product's own rounding (2^-24 of it with
// one fp32 factor) drops out of a score.  lo > 0, so that both parts of a score of
// -inf are -inf (-inf * hi - inf * lo would be a NaN for lo < 0, and for lo = 0).
struct Log2Scale {
  float hi, lo;
};
// c * s - ref in two FMAs, good to an ulp of the larger of ref and the result.
__device__ __forceinline__ float log2_score(float s, Log2Scale c, float ref) {
  return fmaf(s, c.hi, fmaf(s, c.lo, -ref));
}
inline Log2Scale log2_scale(float scale) {
  const double c = static_cast<double>(scale) * 1.4426950408889634;
  float hi = static_cast<float>(c);
  if (static_cast<double>(hi) >= c) hi = nextafterf(hi, 0.f);
  return {hi, fmaxf(static_cast<float>(c - static_cast<double>(hi)), FLT_MIN)};
}

__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.f;
  return z;
}

// bf16 <-> f32.  The conversion to bf16 rounds to nearest even.
__device__ __forceinline__ float bf16_to_f32(uint16_t h) {
  return __uint_as_float(static_cast<uint32_t>(h) << 16);
}
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Value held by the lane 32 positions away (the other half of the wave).
__device__ __forceinline__ float swap_halves(float x) {
  return __shfl_xor(x, 32, 64);
}

__device__ __forceinline__ float fast_exp2(float x) {
  return __builtin_amdgcn_exp2f(x);
}

typedef __attribute__((address_space(3))) void lds_void_t;

// LDS tile layout: D/32 "planes" of [64 keys][32 d] bf16 (64 bytes per key
// row, 4 KB per plane); 16-byte slot s of row r is stored at slot
// s ^ plane_swz(r).  With this swizzle both the K operand reads
// (ds_read_b128: 16 consecutive rows, one slot) and the transposing V reads
// (ds_read_b64_tr_b16: 4 consecutive rows, two slots) are free of bank
// conflicts, and every read address is a lane constant plus an immediate.
__device__ __forceinline__ constexpr int plane_swz(int r) {
  return ((r >> 2) & 1) | ((((r >> 1) ^ (r >> 3)) & 1) << 1);
}

// Copy of 16 bytes per lane, global -> LDS (global_load_lds_dwordx4): lane l
// writes LDS bytes [lds_addr + 16*l, +16) with the 16 bytes at sbase + voff.
// A 64-key tile of a [L][D] bf16 matrix is 4*D such chunks, i.e. 4*D/64 spans
// of 1 KB; chunk i of the tile is LDS byte 16*i = plane i/256, row (i%256)/4,
// physical slot i%4, holding logical slot (i%4) ^ plane_swz(row).
//
// The copy is issued with inline assembly on purpose: the compiler cannot
// tell that an in-flight copy into one buffer does not alias the operand
// reads of the other, and would otherwise wait for every copy (vmcnt(0))
// before the first LDS read that follows it, serialising the pipeline.  The
// kernel orders the buffers itself: s_waitcnt vmcnt(0) and a barrier end
// every iteration, before any copied tile is read or a buffer is refilled.
__device__ __forceinline__ void lds_dma16(const char* sbase, uint32_t voff, uint32_t lds_addr) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %0, %1"
      :
      : "v"(voff), "s"(sbase), "s"(lds_addr)
      : "memory", "m0");
}

__device__ __forceinline__ void wait_dma() {
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
}
// Wait until at most n (< 16) vector-memory operations of this wave are
// outstanding; they complete in issue order.
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 16, "vmcnt field");
  __builtin_amdgcn_s_waitcnt(0x0F70 | N);
}

// A wave's private LDS buffers for 16-row tiles of an fp32 [L][D] matrix that
// feed v_mfma_f32_16x16x4_f32 as one operand: lane (n, gk) = (l % 16, l / 16)
// needs 16 bytes at channel 16i + 4gk of row n.  Loaded straight from memory
// that way, consecutive lanes lie in 16 different rows and the CU's L1 takes
// them one by one (11-14 bytes per cycle measured, the bound of the kernels
// then); copied row by row into LDS they come in at full width.  16-byte
// slot s of row r sits at slot s ^ r, so that the 16 rows of an operand read
// fall into different banks.  Only the wave itself reads a buffer, so its own
// vmcnt wait orders the copy and no barrier is needed.
template <int D>
struct RowTile16 {
  static constexpr int kBytes = 16 * D * 4;     // one tile
  static constexpr int kCopies = kBytes / 1024;  // copy instructions per tile
  const char* lds;          // the wave's two buffers
  uint32_t lds_addr;        // their LDS byte address
  int row[kCopies];         // tile row copied by this lane
  uint32_t col[kCopies];    // byte offset of the lane's source slot in the row
  int rd;                   // lane offset of the operand reads (XOR 64i)

  __device__ __forceinline__ void init(char* wave_lds, int lane) {
    lds = wave_lds;
    lds_addr = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(lds_void_t*)wave_lds);
#pragma unroll
    for (int i = 0; i < kCopies; ++i) {
      const int chunk = 64 * i + lane;
      row[i] = chunk / (D / 4);
      col[i] = 16u * static_cast<uint32_t>((chunk % (D / 4)) ^ row[i]);
    }
    const int n = lane & 15, gk = lane >> 4;
    rd = n * D * 4 + 16 * (gk ^ n);
  }
  // Copy rows [row0, row0 + 16) of src into buffer b; rows past L repeat row
  // L - 1.  row0 is wave-uniform.
  __device__ __forceinline__ void copy(const float* src, int row0, int L, int b) const {
    const int first = __builtin_amdgcn_readfirstlane(min(row0, L - 1));
    const char* base = reinterpret_cast<const char*>(src + static_cast<size_t>(first) * D);
    const int limit = L - 1 - first;
#pragma unroll
    for (int i = 0; i < kCopies; ++i)
      lds_dma16(base, static_cast<uint32_t>(min(row[i], limit) * (D * 4)) + col[i],
                lds_addr + b * kBytes + i * 1024);
  }
  __device__ __forceinline__ void read(int b, f32x4 (&dst)[D / 16]) const {
#pragma unroll
    for (int i = 0; i < D / 16; ++i)
      dst[i] = *reinterpret_cast<const f32x4*>(lds + b * kBytes + (rd ^ (64 * i)));
  }
};

__device__ __forceinline__ u32x4 ldg16(const void* p) {
  return *reinterpret_cast<const u32x4*>(p);
}
// The same load with the nontemporal cache policy (`nt`), for data that a
// pass reads exactly once.  On gfx950 the block pooling's reads of Q^v and
// K^v ran at about 6.1 TB/s with it against 5.0-5.4 TB/s without (same
// kernel and box).
__device__ __forceinline__ u32x4 ldg16_nt(const void* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}
__device__ __forceinline__ void stg16(void* p, u32x4 v) {
  *reinterpret_cast<u32x4*>(p) = v;
}

// Monotone map of a float to an unsigned integer (larger float -> larger
// integer); -0.0 is folded into +0.0 so equal values compare equal.
__device__ __forceinline__ uint32_t float_order_key(float v) {
  uint32_t u = __float_as_uint(v);
  if ((u & 0x7fffffffu) == 0u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Sort key for "value descending, index ascending" as one ascending u64.
__device__ __forceinline__ uint64_t desc_value_asc_index_key(float v,
                                                            uint32_t idx) {
  return (static_cast<uint64_t>(~float_order_key(v)) << 32) | idx;
}

// Sort key for "value descending, index ascending" from a double: the low 12
// bits of the order-preserving image are replaced by the index (idx < 4096),
// so values within 2^-40 relative of each other rank as ties (lower index
// first).
__device__ __forceinline__ uint64_t desc_double_asc_index_key(double v,
                                                             uint32_t idx) {
  uint64_t u = static_cast<uint64_t>(__double_as_longlong(v));
  if ((u & 0x7fffffffffffffffull) == 0ull) u = 0ull;
  const uint64_t ord = (u >> 63) ? ~u : (u | 0x8000000000000000ull);
  return (~ord & ~0xfffull) | idx;
}

// In-place ascending bitonic sort of n (a power of two) keys in LDS by the
// whole workgroup.  Ends with a barrier.
__device__ __forceinline__ void bitonic_sort_lds(uint64_t* keys, int n) {
  const int tid = threadIdx.x;
  const int nt = blockDim.x;
  for (int size = 2; size <= n; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      __syncthreads();
      for (int t = tid; t < (n >> 1); t += nt) {
        const int lo = 2 * t - (t & (stride - 1));
        const int hi = lo + stride;
        const bool up = (lo & size) == 0;
        const uint64_t a = keys[lo];
        const uint64_t b = keys[hi];
        if ((a > b) == up) {
          keys[lo] = b;
          keys[hi] = a;
        }
      }
    }
  }
  __syncthreads();
}

__host__ __device__ constexpr int ceil_div(int a, int b) {
  return (a + b - 1) / b;
}

__host__ __device__ constexpr size_t align_to_8(size_t x) {
  return (x + 7) & ~static_cast<size_t>(7);
}

__host__ __device__ constexpr int next_pow2(int n) {
  int p = 1;
  while (p < n) p <<= 1;
  return p;
}

}  // namespace sa
