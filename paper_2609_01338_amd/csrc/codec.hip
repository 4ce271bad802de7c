// 8-bit group-wise codec of swapped KV chunks (the paper's default codec on
// its in-memory swap path, Sec. 5, after FlexGen's group-wise quantization).
//
// On a run of n halves (n a multiple of 64), groups of 64 consecutive values:
//   mn, mx = min, max (exact in fp32);  d = half(fp32(mx - mn) / 255);  m = mn
//   q_i = d == 0 ? 0 : clamp(rint(fp32(x_i - m) / fp32(d)), 0, 255)
//   x^_i = half(fp32(q_i) * fp32(d) + fp32(m))   (the product is exact)
// with correctly rounded fp32 division and round-half-even, so every code is
// reproducible bit for bit.  Compressed run: n code bytes, then (m, d) as two
// halves per group.
//
// Four lanes take a group, 16 values each (32 bytes in, 16 code bytes out).
// Compression was bound by its vector work, not by memory: with 16 lanes of 4
// values a group's min and max took four exchanges each, and every value a
// correctly rounded division (23.3 us for 22.5 M halves, 14.4 now: 4.8 TB/s;
// decompression 13.5).  Now two exchanges serve 16 values, and
// a value is multiplied by 1 / d; only where that lands within 5e-4 of the
// middle between two codes is it divided (see quantize).
#include "mz_kernels.h"

namespace mzk {
namespace {

// (runs start on 4-byte boundaries only)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));

constexpr int G = 64, PER = 16, LANES = G / PER;   // values per group and per lane

// clamp(rint(RN(a / d)), 0, 255), RN the correctly rounded fp32 quotient.  t =
// a * rd is within 1e-4 of a / d (codes up to 256, rd = 1 / d rounded), so
// rint(t) is the code unless a / d lies that close to the middle between two
// codes; the distance from q d to a, exact to one rounding, tells (by 5e-4: 2 |e|
// within d / 1024 of d), and then the quotient is formed.  (NaN compares false and ends as code 0, as the division's
// does; so do the quotients of an infinite d.)
__device__ __forceinline__ uint32_t quantize(float a, float d, float rd) {
  float q = __builtin_rintf(a * rd);
  const float e = __builtin_fmaf(-q, d, a);
  if (fabsf(fabsf(e + e) - d) <= d * 9.765625e-4f) q = __builtin_rintf(__fdiv_rn(a, d));
  q = fminf(fmaxf(q, 0.0f), 255.0f);
  return (uint32_t)q;
}

// blockIdx.y selects one of n_runs runs: run r reads src + src_off(r) and
// writes dst + r * (n + n/16) (compress) -- see the launchers.
__global__ __launch_bounds__(256) void kv_compress_kernel(const uint8_t* __restrict__ src_base,
                                                          const int32_t* __restrict__ src_slots,
                                                          int64_t src_stride, int64_t n,
                                                          uint8_t* __restrict__ dst) {
  const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * PER;   // first value of the lane
  if (i0 >= n) return;   // whole groups leave together
  const int r = blockIdx.y;
  const _Float16* src = reinterpret_cast<const _Float16*>(
      src_base + (src_slots ? (int64_t)src_slots[r] : (int64_t)r) * src_stride);
  uint8_t* out = dst + (int64_t)r * (n + n / 16);
  uint32_t w[PER / 2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const u32x4 v = reinterpret_cast<const u32x4*>(src + i0)[k];
#pragma unroll
    for (int j = 0; j < 4; ++j) w[4 * k + j] = v[j];
  }
  float x[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) x[i] = (float)__builtin_bit_cast(_Float16, (uint16_t)(w[i / 2] >> (16 * (i & 1))));
  float mn = x[0], mx = x[0];
#pragma unroll
  for (int i = 1; i < PER; ++i) {
    mn = fminf(mn, x[i]);
    mx = fmaxf(mx, x[i]);
  }
#pragma unroll
  for (int o = 1; o < LANES; o <<= 1) {
    mn = fminf(mn, __shfl_xor(mn, o));
    mx = fmaxf(mx, __shfl_xor(mx, o));
  }
  const _Float16 dh = (_Float16)__fdiv_rn(mx - mn, 255.0f);
  const float d = (float)dh;
  u32x4 packed = {};
  if (d != 0.0f) {
    const float rd = __fdiv_rn(1.0f, d);
#pragma unroll
    for (int i = 0; i < PER; ++i) packed[i / 4] |= quantize(x[i] - mn, d, rd) << (8 * (i & 3));
  }
  *reinterpret_cast<u32x4*>(out + i0) = packed;
  if (i0 % G == 0) {
    const _Float16 p[2] = {(_Float16)mn, dh};
    *reinterpret_cast<uint32_t*>(out + n + i0 / G * 4) = __builtin_bit_cast(uint32_t, p);
  }
}

__global__ __launch_bounds__(256) void kv_decompress_kernel(const uint8_t* __restrict__ src, int64_t n,
                                                            uint8_t* __restrict__ dst_base,
                                                            const int32_t* __restrict__ dst_slots,
                                                            int64_t dst_stride) {
  const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * PER;
  if (i0 >= n) return;
  const int r = blockIdx.y;
  const uint8_t* in = src + (int64_t)r * (n + n / 16);
  _Float16* out = reinterpret_cast<_Float16*>(
      dst_base + (dst_slots ? (int64_t)dst_slots[r] : (int64_t)r) * dst_stride);
  const u32x4 codes = *reinterpret_cast<const u32x4*>(in + i0);
  const uint32_t pw = *reinterpret_cast<const uint32_t*>(in + n + i0 / G * 4);
  const float m = (float)__builtin_bit_cast(_Float16, (uint16_t)(pw & 0xFFFFu));
  const float d = (float)__builtin_bit_cast(_Float16, (uint16_t)(pw >> 16));
  uint32_t w[PER / 2];
#pragma unroll
  for (int i = 0; i < PER; i += 2) {
    const uint32_t c = codes[i / 4] >> (8 * (i & 3));
    const _Float16 o[2] = {(_Float16)__builtin_fmaf((float)(c & 0xFFu), d, m),
                           (_Float16)__builtin_fmaf((float)((c >> 8) & 0xFFu), d, m)};
    w[i / 2] = __builtin_bit_cast(uint32_t, o);
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const u32x4 v = {w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]};
    reinterpret_cast<u32x4*>(out + i0)[k] = v;
  }
}

}  // namespace

int64_t kv_compressed_bytes(int64_t n_halves) { return n_halves + n_halves / 16; }

void launch_kv_compress(const void* src_base, const int32_t* src_slots, int64_t src_stride, int64_t n_halves,
                        int n_runs, void* dst, hipStream_t s) {
  if (n_runs < 1 || n_halves < G) return;
  const int64_t threads = n_halves / PER;
  hipLaunchKernelGGL(kv_compress_kernel, dim3((unsigned)((threads + 255) / 256), n_runs), dim3(256), 0, s,
                     reinterpret_cast<const uint8_t*>(src_base), src_slots, src_stride, n_halves,
                     reinterpret_cast<uint8_t*>(dst));
}

void launch_kv_decompress(const void* src, int64_t n_halves, int n_runs, void* dst_base,
                          const int32_t* dst_slots, int64_t dst_stride, hipStream_t s) {
  if (n_runs < 1 || n_halves < G) return;
  const int64_t threads = n_halves / PER;
  hipLaunchKernelGGL(kv_decompress_kernel, dim3((unsigned)((threads + 255) / 256), n_runs), dim3(256), 0, s,
                     reinterpret_cast<const uint8_t*>(src), n_halves, reinterpret_cast<uint8_t*>(dst_base),
                     dst_slots, dst_stride);
}

}  // namespace mzk
