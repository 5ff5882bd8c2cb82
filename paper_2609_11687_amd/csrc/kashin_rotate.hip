// Incoherence pre-rotation of rows (the "+H" preprocessing of Sec. 5): y = R x or y = R^T x,
// R = (H_{2^a} / sqrt(2^a) kron C_b) diag(s) for n = 2^a b, b odd, H the Sylvester Hadamard
// matrix, C_b the orthonormal DCT-II of length b, s_i = -1 when the top bit of the i-th
// splitmix64 output of the seed is set (the generator of the plan's sign mask).
//
// One workgroup per row at a time, the row held in LDS (n <= 16384 floats).  Element n = i b + j; the odd
// factor mixes the b contiguous entries of each segment i, the Hadamard factor mixes entries with
// equal j across segments (kashin_rot_impl.h).  The two factors commute, so R applies signs,
// C_b, H and R^T applies H, C_b^T, signs.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "kashin.h"
#include "kashin_internal.h"
#include "kashin_rot_impl.h"

namespace kashin {
namespace {

constexpr int kRotThreads = 256;
constexpr int kRotMaxN = 16384;
constexpr int kBatch = 16;  // row elements per thread loaded together
constexpr int kPadMaxN = 8192;

// v times the sign of bit k
__device__ __forceinline__ float rot_apply_sign(float v, uint32_t bits, int k) {
  return __uint_as_float(__float_as_uint(v) ^ ((bits << (31 - k)) & 0x80000000u));
}

__device__ __forceinline__ float to_float(float v) { return v; }
__device__ __forceinline__ float to_float(__half v) { return __half2float(v); }
__device__ __forceinline__ float to_float(bf16_t v) { return bf16_to_f32(v); }

// R's factors without signs and scale, or R^T's
template <int B, bool INV, bool PAD>
__device__ __forceinline__ void rot_factors(float* buf, int n, uint32_t huge, int tid) {
  if constexpr (!INV) {
    rot_odd_factor<B, false, kRotThreads>(buf, n, huge, tid);
    rot_hadamard<B, kRotThreads, PAD>(buf, n, tid);
  } else {
    rot_hadamard<B, kRotThreads, PAD>(buf, n, tid);
    rot_odd_factor<B, true, kRotThreads>(buf, n, 0, tid);
  }
}

// Rows of at most 256 K entries (K <= 16; 8 for b = 3): workgroups walk the rows blockIdx.x, blockIdx.x +
// gridDim.x, ..  The row signs, three 64-bit multiplications each, cost as much as the transform, so a
// thread forms those of its elements (tid + 256 k) once, as bits, and keeps them for all its rows;
// and the next row's loads are issued before this row is transformed, so that their latency passes
// under it.  4096 wide, 16384 fp16 rows: 99.7 -> 84.2 us; 256 wide, 65536 rows: 107 -> 50 (a walk
// without the early loads is slower than a workgroup per row: 116 and 167).  Loads past n repeat the
// last entry.
template <int B, bool INV, bool PAD, int K, class IT>
__global__ __launch_bounds__(kRotThreads) void rotate_kernel(int n, uint64_t seed, float scale, const IT* x,
                                                             int64_t ldx, float* y, int64_t ldy, int64_t m) {
  extern __shared__ float buf[];  // n floats, or n + n/16 with PAD (padded slots, rot_slot)
  static_assert(!rot_watch_huge<B, INV>(), "b = 1 and 3 only");
  const int tid = threadIdx.x;
  static_assert(K <= 32, "sign bits per thread");
  IT v[K];
  auto load_row = [&](int64_t row) {
    const IT* xr = x + row * ldx;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = tid + k * kRotThreads;
      v[k] = xr[i < n ? i : n - 1];
    }
  };
  load_row(blockIdx.x);  // gridDim.x <= m
  uint32_t sgn = 0;      // bit k: the sign of element tid + 256 k
  for (int k = 0; k < K; ++k)
    if (rot_sign(seed, tid + k * kRotThreads) < 0.f) sgn |= 1u << k;
  for (int64_t row = blockIdx.x; row < m; row += gridDim.x) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = tid + k * kRotThreads;
      const float f = to_float(v[k]);
      if (i < n) buf[rot_slot<PAD>(i)] = INV ? f : rot_apply_sign(f, sgn, k);
    }
    if (row + gridDim.x < m) load_row(row + gridDim.x);
    lds_barrier();
    rot_factors<B, INV, PAD>(buf, n, 0, tid);
    float* yr = y + row * ldy;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = tid + k * kRotThreads;
      if (i < n) {
        const float f = buf[rot_slot<PAD>(i)] * scale;
        yr[i] = INV ? rot_apply_sign(f, sgn, k) : f;
      }
    }
    lds_barrier();  // the row is read out before the next one is written
  }
}

// Longer rows: a workgroup per row (kept in registers, the next row of a walk would leave too few
// for the transform), loads in batches of kBatch per thread, all issued before the first is used,
// the signs formed while they are in flight.
template <int B, bool INV, bool PAD, class IT>
__global__ __launch_bounds__(kRotThreads) void rotate_long_kernel(int n, uint64_t seed, float scale, const IT* x,
                                                                  int64_t ldx, float* y, int64_t ldy, int64_t row0) {
  extern __shared__ float buf[];
  constexpr bool WATCH = rot_watch_huge<B, INV>() && !std::is_same<IT, __half>::value;  // no fp16 value is huge
  __shared__ uint32_t flags[kRotThreads / 64];
  bool huge = false;
  const int tid = threadIdx.x;
  const int64_t row = row0 + blockIdx.x;
  const IT* xr = x + row * ldx;
  for (int i0 = tid; i0 < n; i0 += kRotThreads * kBatch) {
    float v[kBatch];
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const int i = i0 + k * kRotThreads;
      v[k] = to_float(xr[i < n ? i : n - 1]);
    }
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const int i = i0 + k * kRotThreads;
      if constexpr (WATCH) huge |= fabsf(v[k]) >= kRotHuge;
      if (i < n) buf[rot_slot<PAD>(i)] = INV ? v[k] : v[k] * rot_sign(seed, i);
    }
  }
  if constexpr (WATCH) rot_note_huge(flags, huge, tid);
  lds_barrier();
  uint32_t huge_rows = 0;
  if constexpr (WATCH) huge_rows = rot_huge_rows<kRotThreads / 64>(flags);
  rot_factors<B, INV, PAD>(buf, n, huge_rows, tid);
  float* yr = y + row * ldy;
  for (int i = tid; i < n; i += kRotThreads) {
    const float v = buf[rot_slot<PAD>(i)] * scale;
    yr[i] = INV ? v * rot_sign(seed, i) : v;
  }
}

template <int B, bool INV, bool PAD, class IT>
hipError_t launch_rot_k(int64_t grid, unsigned lds, int n, uint64_t seed, float scale, const IT* x, int64_t ldx, float* y,
                        int64_t ldy, int64_t m, hipStream_t s) {
  const dim3 g(static_cast<unsigned>(grid)), t(kRotThreads);
  const int k = (n + kRotThreads - 1) / kRotThreads;
#define KASHIN_ROT_K(K)                                                                                             \
  if (k <= K) {                                                                                                     \
    hipLaunchKernelGGL((rotate_kernel<B, INV, PAD, K, IT>), g, t, lds, s, n, seed, scale, x, ldx, y, ldy, m);       \
    return hipGetLastError();                                                                                       \
  }
  if constexpr (PAD || B == 3) {  // 43-entry segments leave too few registers for the early loads
    KASHIN_ROT_K(1)
    KASHIN_ROT_K(4)
    KASHIN_ROT_K(8)
    // 16 entries a thread pay for power-of-two rows (4096) only: 3072 = 2^10 3 wide, 10922 fp16 rows, takes
    // 60.7 us walked and 53.6 a row per workgroup
    if constexpr (PAD) {
      KASHIN_ROT_K(16)
    }
  }
#undef KASHIN_ROT_K
  constexpr int64_t kMaxGrid = int64_t(1) << 30;
  for (int64_t r0 = 0; r0 < m; r0 += kMaxGrid) {
    const int64_t r = m - r0 < kMaxGrid ? m - r0 : kMaxGrid;
    hipLaunchKernelGGL((rotate_long_kernel<B, INV, PAD, IT>), dim3(static_cast<unsigned>(r)), t, lds, s, n, seed, scale,
                       x, ldx, y, ldy, r0);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int B, bool INV, class IT>
hipError_t launch_rot(int n, uint64_t seed, const IT* x, int64_t ldx, float* y, int64_t ldy, int64_t m,
                      hipStream_t s) {
  const float scale = static_cast<float>(1.0 / std::sqrt(static_cast<double>(n / B)));  // 1 / sqrt(2^a)
  // power-of-two rows up to kPadMaxN take the padded layout (at most 34 KB of LDS per row)
  const bool pad = B == 1 && n <= kPadMaxN;
  const unsigned lds = static_cast<unsigned>((pad ? n + (n >> 4) : n) * sizeof(float));
  // as many workgroups as are resident at once (160 KB of LDS and 2048 threads on each of 256
  // compute units), so that each keeps its signs over several rows and all walk equally many
  const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(2048 / kRotThreads, 160 * 1024 / std::max(lds, 1u)));
  const int64_t grid = std::min<int64_t>(m, 256 * per_cu);
  if constexpr (B == 1) {
    if (pad) return launch_rot_k<B, INV, true>(grid, lds, n, seed, scale, x, ldx, y, ldy, m, s);
  }
  return launch_rot_k<B, INV, false>(grid, lds, n, seed, scale, x, ldx, y, ldy, m, s);
}

template <int B, class IT>
hipError_t launch_rot_dir(int n, uint64_t seed, bool inverse, const IT* x, int64_t ldx, float* y, int64_t ldy,
                          int64_t m, hipStream_t s) {
  return inverse ? launch_rot<B, true>(n, seed, x, ldx, y, ldy, m, s) : launch_rot<B, false>(n, seed, x, ldx, y, ldy, m, s);
}

template <class IT>
hipError_t launch_rot_odd(int n, uint64_t seed, bool inverse, const IT* x, int64_t ldx, float* y, int64_t ldy,
                          int64_t m, hipStream_t s) {
  const int b = n / (n & -n);
  if (b == 1) return launch_rot_dir<1>(n, seed, inverse, x, ldx, y, ldy, m, s);
  if (b == 3) return launch_rot_dir<3>(n, seed, inverse, x, ldx, y, ldy, m, s);
  return launch_rot_dir<43>(n, seed, inverse, x, ldx, y, ldy, m, s);
}

}  // namespace

bool rotate_supported_n(int n) {
  if (n < 1 || n > kRotMaxN) return false;
  const int b = n / (n & -n);
  return b == 1 || b == 3 || b == 43;
}

hipError_t launch_rotate(int n, uint64_t seed, bool inverse, const void* x, int dtype, int64_t ldx, float* y,
                         int64_t ldy, int64_t m, hipStream_t stream) {
  if (dtype == KASHIN_F16)
    return launch_rot_odd(n, seed, inverse, static_cast<const __half*>(x), ldx, y, ldy, m, stream);
  if (dtype == KASHIN_BF16)
    return launch_rot_odd(n, seed, inverse, static_cast<const bf16_t*>(x), ldx, y, ldy, m, stream);
  return launch_rot_odd(n, seed, inverse, static_cast<const float*>(x), ldx, y, ldy, m, stream);
}

}  // namespace kashin
