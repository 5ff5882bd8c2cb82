// Device pieces of the incoherence rotation R = (H_{2^a} / sqrt(2^a) kron C_b) diag(s) (Sec. 5's
// "+H" preprocessing), shared by the standalone rotation kernel and the fused loads of the pair
// kernels.  Element index i b + j (segment i, position j); values are float (one row) or float2
// (two rows at once, the rotation acting on each component).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "kashin_tables.h"

namespace kashin {

// Barrier that orders the workgroup's LDS accesses and nothing else.  __syncthreads also waits for
// every global access of the wave, so in a kernel that walks rows it holds each row back until the
// stores of the row before have reached memory.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// s_i: -1 when the top bit of the i-th splitmix64 output of `seed` is set: rot_sign_of(rot_state(seed, i)), and
// rot_state(seed, i + d) = rot_state(seed, i) + d kRotStep (one of three 64-bit products saved)
constexpr uint64_t kRotStep = 0x9E3779B97F4A7C15ull;
__device__ __forceinline__ uint64_t rot_state(uint64_t seed, int i) {
  return seed + static_cast<uint64_t>(i + 1) * kRotStep;
}
__device__ __forceinline__ float rot_sign_of(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  return (z >> 63) ? -1.f : 1.f;
}
__device__ __forceinline__ float rot_sign(uint64_t seed, int i) { return rot_sign_of(rot_state(seed, i)); }

__device__ __forceinline__ float rv_fma(float c, float a, float acc) { return fmaf(c, a, acc); }
__device__ __forceinline__ float2 rv_fma(float c, float2 a, float2 acc) {
  return make_float2(fmaf(c, a.x, acc.x), fmaf(c, a.y, acc.y));
}
__device__ __forceinline__ float rv_zero(float) { return 0.f; }
__device__ __forceinline__ float2 rv_zero(float2) { return make_float2(0.f, 0.f); }
__device__ __forceinline__ float rv_add(float a, float b) { return a + b; }
__device__ __forceinline__ float2 rv_add(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float rv_sub(float a, float b) { return a - b; }
__device__ __forceinline__ float2 rv_sub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float rv_scale(float a, float s) { return a * s; }
__device__ __forceinline__ float2 rv_scale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }

// The odd factor C_B, B > 3, by its symmetry m[k][B-1-j] = (-1)^k m[k][j]: with s_j = x_j + x_{B-1-j} and
// d_j = x_j - x_{B-1-j} (j < H = (B-1)/2), output k of C_B x is sum_j m[k][j] s_j + m[k][H] x_H for even
// k and sum_j m[k][j] d_j for odd k; outputs j and B-1-j of C_B^T x are E_j +- O_j, the sums over even
// and odd k.  Half the products of the plain matrix (925 FMAs for B = 43 against 1849).  C_3 is the
// plain product (its nine FMAs hide behind the LDS accesses).  Every sum runs in ascending order
// from zero, in the whole-segment and the chunked form alike, so the fused and the standalone
// rotation agree bit for bit.
//
// The pair sums of C_B double their entries and could overflow where the plain product is finite, so a
// row with an entry of 2^125 or more in magnitude is a quarter of itself inside C_B (a power of two: the
// same bits otherwise).  Below 2^125 no sum of C_43 can overflow (its rows have l1 norms of at most
// sqrt(43) < 8); nor, in a quarter row, one whose plain partial sums are all finite.  C_B^T's E_j and O_j
// are half the sum and the difference of two plain outputs and need no care.
constexpr float kRotHuge = 0x1p125f;
template <int B, bool TRANS>
constexpr bool rot_watch_huge() {
  return B > 3 && !TRANS;
}

// Which of up to two rows hold such an entry, one bit each: every wave notes in flags[wave], before the
// barrier that ends the load, what its threads saw, and reads all NW notes after it (a uniform value).
__device__ __forceinline__ void rot_note_huge(uint32_t* flags, uint32_t rows, int tid) {
  const uint32_t w = (__ballot(rows & 1u) ? 1u : 0u) | (__ballot(rows & 2u) ? 2u : 0u);
  if ((tid & 63) == 0) flags[tid >> 6] = w;
}
template <int NW>
__device__ __forceinline__ uint32_t rot_huge_rows(const uint32_t* flags) {
  uint32_t w = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) w |= flags[i];
  return __builtin_amdgcn_readfirstlane(w);
}
// the noted rows (bit 0: a float's, or .x; bit 1: .y) of the n entries in buf times f, then a barrier
template <int T, class V>
__device__ __forceinline__ void rot_scale_rows(V* buf, int n, uint32_t rows, float f, int tid) {
  for (int i = tid; i < n; i += T) {
    if constexpr (std::is_same<V, float>::value) buf[i] *= f;
    else buf[i] = make_float2(buf[i].x * (rows & 1u ? f : 1.f), buf[i].y * (rows & 2u ? f : 1.f));
  }
  lds_barrier();
}

// one segment of length B: v <- C_B v (or C_B^T v), in place, constants compile-time
template <int B, bool TRANS, class V>
__device__ __forceinline__ void rot_odd_segment(V* seg) {
  constexpr int H = (B - 1) / 2;
  V in[B];
#pragma unroll
  for (int j = 0; j < B; ++j) in[j] = seg[j];
  if constexpr (B <= 3) {
#pragma unroll
    for (int k = 0; k < B; ++k) {
      V acc = rv_zero(in[0]);
#pragma unroll
      for (int j = 0; j < B; ++j) acc = rv_fma(TRANS ? DctTab<B>::m[j * B + k] : DctTab<B>::m[k * B + j], in[j], acc);
      seg[k] = acc;
    }
  } else if constexpr (!TRANS) {
#pragma unroll
    for (int j = 0; j < H; ++j) {
      const V u = in[j], v = in[B - 1 - j];
      in[j] = rv_add(u, v);
      in[B - 1 - j] = rv_sub(u, v);
    }
#pragma unroll
    for (int k = 0; k < B; ++k) {
      V acc = rv_zero(in[0]);
#pragma unroll
      for (int j = 0; j < H; ++j) acc = rv_fma(DctTab<B>::m[k * B + j], k % 2 ? in[B - 1 - j] : in[j], acc);
      if (k % 2 == 0) acc = rv_fma(DctTab<B>::m[k * B + H], in[H], acc);
      seg[k] = acc;
    }
  } else {
#pragma unroll
    for (int j = 0; j <= H; ++j) {
      V e = rv_zero(in[0]), o = rv_zero(in[0]);
#pragma unroll
      for (int k = 0; k < B; k += 2) e = rv_fma(DctTab<B>::m[k * B + j], in[k], e);
      if (j < H) {
#pragma unroll
        for (int k = 1; k < B; k += 2) o = rv_fma(DctTab<B>::m[k * B + j], in[k], o);
        seg[B - 1 - j] = rv_sub(e, o);
        seg[j] = rv_add(e, o);
      } else {
        seg[j] = e;
      }
    }
  }
}

// the odd factor over all n / B segments (one thread per segment), then a barrier; huge: rot_huge_rows's
// (0 unless rot_watch_huge)
template <int B, bool TRANS, int T, class V>
__device__ __forceinline__ void rot_odd_factor(V* buf, int n, uint32_t huge, int tid) {
  if constexpr (B > 1) {
    if (huge != 0) rot_scale_rows<T>(buf, n, huge, 0.25f, tid);
    for (int i = tid; i < n / B; i += T) rot_odd_segment<B, TRANS>(buf + i * B);
    lds_barrier();
    if (huge != 0) rot_scale_rows<T>(buf, n, huge, 4.f, tid);
  }
}

// chunk c of C_B seg (or C_B^T seg) in acc: outputs c KC .. of C_B; of C_B^T the pairs (j, B-1-j),
// j = c KC / 2 .., as E_j + O_j in acc[0 .. KC/2) and E_j - O_j in acc[KC/2 .. KC), the middle output
// (j = H) being the last chunk's last pair
template <int B, bool TRANS, int CH, int KC, class V>
__device__ __forceinline__ void rot_odd_chunk(const V* seg, V (&acc)[KC]) {
  constexpr int H = (B - 1) / 2;
#pragma unroll
  for (int kk = 0; kk < KC; ++kk) acc[kk] = rv_zero(acc[0]);
  if constexpr (!TRANS) {
#pragma unroll
    for (int j = 0; j <= H; ++j) {
      const V u = seg[j], v = j < H ? seg[B - 1 - j] : u;
      const V sm = j < H ? rv_add(u, v) : u, df = rv_sub(u, v);
#pragma unroll
      for (int kk = 0; kk < KC; ++kk) {
        const int k = CH * KC + kk;
        if (k < B && (j < H || k % 2 == 0)) acc[kk] = rv_fma(DctTab<B>::m[k * B + j], k % 2 ? df : sm, acc[kk]);
      }
    }
  } else {
    constexpr int JC = KC / 2;
#pragma unroll
    for (int k = 0; k < B; ++k) {
      const V x = seg[k];
#pragma unroll
      for (int jj = 0; jj < JC; ++jj) {
        const int j = CH * JC + jj;  // even k into acc[jj] (E_j), odd k into acc[JC + jj] (O_j)
        if (j <= H && !(j == H && k % 2)) acc[(k % 2) * JC + jj] = rv_fma(DctTab<B>::m[k * B + j], x, acc[(k % 2) * JC + jj]);
      }
    }
#pragma unroll
    for (int jj = 0; jj < JC; ++jj) {
      const V e = acc[jj], o = acc[JC + jj];
      if (CH * JC + jj < H) {
        acc[jj] = rv_add(e, o);
        acc[JC + jj] = rv_sub(e, o);
      }
    }
  }
}

// The odd factor for a length N known at compile time.  When the workgroup has at least three
// times as many threads as segments and B is large, each segment's outputs are split into NC chunks
// computed by NC threads (all inputs read before the barrier, outputs written after it), so that
// more waves share the work and each holds fewer values; otherwise one thread per segment.
template <int B, bool TRANS, int T, int N, class V>
__device__ __forceinline__ void rot_odd_factor_fixed(V* buf, uint32_t huge, int tid) {
  constexpr int NSEG = N / B;
  constexpr int NC = (B >= 16 && T >= 3 * NSEG) ? 3 : 1;
  if constexpr (NC == 1) {
    rot_odd_factor<B, TRANS, T>(buf, N, huge, tid);
  } else {
    constexpr int H = (B - 1) / 2;
    constexpr int JC = (H + 1 + NC - 1) / NC;              // output pairs per chunk (TRANS)
    constexpr int KC = TRANS ? 2 * JC : (B + NC - 1) / NC;  // values per chunk
    if (huge != 0) rot_scale_rows<T>(buf, N, huge, 0.25f, tid);
    V acc[KC];
    const int c = tid / NSEG, sg = tid - c * NSEG;  // chunk and segment of this thread
    const V* seg = buf + sg * B;
    if (c == 0) {
      rot_odd_chunk<B, TRANS, 0, KC>(seg, acc);
    } else if (c == 1) {
      rot_odd_chunk<B, TRANS, 1, KC>(seg, acc);
    } else if (c == 2) {
      rot_odd_chunk<B, TRANS, 2, KC>(seg, acc);
    }
    lds_barrier();  // every input read before any output is written
    if (c < NC) {
      if constexpr (TRANS) {
        V* out = buf + sg * B + c * JC;
        V* mir = buf + sg * B + B - 1 - c * JC;
#pragma unroll
        for (int jj = 0; jj < JC; ++jj) {
          if (c * JC + jj <= H) out[jj] = acc[jj];
          if (c * JC + jj < H) mir[-jj] = acc[JC + jj];
        }
      } else {
        V* out = buf + sg * B + c * KC;
#pragma unroll
        for (int kk = 0; kk < KC; ++kk)
          if (c * KC + kk < B) out[kk] = acc[kk];
      }
    }
    lds_barrier();
    if (huge != 0) rot_scale_rows<T>(buf, N, huge, 4.f, tid);
  }
}

// Slot of entry e of a row held in LDS: e, or with PAD (B = 1 only) e + e/16, one spare word per
// 16 entries, so that the 16 consecutive entries a thread of the first Hadamard pass takes, the
// stride-16 groups of the second and the row-order loads and stores all spread over the banks.
template <bool PAD>
__device__ __forceinline__ int rot_slot(int e) {
  return PAD ? e + (e >> 4) : e;
}

// One pass of the unnormalised Walsh-Hadamard transform over the segment-index bits
// [lh, lh + log2 R): each thread takes groups of R entries at stride 2^lh B, transforms them in
// registers with radix-2 stages in ascending bit order, and writes them back; then a barrier.
// Consecutive threads take consecutive offsets within a stride, so each access is contiguous.
// With PAD the entries sit at rot_slot<true> (the stride 2^lh is then 1 or a multiple of 16, so
// entries hb apart are hb + hb/16 slots apart).
template <int B, int R, int T, bool PAD = false, class V>
__device__ __forceinline__ void rot_hadamard_pass(V* buf, int n, int lh, int tid) {
  static_assert(!PAD || B == 1, "padded rows are power-of-two rows");
  const int hb = (1 << lh) * B;
  const int st = PAD ? hb + (hb >> 4) : hb;
  for (int q = tid; q < n / R; q += T) {
    const int hi = (q >> lh) / B;  // = q / hb
    V* p = buf + rot_slot<PAD>(hi * (R * hb) + (q - hi * hb));
    V x[R];
#pragma unroll
    for (int m = 0; m < R; ++m) x[m] = p[m * st];
#pragma unroll
    for (int st = 1; st < R; st <<= 1) {
#pragma unroll
      for (int m = 0; m < R; ++m) {
        if (!(m & st)) {
          const V u = x[m], v = x[m + st];
          x[m] = rv_add(u, v);
          x[m + st] = rv_sub(u, v);
        }
      }
    }
#pragma unroll
    for (int m = 0; m < R; ++m) p[m * st] = x[m];
  }
  lds_barrier();
}

// unnormalised Walsh-Hadamard transform over the 2^a segments (stride B), in place: passes of
// radix 16 (a last one of radix 2, 4 or 8), the radix-2 stages in ascending bit order overall
template <int B, int T, bool PAD = false, class V>
__device__ __forceinline__ void rot_hadamard(V* buf, int n, int tid) {
  const int a = __builtin_ctz(static_cast<unsigned>(n));  // n = 2^a B, B odd
  int lh = 0;
  for (; lh + 4 <= a; lh += 4) rot_hadamard_pass<B, 16, T, PAD>(buf, n, lh, tid);
  const int r = a - lh;
  if (r == 3) rot_hadamard_pass<B, 8, T, PAD>(buf, n, lh, tid);
  else if (r == 2) rot_hadamard_pass<B, 4, T, PAD>(buf, n, lh, tid);
  else if (r == 1) rot_hadamard_pass<B, 2, T, PAD>(buf, n, lh, tid);
}

// b, the odd part of n = 2^a b
__host__ __device__ constexpr int rot_odd_part(int n) { return n / (n & -n); }

}  // namespace kashin
