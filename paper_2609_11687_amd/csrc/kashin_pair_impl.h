// Kernel templates (included by the per-size translation units kashin_n*.hip).
// HIP kernels for gfx950: Kashin-DCT decomposition (Alg. 2), the operator
// P = IDCT o diag(eps) o DCT (Sec. 4.1), four-peak 2-bit clustering (Sec. 3.1)
// and reconstitution (App. C).
//
// Data flow of one workgroup ("pair kernel"): two rows a, b of the weight matrix
// are held as one complex vector y = v_a + i v_b, where v is the row in the
// even/odd ("Makhoul") order v_m = x_{2m}, v_{N-1-m} = x_{2m+1}.  Then
//   DCT-II / DCT-III of both rows = one length-N complex FFT / inverse FFT of y,
// and the sign flips between them reduce to a per-frequency gather and scale:
//   Y'_k = f_k * Y_{s(k)},  s(k) = k if eps_k == eps_{N-k} else N - k,
//   f_k = eps_k / N  or  eps_k * exp(i pi k / N) / N.
// Because every greedy step is elementwise or a permutation-invariant l1 sum,
// the factors stay in the permuted order for the whole run; only loads and
// stores translate indices.  P never forms a matrix: each application is a
// forward FFT, the gather above fused into the first inverse pass, and an
// inverse FFT (Stockham, mixed radix, LDS-resident between passes).  Between two
// applications of P the residual sits in registers, where the greedy steps run.
// Rows are pre-scaled by a power of two (exact) so both halves of a pair have
// comparable magnitude; a row with NaN/Inf is zeroed inside the pair and
// reported as NaN, so it cannot contaminate its partner.

#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <cfloat>
#include <cstdint>
#include <type_traits>

#include "kashin.h"
#include "kashin_internal.h"
#include "kashin_rot_impl.h"
#include "kashin_tables.h"

namespace kashin {
namespace {

// ------------------------------------------------------------------ compile-time helpers
template <int B, int E, class F>
__device__ __forceinline__ void sfor(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    sfor<B + 1, E>(f);
  }
}

constexpr int ilog2(int x) {
  int l = 0;
  while ((1 << l) < x) ++l;
  return l;
}
constexpr int bitrev(int x, int bits) {
  int r = 0;
  for (int i = 0; i < bits; ++i) r = (r << 1) | ((x >> i) & 1);
  return r;
}

__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }

// cos / sin (2 pi m / 32) in double, for compile-time constants
struct W32 {
  static constexpr double c[32] = {
      1.0, 0.9807852804032304, 0.9238795325112867, 0.8314696123025452,
      0.7071067811865476, 0.5555702330196023, 0.38268343236508984, 0.19509032201612833,
      0, -0.1950903220161282, -0.3826834323650897, -0.555570233019602,
      -0.7071067811865475, -0.8314696123025453, -0.9238795325112867, -0.9807852804032304,
      -1.0, -0.9807852804032304, -0.9238795325112868, -0.8314696123025455,
      -0.7071067811865477, -0.5555702330196022, -0.38268343236509034, -0.19509032201612866,
      0, 0.1950903220161283, 0.38268343236509, 0.5555702330196018,
      0.7071067811865474, 0.8314696123025452, 0.9238795325112865, 0.9807852804032303};
  static constexpr double s[32] = {
      0, 0.19509032201612825, 0.3826834323650898, 0.5555702330196022,
      0.7071067811865475, 0.8314696123025452, 0.9238795325112867, 0.9807852804032304,
      1.0, 0.9807852804032304, 0.9238795325112867, 0.8314696123025455,
      0.7071067811865476, 0.5555702330196022, 0.3826834323650899, 0.1950903220161286,
      0, -0.19509032201612836, -0.38268343236508967, -0.555570233019602,
      -0.7071067811865475, -0.8314696123025452, -0.9238795325112865, -0.9807852804032303,
      -1.0, -0.9807852804032304, -0.9238795325112866, -0.8314696123025455,
      -0.7071067811865477, -0.5555702330196022, -0.3826834323650904, -0.19509032201612872};
};
constexpr double cabs_d(double v) { return v < 0 ? -v : v; }

// Radix-2 butterfly with a compile-time twiddle w = w32^K (forward, w32 = exp(-2 pi i / 32);
// the inverse uses w32^-K): (x, y) <- (x + w y, x - w y).  A general twiddle is applied as
// w y = m p with p = (w / m) y, m whichever of Re w, Im w is larger in magnitude: p takes
// two FMAs with the ratio t = Im w / Re w or Re w / Im w (|t| <= 1), and x +- m p four more,
// six instructions instead of a complex product followed by four additions.
template <int K, bool INV>
__device__ __forceinline__ void bfly(float2& x, float2& y) {
  constexpr int k = K & 31;
  const float2 a = x;
  if constexpr (k == 0) {
    x = cadd(a, y);
    y = csub(a, y);
  } else if constexpr (k == 16) {
    x = csub(a, y);
    y = cadd(a, y);
  } else if constexpr (k == 8 || k == 24) {
    // w = (0, wi), wi = +-1: w y = (-wi y.y, wi y.x)
    constexpr float wi = static_cast<float>(INV ? W32::s[k] : -W32::s[k]);
    const float2 wy = make_float2(-wi * y.y, wi * y.x);
    x = cadd(a, wy);
    y = csub(a, wy);
  } else {
    constexpr double wr = W32::c[k];
    constexpr double wi = INV ? W32::s[k] : -W32::s[k];
    float2 p;
    float m;
    if constexpr (cabs_d(wr) >= cabs_d(wi)) {
      constexpr float t = static_cast<float>(wi / wr);
      m = static_cast<float>(wr);
      p = make_float2(fmaf(-t, y.y, y.x), fmaf(t, y.x, y.y));  // (w / wr) y
    } else {
      constexpr float t = static_cast<float>(wr / wi);
      m = static_cast<float>(wi);
      p = make_float2(fmaf(t, y.x, -y.y), fmaf(t, y.y, y.x));  // (w / wi) y
    }
    x = make_float2(fmaf(m, p.x, a.x), fmaf(m, p.y, a.y));
    y = make_float2(fmaf(-m, p.x, a.x), fmaf(-m, p.y, a.y));
  }
}

// In-register DFT of a power-of-two length R <= 32: radix-2 decimation in time on the
// bit-reversed input (a compile-time renaming), so every twiddle multiplies the second
// operand of a butterfly and fuses with it; output in natural order.
template <int R, bool INV>
__device__ __forceinline__ void dft_pow2(float2 (&a)[R]) {
  constexpr int L = ilog2(R);
  float2 b[R];
  sfor<0, R>([&](auto iv) { b[decltype(iv)::value] = a[bitrev(decltype(iv)::value, L)]; });
  sfor<1, L + 1>([&](auto sv) {
    constexpr int len = 1 << decltype(sv)::value;
    constexpr int half = len >> 1;
    sfor<0, R / len>([&](auto bv) {
      sfor<0, half>([&](auto jv) {
        constexpr int i0 = decltype(bv)::value * len + decltype(jv)::value;
        bfly<decltype(jv)::value * (32 / len), INV>(b[i0], b[i0 + half]);
      });
    });
  });
  sfor<0, R>([&](auto iv) { a[decltype(iv)::value] = b[decltype(iv)::value]; });
}

// DFT of the twiddled inputs a_r tw(r) (tw(0) = 1; conjugated twiddles on the inverse).
// The first DIT stage pairs a_r with a_{r+R/2} (r = bitrev of the pair index): with
// x = a_r tw(r) and w = tw(r + R/2) it forms X = x + w a_{r+R/2} in four FMAs and the other
// output as 2x - X, so the second twiddle costs no separate complex product.
template <int R, bool INV, class TW>
__device__ __forceinline__ void dft_pow2_tw(float2 (&a)[R], TW&& tw) {
  constexpr int L = ilog2(R);
  constexpr int H = R / 2;
  float2 b[R];
  sfor<0, H>([&](auto mv) {
    constexpr int m = decltype(mv)::value;
    constexpr int r = bitrev(m, L - 1);
    float2 x = a[r];
    if constexpr (r > 0) {
      const float2 t = tw(std::integral_constant<int, r>{});
      x = INV ? make_float2(x.x * t.x + x.y * t.y, x.y * t.x - x.x * t.y)
              : make_float2(x.x * t.x - x.y * t.y, x.x * t.y + x.y * t.x);
    }
    const float2 w = tw(std::integral_constant<int, r + H>{});
    const float2 y = a[r + H];
    const float wy = INV ? -w.y : w.y;
    const float2 X = make_float2(fmaf(w.x, y.x, fmaf(-wy, y.y, x.x)), fmaf(w.x, y.y, fmaf(wy, y.x, x.y)));
    b[2 * m] = X;
    b[2 * m + 1] = make_float2(fmaf(2.f, x.x, -X.x), fmaf(2.f, x.y, -X.y));
  });
  sfor<2, L + 1>([&](auto sv) {
    constexpr int len = 1 << decltype(sv)::value;
    constexpr int half = len >> 1;
    sfor<0, R / len>([&](auto bv) {
      sfor<0, half>([&](auto jv) {
        constexpr int i0 = decltype(bv)::value * len + decltype(jv)::value;
        bfly<decltype(jv)::value * (32 / len), INV>(b[i0], b[i0 + half]);
      });
    });
  });
  sfor<0, R>([&](auto iv) { a[decltype(iv)::value] = b[decltype(iv)::value]; });
}

// In-register DFT of an odd length R, directly from its definition, pairing j with R-j
// so each constant multiplies a sum or a difference.  The sums and differences overwrite
// the inputs in place (a[j] <- a[j] + a[R-j], a[R-j] <- a[j] - a[R-j]) and outputs are
// handed to sink(q, A_q) as soon as they are formed, so no second array is live.
// `pre(r, v)` is applied to input r just before it is paired (the pass twiddles), so a
// twiddled input never waits in a register of its own.
template <int R, bool INV, class Pre, class Sink>
__device__ __forceinline__ void dft_odd(float2 (&a)[R], Pre&& pre, Sink&& sink) {
  constexpr int H = (R - 1) / 2;
  sfor<1, H + 1>([&](auto jv) {
    constexpr int j = decltype(jv)::value;
    const float2 p = pre(j, a[j]), m = pre(R - j, a[R - j]);
    a[j] = cadd(p, m);
    a[R - j] = csub(p, m);
    if constexpr (R > 16 && j % 4 == 0) __builtin_amdgcn_sched_barrier(0);
  });
  const float2 x0 = a[0];
  float2 sum = x0;
  sfor<1, H + 1>([&](auto jv) { sum = cadd(sum, a[decltype(jv)::value]); });
  sfor<1, H + 1>([&](auto qv) {
    constexpr int q = decltype(qv)::value;
    float2 re = x0;
    float2 im = make_float2(0.f, 0.f);
    sfor<1, H + 1>([&](auto jv) {
      constexpr int j = decltype(jv)::value;
      constexpr int m = (j * q) % R;
      constexpr float c = CisTab<R>::c[m];
      constexpr float sn = CisTab<R>::s[m];
      re.x = fmaf(a[j].x, c, re.x);
      re.y = fmaf(a[j].y, c, re.y);
      im.x = fmaf(a[R - j].x, sn, im.x);
      im.y = fmaf(a[R - j].y, sn, im.y);
    });
    // forward: A_q = re - i im, A_{R-q} = re + i im; inverse swaps them
    const float2 minus = make_float2(re.x + im.y, re.y - im.x);
    const float2 plus = make_float2(re.x - im.y, re.y + im.x);
    sink(q, INV ? plus : minus);
    sink(R - q, INV ? minus : plus);
    // keep the scheduler from interleaving all output pairs (each pair needs its own
    // accumulators next to the R inputs)
    if constexpr (R > 16) __builtin_amdgcn_sched_barrier(0);
  });
  sink(0, sum);
}

// The largest power of two that divides R.
constexpr int pow2_part(int r) { return r & -r; }
// k in [0, a b) with k mod a = ka and k mod b = kb (a, b coprime)
constexpr int crt(int a, int b, int ka, int kb) {
  int k = ka;
  while (k % b != kb) k += a;
  return k;
}

// In-register DFT of length R = 2^a b, b odd: the prime-factor (Good-Thomas) split into b DFTs of
// length 2^a and 2^a of length b, whose index maps are compile-time renamings and which needs no
// twiddles between its two halves; R = 25 as 5 x 5 with them.
template <int R, bool INV>
__device__ __forceinline__ void dft_inplace(float2 (&a)[R]) {
  constexpr int N1 = pow2_part(R), N2 = R / N1;
  if constexpr (R == 25) {
    float2 c[25];
    sfor<0, 5>([&](auto nv) {
      constexpr int n2 = decltype(nv)::value;
      float2 b[5];
      sfor<0, 5>([&](auto iv) { b[decltype(iv)::value] = a[5 * decltype(iv)::value + n2]; });
      float2 o[5];
      dft_odd<5, INV>(b, [](int, float2 v) { return v; }, [&](int q, float2 v) { o[q] = v; });
      sfor<0, 5>([&](auto kv) {
        constexpr int k1 = decltype(kv)::value;
        constexpr float wr = CisTab<25>::c[n2 * k1], wi = INV ? CisTab<25>::s[n2 * k1] : -CisTab<25>::s[n2 * k1];
        const float2 v = o[k1];
        c[k1 * 5 + n2] = (n2 == 0 || k1 == 0) ? v : make_float2(v.x * wr - v.y * wi, v.x * wi + v.y * wr);
      });
    });
    sfor<0, 5>([&](auto kv) {
      constexpr int k1 = decltype(kv)::value;
      float2 b[5];
      sfor<0, 5>([&](auto iv) { b[decltype(iv)::value] = c[k1 * 5 + decltype(iv)::value]; });
      dft_odd<5, INV>(b, [](int, float2 v) { return v; }, [&](int q, float2 v) { a[k1 + 5 * q] = v; });
    });
  } else if constexpr (N2 == 1) {
    dft_pow2<R, INV>(a);
  } else {
    float2 c[R];
    sfor<0, N2>([&](auto nv) {
      constexpr int n2 = decltype(nv)::value;
      float2 b[N1];
      sfor<0, N1>([&](auto iv) { b[decltype(iv)::value] = a[(N2 * decltype(iv)::value + N1 * n2) % R]; });
      if constexpr (N1 > 1) dft_pow2<N1, INV>(b);
      sfor<0, N1>([&](auto kv) { c[decltype(kv)::value * N2 + n2] = b[decltype(kv)::value]; });
    });
    sfor<0, N1>([&](auto kv) {
      constexpr int k1 = decltype(kv)::value;
      float2 b[N2];
      sfor<0, N2>([&](auto iv) { b[decltype(iv)::value] = c[k1 * N2 + decltype(iv)::value]; });
      dft_odd<N2, INV>(b, [](int, float2 v) { return v; }, [&](int q, float2 v) { a[crt(N1, N2, k1, q)] = v; });
    });
  }
}

template <bool INV>
__device__ __forceinline__ float2 twmul(float2 v, float2 t) {
  if constexpr (!INV) return make_float2(v.x * t.x - v.y * t.y, v.x * t.y + v.y * t.x);
  else return make_float2(v.x * t.x + v.y * t.y, v.y * t.x - v.x * t.y);
}

// In-register DFT of the twiddled inputs a_r tw(r) (tw(0) = 1; conjugated twiddles on the inverse)
template <int R, bool INV, class TW>
__device__ __forceinline__ void dft_tw(float2 (&a)[R], TW&& tw) {
  if constexpr ((R & (R - 1)) == 0) {
    dft_pow2_tw<R, INV>(a, tw);
  } else {
    sfor<1, R>([&](auto rv) {
      constexpr int r = decltype(rv)::value;
      a[r] = twmul<INV>(a[r], tw(rv));
    });
    dft_inplace<R, INV>(a);
  }
}

// DFT of a[] handed to sink(q, A_q) for every q (power-of-two R: computed in place first).
template <int R, bool INV, class Sink>
__device__ __forceinline__ void dft(float2 (&a)[R], Sink&& sink) {
  if constexpr ((R & (R - 1)) == 0) {
    if constexpr (R > 1) dft_pow2<R, INV>(a);
    sfor<0, R>([&](auto qv) { sink(decltype(qv)::value, a[decltype(qv)::value]); });
  } else {
    static_assert(R % 2 == 1, "composite non-power-of-two radices are not implemented");
    dft_odd<R, INV>(a, [](int, float2 v) { return v; }, sink);
  }
}

// ------------------------------------------------------------------ launch configuration
// N: vector length = complex FFT length of a packed pair.  T: threads per workgroup.
// W: occupancy target (waves per SIMD) given to the register allocator.
// Rs: radices of the forward FFT passes; the first radix also fixes the register layout
// in which the greedy steps run: thread t holds elements j + r * (N / R0) for its
// butterflies j = t + T * i, r < R0.
template <int N_, int T_, int W_, int... Rs>
struct Cfg {
  static constexpr int N = N_;
  static constexpr int T = T_;
  static constexpr int W = W_;  // waves per SIMD the register allocation must allow
  static constexpr int NP = sizeof...(Rs);
  static constexpr int rad[NP] = {Rs...};
  static constexpr int R0 = rad[0];
  static constexpr int NB0 = N / R0;
  static constexpr int B0 = (NB0 + T - 1) / T;
  static constexpr int E = B0 * R0;
  static constexpr int NW = (T + 63) / 64;
  static constexpr int PG = 1 << kPadShift;  // generic path: a spare LDS slot per PG elements
  // three-pass path (N = R0 M R0, one butterfly of the outer passes per thread)
  static constexpr bool RES = three_pass(N_, T_, NP, rad);
  static constexpr int M = RES ? rad[1] : 1;
  static constexpr bool UNI = RES && M == R0 && (R0 & (R0 - 1)) == 0;  // one power-of-two radix throughout
  static constexpr int S1 = NB0 + (R0 == 8 ? 4 : 2);   // row strides of the two exchange layouts (below)
  static constexpr int S2 = NB0 + (R0 == 20 ? 8 : 1);
  static constexpr int LDS = RES ? R0 * (S1 > S2 ? S1 : S2) + 2 : pad_slot(N) + 4;
};

template <class C>
constexpr int ns_fwd(int p) {
  int s = 1;
  for (int i = 0; i < p; ++i) s *= C::rad[i];
  return s;
}
template <class C>
constexpr int ns_inv(int p) {
  int s = 1;
  for (int i = 0; i < p; ++i) s *= C::rad[C::NP - 1 - i];
  return s;
}

// Generic path's LDS layout: element k of the length-N complex vector lives at float2 slot pad<C>(k)
// (a spare slot per C::PG elements, so that both contiguous and stride-16 accesses of a Stockham
// pass spread over the banks).  pad<C>(x + y) = pad<C>(x) + pad<C>(y) whenever x mod PG +
// y mod PG < PG: a base slot plus compile-time offsets addresses a butterfly's elements.
template <class C>
constexpr int pad(int i) { return pad_slot(i); }
// Whether a Stockham write (element q of butterfly j to b + q S, b = (j / S) S R + j mod S,
// q < R) can address slots as pad(b) + pad(q S): S a multiple of PG, or S dividing PG with
// S R a multiple or a divisor of PG (then b mod PG + q S mod PG < PG for every q).
template <class C>
constexpr bool pad_offsets_ok(int S, int R) {
  return S % C::PG == 0 || (C::PG % S == 0 && ((S * R) % C::PG == 0 || C::PG % (S * R) == 0));
}

// Opaque copy of the thread index: without it every twiddle load and LDS address of every
// pass is proven invariant across the block loop, hoisted out of it, and kept live in
// registers at once.
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Position m of the even/odd order -> index in the row.
template <int N>
__device__ __forceinline__ int orig_index(int m) {
  return m < N / 2 ? 2 * m : 2 * (N - 1 - m) + 1;
}

// ------------------------------------------------------------------ reductions
// Cross-lane moves with DPP (no LDS round trip).  update_dpp(old = 0, ...): lanes of rows
// outside ROW_MASK keep 0.
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xf, false));
}
__device__ __forceinline__ float lane63(float v) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Sum over the wave in a fixed order: quad xor 1, 2, half-row mirror, row mirror, then the
// row sums folded into lane 63 by row broadcasts; returned as a wave-uniform value.  With ALT the
// lanes of a row fold in the order xor 2, 4, 8, 1 (lane 15 of a row rotated by 4 and 8 adds exactly
// those pairs): the order of the uniform shapes (N = 512 and 4096), whose step sizes, and so whose
// codes, stay those of earlier builds bit for bit.
template <bool ALT = false>
__device__ __forceinline__ float wave_sum(float v) {
  if constexpr (ALT) {
    v += dpp<0x4e>(v);   // quad_perm [2,3,0,1]
    v += dpp<0x124>(v);  // row_ror:4
    v += dpp<0x128>(v);  // row_ror:8
    v += dpp<0xb1>(v);   // quad_perm [1,0,3,2]
  } else {
    v += dpp<0xb1>(v);   // quad_perm [1,0,3,2]
    v += dpp<0x4e>(v);   // quad_perm [2,3,0,1]
    v += dpp<0x141>(v);  // row_half_mirror
    v += dpp<0x140>(v);  // row_mirror
  }
  v += dpp<0x142, 0xa>(v); // row_bcast:15 into rows 1 and 3
  v += dpp<0x143, 0xc>(v); // row_bcast:31 into rows 2 and 3
  return lane63(v);
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp<0xb1>(v));
  v = fmaxf(v, dpp<0x4e>(v));
  v = fmaxf(v, dpp<0x141>(v));
  v = fmaxf(v, dpp<0x140>(v));
  v = fmaxf(v, dpp<0x142, 0xa>(v));
  v = fmaxf(v, dpp<0x143, 0xc>(v));
  return lane63(v);
}

// Sum of K values over the workgroup in a fixed order (every thread gets the same bits).
// `red` holds 2 * NW * 32 floats; consecutive calls alternate halves, so one barrier per
// call suffices.
template <int T, int K, bool ALT = false>
__device__ __forceinline__ void block_sum(float (&v)[K], float* red, int& slot) {
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = wave_sum<ALT>(v[k]);
  if constexpr (T > 64) {
    constexpr int NW = (T + 63) / 64;
    float* r = red + (slot & 1) * (NW * 32);
    ++slot;
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
      for (int k = 0; k < K; ++k) r[(threadIdx.x >> 6) * K + k] = v[k];
    }
    lds_barrier();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      float s = r[k];
#pragma unroll
      for (int w = 1; w < NW; ++w) s += r[w * K + k];
      v[k] = s;
    }
  }
}

// block_sum for many values over many waves: the workgroup's per-wave partials are summed by the
// lanes of one DPP row (lane w holds wave w's partial; a quad, half-row and row fold, the same in
// every wave), so K values cost K registers after the barrier rather than K x (waves), which
// block_sum's unrolled reads need all at once.  A fixed order again, but another one.
template <int T, int K>
__device__ __forceinline__ void block_sum_lanes(float (&v)[K], float* red, int& slot) {
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = wave_sum(v[k]);
  if constexpr (T > 64) {
    constexpr int NW = (T + 63) / 64;
    static_assert(NW <= 16 && K <= 32, "one DPP row of partials, K values per wave in red");
    float* r = red + (slot & 1) * (NW * 32);
    ++slot;
    const int lane = threadIdx.x & 63;
    if (lane == 0) {
#pragma unroll
      for (int k = 0; k < K; ++k) r[(threadIdx.x >> 6) * K + k] = v[k];
    }
    lds_barrier();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      float t = lane < NW ? r[lane * K + k] : 0.f;
      t += dpp<0xb1>(t);   // quad_perm [1,0,3,2]
      t += dpp<0x4e>(t);   // quad_perm [2,3,0,1]
      t += dpp<0x141>(t);  // row_half_mirror
      t += dpp<0x140>(t);  // row_mirror: every lane of row 0 holds the sum of lanes 0..15
      v[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t), 0));
    }
  }
}

template <int T, int K>
__device__ __forceinline__ void block_max(float (&v)[K], float* red, int& slot) {
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = wave_max(v[k]);
  if constexpr (T > 64) {
    constexpr int NW = (T + 63) / 64;
    float* r = red + (slot & 1) * (NW * 32);
    ++slot;
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
      for (int k = 0; k < K; ++k) r[(threadIdx.x >> 6) * K + k] = v[k];
    }
    lds_barrier();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      float s = r[k];
#pragma unroll
      for (int w = 1; w < NW; ++w) s = fmaxf(s, r[w * K + k]);
      v[k] = s;
    }
  }
}

// ------------------------------------------------------------------ plan tables
// Twiddle tables, one per pass with stride NS > 1, forward passes first then (generic path) inverse
// passes: entry [jm][r] = w_N^(r * jm * N / (NS R)), jm < NS, r < R (each table padded to
// an even length so every table starts 16-byte aligned).  Every thread reads its R
// twiddles contiguously.
template <class C, bool INV>
constexpr int pass_radix(int p) {
  return INV ? C::rad[C::NP - 1 - p] : C::rad[p];
}
template <class C, bool INV>
constexpr int pass_ns(int p) {
  return INV ? ns_inv<C>(p) : ns_fwd<C>(p);
}
template <class C, bool INV>
constexpr int tw_offset(int p) {
  int off = 0;
  for (int q = 1; q < C::NP; ++q) {
    if (!INV && q == p) return off;
    off += (ns_fwd<C>(q) * C::rad[q] + 1) & ~1;
  }
  for (int q = 1; q < C::NP; ++q) {
    if (INV && q == p) return off;
    off += (ns_inv<C>(q) * C::rad[C::NP - 1 - q] + 1) & ~1;
  }
  return off;
}

// ------------------------------------------------------------------ FFT passes
enum { SRC_REGS = 0, SRC_LDS = 1, SRC_MID = 2 };
enum { DST_LDS = 0, DST_REGS = 1 };

// One Stockham pass of radix R with stride NS: butterfly j reads elements j + r * N/R,
// multiplies by the twiddles w_N^(r * (j mod NS) * N/(NS R)), takes a length-R DFT, and
// writes element q to (j / NS) * NS * R + (j mod NS) + q * NS.  In place in LDS: every
// read completes (barrier) before any write.  SRC_MID (first inverse pass) reads through
// the eps table: element k = j + r N/R comes from LDS byte address mid[j R + r].z, scaled by
// the complex factor mid[j R + r].xy.
template <class C, int P, bool INV, int SRC, int DST>
__device__ __forceinline__ void fft_pass(float2 (&z)[C::E], float2* __restrict__ lds,
                                         const float2* __restrict__ tw, const float4* __restrict__ mid) {
  constexpr int N = C::N;
  constexpr int T = C::T;
  constexpr int R = pass_radix<C, INV>(P);
  constexpr int NS = pass_ns<C, INV>(P);
  constexpr int NB = N / R;
  constexpr int BP = (NB + T - 1) / T;
  constexpr bool FULL = (NB % T) == 0;
  static_assert(SRC != SRC_REGS || (R == C::R0 && NS == 1), "register source must be the first pass");
  static_assert(DST != DST_REGS || (R == C::R0 && NS == N / C::R0), "register target must be the last pass");
  const int tid = opaque(threadIdx.x);
  float2 a[BP][R];
  sfor<0, BP>([&](auto iv) {
    constexpr int i = decltype(iv)::value;
    const int j = tid + T * i;
    if constexpr (SRC == SRC_REGS) {
      sfor<0, R>([&](auto rv) { a[i][decltype(rv)::value] = z[i * R + decltype(rv)::value]; });
    } else if (FULL || j < NB) {
      if constexpr (SRC == SRC_MID) {
        const float4* m = mid + j * R;
        const char* lb = reinterpret_cast<const char*>(lds);
        sfor<0, R>([&](auto rv) {
          constexpr int r = decltype(rv)::value;
          const float4 f = m[r];
          const float2 v = *reinterpret_cast<const float2*>(lb + __float_as_int(f.z));
          a[i][r] = make_float2(f.x * v.x - f.y * v.y, f.x * v.y + f.y * v.x);
          if constexpr (R > 16 && r % 8 == 7) __builtin_amdgcn_sched_barrier(0);
        });
      } else if constexpr (NB % C::PG == 0) {
        const float2* base = lds + pad<C>(j);
        sfor<0, R>([&](auto rv) { a[i][decltype(rv)::value] = base[decltype(rv)::value * pad<C>(NB)]; });
      } else {
        sfor<0, R>([&](auto rv) { a[i][decltype(rv)::value] = lds[pad<C>(j + decltype(rv)::value * NB)]; });
      }
    }
  });
  if constexpr (SRC != SRC_REGS) lds_barrier();
  sfor<0, BP>([&](auto iv) {
    constexpr int i = decltype(iv)::value;
    const int j = tid + T * i;
    if (FULL || j < NB) {
      const int jm = (NS > 1) ? (j % NS) : 0;
      if constexpr (NS > 1 && R % 2 == 0) {
        // a_r *= w_N^(r jm N/(NS R)) (conjugate on the inverse), read pairwise from the
        // thread's contiguous table row and applied as soon as it arrives
        const float2* tp = tw + tw_offset<C, INV>(P) + jm * R;
        auto twmul = [&](float2& v, float2 t) {
          if constexpr (!INV) v = make_float2(v.x * t.x - v.y * t.y, v.x * t.y + v.y * t.x);
          else v = make_float2(v.x * t.x + v.y * t.y, v.y * t.x - v.x * t.y);
        };
        if constexpr (R % 2 == 0) {
          const float4* t4 = reinterpret_cast<const float4*>(tp);
          sfor<0, R / 2>([&](auto hv) {
            constexpr int h = decltype(hv)::value;
            const float4 q = t4[h];
            if constexpr (h > 0) twmul(a[i][2 * h], make_float2(q.x, q.y));
            twmul(a[i][2 * h + 1], make_float2(q.z, q.w));
          });
        }
      }
      if constexpr (DST == DST_LDS) {
        const int idx0 = (j / NS) * NS * R + jm;
        if constexpr (R % 2 == 1 && NS > 1) {
          // odd radix: the twiddle of each input is applied inside the DFT's pairing step
          const float2* tp = tw + tw_offset<C, INV>(P) + jm * R;
          auto pre = [&](int r, float2 v) {
            if (r == 0) return v;
            const float2 t = tp[r];
            if constexpr (!INV) return make_float2(v.x * t.x - v.y * t.y, v.x * t.y + v.y * t.x);
            else return make_float2(v.x * t.x + v.y * t.y, v.y * t.x - v.x * t.y);
          };
          if constexpr (pad_offsets_ok<C>(NS, R)) {
            float2* base = lds + pad<C>(idx0);
            dft_odd<R, INV>(a[i], pre, [&](int q, float2 v) { base[pad<C>(q * NS)] = v; });
          } else {
            dft_odd<R, INV>(a[i], pre, [&](int q, float2 v) { lds[pad<C>(idx0 + q * NS)] = v; });
          }
        } else if constexpr (pad_offsets_ok<C>(NS, R)) {
          float2* base = lds + pad<C>(idx0);
          dft<R, INV>(a[i], [&](int q, float2 v) { base[pad<C>(q * NS)] = v; });
        } else {
          dft<R, INV>(a[i], [&](int q, float2 v) { lds[pad<C>(idx0 + q * NS)] = v; });
        }
      } else {
        dft<R, INV>(a[i], [&](int q, float2 v) { z[i * R + q] = v; });
      }
    }
  });
  if constexpr (DST == DST_LDS) lds_barrier();
}

template <class C, int P>
__device__ __forceinline__ void fwd_passes(float2 (&z)[C::E], float2* lds, const float2* tw, const float4* mid) {
  if constexpr (P < C::NP) {
    fft_pass<C, P, false, (P == 0 ? SRC_REGS : SRC_LDS), DST_LDS>(z, lds, tw, mid);
    fwd_passes<C, P + 1>(z, lds, tw, mid);
  }
}
template <class C, int P>
__device__ __forceinline__ void inv_passes(float2 (&z)[C::E], float2* lds, const float2* tw, const float4* mid) {
  if constexpr (P < C::NP) {
    fft_pass<C, P, true, (P == 0 ? SRC_MID : SRC_LDS), (P == C::NP - 1 ? DST_REGS : DST_LDS)>(z, lds, tw, mid);
    inv_passes<C, P + 1>(z, lds, tw, mid);
  }
}

// z <- P z for both rows of the pair (Alg. 2: P z = IDCT(eps * DCT(z))).
template <class C>
__device__ __forceinline__ void apply_P(float2 (&z)[C::E], float2* lds, const float2* tw, const float4* mid) {
  fwd_passes<C, 0>(z, lds, tw, mid);
  inv_passes<C, 0>(z, lds, tw, mid);
}

// ------------------------------------------------------------------ three-pass resident path
// N = R0 M R0 with one butterfly of the two outer passes per thread (C::RES): the transform of
// every length from 256 up.  The operator's constants stay out of memory inside the block loop: the
// twiddles of the last pass (a row of R0 per thread, kept as a few powers) and the eps factors of the
// middle step live in registers, loaded once; the inner pass's twiddles are copied to LDS once.  The
// forward last pass, the eps step and the inverse first pass are fused: thread t holds Y_k for
// k = t + q N/R0 after the forward FFT and needs exactly those elements for the inverse one, plus
// Y_{N-k}, which thread N/R0 - t holds; one LDS exchange brings the partner's values.  The inverse
// runs the same radices in the same order, so it shares every table, conjugated.
//
// Three passes because the exchanges through LDS bound the transform together with the VALU: a
// 64-lane 8-byte write costs the CU 6.5 clocks, an 8-byte read 4, and a 16-byte read, measured at
// twice the bytes per clock, 4.4, against about 190 two-clock instructions of a radix-16 butterfly
// over four SIMDs.  One larger inner radix (M = 20, 24, 25, 32) beats two small ones even where
// some waves idle in it.  Each exchange has a layout of its own, in which the accesses of the passes are
// free of bank conflicts (8-byte reads resolve per 32 lanes over 64 banks, 8-byte writes per 16 lanes
// over 32) except a few for R0 = 20 and 24; the eps step's partner reads, 8 bytes at a lane stride of 16,
// conflict two ways (2.5 % of the CU's cycles at N = 4096; read as 16-byte pairs they cost more):
//   first -> inner   element i = R0 t + q (output q of butterfly t) at slot q S1 + t: written in
//                    lane order; butterfly (jh, jm) of the inner pass reads input r at
//                    jm S1 + jh + r R0, its lanes running over jm and the low bit of jh
//   inner -> last    element jh N/R0 + c at the slot of row pair jh >> 1, column c, half jh & 1:
//                    2 ((jh >> 1) S2 + c) + (jh & 1), so that the last pass (input r of butterfly t =
//                    row r, column t) reads two rows in 16 bytes; the partner exchange reuses it
//                    (8-byte reads throughout instead cost N = 4096 5 %)
// N = 5120 as 16 x 20 x 16 against the four-pass 16 x 16 x 4 x 5 with its tables in memory: see
// the launch shapes in kashin_dispatch.hip for the measured times.
//
// A radix M > 32 is split: its R0^2 butterflies are each shared by S = T / R0^2 threads
// (wave-uniform sub-groups; see split_pass), its twiddles applied by the first pass to its outputs.
template <class C>
constexpr bool resident_ok() {
  return C::RES;
}
template <class C>
constexpr bool has_split_pass() {
  return C::RES && C::M > 32;
}
// LDS slots of the inner pass's twiddle table, after the exchange buffer
template <class C>
constexpr int small_tw_total() {
  return C::RES ? C::R0 * ((C::M + 1) & ~1) : 0;
}

// eps factors f_k of the fused step for the thread's elements k = t + q N/R0: kept as R0 complex
// values, or -- COMPACT, for kernels whose block loop is register-bound (the split shape, radices
// above 16, a 128-register budget) -- as e^{i pi t/N}/D and two masks (bit q: eps_k < 0, and
// eps_k != eps_{N-k}), from which f_k = eps_k / D or eps_k e^{i pi k/N} / D =
// eps_k (e^{i pi t/N} / D) e^{i pi q/R0} is rebuilt at each use (D = N, or p_divisor).
template <class C>
constexpr bool compact_eps() {
  return has_split_pass<C>() || C::R0 > 16 || (C::W >= 4 && C::R0 == 16);
}
template <class C, bool COMPACT>
struct EpsRegs {
  float2 f[C::R0];
};
template <class C>
struct EpsRegs<C, true> {
  float2 base;
  uint32_t neg, swap;
};
// f_k for element q, and whether it takes the partner value (eps_k != eps_{N-k})
template <class C, int q, bool COMPACT>
__device__ __forceinline__ float2 eps_factor(const EpsRegs<C, COMPACT>& e, bool& partner) {
  if constexpr (COMPACT) {
    partner = (e.swap >> q) & 1u;
    const bool neg = (e.neg >> q) & 1u;
    constexpr float cx = HalfTab<C::R0>::c[q], cy = HalfTab<C::R0>::s[q];
    constexpr float inv_n = static_cast<float>(1.0 / p_divisor(C::N, C::R0, C::M));
    const float2 g = partner ? make_float2(e.base.x * cx - e.base.y * cy, e.base.x * cy + e.base.y * cx)
                             : make_float2(inv_n, 0.f);
    return neg ? make_float2(-g.x, -g.y) : g;
  } else {
    const float2 f = e.f[q];
    partner = f.y != 0.f;
    return f;
  }
}

template <class C, bool COMPACT = false>
struct ResRegs {
  static constexpr bool compact = COMPACT && has_split_pass<C>();
  float2 tw[C::R0];         // stored powers of w_N^t (kept_tw); the rest are products of two of these
  EpsRegs<C, COMPACT> eps;  // eps factors of the fused step for elements k = t + r N/R0
};

__device__ __forceinline__ float2 cmulf(float2 x, float2 y) {
  return make_float2(x.x * y.x - x.y * y.y, x.x * y.y + x.y * y.x);
}
// Twiddle r of the last pass, w_N^{r t}: below radix 16 all are kept; else r = 4a + b is the product
// w_{4a} w_b (one rounding) of the kept powers 1, 2, 3, 4, 8, 12, ..  Only the split shape keeps no
// more than 1 and 4, from which w^15 takes five products: at 5120 and 6144 that put P's error up by
// 10 and 7 % (rms 18.9e-8 and 19.5e-8 of the input against 17.0e-8 and 18.1e-8), for 0.2 and 1.2 % of
// the quantiser's time (it spills 21 and 33 registers; with two powers 1 and 21).
template <class C, class RR>
constexpr bool kept_tw(int r) {
  return C::R0 < 16 ? r > 0 : (RR::compact ? (r == 1 || r == 4) : r > 0 && (r < 4 || r % 4 == 0));
}
template <class C, int r, class RR>
__device__ __forceinline__ float2 last_tw(const RR& rr) {
  if constexpr (kept_tw<C, RR>(r)) return rr.tw[r];
  else if constexpr (r == 2) return cmulf(rr.tw[1], rr.tw[1]);
  else if constexpr (r == 3) return cmulf(last_tw<C, 2>(rr), rr.tw[1]);
  else if constexpr (r % 4 == 0) return cmulf(last_tw<C, r - 4>(rr), rr.tw[4]);
  else return cmulf(last_tw<C, (r & ~3)>(rr), last_tw<C, (r & 3)>(rr));
}

__device__ __forceinline__ void launder(float2& v) { asm volatile("" : "+v"(v.x), "+v"(v.y)); }

// Before each last pass: declare the stored powers modified (in place, no instruction), so
// the products formed from them are neither hoisted out of the block loop nor shared between
// the two last passes of one application of P, either of which would keep many more complex
// values live.
template <class C, class RR>
__device__ __forceinline__ void launder_powers(RR& rr) {
  if constexpr (C::R0 >= 16) {
    sfor<1, C::R0>([&](auto rv) {
      constexpr int r = decltype(rv)::value;
      if constexpr (kept_tw<C, RR>(r)) launder(rr.tw[r]);
    });
  }
  // the compact eps factors are rebuilt inside the block loop, not hoisted out of it as R0 live values
  if constexpr (compact_eps<C>() && std::is_same<decltype(rr.eps), EpsRegs<C, true>>::value)
    asm volatile("" : "+v"(rr.eps.base.x), "+v"(rr.eps.base.y), "+v"(rr.eps.neg), "+v"(rr.eps.swap));
}

template <class C, class RR>
__device__ __forceinline__ void resident_load(RR& rr, float2* lds, const float2* __restrict__ tw,
                                              const float4* __restrict__ mid) {
  constexpr int R = C::R0;
  constexpr int NB = C::NB0;
  const int t = threadIdx.x;
  const int tl = (C::T == NB || t < NB) ? t : 0;  // threads past the last butterfly load row 0 (unused)
  const float4* t4 = reinterpret_cast<const float4*>(tw + tw_offset<C, false>(2) + tl * R);
  sfor<0, R / 2>([&](auto hv) {
    constexpr int h = decltype(hv)::value;
    if constexpr (kept_tw<C, RR>(2 * h) || kept_tw<C, RR>(2 * h + 1)) {
      const float4 q = t4[h];
      rr.tw[2 * h] = make_float2(q.x, q.y);
      rr.tw[2 * h + 1] = make_float2(q.z, q.w);
    }
  });
  if constexpr (std::is_same<decltype(rr.eps), EpsRegs<C, true>>::value) {
    uint32_t neg = 0, swap = 0;
    sfor<0, R>([&](auto rv) {
      constexpr int q = decltype(rv)::value;
      const float4 m = mid[tl * R + q];  // {Re f_k, Im f_k, -, eps_k}
      neg |= (m.w < 0.f ? 1u : 0u) << q;
      swap |= (m.y != 0.f ? 1u : 0u) << q;
    });
    float sn, cs;
    sincospif(static_cast<float>(tl) / static_cast<float>(C::N), &sn, &cs);
    rr.eps.neg = neg;
    rr.eps.swap = swap;
    constexpr float inv_n = static_cast<float>(1.0 / p_divisor(C::N, C::R0, C::M));
    rr.eps.base = make_float2(cs * inv_n, sn * inv_n);
  } else {
    sfor<0, R>([&](auto rv) {
      const float4 m = mid[tl * R + decltype(rv)::value];
      rr.eps.f[decltype(rv)::value] = make_float2(m.x, m.y);
    });
  }
  // inner-pass table, entry [jm][r] of the global layout: [r][jm] for a split pass (the first pass
  // reads entries jm, jm + 1), else [r / 2][jm] pairs (entries r and r + 1 side by side, one 16-byte
  // read per pair), the lanes of a wave (consecutive jm) reading consecutive words either way
  float2* small = lds + C::LDS;
  for (int i = t; i < R * C::M; i += C::T) {
    const int jm = i / C::M, r = i % C::M;
    const int at = has_split_pass<C>() ? r * R + jm : 2 * ((r / 2) * R + jm) + (r & 1);
    small[at] = tw[tw_offset<C, false>(1) + i];
  }
  lds_barrier();
}

// Butterfly (jh, jm) = jh R0 + jm of the inner pass that lane l takes: lanes run over the low bit of
// jh first, then jm, so that 16 lanes write 16 consecutive slots of the inner -> last layout.
template <class C>
struct InnerLane {
  int rd, wr, jm;
  __device__ __forceinline__ explicit InnerLane(int l) {
    const int p = l & 1, hq = (l >> 1) / C::R0;
    jm = (l >> 1) % C::R0;
    rd = jm * C::S1 + 2 * hq + p;
    wr = 2 * (hq * C::S2 + jm) + p;
  }
};

// The inner pass: R0^2 butterflies of radix M, thread t taking t, t + T, ..; LDS -> LDS in place
// (every read completes before any write).
template <class C, bool INV>
__device__ __forceinline__ void res_inner_pass(float2* __restrict__ lds) {
  const int t = opaque(threadIdx.x);  // each pass forms its own addresses: none stays live across others
  constexpr int R0 = C::R0;
  constexpr int M = C::M;
  constexpr int NB = R0 * R0;
  constexpr int BPT = (NB + C::T - 1) / C::T;
  static_assert(C::LDS % 2 == 0, "16-byte twiddle pairs");
  float2 a[BPT][M];
  constexpr int MP = (M + 1) / 2;
  // twiddle pairs read before the barrier, so that their latency passes while the waves gather there
  // (eight of them; four where 128 registers hold everything: y = P x at 6144 117 -> 106 us a 5461 rows)
  constexpr int PFM = C::W >= 4 && C::R0 >= 16 ? 4 : 8;
  constexpr int PF = BPT == 1 ? (MP < PFM ? MP : PFM) : 0;
  float4 pf[PF > 0 ? PF : 1];
  sfor<0, BPT>([&](auto iv) {
    constexpr int i = decltype(iv)::value;
    const int l = t + C::T * i;
    if (NB % C::T == 0 || l < NB) {
      const InnerLane<C> il(l);
      const float2* rb = lds + il.rd;
      sfor<0, M>([&](auto rv) { a[i][decltype(rv)::value] = rb[decltype(rv)::value * R0]; });
      if constexpr (PF > 0) {
        const float4* tb = reinterpret_cast<const float4*>(lds + C::LDS) + il.jm;
        sfor<0, PF>([&](auto hv) { pf[decltype(hv)::value] = tb[decltype(hv)::value * R0]; });
      }
    }
  });
  lds_barrier();
  sfor<0, BPT>([&](auto iv) {
    constexpr int i = decltype(iv)::value;
    const int l = t + C::T * i;
    if (NB % C::T == 0 || l < NB) {
      const InnerLane<C> il(l);
      const float4* tb = reinterpret_cast<const float4*>(lds + C::LDS) + il.jm;  // [r / 2][jm]
      dft_tw<M, INV>(a[i], [&](auto rv) {
        constexpr int r = decltype(rv)::value;
        float4 q;
        if constexpr (r / 2 < PF) q = pf[r / 2];
        else q = tb[(r / 2) * R0];
        return (r & 1) ? make_float2(q.z, q.w) : make_float2(q.x, q.y);
      });
      float2* wb = lds + il.wr;
      sfor<0, M>([&](auto qv) { wb[decltype(qv)::value * 2 * R0] = a[i][decltype(qv)::value]; });
    }
  });
  lds_barrier();
}

// Split inner pass: odd radix R = M, R0^2 butterflies, each shared by S = T / R0^2 threads
// t = l + s R0^2 (s is uniform across a wave).  Every sub-group streams the R inputs of butterfly l
// from LDS once, forming the pair sums and differences a_r +- a_{R-r}, and accumulates only its own
// share of the (R-1)/2 output pairs (q, R-q); the twiddles were applied by the pass before.  Each
// sub-group has code of its own with the DFT constants as literals: an FMA with a literal issues
// in two clocks, one with a scalar register (a shared code path with the constants in SGPRs) in
// four, and the 588 FMAs a thread spends here were over half of the N = 11008 kernel's VALU time.
// One copy of that code serves both directions (apply_P_split), so that the block loop stays in
// the instruction cache.
template <class C>
struct SplitShape {
  static constexpr int R = C::M;
  static constexpr int NB = C::R0 * C::R0;
  static constexpr int S = C::T / NB;         // threads per butterfly
  static constexpr int H = (R - 1) / 2;       // output pairs (q, R - q)
  static constexpr int QP = (H + S - 1) / S;  // output pairs per sub-group
};

// sub-group SG's outputs: re +- i im for its pairs (q, R - q), and the sum of all inputs
template <class C, int SG>
__device__ __forceinline__ void split_accumulate(const float2* __restrict__ rb, float2 (&re)[SplitShape<C>::QP],
                                                 float2 (&im)[SplitShape<C>::QP], float2& sum) {
  using SS = SplitShape<C>;
  constexpr int R = SS::R, H = SS::H, QP = SS::QP, R0 = C::R0;
  constexpr int D = 3;  // input pairs in flight
  const float2 x0 = rb[0];
  float2 p[D], m[D];
  sfor<0, D>([&](auto cv) {
    constexpr int c = decltype(cv)::value;
    p[c] = rb[(c + 1) * R0];
    m[c] = rb[(R - 1 - c) * R0];
  });
  sfor<0, QP>([&](auto iv) {
    re[decltype(iv)::value] = x0;
    im[decltype(iv)::value] = make_float2(0.f, 0.f);
  });
  sum = x0;
  sfor<0, H>([&](auto cv) {
    constexpr int c = decltype(cv)::value;
    constexpr int r = c + 1;
    const float2 sp = cadd(p[c % D], m[c % D]), dm = csub(p[c % D], m[c % D]);
    if constexpr (c + D < H) {
      p[c % D] = rb[(r + D) * R0];
      m[c % D] = rb[(R - r - D) * R0];
    }
    if constexpr (SG == 0) sum = cadd(sum, sp);
    sfor<0, QP>([&](auto iv) {
      constexpr int i = decltype(iv)::value;
      constexpr int q = SG * QP + 1 + i;
      if constexpr (q <= H) {
        constexpr float cc = CisTab<R>::c[(r * q) % R], sn = CisTab<R>::s[(r * q) % R];
        re[i].x = fmaf(sp.x, cc, re[i].x);
        re[i].y = fmaf(sp.y, cc, re[i].y);
        im[i].x = r == 1 ? dm.x * sn : fmaf(dm.x, sn, im[i].x);
        im[i].y = r == 1 ? dm.y * sn : fmaf(dm.y, sn, im[i].y);
      }
    });
    __builtin_amdgcn_sched_barrier(0);  // bound the values in flight
  });
}

template <class C>
__device__ __forceinline__ void split_pass(float2* __restrict__ lds, bool inv) {
  using SS = SplitShape<C>;
  constexpr int R = SS::R, NB = SS::NB, S = SS::S, QP = SS::QP, H = SS::H, R0 = C::R0;
  static_assert(R % 2 == 1 && NB % 64 == 0 && C::T % NB == 0 && S == 3 && H % S == 0, "split pass shape");
  const int t = opaque(threadIdx.x);
  const int s = __builtin_amdgcn_readfirstlane(t / NB);  // uniform across a wave
  const InnerLane<C> il(t - s * NB);
  float2 re[QP], im[QP], sum;
  if (s == 0) split_accumulate<C, 0>(lds + il.rd, re, im, sum);
  else if (s == 1) split_accumulate<C, 1>(lds + il.rd, re, im, sum);
  else split_accumulate<C, 2>(lds + il.rd, re, im, sum);
  lds_barrier();
  // forward: A_q = re - i im, A_{R-q} = re + i im; the inverse swaps them, by where they are written
  const int q0 = s * QP + 1;
  float2* wm = lds + il.wr + (inv ? R - q0 : q0) * 2 * R0;
  float2* wp = lds + il.wr + (inv ? q0 : R - q0) * 2 * R0;
  const int st = inv ? -2 * R0 : 2 * R0;
  sfor<0, QP>([&](auto iv) {
    constexpr int i = decltype(iv)::value;
    wm[i * st] = make_float2(re[i].x + im[i].y, re[i].y - im[i].x);
    wp[-i * st] = make_float2(re[i].x - im[i].y, re[i].y + im[i].x);
  });
  if (s == 0) lds[il.wr] = sum;
  lds_barrier();
}

// First pass (stride 1) of either direction: a[] -> LDS.  When the inner pass is split its input
// twiddles are applied here, to the outputs: element t R0 + q is input r = t / R0 of a butterfly
// with jm = q, so its twiddle is entry [r][q] of the LDS copy of that pass's table.
template <class C, bool INV>
__device__ __forceinline__ void res_first_pass(float2 (&a)[C::R0], float2* lds, int t) {
  constexpr int R = C::R0;
  dft_inplace<R, INV>(a);
  if constexpr (has_split_pass<C>()) {
    const float4* tb = reinterpret_cast<const float4*>(lds + C::LDS + (t / R) * R);
    sfor<0, R / 2>([&](auto hv) {
      constexpr int h = decltype(hv)::value;
      const float4 q = tb[h];
      if constexpr (h > 0) a[2 * h] = twmul<INV>(a[2 * h], make_float2(q.x, q.y));
      a[2 * h + 1] = twmul<INV>(a[2 * h + 1], make_float2(q.z, q.w));
    });
  }
  float2* wb = lds + t;
  sfor<0, R>([&](auto qv) { wb[decltype(qv)::value * C::S1] = a[decltype(qv)::value]; });
}

// Column t of the inner -> last layout: the inputs of the last pass's butterfly t.
template <class C>
__device__ __forceinline__ void res_read_column(float2 (&v)[C::R0], const float2* lds, int t) {
  const float4* rb = reinterpret_cast<const float4*>(lds) + t;
  sfor<0, C::R0 / 2>([&](auto hv) {
    constexpr int h = decltype(hv)::value;
    const float4 q = rb[h * C::S2];
    v[2 * h] = make_float2(q.x, q.y);
    v[2 * h + 1] = make_float2(q.z, q.w);
  });
}

// The fused step between the transforms: y[q] = Y_{t + q NB} -> f_k Y_{s(k)}, the values of
// thread N/R0 - t through LDS.  Column t is read and written by thread t alone before the barrier.
// Called by every thread; those without elements (act false) take part in the barriers.
template <class C, class RR>
__device__ __forceinline__ void res_eps_step(float2 (&y)[C::R0], float2* lds, const RR& rr, int t, bool act) {
  constexpr int R = C::R0;
  constexpr int NB = C::NB0;
  constexpr int H = R / 2;
  if (act) {
    float4* rb = reinterpret_cast<float4*>(lds) + t;
    sfor<0, H>([&](auto hv) {
      constexpr int h = decltype(hv)::value;
      rb[h * C::S2] = make_float4(y[2 * h].x, y[2 * h].y, y[2 * h + 1].x, y[2 * h + 1].y);
    });
  }
  lds_barrier();
  if (act) {
    // partner values Y_{N - t - q NB}: row R - 1 - q, column NB - t (thread 0 pairs q with R - q: its
    // bases are one row further, and q = 0 reads the slot past the last row, which is not used
    // since k = 0 pairs with itself).  The reads are issued ahead and used unconditionally: for a
    // select alone the compiler reads under a lane mask, element by element.
    const float2* pe = lds + (t == 0 ? H * 2 * C::S2 : (H - 1) * 2 * C::S2 + 2 * (NB - t) + 1);
    const float2* po = lds + (H - 1) * 2 * C::S2 + (t == 0 ? 1 : 2 * (NB - t));
    // reads in flight (fewer under a tight register budget)
    constexpr int D = R < 16 ? R : (R == 16 && compact_eps<C>() ? 4 : (R > 16 ? 8 : 16));
    float2 o[D];
    sfor<0, D>([&](auto qv) {
      constexpr int q = decltype(qv)::value;
      o[q] = (q & 1 ? po : pe)[-(q / 2) * 2 * C::S2];
    });
    sfor<0, R>([&](auto qv) {
      constexpr int q = decltype(qv)::value;
      float2 oth = o[q % D];
      launder(oth);
      if constexpr (q + D < R) o[q % D] = ((q + D) & 1 ? po : pe)[-((q + D) / 2) * 2 * C::S2];
      bool partner;
      const float2 fq = eps_factor<C, q>(rr.eps, partner);
      const float2 v = partner ? oth : y[q];
      y[q] = make_float2(fq.x * v.x - fq.y * v.y, fq.x * v.y + fq.y * v.x);
      if constexpr (q & 1) __builtin_amdgcn_sched_barrier(0);  // bound the values in flight
    });
  }
  lds_barrier();
}

// apply_P_res with a split inner pass: both transforms in one loop, so that the split pass's code
// (16 KB for its three sub-groups) is there once.
template <class C, class RR>
__device__ __forceinline__ void apply_P_split(float2 (&z)[C::E], float2* lds, RR& rr) {
  constexpr int R = C::R0;
  const bool act = (C::T == C::NB0) || threadIdx.x < C::NB0;
#pragma unroll 1
  for (int dir = 0; dir < 2; ++dir) {
    if (act) {
      if (dir == 0) res_first_pass<C, false>(z, lds, opaque(threadIdx.x));
      else res_first_pass<C, true>(z, lds, opaque(threadIdx.x));
    }
    lds_barrier();
    split_pass<C>(lds, dir != 0);
    const int t = opaque(threadIdx.x);
    launder_powers<C>(rr);
    if (act) {
      res_read_column<C>(z, lds, t);
      if (dir == 0) dft_tw<R, false>(z, [&](auto rv) { return last_tw<C, decltype(rv)::value>(rr); });
      else dft_tw<R, true>(z, [&](auto rv) { return last_tw<C, decltype(rv)::value>(rr); });
    } else {
      sfor<0, R>([&](auto rv) { z[decltype(rv)::value] = make_float2(0.f, 0.f); });
    }
    if (dir == 0) res_eps_step<C>(z, lds, rr, t, act);
  }
}

// z <- P z on the resident path.  Threads past the last outer butterfly (T > N/R0) take part in the
// inner pass and the barriers only.
template <class C, class RR>
__device__ __forceinline__ void apply_P_res(float2 (&z)[C::E], float2* lds, RR& rr) {
  constexpr int R = C::R0;
  if constexpr (has_split_pass<C>()) {
    apply_P_split<C>(z, lds, rr);
    return;
  }
  const bool act = (C::T == C::NB0) || threadIdx.x < C::NB0;
  // forward first pass (stride 1): registers -> LDS
  if (act) {
    float2 a[R];
    sfor<0, R>([&](auto rv) { a[decltype(rv)::value] = z[decltype(rv)::value]; });
    res_first_pass<C, false>(a, lds, opaque(threadIdx.x));
  }
  lds_barrier();
  res_inner_pass<C, false>(lds);
  // forward last pass (stride N/R0), fused with the eps step and the inverse first pass
  float2 y[R];
  const int t = opaque(threadIdx.x);
  if (act) res_read_column<C>(y, lds, t);
  launder_powers<C>(rr);
  if (act) dft_tw<R, false>(y, [&](auto rv) { return last_tw<C, decltype(rv)::value>(rr); });
  res_eps_step<C>(y, lds, rr, t, act);
  if (act) res_first_pass<C, true>(y, lds, opaque(threadIdx.x));
  lds_barrier();
  res_inner_pass<C, true>(lds);
  // inverse last pass: LDS -> registers
  launder_powers<C>(rr);
  if (act) {
    res_read_column<C>(z, lds, opaque(threadIdx.x));
    dft_tw<R, true>(z, [&](auto rv) { return last_tw<C, decltype(rv)::value>(rr); });
  } else {  // threads without elements hold zeros, set here so that z is not live across the transform
    sfor<0, R>([&](auto rv) { z[decltype(rv)::value] = make_float2(0.f, 0.f); });
  }
}

// ------------------------------------------------------------------ greedy step
__device__ __forceinline__ int8_t sgn8(float x) { return x > 0.f ? 1 : (x < 0.f ? -1 : 0); }
// sign(x) * c with sign(0) = 0, as the median of (-c, x 2^160, c): every nonzero float times 2^160
// is at least 2^11 in magnitude (or infinite), above any step size c -- on the normalised rows
// (max |w| < 1) c <= ||x||_2 <= ||w||_2 < sqrt(N) < 2^8, since no step raises the residual norm --
// so the median is exactly +-c; x = +-0 gives +-0, and x -/+ 0 leaves x unchanged up to the sign
// of a zero.  Two VALU operations instead of a compare, a copysign and a select.
__device__ __forceinline__ float sgn_times(float x, float c) {
  return __builtin_amdgcn_fmed3f(-c, __builtin_amdgcn_ldexpf(x, 160), c);
}

// s / N: exact for a power of two; otherwise s times the float nearest 1 / N (within one ulp of the
// quotient, and the step size c only enters the greedy as c itself)
template <int N>
__device__ __forceinline__ float div_n(float s) {
  return s * static_cast<float>(1.0 / N);
}

// One atomic greedy step of Alg. 2 on both rows: c = ||x||_1 / N, delta = sign(x) c
// (sign(0) = 0), x -= delta, and acc += delta when ACC.  Returns (c_a, c_b).  With
// `trace`, the signs of one side are written in row order.
template <class C, bool ACC>
__device__ __forceinline__ float2 greedy_step(float2 (&z)[C::E], float2 (&acc)[C::E], float* red, int& slot,
                                              int8_t* trace, int side) {
  float s[2] = {0.f, 0.f};
#pragma unroll
  for (int e = 0; e < C::E; ++e) {
    s[0] += fabsf(z[e].x);
    s[1] += fabsf(z[e].y);
  }
  block_sum<C::T, 2, C::UNI>(s, red, slot);
  const float ca = div_n<C::N>(s[0]);
  const float cb = div_n<C::N>(s[1]);
  if (trace != nullptr) {
    const int tid = opaque(threadIdx.x);
#pragma unroll
    for (int i = 0; i < C::B0; ++i) {
      const int j = tid + C::T * i;
      if (j < C::NB0) {
#pragma unroll
        for (int r = 0; r < C::R0; ++r) {
          const float2 v = z[i * C::R0 + r];
          trace[orig_index<C::N>(j + r * C::NB0)] = sgn8(side ? v.y : v.x);
        }
      }
    }
  }
#pragma unroll
  for (int e = 0; e < C::E; ++e) {
    const float da = sgn_times(z[e].x, ca);
    const float db = sgn_times(z[e].y, cb);
    if constexpr (ACC) {
      acc[e].x += da;
      acc[e].y += db;
    }
    z[e].x -= da;
    z[e].y -= db;
  }
  return make_float2(ca, cb);
}

// ------------------------------------------------------------------ loads / stores
__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(__half v) { return __half2float(v); }
__device__ __forceinline__ float to_f32(bf16_t v) { return bf16_to_f32(v); }

// Load rows a (and b if >= 0) into the greedy register layout, in even/odd order.
// `tid` is the thread index (a laundered copy in loops whose other values are invariant, so
// that the element offsets are recomputed rather than kept live across the loop).
template <class C, class IT>
__device__ __forceinline__ void load_pair_t(float2 (&z)[C::E], const IT* __restrict__ w, int64_t ldw, int64_t ra,
                                            int64_t rb, int tid = threadIdx.x) {
  const IT* __restrict__ pa = w + ra * ldw;
  const IT* __restrict__ pb = w + (rb >= 0 ? rb : ra) * ldw;
#pragma unroll
  for (int i = 0; i < C::B0; ++i) {
    const int j = tid + C::T * i;
#pragma unroll
    for (int r = 0; r < C::R0; ++r) {
      float2 v = make_float2(0.f, 0.f);
      if (C::NB0 % C::T == 0 || j < C::NB0) {
        const int src = orig_index<C::N>(j + r * C::NB0);
        v.x = to_f32(pa[src]);
        v.y = to_f32(pb[src]);
      }
      z[i * C::R0 + r] = v;
    }
  }
  if (rb < 0) {
#pragma unroll
    for (int e = 0; e < C::E; ++e) z[e].y = 0.f;
  }
}

template <class C, class F>
__device__ __forceinline__ void for_each_elem(F&& f, int tid = threadIdx.x) {
#pragma unroll
  for (int i = 0; i < C::B0; ++i) {
    const int j = tid + C::T * i;
    if (j < C::NB0) {
#pragma unroll
      for (int r = 0; r < C::R0; ++r) f(i * C::R0 + r, orig_index<C::N>(j + r * C::NB0));
    }
  }
}

// Rows a and b of w (b if >= 0, else zeros) into the LDS buffer in row order as float2 (row a
// in .x, row b in .y), times the rotation's sign s_i when ROT.  Each thread issues its loads in
// batches of eight per row before the first store, so that several are in flight at once.  Returns the
// rows (bit 0: a, 1: b) of which the thread saw an entry of at least kRotHuge, where HUGE_ROWS.
template <class C, bool ROT, bool HUGE_ROWS, class IT>
__device__ __forceinline__ uint32_t stage_pair_t(float2* lds, const IT* __restrict__ w, int64_t ldw, int64_t ra,
                                                 int64_t rb, uint64_t seed, int tid) {
  bool huge_a = false, huge_b = false;
  constexpr int K = (C::N + C::T - 1) / C::T;  // entries per thread and row
  constexpr int BATCH = 8;
  const IT* __restrict__ pa = w + ra * ldw;
  const IT* __restrict__ pb = w + (rb >= 0 ? rb : ra) * ldw;
#pragma unroll
  for (int k0 = 0; k0 < K; k0 += BATCH) {
    IT va[BATCH], vb[BATCH];
#pragma unroll
    for (int k = 0; k < BATCH; ++k) {
      const int i = tid + (k0 + k) * C::T;
      if (k0 + k < K && (C::N % C::T == 0 || i < C::N)) {
        va[k] = pa[i];
        vb[k] = pb[i];
      }
    }
#pragma unroll
    for (int k = 0; k < BATCH; ++k) {
      const int i = tid + (k0 + k) * C::T;
      if (k0 + k < K && (C::N % C::T == 0 || i < C::N)) {
        float2 v = make_float2(to_f32(va[k]), rb >= 0 ? to_f32(vb[k]) : 0.f);
        if constexpr (ROT) {
          if constexpr (HUGE_ROWS) {
            huge_a |= fabsf(v.x) >= kRotHuge;
            huge_b |= fabsf(v.y) >= kRotHuge;
          }
          v = rv_scale(v, rot_sign(seed, i));
        }
        lds[i] = v;
      }
    }
  }
  return (huge_a ? 1u : 0u) | (huge_b ? 2u : 0u);
}

// w (or R w when ROT: the rotation fused into the load) for both rows of the pair, handed to
// f(e, t) entry by entry in the greedy register layout (t = both rows' values at that entry,
// times 1 / sqrt(2^a) when ROT).  The rows are staged in the LDS buffer in row order; for ROT
// they are signed there and mixed by C_b and the Hadamard factor -- the operations of the
// standalone rotation kernel in the same order.  Uses the whole buffer, with a barrier on entry
// (a transform may still read it) and on exit (the next transform overwrites it).
template <class C, bool ROT, class F>
__device__ __forceinline__ void load_pair_staged(const void* w, int dtype, int64_t ldw, int64_t ra, int64_t rb,
                                                 uint64_t seed, float scale, float2* lds, F&& f) {
  constexpr int B = rot_odd_part(C::N);
  constexpr bool HUGE_ROWS = ROT && rot_watch_huge<B, false>();
  __shared__ uint32_t flags[HUGE_ROWS ? C::NW : 1];
  const int tid = threadIdx.x;
  uint32_t huge = 0;
  lds_barrier();
  if (dtype == KASHIN_F16)
    huge = stage_pair_t<C, ROT, HUGE_ROWS>(lds, static_cast<const __half*>(w), ldw, ra, rb, seed, tid);
  else if (dtype == KASHIN_BF16)
    huge = stage_pair_t<C, ROT, HUGE_ROWS>(lds, static_cast<const bf16_t*>(w), ldw, ra, rb, seed, tid);
  else huge = stage_pair_t<C, ROT, HUGE_ROWS>(lds, static_cast<const float*>(w), ldw, ra, rb, seed, tid);
  if constexpr (HUGE_ROWS) rot_note_huge(flags, huge, tid);
  lds_barrier();
  if constexpr (ROT) {
    huge = 0;
    if constexpr (HUGE_ROWS) huge = rot_huge_rows<C::NW>(flags);
    rot_odd_factor_fixed<B, false, C::T, C::N>(lds, huge, tid);
    rot_hadamard<B, C::T>(lds, C::N, tid);
  }
  for_each_elem<C>([&](int e, int i) { f(e, ROT ? rv_scale(lds[i], scale) : lds[i]); }, tid);
  lds_barrier();
}

template <class C>
__device__ __forceinline__ void load_pair(float2 (&z)[C::E], const void* w, int dtype, int64_t ldw, int64_t ra,
                                          int64_t rb, int tid = threadIdx.x) {
  if (dtype == KASHIN_F16) load_pair_t<C>(z, static_cast<const __half*>(w), ldw, ra, rb, tid);
  else if (dtype == KASHIN_BF16) load_pair_t<C>(z, static_cast<const bf16_t*>(w), ldw, ra, rb, tid);
  else load_pair_t<C>(z, static_cast<const float*>(w), ldw, ra, rb, tid);
}

// z <- w * scale - z for the pair (rows reloaded in the register layout); zero for a bad row.
template <class C>
__device__ __forceinline__ void sub_from_rows(float2 (&z)[C::E], const void* w, int dtype, int64_t ldw, int64_t ra,
                                              int64_t rb, float2 scale, bool bad_a, bool bad_b) {
  float2 t[C::E];
  load_pair<C>(t, w, dtype, ldw, ra, rb);
#pragma unroll
  for (int e = 0; e < C::E; ++e) {
    z[e].x = bad_a ? 0.f : fmaf(t[e].x, scale.x, -z[e].x);
    z[e].y = bad_b ? 0.f : fmaf(t[e].y, scale.y, -z[e].y);
  }
}



// Per-row power-of-two scale s (|w| * s in [0.5, 1)) and a NaN/Inf flag, for both rows.
// Returns the scales and zeroes a row that is not finite.
template <class C>
__device__ __forceinline__ void normalise_pair(float2 (&z)[C::E], float* red, int& slot, float2& scale,
                                               float2& unscale, bool& bad_a, bool& bad_b) {
  // largest magnitude by its bits (the order of the floats, NaN above infinity): two instructions an
  // entry where a finiteness test, a select and a maximum took six, a tenth of a P-only pair's VALU
  uint32_t ma = 0, mb = 0;
#pragma unroll
  for (int e = 0; e < C::E; ++e) {
    const uint32_t ba = __float_as_uint(z[e].x) & 0x7fffffffu, bb = __float_as_uint(z[e].y) & 0x7fffffffu;
    ma = ma > ba ? ma : ba;
    mb = mb > bb ? mb : bb;
  }
  constexpr uint32_t kInf = 0x7f800000u;
  float v[2] = {__uint_as_float(ma < kInf ? ma : kInf), __uint_as_float(mb < kInf ? mb : kInf)};
  block_max<C::T, 2>(v, red, slot);
  bad_a = v[0] > FLT_MAX;
  bad_b = v[1] > FLT_MAX;
  int ea = 0, eb = 0;
  if (!bad_a && v[0] > 0.f) (void)frexpf(v[0], &ea);
  if (!bad_b && v[1] > 0.f) (void)frexpf(v[1], &eb);
  // a row of subnormals only (max below 2^-126) would need a scale above 2^126: clamp, so that the
  // scale stays finite and the scaled row stays finite and nonzero (it is then below 0.5)
  ea = ea < -126 ? -126 : ea;
  eb = eb < -126 ? -126 : eb;
  scale = make_float2(ldexpf(1.f, -ea), ldexpf(1.f, -eb));
  unscale = make_float2(ldexpf(1.f, ea), ldexpf(1.f, eb));
  if (bad_a || bad_b) {  // uniform over the workgroup
#pragma unroll
    for (int e = 0; e < C::E; ++e) {
      z[e].x = bad_a ? 0.f : z[e].x;
      z[e].y = bad_b ? 0.f : z[e].y;
    }
  }
#pragma unroll
  for (int e = 0; e < C::E; ++e) {
    z[e].x *= scale.x;
    z[e].y *= scale.y;
  }
}

__device__ __forceinline__ void sort4(float (&q)[4]) {
  auto cx = [](float& a, float& b) {
    const float lo = fminf(a, b), hi = fmaxf(a, b);
    a = lo;
    b = hi;
  };
  cx(q[0], q[1]);
  cx(q[2], q[3]);
  cx(q[0], q[2]);
  cx(q[1], q[3]);
  cx(q[1], q[2]);
}

// q[c] for a 2-bit code c held in a register (selects, no indexed access)
__device__ __forceinline__ float pick4(const float (&q)[4], uint32_t c) {
  const float lo = (c & 1) ? q[1] : q[0];
  const float hi = (c & 1) ? q[3] : q[2];
  return (c & 2) ? hi : lo;
}

__device__ __forceinline__ int code_of(float x, const float (&mids)[3]) {
  return (x > mids[0] ? 1 : 0) + (x > mids[1] ? 1 : 0) + (x > mids[2] ? 1 : 0);
}

__device__ __forceinline__ void closed_form(float a, float b, float (&q)[4]) {
  const float s = a + b, d = fabsf(a - b);
  q[0] = -s;
  q[1] = -d;
  q[2] = d;
  q[3] = s;
}

__device__ __forceinline__ void midpoints(const float (&q)[4], float (&m)[3]) {
  m[0] = (q[0] + q[1]) * 0.5f;
  m[1] = (q[1] + q[2]) * 0.5f;
  m[2] = (q[2] + q[3]) * 0.5f;
}

// Closed-form centres of both rows from the two step sizes of block 0 (Sec. 3.1), then
// `lloyd` plain 1-D k-means passes when LLOYD (an emptied cluster keeps its centre;
// centres re-sorted after each pass).  q[side][4], ascending.
template <class C, bool LLOYD>
__device__ __forceinline__ void cluster_factor(const float2 (&x)[C::E], float2 c1, float2 c2, int lloyd, float* red,
                                               int& slot, float (&q)[2][4]) {
  closed_form(c1.x, c2.x, q[0]);
  closed_form(c1.y, c2.y, q[1]);
  if constexpr (LLOYD) {
    // one row at a time, the four counts packed as bytes of one word (a thread holds fewer than
    // 256 entries of a row): 5 accumulators live instead of 16, so the pass fits the registers
    // the block loop leaves (sums and counts accumulate in the same order either way)
    static_assert(C::E < 256, "per-thread counts packed in bytes");
    for (int it = 0; it < lloyd; ++it) {
#pragma unroll
      for (int sd = 0; sd < 2; ++sd) {
        float mids[3];
        midpoints(q[sd], mids);
        float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
        uint32_t cnt = 0;
        for_each_elem<C>([&](int e, int) {
          const float xv = sd ? x[e].y : x[e].x;
          const int cd = code_of(xv, mids);
          s0 += (cd == 0) ? xv : 0.f;
          s1 += (cd == 1) ? xv : 0.f;
          s2 += (cd == 2) ? xv : 0.f;
          s3 += (cd == 3) ? xv : 0.f;
          cnt += 1u << (8 * cd);
        });
        float acc[8] = {s0, s1, s2, s3, static_cast<float>(cnt & 255u), static_cast<float>((cnt >> 8) & 255u),
                        static_cast<float>((cnt >> 16) & 255u), static_cast<float>(cnt >> 24)};
        block_sum<C::T, 8, C::UNI>(acc, red, slot);
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (acc[4 + c] > 0.f) q[sd][c] = acc[c] / acc[4 + c];
        sort4(q[sd]);
      }
    }
  }
}

// 2-bit codes of both rows (code = number of midpoints strictly below the value), staged
// in LDS in row order and packed four per byte: byte b holds elements 4b..4b+3, element
// 4b+k in bits 2k.  Leaves the LDS free (barrier on exit).
template <class C>
__device__ __forceinline__ void write_codes(const float2 (&x)[C::E], const float (&q)[2][4], float2* lds,
                                            uint8_t* dst, int64_t ra, int64_t rb, bool bad_a, bool bad_b) {
  float mids[2][3];
  midpoints(q[0], mids[0]);
  midpoints(q[1], mids[1]);
  uint8_t* cb = reinterpret_cast<uint8_t*>(lds);
  lds_barrier();  // the last FFT pass read this buffer without a closing barrier
  for_each_elem<C>([&](int e, int i) {
    cb[i] = static_cast<uint8_t>(code_of(x[e].x, mids[0]));
    cb[C::N + i] = static_cast<uint8_t>(code_of(x[e].y, mids[1]));
  });
  lds_barrier();
  static_assert(C::N % 4 == 0, "four codes a byte");
  constexpr int NBY = C::N / 4;
  constexpr int K = (NBY + C::T - 1) / C::T;  // bytes per thread and row, unrolled: no read waits for another
  const uint32_t* cw = reinterpret_cast<const uint32_t*>(lds);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int b = threadIdx.x + k * C::T;
    if (NBY % C::T != 0 && b >= NBY) continue;
#pragma unroll
    for (int sd = 0; sd < 2; ++sd) {
      const int64_t row = sd ? rb : ra;
      if (row < 0) continue;
      const uint32_t c = cw[sd * NBY + b];  // one code in the low bits of each byte
      const uint32_t byte = c | (c >> 6) | (c >> 12) | (c >> 18);
      dst[row * NBY + b] = (sd ? bad_b : bad_a) ? 0 : static_cast<uint8_t>(byte);
    }
  }
  lds_barrier();
}

__device__ __forceinline__ void store_centers(float* centers, int f, const float (&q)[2][4], int64_t ra, int64_t rb,
                                              float2 unscale, bool bad_a, bool bad_b) {
  const float qnan = __int_as_float(0x7fc00000);
#pragma unroll
  for (int c = 0; c < 4; ++c) centers[ra * 8 + f * 4 + c] = bad_a ? qnan : q[0][c] * unscale.x;
  if (rb >= 0) {
#pragma unroll
    for (int c = 0; c < 4; ++c) centers[rb * 8 + f * 4 + c] = bad_b ? qnan : q[1][c] * unscale.y;
  }
}

// ------------------------------------------------------------------ greedy kernel
// Alg. 2 for a pair of rows.  Only the residual z and the accumulated vhat live in
// registers across the blocks; after the last block (whose final P is skipped) the
// first factor is recovered exactly as u = w - P(z + vhat), since w = u + P vhat + P z.
// QUANT selects the fused quantizer instance (MODE_QUANTIZE), the other one serves
// MODE_DECOMPOSE and MODE_TRACE; LLOYD (QUANT only) the instance with k-means refinement
// after the closed form; ROT (QUANT only) the instance with the rotation fused into the loads.
// Each instance carries only the code and registers of its own variant.
template <class C, bool LLOYD, bool QUANT, bool ROT>
__global__ __launch_bounds__(C::T) __attribute__((amdgpu_waves_per_eu(C::W))) void pair_greedy_kernel(
    KArgs ka, int64_t item0) {
  __shared__ __align__(16) float2 lds[C::LDS + small_tw_total<C>()];
  __shared__ float red[2 * C::NW * 32];
  int64_t item = item0 + blockIdx.x;
  KArgs a = ka;
  if constexpr (QUANT) {
    if (ka.ngroup > 0) {  // grouped launch: the matrix of this row pair (uniform over the workgroup)
      int gi = 0;
#pragma unroll
      for (int g = 1; g < kMaxGroup; ++g)
        if (g < ka.ngroup && item >= ka.group[g].pair0) gi = g;
      const GroupItem& it = ka.group[gi];
      a.tw = it.tw;
      a.mid4 = it.mid4;
      a.w = it.w;
      a.ldw = it.ldw;
      a.m = it.m;
      a.codes_u = it.codes_u;
      a.codes_v = it.codes_v;
      a.centers = it.centers;
      item -= it.pair0;
    }
  }
  int64_t ra;
  int side = 0;
  if (!QUANT && a.mode == MODE_TRACE) {
    const int64_t row = a.rows[item];
    if (row < 0 || row >= a.m) return;  // uniform: the whole workgroup reads the same entry
    ra = row & ~int64_t(1);
    side = static_cast<int>(row & 1);
  } else {
    ra = 2 * item;
  }
  const int64_t rb = (ra + 1 < a.m) ? ra + 1 : -1;
  int slot = 0;

  constexpr bool RES = resident_ok<C>();
  ResRegs<C, compact_eps<C>()> rr;
  if constexpr (RES) resident_load<C>(rr, lds, a.tw, a.mid4);
  auto applyP = [&](float2(&v)[C::E]) {
    if constexpr (RES) apply_P_res<C>(v, lds, rr);
    else apply_P<C>(v, lds, a.tw, a.mid4);
  };

  float2 z[C::E], vh[C::E];
  if constexpr (ROT) {
#pragma unroll
    for (int e = 0; e < C::E; ++e) z[e] = make_float2(0.f, 0.f);
    load_pair_staged<C, true>(a.w, a.dtype, a.ldw, ra, rb, a.rot_seed, a.rot_scale, lds,
                              [&](int e, float2 t) { z[e] = t; });
  } else {
    load_pair<C>(z, a.w, a.dtype, a.ldw, ra, rb);
  }
  float2 scale, unscale;
  bool bad_a, bad_b;
  normalise_pair<C>(z, red, slot, scale, unscale, bad_a, bad_b);
#pragma unroll
  for (int e = 0; e < C::E; ++e) vh[e] = make_float2(0.f, 0.f);

  const int steps = 4 * a.iters;
  int8_t* trace = nullptr;
  float* trc = nullptr;
  if (!QUANT && a.mode == MODE_TRACE) {
    trace = a.tr_signs + (item * steps) * int64_t(C::N);
    trc = a.tr_c + item * steps;
  }
  // block-0 step sizes (equal in every lane): on the shapes whose block loop sits at its register
  // limit they wait for the epilogue in LDS rather than in registers across the loop, and so they do in
  // the instance that reports them, with thread 0 keeping the sums of the step sizes there too where a
  // workgroup has several waves (in registers both spilled 5 to 11 of them at 1024, 2048 and 4096: 128
  // rows, k = 10, 1024 wide 91.3 -> 85.7 us, 2048 wide 106.1 -> 100.4; a single wave waits for the sums:
  // 512 wide 43.8 -> 45.6)
  constexpr bool CS_LDS = C::RES && (!QUANT || C::R0 > 16 || C::W >= 4 || (C::M & (C::M - 1)) != 0);
  __shared__ float2 cs_lds[4];
  float2 cs_reg[4];
  float2* cs = CS_LDS ? cs_lds : cs_reg;
  constexpr bool CSUM_LDS = !QUANT && C::RES && C::T > 64;
  __shared__ float2 csum_lds[2];  // of the u-steps and the vhat-steps; thread 0's own
  float2 csum_reg[2];
  float2* csum = CSUM_LDS ? csum_lds : csum_reg;
  if (!CSUM_LDS || threadIdx.x == 0) csum[0] = csum[1] = make_float2(0.f, 0.f);
  auto step = [&](int t, int st, float2 c) {
    if (t == 0 && (!CS_LDS || threadIdx.x == 0)) cs[st] = c;
    if constexpr (!QUANT) {
      if (!CSUM_LDS || threadIdx.x == 0) csum[st >> 1] = cadd(csum[st >> 1], c);
      if (trc != nullptr && threadIdx.x == 0) trc[4 * t + st] = (side ? c.y : c.x) * (side ? unscale.y : unscale.x);
    }
  };
  // half-block h = 2t: two steps on the cube Q_N, accumulating into u (u itself is recovered at the
  // end); h = 2t + 1: two steps on P Q_N, in the z = P rho domain, accumulating into vhat.  P between
  // any two half-blocks (P^2 = I)
  auto half_u = [&](int t) {
    int8_t* tr = trace ? trace + int64_t(4 * t) * C::N : nullptr;
    float2 c = greedy_step<C, false>(z, vh, red, slot, tr, side);
    step(t, 0, c);
    c = greedy_step<C, false>(z, vh, red, slot, tr ? tr + C::N : nullptr, side);
    step(t, 1, c);
  };
  auto half_v = [&](int t) {
    int8_t* tr = trace ? trace + int64_t(4 * t + 2) * C::N : nullptr;
    float2 c = greedy_step<C, true>(z, vh, red, slot, tr, side);
    step(t, 2, c);
    c = greedy_step<C, true>(z, vh, red, slot, tr ? tr + C::N : nullptr, side);
    step(t, 3, c);
  };
  if constexpr (has_split_pass<C>()) {
    // one copy of P's code (see split_pass)
#pragma unroll 1
    for (int h = 0; h < 2 * a.iters; ++h) {
      if (h > 0) applyP(z);
      if (h & 1) half_v(h >> 1);
      else half_u(h >> 1);
    }
  } else {
    for (int t = 0; t < a.iters; ++t) {
      if (t > 0) applyP(z);
      half_u(t);
      applyP(z);
      half_v(t);
    }
  }

  if constexpr (CS_LDS) lds_barrier();  // cs (written by thread 0 in the first block) visible to all
  // Epilogue.  vhat is consumed first (written out, or clustered into codes) so that it is
  // not live while u = w - P(z + vhat) is formed: the register peak stays that of the loop.
  const float qnan = __int_as_float(0x7fc00000);
  const bool want_r = !QUANT && (a.mode == MODE_DECOMPOSE) && a.r != nullptr;
  float vmax[2] = {0.f, 0.f};
  if constexpr (QUANT) {
    float qv[2][4];
    cluster_factor<C, LLOYD>(vh, cs[2], cs[3], a.lloyd, red, slot, qv);
    write_codes<C>(vh, qv, lds, a.codes_v, ra, rb, bad_a, bad_b);
    if (threadIdx.x == 0) store_centers(a.centers, 1, qv, ra, rb, unscale, bad_a, bad_b);
  } else {
    int64_t oa = ra, ob = rb;
    bool wa = true, wb = rb >= 0;
    if (a.mode == MODE_TRACE) {
      wa = side == 0;
      wb = side == 1;
      oa = ob = item;
    }
    if (want_r) {  // keep the final z (scaled) in the r buffer until P z is formed below
      for_each_elem<C>([&](int e, int i) {
        a.r[ra * C::N + i] = z[e].x;
        if (rb >= 0) a.r[rb * C::N + i] = z[e].y;
      });
    }
    for_each_elem<C>([&](int e, int i) {
      if (wa) a.vhat[oa * C::N + i] = bad_a ? qnan : vh[e].x * unscale.x;
      if (wb) a.vhat[ob * C::N + i] = bad_b ? qnan : vh[e].y * unscale.y;
    });
#pragma unroll
    for (int e = 0; e < C::E; ++e) {
      vmax[0] = fmaxf(vmax[0], fabsf(vh[e].x));
      vmax[1] = fmaxf(vmax[1], fabsf(vh[e].y));
    }
  }

  // u = w - P(z + vhat) (row reloaded from HBM)
#pragma unroll
  for (int e = 0; e < C::E; ++e) z[e] = cadd(z[e], vh[e]);
  applyP(z);
  if constexpr (ROT) {
    load_pair_staged<C, true>(a.w, a.dtype, a.ldw, ra, rb, a.rot_seed, a.rot_scale, lds, [&](int e, float2 t) {
      z[e].x = bad_a ? 0.f : fmaf(t.x, scale.x, -z[e].x);
      z[e].y = bad_b ? 0.f : fmaf(t.y, scale.y, -z[e].y);
    });
  } else {
    sub_from_rows<C>(z, a.w, a.dtype, a.ldw, ra, rb, scale, bad_a, bad_b);
  }
  float2(&u)[C::E] = z;

  if constexpr (QUANT) {
    float qu[2][4];
    cluster_factor<C, LLOYD>(u, cs[0], cs[1], a.lloyd, red, slot, qu);
    write_codes<C>(u, qu, lds, a.codes_u, ra, rb, bad_a, bad_b);
    if (threadIdx.x == 0) store_centers(a.centers, 0, qu, ra, rb, unscale, bad_a, bad_b);
    return;
  }

  {
    int64_t oa = ra, ob = rb;
    bool wa = true, wb = rb >= 0;
    if (a.mode == MODE_TRACE) {
      wa = side == 0;
      wb = side == 1;
      oa = ob = item;
    }
    for_each_elem<C>([&](int e, int i) {
      if (wa) a.u[oa * C::N + i] = bad_a ? qnan : u[e].x * unscale.x;
      if (wb) a.u[ob * C::N + i] = bad_b ? qnan : u[e].y * unscale.y;
    });
  }
  if (a.mode != MODE_DECOMPOSE) return;
  if (a.bounds != nullptr) {
    float mx[4] = {0.f, vmax[0], 0.f, vmax[1]};
#pragma unroll
    for (int e = 0; e < C::E; ++e) {
      mx[0] = fmaxf(mx[0], fabsf(u[e].x));
      mx[2] = fmaxf(mx[2], fabsf(u[e].y));
    }
    block_max<C::T, 4>(mx, red, slot);
    if (threadIdx.x == 0) {
      float* bo = a.bounds + ra * 4;
      bo[0] = bad_a ? qnan : mx[0] * unscale.x;
      bo[1] = bad_a ? qnan : mx[1] * unscale.x;
      bo[2] = bad_a ? qnan : csum[0].x * unscale.x;
      bo[3] = bad_a ? qnan : csum[1].x * unscale.x;
      if (rb >= 0) {
        bo[4] = bad_b ? qnan : mx[2] * unscale.y;
        bo[5] = bad_b ? qnan : mx[3] * unscale.y;
        bo[6] = bad_b ? qnan : csum[0].y * unscale.y;
        bo[7] = bad_b ? qnan : csum[1].y * unscale.y;
      }
    }
  }
  if (a.cstep != nullptr && threadIdx.x == 0) {
    float* co = a.cstep + ra * 4;
#pragma unroll
    for (int st = 0; st < 4; ++st) co[st] = bad_a ? qnan : cs[st].x * unscale.x;
    if (rb >= 0) {
#pragma unroll
      for (int st = 0; st < 4; ++st) co[4 + st] = bad_b ? qnan : cs[st].y * unscale.y;
    }
  }
  if (want_r) {
    // r = P z_final (the residual of Alg. 2), from the z saved above
    __syncthreads();  // the saved z (in global memory) is read back by other threads of the workgroup
    load_pair_t<C>(z, a.r, C::N, ra, rb);
    applyP(z);
    for_each_elem<C>([&](int e, int i) {
      a.r[ra * C::N + i] = bad_a ? qnan : z[e].x * unscale.x;
      if (rb >= 0) a.r[rb * C::N + i] = bad_b ? qnan : z[e].y * unscale.y;
    });
  }
}

// ------------------------------------------------------------------ P-only kernel
// MODE_APPLY_P: y = P x.  MODE_RECON: w_hat = u_q + P v_q from codes and centres.
// Persistent over pairs: the grid is capped and each workgroup walks items
// blockIdx.x, blockIdx.x + gridDim.x, ... so the operator constants are loaded once per
// workgroup, not once per pair (one application of P is cheap next to them).  The
// reconstruction moves its rows between HBM and the FFT's register layout through the LDS
// buffer, in row order, so codes are read one byte per four elements and w_hat is written in
// contiguous 16-byte vectors; y = P x loads and stores in the register layout directly
// (measured faster for it than staging).
template <class C, bool ROT, bool GROUPED>
__global__ __launch_bounds__(C::T) __attribute__((amdgpu_waves_per_eu(C::W))) void pair_pmap_kernel(
    KArgs ka, int64_t item0, int64_t nitems) {
  __shared__ __align__(16) float2 lds[C::LDS + small_tw_total<C>()];
  __shared__ float red[2 * C::NW * 32];
  constexpr int N = C::N;
  static_assert(N % 4 == 0, "row staging in 16-byte vectors");
  constexpr int NBY = N / 4;
  constexpr int KQ = (NBY + C::T - 1) / C::T;  // code bytes per thread and row
  int slot = 0;
  constexpr bool RES = resident_ok<C>();
  ResRegs<C> rr;
  KArgs a = ka;
  int64_t first = blockIdx.x, stride = gridDim.x;
  if constexpr (GROUPED) {  // grouped reconstruction: this workgroup's matrix (uniform)
    int gi = 0;
#pragma unroll
    for (int g = 1; g < kMaxGroup; ++g)
      if (g < ka.ngroup && static_cast<int64_t>(blockIdx.x) >= ka.group[g].wg0) gi = g;
    const GroupItem& gr = ka.group[gi];
    a.tw = gr.tw;
    a.mid4 = gr.mid4;
    a.m = gr.m;
    a.in_codes_v = gr.codes_v;
    a.in_centers = gr.centers;
    a.w = gr.w;  // codes_u
    a.y = gr.y;
    a.ldy = gr.ldy;
    first = blockIdx.x - gr.wg0;
    stride = (gi + 1 < ka.ngroup ? ka.group[gi + 1].wg0 : static_cast<int64_t>(gridDim.x)) - gr.wg0;
    item0 = 0;
    nitems = (gr.m + 1) / 2;
  }
  if constexpr (RES) resident_load<C>(rr, lds, a.tw, a.mid4);
  const float qnan = __int_as_float(0x7fc00000);
  float* lf = reinterpret_cast<float*>(lds);  // staging: row a at [0, N), row b at [N, 2N)
  float4* lf4 = reinterpret_cast<float4*>(lds);
  const bool recon = a.mode == MODE_RECON;
  const bool vout = (reinterpret_cast<uintptr_t>(a.y) % 16 == 0) && (a.ldy % 4 == 0);
  for (int64_t it = first; it < nitems; it += stride) {
    const int64_t ra = 2 * (item0 + it);
    const int64_t rb = (ra + 1 < a.m) ? ra + 1 : -1;
    const int tid = opaque(threadIdx.x);
    // a thread's bytes of both rows' codes, all loads issued before the first is used: a loop that loads,
    // decodes and stores byte by byte waits for memory KQ times (at 8192, where a thread has eight, 16 rows
    // 24.1 -> 21.5 us and 4096 rows 118 -> 95; 4096 wide, 8192 rows 73.3 -> 65.5)
    auto load_codes = [&](const uint8_t* ca, const uint8_t* cb, uint32_t(&ba)[KQ], uint32_t(&bb)[KQ]) {
#pragma unroll
      for (int k = 0; k < KQ; ++k) {
        const int q = tid + k * C::T;
        ba[k] = ca[NBY % C::T == 0 || q < NBY ? q : NBY - 1];
        bb[k] = cb[NBY % C::T == 0 || q < NBY ? q : NBY - 1];
      }
    };
    float2 z[C::E];
#pragma unroll
    for (int e = 0; e < C::E; ++e) z[e] = make_float2(0.f, 0.f);
    // 1. y = P x reads its rows straight into the register layout; the reconstruction decodes
    // the v codes in row order into LDS (row b zero when absent)
    if (!recon) {
      load_pair<C>(z, a.w, /*fp32*/ 0, a.ldw, ra, rb, tid);
    } else {
      const float* cea = a.in_centers + ra * 8 + 4;
      const float* ceb = a.in_centers + (rb >= 0 ? rb : ra) * 8 + 4;
      const float qa[4] = {cea[0], cea[1], cea[2], cea[3]};
      const float qb[4] = {ceb[0], ceb[1], ceb[2], ceb[3]};
      const uint8_t* cva = a.in_codes_v + ra * NBY;
      const uint8_t* cvb = a.in_codes_v + (rb >= 0 ? rb : ra) * NBY;
      uint32_t bva[KQ], bvb[KQ];
      load_codes(cva, cvb, bva, bvb);
#pragma unroll
      for (int k = 0; k < KQ; ++k) {
        const int q = tid + k * C::T;
        if (NBY % C::T != 0 && q >= NBY) continue;
        const uint32_t ba = bva[k], bb = bvb[k];
        float4 va, vb;
        va.x = pick4(qa, ba & 3);
        va.y = pick4(qa, (ba >> 2) & 3);
        va.z = pick4(qa, (ba >> 4) & 3);
        va.w = pick4(qa, (ba >> 6) & 3);
        vb.x = pick4(qb, bb & 3);
        vb.y = pick4(qb, (bb >> 2) & 3);
        vb.z = pick4(qb, (bb >> 4) & 3);
        vb.w = pick4(qb, (bb >> 6) & 3);
        lf4[q] = va;
        lf4[N / 4 + q] = rb >= 0 ? vb : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
    if (recon) {
      lds_barrier();
      for_each_elem<C>([&](int e, int i) { z[e] = make_float2(lf[i], lf[N + i]); }, tid);
      lds_barrier();  // the staged v_q rows are read before the first pass overwrites the buffer
    }
    float2 scale, unscale;
    bool bad_a, bad_b;
    normalise_pair<C>(z, red, slot, scale, unscale, bad_a, bad_b);
    // a row that is not finite is zero in the pair and becomes NaN by its factor
    unscale.x = bad_a ? qnan : unscale.x;
    unscale.y = bad_b ? qnan : unscale.y;
    if constexpr (RES) apply_P_res<C>(z, lds, rr);
    else apply_P<C>(z, lds, a.tw, a.mid4);
    if (!recon) {
      for_each_elem<C>([&](int e, int i) {
        a.y[ra * a.ldy + i] = z[e].x * unscale.x;
        if (rb >= 0) a.y[rb * a.ldy + i] = z[e].y * unscale.y;
      }, tid);
      lds_barrier();  // the last pass read the buffer the next item's first pass writes
      continue;
    }
    if constexpr (ROT) {
      // w_hat = R^T (P v_q + u_q): both rows in row order as float2, u_q added, then the
      // Hadamard factor, C_b^T, the scale and the signs, as the standalone inverse rotation
      constexpr int B = rot_odd_part(N);
      lds_barrier();  // the last pass read the buffer
      for_each_elem<C>([&](int e, int i) {
        lds[i] = make_float2(z[e].x * unscale.x, z[e].y * unscale.y);
      }, tid);
      lds_barrier();
      const uint8_t* cua = static_cast<const uint8_t*>(a.w) + ra * NBY;
      const uint8_t* cub = static_cast<const uint8_t*>(a.w) + (rb >= 0 ? rb : ra) * NBY;
      const float* cea = a.in_centers + ra * 8;
      const float* ceb = a.in_centers + (rb >= 0 ? rb : ra) * 8;
      const float ua[4] = {cea[0], cea[1], cea[2], cea[3]};
      const float ub[4] = {ceb[0], ceb[1], ceb[2], ceb[3]};
      uint32_t bua[KQ], bub[KQ];
      load_codes(cua, cub, bua, bub);
#pragma unroll
      for (int j = 0; j < KQ; ++j) {
        const int q = tid + j * C::T;
        if (NBY % C::T != 0 && q >= NBY) continue;
        const uint32_t ba = bua[j], bb = bub[j];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          float2 v = lds[4 * q + k];
          v.x += pick4(ua, (ba >> (2 * k)) & 3);
          v.y += pick4(ub, (bb >> (2 * k)) & 3);
          lds[4 * q + k] = v;
        }
      }
      lds_barrier();
      rot_hadamard<B, C::T>(lds, N, tid);
      rot_odd_factor_fixed<B, true, C::T, N>(lds, 0, tid);
      float* ya = a.y + ra * a.ldy;
      float* yb = a.y + (rb >= 0 ? rb : ra) * a.ldy;
      uint64_t st = rot_state(a.rot_seed, tid);
#pragma unroll 4
      for (int i = tid; i < N; i += C::T, st += C::T * kRotStep) {
        const float s = rot_sign_of(st);
        const float2 v = lds[i];
        ya[i] = v.x * a.rot_scale * s;
        if (rb >= 0) yb[i] = v.y * a.rot_scale * s;
      }
      lds_barrier();  // read before the next item's first pass writes the buffer
      continue;
    }
    lds_barrier();  // the last pass read the buffer the outputs are staged in
    for_each_elem<C>([&](int e, int i) {
      lf[i] = z[e].x * unscale.x;
      lf[N + i] = z[e].y * unscale.y;
    }, tid);
    lds_barrier();
    // 2. reconstruction: w_hat = P v_q + u_q in row order, 16-byte stores
    const uint8_t* cua = static_cast<const uint8_t*>(a.w) + ra * NBY;
    const uint8_t* cub = static_cast<const uint8_t*>(a.w) + (rb >= 0 ? rb : ra) * NBY;
    const float* cea = a.in_centers + ra * 8;
    const float* ceb = a.in_centers + (rb >= 0 ? rb : ra) * 8;
    const float ua[4] = {cea[0], cea[1], cea[2], cea[3]};
    const float ub[4] = {ceb[0], ceb[1], ceb[2], ceb[3]};
    float* ya = a.y + ra * a.ldy;
    float* yb = a.y + (rb >= 0 ? rb : ra) * a.ldy;
    uint32_t bua[KQ], bub[KQ];
    load_codes(cua, cub, bua, bub);
#pragma unroll
    for (int k = 0; k < KQ; ++k) {
      const int q = tid + k * C::T;
      if (NBY % C::T != 0 && q >= NBY) continue;
      float4 oa = lf4[q], ob = lf4[N / 4 + q];
      const uint32_t ba = bua[k], bb = bub[k];
      oa.x += pick4(ua, ba & 3);
      oa.y += pick4(ua, (ba >> 2) & 3);
      oa.z += pick4(ua, (ba >> 4) & 3);
      oa.w += pick4(ua, (ba >> 6) & 3);
      ob.x += pick4(ub, bb & 3);
      ob.y += pick4(ub, (bb >> 2) & 3);
      ob.z += pick4(ub, (bb >> 4) & 3);
      ob.w += pick4(ub, (bb >> 6) & 3);
      if (vout) {
        reinterpret_cast<float4*>(ya)[q] = oa;
        if (rb >= 0) reinterpret_cast<float4*>(yb)[q] = ob;
      } else {
        ya[4 * q] = oa.x;
        ya[4 * q + 1] = oa.y;
        ya[4 * q + 2] = oa.z;
        ya[4 * q + 3] = oa.w;
        if (rb >= 0) {
          yb[4 * q] = ob.x;
          yb[4 * q + 1] = ob.y;
          yb[4 * q + 2] = ob.z;
          yb[4 * q + 3] = ob.w;
        }
      }
    }
    lds_barrier();  // staged outputs read before the next item stages its inputs
  }
}

// One output of both rows of a pair (the thread's elements given by f(e) as float2: row a in .x,
// row b in .y) written in row order through the LDS buffer: contiguous 16-byte stores (4-byte
// ones where a row is not 16-byte aligned) instead of the even/odd order's stride-2 stores, which
// leave every line half written per instruction.  out_b may be null (no row b to write).  Starts
// and ends with a barrier, so the buffer is free before and after.
template <class C, class F>
__device__ __forceinline__ void store_pair_staged(float2* lds, float* out_a, float* out_b, F&& f) {
  static_assert(C::N % 4 == 0, "rows staged as float4");
  float* lf = reinterpret_cast<float*>(lds);
  const float4* lf4 = reinterpret_cast<const float4*>(lds);
  lds_barrier();  // earlier readers of the buffer are done
  for_each_elem<C>([&](int e, int i) {
    const float2 v = f(e);
    lf[i] = v.x;
    lf[C::N + i] = v.y;
  });
  lds_barrier();
  const bool vec_a = (reinterpret_cast<uintptr_t>(out_a) & 15) == 0;
  const bool vec_b = (reinterpret_cast<uintptr_t>(out_b) & 15) == 0;
  for (int q = threadIdx.x; q < C::N / 4; q += C::T) {
    if (out_a != nullptr) {
      const float4 o = lf4[q];
      if (vec_a) {
        reinterpret_cast<float4*>(out_a)[q] = o;
      } else {
        out_a[4 * q] = o.x;
        out_a[4 * q + 1] = o.y;
        out_a[4 * q + 2] = o.z;
        out_a[4 * q + 3] = o.w;
      }
    }
    if (out_b != nullptr) {
      const float4 o = lf4[C::N / 4 + q];
      if (vec_b) {
        reinterpret_cast<float4*>(out_b)[q] = o;
      } else {
        out_b[4 * q] = o.x;
        out_b[4 * q + 1] = o.y;
        out_b[4 * q + 2] = o.z;
        out_b[4 * q + 3] = o.w;
      }
    }
  }
  lds_barrier();  // the staged rows are read before the buffer's next writer
}

// ------------------------------------------------------------------ schedule variants
// The greedy over Q_N u P Q_N with another step schedule (MODE_SCHEDULE; a.schedule).  Both
// domains of the residual are kept per row of the pair, rho and z = P rho; a step works in one
// domain per row (the two rows of a pair may choose differently), and one application of P to
// the pair's stepped values refreshes the other domain of both rows (P^2 = I).  That is one P
// per atomic step, twice what the alternating kernel needs; three arrays live across steps (the
// residual in two domains and vhat).  The register budget is relaxed to two waves per SIMD where
// the workgroup allows it.
// With a.rows set, workgroup i decomposes the pair holding row a.rows[i] and records that
// row's signs, step sizes, choices and ||rho||^2 after every step.
//
// Where the workgroup shape caps the registers (more than 512 threads: one workgroup per CU, 168
// VGPRs) or an array has 32 complex values, the arrays do not fit, and vhat lives outside the registers
// between its steps, so that the residual's two domains and the transform's array stay in them: in LDS
// where there is room (sched_vh_lds_values), else (13824, 14336, 16384) in private memory, read and
// written in 16 bytes, the whole array at each vhat-step.
template <class C>
constexpr bool sched_vh_in_memory() {
  return (C::T > 512 || C::E >= 32) && C::E % 2 == 0;
}
// vhat values a thread keeps in LDS beside the transform's buffer, of its 2E (row a's first, then row
// b's; each thread its own slots, touched only at vhat-steps), the rest in registers; 0 if less than row
// a's fit.  8192 keeps all 64 there (134 KB with the buffer: one workgroup of four waves a CU, no spills; k = 10,
// 4096 rows 4114 us, against 5683 for the four passes on 512 threads with vhat in registers), 11008 those
// that fit.  Private memory would be written back to HBM at every vhat-step.
template <class C>
constexpr int sched_vh_lds_values() {
  if constexpr (!sched_vh_in_memory<C>() || C::B0 != 1) {
    return 0;
  } else {
    constexpr int used = (C::LDS + small_tw_total<C>()) * 8 + 2 * C::NW * 32 * 4;
    constexpr int fit = (160 * 1024 - used) / (4 * C::NB0);
    return fit < C::E ? 0 : (fit < 2 * C::E ? fit : 2 * C::E);
  }
}
template <class C, bool TRACE>
__global__ __launch_bounds__(C::T) __attribute__((amdgpu_waves_per_eu(C::T <= 512 ? 2 : C::W))) void
pair_schedule_kernel(KArgs a, int64_t item0) {
  __shared__ __align__(16) float2 lds[C::LDS + small_tw_total<C>()];
  __shared__ float red[2 * C::NW * 32];
  const int64_t item = item0 + blockIdx.x;
  constexpr bool tracing = TRACE;  // an instance of its own: the trace code costs registers
  int64_t ra;
  int side = 0;
  if constexpr (tracing) {
    const int64_t row = a.rows[item];
    if (row < 0 || row >= a.m) return;  // uniform
    ra = row & ~int64_t(1);
    side = static_cast<int>(row & 1);
  } else {
    ra = 2 * item;
  }
  const int64_t rb = (ra + 1 < a.m) ? ra + 1 : -1;
  int slot = 0;
  constexpr bool RES = resident_ok<C>();
  ResRegs<C, compact_eps<C>()> rr;
  if constexpr (RES) resident_load<C>(rr, lds, a.tw, a.mid4);
  auto applyP = [&](float2(&v)[C::E]) {
    if constexpr (RES) apply_P_res<C>(v, lds, rr);
    else apply_P<C>(v, lds, a.tw, a.mid4);
  };
  constexpr int VL = sched_vh_lds_values<C>();  // vhat values per thread in LDS
  constexpr bool VHL = VL > 0;
  constexpr bool VHM = sched_vh_in_memory<C>() && !VHL;
  // The residual of each row in both domains: sv holds it in one domain and y = P sv in the other;
  // za / zb say which (true: sv holds z = P rho for that row).  A step takes each row's chosen
  // domain from sv or y, writes the stepped values to sv and transforms them into y, so no select
  // ever lands on the arrays carried from step to step.
  float2 sv[C::E], y[C::E], vh[VHM || VHL ? 1 : C::E];
  float4 vhm[VHM ? C::E / 2 : 1];  // vhat (VHM); a run-time index keeps it in memory
  // VHL: slot s < VL of thread t at vhl[s * NB0 + t], s = e for row a, E + e for row b; row b's
  // elements e >= VL - E in vhr
  __shared__ float vhl[VHL ? VL * C::NB0 : 1];
  float vhr[VHL && VL < 2 * C::E ? 2 * C::E - VL : 1];
  const int vt = threadIdx.x;
  const bool vown = vt < C::NB0;  // threads past the last butterfly hold no elements
  auto vh_slot = [&](int sl) -> float& { return vhl[sl * C::NB0 + vt]; };
  load_pair<C>(sv, a.w, a.dtype, a.ldw, ra, rb);
  float2 scale, unscale;
  bool bad_a, bad_b;
  normalise_pair<C>(sv, red, slot, scale, unscale, bad_a, bad_b);
#pragma unroll
  for (int e = 0; e < C::E; ++e) y[e] = sv[e];
  if constexpr (VHM) {
    const int b = opaque(0);
#pragma unroll
    for (int h = 0; h < C::E / 2; ++h) vhm[b + h] = make_float4(0.f, 0.f, 0.f, 0.f);
  } else if constexpr (VHL) {
    if (vown) {
#pragma unroll
      for (int sl = 0; sl < VL; ++sl) vh_slot(sl) = 0.f;
    }
#pragma unroll
    for (int k = 0; k < 2 * C::E - VL; ++k) vhr[k] = 0.f;
  } else {
#pragma unroll
    for (int e = 0; e < C::E; ++e) vh[e] = make_float2(0.f, 0.f);
  }
  applyP(y);
  bool za = false, zb = false;
  const int steps = 4 * a.iters;
  const int sched = a.schedule;
  const float tola = a.tol * scale.x, tolb = a.tol * scale.y;
  const float unsel = side ? unscale.y : unscale.x;
  for (int st = 0; st < steps; ++st) {
    // l1 norms, nonzero counts and squared norms of sv and y, both rows
    float s12[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) s12[k] = 0.f;
#pragma unroll
    for (int e = 0; e < C::E; ++e) {
      s12[0] += fabsf(sv[e].x);
      s12[1] += fabsf(sv[e].y);
      s12[2] += fabsf(y[e].x);
      s12[3] += fabsf(y[e].y);
      s12[4] += sv[e].x != 0.f ? 1.f : 0.f;
      s12[5] += sv[e].y != 0.f ? 1.f : 0.f;
      s12[6] += y[e].x != 0.f ? 1.f : 0.f;
      s12[7] += y[e].y != 0.f ? 1.f : 0.f;
      s12[8] += sv[e].x * sv[e].x;
      s12[9] += sv[e].y * sv[e].y;
      s12[10] += y[e].x * y[e].x;
      s12[11] += y[e].y * y[e].y;
    }
    if constexpr (C::NW * 12 > 64) block_sum_lanes<C::T, 12>(s12, red, slot);
    else block_sum<C::T, 12, C::UNI>(s12, red, slot);
    // threads past the last butterfly hold zeros: they add nothing to the counts above
    // v: l1 of rho and z, nonzero counts of rho and z, ||rho||^2 (rows a, b in turn)
    const float v[10] = {za ? s12[2] : s12[0],  zb ? s12[3] : s12[1], za ? s12[0] : s12[2], zb ? s12[1] : s12[3],
                         za ? s12[6] : s12[4],  zb ? s12[7] : s12[5], za ? s12[4] : s12[6], zb ? s12[5] : s12[7],
                         za ? s12[10] : s12[8], zb ? s12[11] : s12[9]};
    const int pos = st & 3;
    bool va, vb;  // true: the vhat-half (step on z)
    if (sched == SCHED_ALTERNATING) {
      va = vb = pos >= 2;
    } else if (sched == SCHED_REVERSE) {
      va = vb = pos < 2;
    } else {
      va = !(v[0] > v[2]);
      vb = !(v[1] > v[3]);
    }
    const bool act_a = !(sched == SCHED_ORIGINAL && a.tol > 0.f && sqrtf(v[8]) < tola);
    const bool act_b = !(sched == SCHED_ORIGINAL && a.tol > 0.f && sqrtf(v[9]) < tolb);
    const float l1a = va ? v[2] : v[0], l1b = vb ? v[3] : v[1];
    const float nza = va ? v[6] : v[4], nzb = vb ? v[7] : v[5];
    float ca = sched == SCHED_ORIGINAL ? (nza > 0.f ? l1a / nza : 0.f) : div_n<C::N>(l1a);
    float cb = sched == SCHED_ORIGINAL ? (nzb > 0.f ? l1b / nzb : 0.f) : div_n<C::N>(l1b);
    ca = act_a ? ca : 0.f;
    cb = act_b ? cb : 0.f;
    // each row's chosen domain: in sv when it is the domain sv holds, else in y
    const bool fa = va == za, fb = vb == zb;
    if constexpr (tracing) {
      const bool vs = side ? vb : va;
      const bool fs = side ? fb : fa;
      const int tid = opaque(threadIdx.x);
      int8_t* trs = a.tr_signs + (item * steps + st) * int64_t(C::N);
#pragma unroll
      for (int i = 0; i < C::B0; ++i) {
        const int j = tid + C::T * i;
        if (j < C::NB0) {
#pragma unroll
          for (int r = 0; r < C::R0; ++r) {
            const float2 xv = fs ? sv[i * C::R0 + r] : y[i * C::R0 + r];
            trs[orig_index<C::N>(j + r * C::NB0)] = sgn8(side ? xv.y : xv.x);
          }
        }
      }
      if (threadIdx.x == 0) {
        a.tr_c[item * steps + st] = (side ? cb : ca) * unsel;
        a.tr_choice[item * steps + st] = (side ? act_b : act_a) ? (vs ? 1 : 0) : -1;
      }
    }
    // vhat += the steps of the rows that step on z (VHM, VHL: the same values, through memory)
    if constexpr (VHL) {
      if (va && vown) {
#pragma unroll
        for (int e = 0; e < C::E; ++e) vh_slot(e) += sgn_times(fa ? sv[e].x : y[e].x, ca);
      }
      if (vb) {
#pragma unroll
        for (int e = 0; e < C::E; ++e) {
          const float d = sgn_times(fb ? sv[e].y : y[e].y, cb);
          if (C::E + e < VL) {
            if (vown) vh_slot(C::E + e) += d;
          } else {
            vhr[e - (VL - C::E)] += d;
          }
        }
      }
    }
    if constexpr (VHM) {
      if (va || vb) {
        const int b = opaque(0);
#pragma unroll
        for (int h = 0; h < C::E / 2; ++h) {
          float4 q = vhm[b + h];
          if (va) {
            q.x += sgn_times(fa ? sv[2 * h].x : y[2 * h].x, ca);
            q.z += sgn_times(fa ? sv[2 * h + 1].x : y[2 * h + 1].x, ca);
          }
          if (vb) {
            q.y += sgn_times(fb ? sv[2 * h].y : y[2 * h].y, cb);
            q.w += sgn_times(fb ? sv[2 * h + 1].y : y[2 * h + 1].y, cb);
          }
          vhm[b + h] = q;
        }
      }
    }
    // the step, in each row's chosen domain; sv collects the stepped values of both rows
#pragma unroll
    for (int e = 0; e < C::E; ++e) {
      float xa = fa ? sv[e].x : y[e].x;
      float xb = fb ? sv[e].y : y[e].y;
      const float da = sgn_times(xa, ca), db = sgn_times(xb, cb);
      xa -= da;
      xb -= db;
      if constexpr (!VHM && !VHL) {
        if (va) vh[e].x += da;
        if (vb) vh[e].y += db;
      }
      sv[e] = make_float2(xa, xb);
      y[e] = sv[e];
    }
    applyP(y);  // the other domain of each row
    za = va;
    zb = vb;
    if constexpr (tracing) {
      float q[1] = {0.f};
      const bool zs = side ? zb : za;  // rho of the traced row: y if sv holds its z
#pragma unroll
      for (int e = 0; e < C::E; ++e) {
        const float2 rv = zs ? y[e] : sv[e];
        q[0] += side ? rv.y * rv.y : rv.x * rv.x;
      }
      block_sum<C::T, 1, C::UNI>(q, red, slot);
      if (threadIdx.x == 0) a.tr_r2[item * steps + st] = q[0] * unsel * unsel;
    }
  }
  // u = w - r - P vhat (row reloaded from HBM), in steps that keep two arrays live: rho of each
  // row into sv and out to r; then sv = w - rho; then y = P vhat and u = sv - y
  const float qnan = __int_as_float(0x7fc00000);
#pragma unroll
  for (int e = 0; e < C::E; ++e) sv[e] = make_float2(za ? y[e].x : sv[e].x, zb ? y[e].y : sv[e].y);
  int64_t oa = ra, ob = rb;
  bool wa = true, wb = rb >= 0;
  if constexpr (tracing) {
    wa = side == 0;
    wb = side == 1;
    oa = ob = item;
  }
  auto out_rows = [&](float* base, float*& pa, float*& pb) {
    pa = wa ? base + oa * C::N : nullptr;
    pb = wb ? base + ob * C::N : nullptr;
  };
  float *pa, *pb;
  if (a.r != nullptr) {
    out_rows(a.r, pa, pb);
    store_pair_staged<C>(lds, pa, pb, [&](int e) {
      return make_float2(bad_a ? qnan : sv[e].x * unscale.x, bad_b ? qnan : sv[e].y * unscale.y);
    });
  }
  {
    float2 t[C::E];
    load_pair<C>(t, a.w, a.dtype, a.ldw, ra, rb);
#pragma unroll
    for (int e = 0; e < C::E; ++e)
      sv[e] = make_float2(fmaf(t[e].x, scale.x, -sv[e].x), fmaf(t[e].y, scale.y, -sv[e].y));
  }
  auto vhat_at = [&](int e) -> float2 {
    if constexpr (VHM) {
      const float4 q = vhm[opaque(0) + e / 2];
      return (e & 1) ? make_float2(q.z, q.w) : make_float2(q.x, q.y);
    } else if constexpr (VHL) {
      const float b = C::E + e < VL ? (vown ? vh_slot(C::E + e) : 0.f) : vhr[e - (VL - C::E)];
      return make_float2(vown ? vh_slot(e) : 0.f, b);
    } else {
      return vh[e];
    }
  };
#pragma unroll
  for (int e = 0; e < C::E; ++e) y[e] = vhat_at(e);
  lds_barrier();  // without an r output nothing else separates the last step's P from this one
  applyP(y);
  out_rows(a.u, pa, pb);
  store_pair_staged<C>(lds, pa, pb, [&](int e) {
    return make_float2(bad_a ? qnan : (sv[e].x - y[e].x) * unscale.x, bad_b ? qnan : (sv[e].y - y[e].y) * unscale.y);
  });
  out_rows(a.vhat, pa, pb);
  store_pair_staged<C>(lds, pa, pb, [&](int e) {
    const float2 vhe = vhat_at(e);
    return make_float2(bad_a ? qnan : vhe.x * unscale.x, bad_b ? qnan : vhe.y * unscale.y);
  });
}

// ------------------------------------------------------------------ dispatch
// Whether the incoherence rotation of length N can be fused into the pair kernels: the odd
// factor C_b has compile-time constants for b = 1, 3 and 43 only (the lengths the rotation kernel
// takes); the host layer rejects the rotated entry points for other lengths before any launch.
constexpr bool rot_fusable(int n) {
  const int b = n / (n & -n);
  return n <= 16384 && (b == 1 || b == 3 || b == 43);
}

template <class C>
hipError_t launch_cfg(const KArgs& a, int64_t grid, hipStream_t s) {
  constexpr int64_t kMaxGrid = int64_t(1) << 30;
  if constexpr (!rot_fusable(C::N)) {
    if (a.rot) return hipErrorInvalidValue;
  }
  for (int64_t i0 = 0; i0 < grid; i0 += kMaxGrid) {
    const int64_t g = (grid - i0 < kMaxGrid) ? grid - i0 : kMaxGrid;
    const dim3 gd(static_cast<unsigned>(g)), bd(C::T);
    if (a.mode == MODE_QUANTIZE) {
      if (a.rot) {
        if constexpr (rot_fusable(C::N)) {
          if (a.lloyd > 0) hipLaunchKernelGGL((pair_greedy_kernel<C, true, true, true>), gd, bd, 0, s, a, i0);
          else hipLaunchKernelGGL((pair_greedy_kernel<C, false, true, true>), gd, bd, 0, s, a, i0);
        }
      } else if (a.lloyd > 0) {
        hipLaunchKernelGGL((pair_greedy_kernel<C, true, true, false>), gd, bd, 0, s, a, i0);
      } else {
        hipLaunchKernelGGL((pair_greedy_kernel<C, false, true, false>), gd, bd, 0, s, a, i0);
      }
    } else if (a.mode <= MODE_TRACE) {
      hipLaunchKernelGGL((pair_greedy_kernel<C, false, false, false>), gd, bd, 0, s, a, i0);
    } else if (a.mode == MODE_SCHEDULE) {
      if (a.rows != nullptr)
        hipLaunchKernelGGL((pair_schedule_kernel<C, true>), dim3(static_cast<unsigned>(g)), dim3(C::T), 0, s, a, i0);
      else
        hipLaunchKernelGGL((pair_schedule_kernel<C, false>), dim3(static_cast<unsigned>(g)), dim3(C::T), 0, s, a, i0);
    } else {
      // grouped reconstruction: `grid` is the launch's workgroup count (the matrices' shares)
      const int64_t pg = a.ngroup > 0 ? g : (g < kPmapGrid ? g : kPmapGrid);
      if (a.rot) {
        if constexpr (rot_fusable(C::N))
          hipLaunchKernelGGL((pair_pmap_kernel<C, true, false>), dim3(static_cast<unsigned>(pg)), bd, 0, s, a, i0, g);
      } else if (a.ngroup > 0) hipLaunchKernelGGL((pair_pmap_kernel<C, false, true>), dim3(static_cast<unsigned>(pg)), bd, 0, s, a, i0, g);
      else hipLaunchKernelGGL((pair_pmap_kernel<C, false, false>), dim3(static_cast<unsigned>(pg)), bd, 0, s, a, i0, g);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

// Defines the external launcher launch_n<N> for one launch configuration.
#define KASHIN_DEFINE_SIZE(N, T, W, ...)                                                     \
  hipError_t launch_n##N(const KArgs& a, int64_t grid, hipStream_t stream) {                \
    return launch_cfg<Cfg<N, T, W, __VA_ARGS__>>(a, grid, stream);                          \
  }

}  // namespace kashin
