// Internal interface between the C-ABI host layer (kashin_api.cpp) and the HIP
// kernels (kashin_kernels.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace kashin {

// bfloat16 input (KASHIN_BF16): the upper 16 bits of an IEEE binary32, widened exactly by a shift
struct bf16_t {
  uint16_t bits;
};
__device__ inline float bf16_to_f32(bf16_t v) {
  return __uint_as_float(static_cast<uint32_t>(v.bits) << 16);
}

enum Mode : int32_t {
  MODE_DECOMPOSE = 0,  // write u, vhat (+ r, cstep, bounds)
  MODE_QUANTIZE = 1,   // fused decompose + cluster + pack, write codes and centres only
  MODE_TRACE = 2,      // decompose listed rows and record every sign decision
  MODE_APPLY_P = 3,    // y = P x
  MODE_RECON = 4,      // w_hat = u_q + P v_q
  MODE_SCHEDULE = 5,   // greedy with another step schedule (writes u, vhat, r; traces listed rows)
};

enum Schedule : int32_t {
  SCHED_ALTERNATING = 0,  // blocks u, u, vhat, vhat (Alg. 2)
  SCHED_REVERSE = 1,      // blocks vhat, vhat, u, u
  SCHED_ADAPTIVE = 2,     // the half with the larger l1 correlation, step ||.||_1 / N
  SCHED_ORIGINAL = 3,     // Alg. 1: that choice, projection step ||.||_1 / nnz, stop at ||rho|| < tol
};

// One matrix of a grouped launch: its plan's tables, rows, codes, centres, output rows, and the
// index of its first row pair among the launch's items.  Quantisation reads w and writes the
// codes and centres; reconstruction reads the codes (w = codes_u) and centres and writes y.
struct GroupItem {
  const float2* tw;
  const float4* mid4;
  const void* w;
  int64_t ldw;
  int64_t m;
  uint8_t* codes_u;
  uint8_t* codes_v;
  float* centers;
  float* y;
  int64_t ldy;
  int64_t pair0;
  int64_t wg0;  // reconstruction: the matrix's first workgroup (it takes wg0 .. next matrix's wg0 - 1)
};
constexpr int kMaxGroup = 16;  // matrices per grouped launch (the table travels in the kernel arguments)
constexpr int64_t kPmapGrid = 2048;  // persistent y = P x / reconstruction grid: resident workgroups, a few times over

// Everything a launch needs, passed to the kernel by value.
struct KArgs {
  // operator tables (plan-owned, device)
  const float2* tw;    // per-pass twiddle tables (layout: see build_tables in kashin_api.cpp)
  const float4* mid4;  // first inverse pass, per (j, r): {f.x, f.y, LDS byte address of the source, 0}
  int32_t iters;       // blocks of Alg. 2
  int32_t mode;
  int32_t dtype;       // input dtype (KASHIN_F32 / KASHIN_F16)
  int32_t lloyd;       // Lloyd passes for the fused clustering
  int64_t m;           // rows in the matrix
  int64_t ldw;         // leading dimension of the input matrix
  const void* w;       // input rows (w, x, or codes_u for MODE_RECON)
  // outputs / other inputs
  float* u;
  float* vhat;
  float* r;
  float* cstep;
  float* bounds;
  uint8_t* codes_u;
  uint8_t* codes_v;
  float* centers;
  const uint8_t* in_codes_v;  // MODE_RECON
  const float* in_centers;    // MODE_RECON
  float* y;                   // MODE_APPLY_P / MODE_RECON output
  int64_t ldy;
  // trace
  const int64_t* rows;
  int64_t nrows;
  int8_t* tr_signs;
  float* tr_c;
  // MODE_SCHEDULE
  int32_t schedule;
  float tol;
  int8_t* tr_choice;
  float* tr_r2;
  // incoherence rotation fused into the load (quantize, decompose, trace) or the store (recon)
  int32_t rot;
  float rot_scale;  // 1 / sqrt(2^a), n = 2^a b
  uint64_t rot_seed;
  // MODE_QUANTIZE over several matrices of one vector length (ngroup > 0): item p is row pair
  // p - group[g].pair0 of the last matrix g with group[g].pair0 <= p.  MODE_RECON: workgroup b
  // serves the last matrix g with group[g].wg0 <= b, walking its row pairs with the stride of
  // that matrix's workgroup count
  int32_t ngroup;
  GroupItem group[kMaxGroup];
};

struct ClusterArgs {
  const float* u;
  const float* vhat;
  const float* cstep;
  int64_t m;
  int32_t n;
  int32_t lloyd;
  uint8_t* codes_u;
  uint8_t* codes_v;
  float* centers;
};

// Radix plan of the pair kernel for vector length n: threads per workgroup and the radices
// of the forward FFT passes.
struct PlanShape {
  int n = 0;
  int threads = 0;
  int np = 0;
  int rad[8] = {};
};
bool plan_shape(int n, PlanShape* out);

// Relative error of the factor m (1, t) by which a butterfly multiplies for e^{i pi a / 16}, a = 1..4
// (the larger of cosine and sine, and their ratio, both rounded to float), along the true value.
constexpr double twiddle_gain(int a) {
  constexpr double c[5] = {1.0, 0.98078528040323044913, 0.92387953251128675613, 0.83146961230254523708,
                           0.70710678118654752440};
  constexpr double s[5] = {0.0, 0.19509032201612826785, 0.38268343236508977173, 0.55557023301960222474,
                           0.70710678118654752440};
  const double m = static_cast<double>(static_cast<float>(c[a]));
  const double t = static_cast<double>(static_cast<float>(s[a] / c[a]));
  return m * (c[a] + t * s[a]) - 1.0;
}
// Relative gain of the in-register transform of length r (its power-of-two part, radix 2): every one of
// these constants rounds down, so that each stage shrinks the half of its energy that goes through its
// twiddles: -1.4e-8 for 16, -2.5e-8 for 32.
constexpr double dft_gain(int r) {
  r &= -r;
  double g = 0.0;
  for (int len = 8; len <= r; len *= 2) {
    double sum = 0.0;
    for (int j = 0; j < len / 2; ++j) {
      const int k = (j * (32 / len)) % 8;
      sum += twiddle_gain(k <= 4 ? k : 8 - k);
    }
    g += 0.5 * sum / (len / 2);
  }
  return g;
}
// The divisor of P's frequency factors for n = r0 m r0: n, times the transforms' gain for the lengths
// above 4096 (without the correction the two radix-32 passes of a transform put 1.1e-7 to 1.3e-7 of
// P's 2.2e-7 rms error into a plain factor).  Below, and with a split pass, P is as exact as it was
// before the three-pass path and its results keep their bits.
constexpr double p_divisor(int n, int r0, int m) {
  return (n > 4096 && m <= 32) ? n * (1.0 + 2.0 * (2.0 * dft_gain(r0) + dft_gain(m))) : n;
}

// Whether a shape (threads per workgroup, np radices) takes the three-pass path: n = r0 m r0, r0 even, one
// butterfly of the outer passes per thread.  The inverse runs the same radices on the same tables there
// and the frequency factors are addressed by the thread's own elements.
constexpr bool three_pass(int n, int threads, int np, const int* rad) {
  return np == 3 && rad[0] == rad[2] && rad[0] % 2 == 0 && threads >= n / rad[0];
}

// LDS layout of the generic path's transform buffer: element i of the vector lives at float2 slot
// i + (i >> kPadShift).
constexpr int kPadShift = 4;
constexpr int pad_slot(int i) { return i + (i >> kPadShift); }

bool supported_n(int n);
// Launch the pair kernel for vector length n; grid = number of work items (pairs or listed rows).
hipError_t launch_pair(int n, const KArgs& a, int64_t grid, hipStream_t stream);
hipError_t launch_cluster(const ClusterArgs& a, hipStream_t stream);

// Error-compensated quantisation (kashin_optq.hip).  optq_factor_device: U (upper, U^T U =
// (H + lambda I)^-1, lambda = damp mean(diag H)) and, if v != null, V = U^-1, both d x d float64
// row-major; allocates and frees its temporaries and synchronises `stream`; *info != 0 when the
// damped Hessian is not positive definite (> 0) or its factor singular (< 0).
hipError_t optq_factor_device(const float* h, int d, int64_t ldh, double damp, double* u, double* v,
                              hipStream_t stream, int* info);
constexpr int kOptqMaxChunk = 128;
int64_t optq_workspace_bytes(int64_t d_in, int n, int chunk);
// kashin_optq_quantize_noalloc's workspace: a static device array of this many bytes per device;
// optq_static_scratch gives its address on the current device
constexpr int64_t kOptqStaticScratchBytes = int64_t(16) << 20;
hipError_t optq_static_scratch(void** out);
hipError_t optq_error(const float* w, int64_t ldw, const float* q, int n, int64_t row0, int rows, const double* u,
                      int64_t ldu, float* e, hipStream_t s);
hipError_t optq_rank1(float* w, int64_t ldw, int n, int64_t i, int64_t j0, int64_t j1, const double* u, int64_t ldu,
                      const float* err, hipStream_t s);
hipError_t optq_chunk_factor(const double* u, const double* v, int64_t ld, int64_t c0, int rows, int64_t c1,
                             int64_t rest, bool exact, float* m, hipStream_t s);
hipError_t optq_update(float* w_rest, int64_t ldw, const float* m, const float* e, int rows, int64_t rest, int n,
                       hipStream_t s);

// Incoherence rotation of rows (kashin_rotate.hip).
bool rotate_supported_n(int n);
hipError_t launch_rotate(int n, uint64_t seed, bool inverse, const void* x, int dtype, int64_t ldx, float* y,
                         int64_t ldy, int64_t m, hipStream_t stream);

}  // namespace kashin
