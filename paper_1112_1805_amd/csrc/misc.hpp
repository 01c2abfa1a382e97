// Small kernels launched by the host code only: filter bank and its windows (plan creation),
// data term, energy dot product, epilogue and reductions.
#pragma once
#include "kernels.hpp"

namespace shs {

// ---------------------------------------------------------------- filter bank (FP64)
// Meyer building blocks of Section 2 (eq. (psi1_psi2), the auxiliary polynomial v, the
// profile b and the scaling-function profile), evaluated in double precision.
__device__ __forceinline__ double mey_v(double x) {
  if (x < 0.0) return 0.0;
  if (x > 1.0) return 1.0;
  const double x2 = x * x;
  return x2 * x2 * (35.0 + x * (-84.0 + x * (70.0 - 20.0 * x)));
}
__device__ __forceinline__ double mey_b(double x) {
  const double a = fabs(x);
  if (a >= 1.0 && a <= 2.0) return sin(0.5 * M_PI * mey_v(a - 1.0));
  if (a > 2.0 && a <= 4.0) return cos(0.5 * M_PI * mey_v(0.5 * a - 1.0));
  return 0.0;
}
__device__ __forceinline__ double mey_psi1(double w) {
  const double b2 = mey_b(2.0 * w), b1 = mey_b(w);
  return sqrt(b2 * b2 + b1 * b1);
}
__device__ __forceinline__ double mey_psi2(double w) { return w <= 0.0 ? sqrt(mey_v(1.0 + w)) : sqrt(mey_v(1.0 - w)); }
__device__ __forceinline__ double mey_phi(double w) {
  const double a = fabs(w);
  if (a <= 0.5) return 1.0;
  if (a < 1.0) return cos(0.5 * M_PI * mey_v(2.0 * a - 1.0));
  return 0.0;
}

// Decode filter index f (documented order) into kind (0 low, 1 h, 2 v, 3 seam), scale, shear.
__device__ __forceinline__ void decode_filter(int f, int& kind, int& j, int& k) {
  if (f == 0) { kind = 0; j = 0; k = 0; return; }
  int rem = f - 1;
  j = 0;
  while (rem >= (4 << j)) { rem -= (4 << j); ++j; }
  const int ns = (2 << j) - 1;      // shears per cone at scale j
  const int half = (1 << j) - 1;
  if (rem < ns) { kind = 1; k = rem - half; }
  else if (rem < 2 * ns) { kind = 2; k = rem - ns - half; }
  else { kind = 3; k = (rem == 2 * ns) ? -(1 << j) : (1 << j); }
}

// psi1(4^-j a) psi2(2^j b/a + k): the sheared, dilated shearlet of Section 2 (a != 0).
__device__ __forceinline__ double shear_val(double a, double b, int j, int k) {
  return mey_psi1(a / double(1 << (2 * j))) * mey_psi2(double(1 << j) * b / a + double(k));
}

// Filter value at integer frequencies (o1, o2) with xi = rho * omega.
static __device__ double filter_value(int kind, int j, int k, int o1, int o2, double rho) {
  const double x1 = rho * o1, x2 = rho * o2;
  const int a1 = o1 < 0 ? -o1 : o1, a2 = o2 < 0 ? -o2 : o2;
  if (kind == 0) return mey_phi(fmax(fabs(x1), fabs(x2)));
  double v = 0.0;
  if (kind != 2 && a2 < a1) v += shear_val(x1, x2, j, k);         // horizontal cone
  if (kind != 1 && a1 < a2) v += shear_val(x2, x1, j, k);         // vertical cone
  if (kind == 3 && a1 == a2 && a1 > 0) v += shear_val(x1, x2, j, k);  // seam line
  return v;
}

__device__ __forceinline__ int freq_of(int idx, int n) { return idx < (n + 1) / 2 ? idx : idx - n; }

// One thread per (filter, k0, k1) of the half spectrum (k1 <= N/2).
static __global__ void k_filter_gen(float* __restrict__ psi, int n, int J, int P, int eta) {
  const int half = n / 2 + 1;
  const long long total = (long long)eta * n * half;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int k1 = int(i % half);
  const int k0 = int((i / half) % n);
  const int f = int(i / ((long long)half * n));
  int kind, j, k;
  decode_filter(f, kind, j, k);
  const double rho = double(1 << (2 * J)) / double(n);
  const int o1 = freq_of(k0, n), o2 = freq_of(k1, n);
  double v = filter_value(kind, j, k, o1, o2, rho);
  if ((n % 2 == 0) && (k0 == n / 2 || k1 == n / 2)) {
    // Nyquist bins: energy-symmetrise with the mirror bin -omega (mod N).
    const int m0 = (n - k0) % n, m1 = (n - k1) % n;
    const double w = filter_value(kind, j, k, freq_of(m0, n), freq_of(m1, n), rho);
    v = sqrt(0.5 * (v * v + w * w));
  }
  psi[((long long)f * n + k0) * P + k1] = float(v);
}

// ---------------------------------------------------------------- data term
struct Codebook { float c[8 * 4]; };
// s[k][p] = sum_c |f[c][p] - cb[k][c]|^p (eq. (computationOfs), colour form of Section 4).
static __global__ void k_datacost(const float* __restrict__ img, int C, Codebook cb, int q, float pw,
                           float* __restrict__ s, long long n2) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n2) return;
  float f[4];
  for (int c = 0; c < C; ++c) f[c] = img[c * n2 + i];
  for (int k = 0; k < q; ++k) {
    float acc = 0.f;
    for (int c = 0; c < C; ++c) {
      const float d = f[c] - cb.c[k * 4 + c];
      acc += (pw == 2.0f) ? d * d : powf(fabsf(d), pw);
    }
    s[k * n2 + i] = acc;
  }
}

// ---------------------------------------------------------------- plan-time filter windows
// For filter j and column k1: the shortest circular interval of k0 holding every nonzero
// of the column (start a, length L; L = 0 for an all-zero column).
static __global__ void k_filter_windows(const float* __restrict__ psi, int n, int P, int eta, int2* __restrict__ win) {
  const int half = n / 2 + 1;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= eta * half) return;
  const int j = i / half, k1 = i % half;
  const float* col = psi + (long long)j * n * P + k1;
  int first = -1, last = -1, prev = -1, gap_best = -1, gap_end = 0;
  for (int k0 = 0; k0 < n; ++k0) {
    if (col[(long long)k0 * P] != 0.f) {
      if (first < 0) first = k0;
      if (prev >= 0 && k0 - prev - 1 > gap_best) { gap_best = k0 - prev - 1; gap_end = k0; }
      prev = k0;
      last = k0;
    }
  }
  if (first < 0) { win[i] = make_int2(0, 0); return; }
  const int wrap = first + n - last - 1;          // zero run across the end of the column
  if (wrap >= gap_best) win[i] = make_int2(first, last - first + 1);
  else win[i] = make_int2(gap_end, n - gap_best);
}

// Gathers the window values: psiw[off + r] = psi[j][(a + r) mod N][k1].
static __global__ void k_filter_compact(const float* __restrict__ psi, int n, int P, int eta, const int4* __restrict__ pwin,
                                 float* __restrict__ psiw) {
  const int half = n / 2 + 1;
  for (int i = blockIdx.y; i < eta * half; i += gridDim.y) {   // (j, k1) pair
    const int j = i / half, k1 = i % half;
    const int4 w = pwin[i];
    for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < w.y; r += gridDim.x * blockDim.x)
      psiw[w.z + r] = psi[((long long)j * n + ((w.x + r) % n)) * P + k1];
  }
}

// ---------------------------------------------------------------- solve tail
// <u, s> partial sums (energy), one per block.
static __global__ __launch_bounds__(256) void k_dot(const float* __restrict__ u, const float* __restrict__ s,
                                             long long n, double* partials) {
  __shared__ double red[4 * 4];
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256)
    acc[SLOT_WS] += double(u[i]) * double(s[i]);
  block_sum4<4>(acc, red);
  if (threadIdx.x == 0) {
    double* o = partials + (long long)blockIdx.x * 4;
    o[0] = acc[0]; o[1] = acc[1]; o[2] = acc[2]; o[3] = acc[3];
  }
}

// Relaxed labelling and label map: u* = w, label = first index of the largest entry.
static __global__ __launch_bounds__(256) void k_epilogue(const float* __restrict__ w, int q, long long n2,
                                                  float* __restrict__ u_out, int32_t* __restrict__ labels) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n2) return;
  float best = w[i];
  int arg = 0;
  if (u_out) u_out[i] = best;
  for (int l = 1; l < q; ++l) {
    const float v = w[l * n2 + i];
    if (u_out) u_out[l * n2 + i] = v;
    if (v > best) { best = v; arg = l; }
  }
  if (labels) labels[i] = arg;
}

// ---------------------------------------------------------------- reductions
// Sums n partial rows of four in a fixed order, in one launch: block b sums rows [b*per,
// min((b+1)*per, n)) and leaves its sums in red; the block that finishes last (counted in
// *done, which it sets back to zero) adds the blocks' sums in block order and writes
// totals[0..3], the history row (r_primal, r_dual, r_combined, surrogate energy) and a
// non-finite flag in totals[4].  With hist_ctr the row is hist_row + 4 * (*hist_ctr) and the
// counter advances by one, so one launch sequence (a captured graph) serves every iteration of
// a solve.  The sums travel between blocks by agent-scope atomics: blocks run on different
// XCDs, whose L2 caches are not coherent with each other.  A launch of few bytes is all
// latency: 3.2 + 2.6 us (128^2) and 4.8 + 4.7 us (1024^2, q = 5) as two launches, 3.4 and 8.6 us as
// one.
static __global__ __launch_bounds__(256) void k_reduce(const double* __restrict__ parts, long long n, long long per,
                                                       double* red_out, unsigned* done, double* __restrict__ totals,
                                                       double* __restrict__ hist_row, double gamma, int* hist_ctr) {
  __shared__ double red[4 * 4];
  __shared__ int last;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  const long long b0 = blockIdx.x * per, b1 = min(b0 + per, n);
  for (long long r = b0 + threadIdx.x; r < b1; r += 256) {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] += parts[r * 4 + i];
  }
  block_sum4<4>(acc, red);
  if (gridDim.x > 1) {
    if (threadIdx.x == 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        __hip_atomic_store(red_out + blockIdx.x * 4 + i, acc[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      last = __hip_atomic_fetch_add(done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    }
    __syncthreads();
    if (!last) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      acc[i] = threadIdx.x < gridDim.x
                   ? __hip_atomic_load(red_out + threadIdx.x * 4 + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                   : 0.0;
    }
    block_sum4<4>(acc, red);
    if (threadIdx.x == 0) __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (threadIdx.x == 0) {
    const double dy2 = acc[SLOT_DY2], db2 = acc[SLOT_DB2];
    totals[0] = acc[0]; totals[1] = acc[1]; totals[2] = acc[2]; totals[3] = acc[3];
    const double comb = dy2 + db2;
    totals[4] = (isfinite(comb) && isfinite(acc[2]) && isfinite(acc[3])) ? 0.0 : 1.0;
    if (hist_row && hist_ctr) hist_row += 4LL * (*hist_ctr)++;
    if (hist_row) {
      hist_row[0] = sqrt(db2);
      hist_row[1] = sqrt(dy2) / gamma;
      hist_row[2] = comb;
      hist_row[3] = acc[SLOT_WS] + acc[SLOT_L1];
    }
  }
}

static __global__ void k_fill_u32(uint32_t* __restrict__ p, long long n, uint32_t v) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

static __global__ void k_copy_f64(const double* __restrict__ src, int n, double* __restrict__ dst) {
  if (int(threadIdx.x) < n) dst[threadIdx.x] = src[threadIdx.x];
}

}  // namespace shs
