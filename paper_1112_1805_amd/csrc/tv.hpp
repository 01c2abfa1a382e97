// TV comparison model of Section 4 (labels coupled per pixel), solved by the ADMM of
// Section 3 with the periodic forward-difference gradient in place of S:
//   u   = (I + grad^T grad)^{-1} [grad^T (v - b_v) + (w - b_w) - gamma s]
//   v   = shrink_{gamma lambda}(b_v + grad u)   (isotropic over the 2q-vector of a pixel)
//   w   = P_C(b_w + u),  b_v, b_w as in Section 3.
// The state keeps g = b_v + grad u ([q][2][N][N]) as for the shearlet model: with P the
// projection onto the ball of radius gamma lambda, v = g - P(g), b_v = P(g), and
// v - b_v = g - 2 P(g).  The u-step runs on the DFT: grad^T grad has the eigenvalues
// e(k0) + e(k1), e(k) = 4 sin^2(pi k / N).
#pragma once
#include "kernels.hpp"

namespace shs {

constexpr int kTvMaxLabels = 8;

struct TvParams {
  void* g;            // state g [q][2][N][N] (rhs: read; update: read and written)
  float* b;           // ball scale of every pixel's g (rhs, update: read; update: written) [N^2]
  float* w;           // [q][N^2] (update: read with statistics, written when write_w)
  float* bw;          // [q][N^2]
  float* t;           // w - b_w, what the next right-hand side needs of the two [q][N^2]
  const float* s;     // [q][N^2]
  const float* u;     // u [q][N^2] (update: read)
  float* rhs;         // [q][N^2] (rhs: written)
  double* partials;   // [blocks][4]
  int n, q;
  float gamma, radius, lambda;   // radius = gamma * lambda
  int fresh;          // first iteration: g = w = b_w = 0 and need not be read
  int write_w;        // update: w is needed after this iteration (its statistics or the result)
};

// Scale of the ball projection of a 2q-vector with squared norm nn: P(x) = x min(1, r/|x|).
__device__ __forceinline__ float ball_scale(float nn, float r) {
  return nn > r * r ? r * rsqrtf(nn) : 1.f;
}

// Both kernels below move bytes and little else: a thread takes two adjacent pixels (vector
// loads), all arrays are indexed by compile-time label counts, and each array is read once:
// the update leaves the ball scale b of every pixel and t = w - b_w, so the right-hand side
// reads of the state only the components its stencil needs at each of the three pixels, and
// the update reads s and w with statistics only and writes w only where it is asked for.  At 1024^2, q = 5,
// FP16: 31 + 33 us with one pixel per thread, the norms formed again at all three pixels and w,
// b_w, s read by both; 13 + 21 us like this.
constexpr int kTvPerBlock = 512;   // pixels

// A pair of pixels of an FP32 image.
__device__ __forceinline__ float2 ld2(const float* p) { return *reinterpret_cast<const float2*>(p); }
__device__ __forceinline__ void st2(float* p, float a, float b) { *reinterpret_cast<float2*>(p) = make_float2(a, b); }

// rhs_l = grad^T d_l + (w - b_w)_l - gamma s_l with d = g - 2 P(g) = (1 - 2 b) g per pixel:
// (grad^T d)(r, c) = d_0(r-1, c) - d_0(r, c) + d_1(r, c-1) - d_1(r, c)  (periodic).
template <int ST, int Q>
__global__ __launch_bounds__(256) void k_tv_rhs(TvParams p) {
  using S = Store<ST>;
  const int n = p.n, n2 = n * n;
  const int i = xcd_chunked(blockIdx.x, gridDim.x) * kTvPerBlock + 2 * int(threadIdx.x);
  if (i >= n2) return;
  const int r = i / n, c = i - r * n;
  if (p.fresh) {
    static_for<Q>([&](auto l) {
      const float2 s = load2_any(p.s + (long long)l * n2 + i);
      st2(p.rhs + (long long)l * n2 + i, -p.gamma * s.x, -p.gamma * s.y);
    });
    return;
  }
  const int iu = (r == 0 ? n - 1 : r - 1) * n + c;   // (r-1, c)
  const int il = r * n + (c == 0 ? n - 1 : c - 1);   // (r, c-1)
  const typename S::T* g = reinterpret_cast<const typename S::T*>(p.g);
  typename S::Pair x0[Q], x1[Q], xu[Q];
  typename S::T xl[Q];
  float2 tt[Q], sv[Q];
  static_for<Q>([&](auto l) {
    const typename S::T* a = g + (long long)(2 * l) * n2;
    x0[l] = S::load_pair(a + i);
    xu[l] = S::load_pair(a + iu);
    x1[l] = S::load_pair(a + n2 + i);
    xl[l] = a[n2 + il];
    tt[l] = ld2(p.t + (long long)l * n2 + i);
    sv[l] = load2_any(p.s + (long long)l * n2 + i);
  });
  const float2 b = ld2(p.b + i), bu = ld2(p.b + iu);
  const float m0 = 1.f - 2.f * b.x, m1 = 1.f - 2.f * b.y;
  const float mu0 = 1.f - 2.f * bu.x, mu1 = 1.f - 2.f * bu.y;
  const float ml = 1.f - 2.f * p.b[il];
  static_for<Q>([&](auto l) {
    float a0, a1, c0, c1, u0, u1;
    S::unpack(x0[l], a0, a1);
    S::unpack(x1[l], c0, c1);
    S::unpack(xu[l], u0, u1);
    // (the second pixel's left product is kept apart from the first pixel's right one, which it
    // equals: shared, the two pixels' sums would be contracted into different FMAs)
    float cl = c0;
    __asm__ volatile("" : "+v"(cl));
    const float d0 = (mu0 * u0 - m0 * a0) + (ml * S::to_float(xl[l]) - m0 * c0);
    const float d1 = (mu1 * u1 - m1 * a1) + (m0 * cl - m1 * c1);
    st2(p.rhs + (long long)l * n2 + i, d0 + tt[l].x - p.gamma * sv[l].x, d1 + tt[l].y - p.gamma * sv[l].y);
  });
}

// g <- P(g) + grad u (the v / b_v update), w = P_C(b_w + u), b_w += u - w, and the
// residual partials (||v' - v||^2 + ||w' - w||^2, ||b' - b||^2, <w', s>, lambda sum |v'|).
template <int ST, int Q, bool STATS>
__global__ __launch_bounds__(256) void k_tv_update(TvParams p) {
  using S = Store<ST>;
  __shared__ double red[4 * 4];
  const int n = p.n, n2 = n * n;
  const int blk = xcd_chunked(blockIdx.x, gridDim.x);
  const int i = blk * kTvPerBlock + 2 * int(threadIdx.x);
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  if (i < n2) {
    const int r = i / n, c = i - r * n;
    const int id = (r == n - 1 ? 0 : r + 1) * n + c;            // (r+1, c)
    const int ir = r * n + (c + 2 == n ? 0 : c + 2);            // (r, c+2), right of the pair
    typename S::T* g = reinterpret_cast<typename S::T*>(p.g);
    typename S::Pair xp[2 * Q];
    float2 uc[Q], ud[Q], bo[Q], sv[Q], wo[Q];
    float ur[Q];
    float2 b = make_float2(0.f, 0.f);
    if (!p.fresh) b = ld2(p.b + i);
    static_for<Q>([&](auto l) {
      const long long o = (long long)l * n2;
      xp[2 * l] = xp[2 * l + 1] = typename S::Pair{};
      bo[l] = wo[l] = make_float2(0.f, 0.f);
      if (!p.fresh) {
        xp[2 * l] = S::load_pair(g + 2 * o + i);
        xp[2 * l + 1] = S::load_pair(g + 2 * o + n2 + i);
        bo[l] = ld2(p.bw + o + i);
        if constexpr (STATS) wo[l] = ld2(p.w + o + i);
      }
      uc[l] = ld2(p.u + o + i);
      ud[l] = ld2(p.u + o + id);
      ur[l] = p.u[o + ir];
      if constexpr (STATS) sv[l] = load2_any(p.s + o + i);
    });
    float mm0 = 0.f, mm1 = 0.f;
    float w0[Q], w1[Q], g0[Q], g1[Q];
    double dv = 0.0, dbv = 0.0;
    float xn[2 * Q][2];
    static_for<Q>([&](auto l) {
      const long long o = (long long)l * n2;
      static_for<2>([&](auto k) {
        float a0, a1;
        S::unpack(xp[2 * l + k], a0, a1);
        // down and right differences of the pair's two pixels
        // (each value is rounded to the storage type by itself: with FP16 one instruction with
        // the product and the sum)
        const typename S::T h0 = S::from_float(fmaf(b.x, a0, (k == 0 ? ud[l].x : uc[l].y) - uc[l].x));
        const typename S::T h1 = S::from_float(fmaf(b.y, a1, (k == 0 ? ud[l].y : ur[l]) - uc[l].y));
        const float n0 = S::to_float(h0), n1 = S::to_float(h1);
        if constexpr (ST == ST_F32) st2(reinterpret_cast<float*>(g) + (2 * l + k) * (long long)n2 + i, n0, n1);
        else S::store_pair(g + (2 * l + k) * (long long)n2 + i, uint32_t(h0) | (uint32_t(h1) << 16));
        mm0 = fmaf(n0, n0, mm0);
        mm1 = fmaf(n1, n1, mm1);
        if constexpr (STATS) {
          xn[2 * l + k][0] = n0;
          xn[2 * l + k][1] = n1;
        }
      });
      g0[l] = w0[l] = bo[l].x + uc[l].x;
      g1[l] = w1[l] = bo[l].y + uc[l].y;
    });
    simplex_project<Q>(w0, Q);
    simplex_project<Q>(w1, Q);
    const float b0 = ball_scale(mm0, p.radius), b1 = ball_scale(mm1, p.radius);
    st2(p.b + i, b0, b1);
    static_for<Q>([&](auto l) {
      const long long o = (long long)l * n2 + i;
      const float bn0 = g0[l] - w0[l], bn1 = g1[l] - w1[l];
      st2(p.bw + o, bn0, bn1);
      st2(p.t + o, w0[l] - bn0, w1[l] - bn1);
      if (p.write_w) st2(p.w + o, w0[l], w1[l]);
      if constexpr (STATS) {
        const float dw0 = w0[l] - wo[l].x, dw1 = w1[l] - wo[l].y, db0 = bn0 - bo[l].x, db1 = bn1 - bo[l].y;
        acc[SLOT_DY2] += double(dw0) * dw0 + double(dw1) * dw1;
        acc[SLOT_DB2] += double(db0) * db0 + double(db1) * db1;
        acc[SLOT_WS] += double(w0[l]) * double(sv[l].x) + double(w1[l]) * double(sv[l].y);
        // v = (1 - b) x, b_v = b x, for the old and the new state vector
        static_for<2>([&](auto k) {
          float a0, a1;
          S::unpack(xp[2 * l + k], a0, a1);
          const float n0 = xn[2 * l + k][0], n1 = xn[2 * l + k][1];
          const float e0 = (1.f - b0) * n0 - (1.f - b.x) * a0, e1 = (1.f - b1) * n1 - (1.f - b.y) * a1;
          const float f0 = b0 * n0 - b.x * a0, f1 = b1 * n1 - b.y * a1;
          dv += double(e0) * e0 + double(e1) * e1;
          dbv += double(f0) * f0 + double(f1) * f1;
        });
      }
    });
    if constexpr (STATS) {
      acc[SLOT_DY2] += dv;
      acc[SLOT_DB2] += dbv;
      acc[SLOT_L1] += double(p.lambda) * (double(1.f - b0) * sqrt(double(mm0)) + double(1.f - b1) * sqrt(double(mm1)));
    }
  }
  if constexpr (STATS) {
    block_sum4<4>(acc, red);
    if (threadIdx.x == 0) {
      double* o = p.partials + (long long)blk * 4;
      o[0] = acc[0]; o[1] = acc[1]; o[2] = acc[2]; o[3] = acc[3];
    }
  }
}

// Exact energy partials of w: <w, s> and lambda sum_pixels (sum_l |grad w_l|^2)^(1/2).
static __global__ __launch_bounds__(256) void k_tv_energy(TvParams p) {
  __shared__ double red[4 * 4];
  const long long n2 = (long long)p.n * p.n;
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  if (i < n2) {
    const int r = int(i / p.n), c = int(i - (long long)r * p.n);
    const long long id = (long long)(r == p.n - 1 ? 0 : r + 1) * p.n + c;
    const long long ir = (long long)r * p.n + (c == p.n - 1 ? 0 : c + 1);
    double nn = 0.0;
    for (int l = 0; l < p.q; ++l) {
      const long long o = l * n2;
      const double wc = p.w[o + i];
      const double d0 = double(p.w[o + id]) - wc, d1 = double(p.w[o + ir]) - wc;
      nn += d0 * d0 + d1 * d1;
      acc[SLOT_WS] += wc * double(p.s[o + i]);
    }
    acc[SLOT_L1] = double(p.lambda) * sqrt(nn);
  }
  block_sum4<4>(acc, red);
  if (threadIdx.x == 0) {
    double* o = p.partials + (long long)blockIdx.x * 4;
    o[0] = acc[0]; o[1] = acc[1]; o[2] = acc[2]; o[3] = acc[3];
  }
}

}  // namespace shs
