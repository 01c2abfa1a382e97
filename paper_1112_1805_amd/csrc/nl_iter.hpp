// Primal-dual iteration of the nonlocal model,  <u, s> + lambda sum_i ||(D u)(i)|| + iota_C(u)
// with D the difference operator of the neighbour graph (nl.hpp).
//
// Both steps gather from a pixel's neighbours, which lie anywhere in a 15 x 15 window.  What is
// gathered is stored as one record of all labels per pixel, so that a neighbour costs one
// vector load instead of one scalar load per label:
//   ubar  [pixel][q] float
//   y     [block][pixel][QP] storage type (QP = q, for 16-bit types rounded up to even so that
//         records are whole words; 12 bytes at q = 5)
// The dual step keeps its vector in registers between the norm and the projection (one pass
// over y) and leaves sum_b y_b per pixel, so the primal step reads of y only what it gathers;
// the neighbour and its block are one index.  At 512^2, q = 5, ten blocks, FP16: 62 + 50 us with
// label planes, 19 + 22 us with records.
#pragma once
#include "kernels.hpp"

namespace shs {

constexpr int kNlMaxBlocks = 16;

struct NlParams {
  void* y;              // dual variable, records (see above)
  float* u;             // primal u [q][n^2] (read, written)
  float* ubar;          // extrapolation, records (read by the dual step, written by the primal step)
  float* ysum;          // sum of a pixel's y over its blocks, records [pixel][q]
  const float* s;       // data term [q][n^2]
  const int32_t* nbr;   // [M2][n^2]
  const int32_t* rev;   // [M2][n^2]
  int32_t* src;         // [M2][n^2] record index rev * n^2 + nbr of the neighbour's entry, -1 without
  double* partials;     // [blocks][4]
  long long n2;
  int q, M2;
  float lambda, tau, sigma;
  int fresh;            // y and ubar are zero and need not be read
  int stats;
};

// Records of Q FP32 values, and of Q values of a storage type padded to QP.
template <int Q> struct NlVec { float v[Q]; };
template <int Q>
__device__ __forceinline__ NlVec<Q> nl_load(const float* p) {
  NlVec<Q> r;
  static_for<Q>([&](auto l) { r.v[l] = p[l]; });
  return r;
}
template <int ST, int Q> constexpr int nl_pad() { return ST == ST_F32 || Q == 1 ? Q : (Q + 1) / 2 * 2; }
template <int ST, int Q>
__device__ __forceinline__ NlVec<Q> nl_load_y(const void* y, long long rec) {
  using S = Store<ST>;
  constexpr int QP = nl_pad<ST, Q>();
  NlVec<Q> r;
  if constexpr (ST == ST_F32 || Q == 1) {
    const typename S::T* p = reinterpret_cast<const typename S::T*>(y) + rec * QP;
    static_for<Q>([&](auto l) { r.v[l] = S::to_float(p[l]); });
  } else {
    const uint32_t* p = reinterpret_cast<const uint32_t*>(y) + rec * (QP / 2);
    uint32_t w[QP / 2];
    static_for<QP / 2>([&](auto h) { w[h] = p[h]; });
    static_for<QP / 2>([&](auto h) {
      float a, b;
      S::unpack(w[h], a, b);
      r.v[2 * h] = a;
      if constexpr (2 * h + 1 < Q) r.v[2 * h + 1] = b;
    });
  }
  return r;
}
// Stores a record; on return `r` holds the stored (rounded) values.
template <int ST, int Q>
__device__ __forceinline__ void nl_store_y(void* y, long long rec, NlVec<Q>& r) {
  using S = Store<ST>;
  constexpr int QP = nl_pad<ST, Q>();
  if constexpr (ST == ST_F32 || Q == 1) {
    typename S::T* p = reinterpret_cast<typename S::T*>(y) + rec * QP;
    static_for<Q>([&](auto l) {
      p[l] = S::from_float(r.v[l]);
      r.v[l] = S::round(r.v[l]);
    });
  } else {
    uint32_t* p = reinterpret_cast<uint32_t*>(y) + rec * (QP / 2);
    static_for<QP / 2>([&](auto h) {
      float a = r.v[2 * h], b = 0.f;
      if constexpr (2 * h + 1 < Q) b = r.v[2 * h + 1];
      p[h] = S::round2(a, b);
      r.v[2 * h] = a;
      if constexpr (2 * h + 1 < Q) r.v[2 * h + 1] = b;
    });
  }
}

// src = the record of y that a pixel's neighbour holds for it (once per solve).
static __global__ __launch_bounds__(256) void k_nl_index(NlParams p) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= p.n2) return;
  for (int b = 0; b < p.M2; ++b) {
    const int j = p.nbr[b * p.n2 + i];
    p.src[b * p.n2 + i] = j >= 0 ? int(p.rev[b * p.n2 + i] * p.n2) + j : -1;
  }
}

__device__ __forceinline__ void nl_partials(const NlParams& p, double (&acc)[4], double* red, int block) {
  block_sum4<4>(acc, red);
  if (threadIdx.x == 0) {
    double* o = p.partials + (long long)block * 4;
    o[0] = acc[0]; o[1] = acc[1]; o[2] = acc[2]; o[3] = acc[3];
  }
}

// y <- P_ball(y + sigma D ubar) per pixel over (label, block), radius lambda.  Partials:
// ||y' - y||^2 and lambda ||(D ubar)(i)||.  B: the most blocks this instance takes; its Q B
// values stay in registers where that is at most 80 of them, else the second pass forms them
// again.
template <int ST, int Q, int B>
__global__ __launch_bounds__(256) void k_nl_dual(NlParams p) {
  __shared__ double red[4 * 4];
  constexpr bool KEEP = Q * B <= 80;
  const int blk = xcd_chunked(blockIdx.x, gridDim.x);
  const long long i = (long long)blk * 256 + threadIdx.x;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  if (i < p.n2) {
    int nj[B];
    static_for<B>([&](auto b) {
      nj[b] = -1;
      if (b < p.M2) nj[b] = p.nbr[b * p.n2 + i];
    });
    NlVec<Q> ui{};
    if (!p.fresh) ui = nl_load<Q>(p.ubar + i * Q);
    // a missing neighbour stands for the pixel itself: its difference is zero
    const auto diff = [&](int b, int j) {
      NlVec<Q> z{};
      if (!p.fresh) {
        z = nl_load<Q>(p.ubar + (j >= 0 ? (long long)j : i) * Q);
        static_for<Q>([&](auto l) { z.v[l] -= ui.v[l]; });
      }
      return z;
    };
    const auto old = [&](int b) {
      NlVec<Q> y{};
      if (!p.fresh) y = nl_load_y<ST, Q>(p.y, b * p.n2 + i);
      return y;
    };
    NlVec<Q> v[KEEP ? B : 1];
    float nn = 0.f, kk = 0.f;
    static_for<B>([&](auto b) {
      if (b < p.M2) {
        const NlVec<Q> z = diff(b, nj[b]), y = old(b);
        NlVec<Q> t;
        static_for<Q>([&](auto l) {
          t.v[l] = fmaf(p.sigma, z.v[l], y.v[l]);
          nn = fmaf(t.v[l], t.v[l], nn);
          kk = fmaf(z.v[l], z.v[l], kk);
        });
        if constexpr (KEEP) v[b] = t;
      }
    });
    const float sc = nn > p.lambda * p.lambda ? p.lambda * rsqrtf(nn) : 1.f;
    float d2 = 0.f;
    NlVec<Q> sum{};
    static_for<B>([&](auto b) {
      if (b < p.M2) {
        NlVec<Q> t, y{};
        if constexpr (KEEP) {
          t = v[b];
          if (p.stats) y = old(b);
        } else {
          const NlVec<Q> z = diff(b, nj[b]);
          y = old(b);
          static_for<Q>([&](auto l) { t.v[l] = fmaf(p.sigma, z.v[l], y.v[l]); });
        }
        static_for<Q>([&](auto l) { t.v[l] *= sc; });
        nl_store_y<ST, Q>(p.y, b * p.n2 + i, t);
        static_for<Q>([&](auto l) {
          sum.v[l] += t.v[l];
          d2 = fmaf(t.v[l] - y.v[l], t.v[l] - y.v[l], d2);
        });
      }
    });
    static_for<Q>([&](auto l) { p.ysum[i * Q + l] = sum.v[l]; });
    acc[SLOT_DY2] = d2;
    acc[SLOT_L1] = double(p.lambda) * sqrt(double(kk));
  }
  if (p.stats) nl_partials(p, acc, red, blk);
}

// u' = P_C(u - tau (D^T y + s)), ubar = 2 u' - u, with
// (D^T y)(j) = sum_c [j has a c-th neighbour i] y_{rev_c(j)}(i) - sum_c y_c(j).
template <int ST, int Q, int B>
__global__ __launch_bounds__(256) void k_nl_primal(NlParams p) {
  __shared__ double red[4 * 4];
  const int blk = xcd_chunked(blockIdx.x, gridDim.x);
  const long long j = (long long)blk * 256 + threadIdx.x;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  if (j < p.n2) {
    int src[B];
    static_for<B>([&](auto c) {
      src[c] = -1;
      if (c < p.M2) src[c] = p.src[c * p.n2 + j];
    });
    float un[Q], uo[Q], sv[Q];
    static_for<Q>([&](auto l) {
      uo[l] = p.u[l * p.n2 + j];
      sv[l] = p.s[l * p.n2 + j];
    });
    const NlVec<Q> own = nl_load<Q>(p.ysum + j * Q);
    NlVec<Q> kt{};
    static_for<B>([&](auto c) {
      if (c < p.M2) {
        const NlVec<Q> y = nl_load_y<ST, Q>(p.y, src[c] >= 0 ? (long long)src[c] : j);
        static_for<Q>([&](auto l) { kt.v[l] += src[c] >= 0 ? y.v[l] : 0.f; });
      }
    });
    static_for<Q>([&](auto l) { un[l] = uo[l] - p.tau * ((kt.v[l] - own.v[l]) + sv[l]); });
    simplex_project<Q>(un, Q);
    static_for<Q>([&](auto l) {
      p.u[l * p.n2 + j] = un[l];
      p.ubar[j * Q + l] = 2.f * un[l] - uo[l];
      const float du = un[l] - uo[l];
      acc[SLOT_DB2] += double(du) * du;
      acc[SLOT_WS] += double(un[l]) * double(sv[l]);
    });
  }
  if (p.stats) nl_partials(p, acc, red, blk);
}

// Energy partials of u: <u, s> and lambda sum_i (sum_{l, b} (D_b u_l)(i)^2)^(1/2), FP64.
static __global__ __launch_bounds__(256) void k_nl_energy(NlParams p) {
  __shared__ double red[4 * 4];
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  if (i < p.n2) {
    double nn = 0.0;
    for (int l = 0; l < p.q; ++l) {
      const float* u = p.u + l * p.n2;
      const double ui = u[i];
      acc[SLOT_WS] += ui * double(p.s[l * p.n2 + i]);
      for (int b = 0; b < p.M2; ++b) {
        const int jb = p.nbr[b * p.n2 + i];
        if (jb >= 0) {
          const double d = double(u[jb]) - ui;
          nn += d * d;
        }
      }
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
