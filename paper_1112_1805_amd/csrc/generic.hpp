// Row and column passes for image sizes that are not a power of two (N = 2^a * m with
// m's prime factors in {3, 5, 7, 11, 13, 17, 19, 23}), e.g. the 32 * {3..24} sizes of a
// batch of mixed images.  The data of a transform stays in LDS between stages; every stage
// of the mixed-radix Stockham FFT has a runtime radix from a small set, each with a
// compile-time butterfly: power-of-two radices use the register DFTs of fft.hpp, radix 9 a
// 3 x 3 split, odd primes the symmetric-pair form
//   X[k]   = a0 + sum_n (a_n + a_{P-n}) cos(2 pi n k/P) - i (a_n - a_{P-n}) sin(2 pi n k/P)
//   X[P-k] = a0 + sum_n (a_n + a_{P-n}) cos(2 pi n k/P) + i (a_n - a_{P-n}) sin(2 pi n k/P)
// (forward; the inverse swaps the signs of the sine terms).
#pragma once
#include "kernels.hpp"
#include "schedule.hpp"

namespace shs {

using PlanRef = const __attribute__((address_space(4))) FftPlan*;   // in constant memory

// ---------------------------------------------------------------- small DFTs
template <int P, bool INV>
__device__ __forceinline__ void dft_odd_prime(cpx (&a)[P]) {
  constexpr int H = (P - 1) / 2;
  cpx s[H], d[H];
  cpx sum = a[0];
  static_for<H>([&](auto i) {
    s[i] = a[i + 1] + a[P - 1 - i];
    d[i] = a[i + 1] - a[P - 1 - i];
    sum = sum + s[i];
  });
  const cpx a0 = a[0];
  a[0] = sum;
  static_for<H>([&](auto kk) {
    constexpr int k = kk + 1;
    cpx re = a0, im = cpx{0.f, 0.f};
    static_for<H>([&](auto i) {
      constexpr int n = i + 1;
      constexpr float c = float(cos2pi(n * k, P));
      constexpr float sn = float(sin2pi(n * k, P));
      re = cpx{fmaf(s[i].x, c, re.x), fmaf(s[i].y, c, re.y)};
      im = cpx{fmaf(d[i].x, sn, im.x), fmaf(d[i].y, sn, im.y)};
    });
    // forward: X[k] = re - i im, X[P-k] = re + i im
    const cpx t = INV ? mul_i(im) : mul_mi(im);
    a[k] = re + t;
    a[P - k] = re - t;
  });
}

// Composite radices: they halve the trips through LDS of most sides (32 m needs two stages
// instead of three).  A * B with coprime factors by the Good-Thomas prime-factor map: input
// n = (B n1 + A n2) mod R, output k = (B (B^-1 mod A) k1 + A (A^-1 mod B) k2) mod R turn the
// DFT into an A x B two-dimensional one without twiddles (all index maps are compile-time).
constexpr int inv_mod(int a, int m) {
  for (int x = 1; x < m; ++x)
    if (a * x % m == 1) return x;
  return 1;
}
template <int R, bool INV>
__device__ __forceinline__ void dft_any(cpx (&a)[R]);
template <int A, int B, bool INV>
__device__ __forceinline__ void dft_pfa(cpx (&a)[A * B]) {
  constexpr int R = A * B, EA = B * inv_mod(B % A, A), EB = A * inv_mod(A % B, B);
  cpx y[A][B];
  static_for<A>([&](auto i) {
    static_for<B>([&](auto j) { y[i][j] = a[(B * i + A * j) % R]; });
    dft_any<B, INV>(y[i]);
  });
  static_for<B>([&](auto j) {
    cpx z[A];
    static_for<A>([&](auto i) { z[i] = y[i][j]; });
    dft_any<A, INV>(z);
    static_for<A>([&](auto i) { a[(EA * i + EB * j) % R] = z[i]; });
  });
}

template <int R, bool INV>
__device__ __forceinline__ void dft_any(cpx (&a)[R]) {
  if constexpr (R == 2 || R == 3 || R == 4 || R == 8 || R == 16 || R == 32) RegDFT<R, INV>::run(a);
  else if constexpr (R == 9) reg_dft_split<9, 3, 3, INV>(a);
  else if constexpr (R == 6) dft_pfa<2, 3, INV>(a);
  else if constexpr (R == 10) dft_pfa<2, 5, INV>(a);
  else if constexpr (R == 12) dft_pfa<4, 3, INV>(a);
  else if constexpr (R == 14) dft_pfa<2, 7, INV>(a);
  else if constexpr (R == 15) dft_pfa<3, 5, INV>(a);
  else if constexpr (R == 18) dft_pfa<2, 9, INV>(a);
  else if constexpr (R == 20) dft_pfa<4, 5, INV>(a);
  else if constexpr (R == 22) dft_pfa<2, 11, INV>(a);
  else if constexpr (R == 24) dft_pfa<8, 3, INV>(a);
  else dft_odd_prime<R, INV>(a);
}

template <class F>
__device__ __forceinline__ void with_radix(int r, F&& f) {
  switch (r) {
#define SHS_CASE(RR) \
    case RR: f(std::integral_constant<int, RR>{}); break;
    SHS_RADICES(SHS_CASE)
#undef SHS_CASE
    default: break;
  }
}

// ---------------------------------------------------------------- one Stockham stage
// `items` = 2^lw interleaved transforms x (L / R) butterflies, spread over nthr threads;
// item it is butterfly it >> lw of transform it mod 2^lw.
// `early(bf, c)` issues loads whose values only `done` needs; `load(a, bf, nb, c)` fills the
// inputs, a[i] = element bf + i nb (nb = L/R) of transform c; `done(a, ob, bf, c, e)` takes
// the R outputs, output i belonging to position ob + i Ns, and what `early` returned.  So a
// transform's first stage can read global memory and its last one can write there (or go on
// with the data in registers): in the last stage ob = bf and Ns = nb, so a butterfly's outputs
// are the positions of its inputs.  Loads are issued for the whole butterfly before any is
// used: a wave runs alone with its latencies where the GPU is not full.
// sw: stage twiddles of the whole transform in thread read order (LDS), W_{Ns R}^{i k} at
// sw[i Ns + k - 1] (1 <= i < R, k < Ns) for the stage of stride Ns and radix R; the stages'
// ranges [Ns - 1, Ns R - 1) tile [0, L - 1), and consecutive butterflies read consecutive
// entries.
struct StageGeom {
  int L, Ns;
  unsigned mag;
  int sh;
};
__device__ __forceinline__ StageGeom stage_geom(PlanRef pl, int s, int Ns) {
  return StageGeom{pl->L, Ns, pl->mag[s], pl->sh[s]};
}
// What `early` loaded, or (EARLY = false) what `now` loads.
template <bool EARLY, class E, class F>
__device__ __forceinline__ auto early_or(const E& e, F&& now) {
  if constexpr (EARLY) return e;
  else return now();
}
struct NoEarly {
  __device__ __forceinline__ int operator()(int, int) const { return 0; }
};
template <int R, bool INV, class Early, class Load, class Done>
__device__ __forceinline__ void gstage(const StageGeom& q, int lw, int nthr, int tid, const float2* sw, Early&& early,
                                       Load&& load, Done&& done) {
  const int nb = q.L / R;
  const int items = nb << lw;
  for (int it = tid; it < items; it += nthr) {
    const int c = it & ((1 << lw) - 1);
    const unsigned bf = unsigned(it) >> lw;
    unsigned g = bf;
    int k = 0;
    if (q.Ns > 1) {
      g = (__umulhi(bf, q.mag) + bf) >> q.sh;     // bf / Ns
      k = int(bf - g * unsigned(q.Ns));
    }
    const auto e = early(int(bf), c);
    cpx a[R];
    load(a, int(bf), nb, c);
    if (q.Ns > 1) {
      static_for<R - 1>([&](auto i1) {
        constexpr int i = i1 + 1;
        const cpx w = ld(sw + (i * q.Ns + k - 1));
        a[i] = INV ? cmulc(a[i], w) : cmul(a[i], w);
      });
    }
    dft_any<R, INV>(a);
    done(a, int(g) * q.Ns * R + k, int(bf), c, e);
  }
}

// Element accesses of LDS-resident data: position pos of transform c at buf[pos 2^lw + c].
struct LdsRead {
  const float2* buf;
  int lw;
  template <int R>
  __device__ __forceinline__ void operator()(cpx (&a)[R], int bf, int nb, int c) const {
    static_for<R>([&](auto i) { a[i] = ld(buf + (((bf + i * nb) << lw) + c)); });
  }
};
struct LdsWrite {
  float2* buf;
  int lw, Ns;
  template <int R>
  __device__ __forceinline__ void operator()(cpx (&a)[R], int ob, int, int c, int = 0) const {
    static_for<R>([&](auto i) { st(buf + (((ob + i * Ns) << lw) + c), a[i]); });
  }
};

// The stages [s0, s1) of a transform between LDS buffers, starting in `cur`; returns the
// buffer that holds the result (alt == cur is allowed where every stage is one pass of one
// wave, whose reads all precede its writes).  Ns: stride of stage s0 on entry, of s1 on exit.
template <bool INV, int SK>
__device__ __forceinline__ float2* gfft_stages(PlanRef pl, int s0, int s1, int& Ns, float2* cur, float2* alt,
                                               int lw, int nthr, int tid, const float2* sw) {
  for (int s = s0; s < s1; ++s) {
    const int r = pl->radix[s];
    const StageGeom q = stage_geom(pl, s, Ns);
    with_radix(r, [&](auto R) __attribute__((always_inline)) {
      gstage<R, INV>(q, lw, nthr, tid, sw, NoEarly{}, LdsRead{cur, lw}, LdsWrite{alt, lw, q.Ns});
    });
    fft_sync<SK>();
    float2* t = cur;
    cur = alt;
    alt = t;
    Ns *= r;
  }
  return cur;
}

// ---------------------------------------------------------------- generic geometry
constexpr int kGW = 4;          // strip width of the generic path
constexpr int kGLW = 2;         // its logarithm

// The launch parameters of the path.  The stage lists stay in device memory and are read
// through constant-memory (scalar) loads: they are indexed by a runtime stage number, for which
// the compiler would copy a by-value kernel argument to scratch memory and read it back from
// there before every stage (middle step at 360^2, q = 2: 37 us against 21 us).
enum { FFT_INV = 0, FFT_FWD = 1, FFT_COL = 2 };   // inverse rows, forward rows (reversed), columns
struct GenParams {
  const FftPlan* plans;   // [3]
  int n;
  int wpb;        // waves per row-pass block (1, 2 or 4; the block is 64 wpb threads)
  int lrw;        // log2 of the rows per wave
  int nbuf;       // LDS buffers per row-pass wave: 1 where every stage is one pass, else 2
  int lrb;        // middle step: log2 of the rows per block
  __device__ __forceinline__ PlanRef inv() const { return (PlanRef)(plans + FFT_INV); }
  __device__ __forceinline__ PlanRef fwd() const { return (PlanRef)(plans + FFT_FWD); }
  __device__ __forceinline__ PlanRef col() const { return (PlanRef)(plans + FFT_COL); }
};
// Twiddle table of a mixed-radix plan, one device array: [0, N) exp(-2 pi i m / N); then what
// a row pass copies, 3 N/2 entries (see row_tab_len); then the column transform's stage table
// (N entries).
__device__ __forceinline__ const float2* row_sw_g(const float2* tw, int n) { return tw + n; }
__device__ __forceinline__ const float2* col_sw_g(const float2* tw, int n) { return tw + n + 3 * (n / 2); }

// The kernels below keep their twiddles in LDS, at the start of the dynamic shared memory
// (loaded once per block): the mixed-radix stages read one table entry per twiddle, where
// loads from global memory would compete with the data for the vector-memory path.
//   row pass:     exp(-2 pi i k / N) for k <= N/2, then the two stage tables (N/2 - 1 each)
//   column pass:  the column FFT's stage table (N - 1 entries, padded to N)
// (row_tab_len and col_tab_len entries, schedule.hpp.)
__device__ __forceinline__ void load_table(float2* dst, const float2* __restrict__ src, int len) {
#pragma unroll 4
  for (int e = threadIdx.x; e < len; e += blockDim.x) dst[e] = src[e];   // loads of four entries in flight
}

// ---------------------------------------------------------------- generic row pass
// Same modes and data contract as k_row.  Each wave transforms 2^lrw rows at once, stored
// interleaved in LDS (bin k of row c at k 2^lrw + c), so that a stage's butterflies of all
// its rows share the wave's lanes.  A block holds gp.wpb waves: more rows per wave fill the
// lanes in stages with few butterflies (a large radix), fewer waves per block keep such
// blocks within their LDS share.
//
// The pass is bound by VALU issue and LDS traffic together, so the data stay in registers
// wherever one butterfly's outputs are another's inputs: the inverse transform's first stage
// reads the spectrum from global memory (with the real-FFT pre-processing), and its last
// stage, the state update and the forward transform's first stage are one butterfly, because
// the forward transform runs the same radices in reverse order (outputs and inputs of both
// are the positions bf + i M/R).  Measured with the column passes' like change, against every
// stage as a pass over LDS with power-of-two and prime radices: 32 images of 96..768, FP32
// state, 10.7 -> 7.4 ms per iteration; 360^2, q = 2, FP16, 143 -> 100 us; adjoint of five
// 736^2 images 632 -> 407 us.
__device__ __forceinline__ int tix_g(int ip, int row, int n) {
  return (ip >> 2) * (n * kGW) + row * kGW + (ip & (kGW - 1));     // floor for negative ip
}

// Inputs of a butterfly of the inverse row transform's first stage from a half spectrum:
// z[k] = s + i d W_N^{-k} with s = X[k] + conj(X[M-k]), d = X[k] - conj(X[M-k]), k = bf + i nb.
// load(k) returns X[k]; only the columns [cb, cb + pitch) exist, and whole chunks [i nb, i nb +
// nb) that miss them directly or mirrored are skipped.
template <int R, class Load>
__device__ __forceinline__ void real_pre(cpx (&a)[R], int bf, int nb, int M, int cb, int pitch, const float2* ltw,
                                         Load&& load) {
  const auto in_p = [&](int k0) { return k0 < cb + pitch && k0 + nb > cb; };
  const auto in_m = [&](int k0) { return k0 <= M - cb && k0 + nb > M - cb - pitch; };
  // in groups of 8 bins: their mirrored bins' registers bound the butterfly's footprint
  constexpr int H = 8;
  static_for<(R + H - 1) / H>([&](auto h) {
    constexpr int i0 = h * H, cnt = R - i0 < H ? R - i0 : H;
    cpx xm[H];
    static_for<cnt>([&](auto m) {
      constexpr int i = i0 + m;
      const int k = bf + i * nb;
      a[i] = cpx{0.f, 0.f};
      xm[m] = cpx{0.f, 0.f};
      if (in_p(i * nb)) a[i] = load(k);
      if (in_m(i * nb)) xm[m] = load(M - k);
    });
    static_for<cnt>([&](auto m) {
      constexpr int i = i0 + m;
      if (in_p(i * nb) || in_m(i * nb)) {
        const cpx s = a[i] + conj(xm[m]), d = a[i] - conj(xm[m]);
        const cpx w = ld(ltw + (bf + i * nb));   // W_N^k
        a[i] = cpx{fmaf(d.x, w.y, fmaf(-d.y, w.x, s.x)), fmaf(d.x, w.x, fmaf(d.y, w.y, s.y))};
      }
    });
  });
}
// Half spectra of the 2^lw rows whose forward transforms Y sit interleaved in LDS: bins k and
// M - k come from the same two points, X[k] = (s - i d W^k) / 2 and X[M-k] = conj(s + i d W^k) / 2
// with s = Y[k] + conj(Y[M-k]), d = Y[k] - conj(Y[M-k]).  hs: 1/2, or 1 where the rows were passed
// in halved.  store(c, k, x) takes bin k of row c.
template <class Store>
__device__ __forceinline__ void real_post(const float2* Y, int M, int lw, int lane, const float2* ltw, float hs,
                                          Store&& store) {
  const int items = (M / 2 + 1) << lw;
  for (int it = lane; it < items; it += 64) {
    const int c = it & ((1 << lw) - 1), k = it >> lw;
    const cpx yk = ld(Y + it);
    const cpx ym = conj(ld(Y + (((k == 0 ? 0 : M - k) << lw) + c)));
    const cpx s = yk + ym, d = yk - ym;
    const cpx e = mul_i(cmul(d, ld(ltw + k)));
    store(c, k, (s - e) * hs);
    store(c, M - k, conj(s + e) * hs);
  }
}

template <class Pair, int R> struct StatePairs { Pair v[R]; };
// Raw buffer view of one channel's state image; with `bytes` = 0 every load reads zero (a state
// that need not be read).  A branch per load in its place splits the butterfly into blocks that
// the scheduler cannot move loads between: the largest radices then kept their loaded pairs and
// the unfinished outputs live together, past the 128 registers of four waves per SIMD (92..108
// bytes of scratch per lane in the FP32 forms; none like this).  With the analysis pass's like
// change, per iteration: 768^2, q = 3, FP32 430 -> 413 us, q = 5, FP16 620 -> 586; 184^2, q = 2 73
// -> 67; sides of small radices within 1.5%.
template <class S> struct StateBuf {
  using Pair = typename S::Pair;
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ StateBuf(const void* base, int bytes)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), short(0), bytes, 0x00020000)) {}
  __device__ __forceinline__ Pair load_pair(int pair) const {
    const unsigned at = unsigned(pair) * unsigned(sizeof(Pair));
    if constexpr (sizeof(Pair) == 8) {
      const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, at, 0, 0);
      const unsigned lo = v[0], hi = v[1];
      return make_float2(__uint_as_float(lo), __uint_as_float(hi));
    } else {
      return __builtin_amdgcn_raw_buffer_load_b32(r, at, 0, 0);
    }
  }
};

template <int MODE, int ST, bool STATS>
__device__ __forceinline__ void row_g_body(const RowParams& p, const GenParams& gp, BlockId bid) {
  static_assert(kGW == 4, "tix_g assumes strips of 4 columns");
  using S = Store<ST>;
  extern __shared__ float2 gsm[];
  __shared__ double red[4 * 4];
  constexpr bool HALVED = MODE == ROW_SOLVE || MODE == ROW_PRIME;   // next adjoint input passed on halved
  const int n = gp.n, M = n / 2, lw = gp.lrw;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row0 = (bid.x * gp.wpb + wave) << lw;
  const int ch = bid.y;
  const int j = ch % p.eta;
  const int last = gp.inv()->ns - 1;
  float2* ltw = gsm;                     // exp(-2 pi i k / N), k <= M
  float2* isw = gsm + M + 1;             // inverse row transform's stage table
  float2* fsw = isw + M - 1;             // forward row transform's
  load_table(ltw, row_sw_g(p.tw, n), 3 * M - 1);
  float2* cur = gsm + row_tab_len(n) + ((wave * gp.nbuf * M) << lw);
  float2* alt = cur + (gp.nbuf == 2 ? (M << lw) : 0);
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  bool emit = true;
  if constexpr (MODE == ROW_SOLVE) emit = p.emit != 0;
  __syncthreads();

  const float th = p.fw.thr[j];
  const auto state = [&](int c) {
    return reinterpret_cast<typename S::T*>(p.g) + (long long)ch * n * n + (long long)(row0 + c) * n;
  };
  if constexpr (MODE == ROW_SOLVE || MODE == ROW_C2R || MODE == ROW_ENERGY || MODE == ROW_SHRINK || MODE == ROW_PD) {
    int cb, pitch;
    long long off;
    plane_geom(p.lin, ch % p.lin.nf, cb, pitch, off);
    const PlaneBuf B(p.spec_in + (ch / p.lin.nf) * p.lin.ls + off, pitch * n);
    const StateBuf<S> G(reinterpret_cast<const typename S::T*>(p.g) + (long long)ch * n * n,
                        p.fresh ? 0 : n * n * int(sizeof(typename S::T)));
    // first stage (bins outside the plane's columns are out-of-range buffer loads: zero)
    with_radix(gp.inv()->radix[0], [&](auto R) __attribute__((always_inline)) {
      gstage<R, true>(stage_geom(gp.inv(), 0, 1), lw, 64, lane, isw, NoEarly{}, [&](cpx (&a)[R], int bf, int nb, int c) {
        real_pre(a, bf, nb, M, cb, pitch, ltw, [&](int k) { return B.load(tix_g(k - cb, row0 + c, n)); });
      }, LdsWrite{cur, lw, 1});
    });
    fft_sync<SYNC_WAVE>();
    int Ns = gp.inv()->radix[0];
    float2* res = gfft_stages<true, SYNC_WAVE>(gp.inv(), 1, last, Ns, cur, alt, lw, 64, lane, isw);
    alt = res == cur ? alt : cur;
    cur = res;
    // last stage, update, and the forward transform's first stage
    with_radix(gp.inv()->radix[last], [&](auto R) __attribute__((always_inline)) {
      const int nb = M / R;
      // the state's pairs: loaded before the butterfly where its registers allow, else after it
      constexpr bool STATE = MODE == ROW_SOLVE || MODE == ROW_PD;
      constexpr bool EARLY = STATE && R * sizeof(typename S::Pair) <= 64;
      const auto load_state = [&](int bf, int c) {
        StatePairs<typename S::Pair, STATE ? int(R) : 1> e;
        const int at = (row0 + c) * M + bf;
        static_for<R>([&](auto i) { e.v[i] = G.load_pair(at + i * nb); });
        return e;
      };
      const auto early = [&](int bf, int c) {
        if constexpr (EARLY) return load_state(bf, c);
        else return 0;
      };
      gstage<R, true>(stage_geom(gp.inv(), last, Ns), lw, 64, lane, isw, early, LdsRead{cur, lw},
                      [&](cpx (&a)[R], int, int bf, int c, const auto& e0) {
        if constexpr (MODE == ROW_C2R) {
          float* out = p.real_out + ch * p.real_cs + (long long)(row0 + c) * n;
          static_for<R>([&](auto i) {
            *reinterpret_cast<float2*>(out + 2 * (bf + i * nb)) = make_float2(a[i].x, a[i].y);
          });
        }
        if constexpr (MODE == ROW_ENERGY) {
          static_for<R>([&](auto i) { acc[SLOT_L1] += fabsf(a[i].x) + fabsf(a[i].y); });
        }
        if constexpr (MODE == ROW_SOLVE) {
          typename S::T* g = state(c);
          const auto e = early_or<EARLY>(e0, [&] { return load_state(bf, c); });
          static_for<R>([&](auto i) {
            const int k = bf + i * nb;
            float g0, g1;
            S::unpack(e.v[i], g0, g1);
            const float b0v = clip(g0, th), b1v = clip(g1, th);
            // g <- clip(g) + S_j u  (v = shrink(g), b_v = clip(g); Section 3 v- and b_v-updates)
            float n0 = b0v + a[i].x, n1 = b1v + a[i].y;
            S::store_pair(g + 2 * k, S::round2(n0, n1));
            const float nb0 = clip(n0, th), nb1 = clip(n1, th);
            if constexpr (STATS) {
              const float dv0 = (n0 - nb0) - (g0 - b0v), dv1 = (n1 - nb1) - (g1 - b1v);
              const float db0 = nb0 - b0v, db1 = nb1 - b1v;
              acc[SLOT_DY2] = fmaf(dv0, dv0, acc[SLOT_DY2]);
              acc[SLOT_DY2] = fmaf(dv1, dv1, acc[SLOT_DY2]);
              acc[SLOT_DB2] = fmaf(db0, db0, acc[SLOT_DB2]);
              acc[SLOT_DB2] = fmaf(db1, db1, acc[SLOT_DB2]);
              acc[SLOT_L1] += fabsf(n0 - nb0);
              acc[SLOT_L1] += fabsf(n1 - nb1);
            }
            a[i] = cpx{fmaf(0.5f, n0, -nb0), fmaf(0.5f, n1, -nb1)};
          });
          // complete the residual sums here: sunk past the next butterfly they would keep
          // every per-pixel term live
          if constexpr (STATS) __asm__ volatile("" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[3]));
        }
        if constexpr (MODE == ROW_PD) {
          // dual step of the primal-dual iteration: y <- clip(y + sigma c, +-lambda_j), c = (K ubar)_j
          typename S::T* g = state(c);
          const auto e = early_or<EARLY>(e0, [&] { return load_state(bf, c); });
          static_for<R>([&](auto i) {
            const int k = bf + i * nb;
            float y0, y1;
            S::unpack(e.v[i], y0, y1);
            float n0 = clip(fmaf(p.sigma, a[i].x, y0), th);
            float n1 = clip(fmaf(p.sigma, a[i].y, y1), th);
            S::store_pair(g + 2 * k, S::round2(n0, n1));
            if constexpr (STATS) {
              const float d0 = n0 - y0, d1 = n1 - y1;
              acc[SLOT_DY2] += d0 * d0 + d1 * d1;
              acc[SLOT_L1] += fabsf(a[i].x) + fabsf(a[i].y);
            }
            a[i] = cpx{n0, n1};
          });
          if constexpr (STATS) __asm__ volatile("" : "+v"(acc[0]), "+v"(acc[3]));
        }
        if constexpr (MODE == ROW_SHRINK) {
          static_for<R>([&](auto i) { a[i] = cpx{a[i].x - clip(a[i].x, th), a[i].y - clip(a[i].y, th)}; });
        }
        if constexpr (MODE == ROW_SOLVE || MODE == ROW_PD || MODE == ROW_SHRINK) {
          if (emit) {
            dft_any<R, false>(a);
            LdsWrite{alt, lw, 1}(a, bf * R, bf, c);
          }
        }
      });
    });
  }
  if constexpr (MODE == ROW_C2R) return;
  if constexpr (MODE == ROW_R2C || MODE == ROW_PRIME) {
    with_radix(gp.fwd()->radix[0], [&](auto R) __attribute__((always_inline)) {
      gstage<R, false>(stage_geom(gp.fwd(), 0, 1), lw, 64, lane, fsw, NoEarly{}, [&](cpx (&a)[R], int bf, int nb, int c) {
        if constexpr (MODE == ROW_R2C) {
          const float* in = p.real_in + ch * p.real_cs + (long long)(row0 + c) * n;
          static_for<R>([&](auto i) { a[i] = ld(reinterpret_cast<const float2*>(in + 2 * (bf + i * nb))); });
        } else {
          const typename S::T* g = state(c);
          static_for<R>([&](auto i) {
            float g0, g1;
            S::unpack(S::load_pair(g + 2 * (bf + i * nb)), g0, g1);
            a[i] = cpx{fmaf(0.5f, g0, -clip(g0, th)), fmaf(0.5f, g1, -clip(g1, th))};
          });
        }
      }, LdsWrite{alt, lw, 1});
    });
  }
  if constexpr (MODE != ROW_ENERGY) {
    if (emit) {
      fft_sync<SYNC_WAVE>();
      int Ns = gp.fwd()->radix[0];
      const float2* Y = gfft_stages<false, SYNC_WAVE>(gp.fwd(), 1, last + 1, Ns, alt, cur, lw, 64, lane, fsw);
      int cb, pitch;
      long long off;
      plane_geom(p.lout, ch % p.lout.nf, cb, pitch, off);
      const PlaneBuf B(p.spec_out + (ch / p.lout.nf) * p.lout.ls + off, pitch * n);
      real_post(Y, M, lw, lane, ltw, HALVED ? 1.f : 0.5f, [&](int c, int k, cpx x) {
        B.store(tix_g(k - cb, row0 + c, n), x);      // outside the plane's columns: dropped
      });
    }
  }
  if constexpr (STATS) {
    double dd[4] = {double(acc[0]), double(acc[1]), double(acc[2]), double(acc[3])};
    dd[SLOT_L1] *= double(p.fw.lam[j]);
    block_sum4_n(dd, red, gp.wpb);
    if (threadIdx.x == 0) {
      double* o = p.partials + ((long long)bid.y * bid.gx + bid.x) * 4;
      o[0] = dd[0]; o[1] = dd[1]; o[2] = dd[2]; o[3] = dd[3];
    }
  }
}

template <int MODE, int ST, bool STATS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_row_g(RowParams p, GenParams gp) {
  row_g_body<MODE, ST, STATS>(p, gp, own_block());
}

// ---------------------------------------------------------------- generic middle step
// As mid_body: slot l RB + r is row r of label l, a wave transforms 2^lrw slots at a time.
// Dynamic LDS: the twiddle tables, the slots' rows (2^lrw interleaved), and with two buffers
// one more per wave.
template <int MODE, bool STATS>
__device__ __forceinline__ void mid_g_body(const MidParams& p, const GenParams& gp, BlockId bid) {
  extern __shared__ float2 gsm[];
  __shared__ double red[16 * 4];
  const int n = gp.n, M = n / 2, lw = gp.lrw, lrb = gp.lrb, RB = 1 << lrb;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int row0 = xcd_chunked(bid.x, bid.gx) * RB, groups = (RB * p.q) >> lw;
  float2* ltw = gsm;                     // as in the row pass
  float2* isw = gsm + M + 1;
  float2* fsw = isw + M - 1;
  float2* res = gsm + row_tab_len(n);
  float2* alt = res + ((groups * M) << lw) + ((wave * M) << lw);   // two buffers only
  load_table(ltw, row_sw_g(p.tw, n), 3 * M - 1);
  __syncthreads();
  if (p.z) {
    const PlaneBuf B(p.z, p.q * n * p.P);
    for (int g = wave; g < groups; g += nw) {
      float2* r = res + ((g * M) << lw);
      // the transform's result lands in r: start there or in the second buffer by its parity
      float2* a0 = gp.nbuf == 1 || gp.inv()->ns % 2 == 1 ? r : alt;
      float2* a1 = gp.nbuf == 1 ? r : (a0 == r ? alt : r);
      with_radix(gp.inv()->radix[0], [&](auto R) __attribute__((always_inline)) {
        gstage<R, true>(stage_geom(gp.inv(), 0, 1), lw, 64, lane, isw, NoEarly{}, [&](cpx (&a)[R], int bf, int nb, int c) {
          const int s = (g << lw) + c, l = s >> lrb;
          const int base = l * n * p.P, row = row0 + (s & (RB - 1));
          real_pre(a, bf, nb, M, 0, p.P, ltw, [&](int k) { return B.load(base + tix_g(k, row, n)); });
        }, LdsWrite{a0, lw, 1});
      });
      fft_sync<SYNC_WAVE>();
      int Ns = gp.inv()->radix[0];
      gfft_stages<true, SYNC_WAVE>(gp.inv(), 1, gp.inv()->ns, Ns, a0, a1, lw, 64, lane, isw);
    }
  }
  __syncthreads();
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  pixel_rows_q<MODE, STATS>(p, row0, RB, n, blockDim.x, acc, [&](int l, int r, int k) {
    const int s = (l << lrb) + r;
    return res + ((((s >> lw) * M + k) << lw) + (s & ((1 << lw) - 1)));
  });
  __syncthreads();
  if (p.emit) {
    const PlaneBuf B(p.v, p.q * n * p.P);
    for (int g = wave; g < groups; g += nw) {
      float2* r = res + ((g * M) << lw);
      int Ns = 1;
      const float2* Y = gfft_stages<false, SYNC_WAVE>(gp.fwd(), 0, gp.fwd()->ns, Ns, r, gp.nbuf == 1 ? r : alt, lw, 64, lane, fsw);
      real_post(Y, M, lw, lane, ltw, 0.5f, [&](int c, int k, cpx x) {
        const int s = (g << lw) + c, l = s >> lrb;
        B.store(l * n * p.P + tix_g(k, row0 + (s & (RB - 1)), n), x);
      });
      fft_sync<SYNC_WAVE>();   // the next group's second buffer is this one's
    }
  }
  if constexpr (STATS) mid_partials(p, acc, red, nw, bid);
}
template <int MODE, bool STATS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void k_mid_g(MidParams p, GenParams gp) {
  mid_g_body<MODE, STATS>(p, gp, own_block());
}

}  // namespace shs
