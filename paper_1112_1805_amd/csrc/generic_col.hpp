// Column passes of the mixed-radix path (runtime N): single-image and grouped kernels, and
// the TV model's column solve.
//
// One strip (kGW columns) per block; a strip's N x kGW bins are one contiguous block in
// memory and in LDS (bin (k0, c) at k0 * kGW + c).  A transform's first stage takes its
// inputs from where they are (global memory, or the strip's spectrum times the filter) and
// its last stage hands its outputs on (to global memory, or into the accumulator), so LDS
// holds the data only between stages and a two-stage transform needs one buffer and two
// barriers.  The block is as wide as the stages have butterflies (col_g_threads): wider
// blocks would hold LDS for waves that only wait at barriers.
#pragma once
#include "mixed.hpp"

namespace shs {

// col_final: the summing of the partials wants many threads.  512 / 256 / 128 per block, per
// iteration: 360^2, q = 2 alone 102 / 104 / 109 us; in grouped launches 64 images 12.0 / 12.1 / 12.3 ms, 32
// images of 96..256 1.04 / 1.03 / 1.03, eight of 360^2 460 / 459 / 465 us.
constexpr int kFinalThreads = 512;

// Filter values psi_j(k0, k1) of one column window at k0 = bf + i nb: every value is one
// unconditional buffer load, out of range (zero) outside the window, so all are in flight
// together.
template <int R> struct PsiVals { float v[R]; };
template <int R>
__device__ __forceinline__ PsiVals<R> psi_load_g(const PsiBuf& pb, int4 win, int bf, int nb, int n) {
  PsiVals<R> o;
  static_for<R>([&](auto i) {
    int rel = bf + i * nb - win.x;
    if (rel < 0) rel += n;
    const unsigned at = rel < win.y ? unsigned(win.z + rel) * 4u : ~0u;
    o.v[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(pb.r, at, 0, 0));
  });
  return o;
}

// Plane geometry of the item's filter i, in scalar registers: the same for the whole block (read
// from LDS it counts as divergent, and every access through it became a loop over the lanes).
__device__ __forceinline__ int4 item_geo(const ItemStage<kGW>& stg, int i) {
  const int4 g = stg.geo[i];
  return make_int4(__builtin_amdgcn_readfirstlane(g.x), __builtin_amdgcn_readfirstlane(g.y),
                   __builtin_amdgcn_readfirstlane(g.z), __builtin_amdgcn_readfirstlane(g.w));
}

// A strip's transform between `load` (first stage: fills the butterfly's inputs) and `done`
// (last stage: outputs i at positions bf + i nb, with what `early` loaded); b0/b1: the LDS
// buffers of the stages between (b1 is used by transforms of more than two stages).  Ends
// without a barrier: the caller separates the last stage's reads from the next write to b0.
struct NoEarlyCol {
  template <class R>
  __device__ __forceinline__ int operator()(R, int, int, int) const { return 0; }
};
template <bool INV, class Early, class Load, class Done>
__device__ __forceinline__ void col_transform_g(const GenParams& gp, const float2* lsw, float2* b0, float2* b1,
                                                Early&& early, Load&& load, Done&& done) {
  const PlanRef pl = gp.col();
  const int last = pl->ns - 1, nthr = blockDim.x, tid = threadIdx.x;
  const auto first = [&](auto R) __attribute__((always_inline)) {
    gstage<R, INV>(stage_geom(pl, 0, 1), kGLW, nthr, tid, lsw, NoEarly{}, load, LdsWrite{b0, kGLW, 1});
  };
  if (pl->radix[0] == kFirstRadix) first(std::integral_constant<int, kFirstRadix>{});
  else with_radix(pl->radix[0], first);
  __syncthreads();
  int Ns = pl->radix[0];
  const float2* cur = gfft_stages<INV, SYNC_BLOCK>(pl, 1, last, Ns, b0, b1, kGLW, nthr, tid, lsw);
  with_radix(pl->radix[last], [&](auto R) __attribute__((always_inline)) {
    const int nb = pl->L / R;
    gstage<R, INV>(stage_geom(pl, last, Ns), kGLW, nthr, tid, lsw,
                   [&](int bf, int c) { return early(R, bf, nb, c); }, LdsRead{cur, kGLW},
                   [&](cpx (&a)[R], int, int bf, int c, const auto& e) { done(a, bf, nb, c, e); });
  });
}

// Loads and stores of a strip's bins at k0 = bf + i nb, column c, in global memory.  Columns
// past N/2 read as zero and are not written (plane = false there).
struct StripRead {
  PlaneBuf b;
  bool full;
  int cols;      // valid columns of the strip where it is not full
  template <int R>
  __device__ __forceinline__ void operator()(cpx (&a)[R], int bf, int nb, int c) const {
    const int base = full || c < cols ? bf * kGW + c : kOutOfPlane;
    static_for<R>([&](auto i) { a[i] = b.load(base + i * nb * kGW); });
  }
};
struct StripWrite {
  PlaneBuf b;
  bool full;
  int cols;
  template <int R, class E>
  __device__ __forceinline__ void operator()(cpx (&a)[R], int bf, int nb, int c, const E&) const {
    const int base = full || c < cols ? bf * kGW + c : kOutOfPlane;
    static_for<R>([&](auto i) { b.store(base + i * nb * kGW, a[i]); });
  }
};
// Valid columns of strip s (of those <= M).
__device__ __forceinline__ int strip_cols(int s, int M) { return M + 1 - s * kGW; }

__device__ __forceinline__ void colg_fwd_body(const ColParams& p, const GenParams& gp, BlockId bid) {
  extern __shared__ float2 gsm[];
  const int n = gp.n, E = n * kGW, cols = strip_cols(bid.x, n / 2);
  float2* lsw = gsm;
  float2* b0 = gsm + col_tab_len(n);
  load_table(lsw, col_sw_g(p.tw, n), n - 1);
  const long long strip = bid.y * (long long)n * p.P + (long long)bid.x * E;
  __syncthreads();
  col_transform_g<false>(gp, lsw, b0, b0 + E, NoEarlyCol{}, StripRead{PlaneBuf(p.in + strip, E), cols >= kGW, cols},
                         StripWrite{PlaneBuf(p.out + strip, E), cols >= kGW, cols});
}

__device__ __forceinline__ void colg_syn_body(const ColParams& p, const GenParams& gp, BlockId bid) {
  extern __shared__ float2 gsm[];
  const int n = gp.n, E = n * kGW, M = n / 2;
  float2* lsw = gsm;
  float2* b0 = gsm + col_tab_len(n);
  __shared__ ItemStage<kGW> stg;
  const int4 it = p.items[bid.x];
  const int l = bid.y, cols = strip_cols(it.x, M);
  stage_item(p, it, stg, blockDim.x);
  load_table(lsw, col_sw_g(p.tw, n), n - 1);
  // the strip's spectrum is read again for every filter (from the cache): kept in LDS it would
  // cost a trip through LDS before the first filter and a third of the block's LDS
  const PlaneBuf U(p.in + l * (long long)n * p.P + (long long)it.x * E, E);
  const PsiBuf pb(p);
  __syncthreads();
  for (int i = 0; i < it.z; ++i) {
    const int4 geo = item_geo(stg, i);
    float2* o = p.out + l * p.tl.ls + geo_off(geo) + (long long)(it.x - geo.x / kGW) * E;
    col_transform_g<true>(gp, lsw, b0, b0 + E, NoEarlyCol{},
      [&](auto& a, int bf, int nb, int c) {
        constexpr int R = sizeof(a) / sizeof(cpx);
        const auto f = psi_load_g<R>(pb, stg.win[i][c], bf, nb, n);   // zero window past N/2
        static_for<R>([&](auto k) { a[k] = U.load((bf + k * nb) * kGW + c); });
        // columns past N/2 of the strip hold no spectrum
        static_for<R>([&](auto k) { a[k] = cols >= kGW || c < cols ? a[k] * (f.v[k] * p.inv_n2) : cpx{0.f, 0.f}; });
      },
      StripWrite{PlaneBuf(o, E), cols >= kGW, cols});
    __syncthreads();
  }
}

__device__ __forceinline__ void colg_ana_body(const ColParams& p, const GenParams& gp, BlockId bid) {
  extern __shared__ float2 gsm[];
  const int n = gp.n, E = n * kGW, M = n / 2;
  float2* lsw = gsm;
  float2* ba = gsm + col_tab_len(n);
  float2* b0 = ba + E;
  __shared__ ItemStage<kGW> stg;
  const int4 it = p.items[bid.x];
  const int l = bid.y, cols = strip_cols(it.x, M);
  stage_item(p, it, stg, blockDim.x);
  load_table(lsw, col_sw_g(p.tw, n), n - 1);
  const PsiBuf pb(p);
  // ba: the accumulator; a thread adds to the positions of its own last-stage butterflies, the
  // same ones for every filter (zeroed here: a branch on the first filter at every addition kept
  // the butterfly's outputs live across blocks, 80..108 bytes of scratch per lane)
  for (int e = threadIdx.x; e < E; e += blockDim.x) ba[e] = make_float2(0.f, 0.f);
  __syncthreads();
  for (int i = 0; i < it.z; ++i) {
    const int4 geo = item_geo(stg, i);
    const float2* in = p.in + l * p.tl.ls + geo_off(geo) + (long long)(it.x - geo.x / kGW) * E;
    col_transform_g<false>(gp, lsw, b0, b0 + E,
      [&](auto R, int bf, int nb, int c) {
        if constexpr (R <= 16) return psi_load_g<R>(pb, stg.win[i][c], bf, nb, n);
        else return 0;      // large butterflies: after the transform, in groups (registers)
      },
      StripRead{PlaneBuf(in, E), cols >= kGW, cols},
      [&](auto& a, int bf, int nb, int c, const auto& f0) {
        constexpr int R = sizeof(a) / sizeof(cpx);
        const auto add = [&](int k, cpx x, float f) {
          float2* o = ba + (bf + k * nb) * kGW + c;
          const cpx old = ld(o);
          st(o, cpx{fmaf(x.x, f, old.x), fmaf(x.y, f, old.y)});
        };
        if constexpr (R <= 16) {
          static_for<R>([&](auto k) { add(k, a[k], f0.v[k]); });
        } else {
          constexpr int H = 8;
          static_for<(R + H - 1) / H>([&](auto h) {
            constexpr int k0 = h * H, cnt = R - k0 < H ? R - k0 : H;
            const auto f = psi_load_g<cnt>(pb, stg.win[i][c], bf + k0 * nb, nb, n);
            static_for<cnt>([&](auto m) { add(k0 + m, a[k0 + m], f.v[m]); });
          });
        }
      });
    __syncthreads();
  }
  if (it.w < 0) {
    col_transform_g<true>(gp, lsw, b0, b0 + E, NoEarlyCol{},
      [&](auto& a, int bf, int nb, int c) {
        constexpr int R = sizeof(a) / sizeof(cpx);
        static_for<R>([&](auto k) { a[k] = ld(ba + (bf + k * nb) * kGW + c) * p.inv_n2; });
      },
      StripWrite{PlaneBuf(p.out + l * (long long)n * p.P + (long long)it.x * E, E), cols >= kGW, cols});
  } else {
    float2* o = p.part + ((long long)it.w * p.labels + l) * E;
    for (int e = threadIdx.x; e < E; e += blockDim.x) o[e] = ba[e];
  }
}

// A strip's partial accumulators (consecutive slots) summed in order, then its inverse
// transform.  The sum is a chain of dependent adds on data just written by other CUs, in a
// launch of few blocks: all the block's threads take part, each with several slots' loads in
// flight.
__device__ __forceinline__ void colg_final_body(const ColParams& p, const GenParams& gp, BlockId bid) {
  extern __shared__ float2 gsm[];
  const int n = gp.n, E = n * kGW, M = n / 2;
  const int2 si = p.strips[bid.x];
  if (si.y <= 1) return;
  float2* lsw = gsm;
  float2* ba = gsm + col_tab_len(n);
  float2* b0 = ba + E;
  const int l = bid.y, cols = strip_cols(bid.x, M);
  load_table(lsw, col_sw_g(p.tw, n), n - 1);
  const float4* in = reinterpret_cast<const float4*>(p.part + ((long long)p.items[si.x].w * p.labels + l) * E);
  const long long step = (long long)p.labels * E / 2;
  for (int e = threadIdx.x; e < E / 2; e += blockDim.x) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
    for (int i = 0; i < si.y; ++i) {
      const float4 x = in[i * step + e];
      v.x += x.x; v.y += x.y; v.z += x.z; v.w += x.w;
    }
    reinterpret_cast<float4*>(ba)[e] = v;
  }
  __syncthreads();
  col_transform_g<true>(gp, lsw, b0, b0 + E, NoEarlyCol{},
    [&](auto& a, int bf, int nb, int c) {
      constexpr int R = sizeof(a) / sizeof(cpx);
      static_for<R>([&](auto k) { a[k] = ld(ba + (bf + k * nb) * kGW + c) * p.inv_n2; });
    },
    StripWrite{PlaneBuf(p.out + l * (long long)n * p.P + (long long)bid.x * E, E), cols >= kGW, cols});
}

// One kernel per kind of column pass, plain and grouped; instantiated per translation unit.
template <int KIND>
__device__ __forceinline__ void colg_body(const ColParams& p, const GenParams& gp, BlockId bid) {
  if constexpr (KIND == COL_FWD) colg_fwd_body(p, gp, bid);
  else if constexpr (KIND == COL_SYN) colg_syn_body(p, gp, bid);
  else if constexpr (KIND == COL_ANA) colg_ana_body(p, gp, bid);
  else colg_final_body(p, gp, bid);
}
template <int KIND>
__global__ __launch_bounds__(KIND == COL_FINAL ? kFinalThreads : 256) __attribute__((amdgpu_waves_per_eu(4)))
void k_colg(ColParams p, GenParams gp) {
  colg_body<KIND>(p, gp, own_block());
}
template <int KIND>
__global__ __launch_bounds__(KIND == COL_FINAL ? kFinalThreads : 256) __attribute__((amdgpu_waves_per_eu(4)))
void kg_colg(const GroupTask<ColParams>* __restrict__ tasks, const uint16_t* __restrict__ bt) {
  const GroupTask<ColParams>& T = group_task(tasks, bt);
  colg_body<KIND>(T.p, T.gp, group_block(T));
}

template <int KIND>
void mixed_col(const shs_plan* p, const ColParams& cp, int nblocks, int labels, hipStream_t s) {
  const int threads = KIND == COL_FINAL ? kFinalThreads : col_g_threads(p->pcol);
  const GenParams gp = mixed_params(p);
  const size_t lds = col_g_lds_bytes(p, KIND == COL_ANA || KIND == COL_FINAL ? 1 : 0);
  if (g_rec) {
    LaunchRec& r = rec_add(RK_COL, &kg_colg<KIND>, threads, nblocks, labels, lds);
    r.cp = cp;
    r.gp = gp;
    return;
  }
  hipLaunchKernelGGL((k_colg<KIND>), dim3(nblocks, labels), dim3(threads), lds, s, cp, gp);
}
// Lets the column kernels take the dynamic LDS of the largest supported side.
template <int KIND>
bool mixed_col_reserve() {
  const int bytes = (3 * kGenericMaxN * kGW + col_tab_len(kGenericMaxN)) * int(sizeof(float2));
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_colg<KIND>), hipFuncAttributeMaxDynamicSharedMemorySize,
                             bytes) == hipSuccess &&
         hipFuncSetAttribute(reinterpret_cast<const void*>(&kg_colg<KIND>), hipFuncAttributeMaxDynamicSharedMemorySize,
                             bytes) == hipSuccess;
}
#define SHS_MIXED_COL_EXTERN(KIND)                                                                                  \
  extern template void mixed_col<KIND>(const shs_plan*, const ColParams&, int, int, hipStream_t);                    \
  extern template bool mixed_col_reserve<KIND>();
#define SHS_MIXED_COL_HERE(KIND)                                                                                    \
  template void shs::mixed_col<KIND>(const shs_plan*, const ColParams&, int, int, hipStream_t);                      \
  template bool shs::mixed_col_reserve<KIND>();

}  // namespace shs
