// Column passes of the mixed-radix path (runtime N): single-image and grouped kernels, and
// the TV model's column solve.
#pragma once
#include "generic.hpp"
#include "grouped.hpp"

namespace shs {

// ---------------------------------------------------------------- generic column passes
// One strip (kGW columns) per block of 256 threads; a strip's N x kGW bins are one
// contiguous block in memory and in LDS (bin (k0, c) at k0 * kGW + c).
__device__ __forceinline__ float psi_at_rt(const ColParams& p, int4 win, int k0, int n) {
  int rel = k0 - win.x;
  if (rel < 0) rel += n;
  return rel < win.y ? p.psiw[win.z + rel] : 0.f;
}

// The item's filter windows and plane geometry in LDS (as stage_item of the fixed sizes).
__device__ __forceinline__ void stage_item_g(const ColParams& p, int4 it, int M, ItemStage<kGW>& st) {
  for (int e = threadIdx.x; e < it.z * kGW; e += 256) {
    const int i = e / kGW, cc = e % kGW;
    const int j = p.flist[it.y + i];
    const int k1 = it.x * kGW + cc;
    st.win[i][cc] = k1 <= M ? p.pwin[j * (M + 1) + k1] : make_int4(0, 0, 0, 0);
    if (cc == 0) st.geo[i] = p.tl.tab[j];
  }
}

__device__ __forceinline__ void colg_fwd_body(const ColParams& p, const GenParams& gp, BlockId bid) {
  extern __shared__ float2 gsm[];
  const int n = gp.n, E = n * kGW;
  float2* lsw = gsm;
  float2* b0 = gsm + col_tab_len(n);
  float2* b1 = b0 + E;
  load_table(lsw, col_sw_g(p.tw, n), n - 1);
  const long long strip = bid.y * (long long)n * p.P + (long long)bid.x * E;
  for (int e = threadIdx.x; e < E; e += 256) b0[e] = p.in[strip + e];
  __syncthreads();
  float2* r = gfft<false, SYNC_BLOCK, kGW, true>(b0, b1, gp.pcol, 256, threadIdx.x, lsw);
  const int M = n / 2;
  for (int e = threadIdx.x; e < E; e += 256)
    if (bid.x * kGW + (e % kGW) <= M) p.out[strip + e] = r[e];
}

static __global__ __launch_bounds__(256) void k_colg_fwd(ColParams p, GenParams gp) {
  colg_fwd_body(p, gp, own_block());
}

__device__ __forceinline__ void colg_syn_body(const ColParams& p, const GenParams& gp, BlockId bid) {
  extern __shared__ float2 gsm[];
  const int n = gp.n, E = n * kGW, M = n / 2;
  float2* lsw = gsm;
  float2* bu = gsm + col_tab_len(n);
  float2* b0 = bu + E;
  float2* b1 = bu + 2 * E;
  __shared__ ItemStage<kGW> stg;
  const int4 it = p.items[bid.x];
  const int l = bid.y;
  load_table(lsw, col_sw_g(p.tw, n), n - 1);
  stage_item_g(p, it, M, stg);
  const float2* U = p.in + l * (long long)n * p.P + (long long)it.x * E;
  for (int e = threadIdx.x; e < E; e += 256) bu[e] = U[e];
  __syncthreads();
  for (int i = 0; i < it.z; ++i) {
    for (int e = threadIdx.x; e < E; e += 256) {
      const float f = psi_at_rt(p, stg.win[i][e % kGW], e / kGW, n);   // zero window past N/2
      b0[e] = make_float2(bu[e].x * f * p.inv_n2, bu[e].y * f * p.inv_n2);
    }
    __syncthreads();
    float2* r = gfft<true, SYNC_BLOCK, kGW, true>(b0, b1, gp.pcol, 256, threadIdx.x, lsw);
    const int4 geo = stg.geo[i];
    float2* o = p.out + l * p.tl.ls + geo_off(geo) + (long long)(it.x - geo.x / kGW) * E;
    for (int e = threadIdx.x; e < E; e += 256)
      if (it.x * kGW + (e % kGW) <= M) o[e] = r[e];
    __syncthreads();
  }
}

static __global__ __launch_bounds__(256) void k_colg_syn(ColParams p, GenParams gp) {
  colg_syn_body(p, gp, own_block());
}

__device__ __forceinline__ void colg_finish(const ColParams& p, const GenParams& gp, const float2* lsw, float2* acc,
                                            float2* b1, int strip, int l) {
  const int n = gp.n, E = n * kGW, M = n / 2;
  for (int e = threadIdx.x; e < E; e += 256) acc[e] = make_float2(acc[e].x * p.inv_n2, acc[e].y * p.inv_n2);
  __syncthreads();
  float2* r = gfft<true, SYNC_BLOCK, kGW, true>(acc, b1, gp.pcol, 256, threadIdx.x, lsw);
  float2* o = p.out + l * (long long)n * p.P + (long long)strip * E;
  for (int e = threadIdx.x; e < E; e += 256)
    if (strip * kGW + (e % kGW) <= M) o[e] = r[e];
}

__device__ __forceinline__ void colg_ana_body(const ColParams& p, const GenParams& gp, BlockId bid) {
  extern __shared__ float2 gsm[];
  const int n = gp.n, E = n * kGW, M = n / 2;
  float2* lsw = gsm;
  float2* ba = gsm + col_tab_len(n);
  float2* b0 = ba + E;
  float2* b1 = ba + 2 * E;
  __shared__ ItemStage<kGW> stg;
  const int4 it = p.items[bid.x];
  const int l = bid.y;
  load_table(lsw, col_sw_g(p.tw, n), n - 1);
  stage_item_g(p, it, M, stg);
  for (int e = threadIdx.x; e < E; e += 256) ba[e] = make_float2(0.f, 0.f);
  __syncthreads();
  for (int i = 0; i < it.z; ++i) {
    const int4 geo = stg.geo[i];
    const float2* in = p.in + l * p.tl.ls + geo_off(geo) + (long long)(it.x - geo.x / kGW) * E;
    for (int e = threadIdx.x; e < E; e += 256) {
      const int k1 = it.x * kGW + (e % kGW);
      b0[e] = k1 <= M ? in[e] : make_float2(0.f, 0.f);
    }
    __syncthreads();
    float2* r = gfft<false, SYNC_BLOCK, kGW, true>(b0, b1, gp.pcol, 256, threadIdx.x, lsw);
    for (int e = threadIdx.x; e < E; e += 256) {
      const float f = psi_at_rt(p, stg.win[i][e % kGW], e / kGW, n);   // zero window past N/2
      ba[e] = make_float2(ba[e].x + r[e].x * f, ba[e].y + r[e].y * f);
    }
    __syncthreads();
  }
  if (it.w < 0) {
    colg_finish(p, gp, lsw, ba, b1, it.x, l);
  } else {
    float2* o = p.part + ((long long)it.w * p.labels + l) * E;
    for (int e = threadIdx.x; e < E; e += 256) o[e] = ba[e];
  }
}

static __global__ __launch_bounds__(256) void k_colg_ana(ColParams p, GenParams gp) {
  colg_ana_body(p, gp, own_block());
}

__device__ __forceinline__ void colg_final_body(const ColParams& p, const GenParams& gp, BlockId bid) {
  extern __shared__ float2 gsm[];
  const int n = gp.n, E = n * kGW;
  const int2 si = p.strips[bid.x];
  if (si.y <= 1) return;
  float2* lsw = gsm;
  float2* ba = gsm + col_tab_len(n);
  float2* b1 = ba + E;
  const int l = bid.y;
  load_table(lsw, col_sw_g(p.tw, n), n - 1);
  for (int e = threadIdx.x; e < E; e += 256) ba[e] = make_float2(0.f, 0.f);
  for (int i = 0; i < si.y; ++i) {
    const float2* in = p.part + ((long long)p.items[si.x + i].w * p.labels + l) * E;
    for (int e = threadIdx.x; e < E; e += 256) ba[e] = make_float2(ba[e].x + in[e].x, ba[e].y + in[e].y);
  }
  __syncthreads();
  colg_finish(p, gp, lsw, ba, b1, bid.x, l);
}

static __global__ __launch_bounds__(256) void k_colg_final(ColParams p, GenParams gp) {
  colg_final_body(p, gp, own_block());
}

// ---- grouped launches
static __global__ __launch_bounds__(256) void kg_colg_fwd(const GroupTask<ColParams>* __restrict__ tasks,
                                                  const uint16_t* __restrict__ bt) {
  const GroupTask<ColParams>& T = group_task(tasks, bt);
  colg_fwd_body(T.p, T.gp, group_block(T));
}
static __global__ __launch_bounds__(256) void kg_colg_syn(const GroupTask<ColParams>* __restrict__ tasks,
                                                  const uint16_t* __restrict__ bt) {
  const GroupTask<ColParams>& T = group_task(tasks, bt);
  colg_syn_body(T.p, T.gp, group_block(T));
}
static __global__ __launch_bounds__(256) void kg_colg_ana(const GroupTask<ColParams>* __restrict__ tasks,
                                                  const uint16_t* __restrict__ bt) {
  const GroupTask<ColParams>& T = group_task(tasks, bt);
  colg_ana_body(T.p, T.gp, group_block(T));
}
static __global__ __launch_bounds__(256) void kg_colg_final(const GroupTask<ColParams>* __restrict__ tasks,
                                                    const uint16_t* __restrict__ bt) {
  const GroupTask<ColParams>& T = group_task(tasks, bt);
  colg_final_body(T.p, T.gp, group_block(T));
}

// ---------------------------------------------------------------- TV column solve
static __global__ __launch_bounds__(256) void k_colg_solve(ColParams p, GenParams gp, const float* __restrict__ eig) {
  extern __shared__ float2 gsm[];
  const int n = gp.n, E = n * kGW, M = n / 2;
  float2* b0 = gsm;
  float2* b1 = gsm + E;
  const long long strip = blockIdx.y * (long long)n * p.P + (long long)blockIdx.x * E;
  for (int e = threadIdx.x; e < E; e += 256) b0[e] = p.in[strip + e];
  __syncthreads();
  float2* r = gfft<false, SYNC_BLOCK, kGW>(b0, b1, gp.pcol, 256, threadIdx.x, col_sw_g(p.tw, gp.n));
  float2* o = r == b0 ? b1 : b0;
  for (int e = threadIdx.x; e < E; e += 256) {
    const int k1 = blockIdx.x * kGW + (e % kGW);
    const float m = k1 <= M ? p.inv_n2 / (1.f + eig[e / kGW] + eig[k1]) : 0.f;
    r[e] = make_float2(r[e].x * m, r[e].y * m);
  }
  __syncthreads();
  float2* z = gfft<true, SYNC_BLOCK, kGW>(r, o, gp.pcol, 256, threadIdx.x, col_sw_g(p.tw, gp.n));
  for (int e = threadIdx.x; e < E; e += 256)
    if (blockIdx.x * kGW + (e % kGW) <= M) p.out[strip + e] = z[e];
}

}  // namespace shs
