// Skinny LoRA down-projection U = scale * X A^T for up to three adapter targets
// that read the same input (q/k/v, gate/up, o or down).  The input is read
// once; the r x K factors stay in L2.  HBM-bound.
#include <algorithm>

#include "kernels.hpp"

namespace crf {
namespace {

constexpr int MAXT = 3;
constexpr int MAXB = 12;  // 16-row blocks over all targets (3 targets x rank 64)
// block counts n_targets * rank_pad / 16 that occur: {1,2,3} targets x rank_pad {16,32,48,64}

struct LdArgs {
  const bf16 *X;
  int64_t ldx;
  int M, K;
  const bf16 *A[MAXT];
  int rank[MAXT];
  float scale[MAXT];
  int ucol[MAXT];
  int n_targets, rank_pad;
  bf16 *U;
  int ldu;
  int spw;      // k-steps of 32 per workgroup along grid.y
  float *part;  // non-null: fp32 partial sums [grid.y][16][n_targets * rank_pad], unscaled
  // non-null: K split over grid.y workgroups, whose partial blocks go to
  // `blocks` [token block][grid.y][NB][64][4] and are summed by the last of
  // them; one ticket per token block, zero between launches
  unsigned *tickets;
  float *blocks;
};

// Workgroup: TB blocks of 16 tokens, NW waves splitting K (wave w takes k-steps
// w, w+NW, ...).  Per k-step of 32: D[j, token] += A_t[j, k..k+32] .
// X[token, k..k+32] on the 16x16x32 MFMA, one MFMA per (16-row block of the
// concatenated factors, token block): the factors are read once per TB*16
// tokens.  The loads of UNROLL k-steps are issued before their MFMAs so enough
// bytes are in flight to keep HBM busy; the factors (a few hundred KB) stay in
// L2.
template <int NB, int UNROLL, int TB, int NW = 4>
__global__ __launch_bounds__(64 * NW) void lora_down_kernel(LdArgs a) {
  __shared__ f32x4 red[NW][NB * TB][64];
  // wave-uniform in a scalar register: the k-step guards below are then scalar
  // branches.  Derived per lane, they become EXEC-masked blocks, and an MFMA in
  // such a block still updates its accumulators when the mask is empty, adding
  // the previous batch's fragments once more.
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int m0 = blockIdx.x * 16 * TB;
  const int kq = (lane / 16) * 8;
  const bf16 *xrow[TB];
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) xrow[tb] = a.X + (int64_t)min(m0 + 16 * tb + lane % 16, a.M - 1) * a.ldx + kq;
  // per block: the target's factor as a buffer resource and this lane's row
  // offset; rows past the rank (and absent targets) lie out of range and read
  // as zero, so the loads need no branch
  __amdgpu_buffer_rsrc_t ares[NB];
  uint32_t aoff[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int t = (b * 16) / a.rank_pad;
    const int j = b * 16 - t * a.rank_pad + lane % 16;
    const bool on = a.A[t] != nullptr;
    ares[b] = make_rsrc(on ? (const void *)a.A[t] : (const void *)a.X, on ? (uint32_t)(a.rank[t] * a.K * 2) : 0u);
    aoff[b] = on && j < a.rank[t] ? (uint32_t)((j * a.K + kq) * 2) : CRF_OOB;
  }
  f32x4 acc[NB][TB];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) acc[b][tb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int s0 = blockIdx.y * a.spw, s1 = min(a.K / 32, s0 + a.spw);
  for (int st = s0 + wave; st < s1; st += NW * UNROLL) {
    bf16x8 xb[UNROLL][TB], ab[UNROLL][NB];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      if (st + NW * u < s1) {  // wave-uniform
        const int k = (st + NW * u) * 32;
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) xb[u][tb] = as_bf16x8(ld16(xrow[tb] + k));
#pragma unroll
        for (int b = 0; b < NB; ++b)
          ab[u][b] = as_bf16x8(bld16(ares[b], aoff[b], (uint32_t)k * 2));
      }
    }
    __builtin_amdgcn_sched_barrier(0);  // every load of the batch in flight before the first MFMA
#pragma unroll
    for (int u = 0; u < UNROLL; ++u)
      if (st + NW * u < s1)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int tb = 0; tb < TB; ++tb) acc[b][tb] = mfma16(ab[u][b], xb[u][tb], acc[b][tb]);
  }
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) red[wave][b * TB + tb][lane] = acc[b][tb];
  __syncthreads();
  // the waves share the blocks' final sums
  for (int i = wave; i < NB * TB; i += NW) {
    const int b = i / TB, tb = i % TB, m = m0 + 16 * tb + lane % 16;
    f32x4 v = red[0][i][lane];
#pragma unroll
    for (int w = 1; w < NW; ++w) v += red[w][i][lane];
    if (a.tickets) {
      st_agent16(a.blocks + ((((int64_t)blockIdx.x * gridDim.y + blockIdx.y) * NB + b) * 64 + lane) * 4, v);
      continue;
    }
    if (m >= a.M) continue;
    if (a.part) {  // K split over workgroups: unscaled part, summed by the projection
      const int ncols = a.n_targets * a.rank_pad;
      *reinterpret_cast<f32x4 *>(a.part + ((int64_t)blockIdx.y * 16 + m) * ncols + b * 16 + (lane / 16) * 4) = v;
      continue;
    }
    const int t = (b * 16) / a.rank_pad;
    const int jb = b * 16 - t * a.rank_pad + (lane / 16) * 4;  // first of 4 rows held by this lane
    const float sc = a.scale[t];
    st8(a.U + (int64_t)m * a.ldu + a.ucol[t] + jb, pack_bf16x4(v[0] * sc, v[1] * sc, v[2] * sc, v[3] * sc));
  }
  if (TB > 1 || !a.tickets) return;
  __shared__ bool is_last;
  agent_flush();
  __syncthreads();
  if (threadIdx.x == 0) {
    is_last = agent_ticket(a.tickets + blockIdx.x) == gridDim.y - 1;
    if (is_last) __hip_atomic_store(a.tickets + blockIdx.x, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (!is_last) return;
  for (int b = wave; b < NB; b += NW) {
    const float *q = a.blocks + (((int64_t)blockIdx.x * gridDim.y * NB + b) * 64 + lane) * 4;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    for (int y0 = 0; y0 < (int)gridDim.y; y0 += 4) {
      f32x4 t[4];
#pragma unroll
      for (int y = 0; y < 4; ++y) t[y] = ld_agent16(q + (int64_t)min(y0 + y, (int)gridDim.y - 1) * NB * 256);
#pragma unroll
      for (int y = 0; y < 4; ++y)
        if (y0 + y < (int)gridDim.y) v += t[y];
    }
    const int m = m0 + lane % 16;
    if (m >= a.M) continue;
    const int t = (b * 16) / a.rank_pad;
    const int jb = b * 16 - t * a.rank_pad + (lane / 16) * 4;
    const float sc = a.scale[t];
    st8(a.U + (int64_t)m * a.ldu + a.ucol[t] + jb, pack_bf16x4(v[0] * sc, v[1] * sc, v[2] * sc, v[3] * sc));
  }
}

template <int NB>
hipError_t go(hipStream_t s, LdArgs a, float *ws, int64_t ws_floats, int *n_parts, const LoraWs &lw) {
  constexpr int UNROLL = NB <= 4 ? 8 : 2;
  const int nsteps = a.K / 32;
  if (n_parts) {
    // a few token rows: K split over workgroups (one batch of loads per wave),
    // the parts summed by the projection that uses U
    a.spw = 4 * UNROLL;
    const int n = (nsteps + a.spw - 1) / a.spw;
    if (a.M > 16 || !ws || (int64_t)n * 16 * a.n_targets * a.rank_pad > ws_floats) return hipErrorInvalidValue;
    a.part = ws;
    *n_parts = n;
    hipLaunchKernelGGL((lora_down_kernel<NB, UNROLL, 1>), dim3(1, n), dim3(256), 0, s, a);
    return hipSuccess;
  }
  a.spw = nsteps;
  a.part = nullptr;
  if constexpr (NB <= 4) {
    if (a.M >= 8192) {
      // 64 tokens per workgroup (the factors are read once per 64 tokens) and
      // 8 waves splitting K, so that enough loads are in flight per CU
      hipLaunchKernelGGL((lora_down_kernel<NB, 4, 4, 8>), dim3((a.M + 63) / 64), dim3(512), 0, s, a);
      return hipSuccess;
    }
  }
  // Fewer tokens: 16 per workgroup.  A workgroup is bound by what one CU can
  // read (its tokens and all of the factors), so K is split over workgroups
  // until there are about two to a CU, of at least 16 k-steps.  777 tokens of 7B
  // shapes, rank 32: down (K = 18944) 85 -> 19 us, o (K = 3584) 22 -> 8, gate/up
  // 22 -> 12.  Two parts of 256 token blocks are slower than none (4096 tokens of
  // 1.5B shapes, q/k/v: 12.4 against 11.2 us), three of 129 to 170 faster (a layer of
  // 7B shapes, rank 64 on all: 2064 tokens 1269 -> 1206 us, 2720: 1573 -> 1514; rank 16
  // on q, k, v, o: the same within 1 %).
  const int mb = (a.M + 15) / 16;
  const int64_t cap = lw.blocks ? lw.floats / ((int64_t)mb * NB * 256) : 0;
  const int64_t split = std::min<int64_t>({512 / mb, nsteps / 16, cap, 64});
  if (split >= 3 && lw.tickets && mb <= lw.n_tickets) {
    a.spw = (int)((nsteps + split - 1) / split);
    a.tickets = lw.tickets;
    a.blocks = lw.blocks;
    hipLaunchKernelGGL((lora_down_kernel<NB, UNROLL, 1>), dim3(mb, (nsteps + a.spw - 1) / a.spw), dim3(256), 0, s, a);
    return hipSuccess;
  }
  hipLaunchKernelGGL((lora_down_kernel<NB, UNROLL, 1>), dim3(mb), dim3(256), 0, s, a);
  return hipSuccess;
}

}  // namespace

hipError_t launch_lora_down_bf16(hipStream_t s, const bf16 *X, int64_t ldx, int M, int K, const LoraDownTarget *t,
                                 int n_targets, int rank_pad, bf16 *U, int ldu, float *ws, int64_t ws_floats,
                                 int *n_parts, const LoraWs &lw) {
  if (n_parts) *n_parts = 0;
  if (M <= 0 || n_targets <= 0) return hipSuccess;
  if (n_targets > MAXT || n_targets * rank_pad > MAXB * 16 || rank_pad % 16 || K % 32) return hipErrorInvalidValue;
  LdArgs a{};
  a.X = X;
  a.ldx = ldx;
  a.M = M;
  a.K = K;
  for (int i = 0; i < n_targets; ++i) {
    a.A[i] = t[i].A;
    a.rank[i] = t[i].A ? t[i].rank : 0;
    a.scale[i] = t[i].scale;
    a.ucol[i] = t[i].ucol;
  }
  a.n_targets = n_targets;
  a.rank_pad = rank_pad;
  a.U = U;
  a.ldu = ldu;
  hipError_t e;
  switch (n_targets * rank_pad / 16) {
    case 1: e = go<1>(s, a, ws, ws_floats, n_parts, lw); break;
    case 2: e = go<2>(s, a, ws, ws_floats, n_parts, lw); break;
    case 3: e = go<3>(s, a, ws, ws_floats, n_parts, lw); break;
    case 4: e = go<4>(s, a, ws, ws_floats, n_parts, lw); break;
    case 6: e = go<6>(s, a, ws, ws_floats, n_parts, lw); break;
    case 8: e = go<8>(s, a, ws, ws_floats, n_parts, lw); break;
    case 9: e = go<9>(s, a, ws, ws_floats, n_parts, lw); break;
    case 12: e = go<12>(s, a, ws, ws_floats, n_parts, lw); break;
    default: return hipErrorInvalidValue;
  }
  return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace crf
