// Projections of a few token rows (M <= 16: the new tokens of a decoding step,
// or a very short window).  There the weights are streamed once and used M
// times, so the work is HBM-bound and the 256-row tiles of gemm_bf16 would sit
// mostly empty.  Instead, one workgroup owns 16 output features (32 for
// gate/up: the same 16 features of both) for all M tokens: its 4-16 waves split K,
// each issuing v_mfma_f32_16x16x32_bf16 with the weight rows as operand A and
// the token rows as operand B, several k-steps of loads in flight; the partial
// sums meet in LDS, wave 0 adds the adapter delta (U B^T, one more MFMA step
// per 32 of rank) and runs the epilogue.  A lane ends up with 4 consecutive
// features of one token, as in gemm_bf16:
//   EPI_RESID  resid[m, f] (+)= acc, optional bf16 copy;
//   EPI_SWIGLU act[m, f] = silu(gate) * up;
//   EPI_QKV    8 features of a head and their rotary partners: bias, rotation,
//              Q to its buffer, K and V to their pages.
// U comes as K-split parts of the launch before (norm_lora below, the attention
// merge, or lora_down), which every workgroup sums while its weights stream: a
// layer of a decoding step is a chain of launches whose start and end cost as
// much as their bytes, so each one saved is worth 3 to 5 us.  A 7B-shaped layer
// over a 16384-token prefix (rank 16 on all seven) takes 9 launches where it
// took 14; whole step of 28 layers and a 152064-row head, 15.2 GB: 4.62 -> 3.99
// ms (3.8 TB/s); 1.5B shapes, 5 tokens over 3001: 2.22 -> 1.87 ms.  The head
// alone streams at 6.2 TB/s, gate/up at 5.1, down at 4.9, QKV at 2.6 (33 MB in
// 13 us: about 6 us of every launch are its start and end).
#include <algorithm>

#include "kernels.hpp"

namespace crf {
namespace {

CRF_DEV void load8f(const float *p, float (&v)[8]) {
  const f32x4 a = *reinterpret_cast<const f32x4 *>(p), b = *reinterpret_cast<const f32x4 *>(p + 4);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[i] = a[i];
    v[i + 4] = b[i];
  }
}
CRF_DEV void load8f(const bf16 *p, float (&v)[8]) {
  const bf16x8 a = as_bf16x8(ld16(p));
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = bf2f(a[i]);
}

constexpr int SKINNY_MAX_PARTS = 8;
// k-steps of loads issued before their MFMAs (8; 4 where 16 waves of two blocks
// and an adapter's sums would not fit the registers)
template <int W, int NB, int KB>
constexpr int unroll_of() {
  return W == 16 && NB == 2 && KB > 0 ? 4 : 8;
}

// Row `i` (0..15) of block `block` of workgroup tile `t` and its segment.
// Gate/up: block 0 gate rows, block 1 up rows of the same features.  QKV: 8
// in-head features of the first half, then their 8 rotary partners.
template <int EPI>
CRF_DEV const bf16 *skinny_weight_row(const GemmParams &p, int t, int i, int block, int &seg, int &local) {
  if (EPI == EPI_SWIGLU) {
    seg = block;
    local = min(16 * t + i, p.d_ffn - 1);
  } else if (EPI == EPI_QKV) {
    // (head sizes are 64 and 128; a division would stand before the first load)
    const int half = p.hd / 2, sh = p.hd == 128 ? 3 : 2;  // tiles per head: 8 or 4
    const int r = (t >> sh) * p.hd + (t & ((1 << sh) - 1)) * 8;  // one head: one segment
    seg = r < p.seg1 ? 0 : (r < p.seg2 ? 1 : 2);
    local = r - (seg == 0 ? 0 : (seg == 1 ? p.seg1 : p.seg2)) + (i < 8 ? i : half + i - 8);
  } else {
    seg = 0;
    local = min(16 * t + i, p.N - 1);
  }
  return p.w[seg] + (int64_t)local * p.K;
}

// KB: rank steps of 32 of the adapter (0: no adapter)
// SPLIT: grid.y workgroups share a tile's K, kpairs pairs of k-steps each
template <int EPI, int NB, int W, int KB, bool SPLIT>
__global__ __launch_bounds__(64 * W) void gemm_skinny_kernel(const GemmParams p) {
  constexpr bool LORA = KB > 0;
  constexpr int UNROLL = unroll_of<W, NB, KB>();
  constexpr int NU = LORA ? (EPI == EPI_SWIGLU ? 2 : 1) : 0;  // adapter targets of the tile
  constexpr int UW = NU == 2 ? 2 : (W < 8 ? W : 8);           // waves that sum U's parts
  __shared__ f32x4 red[W][NB][64];
  __shared__ f32x4 ured[LORA ? UW : 1][LORA ? NU * 2 * KB : 1][LORA ? 64 : 1];
  // wave-uniform in a scalar register, so that the k-step guards are scalar
  // branches: an MFMA in an EXEC-masked block still updates its accumulators
  // when the mask is empty
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int tile = blockIdx.x;
  const int tok = min(lane % 16, p.M - 1);  // rows past M repeat the last token; never stored
  const int kq = (lane / 16) * 8;
  const bf16 *xrow = p.X + (int64_t)tok * p.ldx + kq;
  const bf16 *wrow[NB];
  int seg[NB], local[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) wrow[b] = skinny_weight_row<EPI>(p, tile, lane % 16, b, seg[b], local[b]) + kq;

  // the adapter's U arrives as unscaled K-split parts: a few waves take every
  // UW-th part, ahead of the weights' stream (the sums are used at its end)
  f32x4 us[LORA ? NU * 2 * KB : 1];
  if (LORA && wave < UW) {
#pragma unroll
    for (int b = 0; b < NU; ++b)
#pragma unroll
      for (int q = 0; q < KB; ++q) {
        f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = {0.f, 0.f, 0.f, 0.f};
        const int j = 32 * q + kq;
        if (p.lb[seg[b]] && j < p.rank) {
          const float *pp = p.upart + (int64_t)tok * p.upart_cols + p.ucol[seg[b]] + j;
#pragma unroll 4
          for (int y = wave; y < p.upart_n; y += UW) {
            lo += *reinterpret_cast<const f32x4 *>(pp + (int64_t)y * 16 * p.upart_cols);
            hi += *reinterpret_cast<const f32x4 *>(pp + (int64_t)y * 16 * p.upart_cols + 4);
          }
        }
        us[(b * KB + q) * 2] = lo;
        us[(b * KB + q) * 2 + 1] = hi;
      }
  }

  f32x4 acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  // wave w takes the k-step pairs w, w + W, ... (a pair covers 128 bytes of
  // each weight row: whole cache lines per wave); UNROLL steps are loaded
  // before their MFMAs (the scheduling barrier keeps every load of a batch in
  // flight at once)
  const int y = SPLIT ? blockIdx.y : 0, n_parts = SPLIT ? gridDim.y : 1;
  const int nsteps = SPLIT ? min(p.K / 32, 2 * (y + 1) * p.kpairs) : p.K / 32;
  for (int sp = (SPLIT ? y * p.kpairs : 0) + wave; 2 * sp < nsteps; sp += W * UNROLL / 2) {
    bf16x8 xb[UNROLL], wb[UNROLL][NB];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int st = 2 * (sp + W * (u / 2)) + u % 2;
      if (st < nsteps) {  // wave-uniform
        const int k = st * 32;
        xb[u] = as_bf16x8(ld16(xrow + k));
#pragma unroll
        for (int b = 0; b < NB; ++b) wb[u][b] = as_bf16x8(ld16(wrow[b] + k));
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < UNROLL; ++u)
      if (2 * (sp + W * (u / 2)) + u % 2 < nsteps)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b] = mfma16(wb[u][b], xb[u], acc[b]);
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) red[wave][b][lane] = acc[b];
  if (LORA && wave < UW)
#pragma unroll
    for (int i = 0; i < NU * 2 * KB; ++i) ured[wave][i][lane] = us[i];
  __syncthreads();
  if (wave != 0) return;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    acc[b] = red[0][b][lane];
#pragma unroll
    for (int w = 1; w < W; ++w) acc[b] += red[w][b][lane];
  }
  if constexpr (SPLIT) {
    // the last of the tile's workgroups to get here adds the parts in order
    float *q = p.split_part + ((int64_t)tile * n_parts * NB * 64 + lane) * 4;
#pragma unroll
    for (int b = 0; b < NB; ++b) st_agent16(q + (y * NB + b) * 256, acc[b]);
    agent_flush();
    unsigned t = 0;
    if (lane == 0) t = agent_ticket(p.tickets + tile);
    if (__builtin_amdgcn_readfirstlane(t) != (unsigned)n_parts - 1) return;
    if (lane == 0) __hip_atomic_store(p.tickets + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      f32x4 v[SKINNY_MAX_PARTS];
#pragma unroll
      for (int i = 0; i < SKINNY_MAX_PARTS; ++i) v[i] = ld_agent16(q + (min(i, n_parts - 1) * NB + b) * 256);
      acc[b] = v[0];
#pragma unroll
      for (int i = 1; i < SKINNY_MAX_PARTS; ++i)
        if (i < n_parts) acc[b] += v[i];
    }
  }
  // adapter delta: acc += U[token, j] * lb[row, j], j < rank (zero-padded to 32)
  if (LORA) {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const bf16 *lb = p.lb[seg[b]];
      if (!lb) continue;
#pragma unroll
      for (int q = 0; q < KB; ++q) {
        if (32 * q >= p.rank) break;
        const int j = 32 * q + kq, i = ((NU == 2 ? b : 0) * KB + q) * 2;
        f32x4 lo = ured[0][i][lane], hi = ured[0][i + 1][lane];
#pragma unroll
        for (int w = 1; w < UW; ++w) {
          lo += ured[w][i][lane];
          hi += ured[w][i + 1][lane];
        }
        lo *= p.uscale;
        hi *= p.uscale;
        const bf16x8 u8 = {f2bf(lo[0]), f2bf(lo[1]), f2bf(lo[2]), f2bf(lo[3]),
                           f2bf(hi[0]), f2bf(hi[1]), f2bf(hi[2]), f2bf(hi[3])};
        u32x4 av = {0u, 0u, 0u, 0u};
        if (j < p.rank) av = ld16(lb + (int64_t)local[b] * p.rank + j);
        acc[b] = mfma16(as_bf16x8(av), u8, acc[b]);
      }
    }
  }
  const int m = lane % 16;
  const int f = 16 * tile + 4 * (lane / 16);  // first of this lane's 4 features
  if (m >= p.M) return;
  if (EPI == EPI_RESID) {
    if (f >= p.N) return;
    float *rp = p.resid + (int64_t)m * p.ldr + f;
    f32x4 r = p.resid_overwrite ? f32x4{0.f, 0.f, 0.f, 0.f} : *reinterpret_cast<f32x4 *>(rp);
    r += acc[0];
    *reinterpret_cast<f32x4 *>(rp) = r;
    if (p.resid_out) st8(p.resid_out + (int64_t)m * p.ldr + f, pack_bf16x4(r[0], r[1], r[2], r[3]));
  } else if (EPI == EPI_SWIGLU) {
    if (f >= p.d_ffn) return;
    float o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float g = acc[0][i], u = acc[NB - 1][i];
      o[i] = g / (1.0f + __expf(-g)) * u;
    }
    st8(p.act + (int64_t)m * p.d_ffn + f, pack_bf16x4(o[0], o[1], o[2], o[3]));
  } else {  // bias, rotation (token row m at position pos0 + m), Q to its buffer, K and V to their pages
    // lanes l and l ^ 32 hold rotary partners: rows 4 g .. 4 g + 3 and 8 further
    const int half = p.hd / 2, g = lane / 16;
    const bool first = g < 2;
    const int r0 = local[0] - (lane % 16 < 8 ? lane % 16 : half + lane % 16 - 8) + 4 * (g & 1) + (first ? 0 : half);
    const int head = r0 >> (p.hd == 128 ? 7 : 6), fh = r0 & (p.hd - 1);
    f32x4 x = acc[0];
    if (const bf16 *bias = p.bias[seg[0]])
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] += bf2f(bias[r0 + i]);
    if (seg[0] < 2) {
      const float2 *cs = p.rope_cs + (int64_t)(p.pos0 + m) * half + (fh & (half - 1));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float2 c = cs[i];
        const float o = __shfl_xor(x[i], 32, 64);  // (every lane of a pair has the same token: both are here)
        x[i] = first ? x[i] * c.x - o * c.y : x[i] * c.x + o * c.y;
      }
    }
    bf16 *dst;
    if (seg[0] == 0) {
      dst = p.q_out + (int64_t)m * p.dq + r0;
      x *= p.q_scale;
    } else {
      const int64_t row = paged_row(p.kv, p.pos0 + m, head, p.hd);
      if (row < 0) return;
      dst = (bf16 *)(seg[0] == 1 ? p.kv.k : p.kv.v) + row + fh;
    }
    st8(dst, pack_bf16x4(x[0], x[1], x[2], x[3]));
  }
}

// RMSNorm of up to 16 rows and the adapters' down-projection of the result, in
// one launch: workgroup y owns 512 columns.  Every workgroup sums the squares of
// the whole rows (a few KB from L2, while its factors are on their way), writes
// its slice of the normalised rows and leaves the slice's part of U.
// NB: 16-row blocks of the concatenated factors (0: none).
template <typename TX, int NB>
__global__ __launch_bounds__(256) void norm_lora_kernel(const NormLora p) {
  constexpr int SL = 512;
  constexpr bool EARLY = NB > 0 && NB <= 4;  // factors loaded ahead of the norm
  constexpr int NBA = NB > 0 ? NB : 1;
  __shared__ __align__(16) bf16 xs[16][SL + 8];
  __shared__ float rs[16][4];
  __shared__ f32x4 red[4][NBA][64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int k0 = blockIdx.x * SL, kend = min(p.d, k0 + SL);
  const int kq = (lane / 16) * 8;
  const TX *x = (const TX *)p.x;
  bf16x8 ab[4][NBA];
  const bf16 *arow[NBA];
  bool on[NBA];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int t = (b * 16) / p.rank_pad, j = b * 16 - t * p.rank_pad + lane % 16;
    on[b] = p.A[t] && j < p.rank;
    arow[b] = on[b] ? p.A[t] + (int64_t)j * p.d + kq : nullptr;
  }
  auto load_a = [&](int u) {
    const int k = k0 + 32 * (wave + 4 * u);
#pragma unroll
    for (int b = 0; b < NB; ++b)
      ab[u][b] = as_bf16x8(on[b] && k < kend ? ld16(arow[b] + k) : u32x4{0u, 0u, 0u, 0u});
  };
  // Squares: every thread takes 8 columns in 2048, for four rows at a time.  The
  // first rows' loads go out ahead of the factors', whose wait would hold them.
  float ss[4] = {0.f, 0.f, 0.f, 0.f};
  for (int m0 = 0; m0 < p.M; m0 += 4) {
#pragma unroll
    for (int q = 0; q < 4; ++q) ss[q] = 0.f;
#pragma unroll 2
    for (int c = threadIdx.x * 8; c < p.d; c += 2048) {
      float v[4][8];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (m0 + q < p.M) load8f(x + (int64_t)(m0 + q) * p.d + c, v[q]);  // uniform
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (m0 + q < p.M)
#pragma unroll
          for (int i = 0; i < 8; ++i) ss[q] = fmaf(v[q][i], v[q][i], ss[q]);
    }
    if (EARLY && m0 == 0)
#pragma unroll
      for (int u = 0; u < 4; ++u) load_a(u);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (m0 + q < p.M) {
        const float t = wave_sum(ss[q]);
        if (lane == 0) rs[m0 + q][wave] = t;
      }
  }
  __syncthreads();
  {
    const int c = k0 + 8 * lane;  // a wave covers the slice
    float gv[8];
    if (c < kend) load8f(p.g + c, gv);
    for (int m = wave; m < p.M && c < kend; m += 4) {
      float v[8];
      load8f(x + (int64_t)m * p.d + c, v);
      if (p.copy_out) {
        float *o = p.copy_out + (int64_t)m * p.d + c;
        *reinterpret_cast<f32x4 *>(o) = f32x4{v[0], v[1], v[2], v[3]};
        *reinterpret_cast<f32x4 *>(o + 4) = f32x4{v[4], v[5], v[6], v[7]};
      }
      const float r = 1.0f / sqrtf(((rs[m][0] + rs[m][1]) + (rs[m][2] + rs[m][3])) / (float)p.d + p.eps);
      bf16x8 o;
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = f2bf(v[i] * r * gv[i]);
      st16(p.y + (int64_t)m * p.d + c, as_u32x4(o));
      st16(&xs[m][8 * lane], as_u32x4(o));
    }
  }
  if constexpr (NB > 0) {
    __syncthreads();
    f32x4 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int tok = min(lane % 16, p.M - 1);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = 32 * (wave + 4 * u);
      if (!EARLY) load_a(u);
      if (k0 + k < kend) {  // uniform; (past the end LDS holds nothing)
        const bf16x8 xb = as_bf16x8(ld16(&xs[tok][k + kq]));
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b] = mfma16(ab[u][b], xb, acc[b]);
      }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) red[wave][b][lane] = acc[b];
    __syncthreads();
    const int m = lane % 16;
    for (int b = wave; b < NB; b += 4) {
      const f32x4 v = (red[0][b][lane] + red[1][b][lane]) + (red[2][b][lane] + red[3][b][lane]);
      if (m < p.M)
        *reinterpret_cast<f32x4 *>(p.part + ((int64_t)blockIdx.x * 16 + m) * (16 * NB) + b * 16 + (lane / 16) * 4) = v;
    }
  }
}

// Waves per workgroup (the K split inside one workgroup): enough waves in the
// whole grid to keep HBM busy when there are few 16-feature workgroups.
template <int EPI, int NB, int KB>
void go(hipStream_t s, int n_wg, const GemmParams &p) {
  const int CUS = p.n_cu > 0 ? p.n_cu : 256;  // compute units of the device
  // A long K over fewer workgroups than half the CUs (the down projection of
  // narrow models): K is split over workgroups too, two to a CU in all (1.5B
  // shapes, 96 workgroups: 14.5 -> 11.2 us).  With most CUs in use 16 waves on
  // each stream better than 8 twice (7B shapes, 224 workgroups: 28 against 35
  // us), and with a short K the tickets cost what the split gains.
  if constexpr (EPI == EPI_RESID) {
    int parts = 1;
    if (2 * n_wg <= CUS && p.K >= 4096 && p.tickets && n_wg <= p.n_tickets)
      parts = (int)std::min<int64_t>({2 * CUS / n_wg, SKINNY_MAX_PARTS, p.split_cap / (n_wg * NB * 256)});
    if (parts > 1) {
      GemmParams q = p;
      q.kpairs = (p.K / 64 + parts - 1) / parts;
      const dim3 grid(n_wg, (p.K / 64 + q.kpairs - 1) / q.kpairs);
      hipLaunchKernelGGL((gemm_skinny_kernel<EPI, NB, 8, KB, true>), grid, dim3(512), 0, s, q);
      return;
    }
  }
  // about 16 resident waves per CU: one round of 16-wave workgroups up to one
  // per CU, of 8-wave ones up to two per CU, else 4 waves (2 were no faster)
  if (n_wg > 2 * CUS)
    hipLaunchKernelGGL((gemm_skinny_kernel<EPI, NB, 4, KB, false>), dim3(n_wg), dim3(256), 0, s, p);
  else if (n_wg > CUS)
    hipLaunchKernelGGL((gemm_skinny_kernel<EPI, NB, 8, KB, false>), dim3(n_wg), dim3(512), 0, s, p);
  else
    hipLaunchKernelGGL((gemm_skinny_kernel<EPI, NB, 16, KB, false>), dim3(n_wg), dim3(1024), 0, s, p);
}

template <int EPI, int NB>
void launch_skinny(hipStream_t s, int n_wg, const GemmParams &p) {
  if (p.upart_n == 0)
    go<EPI, NB, 0>(s, n_wg, p);
  else if (p.rank <= 32)
    go<EPI, NB, 1>(s, n_wg, p);
  else
    go<EPI, NB, 2>(s, n_wg, p);
}

}  // namespace

hipError_t launch_gemm_skinny_bf16(hipStream_t s, GemmEpi epi, const GemmParams &p) {
  if (p.M <= 0 || p.N <= 0) return hipSuccess;
  if (p.M > 16 || p.K % 64 || (p.upart_n > 0 && (p.rank % 8 || p.rank > 64))) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_RESID:
      if (p.N % 4) return hipErrorInvalidValue;
      launch_skinny<EPI_RESID, 1>(s, (p.N + 15) / 16, p);
      break;
    case EPI_SWIGLU:
      if (p.d_ffn % 16) return hipErrorInvalidValue;
      launch_skinny<EPI_SWIGLU, 2>(s, p.d_ffn / 16, p);
      break;
    case EPI_QKV:
      if ((p.hd != 64 && p.hd != 128) || p.N % p.hd || p.seg1 % p.hd || p.seg2 % p.hd) return hipErrorInvalidValue;
      launch_skinny<EPI_QKV, 1>(s, p.N / 16, p);
      break;
  }
  return hipGetLastError();
}

int norm_lora_parts(int d) { return (d + 511) / 512; }

hipError_t launch_norm_lora(hipStream_t s, bool x_f32, const NormLora &p, int n_blocks) {
  if (p.M < 1 || p.M > 16 || p.d % 32) return hipErrorInvalidValue;
  const dim3 grid(norm_lora_parts(p.d));
#define CRF_NL(nb)                                                                             \
  case nb:                                                                                     \
    if (x_f32)                                                                                 \
      hipLaunchKernelGGL((norm_lora_kernel<float, nb>), grid, dim3(256), 0, s, p);             \
    else                                                                                       \
      hipLaunchKernelGGL((norm_lora_kernel<bf16, nb>), grid, dim3(256), 0, s, p);              \
    break;
  switch (n_blocks) {  // {1, 2, 3} targets x 16-row blocks per rank {1, 2, 3, 4}
    CRF_NL(0) CRF_NL(1) CRF_NL(2) CRF_NL(3) CRF_NL(4) CRF_NL(6) CRF_NL(8) CRF_NL(9) CRF_NL(12)
    default: return hipErrorInvalidValue;
  }
#undef CRF_NL
  return hipGetLastError();
}

}  // namespace crf
