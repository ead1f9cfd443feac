// bf16 projections of 17 token rows and more, with large adapters of 13 (a short
// prefix, the new tokens of a decoding step), up to where the large tiles win (mid_rows in api.cpp: about 600
// rows of 7B shapes, 1800 of 1.5B, several thousand of small decoders, fewer with
// large adapters).  There 256x256 tiles leave most CUs without
// one and the weights, read once, are a large share of the time, so the tiles
// are 128 weight rows x 64 or 128 tokens, two or three workgroups per CU, and
// K is split over workgroups until every CU has its share.
//
// QKV, O and down write fp32 K-parts [part][M][rows]; one kernel then sums the
// parts of a token in order and does everything that follows on that token:
//   reduce_qkv    adapter delta, bias, rotary rotation, Q buffer, K/V pages;
//   reduce_resid  adapter delta, residual update, RMSNorm of the next block.
// The adapters' A rows are weight rows like any other, appended to the base
// rows, so U comes out of the same launch.  Gate/up has rows enough unsplit:
// its SwiGLU (and its adapters' delta, from a U formed before) is the epilogue.
//
// What bounds it: the weights' bytes at the shortest counts, above that the
// latency of a tile's slices with one or two workgroups on a CU, and the chain
// of launches (seven a layer, without adapters on gate/up).  Two layers of
// 1.5B shapes (rank 16 on q, k, v, o) over 17 / 200 / 1024 tokens: 291 / 315 /
// 485 -> 127 / 190 / 410 us; of 7B shapes (rank 16 on all) over 17 / 200 / 512
// tokens: 622 / 673 / 938 -> 354 / 540 / 831 us.
#include <algorithm>
#include <type_traits>

#include "kernels.hpp"

namespace crf {
namespace {

constexpr int BN = 128, BK = 64, STAGES = 2;

// 16-byte chunk c of slice row r sits at position c ^ (r / 2) % 8: conflict-free
// fragment reads (16 rows of one chunk on 16 bank groups).
CRF_DEV int swz(int row, int chunk) { return row * BK + ((chunk ^ ((row >> 1) & 7)) << 3); }

// Source segment and row of tile-space row r.  Gate/up: within each wave's 64
// rows 32 gate rows, then the 32 up rows of the same features.
template <bool GU>
CRF_DEV int mid_row(const MidGemm &p, int r, int &local) {
  if (GU) {
    local = (r >> 7) * 64 + ((r >> 6) & 1) * 32 + (r & 31);
    return (r >> 5) & 1;
  }
  int s = 0, first = 0;
#pragma unroll
  for (int i = 0; i < MID_SEGS - 1; ++i)
    if (r >= p.seg_end[i]) {
      s = i + 1;
      first = p.seg_end[i];
    }
  local = r - first;
  return s;
}

// Tile (tm, tn) and K-part of workgroup b: consecutive items (token tiles of
// one weight panel and part) go to one XCD, which fetches the panel once.
CRF_DEV void mid_item(const MidGemm &p, int b, int n, int &tm, int &tn, int &part) {
  const int x = b % 8, q = n / 8, r = n % 8;
  int i = x * q + min(x, r) + b / 8;
  tm = i % p.tiles_m;
  i /= p.tiles_m;
  part = i % p.parts;
  tn = i / p.parts;
}

// 4 waves, wave (wn, wm): 64 rows x 32 NJ tokens.
template <bool GU, int NJ>
__global__ __launch_bounds__(256, NJ == 2 ? 2 : 3) void gemm_mid_kernel(const MidGemm p) {
  constexpr int BM = 64 * NJ;
  constexpr int WB = BN / 8 / 4, XB = BM / 8 / 4;  // 1 KB DMA blocks (8 rows) per wave and slice
  extern __shared__ __align__(16) bf16 smem[];
  bf16 *const lds_x = smem, *const lds_w = smem + STAGES * BM * BK;
  const int tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int wn = wave / 2, wm = wave % 2, g = lane / 32, l32 = lane % 32;
  int tm, tn, part;
  mid_item(p, blockIdx.x, gridDim.x, tm, tn, part);
  const int m0 = tm * BM, n0 = tn * BN, nk = p.K / BK;
  const int kb = part * nk / p.parts, ke = (part + 1) * nk / p.parts;

  // DMA: wave w moves the 8-row blocks 4 j + w; lane L writes 16 bytes, row
  // L / 8, position L % 8.  Rows past the end arrive as zeros.
  const __amdgpu_buffer_rsrc_t xres = make_rsrc(p.X, (uint32_t)((int64_t)p.M * p.ldx * 2));
  uint32_t xoff[XB], woff[WB];
  __amdgpu_buffer_rsrc_t wres[WB];
#pragma unroll
  for (int j = 0; j < XB; ++j) {
    const int row = (4 * j + wave) * 8 + lane / 8, c = (lane % 8) ^ ((row >> 1) & 7), m = m0 + row;
    xoff[j] = m < p.M ? (uint32_t)(((int64_t)m * p.ldx + c * 8) * 2) : CRF_OOB;
  }
#pragma unroll
  for (int j = 0; j < WB; ++j) {
    const int blk = 4 * j + wave, row = blk * 8 + lane / 8, c = (lane % 8) ^ ((row >> 1) & 7);
    int l0, local;
    const int sg = mid_row<GU>(p, min(n0 + blk * 8, p.N - 1), l0);  // a block lies in one segment
    mid_row<GU>(p, min(n0 + row, p.N - 1), local);
    wres[j] = make_rsrc(p.w[sg], (uint32_t)((int64_t)p.w_rows[sg] * p.K * 2));
    woff[j] = n0 + row < p.N ? (uint32_t)(((int64_t)local * p.K + c * 8) * 2) : CRF_OOB;
  }
  auto produce = [&](int k, int stage) {
    const uint32_t k0 = (uint32_t)k * BK * 2;
    lds_char *dx = (lds_char *)(lds_x + stage * BM * BK), *dw = (lds_char *)(lds_w + stage * BN * BK);
#pragma unroll
    for (int j = 0; j < WB; ++j) dma16(wres[j], dw + (4 * j + wave) * 1024, woff[j], k0);
#pragma unroll
    for (int j = 0; j < XB; ++j) dma16(xres, dx + (4 * j + wave) * 1024, xoff[j], k0);
  };
  f32x16 acc[2][NJ];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  auto frag = [&](int stage, int s, bf16x8 (&fa)[2], bf16x8 (&fb)[NJ]) {
    const bf16 *sx = lds_x + stage * BM * BK, *sw = lds_w + stage * BN * BK;
#pragma unroll
    for (int i = 0; i < 2; ++i) fa[i] = as_bf16x8(ld16(sw + swz(wn * 64 + 32 * i + l32, 2 * s + g)));
#pragma unroll
    for (int j = 0; j < NJ; ++j) fb[j] = as_bf16x8(ld16(sx + swz(wm * 32 * NJ + 32 * j + l32, 2 * s + g)));
  };
  auto mm = [&](bf16x8 (&fa)[2], bf16x8 (&fb)[NJ]) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = mfma32(fa[i], fb[j], acc[i][j]);
  };
  // one MFMA, one LDS read (and, where they are issued, one DMA) in turn
  auto interleave = [&](auto n_dma) {
    constexpr int ND = decltype(n_dma)::value;
#pragma unroll
    for (int i = 0; i < 2 * NJ; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (2 * i < ND) __builtin_amdgcn_sched_group_barrier(0x020, 2, 0);
      if (i < 2 + NJ) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  constexpr int PER_SLICE = WB + XB;
  produce(kb, 0);
  if (kb + 1 < ke) {
    produce(kb + 1, 1);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER_SLICE) : "memory");
  } else {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  asm volatile("s_barrier" ::: "memory");
  bf16x8 a0[2], b0[NJ], a1[2], b1[NJ];
  frag(0, 0, a0, b0);
  // One slice: its fragments are read one k-step ahead; the last step's MFMAs
  // follow the barrier that ends all reads of the stage, next to its refill
  // (slices before the last two) and the next slice's first reads.
  int st = 0;
  auto slice = [&](int kt, auto left_t) {
    constexpr int LEFT = decltype(left_t)::value;  // slices after this one: 0, 1, or 2 and more
    __builtin_amdgcn_sched_barrier(0);
    frag(st, 1, a1, b1);
    mm(a0, b0);
    interleave(std::integral_constant<int, 0>());
    frag(st, 2, a0, b0);
    mm(a1, b1);
    interleave(std::integral_constant<int, 0>());
    frag(st, 3, a1, b1);
    mm(a0, b0);
    interleave(std::integral_constant<int, 0>());
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (LEFT >= 2) produce(kt + 2, st);
    if constexpr (LEFT >= 1) frag(st ^ 1, 0, a0, b0);
    mm(a1, b1);
    interleave(std::integral_constant<int, LEFT >= 2 ? PER_SLICE : 0>());
    st ^= 1;
  };
  int kt = kb;
  for (; kt + 2 < ke; ++kt) slice(kt, std::integral_constant<int, 2>());
  if (kt + 1 < ke) slice(kt++, std::integral_constant<int, 1>());
  slice(kt, std::integral_constant<int, 0>());

  if (!GU) {
    float *pp = p.part + (int64_t)part * p.M * p.N;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int m = m0 + wm * 32 * NJ + 32 * j + l32;
      if (m >= p.M) continue;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int n = n0 + wn * 64 + 32 * i + 8 * q + 4 * g;
          if (n < p.N)
            *reinterpret_cast<f32x4 *>(pp + (int64_t)m * p.N + n) =
                f32x4{acc[i][j][q * 4], acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2], acc[i][j][q * 4 + 3]};
        }
    }
    return;
  }
  // ---- gate/up: adapter delta, then act = silu(gate) * up
  const int f0 = tn * 64 + wn * 32;  // first feature of the wave
  if (p.U) {
    for (int kk = 0; kk < p.rank; kk += 16) {
      const int k = kk + 8 * g;
      bf16x8 lbf[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        u32x4 v = {0u, 0u, 0u, 0u};
        if (p.lb[i] && k < p.rank) v = ld16(p.lb[i] + (int64_t)(f0 + l32) * p.rank + k);
        lbf[i] = as_bf16x8(v);
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int m = min(m0 + wm * 32 * NJ + 32 * j + l32, p.M - 1);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          // (past the rank the factor is zero, and U may end there)
          u32x4 u = {0u, 0u, 0u, 0u};
          if (k < p.rank) u = ld16(p.U + (int64_t)m * p.ldu + p.ucol[i] + k);
          acc[i][j] = mfma32(lbf[i], as_bf16x8(u), acc[i][j]);
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int m = m0 + wm * 32 * NJ + 32 * j + l32;
    if (m >= p.M) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float gt = acc[0][j][q * 4 + e], up = acc[1][j][q * 4 + e];
        o[e] = gt * __builtin_amdgcn_rcpf(1.0f + __expf(-gt)) * up;
      }
      st8(p.act + (int64_t)m * p.d_ffn + f0 + 8 * q + 4 * g, pack_bf16x4(o[0], o[1], o[2], o[3]));
    }
  }
}

// ---- reductions.  U of a token: the summed parts of its adapter columns
// (after the base rows), scaled and rounded to bf16 as the large-M path stores
// it; the delta of a feature is the fp32 dot product with its factor row.

typedef float f32x2 __attribute__((ext_vector_type(2)));

// v[i] = sum over the parts, in order, of the values at p[i]: the parts are the
// outer loop, so that the loads of UP parts of every value go out together.
template <int UP, int N, typename V>
CRF_DEV void sum_parts(const float *const (&p)[N], int64_t stride, int parts, V (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = *reinterpret_cast<const V *>(p[i]);
  for (int s = 1; s < parts; s += UP) {
    V t[UP][N];
#pragma unroll
    for (int q = 0; q < UP; ++q)
#pragma unroll
      for (int i = 0; i < N; ++i) t[q][i] = *reinterpret_cast<const V *>(p[i] + min(s + q, parts - 1) * stride);
#pragma unroll
    for (int q = 0; q < UP; ++q)
      if (s + q < parts)
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] += t[q][i];
  }
}

// U of R tokens from m0, in two steps so that the loads of a row's own parts
// can go out in between: columns c .. c + 4 of token r of thread i < R * n_u / 4.
template <int R>
struct ULoad {
  static constexpr int NK = (R * 3 * 64 / 4 + 255) / 256;
  f32x4 u[NK];
  CRF_DEV void load(const MidReduce &p, int m0) {
    const int n4 = p.n_u / 4;
    const float *q[NK];
#pragma unroll
    for (int k = 0; k < NK; ++k) {  // threads past the end repeat the last item
      const int i = min((int)threadIdx.x + 256 * k, R * n4 - 1);
      q[k] = p.part + (int64_t)min(m0 + i / n4, p.M - 1) * p.ld + p.n_base + 4 * (i % n4);
    }
    sum_parts<4>(q, (int64_t)p.M * p.ld, p.parts, u);
  }
  CRF_DEV void store(const MidReduce &p, float (&ush)[R][3 * 64]) {
    const int n4 = p.n_u / 4;
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const int i = threadIdx.x + 256 * k;
      if (i >= R * n4) break;
#pragma unroll
      for (int e = 0; e < 4; ++e) ush[i / n4][4 * (i % n4) + e] = bf2f(f2bf(u[k][e] * p.scale));
    }
    __syncthreads();
  }
};

// v[r] += sum_k lb[row, k] ush[r][col + k] for 2 consecutive rows (a wave then
// reads 128 consecutive factor rows, which its cache holds while it walks k)
template <int R>
CRF_DEV void add_delta(const MidReduce &p, const bf16 *lb, int row, int col, const float (&ush)[R][3 * 64],
                       f32x2 (&v)[R]) {
  if (!lb) return;
  for (int k = 0; k < p.rank; k += 8) {
    bf16x8 b[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) b[i] = as_bf16x8(ld16(lb + (int64_t)(row + i) * p.rank + k));
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const float u = ush[r][col + k + e];
#pragma unroll
        for (int i = 0; i < 2; ++i) v[r][i] = fmaf(bf2f(b[i][e]), u, v[r][i]);
      }
  }
}

CRF_DEV f32x2 ld_bf16x2(const bf16 *p) {
  const uint32_t v = *reinterpret_cast<const uint32_t *>(p);
  return f32x2{__builtin_bit_cast(float, v << 16), __builtin_bit_cast(float, v & 0xffff0000u)};
}
CRF_DEV void st_bf16x2(bf16 *p, f32x2 v) {
  const bf16x2 o = {f2bf(v[0]), f2bf(v[1])};
  *reinterpret_cast<bf16x2 *>(p) = o;
}

// One thread: 2 in-head features and their rotary partners, for R tokens.
template <int R>
__global__ __launch_bounds__(256) void reduce_qkv_kernel(const MidReduce p) {
  __shared__ float ush[R][3 * 64];
  const int m0 = blockIdx.x * R;
  ULoad<R> ul;
  if (p.n_u) ul.load(p, m0);
  const int t = blockIdx.y * 256 + threadIdx.x, half = p.hd / 2, per = half / 2;
  const int head = t / per, f = 2 * (t % per), n = head * p.hd + f;
  const bool on = n < p.n_base;
  const int64_t stride = (int64_t)p.M * p.ld;
  f32x2 x[2 * R], x1[R], x2[R];
  const float *src[2 * R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    src[r] = p.part + (int64_t)min(m0 + r, p.M - 1) * p.ld + (on ? n : 0);
    src[R + r] = src[r] + half;
  }
  sum_parts<4>(src, stride, p.parts, x);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    x1[r] = x[r];
    x2[r] = x[R + r];
  }
  if (p.n_u) ul.store(p, ush);
  if (!on) return;
  const int sg = n < p.seg1 ? 0 : (n < p.seg2 ? 1 : 2);
  const int local = n - (sg == 0 ? 0 : (sg == 1 ? p.seg1 : p.seg2));
  if (p.n_u) {
    add_delta<R>(p, p.lb[sg], local, p.ucol[sg], ush, x1);
    add_delta<R>(p, p.lb[sg], local + half, p.ucol[sg], ush, x2);
  }
  const bf16 *bias = p.bias[sg];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int m = m0 + r;
    if (m >= p.M) break;
    f32x2 y1 = x1[r], y2 = x2[r];
    if (bias) {  // (a bias may start at any element)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        y1[i] += bf2f(bias[local + i]);
        y2[i] += bf2f(bias[local + half + i]);
      }
    }
    if (sg < 2) {
      const float2 *cs = p.rope_cs + (int64_t)(p.pos0 + m) * half + f;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float2 c = cs[i];
        const float a = y1[i] * c.x - y2[i] * c.y, b = y2[i] * c.x + y1[i] * c.y;
        y1[i] = a;
        y2[i] = b;
      }
    }
    bf16 *dst;
    if (sg == 0) {
      dst = p.q_out + (int64_t)m * p.dq + local;
      y1 *= p.q_scale;
      y2 *= p.q_scale;
    } else {
      const int64_t row = paged_row(p.kv, p.pos0 + m, local / p.hd, p.hd);
      if (row < 0) continue;
      dst = (bf16 *)(sg == 1 ? p.kv.k : p.kv.v) + row + f;
    }
    st_bf16x2(dst, y1);
    st_bf16x2(dst + half, y2);
  }
}

// One workgroup: R whole rows (n_base <= 512 NV), so the row's RMSNorm for the
// next block comes with it.
template <int R, int NV>
__global__ __launch_bounds__(256) void reduce_resid_kernel(const MidReduce p) {
  __shared__ float ush[R][3 * 64];
  __shared__ float ssh[4][R];
  const int m0 = blockIdx.x * R;
  ULoad<R> ul;
  if (p.n_u) ul.load(p, m0);
  const int64_t stride = (int64_t)p.M * p.ld;
  f32x2 v[NV][R], x[NV * R], old[NV * R];
  const float *src[NV * R];
#pragma unroll
  for (int c = 0; c < NV; ++c)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int m = min(m0 + r, p.M - 1), n = min(512 * c + 2 * (int)threadIdx.x, p.n_base - 2);
      const int64_t o = (int64_t)m * p.n_base + n;
      src[c * R + r] = p.part + (int64_t)m * p.ld + n;
      old[c * R + r] = p.resid_in ? ld_bf16x2(p.resid_in + o) : *reinterpret_cast<const f32x2 *>(p.resid + o);
    }
  sum_parts<(NV * R <= 4 ? 4 : NV * R <= 8 ? 2 : 1)>(src, stride, p.parts, x);
#pragma unroll
  for (int c = 0; c < NV; ++c)
#pragma unroll
    for (int r = 0; r < R; ++r) v[c][r] = x[c * R + r] + old[c * R + r];
  if (p.n_u) ul.store(p, ush);
  float ss[R];
#pragma unroll
  for (int r = 0; r < R; ++r) ss[r] = 0.f;
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    const int n = 512 * c + 2 * threadIdx.x;
    if (n >= p.n_base) continue;
    if (p.n_u) add_delta<R>(p, p.lb[0], n, 0, ush, v[c]);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      ss[r] = fmaf(v[c][r][0], v[c][r][0], fmaf(v[c][r][1], v[c][r][1], ss[r]));
      if (m0 + r >= p.M) continue;
      const int64_t o = (int64_t)(m0 + r) * p.n_base + n;
      if (p.resid_out)
        st_bf16x2(p.resid_out + o, v[c][r]);
      else
        *reinterpret_cast<f32x2 *>(p.resid + o) = v[c][r];
    }
  }
  if (!p.gain) return;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const float s = wave_sum(ss[r]);
    if (threadIdx.x % 64 == 0) ssh[threadIdx.x / 64][r] = s;
  }
  __syncthreads();
  float k[R];
#pragma unroll
  for (int r = 0; r < R; ++r)
    k[r] = 1.0f / sqrtf(((ssh[0][r] + ssh[1][r]) + (ssh[2][r] + ssh[3][r])) / (float)p.n_base + p.eps);
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    const int n = 512 * c + 2 * threadIdx.x;
    if (n >= p.n_base) continue;
    const f32x2 gv = ld_bf16x2(p.gain + n);
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (m0 + r < p.M) st_bf16x2(p.xn + (int64_t)(m0 + r) * p.n_base + n, v[c][r] * k[r] * gv);
  }
}

}  // namespace

// Token tiles of 64 up to these counts, of 128 from there on (2 layers of 7B
// shapes): a product whose K is split has its slots filled by parts and reads
// each weight once per token tile, so it keeps 64 only up to two of them (100
// tokens: 429 against 446 us, 200 tokens: 575 against 558); unsplit gate/up
// fills the slots with them up to four (256 tokens: 601 against 636 us, 300
// tokens: 629 against 600).
constexpr int SMALL_SPLIT = 128, SMALL_GATE_UP = 256;
constexpr int ONE_ROW = 512;  // tokens up to which the reductions take one per thread

int mid_parts(int M, int N, int K, int n_cu, int64_t part_floats) {
  const int bm = M <= SMALL_SPLIT ? 64 : 128;
  const int tiles = ((M + bm - 1) / bm) * ((N + BN - 1) / BN);
  // fill the resident slots (two workgroups per CU), at least 4 slices a part
  const int64_t s = std::min<int64_t>({2 * n_cu / std::max(tiles, 1), K / BK / 4, part_floats / ((int64_t)M * N), 16});
  return (int)std::max<int64_t>(1, s);
}

hipError_t launch_gemm_mid(hipStream_t s, bool gate_up, const MidGemm &p0) {
  MidGemm p = p0;
  if (p.M <= 0 || p.N <= 0) return hipSuccess;
  if (p.K % BK || p.parts < 1 || (int64_t)p.M * p.ldx * 2 >= (int64_t)CRF_OOB) return hipErrorInvalidValue;
  const bool small = p.M <= (gate_up ? SMALL_GATE_UP : SMALL_SPLIT);
  p.tiles_m = small ? (p.M + 63) / 64 : (p.M + 127) / 128;
  const int tiles_n = (p.N + BN - 1) / BN;
  const dim3 grid(p.tiles_m * tiles_n * p.parts);
  const size_t lds = (size_t)STAGES * ((small ? 64 : 128) + BN) * BK * 2;  // at most 64 KB
  if (gate_up) {
    if (small)
      hipLaunchKernelGGL((gemm_mid_kernel<true, 1>), grid, dim3(256), lds, s, p);
    else
      hipLaunchKernelGGL((gemm_mid_kernel<true, 2>), grid, dim3(256), lds, s, p);
  } else {
    if (small)
      hipLaunchKernelGGL((gemm_mid_kernel<false, 1>), grid, dim3(256), lds, s, p);
    else
      hipLaunchKernelGGL((gemm_mid_kernel<false, 2>), grid, dim3(256), lds, s, p);
  }
  return hipGetLastError();
}

hipError_t launch_mid_reduce_qkv(hipStream_t s, const MidReduce &p) {
  const int threads = p.n_base / 4;
  // several tokens a thread read the factor rows once for them; a few rows want the threads
  if (p.M <= ONE_ROW)
    hipLaunchKernelGGL((reduce_qkv_kernel<1>), dim3(p.M, (threads + 255) / 256), dim3(256), 0, s, p);
  else
    hipLaunchKernelGGL((reduce_qkv_kernel<4>), dim3((p.M + 3) / 4, (threads + 255) / 256), dim3(256), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_mid_reduce_resid(hipStream_t s, const MidReduce &p) {
#define CRF_RR(nv)                                                                                      \
  if (p.n_base <= 512 * nv) {                                                                           \
    if (p.M <= ONE_ROW)                                                                                     \
      hipLaunchKernelGGL((reduce_resid_kernel<1, nv>), dim3(p.M), dim3(256), 0, s, p);                  \
    else                                                                                                \
      hipLaunchKernelGGL((reduce_resid_kernel<2, nv>), dim3((p.M + 1) / 2), dim3(256), 0, s, p);        \
    return hipGetLastError();                                                                           \
  }
  CRF_RR(2) CRF_RR(3) CRF_RR(4) CRF_RR(7) CRF_RR(10) CRF_RR(16)
#undef CRF_RR
  return hipErrorInvalidValue;
}

}  // namespace crf
