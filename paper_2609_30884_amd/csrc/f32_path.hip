// fp32 storage path (small decoders): the projections of a layer with their
// RMSNorm, adapter, rotary, SwiGLU and residual work fused around one fp32 MFMA
// kernel, and a causal attention on the same instruction.  Every product and
// sum is fp32 (v_mfma_f32_16x16x4_f32).
//
// What bounds it: at these widths a layer is a few MFLOP to 1 GFLOP per
// launch, so the number of dependent launches and the latency inside each
// count, not the matrix rate.  Five launches per layer (QKV, attention, O,
// gate/up, down) where one kernel per operation took 20; every launch splits K
// over the waves of a workgroup so that its chain of loads stays short.
// Measured: 2 layers of d = 256 over 128 tokens (rank 8 on q, k, v, o) 966 ->
// 66 us, 4 layers over 1511 tokens (rank 8 on all seven) 4399 -> 473 us (30
// TFLOP/s); attention over the 1511 tokens 505 -> 42 us per layer.  Matrix cores
// are 31 % busy while a CU has work there: the rest is the start of each launch,
// whose waves all load first and multiply after.
#include <math.h>

#include "kernels.hpp"

namespace crf {
namespace {

CRF_DEV f32x4 mfma_f32(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
CRF_DEV f32x4 ldf4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }
constexpr f32x4 ZERO4 = {0.f, 0.f, 0.f, 0.f};
// Tiles of 2 x 2 blocks (32 rows x 32 tokens) up to which each token half is a
// tile of its own: below one tile per CU the chain inside a tile is the time
// (2 layers of d = 256 over 128 tokens: 81 us with 2 x 2, 66 us with 2 x 1).
constexpr int F32_FEW_TILES = 256;
// ... and from which 4 x 4 blocks take over (1511 tokens, d_ffn = 704, 2112
// tiles: 557 us a pass with 4 x 4 in gate/up, 584 us with 2 x 2; taken from 512
// tiles on it is 590 us, the last wave of tiles being too thin).
constexpr int F32_BIG_TILES = 2048;

// Weight row of tile row `i` (0..15) in block b of feature tile tn, its LoRA
// target, and whether it exists (rows past the end are clamped, never stored).
// Blocks come in pairs (b, b + FB/2) that share their columns' consumers: gate
// and up rows of the same feature, or the rotary partners f and f + hd/2 of one
// head; a tile therefore lies in one head.
template <int EPI, int FB>
CRF_DEV void tile_row(const F32Gemm &p, int tn, int b, int i, int &seg, int &row) {
  if (EPI == F32_SWIGLU) {
    seg = b / (FB / 2);
    row = tn * 8 * FB + 16 * (b % (FB / 2)) + i;
  } else if (EPI == F32_QKV) {
    const int half = p.hd / 2, per_head = half / (8 * FB);
    const int head = tn / per_head;
    const int r = head * p.hd + (tn % per_head) * 8 * FB + 16 * (b % (FB / 2)) + (b / (FB / 2)) * half;
    seg = r < p.seg1 ? 0 : (r < p.seg2 ? 1 : 2);
    row = r - (seg == 0 ? 0 : (seg == 1 ? p.seg1 : p.seg2)) + i;
  } else {
    seg = 0;
    row = tn * 16 * FB + 16 * b + i;
  }
}

// Workgroup: FB blocks of 16 weight rows x TB blocks of 16 tokens, NW waves
// splitting K in steps of 16 (wave w takes steps w, w + NW, ...).  A lane loads
// 4 consecutive k of its row, and MFMA i of a step multiplies element i of both
// operands: the k order is permuted the same way on both sides.  With a norm
// gain the tokens are multiplied by it as they are loaded, their squares are
// summed alongside (the workgroup sees every k of its tokens), and the row
// factor 1/rms multiplies the sums at the end.  LORA = 1: the adapter's rank rows
// (rank <= 16) are one more block per target, so U never leaves the workgroup;
// LORA = 2 (rank <= 8): gate's are rows 0-7 and up's rows 8-15 of one block, a
// sixth of a 4 x 4 tile's products less (1511 tokens, d_ffn = 704: 39.6 -> 34.3
// us); larger ranks read U from memory (formed
// by the F32_PLAIN launch).
// Small tiles (2 x 1 or 2 x 2 blocks, 4 waves) keep a few hundred rows spread
// over the CUs; big ones (4 x 4 blocks, 2 waves) read half the bytes per FLOP.
template <int EPI, int FB, int TB, int NW, int LORA>
__global__ __launch_bounds__(64 * NW) void gemm_f32_kernel(const F32Gemm p) {
  constexpr bool PACK = LORA == 2;
  constexpr int XB = LORA ? (EPI == F32_SWIGLU && !PACK ? 2 : 1) : 0;  // adapter blocks
  constexpr int NB = FB + XB;
  constexpr int UNROLL = FB * TB <= 4 ? 2 : 1;  // k-steps per batch; two batches in flight
  __shared__ f32x4 red[NW][NB * TB][64];
  __shared__ float ssred[NW][TB][64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int r16 = lane % 16, kg = lane / 16;
  const int tn = blockIdx.x, m0 = blockIdx.y * 16 * TB;
  // row offsets in elements from the tensors' bases.  Every load is
  // unconditional: rows past the end repeat the last one (never stored), rank
  // rows past the rank repeat the last one (their factor column is zero), and
  // an absent adapter's block reads weight rows that nothing uses.
  const float *xp[TB], *wp[NB];
#pragma unroll
  for (int t = 0; t < TB; ++t) xp[t] = p.x + (int64_t)min(m0 + 16 * t + r16, p.M - 1) * p.ldx;
  int seg0 = 0, seg1 = 0;
#pragma unroll
  for (int b = 0; b < FB; ++b) {
    int seg, row;
    tile_row<EPI, FB>(p, tn, b, r16, seg, row);
    if (b == 0) seg0 = seg;
    if (b == FB - 1) seg1 = seg;
    wp[b] = p.w[seg] + (int64_t)min(row, p.seg_rows[seg] - 1) * p.K;
  }
#pragma unroll
  for (int x = 0; x < XB; ++x) {
    const float *a = p.la[(PACK ? r16 >= 8 : x > 0) ? seg1 : seg0];
    wp[FB + x] = a ? a + (int64_t)min(PACK ? r16 % 8 : r16, p.rank - 1) * p.K : wp[0];
  }
  f32x4 acc[NB][TB];
  float ss[TB];
#pragma unroll
  for (int t = 0; t < TB; ++t) {
    ss[t] = 0.f;
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b][t] = ZERO4;
  }
  const int nsteps = (p.K + 15) / 16;
  const bool norm = p.gain != nullptr;
  struct Batch {
    f32x4 w[UNROLL][NB], x[UNROLL][TB], g[UNROLL];
  };
  auto load = [&](int st, Batch &q) {
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      // this lane's 4 k; past the end (K is a multiple of 4) the last 4, dropped in `mul`
      const int k = min((st + NW * u) * 16 + 4 * kg, p.K - 4);
#pragma unroll
      for (int t = 0; t < TB; ++t) q.x[u][t] = ldf4(xp[t] + k);
#pragma unroll
      for (int b = 0; b < NB; ++b) q.w[u][b] = ldf4(wp[b] + k);
      if (norm) q.g[u] = ldf4(p.gain + k);
    }
  };
  auto mul = [&](int st, Batch &q) {
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int k = (st + NW * u) * 16;
      if (k >= p.K) break;   // uniform
      if (k + 16 > p.K) {    // the last, partial step
        const bool in = k + 4 * kg < p.K;
#pragma unroll
        for (int t = 0; t < TB; ++t) q.x[u][t] = in ? q.x[u][t] : ZERO4;
#pragma unroll
        for (int b = 0; b < NB; ++b) q.w[u][b] = in ? q.w[u][b] : ZERO4;
      }
      if (norm) {
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            ss[t] = fmaf(q.x[u][t][i], q.x[u][t][i], ss[t]);
            q.x[u][t][i] *= q.g[u][i];
          }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int t = 0; t < TB; ++t) acc[b][t] = mfma_f32(q.w[u][b][i], q.x[u][t][i], acc[b][t]);
    }
  };
  constexpr int STRIDE = NW * UNROLL;
  // what the epilogue of this wave's first token block reads, loaded ahead of
  // the products: the adapter's output factor rows (fused ranks), the old residual
  f32x4 lbv[FB], rin[FB];
  const int m1 = min(m0 + 16 * wave + r16, p.M - 1);
  if (wave < TB) {
#pragma unroll
    for (int b = 0; b < FB; ++b) {
      int seg, row;
      tile_row<EPI, FB>(p, tn, b, r16, seg, row);
      if (LORA && p.lb[seg]) {
        const float *lb = p.lb[seg] + (int64_t)min(row, p.seg_rows[seg] - 1) * p.rank;
        const int j = PACK ? (kg / 2 == (b >= FB / 2) ? 4 * (kg % 2) : p.rank) : 4 * kg;
#pragma unroll
        for (int i = 0; i < 4; ++i) lbv[b][i] = j + i < p.rank ? lb[j + i] : 0.f;
      }
      if (EPI == F32_RESID)
        rin[b] = ldf4(p.resid_in + (int64_t)m1 * p.ldo + min(tn * 16 * FB + 16 * b + 4 * kg, p.seg_rows[0] - 4));
    }
  }
  Batch qa, qb;
  load(wave, qa);
  for (int st = wave; st < nsteps; st += 2 * STRIDE) {
    load(st + STRIDE, qb);
    mul(st, qa);
    load(st + 2 * STRIDE, qa);
    mul(st + STRIDE, qb);
  }
#pragma unroll
  for (int t = 0; t < TB; ++t) {
    ssred[wave][t][lane] = ss[t];
#pragma unroll
    for (int b = 0; b < NB; ++b) red[wave][b * TB + t][lane] = acc[b][t];
  }
  __syncthreads();
  // wave w finishes token blocks w, w + NW, ...
  for (int t = wave; t < TB; t += NW) {
    const int m = m0 + 16 * t + r16;
    f32x4 v[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      v[b] = red[0][b * TB + t][lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) v[b] += red[w][b * TB + t][lane];
    }
    if (norm) {
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w)
#pragma unroll
        for (int q = 0; q < 4; ++q) s += ssred[w][t][16 * q + r16];
      const float r = 1.0f / sqrtf(s / (float)p.K + p.eps);
#pragma unroll
      for (int b = 0; b < NB; ++b) v[b] *= r;
    }
    // adapter: v[b] += B[row, :rank] . U[:rank, token]; U sits in the lanes as
    // the MFMA's token operand already (rank 4 kg + i in element i)
    if (EPI != F32_PLAIN && p.rank > 0) {
      for (int kk = 0; kk < p.rank; kk += 16) {
        f32x4 u[2];
#pragma unroll
        for (int x = 0; x < (EPI == F32_SWIGLU ? 2 : 1); ++x) {
          const int seg = x ? seg1 : seg0;
          if (LORA) {  // (rows past the rank, and PACK's other target, take no part: 0 times an infinity would)
            const bool own = !PACK || kg / 2 == x;
#pragma unroll
            for (int i = 0; i < 4; ++i)
              u[x][i] = own && 4 * (PACK ? kg % 2 : kg) + i < p.rank ? v[FB + (XB > 1 ? x : 0)][i] * p.scale : 0.f;
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int j = kk + 4 * kg + i;
              u[x][i] = p.lb[seg] && j < p.rank ? p.U[(int64_t)min(m, p.M - 1) * p.ldu + seg * p.rank + j] : 0.f;
            }
          }
        }
#pragma unroll
        for (int b = 0; b < FB; ++b) {
          int seg, row;
          tile_row<EPI, FB>(p, tn, b, r16, seg, row);
          const float *lb = p.lb[seg];
          if (!lb) continue;  // uniform: a tile's block lies in one segment
          lb += (int64_t)min(row, p.seg_rows[seg] - 1) * p.rank;
          const f32x4 ub = EPI == F32_SWIGLU && b >= FB / 2 ? u[1] : u[0];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int j = kk + 4 * kg + i;
            v[b] = mfma_f32(LORA ? lbv[b][i] : (j < p.rank ? lb[j] : 0.f), ub[i], v[b]);
          }
        }
      }
    }
    if (m >= p.M) continue;
    // epilogues: the lane holds rows 4 kg .. 4 kg + 3 of each block, token m
    if (EPI == F32_PLAIN) {  // U[m, row] = scale * v
#pragma unroll
      for (int b = 0; b < FB; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = tn * 16 * FB + 16 * b + 4 * kg + i;
          if (row < p.seg_rows[0]) p.out[(int64_t)m * p.ldo + row] = v[b][i] * p.scale;
        }
    } else if (EPI == F32_RESID) {
#pragma unroll
      for (int b = 0; b < FB; ++b) {
        const int row = tn * 16 * FB + 16 * b + 4 * kg;
        if (row >= p.seg_rows[0]) continue;  // rows are a multiple of 8
        const int64_t o = (int64_t)m * p.ldo + row;
        *reinterpret_cast<f32x4 *>(p.out + o) = (t == wave ? rin[b] : ldf4(p.resid_in + o)) + v[b];
      }
    } else if (EPI == F32_SWIGLU) {
#pragma unroll
      for (int b = 0; b < FB / 2; ++b) {
        const int row = tn * 8 * FB + 16 * b + 4 * kg;
        if (row >= p.seg_rows[0]) continue;
        f32x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float g = v[b][i];
          o[i] = g / (1.0f + expf(-g)) * v[b + FB / 2][i];
        }
        *reinterpret_cast<f32x4 *>(p.out + (int64_t)m * p.ldo + row) = o;
      }
    } else {  // F32_QKV: bias, rotation of Q and K, Q to its buffer, K and V to their pages
#pragma unroll
      for (int b = 0; b < FB / 2; ++b) {
        int seg, row;
        tile_row<EPI, FB>(p, tn, b, 4 * kg, seg, row);
        const int head = row / p.hd, f = row % p.hd, half = p.hd / 2;
        f32x4 x1 = v[b], x2 = v[b + FB / 2];
        if (p.bias[seg]) {
          for (int i = 0; i < 4; ++i) {  // (a bias may start at any element)
            x1[i] += p.bias[seg][row + i];
            x2[i] += p.bias[seg][row + half + i];
          }
        }
        if (seg < 2) {
          const float2 *cs = p.rope_cs + (int64_t)m * half + f;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float2 c = cs[i];
            const float y1 = x1[i] * c.x - x2[i] * c.y, y2 = x2[i] * c.x + x1[i] * c.y;
            x1[i] = y1;
            x2[i] = y2;
          }
        }
        float *dst;
        if (seg == 0) {
          dst = p.out + (int64_t)m * p.ldo + head * p.hd;
        } else {
          const int64_t r = paged_row(p.kv, m, head, p.hd);
          if (r < 0) continue;
          dst = (float *)(seg == 1 ? p.kv.k : p.kv.v) + r;
        }
        *reinterpret_cast<f32x4 *>(dst + f) = x1;
        *reinterpret_cast<f32x4 *>(dst + f + half) = x2;
      }
    }
  }
}

constexpr int AW = 8;  // waves per attention workgroup

// Causal attention: one workgroup per 16 queries of a head, its 8 waves taking
// every eighth tile of 32 keys with an online softmax each, merged at the end
// through LDS.  S^T = K Q^T (keys on MFMA rows) leaves a lane with 4 keys of
// one query, which is the token operand of O^T = V^T P^T as it stands; the V
// rows are taken in an order that lets a lane load 4 consecutive values.
// Keys on a rejected page count as zero keys and values.  A key that some of the
// block's queries do not see has probability 0 there, and 0 times a non-finite
// value would be NaN: where a tile on the diagonal holds such a value, its keys
// past the first query are added by a loop of their own, for those that see them.
template <int HD>
__global__ __launch_bounds__(64 * AW) void attn_f32_kernel(const float *__restrict__ Q, PagedKV kv,
                                                       float *__restrict__ O, int M, int nq, int nkv) {
  constexpr int KS = HD / 16, VC = HD / 64;
  __shared__ float osh[AW][16][HD + 4];
  __shared__ float msh[AW][16], lsh[AW][16];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int r16 = lane % 16, kg = lane / 16;
  const int q0 = ((int)gridDim.x - 1 - (int)blockIdx.x) * 16;  // longest rows first
  const int h = blockIdx.y, hk = h / (nq / nkv);
  const int qi = q0 + r16;
  const float scale = 1.0f / sqrtf((float)HD);
  const float *K = (const float *)kv.k, *V = (const float *)kv.v;
  f32x4 qf[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) qf[s] = ldf4(Q + ((int64_t)min(qi, M - 1) * nq + h) * HD + 16 * s + 4 * kg);
  f32x4 o[VC][4];
#pragma unroll
  for (int c = 0; c < VC; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) o[c][e] = ZERO4;
  float m = -INFINITY, l = 0.f;
  const int last = min(q0 + 15, M - 1);
  // Tile rows: element offsets of keys k0 + 16 b + r16 in the pools, -1 for a
  // rejected page (and for keys past the last query, which are not looked up:
  // their scores are masked).  The loads are unconditional (row 0 of the pool
  // stands in) so that K of the next tile and V of this one are in flight
  // under the products.
  int64_t krow[2], nrow[2];
  f32x4 kf[2][KS];
  auto rows = [&](int k0, int64_t (&r)[2]) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int key = k0 + 16 * b + r16;
      r[b] = key <= last ? paged_row(kv, key, hk, HD) : -1;
    }
  };
  auto load_k = [&](const int64_t (&r)[2]) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const float *kp = K + (r[b] >= 0 ? r[b] : 0) + 4 * kg;
#pragma unroll
      for (int st = 0; st < KS; ++st) kf[b][st] = ldf4(kp + 16 * st);
    }
  };
  rows(32 * wave, krow);
  load_k(krow);
  for (int k0 = 32 * wave; k0 <= last; k0 += 32 * AW) {
    rows(k0 + 32 * AW, nrow);
    f32x4 vf[2][4][VC];
    bool vok[2][4];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t r = __shfl(krow[b], 4 * kg + i, 64);
        vok[b][i] = r >= 0;
        const float *vp = V + (r >= 0 ? r : 0) + 4 * r16;
#pragma unroll
        for (int c = 0; c < VC; ++c) vf[b][i][c] = ldf4(vp + 64 * c);
      }
    f32x4 s[2] = {ZERO4, ZERO4};
#pragma unroll
    for (int st = 0; st < KS; ++st)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int b = 0; b < 2; ++b) s[b] = mfma_f32(krow[b] >= 0 ? kf[b][st][i] : 0.f, qf[st][i], s[b]);
    load_k(nrow);
    float mt = -INFINITY;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s[b][i] = k0 + 16 * b + 4 * kg + i <= qi ? s[b][i] * scale : -INFINITY;
        mt = fmaxf(mt, s[b][i]);
      }
    mt = fmaxf(mt, __shfl_xor(mt, 16, 64));
    mt = fmaxf(mt, __shfl_xor(mt, 32, 64));
    bool apart = false;  // (uniform) keys past q0 are added apart
    if (k0 + 31 > q0) {
      float z = 0.f;  // NaN where a value is not finite
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int c = 0; c < VC; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) z = fmaf(vok[b][i] ? vf[b][i][c][e] : 0.f, 0.f, z);
      apart = __builtin_amdgcn_ballot_w64(!(z == 0.f)) != 0;
    }
    const float mn = fmaxf(m, mt);
    const float ref = mn == -INFINITY ? 0.f : mn;  // no key of this wave seen yet
    const float alpha = expf(m - ref);
    m = mn;
    l *= alpha;
#pragma unroll
    for (int c = 0; c < VC; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) o[c][e] *= alpha;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float pr = expf(s[b][i] - ref);
        l += pr;
        const bool in = vok[b][i] && !(apart && k0 + 16 * b + 4 * kg + i > q0);
#pragma unroll
        for (int c = 0; c < VC; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) o[c][e] = mfma_f32(in ? vf[b][i][c][e] : 0.f, pr, o[c][e]);
        if (apart)
          for (int g = 0; g < 4; ++g) {
            const int key = k0 + 16 * b + 4 * g + i;
            const float pk = __shfl(pr, 16 * g + r16, 64);
            const int64_t r = __shfl(krow[b], 4 * g + i, 64);
            if (key <= q0 || key > qi || r < 0) continue;
#pragma unroll
            for (int c = 0; c < VC; ++c)
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                const f32x4 x = ldf4(V + r + 64 * c + 16 * kg + 4 * j);
#pragma unroll
                for (int e = 0; e < 4; ++e) o[c][e][j] = fmaf(pk, x[e], o[c][e][j]);
              }
          }
      }
#pragma unroll
    for (int b = 0; b < 2; ++b) krow[b] = nrow[b];
  }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  if (kg == 0) {
    msh[wave][r16] = m;
    lsh[wave][r16] = l;
  }
  // MFMA row 4 kg + i of block (c, e) is hd 64 c + 4 (4 kg + i) + e
#pragma unroll
  for (int c = 0; c < VC; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *reinterpret_cast<f32x4 *>(&osh[wave][r16][64 * c + 16 * kg + 4 * i]) =
          f32x4{o[c][0][i], o[c][1][i], o[c][2][i], o[c][3][i]};
  __syncthreads();
  for (int idx = threadIdx.x; idx < 16 * HD / 4; idx += 64 * AW) {
    const int r = idx / (HD / 4), e = 4 * (idx % (HD / 4));
    if (q0 + r >= M) continue;
    float mx = msh[0][r];
#pragma unroll
    for (int w = 1; w < AW; ++w) mx = fmaxf(mx, msh[w][r]);
    const float ref = mx == -INFINITY ? 0.f : mx;
    f32x4 acc = ZERO4;
    float lt = 0.f;
#pragma unroll
    for (int w = 0; w < AW; ++w) {
      const float a = expf(msh[w][r] - ref);
      lt += a * lsh[w][r];
      acc += a * *reinterpret_cast<const f32x4 *>(&osh[w][r][e]);
    }
    acc /= lt;
    *reinterpret_cast<f32x4 *>(O + ((int64_t)(q0 + r) * nq + h) * HD + e) = acc;
  }
}

// Feature tiles of `rows` output rows (gate/up: rows of one of the two).
template <int EPI, int FB>
int n_tiles(const F32Gemm &p) {
  if (EPI == F32_QKV) return (p.N / p.hd) * (p.hd / 2 / (8 * FB));
  const int per = EPI == F32_SWIGLU ? 8 * FB : 16 * FB;
  return (p.seg_rows[0] + per - 1) / per;
}

// (A QKV launch without Q takes the form that it would take with Q: the forms
// split K over four waves or two, and K and V are the same to the bit either way.)
template <int EPI, int LORA>
void go(hipStream_t s, const F32Gemm &p) {
  F32Gemm whole = p;
  if (EPI == F32_QKV) whole.N = p.n_form;
  const int small = n_tiles<EPI, 2>(whole) * ((p.M + 31) / 32);
  if (small <= F32_FEW_TILES) {
    hipLaunchKernelGGL((gemm_f32_kernel<EPI, 2, 1, 4, LORA>), dim3(n_tiles<EPI, 2>(p), (p.M + 15) / 16), dim3(256), 0,
                       s, p);
  } else if (small < F32_BIG_TILES) {
    hipLaunchKernelGGL((gemm_f32_kernel<EPI, 2, 2, 4, LORA>), dim3(n_tiles<EPI, 2>(p), (p.M + 31) / 32), dim3(256), 0,
                       s, p);
  } else {
    hipLaunchKernelGGL((gemm_f32_kernel<EPI, 4, 4, 2, LORA>), dim3(n_tiles<EPI, 4>(p), (p.M + 63) / 64), dim3(128), 0,
                       s, p);
  }
}

}  // namespace

hipError_t launch_gemm_f32(hipStream_t s, F32Epi epi, const F32Gemm &p0) {
  F32Gemm p = p0;
  if (p.M <= 0) return hipSuccess;
  if (p.K % 4 || p.ldx % 4) return hipErrorInvalidValue;
  bool any = false;
  for (int i = 0; i < 3; ++i) any |= p.lb[i] != nullptr;
  if (!any) p.rank = 0;
  const bool fused = p.rank > 0 && p.rank <= F32_FUSED_RANK;
  switch (epi) {
    case F32_PLAIN: go<F32_PLAIN, 0>(s, p); break;
    case F32_RESID: fused ? go<F32_RESID, 1>(s, p) : go<F32_RESID, 0>(s, p); break;
    case F32_SWIGLU:
      if (fused && p.rank <= 8)
        go<F32_SWIGLU, 2>(s, p);
      else
        fused ? go<F32_SWIGLU, 1>(s, p) : go<F32_SWIGLU, 0>(s, p);
      break;
    case F32_QKV: fused ? go<F32_QKV, 1>(s, p) : go<F32_QKV, 0>(s, p); break;
  }
  return hipGetLastError();
}

hipError_t launch_attn_f32(hipStream_t s, const float *Q, const PagedKV &kv, float *O, int M, int nq, int nkv,
                           int hd) {
  if (M <= 0) return hipSuccess;
  const dim3 grid((M + 15) / 16, nq);
  if (hd == 64)
    hipLaunchKernelGGL(attn_f32_kernel<64>, grid, dim3(64 * AW), 0, s, Q, kv, O, M, nq, nkv);
  else if (hd == 128)
    hipLaunchKernelGGL(attn_f32_kernel<128>, grid, dim3(64 * AW), 0, s, Q, kv, O, M, nq, nkv);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace crf
