// Causal grouped-query softmax attention over the full prefix, reading K/V from
// the paged cache (flash-style: K/V tiles staged in LDS, online softmax).
//
// Workgroup = one query head x 128 queries: 4 waves of 32 queries, two
// workgroups per CU (two waves per SIMD from independent workgroups, so one
// wave's softmax overlaps the other's MFMAs).  Each wave computes S^T = K Q^T
// (keys on MFMA rows, queries on columns), so a lane owns one query and 16 of
// the 32 keys of a block: the online-softmax max and sum are in-lane plus one
// exchange with lane^32.  The probabilities feed O^T = V^T P^T straight from
// the S accumulators: the 8 accumulator registers of a key half-block are the
// 8 k-slots a lane supplies, so the V^T operand takes keys in the same order
// (slots 0-3: keys 4*(lane/32) + 0..3, slots 4-7: the same plus 8).
//
// K and V tiles go from the pages straight into LDS (buffer loads with an LDS
// destination, no register staging), both in their natural [key][hd] layout
// with XOR-swizzled 16-byte chunks.  The V^T operand is read with the gfx950
// LDS transpose read: within each 16-lane group, lane 4r+c points at 4
// consecutive hd values of key row r, and lane j receives hd column j of the 4
// rows.  A two-stage ring lets the loads of tile i+1 run under the MFMAs of
// tile i, with one barrier per tile.
//
// The workgroup's page bases are staged in LDS once (validated there); a key
// past the prefix or on a rejected page gets an out-of-range buffer offset,
// which the hardware returns as zero.
//
// Online softmax without a per-block maximum: the query rows come scaled by
// log2(e)/sqrt(hd) (attn_query_scale, applied where Q is stored) and each S
// accumulator starts at -ref, the lane's current reference, so the MFMAs hand
// back scores in log2 units already shifted and the probabilities are plain
// exp2 of the accumulators.  The reference is the row maximum of the first
// key block and is raised only when a half-block's probabilities sum past
// 2^8, which bounds every probability by 2^8; only then is the block maximum
// formed and O rescaled.  The result is the softmax of the definition (the
// reference cancels between O and the row sum).
//
// Launch order: workgroup b runs on XCD b % 8.  When the KV-head count divides
// 8, each XCD serves one KV head and every R-th query block (R = 8 / n_kv),
// longest causal rows first, with the G query heads of that KV head adjacent:
// the work per XCD is balanced and the heads that share K/V tiles run side by
// side on one L2.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "kernels.hpp"

namespace crf {
namespace {

#ifndef CRF_ATTN_WAVES
#define CRF_ATTN_WAVES 4
#endif
constexpr int NW = CRF_ATTN_WAVES;  // waves per workgroup, 32 queries each
constexpr int BQ = 32 * NW;         // queries per workgroup
constexpr int NT = 64 * NW;         // threads per workgroup
constexpr int BKV = 64;   // keys per tile
constexpr float PSUM_MAX = 256.0f;  // bound on a half-block's probability sum (and each probability)
constexpr int PGCAP = 2048;  // page bases staged in LDS at a time
// Workgroups aimed at when a few query rows are split over the keys: the
// resident ones (16385 keys, 4 KV heads of 128: 1024 -> 12.3 + 6.0 us with the
// merge, 512 -> 11.0 + 4.8, 384 the same).
constexpr int SPLIT_WG = 512;
constexpr int ATTN_SLOTS = 512;  // resident workgroups of the GPU (two per CU)

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// 16-byte chunk slot of chunk c in K row r: conflict-free 16-byte fragment reads.
template <int HD>
CRF_DEV int kslot(int r, int c) {
  return c ^ (r & (HD / 8 - 1));
}
// Chunk slot in V row r: every transpose read (4 rows x 32 bytes per 16 lanes,
// 4 rows x 64 bytes per 32 lanes) lands on distinct banks.
template <int HD>
CRF_DEV int vslot(int r, int c) {
  if (HD == 128) return c ^ ((0xCA60 >> (4 * (r & 3))) & 15);
  return c ^ (2 * (r & 3));
}

CRF_DEV float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

CRF_DEV s16x4 ld_tr(const bf16 *p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(const __attribute__((address_space(3))) void *)p);
}

// Byte offset of the first key of logical page p for this KV head, or CRF_OOB.
struct PageMap {
  const int32_t *bt;
  int n_pages;
  uint32_t page_bytes, head_bytes;
  int *err;
  CRF_DEV uint32_t base(int p) const {
    const int q = bt[p];
    if (q < 0 || q >= n_pages) {
      atomicOr(err, (int)CRF_DEVERR_BLOCK_TABLE);
      return CRF_OOB;
    }
    return (uint32_t)q * page_bytes + head_bytes;
  }
};

// Query head and query block of workgroup `bid` over nqb blocks of BQ rows;
// false for padding at the end of a per-XCD list (uniform per workgroup).
// Packed: one workgroup per KV head carries the group's query heads stacked on
// the rows of one tile.  xcd_r > 0: XCD x (= bid % 8) serves KV head x / xcd_r
// and every xcd_r-th query block from x % xcd_r, longest causal rows first,
// with the group's query heads adjacent.  Otherwise head-major, longest rows
// first.
__host__ __device__ inline bool attn_block(int bid, int nq, int nkv, int nqb, int xcd_r, int packed, int &head,
                                           int &qblk) {
  const int group = nq / nkv;
  if (packed) {
    head = bid * group;
    qblk = 0;
    return true;
  }
  if (xcd_r > 0) {
    const int x = bid % 8, j = bid / 8;
    const int qi = j / group;
    head = (x / xcd_r) * group + j % group;
    qblk = nqb - 1 - (qi * xcd_r + x % xcd_r);
    return qblk >= 0;
  }
  head = bid % nq;
  qblk = nqb - 1 - bid / nq;
  return true;
}

// Workgroups of a window launch (no key split); sets xcd_r for attn_block
// (0 when the KV-head count does not divide the XCD count).
inline int attn_window_grid(int nq, int nkv, int nqb, int &xcd_r) {
  if (nkv <= 8 && 8 % nkv == 0) {
    xcd_r = 8 / nkv;
    return 8 * (nq / nkv) * ((nqb + xcd_r - 1) / xcd_r);
  }
  xcd_r = 0;
  return nqb * nq;
}

// Query head, query block and key split of workgroup `bid` of a key-split
// launch; false for padding.  A unit is one split of one KV head: its workgroups
// (every query block of the group's heads, or one when packed) read the same
// K/V tiles.  The XCDs share the list of all units' workgroups evenly, each
// taking a run of it, so that none idles however few the units are and a unit's
// workgroups lie on as few XCDs as that allows.
__host__ __device__ inline bool attn_split_block(int bid, int nq, int nkv, int nqb, int n_splits, int packed,
                                                 int &head, int &qblk, int &split) {
  const int group = nq / nkv, per = packed ? 1 : group * nqb;
  const int n = nkv * n_splits * per, x = bid % 8, j = bid / 8;
  if (j >= n / 8 + (x < n % 8)) return false;
  const int i = x * (n / 8) + (x < n % 8 ? x : n % 8) + j, u = i / per, w = i % per;
  split = u / nkv;
  attn_block(packed ? u % nkv : 0, nq, nkv, nqb, 0, packed, head, qblk);
  if (!packed) {
    head = (u % nkv) * group + w / nqb;
    qblk = nqb - 1 - w % nqb;
  }
  return true;
}

inline int attn_split_grid(int nq, int nkv, int nqb, int n_splits, int packed) {
  return 8 * ((nkv * n_splits * (packed ? 1 : nq / nkv * nqb) + 7) / 8);
}

// Window launch whose query blocks from `long0` on have their keys in two parts
// (per-XCD order, xcd_r > 0): query head, query block and part of workgroup
// `bid`; false for padding.  Longest first along an XCD's list: the first parts
// of its long blocks, then their second parts and the short blocks in turn.
__host__ __device__ inline bool attn_halves_block(int bid, int nq, int nkv, int nqb, int xcd_r, int long0, int &head,
                                                  int &qblk, int &split) {
  const int group = nq / nkv, x = bid % 8, r = x % xcd_r, j = bid / 8;
  head = (x / xcd_r) * group + j % group;
  const int last = nqb - 1 - r;  // the XCD's longest block; its others are xcd_r apart
  const int blocks = last < 0 ? 0 : last / xcd_r + 1, n_long = last < long0 ? 0 : (last - long0) / xcd_r + 1;
  int q = j / group;
  if (q >= blocks + n_long) return false;
  split = 0;
  if (q >= n_long) {
    q -= n_long;
    const int n_short = blocks - n_long, both = 2 * (n_long < n_short ? n_long : n_short);
    if (q < both) {
      split = (q & 1) == 0;
      q = split ? q / 2 : n_long + q / 2;
    } else if (n_long > n_short) {
      split = 1;
      q -= n_short;
    }  // else short block q - n_long of the list, whose index is q
  }
  qblk = last - q * xcd_r;
  return true;
}

inline int attn_halves_grid(int nq, int nkv, int nqb, int xcd_r, int long0) {
  return 8 * (nq / nkv) * ((nqb + xcd_r - 1) / xcd_r + (nqb - long0 + xcd_r - 1) / xcd_r);
}

// Logical pages that a query block whose last query sits at `last_key` may load
// from: it loads whole tiles, of which the last can run on past last_key, over
// the keys of the block's successors, up to the M keys there are.
__host__ __device__ inline int attn_pages(int last_key, int M, int ps) {
  const int end = (last_key / BKV + 1) * BKV;
  return ((end < M ? end : M) - 1) / ps + 1;
}

// PS: page size when fixed at compile time (16), 0 = runtime kv.page_size.
template <int HD, int PS>
__global__ __launch_bounds__(NT, 8 / NW) void attn_bf16_kernel(const bf16 *__restrict__ Q, PagedKV kv,
                                                           bf16 *__restrict__ O, int Mq, int q_off, int nq,
                                                           int nkv, uint32_t pool_bytes, int xcd_r,
                                                           int split_tiles, int n_splits, int packed, int long0,
                                                           float *__restrict__ part) {
  constexpr int CH = HD / 8;             // 16-byte chunks per row
  constexpr int KS = HD / 16;            // MFMA k-steps for S
  constexpr int HB = HD / 32;            // 32-row hd blocks of O^T
  constexpr int RPI = 64 / CH;           // rows per 64-lane load instruction
  constexpr int RPW = BKV / NW;          // key rows each wave loads per tile
  constexpr int IPW = RPW / RPI;         // load instructions per wave per tile (each of K and V)
  constexpr int TILE = BKV * HD;         // elements per K (or V) tile
  // one array per stage and operand, so the compiler sees that loads into one
  // stage never alias reads of the other
  __shared__ __align__(16) bf16 ks0[TILE], ks1[TILE], vs0[TILE], vs1[TILE];
  __shared__ uint32_t pgbase[PGCAP];

  // Query rows 0..Mq-1 sit at positions q_off..q_off+Mq-1 and attend to keys
  // 0..q_off+row: the cached prefix and the rows before them (q_off = 0 and
  // Mq = the prefix length for a window).
  const int M = q_off + Mq;  // keys
  const int nqb = (Mq + BQ - 1) / BQ;
  const int group = nq / nkv;
  int head, qblk, split = 0;
  if (long0 >= 0) {
    if (!attn_halves_block(blockIdx.x, nq, nkv, nqb, xcd_r, long0, head, qblk, split)) return;
  } else if (split_tiles > 0) {
    if (!attn_split_block(blockIdx.x, nq, nkv, nqb, n_splits, packed, head, qblk, split)) return;
  } else if (!attn_block(blockIdx.x, nq, nkv, nqb, xcd_r, packed, head, qblk)) {
    return;
  }
  const int g_kv = head / group;
  const int ps = PS > 0 ? PS : kv.page_size;
  const int tid = threadIdx.x, lane = tid % 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int g = lane / 32, l32 = lane % 32;
  const int q0 = qblk * BQ;
  const int q0w = q0 + wave * 32;
  const int qi = q0w + l32;
  const int dq = nq * HD;
  // This lane's query: row qrow of head qhead.  Packed, tile row qi holds
  // (query head qi / Mq of the group, query row qi % Mq).
  const int n_rows = packed ? group * Mq : Mq;
  const int qrow = packed ? qi % Mq : qi;
  const int qhead = packed ? head + min(qi / Mq, group - 1) : head;
  // first and last position of the wave's queries
  const int pos_lo = packed ? q_off : q_off + q0w;
  const int pos_hi = packed ? q_off + Mq - 1 : q_off + q0w + 31;

  bf16x8 qf[KS];
  {
    const bf16 *qrow_p = Q + (int64_t)min(qrow, Mq - 1) * dq + qhead * HD + 8 * g;
#pragma unroll
    for (int s = 0; s < KS; ++s) qf[s] = as_bf16x8(ld16(qrow_p + 16 * s));
  }

  const __amdgpu_buffer_rsrc_t kres = make_rsrc(kv.k, pool_bytes);
  const __amdgpu_buffer_rsrc_t vres = make_rsrc(kv.v, pool_bytes);
  const PageMap pm{kv.block_table, kv.n_pages, (uint32_t)(kv.page_stride * 2), (uint32_t)(g_kv * ps * HD * 2),
                   kv.err};

  const int last_key = min(q_off + q0 + BQ, M) - 1;
  const int ntiles = last_key / BKV + 1;
  // Split over keys (few query blocks over a long prefix): this workgroup takes
  // tiles [t_begin, t_end) and leaves an unnormalised partial for the merge (of
  // weight 0 where the range lies past every key of its rows).  long0 >= 0: only
  // the query blocks from long0 on are split.
  const bool partial = split_tiles > 0 && qblk >= long0;
  int t_begin = 0, t_end = ntiles;
  if (partial) {
    t_begin = split * split_tiles;
    t_end = min(ntiles, t_begin + split_tiles);
  }
  const int n_pages_needed = attn_pages(last_key, M, ps);

  // pgbase[i] = base of logical page pg_first + i; refilled only between barriers.
  int pg_first = 0;
  auto fill_pages = [&](int first) {
    pg_first = first;
    for (int i = tid; i < min(PGCAP, n_pages_needed - first); i += NT) pgbase[i] = pm.base(first + i);
  };

  // This lane's row and chunk in each of the wave's load instructions.  A wave
  // loads RPW consecutive rows (keys) of the tile; the in-page part of each
  // lane's offset (row in the page, swizzled chunk) is fixed for the kernel
  // when the page size is a multiple of 16.
  const int lrow = lane / CH, lslot = lane % CH;
  uint32_t koff[IPW], voff[IPW];
#pragma unroll
  for (int i = 0; i < IPW; ++i) {
    const int row = RPI * i + lrow;    // row within the wave's rows
    const int trow = wave * RPW + row;  // row within the tile (the LDS swizzle's row)
    koff[i] = (uint32_t)(row * HD * 2 + kslot<HD>(trow, lslot) * 16);
    voff[i] = (uint32_t)(row * HD * 2 + vslot<HD>(trow, lslot) * 16);
  }
  auto dma = [&](int kt0, bf16 *kdst, bf16 *vdst) {
    const int wrow0 = kt0 + wave * RPW;  // first key of this wave's rows
    if (PS > 0 && PS % 16 == 0) {
      // the wave's rows share one page: one uniform base (CRF_OOB plus an
      // in-page offset stays out of range, pool sizes being below 2^31)
      const int pidx = min(max(wrow0 / PS - pg_first, 0), PGCAP - 1);
      const uint32_t b =
          (uint32_t)__builtin_amdgcn_readfirstlane((int)pgbase[pidx]) + (uint32_t)((wrow0 % PS) * HD * 2);
      if (wrow0 + RPW <= M) {  // uniform: all the wave's rows inside the prefix
#pragma unroll
        for (int i = 0; i < IPW; ++i) {
          const int ldsoff = (wave * RPW + RPI * i) * HD;  // wave-uniform first row of this instruction
          dma16(kres, (lds_char *)(kdst + ldsoff), b + koff[i], 0);
          dma16(vres, (lds_char *)(vdst + ldsoff), b + voff[i], 0);
        }
      } else {
#pragma unroll
        for (int i = 0; i < IPW; ++i) {
          const int ldsoff = (wave * RPW + RPI * i) * HD;
          const bool in = wrow0 + RPI * i + lrow < M;
          dma16(kres, (lds_char *)(kdst + ldsoff), in ? b + koff[i] : CRF_OOB, 0);
          dma16(vres, (lds_char *)(vdst + ldsoff), in ? b + voff[i] : CRF_OOB, 0);
        }
      }
    } else {
      uint32_t b[IPW];
#pragma unroll
      for (int i = 0; i < IPW; ++i) {
        const int tok = wrow0 + RPI * i + lrow;
        b[i] = pgbase[min(max(tok / ps - pg_first, 0), PGCAP - 1)];  // clamped: used only when tok < M
      }
#pragma unroll
      for (int i = 0; i < IPW; ++i) {
        const int row = wave * RPW + RPI * i + lrow;  // key within the tile
        const int tok = kt0 + row;
        const bool ok = tok < M && b[i] != CRF_OOB;
        const uint32_t rowoff = b[i] + (uint32_t)((tok % ps) * HD * 2);
        const int ldsoff = (wave * RPW + RPI * i) * HD;
        dma16(kres, (lds_char *)(kdst + ldsoff), ok ? rowoff + (uint32_t)(kslot<HD>(row, lslot) * 16) : CRF_OOB, 0);
        dma16(vres, (lds_char *)(vdst + ldsoff), ok ? rowoff + (uint32_t)(vslot<HD>(row, lslot) * 16) : CRF_OOB, 0);
      }
    }
  };

  f32x16 oacc[HB];
#pragma unroll
  for (int b = 0; b < HB; ++b)
#pragma unroll
    for (int v = 0; v < 16; ++v) oacc[b][v] = 0.f;
  // Scores arrive in log2 units (the query rows are stored pre-multiplied by
  // log2(e)/sqrt(hd)) and relative to the lane's reference `ref`: the S
  // accumulators start at -ref (negm), so exp2 of an accumulator is the
  // probability up to the common factor 2^ref.  The reference is set to the
  // row maximum on the wave's first key block and afterwards only raised,
  // when the probabilities of a 32-key half-block sum past PSUM_MAX (which
  // bounds each of them); most half-blocks therefore need no maximum at all.
  float ref = 0.f, l_run = 0.f;
  f32x16 negm;
#pragma unroll
  for (int v = 0; v < 16; ++v) negm[v] = 0.f;

  // Transpose-read coordinates: 16-lane group gq covers hd 16*(gq&1) .. +15 of a
  // 32-row block and key rows 4*(gq>>1) + r; lane 4r + c reads hd chunk c*4.
  const int tr_r = (lane % 16) / 4, tr_c = lane % 4, tr_g = lane / 16;
  const int tr_key = 4 * (tr_g >> 1) + tr_r;            // + key half-block base (+8 for slots 4-7)
  const int tr_hd = 16 * (tr_g & 1) + 4 * tr_c;         // + 32*b

  // One tile: wait for its loads, publish them, start the next tile's loads
  // into the other stage, then compute.  FIRST: the range's first tile, where
  // the reference is set (a row that sees any key of the range sees that
  // tile's first key, which lies in its first half-block).
  auto tile = [&](int it, const bf16 *kt, const bf16 *vt, bf16 *kn, bf16 *vn, auto first_t) {
    constexpr bool FIRST = decltype(first_t)::value;
    const int kt0 = it * BKV;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (it + 1 < t_end) {
      const int next_last_page = (min(kt0 + 2 * BKV, M) - 1) / ps;
      if (next_last_page >= pg_first + PGCAP) {
        fill_pages((kt0 + BKV) / ps);
        __syncthreads();
      }
      dma(kt0 + BKV, kn, vn);
    }
    // every key of this tile is in this wave's future, or every row of the wave is padding
    if (kt0 > pos_hi || q0w >= n_rows) return;
    f32x16 sacc[2];
    // K fragments are read two k-steps ahead of the MFMAs that use them (the
    // scheduling barriers keep the compiler from regrouping them)
    bf16x8 kf[3][2];
    auto kread = [&](int s, bf16x8 (&f)[2]) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const int r = kb * 32 + l32;
        f[kb] = as_bf16x8(ld16(kt + r * HD + kslot<HD>(r, 2 * s + g) * 8));
      }
    };
    kread(0, kf[0]);
    kread(1, kf[1]);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      if (s + 2 < KS) kread(s + 2, kf[(s + 2) % 3]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) sacc[kb] = mfma32(kf[s % 3][kb], qf[s], s == 0 ? negm : sacc[kb]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // causal mask (also hides keys >= M, which are always > q_off + qrow for a valid row)
    if (kt0 + BKV - 1 > pos_lo) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int key = kt0 + kb * 32 + 8 * (v / 4) + 4 * g + (v % 4);
          if (key > q_off + qrow) sacc[kb][v] = -INFINITY;
        }
    }
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      float pr[16];
      float psum = 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        pr[v] = fast_exp2(sacc[kb][v]);
        psum += pr[v];
      }
      // (the negated test also catches an infinite sum)
      if ((FIRST && kb == 0) || __builtin_amdgcn_ballot_w64(!(psum <= PSUM_MAX))) {
        float mx = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sacc[kb][v]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        float shift;
        if (FIRST && kb == 0) {
          // the reference jumps to the row maximum (a row that sees no key
          // here sees none of the range: it keeps l = 0)
          shift = mx > -INFINITY ? mx : 0.f;
        } else {
          shift = fmaxf(mx, 0.f);
          const float alpha = fast_exp2(-shift);
          l_run *= alpha;
#pragma unroll
          for (int b = 0; b < HB; ++b) oacc[b] *= alpha;
        }
        ref += shift;
#pragma unroll
        for (int v = 0; v < 16; ++v) negm[v] = -ref;
#pragma unroll
        for (int k2 = kb; k2 < 2; ++k2)
#pragma unroll
          for (int v = 0; v < 16; ++v) sacc[k2][v] -= shift;
        psum = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          pr[v] = fast_exp2(sacc[kb][v]);
          psum += pr[v];
        }
      }
      l_run += psum;
      bf16x8 pf[2];
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
#pragma unroll
        for (int e = 0; e < 8; ++e) pf[hh][e] = f2bf(pr[8 * hh + e]);
      // O^T[hd, q] += V^T[hd, keys] P^T[keys, q]
#pragma unroll
      for (int b = 0; b < HB; ++b) {
        const int hd = 32 * b + tr_hd;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          const int r0 = kb * 32 + 16 * hh + tr_key, r1 = r0 + 8;
          const s16x4 lo = ld_tr(vt + r0 * HD + vslot<HD>(r0, hd / 8) * 8 + hd % 8);
          const s16x4 hi = ld_tr(vt + r1 * HD + vslot<HD>(r1, hd / 8) * 8 + hd % 8);
          const s16x4 lohi[2] = {lo, hi};
          oacc[b] = mfma32(__builtin_bit_cast(bf16x8, lohi), pf[hh], oacc[b]);
        }
      }
    }
  };

  if (t_begin < t_end) {  // (a part past the block's last key loads nothing)
    fill_pages(t_begin * BKV / ps);
    __syncthreads();
    dma(t_begin * BKV, ks0, vs0);
    tile(t_begin, ks0, vs0, ks1, vs1, std::true_type());
  }
  for (int it = t_begin + 1; it < t_end; it += 2) {
    tile(it, ks1, vs1, ks0, vs0, std::false_type());
    if (it + 1 < t_end) tile(it + 1, ks0, vs0, ks1, vs1, std::false_type());
  }

  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  if (qi >= n_rows) return;
  if (partial) {  // unnormalised O^T row, then the running max and sum
    const int row0 = max(long0, 0) * BQ;  // first row with partials
    float *prow = part + (((int64_t)split * nq + qhead) * (Mq - row0) + qrow - row0) * (HD + 4);
#pragma unroll
    for (int b = 0; b < HB; ++b)
#pragma unroll
      for (int ii = 0; ii < 4; ++ii)
        *reinterpret_cast<f32x4 *>(prow + b * 32 + 8 * ii + 4 * g) =
            f32x4{oacc[b][ii * 4], oacc[b][ii * 4 + 1], oacc[b][ii * 4 + 2], oacc[b][ii * 4 + 3]};
    if (g == 0) {
      prow[HD] = l_tot > 0.f ? ref : -1e30f;  // a row that saw no key weighs 0 in the merge
      prow[HD + 1] = l_tot;
    }
    return;
  }
  const float inv = 1.0f / l_tot;
  bf16 *orow = O + (int64_t)qrow * dq + qhead * HD;
#pragma unroll
  for (int b = 0; b < HB; ++b)
#pragma unroll
    for (int ii = 0; ii < 4; ++ii) {
      const int e = b * 32 + 8 * ii + 4 * g;
      st8(orow + e, pack_bf16x4(oacc[b][ii * 4] * inv, oacc[b][ii * 4 + 1] * inv, oacc[b][ii * 4 + 2] * inv,
                                oacc[b][ii * 4 + 3] * inv));
    }
}

// Merge of the key splits of one (query row, head): O = sum_s 2^(m_s - m) O_s /
// sum_s 2^(m_s - m) l_s with m = max_s m_s (scores in log2 units).  Groups of
// HD / 4 threads take every NG-th split, 4 output elements per thread, with the
// group's own running maximum (no pass over the maxima first), four splits'
// loads in flight.
template <int HD>
__global__ __launch_bounds__(256) void attn_merge_kernel(const float *__restrict__ part, bf16 *__restrict__ O,
                                                         int Mq, int nq, int n_splits, const AttnLora lora) {
  constexpr int TPG = HD / 4, NG = 256 / TPG, UN = 4;
  __shared__ f32x4 osum[NG][TPG];
  __shared__ float lsum[NG], gmax[NG];
  const int qi = blockIdx.x / nq, head = blockIdx.x % nq;
  const int tid = threadIdx.x;
  const int64_t stride = (int64_t)nq * Mq * (HD + 4);
  const float *p0 = part + ((int64_t)head * Mq + qi) * (HD + 4);
  const int gi = tid / TPG, e = 4 * (tid % TPG);
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
  float l = 0.f, m = -INFINITY;
  for (int sp0 = gi; sp0 < n_splits; sp0 += UN * NG) {
    f32x4 t[UN];
    float ms[UN], ls[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {  // past the end: the last split again, of weight 0
      const int sp = sp0 + u * NG;
      const float *ps = p0 + min(sp, n_splits - 1) * stride;
      t[u] = *reinterpret_cast<const f32x4 *>(ps + e);
      ms[u] = sp < n_splits ? ps[HD] : -INFINITY;
      ls[u] = ps[HD + 1];
    }
    float mn = m;
#pragma unroll
    for (int u = 0; u < UN; ++u) mn = fmaxf(mn, ms[u]);  // finite: the first split of a batch is a real one
    const float a = exp2f(m - mn);
    o *= a;
    l *= a;
    m = mn;
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const float w = exp2f(ms[u] - mn);
      l += w * ls[u];
      o += w * t[u];
    }
  }
  osum[gi][tid % TPG] = o;
  if (tid % TPG == 0) {
    lsum[gi] = l;
    gmax[gi] = m;
  }
  __syncthreads();
  __shared__ __align__(16) bf16 osh[HD];
  if (tid < TPG) {
    float mt = gmax[0];
#pragma unroll
    for (int g2 = 1; g2 < NG; ++g2) mt = fmaxf(mt, gmax[g2]);
    f32x4 ot = {0.f, 0.f, 0.f, 0.f};
    float lt = 0.f;
#pragma unroll
    for (int g2 = 0; g2 < NG; ++g2) {
      const float w = exp2f(gmax[g2] - mt);  // (a group without a split weighs 0)
      ot += w * osum[g2][tid];
      lt += w * lsum[g2];
    }
    const float inv = 1.0f / lt;
    const u32x2 o4 = pack_bf16x4(ot[0] * inv, ot[1] * inv, ot[2] * inv, ot[3] * inv);
    st8(O + (int64_t)qi * nq * HD + head * HD + e, o4);
    st8(&osh[e], o4);
  }
  if (!lora.A) return;
  // this head's part of the output adapter's U: HD / 8 lanes per rank
  constexpr int LPK = HD / 8;
  const int l8 = tid % LPK;
  u32x4 a0 = {0u, 0u, 0u, 0u};
  const bf16 *ap = lora.A + (int64_t)(tid / LPK) * nq * HD + head * HD + 8 * l8;
  if (tid / LPK < lora.rank) a0 = ld16(ap);
  __syncthreads();
  const bf16x8 x = as_bf16x8(ld16(&osh[8 * l8]));
  for (int r = tid / LPK; r < lora.rank; r += 256 / LPK) {
    const bf16x8 a = as_bf16x8(a0);
    if (r + 256 / LPK < lora.rank) a0 = ld16(ap += (int64_t)(256 / LPK) * nq * HD);
    float v = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) v = fmaf(bf2f(a[i]), bf2f(x[i]), v);
#pragma unroll
    for (int o = LPK / 2; o >= 1; o >>= 1) v += __shfl_xor(v, o, LPK);
    if (l8 == 0) lora.part[((int64_t)head * 16 + qi) * lora.cols + r] = v;
  }
}

// The same for the two parts of every row from row0 on: HD / 4 lanes per (row,
// head), 256 * 4 / HD of them to a workgroup.
template <int HD>
__global__ __launch_bounds__(256) void attn_halves_merge_kernel(const float *__restrict__ part, bf16 *__restrict__ O,
                                                                int row0, int n_rows, int nq) {
  constexpr int TPG = HD / 4;
  const int64_t i = (int64_t)blockIdx.x * (256 / TPG) + threadIdx.x / TPG;  // row * nq + head
  if (i >= (int64_t)n_rows * nq) return;
  const int r = (int)(i / nq), head = (int)(i % nq), e = 4 * (threadIdx.x % TPG);
  const float *p0 = part + ((int64_t)head * n_rows + r) * (HD + 4), *p1 = p0 + (int64_t)nq * n_rows * (HD + 4);
  const f32x4 a = *reinterpret_cast<const f32x4 *>(p0 + e), b = *reinterpret_cast<const f32x4 *>(p1 + e);
  const float ma = p0[HD], la = p0[HD + 1], mb = p1[HD], lb = p1[HD + 1];
  const float m = fmaxf(ma, mb), wa = exp2f(ma - m), wb = exp2f(mb - m);
  const float inv = 1.0f / (wa * la + wb * lb);
  const f32x4 o = (wa * a + wb * b) * inv;
  st8(O + (int64_t)(row0 + r) * nq * HD + head * HD + e, pack_bf16x4(o[0], o[1], o[2], o[3]));
}

// First query block whose keys a window launch takes in two parts of split_tiles
// tiles (-1: none).  A workgroup alone on a CU computes a tile more slowly than a
// CU with all its workgroups (two at head size 128, three at 64), so with few
// blocks the longest chain of tiles outlasts the GPU's share of all tiles; the
// parts cost 52 MB of partials at 4096 tokens of 12 heads (attention 94 -> 77 us
// and a merge of 8).  The line, as the chain's tiles over a CU's share of all:
// 12 heads of 128, 3000 tokens (1.7) 865 -> 843 us for two layers, 5000 (1.04)
// 1285 -> 1276, 6100 (0.87) 1593 -> 1612; 28 heads, 2060 tokens (1.01) 1056 ->
// 1070 for one; 12 heads of 64, 6100 tokens (0.87) 514 -> 501.  Where the partials
// have room for the last blocks only (a context of less than 2048 tokens) the parts
// neither win nor lose more than 0.6 % (2000 tokens, seven layouts).
inline int attn_halves(int Mq, int q_off, int nq, int nqb, int hd, int64_t part_floats, int &split_tiles) {
  const int nt = (q_off + Mq + BKV - 1) / BKV, nt0 = (q_off + std::min(Mq, BQ) + BKV - 1) / BKV;
  if (nt < 32) return -1;  // a part of at least 16 tiles
  const double share = 0.5 * nq * nqb * (nt + nt0) / (ATTN_SLOTS / 2);
  if (nt <= (hd == 128 ? 1.03 : 0.8) * share) return -1;
  // the middle, or as far past it as the partials fit
  for (int st = (nt + 1) / 2; st < nt; ++st) {
    // blocks from here on end past tile st: q_off + (b + 1) * BQ > st * BKV
    const int b = std::max(0, (int)(((int64_t)st * BKV - q_off) / BQ));
    if (b >= nqb) break;
    if (2 * (int64_t)nq * (Mq - b * BQ) * (hd + 4) > part_floats) continue;
    split_tiles = st;
    return b;
  }
  return -1;
}

// Tiles of keys per split of a launch whose keys are split over workgroups (0:
// none), for room of max_splits partials of every row.
//   A few query rows (<= 16): when the group's heads fit one tile (packed), one
// workgroup serves all of them, so the K/V tiles are read once per KV head.
//   A few query blocks (the new tokens of a decoding step over a long prefix)
// leave most of the GPU idle: split until every slot has a workgroup.  Every row
// is then written as partials and merged, which only pays where every block has
// the prefix to share out, from a prefix of twice the new tokens on.  Four-layer
// steps, whole against split: 12/2 heads of 64, 2000 + 400 tokens 302 -> 292 us
// and 4000 + 300 338 -> 296, but 1500 + 800 355 -> 367 and 1000 + 2000 502 -> 599;
// 16/2 heads of 128, 2000 + 1500 tokens 1289 -> 1371.  A window has no prefix
// (one layer of 1.5B shapes over 2048 / 2688 tokens 329 -> 360 / 419 -> 451 us;
// its long blocks are attn_halves' business).
inline int attn_split(int Mq, int q_off, int nq, int nkv, int64_t max_splits, int &packed) {
  const int nqb = (Mq + BQ - 1) / BQ, ntiles = (q_off + Mq + BKV - 1) / BKV;
  packed = 0;
  if (max_splits < 2) return 0;
  if (Mq <= 16 && ntiles >= 8) {
    packed = (nq / nkv) * Mq <= BQ;
    const int units = packed ? nkv : nq;
    return std::max<int>(std::max<int>(1, (ntiles * units + SPLIT_WG - 1) / SPLIT_WG),
                         (int)((ntiles + max_splits - 1) / max_splits));
  }
  if (Mq > 16 && q_off >= 2 * (int64_t)Mq && nq * nqb * 2 <= ATTN_SLOTS && ntiles >= 32) {
    const int sp = std::min<int>(ATTN_SLOTS / (nq * nqb), (int)std::min<int64_t>(max_splits, ntiles / 8));
    if (sp >= 2) return (ntiles + sp - 1) / sp;
  }
  return 0;
}

template <int HD>
void launch(hipStream_t s, const bf16 *Q, const PagedKV &kv, bf16 *O, int Mq, int q_off, int nq, int nkv,
            uint32_t pool_bytes, float *part, int64_t part_floats, AttnLora *lora) {
  const int nqb = (Mq + BQ - 1) / BQ;
  int xcd_r = 0, grid = nqb * nq, n_splits = 1, packed = 0, long0 = -1;
  const int64_t keys = (int64_t)q_off + Mq;
  const int ntiles = (int)((keys + BKV - 1) / BKV);
  const int64_t max_splits = part ? part_floats / ((int64_t)nq * Mq * (HD + 4)) : 0;
  int split_tiles = attn_split(Mq, q_off, nq, nkv, max_splits, packed);
  if (split_tiles > 0) {
    n_splits = (ntiles + split_tiles - 1) / split_tiles;
    grid = attn_split_grid(nq, nkv, nqb, n_splits, packed);
  } else {
    grid = attn_window_grid(nq, nkv, nqb, xcd_r);
    if (xcd_r > 0 && part) long0 = attn_halves(Mq, q_off, nq, nqb, HD, part_floats, split_tiles);
    if (long0 >= 0) grid = attn_halves_grid(nq, nkv, nqb, xcd_r, long0);
  }
  const dim3 g3(grid);
  if (kv.page_size == 16)
    hipLaunchKernelGGL((attn_bf16_kernel<HD, 16>), g3, dim3(NT), 0, s, Q, kv, O, Mq, q_off, nq, nkv, pool_bytes,
                       xcd_r, split_tiles, n_splits, packed, long0, part);
  else
    hipLaunchKernelGGL((attn_bf16_kernel<HD, 0>), g3, dim3(NT), 0, s, Q, kv, O, Mq, q_off, nq, nkv, pool_bytes,
                       xcd_r, split_tiles, n_splits, packed, long0, part);
  if (long0 >= 0) {
    const int rows = Mq - long0 * BQ;
    const int64_t threads = (int64_t)rows * nq * (HD / 4);
    hipLaunchKernelGGL((attn_halves_merge_kernel<HD>), dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, part, O,
                       long0 * BQ, rows, nq);
  } else if (split_tiles > 0) {
    if (lora && Mq <= 16) lora->n_parts = nq;
    const AttnLora al = lora && Mq <= 16 ? *lora : AttnLora{};
    hipLaunchKernelGGL((attn_merge_kernel<HD>), dim3(Mq * nq), dim3(256), 0, s, part, O, Mq, nq, n_splits, al);
  }
}

}  // namespace

hipError_t launch_attn_bf16(hipStream_t s, const bf16 *Q, const PagedKV &kv, bf16 *O, int Mq, int q_off, int nq,
                            int nkv, int hd, float *part, int64_t part_floats, AttnLora *lora) {
  if (lora) lora->n_parts = 0;
  if (Mq <= 0) return hipSuccess;
  if (q_off < 0) return hipErrorInvalidValue;
  const int64_t bytes = (int64_t)kv.n_pages * kv.page_stride * 2;
  if (bytes >= (int64_t)CRF_OOB) return hipErrorInvalidValue;
  if (hd == 128)
    launch<128>(s, Q, kv, O, Mq, q_off, nq, nkv, (uint32_t)bytes, part, part_floats, lora);
  else if (hd == 64)
    launch<64>(s, Q, kv, O, Mq, q_off, nq, nkv, (uint32_t)bytes, part, part_floats, lora);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace crf
