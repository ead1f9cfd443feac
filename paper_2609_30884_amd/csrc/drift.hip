// Adapter drift: squared distances between the current adapter and every stored
// version, in chunks of its factor tensors, then summed in a fixed order
// (deterministic).  Accumulation in fp64.
//
// HBM-bound once enough bytes are in flight: a workgroup reads its chunk of the
// current adapter once for four versions, 16 bytes per lane and four loads per
// tensor ahead of the sums, and the workgroup that finishes last forms the
// outputs, so that there is no second launch.  Measured: 28 layers x 4 versions at 1.5B shapes
// (44 MB) 32 + 5 -> 20 us on the GPU, 57 -> 26 us a call; x 2 versions at 7B
// shapes (242 MB) 85 + 8 -> 51 us (4.7 TB/s), 153 -> 71 us a call, issued one after
// another (each waited for: 69 -> 48 and 165 -> 84 us; the first on new adapters 217
// -> 164 and 170 -> 127).  The first
// is all latency: tables, chunk, and the last workgroup's two rounds of loads.
#include <math.h>

#include <algorithm>

#include <mutex>

#include "../../include/crf.h"
#include "kernels.hpp"

// Fixed device scratch of crf_layer_drift_noalloc (tables and partials), one
// copy per device, held until the process ends.  Host code never passes this
// name to a kernel: the device address comes from hipGetSymbolAddress.
static __device__ __align__(256) char scratch[CRF_DRIFT_NOALLOC_MAX_BYTES];

namespace crf {
namespace {

template <typename T>
CRF_DEV double tod(T x);
template <>
CRF_DEV double tod<float>(float x) { return (double)x; }
template <>
CRF_DEV double tod<bf16>(bf16 x) { return (double)bf2f(x); }

// Partials cross workgroups (and XCDs, whose L2 caches are not coherent with
// each other) as agent-scope accesses, which go to memory.
CRF_DEV void st_agent(double *p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
CRF_DEV double ld_agent(const double *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
CRF_DEV double sum16(double v) {  // over 16 consecutive lanes, in every lane
#pragma unroll
  for (int o = 8; o >= 1; o >>= 1) v += __shfl_xor(v, o, 16);
  return v;
}

template <typename T>
CRF_DEV void add_vec(double &acc, u32x4 a, u32x4 b) {
  constexpr int VE = 16 / sizeof(T);
  typedef T vec __attribute__((ext_vector_type(VE)));
  const vec av = __builtin_bit_cast(vec, a), bv = __builtin_bit_cast(vec, b);
#pragma unroll
  for (int e = 0; e < VE; ++e) {
    const double d = tod<T>(av[e]) - tod<T>(bv[e]);
    acc = fma(d, d, acc);
  }
}

constexpr int SQ_LDS = 512;  // squared distances the last workgroup keeps at hand

template <typename T>
__global__ __launch_bounds__(256) void drift_kernel(const DriftArgs p) {
  constexpr int VE = 16 / sizeof(T);  // elements per load
  constexpr int VB = 4, UN = 4;       // versions and loads per tensor in flight
  __shared__ double red[4][VB];
  __shared__ bool is_last;
  __shared__ double sq_lds[SQ_LDS];
  const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
  // (the next chunk's descriptors are read one chunk ahead)
  DriftChunk ch{}, chn{};
  DriftSeg sg{}, sgn{};
  if ((int)blockIdx.x < p.n_chunks) {
    chn = p.chunks[blockIdx.x];
    sgn = p.segs[chn.seg];
  }
  for (int c = blockIdx.x; c < p.n_chunks; c += gridDim.x) {
    ch = chn;
    sg = sgn;
    if (c + (int)gridDim.x < p.n_chunks) {
      chn = p.chunks[c + gridDim.x];
      sgn = p.segs[chn.seg];
    }
    const int64_t start = (int64_t)ch.idx * p.chunk;
    const int len = (int)min((int64_t)p.chunk, sg.count - start);
    const T *a = (const T *)sg.a + start;
    for (int v0 = 0; v0 < p.n_versions; v0 += VB) {
      const T *b[VB];
      uintptr_t bits = (uintptr_t)a;
#pragma unroll
      for (int v = 0; v < VB; ++v) {  // a version past the last repeats it (its sum is dropped)
        b[v] = (const T *)p.b[(int64_t)ch.seg * p.n_versions + min(v0 + v, p.n_versions - 1)] + start;
        bits |= (uintptr_t)b[v];
      }
      const int nv = min(VB, p.n_versions - v0);
      double acc[VB] = {0.0, 0.0, 0.0, 0.0};
      int done = 0;  // elements summed by the vector loop
      if ((bits & 15) == 0) {
        const int nvec = len / VE;
        for (int i0 = 0; i0 < nvec; i0 += 256 * UN) {
          u32x4 av[UN], bv[VB][UN];
#pragma unroll
          for (int u = 0; u < UN; ++u) {
            // lanes past the end load the chunk's first vector and drop it
            const int i = i0 + 256 * u + tid;
            const int64_t o = (int64_t)(i < nvec ? i : 0) * VE;
            av[u] = ld16(a + o);
#pragma unroll
            for (int v = 0; v < VB; ++v)
              if (v < nv) bv[v][u] = ld16(b[v] + o);
          }
#pragma unroll
          for (int u = 0; u < UN; ++u)
            if (i0 + 256 * u + tid < nvec)
#pragma unroll
              for (int v = 0; v < VB; ++v)
                if (v < nv) add_vec<T>(acc[v], av[u], bv[v][u]);
        }
        done = nvec * VE;
      }
      for (int i = done + tid; i < len; i += 256)  // the remainder, or everything when a tensor is not 16-byte aligned
#pragma unroll
        for (int v = 0; v < VB; ++v)
          if (v < nv) {
            const double d = tod<T>(a[i]) - tod<T>(b[v][i]);
            acc[v] = fma(d, d, acc[v]);
          }
#pragma unroll
      for (int v = 0; v < VB; ++v) {
        double s = sum16(acc[v]);
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        if (lane == 0) red[wave][v] = s;
      }
      __syncthreads();
      if (tid < nv)
        st_agent(p.partials + (int64_t)(v0 + tid) * p.n_chunks + c,
                 (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]));
      __syncthreads();
    }
  }
  // the last workgroup to get here sums everybody's partials
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's partials have reached memory
  __syncthreads();
  if (tid == 0)
    is_last = __hip_atomic_fetch_add(p.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
  __syncthreads();
  if (!is_last) return;
  // 16 lanes per output: sq[v, l] = sum of layer l's chunks, then per layer
  // d_l = sqrt(sum_k sq[anchor(l), k]) (or of its own slice).  One workgroup is
  // all latency here, so four outputs' loads go out before the first sum.
  const int g = tid / 16, l16 = tid % 16, n_out = p.n_versions * p.n_layers;
  for (int o0 = g; o0 < n_out; o0 += 64) {
    double s[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int o = o0 + 16 * j;
      s[j] = 0.0;
      if (o < n_out) {
        const int v = o / p.n_layers, l = o % p.n_layers;
        const double *q = p.partials + (int64_t)v * p.n_chunks;
#pragma unroll 4
        for (int c = p.first[l] + l16; c < p.first[l + 1]; c += 16) s[j] += ld_agent(q + c);
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int o = o0 + 16 * j;
      s[j] = sum16(s[j]);
      if (l16 == 0 && o < n_out) {
        if (o < SQ_LDS) sq_lds[o] = s[j];
        st_agent(p.sq + o, s[j]);
        if (p.sq_out) p.sq_out[o] = (float)s[j];
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  for (int l = g; l < p.n_layers; l += 16) {
    const int q0 = p.anchor[l] * p.n_layers;
    double s = 0.0;
    if (p.per_layer_only) {
      s = q0 + l < SQ_LDS ? sq_lds[q0 + l] : ld_agent(p.sq + q0 + l);
    } else {
      for (int k = l16; k < p.n_layers; k += 16) s += q0 + k < SQ_LDS ? sq_lds[q0 + k] : ld_agent(p.sq + q0 + k);
      s = sum16(s);
    }
    if (l16 == 0) {
      const double d = sqrt(s);
      p.drift[l] = (float)d;
      p.risk[l] = (float)(d * (p.sens ? (double)p.sens[l] : 1.0));
    }
  }
}

// Workgroups of a launch: 3 of 256 threads fit a CU.  28 layers of 7B shapes x 2
// versions (242 MB): 256 -> 101 us a call, 512 -> 75, 768 -> 67, 1024 -> 73.
constexpr int DRIFT_GRID = 768;
constexpr int MAX_DEVICES = 64;
void *g_scratch[MAX_DEVICES];
std::once_flag g_scratch_once[MAX_DEVICES];
hipError_t g_scratch_err[MAX_DEVICES];

}  // namespace

hipError_t drift_noalloc_scratch(void **out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  // once per device, with that device current (it is: hipGetDevice above)
  std::call_once(g_scratch_once[dev], [dev] {
    void *p = nullptr;
    g_scratch_err[dev] = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    g_scratch[dev] = g_scratch_err[dev] == hipSuccess ? p : nullptr;
  });
  *out = g_scratch[dev];
  return g_scratch_err[dev];
}

hipError_t launch_drift(hipStream_t s, bool f32, const DriftArgs &a) {
  // at most DRIFT_GRID workgroups, each with every DRIFT_GRID-th chunk: the
  // tickets are atomics on one address (no adapter at all: one, which writes zeros)
  const dim3 grid(std::max(1, std::min(a.n_chunks, DRIFT_GRID)));
  if (f32)
    hipLaunchKernelGGL(drift_kernel<float>, grid, dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(drift_kernel<bf16>, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace crf
