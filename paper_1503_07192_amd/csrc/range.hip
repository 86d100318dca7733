// Exactness certificate for graphs whose total edge weight reaches INF.
//
// Every stored distance is min(exact distance, INF) (see tiles.h), so the
// only possible error is a finite distance at or above INF shown as INF.  The
// build proves that none exists:
//   (i)   every component's edge weights sum below INF, so APSP(C) is exact;
//   (ii)  no BG entry is INF between two boundary vertices that are connected
//         in G (connected components computed here), so BG is exact;
//   (iii) 2 * max finite APSP(C) entry + max finite BG entry < INF, so every
//         sum a query forms on an optimal decomposition stays below INF.
// Under (i)-(iii) all answers are exact; otherwise the build reports
// SPQ_ERANGE.
#include "spq_internal.h"
#include "tiles.h"

namespace spq {

__global__ void k_cc_init(int32_t n, int32_t* __restrict__ label) {
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
       v += (int64_t)gridDim.x * blockDim.x)
    label[v] = (int32_t)v;
}

// Labels only decrease and always point to a smaller or equal id, so every
// chain ends at a root.  They are read through the caches: an older label is
// an earlier ancestor, and a pass that hooks nothing reads settled ones.
__device__ __forceinline__ int32_t cc_label(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ int32_t cc_root(const int32_t* label, int32_t x) {
  for (;;) {
    const int32_t p = cc_label(label + x);
    if (p == x) return x;
    x = p;
  }
}

// The same, halving the chain on the way (every vertex passed points past its
// parent afterwards; atomicMin, as another thread may have lowered it further).
__device__ __forceinline__ int32_t cc_root_halve(int32_t* label, int32_t x) {
  for (;;) {
    const int32_t p = cc_label(label + x);
    if (p == x) return x;
    const int32_t g = cc_label(label + p);
    if (g == p) return p;
    atomicMin(label + x, g);
    x = g;
  }
}

// Hooks the larger root of every edge under the smaller one.  Bound by the
// chains' dependent loads and by the atomics on the same few roots in the second
// pass; `changed` is a plain store by one lane per wave.  1.2 million edges, three
// passes: 3.4 -> 0.7 ms (an atomicOr per hooked edge on the one word, loads past
// every cache and an atomicMin per edge between the last trees before).
__global__ void k_cc_hook(int64_t m, const int32_t* __restrict__ eu, const int32_t* __restrict__ ev,
                          int32_t* label, u32* __restrict__ changed) {
  bool hooked = false;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int32_t a = cc_root_halve(label, eu[e]), b = cc_root_halve(label, ev[e]);
    if (a != b) {
      // in the later passes many edges join the same two trees: most find the
      // root already hooked at least as low
      const int32_t hi = max(a, b), lo = min(a, b);
      if (__hip_atomic_load(label + hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > lo)
        atomicMin(label + hi, lo);
      hooked = true;
    }
  }
  const unsigned long long any = __ballot(hooked);
  if (any && (threadIdx.x & 63) == __ffsll((unsigned long long)any) - 1) *changed = 1u;
}

__global__ void k_cc_flatten(int32_t n, int32_t* label) {
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
       v += (int64_t)gridDim.x * blockDim.x)
    label[v] = cc_root(label, (int32_t)v);
}

__global__ void k_bg_label(int32_t V, const int32_t* __restrict__ bgvert, const int32_t* __restrict__ label,
                           int32_t* __restrict__ bglabel) {
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < V;
       x += (int64_t)gridDim.x * blockDim.x)
    bglabel[x] = label[bgvert[x]];
}

__device__ __forceinline__ u32 wave_max(u32 v) {
  for (int o = 32; o > 0; o >>= 1) v = max(v, (u32)__shfl_xor((int)v, o));
  return v;
}

// Largest entry below INF of a contiguous array (16-byte aligned, count a
// multiple of 4: whole 64-tiles).  Bound by reading it: at most 2,048
// workgroups with 16-byte loads and one atomic each (an atomic per wave of
// 65,535 workgroups on the one word read 537 MB in 3.0 ms, now 0.11 ms).
__global__ __launch_bounds__(256) void k_max_finite(int64_t count4, const uint4* __restrict__ a,
                                                    u32* __restrict__ out) {
  __shared__ u32 part[4];
  u32 best = 0;  // largest finite value plus one: INF becomes 0
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count4; i += 2 * step) {
    const uint4 v = a[i], w = i + step < count4 ? a[i + step] : make_uint4(INF, INF, INF, INF);
    best = max(max(max(best, (v.x + 1) & INF), max((v.y + 1) & INF, (v.z + 1) & INF)), (v.w + 1) & INF);
    best = max(max(max(best, (w.x + 1) & INF), max((w.y + 1) & INF, (w.z + 1) & INF)), (w.w + 1) & INF);
  }
  best = wave_max(best);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = best;
  __syncthreads();
  if (threadIdx.x == 0) {
    best = max(max(part[0], part[1]), max(part[2], part[3]));
    if (best) atomicMax(out, best - 1);
  }
}

// Flat BG: rows p < V, columns q < V.
__global__ void k_check_flat(int32_t V, int64_t Vp, const u32* __restrict__ BG,
                             const int32_t* __restrict__ bglabel, u32* __restrict__ bad,
                             u32* __restrict__ mbg) {
  const int64_t p = blockIdx.x;
  const u32* row = BG + p * Vp;
  const int32_t lp = bglabel[p];
  u32 best = 0, wrong = 0;
  for (int64_t q = threadIdx.x; q < V; q += blockDim.x) {
    const u32 v = row[q];
    if (v < INF) best = max(best, v);
    else if (bglabel[q] == lp) wrong = 1;
  }
  best = wave_max(best);
  wrong = wave_max(wrong);
  if ((threadIdx.x & 63) == 0) {
    if (best) atomicMax(mbg, best);
    if (wrong) atomicOr(bad, 1u);
  }
}

// Two-level store: block (pair (s1, s2), 16-row chunk of group s1), s1 <= s2.
__global__ void k_check_hier(int32_t ngroups, const int32_t* __restrict__ gV,
                             const int32_t* __restrict__ gbg0, const int64_t* __restrict__ pairbase,
                             const int32_t* __restrict__ bgrow, const int32_t* __restrict__ bgnb,
                             const int32_t* __restrict__ bglocal, const int32_t* __restrict__ bglabel,
                             const u32* __restrict__ H, u32* __restrict__ bad, u32* __restrict__ mbg) {
  const int32_t s1 = (int32_t)(blockIdx.x / ngroups), s2 = (int32_t)(blockIdx.x % ngroups);
  if (s1 > s2) return;
  const int32_t V1 = gV[s1], V2 = gV[s2], g1 = gbg0[s1], g2 = gbg0[s2];
  const u32* base = H + pairbase[(int64_t)s1 * ngroups + s2];
  u32 best = 0, wrong = 0;
  for (int32_t r = 0; r < 16; r++) {
    const int32_t x = (int32_t)blockIdx.y * 16 + r;
    if (x >= V1) break;
    const int32_t xg = g1 + x;
    const int64_t rb = (int64_t)bgrow[xg] * V2;
    const int64_t nbx = bgnb[xg], locx = bglocal[xg];
    const int32_t lx = bglabel[xg];
    for (int32_t y = threadIdx.x; y < V2; y += blockDim.x) {
      const int32_t yg = g2 + y;
      const u32 v = base[rb + nbx * bgrow[yg] + locx * bgnb[yg] + bglocal[yg]];
      if (v < INF) best = max(best, v);
      else if (bglabel[yg] == lx) wrong = 1;
    }
  }
  best = wave_max(best);
  wrong = wave_max(wrong);
  if ((threadIdx.x & 63) == 0) {
    if (best) atomicMax(mbg, best);
    if (wrong) atomicOr(bad, 1u);
  }
}

static inline unsigned rblocks(int64_t items) {
  int64_t b = (items + 255) / 256;
  if (b < 1) b = 1;
  if (b > 65535) b = 65535;
  return (unsigned)b;
}

hipError_t launch_cc_init(int32_t n, int32_t* label, hipStream_t s) {
  k_cc_init<<<rblocks(n), 256, 0, s>>>(n, label);
  return hipGetLastError();
}

hipError_t launch_cc_round(int64_t m, const int32_t* eu, const int32_t* ev, int32_t n, int32_t* label,
                           u32* changed, hipStream_t s) {
  if (m > 0) k_cc_hook<<<rblocks(m), 256, 0, s>>>(m, eu, ev, label, changed);
  k_cc_flatten<<<rblocks(n), 256, 0, s>>>(n, label);
  return hipGetLastError();
}

hipError_t launch_bg_label(int32_t V, const int32_t* bgvert, const int32_t* label, int32_t* bglabel,
                           hipStream_t s) {
  if (V > 0) k_bg_label<<<rblocks(V), 256, 0, s>>>(V, bgvert, label, bglabel);
  return hipGetLastError();
}

hipError_t launch_certificate(const CertArgs& a, hipStream_t s) {
  if (a.comp_elems > 0) {
    const unsigned g = rblocks(a.comp_elems / 8);
    k_max_finite<<<g < 2048 ? g : 2048, 256, 0, s>>>(a.comp_elems / 4, reinterpret_cast<const uint4*>(a.M), a.mc);
  }
  if (a.V > 0 && !a.bg_checked) {
    if (a.H) {
      dim3 grid((unsigned)((int64_t)a.ngroups * a.ngroups), (unsigned)((a.Vgp + 15) / 16));
      k_check_hier<<<grid, 256, 0, s>>>(a.ngroups, a.gV, a.gbg0, a.pairbase, a.bgrow, a.bgnb,
                                         a.bglocal, a.bglabel, a.H, a.bad, a.mbg);
    } else {
      k_check_flat<<<(unsigned)a.V, 256, 0, s>>>(a.V, a.Vp, a.BG, a.bglabel, a.bad, a.mbg);
    }
  }
  return hipGetLastError();
}

}  // namespace spq
