// Two-level all-pairs distances in BG.
//
// The preprocessing of Algorithm 1 applied once more, one level up: BG itself
// is partitioned into groups of consecutive components.  For a group S:
//   * BG_S = the subgraph of BG induced by S's boundary vertices (the clique
//     edges of S's components plus the G edges between them), closed by
//     Floyd-Warshall: d_S (a batch of equally sized matrices);
//   * B2(S) = vertices of BG_S with a BG edge leaving S (the boundary of the
//     group partition, Section 2's definition applied to BG).
// BG2 = the B2 vertices of all groups, joined by d_S between the B2 vertices
// of one group and by the G edges between groups; closed by Floyd-Warshall it
// holds d_BG between B2 vertices (Lemma 1 for the group partition).  Every
// other BG distance is Algorithm 2's formula at the group level (Lemma 3):
//   D(S1,S2)[x][y] = min over a in B2(S1), b in B2(S2) of
//                    d_S1(x,a) + d_BG2(a,b) + d_S2(b,y),
//   and when S1 = S2 also d_S1(x,y).
// It is evaluated as two min-plus products, XT = D2(S1,S2)^T (x) R_S1 and
// D = XT^T (x) R_S2, where R_S = rows B2(S) of d_S (by symmetry, the columns
// too).  Only S1 <= S2 is stored; a query swaps its endpoints otherwise.
//
// Storage of D(S1,S2) (V_S1 x V_S2 values at pairbase[S1][S2]): the rows of
// one component C1 of S1 form a band; inside it, the block of component C2 of
// S2 is nb(C1) x nb(C2) contiguous values, so a query reads one contiguous
// block.  Element (x, y) is at
//   rowoff(x) * V_S2 + nb(x) * rowoff(y) + loc(x) * nb(y) + loc(y)
// with rowoff = first BG id of the component inside its group, loc = index
// inside the component's boundary.
#include "spq_internal.h"
#include "tiles.h"

namespace spq {

// Group matrix init: 0 on the diagonal, the APSP(C) distance inside one
// component, INF elsewhere and on the padding.
__global__ void k_grp_init(int32_t Vgp, const int32_t* __restrict__ gbg0, const int32_t* __restrict__ gV,
                           const int32_t* __restrict__ bgcomp, const int32_t* __restrict__ bglocal,
                           const int32_t* __restrict__ bgoff, const int32_t* __restrict__ nb,
                           const int32_t* __restrict__ P, const int64_t* __restrict__ moff,
                           const u32* __restrict__ M, u32* __restrict__ Mg) {
  const int s = blockIdx.y;
  const int64_t p = blockIdx.x;
  u32* out = Mg + ((int64_t)s * Vgp + p) * Vgp;
  const int32_t g0 = gbg0[s];
  int64_t lo = 0, hi = 0;
  const u32* mrow = nullptr;
  if (p < gV[s]) {
    const int32_t x = g0 + (int32_t)p;
    const int32_t c = bgcomp[x];
    lo = bgoff[c] - g0;
    hi = lo + nb[c];
    mrow = M + moff[c] + (int64_t)bglocal[x] * P[c] - lo;
  }
  for (int64_t q0 = (int64_t)threadIdx.x * 4; q0 < Vgp; q0 += (int64_t)blockDim.x * 4) {
    u32 v[4];
#pragma unroll
    for (int t = 0; t < 4; t++) {
      const int64_t q = q0 + t;
      v[t] = (q == p) ? 0u : (q >= lo && q < hi) ? mrow[q] : INF;
    }
    *reinterpret_cast<uint4*>(out + q0) = make_uint4(v[0], v[1], v[2], v[3]);
  }
}

// G edges between boundary vertices of different components: inside a group
// they become entries of the group matrix; between groups they mark both ends
// as level-2 boundary vertices.
__global__ void k_grp_edges(int64_t m, const int32_t* __restrict__ eu, const int32_t* __restrict__ ev,
                            const int32_t* __restrict__ w, const int32_t* __restrict__ comp,
                            const int32_t* __restrict__ local, const int32_t* __restrict__ bgoff,
                            const int32_t* __restrict__ grp, const int32_t* __restrict__ gbg0,
                            int32_t Vgp, u32* __restrict__ Mg, uint8_t* __restrict__ flag2) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int32_t u = eu[e], v = ev[e];
    const int32_t cu = comp[u], cv = comp[v];
    if (cu == cv) continue;
    const int32_t su = grp[cu], sv = grp[cv];
    const int32_t xu = bgoff[cu] + local[u], xv = bgoff[cv] + local[v];
    if (su == sv) {
      u32* base = Mg + (int64_t)su * Vgp * Vgp;
      const int64_t a = xu - gbg0[su], b = xv - gbg0[su];
      atomicMin(base + a * Vgp + b, (u32)w[e]);
      atomicMin(base + b * Vgp + a, (u32)w[e]);
    } else {
      flag2[xu] = 1;
      flag2[xv] = 1;
    }
  }
}

// One workgroup per group: lists the level-2 boundary vertices of the group in
// ascending order (b2list), their rank (b2rank, -1 if not one) and count.
__global__ __launch_bounds__(256) void k_b2_scan(const int32_t* __restrict__ gbg0,
                                                 const int32_t* __restrict__ gV,
                                                 const uint8_t* __restrict__ flag2, int32_t Vgp,
                                                 int32_t* __restrict__ b2list, int32_t* __restrict__ b2rank,
                                                 int32_t* __restrict__ m2) {
  __shared__ int32_t wsum[4];
  const int s = blockIdx.x;
  const int32_t g0 = gbg0[s], V = gV[s];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  int32_t base = 0;
  for (int32_t c0 = 0; c0 < V; c0 += 256) {
    const int32_t p = c0 + (int32_t)threadIdx.x;
    const bool f = p < V && flag2[g0 + p];
    const unsigned long long bal = __ballot(f);
    const int32_t before = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) wsum[wid] = __popcll(bal);
    __syncthreads();
    int32_t woff = 0, tot = 0;
    for (int i = 0; i < 4; i++) {
      if (i < wid) woff += wsum[i];
      tot += wsum[i];
    }
    if (p < V) {
      if (f) {
        const int32_t r = base + woff + before;
        b2list[(int64_t)s * Vgp + r] = p;
        b2rank[g0 + p] = r;
      } else {
        b2rank[g0 + p] = -1;
      }
    }
    base += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) m2[s] = base;
}

// R_S: rows B2(S) of d_S (m2pmax rows per group, INF rows past m2[S]).
__global__ void k_r_gather(int32_t Vgp, int32_t m2pmax, const int32_t* __restrict__ m2,
                           const int32_t* __restrict__ b2list, const u32* __restrict__ Mg,
                           u32* __restrict__ R) {
  const int s = blockIdx.y;
  const int32_t i = blockIdx.x;
  uint4* dst = reinterpret_cast<uint4*>(R + ((int64_t)s * m2pmax + i) * Vgp);
  const int32_t n4 = Vgp / 4;
  if (i < m2[s]) {
    const uint4* src =
        reinterpret_cast<const uint4*>(Mg + ((int64_t)s * Vgp + b2list[(int64_t)s * Vgp + i]) * Vgp);
    for (int32_t q = threadIdx.x; q < n4; q += blockDim.x) dst[q] = src[q];
  } else {
    for (int32_t q = threadIdx.x; q < n4; q += blockDim.x) dst[q] = make_uint4(INF, INF, INF, INF);
  }
}

// BG2 matrix init: d_S between B2 vertices of one group, 0 on the diagonal,
// INF elsewhere and on the padding.  With super-groups (tbase, tsize: their first
// BG2 ids and sizes) matrix blockIdx.y is BG2 on super-group blockIdx.y's vertices
// alone: level 3 overwrites the rest of BG2, so nothing else of it is made first
// (29,499 BG2 vertices in 16 super-groups: all of BG2, then its blocks gathered,
// 0.81 ms; the blocks alone 0.09).
__global__ void k_bg2_init(int32_t V2, int64_t ld, int32_t ngroups, const int32_t* __restrict__ b2off,
                           const int32_t* __restrict__ b2list, int32_t Vgp, const u32* __restrict__ Mg,
                           const int32_t* __restrict__ tbase, const int32_t* __restrict__ tsize,
                           u32* __restrict__ BG2) {
  const int64_t p = blockIdx.x, base = tbase ? tbase[blockIdx.y] : 0, i = base + p;
  u32* out = BG2 + (blockIdx.y * ld + p) * ld;
  int64_t lo = 0, hi = 0;
  const u32* prow = nullptr;
  const int32_t* list = nullptr;
  if (p < (tbase ? tsize[blockIdx.y] : V2)) {
    int32_t a = 0, b = ngroups - 1;  // group of B2 id i: largest s with b2off[s] <= i
    while (a < b) {
      const int32_t mid = (a + b + 1) >> 1;
      if (b2off[mid] <= i) a = mid; else b = mid - 1;
    }
    lo = b2off[a] - base;
    hi = b2off[a + 1] - base;
    list = b2list + (int64_t)a * Vgp;
    prow = Mg + ((int64_t)a * Vgp + list[p - lo]) * Vgp;
  }
  for (int64_t q0 = (int64_t)threadIdx.x * 4; q0 < ld; q0 += (int64_t)blockDim.x * 4) {
    u32 v[4];
#pragma unroll
    for (int t = 0; t < 4; t++) {
      const int64_t q = q0 + t;
      v[t] = (q == p) ? 0u : (q >= lo && q < hi) ? prow[list[q - lo]] : INF;
    }
    *reinterpret_cast<uint4*>(out + q0) = make_uint4(v[0], v[1], v[2], v[3]);
  }
}

// G edges between groups into BG2, or (tbase not null, super-groups of gpt
// groups) those inside a super-group into its matrix.
__global__ void k_bg2_edges(int64_t m, const int32_t* __restrict__ eu, const int32_t* __restrict__ ev,
                            const int32_t* __restrict__ w, const int32_t* __restrict__ comp,
                            const int32_t* __restrict__ local, const int32_t* __restrict__ bgoff,
                            const int32_t* __restrict__ grp, const int32_t* __restrict__ b2off,
                            const int32_t* __restrict__ b2rank, int64_t ld, int32_t gpt,
                            const int32_t* __restrict__ tbase, u32* __restrict__ BG2) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int32_t u = eu[e], v = ev[e];
    const int32_t cu = comp[u], cv = comp[v];
    if (cu == cv) continue;
    const int32_t su = grp[cu], sv = grp[cv];
    if (su == sv) continue;
    u32* M = BG2;
    int64_t base = 0;
    if (tbase) {
      const int32_t t = su / gpt;
      if (sv / gpt != t) continue;
      base = tbase[t];
      M += t * ld * ld;
    }
    const int64_t a = b2off[su] + b2rank[bgoff[cu] + local[u]] - base;
    const int64_t b = b2off[sv] + b2rank[bgoff[cv] + local[v]] - base;
    atomicMin(M + a * ld + b, (u32)w[e]);
    atomicMin(M + b * ld + a, (u32)w[e]);
  }
}

// Per BG vertex: first BG id of its component inside its group, and the
// component's boundary count (the layout terms of D(S1,S2)).
__global__ void k_hier_vmeta(int32_t V, const int32_t* __restrict__ bgcomp, const int32_t* __restrict__ bgoff,
                             const int32_t* __restrict__ nb, const int32_t* __restrict__ grp,
                             const int32_t* __restrict__ gbg0, const int32_t* __restrict__ bglocal,
                             int32_t* __restrict__ bgrow, int32_t* __restrict__ bgnb,
                             int32_t* __restrict__ bggrp, int4* __restrict__ meta) {
  const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= V) return;
  const int32_t c = bgcomp[x], s = grp[c];
  bgrow[x] = bgoff[c] - gbg0[s];
  bgnb[x] = nb[c];
  bggrp[x] = s;
  if (meta) meta[x] = make_int4(bgoff[c] - gbg0[s], nb[c], bglocal[x], 0);
}

// The counters' sums into `out` (pinned host memory; see launch_counts), and the
// counters cleared for the next replay.  By one wave.
__device__ __forceinline__ void counts_out(unsigned long long* exec, unsigned long long* out) {
  static_assert(MP_EXEC == 32, "two times sixteen counters, summed by sixteen lanes");
  const int l = threadIdx.x;
  unsigned long long n = l < EXEC_WORDS ? exec[l] : 0ull;
  if (l < EXEC_WORDS) exec[l] = 0ull;
  const unsigned long long comps = __shfl(n, MP_EXEC), bg = __shfl(n, MP_EXEC + 1);
  for (int o = 8; o > 0; o >>= 1) n += __shfl_xor(n, o);
  const unsigned long long second = __shfl(n, MP_EXEC / 2);
  if (l == 0) {
    out[0] = n + second + bg;
    out[1] = second;
    out[2] = comps;
  }
}

__global__ __launch_bounds__(64) void k_counts(unsigned long long* exec, unsigned long long* out) {
  counts_out(exec, out);
}

// Flat method: row x of the closed BG matrix into the blocked store of one
// group (the layout above with S1 = S2 = the only group).
__global__ void k_flat_store(int32_t V, int64_t Vp, const u32* __restrict__ BG,
                             const int32_t* __restrict__ bgrow, const int32_t* __restrict__ bgnb,
                             const int32_t* __restrict__ bglocal, u32* __restrict__ H,
                             unsigned long long* exec, unsigned long long* counted) {
  const int64_t x = blockIdx.x;
  if (x == 0 && threadIdx.x < 64) counts_out(exec, counted);
  const u32* row = BG + x * Vp;
  const int64_t rb = (int64_t)bgrow[x] * V, nbx = bgnb[x], locx = bglocal[x];
  for (int32_t y = threadIdx.x; y < V; y += blockDim.x)
    H[rb + nbx * bgrow[y] + locx * bgnb[y] + bglocal[y]] = row[y];
}

// ------------------------------------------------------- min-plus products --
// c = min(c, min over k < cnt of At[rows[k]][i] + B[bmap[rows[k]]][j]): the K
// rows are gathered through the list `rows` (rows k themselves when it is
// null; cnt of them), and B's rows once more through bmap.  Sixteen rows at a
// time straight to LDS, double buffered; a lane has the row numbers of the chunk
// after the one in flight in registers, so that a chunk waits for one load, not
// for three in a row.  Rows past cnt repeat the last one and are not multiplied
// beyond an even count.  118 VGPRs, four waves per SIMD (staged through
// registers it took 131 and three): the last product of a 30,700-row share 5.0 ->
// 4.7 ms, its 40 rounds' 7.5 -> 6.3.
__device__ __forceinline__ void mp_stream128_rows(u32 (&c)[8][8], const u32* At, int64_t ldA,
                                                  const u32* B, int64_t ldB,
                                                  const int32_t* __restrict__ rows, int cnt,
                                                  u32* sA, u32* sB, const int32_t* __restrict__ bmap) {
  constexpr int T = 128, KC = 16;
  if (cnt <= 0) return;
  const int wv = (int)threadIdx.x >> 6, r0 = (int)threadIdx.x >> 5, col = ((int)threadIdx.x & 31) * 4;
  int32_t ra[2], rb[2];  // this thread's rows of A and B, of the next chunk
  auto index = [&](int k0) {
#pragma unroll
    for (int h = 0; h < 2; h++) {
      const int k = min(k0 + h * 8 + r0, cnt - 1);
      ra[h] = rows ? rows[k] : k;
      rb[h] = bmap[ra[h]];
    }
  };
  auto load = [&](int buf) {
#pragma unroll
    for (int h = 0; h < 2; h++) {
      lds_load16(At + ra[h] * ldA + col, sA + buf * KC * T + (h * 256 + wv * 64) * 4);
      lds_load16(B + rb[h] * ldB + col, sB + buf * KC * T + (h * 256 + wv * 64) * 4);
    }
  };
  index(0);
  load(0);
  index(KC);
  wait_loads();
  __syncthreads();
#pragma unroll 1
  for (int k = 0; k < cnt; k += KC) {
    const int cur = (k / KC) & 1;
    if (k + KC < cnt) {
      load(cur ^ 1);
      index(k + 2 * KC);
    }
    minplus_lds<T, 1>(c, sA + cur * KC * T, sB + cur * KC * T, min(KC, (cnt - k + 1) & ~1));
    wait_loads();
    __syncthreads();
  }
}

// The composition kernels fit in 128 VGPRs without spilling: four waves per
// SIMD (four workgroups per CU) instead of two or three.
#define SPQ_MP_ATTR __attribute__((amdgpu_waves_per_eu(4, 4)))

__device__ __forceinline__ void fill_inf(u32 (&c)[8][8]) {
#pragma unroll
  for (int i = 0; i < 8; i++)
#pragma unroll
    for (int j = 0; j < 8; j++) c[i][j] = INF;
}

// The certificate's per-wave reduction: largest finite value, and whether
// an INF joins two vertices connected in G.  seen: *cert_mbg as read before; a
// wave that does not raise it leaves the word alone (one atomic per wave on it, 14 ns
// each, was what bound the products of a 400,000-vertex graph: 23.7 -> 19.0 ms).
__device__ __forceinline__ void cert_reduce(u32 best, u32 wrong, u32 seen, u32* cert_bad, u32* cert_mbg) {
  for (int o = 32; o > 0; o >>= 1) {
    best = max(best, (u32)__shfl_xor((int)best, o));
    wrong |= (u32)__shfl_xor((int)wrong, o);
  }
  if ((threadIdx.x & 63) == 0) {
    if (best > seen) atomicMax(cert_mbg, best);
    if (wrong) atomicOr(cert_bad, 1u);
  }
}

// Where the composition's results go: the query layout (with or without the
// certificate), or (level 3) the dense BG2 matrix.
struct CompStore {
  const int32_t* g0;       // first BG (level 3: BG2) id of every group
  const int32_t* rank;     // per such id its index among the group's boundary vertices, -1 if
                           // none (NULL, test hooks: every column is multiplied)
  const int4* meta;        // per id: row offset, |B|, index inside its component
  const u32* Mg;           // the groups' closures (leading dimension Vp)
  int32_t ngroups;
  const int64_t* pairbase;
  u32* H;
  const int32_t* bglabel;  // certificate
  u32 *cert_bad, *cert_mbg;
  // dense store (level 3): element (x, y) of the pair block (S1, S2) at
  // dense[(g0[S1] + x) * ldo + g0[S2] + y]; NULL: the query layout
  u32* dense;
  int64_t ldo;
};

// The composition's products, pruned.
//
// Both products have the form out[x][y] = min over k < K of A[k][x] + B[k][y]
// with K boundary vertices of one group, A the distances to them from far
// away (the other group's vertices) and B rows of the group's own closure.
// Most k never give a minimum: shortest paths from a whole region enter a
// group through few of its boundary vertices.  For a row tile X (MP_SR rows)
// let r(x) be any value per row and mn[k] <= A[k][x] - r(x) <= mx[k] for x in
// X.  If mx[k'] + B[k'][y] <= mn[k] + B[k][y], then A[k'][x] + B[k'][y] <=
// A[k][x] + B[k][y] for every x of X: column y needs k no more once it has
// k'.  So with U[y] = min over k' of mx[k'] + B[k'][y], reached first at
// arg[y], the rows X x columns Y of the product need only the k that some y
// of Y has as arg[y] or with mn[k] + B[k][y] < U[y]: exactly the same minima
// from (measured) a seventh to a half of the K.  r is near a row's minimum,
// so that mx - mn stays small.
//
// A column y that is itself one of the K (y in B2 of its group) takes part in
// neither: out[x][y] = A[y][x], its minimum (B[y][y] = 0, and no other k goes
// lower, A being distances in a closed graph and B at least those distances), and the
// product starts from it.
//
// Measured (MI355X): 400,000 Delaunay vertices in 128 groups, both levels'
// products 79 -> 40 ms with all tests, the second one executing 0.48e12
// relaxations instead of 1.45e12; build 117 -> 58.5 ms.  A 30,700-row share of a
// 1024 x 1024 grid: 45 -> 19 ms, 0.13e12 of 0.93e12 relaxations; build 79.5 ->
// 46.7 ms.  The test stays exact and costs little on operands it cannot prune.
//
// Three kernels per product and chunk of pairs: k_mp_stats (mn, mx per row
// tile and k), k_mp_keep (per row tile and 64 columns a bit mask of the k to
// keep), k_mp_prod (the product over the kept k).  The test costs 6 VALU
// instructions per (k, 64 columns, row tile), 1/16 of the full product at 64
// rows.
// rows per tile of the statistics, row tiles per wave of k_mp_keep: the first
// product has few rows (a group's boundary, 200 or so), the second a whole
// group's.  There 128 rows per tile test half as often as 64 and keep 10 - 17%
// more: second product and test 21.6 + 5.4 ms against 20.6 + 8.2 on 400,000
// Delaunay vertices in 128 groups, 12.4 + 3.5 against 11.8 + 6.6 ms on a share
// of 32 of a 1024 x 1024 grid's 256 groups (now, at 128: 18.9 + 4.8 and 10.5 + 2.4)
template <int SIDE>
constexpr int MP_SR = SIDE ? 128 : 64;
template <int SIDE>
constexpr int MP_RG = SIDE ? 8 : 4;
template <int SIDE>
constexpr int MP_KU = 32 / MP_RG<SIDE>;  // k per step of k_mp_keep
constexpr int MP_T = 64;           // rows and columns of a product tile (one wave)
constexpr int MP_KC = 4;           // k per LDS step of a product
constexpr int MP_RING = 4;         // steps in LDS
// Statistics are kept above MP_SHIFT (only their differences matter), the
// upper ones clamped to [0, MP_BIG], the lower ones to [-MP_BIG - 1, MP_BIG],
// B to MP_BIG: no sum overflows.  A bound with a term at MP_BIG is none; a lower
// one at -MP_BIG - 1 is below every bound.
constexpr int32_t MP_BIG = (1 << 29) - 1, MP_SHIFT = 1 << 27;
constexpr int32_t MP_ALL = 1 << 30, MP_NONE = -(1 << 30);  // bounds above and below every sum

typedef const __attribute__((address_space(4))) int32_t* cptr32;  // scalar loads

// One chunk of the composition's pairs, as its kernels take it.
struct MpArgs {
  const int2* plist;     // pair of slot i: plist[pbase + i]
  int32_t pbase, np;     // pairs of the launch
  int32_t Vp, Kp;        // row length and rows per slot of XT, R
  int32_t NT, NC, NW;    // row tiles (whole MP_RG), column tiles, mask words
  const int32_t *m2, *gV, *b2off;
  const u32* D2;         // D2: dense (pstride 0), or a column panel per group S2
  int64_t ldd, pstride;  //   (pstride apart, column j = its j-th boundary vertex)
  const u32* D2t;        // D2 transposed, for swapped pairs
  int64_t ldt;
  const u32* R;
  u32* XT;
  int32_t* stats;
  unsigned long long* mask;
  unsigned long long* exec;  // 16 counters
  CompStore cs;
  // side 2, the last product of a share's Bellman-Ford: rows (share sources), the blocks'
  // first level-2 ids, their rows outside B3 (nstride apart) and the table they lie in
  int32_t rows, nstride;
  const int32_t *boff, *nlist;
  u32* DT;
};

// One side of the composition for the pair of a slot: 0 the first product,
// 1 the second; 2: block `slot` of the Bellman-Ford's last product, K its B3 rows (of
// DT, gathered into XT; leading dimension ldd), columns its other rows.
struct MpSide {
  int32_t g;      // the group whose boundary vertices are the K and whose closure rows are B
  int32_t K;      // its boundary vertices
  int32_t W;      // its vertices: columns of the product
  int32_t rows;   // rows of the product
  const u32* A;   // A[k * lda + row]
  int64_t lda;
};

__device__ __forceinline__ MpSide mp_side(int side, const MpArgs& a, int32_t slot) {
  MpSide m;
  if (side == 2) {
    m.g = slot;
    m.K = a.m2[slot];
    m.W = a.gV[slot];
    m.rows = a.rows;
    m.A = a.XT + (int64_t)slot * a.Kp * a.ldd;
    m.lda = a.ldd;
    return m;
  }
  const int2 pr = a.plist[a.pbase + slot];
  const bool sw = (pr.y & PAIR_SWAP) != 0;
  const int32_t s1 = pr.x, s2 = pr.y & ~PAIR_SWAP;
  m.g = side ? s2 : s1;
  m.K = a.m2[m.g];
  m.W = a.gV[m.g];
  if (side) {
    m.rows = a.gV[s1];
    m.A = a.XT + (int64_t)slot * a.Kp * a.Vp;
    m.lda = a.Vp;
  } else {
    // D2[B2(s1)][B2(s2)] (row a, column b); a swapped pair reads it from the
    // transposed table (rows: level-2 ids)
    m.rows = a.m2[s2];
    m.A = sw ? a.D2t + (int64_t)a.b2off[s1] * a.ldt + a.b2off[s2]
             : a.D2 + (int64_t)s2 * a.pstride + (int64_t)a.b2off[s1] * a.ldd +
                   (a.pstride ? 0 : a.b2off[s2]);
    m.lda = sw ? a.ldt : a.ldd;
  }
  return m;
}

// mn, mx of every k for the row tile of blockIdx.x (pair blockIdx.y), laid out as
// k_mp_keep reads them (one wave's MP_RG row tiles and MP_KU k in a row; k from K on
// to a whole MP_KU bound nothing).  r(x) = the minimum over up to 16 of the K rows,
// spread evenly.  Sixteen-byte loads, MP_SR / 4 lanes per k:
// bound by reading A once (plus the sampled rows).  Rows that are INF for every
// k (unreachable) are left out; a tile without any other row keeps each
// column's arg only.  Where a row is INF in the sample only, the tile's
// statistics are made to keep every k.
template <int SIDE>
__global__ __launch_bounds__(256) void k_mp_stats(MpArgs a) {
  constexpr int SR = MP_SR<SIDE>, L = SR / 4, G = 256 / L;  // lanes per k, k per step
  static_assert(L == 16 || L == 32, "the reduction's lanes");
  __shared__ u32 smin[16][SR];
  __shared__ int odd, live;
  const int32_t slot = blockIdx.y, tile = blockIdx.x;
  const MpSide m = mp_side(SIDE, a, slot);
  constexpr int RG = MP_RG<SIDE>, KU = MP_KU<SIDE>;
  int32_t* out = a.stats + ((int64_t)slot * a.NT + tile / RG * RG) * 2 * a.Kp + tile % RG;
  auto put = [&](int32_t k, int32_t mn, int32_t mx) {
    out[(int64_t)k * RG] = mn;
    out[((int64_t)a.Kp + k) * RG] = mx;
  };
  const int32_t Kr = (m.K + KU - 1) / KU * KU;
  if ((int32_t)threadIdx.x < Kr - m.K) put(m.K + threadIdx.x, MP_BIG, MP_BIG);
  const int32_t x0 = tile * SR, nx = min(m.rows - x0, SR);
  if (nx <= 0) {  // k_mp_keep reads whole groups of row tiles
    for (int32_t k = threadIdx.x; k < m.K; k += 256) put(k, MP_BIG, 0);
    return;
  }
  if (threadIdx.x == 0) odd = live = 0;
  const int l = threadIdx.x % L, kg = threadIdx.x / L, x = l * 4;
  const u32* A = m.A + x0;
  auto load = [&](int32_t k) -> uint4 {
    const u32* p = A + (int64_t)k * m.lda + x;
    if (x + 3 < nx) return load_words4(p);  // (the first product's rows start anywhere)
    return make_uint4(x < nx ? p[0] : INF, x + 1 < nx ? p[1] : INF, x + 2 < nx ? p[2] : INF, INF);
  };
  {
    const int32_t ns = min(m.K, 16);
    for (int i = kg; i < 16; i += G) {
      uint4 v = make_uint4(INF, INF, INF, INF);
      if (i < ns) v = load((int32_t)((int64_t)i * m.K / ns));
      *reinterpret_cast<uint4*>(&smin[i][x]) = v;
    }
  }
  __syncthreads();
  u32 r[4] = {INF, INF, INF, INF};
#pragma unroll
  for (int i = 0; i < 16; i++) {
    const uint4 v = *reinterpret_cast<const uint4*>(&smin[i][x]);
    r[0] = min(r[0], v.x);
    r[1] = min(r[1], v.y);
    r[2] = min(r[2], v.z);
    r[3] = min(r[3], v.w);
  }
  bool bad = false;
  if (r[0] < INF || r[1] < INF || r[2] < INF || r[3] < INF) live = 1;
  constexpr int KQ = 4;  // k per lane and step
  for (int32_t k0 = 0; k0 < m.K; k0 += G * KQ) {
    uint4 v4[KQ];
#pragma unroll
    for (int q = 0; q < KQ; q++) v4[q] = load(min(k0 + q * G + kg, m.K - 1));
#pragma unroll
    for (int q = 0; q < KQ; q++) {
      const int32_t k = k0 + q * G + kg;
      int32_t mn = 0x7fffffff, mx = -0x7fffffff;
      const u32 v[4] = {v4[q].x, v4[q].y, v4[q].z, v4[q].w};
#pragma unroll
      for (int j = 0; j < 4; j++) {
        if (r[j] < INF) {
          const int32_t d = (int32_t)(v[j] - r[j]);  // both in [0, INF]: no overflow
          mn = min(mn, d);
          mx = max(mx, d);
        } else {
          bad |= v[j] < INF;
        }
      }
      // over the 16 (or 32) lanes of the k
#define DPP_STEP(c)                                                        \
  mn = min(mn, __builtin_amdgcn_update_dpp(mn, mn, c, 0xf, 0xf, false));   \
  mx = max(mx, __builtin_amdgcn_update_dpp(mx, mx, c, 0xf, 0xf, false));
      DPP_STEP(0xb1) DPP_STEP(0x4e) DPP_STEP(0x141) DPP_STEP(0x140)
#undef DPP_STEP
      if (L == 32) {
        mn = min(mn, __shfl_xor(mn, 16));
        mx = max(mx, __shfl_xor(mx, 16));
      }
      if (l == 0 && k < m.K)
        put(k, max(min(mn, MP_BIG - MP_SHIFT) + MP_SHIFT, -MP_BIG - 1),
            max(min(mx, MP_BIG - MP_SHIFT) + MP_SHIFT, 0));
    }
  }
  if (bad) odd = 1;
  __syncthreads();
  if (odd || !live)
    for (int32_t k = threadIdx.x; k < m.K; k += 256)
      put(k, odd ? -MP_BIG - 1 : MP_BIG, odd ? MP_BIG : 0);
}

// The bit masks of the k to keep: mask[((slot * NT + row tile) * NC + column
// tile) * NW + k / 64].  A wave takes 64 columns (one per lane) and MP_RG row
// tiles, whose statistics are scalar loads; B is read twice, from L2.  exec
// counts the relaxations of the product the masks leave.
constexpr int MP_SEG = 64;  // mask words per LDS segment (4,096 k)

// OR over the wave's lanes, in every lane.
__device__ __forceinline__ u32 wave_or(u32 v) {
  int x = (int)v;
  x |= __builtin_amdgcn_update_dpp(0, x, 0xb1, 0xf, 0xf, false);   // quad_perm 1 0 3 2
  x |= __builtin_amdgcn_update_dpp(0, x, 0x4e, 0xf, 0xf, false);   // quad_perm 2 3 0 1
  x |= __builtin_amdgcn_update_dpp(0, x, 0x141, 0xf, 0xf, false);  // row_half_mirror
  x |= __builtin_amdgcn_update_dpp(0, x, 0x140, 0xf, 0xf, false);  // row_mirror: OR of the row
  return (u32)(__builtin_amdgcn_readlane(x, 0) | __builtin_amdgcn_readlane(x, 16) |
               __builtin_amdgcn_readlane(x, 32) | __builtin_amdgcn_readlane(x, 48));
}
template <int SIDE>
__global__ __launch_bounds__(256) void k_mp_keep(MpArgs a) {
  constexpr int SR = MP_SR<SIDE>, RG = MP_RG<SIDE>;
  static_assert(RG % 2 == 0, "the bounds are raised two row tiles at a time");
  __shared__ u32 seg[4][RG][MP_SEG * 2];
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int32_t slot = blockIdx.y;
  const MpSide m = mp_side(SIDE, a, slot);
  const int ncg = (a.NC + 3) / 4;
  const int32_t tj = ((int32_t)blockIdx.x % ncg) * 4 + w, t0 = ((int32_t)blockIdx.x / ncg) * RG;
  const int32_t p = tj * MP_T;
  if (p >= m.W || t0 * SR >= m.rows) return;  // (no barrier below: waves are on their own)
  const u32* B = a.R + (int64_t)m.g * a.Kp * a.Vp + min(p + lane, m.W - 1);
  const int64_t ldb = a.Vp;
  const int32_t K = m.K;
  int32_t U[RG], arg[RG];
#pragma unroll
  for (int r = 0; r < RG; r++) {
    U[r] = MP_ALL;
    arg[r] = -1;
  }
  u32 bmin = INF;
  constexpr int KU = MP_KU<SIDE>;
  const int32_t Kr = (K + KU - 1) / KU * KU;
  // a step's B entries (rows past K are there: Kp is a multiple of 128) and statistics
  // (side: 0 the lower, 1 the upper ones); the next step's are on their way while one
  // is worked on
  struct Step {
    u32 b[KU];
    int32_t m[KU * RG];
  };
  const int32_t* stats = a.stats + ((int64_t)slot * a.NT + t0) * 2 * a.Kp;
  auto fetch = [&](Step& t, int32_t k0, int side) {
    k0 = max(min(k0, Kr - KU), 0);
    const u32* bp = B + (int64_t)k0 * ldb;
    const cptr32 m = (cptr32)(stats + ((int64_t)side * a.Kp + k0) * RG);
#pragma unroll
    for (int q = 0; q < KU; q++, bp += ldb) t.b[q] = *bp;
#pragma unroll
    for (int i = 0; i < KU * RG; i++) t.m[i] = m[i];
  };
  Step cur, nxt;
  fetch(nxt, 0, 1);
#pragma unroll 1
  for (int32_t k0 = 0; k0 < K; k0 += KU) {
    cur = nxt;
    fetch(nxt, k0 + KU, 1);
#pragma unroll
    for (int q = 0; q < KU; q++) {
      bmin = min(bmin, cur.b[q]);
      const int32_t bu = (int32_t)min(cur.b[q], (u32)MP_BIG);
#pragma unroll
      for (int r = 0; r < RG; r += 2) {
        // v = mx + b;  if (v < U) arg = k;  U = min(U, v).  Two row tiles at a time, with a
        // mask each: v_cndmask may read a mask two wait states after the v_cmp that
        // wrote it, which the other tile's instructions fill.
        int32_t v0, v1;
        unsigned long long below;
        asm("v_add_u32 %4, %7, %9\n\tv_add_u32 %5, %8, %9\n\t"
            "v_cmp_lt_i32 vcc, %4, %0\n\tv_cmp_lt_i32_e64 %6, %5, %2\n\t"
            "v_min_i32 %0, %0, %4\n\tv_cndmask_b32 %1, %1, %10, vcc\n\t"
            "v_min_i32 %2, %2, %5\n\tv_cndmask_b32_e64 %3, %3, %10, %6"
            : "+&v"(U[r]), "+&v"(arg[r]), "+&v"(U[r + 1]), "+v"(arg[r + 1]), "=&v"(v0), "=&v"(v1), "=&s"(below)
            : "s"(cur.m[q * RG + r]), "s"(cur.m[q * RG + r + 1]), "v"(bu), "v"(k0 + q)
            : "vcc");
      }
    }
  }
  // a column that no k reaches, one of the K itself or past the end keeps nothing
  const bool off = bmin >= INF || p + lane >= m.W ||
                   (a.cs.rank && a.cs.rank[a.cs.g0[m.g] + p + lane] >= 0);
  int32_t nU[RG];
#pragma unroll
  for (int r = 0; r < RG; r++) {
    if (U[r] >= MP_BIG) {
      U[r] = MP_ALL;
      arg[r] = -1;
    }
    if (off) {
      U[r] = MP_NONE;
      arg[r] = -1;
    }
    nU[r] = -U[r];
  }
  const int32_t nrt = min(RG, (m.rows - t0 * SR + SR - 1) / SR);
  u32 kept[RG];
#pragma unroll
  for (int r = 0; r < RG; r++) kept[r] = 0;
  fetch(nxt, 0, 0);
  for (int32_t s0 = 0; s0 < K; s0 += MP_SEG * 64) {
    const int32_t s1 = min(K, s0 + MP_SEG * 64);
    for (int32_t k0 = s0; k0 < s1; k0 += 32) {
      // bit 31 - q of a lane's word: its column needs k0 + q (the sign of
      // mn + b - U)
      u32 word[RG];
#pragma unroll
      for (int r = 0; r < RG; r++) word[r] = 0;
#pragma unroll 1
      for (int q0 = 0; q0 < 32; q0 += KU) {
        cur = nxt;
        fetch(nxt, k0 + q0 + KU, 0);
#pragma unroll
        for (int q = 0; q < KU; q++) {
          const int32_t b = (int32_t)min(cur.b[q], (u32)MP_BIG);
          int32_t t;
#pragma unroll
          for (int r = 0; r < RG; r++)
            asm("v_add3_u32 %1, %2, %3, %4\n\tv_alignbit_b32 %0, %0, %1, 31"
                : "+v"(word[r]), "=&v"(t)
                : "s"(cur.m[q * RG + r]), "v"(b), "v"(nU[r]));
        }
      }
      const u32 valid = K - k0 >= 32 ? 0xffffffffu : (1u << (K - k0)) - 1;
#pragma unroll
      for (int r = 0; r < RG; r++) {
        const u32 x = __builtin_bitreverse32(wave_or(word[r])) & valid;
        if (lane == 0) seg[w][r][(k0 - s0) >> 5] = x;
      }
    }
    const int32_t nh = (s1 - s0 + 31) >> 5;  // 32-bit words
    if ((nh & 1) && lane < RG) seg[w][lane][nh] = 0;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < RG; r++)
      if (arg[r] >= s0 && arg[r] < s1) atomicOr(&seg[w][r][(arg[r] - s0) >> 5], 1u << (arg[r] & 31));
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < RG; r++) {
      if (r >= nrt) break;
      u32* out = reinterpret_cast<u32*>(
          a.mask + (((int64_t)slot * a.NT + t0 + r) * a.NC + tj) * a.NW + (s0 >> 6));
      for (int32_t i = lane; i < nh + (nh & 1); i += 64) {
        const u32 x = seg[w][r][i];
        out[i] = x;
        kept[r] += __popc(x);
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
  // relaxations: pairs of k on whole tiles
  unsigned long long n = 0;
#pragma unroll
  for (int r = 0; r < RG; r++) {
    if (r >= nrt) break;
    u32 x = kept[r];
    for (int o = 32; o > 0; o >>= 1) x += (u32)__shfl_xor((int)x, o);
    const u32 tiles = (u32)(min(m.rows - (t0 + r) * SR, SR) + MP_T - 1) / MP_T;
    n += (unsigned long long)((x + 1) & ~1u) * (MP_T * MP_T) * tiles;
  }
  if (lane == 0 && n) atomicAdd(a.exec + ((blockIdx.x + blockIdx.y) & 15), n);
}

// The relaxations of one LDS step, its first n k (even): MP_KC rows of A's 64
// rows, then as many of B's 64 columns.  Lane (ly, lx) = (lane / 8, lane % 8)
// holds rows h*32 + ly*4 + a and columns h*32 + lx*4 + a of the tile, h < 2, a < 4.
__device__ __forceinline__ void mp_wave_step(u32 (&c)[8][8], const u32* s, int n, int ly, int lx) {
  const u32* ap = s + ly * 4;
  const u32* bp = s + MP_KC * MP_T + lx * 4;
#pragma unroll 1
  for (int k = 0; k < n; k += 2) {
    u32 a0[8], a1[8], b0[8], b1[8];
#pragma unroll
    for (int h = 0; h < 2; h++) {
      const uint4 x0 = *reinterpret_cast<const uint4*>(ap + h * 32);
      const uint4 x1 = *reinterpret_cast<const uint4*>(ap + MP_T + h * 32);
      const uint4 y0 = *reinterpret_cast<const uint4*>(bp + h * 32);
      const uint4 y1 = *reinterpret_cast<const uint4*>(bp + MP_T + h * 32);
      a0[h * 4 + 0] = x0.x; a0[h * 4 + 1] = x0.y; a0[h * 4 + 2] = x0.z; a0[h * 4 + 3] = x0.w;
      a1[h * 4 + 0] = x1.x; a1[h * 4 + 1] = x1.y; a1[h * 4 + 2] = x1.z; a1[h * 4 + 3] = x1.w;
      b0[h * 4 + 0] = y0.x; b0[h * 4 + 1] = y0.y; b0[h * 4 + 2] = y0.z; b0[h * 4 + 3] = y0.w;
      b1[h * 4 + 0] = y1.x; b1[h * 4 + 1] = y1.y; b1[h * 4 + 2] = y1.z; b1[h * 4 + 3] = y1.w;
    }
    ap += 2 * MP_T;
    bp += 2 * MP_T;
#pragma unroll
    for (int i = 0; i < 8; i++)
#pragma unroll
      for (int j = 0; j < 8; j++) relax2(c[i][j], a0[i], b0[j], a1[i], b1[j]);
  }
}

// Half h of a wave's tile through LDS, so that a wave stores 64 consecutive
// columns (BYROW: rows h*32 .., lane = column) or rows (columns h*32 ..,
// lane = row) at a time.
constexpr int MP_ST = 68;  // row length of the staged half: 16-byte aligned, banks spread
template <bool BYROW>
__device__ __forceinline__ void mp_stage(const u32 (&c)[8][8], u32* s, int h, int ly, int lx) {
#pragma unroll
  for (int q = 0; q < 4; q++)
#pragma unroll
    for (int g = 0; g < 2; g++) {
      uint4 v;
      if (BYROW)
        v = h ? make_uint4(c[4 + q][g * 4], c[4 + q][g * 4 + 1], c[4 + q][g * 4 + 2], c[4 + q][g * 4 + 3])
              : make_uint4(c[q][g * 4], c[q][g * 4 + 1], c[q][g * 4 + 2], c[q][g * 4 + 3]);
      else
        v = h ? make_uint4(c[g * 4][4 + q], c[g * 4 + 1][4 + q], c[g * 4 + 2][4 + q], c[g * 4 + 3][4 + q])
              : make_uint4(c[g * 4][q], c[g * 4 + 1][q], c[g * 4 + 2][q], c[g * 4 + 3][q]);
      const int row = (BYROW ? ly : lx) * 4 + q, col = g * 32 + (BYROW ? lx : ly) * 4;
      *reinterpret_cast<uint4*>(s + row * MP_ST + col) = v;
    }
}

// What a lane holds of the query layout for the store of a tile: the terms of
// its column (byte offsets) and of the row of the same number.
struct MpTerms {
  u32 lo, ln, ll;  // column (block's y): rowoff, |B|, local index, times 4
  u32 uo, un, ul;  // row (block's x): rowoff, |B|, local index
};

// (Eight rows are read from LDS before the first is stored: one at a time each store
// waited for its read: a 30,700-row share's build 53.0 -> 52.5 ms.)
// Stores the staged half: staged row q (of n) is the block's row u0 + q, the
// lane's column its column l (-1: none), so the 64 stores are consecutive inside
// a component's run.  Query layout: element (x, y) at rowoff(x) |Y| + nb(x)
// rowoff(y) + loc(x) nb(y) + loc(y) (bytes below 2^32): the rows of one
// component follow each other nb(y) apart.  h: which half, row q's terms in
// lane h*32 + q.  Mg (not null: S1 = S2): the group's closure is folded in.
// CERT: worst gets the largest value.
template <bool CERT>
__device__ __forceinline__ void mp_store_half(const u32* s, const MpTerms& t, u32* base, int h, int32_t n,
                                              int32_t l, u32 nY, const u32* Mg, int32_t Vp, u32& worst) {
  const int lane = threadIdx.x;
  if (l < 0) return;
  char* row = nullptr;
  u32 off = 0;
  int e = 0;  // where the component's rows end
  for (int q0 = 0; q0 < n; q0 += 8) {
    u32 v[8];
#pragma unroll
    for (int i = 0; i < 8; i++) v[i] = s[(q0 + i) * MP_ST + lane];
    if (Mg) {
#pragma unroll
      for (int i = 0; i < 8; i++) v[i] = min(v[i], Mg[(int64_t)min(q0 + i, n - 1) * Vp + l]);
    }
#pragma unroll
    for (int i = 0; i < 8; i++) {
      const int q = q0 + i;
      if (q >= n) break;
      if (q == e) {
        const int r = h * 32 + q;
        const u32 uo = (u32)__builtin_amdgcn_readlane((int)t.uo, r), un = (u32)__builtin_amdgcn_readlane((int)t.un, r),
                  ul = (u32)__builtin_amdgcn_readlane((int)t.ul, r);
        row = reinterpret_cast<char*>(base) + (uint64_t)uo * nY * 4;
        off = __umul24(un, t.lo) + (__umul24(ul, t.ln) + t.ll);
        e = q + (int)(un - ul);
      }
      *reinterpret_cast<u32*>(row + off) = v[i];
      off += t.ln;
      if (CERT) worst = max(worst, v[i]);
    }
  }
}

// The same into the dense matrix of level 3, from its row `out`.
__device__ __forceinline__ void mp_store_half_dense(const u32* s, u32* out, int64_t ldo, int32_t n,
                                                    int32_t l, const u32* Mg, int32_t Vp) {
  const int lane = threadIdx.x;
  if (l < 0) return;
  for (int q0 = 0; q0 < n; q0 += 8) {
    u32 v[8];
#pragma unroll
    for (int i = 0; i < 8; i++) v[i] = s[(q0 + i) * MP_ST + lane];
    if (Mg) {
#pragma unroll
      for (int i = 0; i < 8; i++) v[i] = min(v[i], Mg[(int64_t)min(q0 + i, n - 1) * Vp + l]);
    }
#pragma unroll
    for (int i = 0; i < 8; i++)
      if (q0 + i < n) out[(q0 + i) * ldo + l] = v[i];
  }
}

// Pair slot and tile of a workgroup.  Workgroups go round-robin to the eight
// XCDs (an L2 each) in order of their linear id: pairs c, c + 8, ... all stay on
// XCD c, so its L2 serves the reuse of a pair's operands.  With few pairs that
// would leave XCDs idle at the end (level 3, 36 pairs: 3.0 against 2.1 ms), so
// there a pair's tiles spread over all of them, rotated by the pair (the tiles
// past a group's last vertex would otherwise all fall to the same XCDs).
constexpr int MP_XCD_PAIRS = 128;
__device__ __forceinline__ void mp_place(const MpArgs& a, int32_t& slot, int32_t& tile) {
  if (a.np >= MP_XCD_PAIRS) {
    const u32 id = blockIdx.y * gridDim.x + blockIdx.x, q = id >> 3;
    slot = (int32_t)(q / gridDim.x * 8 + (id & 7));
    tile = (int32_t)(q % gridDim.x);
  } else {
    slot = blockIdx.y;
    tile = (int32_t)((blockIdx.x + blockIdx.y) % gridDim.x);
  }
}

// One wave per 64 x 64 tile of a product, over the kept k.  The two 256-byte
// operand rows of a kept k go straight to LDS, into a ring of MP_RING steps of
// MP_KC k; waves share nothing, so no barrier holds one up.  8 x 8
// entries per lane: 128 VGPRs, 9.2 KB of LDS, four waves per SIMD.
//
// SIDE 0, the first product: rows b in B2(S2), columns x of S1, stored as XT.
// SIDE 1: rows x of S1, columns y of S2, stored as the block D(S1, S2) (D(S2,
// S1) for a swapped pair).  CERT: with the certificate.
// SIDE 2: rows: share sources, columns: rows of DT, lowered in place.
template <int SIDE, bool CERT>
__global__ __launch_bounds__(64) SPQ_MP_ATTR void k_mp_prod(MpArgs a) {
  __shared__ __attribute__((aligned(16))) u32 s[32 * MP_ST];
  __shared__ uint16_t kl[256 + MP_KC];
  static_assert(MP_RING * MP_KC * 2 * MP_T <= 32 * MP_ST, "the ring fits in the staging buffer");
  static_assert(MP_KC == 4 && MP_RING == 4, "the waits below");
  int32_t slot, tile;
  mp_place(a, slot, tile);
  if (slot >= a.np) return;
  const MpSide m = mp_side(SIDE, a, slot);
  const int32_t ti = tile / a.NC, tj = tile % a.NC;
  const int32_t x0 = ti * MP_T, p0 = tj * MP_T;
  if (x0 >= m.rows || p0 >= m.W) return;
  const CompStore& cs = a.cs;
  const int lane = threadIdx.x, ly = lane >> 3, lx = lane & 7;
  const int2 pr = SIDE == 2 ? make_int2(slot, slot) : a.plist[a.pbase + slot];
  const bool sw = (pr.y & PAIR_SWAP) != 0;
  const int32_t s1 = pr.x, s2 = pr.y & ~PAIR_SWAP;
  // the block's rows (of a swapped pair the tile's columns) and columns
  const int32_t u0 = sw ? p0 : x0, ulim = sw ? m.W : m.rows;
  const int32_t l0 = sw ? x0 : p0, llim = sw ? m.rows : m.W;
  const int32_t gu = SIDE == 1 ? cs.g0[sw ? s2 : s1] : 0, gl = SIDE == 1 ? cs.g0[sw ? s1 : s2] : 0;
  u32* base = nullptr;
  MpTerms t{};
  u32 c[8][8];
  fill_inf(c);
  {
    const u32* A = m.A + x0;
    const u32* B = a.R + (int64_t)m.g * a.Kp * a.Vp + p0;
    const auto mk = (const __attribute__((address_space(4))) unsigned long long*)(
        a.mask + (((int64_t)slot * a.NT + x0 / MP_SR<SIDE>) * a.NC + tj) * a.NW);
    const int32_t nw = (m.K + 63) >> 6;
    // the kept k of up to four mask words, padded by repeating the last to a whole
    // chunk (harmless in a minimum); returns their number
    auto list_window = [&](int32_t w0) -> int32_t {
      int32_t n = 0, last = 0;
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const unsigned long long word = w0 + i < nw ? mk[w0 + i] : 0ull;
        if (word >> lane & 1)
          kl[n + __builtin_amdgcn_mbcnt_hi((u32)(word >> 32), __builtin_amdgcn_mbcnt_lo((u32)word, 0))] =
              (uint16_t)(i * 64 + lane);
        if (word) last = i * 64 + 63 - __builtin_clzll(word);
        n += __popcll(word);
      }
      if (lane < MP_KC) kl[n + lane] = (uint16_t)last;
      return n;
    };
    // sixteen lanes fetch a row of 64 words (B, and A in the second product,
    // whose rows are 16-byte aligned; A's in the first start anywhere: one
    // word per lane)
    const u32 acol = min((u32)lane, (u32)(m.rows - x0 - 1)) & 63u;
    constexpr int LOADS = SIDE ? 2 : 1 + MP_KC;  // per step
    auto load_step = [&](int32_t kw, int32_t st) {
      u32* d = s + (st % MP_RING) * MP_KC * 2 * MP_T;
      const u32 k = (u32)kw + kl[st * MP_KC + (lane >> 4)];
      const u32* bp = B + (uint64_t)k * (u32)a.Vp + (lane & 15) * 4;
      lds_load16(bp, d + MP_KC * MP_T);
      if (SIDE) {
        const u32* ap = A + (uint64_t)k * (u32)m.lda + (lane & 15) * 4;
        lds_load16(ap, d);
      } else {
#pragma unroll
        for (int i = 0; i < MP_KC; i++) {
          const int32_t ki = __builtin_amdgcn_readlane((int)k, i * 16);
          lds_load4(A + (int64_t)ki * m.lda + acol, d + i * MP_T);
        }
      }
    };
    int32_t n = list_window(0);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < MP_RING; i++)
      if (i * MP_KC < n) load_step(0, i);
    if (SIDE == 1 && !cs.dense) {  // the store's terms, before they are needed
      base = cs.H + (sw ? cs.pairbase[(int64_t)s2 * cs.ngroups + s1]
                        : cs.pairbase[(int64_t)s1 * cs.ngroups + s2]);
      const int32_t ug = gu + min(u0 + lane, ulim - 1), lg = gl + min(l0 + lane, llim - 1);
      const int4 um = cs.meta[ug], lm = cs.meta[lg];
      t.lo = (u32)lm.x * 4;
      t.ln = (u32)lm.y * 4;
      t.ll = (u32)lm.z * 4;
      t.uo = (u32)um.x;
      t.un = (u32)um.y;
      t.ul = (u32)um.z;
    }
    if (cs.rank) {  // the columns that are boundary vertices themselves
      const int32_t rk = p0 + lane < m.W ? cs.rank[cs.g0[m.g] + p0 + lane] : -1;
      if (__ballot(rk >= 0)) {
#pragma unroll
        for (int j = 0; j < 8; j++) {
          const int32_t r = __shfl(rk, (j >> 2) * 32 + lx * 4 + (j & 3));
          if (r < 0) continue;
#pragma unroll
          for (int h = 0; h < 2; h++) {
            const int32_t x = h * 32 + ly * 4, nx = m.rows - x0 - x;
            const u32* ap = A + (int64_t)r * m.lda + x;
            if (nx >= 4) {
              const uint4 v = load_words4(ap);
              c[h * 4][j] = v.x;
              c[h * 4 + 1][j] = v.y;
              c[h * 4 + 2][j] = v.z;
              c[h * 4 + 3][j] = v.w;
            } else {
              if (nx > 0) c[h * 4][j] = ap[0];
              if (nx > 1) c[h * 4 + 1][j] = ap[1];
              if (nx > 2) c[h * 4 + 2][j] = ap[2];
            }
          }
        }
        wait_loads();  // else the compiler waits for them in every step of the loop below
      }
    }
    for (int32_t w0 = 0;;) {
      const int32_t ns = (n + MP_KC - 1) / MP_KC;
#pragma unroll 1
      for (int32_t st = 0; st < ns; st++) {
        // step st has arrived (the loads behind it may still be in flight), and
        // every LDS read of the step before it is over
        const int32_t behind = ns - 1 - st;
        if (behind >= 3)
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(3 * LOADS) : "memory");
        else if (behind == 2)
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(2 * LOADS) : "memory");
        else if (behind == 1)
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(LOADS) : "memory");
        else
          asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        mp_wave_step(c, s + (st % MP_RING) * MP_KC * 2 * MP_T, min(MP_KC, (n - st * MP_KC + 1) & ~1), ly, lx);
        // its slot is free once its LDS reads are over (their values are used above)
        if (st + MP_RING < ns) {
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          load_step(w0 * 64, st + MP_RING);
        }
      }
      w0 += 4;
      if (w0 >= nw) break;
      n = list_window(w0);
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int i = 0; i < MP_RING; i++)
        if (i * MP_KC < n) load_step(w0 * 64, i);
    }
  }
  __builtin_amdgcn_wave_barrier();
  if (SIDE == 0) {
    // XT rows b: 64 consecutive x per store (those past the group, and rows past
    // its boundary, are unused)
    u32* xt = a.XT + ((int64_t)slot * a.Kp + x0) * a.Vp + p0;
#pragma unroll
    for (int h = 0; h < 2; h++) {
      mp_stage<true>(c, s, h, ly, lx);
      __builtin_amdgcn_wave_barrier();
#pragma unroll 8
      for (int q = 0; q < 32; q++) xt[(int64_t)(h * 32 + q) * a.Vp + lane] = s[q * MP_ST + lane];
      __builtin_amdgcn_wave_barrier();
    }
    return;
  }
  if (SIDE == 2) {
    // DT's rows of the tile's columns, 64 consecutive sources per store
    const int32_t* nl = a.nlist + (int64_t)slot * a.nstride + p0;
    u32* D = a.DT + (int64_t)a.boff[slot] * a.ldd + x0 + lane;
#pragma unroll
    for (int h = 0; h < 2; h++) {
      mp_stage<false>(c, s, h, ly, lx);
      __builtin_amdgcn_wave_barrier();
      const int32_t n = min(m.W - p0 - h * 32, 32);
      for (int q0 = 0; q0 < n; q0 += 8) {
        u32 v[8], old[8];
        int32_t row[8];
#pragma unroll
        for (int i = 0; i < 8; i++) row[i] = nl[h * 32 + min(q0 + i, n - 1)];
#pragma unroll
        for (int i = 0; i < 8; i++) {
          v[i] = s[(q0 + i) * MP_ST + lane];
          old[i] = D[row[i] * a.ldd];
        }
#pragma unroll
        for (int i = 0; i < 8; i++)
          if (q0 + i < n) D[row[i] * a.ldd] = min(v[i], old[i]);
      }
      __builtin_amdgcn_wave_barrier();
    }
    return;
  }
  const u32* Mg = s1 == s2 ? cs.Mg + ((int64_t)s1 * a.Vp + u0) * a.Vp : nullptr;
  const int32_t l = l0 + lane < llim ? l0 + lane : -1;
  u32 worst = 0, seen = 0;
  if (CERT) seen = __hip_atomic_load(cs.cert_mbg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
  for (int h = 0; h < 2; h++) {
    const int32_t n = min(ulim - u0 - h * 32, 32);
    if (n <= 0) break;
    if (sw)
      mp_stage<false>(c, s, h, ly, lx);
    else
      mp_stage<true>(c, s, h, ly, lx);
    __builtin_amdgcn_wave_barrier();
    const u32* Mh = Mg ? Mg + (int64_t)h * 32 * a.Vp : nullptr;
    if (cs.dense)
      mp_store_half_dense(s, cs.dense + (int64_t)(gu + u0 + h * 32) * cs.ldo + gl, cs.ldo, n, l, Mh, a.Vp);
    else
      mp_store_half<CERT>(s, t, base, h, n, l, (u32)llim, Mh, a.Vp, worst);
    __builtin_amdgcn_wave_barrier();
  }
  if (CERT) {
    // an INF somewhere (rare): the largest finite value, and whether an INF joins
    // vertices connected in G, from the stored entries (this lane wrote them)
    u32 wrong = 0, best = worst;
    if (worst >= INF) {
      best = 0;
      const int32_t lab = cs.bglabel[gl + l];
      for (int32_t x = u0; x < min(ulim, u0 + MP_T); x++) {
        const int4 um = cs.meta[gu + x];
        const u32 off = __umul24((u32)um.y, t.lo) + (__umul24((u32)um.z, t.ln) + t.ll);
        const u32 v = *reinterpret_cast<const u32*>(reinterpret_cast<const char*>(base) +
                                                    (uint64_t)(u32)um.x * (u32)llim * 4 + off);
        if (v < INF)
          best = max(best, v);
        else
          wrong |= (u32)(cs.bglabel[gu + x] == lab);
      }
    }
    cert_reduce(best, wrong, seen, cs.cert_bad, cs.cert_mbg);
  }
}

// ------------------------------------------------------------- level 3
// The construction once more, on BG2, when BG2 itself is too large for one
// flat Floyd-Warshall: super-groups T of consecutive groups; M3[T] = BG2
// induced on T's vertices, closed (d_T); B3(T) = vertices of T with a G edge
// to another super-group (the only BG2 edges that leave T); BG3 on the B3
// vertices, closed by flat Floyd-Warshall (= d_BG2 on B3, Lemma 1 for the
// super-group partition); then, by Lemma 3 at this level,
//   d_BG2(x,y) = min over a in B3(T1), b in B3(T2) of
//                d_T1(x,a) + d_BG3(a,b) + d_T2(b,y)   (and d_T1(x,y) if T1 = T2),
// evaluated with the same two products and written straight into the dense
// BG2 matrix for T1 <= T2: the block upper triangle the level-2 composition
// reads (rows of a group S1, columns of a group S2 >= S1).

// G edges between super-groups (both ends are level-2 vertices).  BG3 ==
// NULL: flags both ends as level-3 boundary vertices; otherwise enters the
// edge into BG3 (ids b3off[T] + rank inside T).
__global__ void k_l3_edges(int64_t m, const int32_t* __restrict__ eu, const int32_t* __restrict__ ev,
                           const int32_t* __restrict__ w, const int32_t* __restrict__ comp,
                           const int32_t* __restrict__ local, const int32_t* __restrict__ bgoff,
                           const int32_t* __restrict__ grp, int32_t gpt, const int32_t* __restrict__ b2off,
                           const int32_t* __restrict__ b2rank, uint8_t* __restrict__ flag3,
                           const int32_t* __restrict__ b3off, const int32_t* __restrict__ b3rank,
                           int64_t V3p, u32* __restrict__ BG3) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int32_t u = eu[e], v = ev[e];
    const int32_t cu = comp[u], cv = comp[v];
    if (cu == cv) continue;
    const int32_t su = grp[cu], sv = grp[cv];
    const int32_t tu = su / gpt, tv = sv / gpt;
    if (tu == tv) continue;
    const int32_t xu = b2off[su] + b2rank[bgoff[cu] + local[u]];
    const int32_t xv = b2off[sv] + b2rank[bgoff[cv] + local[v]];
    if (!BG3) {
      flag3[xu] = 1;
      flag3[xv] = 1;
      continue;
    }
    const int64_t a = b3off[tu] + b3rank[xu], b = b3off[tv] + b3rank[xv];
    atomicMin(BG3 + a * V3p + b, (u32)w[e]);
    atomicMin(BG3 + b * V3p + a, (u32)w[e]);
  }
}

// One BG row (BG id x) gathered from the two-level store, for inspection.
__global__ void k_hier_row(int32_t x, int32_t swap, int32_t V, int32_t ngroups,
                           const int32_t* __restrict__ bggrp,
                           const int32_t* __restrict__ bgrow, const int32_t* __restrict__ bgnb,
                           const int32_t* __restrict__ bglocal, const int32_t* __restrict__ gV,
                           const int64_t* __restrict__ pairbase, const u32* __restrict__ H,
                           u32* __restrict__ out) {
  const int64_t y = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (y >= V) return;
  int32_t a = x, b = (int32_t)y;
  if (swap && bggrp[a] > bggrp[b]) {
    a = (int32_t)y;
    b = x;
  }
  const int32_t sa = bggrp[a], sb = bggrp[b];
  const int64_t off = pairbase[(int64_t)sa * ngroups + sb] + (int64_t)bgrow[a] * gV[sb] +
                      (int64_t)bgnb[a] * bgrow[b] + (int64_t)bglocal[a] * bgnb[b] + bglocal[b];
  out[y] = H[off];
}


// ------------------------------------------------------------ share mode --
// Distances from the level-2 boundary vertices of the share groups (the
// first share_groups groups; their level-2 ids are 0 .. S2-1) to all level-2
// vertices, by Bellman-Ford over blocks of consecutive groups on BG2, without
// building BG2.  A block T is a run of consecutive groups (one group: the
// Bellman-Ford over groups); A_T = BG2 induced on T's level-2 vertices (d_S
// between the B2
// vertices of one group S, the G edges between groups of T), closed.  DT[b][i]
// (row b = any level-2 id, column i = share source) alternates
//   intra-block:  DT[T] = min(DT[T], A_T (x) DT[T])   (A_T closed: one product
//                 covers any walk that stays inside T)
//   cross edges:  DT[b] = min(DT[b], DT[a] + w(a,b))  for each G edge between blocks
// until nothing changes.  Every walk of BG2 is a sequence of pieces inside one
// block joined by G edges between blocks, so the fixed point is d_BG2 from
// every share source (Lemma 1 for the block partition of BG2).  Larger blocks
// mean fewer rounds (a round crosses one block) and fewer cross edges, at the
// price of larger products.

// A_T before its closure (bpmax x bpmax per block, local level-2 indices):
// d_S between the B2 vertices of one group, 0 on the diagonal, INF elsewhere
// and on the padding.  Block t holds groups [bfirst[t], bfirst[t+1]); a block
// of one group: A_T = d_S on B2(S), already closed.
__global__ void k_blk_init(int32_t Vgp, int32_t bpmax, const int32_t* __restrict__ bfirst,
                           const int32_t* __restrict__ b2off, const int32_t* __restrict__ b2list,
                           const u32* __restrict__ Mg, u32* __restrict__ A) {
  const int t = blockIdx.y;
  const int32_t p = blockIdx.x;
  const int32_t g0 = bfirst[t], g1 = bfirst[t + 1];
  const int32_t base = b2off[g0], size = b2off[g1] - base;
  u32* out = A + ((int64_t)t * bpmax + p) * bpmax;
  int32_t lo = 0, hi = 0;
  const u32* prow = nullptr;
  const int32_t* list = nullptr;
  if (p < size) {
    int32_t a = g0;  // the row's group (a block holds few groups)
    while (a + 1 < g1 && b2off[a + 1] - base <= p) a++;
    lo = b2off[a] - base;
    hi = b2off[a + 1] - base;
    list = b2list + (int64_t)a * Vgp;
    prow = Mg + ((int64_t)a * Vgp + list[p - lo]) * Vgp;
  }
  for (int32_t q = threadIdx.x; q < bpmax; q += blockDim.x)
    out[q] = (q == p) ? 0u : (q >= lo && q < hi) ? prow[list[q - lo]] : INF;
}

// G edges between groups of the same block, into A_T (both directions).
__global__ void k_blk_edges(int64_t m, const int32_t* __restrict__ eu, const int32_t* __restrict__ ev,
                            const int32_t* __restrict__ w, const int32_t* __restrict__ comp,
                            const int32_t* __restrict__ local, const int32_t* __restrict__ bgoff,
                            const int32_t* __restrict__ grp, const int32_t* __restrict__ gblk,
                            const int32_t* __restrict__ bfirst,
                            const int32_t* __restrict__ b2off, const int32_t* __restrict__ b2rank,
                            int32_t bpmax, u32* __restrict__ A) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int32_t u = eu[e], v = ev[e];
    const int32_t cu = comp[u], cv = comp[v];
    if (cu == cv) continue;
    const int32_t su = grp[cu], sv = grp[cv];
    if (su == sv || gblk[su] != gblk[sv]) continue;
    const int32_t t = gblk[su], base = b2off[bfirst[t]];
    const int64_t a = b2off[su] + b2rank[bgoff[cu] + local[u]] - base;
    const int64_t b = b2off[sv] + b2rank[bgoff[cv] + local[v]] - base;
    u32* At = A + (int64_t)t * bpmax * bpmax;
    atomicMin(At + a * bpmax + b, (u32)w[e]);
    atomicMin(At + b * bpmax + a, (u32)w[e]);
  }
}

// DT init: row b (level-2 id), column i (share source): the distance inside
// b's block when i lies in it (row b of the closed A_T), 0 for b = i, INF
// otherwise.  boff: first level-2 id of each block (nblk + 1 entries).
__global__ void k_dt_init(int32_t V2, int32_t S2, int64_t S2p, int32_t nblk,
                          const int32_t* __restrict__ boff, int32_t bpmax, const u32* __restrict__ A,
                          u32* __restrict__ DT) {
  const int64_t b = blockIdx.x;
  u32* out = DT + b * S2p;
  int64_t lo = 0, hi = 0;
  const u32* arow = nullptr;
  if (b < V2) {
    int32_t a = 0, z = nblk - 1;
    while (a < z) {
      const int32_t mid = (a + z + 1) >> 1;
      if (boff[mid] <= b) a = mid; else z = mid - 1;
    }
    lo = boff[a];
    hi = min((int64_t)boff[a + 1], (int64_t)S2);
    arow = A + ((int64_t)a * bpmax + (b - lo)) * bpmax;
  }
  for (int64_t i = threadIdx.x; i < S2p; i += blockDim.x)
    out[i] = (i == b) ? 0u : (i >= lo && i < hi) ? arow[i - lo] : INF;
}

// Dirty flags of the Bellman-Ford rounds: per block (a group or a run of
// groups), one word per column tile of 128 share sources, then one word "any
// tile" (stride ntc + 1).  Beside them, per (block, column tile), the B3 rows
// (indices in the block's b3list) that the cross edges lowered since the
// block's last intra step: a count and a list (count BF_ALL_ROWS: every row).
//
// Intra-block step, in place: the block's rows x column tile of DT = min(DT,
// A (x) DT) for the (block, tile) pairs whose values changed in the previous
// round.  One product with the closed A leaves the rows closed.  The rows were
// closed before the cross edges lowered some of them, and for an unchanged
// row k, A[x][k] + DT[k] >= DT[x] already; so only the lowered rows need to
// be the K of the product.  Tiles of one block read rows that other tiles of
// the block are lowering: every value read is the old or the new one, both
// lengths of real walks and each at most the old value, and A being closed,
// the old values already give the closed result, so the step is exact in any
// interleaving.  The rounds run this step on the B3 rows only (k_bf_intra3
// below, with A restricted to B3 x B3, which is closed as well: a shortest
// path inside the block between two B3 vertices needs no other row of DT).

// Cross edges between blocks, as directed level-2 pairs (a -> b, w), tagged
// (source block << 16) | destination block.
__global__ void k_cross_collect(int64_t m, const int32_t* __restrict__ eu, const int32_t* __restrict__ ev,
                                const int32_t* __restrict__ w, const int32_t* __restrict__ comp,
                                const int32_t* __restrict__ local, const int32_t* __restrict__ bgoff,
                                const int32_t* __restrict__ grp, const int32_t* __restrict__ gblk,
                                const int32_t* __restrict__ b2off,
                                const int32_t* __restrict__ b2rank, int32_t* __restrict__ count,
                                int4* __restrict__ xe) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int32_t u = eu[e], v = ev[e];
    const int32_t cu = comp[u], cv = comp[v];
    if (cu == cv) continue;
    const int32_t su = grp[cu], sv = grp[cv];
    const int32_t tu = gblk[su], tv = gblk[sv];  // blocks
    if (tu == tv) continue;
    const int32_t a = b2off[su] + b2rank[bgoff[cu] + local[u]];
    const int32_t b = b2off[sv] + b2rank[bgoff[cv] + local[v]];
    const int32_t slot = atomicAdd(count, 2);
    xe[slot] = make_int4(a, b, w[e], (tu << 16) | tv);
    xe[slot + 1] = make_int4(b, a, w[e], (tv << 16) | tu);
  }
}

// DT[b][i] = min(DT[b][i], DT[a][i] + w) for every directed cross edge, on
// the column tiles that are dirty for the source block (values that have not
// changed since they were last propagated need no new pass); a lowered value
// marks its (block, tile) dirty for the next round and, once per round (the
// stamp of (row, tile) holds the round that last listed it), adds its row to
// that (block, tile)'s list as its index among the block's B3 rows (b3rank;
// a cross edge ends in B3 by definition; lstride: list slots per (block,
// tile)).
__global__ void k_bf_cross(int32_t nxe, const int4* __restrict__ xe, int32_t S2, int64_t S2p, u32* DT,
                           const u32* __restrict__ dirty, u32* __restrict__ dirty_next,
                           const int32_t* __restrict__ b3rank, int32_t lstride, u32 round,
                           u32* __restrict__ stamp, int32_t* __restrict__ rcnt_next,
                           int32_t* __restrict__ rlist_next) {
  const int32_t e = blockIdx.x;
  if (e >= nxe) return;
  const int4 t = xe[e];
  const int ntc = (int)(S2p / 128);
  const u32* dsrc = dirty + (int64_t)(t.w >> 16) * (ntc + 1);
  if (!dsrc[ntc]) return;
  const int32_t sv = t.w & 0xffff;
  u32* dnext = dirty_next + (int64_t)sv * (ntc + 1);
  const u32* src = DT + (int64_t)t.x * S2p;
  u32* dst = DT + (int64_t)t.y * S2p;
  // tiles this workgroup has already listed its row for (LDS, when they fit):
  // the global stamp is then touched once per tile, not once per element
  __shared__ u32 listed[BF_LDS_TILES];
  const bool local = ntc <= BF_LDS_TILES;
  if (local) {
    for (int q = threadIdx.x; q < ntc; q += blockDim.x) listed[q] = 0u;
    __syncthreads();
  }
  // four consecutive columns per thread and step (one 16-byte load of each
  // row; rows are S2p words apart, a multiple of 128, and the four lie in
  // one column tile)
  for (int32_t i0 = 4 * (int32_t)threadIdx.x; i0 < S2; i0 += 4 * (int32_t)blockDim.x) {
    const int tile = i0 >> 7;
    if (!dsrc[tile]) continue;
    const uint4 a4 = *reinterpret_cast<const uint4*>(src + i0);
    const uint4 d4 = *reinterpret_cast<const uint4*>(dst + i0);
    const u32 av[4] = {a4.x, a4.y, a4.z, a4.w}, dv[4] = {d4.x, d4.y, d4.z, d4.w};
    bool lowered = false;
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const u32 v = min(av[q] + (u32)t.z, INF);
      if (i0 + q < S2 && v < dv[q]) {
        atomicMin(dst + i0 + q, v);
        lowered = true;
      }
    }
    if (!lowered) continue;
    dnext[tile] = 1u;
    dnext[ntc] = 1u;
    if (local && atomicExch(listed + tile, 1u) != 0u) continue;
    if (atomicExch(stamp + (int64_t)t.y * ntc + tile, round) != round) {
      const int64_t st = (int64_t)sv * ntc + tile;
      const int32_t slot = atomicAdd(rcnt_next + st, 1);
      rlist_next[st * lstride + slot] = b3rank[t.y];
    }
  }
}

// ------------------------------------------------------------- block boundary
// Only the B3 rows of a block (level-2 vertices with a G edge to another
// block) are lowered by cross edges and read by them, so the rounds keep
// just those rows settled; a path from a source to any other row v of block
// T either stays in T (DT's initial row, from the closed A_T) or enters T
// last through some b in B3(T), so once the B3 rows are exact
//   DT[v] = min(DT[v], min over b in B3(T) of A_T[v][b] + DT[b])
// gives the rest in one product per block.

// flag3[a] = 1 for every source a of a directed cross edge (both directions
// are listed, so every endpoint); the count is read on the device.
__global__ void k_b3_mark(const int32_t* __restrict__ xcount, const int4* __restrict__ xe,
                          uint8_t* __restrict__ flag3) {
  const int32_t n = *xcount;
  for (int32_t e = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x); e < n;
       e += (int32_t)(gridDim.x * blockDim.x))
    flag3[xe[e].x] = 1;
}

__global__ void k_flag_not(int32_t n, const uint8_t* __restrict__ f, uint8_t* __restrict__ g) {
  for (int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x); i < n;
       i += (int32_t)(gridDim.x * blockDim.x))
    g[i] = f[i] ? 0 : 1;
}

// Row i of block t's A3: A_T[b3[i]][b3[j]] for i, j < m3[t]; INF elsewhere.
__global__ void k_a3_gather(int32_t bpmax, int32_t b3pmax, const int32_t* __restrict__ m3,
                            const int32_t* __restrict__ b3list, const u32* __restrict__ A,
                            u32* __restrict__ A3) {
  const int t = blockIdx.y;
  const int32_t i = blockIdx.x, mt = m3[t];
  const int32_t* bl = b3list + (int64_t)t * bpmax;
  u32* out = A3 + ((int64_t)t * b3pmax + i) * b3pmax;
  const u32* arow = i < mt ? A + ((int64_t)t * bpmax + bl[i]) * bpmax : nullptr;
  for (int32_t j = threadIdx.x; j < b3pmax; j += blockDim.x) out[j] = (arow && j < mt) ? arow[bl[j]] : INF;
}

// Row k of block t's Aout: A_T[b3[k]][nb3[i]] for k < m3[t], i < n3[t]; INF
// elsewhere (A_T is symmetric: row b3[k] holds column b3[k]).
__global__ void k_aout_gather(int32_t bpmax, int32_t b3pmax, int32_t n3pmax,
                              const int32_t* __restrict__ m3, const int32_t* __restrict__ n3,
                              const int32_t* __restrict__ b3list, const int32_t* __restrict__ nb3list,
                              const u32* __restrict__ A, u32* __restrict__ Aout) {
  const int t = blockIdx.y;
  const int32_t k = blockIdx.x, nt = n3[t];
  const int32_t* bl = b3list + (int64_t)t * bpmax;
  const int32_t* nl = nb3list + (int64_t)t * bpmax;
  u32* out = Aout + ((int64_t)t * b3pmax + k) * n3pmax;
  const u32* arow = k < m3[t] ? A + ((int64_t)t * bpmax + bl[k]) * bpmax : nullptr;
  for (int32_t i = threadIdx.x; i < n3pmax; i += blockDim.x) out[i] = (arow && i < nt) ? arow[nl[i]] : INF;
}

// The B3 rows of DT, block by block: row k of block t at rows3[(t * b3pmax + k) * S2p].
__global__ void k_b3_rows(int32_t bpmax, int64_t S2p, const int32_t* __restrict__ m3,
                          const int32_t* __restrict__ b3list, const int32_t* __restrict__ boff,
                          const u32* __restrict__ DT, u32* __restrict__ rows3) {
  const int t = blockIdx.y;
  const int32_t k = blockIdx.x;
  if (k >= m3[t]) return;
  const uint4* src = reinterpret_cast<const uint4*>(DT + ((int64_t)boff[t] + b3list[(int64_t)t * bpmax + k]) * S2p);
  uint4* dst = reinterpret_cast<uint4*>(rows3 + ((int64_t)t * gridDim.x + k) * S2p);
  for (int64_t i = threadIdx.x; i < S2p / 4; i += blockDim.x) dst[i] = src[i];
}

// The 128 x 128 tile whose row r is g + rows[r] * ld, in the register layout
// of tile_load; rows r >= nvalid read as INF and are not stored.
__device__ __forceinline__ void tile_load_rows(u32 (&c)[8][8], const u32* g, int64_t ld,
                                               const int32_t* __restrict__ rows, int nvalid) {
  const int tx = tid_x(), ty = tid_y();
#pragma unroll
  for (int h = 0; h < 2; h++)
#pragma unroll
    for (int a = 0; a < 4; a++) {
      const int r = h * 64 + ty * 4 + a;
      if (r < nvalid) {
        const u32* row = g + (int64_t)rows[r] * ld + tx * 4;
#pragma unroll
        for (int h2 = 0; h2 < 2; h2++) {
          const uint4 v = *reinterpret_cast<const uint4*>(row + h2 * 64);
          u32* d = c[h * 4 + a] + h2 * 4;
          d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
        }
      } else {
#pragma unroll
        for (int j = 0; j < 8; j++) c[h * 4 + a][j] = INF;
      }
    }
}

__device__ __forceinline__ void tile_store_rows(const u32 (&c)[8][8], u32* g, int64_t ld,
                                                const int32_t* __restrict__ rows, int nvalid) {
  const int tx = tid_x(), ty = tid_y();
#pragma unroll
  for (int h = 0; h < 2; h++)
#pragma unroll
    for (int a = 0; a < 4; a++) {
      const int r = h * 64 + ty * 4 + a;
      if (r >= nvalid) continue;
      u32* row = g + (int64_t)rows[r] * ld + tx * 4;
#pragma unroll
      for (int h2 = 0; h2 < 2; h2++) {
        const u32* v = c[h * 4 + a] + h2 * 4;
        *reinterpret_cast<uint4*>(row + h2 * 64) = make_uint4(v[0], v[1], v[2], v[3]);
      }
    }
}

// The intra-block step of a round on the B3 rows only (see the Intra-block
// step above for why the listed rows suffice and why in place is exact): rows
// b3[ti*128 ..] x column tile tj of block s = min(DT, A3 (x) DT) over the
// listed B3 rows (their indices in b3list).
__global__ __launch_bounds__(256) SPQ_MP_ATTR void k_bf_intra3(int32_t bpmax, int32_t b3pmax, int64_t S2p,
                                                   const int32_t* __restrict__ m3,
                                                   const int32_t* __restrict__ boff,
                                                   const int32_t* __restrict__ b3list,
                                                   const u32* __restrict__ A3, u32* DT,
                                                   const u32* __restrict__ dirty,
                                                   const int32_t* __restrict__ rcnt,
                                                   const int32_t* __restrict__ rlist) {
  __shared__ __attribute__((aligned(16))) u32 sA[2 * 16 * 128];
  __shared__ __attribute__((aligned(16))) u32 sB[2 * 16 * 128];
  const int s = blockIdx.y;
  const int32_t ms = m3[s];
  const int ntc = (int)(S2p / 128);
  const int ti = (int)blockIdx.x / ntc, tj = (int)blockIdx.x % ntc;
  if (ti * 128 >= ms || !dirty[(int64_t)s * (ntc + 1) + tj]) return;
  const int64_t st = (int64_t)s * ntc + tj;
  const int32_t cnt = rcnt[st];
  if (cnt == 0) return;
  const int32_t* bl = b3list + (int64_t)s * bpmax;
  u32* D = DT + (int64_t)boff[s] * S2p + tj * 128;  // the block's rows, this column tile
  const int nv = min(128, ms - ti * 128);
  u32 c[8][8];
  tile_load_rows(c, D, S2p, bl + ti * 128, nv);
  const u32* At = A3 + (int64_t)s * b3pmax * b3pmax + ti * 128;  // symmetric: At[k][i] = A3[i][k]
  const bool all = cnt == BF_ALL_ROWS;
  mp_stream128_rows(c, At, b3pmax, D, S2p, all ? nullptr : rlist + st * b3pmax, all ? ms : cnt, sA, sB,
                    bl);
  tile_store_rows(c, D, S2p, bl + ti * 128, nv);
}

// The rows outside B3, once the rounds have settled: rows nb3[ti*128 ..] x
// column tile tj of block s = min(DT, Aout^T (x) DT[B3 rows]).
__global__ __launch_bounds__(256) SPQ_MP_ATTR void k_bf_final(int32_t bpmax, int32_t b3pmax, int32_t n3pmax,
                                                  int64_t S2p, const int32_t* __restrict__ m3,
                                                  const int32_t* __restrict__ n3,
                                                  const int32_t* __restrict__ boff,
                                                  const int32_t* __restrict__ b3list,
                                                  const int32_t* __restrict__ nb3list,
                                                  const u32* __restrict__ Aout, u32* DT) {
  __shared__ __attribute__((aligned(16))) u32 sA[2 * 16 * 128];
  __shared__ __attribute__((aligned(16))) u32 sB[2 * 16 * 128];
  const int s = blockIdx.y;
  const int32_t nn = n3[s], kk = m3[s];
  const int ntc = (int)(S2p / 128);
  const int ti = (int)blockIdx.x / ntc, tj = (int)blockIdx.x % ntc;
  if (ti * 128 >= nn || kk == 0) return;
  const int32_t* nl = nb3list + (int64_t)s * bpmax;
  u32* D = DT + (int64_t)boff[s] * S2p + tj * 128;
  const int nv = min(128, nn - ti * 128);
  u32 c[8][8];
  tile_load_rows(c, D, S2p, nl + ti * 128, nv);
  const u32* At = Aout + (int64_t)s * b3pmax * n3pmax + ti * 128;  // At[k][i] = A_T[b3[k]][nb3[i]]
  mp_stream128_rows(c, At, n3pmax, D, S2p, nullptr, kk, sA, sB, b3list + (int64_t)s * bpmax);
  tile_store_rows(c, D, S2p, nl + ti * 128, nv);
}

// The share's D2 in column panels: panel S (one per group, S2p x m2pmax
// elements) holds D2[i][j] = DT[b2off[S] + j][i] for the share sources i and
// the B2(S) vertices j < m2[S], INF in the columns past m2[S].  32 x 32 tiles
// through LDS; blockIdx.z = the group.
__global__ void k_panel_transpose(const u32* __restrict__ DT, int64_t S2p, int32_t m2pmax,
                                  const int32_t* __restrict__ m2, const int32_t* __restrict__ b2off,
                                  u32* __restrict__ D2) {
  __shared__ u32 t[32][33];
  const int g = blockIdx.z;
  const int32_t ms = m2[g], r0 = b2off[g];
  const int64_t i0 = (int64_t)blockIdx.x * 32;  // share sources (panel rows)
  const int32_t j0 = (int32_t)blockIdx.y * 32;  // B2(S) vertices (panel columns)
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int k = ty; k < 32; k += 8)
    if (j0 + k < ms && i0 + tx < S2p) t[k][tx] = DT[(int64_t)(r0 + j0 + k) * S2p + i0 + tx];
  __syncthreads();
  u32* panel = D2 + (int64_t)g * S2p * m2pmax;
  for (int k = ty; k < 32; k += 8)
    if (i0 + k < S2p) panel[(i0 + k) * m2pmax + j0 + tx] = j0 + tx < ms ? t[tx][k] : INF;
}

// ---------------------------------------------------------------- launch --
static inline unsigned hblocks(int64_t items) {
  int64_t b = (items + 255) / 256;
  if (b < 1) b = 1;
  if (b > 8192) b = 8192;
  return (unsigned)b;
}

hipError_t launch_hier_level1(const HierArgs& a, hipStream_t s) {
  k_hier_vmeta<<<hblocks(a.V), 256, 0, s>>>(a.V, a.bgcomp, a.bgoff, a.nb, a.grp, a.gbg0,
                                                              a.bglocal, a.bgrow, a.bgnb, a.bggrp, a.meta);
  k_grp_init<<<dim3((unsigned)a.Vgp, (unsigned)a.ngroups), 256, 0, s>>>(
      a.Vgp, a.gbg0, a.gV, a.bgcomp, a.bglocal, a.bgoff, a.nb, a.P, a.moff, a.M, a.Mg);
  if (a.m > 0)
    k_grp_edges<<<hblocks(a.m), 256, 0, s>>>(a.m, a.eu, a.ev, a.w, a.comp, a.local, a.bgoff, a.grp,
                                             a.gbg0, a.Vgp, a.Mg, a.flag2);
  const int ntg = a.Vgp / 128;
  hipError_t e = (a.side && ntg > 1)
                     ? launch_dense_fw_batch_lookahead(a.Mg, a.Vgp, 128, ntg, a.ngroups,
                                                       (int64_t)a.Vgp * a.Vgp, s, a.side, a.sync,
                                                       nullptr, a.kc, a.pivot, a.fw, FwSizes{a.gV, a.h_gV})
                     : launch_dense_fw_batch(a.Mg, a.Vgp, 128, ntg, a.ngroups, (int64_t)a.Vgp * a.Vgp,
                                             s, nullptr, a.kc, a.pivot, a.fw, FwSizes{a.gV, a.h_gV});
  if (e != hipSuccess) return e;
  k_b2_scan<<<(unsigned)a.ngroups, 256, 0, s>>>(a.gbg0, a.gV, a.flag2, a.Vgp, a.b2list, a.b2rank, a.m2);
  return hipGetLastError();
}

// R_S of every group.
static void launch_r(const HierArgs& a, hipStream_t s) {
  k_r_gather<<<dim3((unsigned)a.m2pmax, (unsigned)a.ngroups), 256, 0, s>>>(a.Vgp, a.m2pmax, a.m2, a.b2list,
                                                                            a.Mg, a.R);
}

hipError_t launch_hier_level2_prep(const HierArgs& a, bool bg2, hipStream_t s) {
  launch_r(a, s);
  if (bg2 && a.V2p > 0) {
    k_bg2_init<<<(unsigned)a.V2p, 256, 0, s>>>(a.V2, a.V2p, a.ngroups, a.b2off, a.b2list, a.Vgp, a.Mg,
                                               nullptr, nullptr, a.BG2);
    if (a.m > 0)
      k_bg2_edges<<<hblocks(a.m), 256, 0, s>>>(a.m, a.eu, a.ev, a.w, a.comp, a.local, a.bgoff, a.grp,
                                               a.b2off, a.b2rank, a.V2p, 0, nullptr, a.BG2);
  }
  return hipGetLastError();
}

hipError_t launch_hier_level2_close(const HierArgs& a, hipStream_t s) {
  if (a.V2p <= 0) return hipSuccess;
  const int nt = (int)(a.V2p / 128);
  if (a.side && nt > 1)
    return launch_dense_fw_lookahead(a.BG2, a.V2p, 128, nt, s, a.side, a.sync, nullptr, a.kc, a.pivot,
                                     nullptr, a.fw);
  return launch_dense_fw(a.BG2, a.V2p, 128, nt, s, nullptr, a.kc, a.pivot, a.fw);
}

// Buffers and launch shapes of the composition's kernels (Kp: rows per slot,
// Vp: row length; side 0 the first product's row tiles, 1 the second's).
template <int SIDE>
static int mp_row_tiles(int32_t rows) {
  constexpr int step = MP_SR<SIDE> * MP_RG<SIDE>;
  return (rows + step - 1) / step * MP_RG<SIDE>;
}
static int64_t mp_max_tiles(int32_t Kp, int32_t Vp) { return max(mp_row_tiles<0>(Kp), mp_row_tiles<1>(Vp)); }

int64_t mp_stats_words(int32_t Kp, int32_t Vp) { return Kp * mp_max_tiles(Kp, Vp) * 2; }
int64_t mp_mask_words(int32_t Kp, int32_t Vp) {
  return mp_max_tiles(Kp, Vp) * (Vp / MP_T) * (Kp / 64);
}

template <int SIDE>
static void mp_product(MpArgs a, bool cert, const MpWork& w, hipEvent_t* evt, hipStream_t s) {
  const int32_t rows = SIDE == 2 ? (int32_t)a.ldd : SIDE ? a.Vp : a.Kp;
  a.NT = mp_row_tiles<SIDE>(rows);
  a.exec = w.exec + (SIDE == 1 && !a.cs.dense ? 16 : 0);
  const unsigned np = (unsigned)a.np;
  k_mp_stats<SIDE><<<dim3((unsigned)a.NT, np), 256, 0, s>>>(a);
  k_mp_keep<SIDE><<<dim3((unsigned)((a.NC + 3) / 4 * (a.NT / MP_RG<SIDE>)), np), 256, 0, s>>>(a);
  if (evt) (void)hipEventRecord(evt[0], s);
  const dim3 g((unsigned)(rows / MP_T * a.NC), (np + 7) / 8 * 8);
  if (SIDE == 1 && cert)
    k_mp_prod<SIDE, SIDE == 1><<<g, 64, 0, s>>>(a);
  else
    k_mp_prod<SIDE, false><<<g, 64, 0, s>>>(a);
  if (evt) (void)hipEventRecord(evt[1], s);
}

// The two products of one chunk; evt (optional): two events around the second.
static void mp_chunk_products(const MpArgs& a, bool first, bool cert, const MpWork& w, hipEvent_t* evt,
                              hipStream_t s) {
  if (first) mp_product<0>(a, cert, w, nullptr, s);
  mp_product<1>(a, cert, w, evt, s);
}

// Composition over the pair list a.plist (a.npairs pairs), a.chunk pairs per
// launch of each product.  evt (optional) gets a pair of events around every
// second product.  The share's BG2 rows come from its Bellman-Ford (DT^T).
static hipError_t compose_level2(const HierArgs& a, const int32_t* bglabel, u32* cert_bad,
                                 u32* cert_mbg, hipStream_t s) {
  MpArgs m{};
  m.plist = a.plist;
  m.Vp = a.Vgp;
  m.Kp = a.m2pmax;
  m.NC = m.Vp / MP_T;
  m.NW = m.Kp / 64;
  m.m2 = a.m2; m.gV = a.gV; m.b2off = a.b2off;
  m.D2 = a.BG2; m.ldd = a.d2pstride ? a.d2ld : a.V2p; m.pstride = a.d2pstride;
  m.D2t = a.D2t; m.ldt = a.d2tld;
  m.R = a.R; m.XT = a.XT; m.stats = a.work.stats; m.mask = a.work.mask;
  m.cs = CompStore{a.gbg0, a.b2rank, a.meta, a.Mg, a.ngroups, a.pairbase, a.H, bglabel,
                   cert_bad, cert_mbg, nullptr, 0};
  for (int32_t p0 = 0, c = 0; p0 < a.npairs; p0 += a.chunk, c++) {
    m.pbase = p0;
    m.np = min(a.chunk, a.npairs - p0);
    mp_chunk_products(m, a.V2p > 0, bglabel != nullptr, a.work, a.evt ? a.evt + 2 * c : nullptr, s);
  }
  return hipGetLastError();
}

hipError_t launch_counts(unsigned long long* exec, unsigned long long* out, hipStream_t s) {
  k_counts<<<1, 64, 0, s>>>(exec, out);
  return hipGetLastError();
}

hipError_t launch_hier_level2_compose(const HierArgs& a, hipStream_t s) {
  return compose_level2(a, a.bglabel, a.cert_bad, a.cert_mbg, s);
}

hipError_t launch_flat_store(int32_t V, int64_t Vp, const u32* BG, const int32_t* bgcomp,
                             const int32_t* bgoff, const int32_t* nb, const int32_t* grp,
                             const int32_t* gbg0, int32_t* bgrow, int32_t* bgnb, int32_t* bggrp,
                             const int32_t* bglocal, u32* H, unsigned long long* exec,
                             unsigned long long* counted, hipStream_t s) {
  if (V <= 0) return launch_counts(exec, counted, s);
  k_hier_vmeta<<<hblocks(V), 256, 0, s>>>(V, bgcomp, bgoff, nb, grp, gbg0, bglocal, bgrow, bgnb, bggrp,
                                          nullptr);
  k_flat_store<<<(unsigned)V, 256, 0, s>>>(V, Vp, BG, bgrow, bgnb, bglocal, H, exec, counted);
  return hipGetLastError();
}

hipError_t launch_level3_a(const L3Args& a, hipStream_t s) {
  k_bg2_init<<<dim3((unsigned)a.V3gp, (unsigned)a.nT), 256, 0, s>>>(
      0, a.V3gp, a.ngroups, a.b2off, a.b2list, a.Vgp, a.Mg, a.tbase, a.tsize, a.M3);
  if (a.m > 0)
    k_bg2_edges<<<hblocks(a.m), 256, 0, s>>>(a.m, a.eu, a.ev, a.w, a.comp, a.local, a.bgoff, a.grp, a.b2off,
                                             a.b2rank, a.V3gp, a.gpt, a.tbase, a.M3);
  const int ntt = a.V3gp / 128;
  hipError_t e = (a.side && ntt > 1)
                     ? launch_dense_fw_batch_lookahead(a.M3, a.V3gp, 128, ntt, a.nT,
                                                       (int64_t)a.V3gp * a.V3gp, s, a.side, a.sync,
                                                       nullptr, a.kc, a.pivot, a.fw, FwSizes{a.tsize, a.h_tsize})
                     : launch_dense_fw_batch(a.M3, a.V3gp, 128, ntt, a.nT, (int64_t)a.V3gp * a.V3gp,
                                             s, nullptr, a.kc, a.pivot, a.fw, FwSizes{a.tsize, a.h_tsize});
  if (e != hipSuccess) return e;
  if (a.m > 0)
    k_l3_edges<<<hblocks(a.m), 256, 0, s>>>(a.m, a.eu, a.ev, a.w, a.comp, a.local, a.bgoff, a.grp,
                                            a.gpt, a.b2off, a.b2rank, a.flag3, nullptr, nullptr, 0,
                                            nullptr);
  k_b2_scan<<<(unsigned)a.nT, 256, 0, s>>>(a.tbase, a.tsize, a.flag3, a.V3gp, a.b3list, a.b3rank, a.m3);
  return hipGetLastError();
}

hipError_t launch_level3_b(const L3Args& a, hipStream_t s) {
  k_r_gather<<<dim3((unsigned)a.m3pmax, (unsigned)a.nT), 256, 0, s>>>(a.V3gp, a.m3pmax, a.m3,
                                                                         a.b3list, a.M3, a.R3);
  if (a.V3p > 0) {
    k_bg2_init<<<(unsigned)a.V3p, 256, 0, s>>>(a.V3, a.V3p, a.nT, a.b3off, a.b3list, a.V3gp, a.M3,
                                               nullptr, nullptr, a.BG3);
    if (a.m > 0)
      k_l3_edges<<<hblocks(a.m), 256, 0, s>>>(a.m, a.eu, a.ev, a.w, a.comp, a.local, a.bgoff, a.grp,
                                              a.gpt, a.b2off, a.b2rank, nullptr, a.b3off, a.b3rank,
                                              a.V3p, a.BG3);
    const int nt = (int)(a.V3p / 128);
    hipError_t e = (a.side && nt > 1)
                       ? launch_dense_fw_lookahead(a.BG3, a.V3p, 128, nt, s, a.side, a.sync, nullptr,
                                                   a.kc, a.pivot, nullptr, a.fw)
                       : launch_dense_fw(a.BG3, a.V3p, 128, nt, s, nullptr, a.kc, a.pivot, a.fw);
    if (e != hipSuccess) return e;
  }
  return launch_level3_compose(a, s);
}

hipError_t launch_level3_compose(const L3Args& a, hipStream_t s) {
  MpArgs m{};
  m.plist = a.plist;
  m.Vp = a.V3gp;
  m.Kp = a.m3pmax;
  m.NC = m.Vp / MP_T;
  m.NW = m.Kp / 64;
  m.m2 = a.m3; m.gV = a.tsize; m.b2off = a.b3off;
  m.D2 = a.BG3; m.ldd = a.V3p;
  m.R = a.R3; m.XT = a.XT3; m.stats = a.work.stats; m.mask = a.work.mask;
  m.cs.g0 = a.tbase; m.cs.rank = a.b3rank; m.cs.Mg = a.M3; m.cs.ngroups = a.nT;
  m.cs.dense = a.BG2; m.cs.ldo = a.V2p;
  for (int32_t p0 = 0; p0 < a.npairs; p0 += a.chunk) {
    m.pbase = p0;
    m.np = min(a.chunk, a.npairs - p0);
    mp_chunk_products(m, a.V3p > 0, false, a.work, nullptr, s);
  }
  return hipGetLastError();
}

hipError_t launch_hier_row(const HierArgs& a, int32_t x, u32* out, hipStream_t s) {
  k_hier_row<<<(unsigned)((a.V + 255) / 256 > 0 ? (a.V + 255) / 256 : 1), 256, 0, s>>>(
      x, a.share_groups > 0 ? 0 : 1, a.V, a.ngroups, a.bggrp, a.bgrow, a.bgnb, a.bglocal, a.gV,
      a.pairbase, a.H, out);
  return hipGetLastError();
}

}  // namespace spq

namespace spq {

hipError_t launch_share_prepare(const HierArgs& a, const ShareBlocks& b, hipStream_t s) {
  launch_r(a, s);
  k_blk_init<<<dim3((unsigned)b.bpmax, (unsigned)b.nblk), 256, 0, s>>>(a.Vgp, b.bpmax, b.bfirst,
                                                                       a.b2off, a.b2list, a.Mg,
                                                                       b.A);
  if (b.multi) {
    if (a.m > 0)
      k_blk_edges<<<hblocks(a.m), 256, 0, s>>>(a.m, a.eu, a.ev, a.w, a.comp, a.local, a.bgoff, a.grp,
                                               b.gblk, b.bfirst, a.b2off, a.b2rank, b.bpmax, b.A);
    hipError_t e = launch_dense_fw_batch(b.A, b.bpmax, 128, b.bpmax / 128, b.nblk,
                                         (int64_t)b.bpmax * b.bpmax, s, nullptr, a.kc, a.pivot,
                                         a.fw, FwSizes{b.bsize, b.h_bsize});
    if (e != hipSuccess) return e;
  }
  k_dt_init<<<(unsigned)a.V2p, 256, 0, s>>>(a.V2, a.S2, a.S2p, b.nblk, b.boff, b.bpmax, b.A, a.DT);
  if (a.m > 0)
    k_cross_collect<<<hblocks(a.m), 256, 0, s>>>(a.m, a.eu, a.ev, a.w, a.comp, a.local, a.bgoff, a.grp,
                                                 b.gblk, a.b2off, a.b2rank, a.xcount, a.xe);
  return hipGetLastError();
}

hipError_t launch_share_b3_lists(const HierArgs& a, const ShareBlocks& b, uint8_t* flag3,
                                 uint8_t* flagn, int32_t* b3list, int32_t* nb3list, int32_t* b3rank,
                                 int32_t* nrank, int32_t* m3, int32_t* n3, hipStream_t s) {
  hipError_t e = hipMemsetAsync(flag3, 0, (size_t)(a.V2 > 0 ? a.V2 : 1), s);
  if (e != hipSuccess) return e;
  if (a.m > 0) k_b3_mark<<<hblocks(2 * a.m), 256, 0, s>>>(a.xcount, a.xe, flag3);
  if (a.V2 > 0) k_flag_not<<<hblocks(a.V2), 256, 0, s>>>(a.V2, flag3, flagn);
  k_b2_scan<<<(unsigned)b.nblk, 256, 0, s>>>(b.boff, b.bsize, flag3, b.bpmax, b3list, b3rank, m3);
  k_b2_scan<<<(unsigned)b.nblk, 256, 0, s>>>(b.boff, b.bsize, flagn, b.bpmax, nb3list, nrank, n3);
  return hipGetLastError();
}

hipError_t launch_share_b3_gather(const ShareBlocks& b, const ShareB3& c, hipStream_t s) {
  k_a3_gather<<<dim3((unsigned)c.b3pmax, (unsigned)b.nblk), 256, 0, s>>>(b.bpmax, c.b3pmax, c.m3,
                                                                          c.b3list, b.A, c.A3);
  k_aout_gather<<<dim3((unsigned)c.b3pmax, (unsigned)b.nblk), 256, 0, s>>>(
      b.bpmax, c.b3pmax, c.n3pmax, c.m3, c.n3, c.b3list, c.nb3list, b.A, c.Aout);
  return hipGetLastError();
}

// One Bellman-Ford round, in place on DT: intra-block step on the B3 rows,
// then cross edges.
hipError_t launch_share_round(const HierArgs& a, const ShareBlocks& b, const ShareB3& c, int32_t nxe,
                              const BfRound& r, hipStream_t s) {
  const int ntm = c.b3pmax / 128, ntc = (int)(a.S2p / 128);
  k_bf_intra3<<<dim3((unsigned)(ntm * ntc), (unsigned)b.nblk), 256, 0, s>>>(
      b.bpmax, c.b3pmax, a.S2p, c.m3, b.boff, c.b3list, c.A3, a.DT, r.dirty, r.cnt, r.list);
  if (nxe > 0)
    k_bf_cross<<<(unsigned)nxe, 256, 0, s>>>(nxe, a.xe, a.S2, a.S2p, a.DT, r.dirty, r.dirty_next,
                                             c.b3rank, c.b3pmax, r.round, r.stamp, r.cnt_next,
                                             r.list_next);
  return hipGetLastError();
}

// The rows outside B3 from the settled B3 rows, pruned like the composition's products
// (the B3 rows of DT are distances from far away, Aout is part of a closed matrix): the
// B3 rows are gathered into rows3, then the same three kernels, masks and statistics in
// `scratch`.  By one product of every B3 row (k_bf_final, where the scratch is too
// small) a 30,700-row share took 4.6 ms, so 1.8 (build 49.3 -> 46.7).
int64_t share_final_words(const ShareBlocks& b, const ShareB3& c, int64_t S2p, int64_t* rows3) {
  *rows3 = (int64_t)b.nblk * c.b3pmax * S2p;
  const int64_t nt = mp_row_tiles<2>((int32_t)S2p);
  return (int64_t)b.nblk * (nt * (c.n3pmax / MP_T) * (c.b3pmax / 64) * 2 + nt * 2 * c.b3pmax);
}

hipError_t launch_share_final(const HierArgs& a, const ShareBlocks& b, const ShareB3& c, u32* rows3,
                              u32* scratch, hipStream_t s) {
  if (!rows3) {
    const int ntm = c.n3pmax / 128, ntc = (int)(a.S2p / 128);
    k_bf_final<<<dim3((unsigned)(ntm * ntc), (unsigned)b.nblk), 256, 0, s>>>(
        b.bpmax, c.b3pmax, c.n3pmax, a.S2p, c.m3, c.n3, b.boff, c.b3list, c.nb3list, c.Aout, a.DT);
    return hipGetLastError();
  }
  k_b3_rows<<<dim3((unsigned)c.b3pmax, (unsigned)b.nblk), 256, 0, s>>>(b.bpmax, a.S2p, c.m3, c.b3list,
                                                                       b.boff, a.DT, rows3);
  MpArgs m{};
  m.np = b.nblk;
  m.Vp = c.n3pmax;
  m.Kp = c.b3pmax;
  m.NC = m.Vp / MP_T;
  m.NW = m.Kp / 64;
  m.m2 = c.m3; m.gV = c.n3;
  m.ldd = a.S2p;
  m.R = c.Aout; m.XT = rows3;
  m.rows = a.S2; m.nstride = b.bpmax; m.boff = b.boff; m.nlist = c.nb3list; m.DT = a.DT;
  const int64_t nt = mp_row_tiles<2>((int32_t)a.S2p);
  m.mask = reinterpret_cast<unsigned long long*>(scratch);
  m.stats = reinterpret_cast<int32_t*>(scratch + (int64_t)b.nblk * nt * m.NC * m.NW * 2);
  mp_product<2>(m, false, a.work, nullptr, s);
  return hipGetLastError();
}

hipError_t launch_bf_rows(int32_t ngroups, int32_t lstride, int32_t kp, int64_t ldc,
                          const int32_t* nk, const int32_t* zero, const int32_t* own, const u32* A,
                          u32* C, const u32* dirty, const int32_t* rcnt, const int32_t* rlist,
                          hipStream_t s) {
  const int ntm = kp / 128, ntc = (int)(ldc / 128);
  k_bf_intra3<<<dim3((unsigned)(ntm * ntc), (unsigned)ngroups), 256, 0, s>>>(
      lstride, kp, ldc, nk, zero, own, A, C, dirty, rcnt, rlist);
  return hipGetLastError();
}

hipError_t launch_bf_gather(int32_t ngroups, int32_t lstride, int32_t kp, int32_t np, int64_t ldc,
                            const int32_t* nk, const int32_t* nout, const int32_t* zero,
                            const int32_t* own, const int32_t* out, const u32* Aout, u32* C,
                            hipStream_t s) {
  const int ntm = np / 128, ntc = (int)(ldc / 128);
  k_bf_final<<<dim3((unsigned)(ntm * ntc), (unsigned)ngroups), 256, 0, s>>>(
      lstride, kp, np, ldc, nk, nout, zero, own, out, Aout, C);
  return hipGetLastError();
}

hipError_t launch_share_compose(const HierArgs& a, const u32* DT, hipStream_t s) {
  dim3 tg((unsigned)((a.S2p + 31) / 32), (unsigned)(a.m2pmax / 32), (unsigned)a.ngroups);
  k_panel_transpose<<<tg, 256, 0, s>>>(DT, a.S2p, a.m2pmax, a.m2, a.b2off, a.BG2);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  HierArgs p = a;
  p.d2ld = a.m2pmax;
  p.d2pstride = a.S2p * a.m2pmax;
  return compose_level2(p, nullptr, nullptr, nullptr, s);
}

}  // namespace spq
