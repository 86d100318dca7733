// Blocked Floyd-Warshall (min-plus) on dense symmetric matrices: the
// closure of BG (Algorithm 1, Phase 3, by Floyd-Warshall instead of the
// paper's Dijkstra), of large components (Phase 2) and of the group and
// level-2/3 matrices of the two-level method.
#include "spq_internal.h"
#include "tiles.h"

#include <algorithm>
#include <vector>

namespace spq {

#define LAUNCH_CHECK() return hipGetLastError()

// Blocked Floyd-Warshall on one symmetric matrix of nt x nt tiles, in rounds
// over pivot blocks of one, two or four tiles (the tiles left at the end form
// smaller blocks):
//   close    the pivot block: k_fw_diag64 or k_fw_diag128 for one tile; a larger block by
//            squarings (k_fw_square) or, in large batches, by the same rounds on
//            the sub-matrix, over blocks of half its size
//   panel    tile (a, j), a in the block, j outside it: tile (a, j) =
//            D (x) tile (a, j), stored twice (as (a, j) and transposed as
//            (j, a)); k_fw_inner part 3 (k_fw_panel in fw_rounds, the
//            one-tile rounds of a batch)
//   interior tile (i, j) = min(tile (i, j),
//            (block rows, tile i)^T (x) (block rows, tile j)), k_fw_inner
// A two-tile block doubles the K of every interior product (256 instead of
// 128 for 128-tiles): the fixed cost of a tile (loading and storing C) is
// spread over twice the relaxations, and there are half as many rounds.
//
// A batch of equally sized matrices is handled by blockIdx.y: matrix y starts
// gstride elements after matrix y-1, or (components of one padded size) at
// moff[order[y]].
struct FwAt {
  int64_t gstride;
  const int32_t* order;
  const int64_t* moff;
  FwWork work;  // or none: see k_fw_square
  // null, or the vertices of each matrix, `first` of them before A's first row: the
  // tiles past them are padding, which no closure changes, and are left out.  Groups
  // differ in size (a 400,000-vertex graph: 128 of 930 vertices on average in 1,152
  // rows, 16 super-groups of 1,850 in 2,048: build 71.4 -> 70.6 ms).
  const int32_t* sizes;
  int first;
};
// Whether tile t (of T rows) of this workgroup's matrix is padding.
__device__ __forceinline__ bool fw_pad(const FwAt& at, int t, int T) {
  return at.sizes && at.first + t * T >= at.sizes[blockIdx.y];
}
__device__ __forceinline__ u32* fw_at(u32* A, const FwAt& at) {
  return A + (at.order ? at.moff[at.order[blockIdx.y]] : (int64_t)blockIdx.y * at.gstride);
}

template <int T>
__global__ __launch_bounds__(256) void k_fw_diag64(u32* __restrict__ A, int64_t ld, int r, FwAt at) {
  __shared__ __attribute__((aligned(16))) u32 rb[4 * T];
  if (fw_pad(at, r, T)) return;
  A = fw_at(A, at);
  u32 t[T / 16][T / 16];
  u32* D = A + (int64_t)r * T * ld + (int64_t)r * T;
  tile_load<T>(t, D, ld);
  fw_tile<T>(t, rb);
  tile_store<T>(t, D, ld);
}

// A 128-tile by 1,024 threads, 4 x 4 entries each (rows ty*4 + a, columns tx*4 +
// a): fw_tile's two pivots per barrier, with four waves per SIMD to cover the
// LDS reads and the barrier.  Bound by one CU's VALU (768 cycles for each of the
// 64 steps' relaxations).  A grid32-sized closure through it 0.87 -> 0.62 ms;
// 256 threads of 8 x 8, one wave per SIMD, took 53 us a tile.
__global__ __launch_bounds__(1024) void k_fw_diag128(u32* __restrict__ A, int64_t ld, int r, FwAt at) {
  constexpr int T = 128;
  __shared__ __attribute__((aligned(16))) u32 rb[4 * T];
  if (fw_pad(at, r, T)) return;
  u32* D = fw_at(A, at) + (int64_t)r * T * ld + (int64_t)r * T;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  u32 c[4][4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const uint4 v = *reinterpret_cast<const uint4*>(D + (int64_t)(ty * 4 + i) * ld + tx * 4);
    c[i][0] = v.x; c[i][1] = v.y; c[i][2] = v.z; c[i][3] = v.w;
  }
  auto put = [&](u32* buf, int i) {
    *reinterpret_cast<uint4*>(buf + tx * 4) = make_uint4(c[i][0], c[i][1], c[i][2], c[i][3]);
  };
  for (int k = 0; k < T; k += 2) {
    u32* buf = rb + ((k >> 1) & 1) * 2 * T;
    if (ty == k >> 2) {  // rows k, k + 1
      if (k & 2) {
        put(buf, 2);
        put(buf + T, 3);
      } else {
        put(buf, 0);
        put(buf + T, 1);
      }
    }
    __syncthreads();
    const u32 s = buf[T + k];  // M[k+1][k]
    const uint4 x = *reinterpret_cast<const uint4*>(buf + tx * 4);
    const uint4 y = *reinterpret_cast<const uint4*>(buf + T + tx * 4);
    const uint4 p = *reinterpret_cast<const uint4*>(buf + ty * 4);
    const uint4 q = *reinterpret_cast<const uint4*>(buf + T + ty * 4);
    const u32 kc[4] = {x.x, x.y, x.z, x.w}, kr[4] = {p.x, p.y, p.z, p.w};
    const u32 k1c[4] = {min(y.x, s + x.x), min(y.y, s + x.y), min(y.z, s + x.z), min(y.w, s + x.w)};
    const u32 k1r[4] = {min(q.x, s + p.x), min(q.y, s + p.y), min(q.z, s + p.z), min(q.w, s + p.w)};
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
      for (int j = 0; j < 4; j++) relax2(c[i][j], kr[i], kc[j], k1r[i], k1c[j]);
  }
#pragma unroll
  for (int i = 0; i < 4; i++)
    *reinterpret_cast<uint4*>(D + (int64_t)(ty * 4 + i) * ld + tx * 4) =
        make_uint4(c[i][0], c[i][1], c[i][2], c[i][3]);
}

template <int T>
static void fw_diag(u32* A, int64_t ld, int r, int batch, FwAt at, hipStream_t s) {
  if (T == 128)
    k_fw_diag128<<<dim3(1, batch), 1024, 0, s>>>(A, ld, r, at);
  else
    k_fw_diag64<64><<<dim3(1, batch), 256, 0, s>>>(A, ld, r, at);
}

template <int T>
__global__ __launch_bounds__(256) void k_fw_panel(u32* __restrict__ A, int64_t ld, int r, FwAt at) {
  __shared__ __attribute__((aligned(16))) u32 sD[T * T];
  __shared__ __attribute__((aligned(16))) u32 sB[T * T];
  A = fw_at(A, at);
  const int j = (int)blockIdx.x + ((int)blockIdx.x >= r);
  if (fw_pad(at, max(r, j), T)) return;
  u32 t[T / 16][T / 16];
  tile_load<T>(t, A + (int64_t)r * T * ld + (int64_t)r * T, ld);
  tile_to_lds<T>(t, sD);
  u32* Rj = A + (int64_t)r * T * ld + (int64_t)j * T;
  tile_load<T>(t, Rj, ld);
  tile_to_lds<T>(t, sB);
  __syncthreads();
  minplus_lds<T>(t, sD, sB, T);
  tile_store<T>(t, Rj, ld);
  tile_store_t<T>(t, A + (int64_t)j * T * ld + (int64_t)r * T, ld);
}

// Upper-triangle enumeration: block b -> (bi, bj), 0 <= bi <= bj < m, row by
// row (row bi holds m - bi blocks).
__device__ __forceinline__ void tri_index(int b, int m, int& bi, int& bj) {
  const float fm = 2.0f * m + 1.0f;
  int i = (int)((fm - sqrtf(fm * fm - 8.0f * (float)b)) * 0.5f);
  if (i < 0) i = 0;
  if (i > m - 1) i = m - 1;
  while (i > 0 && i * (2 * m - i + 1) / 2 > b) i--;
  while (i + 1 < m && (i + 1) * (2 * m - i) / 2 <= b) i++;
  bi = i;
  bj = i + (b - i * (2 * m - i + 1) / 2);
}

// Interior tiles.  The matrix is symmetric, so only tiles (i, j) with i <= j
// are computed; tile (j, i) receives the transpose.  The k dimension (the
// PT * T rows of the pivot block) is streamed through LDS in chunks of KC rows
// of the two operand tiles (double buffered, next chunk prefetched into
// registers while the current one is consumed).
//
// The pivot block is tiles [c0, c0 + PT); nn = tiles of the next block
// (parts 1 and 2).  part selects the tiles of the launch:
//   0  every tile outside the pivot block (i <= j)
//   1  the tiles with a row or column in the next block (what the next
//      round's diagonal and panel read)
//   2  every tile outside both blocks
//   3  the panel: (a, j) for a in the pivot block, j outside it (PT = 2)
template <int PT>
__device__ __forceinline__ void inner_tile(int part, int b, int c0, int nt, int nn, int& i, int& j) {
  int bi, bj;
  if (part == 0) {
    tri_index(b, nt - PT, bi, bj);
    i = bi + (bi >= c0 ? PT : 0);
    j = bj + (bj >= c0 ? PT : 0);
  } else if (part == 1) {
    const int no = nt - PT - nn;  // tiles outside both blocks
    if (b < nn * no) {
      const int x = c0 + PT + b / no, o = b % no;
      const int y = o + (o >= c0 ? PT + nn : 0);
      i = min(x, y);
      j = max(x, y);
    } else {
      tri_index(b - nn * no, nn, bi, bj);
      i = c0 + PT + bi;
      j = c0 + PT + bj;
    }
  } else if (part == 2) {
    tri_index(b, nt - PT - nn, bi, bj);
    i = bi + (bi >= c0 ? PT + nn : 0);
    j = bj + (bj >= c0 ? PT + nn : 0);
  } else {
    const int m = nt - PT, o = b % m;
    i = c0 + b / m;
    j = o + (o >= c0 ? PT : 0);
  }
}

// Four workgroups per CU while their chunks take 32 KB of LDS each, two at 64 KB.
template <int T, int KC, int PT>
__global__ __launch_bounds__(256, KC * T <= 2048 ? 4 : 2) void k_fw_inner(u32* __restrict__ A, int64_t ld, int c0, int nt,
                                                                FwAt at, int part, int nn) {
  constexpr int Q = KC * T / 4 / 256;  // uint4 per thread per operand chunk
  static_assert(Q >= 1 && KC * T / 4 % 256 == 0, "chunk must split evenly");
  __shared__ __attribute__((aligned(16))) u32 sA[2][KC * T];
  __shared__ __attribute__((aligned(16))) u32 sB[2][KC * T];
  A = fw_at(A, at);
  int i, j;
  inner_tile<PT>(part, (int)blockIdx.x, c0, nt, nn, i, j);
  if (fw_pad(at, max(c0, max(i, j)), T)) return;
  const u32* Ar = A + (int64_t)c0 * T * ld + (int64_t)i * T;  // block rows, tile column i
  const u32* Br = A + (int64_t)c0 * T * ld + (int64_t)j * T;  // block rows, tile column j
  u32* Cij = A + (int64_t)i * T * ld + (int64_t)j * T;
  u32 t[T / 16][T / 16];
  tile_load<T>(t, Cij, ld);
  // The operand chunks go from global memory straight to LDS
  // (global_load_lds_dwordx4, gfx950): no staging registers and no LDS
  // stores.  Element e (in 16-byte units) of a chunk is row e / (T/4),
  // column 4 (e % (T/4)); lane l of wave w loads e = s*256 + w*64 + l, and a
  // wave's 64 lanes fill 1 KB of LDS in that order.  A chunk is complete once
  // every wave's loads have arrived: vmcnt(0), then the barrier.
  const int wv = (int)threadIdx.x >> 6;
  auto load_chunk = [&](int kc, int buf) {
#pragma unroll
    for (int s = 0; s < Q; s++) {
      const int e = threadIdx.x + s * 256;
      const int row = e / (T / 4), c4 = e % (T / 4);
      const int64_t off = (int64_t)(kc + row) * ld + c4 * 4;
      lds_load16(Ar + off, &sA[buf][(s * 256 + wv * 64) * 4]);
      lds_load16(Br + off, &sB[buf][(s * 256 + wv * 64) * 4]);
    }
  };
  load_chunk(0, 0);
  wait_loads();
  __syncthreads();
  // The chunk loop stays rolled (unrolled, the staged version needed 136
  // VGPRs and three waves per SIMD).
  constexpr int NCH = PT * T / KC;
#pragma unroll 1
  for (int ch = 0; ch < NCH; ch++) {
    if (ch + 1 < NCH) load_chunk((ch + 1) * KC, (ch + 1) & 1);
    minplus_lds<T>(t, sA[ch & 1], sB[ch & 1], KC);
    wait_loads();
    __syncthreads();
  }
  tile_store<T>(t, Cij, ld);
  if (i != j) tile_store_t<T>(t, A + (int64_t)j * T * ld + (int64_t)i * T, ld);
}

// One squaring of the B x B block at A (B = 32 nb), in place: every entry takes
// the minimum over two-step walks.  After ceil(log2(B - 1)) squarings any walk of
// the block's at most B - 1 steps is covered: the closure, without the serial
// chain of B pivots in one workgroup.  In place is exact in any
// interleaving: every value read is the length of a real walk and at most the
// old value.  One workgroup per 32 x 32 tile i <= j (the other triangle gets the
// transpose); its four waves take a quarter of the K each, 4 x 4 entries per
// lane, operand rows straight to LDS 16 at a time, double buffered: 32 KB, which
// fits beside a running interior launch.  Bound by launch and load latency: a
// 256-wide block closes in 8 launches of 8.7 us (70 us; the rounds over its two
// 128-tiles took 258: two diagonal tiles of 52 us and four one-tile products of 39
// us in a row).
//
// q: which of the nq squarings.  Few hops inside a block suffice in most graphs
// (blocks of closed cliques: 2 or 3 squarings of 8), and once a squaring of the
// whole batch lowers nothing the block is closed: flags[q] is raised by one that
// does, and the ones after the first that does not end at once.  Launch 0 clears
// the flags from 1 on, launch 2 flag 0 (read by launch 1) for the next closure.
// The next round's closure runs beside this round's interior and is the longer
// of the two where matrices are small: its waves go first on a SIMD they share
// (13 -> 9 us a launch).  Both: the closures of a 27,900-vertex BG in three levels
// 1.5 of 14.0 ms less, a 400,000-vertex graph's 1.6 of 74.2.  relax: what this squaring
// executes in the whole batch, counted if it runs.
__global__ __launch_bounds__(256) void k_fw_square(u32* A, int64_t ld, int nb, FwAt at, int q, int nq,
                                                   unsigned long long relax) {
  constexpr int KC = 16;
  __shared__ __attribute__((aligned(16))) u32 sm[4][2][2][KC * 32];
  u32* flags = at.work.flags;
  const bool first = blockIdx.x == 0 && blockIdx.y == 0;
  if (flags) {
    if (first) {
      if (q == 0 && threadIdx.x >= 1 && (int)threadIdx.x < nq) flags[threadIdx.x] = 0;
      if (q == 2 && threadIdx.x == 0) flags[0] = 0;
    }
    if (q > 0 && flags[q - 1] == 0) return;
  }
  if (at.work.ran && first && threadIdx.x == 0) atomicAdd(at.work.ran, relax);
  __builtin_amdgcn_s_setprio(3);
  A = fw_at(A, at);
  int bi, bj;
  tri_index((int)blockIdx.x, nb, bi, bj);
  if (fw_pad(at, bj, 32)) return;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int ly = lane >> 3, lx = lane & 7, kn = nb * 8;  // K rows per wave
  const u32* Ar = A + (int64_t)(w * kn + ly) * ld + bi * 32 + lx * 4;
  const u32* Br = A + (int64_t)(w * kn + ly) * ld + bj * 32 + lx * 4;
  // eight lanes fetch a row's 32 words: a wave's load fills eight rows
  auto load = [&](int k, int buf) {
#pragma unroll
    for (int i = 0; i < KC / 8; i++) {
      lds_load16(Ar + (int64_t)(k + i * 8) * ld, &sm[w][buf][0][i * 256]);
      lds_load16(Br + (int64_t)(k + i * 8) * ld, &sm[w][buf][1][i * 256]);
    }
  };
  // thread t keeps four entries of the tile for the end
  const int er = threadIdx.x >> 3, ec = (threadIdx.x & 7) * 4;
  u32* Cp = A + (int64_t)(bi * 32 + er) * ld + bj * 32 + ec;
  load(0, 0);
  const uint4 old = *reinterpret_cast<const uint4*>(Cp);
  u32 c[4][4];
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int j = 0; j < 4; j++) c[i][j] = INF;
  for (int k = 0; k < kn; k += KC) {
    const int buf = (k / KC) & 1;
    // the chunk has arrived, and every LDS read of the other buffer is over
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    if (k + KC < kn) load(k + KC, buf ^ 1);
    const u32 *sa = sm[w][buf][0] + ly * 4, *sb = sm[w][buf][1] + lx * 4;
#pragma unroll
    for (int q = 0; q < KC; q += 2) {
      const uint4 a0 = *reinterpret_cast<const uint4*>(sa + q * 32);
      const uint4 a1 = *reinterpret_cast<const uint4*>(sa + q * 32 + 32);
      const uint4 b0 = *reinterpret_cast<const uint4*>(sb + q * 32);
      const uint4 b1 = *reinterpret_cast<const uint4*>(sb + q * 32 + 32);
      const u32 av[4] = {a0.x, a0.y, a0.z, a0.w}, aw[4] = {a1.x, a1.y, a1.z, a1.w};
      const u32 bv[4] = {b0.x, b0.y, b0.z, b0.w}, bw[4] = {b1.x, b1.y, b1.z, b1.w};
#pragma unroll
      for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) relax2(c[i][j], av[i], bv[j], aw[i], bw[j]);
    }
  }
  __syncthreads();
  u32* red = &sm[0][0][0][0];  // [4][32][32]: the waves' minima
#pragma unroll
  for (int i = 0; i < 4; i++)
    *reinterpret_cast<uint4*>(red + w * 1024 + (ly * 4 + i) * 32 + lx * 4) =
        make_uint4(c[i][0], c[i][1], c[i][2], c[i][3]);
  __syncthreads();
  uint4 v = old;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const uint4 x = *reinterpret_cast<const uint4*>(red + i * 1024 + er * 32 + ec);
    v.x = min(v.x, x.x);
    v.y = min(v.y, x.y);
    v.z = min(v.z, x.z);
    v.w = min(v.w, x.w);
  }
  if (flags && (v.x != old.x || v.y != old.y || v.z != old.z || v.w != old.w)) flags[q] = 1;
  *reinterpret_cast<uint4*>(Cp) = v;
  if (bi == bj) return;
  u32* tr = red + 4096;  // [32][33]
  tr[(ec + 0) * 33 + er] = v.x;
  tr[(ec + 1) * 33 + er] = v.y;
  tr[(ec + 2) * 33 + er] = v.z;
  tr[(ec + 3) * 33 + er] = v.w;
  __syncthreads();
  *reinterpret_cast<uint4*>(A + (int64_t)(bj * 32 + er) * ld + bi * 32 + ec) =
      make_uint4(tr[er * 33 + ec], tr[er * 33 + ec + 1], tr[er * 33 + ec + 2], tr[er * 33 + ec + 3]);
}

#ifndef SPQ_INNER_KC
#define SPQ_INNER_KC 16
#endif

template <int T, int KC>
static hipError_t fw_rounds(u32* A, int64_t ld, int nt, int batch, FwAt at, hipStream_t s,
                           hipEvent_t* ev) {
  for (int r = 0; r < nt; r++) {
    fw_diag<T>(A, ld, r, batch, at, s);
    if (nt > 1) {
      k_fw_panel<T><<<dim3(nt - 1, batch), 256, 0, s>>>(A, ld, r, at);
      if (ev) {
        hipError_t e = hipEventRecord(ev[2 * r], s);
        if (e != hipSuccess) return e;
      }
      k_fw_inner<T, KC, 1><<<dim3((unsigned)((nt - 1) * nt / 2), batch), 256, 0, s>>>(
          A, ld, r, nt, at, 0, 1);
      if (ev) {
        hipError_t e = hipEventRecord(ev[2 * r + 1], s);
        if (e != hipSuccess) return e;
      }
    }
  }
  LAUNCH_CHECK();
}

// Workgroups of a squaring launch, and 128-tiles of an interior launch, up to
// which the block closure and the split into 64-tiles above are taken.
constexpr int64_t SQUARE_WGS = 1024, SPLIT_TILES = 512;

// Pivot blocks of a single matrix: pivot_tiles (1, 2 or 4) tiles each; the
// tiles left at the end form blocks of two and one.
struct FwBlock {
  int c0, pt;
};

static int fw_blocks(int nt, int pivot_tiles, FwBlock* out) {
  int nb = 0;
  for (int c0 = 0; c0 < nt; nb++) {
    int pt = pivot_tiles;
    while (pt > nt - c0) pt >>= 1;
    if (out) out[nb] = FwBlock{c0, pt};
    c0 += pt;
  }
  return nb;
}

static int64_t tri_count(int64_t m) { return m > 0 ? m * (m + 1) / 2 : 0; }

// tiles of an interior launch of block b (parts 0-2; nn = next block's tiles)
static int64_t inner_count(int nt, FwBlock b, int part, int nn) {
  if (part == 0) return tri_count(nt - b.pt);
  if (part == 1) return (int64_t)nn * (nt - b.pt - nn) + tri_count(nn);
  return tri_count(nt - b.pt - nn);
}

// `batch` equally sized matrices (blockIdx.y)
struct FwBatch {
  int batch;
  FwAt at;
  const int32_t* hsizes;  // at.sizes on the host
};

template <int T, int KC>
static hipError_t fw_rounds_blocks(u32* A, int64_t ld, int nt, int pivot_tiles, FwBatch bt,
                                   hipStream_t s, hipEvent_t* ev);

// Squarings that close a block of n vertices.
static int fw_squarings(int n) {
  int q = 0;
  while ((1 << q) < n - 1) q++;
  return q;
}

// Whether the pivot blocks of `pt` tiles of a batch are closed by squarings:
// they execute more relaxations than the rounds over half-size blocks (8 x 256^3
// / 2 against 6 x 128^3 for two 128-tiles) but in short launches of many
// workgroups.  While a launch is at most four workgroups per CU they are the faster
// way: 70 against 258 us for one 256-row block, 16 blocks in a batch 130 against
// about 270 (a batch of 128 such blocks: 850 against about 300).
static bool fw_by_squaring(int tile, int pt, int batch) {
  return pt > 1 && tri_count(pt * tile / 32) * batch <= SQUARE_WGS;
}

// Relaxations of one squaring of a block of n vertices, of which the first `size` (< 0:
// all) are not padding.
static double square_relax(int64_t n, int64_t size) {
  const int64_t used = size < 0 ? n : std::max<int64_t>(0, std::min(n, size));
  return (double)tri_count((used + 31) / 32) * 1024.0 * (double)n;
}

static void fw_square_all(u32* D, int64_t ld, int n, FwBatch bt, hipStream_t s) {
  const int nq = fw_squarings(n);
  double relax = bt.hsizes ? 0 : bt.batch * square_relax(n, -1);
  for (int i = 0; bt.hsizes && i < bt.batch; i++)
    relax += square_relax(n, std::max(0, bt.hsizes[i] - bt.at.first));
  for (int q = 0; q < nq; q++)
    k_fw_square<<<dim3((unsigned)tri_count(n / 32), (unsigned)bt.batch), 256, 0, s>>>(D, ld, n / 32, bt.at,
                                                                                     q, nq, (unsigned long long)relax);
}

// A whole matrix of up to 512 vertices is one block.
static bool fw_all_squaring(int tile, int nt, int pt, int batch) {
  return pt > 1 && nt > 1 && nt * tile <= 512 && fw_by_squaring(tile, nt, batch);
}

// Closes the diagonal block: one tile in one workgroup (fw_diag); a block of
// two or four tiles by squarings or by the rounds of this file on the
// sub-matrix, over blocks of half its size.  Every launch of a block closure is
// small (32 KB LDS at most), so beside a running interior launch it finds room
// on a CU at once; one workgroup holding two tiles in LDS (130 KB) waited for
// a whole CU to drain, about as long as the interior.
template <int T, int KC>
static hipError_t fw_close(u32* A, int64_t ld, FwBlock b, FwBatch bt, hipStream_t s) {
  if (b.pt == 1) {
    fw_diag<T>(A, ld, b.c0, bt.batch, bt.at, s);
    return hipGetLastError();
  }
  u32* D = A + (int64_t)b.c0 * T * ld + (int64_t)b.c0 * T;
  bt.at.first += b.c0 * T;
  if (fw_by_squaring(T, b.pt, bt.batch)) {
    fw_square_all(D, ld, b.pt * T, bt, s);
    return hipGetLastError();
  }
  return fw_rounds_blocks<T, KC>(D, ld, b.pt, b.pt / 2, bt, s, nullptr);
}

// One launch of the interior kernel, part as in inner_tile, on `count` T-tiles
// per matrix.  A launch that leaves most CUs idle runs on 64-tiles instead: four
// times the workgroups, each with a quarter of the serial work (116 tiles of 128
// through 256 pivot rows 77 us, as 464 of 64 32 us; up to 512 tiles, two per CU,
// measured no slower split).
template <int T, int KC>
static void inner_launch(u32* A, int64_t ld, int nt, FwBlock b, int part, int nn, int64_t count,
                         FwBatch bt, hipStream_t s) {
  const dim3 grid((unsigned)count, (unsigned)bt.batch);
  if (b.pt == 1)
    k_fw_inner<T, KC, 1><<<grid, 256, 0, s>>>(A, ld, b.c0, nt, bt.at, part, nn);
  else if (b.pt == 2)
    k_fw_inner<T, KC, 2><<<grid, 256, 0, s>>>(A, ld, b.c0, nt, bt.at, part, nn);
  else if (b.pt == 4)
    k_fw_inner<T, KC, 4><<<grid, 256, 0, s>>>(A, ld, b.c0, nt, bt.at, part, nn);
  else if constexpr (T == 64 && KC == 16)  // four 128-tiles, split
    k_fw_inner<T, KC, 8><<<grid, 256, 0, s>>>(A, ld, b.c0, nt, bt.at, part, nn);
}

static int64_t part_count(int nt, FwBlock b, int part, int nn) {
  return part == 3 ? (int64_t)b.pt * (nt - b.pt) : inner_count(nt, b, part, nn);
}

template <int T, int KC>
static hipError_t fw_inner(u32* A, int64_t ld, int nt, FwBlock b, int part, int nn, FwBatch bt,
                           hipStream_t s) {
  const int64_t count = part_count(nt, b, part, nn);
  if (count <= 0) return hipSuccess;
  if (T == 128 && count * bt.batch <= SPLIT_TILES) {
    const FwBlock h{b.c0 * 2, b.pt * 2};
    inner_launch<64, 16>(A, ld, nt * 2, h, part, nn * 2, part_count(nt * 2, h, part, nn * 2), bt, s);
  } else {
    inner_launch<T, KC>(A, ld, nt, b, part, nn, count, bt, s);
  }
  return hipGetLastError();
}

// The panel of block b: tiles (a, j), a in the block, j outside it, by the
// interior kernel (part 3; 32 KB LDS, not k_fw_panel's 128 KB, for the same
// reason as above).
template <int T, int KC>
static hipError_t fw_panel(u32* A, int64_t ld, int nt, FwBlock b, FwBatch bt, hipStream_t s) {
  return fw_inner<T, KC>(A, ld, nt, b, 3, 0, bt, s);
}

#define CHK(x)                              \
  do {                                      \
    hipError_t e_ = (x);                    \
    if (e_ != hipSuccess) return e_;        \
  } while (0)

// Rounds over the pivot blocks on one stream (a batch of matrices at once).
// ev (optional) gets one pair per round around its interior launch.
template <int T, int KC>
static hipError_t fw_rounds_blocks(u32* A, int64_t ld, int nt, int pivot_tiles, FwBatch bt,
                                   hipStream_t s, hipEvent_t* ev) {
  std::vector<FwBlock> blk(fw_blocks(nt, pivot_tiles, nullptr));
  fw_blocks(nt, pivot_tiles, blk.data());
  for (size_t q = 0; q < blk.size(); q++) {
    CHK((fw_close<T, KC>(A, ld, blk[q], bt, s)));
    if (nt <= blk[q].pt) continue;
    CHK((fw_panel<T, KC>(A, ld, nt, blk[q], bt, s)));
    if (ev) CHK(hipEventRecord(ev[2 * q], s));
    CHK((fw_inner<T, KC>(A, ld, nt, blk[q], 0, 0, bt, s)));
    if (ev) CHK(hipEventRecord(ev[2 * q + 1], s));
  }
  return hipSuccess;
}

// The same rounds with a lookahead: the interior tiles with a row or column
// in the next pivot block go first (part 1); as soon as they are done, the
// next round's diagonal block and panel run on the side stream while the rest
// of this round's interior (part 2) runs on the main stream.  Part 2 neither
// reads nor writes a tile that the next round's diagonal or panel touches
// (rows and columns of the next block: the panel also writes the tiles of the
// current block's rows in those columns, which part 2 does not read), so the
// two overlap safely.  A batch of matrices runs the same rounds side by side
// (the argument holds for each).  With a third stream p1, part 1 runs there
// beside part 2 instead of before it (part 1 alone leaves workgroup slots
// idle); the round still ends only when both are done.  ev (optional) gets
// one pair per round around parts 1 + 2.
template <int T, int KC>
static hipError_t fw_rounds_lookahead(u32* A, int64_t ld, int nt, int pivot_tiles, FwBatch bt,
                                      hipStream_t s, hipStream_t side, hipStream_t p1,
                                      hipEvent_t* sync, hipEvent_t* ev) {
  std::vector<FwBlock> blk(fw_blocks(nt, pivot_tiles, nullptr));
  fw_blocks(nt, pivot_tiles, blk.data());
  // sync[0] = side stream may start the next round (part 1 of this one done);
  // sync[1] = main stream may start the next round's interior (its panel done);
  // sync[2] (with p1) = p1 may start this round's part 1
  CHK(hipEventRecord(sync[0], s));
  CHK(hipStreamWaitEvent(side, sync[0], 0));
  CHK((fw_close<T, KC>(A, ld, blk[0], bt, side)));
  CHK((fw_panel<T, KC>(A, ld, nt, blk[0], bt, side)));
  CHK(hipEventRecord(sync[1], side));
  for (size_t q = 0; q < blk.size(); q++) {
    CHK(hipStreamWaitEvent(s, sync[1], 0));
    if (nt <= blk[q].pt) continue;  // a single block: closed, nothing else
    if (ev) CHK(hipEventRecord(ev[2 * q], s));
    if (q + 1 < blk.size()) {
      const int nn = blk[q + 1].pt;
      hipStream_t s1 = s;
      if (p1) {
        CHK(hipEventRecord(sync[2], s));
        CHK(hipStreamWaitEvent(p1, sync[2], 0));
        s1 = p1;
      }
      CHK((fw_inner<T, KC>(A, ld, nt, blk[q], 1, nn, bt, s1)));
      CHK(hipEventRecord(sync[0], s1));
      CHK(hipStreamWaitEvent(side, sync[0], 0));
      CHK((fw_close<T, KC>(A, ld, blk[q + 1], bt, side)));
      CHK((fw_panel<T, KC>(A, ld, nt, blk[q + 1], bt, side)));
      CHK((fw_inner<T, KC>(A, ld, nt, blk[q], 2, nn, bt, s)));
      CHK(hipEventRecord(sync[1], side));
      if (p1) CHK(hipStreamWaitEvent(s, sync[0], 0));  // the round ends with part 1 too
    } else {
      // last round: nothing to look ahead to
      CHK((fw_inner<T, KC>(A, ld, nt, blk[q], 0, 0, bt, s)));
    }
    if (ev) CHK(hipEventRecord(ev[2 * q + 1], s));
  }
  return hipSuccess;
}

static int pivot_tiles_of(int tile, int pivot) { return pivot <= tile ? 1 : pivot / tile; }

int fw_rounds_count(int nt, int tile, int pivot) {
  return fw_blocks(nt, pivot_tiles_of(tile, pivot), nullptr);
}

hipError_t launch_dense_fw(u32* A, int64_t ld, int tile, int nt, hipStream_t s, hipEvent_t* ev,
                           int kc, int pivot, FwWork work) {
  return launch_dense_fw_batch(A, ld, tile, nt, 1, 0, s, ev, kc, pivot, work);
}

static hipError_t dense_lookahead(u32* A, int64_t ld, int tile, int nt, FwBatch bt, hipStream_t s,
                                  hipStream_t side, hipStream_t p1, hipEvent_t* sync,
                                  hipEvent_t* ev, int kc, int pivot) {
  if (nt <= 0 || bt.batch <= 0) return hipSuccess;
  const int pt = pivot_tiles_of(tile, pivot);
  if (!ev && fw_all_squaring(tile, nt, pt, bt.batch)) {
    fw_square_all(A, ld, nt * tile, bt, s);
    return hipGetLastError();
  }
  if (kc == 0) kc = SPQ_INNER_KC;
  if (tile == 64)
    return kc == 32 ? fw_rounds_lookahead<64, 32>(A, ld, nt, pt, bt, s, side, p1, sync, ev)
                    : fw_rounds_lookahead<64, 16>(A, ld, nt, pt, bt, s, side, p1, sync, ev);
  return kc == 32 ? fw_rounds_lookahead<128, 32>(A, ld, nt, pt, bt, s, side, p1, sync, ev)
                  : fw_rounds_lookahead<128, 16>(A, ld, nt, pt, bt, s, side, p1, sync, ev);
}

hipError_t launch_dense_fw_lookahead(u32* A, int64_t ld, int tile, int nt, hipStream_t s,
                                     hipStream_t side, hipEvent_t* sync, hipEvent_t* ev, int kc,
                                     int pivot, hipStream_t p1, FwWork work) {
  return dense_lookahead(A, ld, tile, nt, FwBatch{1, FwAt{0, nullptr, nullptr, work, nullptr, 0}, nullptr}, s, side, p1, sync, ev, kc, pivot);
}

hipError_t launch_dense_fw_batch_lookahead(u32* A, int64_t ld, int tile, int nt, int batch,
                                           int64_t gstride, hipStream_t s, hipStream_t side,
                                           hipEvent_t* sync, hipEvent_t* ev, int kc, int pivot, FwWork work,
                                           FwSizes sizes) {
  return dense_lookahead(A, ld, tile, nt, FwBatch{batch, FwAt{gstride, nullptr, nullptr, work, sizes.dev, 0}, sizes.host}, s, side,
                         nullptr, sync, ev, kc, pivot);
}
#undef CHK

// kc: K chunk of the interior-tile kernel (16 or 32; 0 = SPQ_INNER_KC)
static hipError_t dense_rounds(u32* A, int64_t ld, int tile, int nt, FwBatch bt, hipStream_t s,
                               hipEvent_t* ev, int kc, int pivot) {
  if (nt <= 0 || bt.batch <= 0) return hipSuccess;
  if (kc == 0) kc = SPQ_INNER_KC;
  const int pt = pivot_tiles_of(tile, pivot);
  if (pt > 1) {
    if (!ev && fw_all_squaring(tile, nt, pt, bt.batch)) {
      fw_square_all(A, ld, nt * tile, bt, s);
      return hipGetLastError();
    }
    if (tile == 64)
      return kc == 32 ? fw_rounds_blocks<64, 32>(A, ld, nt, pt, bt, s, ev)
                      : fw_rounds_blocks<64, 16>(A, ld, nt, pt, bt, s, ev);
    return kc == 32 ? fw_rounds_blocks<128, 32>(A, ld, nt, pt, bt, s, ev)
                    : fw_rounds_blocks<128, 16>(A, ld, nt, pt, bt, s, ev);
  }
  if (tile == 64)
    return kc == 32 ? fw_rounds<64, 32>(A, ld, nt, bt.batch, bt.at, s, ev)
                    : fw_rounds<64, 16>(A, ld, nt, bt.batch, bt.at, s, ev);
  return kc == 32 ? fw_rounds<128, 32>(A, ld, nt, bt.batch, bt.at, s, ev)
                  : fw_rounds<128, 16>(A, ld, nt, bt.batch, bt.at, s, ev);
}

hipError_t launch_dense_fw_batch(u32* A, int64_t ld, int tile, int nt, int batch, int64_t gstride,
                                 hipStream_t s, hipEvent_t* ev, int kc, int pivot, FwWork work, FwSizes sizes) {
  return dense_rounds(A, ld, tile, nt, FwBatch{batch, FwAt{gstride, nullptr, nullptr, work, sizes.dev, 0}, sizes.host}, s, ev, kc,
                      pivot);
}

hipError_t launch_dense_fw_list(u32* A, int64_t ld, int tile, int nt, int batch, const int32_t* order,
                                const int64_t* moff, hipStream_t s, int kc, int pivot, FwWork work) {
  return dense_rounds(A, ld, tile, nt, FwBatch{batch, FwAt{0, order, moff, work, nullptr, 0}, nullptr}, s, nullptr, kc, pivot);
}

// Executed relaxations of a matrix closed in a batch of `batch`: per round the
// pivot block (one tile: T^3; more: squarings, which are counted as they run, or the
// rounds over half-size blocks on it), the panel (each of its tiles K = block rows) and the
// upper-triangle interior tiles; `inner` gets the interior part.
double dense_fw_exec_relax(int64_t nt, int tile, int pivot, double* inner, int batch, int64_t size) {
  const double t3 = (double)tile * tile * tile;
  const int ptiles = pivot_tiles_of(tile, pivot);
  const int64_t used = size < 0 ? nt : std::min(nt, (size + tile - 1) / tile);  // tiles not padding
  if (inner) *inner = 0;
  if (fw_all_squaring(tile, (int)nt, ptiles, batch)) return 0;
  std::vector<FwBlock> blk(fw_blocks((int)nt, ptiles, nullptr));
  fw_blocks((int)nt, ptiles, blk.data());
  double all = 0, in = 0;
  for (const FwBlock& b : blk) {
    const int64_t mine = std::min<int64_t>(b.pt, used - b.c0);  // of the block's tiles
    if (mine <= 0) break;
    const int64_t left = size < 0 ? -1 : size - (int64_t)b.c0 * tile;
    all += b.pt == 1                           ? t3
           : fw_by_squaring(tile, b.pt, batch) ? 0.0
                                               : dense_fw_exec_relax(b.pt, tile, b.pt / 2 * tile, nullptr, batch, left);
    if (nt <= b.pt) continue;
    all += (double)mine * (used - mine) * b.pt * t3;
    const double x = (double)tri_count(used - mine) * b.pt * t3;
    all += x;
    in += x;
  }
  if (inner) *inner = in;
  return all;
}

}  // namespace spq
