// Particle binning by grid tile and the LDS-privatised charge deposition of the tracking loop.
//
// Every step the particles are counting-sorted by the tile of their stencil's first node
// (tiles of T_x x T_y x T_z cells, at most 4096 tiles).  Particles move several cells per step,
// so the order is rebuilt each step; the previous step's order keeps every pass coherent:
//   k_key_rank     tile key of each particle and its rank within the tile, packed in 4 B: the
//                  rank inside the workgroup from a histogram in LDS, the workgroup's base from
//                  the global atomic (one per non-empty bin) that flushes it.  The last
//                  workgroup to finish scans the tile counts (sort offsets) and writes the work
//                  list of (tile, begin, end) chunks of at most `chunk` particles;
//   k_scatter      moves phase space and particle ids to their sorted slots: each block
//                  counts its keys in LDS, reserves one contiguous range per key with a single
//                  global atomic, then ranks its particles with LDS atomics, so particles of one
//                  key leave a block as one contiguous run (first step of a call, where the
//                  caller's order is unrelated to the tiles);
//   k_place        the order without moving anything: the source index of every sorted slot,
//                  perm[tile offset + rank] = i (8 B per particle instead of 104).  Later steps,
//                  and the first step of a small beam, read the particles through it, and the
//                  gather-kick writes the new state in sorted order, so the phase space crosses
//                  HBM once per step fewer;
//   k_deposit_tiles each workgroup takes a chunk, accumulates the (T + S)^3 window of its tile
//                  with 64-bit fixed-point LDS atomics, and adds the non-zero window entries to
//                  the tile's own 64-bit integer window in HBM with one integer atomic each;
//   k_tile_reduce  forms the charge grid from the tiles' integer windows in a fixed order, so
//                  the grid depends neither on the particle order nor on that of the atomics;
//   k_gkd_tiles    the gather, kick and push of a chunk from its tile's E' window in LDS,
//                  reading through the ranking and writing the new state in sorted order.
#include "device_common.hpp"
#include "internal.hpp"

namespace pic {

namespace {

constexpr int kBlk = 256;
constexpr int kItems = 4096;               // particles per block in key_hist / scatter
constexpr int kPer = kItems / kBlk;         // 16 per thread

// the tile key's bits of a packed (rank, key) word
__host__ __device__ __forceinline__ uint32_t key_mask(const SortPlan& sp) {
  return (1u << sp.kbits) - 1u;
}

// stencil base node along one axis: the very function the deposit and gather kernels use
template <int S>
__device__ __forceinline__ int base_node(double u, int n) {
  double w[S + 1];
  return stencil<S>(u, n, w);
}

template <int S>
__device__ __forceinline__ uint32_t tile_key(double x, double y, double z, const double* o,
                                             const double* ih, const Consts& c,
                                             const SortPlan& sp) {
  int bx = base_node<S>((x - o[0]) * ih[0], c.nx);
  int by = base_node<S>((y - o[1]) * ih[1], c.ny);
  int bz = base_node<S>((z - o[2]) * ih[2], c.nz);
  return (uint32_t)(((bz / sp.T[2]) * sp.NT[1] + (by / sp.T[1])) * sp.NT[0] + (bx / sp.T[0]));
}

// Exclusive scan of v over the workgroup's NT threads, by wave scans; total: the sum of all.
template <int NT>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* total) {
  __shared__ uint32_t wsum[NT / 64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t incl = v;
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t up = __shfl_up(incl, off);
    if (lane >= off) incl += up;
  }
  __syncthreads();  // readers of a previous scan are done with wsum
  if (lane == 63) wsum[wv] = incl;
  __syncthreads();
  uint32_t base = 0, all = 0;
  for (int q = 0; q < NT / 64; ++q) {
    base += q < wv ? wsum[q] : 0u;
    all += wsum[q];
  }
  *total = all;
  return base + incl - v;
}

// In-place exclusive scan of a[0..count) (count <= kMaxTiles) by one block of NT threads;
// each thread owns a run of consecutive entries.  Returns the sum of all entries.
template <int NT>
__device__ uint32_t block_exclusive_scan_lds(uint32_t* a, int count) {
  const int per = (count + NT - 1) / NT;
  const int b = threadIdx.x * per;
  const int e = min(b + per, count);
  uint32_t sum = 0, total;
  for (int t = b; t < e; ++t) sum += a[t];
  uint32_t run = block_exclusive_scan<NT>(sum, &total);
  for (int t = b; t < e; ++t) {
    const uint32_t v = a[t];
    a[t] = run;
    run += v;
  }
  __syncthreads();
  return total;
}

// nchunks[0]: entries of the work list; [1]: workgroups of k_key_rank that have finished (zero
// between launches); [2]: non-zero if a tile's ranks do not fit the packed key
constexpr int kNck = 0, kTicket = 1, kOverflow = 2;

// Sort offsets (cursor) and work list from the tile counts in hist (left zero), by one block of
// NT threads; lh: kMaxTiles words of LDS.  Thread t takes tiles t, t + NT, ..., so that the dense
// tiles in the middle of the grid, whose chunks are many, are spread over the threads.  The
// counts are read with agent-scope atomic loads: other workgroups of the same launch may have
// added to them.  Counts that do not hold every one of the n particles once, or a list that would
// not fit (neither can be with a histogram that started at zero), are a fault of the library: no
// list is written and the status says so, on which the passes behind it do nothing.
// A thread writes up to kOwnItems items of a tile; the workgroup writes the rest of up to kWideTiles
// such tiles together.  On a grid of a few tiles one thread's chain of stores was the length of the
// pass otherwise: k_key_rank 115 us at 1.77e6 particles in one tile of a 4^3 grid, 95 at 2e6 in 27 of
// 12^3, 19 and 22 so.
constexpr int kOwnItems = 32, kWideTiles = 128;
template <int NT>
__device__ __forceinline__ void build_chunks_body(const Geom* g, int64_t n, const SortPlan& sp,
                                                  uint32_t* __restrict__ hist,
                                                  uint32_t* __restrict__ cursor,
                                                  int4* __restrict__ chunks,
                                                  uint32_t* __restrict__ nchunks, uint32_t* lh) {
  constexpr int Q = kMaxTiles / NT;
  __shared__ uint32_t nwide;
  __shared__ uint4 wide[kWideTiles];  // first entry, first particle, particles, tile
  uint32_t cnt[Q], off[Q];
  bool over = false;
  if (threadIdx.x == 0) nwide = 0u;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int t = q * NT + threadIdx.x;
    cnt[q] = 0u;
    if (t < sp.ntiles) {
      cnt[q] = __hip_atomic_load(&hist[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      hist[t] = 0u;  // ready for the next step
      lh[t] = cnt[q];
      over |= cnt[q] && ((uint64_t)(cnt[q] - 1u) >> (32 - sp.kbits)) != 0ull;
    }
  }
  __syncthreads();
  const uint32_t tot_c = block_exclusive_scan_lds<NT>(lh, sp.ntiles);
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int t = q * NT + threadIdx.x;
    if (t < sp.ntiles) {
      off[q] = lh[t];
      cursor[t] = off[q];
      lh[t] = (cnt[q] + sp.chunk - 1) / sp.chunk;
    }
  }
  over = __syncthreads_or(over);
  const uint32_t tot_k = block_exclusive_scan_lds<NT>(lh, sp.ntiles);
  const bool fault = tot_c != (uint32_t)n || (int64_t)tot_k > sp.max_chunks;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int t = q * NT + threadIdx.x;
    if (t < sp.ntiles && !fault) {
      int4* out = chunks + lh[t];
      const uint32_t end = off[q] + cnt[q];
      uint32_t own = end;
      if (cnt[q] > (uint64_t)kOwnItems * sp.chunk) {
        const uint32_t w = atomicAdd(&nwide, 1u);
        if (w < kWideTiles) {
          wide[w] = make_uint4(lh[t], off[q], cnt[q], (uint32_t)t);
          own = off[q] + (uint32_t)kOwnItems * sp.chunk;
        }
      }
      for (uint32_t b = off[q]; b < own; b += sp.chunk)
        *out++ = make_int4(t, (int)b, (int)min(b + sp.chunk, end), (int)cnt[q]);  // w: the tile's
    }
  }
  __syncthreads();
  const uint32_t nw = min(nwide, (uint32_t)kWideTiles);
  for (uint32_t w = 0; w < nw; ++w) {
    const uint4 x = wide[w];
    const uint32_t end = x.y + x.z, items = (x.z + sp.chunk - 1) / sp.chunk;
    for (uint32_t k = kOwnItems + threadIdx.x; k < items; k += NT) {
      const uint32_t b = x.y + k * sp.chunk;
      chunks[x.x + k] = make_int4((int)x.w, (int)b, (int)min(b + sp.chunk, end), (int)x.z);
    }
  }
  if (threadIdx.x == 0) {
    if (fault) atomicCAS(const_cast<int*>(&g->status), 0, -7);
    nchunks[kNck] = fault ? 0u : tot_k;
    nchunks[kTicket] = 0u;
    nchunks[kOverflow] = over ? 1u : 0u;
  }
}

__global__ __launch_bounds__(1024) void k_build_chunks(const Geom* g, int64_t n, SortPlan sp,
                                                       uint32_t* __restrict__ hist,
                                                       uint32_t* __restrict__ cursor,
                                                       int4* __restrict__ chunks,
                                                       uint32_t* __restrict__ nchunks) {
  __shared__ uint32_t lh[kMaxTiles];
  if (g->status) {
    if (threadIdx.x == 0) nchunks[kNck] = 0u;
    return;
  }
  build_chunks_body<1024>(g, n, sp, hist, cursor, chunks, nchunks, lh);
}

// Keys, ranks, sort offsets and work list of the particles in X (see the list at the top of the
// file), PER particles per thread.  keys[i] = rank << sp.kbits | key; a rank that does not fit
// (a tile of more than 2^(32 - kbits) particles, at least 2^20) loses its upper bits and the
// work list's overflow word is set, on which k_place ranks anew from the keys.
// The last workgroup is found with a counter: a workgroup adds to it only after its own atomics
// on hist have returned (their results are in LDS, and the barrier stands between), and the
// counts are read and changed by agent-scope atomics alone, so the last one reads them whole.
template <int S, int PER>
__device__ __forceinline__ void key_rank_body(const double* __restrict__ X, const Geom* g,
                                              const Consts& c,
                                              const SortPlan& sp, uint32_t* __restrict__ keys,
                                              uint32_t* __restrict__ hist,
                                              uint32_t* __restrict__ cursor,
                                              int4* __restrict__ chunks,
                                              uint32_t* __restrict__ nchunks, int blk, int nblk) {
  __shared__ uint32_t lh[kMaxTiles];
  __shared__ bool s_last;
  if (g->status) {
    if (blk == 0 && threadIdx.x == 0) nchunks[kNck] = 0u;
    return;
  }
  const double o[3] = {g->origin[0], g->origin[1], g->origin[2]};
  const double ih[3] = {g->inv_h[0], g->inv_h[1], g->inv_h[2]};
  for (int t = threadIdx.x; t < sp.ntiles; t += kBlk) lh[t] = 0u;
  __syncthreads();
  const int64_t n = c.n;
  const int64_t base = (int64_t)blk * (kBlk * PER) + threadIdx.x;
  uint32_t key[PER], rank[PER];
  // loads of up to four particles in flight, without a branch around them (clamped to the last)
  constexpr int G = PER < 4 ? PER : 4;
#pragma unroll
  for (int k0 = 0; k0 < PER; k0 += G) {
    double p[G][3];
#pragma unroll
    for (int k = 0; k < G; ++k) {
      const int64_t i = min(base + (k0 + k) * kBlk, n - 1);
      for (int a = 0; a < 3; ++a) p[k][a] = X[2 * a * n + i];
    }
#pragma unroll
    for (int k = 0; k < G; ++k) {
      key[k0 + k] = tile_key<S>(p[k][0], p[k][1], p[k][2], o, ih, c, sp);
      if (base + (k0 + k) * kBlk < n) rank[k0 + k] = atomicAdd(&lh[key[k0 + k]], 1u);
    }
  }
  __syncthreads();
  // four of a thread's counters at a time, so that the returns of their atomics overlap
  for (int t0 = threadIdx.x; t0 < sp.ntiles; t0 += 4 * kBlk) {
    uint32_t cnt[4], old[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = t0 + u * kBlk;
      cnt[u] = t < sp.ntiles ? lh[t] : 0u;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (cnt[u]) old[u] = atomicAdd(&hist[t0 + u * kBlk], cnt[u]);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (cnt[u]) lh[t0 + u * kBlk] = old[u];
  }
  __syncthreads();
  if (threadIdx.x == 0) s_last = atomicAdd(&nchunks[kTicket], 1u) == (uint32_t)nblk - 1u;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int64_t i = base + k * kBlk;
    if (i < n) keys[i] = ((rank[k] + lh[key[k]]) << sp.kbits) | key[k];
  }
  __syncthreads();
  if (s_last) build_chunks_body<kBlk>(g, n, sp, hist, cursor, chunks, nchunks, lh);
}

template <int S, int PER>
__global__ __launch_bounds__(kBlk) void k_key_rank(const double* __restrict__ X,
                                                   const Geom* g, Consts c,
                                                   SortPlan sp, uint32_t* __restrict__ keys,
                                                   uint32_t* __restrict__ hist,
                                                   uint32_t* __restrict__ cursor,
                                                   int4* __restrict__ chunks,
                                                   uint32_t* __restrict__ nchunks) {
  key_rank_body<S, PER>(X, g, c, sp, keys, hist, cursor, chunks, nchunks, blockIdx.x, gridDim.x);
}

// LDS atomic add of 1 per active lane to lh[key], aggregated over the wave: one atomic per
// distinct key among the active lanes (their count), each lane getting the value it would
// have had from its own atomic in lane order.  Called by all lanes of the wave (the loop is
// wave-uniform).  After the first step of a call the particles arrive in the previous step's
// tile order, so a wave holds only a few distinct keys and the same-address atomics that
// would serialise lane by lane collapse into one per key.
__device__ __forceinline__ uint32_t wave_aggregated_add(uint32_t* lh, uint32_t key, bool active) {
  const int lane = (int)__lane_id();
  const uint64_t below = (1ull << lane) - 1ull;
  uint64_t todo = __ballot(active);
  uint32_t out = 0u;
  while (todo) {
    const int leader = __ffsll((unsigned long long)todo) - 1;  // wave-uniform
    const uint32_t k0 = (uint32_t)__builtin_amdgcn_readlane((int)key, leader);
    const uint64_t grp = todo & __ballot(key == k0);
    uint32_t b = 0u;
    if (lane == leader) b = atomicAdd(&lh[k0], (uint32_t)__popcll(grp));
    b = (uint32_t)__builtin_amdgcn_readlane((int)b, leader);
    if ((grp >> lane) & 1ull) out = b + (uint32_t)__popcll(grp & below);
    todo &= ~grp;
  }
  return out;
}

// Counting-sort scatter of one block of kItems particles, staged: the block ranks its items by
// key in LDS (local offsets by a scan of its key counts, one global atomic per key present to
// reserve the key's run in the output), then moves each row through LDS in ranked order, so
// every key's run leaves the block as consecutive lanes writing consecutive addresses.  Used
// where the input order is unrelated to the keys (the caller's order, the id buckets of the
// final reordering): there it writes 3.6 times fewer bytes than the direct form.
__device__ __forceinline__ void scatter_staged_body(const double* __restrict__ A,
                                                  const uint32_t* __restrict__ idA,
                                                  const uint32_t* __restrict__ keys,
                                                  uint32_t kmask,
                                                  const Geom* __restrict__ g, int64_t n,
                                                  int ntiles, uint32_t* __restrict__ cursor,
                                                  double* __restrict__ B,
                                                  uint32_t* __restrict__ idB, int blk, int nblk) {
  // cur/delta (ranking) and the row buffer share storage
  __shared__ __align__(16) unsigned char stage[2 * kMaxTiles * sizeof(uint32_t)];
  __shared__ uint32_t dest[kItems];
  static_assert(kItems * sizeof(double) <= sizeof(stage), "row buffer exceeds its storage");
  uint32_t* cur = reinterpret_cast<uint32_t*>(stage);
  uint32_t* delta = cur + kMaxTiles;
  double* rowbuf = reinterpret_cast<double*>(stage);
  uint32_t* idbuf = reinterpret_cast<uint32_t*>(stage);
  if (g->status) return;
  const int64_t base = (int64_t)blk * kItems;
  const int m = (int)min((int64_t)kItems, n - base);
  for (int t = threadIdx.x; t < ntiles; t += kBlk) cur[t] = 0u;
  __syncthreads();
  uint32_t key[kPer];
  for (int k = 0; k < kPer; ++k) {
    const int l = k * kBlk + threadIdx.x;
    key[k] = l < m ? keys[base + l] & kmask : 0u;
    if (l < m) atomicAdd(&cur[key[k]], 1u);
  }
  __syncthreads();
  // reserve each present key's run in the output
  for (int t = threadIdx.x; t < ntiles; t += kBlk) {
    const uint32_t c = cur[t];
    delta[t] = c ? atomicAdd(&cursor[t], c) : 0u;
  }
  __syncthreads();
  block_exclusive_scan_lds<kBlk>(cur, ntiles);  // cur[t] = local offset of key t
  for (int t = threadIdx.x; t < ntiles; t += kBlk) delta[t] -= cur[t];
  __syncthreads();
  uint32_t slot[kPer];
  for (int k = 0; k < kPer; ++k) {
    const int l = k * kBlk + threadIdx.x;
    if (l < m) {
      slot[k] = atomicAdd(&cur[key[k]], 1u);
      dest[slot[k]] = delta[key[k]] + slot[k];
    }
  }
  __syncthreads();
  const int rows = idA ? 7 : 6;  // the ids travel as a seventh row when there are any
  for (int r = 0; r < rows; ++r) {
    for (int k = 0; k < kPer; ++k) {
      const int l = k * kBlk + threadIdx.x;
      if (l < m) {
        if (r < 6)
          rowbuf[slot[k]] = A[r * n + base + l];
        else
          idbuf[slot[k]] = idA[base + l];
      }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < m; q += kBlk) {
      const uint32_t d = dest[q];
      if (d < (uint64_t)n) {  // always true for a consistent histogram; keeps writes in bounds
        if (r < 6)
          B[r * n + d] = rowbuf[q];
        else
          idB[d] = idbuf[q];
      }
    }
    __syncthreads();
  }
}

// Counting-sort scatter of one block of kItems particles, written straight from registers: the
// block counts its keys in LDS, reserves one run per key with a global atomic, and ranks its
// particles with LDS atomics.  When the input is already close to the key order (the previous
// step's binning), the lanes of a wave mostly share a key and get consecutive slots, so the
// writes coalesce without staging.
__device__ __forceinline__ void scatter_direct_body(const double* __restrict__ A,
                                                  const uint32_t* __restrict__ idA,
                                                  const uint32_t* __restrict__ keys,
                                                  uint32_t kmask,
                                                  const Geom* __restrict__ g, int64_t n,
                                                  int ntiles, uint32_t* __restrict__ cursor,
                                                  double* __restrict__ B,
                                                  uint32_t* __restrict__ idB, int blk, int nblk) {
  __shared__ uint32_t lh[kMaxTiles];
  if (g->status) return;
  for (int t = threadIdx.x; t < ntiles; t += kBlk) lh[t] = 0u;
  __syncthreads();
  const int64_t base = (int64_t)blk * kItems;
  uint32_t key[kPer];
  for (int k = 0; k < kPer; ++k) {
    int64_t i = base + k * kBlk + threadIdx.x;
    key[k] = i < n ? keys[i] & kmask : 0u;
    if (i < n) atomicAdd(&lh[key[k]], 1u);
  }
  __syncthreads();
  for (int t = threadIdx.x; t < ntiles; t += kBlk)
    if (lh[t]) lh[t] = atomicAdd(&cursor[t], lh[t]);
  __syncthreads();
  for (int k = 0; k < kPer; ++k) {
    int64_t i = base + k * kBlk + threadIdx.x;
    if (i < n) {
      uint32_t pos = atomicAdd(&lh[key[k]], 1u);
      if (pos < (uint64_t)n) {  // always true for a consistent histogram; keeps writes in bounds
        for (int r = 0; r < 6; ++r) B[r * n + pos] = A[r * n + i];
        if (idA) idB[pos] = idA[i];
      }
    }
  }
}

// Ranking of one block of kItems particles as in the direct form, writing only the source
// index of each slot: perm[slot] = i.  Only for a tile whose ranks overflowed the packed keys.
__device__ __forceinline__ void rank_again_body(const uint32_t* __restrict__ keys, uint32_t kmask,
                                                int64_t n, int ntiles,
                                                uint32_t* __restrict__ cursor,
                                                uint32_t* __restrict__ perm, int blk) {
  __shared__ uint32_t lh[kMaxTiles];
  for (int t = threadIdx.x; t < ntiles; t += kBlk) lh[t] = 0u;
  __syncthreads();
  const int64_t base = (int64_t)blk * kItems;
  // all of the thread's keys are loaded before the first (wave-uniform, branching) histogram
  // add, so that the loads overlap instead of each waiting behind the previous add
  uint32_t key[kPer];
  for (int k = 0; k < kPer; ++k) {
    int64_t i = base + k * kBlk + threadIdx.x;
    key[k] = i < n ? keys[i] & kmask : 0u;
  }
  for (int k = 0; k < kPer; ++k)
    (void)wave_aggregated_add(lh, key[k], base + k * kBlk + threadIdx.x < n);
  __syncthreads();
  for (int t = threadIdx.x; t < ntiles; t += kBlk)
    if (lh[t]) lh[t] = atomicAdd(&cursor[t], lh[t]);
  __syncthreads();
  for (int k = 0; k < kPer; ++k) {
    int64_t i = base + k * kBlk + threadIdx.x;
    const uint32_t pos = wave_aggregated_add(lh, key[k], i < n);
    // in bounds for a consistent histogram
    if (i < n && pos < (uint64_t)n) perm[pos] = (uint32_t)i;
  }
}

// The source index of every sorted slot from the packed keys, PER particles per thread:
// perm[cursor[key] + rank] = i.  PER < kPer only where no tile can overflow (n < 2^20).
template <int PER>
__device__ __forceinline__ void place_body(const uint32_t* __restrict__ keys,
                                           const Geom* __restrict__ g, int64_t n,
                                           const SortPlan& sp, uint32_t* __restrict__ cursor,
                                           const uint32_t* __restrict__ nchunks,
                                           uint32_t* __restrict__ perm, int blk) {
  if (g->status) return;
  const uint32_t kmask = key_mask(sp);
  if constexpr (PER == kPer)
    if (nchunks[kOverflow]) {
      rank_again_body(keys, kmask, n, sp.ntiles, cursor, perm, blk);
      return;
    }
  const int64_t base = (int64_t)blk * (kBlk * PER) + threadIdx.x;
  uint32_t k[PER], pos[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) k[q] = keys[min(base + q * kBlk, n - 1)];
#pragma unroll
  for (int q = 0; q < PER; ++q) pos[q] = cursor[k[q] & kmask] + (k[q] >> sp.kbits);
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int64_t i = base + q * kBlk;
    // in bounds for a consistent histogram
    if (i < n && pos[q] < (uint64_t)n) perm[pos[q]] = (uint32_t)i;
  }
}

template <int PER>
__global__ __launch_bounds__(kBlk) void k_place(const uint32_t* __restrict__ keys,
                                                const Geom* __restrict__ g, int64_t n,
                                                SortPlan sp, uint32_t* __restrict__ cursor,
                                                const uint32_t* __restrict__ nchunks,
                                                uint32_t* __restrict__ perm) {
  place_body<PER>(keys, g, n, sp, cursor, nchunks, perm, blockIdx.x);
}

template <bool STAGED>
__device__ __forceinline__ void scatter_body(const double* __restrict__ A,
                                             const uint32_t* __restrict__ idA,
                                             const uint32_t* __restrict__ keys, uint32_t kmask,
                                             const Geom* __restrict__ g, int64_t n, int ntiles,
                                             uint32_t* __restrict__ cursor, double* __restrict__ B,
                                             uint32_t* __restrict__ idB, int blk, int nblk) {
  if constexpr (STAGED)
    scatter_staged_body(A, idA, keys, kmask, g, n, ntiles, cursor, B, idB, blk, nblk);
  else
    scatter_direct_body(A, idA, keys, kmask, g, n, ntiles, cursor, B, idB, blk, nblk);
}

template <bool STAGED>
__global__ __launch_bounds__(kBlk) void k_scatter(const double* __restrict__ A,
                                                  const uint32_t* __restrict__ idA,
                                                  const uint32_t* __restrict__ keys,
                                                  uint32_t kmask,
                                                  const Geom* __restrict__ g, int64_t n,
                                                  int ntiles, uint32_t* __restrict__ cursor,
                                                  double* __restrict__ B,
                                                  uint32_t* __restrict__ idB) {
  scatter_body<STAGED>(A, idA, keys, kmask, g, n, ntiles, cursor, B, idB, blockIdx.x, gridDim.x);
}

// The staged scatter over wide blocks, for inputs whose order is unrelated to the keys (the
// caller's order on a call's first step, the id buckets of the final reordering).  A block of
// kWBlk threads takes kWItems particles, four times the items of k_scatter<true>, so that every
// key's run in the output is four times longer (at 2048 tiles about 8 particles, 64 B per row,
// instead of 2): the runs' writes then fill whole 64-byte pieces of memory instead of a
// fraction of one.  The ranking is that of the staged form; the rows then move through a
// kWHalf-slot LDS buffer in two halves of the ranked slots, each item's value read from HBM in
// the half its slot falls in.
constexpr int kWBlk = 1024;
constexpr int kWPer = 16;
constexpr int kWItems = kWBlk * kWPer;  // 16384
constexpr int kWHalf = kWItems / 2;     // slots staged per pass

__global__ __launch_bounds__(kWBlk) void k_scatter_wide(const double* __restrict__ A,
                                                        const uint32_t* __restrict__ idA,
                                                        const uint32_t* __restrict__ keys,
                                                        uint32_t kmask,
                                                        const Geom* __restrict__ g, int64_t n,
                                                        int ntiles, uint32_t* __restrict__ cursor,
                                                        double* __restrict__ B,
                                                        uint32_t* __restrict__ idB) {
  // cur/delta (ranking, 2 x kMaxTiles words) and the row buffer (kWHalf doubles) share storage
  __shared__ __align__(16) unsigned char stage[kWHalf * sizeof(double)];
  __shared__ uint32_t dest[kWItems];
  static_assert(2 * kMaxTiles * sizeof(uint32_t) <= sizeof(stage), "ranking exceeds storage");
  uint32_t* cur = reinterpret_cast<uint32_t*>(stage);
  uint32_t* delta = cur + kMaxTiles;
  double* rowbuf = reinterpret_cast<double*>(stage);
  uint32_t* idbuf = reinterpret_cast<uint32_t*>(stage);
  if (g->status) return;
  const int64_t base = (int64_t)blockIdx.x * kWItems;
  const int m = (int)min((int64_t)kWItems, n - base);
  for (int t = threadIdx.x; t < ntiles; t += kWBlk) cur[t] = 0u;
  __syncthreads();
  uint32_t key[kWPer];
  for (int k = 0; k < kWPer; ++k) {
    const int l = k * kWBlk + threadIdx.x;
    key[k] = l < m ? keys[base + l] & kmask : 0u;
  }
  for (int k = 0; k < kWPer; ++k)
    if (k * kWBlk + (int)threadIdx.x < m) atomicAdd(&cur[key[k]], 1u);
  __syncthreads();
  // reserve each present key's run in the output
  for (int t = threadIdx.x; t < ntiles; t += kWBlk) {
    const uint32_t c = cur[t];
    delta[t] = c ? atomicAdd(&cursor[t], c) : 0u;
  }
  __syncthreads();
  block_exclusive_scan_lds<kWBlk>(cur, ntiles);  // cur[t] = local offset of key t
  for (int t = threadIdx.x; t < ntiles; t += kWBlk) delta[t] -= cur[t];
  __syncthreads();
  uint32_t slot[kWPer];
  for (int k = 0; k < kWPer; ++k) {
    const int l = k * kWBlk + threadIdx.x;
    slot[k] = 0u;
    if (l < m) {
      slot[k] = atomicAdd(&cur[key[k]], 1u);
      dest[slot[k]] = delta[key[k]] + slot[k];
    }
  }
  __syncthreads();  // the ranking's words are dead from here: the row buffer takes them over
  const int rows = idA ? 7 : 6;  // the ids travel as a seventh row when there are any
  for (int r = 0; r < rows; ++r) {
    for (int h = 0; h < 2; ++h) {
      const uint32_t lo = (uint32_t)(h * kWHalf);
      for (int k = 0; k < kWPer; ++k) {
        const int l = k * kWBlk + threadIdx.x;
        if (l < m && slot[k] - lo < (uint32_t)kWHalf) {
          if (r < 6)
            rowbuf[slot[k] - lo] = A[r * n + base + l];
          else
            idbuf[slot[k] - lo] = idA[base + l];
        }
      }
      __syncthreads();
      const int cnt = min(kWHalf, m - (int)lo);
      for (int q = threadIdx.x; q < cnt; q += kWBlk) {
        const uint32_t d = dest[lo + q];
        if (d < (uint64_t)n) {  // always true for a consistent histogram; keeps writes in bounds
          if (r < 6)
            B[r * n + d] = rowbuf[q];
          else
            idB[d] = idbuf[q];
        }
      }
      __syncthreads();
    }
  }
}

template <typename T>
__device__ __forceinline__ void add_global(T* p, T v) {
  unsafeAtomicAdd(p, v);
}

// Charge of one chunk in its tile's (T + S)^3 window, accumulated in LDS as 64-bit fixed point:
// every contribution q_m w is scaled by a power of two 2^k chosen from the whole charge of the
// chunk's tile, |q_m| * count_tile 2^k <= 2^62 (no overflow in any node, whatever the order;
// the same k for all chunks of the tile), with a single contribution below 2^50, rounded to
// the nearest integer (error below 2^-(k+1) |q_m|) and added with integer LDS atomics, which
// are exact, so the window sum does not depend on the order of the lanes.  Integer LDS atomics
// also run faster here than floating-point ones (1.13 ms against 1.85 ms with float64 and 13 ms
// with float32 atomics for 1e8 TSC particles on MI355X).  The non-zero window entries are then
// added, still as integers, to the tile's own window in tacc (tacc[t nw + w], one 64-bit
// integer atomic each, exact in any order); the tile's exponent goes to tscale[t], and
// k_tile_reduce forms the grid, which then depends neither on the order of the particles nor
// on that of the atomics.
template <int S, bool PERM>
__device__ __forceinline__ void deposit_tiles_body(const double* __restrict__ B,
                                                        const uint32_t* __restrict__ perm,
                                                        const Geom* __restrict__ g, Consts c,
                                                        SortPlan sp,
                                                        const int4* __restrict__ chunks,
                                                        const uint32_t* __restrict__ nchunks,
                                                        int blk, int nblk,
                                                        unsigned long long* __restrict__ tacc,
                                                        int* __restrict__ tscale) {
  extern __shared__ unsigned char smem_raw[];
  unsigned long long* win = reinterpret_cast<unsigned long long*>(smem_raw);
  if (g->status) return;
  const double o[3] = {g->origin[0], g->origin[1], g->origin[2]};
  const double ih[3] = {g->inv_h[0], g->inv_h[1], g->inv_h[2]};
  const int Wx = sp.T[0] + S, Wy = sp.T[1] + S, Wz = sp.T[2] + S;
  const int nw = Wx * Wy * Wz;
  int rowoff[S + 1][S + 1];  // window offset of stencil row (a, b)
  for (int a = 0; a <= S; ++a)
    for (int b = 0; b <= S; ++b) rowoff[a][b] = (a * Wy + b) * Wx;
  const int64_t n = c.n;
  bool bin_fault = false;
  const uint32_t nck = *nchunks;
  for (uint32_t ci = blk; ci < nck; ci += nblk) {
    const int4 ch = chunks[ci];
    const int t = ch.x;
    const int tx = t % sp.NT[0], ty = (t / sp.NT[0]) % sp.NT[1], tz = t / (sp.NT[0] * sp.NT[1]);
    const int ox = tx * sp.T[0], oy = ty * sp.T[1], oz = tz * sp.T[2];
    // scale 2^k with |q_m| * count * 2^k <= 2^62 (no node overflows) and |q_m| 2^k <= 2^50
    // (every scaled contribution converts exactly below); a zero charge gives zero
    const double qa = fabs(c.q_macro);
    const double qc = qa * (double)ch.w;  // the tile's particle count
    const int k = qc > 0.0 ? min(62 - max(ilogb(qc) + 1, -960), 50 - max(ilogb(qa) + 1, -960)) : 0;
    const double qs = c.q_macro * ldexp(1.0, k);
    if (threadIdx.x == 0) tscale[t] = k;  // every chunk of the tile writes the same k
    for (int w = threadIdx.x; w < nw; w += (int)blockDim.x) win[w] = 0ull;
    __syncthreads();
    // Software-pipelined over the lane's slots i, i + stride, ... in pairs (a, b): before the
    // atomics of one slot the positions of the lane's next slot and the index of the slot after
    // that are loaded.  No branch surrounds these loads (slot indices are clamped into the chunk
    // and particle indices into [0, n), and a result is used only where it is valid), so the
    // waits for them fall at their first use and they stay in flight during the LDS atomics; a
    // load inside a branch makes the join wait for every load the wave has issued.  Slot i
    // holds particle perm[i] of B (B itself in slot order without a permutation); an index past
    // n, impossible for a consistent ranking, is flagged and its particle skipped.
    const int64_t stride = (int)blockDim.x;
    const int64_t last = ch.z - 1;  // a work item holds at least one slot
    auto index_of = [&](int64_t j) -> int64_t {
      j = j < last ? j : last;
      if constexpr (PERM) return (int64_t)perm[j];
      return j;
    };
    auto load_pos = [&](int64_t r, double* p) {
      const int64_t q = r < n ? r : 0;
      p[0] = B[q];
      p[1] = B[2 * n + q];
      p[2] = B[4 * n + q];
    };
    auto deposit_one = [&](const double* p, int64_t r) {
      const bool valid = r < n;
      if (!valid) bin_fault = true;
      double wx[S + 1], wy[S + 1], wz[S + 1];
      const int bx = stencil<S>((p[0] - o[0]) * ih[0], c.nx, wx);
      const int by = stencil<S>((p[1] - o[1]) * ih[1], c.ny, wy);
      const int bz = stencil<S>((p[2] - o[2]) * ih[2], c.nz, wz);
      const int lx = bx - ox, ly = by - oy, lz = bz - oz;
      const bool inside = lx >= 0 && lx < sp.T[0] && ly >= 0 && ly < sp.T[1] && lz >= 0 &&
                          lz < sp.T[2];
      // the binning put the particle in the chunk's tile with this very stencil function, so
      // its stencil lies in the window; a violation is a library fault, flagged as the
      // gather-kick flags it (PIC_EINTERNAL), and the particle is not deposited
      if (valid && !inside) bin_fault = true;
      if (valid && inside) {
        // q_m 2^k w rounded to the nearest integer by one fused multiply-add with 1.5 2^52
        // (the sum then has the integer in its low mantissa bits, |value| < 2^51), read back
        // as a two's-complement int64 by subtracting the constant's bit pattern
        constexpr double kMagic = 6755399441055744.0;  // 1.5 * 2^52
        constexpr unsigned long long kMagicBits = 0x4338000000000000ull;
        unsigned long long* w0 = win + (lz * Wy + ly) * Wx + lx;
        for (int a = 0; a <= S; ++a) {
          const double wzs = qs * wz[a];
          for (int b = 0; b <= S; ++b) {
            const double wzy = wzs * wy[b];
            unsigned long long* row = w0 + rowoff[a][b];
            for (int q = 0; q <= S; ++q) {
              const double d = __builtin_fma(wzy, wx[q], kMagic);
              atomicAdd(row + q, (unsigned long long)__double_as_longlong(d) - kMagicBits);
            }
          }
        }
      }
    };
    int64_t i = ch.y + threadIdx.x;
    int64_t ra = index_of(i), rb = index_of(i + stride);
    double pa[3], pb[3];
    load_pos(ra, pa);
    for (; i < ch.z; i += 2 * stride) {
      const int64_t ra2 = index_of(i + 2 * stride);
      load_pos(rb, pb);
      deposit_one(pa, ra);  // slot i
      const int64_t rb2 = index_of(i + 3 * stride);
      load_pos(ra2, pa);
      if (i + stride < ch.z) deposit_one(pb, rb);  // slot i + stride
      ra = ra2;
      rb = rb2;
    }
    __syncthreads();
    for (int w = threadIdx.x; w < nw; w += (int)blockDim.x) {
      const long long v = (long long)win[w];
      int wx_ = w % Wx, wy_ = (w / Wx) % Wy, wz_ = w / (Wx * Wy);
      int gx = ox + wx_, gy = oy + wy_, gz = oz + wz_;
      if (v != 0 && gx < c.nx && gy < c.ny && gz < c.nz)
        atomicAdd(&tacc[(int64_t)t * nw + w], (unsigned long long)v);
    }
    __syncthreads();
  }
  if (bin_fault) atomicCAS(const_cast<int*>(&g->status), 0, -7);
}

// The charge grid from the tiles' integer windows: every node sums, in ascending tile order
// (z, then y, then x), the windows of the tiles that cover it, each scaled back by its tile's
// 2^-k, and clears the entries it read, so that tacc is zero again for the next step (entries
// outside the grid are never written).  Every node is written (zero after a device error), so
// the grid needs no clearing pass.
template <int S, typename T>
__device__ __forceinline__ void tile_reduce_body(const Geom* __restrict__ g, Consts c,
                                                 SortPlan sp,
                                                 unsigned long long* __restrict__ tacc,
                                                 const int* __restrict__ tscale,
                                                 T* __restrict__ rho, int blk, int nblk) {
  const bool err = g->status != 0;
  const int Wx = sp.T[0] + S, Wy = sp.T[1] + S, Wz = sp.T[2] + S;
  const int64_t nw = (int64_t)Wx * Wy * Wz;
  const int64_t total = (int64_t)c.nx * c.ny * c.nz;
  for (int64_t node = blk * 256ll + threadIdx.x; node < total; node += (int64_t)nblk * 256) {
    const Idx3 g3 = split3(node, c.nx, c.ny);
    const int gx = g3.x, gy = g3.y, gz = g3.z;
    const int p[3] = {gx, gy, gz};
    int lo[3], hi[3];
    for (int a = 0; a < 3; ++a) {  // tiles whose window [t T, t T + T + S) holds p[a]
      hi[a] = min(p[a] / sp.T[a], sp.NT[a] - 1);
      lo[a] = hi[a];
      while (lo[a] > 0 && (lo[a] - 1) * sp.T[a] + sp.T[a] + S > p[a]) --lo[a];
    }
    double val = 0.0;
    if (err) {
      rho[node] = T(0);
      continue;
    }
    for (int tz = lo[2]; tz <= hi[2]; ++tz)
      for (int ty = lo[1]; ty <= hi[1]; ++ty)
        for (int tx = lo[0]; tx <= hi[0]; ++tx) {
          const int t = (tz * sp.NT[1] + ty) * sp.NT[0] + tx;
          const int64_t w = ((int64_t)(gz - tz * sp.T[2]) * Wy + (gy - ty * sp.T[1])) * Wx +
                            (gx - tx * sp.T[0]);
          unsigned long long* e = &tacc[t * nw + w];
          const long long v = (long long)*e;
          if (v != 0) {
            val += ldexp((double)v, -tscale[t]);
            *e = 0ull;
          }
        }
    rho[node] = (T)val;
  }
}

template <int S, typename T>
__global__ __launch_bounds__(256) void k_tile_reduce(const Geom* __restrict__ g, Consts c,
                                                     SortPlan sp,
                                                     unsigned long long* __restrict__ tacc,
                                                     const int* __restrict__ tscale,
                                                     T* __restrict__ rho) {
  tile_reduce_body<S, T>(g, c, sp, tacc, tscale, rho, blockIdx.x, gridDim.x);
}

// Vector deposit e_c(node) = sum_i W(r_i - node) a_c,i of the records, read through their ranking
// perm (the reverse sweep's transposed gather), one chunk per workgroup: three
// float64 LDS windows (the values have both signs), flushed with global atomics.
template <int S, typename T>
__device__ __forceinline__ void vdeposit_tiles_body(const AdjRecord* __restrict__ recs,
                                                    const uint32_t* __restrict__ perm,
                                                    const Geom* __restrict__ g, Consts c,
                                                    SortPlan sp,
                                                    const int4* __restrict__ chunks,
                                                    const uint32_t* __restrict__ nchunks,
                                                    T* __restrict__ e, int blk, int nblk) {
  extern __shared__ unsigned char smem_raw[];
  double* win = reinterpret_cast<double*>(smem_raw);
  if (g->status) return;
  const double o[3] = {g->origin[0], g->origin[1], g->origin[2]};
  const double ih[3] = {g->inv_h[0], g->inv_h[1], g->inv_h[2]};
  const int Wx = sp.T[0] + S, Wy = sp.T[1] + S, Wz = sp.T[2] + S;
  const int nw = Wx * Wy * Wz;
  const int64_t ng = (int64_t)c.nx * c.ny * c.nz;
  const uint32_t nck = *nchunks;
  for (uint32_t ci = blk; ci < nck; ci += nblk) {
    const int4 ch = chunks[ci];
    const int t = ch.x;
    const int tx = t % sp.NT[0], ty = (t / sp.NT[0]) % sp.NT[1], tz = t / (sp.NT[0] * sp.NT[1]);
    const int ox = tx * sp.T[0], oy = ty * sp.T[1], oz = tz * sp.T[2];
    for (int w = threadIdx.x; w < 3 * nw; w += (int)blockDim.x) win[w] = 0.0;
    __syncthreads();
    for (int64_t slot = ch.y + threadIdx.x; slot < ch.z; slot += (int)blockDim.x) {
      const AdjRecord p = recs[perm[slot]];
      const double* v = p.a;
      double wx[S + 1], wy[S + 1], wz[S + 1];
      const int bx = stencil<S>((p.r[0] - o[0]) * ih[0], c.nx, wx);
      const int by = stencil<S>((p.r[1] - o[1]) * ih[1], c.ny, wy);
      const int bz = stencil<S>((p.r[2] - o[2]) * ih[2], c.nz, wz);
      const int lx = bx - ox, ly = by - oy, lz = bz - oz;
      const bool inside = lx >= 0 && lx < sp.T[0] && ly >= 0 && ly < sp.T[1] && lz >= 0 &&
                          lz < sp.T[2];
      for (int a = 0; a <= S; ++a)
        for (int b = 0; b <= S; ++b) {
          const double wzy = wz[a] * wy[b];
          for (int q = 0; q <= S; ++q) {
            const double w = wzy * wx[q];
            if (inside) {
              const int idx = ((lz + a) * Wy + (ly + b)) * Wx + (lx + q);
              for (int comp = 0; comp < 3; ++comp) atomicAdd(&win[comp * nw + idx], w * v[comp]);
            } else {
              const int64_t node = ((int64_t)(bz + a) * c.ny + (by + b)) * c.nx + (bx + q);
              for (int comp = 0; comp < 3; ++comp) add_global(&e[comp * ng + node], (T)(w * v[comp]));
            }
          }
        }
    }
    __syncthreads();
    for (int w = threadIdx.x; w < nw; w += (int)blockDim.x) {
      const int wx_ = w % Wx, wy_ = (w / Wx) % Wy, wz_ = w / (Wx * Wy);
      const int gx = ox + wx_, gy = oy + wy_, gz = oz + wz_;
      if (gx < c.nx && gy < c.ny && gz < c.nz) {
        const int64_t node = ((int64_t)gz * c.ny + gy) * c.nx + gx;
        for (int comp = 0; comp < 3; ++comp) {
          const double v = win[comp * nw + w];
          if (v != 0.0) add_global(&e[comp * ng + node], (T)v);
        }
      }
    }
    __syncthreads();
  }
}

template <int S, typename T>
__global__ __launch_bounds__(kMaxThreads) void k_vdeposit_tiles(const AdjRecord* __restrict__ recs,
                                                         const uint32_t* __restrict__ perm,
                                                         const Geom* __restrict__ g, Consts c,
                                                         SortPlan sp,
                                                         const int4* __restrict__ chunks,
                                                         const uint32_t* __restrict__ nchunks,
                                                         T* __restrict__ e) {
  vdeposit_tiles_body<S, T>(recs, perm, g, c, sp, chunks, nchunks, e, blockIdx.x, gridDim.x);
}

template <int S>
__global__ __launch_bounds__(kMaxThreads) void k_deposit_tiles(const double* __restrict__ B,
                                                        const uint32_t* __restrict__ perm,
                                                        const Geom* __restrict__ g, Consts c,
                                                        SortPlan sp,
                                                        const int4* __restrict__ chunks,
                                                        const uint32_t* __restrict__ nchunks,
                                                        unsigned long long* __restrict__ tacc,
                                                        int* __restrict__ tscale) {
  // the permutation's presence as a template argument: a uniform branch around its loads
  // inside the loop would make the join wait for all of the wave's loads
  if (perm)
    deposit_tiles_body<S, true>(B, perm, g, c, sp, chunks, nchunks, blockIdx.x, gridDim.x, tacc,
                                tscale);
  else
    deposit_tiles_body<S, false>(B, nullptr, g, c, sp, chunks, nchunks, blockIdx.x, gridDim.x,
                                 tacc, tscale);
}

// Fused second half of step j and first half of step j+1 on the sorted array, one chunk per
// workgroup: the (T + S)^3 window of E' around the chunk's tile is staged in LDS (coalesced
// rows), the particles gather from LDS, get the space-charge kick over L and the slice's second
// half map, then (has_next) the next slice's first half map (without DIAG the two as one
// product), and the box of the new positions is accumulated.  PERM false: B is in slot order and updated in place.  PERM true: slot i
// reads particle perm[i] of src (and its id) and writes the new state to slot i of B, so B
// leaves in sorted order.  The gather reads LDS only (a per-lane choice between LDS and global memory
// compiles to flat loads, which go through the vector memory pipeline); a stencil outside the
// window, impossible for a consistent binning, sets status -7 (PIC_EINTERNAL).
// PERM with a next step and no DIAG: the chunk's slots [begin, end) are refilled from both
// ends, the particles whose next kick-point position lies in the same tile of the current grid
// from the bottom and the others from the top (one LDS atomic per wavefront and end), so that
// the particles likely to change tile next step lie together in a short stretch of the order:
// neighbouring tiles then read them through the next permutation from fewer cache lines.
// DIAG: the particles' state at the end of the step (after the second half map, before the
// next first half map) is also summed into the moment accumulators diag_part[q kDiagSlots + ...]:
// 6 sums of d = v - shift and the 21 products d_a d_b (a <= b, row-major), with the
// 6-double shift read from diag_shift (close to the mean, so that the centred moments formed
// from these sums lose no digits).
template <int S, typename T, bool PERM, bool DIAG = false>
__device__ __forceinline__ void gkd_tiles_body(double* __restrict__ B,
                                                    const double* __restrict__ src,
                                                    const uint32_t* __restrict__ perm,
                                                    const uint32_t* __restrict__ idsrc,
                                                    uint32_t* __restrict__ iddst,
                                                    Geom* g, const T* __restrict__ E,
                                                    const T* __restrict__ phi, const Consts& c,
                                                    SortPlan sp,
                                                    const int4* __restrict__ chunks,
                                                    const uint32_t* __restrict__ nchunks,
                                                    double L, const HalfMap& second,
                                                    int has_next, const HalfMap& first_next,
                                                    Box* box, int blk, int nblk,
                                                    double* __restrict__ diag_part = nullptr,
                                                    const double* __restrict__ diag_shift = nullptr) {
  extern __shared__ unsigned char smem_raw[];
  __shared__ uint32_t s_up, s_down;  // the next free slot from either end of the chunk
  T* win = reinterpret_cast<T*>(smem_raw);
  if (g->status) return;
  const bool reorder = PERM && !DIAG && has_next;  // with DIAG it cost more time than it saved
  double sh[6], acc[DIAG ? kMomentSlots : 1];
  if constexpr (DIAG) {
    for (int r = 0; r < 6; ++r) sh[r] = diag_shift[r];
    for (int q = 0; q < kMomentSlots; ++q) acc[q] = 0.0;
  }
  // Without the moment sums, the slice's second half map and the next slice's first act back
  // to back on the kicked state: they are applied as their product (one matrix per plane, the
  // longitudinal coefficients summed), the same linear map in half the arithmetic and with few
  // enough uniform values to stay in scalar registers.
  // With the moment sums the two maps stay apart (the sums are taken between them), each in
  // matrix form.
  HalfMap maps, next_map;
  if constexpr (!DIAG) {
    maps = half_product(second, first_next, has_next != 0);
  } else {
    maps = half_product(second, second, false);
    next_map = half_product(first_next, first_next, false);
  }
  const double o[3] = {g->origin[0], g->origin[1], g->origin[2]};
  const double ih[3] = {g->inv_h[0], g->inv_h[1], g->inv_h[2]};
  T dif[3];  // 1/(2h) of the centred differences
  for (int a = 0; a < 3; ++a) dif[a] = (T)(1.0 / (2.0 * g->h_rest[a]));
  const int Wx = sp.T[0] + S, Wy = sp.T[1] + S, Wz = sp.T[2] + S;
  const int nw = Wx * Wy * Wz;
  int rowoff[S + 1][S + 1];  // window offset of stencil row (a, b)
  for (int a = 0; a <= S; ++a)
    for (int b = 0; b <= S; ++b) rowoff[a][b] = (a * Wy + b) * Wx;
  const int64_t n = c.n;
  const int64_t plane = (int64_t)c.nx * c.ny * c.nz;
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  bool bad = false, bin_fault = false;
  // the thread's first window entry and the block size, both split into (x, y, z) offsets
  const int w0x = (int)threadIdx.x % Wx, w0y = ((int)threadIdx.x / Wx) % Wy,
            w0z = (int)threadIdx.x / (Wx * Wy);
  const int stx = (int)blockDim.x % Wx, sty = ((int)blockDim.x / Wx) % Wy,
            stz = (int)blockDim.x / (Wx * Wy);
  const uint32_t nck = *nchunks;
  for (uint32_t ci = blk; ci < nck; ci += nblk) {
    const int4 ch = chunks[ci];
    const int t = ch.x;
    const int tx = t % sp.NT[0], ty = (t / sp.NT[0]) % sp.NT[1], tz = t / (sp.NT[0] * sp.NT[1]);
    const int ox = tx * sp.T[0], oy = ty * sp.T[1], oz = tz * sp.T[2];
    __syncthreads();  // the previous chunk's readers are done with the window and counters
    if (reorder && threadIdx.x == 0) {
      s_up = (uint32_t)ch.y;
      s_down = (uint32_t)ch.z;
    }
    // window entry w = (wz_ Wy + wy_) Wx + wx_, stepped by the block size with carries
    int wx_ = w0x, wy_ = w0y, wz_ = w0z;
    for (int w = threadIdx.x; w < nw; w += (int)blockDim.x) {
      int gx = ox + wx_, gy = oy + wy_, gz = oz + wz_;
      bool in = gx < c.nx && gy < c.ny && gz < c.nz;
      int64_t gi = ((int64_t)gz * c.ny + gy) * c.nx + gx;
      if (phi) {  // the centred differences of grad_body
        T e0 = 0, e1 = 0, e2 = 0;
        if (in) {
          const T* p = phi + ((int64_t)(gz + 1) * (c.ny + 2) + (gy + 1)) * (c.nx + 2) + (gx + 1);
          const int64_t sy = c.nx + 2, sz = sy * (c.ny + 2);
          e0 = -(p[1] - p[-1]) * dif[0];
          e1 = -(p[sy] - p[-sy]) * dif[1];
          e2 = -(p[sz] - p[-sz]) * dif[2];
        }
        win[w] = e0;
        win[nw + w] = e1;
        win[2 * nw + w] = e2;
      } else {
        win[w] = in ? E[gi] : T(0);
        win[nw + w] = in ? E[plane + gi] : T(0);
        win[2 * nw + w] = in ? E[2 * plane + gi] : T(0);
      }
      wx_ += stx;
      const int cx = wx_ >= Wx;
      wx_ -= cx ? Wx : 0;
      wy_ += sty + cx;
      const int cy = wy_ >= Wy;
      wy_ -= cy ? Wy : 0;
      wz_ += stz + cy;
    }
    __syncthreads();
    // every thread of the block runs the same number of rounds (the wavefront-wide slot
    // assignment below needs all lanes); lanes past the chunk's end are inactive
    for (int64_t ib = ch.y; ib < ch.z; ib += (int)blockDim.x) {
      const int64_t i = ib + threadIdx.x;
      const bool act = i < ch.z;
      double v[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
      int64_t i0 = i;
      if (act) {
        if constexpr (PERM) {
          i0 = perm[i];
          if (i0 >= n) {  // impossible for a consistent ranking; keeps the reads in bounds
            bin_fault = true;
            i0 = 0;
          }
          for (int r = 0; r < 6; ++r) v[r] = src[r * n + i0];
        } else {
          for (int r = 0; r < 6; ++r) v[r] = B[r * n + i];
        }
        double wx[S + 1], wy[S + 1], wz[S + 1];
        const int bx = stencil<S>((v[0] - o[0]) * ih[0], c.nx, wx);
        const int by = stencil<S>((v[2] - o[1]) * ih[1], c.ny, wy);
        const int bz = stencil<S>((v[4] - o[2]) * ih[2], c.nz, wz);
        // the binning put this particle in the chunk's tile, so its stencil lies in the window;
        // a violation is a library fault: flagged, and the indices clamped to stay in bounds
        int lx = bx - ox, ly = by - oy, lz = bz - oz;
        if (lx < 0 || lx >= sp.T[0] || ly < 0 || ly >= sp.T[1] || lz < 0 || lz >= sp.T[2]) {
          bin_fault = true;
          lx = min(max(lx, 0), sp.T[0] - 1);
          ly = min(max(ly, 0), sp.T[1] - 1);
          lz = min(max(lz, 0), sp.T[2] - 1);
        }
        T ex = 0, ey = 0, ez = 0;
        const T* w0 = win + (lz * Wy + ly) * Wx + lx;
        for (int a = 0; a <= S; ++a)
          for (int b = 0; b <= S; ++b) {
            const double wzy = wz[a] * wy[b];
            const T* row = w0 + rowoff[a][b];
            for (int q = 0; q <= S; ++q) {
              const T w = (T)(wzy * wx[q]);
              ex += w * row[q];
              ey += w * row[nw + q];
              ez += w * row[2 * nw + q];
            }
          }
        v[1] = v[1] + c.C * (double)ex * L;
        v[3] = v[3] + c.C * (double)ey * L;
        v[5] = v[5] + c.gamma * c.C * (double)ez * L;
        if constexpr (DIAG) {
          apply_matrix(maps, v, c.inv_gamma2);
          double d[6];
          for (int r = 0; r < 6; ++r) {
            d[r] = v[r] - sh[r];
            acc[r] += d[r];
          }
          int q = 6;
          for (int a = 0; a < 6; ++a)
            for (int b = a; b < 6; ++b) acc[q++] += d[a] * d[b];
          if (has_next) apply_matrix(next_map, v, c.inv_gamma2);
        } else {
          apply_matrix(maps, v, c.inv_gamma2);
        }
        if (has_next) {
          const double p[3] = {v[0], v[2], v[4]};
          for (int a = 0; a < 3; ++a) {
            bad |= !isfinite(p[a]);
            lo[a] = fmin(lo[a], p[a]);
            hi[a] = fmax(hi[a], p[a]);
          }
        }
      }
      int64_t slot = i;
      if (reorder) {
        // the particle keeps tile t when its new stencil base lies in t's node range: the same
        // test as tile_key(...) == t, without the divisions
        bool stay = false;
        if (act) {
          const int nx_ = base_node<S>((v[0] - o[0]) * ih[0], c.nx) - ox;
          const int ny_ = base_node<S>((v[2] - o[1]) * ih[1], c.ny) - oy;
          const int nz_ = base_node<S>((v[4] - o[2]) * ih[2], c.nz) - oz;
          stay = (unsigned)nx_ < (unsigned)sp.T[0] && (unsigned)ny_ < (unsigned)sp.T[1] &&
                 (unsigned)nz_ < (unsigned)sp.T[2];
        }
        const uint64_t m_s = __ballot(stay), m_m = __ballot(act && !stay);
        const int lane = (int)__lane_id();
        const uint64_t below = (1ull << lane) - 1ull;
        uint32_t b_s = 0u, b_m = 0u;
        if (lane == 0) {
          if (m_s) b_s = atomicAdd(&s_up, (uint32_t)__popcll(m_s));
          if (m_m) b_m = atomicSub(&s_down, (uint32_t)__popcll(m_m));
        }
        b_s = __shfl(b_s, 0);
        b_m = __shfl(b_m, 0);
        slot = stay ? (int64_t)b_s + __popcll(m_s & below)
                    : (int64_t)b_m - __popcll(m_m) + __popcll(m_m & below);
        if (act && (slot < ch.y || slot >= ch.z)) {  // impossible: the two ends tile the chunk
          bin_fault = true;
          slot = i;
        }
      }
      if (act) {
        for (int r = 0; r < 6; ++r) B[r * n + slot] = v[r];
        if constexpr (PERM)
          if (iddst) iddst[slot] = idsrc[i0];
      }
    }
  }
  if (bin_fault) atomicCAS(const_cast<int*>(&g->status), 0, -7);
  if (has_next) box_geometry_block(lo, hi, bad, box, g, c, nblk);
  if constexpr (DIAG) {
    // wave sums, then the waves' sums through LDS (the window is free after the barrier; the
    // launch gives at least kMaxThreads / 64 * 27 doubles)
    for (int q = 0; q < kMomentSlots; ++q)
      for (int off = 32; off > 0; off >>= 1) acc[q] += __shfl_xor(acc[q], off);
    double* red = reinterpret_cast<double*>(smem_raw);
    const int wave = threadIdx.x >> 6, nwave = (int)(blockDim.x + 63) >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0)
      for (int q = 0; q < kMomentSlots; ++q) red[wave * kMomentSlots + q] = acc[q];
    __syncthreads();
    // the blocks' sums go to kDiagSlots accumulators (zero between launches), which k_diag_combine
    // sums: one partial per block took it 16 us of a 154 us step of 1e5 particles
    if (threadIdx.x < kMomentSlots) {
      double t = 0.0;
      for (int w = 0; w < nwave; ++w) t += red[w * kMomentSlots + threadIdx.x];
      unsafeAtomicAdd(&diag_part[threadIdx.x * kDiagSlots + blk % kDiagSlots], t);
    }
  }
}

// With DIAG the 27 moment sums stay in registers beside the particle's state: the kernel is
// built for at most kDiagThreads lanes per workgroup, which doubles the registers a lane may
// hold and keeps the sums out of scratch memory.
constexpr int kDiagThreads = 512;

template <int S, typename T, bool PERM, bool DIAG>
__global__ __launch_bounds__(DIAG ? kDiagThreads : kMaxThreads) void k_gkd_tiles(double* __restrict__ B,
                                                    const double* __restrict__ src,
                                                    const uint32_t* __restrict__ perm,
                                                    const uint32_t* __restrict__ idsrc,
                                                    uint32_t* __restrict__ iddst,
                                                    Geom* g, const T* __restrict__ E,
                                                    const T* __restrict__ phi, Consts c,
                                                    SortPlan sp,
                                                    const int4* __restrict__ chunks,
                                                    const uint32_t* __restrict__ nchunks,
                                                    double L, HalfMap second, int has_next,
                                                    HalfMap first_next, Box* box,
                                                    double* __restrict__ diag_part,
                                                    const double* __restrict__ diag_shift) {
  gkd_tiles_body<S, T, PERM, DIAG>(B, src, perm, idsrc, iddst, g, E, phi, c, sp, chunks, nchunks,
                                   L, second, has_next, first_next, box, blockIdx.x, gridDim.x,
                                   diag_part, diag_shift);
}

// The first step's shift of the fused moment sums: the centre of the step's grid for the positions
// and 0 for the momenta (later steps: the previous step's means, from k_diag_combine).  Also
// empties the accumulators.
__global__ __launch_bounds__(256) void k_diag_start(const Geom* __restrict__ g, Consts c,
                                                    double* __restrict__ part,
                                                    double* __restrict__ shift) {
  for (int t = threadIdx.x; t < kMomentSlots * kDiagSlots; t += 256) part[t] = 0.0;
  const int r = threadIdx.x;
  if (r >= 6) return;
  if (r & 1) {
    shift[r] = 0.0;
  } else {
    const int a = r >> 1;
    const int na = a == 0 ? c.nx : (a == 1 ? c.ny : c.nz);
    shift[r] = g->origin[a] + 0.5 * (na - 1) * g->h[a];
  }
}

// Moments from the accumulators: one wave per sum, one lane per accumulator (left zero); then
// mean_r = shift_r + S_r / n and the centred products S_ab / n - (S_a / n)(S_b / n), and the
// next step's shift.  A device error state (status != 0) writes NaN.
__global__ __launch_bounds__(1024) void k_diag_combine(const Geom* __restrict__ g, double* part,
                                                       double* __restrict__ shift, int64_t n,
                                                       double* __restrict__ out) {
  __shared__ double tot[kMomentSlots];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nwave = (int)blockDim.x >> 6;
  static_assert(kDiagSlots == 64, "one accumulator per lane");
  for (int q = wave; q < kMomentSlots; q += nwave) {
    double t = part[q * kDiagSlots + lane];
    part[q * kDiagSlots + lane] = 0.0;
    for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off);
    if (lane == 0) tot[q] = t;
  }
  __syncthreads();
  if (threadIdx.x >= kMomentSlots) return;
  const int q = threadIdx.x;
  if (g->status) {
    out[q] = NAN;
    return;
  }
  const double inv = 1.0 / (double)n;
  if (q < 6) {
    const double m = shift[q] + tot[q] * inv;
    out[q] = m;
    shift[q] = m;
    return;
  }
  int a = 0, k = q - 6;
  while (k >= 6 - a) {
    k -= 6 - a;
    ++a;
  }
  const int b = a + k;
  out[q] = tot[q] * inv - (tot[a] * inv) * (tot[b] * inv);
}

// First half of the first step out of the caller's array: A = drift(quad(X)), ids, box.  The
// ids are the caller's labels ids_in (binned order) or the indices in X; idA == nullptr: none.
__device__ __forceinline__ void prologue_body(const double* __restrict__ X,
                                                   double* __restrict__ A,
                                                   uint32_t* __restrict__ idA,
                                                   const uint32_t* __restrict__ ids_in,
                                                   const HalfMap& first, const Consts& c,
                                                   Box* box, Geom* g, int blk, int nblk) {
  const int64_t n = c.n;
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  bool bad = false;
  for (int64_t i = blk * (int64_t)kBlk + threadIdx.x; i < n;
       i += (int64_t)nblk * kBlk) {
    double v[6];
    for (int r = 0; r < 6; ++r) v[r] = X[r * n + i];
    apply_half(first, v, c.inv_gamma2);
    for (int r = 0; r < 6; ++r) A[r * n + i] = v[r];
    if (idA) idA[i] = ids_in ? ids_in[i] : (uint32_t)i;
    double p[3] = {v[0], v[2], v[4]};
    for (int a = 0; a < 3; ++a) {
      bad |= !isfinite(p[a]);
      lo[a] = fmin(lo[a], p[a]);
      hi[a] = fmax(hi[a], p[a]);
    }
  }
  box_geometry_block(lo, hi, bad, box, g, c, nblk);
}

__global__ __launch_bounds__(kBlk) void k_prologue(const double* __restrict__ X,
                                                   double* __restrict__ A,
                                                   uint32_t* __restrict__ idA,
                                                   const uint32_t* __restrict__ ids_in,
                                                   HalfMap first, Consts c, Box* box,
                                                   Geom* g) {
  prologue_body(X, A, idA, ids_in, first, c, box, g, blockIdx.x, gridDim.x);
}

// Bucket keys for the return to the caller's order: key = id >> shift (at most 4096 buckets of
// consecutive original indices), with a block-privatised histogram.  After a device error nothing:
// the pass that takes the counts out of hist again does not run then.
__device__ __forceinline__ void id_hist_body(const Geom* __restrict__ g,
                                                  const uint32_t* __restrict__ ids, int64_t n,
                                                  int shift, int nbuckets,
                                                  uint32_t* __restrict__ keys,
                                                  uint32_t* __restrict__ hist, int blk, int nblk) {
  __shared__ uint32_t lh[kMaxTiles];
  if (g->status) return;
  for (int t = threadIdx.x; t < nbuckets; t += kBlk) lh[t] = 0u;
  __syncthreads();
  const int64_t base = (int64_t)blk * kItems;
  for (int k = 0; k < kPer; ++k) {
    int64_t i = base + k * kBlk + threadIdx.x;
    if (i < n) {
      uint32_t key = ids[i] >> shift;
      key = key < (uint32_t)nbuckets ? key : (uint32_t)nbuckets - 1u;
      keys[i] = key;
      atomicAdd(&lh[key], 1u);
    }
  }
  __syncthreads();
  for (int t = threadIdx.x; t < nbuckets; t += kBlk)
    if (lh[t]) atomicAdd(&hist[t], lh[t]);
}

__global__ __launch_bounds__(kBlk) void k_id_hist(const Geom* __restrict__ g,
                                                  const uint32_t* __restrict__ ids, int64_t n,
                                                  int shift, int nbuckets,
                                                  uint32_t* __restrict__ keys,
                                                  uint32_t* __restrict__ hist) {
  id_hist_body(g, ids, n, shift, nbuckets, keys, hist, blockIdx.x, gridDim.x);
}

// Back to the caller's order: X[r][id[i]] = A[r][i].  After the bucket pass, the particles a
// block handles have ids in a narrow range, so its writes stay within an L2-sized window.
__device__ __forceinline__ void unpermute_body(const double* __restrict__ A,
                                                    const uint32_t* __restrict__ idA, int64_t n,
                                                    const Geom* __restrict__ g,
                                                    double* __restrict__ X, int blk, int nblk) {
  if (g->status) return;  // after a device error X keeps the caller's input
  for (int64_t i = blk * (int64_t)kBlk + threadIdx.x; i < n;
       i += (int64_t)nblk * kBlk) {
    uint32_t j = idA[i];
    if (j < (uint64_t)n)
      for (int r = 0; r < 6; ++r) X[r * n + j] = A[r * n + i];
  }
}

__global__ __launch_bounds__(kBlk) void k_unpermute(const double* __restrict__ A,
                                                    const uint32_t* __restrict__ idA, int64_t n,
                                                    const Geom* __restrict__ g,
                                                    double* __restrict__ X) {
  unpermute_body(A, idA, n, g, X, blockIdx.x, gridDim.x);
}


// Final placement through LDS.  After the bucket scatter, bucket b holds exactly the particles
// with ids [b 2^sh, (b + 1) 2^sh) (the ids are a permutation of 0..n-1), at those same
// positions of A.  One workgroup of kUBlk threads takes a bucket: each thread keeps the local
// offsets (id - b 2^sh) of its PER items; then, row by row, the values are dropped into an
// LDS buffer at their offsets, STAGE at a time, and written back to X contiguously, so every
// store is coalesced.  Requires 2^sh <= kUBlk * PER; PER is the smallest that fits, because a
// thread issues all PER loads (clamped into the bucket) whatever the bucket holds.  Up to PER = 8
// a row's items stay in registers and the next row's loads are issued before this row's
// barriers; above, a row is loaded eight items at a time in each pass (the second pass from L2).
constexpr int kUBlk = 1024;
constexpr int kUMaxPer = 32;
constexpr int kUStage = 16384;

template <int PER>
__global__ __launch_bounds__(kUBlk) void k_unpermute_lds(const double* __restrict__ A,
                                                         const uint32_t* __restrict__ idA,
                                                         int64_t n, int sh,
                                                         const Geom* __restrict__ g,
                                                         double* __restrict__ X) {
  constexpr int STAGE = PER * kUBlk < kUStage ? PER * kUBlk : kUStage;
  constexpr int G = PER < 8 ? PER : 8;  // loads in flight per thread
  __shared__ double stage[STAGE];
  if (g->status) return;  // after a device error X keeps the caller's input
  const int64_t b0 = (int64_t)blockIdx.x << sh;
  const int cnt = (int)min((int64_t)1 << sh, n - b0);
  // 16-bit offsets, two per register (2^sh <= 32768); 0xffff marks no item.  An id outside
  // the bucket (impossible for a permutation) is dropped, so LDS stays in bounds.
  uint32_t offp[PER / 2];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int l = threadIdx.x + k * kUBlk;
    uint32_t o = 0xffffu;
    if (l < cnt) {
      const int64_t d = (int64_t)idA[b0 + l] - b0;
      if (d >= 0 && d < cnt) o = (uint32_t)d;
    }
    if (k & 1)
      offp[k >> 1] |= o << 16;
    else
      offp[k >> 1] = o;
  }
  // G loads, unconditional (clamped into the bucket, cnt >= 1)
  auto load = [&](int r, int k0, double* v) {
#pragma unroll
    for (int j = 0; j < G; ++j)
      v[j] = A[r * n + b0 + min((int)threadIdx.x + (k0 + j) * kUBlk, cnt - 1)];
  };
  auto drop = [&](int k0, int q, const double* v) {
#pragma unroll
    for (int j = 0; j < G; ++j) {
      const int k = k0 + j;
      const uint32_t o = (offp[k >> 1] >> (16 * (k & 1))) & 0xffffu;
      if (o != 0xffffu && (int)(o / STAGE) == q) stage[o % STAGE] = v[j];
    }
  };
  auto flush = [&](int r, int q) {
    const int len = min(STAGE, cnt - q * STAGE);
    for (int t = threadIdx.x; t < len; t += kUBlk) X[r * n + b0 + q * STAGE + t] = stage[t];
  };
  if constexpr (PER <= 8) {  // one pass per row: the bucket fits the stage
    double v[2][G];
    load(0, 0, v[0]);
#pragma unroll
    for (int r = 0; r < 6; ++r) {
      if (r < 5) load(r + 1, 0, v[(r + 1) & 1]);
      drop(0, 0, v[r & 1]);
      __syncthreads();
      flush(r, 0);
      __syncthreads();
    }
  } else {
    const int nq = (cnt + STAGE - 1) / STAGE;
    for (int r = 0; r < 6; ++r) {
      for (int q = 0; q < nq; ++q) {
#pragma unroll 1
        for (int k0 = 0; k0 < PER; k0 += G) {
          double v[G];
          load(r, k0, v);
#pragma unroll
          for (int k1 = 0; k1 < PER; k1 += G)  // constant indices into offp
            if (k1 == k0) drop(k1, q, v);
        }
        __syncthreads();
        flush(r, q);
        __syncthreads();
      }
    }
  }
}

// ------------------------------------------------------------------------ batched wrappers
// beam = blockIdx.y; the current phase-space copy of step j is XA for even j (parity 0).

__device__ __forceinline__ double* cur_X(const BeamDev& d, int parity) { return parity ? d.XB : d.XA; }
__device__ __forceinline__ double* nxt_X(const BeamDev& d, int parity) { return parity ? d.XA : d.XB; }
__device__ __forceinline__ uint32_t* cur_id(const BeamDev& d, int parity) { return parity ? d.idB : d.idA; }
__device__ __forceinline__ uint32_t* nxt_id(const BeamDev& d, int parity) { return parity ? d.idA : d.idB; }

__global__ __launch_bounds__(kBlk) void k_prologue_batch(const BeamDev* __restrict__ beams) {
  const BeamDev& d = beams[blockIdx.y];
  // workgroups past the beam's own particles only cost their dispatch
  const int nblk = (int)min((int64_t)gridDim.x, (d.c.n + kBlk - 1) / kBlk);
  if ((int)blockIdx.x >= nblk) return;
  prologue_body(d.X, d.XA, d.idA, nullptr, d.slices[0].first, d.c, d.box, d.geom, blockIdx.x,
                nblk);
}

template <int S>
__global__ __launch_bounds__(kBlk) void k_key_rank_batch(const BeamDev* __restrict__ beams,
                                                         int parity) {
  const BeamDev& d = beams[blockIdx.y];
  const int nblk = (int)((d.c.n + kItems - 1) / kItems);
  if ((int)blockIdx.x >= nblk) return;
  key_rank_body<S, kPer>(cur_X(d, parity), d.geom, d.c, d.sp, d.keys, d.hist, d.cursor, d.chunks,
                         d.nchunks, blockIdx.x, nblk);
}

// after a call's first step: the order only (cur_X stays where it is)
__global__ __launch_bounds__(kBlk) void k_place_batch(const BeamDev* __restrict__ beams) {
  const BeamDev& d = beams[blockIdx.y];
  if ((int64_t)blockIdx.x * kItems >= d.c.n) return;
  place_body<kPer>(d.keys, d.geom, d.c.n, d.sp, d.cursor, d.nchunks, d.perm, blockIdx.x);
}

template <bool STAGED>
__global__ __launch_bounds__(kBlk) void k_scatter_batch(const BeamDev* __restrict__ beams,
                                                        int parity) {
  const BeamDev& d = beams[blockIdx.y];
  if ((int64_t)blockIdx.x * kItems >= d.c.n) return;
  scatter_body<STAGED>(cur_X(d, parity), cur_id(d, parity), d.keys, key_mask(d.sp), d.geom, d.c.n, d.sp.ntiles, d.cursor,
               nxt_X(d, parity), nxt_id(d, parity), blockIdx.x, gridDim.x);
}

// PERM: the step's input cur_X through the ranking; else nxt_X, in slot order
template <int S, bool PERM>
__global__ __launch_bounds__(kBlk) void k_deposit_tiles_batch(const BeamDev* __restrict__ beams,
                                                              int parity) {
  const BeamDev& d = beams[blockIdx.y];
  deposit_tiles_body<S, PERM>(PERM ? cur_X(d, parity) : nxt_X(d, parity), PERM ? d.perm : nullptr,
                              d.geom, d.c, d.sp, d.chunks, d.nchunks, blockIdx.x, gridDim.x,
                              d.tacc, d.tscale);
}

template <int S, typename T>
__global__ __launch_bounds__(256) void k_tile_reduce_batch(const BeamDev* __restrict__ beams) {
  const BeamDev& d = beams[blockIdx.y];
  tile_reduce_body<S, T>(d.geom, d.c, d.sp, d.tacc, d.tscale, (T*)d.rho, blockIdx.x, gridDim.x);
}

// PERM: reads cur_X (and its ids) through the ranking and writes nxt_X in slot order; else
// updates nxt_X in place
template <int S, typename T, bool PERM>
__global__ __launch_bounds__(kBlk) void k_gkd_tiles_batch(const BeamDev* __restrict__ beams,
                                                          int parity, int j, int n_steps) {
  const BeamDev& d = beams[blockIdx.y];
  const SliceDev& sl = d.slices[j % d.n_slices];
  const SliceDev& sn = d.slices[(j + 1) % d.n_slices];
  gkd_tiles_body<S, T, PERM, false>(nxt_X(d, parity), PERM ? cur_X(d, parity) : nullptr,
                                    PERM ? d.perm : nullptr, PERM ? cur_id(d, parity) : nullptr,
                                    PERM ? nxt_id(d, parity) : nullptr, d.geom, nullptr,
                                    (const T*)d.phi, d.c, d.sp, d.chunks, d.nchunks, sl.L, sl.second,
                                    j + 1 < n_steps, sn.first, d.box, blockIdx.x, gridDim.x);
}

// reordering at the end: bucket keys of the ids, bucket offsets, bucket scatter, final scatter
// Buckets of 2^shift consecutive original indices, at most kMaxTiles of them.  A single beam
// takes at least 2^kMinShift indices per bucket: a block of the bucket scatter then writes runs
// of many particles per bucket, and the LDS placement's workgroups are full.  A batch places
// directly (k_unpermute_batch), for which the narrowest buckets are the best (2.4 ms of 167 less
// per call over 256 beams than with kMinShift).
constexpr int kMinShift = 12;
__host__ __device__ __forceinline__ SortPlan bucket_sort_plan(int nb) {
  SortPlan bp{};
  bp.T[0] = bp.T[1] = bp.T[2] = 1;
  bp.NT[0] = nb;
  bp.NT[1] = bp.NT[2] = 1;
  bp.ntiles = nb;
  bp.kbits = 1;
  bp.chunk = 1 << 30;  // the work list is not used; one entry per bucket
  bp.max_chunks = nb + 1;
  return bp;
}
__host__ __device__ __forceinline__ void bucket_plan(int64_t n, int min_shift, int* shift,
                                                     int* nb) {
  int sh = min_shift;
  while (((n - 1) >> sh) >= kMaxTiles) ++sh;
  *shift = sh;
  *nb = (int)(((n - 1) >> sh) + 1);
}

__global__ __launch_bounds__(kBlk) void k_id_hist_batch(const BeamDev* __restrict__ beams,
                                                        int parity) {
  const BeamDev& d = beams[blockIdx.y];
  if ((int64_t)blockIdx.x * kItems >= d.c.n) return;
  int sh, nb;
  bucket_plan(d.c.n, 0, &sh, &nb);
  id_hist_body(d.geom, cur_id(d, parity), d.c.n, sh, nb, d.keys, d.hist, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(1024) void k_bucket_chunks_batch(const BeamDev* __restrict__ beams) {
  const BeamDev& d = beams[blockIdx.x];
  __shared__ uint32_t lh[kMaxTiles];
  if (d.geom->status) return;
  int sh, nb;
  bucket_plan(d.c.n, 0, &sh, &nb);
  build_chunks_body<1024>(d.geom, d.c.n, bucket_sort_plan(nb), d.hist, d.cursor, d.chunks,
                          d.nchunks, lh);
}

__global__ __launch_bounds__(kBlk) void k_bucket_scatter_batch(const BeamDev* __restrict__ beams,
                                                               int parity) {
  const BeamDev& d = beams[blockIdx.y];
  if ((int64_t)blockIdx.x * kItems >= d.c.n) return;
  int sh, nb;
  bucket_plan(d.c.n, 0, &sh, &nb);
  scatter_body<true>(cur_X(d, parity), cur_id(d, parity), d.keys, ~0u, d.geom, d.c.n, nb, d.cursor,
               nxt_X(d, parity), nxt_id(d, parity), blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(kBlk) void k_unpermute_batch(const BeamDev* __restrict__ beams,
                                                          int parity) {
  const BeamDev& d = beams[blockIdx.y];
  unpermute_body(nxt_X(d, parity), nxt_id(d, parity), d.c.n, d.geom, d.X, blockIdx.x, gridDim.x);
}

int grid_per(int64_t n, int per) { return (int)((n + kBlk * per - 1) / (kBlk * per)); }
int grid_items(int64_t n) { return grid_per(n, kPer); }
// Particles per thread of the ranking: one while a workgroup's chain of loads and atomics is the
// length of the pass, kPer once every CU has a workgroup, since each workgroup clears and flushes
// the counters of all tiles (4 per thread took 20.6 us at 1e6 particles, 256 tiles, where kPer
// takes 14.8; kPer took 23 us at 1e4 particles, where one takes 8).
int per_thread(int64_t n) { return n <= (1 << 17) ? 1 : kPer; }
int grid_wide(int64_t n) { return (int)((n + kWItems - 1) / kWItems); }
// the wide staged scatter once it still fills every CU with a block (256 CUs); below that the
// 4096-particle blocks of k_scatter<true> keep the device busy
bool wide_pays(int64_t n) { return grid_wide(n) >= 256; }

// Up to this count the return to the caller's order writes X directly in one launch: the state
// (48 MB) stays in the 256 MB last-level cache, which takes the scattered 8-byte writes.  Direct
// against histogram, bucket scatter and LDS placement, us per return: 6.3 / 75 at 1e4 particles,
// 19 / 77 at 2e5, 81 / 94 at 1e6, 238 / 147 at 2e6, 2343 / 966 at 1.25e7.  (With buckets of 1 to
// 256 particles the second form took 313 at 1e4, 484 at 1e6 and 1181 at 1.25e7.)
constexpr int64_t kDirectReturn = 1 << 20;

int grid_stride(int64_t n) {
  int64_t b = (n + kBlk - 1) / kBlk;
  if (b > 8192) b = 8192;
  return (int)(b < 1 ? 1 : b);
}

}  // namespace

// Particles per work item where the caller gives none: n / 6144 rounded down to a power of two,
// 512..8192.  A work item is one workgroup's serial chain of rounds, and the densest tiles of a
// bunch hold many items, so with 8192 for every size a few workgroups worked through the middle
// of the beam while the rest of the device was idle; below 512 the window's fill and flush per
// item outweigh that.  Deposit + gather-kick, us per step with 8192 and as chosen: 65 and 39 at
// 1e5 TSC (48^3), 112 and 71 at 1e6 CIC and 186 and 88 at 1e6 TSC (64^3), 416 and 221 at 3e6 TSC
// (96^3), 776 and 671 at 1.25e7 TSC and 2259 and 2220 at 4e7 TSC (128^3).  The results do not
// depend on it.
// On a grid of few tiles (64 at 16^3) so small an item flushes its window into one that hundreds of
// others flush into, all atomics on a few hundred addresses: there an item holds n / (32 tiles), as
// long as 768 items, three per CU, are left, and at most 4096.  A binned step of 6e6 CIC particles,
// us, by n alone (512) and so: 570 and 319 on 12^3 (27 tiles; 331 with 8192), 433 and 410 on 8^3, 392
// and 328 on 16^3; of 2e6 232 and 160 on 12^3, 225 and 172 (TSC) on 4^3.  From 24^3 (216 tiles) on it
// is the rule by n.
int default_chunk(int64_t n, int ntiles) {
  const int64_t by_n = std::min<int64_t>(n / 6144, 8192);
  const int64_t by_tiles = std::min<int64_t>(std::min(n / (32 * (int64_t)ntiles), n / 768), 4096);
  const int64_t most = std::max(by_n, by_tiles);
  int c = 512;
  while (2 * (int64_t)c <= most) c *= 2;
  return c;
}

SortPlan make_sort_plan(int nx, int ny, int nz, int64_t n, const int tile[3], int chunk,
                        int blocks, int threads, int deposit_threads) {
  SortPlan sp;
  int nn[3] = {nx, ny, nz};
  for (int a = 0; a < 3; ++a) {
    int t = (nn[a] + 15) / 16;
    if (t < 4) t = 4;
    sp.T[a] = tile && tile[a] > 0 ? tile[a] : t;
    sp.NT[a] = (nn[a] + sp.T[a] - 1) / sp.T[a];
  }
  sp.ntiles = sp.NT[0] * sp.NT[1] * sp.NT[2];
  sp.kbits = 1;
  while ((1 << sp.kbits) < sp.ntiles) ++sp.kbits;
  sp.chunk = chunk > 0 ? chunk : default_chunk(n, sp.ntiles);
  // every tile adds at most one partial work item
  const int64_t items = (int64_t)(n / sp.chunk) + sp.ntiles + 1;
  sp.max_chunks = items;
  // the work list also serves the id buckets of the final reordering (up to kMaxTiles entries)
  if (sp.max_chunks < kMaxTiles + 1) sp.max_chunks = kMaxTiles + 1;
  sp.blocks = blocks > 0 ? blocks : (int)(items < 4096 ? items : 4096);
  sp.threads = threads > 0 ? threads : kBlk;
  sp.dep_threads = deposit_threads > 0 ? deposit_threads : sp.threads;
  return sp;
}

namespace {
// Dynamic LDS above 64 KB needs the kernel's limit raised first; the runtime accepts a limit up
// to the device's 160 KB less the kernel's static LDS.
template <typename K>
hipError_t lds_optin(K kernel, size_t bytes) {
  if (bytes > kMaxLdsBytes) return hipErrorInvalidConfiguration;
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}
}  // namespace

#define PIC_TRY_LDS(kernel, bytes)            \
  do {                                        \
    hipError_t e_ = lds_optin(kernel, bytes); \
    if (e_ != hipSuccess) return e_;          \
  } while (0)

hipError_t launch_prologue(const double* X, double* A, uint32_t* idA, const uint32_t* ids_in,
                           const HalfMap& first, Consts c, Box* box, Geom* g, hipStream_t s) {
  hipLaunchKernelGGL(k_prologue, dim3(grid_stride(c.n)), dim3(kBlk), 0, s, X, A, idA, ids_in,
                     first, c, box, g);
  return hipGetLastError();
}

namespace {
// tile keys, ranks, sort offsets and the deposit work list of the particles in A
template <int S>
hipError_t launch_key_rank(const double* A, const Geom* g, Consts c, const SortPlan& sp,
                           uint32_t* keys, uint32_t* hist, uint32_t* cursor, int4* chunks,
                           uint32_t* nchunks, hipStream_t s) {
  if (per_thread(c.n) == 1)
    hipLaunchKernelGGL((k_key_rank<S, 1>), dim3(grid_per(c.n, 1)), dim3(kBlk), 0, s, A, g, c, sp,
                       keys, hist, cursor, chunks, nchunks);
  else
    hipLaunchKernelGGL((k_key_rank<S, kPer>), dim3(grid_per(c.n, kPer)), dim3(kBlk), 0, s, A, g,
                       c, sp, keys, hist, cursor, chunks, nchunks);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_bin(const double* A, const uint32_t* idA, const Geom* g, Consts c,
                      const SortPlan& sp, uint32_t* keys, uint32_t* hist, uint32_t* cursor,
                      int4* chunks, uint32_t* nchunks, double* B, uint32_t* idB, bool staged,
                      hipStream_t s) {
  hipError_t e =
      c.shape == 1 ? launch_key_rank<1>(A, g, c, sp, keys, hist, cursor, chunks, nchunks, s)
                   : launch_key_rank<2>(A, g, c, sp, keys, hist, cursor, chunks, nchunks, s);
  if (e != hipSuccess) return e;
  const uint32_t kmask = key_mask(sp);
  if (staged && wide_pays(c.n))
    hipLaunchKernelGGL(k_scatter_wide, dim3(grid_wide(c.n)), dim3(kWBlk), 0, s, A, idA, keys,
                       kmask, g, c.n, sp.ntiles, cursor, B, idB);
  else if (staged)
    hipLaunchKernelGGL(k_scatter<true>, dim3(grid_items(c.n)), dim3(kBlk), 0, s, A, idA, keys,
                       kmask, g, c.n, sp.ntiles, cursor, B, idB);
  else
    hipLaunchKernelGGL(k_scatter<false>, dim3(grid_items(c.n)), dim3(kBlk), 0, s, A, idA, keys,
                       kmask, g, c.n, sp.ntiles, cursor, B, idB);
  return hipGetLastError();
}

hipError_t launch_bin_perm(const double* A, const Geom* g, Consts c, const SortPlan& sp,
                           uint32_t* keys, uint32_t* hist, uint32_t* cursor, int4* chunks,
                           uint32_t* nchunks, uint32_t* perm, hipStream_t s) {
  hipError_t e =
      c.shape == 1 ? launch_key_rank<1>(A, g, c, sp, keys, hist, cursor, chunks, nchunks, s)
                   : launch_key_rank<2>(A, g, c, sp, keys, hist, cursor, chunks, nchunks, s);
  if (e != hipSuccess) return e;
  if (per_thread(c.n) < kPer)
    hipLaunchKernelGGL(k_place<4>, dim3(grid_per(c.n, 4)), dim3(kBlk), 0, s, keys, g, c.n, sp,
                       cursor, nchunks, perm);
  else
    hipLaunchKernelGGL(k_place<kPer>, dim3(grid_per(c.n, kPer)), dim3(kBlk), 0, s, keys, g, c.n,
                       sp, cursor, nchunks, perm);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_deposit_tiles(const double* B, const uint32_t* perm, const Geom* g, Consts c,
                                const SortPlan& sp, const int4* chunks, const uint32_t* nchunks,
                                T* rho, hipStream_t s, unsigned long long* tacc, int* tscale) {
  const int S = c.shape;
  size_t lds = sizeof(unsigned long long) * (size_t)(sp.T[0] + S) * (sp.T[1] + S) * (sp.T[2] + S);
  const dim3 grid((unsigned)sp.blocks), block((unsigned)sp.dep_threads);
  if (!tacc || !tscale) return hipErrorInvalidValue;
  const int64_t nodes = (int64_t)c.nx * c.ny * c.nz;
  int rb = (int)((nodes + 255) / 256);
  if (rb > 16384) rb = 16384;
  if (S == 1) {
    PIC_TRY_LDS(k_deposit_tiles<1>, lds);
    hipLaunchKernelGGL(k_deposit_tiles<1>, grid, block, lds, s, B, perm, g, c, sp, chunks, nchunks,
                       tacc, tscale);
    PIC_TRY(hipGetLastError());
    hipLaunchKernelGGL((k_tile_reduce<1, T>), dim3(rb), dim3(256), 0, s, g, c, sp, tacc, tscale,
                       rho);
  } else {
    PIC_TRY_LDS(k_deposit_tiles<2>, lds);
    hipLaunchKernelGGL(k_deposit_tiles<2>, grid, block, lds, s, B, perm, g, c, sp, chunks, nchunks,
                       tacc, tscale);
    PIC_TRY(hipGetLastError());
    hipLaunchKernelGGL((k_tile_reduce<2, T>), dim3(rb), dim3(256), 0, s, g, c, sp, tacc, tscale,
                       rho);
  }
  return hipGetLastError();
}

template <typename T>
hipError_t launch_vdeposit_tiles(const AdjRecord* recs, const uint32_t* perm,
                                 const Geom* g, Consts c, const SortPlan& sp, const int4* chunks,
                                 const uint32_t* nchunks, T* e, hipStream_t s) {
  const int S = c.shape;
  const size_t lds = 3 * sizeof(double) * (size_t)(sp.T[0] + S) * (sp.T[1] + S) * (sp.T[2] + S);
  const dim3 grid((unsigned)sp.blocks), block((unsigned)sp.threads);
  if (S == 1) {
    PIC_TRY_LDS((k_vdeposit_tiles<1, T>), lds);
    hipLaunchKernelGGL((k_vdeposit_tiles<1, T>), grid, block, lds, s, recs, perm, g, c, sp, chunks, nchunks,
                       e);
  } else {
    PIC_TRY_LDS((k_vdeposit_tiles<2, T>), lds);
    hipLaunchKernelGGL((k_vdeposit_tiles<2, T>), grid, block, lds, s, recs, perm, g, c, sp, chunks, nchunks,
                       e);
  }
  return hipGetLastError();
}

template hipError_t launch_vdeposit_tiles<double>(const AdjRecord*, const uint32_t*,
                                                  const Geom*, Consts, const SortPlan&,
                                                  const int4*, const uint32_t*, double*,
                                                  hipStream_t);
template hipError_t launch_vdeposit_tiles<float>(const AdjRecord*, const uint32_t*,
                                                 const Geom*, Consts, const SortPlan&,
                                                 const int4*, const uint32_t*, float*,
                                                 hipStream_t);

template <typename T>
hipError_t launch_gkd_tiles(double* B, const double* src, const uint32_t* perm,
                            const uint32_t* idsrc, uint32_t* iddst, Geom* g, const T* E,
                            const T* phi, Consts c, const SortPlan& sp, const int4* chunks,
                            const uint32_t* nchunks, double L, const HalfMap& second,
                            int has_next, const HalfMap& first_next, Box* box, hipStream_t s,
                            double* diag_part, double* diag_shift, const double* diag_prev,
                            double* diag_out) {
  const int S = c.shape;
  size_t lds = 3 * sizeof(T) * (size_t)(sp.T[0] + S) * (sp.T[1] + S) * (sp.T[2] + S);
  const bool diag = diag_out != nullptr;
  // With diagnostics each workgroup ends with a reduction of its 27 sums, so fewer, longer ones pay
  // although they balance less well.  Measured, us, at 512 / 768 / 2048 / 4096 workgroups:
  // 1e5 TSC 48^3 32 / 37 / 58 / 93; 1e6 TSC 64^3 70 / 71 / 89 / 117; 4e6 TSC 96^3 224 / 207 / 233 /
  // 253; 1.25e7 TSC 128^3 590 / 533 / 580 / 576.  Beyond 2^25 the reduction is paid back in any
  // workgroup and balance counts: 5e7 2494 (768) / 2523 (the plan's), 1e8 with 16384-particle work
  // items 4491 / 4078.
  const int diag_blocks = c.n <= (1 << 21) ? 512 : (c.n <= (1 << 25) ? 768 : sp.blocks);
  const dim3 grid((unsigned)(diag ? std::min(sp.blocks, diag_blocks) : sp.blocks)),
      block((unsigned)(diag ? std::min(sp.threads, kDiagThreads) : sp.threads));
  // the ids are optional, as a pair
  if (perm && (!src || src == B || (!idsrc != !iddst) || (idsrc && idsrc == iddst)))
    return hipErrorInvalidValue;
  if (diag) {
    if (!diag_part || !diag_shift) return hipErrorInvalidValue;
    const size_t red = sizeof(double) * kMomentSlots * (kMaxThreads / 64);
    if (lds < red) lds = red;
    if (!diag_prev) {
      hipLaunchKernelGGL(k_diag_start, dim3(1), dim3(256), 0, s, g, c, diag_part, diag_shift);
      PIC_TRY(hipGetLastError());
    }
  }
#define PIC_GKD(SS, PP, DD)                                                                   \
  do {                                                                                        \
    PIC_TRY_LDS((k_gkd_tiles<SS, T, PP, DD>), lds);                                           \
    hipLaunchKernelGGL((k_gkd_tiles<SS, T, PP, DD>), grid, block, lds, s, B, src, perm, idsrc,\
                       iddst, g, E, phi, c, sp, chunks, nchunks, L, second, has_next,         \
                       first_next, box, diag_part, diag_shift);                               \
  } while (0)
  if (diag) {
    if (S == 1) {
      if (perm) PIC_GKD(1, true, true); else PIC_GKD(1, false, true);
    } else {
      if (perm) PIC_GKD(2, true, true); else PIC_GKD(2, false, true);
    }
  } else {
    if (S == 1) {
      if (perm) PIC_GKD(1, true, false); else PIC_GKD(1, false, false);
    } else {
      if (perm) PIC_GKD(2, true, false); else PIC_GKD(2, false, false);
    }
  }
#undef PIC_GKD
  PIC_TRY(hipGetLastError());
  if (diag) {
    hipLaunchKernelGGL(k_diag_combine, dim3(1), dim3(1024), 0, s, g, diag_part, diag_shift, c.n,
                       diag_out);
    PIC_TRY(hipGetLastError());
  }
  return hipSuccess;
}

template hipError_t launch_gkd_tiles<double>(double*, const double*, const uint32_t*,
                                             const uint32_t*, uint32_t*, Geom*, const double*,
                                             const double*, Consts, const SortPlan&, const int4*,
                                             const uint32_t*, double, const HalfMap&, int,
                                             const HalfMap&, Box*, hipStream_t, double*, double*,
                                             const double*, double*);
template hipError_t launch_gkd_tiles<float>(double*, const double*, const uint32_t*,
                                            const uint32_t*, uint32_t*, Geom*, const float*,
                                            const float*, Consts, const SortPlan&, const int4*, const uint32_t*,
                                            double, const HalfMap&, int, const HalfMap&, Box*,
                                            hipStream_t, double*, double*, const double*,
                                            double*);

hipError_t launch_unpermute(const double* A, const uint32_t* idA, int64_t n, double* X,
                            uint32_t* keys, uint32_t* hist, uint32_t* cursor, int4* chunks,
                            uint32_t* nchunks, double* B, uint32_t* idB, const Geom* g,
                            hipStream_t s) {
  if (n <= kDirectReturn) {
    hipLaunchKernelGGL(k_unpermute, dim3(grid_stride(n)), dim3(kBlk), 0, s, A, idA, n, g, X);
    return hipGetLastError();
  }
  int shift, nb;
  bucket_plan(n, kMinShift, &shift, &nb);
  const SortPlan bp = bucket_sort_plan(nb);
  hipLaunchKernelGGL(k_id_hist, dim3(grid_items(n)), dim3(kBlk), 0, s, g, idA, n, shift, nb, keys,
                     hist);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_build_chunks, dim3(1), dim3(1024), 0, s, g, n, bp, hist, cursor, chunks,
                     nchunks);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (wide_pays(n))
    hipLaunchKernelGGL(k_scatter_wide, dim3(grid_wide(n)), dim3(kWBlk), 0, s, A, idA, keys, ~0u, g,
                       n, nb, cursor, B, idB);
  else
    hipLaunchKernelGGL(k_scatter<true>, dim3(grid_items(n)), dim3(kBlk), 0, s, A, idA, keys, ~0u, g,
                       n, nb, cursor, B, idB);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t bucket = (int64_t)1 << shift;
  if (bucket <= kUBlk * 4)
    hipLaunchKernelGGL(k_unpermute_lds<4>, dim3(nb), dim3(kUBlk), 0, s, B, idB, n, shift, g, X);
  else if (bucket <= kUBlk * 8)
    hipLaunchKernelGGL(k_unpermute_lds<8>, dim3(nb), dim3(kUBlk), 0, s, B, idB, n, shift, g, X);
  else if (bucket <= kUBlk * kUMaxPer)
    hipLaunchKernelGGL(k_unpermute_lds<kUMaxPer>, dim3(nb), dim3(kUBlk), 0, s, B, idB, n, shift,
                       g, X);
  else
    hipLaunchKernelGGL(k_unpermute, dim3(grid_stride(n)), dim3(kBlk), 0, s, B, idB, n, g, X);
  return hipGetLastError();
}

// ------------------------------------------------------------------------ batched launches

hipError_t launch_batch_prologue_particles(const BeamDev* beams, int nb, const BatchDims& bd,
                                           hipStream_t s) {
  hipLaunchKernelGGL(k_prologue_batch, dim3(std::min(grid_stride(bd.max_n), 1024), nb), dim3(kBlk), 0, s, beams);
  return hipGetLastError();
}

hipError_t launch_batch_particles_bin(const BeamDev* beams, int nb, const BatchDims& bd, int shape,
                                      int parity, bool first, hipStream_t s) {
  const dim3 grid(grid_items(bd.max_n), nb);
  if (shape == 1)
    hipLaunchKernelGGL(k_key_rank_batch<1>, grid, dim3(kBlk), 0, s, beams, parity);
  else
    hipLaunchKernelGGL(k_key_rank_batch<2>, grid, dim3(kBlk), 0, s, beams, parity);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the first step moves the caller's order into tile order (staged scatter); later steps, whose
  // input is in the previous step's tile order, only rank
  if (first)
    hipLaunchKernelGGL(k_scatter_batch<true>, grid, dim3(kBlk), 0, s, beams, parity);
  else
    hipLaunchKernelGGL(k_place_batch, grid, dim3(kBlk), 0, s, beams);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_batch_deposit(const BeamDev* beams, int nb, const BatchDims& bd, int shape,
                                int parity, bool first, hipStream_t s) {
  const dim3 grid(bd.max_chunks, nb);
  int rb = (int)(((int64_t)bd.max_nx * bd.max_ny * bd.max_nz + 255) / 256);
  if (rb > 16384) rb = 16384;
#define PIC_DEP_BATCH(SS, PP)                                                                 \
  do {                                                                                        \
    PIC_TRY_LDS((k_deposit_tiles_batch<SS, PP>), bd.dep_lds);                                 \
    hipLaunchKernelGGL((k_deposit_tiles_batch<SS, PP>), grid, dim3(kBlk), bd.dep_lds, s,      \
                       beams, parity);                                                        \
    PIC_TRY(hipGetLastError());                                                               \
    hipLaunchKernelGGL((k_tile_reduce_batch<SS, T>), dim3(rb, nb), dim3(256), 0, s, beams);   \
  } while (0)
  if (shape == 1) {
    if (first) PIC_DEP_BATCH(1, false); else PIC_DEP_BATCH(1, true);
  } else {
    if (first) PIC_DEP_BATCH(2, false); else PIC_DEP_BATCH(2, true);
  }
#undef PIC_DEP_BATCH
  return hipGetLastError();
}

template <typename T>
hipError_t launch_batch_gkd(const BeamDev* beams, int nb, const BatchDims& bd, int shape,
                            int parity, int j, int n_steps, bool first, hipStream_t s) {
  const dim3 grid(bd.max_chunks, nb);
#define PIC_GKD_BATCH(SS, PP)                                                                 \
  do {                                                                                        \
    PIC_TRY_LDS((k_gkd_tiles_batch<SS, T, PP>), bd.gkd_lds);                                  \
    hipLaunchKernelGGL((k_gkd_tiles_batch<SS, T, PP>), grid, dim3(kBlk), bd.gkd_lds, s, beams, \
                       parity, j, n_steps);                                                   \
  } while (0)
  if (shape == 1) {
    if (first) PIC_GKD_BATCH(1, false); else PIC_GKD_BATCH(1, true);
  } else {
    if (first) PIC_GKD_BATCH(2, false); else PIC_GKD_BATCH(2, true);
  }
#undef PIC_GKD_BATCH
  return hipGetLastError();
}

hipError_t launch_batch_unpermute(const BeamDev* beams, int nb, const BatchDims& bd, int parity,
                                  hipStream_t s) {
  const dim3 grid(grid_items(bd.max_n), nb);
  hipLaunchKernelGGL(k_id_hist_batch, grid, dim3(kBlk), 0, s, beams, parity);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_bucket_chunks_batch, dim3(nb), dim3(1024), 0, s, beams);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_bucket_scatter_batch, grid, dim3(kBlk), 0, s, beams, parity);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_unpermute_batch, dim3(grid_stride(bd.max_n), nb), dim3(kBlk), 0, s, beams,
                     parity);
  return hipGetLastError();
}

template hipError_t launch_batch_deposit<double>(const BeamDev*, int, const BatchDims&, int, int,
                                                 bool, hipStream_t);
template hipError_t launch_batch_deposit<float>(const BeamDev*, int, const BatchDims&, int, int,
                                                bool, hipStream_t);
template hipError_t launch_batch_gkd<double>(const BeamDev*, int, const BatchDims&, int, int, int,
                                             int, bool, hipStream_t);
template hipError_t launch_batch_gkd<float>(const BeamDev*, int, const BatchDims&, int, int, int,
                                            int, bool, hipStream_t);

template hipError_t launch_deposit_tiles<double>(const double*, const uint32_t*, const Geom*,
                                                 Consts, const SortPlan&, const int4*,
                                                 const uint32_t*, double*, hipStream_t,
                                                 unsigned long long*, int*);
template hipError_t launch_deposit_tiles<float>(const double*, const uint32_t*, const Geom*,
                                                Consts, const SortPlan&, const int4*,
                                                const uint32_t*, float*, hipStream_t,
                                                unsigned long long*, int*);

}  // namespace pic
