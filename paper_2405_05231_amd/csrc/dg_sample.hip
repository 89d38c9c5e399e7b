// Group sampling: node-wise fan-out neighbour sampling (DiskGNN §2, Fig. 1) for
// up to 64 mini-batches in one pass (offline sampling, §3).
//
// Device state: a node-major membership mask visited[u] (bit b = u is in
// mini-batch b) and its copy prev[u] as of the start of the current hop.  A
// hop is:
//   frontier pass (the seeds enter with the first one): degrees, and edge slots
//     by an exclusive scan within tiles of one batch ->
//   draw + mark: 1-8 lanes per frontier node, a fire-and-forget atomicOr on
//     visited per sampled edge; a hop that can reach only a small share of the
//     nodes also marks the 8-node lines of the mask it touches ->
//   compaction of visited & ~prev (the nodes new at this hop) into each
//     batch's new segment, ascending, with no sort; it also brings prev up to
//     date (the last hop instead clears prev with DG_SAMPLE_EXIT_CLEAR, and
//     writes the member-lines map when asked) ->
//   one read-back of the hop's counts.
// Sampled neighbours are relabelled from global to local IDs at the end,
// through one of two tables: a direct [N][B] array of local indices that the
// compaction fills as it assigns them (DG_SAMPLE_DIRECT), or a (node, batch)
// hash table sized for the group and filled after the last hop.  The last
// hop's own new nodes are found by search in their ascending segment instead.
#include <string.h>

#include <type_traits>

#include "dg_passes.h"

namespace dg {
namespace {

constexpr int THREADS = 256;
constexpr int FMAX = 32;  // fan-outs up to this take the register path

__host__ __device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
constexpr uint64_t GAMMA = 0x9E3779B97F4A7C15ull;

// Per-hop description of the frontier, passed by value.  It is cut into tiles of
// F_TILE entries of one batch each, so that a block's batch is the same for all
// its threads.
constexpr int F_TILE = THREADS;
struct Hop {
  int B;
  int32_t f;        // fan-out of this hop (< 0: all)
  int32_t k;        // hop number, 1-based (RNG key)
  int32_t filter;   // the draws filter their membership atomics (see emit_chunk)
  int32_t scanned;  // the tiles' sums are scanned (see k_tile_scan)
  int32_t tstart[DG_MAX_BATCHES + 1];  // prefix of the batches' tiles
  int64_t fstart[DG_MAX_BATCHES + 1];  // prefix of frontier sizes
  int64_t fpos[DG_MAX_BATCHES];        // local position of b's first frontier node
  int64_t ebase[DG_MAX_BATCHES];       // edges of b before this hop
  uint64_t bstate[DG_MAX_BATCHES];     // mix64(rng_seed + gamma*(g+1)) per batch
  uint8_t *touched;                    // nullable: a byte per 2^MC_TOUCH_SHIFT nodes, set
                                       // for every node that gains a membership bit
};

__device__ __forceinline__ int tile_batch(const Hop &h, int32_t t) {
  int lo = 0, hi = h.B;  // invariant tstart[lo] <= t < tstart[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (h.tstart[mid] <= t) lo = mid; else hi = mid;
  }
  return lo;
}

// What the seeds need before the first hop.
struct SeedInit {
  const int32_t *seeds;
  int S;
  int32_t *nodes;
  uint64_t *visited, *prev;
  uint8_t *plines;
  int32_t *local;  // nullable: the direct table
  const int32_t *cache_slot;
  int32_t *loc;  // nullable
};

// Frontier pass: each entry's CSR row and degree, its edge slots' exclusive scan
// within its tile, and each tile's sum.  The draw kernel adds the sums of its
// batch's earlier tiles itself, or finds them scanned (k_tile_scan).  (Scanning the
// entries by kernels of their own took 16 to 20 us a hop on short frontiers, 39 us at
// 3.2M entries.)
// SEEDS: the first hop's frontier, straight from the seeds; each also enters its
// node list, the membership words and the local indices, with loc its address-
// table entry (final for a cached seed, pending otherwise).  degree = false: that
// part alone, and a frontier pass over the list it leaves follows: from SEEDS_APART
// seeds on, where the two kinds of scattered access are faster one after the other
// (one pass against both: 1M seeds 150 / 161 us, 4.2M 595 / 570 (one mini-batch 527 /
// 564), 8.4M 1159 / 1088, 33.6M 4657 / 4307).
constexpr int64_t SEEDS_APART = 1 << 23;
template <bool SEEDS>
__global__ __launch_bounds__(THREADS) void k_frontier(Hop h, SeedInit sd, bool degree,
                                                      const int32_t *nodes, int64_t node_cap,
                                                      const int64_t *off, int64_t N, int64_t E,
                                                      int64_t *f_off, int64_t *f_deg,
                                                      int64_t *f_eoff, int64_t *tile_sum,
                                                      uint32_t *err) {
  const int32_t t = blockIdx.x;
  const int b = tile_batch(h, t);
  const int64_t j = (int64_t)(t - h.tstart[b]) * F_TILE + threadIdx.x;
  const int64_t i = h.fstart[b] + j;
  const bool valid = i < h.fstart[b + 1];
  int32_t v = -1;
  if (valid) v = SEEDS ? sd.seeds[(int64_t)b * sd.S + j] : nodes[(int64_t)b * node_cap + h.fpos[b] + j];
  const bool in = v >= 0 && (int64_t)v < N;
  int64_t o0 = 0, d = 0;
  if (in && degree) {
    o0 = off[v];
    const int64_t o1 = off[v + 1];
    if (o0 < 0 || o1 < o0 || o1 > E) {
      atomicOr(err, ERR_CSR);
    } else {
      d = o1 - o0;
    }
  }
  if (SEEDS && valid) {
    sd.nodes[(int64_t)b * node_cap + j] = v;
    if (!in) {
      atomicOr(err, ERR_NODE_RANGE);
    } else {
      if (sd.loc) {
        const int32_t sl = sd.cache_slot[v];
        if (sl < -1) atomicOr(err, ERR_CACHE_SLOT);
        sd.loc[(int64_t)b * node_cap + j] = sl >= 0 ? -(sl + 1) : (int32_t)DG_LOC_PENDING;
      }
      const unsigned long long bit = 1ull << b;
      const unsigned long long old = atomicOr((unsigned long long *)&sd.visited[v], bit);
      if (old & bit) atomicOr(err, ERR_DUP_NODE);
      atomicOr((unsigned long long *)&sd.prev[v], bit);  // seeds are not new at hop 1
      sd.plines[v >> MC_TOUCH_SHIFT] = 1;
      if (sd.local) sd.local[(int64_t)v * h.B + b] = (int32_t)j;
    }
  }
  if (!degree) return;  // whole grid
  const int64_t cnt = (h.f < 0 || d <= (int64_t)h.f) ? d : (int64_t)h.f;
  int64_t total;
  const int64_t eoff = block_excl_scan<THREADS>(cnt, &total);
  if (valid) {
    f_off[i] = o0;
    f_deg[i] = d;
    f_eoff[i] = eoff;
  }
  if (threadIdx.x == 0) tile_sum[t] = total;
}

// Exclusive scan of each batch's tile sums in place, a block per batch, and the
// batches' edges of the hop: for frontiers of more than TILES_DIRECT tiles in a batch.
// Up to that many the draw kernel adds the sums of its batch's earlier tiles itself,
// which costs no launch but grows with the square of the frontier (whole call, fan-out 1,
// adding / scanning: one mini-batch, 1024 tiles 383 / 391 us, 4096 688 / 703, 16384
// 1727 / 1738, 65536 5916 / 5318; 8 mini-batches, 4096 3072 / 3084, 16384 11772 / 11635;
// fan-out 5: 8 mini-batches, 4096 7279 / 7266, 16384 26492 / 26066).
constexpr int32_t TILES_DIRECT = 8192;
constexpr int TS_THREADS = 1024;
constexpr int TS_ITEMS = 8;
__global__ __launch_bounds__(TS_THREADS) void k_tile_scan(Hop h, int64_t *tile_sum,
                                                          int64_t *bounds) {
  const int b = blockIdx.x;
  const int32_t n = h.tstart[b + 1] - h.tstart[b];
  int64_t *p = tile_sum + h.tstart[b];
  int64_t carry = 0;
  for (int32_t c0 = 0; c0 < n; c0 += TS_THREADS * TS_ITEMS) {
    // a thread's items lie next to each other: one block scan per chunk
    const int32_t i0 = c0 + (int32_t)threadIdx.x * TS_ITEMS;
    int64_t v[TS_ITEMS], x = 0;
#pragma unroll
    for (int q = 0; q < TS_ITEMS; ++q) v[q] = i0 + q < n ? p[i0 + q] : 0;
#pragma unroll
    for (int q = 0; q < TS_ITEMS; ++q) x += v[q];
    int64_t total;
    int64_t run = carry + block_excl_scan<TS_THREADS>(x, &total);
#pragma unroll
    for (int q = 0; q < TS_ITEMS; ++q) {
      if (i0 + q < n) p[i0 + q] = run;
      run += v[q];
    }
    carry += total;
  }
  if (threadIdx.x == 0) bounds[b] = carry;
}

// Emits up to EMIT sampled edges whose neighbour IDs are already loaded: the
// edge stores, then a fire-and-forget atomicOr of the batch's bit into each
// neighbour's membership word (setting a bit that is already set changes
// nothing, and skipping the atomic for seen pairs would cost a dependent read
// of the word, which measures slower than the atomics it saves).  The atomics
// are what bounds the draws: 27 G/s on this chip whatever their locality, and
// half that where many meet in the words of the hubs.  So on hops with many
// draws a block keeps the nodes it has marked lately in LDS (tag, one per hash
// value; a block serves one batch) and leaves their atomics out.  The filter is
// plain reads and writes: a lost entry costs an atomic, and an entry is only
// ever there because its writer issues the atomic.  Last hop at 1M nodes, 32
// mini-batches (2.1M draws), without and with the filter: 261 and 208 us; 64
// mini-batches: 32M nodes (15M draws) 755 and 717, 100M nodes 805 and 814 (the hop
// before it 229 and 222); no difference on uniform graphs.
constexpr int EMIT = 8;
constexpr int TAG_BITS = 11;
constexpr int64_t TAG_MIN_DRAWS = 1 << 18;

__device__ __forceinline__ void emit_chunk(const int32_t (&u)[EMIT], const int64_t (&slot)[EMIT],
                                           int cnt, int b, int32_t parent, int32_t *edge_src,
                                           int32_t *edge_dst, uint64_t *visited, int64_t N,
                                           uint8_t *touched, uint32_t *err, int32_t *tag) {
  const unsigned long long bit = 1ull << b;
#pragma unroll
  for (int k = 0; k < EMIT; ++k) {
    if (k < cnt) {
      edge_src[slot[k]] = parent;
      edge_dst[slot[k]] = u[k];
    }
  }
#pragma unroll
  for (int k = 0; k < EMIT; ++k) {
    if (k >= cnt) continue;
    if (u[k] >= 0 && (int64_t)u[k] < N) {
      if (tag) {  // uniform
        int32_t *at = &tag[((uint32_t)u[k] * 0x9E3779B1u) >> (32 - TAG_BITS)];
        if (*at == u[k]) continue;
        *at = u[k];
      }
      atomicOr((unsigned long long *)&visited[u[k]], bit);
      if (touched) touched[u[k] >> MC_TOUCH_SHIFT] = 1;
    } else {
      atomicOr(err, ERR_NBR_RANGE);
    }
  }
}

// LPN lanes per frontier node (LPN = 1, 2, 4 or 8; more lanes when the
// frontier is small, so that short hops still keep enough loads in flight).
// Floyd's subset is built in registers (fully unrolled, so the arrays stay in
// VGPRs) when f <= FM, by every lane of the node; FM (8, 16 or 32) is the
// smallest capacity that holds the hop's fan-out, since the arrays' registers
// bound the waves per SIMD and so the loads in flight; each drawn position's rank among the f
// positions gives its slot, so no sort is needed, and lane `sub` takes the
// draws s with s mod LPN = sub.  Neighbour loads and membership atomics are
// issued EMIT at a time so their latencies overlap.  A block takes F_TILE/LPN
// consecutive entries of one tile.  The block of a batch's last tile leaves the
// batch's edges of this hop in bounds[b].  A
// node whose edges would pass edge_cap writes nothing; the host sees the
// overflow in the edge counts and reports it.
template <int LPN, int FM>
__global__ __launch_bounds__(THREADS) void k_hop_sample(
    Hop h, const int32_t *nodes, int64_t node_cap, const int32_t *idx, const int64_t *f_off,
    const int64_t *f_deg, const int64_t *f_eoff, const int64_t *tile_sum, int64_t *bounds,
    int64_t edge_cap, int32_t *edge_src, int32_t *edge_dst, uint64_t *visited, int64_t N,
    uint32_t *err) {
  const int32_t t = (int32_t)(blockIdx.x / LPN);
  const int part = (int)(blockIdx.x % LPN);
  const int b = tile_batch(h, t);
  const int32_t t0 = h.tstart[b];
  const int64_t j =
      (int64_t)(t - t0) * F_TILE + part * (F_TILE / LPN) + (int)threadIdx.x / LPN;
  const int64_t i = h.fstart[b] + j;
  const int sub = (int)threadIdx.x % LPN;
  const bool valid = i < h.fstart[b + 1];
  int64_t o0 = 0, d = 0, eoff = 0;
  if (valid) {
    o0 = f_off[i];
    d = f_deg[i];
    eoff = f_eoff[i];
  }
  __shared__ int32_t s_tag[1 << TAG_BITS];
  int32_t *tag = h.filter ? s_tag : nullptr;
  if (h.filter) {
    for (int q = threadIdx.x; q < (1 << TAG_BITS); q += THREADS) s_tag[q] = -1;
    __syncthreads();
  }
  int64_t before = 0;  // edges of the batch's earlier tiles
  if (h.scanned) {     // uniform
    before = tile_sum[t];
  } else if (t > t0) {  // uniform
    int64_t x = 0;
    for (int32_t q = t0 + (int32_t)threadIdx.x; q < t; q += THREADS) x += tile_sum[q];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    __shared__ int64_t s_x[THREADS / 64];
    if ((threadIdx.x & 63) == 0) s_x[threadIdx.x >> 6] = x;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < THREADS / 64; ++q) before += s_x[q];
  }
  if (!h.scanned && threadIdx.x == 0 && part == 0 && t + 1 == h.tstart[b + 1])
    bounds[b] = before + tile_sum[t];
  if (!valid) return;
  const int64_t p = h.fpos[b] + j;
  const int64_t first = h.ebase[b] + before + eoff;  // local index of the 1st edge
  const int64_t cnt = (h.f < 0 || d <= (int64_t)h.f) ? d : (int64_t)h.f;
  if (first + cnt > edge_cap) return;
  int64_t base = (int64_t)b * edge_cap + first;
  int32_t parent = (int32_t)p;
  int32_t u[EMIT];
  int64_t slot[EMIT];
  if (h.f < 0 || d <= (int64_t)h.f) {  // every neighbour, in CSR order
    // lane sub takes positions q0 + sub + LPN*k, so the lanes of a node read
    // consecutive positions in one instruction
    for (int64_t q0 = 0; q0 < d; q0 += (int64_t)LPN * EMIT) {
      int n = 0;
#pragma unroll
      for (int k = 0; k < EMIT; ++k) {
        const int64_t q = q0 + sub + (int64_t)LPN * k;
        slot[k] = base + q;
        u[k] = q < d ? idx[o0 + q] : 0;
        n += q < d ? 1 : 0;
      }
      emit_chunk(u, slot, n, b, parent, edge_src, edge_dst, visited, N, h.touched, err,
                 tag);
    }
    return;
  }
  const int32_t f = h.f;
  int32_t v = nodes[(int64_t)b * node_cap + p];
  uint64_t key = mix64(h.bstate[b] ^ (((uint64_t)(uint32_t)h.k << 32) | (uint64_t)(uint32_t)v));
  if (d > 0x7fffffffll) {  // positions are kept as 32-bit values
    if (sub == 0) atomicOr(err, ERR_CSR);
    return;
  }
  if (f <= FM) {
    uint32_t r[FM];
#pragma unroll
    for (int s = 0; s < FM; ++s) {
      r[s] = 0xffffffffu;
      if (s < f) {
        uint32_t j = (uint32_t)(d - f + s);
        uint64_t hs = mix64(key + GAMMA * (uint64_t)(s + 1));
        uint32_t tt = (uint32_t)__umul64hi(hs, (uint64_t)j + 1ull);
        bool seen = false;
#pragma unroll
        for (int m = 0; m < s; ++m) seen |= (r[m] == tt);
        r[s] = seen ? j : tt;
      }
    }
    // this lane's draws: s = j*LPN + sub for j = 0, 1, ... (a static j, so the
    // register arrays are indexed by constants only)
    constexpr int SPL = FM / LPN;
    uint32_t rv[SPL];
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      rv[j] = 0xffffffffu;
#pragma unroll
      for (int q = 0; q < LPN; ++q)
        if (q == sub) rv[j] = r[j * LPN + q];
    }
#pragma unroll
    for (int j0 = 0; j0 < SPL; j0 += EMIT) {
      if (j0 * LPN < f) {
        int n = 0;
#pragma unroll
        for (int k = 0; k < EMIT; ++k) {
          const int j = j0 + k;
          const bool mine = j < SPL && j * LPN + sub < f;
          const uint32_t x = j < SPL ? rv[j] : 0xffffffffu;
          int rank = 0;
#pragma unroll
          for (int m = 0; m < FM; ++m) rank += (m < f && r[m] < x) ? 1 : 0;
          slot[k] = base + rank;
          u[k] = mine ? idx[o0 + x] : 0;
          n += mine ? 1 : 0;
        }
        emit_chunk(u, slot, n, b, parent, edge_src, edge_dst, visited, N, h.touched, err,
                 tag);
      }
    }
    return;
  }
  // Larger fan-outs (one lane per node): the subset is built in this node's
  // edge slots, then sorted.
  if (sub != 0) return;
  int32_t *r = edge_dst + base;
  for (int s = 0; s < f; ++s) {
    int64_t j = d - f + s;
    uint64_t hs = mix64(key + GAMMA * (uint64_t)(s + 1));
    int32_t tt = (int32_t)__umul64hi(hs, (uint64_t)(j + 1));
    bool seen = false;
    for (int m = 0; m < s; ++m) seen |= (r[m] == tt);
    r[s] = seen ? (int32_t)j : tt;
  }
  for (int s = 1; s < f; ++s) {  // insertion sort
    int32_t x = r[s];
    int m = s - 1;
    while (m >= 0 && r[m] > x) {
      r[m + 1] = r[m];
      --m;
    }
    r[m + 1] = x;
  }
  for (int s0 = 0; s0 < f; s0 += EMIT) {
    const int n = f - s0 < EMIT ? f - s0 : EMIT;
#pragma unroll
    for (int k = 0; k < EMIT; ++k) {
      slot[k] = base + s0 + k;
      u[k] = k < n ? idx[o0 + r[s0 + k]] : 0;
    }
    emit_chunk(u, slot, n, b, parent, edge_src, edge_dst, visited, N, h.touched, err,
                 tag);
  }
}

// List segments: batch b's segment starts at local index seg0[b].
struct Segs {
  int B;
  int64_t start[DG_MAX_BATCHES + 1];  // prefix of segment lengths
  int64_t seg0[DG_MAX_BATCHES];
};

// Records the local index of every node of the given list segments.
__global__ __launch_bounds__(THREADS) void k_table_insert(Segs L, const int32_t *nodes,
                                                          int64_t node_cap, LocalTable table,
                                                          uint32_t *err) {
  int64_t i = (int64_t)blockIdx.x * THREADS + threadIdx.x;
  if (i >= L.start[L.B]) return;
  int b = find_batch_wave(L.start, L.B, i);
  int64_t j = L.seg0[b] + (i - L.start[b]);
  if (!lt_insert(table, nodes[(int64_t)b * node_cap + j], b, j)) atomicOr(err, ERR_INTERNAL);
}

// ---------------------------------------------------------------- last-hop relabelling by search
// The last hop's new nodes form one ascending segment at the end of each
// batch's list, so a last-hop edge whose neighbour is one of them gets its
// local index as the neighbour's rank in that segment; only edges into nodes
// listed earlier look a table up (the direct one, or the hash table, which then
// holds the earlier nodes alone).  Each batch has a sparse index of its segment
// (the first element of every block of S); a block of threads stages its batch's
// index in LDS, searches it, and reads one block of the list (from L2: thread
// blocks are ordered so that all of a batch run on one XCD).
//
// The segment is read where it lies, in blocks that start at multiples of S in
// memory, so the first and the last may reach past it.  (A padded copy of every
// segment takes 55 us for 10M entries (32M nodes, 64 batches), the index alone 13;
// blocks at any alignment cost the search 10 to 40%, two lines per block.)
constexpr int RL_THREADS = 512;
constexpr int RL_CHUNKS = 4;          // edge chunks per block (one staging of the index)
constexpr int RL_SPARSE_MAX = 16384;  // sparse-index entries per batch (64 KB of LDS)
constexpr int RL_S_MAX_LOG2 = 6;      // block length S = 16, 32 or 64
constexpr int RL_S_MIN_LOG2 = 4;
constexpr int64_t RL_SEGMENT_MAX =
    (int64_t)(RL_SPARSE_MAX - 1) << RL_S_MAX_LOG2;  // one block more where it starts inside one

// edges per thread for block length 2^SLOG2 (keeps the block reads within registers)
__host__ __device__ constexpr int rl_edges(int slog2) { return slog2 <= 4 ? 4 : (slog2 == 5 ? 2 : 1); }

// Sparse-index entries a batch has room for: the index lies in the frontier
// arrays, which are free by then (8 bytes per list entry).  m nodes need at most
// (m + 30) / 16 entries, and m <= node_cap.
inline int rl_sparse_cap(int64_t node_cap) {
  return (int)(2 * node_cap < RL_SPARSE_MAX ? 2 * node_cap : RL_SPARSE_MAX);
}

struct LastHop {
  int B;
  int s_log2;                           // block length S = 2^s_log2
  int chunks;                           // edge chunks per block
  int32_t bstart[DG_MAX_BATCHES + 1];   // logical blocks before batch b
  int32_t m[DG_MAX_BATCHES];            // length of b's last-hop segment
  int32_t a[DG_MAX_BATCHES];            // its first node's place in its block
  int32_t ecount[DG_MAX_BATCHES];       // b's last-hop edges
  int64_t seg0[DG_MAX_BATCHES];         // local index of the segment's first node
  int64_t e0[DG_MAX_BATCHES];           // index of b's first last-hop edge
  int32_t rstart[DG_MAX_BATCHES + 1];   // sparse-index entries before batch b
};

// A node listed before the last hop: its local index by the direct table or by
// the hash table (< 0: absent).
struct OlderNodes {
  const int32_t *local;  // nullable: [N][B]
  LocalTable table;
};
template <bool DIRECT>
__device__ __forceinline__ int64_t older_index(const OlderNodes &o, int32_t u, int b, int B) {
  return DIRECT ? (int64_t)o.local[(int64_t)u * B + b] : lt_find(o.table, u, b);
}

// What the relabelling does beside the last hop's search: three independent
// parts of one launch, each a run of its blocks.  As three launches the whole step
// took 135.5 us against 131 (10,000 nodes), 213 against 208 (one mini-batch at 1M
// nodes) and 1092 against 1084 (32 of them).
struct TailEdges {  // edges whose neighbours the table knows: of b, the first ones
  int B;
  unsigned blocks;
  int64_t start[DG_MAX_BATCHES + 1];  // prefix of the edges
  int64_t limit[DG_MAX_BATCHES];      // b's local indices (of pairs too) lie below
};
struct TailSparse {  // the index of the last-hop segments
  unsigned blocks;
  int s_log2, cap;
  int32_t rstart[DG_MAX_BATCHES + 1];
  int32_t a[DG_MAX_BATCHES];
  int64_t seg0[DG_MAX_BATCHES];
  int32_t *sparse;
};
struct TailLoc {  // P_b and the address tables of the packed pairs
  unsigned blocks;
  int64_t start[DG_MAX_BATCHES + 1];  // packed_ptr
  const uint64_t *pinfo;
  int32_t *packed_ids, *loc;
};

// Edges: sampled neighbours' global IDs -> local indices through the direct [N][B]
// table or the group's (node, batch) hash table.  Every looked-up pair was
// entered when its node entered the batch; the range check guards that.
// Sparse index: the first element of every block of each batch's last-hop segment.
// Packed pairs, after a fused compaction: packed row i of chunk b holds node u (low
// half of pinfo[i]), which is entry j of nodes_b, with j the list slot in the high
// half for a pair new at the last hop, else u's local index in the direct table;
// packed_ids[i] = u and loc_b[j] = i - packed_ptr[b], u's rank in P_b.  Every
// non-cached list entry is reached once this way (its pair is in P_b).
template <bool DIRECT>
__global__ __launch_bounds__(THREADS) void k_relabel_tail(TailEdges te, TailSparse ts, TailLoc tl,
                                                          const int32_t *nodes, int64_t node_cap,
                                                          int64_t edge_cap, int32_t *edge_dst,
                                                          OlderNodes older, int64_t N,
                                                          uint32_t *err) {
  unsigned blk = blockIdx.x;
  if (blk < te.blocks) {
    const int64_t i = (int64_t)blk * THREADS + threadIdx.x;
    if (i >= te.start[te.B]) return;
    const int b = find_batch_wave(te.start, te.B, i);
    const int64_t e = (int64_t)b * edge_cap + (i - te.start[b]);
    const int32_t u = edge_dst[e];
    if (u < 0 || (int64_t)u >= N) return;  // already reported
    const int64_t j = older_index<DIRECT>(older, u, b, te.B);
    if (j < 0 || j >= te.limit[b]) {
      atomicOr(err, ERR_INTERNAL);
      return;
    }
    edge_dst[e] = (int32_t)j;
    return;
  }
  blk -= te.blocks;
  if (blk < ts.blocks) {
    const int32_t i = (int32_t)(blk * THREADS + threadIdx.x);
    if (i >= ts.rstart[te.B]) return;
    int b = 0, top = te.B;  // invariant rstart[b] <= i < rstart[top]
    while (top - b > 1) {
      const int mid = (b + top) >> 1;
      if (ts.rstart[mid] <= i) b = mid; else top = mid;
    }
    const int32_t r = i - ts.rstart[b];
    const int32_t at = max((r << ts.s_log2) - ts.a[b], 0);
    ts.sparse[(int64_t)b * ts.cap + r] = nodes[(int64_t)b * node_cap + ts.seg0[b] + at];
    return;
  }
  blk -= ts.blocks;
  const int64_t i = (int64_t)blk * THREADS + threadIdx.x;
  if (i >= tl.start[te.B]) return;
  const int b = find_batch_wave(tl.start, te.B, i);
  const uint64_t x = tl.pinfo[i];
  const int32_t u = (int32_t)(uint32_t)x;
  int64_t j = (int32_t)(x >> 32);
  tl.packed_ids[i] = u;
  if (j < 0) j = older_index<DIRECT>(older, u, b, te.B);
  if (j < 0 || j >= te.limit[b]) {
    atomicOr(err, ERR_INTERNAL);
    return;
  }
  tl.loc[(int64_t)b * node_cap + j] = (int32_t)(i - tl.start[b]);
}

typedef uint32_t u4_any __attribute__((ext_vector_type(4), aligned(4)));

// v of the lane whose number differs in bit X (1, 2, 4 or 8).
template <int X>
__device__ __forceinline__ int xor_lane(int v) {
  if constexpr (X == 1) return __builtin_amdgcn_update_dpp(0, v, 0xb1, 0xf, 0xf, false);
  else if constexpr (X == 2) return __builtin_amdgcn_update_dpp(0, v, 0x4e, 0xf, 0xf, false);
  else return __builtin_amdgcn_ds_swizzle(v, (X << 10) | 0x1f);
}

// The elements of the S-element window seg[start..] below u, and whether it holds
// u (bit 16), for each lane's u and start; pos = 0: the lane has no window.  What
// bounds the search is lines per load instruction: the windows are scattered.
// S = 16: a lane reads its own 64 bytes, and lanes without a window read nothing
// (15M last-hop edges of 64 mini-batches at 32M nodes: 228 us, 250 when they
// read).  Longer windows are read by S/4 lanes together, 16 bytes each, so that an
// instruction touches 256/S of them and not 64 (S = 32, 3M edges: 115 us
// against 153; at S = 16 the shuffles cost what that gains, 247 us).
template <int S>
__device__ __forceinline__ int window_count(const int32_t *seg, int u, int start, int pos,
                                            int lane) {
  if constexpr (S == 16) {
    int t = 0;
    if (pos > 0) {
      const u4_any *bp = reinterpret_cast<const u4_any *>(seg + start);
#pragma unroll
      for (int q = 0; q < S / 4; ++q) {
        const u4_any x = bp[q];
        const int a0 = (int)x.x, a1 = (int)x.y, a2 = (int)x.z, a3 = (int)x.w;
        t += (a0 < u) + (a1 < u) + (a2 < u) + (a3 < u);
        t |= (int)((a0 == u) | (a1 == u) | (a2 == u) | (a3 == u)) << 16;
      }
    }
    return t;
  }
  constexpr int G = S / 4, PER = 64 / G;  // lanes per window, windows per load
  int mine = 0;
#pragma unroll
  for (int it = 0; it < G; ++it) {
    const int src = it * PER + lane / G;
    const int uu = __shfl(u, src, 64), st = __shfl(start, src, 64);
    const u4_any x = *reinterpret_cast<const u4_any *>(seg + st + 4 * (lane % G));
    const int a0 = (int)x.x, a1 = (int)x.y, a2 = (int)x.z, a3 = (int)x.w;
    int t = (a0 < uu) + (a1 < uu) + (a2 < uu) + (a3 < uu) +
            ((int)((a0 == uu) | (a1 == uu) | (a2 == uu) | (a3 == uu)) << 16);
    t += xor_lane<1>(t);
    t += xor_lane<2>(t);
    if constexpr (G >= 8) t += xor_lane<4>(t);
    if constexpr (G >= 16) t += xor_lane<8>(t);
    const int got = __shfl(t, (lane % PER) * G, 64);
    if (lane / PER == it) mine = got;
  }
  return mine;
}

template <int SLOG2, bool DIRECT>
__global__ __launch_bounds__(RL_THREADS) void k_relabel_last(LastHop h, const int32_t *nodes,
                                                             int64_t node_cap,
                                                             const int32_t *sparse,
                                                             int sparse_cap, int64_t edge_cap,
                                                             int32_t *edge_dst, OlderNodes older,
                                                             int64_t N, uint32_t *err) {
  constexpr int S = 1 << SLOG2;
  constexpr int EPT = rl_edges(SLOG2);
  constexpr int PER_CHUNK = RL_THREADS * EPT;
  extern __shared__ int32_t s_sp[];
  // Each XCD takes one contiguous run of logical blocks, i.e. whole batches, one
  // after the other.
  const int lb = (int)xcd_block(blockIdx.x, gridDim.x);
  if (lb >= h.bstart[h.B]) return;  // whole block
  int b = 0;
  while (b + 1 < h.B && h.bstart[b + 1] <= lb) ++b;
  const int m = h.m[b], a = h.a[b];
  const int R = h.rstart[b + 1] - h.rstart[b];
  const int32_t *sp = sparse + (int64_t)b * sparse_cap;
  for (int i = threadIdx.x; i < R; i += RL_THREADS) s_sp[i] = sp[i];
  __syncthreads();
  int top = 1;  // highest power of two <= R (uniform)
  while (top * 2 <= R) top *= 2;
  const int64_t eend = h.e0[b] + h.ecount[b];
  int32_t *ed = edge_dst + (int64_t)b * edge_cap;
  const int64_t seg0 = h.seg0[b];
  const int32_t *seg = nodes + (int64_t)b * node_cap + seg0;
  for (int ch = 0; ch < h.chunks; ++ch) {
    const int64_t ebase = h.e0[b] +
                          ((int64_t)(lb - h.bstart[b]) * h.chunks + ch) * PER_CHUNK + threadIdx.x;
    if (ebase - threadIdx.x >= eend) break;  // uniform
    int32_t u[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      const int64_t e = ebase + (int64_t)k * RL_THREADS;
      u[k] = e < eend ? ed[e] : -1;
    }
    // pos = number of sparse entries <= u: the block that may hold u is pos - 1.
    // No branch between the reads of a step, so that they are in flight together.
    int pos[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) pos[k] = 0;
    if (R > 0) {  // uniform
      for (int step = top; step > 0; step >>= 1) {
        int32_t x[EPT];
#pragma unroll
        for (int k = 0; k < EPT; ++k) x[k] = s_sp[min(pos[k] + step, R) - 1];
#pragma unroll
        for (int k = 0; k < EPT; ++k)
          pos[k] += pos[k] + step <= R && x[k] <= u[k] ? step : 0;
      }
    }
    // The block's elements below u and whether it holds u.  A window that would
    // reach past the segment is moved inside it: what it gains lies below u (on
    // the left) or above (on the right).
    int below[EPT];
    bool found[EPT];
    if (m >= S) {  // uniform
#pragma unroll
      for (int k = 0; k < EPT; ++k) {
        const int start = min(max(((pos[k] - 1) << SLOG2) - a, 0), m - S);
        const int t = window_count<S>(seg, u[k], start, pos[k], (int)threadIdx.x & 63);
        below[k] = start + (t & 0xffff);
        found[k] = t >> 16;
      }
    } else {
#pragma unroll
      for (int k = 0; k < EPT; ++k) {
        below[k] = 0;
        found[k] = false;
        for (int q = 0; q < m; ++q) {
          below[k] += seg[q] < u[k];
          found[k] |= seg[q] == u[k];
        }
      }
    }
    // The lookups of the nodes listed before the hop, all before any is used.
    int64_t j[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      const bool ok = u[k] >= 0 && (int64_t)u[k] < N;  // bad IDs already reported
      j[k] = seg0 + below[k];
      if (!ok) j[k] = -2;
      else if (!found[k]) j[k] = older_index<DIRECT>(older, u[k], b, h.B);
    }
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      const int64_t e = ebase + (int64_t)k * RL_THREADS;
      if (j[k] == -2 || e >= eend) continue;
      if (!found[k] && (j[k] < 0 || j[k] >= seg0)) {
        atomicOr(err, ERR_INTERNAL);
        continue;
      }
      ed[e] = (int32_t)j[k];
    }
  }
}

// Host staging block (int64 entries): the hop's edges per batch, compaction totals,
// error word.
constexpr int ST_BOUNDS = 0;                              // [B]
constexpr int ST_TOTALS = ST_BOUNDS + DG_MAX_BATCHES + 1; // [B+4]
constexpr int ST_ERR = ST_TOTALS + DG_MAX_BATCHES + 4;
constexpr int ST_PTOTALS = ST_ERR + 1;                      // [B+4] packing's, fused pass
constexpr int ST_SIZE = ST_PTOTALS + DG_MAX_BATCHES + 4;

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + THREADS - 1) / THREADS); }

constexpr uint32_t SAMPLE_FLAGS =
    DG_SAMPLE_LAYERED | DG_SAMPLE_DIRECT | DG_SAMPLE_EXIT_CLEAR | DG_SAMPLE_ENTRY_CLEAR;

struct SampleWs {
  uint32_t *err;
  uint64_t *visited, *prev;
  uint8_t *plines;  // lines of prev that hold a bit (a byte per 8 nodes)
  uint8_t *touched;  // touched marks (a byte per 2^MC_TOUCH_SHIFT nodes)
  size_t state_words;  // 8-byte words from prev to the end of touched
  int64_t *f_off, *f_deg, *f_eoff, *tiles;
  LocalTable table;  // hash relabelling
  int32_t *local;    // direct relabelling: [N][B]
  int64_t *small;    // staging for a few counts
  MaskScan ms;
};

// The state that DG_SAMPLE_EXIT_CLEAR leaves clear (err, prev, plines, touched; with
// visited in the caller's membership words) comes first, at places that depend on N
// alone.
void carve_sample(SampleWs &w, Carve &c, int64_t N, int B, int64_t node_cap, bool direct,
                  int rounds) {
  int64_t fmax = (int64_t)B * node_cap;  // frontier entries never exceed the node lists
  w.err = c.take<uint32_t>(64);
  w.visited = c.take<uint64_t>((size_t)N);
  const size_t state = c.used;
  w.prev = c.take<uint64_t>((size_t)N);
  w.plines = c.take<uint8_t>((size_t)mc_touch_bytes(N));
  w.touched = c.take<uint8_t>((size_t)mc_touch_bytes(N));
  w.state_words = (c.used - state) / 8;
  w.f_off = c.take<int64_t>((size_t)fmax);
  w.f_deg = c.take<int64_t>((size_t)fmax);
  w.f_eoff = c.take<int64_t>((size_t)fmax);
  // tiles of one batch each, none of them empty
  const int64_t tiles = fmax / F_TILE + B;
  w.tiles = c.take<int64_t>((size_t)(tiles < fmax ? tiles : fmax));
  w.table.bits = direct ? 0 : lt_bits_for(fmax);
  w.table.slots = direct ? nullptr : c.take<uint64_t>((size_t)1 << w.table.bits);
  w.local = direct ? c.take<int32_t>((size_t)N * (size_t)B) : nullptr;
  w.small = c.take<int64_t>(ST_SIZE);
  w.ms = MaskScan{};
  w.ms.N = N;
  w.ms.B = B;
  mask_scan_carve(w.ms, c, rounds);
}

int check_err(uint32_t *err_dev, hipStream_t s) {
  uint32_t bits = 0;
  DG_TRY(read_to_host(&bits, err_dev, sizeof(bits), s));
  if (bits) return set_error(DG_EINVAL, "invalid input data: %s", describe_device_error(bits));
  return DG_OK;
}

}  // namespace
}  // namespace dg

using namespace dg;

extern "C" int dg_sample_bounds(int64_t num_nodes, int64_t num_edges, int32_t S,
                                const int32_t *fanouts, int32_t K, uint32_t flags,
                                int64_t *node_cap, int64_t *edge_cap) {
  if (!node_cap || !edge_cap || (K > 0 && !fanouts) || S < 1 || K < 0 || num_nodes < 1 ||
      num_edges < 0 || (flags & ~SAMPLE_FLAGS))
    return set_error(DG_EINVAL, "dg_sample_bounds: bad argument");
  const bool layered = flags & DG_SAMPLE_LAYERED;
  // Saturating arithmetic: once a count reaches its graph bound it stays there.
  // n = nodes so far, front = nodes that sample at the next hop; per hop the
  // edges are distinct CSR edges (each frontier node samples once), so a hop
  // adds at most min(f * front, E) edges.
  const int64_t big = INT64_MAX / 4;
  int64_t n = S, e = 0, front = S;
  for (int k = 0; k < K; ++k) {
    const int32_t f = fanouts[k];
    int64_t hop_e = f < 0 ? num_edges : (front > big / (f > 0 ? f : 1) ? big : front * f);
    if (hop_e > num_edges) hop_e = num_edges;
    e = e > big - hop_e ? big : e + hop_e;
    const int64_t grown = n > big - hop_e ? big : n + hop_e;
    front = layered ? (grown < num_nodes ? grown : num_nodes) : hop_e;
    n = grown < num_nodes ? grown : num_nodes;
    if (front > num_nodes) front = num_nodes;
  }
  // without layering a node samples at most once, so a batch's edges are
  // distinct CSR edges
  if (!layered && e > num_edges) e = num_edges;
  *node_cap = n;
  *edge_cap = e < 1 ? 1 : e;
  return DG_OK;
}

extern "C" size_t dg_sample_workspace_bytes(int64_t num_nodes, int32_t B, int64_t node_cap,
                                            int64_t edge_cap, uint32_t flags) {
  (void)edge_cap;
  if (num_nodes < 1 || B < 1 || B > DG_MAX_BATCHES || node_cap < 1 || (flags & ~SAMPLE_FLAGS))
    return 0;
  return mc_most_bytes(num_nodes, [&](int64_t n) {
    Carve c(nullptr);
    SampleWs w;
    carve_sample(w, c, n, B, node_cap, (flags & DG_SAMPLE_DIRECT) != 0, mc_rounds(n));
    return c.used;
  });
}

namespace dg {
namespace {

// Event indices of a sampling call's phases (read once the call's work is done).
struct SampleMarks {
  int start = -1, r0 = -1, r1 = -1, nhop = 0;
  int hop[8][3];
};

// Packing state of dg_sample_pack_group, carved from its packing workspace:
// what the fused last hop writes besides sampling's outputs, and what it
// reports back.
struct PackInto {
  PackWs pw;          // packing's workspace (last in the carve, see carve_sample_pack)
  size_t pw_offset;   // its offset in the packing workspace
  uint64_t *pinfo;    // [pinfo_cap] node and list slot of each packed pair (fused pass)
  int64_t pinfo_cap;
  int32_t *cw_slot;   // the fused pass's cache slot per listed word
  uint8_t *lines;     // member lines, for a group packed by packing's own passes
  int64_t unc_cap, pair_cap;
  int64_t *packed_ptr;
  int64_t packed_cap;
  int32_t *packed_ids;
  int32_t *group_unique;
  int64_t unique_cap;
  // set by sample_impl
  bool fits = false;                  // the totals match and fit the outputs
  bool loc_done = false;              // P_b and the address tables are queued
  bool fused = false;                 // the last hop's compaction did packing's pass
  int64_t ptot[DG_MAX_BATCHES + 4];  // packing's row totals (fused)
  uint32_t *err = nullptr;            // sampling's device error word, not yet checked
  uint64_t *visited = nullptr;        // the membership words sampling used
  int32_t *local = nullptr;           // the direct table (DG_SAMPLE_DIRECT)
};

void carve_sample_pack(PackInto &pk, Carve &c, int64_t N, int B, int64_t node_cap, int rounds) {
  const int64_t total = (int64_t)B * node_cap;
  pk.pinfo = c.take<uint64_t>((size_t)total);
  pk.pinfo_cap = total;
  pk.cw_slot = c.take<int32_t>((size_t)mc_pad_nodes(N));
  pk.lines = c.take<uint8_t>((size_t)mc_touch_bytes(N));
  pk.pw_offset = c.used;  // packing's own workspace last: the unfused path hands it on whole
  carve_pack(pk.pw, c, N, B, total, rounds);
  pk.unc_cap = (total < N ? total : N) + 1;
  pk.pair_cap = total + 1;
}

int sample_impl(const dg_csr *g, const int32_t *seeds, int32_t B, int32_t S, int64_t batch_base,
                const int32_t *fanouts, int32_t K, uint64_t rng_seed, uint32_t flags,
                int64_t node_cap, int32_t *nodes, int64_t *hop_ptr, int64_t edge_cap,
                int32_t *edge_src, int32_t *edge_dst, int64_t *edge_ptr, uint64_t *membership,
                uint8_t *member_lines, const int32_t *cache_slot, int32_t *loc, void *ws,
                size_t ws_bytes, hipStream_t stream, dg_sizes *sizes, PhaseTimer &tm,
                SampleMarks &mk, PackInto *pk) {
  if (!g || !seeds || !nodes || !hop_ptr || !edge_src || !edge_dst || !edge_ptr || !sizes ||
      (K > 0 && !fanouts))
    return set_error(DG_EINVAL, "dg_sample_group: null pointer argument");
  if (!cache_slot != !loc)
    return set_error(DG_EINVAL, "dg_sample_group: cache_slot and loc go together");
  if (!g->offsets || (g->num_edges > 0 && !g->indices) || g->num_nodes < 1 ||
      g->num_nodes > 0x7fffffffll || g->num_edges < 0)
    return set_error(DG_EINVAL, "dg_sample_group: bad CSR description");
  if (flags & ~SAMPLE_FLAGS)
    return set_error(DG_EINVAL, "dg_sample_group: unknown flags 0x%x", flags);
  const bool layered = flags & DG_SAMPLE_LAYERED;
  const bool direct = flags & DG_SAMPLE_DIRECT;
  const bool entry_clear = flags & DG_SAMPLE_ENTRY_CLEAR;
  const bool exit_clear = flags & DG_SAMPLE_EXIT_CLEAR;
  if (entry_clear && !membership)
    return set_error(DG_EINVAL, "dg_sample_group: DG_SAMPLE_ENTRY_CLEAR needs membership");
  if (B < 1 || B > DG_MAX_BATCHES || S < 1 || K < 0 || node_cap < S || edge_cap < 0 ||
      (int64_t)S > g->num_nodes)
    return set_error(DG_EINVAL, "dg_sample_group: bad sizes (B=%d S=%d K=%d node_cap=%lld)", B,
                     S, K, (long long)node_cap);
  if (node_cap > LT_MAX_VALUE)
    return set_error(DG_EINVAL, "dg_sample_group: node_cap above 2^27 - 1 is not supported");
  // Short tiles need a larger count matrix: where it does not fit (or packing's
  // workspace has longer ones), the longest.
  SampleWs w;
  size_t need_ws = 0;
  for (int rounds : {pk ? pk->pw.ms.rounds : mc_rounds(g->num_nodes), MC_ROUNDS_MAX}) {
    Carve c(ws);
    carve_sample(w, c, g->num_nodes, B, node_cap, direct, rounds);
    need_ws = c.used;
    if (need_ws <= ws_bytes) break;
  }
  if (!ws || ws_bytes < need_ws || ((uintptr_t)ws & 255))
    return set_error(DG_EWORKSPACE, "dg_sample_group: workspace needs %zu bytes, 256-aligned",
                     need_ws);

  const int64_t N = g->num_nodes, E = g->num_edges;
  hipStream_t s = stream;
  w.ms.err = w.err;

  memset(sizes, 0, sizeof(*sizes));
  sizes->packed_rows = sizes->unique_nodes = sizes->unique_packed = -1;
  sizes->exact = 1;
  mk.nhop = 0;
  mk.start = tm.mark();

  int rc;
  if (membership) w.visited = membership;
  // The error word, visited and prev with its lines, and the touched marks must
  // start all-zero: cleared here unless the caller asserts that they already are
  // (see DG_SAMPLE_ENTRY_CLEAR).
  if (!entry_clear) {
    ZeroRanges z;
    z.add(w.err, 32);
    z.add(w.visited, (size_t)N);
    z.add(w.prev, w.state_words);
    if ((rc = zero_ranges(z, s))) return rc;
  }
  bool prev_cleared = false;  // the last hop's count pass zeroed prev
  bool lines_done = false;    // the last hop's count pass wrote member_lines
  bool rl_search = false;     // the last hop's edges are relabelled by search
  int64_t n_b[DG_MAX_BATCHES], e_b[DG_MAX_BATCHES];
  for (int b = 0; b < B; ++b) {
    n_b[b] = S;
    e_b[b] = 0;
    hop_ptr[(int64_t)b * (K + 2) + 0] = 0;
    hop_ptr[(int64_t)b * (K + 2) + 1] = S;
  }

  Hop h;
  memset(&h, 0, sizeof(h));
  h.B = B;
  for (int b = 0; b < B; ++b)
    h.bstate[b] = mix64(rng_seed + GAMMA * ((uint64_t)(batch_base + b) + 1ull));
  int64_t fbeg[DG_MAX_BATCHES], fend[DG_MAX_BATCHES];
  for (int b = 0; b < B; ++b) {
    fbeg[b] = 0;
    fend[b] = S;
  }
  // Frontier pass of the hop that h describes; the first one also enters the
  // seeds (bad seeds are reported at the first hop's round trip).
  auto frontier = [&](bool seeding, bool degree) {
    const SeedInit sd{seeds, S, nodes, w.visited, w.prev, w.plines, w.local, cache_slot, loc};
    const dim3 grid((unsigned)h.tstart[B]);
    const bool apart = seeding && degree && h.fstart[B] >= SEEDS_APART;
    if (seeding)
      hipLaunchKernelGGL(k_frontier<true>, grid, dim3(THREADS), 0, s, h, sd, degree && !apart,
                         nodes, node_cap, g->offsets, N, E, w.f_off, w.f_deg, w.f_eoff, w.tiles,
                         w.err);
    if (!seeding || apart)
      hipLaunchKernelGGL(k_frontier<false>, grid, dim3(THREADS), 0, s, h, sd, degree, nodes,
                         node_cap, g->offsets, N, E, w.f_off, w.f_deg, w.f_eoff, w.tiles, w.err);
  };
  // Frontier positions, and their tiles, of the next hop.
  auto lay_out = [&] {
    h.fstart[0] = 0;
    h.tstart[0] = 0;
    for (int b = 0; b < B; ++b) {
      h.fpos[b] = fbeg[b];
      h.fstart[b + 1] = h.fstart[b] + (fend[b] - fbeg[b]);
      h.tstart[b + 1] = h.tstart[b] + (int32_t)((fend[b] - fbeg[b] + F_TILE - 1) / F_TILE);
      h.ebase[b] = e_b[b];
    }
  };
  bool seeded = false;
  for (int k = 1; k <= K; ++k) {
    for (int b = 0; b < B; ++b) edge_ptr[(int64_t)b * (K + 1) + (k - 1)] = e_b[b];
    const int32_t f = fanouts[k - 1];
    h.f = f;
    h.k = k;
    lay_out();
    const int64_t ftot = h.fstart[B];
    int64_t new_b[DG_MAX_BATCHES];
    if (ftot == 0 || f == 0) {
      for (int b = 0; b < B; ++b) new_b[b] = 0;
    } else {
      const int ev0 = tm.mark();
      // A hop whose edges can reach at most N/16 nodes marks the mask lines it
      // touches (a byte store per edge), and its count pass reads only those.
      // On larger hops the stores cost more time than the lines they spare.
      // The last hop never marks when the call must write the member-lines map
      // or leave prev clear: its count pass then reads every word anyway and
      // does both on the way, where marks would need a pass over the whole mask
      // for the map and a fill of prev afterwards.
      const int64_t ebound = f < 0 ? E : ftot * (int64_t)f;
      h.filter = ebound >= TAG_MIN_DRAWS;
      // With a packing state (and the direct table, which gives older pairs'
      // list slots) the last hop's compaction also does packing's pass.
      const bool fuse = pk && direct && k == K;
      const bool full_last = k == K && (member_lines || exit_clear || fuse);
      h.touched = (ebound <= N / 16 && !full_last) ? w.touched : nullptr;
      frontier(!seeded, true);
      seeded = true;
      h.scanned = 0;
      for (int b = 0; b < B; ++b) h.scanned |= h.tstart[b + 1] - h.tstart[b] > TILES_DIRECT;
      if (h.scanned)
        hipLaunchKernelGGL(k_tile_scan, dim3(B), dim3(TS_THREADS), 0, s, h, w.tiles,
                           w.small + ST_BOUNDS);
      DG_HIP(hipGetLastError());
      // lanes per frontier node: up to 8 while the frontier has fewer than 2^20
      // entries (never more lanes than draws; fan-outs above FMAX keep one)
      int lpn = 1;
      while (lpn < 8 && ftot * lpn < (1 << 20) && (f < 0 || (f <= FMAX && 2 * lpn <= f)))
        lpn *= 2;
      const dim3 hg((unsigned)(h.tstart[B] * lpn)), hb(THREADS);
      // register-path capacity: the smallest that holds f (8 when f does not
      // take the register path at all)
      const int fm = (f < 0 || f > FMAX || f <= 8) ? 8 : (f <= 16 ? 16 : 32);
      auto launch = [&](auto lpn_c, auto fm_c) {
        hipLaunchKernelGGL((k_hop_sample<decltype(lpn_c)::value, decltype(fm_c)::value>), hg, hb,
                           0, s, h, nodes, node_cap, g->indices, w.f_off, w.f_deg, w.f_eoff,
                           w.tiles, w.small + ST_BOUNDS, edge_cap, edge_src, edge_dst,
                           w.visited, N, w.err);
      };
      auto launch_fm = [&](auto lpn_c) {
        if (fm == 8) launch(lpn_c, std::integral_constant<int, 8>());
        else if (fm == 16) launch(lpn_c, std::integral_constant<int, 16>());
        else launch(lpn_c, std::integral_constant<int, 32>());
      };
      if (lpn == 8) launch_fm(std::integral_constant<int, 8>());
      else if (lpn == 4) launch_fm(std::integral_constant<int, 4>());
      else if (lpn == 2) launch_fm(std::integral_constant<int, 2>());
      else launch_fm(std::integral_constant<int, 1>());
      DG_HIP(hipGetLastError());
      const int ev1 = tm.mark();
      // new nodes of this hop, per batch, ascending; the write pass needs only
      // the list starts known before the hop, so it is queued before the host
      // reads this hop's counts (it stops at each list's capacity)
      w.ms.mask = w.visited;
      w.ms.prev = w.prev;
      w.ms.plines = w.plines;
      w.ms.keep_prev = k < K;  // after the last hop nothing reads prev
      w.ms.touched = h.touched;
      w.ms.touched_clear = h.touched;  // read by this hop's count pass only
      // With DG_SAMPLE_EXIT_CLEAR the last hop's count pass zeroes every prev
      // word it reads; that is all non-zero ones (prev is a subset of visited)
      // unless touched marks leave some lines unread.
      w.ms.clear_prev = exit_clear && k == K && !h.touched;
      prev_cleared = w.ms.clear_prev;
      // the last hop's count pass reads every word unless touched marks limit it
      w.ms.lines_out = (member_lines && k == K && !h.touched) ? member_lines : nullptr;
      lines_done = w.ms.lines_out != nullptr;
      w.ms.cache_slot = nullptr;
      w.ms.totals = w.small + ST_TOTALS;
      w.ms.err_stage = w.small + ST_ERR;
      FuseScan F;
      if (fuse) {
        MaskScan &vp = pk->pw.ms;
        vp.totals = w.small + ST_PTOTALS;
        vp.err_stage = nullptr;
        vp.err = w.err;
        memset(&F, 0, sizeof(F));
        F.mask = w.visited;
        F.prev = w.prev;
        F.plines = w.plines;
        F.cache_slot = cache_slot;
        F.N = N;
        F.B = B;
        F.rounds = w.ms.rounds;
        F.nblk = w.ms.nblk;
        F.clear_prev = w.ms.clear_prev;
        F.err = w.err;
        F.wcnt = w.ms.wcnt;
        F.cw_mask = w.ms.cw_mask;
        F.cw_new = vp.cw_mask;
        F.cw_off = w.ms.cw_off;
        F.cw_slot = pk->cw_slot;
        F.cnt_s = w.ms.cnt;
        F.wpre_s = w.ms.wpre;
        F.cnt_p = vp.cnt;
        F.wpre_p = vp.wpre;
        F.base_s = w.ms.base;
        F.base_p = vp.base;
        w.ms.lines_out = nullptr;
        lines_done = false;
        if ((rc = fuse_scan_count(F, w.ms, vp, s))) return rc;
      } else if ((rc = mask_scan_count(w.ms, s))) {
        return rc;
      }
      for (int b = 0; b < B; ++b) {
        w.ms.seg_base[b] = (int64_t)b * node_cap + n_b[b];
        w.ms.seg_end[b] = (int64_t)(b + 1) * node_cap;
        w.ms.local_base[b] = n_b[b];
      }
      // The last hop's edges find their new neighbours by search in the hop's
      // segment, so that hop enters no table, unless a segment could outgrow the
      // sparse index (an upper bound is all that is known before the hop's counts
      // come back).
      if (k == K) {
        int64_t mbound = 0, ebound = 0;
        for (int b = 0; b < B; ++b) {
          const int64_t front = h.fstart[b + 1] - h.fstart[b];
          int64_t mb = node_cap - n_b[b];
          const int64_t eb = f < 0 ? E : (front > E / (f > 0 ? f : 1) ? E : front * f);
          if (eb < mb) mb = eb;
          if (N < mb) mb = N;
          if (mb > mbound) mbound = mb;
          if (eb > ebound) ebound = eb;
        }
        rl_search = mbound <= RL_SEGMENT_MAX && ebound <= INT32_MAX;
      }
      w.ms.seg_out = nodes;
      w.ms.local_out = (k == K && rl_search) ? nullptr : w.local;
      w.ms.loc_slot = cache_slot;  // the list's address-table entries beside it
      w.ms.loc_out = loc;
      w.ms.uniq_out = nullptr;
      w.ms.unc_ids = nullptr;
      w.ms.unc_off = nullptr;
      w.ms.nodeoff = nullptr;
      w.ms.pairdest = nullptr;
      if (fuse) {
        F.node_cap = node_cap;
        for (int b = 0; b < B; ++b) {
          F.seg_base[b] = w.ms.seg_base[b];
          F.seg_end[b] = w.ms.seg_end[b];
        }
        F.seg_out = nodes;
        F.loc_out = loc;
        F.local_out = w.ms.local_out;
        F.totals_p = w.small + ST_PTOTALS;
        F.packed_ptr = pk->packed_ptr;
        F.packed_cap = pk->packed_cap < pk->pinfo_cap ? pk->packed_cap : pk->pinfo_cap;
        F.pinfo = pk->pinfo;
        F.uniq_out = pk->group_unique;
        F.unique_cap = pk->unique_cap;
        F.unc_ids = pk->pw.unc_ids;
        F.unc_off = pk->pw.unc_off;
        F.unc_cap = pk->unc_cap;
        F.nodeoff = nullptr;  // the address tables come from pinfo
        F.pairdest = pk->pw.pairdest;
        F.pair_cap = pk->pair_cap;
        if ((rc = fuse_scan_write(F, s))) return rc;
      } else if ((rc = mask_scan_write(w.ms, s))) {
        return rc;
      }
      const int ev2 = tm.mark();
      // one round trip per hop: edge bounds, node counts and the error word
      // (and packing's totals after a fused pass)
      int64_t st[ST_SIZE];
      DG_TRY(read_to_host(st, w.small, sizeof(int64_t) * (fuse ? ST_SIZE : ST_PTOTALS), s));
      if (st[ST_ERR])
        return set_error(DG_EINVAL, "invalid input data: %s",
                         describe_device_error((uint32_t)st[ST_ERR]));
      const int64_t *edges = st + ST_BOUNDS;
      bool over = false, nover = false;
      for (int b = 0; b < B; ++b) {
        const int64_t cnt = h.fstart[b + 1] > h.fstart[b] ? edges[b] : 0;
        new_b[b] = st[ST_TOTALS + b];
        if (e_b[b] + cnt > edge_cap) over = true;
        if (n_b[b] + new_b[b] > node_cap) nover = true;
        if (e_b[b] + cnt > sizes->max_batch_edges) sizes->max_batch_edges = e_b[b] + cnt;
        e_b[b] += cnt;
      }
      if (over) {  // the node counts of this hop are not meaningful
        sizes->exact = 0;
        for (int b = 0; b < B; ++b)
          if (n_b[b] > sizes->max_batch_nodes) sizes->max_batch_nodes = n_b[b];
        return set_error(DG_ECAPACITY, "dg_sample_group: edge_cap %lld too small at hop %d",
                         (long long)edge_cap, k);
      }
      for (int b = 0; b < B; ++b)
        if (n_b[b] + new_b[b] > sizes->max_batch_nodes) sizes->max_batch_nodes = n_b[b] + new_b[b];
      if (nover) {
        sizes->exact = 0;
        return set_error(DG_ECAPACITY, "dg_sample_group: node_cap %lld too small at hop %d",
                         (long long)node_cap, k);
      }
      if (fuse) {
        pk->fused = true;
        for (int r = 0; r < mc_rows(B); ++r) pk->ptot[r] = st[ST_PTOTALS + r];
        // the caller reports what does not fit or match
        pk->fits = pk->ptot[row_pairs(B)] <= pk->packed_cap &&
                   (!pk->group_unique || pk->ptot[row_all(B)] <= pk->unique_cap);
        int64_t rows = 0;
        for (int b = 0; b < B; ++b) rows += pk->ptot[b];
        pk->fits = pk->fits && rows == pk->ptot[row_pairs(B)];
      }
      if (mk.nhop < 8) {
        mk.hop[mk.nhop][0] = ev0;
        mk.hop[mk.nhop][1] = ev1;
        mk.hop[mk.nhop][2] = ev2;
        ++mk.nhop;
      }
    }
    for (int b = 0; b < B; ++b) {
      // next frontier: the nodes new at this hop, or (layered) every node so far
      fbeg[b] = layered ? 0 : n_b[b];
      n_b[b] += new_b[b];
      fend[b] = n_b[b];
      hop_ptr[(int64_t)b * (K + 2) + k + 1] = n_b[b];
    }
  }
  for (int b = 0; b < B; ++b) edge_ptr[(int64_t)b * (K + 1) + K] = e_b[b];
  if (!seeded) {  // no hop sampled: the seeds alone
    for (int b = 0; b < B; ++b) {
      fbeg[b] = 0;
      fend[b] = S;
    }
    lay_out();
    frontier(true, false);
    DG_HIP(hipGetLastError());
  }

  // Local IDs through the (node, batch) table.
  mk.r0 = tm.mark();
  TailEdges te;
  TailSparse ts;
  TailLoc tl;
  memset(&te, 0, sizeof(te));
  memset(&ts, 0, sizeof(ts));
  memset(&tl, 0, sizeof(tl));
  te.B = B;
  for (int b = 0; b < B; ++b) {
    te.start[b + 1] = te.start[b] + e_b[b];
    te.limit[b] = n_b[b];
  }
  const bool any_edges = te.start[B] > 0;
  // The hash table of the nodes listed before hop `hops` (at load <= 1/2).
  LocalTable table = w.table;
  auto hash_lists = [&](int hops) -> int {
    Segs LS;
    LS.B = B;
    LS.start[0] = 0;
    for (int b = 0; b < B; ++b) {
      LS.start[b + 1] = LS.start[b] + hop_ptr[(int64_t)b * (K + 2) + hops];
      LS.seg0[b] = 0;
    }
    table.bits = lt_bits_for(LS.start[B]);
    DG_TRY(fill_u64(table.slots, (size_t)1 << table.bits, 0, s));
    hipLaunchKernelGGL(k_table_insert, dim3(blocks_for(LS.start[B])), dim3(THREADS), 0, s, LS,
                       nodes, node_cap, table, w.err);
    DG_HIP(hipGetLastError());
    return DG_OK;
  };
  // The fused pass's packed pairs go with the relabelling, unless phases are timed.
  if (pk && pk->fused && pk->fits && !tm.on) {
    for (int b = 0; b < B; ++b) tl.start[b + 1] = tl.start[b] + pk->ptot[b];
    tl.blocks = blocks_for(tl.start[B]);
    tl.pinfo = pk->pinfo;
    tl.packed_ids = pk->packed_ids;
    tl.loc = loc;
    pk->loc_done = true;
  }
  auto launch_part = [&] {
    const OlderNodes older{w.local, table};
    const unsigned grid = te.blocks + ts.blocks + tl.blocks;
    if (grid == 0) return;
    if (direct)
      hipLaunchKernelGGL(k_relabel_tail<true>, dim3(grid), dim3(THREADS), 0, s, te, ts, tl, nodes,
                         node_cap, edge_cap, edge_dst, older, N, w.err);
    else
      hipLaunchKernelGGL(k_relabel_tail<false>, dim3(grid), dim3(THREADS), 0, s, te, ts, tl, nodes,
                         node_cap, edge_cap, edge_dst, older, N, w.err);
  };
  // One launch, unless its threads would pass the 32-bit count that a launch takes.
  auto launch_tail = [&] {
    const unsigned parts[3] = {te.blocks, ts.blocks, tl.blocks};
    if ((uint64_t)parts[0] + parts[1] + parts[2] <= UINT32_MAX / THREADS) return launch_part();
    for (int q = 0; q < 3; ++q) {
      te.blocks = q == 0 ? parts[0] : 0;
      ts.blocks = q == 1 ? parts[1] : 0;
      tl.blocks = q == 2 ? parts[2] : 0;
      launch_part();
    }
  };
  if (any_edges && rl_search) {
    // edges of the hops before the last through the table, the last hop's by
    // search in its segment (and the table for nodes listed before the hop)
    LastHop lh;
    memset(&lh, 0, sizeof(lh));
    lh.B = B;
    int64_t m_max = 0, last_edges = 0;
    for (int b = 0; b < B; ++b) {
      const int64_t before = edge_ptr[(int64_t)b * (K + 1) + (K - 1)];
      te.start[b + 1] = te.start[b] + before;
      lh.seg0[b] = hop_ptr[(int64_t)b * (K + 2) + K];
      lh.m[b] = (int32_t)(n_b[b] - lh.seg0[b]);
      lh.e0[b] = before;
      lh.ecount[b] = (int32_t)(e_b[b] - before);
      last_edges += lh.ecount[b];
      if (lh.m[b] > m_max) m_max = lh.m[b];
    }
    const int sparse_cap = rl_sparse_cap(node_cap);
    int32_t *sparse = reinterpret_cast<int32_t *>(w.f_off);
    lh.s_log2 = RL_S_MIN_LOG2;
    while (lh.s_log2 < RL_S_MAX_LOG2 &&
           (m_max >> lh.s_log2) + 2 > sparse_cap)  // blocks a segment of m_max can touch
      ++lh.s_log2;
    const int S = 1 << lh.s_log2;
    const int per_chunk = RL_THREADS * rl_edges(lh.s_log2);
    lh.rstart[0] = 0;
    lh.bstart[0] = 0;
    int r_max = 0;
    for (int b = 0; b < B; ++b) {
      lh.a[b] = (int32_t)(((uintptr_t)nodes / 4 + (uintptr_t)b * (uintptr_t)node_cap +
                           (uintptr_t)lh.seg0[b]) & (uintptr_t)(S - 1));
      const int r = lh.m[b] == 0 ? 0 : (int)(((int64_t)lh.m[b] + lh.a[b] + S - 1) / S);
      if (r > r_max) r_max = r;
      lh.rstart[b + 1] = lh.rstart[b] + r;
    }
    // Several chunks per block share one staging of the index where that is longer
    // than half a chunk, as long as every CU gets two blocks (one mini-batch of
    // 130k edges: 44 us with four chunks, i.e. 16 blocks, 16 us with one; 3M edges
    // of 8 mini-batches, index of 9600 entries: 152 us with two, 129 with four).
    lh.chunks = 1;
    while (lh.chunks < RL_CHUNKS && per_chunk * lh.chunks < 2 * r_max &&
           last_edges >= (int64_t)512 * per_chunk * 2 * lh.chunks)
      lh.chunks *= 2;
    const int per_block = per_chunk * lh.chunks;
    for (int b = 0; b < B; ++b) {
      lh.bstart[b + 1] = lh.bstart[b] + (int32_t)((lh.ecount[b] + (int64_t)per_block - 1) / per_block);
    }
    if (r_max > sparse_cap)
      return set_error(DG_EINVAL, "internal: last-hop segment of %lld nodes", (long long)m_max);
    if (!direct && (rc = hash_lists(K))) return rc;
    te.blocks = blocks_for(te.start[B]);
    ts.blocks = blocks_for(lh.rstart[B]);
    ts.s_log2 = lh.s_log2;
    ts.cap = sparse_cap;
    ts.sparse = sparse;
    memcpy(ts.rstart, lh.rstart, sizeof(ts.rstart));
    memcpy(ts.a, lh.a, sizeof(ts.a));
    memcpy(ts.seg0, lh.seg0, sizeof(ts.seg0));
    launch_tail();
    if (lh.bstart[B] > 0) {
      const unsigned grid = (unsigned)((lh.bstart[B] + 7) & ~7);
      const size_t lds = (size_t)(r_max > 0 ? r_max : 1) * sizeof(int32_t);
      const OlderNodes older{w.local, table};
      auto go = [&](auto slog2) {
        constexpr int SL = decltype(slog2)::value;
        if (direct)
          hipLaunchKernelGGL((k_relabel_last<SL, true>), dim3(grid), dim3(RL_THREADS), lds, s, lh,
                             nodes, node_cap, sparse, sparse_cap, edge_cap, edge_dst, older, N,
                             w.err);
        else
          hipLaunchKernelGGL((k_relabel_last<SL, false>), dim3(grid), dim3(RL_THREADS), lds, s,
                             lh, nodes, node_cap, sparse, sparse_cap, edge_cap, edge_dst, older,
                             N, w.err);
      };
      if (lh.s_log2 == 4) go(std::integral_constant<int, 4>());
      else if (lh.s_log2 == 5) go(std::integral_constant<int, 5>());
      else go(std::integral_constant<int, 6>());
    }
    DG_HIP(hipGetLastError());
  } else if (any_edges) {
    if (!direct && (rc = hash_lists(K + 1))) return rc;
    te.blocks = blocks_for(te.start[B]);
    launch_tail();
    DG_HIP(hipGetLastError());
  } else if (tl.blocks > 0) {
    launch_tail();
    DG_HIP(hipGetLastError());
  }
  mk.r1 = tm.mark();
  if (exit_clear && !prev_cleared &&
      ((rc = fill_u64(w.prev, (size_t)N, 0, s)) ||
       (rc = fill_u64(reinterpret_cast<uint64_t *>(w.plines), (size_t)mc_touch_bytes(N) / 8, 0,
                      s))))
    return rc;
  if (member_lines && !lines_done && !(pk && pk->fused) &&
      (rc = member_lines_pass(w.visited, N, B, member_lines, s)))
    return rc;
  if (pk) {  // the caller checks the error word after its own work
    pk->err = w.err;
    pk->visited = w.visited;
    pk->local = w.local;
  } else if ((rc = check_err(w.err, s))) {
    return rc;
  }

  int64_t sum_n = 0, sum_e = 0, mn = 0, me = 0;
  for (int b = 0; b < B; ++b) {
    sum_n += n_b[b];
    sum_e += e_b[b];
    if (n_b[b] > mn) mn = n_b[b];
    if (e_b[b] > me) me = e_b[b];
  }
  sizes->max_batch_nodes = mn;
  sizes->max_batch_edges = me;
  sizes->total_nodes = sum_n;
  sizes->total_edges = sum_e;
  return DG_OK;
}

// Sampling's phase times from the marks of a finished call.
void sample_times(const PhaseTimer &tm, const SampleMarks &mk, dg_timing *timing) {
  float t_sample = 0.f, t_dedup = 0.f;
  for (int i = 0; i < mk.nhop && i < 8; ++i) {
    t_sample += tm.ms(mk.hop[i][0], mk.hop[i][1]);
    t_dedup += tm.ms(mk.hop[i][1], mk.hop[i][2]);
  }
  timing->sample_ms = t_sample;
  timing->dedup_ms = t_dedup;
  timing->relabel_ms = tm.ms(mk.r0, mk.r1);
  timing->total_ms = tm.ms(mk.start, mk.r1);
}

}  // namespace
}  // namespace dg

extern "C" int dg_sample_group(const dg_csr *g, const int32_t *seeds, int32_t B, int32_t S,
                               int64_t batch_base, const int32_t *fanouts, int32_t K,
                               uint64_t rng_seed, uint32_t flags, int64_t node_cap,
                               int32_t *nodes,
                               int64_t *hop_ptr, int64_t edge_cap, int32_t *edge_src,
                               int32_t *edge_dst, int64_t *edge_ptr, uint64_t *membership,
                               uint8_t *member_lines, const int32_t *cache_slot, int32_t *loc,
                               void *ws, size_t ws_bytes, hipStream_t stream, dg_sizes *sizes,
                               dg_timing *timing) {
  if (timing) memset(timing, 0, sizeof(*timing));
  PhaseTimer tm(timing != nullptr, stream);
  SampleMarks mk;
  const int rc = sample_impl(g, seeds, B, S, batch_base, fanouts, K, rng_seed, flags, node_cap,
                             nodes, hop_ptr, edge_cap, edge_src, edge_dst, edge_ptr, membership,
                             member_lines, cache_slot, loc, ws, ws_bytes, stream, sizes, tm, mk,
                             nullptr);
  if (rc == DG_OK && timing) sample_times(tm, mk, timing);
  return rc;
}

extern "C" size_t dg_sample_pack_workspace_bytes(int64_t num_nodes, int32_t B,
                                                 int64_t node_cap) {
  if (num_nodes < 1 || B < 1 || B > DG_MAX_BATCHES || node_cap < 1 ||
      node_cap > INT64_MAX / DG_MAX_BATCHES)
    return 0;
  return mc_most_bytes(num_nodes, [&](int64_t n) {
    Carve c(nullptr);
    PackInto pk;
    carve_sample_pack(pk, c, n, B, node_cap, mc_rounds(n));
    return c.used;
  });
}

extern "C" int dg_sample_pack_group(
    const dg_csr *g, const int32_t *seeds, int32_t B, int32_t S, int64_t batch_base,
    const int32_t *fanouts, int32_t K, uint64_t rng_seed, uint32_t flags, int64_t node_cap,
    int32_t *nodes, int64_t *hop_ptr, int64_t edge_cap, int32_t *edge_src, int32_t *edge_dst,
    int64_t *edge_ptr, uint64_t *membership, const int32_t *cache_slot, int32_t *loc,
    const void *feats, int64_t row_bytes, int64_t packed_cap, void *packed, int32_t *packed_ids,
    int64_t *packed_ptr, int64_t *packed_ptr_host, int32_t *group_unique, int64_t unique_cap,
    uint32_t pack_flags, void *ws, size_t ws_bytes, void *pack_ws, size_t pack_ws_bytes,
    hipStream_t stream, hipStream_t rows_stream, dg_sizes *sizes, dg_timing *timing) {
  if (!g || !cache_slot || !loc || !feats || !packed_ptr || !packed_ptr_host || !sizes ||
      !hop_ptr)
    return set_error(DG_EINVAL, "dg_sample_pack_group: null pointer argument");
  if (row_bytes < 1 || packed_cap < 0 || unique_cap < 0 || (packed_cap > 0 && !packed_ids))
    return set_error(DG_EINVAL, "dg_sample_pack_group: bad packing sizes");
  if (pack_flags & ~DG_PACK_ROWS_STREAM)
    return set_error(DG_EINVAL, "dg_sample_pack_group: unknown pack flags 0x%x", pack_flags);
  if ((pack_flags & DG_PACK_ROWS_STREAM) && timing)
    return set_error(DG_EINVAL, "dg_sample_pack_group: timing cannot be combined with "
                                "DG_PACK_ROWS_STREAM");
  if (dg_sample_pack_workspace_bytes(g->num_nodes, B, node_cap) == 0 || K < 0)
    return set_error(DG_EINVAL, "dg_sample_pack_group: bad sizes (B=%d K=%d node_cap=%lld)", B,
                     K, (long long)node_cap);
  // Both workspaces take the same tiles: short ones where they fit, else the longest.
  PackInto pk;
  size_t need = 0;
  for (int rounds : {mc_rounds(g->num_nodes), MC_ROUNDS_MAX}) {
    Carve c(pack_ws), cs(nullptr);
    carve_sample_pack(pk, c, g->num_nodes, B, node_cap, rounds);
    SampleWs sw;
    carve_sample(sw, cs, g->num_nodes, B, node_cap, (flags & DG_SAMPLE_DIRECT) != 0, rounds);
    need = c.used;
    if (need <= pack_ws_bytes && cs.used <= ws_bytes) break;
  }
  if (!pack_ws || pack_ws_bytes < need || ((uintptr_t)pack_ws & 255))
    return set_error(DG_EWORKSPACE,
                     "dg_sample_pack_group: packing workspace needs %zu bytes, 256-aligned",
                     need);
  const bool rows_async = (pack_flags & DG_PACK_ROWS_STREAM) && packed;
  const int64_t N = g->num_nodes;
  pk.packed_ptr = packed_ptr;
  pk.packed_cap = packed_cap;
  pk.packed_ids = packed_ids;
  pk.group_unique = group_unique;
  pk.unique_cap = group_unique ? unique_cap : 0;
  if (timing) memset(timing, 0, sizeof(*timing));
  PhaseTimer tm(timing != nullptr, stream);
  SampleMarks mk;
  int rc = sample_impl(g, seeds, B, S, batch_base, fanouts, K, rng_seed, flags, node_cap, nodes,
                       hop_ptr, edge_cap, edge_src, edge_dst, edge_ptr, membership, pk.lines,
                       cache_slot, loc, ws, ws_bytes, stream, sizes, tm, mk, &pk);
  if (rc) return rc;
  int64_t n_b[DG_MAX_BATCHES];
  for (int b = 0; b < B; ++b) n_b[b] = hop_ptr[(int64_t)b * (K + 2) + K + 1];

  if (!pk.fused) {
    // No fused pass (hash relabelling, or a last hop with nothing to sample):
    // packing's own passes over the lists sampling wrote.
    if ((rc = check_err(pk.err, stream))) return rc;
    if (timing) sample_times(tm, mk, timing);
    dg_sizes ps;
    dg_timing pt;
    rc = pack_impl(feats, N, row_bytes, cache_slot, B, nodes, node_cap, n_b, packed_cap, packed,
                   packed_ids, packed_ptr, packed_ptr_host, loc, group_unique, unique_cap,
                   membership ? membership : pk.visited, pk.lines, nullptr, 0, nullptr,
                   DG_PACK_CLEAR_MEMBERSHIP | DG_PACK_LOC_PENDING |
                       (pack_flags & DG_PACK_ROWS_STREAM),
                   static_cast<char *>(pack_ws) + pk.pw_offset, pack_ws_bytes - pk.pw_offset,
                   stream, rows_stream, &ps, timing ? &pt : nullptr, false);
    sizes->packed_rows = ps.packed_rows;
    sizes->unique_nodes = ps.unique_nodes;
    sizes->unique_packed = ps.unique_packed;
    if (rc) return rc;
    if (timing) {
      timing->mark_ms = pt.mark_ms;
      timing->order_ms = pt.order_ms;
      timing->loc_ms = pt.loc_ms;
      timing->gather_ms = pt.gather_ms;
      timing->total_ms += pt.total_ms;
    }
    return DG_OK;
  }

  // Packing's sizes came back with the last hop's counts.
  int64_t rows = 0;
  packed_ptr_host[0] = 0;
  for (int b = 0; b < B; ++b) {
    rows += pk.ptot[b];
    packed_ptr_host[b + 1] = rows;
  }
  sizes->packed_rows = rows;
  sizes->unique_nodes = pk.ptot[row_all(B)];
  sizes->unique_packed = pk.ptot[row_packed(B)];
  if (rows != pk.ptot[row_pairs(B)] || pk.ptot[row_all_pairs(B)] != sizes->total_nodes)
    return set_error(DG_EINVAL, "dg_sample_pack_group: internal pair count mismatch");
  if (rows > packed_cap || (group_unique && sizes->unique_nodes > unique_cap))
    return set_error(DG_ECAPACITY,
                     "dg_sample_pack_group: need packed_cap >= %lld and unique_cap >= %lld",
                     (long long)rows, (long long)sizes->unique_nodes);
  const FusedRows t{feats,  N,      row_bytes,       packed, pk.pw.unc_ids, pk.pw.unc_off,
                    pk.pw.pairdest, sizes->unique_packed, rows,   pk.err};
  // On a second stream the row copy starts behind the relabelling, so that it runs beside
  // the caller's next call.  It needs the last hop's lists alone, but handed over ahead of
  // the relabelling it slows that, which this call waits for: a loop with the copy and the
  // assembly on a second stream, handed over here / ahead, a step: 1M nodes 943 / 1007 us,
  // 8M 2146 / 2251 and 806 / 894, 32M 4733 / 4800, 100M about 5.6 / 5.9 ms.
  if (rows_async && (rc = pack_fused_rows(t, true, stream, rows_stream))) return rc;
  if (!pk.loc_done && rows > 0) {  // phases are timed: the address tables by themselves
    TailEdges te;
    TailSparse ts;
    TailLoc tl;
    memset(&te, 0, sizeof(te));
    memset(&ts, 0, sizeof(ts));
    te.B = B;
    for (int b = 0; b < B; ++b) te.limit[b] = n_b[b];
    for (int b = 0; b <= B; ++b) tl.start[b] = packed_ptr_host[b];
    tl.blocks = blocks_for(rows);
    tl.pinfo = pk.pinfo;
    tl.packed_ids = packed_ids;
    tl.loc = loc;
    hipLaunchKernelGGL(k_relabel_tail<true>, dim3(tl.blocks), dim3(THREADS), 0, stream, te, ts, tl,
                       nodes, node_cap, edge_cap, edge_dst, OlderNodes{pk.local, LocalTable{}}, N,
                       pk.err);
    DG_HIP(hipGetLastError());
  }
  const int ev_loc = tm.mark();
  if (!rows_async && (rc = pack_fused_rows(t, false, stream, nullptr))) return rc;
  const int ev_gather = tm.mark();
  if ((rc = check_err(pk.err, stream))) return rc;
  if (timing) {
    sample_times(tm, mk, timing);
    timing->loc_ms = tm.ms(mk.r1, ev_loc);
    timing->gather_ms = tm.ms(ev_loc, ev_gather);
    timing->total_ms = tm.ms(mk.start, ev_gather);
  }
  return DG_OK;
}
