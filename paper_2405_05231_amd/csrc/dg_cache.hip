// Cache configuration by access frequency (DiskGNN §4 "Four-level hierarchical
// feature store": one counter per node, streamed over the graph samples, and
// the most popular features go to the fastest tier; §3: this placement
// minimises the features fetched from slower storage) and the row gather that
// fills the cache table, which the paper does by treating the cache as a
// special mini-batch of batched packing (§5.2).  The same gather, run once per
// mini-batch over that batch's packed IDs, is the individual packing of §5.2
// (Fig. 6a).
//
// Frequencies: a node's count is the number of mini-batches of the group that
// require it, i.e. the popcount of its membership word.  Ranking (count
// descending, then ID ascending) is a stable counting sort over 65 keys.
//
// The same counting sort orders the disk-cache entries by MinHash value
// (§5.1, Alg. 1): with k hash functions H_j (permutations of the sample IDs,
// given as input), S(v) is the minimum of H_j(i) over every hash function j
// and every sample i that requires v, which equals the minimum over those
// samples of M(i) = min_j H_j(i); entries are then sorted by S.
#include <initializer_list>
#include <string.h>

#include "dg_rows.h"

namespace dg {
namespace {

constexpr int KEYS = 65;  // keys 0..64
constexpr int CF_WAVES = 4;
constexpr int CF_THREADS = 64 * CF_WAVES;
constexpr int CF_FLIGHT = 16;  // rounds of 64 elements whose keys are loaded together

// A stable counting sort of a list by a key in 0..64.  Each wave owns 64*R
// consecutive elements (a column of the count matrix): it counts its keys, a
// scan runs along each key's row, and the ranks are the wave's base of the key
// plus earlier rounds plus the lanes below with the same key.  Two uses:
//   FREQ:    list = nodes 0..N-1, key = access count (popcount of the
//            membership word), ranked by count descending; key 0 (not
//            accessed) is neither counted nor ranked;
//   MINHASH: list = the disk-cache entries V_d, key = the entry's MinHash
//            value (64 = in no sample), ranked ascending.
// The count pass leaves each element's key as a byte for the place pass, where
// the workspace has room: the membership words are read once.  Bound by HBM
// (FREQ at 50M nodes: 400 MB of words, 2 x 50 MB of keys, 200 MB of slots; 238 us
// the whole call) or by the scattered words (MINHASH: 1M entries, 63 us).  With the
// words read twice and one step per distinct key of a round the passes are bound by
// issue: 120 + 207 us at 50M nodes against 92 + 110 (the calls: 393 and 275 us).
enum Mode { FREQ = 0, MINHASH = 1 };

struct KeySort {
  const uint64_t *mask;
  uint64_t keep;      // bits of the group's batches
  int64_t N;          // nodes
  int64_t n;          // list length
  int64_t ncol;       // waves
  bool wide;          // ranks of more than 31 bits
  void *cnt;          // [KEYS + 1][ncol] counts, then exclusive scans along each key's
                      // row, 4 bytes each, or 8 if wide; the last row holds each
                      // wave's error bits (MINHASH)
  int64_t *totals;    // [KEYS + 1]: per key; the error bits
  uint8_t *keys;      // [n] each element's key; NULL: the place pass finds it again
  // FREQ outputs
  int64_t cap;
  int32_t *cache_slot;
  int32_t *cache_nodes;
  // MINHASH input / outputs
  const int32_t *ids;    // V_d
  const int32_t *perms;  // [k][B]
  int32_t k, B;
  int8_t *minv;          // [64] behind totals: minima over many hash functions
  bool min_done;         // minv holds them
  int32_t *order;        // V_r
  int32_t *signature;    // S(v) per entry (-1: in no sample)
};

// M(i) = min over the k hash functions of H_j(i) for i < B, or -1 if one of the values
// is outside [0, B).  Every block of the count pass (and of the place pass without
// keys) takes the minima for its table itself; above K_ITSELF functions that chain of k
// loads per block costs more than this launch, which does it once (blocks themselves
// against this launch, whole call: 30M entries 728 / 725 us at 17 functions, 820 / 725
// at 64, 2018 / 736 at 512; 1000 entries 37.6 / 38.7, 43.1 / 38.6 and 91 / 41).
constexpr int K_ITSELF = 16;
constexpr int MV_PARTS = 16;
__global__ __launch_bounds__(64 * MV_PARTS) void k_minhash_min(KeySort a) {
  __shared__ int32_t s_m[MV_PARTS][64];
  const int i = threadIdx.x & 63, part = threadIdx.x >> 6;
  int32_t m = 64;
  if (i < a.B) {
    for (int j = part; j < a.k; j += MV_PARTS) {
      const int32_t h = a.perms[(int64_t)j * a.B + i];
      m = min(m, h < a.B ? h : -1);
    }
  }
  s_m[part][i] = m;
  __syncthreads();
  if (part == 0) {
#pragma unroll
    for (int q = 1; q < MV_PARTS; ++q) m = min(m, s_m[q][i]);
    a.minv[i] = (int8_t)max(m, -1);
  }
}

// MINHASH: the smallest value of each set of samples is found a byte of the
// membership word at a time: s_low[q][x] = min over the bits of x of the
// values M(8q + bit), M(i) = min_j H_j(i); 64 for no bit.
struct LowTable {
  uint8_t v[8][256];
};

// Fills the table (whole block); returns the block's error bits to thread 0.
template <int MODE>
__device__ __forceinline__ uint32_t stage_low(const KeySort &a, LowTable *t) {
  uint32_t bad = 0;
  if (MODE == MINHASH) {
    __shared__ uint8_t s_min[64];
    if (threadIdx.x < 64) {
      const int i = threadIdx.x;
      int m = 64;
      if (i < a.B && a.min_done) {
        m = a.minv[i];
        if (m < 0) bad = ERR_ROW_RANGE;
      } else if (i < a.B) {
        for (int j = 0; j < a.k; ++j) {
          const int32_t h = a.perms[(int64_t)j * a.B + i];
          if (h < 0 || h >= a.B) bad = ERR_ROW_RANGE;
          else m = min(m, (int)h);
        }
      }
      s_min[i] = (uint8_t)m;
      bad = __ballot(bad != 0) ? ERR_ROW_RANGE : 0u;
    }
    __syncthreads();
    for (int x = threadIdx.x; x < 8 * 256; x += CF_THREADS) {
      const int q = x >> 8;
      int m = 64;
#pragma unroll
      for (int bit = 0; bit < 8; ++bit)
        if ((x >> bit) & 1) m = min(m, (int)s_min[8 * q + bit]);
      t->v[q][x & 255] = (uint8_t)m;
    }
    __syncthreads();
  }
  return bad;
}

// Keys of U rounds from element t0 (-1 past the list), all their loads issued
// before any is used.
template <int MODE, int U>
__device__ __forceinline__ void load_keys(const KeySort &a, int64_t t0, int lane,
                                          const LowTable *low, int (&k)[U], uint32_t *bad) {
  uint64_t m[U];
  if (MODE == FREQ) {
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const int64_t i = t0 + r * 64 + lane;
      m[r] = a.mask[i < a.n ? i : a.n - 1];
    }
  } else {
    int32_t v[U];
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const int64_t i = t0 + r * 64 + lane;
      v[r] = i < a.n ? a.ids[i] : 0;
    }
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const bool ok = v[r] >= 0 && (int64_t)v[r] < a.N;
      if (!ok) *bad |= ERR_NODE_RANGE;
      m[r] = ok ? a.mask[v[r]] : 0ull;
    }
  }
#pragma unroll
  for (int r = 0; r < U; ++r) {
    const int64_t i = t0 + r * 64 + lane;
    const uint64_t x = m[r] & a.keep;
    int key;
    if (MODE == FREQ) {
      key = __popcll(x);
    } else {
      key = 64;  // S(v) = inf: v is required by no sample
#pragma unroll
      for (int q = 0; q < 8; ++q) key = min(key, (int)low->v[q][(x >> (8 * q)) & 255u]);
    }
    k[r] = i < a.n ? key : -1;
  }
}

// The lanes of `act` that hold this lane's key (for a lane of act), by one
// ballot per key bit.
__device__ __forceinline__ uint64_t same_key(int key, uint64_t act) {
  uint64_t m = act;
#pragma unroll
  for (int bit = 0; bit < 7; ++bit) {
    const bool one = (key >> bit) & 1;
    const uint64_t b = __ballot(one);
    m &= one ? b : ~b;
  }
  return m;
}

// P: unsigned integer that holds a rank (uint64_t if wide).
template <int MODE, int R, typename P>
__global__ __launch_bounds__(CF_THREADS) void k_key_count(KeySort a) {
  constexpr int U = R < CF_FLIGHT ? R : CF_FLIGHT;
  __shared__ uint32_t s_cnt[CF_WAVES][KEYS + 3];
  __shared__ LowTable s_low[1];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t bad = stage_low<MODE>(a, s_low);
  const int64_t col = (int64_t)blockIdx.x * CF_WAVES + w;
  uint32_t *cnt = s_cnt[w];  // this wave's own: its LDS operations run in order
  cnt[lane] = 0u;
  if (lane == 0) cnt[64] = 0u;
  __builtin_amdgcn_wave_barrier();
  for (int c = 0; c < R; c += U) {
    const int64_t t0 = (col * R + c) * 64;
    if (t0 >= a.n) break;  // uniform
    int k[U];
    load_keys<MODE, U>(a, t0, lane, s_low, k, &bad);
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const int64_t i = t0 + r * 64 + lane;
      if (a.keys && k[r] >= 0) a.keys[i] = (uint8_t)k[r];
      const bool counted = k[r] >= (MODE == FREQ ? 1 : 0);
      const uint64_t act = __ballot(counted);
      if (!act) continue;  // uniform
      if (__popcll(act) <= 16) {  // few: one LDS add each
        if (counted) atomicAdd(&cnt[k[r]], 1u);
      } else {  // many, perhaps of one key: one add per key
        const uint64_t same = same_key(k[r], act);
        if (counted && __builtin_ctzll(same) == lane) atomicAdd(&cnt[k[r]], (uint32_t)__popcll(same));
      }
    }
  }
  __builtin_amdgcn_wave_barrier();
  if (col < a.ncol) {
    P *out = static_cast<P *>(a.cnt);
    out[(int64_t)lane * a.ncol + col] = cnt[lane];
    if (lane == 0) out[64 * a.ncol + col] = cnt[64];
    if (MODE == MINHASH) {
      const uint32_t node = __ballot((bad & ERR_NODE_RANGE) != 0) ? (uint32_t)ERR_NODE_RANGE : 0u;
      const uint32_t row = __ballot((bad & ERR_ROW_RANGE) != 0) ? (uint32_t)ERR_ROW_RANGE : 0u;
      if (lane == 0) out[65 * a.ncol + col] = node | row;
    }
  }
}

// One block per row: exclusive scan in place of a key's counts, or (row KEYS) the
// OR of the error bits.
constexpr int KS_ITEMS = 8;
template <typename P>
__global__ __launch_bounds__(1024) void k_key_scan(KeySort a) {
  __shared__ uint32_t s_w[KS_ITEMS][16];
  const int row = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  P *p = static_cast<P *>(a.cnt) + (int64_t)row * a.ncol;
  P carry = 0;
  for (int64_t c0 = 0; c0 < a.ncol; c0 += 1024 * KS_ITEMS) {
    uint32_t v[KS_ITEMS], incl[KS_ITEMS];  // a chunk's sum fits 32 bits
#pragma unroll
    for (int q = 0; q < KS_ITEMS; ++q) {
      const int64_t i = c0 + q * 1024 + threadIdx.x;
      v[q] = i < a.ncol ? (uint32_t)p[i] : 0u;
    }
    if (row == KEYS) {
#pragma unroll
      for (int q = 0; q < KS_ITEMS; ++q) carry |= v[q];
      continue;
    }
#pragma unroll
    for (int q = 0; q < KS_ITEMS; ++q) {
      incl[q] = (uint32_t)wave_incl_sum_i32((int32_t)v[q]);
      if (lane == 63) s_w[q][w] = incl[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < KS_ITEMS; ++q) {
      uint32_t before = 0, sum = 0;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const uint32_t x = s_w[q][j];
        before += j < w ? x : 0u;
        sum += x;
      }
      const int64_t i = c0 + q * 1024 + threadIdx.x;
      if (i < a.ncol) p[i] = carry + before + incl[q] - v[q];
      carry += sum;
    }
    __syncthreads();
  }
  if (row == KEYS) {
    const uint32_t node = __syncthreads_or((int)(carry & ERR_NODE_RANGE)) ? (uint32_t)ERR_NODE_RANGE : 0u;
    const uint32_t hash = __syncthreads_or((int)(carry & ERR_ROW_RANGE)) ? (uint32_t)ERR_ROW_RANGE : 0u;
    carry = node | hash;
  }
  if (threadIdx.x == 0) a.totals[row] = (int64_t)carry;
}

template <int MODE, int R, typename P>
__global__ __launch_bounds__(CF_THREADS) void k_key_place(KeySort a) {
  constexpr int U = R < CF_FLIGHT ? R : CF_FLIGHT;
  __shared__ P s_run[CF_WAVES][KEYS + 3];  // next rank of each key
  __shared__ LowTable s_low[1];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t bad = 0;
  if (!a.keys) (void)stage_low<MODE>(a, s_low);
  const int64_t col = (int64_t)blockIdx.x * CF_WAVES + w;
  const int64_t at = col < a.ncol ? col : a.ncol - 1;
  // rank of the first element of each key (lane k: key k), and key 64's
  const P tot = (P)a.totals[lane], tot64 = (P)a.totals[64];
  const P incl = sizeof(P) == 8 ? (P)wave_incl_sum((int64_t)tot)
                                : (P)(uint32_t)wave_incl_sum_i32((int32_t)tot);
  const P all = (P)read_lane((int64_t)incl, 63);  // keys 0..63 (FREQ: 1..63)
  const P first = MODE == FREQ ? tot64 + all - incl : incl - tot;
  const P first64 = MODE == FREQ ? 0 : all;
  P *run = s_run[w];  // this wave's own
  const P *base = static_cast<const P *>(a.cnt);
  run[lane] = first + base[(int64_t)lane * a.ncol + at];
  if (lane == 0) run[64] = first64 + base[64 * a.ncol + at];
  // FREQ: keys from `cut` on have a rank below cap (first is non-increasing in
  // the key); cut = 65: none has
  int cut = 0;
  if (MODE == FREQ) {
    const uint64_t in = __ballot(lane > 0 && (int64_t)first < a.cap);
    cut = in ? __builtin_ctzll(in) : ((int64_t)first64 < a.cap ? 64 : 65);
    // slots no node takes
    const int64_t used = (int64_t)(tot64 + all);
    for (int64_t r = used + (int64_t)blockIdx.x * CF_THREADS + threadIdx.x; r < a.cap;
         r += (int64_t)gridDim.x * CF_THREADS)
      a.cache_nodes[r] = -1;
  }
  __builtin_amdgcn_wave_barrier();
  const uint64_t lt = lanes_below();
  for (int c = 0; c < R; c += U) {
    const int64_t t0 = (col * R + c) * 64;
    if (t0 >= a.n) break;  // uniform
    int k[U];
    int32_t id[U];
    if (a.keys) {
#pragma unroll
      for (int r = 0; r < U; ++r) {
        const int64_t i = t0 + r * 64 + lane;
        k[r] = i < a.n ? (int)a.keys[i] : -1;
      }
    } else {
      load_keys<MODE, U>(a, t0, lane, s_low, k, &bad);
    }
    if (MODE == MINHASH) {
#pragma unroll
      for (int r = 0; r < U; ++r) {
        const int64_t i = t0 + r * 64 + lane;
        id[r] = i < a.n ? a.ids[i] : 0;
      }
    }
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const int64_t i = t0 + r * 64 + lane;
      const bool cand = k[r] >= cut;  // past the list: -1, never
      const uint64_t act = __ballot(cand);
      int64_t rank = -1;
      if (act) {  // uniform
        if (__popcll(act) <= 6) {  // few: one step per key present
          uint64_t todo = act;
          while (todo) {
            const int src = __builtin_ctzll(todo);
            const int kk = __builtin_amdgcn_readlane(k[r], src);
            const uint64_t same = __ballot(k[r] == kk);
            todo &= ~same;
            const P at0 = run[kk];
            if (k[r] == kk) rank = (int64_t)at0 + __popcll(same & lt);
            if (lane == src) run[kk] = at0 + (P)__popcll(same);
            __builtin_amdgcn_wave_barrier();
          }
        } else {
          const uint64_t same = same_key(k[r], act);
          if (cand) {
            const P at0 = run[k[r]];
            rank = (int64_t)at0 + __popcll(same & lt);
            __builtin_amdgcn_wave_barrier();
            if (__builtin_ctzll(same) == lane) run[k[r]] = at0 + (P)__popcll(same);
          }
          __builtin_amdgcn_wave_barrier();
        }
      }
      if (k[r] < 0) continue;
      if (MODE == FREQ) {
        const bool cached = cand && rank < a.cap;
        a.cache_slot[i] = cached ? (int32_t)rank : -1;
        if (cached) a.cache_nodes[rank] = (int32_t)i;
      } else {
        a.order[rank] = id[r];
        if (a.signature) a.signature[i] = k[r] == 64 ? -1 : k[r];
      }
    }
  }
}

// Rounds per wave: short tiles until the chip's 8192 wave slots are filled, then
// longer ones, so that the count matrix stays small.  Count, scan and place of
// the frequency ranking (5% of the nodes cached, 10% accessed): 20M nodes 86 us
// with 16 rounds, 99 with 64; 50M nodes 215 and 219, and a quarter of the matrix.
constexpr int64_t KEYS_16 = (int64_t)8192 * 64 * 8, KEYS_64 = (int64_t)8192 * 64 * 64;
int key_rounds(int64_t n) { return n >= KEYS_64 ? 64 : n >= KEYS_16 ? 16 : 4; }
int64_t key_cols(int64_t n, int rounds) {
  const int64_t c = (n + 64 * rounds - 1) / (64 * rounds);
  return c < 1 ? 1 : c;  // an empty list: one wave (MINHASH checks the permutations)
}

// The layout with tiles of `rounds` and, with_keys, room for the key bytes.
void carve_keysort(KeySort &a, Carve &c, int rounds, bool with_keys) {
  a.ncol = key_cols(a.n, rounds);
  a.wide = a.n > 0x7fffffffll;
  a.cnt = c.take<char>((size_t)(KEYS + 1) * (size_t)a.ncol *
                       (a.wide ? sizeof(uint64_t) : sizeof(uint32_t)));
  a.totals = c.take<int64_t>(KEYS + 1 + 64 / sizeof(int64_t));
  a.minv = a.totals ? reinterpret_cast<int8_t *>(a.totals + KEYS + 1) : nullptr;
  a.keys = with_keys ? c.take<uint8_t>((size_t)a.n) : nullptr;
}

// Carves the first layout that ws_bytes hold: the tile that suits n, longer ones (a
// smaller matrix), then no keys, as a workspace sized when the keys were read twice
// needs it.  Returns the rounds per wave, 0 if none fits.
int fit_keysort(KeySort &a, void *ws, size_t ws_bytes) {
  for (bool with_keys : {true, false})
    for (int rounds : {4, 16, 64}) {
      if (with_keys ? rounds < key_rounds(a.n) : rounds < 64) continue;
      Carve c(ws);
      carve_keysort(a, c, rounds, with_keys);
      if (c.used <= ws_bytes) return rounds;
    }
  return 0;
}

// What the preferred layout takes at the worst list of up to n elements (the tiles get
// longer, and the matrix smaller, at the steps of key_rounds), so that a workspace
// sized for the longest list suits every shorter one.
size_t keysort_bytes(int64_t n) {
  size_t most = 0;
  for (int64_t len : {n, KEYS_16 - 1, KEYS_64 - 1}) {
    if (len > n) continue;
    KeySort a;
    memset(&a, 0, sizeof(a));
    a.n = len;
    Carve c(nullptr);
    carve_keysort(a, c, key_rounds(len), true);
    if (c.used > most) most = c.used;
  }
  return most;
}

// What the smallest layout takes.
size_t keysort_least(KeySort a) {
  Carve c(nullptr);
  carve_keysort(a, c, 64, false);
  return c.used;
}

// Count pass, scans and place pass; the totals come back to the host.
template <int MODE>
int keysort_run(KeySort &a, int rounds, int64_t *totals, hipStream_t s) {
  const dim3 g((unsigned)((a.ncol + CF_WAVES - 1) / CF_WAVES)), b(CF_THREADS);
  if (MODE == MINHASH && a.k > K_ITSELF) {
    hipLaunchKernelGGL(k_minhash_min, dim3(1), dim3(64 * MV_PARTS), 0, s, a);
    a.min_done = true;
  }
  auto go = [&](auto r, auto p) {
    constexpr int R = decltype(r)::value;
    using P = decltype(p);
    hipLaunchKernelGGL((k_key_count<MODE, R, P>), g, b, 0, s, a);
    hipLaunchKernelGGL(k_key_scan<P>, dim3(MODE == MINHASH ? KEYS + 1 : KEYS), dim3(1024), 0, s,
                       a);
    hipLaunchKernelGGL((k_key_place<MODE, R, P>), g, b, 0, s, a);
  };
  // (FREQ lists are never that long)
  using Wide = std::conditional_t<MODE == MINHASH, uint64_t, uint32_t>;
  if (a.wide) go(std::integral_constant<int, 64>(), Wide());
  else if (rounds == 64) go(std::integral_constant<int, 64>(), uint32_t());
  else if (rounds == 16) go(std::integral_constant<int, 16>(), uint32_t());
  else go(std::integral_constant<int, 4>(), uint32_t());
  DG_HIP(hipGetLastError());
  DG_TRY(read_to_host(totals, a.totals, sizeof(int64_t) * (KEYS + 1), s));
  return DG_OK;
}

// ------------------------------------------------------------------ row gather
constexpr int G_THREADS = 256;
constexpr int G_UNROLL = 4;

// Bound by HBM.  NT: nontemporal stores (gather_nt).  A row that does not end on a
// 128-byte line shares that line with the next row, and plain stores let the two merge
// in L2; that is worth less the longer the rows and the fewer of their 64-byte halves,
// 32-byte sectors and 16-byte vectors are partial.  Outputs of up to STREAM_BYTES, which
// the 256 MB last-level cache largely holds, take plain stores as well (nontemporal over
// plain: 280 MB 1.05 to 1.21, 360 MB 0.88 to 0.97 for the rows below that take them).
// Plain against nontemporal, us: 4M rows: 48 B 148 / 291, 100 B 290 / 453; 2M rows:
// 64 B 64 / 77, 132 B 125 / 224, 160 B 161 / 190, 192 B 176 / 159, 200 B 215 / 284,
// 300 B 280 / 343, 320 B 260 / 248, 400 B 362 / 399, 448 B 371 / 347, 544 B 437 / 440;
// 1.2 GB of rows: 608 B 485 / 476, 704 B 472 / 434, 800 B 495 / 480, 1204 B 488 / 518,
// 1232 B 481 / 486, 1600 B 474 / 439, 1616 B 487 / 477, 1700 B 491 / 497, 2000 B
// 490 / 485, 2032 B 495 / 505, 2408 B 474 / 468, 2700 B 475 / 455, 3601 B 480 / 481,
// 4000 B 472 / 456.
inline bool gather_nt(int R, int64_t n) {
  if (R % 128 == 0) return true;
  return n * R > STREAM_BYTES &&
         ((R % 64 == 0 && R >= 128) || (R % 32 == 0 && R >= 608) || (R % 16 == 0 && R >= 1600) ||
          (R % 4 == 0 && R >= 2400));
}
template <int LPR, int CPL, bool NT>
__global__ __launch_bounds__(G_THREADS) void k_gather16(const char *X, int64_t N,
                                                        const int32_t *ids, int64_t n, int R,
                                                        char *out, uint32_t *err) {
  constexpr int GPB = G_THREADS / LPR;
  const int sub = threadIdx.x % LPR;
  const int64_t grp = (int64_t)blockIdx.x * GPB + threadIdx.x / LPR;
  const int64_t ngrp = (int64_t)gridDim.x * GPB;
  for (int64_t j0 = grp * G_UNROLL; j0 < n; j0 += ngrp * G_UNROLL) {
    // Unconditional loads at always-valid addresses, as in the assembly
    // kernel: ids of positions past n are read at n - 1, an id outside [0, N)
    // reads the output row it would write (its row is written as zeros and
    // the error flag set), and a lane past the row reads the row's last vector.
    int32_t id[G_UNROLL];
#pragma unroll
    for (int u = 0; u < G_UNROLL; ++u) id[u] = ids[j0 + u < n ? j0 + u : n - 1];
    const char *src[G_UNROLL];
    bool ok[G_UNROLL];
    bool bad = false;
#pragma unroll
    for (int u = 0; u < G_UNROLL; ++u) {
      const int64_t j = j0 + u < n ? j0 + u : n - 1;
      ok[u] = id[u] >= 0 && (int64_t)id[u] < N;
      bad |= j0 + u < n && !ok[u];
      src[u] = ok[u] ? X + (int64_t)id[u] * R : out + j * R;
    }
    v4u v[G_UNROLL][CPL];
#pragma unroll
    for (int u = 0; u < G_UNROLL; ++u)
#pragma unroll
      for (int c = 0; c < CPL; ++c)
        v[u][c] = ld_stream(src[u] + row_vec(sub + c * LPR, R));
    if (bad && sub == 0 && err) atomicOr(err, ERR_NODE_RANGE);
#pragma unroll
    for (int u = 0; u < G_UNROLL; ++u) {
      const int64_t j = j0 + u;
      if (j < n) {
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
          const int ch = sub + c * LPR;
          if (row_has(ch, R))
            st_vec<NT>(ok[u] ? v[u][c] : v4u{0u, 0u, 0u, 0u}, out + j * R + row_vec(ch, R));
        }
      }
    }
  }
}

template <typename T>
__global__ __launch_bounds__(G_THREADS) void k_gather_any(const T *X, int64_t N, const int32_t *ids,
                                                          int64_t n, int64_t W, T *out,
                                                          uint32_t *err) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * G_THREADS + threadIdx.x) >> 6;
  const int64_t nwave = ((int64_t)gridDim.x * G_THREADS) >> 6;
  for (int64_t j = wave; j < n; j += nwave) {
    const int32_t id = ids[j];
    const bool ok = id >= 0 && (int64_t)id < N;
    if (!ok && lane == 0 && err) atomicOr(err, ERR_NODE_RANGE);
    for (int64_t c = lane; c < W; c += 64)
      out[j * W + c] = ok ? X[(int64_t)id * W + c] : zero_word<T>();
  }
}

template <int LPR, int CPL>
int gather16(const void *X, int64_t N, const int32_t *ids, int64_t n, int R, void *out,
             uint32_t *err, hipStream_t s) {
  constexpr int GPB = G_THREADS / LPR;
  int64_t blocks = ((n + G_UNROLL - 1) / G_UNROLL + GPB - 1) / GPB;
  if (blocks > (1ll << 20)) blocks = 1ll << 20;
  auto go = [&](auto nt) {
    hipLaunchKernelGGL((k_gather16<LPR, CPL, decltype(nt)::value>), dim3((unsigned)blocks),
                       dim3(G_THREADS), 0, s, (const char *)X, N, ids, n, R, (char *)out, err);
  };
  if (gather_nt(R, n)) go(std::true_type());
  else go(std::false_type());
  return DG_OK;
}

template <typename T>
void gather_any(const void *X, int64_t N, const int32_t *ids, int64_t n, int64_t row_bytes,
                void *out, uint32_t *err, hipStream_t s) {
  int64_t blocks = (n + 3) / 4;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_gather_any<T>, dim3((unsigned)blocks), dim3(G_THREADS), 0, s,
                     (const T *)X, N, ids, n, row_bytes / (int64_t)sizeof(T), (T *)out, err);
}

bool overlaps(const void *a, int64_t an, const void *b, int64_t bn) {
  if (!a || !b || an <= 0 || bn <= 0) return false;
  uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + (uintptr_t)bn && y < x + (uintptr_t)an;
}

}  // namespace

int launch_gather(const void *X, int64_t N, int64_t row_bytes, const int32_t *ids, int64_t n,
                  void *out, uint32_t *err, hipStream_t s) {
  if (n == 0) return DG_OK;
  const int w = word_bytes(row_bytes, {X, out});
  RowShape sh;
  if (row_shape16(row_bytes, &sh)) {
    with_shape(sh, [&](auto lpr, auto cpl) {
      return gather16<decltype(lpr)::value, decltype(cpl)::value>(X, N, ids, n, (int)row_bytes,
                                                                  out, err, s);
    });
  } else if (w == 16) {
    gather_any<uint4>(X, N, ids, n, row_bytes, out, err, s);
  } else if (w == 8) {
    gather_any<uint2>(X, N, ids, n, row_bytes, out, err, s);
  } else if (w == 4) {
    gather_any<uint32_t>(X, N, ids, n, row_bytes, out, err, s);
  } else if (w == 2) {
    gather_any<uint16_t>(X, N, ids, n, row_bytes, out, err, s);
  } else {
    gather_any<uint8_t>(X, N, ids, n, row_bytes, out, err, s);
  }
  DG_HIP(hipGetLastError());
  return DG_OK;
}

}  // namespace dg

using namespace dg;

extern "C" size_t dg_cache_workspace_bytes(int64_t num_nodes) {
  return num_nodes < 1 ? 0 : keysort_bytes(num_nodes);
}

extern "C" int dg_cache_by_frequency(const uint64_t *membership, int64_t N, int32_t B,
                                     int64_t cache_rows, int32_t *cache_slot,
                                     int32_t *cache_nodes, int64_t *cached, void *ws,
                                     size_t ws_bytes, hipStream_t stream) {
  if (!membership || !cache_slot || !cached || (cache_rows > 0 && !cache_nodes))
    return set_error(DG_EINVAL, "dg_cache_by_frequency: null pointer argument");
  if (N < 1 || N > 0x7fffffffll || B < 1 || B > DG_MAX_BATCHES || cache_rows < 0 ||
      cache_rows > N)
    return set_error(DG_EINVAL, "dg_cache_by_frequency: bad sizes");
  KeySort a;
  memset(&a, 0, sizeof(a));
  a.mask = membership;
  a.keep = B == 64 ? ~0ull : ((1ull << B) - 1ull);
  a.N = N;
  a.n = N;
  a.cap = cache_rows;
  a.cache_slot = cache_slot;
  a.cache_nodes = cache_nodes;
  const int rounds = fit_keysort(a, ws, ws_bytes);
  if (!ws || !rounds || ((uintptr_t)ws & 255))
    return set_error(DG_EWORKSPACE, "dg_cache_by_frequency: workspace needs %zu bytes",
                     keysort_least(a));
  int64_t totals[KEYS + 1];
  DG_TRY(keysort_run<FREQ>(a, rounds, totals, stream));
  int64_t accessed = 0;
  for (int k = 1; k < KEYS; ++k) accessed += totals[k];
  *cached = accessed < cache_rows ? accessed : cache_rows;
  return DG_OK;
}

extern "C" size_t dg_minhash_workspace_bytes(int64_t m) { return m < 0 ? 0 : keysort_bytes(m); }

extern "C" int dg_minhash_order(const uint64_t *membership, int64_t N, int32_t B,
                                const int32_t *entries, int64_t m, const int32_t *perms,
                                int32_t k, int32_t *order, int32_t *signature, void *ws,
                                size_t ws_bytes, hipStream_t stream) {
  if (!membership || (m > 0 && (!entries || !order)) || (k > 0 && !perms))
    return set_error(DG_EINVAL, "dg_minhash_order: null pointer argument");
  if (N < 1 || N > 0x7fffffffll || B < 1 || B > DG_MAX_BATCHES || m < 0 || k < 1)
    return set_error(DG_EINVAL, "dg_minhash_order: bad sizes");
  KeySort a;
  memset(&a, 0, sizeof(a));
  a.mask = membership;
  a.keep = B == 64 ? ~0ull : ((1ull << B) - 1ull);
  a.N = N;
  a.n = m;
  a.ids = entries;
  a.perms = perms;
  a.k = k;
  a.B = B;
  a.order = order;
  a.signature = signature;
  const int rounds = fit_keysort(a, ws, ws_bytes);
  if (!ws || !rounds || ((uintptr_t)ws & 255))
    return set_error(DG_EWORKSPACE, "dg_minhash_order: workspace needs %zu bytes",
                     keysort_least(a));
  int64_t totals[KEYS + 1];
  DG_TRY(keysort_run<MINHASH>(a, rounds, totals, stream));
  const uint32_t bits = (uint32_t)totals[KEYS];
  if (bits & ERR_ROW_RANGE)
    return set_error(DG_EINVAL, "dg_minhash_order: a hash value is outside [0, B)");
  if (bits) return set_error(DG_EINVAL, "invalid input data: %s", describe_device_error(bits));
  return DG_OK;
}

extern "C" int dg_gather_rows(const void *feats, int64_t N, int64_t row_bytes,
                              const int32_t *ids, int64_t n, void *out, int32_t *status,
                              hipStream_t stream) {
  if (n < 0 || row_bytes < 1 || N < 1)
    return set_error(DG_EINVAL, "dg_gather_rows: bad sizes");
  if (n == 0) return DG_OK;
  if (!feats || !ids || !out) return set_error(DG_EINVAL, "dg_gather_rows: null pointer argument");
  if (overlaps(out, n * row_bytes, feats, N * row_bytes) || overlaps(out, n * row_bytes, ids, n * 4))
    return set_error(DG_EINVAL, "dg_gather_rows: output overlaps an input");
  return launch_gather(feats, N, row_bytes, ids, n, out, reinterpret_cast<uint32_t *>(status),
                       stream);
}
