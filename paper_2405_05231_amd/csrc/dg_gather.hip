// The fan-out gather of batched packing (DiskGNN §5.2, Fig. 6b): each row of
// the group's non-cached unique set is read once from the feature table and
// written to every packed row that holds it, and (with a cache table) the
// cache rows are filled in the same launch, the cache taken as one more
// mini-batch.
#include <initializer_list>

#include "dg_rows.h"

namespace dg {
namespace {

constexpr int THREADS = 256;

// Which rows take nontemporal stores: as in the row gather, but the packed rows of a
// node lie apart, so that fewer lines merge in L2 and the line lies lower.  Nontemporal
// over plain, the whole packing: packed rows of 232 MB (900 B) 1.13, 310 MB (1200 B) 1.00,
// 400 MB (1540 B) 0.98, 517 MB (2000 B) 0.95.  Packing of 8 lists, plain against
// nontemporal, us: 2M rows in all: 132 B 460 / 513, 192 B 473 / 466, 288 B 568 / 583,
// 320 B 572 / 562, 400 B 653 / 672, 448 B 649 / 625, 544 B 778 / 779; 1.2 GB: 672 B
// 766 / 757, 688 B 773 / 781, 700 B 776 / 788, 850 B 743 / 747, 900 B 712 / 712, 944 B
// 693 / 686, 1204 B 662 / 648, 1601 B 626 / 610, 2400 B 554 / 532, 4000 B 520 / 495.
inline bool fanout_nt(int64_t R, int64_t rows) {
  if (R % 128 == 0) return true;
  return rows * R > STREAM_BYTES &&
         ((R % 64 == 0 && R >= 128) || (R % 32 == 0 && R >= 640) || R >= 900);
}

// Fan-out gather, vector path: a group of LPR lanes reads the row of one U_nc
// node once and stores it into each of its destination rows.  Every U_nc node
// has at least one destination; its first destination index is loaded together
// with the row, so the common single-destination case needs two dependent
// round trips (indices, then row + destination) before its stores.  Bound by
// HBM; nontemporal loads, and nontemporal stores (NT) where fanout_nt says so: for
// 512-byte rows a launch with plain stores is up to 15% shorter (1M nodes: 88 against
// 104 us), but the assembly that follows takes that time back (whole step 1.339
// against 1.332 ms).
// Items n_unc .. n_unc + n_cache - 1 fill the cache table, the cache taken as
// one more mini-batch of the same pass: item n_unc + s copies the row of
// cache_nodes[s] into cache row s (a slot holding -1 is left as it is; an ID
// outside [0, N) is reported and its row left as it is).
template <int LPR, int CPL, bool NT>
__global__ __launch_bounds__(THREADS) void k_fanout16(const char *X, int64_t N,
                                                      const int32_t *unc_ids,
                                                      const int64_t *unc_off, int64_t n_unc,
                                                      int64_t n_pairs, const int64_t *pairdest,
                                                      int R, char *packed,
                                                      const int32_t *cache_nodes,
                                                      int64_t n_cache, char *cache_table,
                                                      uint32_t *err) {
  constexpr int UNROLL = rows_in_flight(CPL);
  constexpr int GPB = THREADS / LPR;
  const int sub = threadIdx.x % LPR;
  const int64_t grp = (int64_t)blockIdx.x * GPB + threadIdx.x / LPR;
  const int64_t ngrp = (int64_t)gridDim.x * GPB;
  const int64_t n_items = n_unc + n_cache;
  for (int64_t i0 = grp * UNROLL; i0 < n_items; i0 += ngrp * UNROLL) {
    int64_t p0[UNROLL], p1[UNROLL], d0[UNROLL];
    int32_t id[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int64_t i = i0 + u;
      p0[u] = p1[u] = 0;
      id[u] = -1;
      if (i < n_unc) {
        id[u] = unc_ids[i];
        p0[u] = unc_off[i];
        p1[u] = i + 1 < n_unc ? unc_off[i + 1] : n_pairs;
      } else if (i < n_items) {
        const int32_t v = cache_nodes[i - n_unc];
        if (v >= 0 && (int64_t)v < N) id[u] = v;
        else if (v != -1 && sub == 0) atomicOr(err, ERR_NODE_RANGE);
      }
    }
    v4u v[UNROLL][CPL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      d0[u] = p1[u] > p0[u] ? pairdest[p0[u]] : -1;
      const char *src = id[u] >= 0 ? X + (int64_t)id[u] * R : nullptr;
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const int ch = sub + c * LPR;
        v[u][c] = (src && row_has(ch, R)) ? ld_stream(src + row_vec(ch, R))
                                          : v4u{0u, 0u, 0u, 0u};
      }
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int64_t i = i0 + u;
      char *dst;
      if (i >= n_unc) {  // a cache row
        if (i >= n_items || id[u] < 0) continue;
        dst = cache_table + (i - n_unc) * R;
      } else {
        if (d0[u] < 0) continue;
        dst = packed + d0[u] * R;
      }
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const int ch = sub + c * LPR;
        if (row_has(ch, R)) st_vec<NT>(v[u][c], dst + row_vec(ch, R));
      }
      for (int64_t p = p0[u] + 1; p < p1[u]; ++p) {
        dst = packed + pairdest[p] * R;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
          const int ch = sub + c * LPR;
          if (row_has(ch, R)) st_vec<NT>(v[u][c], dst + row_vec(ch, R));
        }
      }
    }
  }
}

// Any row size / alignment: one wave per item (U_nc node, then cache row), words
// of sizeof(T).
template <typename T>
__global__ __launch_bounds__(THREADS) void k_fanout_any(const T *X, int64_t N,
                                                        const int32_t *unc_ids,
                                                        const int64_t *unc_off, int64_t n_unc,
                                                        int64_t n_pairs, const int64_t *pairdest,
                                                        int64_t W, T *packed,
                                                        const int32_t *cache_nodes,
                                                        int64_t n_cache, T *cache_table,
                                                        uint32_t *err) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * THREADS + threadIdx.x) >> 6;
  const int64_t nwave = ((int64_t)gridDim.x * THREADS) >> 6;
  for (int64_t i = wave; i < n_unc + n_cache; i += nwave) {
    if (i >= n_unc) {
      const int64_t s = i - n_unc;
      const int32_t v = cache_nodes[s];
      if (v < 0 || (int64_t)v >= N) {
        if (v != -1 && lane == 0) atomicOr(err, ERR_NODE_RANGE);
        continue;
      }
      for (int64_t c = lane; c < W; c += 64) cache_table[s * W + c] = X[(int64_t)v * W + c];
      continue;
    }
    const T *src = X + (int64_t)unc_ids[i] * W;
    int64_t p0 = unc_off[i], p1 = i + 1 < n_unc ? unc_off[i + 1] : n_pairs;
    for (int64_t c = lane; c < W; c += 64) {
      T x = src[c];
      for (int64_t p = p0; p < p1; ++p) packed[pairdest[p] * W + c] = x;
    }
  }
}


template <int LPR, int CPL>
int launch16(const RowCopy &r, hipStream_t s) {
  constexpr int GPB = THREADS / LPR;
  constexpr int UNROLL = rows_in_flight(CPL);
  int64_t groups = (r.n + r.n_cache + UNROLL - 1) / UNROLL;
  int64_t blocks = (groups + GPB - 1) / GPB;
  if (blocks > (1ll << 20)) blocks = 1ll << 20;
  auto go = [&](auto nt) {
    hipLaunchKernelGGL((k_fanout16<LPR, CPL, decltype(nt)::value>), dim3((unsigned)blocks),
                       dim3(THREADS), 0, s, (const char *)r.X, r.N, r.ids, r.off, r.n, r.pairs,
                       r.dest, (int)r.row_bytes, (char *)r.packed, r.cache_nodes, r.n_cache,
                       (char *)r.cache_table, r.err);
  };
  if (fanout_nt(r.row_bytes, r.pairs + r.n_cache)) go(std::true_type());
  else go(std::false_type());
  return DG_OK;
}

template <typename T>
void launch_any(const RowCopy &r, hipStream_t s) {
  int64_t blocks = (r.n + r.n_cache + 3) / 4;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_fanout_any<T>, dim3((unsigned)blocks), dim3(THREADS), 0, s,
                     (const T *)r.X, r.N, r.ids, r.off, r.n, r.pairs, r.dest,
                     r.row_bytes / (int64_t)sizeof(T), (T *)r.packed, r.cache_nodes, r.n_cache,
                     (T *)r.cache_table, r.err);
}

}  // namespace

int launch_fanout(const RowCopy &r, hipStream_t s) {
  if (r.n + r.n_cache == 0) return DG_OK;
  const int w = word_bytes(r.row_bytes, {r.X, r.packed, r.cache_table});
  RowShape sh;
  if (row_shape16(r.row_bytes, &sh)) {
    with_shape(sh, [&](auto lpr, auto cpl) {
      return launch16<decltype(lpr)::value, decltype(cpl)::value>(r, s);
    });
  } else if (w == 16) {
    launch_any<uint4>(r, s);
  } else if (w == 8) {
    launch_any<uint2>(r, s);
  } else if (w == 4) {
    launch_any<uint32_t>(r, s);
  } else if (w == 2) {
    launch_any<uint16_t>(r, s);
  } else {
    launch_any<uint8_t>(r, s);
  }
  DG_HIP(hipGetLastError());
  return DG_OK;
}

}  // namespace dg
