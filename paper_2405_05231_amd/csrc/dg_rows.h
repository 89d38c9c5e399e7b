// Feature-row movement shared by the packing gather and the assembly kernel.
//
// A feature row is row_bytes opaque bytes.  A row of 16 to 4096 bytes moves as
// C = ceil(row_bytes/16) 16-byte vectors: vector c starts at byte 16*c, the last
// one at row_bytes - 16, so where row_bytes is no multiple of 16 the last two
// overlap and write the bytes they share with the same values.  A group of LPR
// lanes owns one row and each lane moves CPL vectors of it (vector c of the row
// goes to lane c % LPR), so each load instruction of a group covers LPR*16
// contiguous bytes.  Neither rows nor base pointers need any alignment: the
// vectors are read and written by plain 16-byte global accesses, which gfx950
// takes at any byte address.  Each group handles UNROLL rows per iteration and
// issues all their loads before any store, to keep enough bytes in flight to
// cover HBM latency.  Shorter and longer rows take narrower words and one wave
// per row.
#pragma once

#include <type_traits>

#include "dg_common.h"

namespace dg {

struct RowShape {
  int lpr;  // lanes per row
  int cpl;  // vectors per lane
};

// Launch shapes of the vector path, by row size; false: the row takes the
// generic path.  Rows of 129 to 192 vectors take three vectors per lane only where
// they are no multiple of 4 bytes, since a lane past the row still reads the row's
// last vector, which costs more unaligned (3 against 4 vectors, gather / assembly of
// 1.2 GB: 2155 B 494 / 542 and 504 / 546 us, 2601 B 481 / 505 and 482 / 503; but
// 2064 B 470 / 455 and 555 / 531, 2408 B 488 / 474 and 513 / 490, 3000 B 492 / 487 and
// 493 / 472).
inline bool row_shape16(int64_t row_bytes, RowShape *s) {
  if (row_bytes < 16) return false;
  const int64_t C = (row_bytes + 15) / 16;
  if (C <= 1) { *s = {1, 1}; return true; }
  if (C <= 2) { *s = {2, 1}; return true; }
  if (C <= 4) { *s = {4, 1}; return true; }
  if (C <= 8) { *s = {8, 1}; return true; }
  if (C <= 16) { *s = {16, 1}; return true; }
  if (C <= 32) { *s = {32, 1}; return true; }
  if (C <= 64) { *s = {64, 1}; return true; }
  if (C <= 128) { *s = {64, 2}; return true; }
  if (C <= 192 && row_bytes % 4 != 0) { *s = {64, 3}; return true; }
  if (C <= 256) { *s = {64, 4}; return true; }
  return false;
}

// Calls f(LPR, CPL) with the shape's values as compile-time constants.
template <typename F>
inline int with_shape(const RowShape &s, F f) {
  using std::integral_constant;
  if (s.lpr == 1) return f(integral_constant<int, 1>(), integral_constant<int, 1>());
  if (s.lpr == 2) return f(integral_constant<int, 2>(), integral_constant<int, 1>());
  if (s.lpr == 4) return f(integral_constant<int, 4>(), integral_constant<int, 1>());
  if (s.lpr == 8) return f(integral_constant<int, 8>(), integral_constant<int, 1>());
  if (s.lpr == 16) return f(integral_constant<int, 16>(), integral_constant<int, 1>());
  if (s.lpr == 32) return f(integral_constant<int, 32>(), integral_constant<int, 1>());
  if (s.cpl == 1) return f(integral_constant<int, 64>(), integral_constant<int, 1>());
  if (s.cpl == 2) return f(integral_constant<int, 64>(), integral_constant<int, 2>());
  if (s.cpl == 3) return f(integral_constant<int, 64>(), integral_constant<int, 3>());
  return f(integral_constant<int, 64>(), integral_constant<int, 4>());
}

// Rows in flight per lane group: four for rows of one vector per lane, two
// when each lane moves two or more vectors of a row (keeps registers, and so
// occupancy, in check for wide rows).
__host__ __device__ constexpr int rows_in_flight(int cpl) { return cpl >= 2 ? 2 : 4; }

inline int word_bytes(int64_t row_bytes, std::initializer_list<const void *> ptrs) {
  int w = 16;
  auto fits = [&](int a) {
    if (row_bytes % a) return false;
    for (const void *p : ptrs)
      if (p && ((uintptr_t)p % a)) return false;
    return true;
  };
  while (w > 1 && !fits(w)) w >>= 1;
  return w;
}

// Outputs of more bytes than this leave the caches anyway (256 MB at the last level).
constexpr int64_t STREAM_BYTES = 320 * 1000 * 1000;

// 16-byte row vector as a native vector type, so the nontemporal builtins
// apply.  Its address may have any alignment.  A nontemporal store leaves the
// caches to reusable lines, but a row that ends inside a 128-byte line then
// reaches memory as a partial line more often; each kernel states which of the
// two it stores with and what both measured.
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef v4u v4u_any __attribute__((aligned(1)));

__device__ __forceinline__ v4u ld_row(const char *p) {
  return *reinterpret_cast<const v4u_any *>(p);
}
__device__ __forceinline__ v4u ld_stream(const char *p) {
  return __builtin_nontemporal_load(reinterpret_cast<const v4u_any *>(p));
}
__device__ __forceinline__ void st_row(v4u x, char *p) {
  *reinterpret_cast<v4u_any *>(p) = x;
}
__device__ __forceinline__ void st_stream(v4u x, char *p) {
  __builtin_nontemporal_store(x, reinterpret_cast<v4u_any *>(p));
}
template <bool NT>
__device__ __forceinline__ void st_vec(v4u x, char *p) {
  if (NT) st_stream(x, p);
  else st_row(x, p);
}
// Byte offset of vector ch in a row of R bytes; a vector past the row is its
// last one (loaded and dropped, so that no load needs a branch).
__device__ __forceinline__ int row_vec(int ch, int R) { return min(16 * ch, R - 16); }
__device__ __forceinline__ bool row_has(int ch, int R) { return 16 * ch < R; }

// The row copy of one packing call: the fan-out gather over U_nc, plus the
// cache rows when a cache table is given.
struct RowCopy {
  const void *X;
  int64_t N, row_bytes;
  const int32_t *ids;
  const int64_t *off;
  int64_t n, pairs;
  const int64_t *dest;
  void *packed;
  const int32_t *cache_nodes;
  int64_t n_cache;
  void *cache_table;
  uint32_t *err;
};
// Launches the fan-out gather of one RowCopy on stream s (nothing when it has
// no item); DG_EHIP when the launch fails.
int launch_fanout(const RowCopy &r, hipStream_t s);

template <typename T>
__device__ __forceinline__ T zero_word() {
  T z;
  memset(&z, 0, sizeof(T));
  return z;
}

}  // namespace dg
