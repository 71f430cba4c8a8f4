// Device helpers over exported rows (keys of W words, most significant
// first, the k-mer right-aligned in 2k bits, rows in ascending key order):
// one-base shifts of a k-mer, binary search over sorted rows, and lookups
// through an index of the rows by their top key bits.  Used by the traversal,
// merge, pruning and localisation kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace kh {

// S[1..k) + b, in the export layout (W words, most significant first, the
// k-mer right-aligned in 2k bits; `top` bits live in word 0).
template <int W>
__device__ __forceinline__ void push_right(const uint64_t (&s)[W], int b, int top,
                                           uint64_t (&t)[W]) {
#pragma unroll
  for (int j = 0; j < W - 1; ++j) t[j] = (s[j] << 2) | (s[j + 1] >> 62);
  t[W - 1] = (s[W - 1] << 2) | (uint64_t)b;
  if (top < 64) t[0] &= (1ull << top) - 1;
}

// b + S[0..k-1).
template <int W>
__device__ __forceinline__ void push_left(const uint64_t (&s)[W], int b, int top,
                                          uint64_t (&t)[W]) {
#pragma unroll
  for (int j = W - 1; j > 0; --j) t[j] = (s[j] >> 2) | (s[j - 1] << 62);
  t[0] = (s[0] >> 2) | ((uint64_t)b << (top - 2));
}

template <int W>
__device__ __forceinline__ int cmp_rows(const uint64_t* a, const uint64_t* b) {
#pragma unroll
  for (int j = 0; j < W; ++j)
    if (a[j] != b[j]) return a[j] < b[j] ? -1 : 1;
  return 0;
}

// First row of keys[0..n) not less than q.
template <int W>
__device__ __forceinline__ int64_t lower_bound_rows(const uint64_t* keys, int64_t n,
                                                    const uint64_t* q) {
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = lo + (hi - lo) / 2;
    if (cmp_rows<W>(keys + mid * W, q) < 0)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

// Index of sorted rows by the top `bits` bits of the 2k-bit key: the rows of
// prefix p are [start[p], start[p + 1]) (2^bits + 1 entries).  The rows are
// sorted already, so it is built by one streaming pass over the keys (no
// hashing, no atomics), and a lookup costs one entry pair and the few rows of
// its bucket (kh_rowindex.hip).
struct RowIndex {
  const uint32_t* start;
  int bits;  // 1 .. 32, at most 2k
};

// The top `bits` bits of a key whose word 0 holds `top` bits.
template <int W>
__device__ __forceinline__ uint32_t row_prefix(const uint64_t* w, int top, int bits) {
  if (W == 1 || bits <= top) return (uint32_t)(w[0] >> (top - bits));
  const int low = bits - top;  // bits of word 1, 1 .. 31
  return (uint32_t)((w[0] << low) | (w[W > 1 ? 1 : 0] >> (64 - low)));
}

// Row of key q among the sorted rows [lo, hi), or -1.
template <int W>
__device__ __forceinline__ int64_t find_between(const uint64_t* keys, int64_t lo, int64_t hi,
                                                const uint64_t (&q)[W]) {
  while (lo < hi) {
    const int64_t mid = lo + (hi - lo) / 2;
    uint64_t w[W];  // the whole row at once: one round trip per probe
#pragma unroll
    for (int j = 0; j < W; ++j) w[j] = keys[mid * W + j];
    const int c = cmp_rows<W>(w, q);
    if (c == 0) return mid;
    if (c < 0)
      lo = mid + 1;
    else
      hi = mid;
  }
  return -1;
}

// Row of key q, or -1.
template <int W>
__device__ __forceinline__ int64_t find_row(const uint64_t* keys, const RowIndex& ix, int top,
                                            const uint64_t (&q)[W]) {
  const uint32_t p = row_prefix<W>(q, top, ix.bits);
  return find_between<W>(keys, ix.start[p], ix.start[(uint64_t)p + 1], q);
}

// No index: all n rows.  Some 26 probes, one after another, and few of them
// equal: the plain search looks at no more of a row than decides its side.
struct AllRows {
  int64_t n;
};

template <int W>
__device__ __forceinline__ int64_t find_row(const uint64_t* keys, const AllRows& rows, int,
                                            const uint64_t (&q)[W]) {
  const int64_t r = lower_bound_rows<W>(keys, rows.n, q);
  return r < rows.n && cmp_rows<W>(keys + r * W, q) == 0 ? r : -1;
}

// The index with, beside each entry's first row, a bit per next key digit
// (`sub` more bits, up to 32 digits) that some row of the bucket has: a key
// that is no row is told so by the entry's line alone, mostly.
struct MaskedIndex {
  const uint2* entry;  // (first row, digits), 2^bits + 1 of them
  int bits, sub;       // bits + sub <= 32 and 2k
};

template <int W>
__device__ __forceinline__ int64_t find_row(const uint64_t* keys, const MaskedIndex& ix, int top,
                                            const uint64_t (&q)[W]) {
  const uint32_t p = row_prefix<W>(q, top, ix.bits + ix.sub);
  const uint64_t b = p >> ix.sub;
  const uint2 x = ix.entry[b];
  const int64_t hi = ix.entry[b + 1].x;
  if (!((x.y >> (p & ((1u << ix.sub) - 1u))) & 1u)) return -1;
  return find_between<W>(keys, x.x, hi, q);
}

}  // namespace kh
