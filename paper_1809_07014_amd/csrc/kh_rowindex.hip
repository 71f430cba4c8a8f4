// Index of sorted rows by their top key bits (RowIndex, kh_rows.hpp).
#include "kh_host.hpp"
#include "kh_rows.hpp"

using namespace kh;

namespace {

constexpr int kXB = 256;

// start[p] = first row whose prefix is at least p, for p in [0, 2^bits].
// Row i owns the entries after row i - 1's prefix up to its own (row n those
// to the end).  Most gaps are short; a long one (keys crowd where the
// canonical form and the genomes' composition put them, and leave stretches
// empty) is written by the whole wave.
//
// Bound by the streams: 8W bytes of key in and 4 bytes per entry out.
template <int W>
__global__ __launch_bounds__(kXB) void k_row_index(const uint64_t* keys, int64_t n, int top,
                                                   int bits, uint32_t* start) {
  const int64_t i = (int64_t)blockIdx.x * kXB + threadIdx.x;
  uint64_t lo = 1, hi = 0;  // entries [lo, hi] get i
  if (i <= n) {
    lo = i == 0 ? 0 : (uint64_t)row_prefix<W>(keys + (i - 1) * W, top, bits) + 1;
    hi = i < n ? (uint64_t)row_prefix<W>(keys + i * W, top, bits) : 1ull << bits;
  }
  const bool wide = lo + 8 <= hi;
  if (!wide)
    for (uint64_t e = lo; e <= hi; ++e) start[e] = (uint32_t)i;
  uint64_t todo = __ballot(wide);
  while (todo) {
    const int src = __ffsll((long long)todo) - 1;
    todo &= todo - 1;
    const uint64_t l = __shfl((unsigned long long)lo, src);
    const uint64_t h = __shfl((unsigned long long)hi, src);
    const uint32_t v = (uint32_t)__shfl((unsigned long long)i, src);
    for (uint64_t e = l + (threadIdx.x & 63); e <= h; e += 64) start[e] = v;
  }
}

// Entry p with the digits its rows have; all of them for a bucket of more rows
// than a thread should look through.
constexpr uint32_t kMaskRows = 64;

template <int W>
__global__ __launch_bounds__(kXB) void k_row_masks(const uint64_t* keys, int top, RowIndex ix,
                                                   int sub, uint2* entry) {
  const uint64_t p = (uint64_t)blockIdx.x * kXB + threadIdx.x;
  if (p > 1ull << ix.bits) return;
  const uint32_t r0 = ix.start[p], r1 = p < 1ull << ix.bits ? ix.start[p + 1] : r0;
  uint32_t m = r1 - r0 > kMaskRows ? ~0u : 0u;
  if (!m)
    for (uint32_t r = r0; r < r1; ++r)
      m |= 1u << (row_prefix<W>(keys + (uint64_t)r * W, top, ix.bits + sub) & ((1u << sub) - 1u));
  entry[p] = make_uint2(r0, m);
}

}  // namespace

// A quarter to half an entry per row: a bucket holds two to four rows where
// keys are spread evenly, so a lookup's binary search stays within a line or
// two, and the index is small enough that part of it stays in the memory-side
// cache.  1.6e8 rows (k_link, 1.6e8 lookups): 12.0 ms at ceil(log2 n) bits,
// 11.6 with one bit less, 11.3 with two; the build 1.6, 1.2 and 1.0 ms.
// Where there is no memory for that many entries, fewer do (longer searches).
int kh::row_index_build(Pool* pool, const uint64_t* keys, int64_t n, uint32_t k,
                        Buf<uint32_t>& start, RowIndex* ix, hipStream_t s, int most_bits) {
  int bits = 1;
  while (bits < most_bits && bits < 2 * (int)k && (4ll << bits) < n) ++bits;
  start.pool = pool;
  for (;; bits = bits > 4 ? bits - 3 : 1) {
    const int rc = start.alloc((1ull << bits) + 1);
    if (rc == KH_OK) break;
    if (rc != KH_ENOMEM || bits == 1) return rc;
  }
  const int W = (int)(k + 31) / 32, top = 2 * (int)k - 64 * (W - 1);
  const dim3 g((unsigned)((n + 1 + kXB - 1) / kXB)), t(kXB);
  switch (W) {
    case 1: hipLaunchKernelGGL(k_row_index<1>, g, t, 0, s, keys, n, top, bits, start.p); break;
    case 2: hipLaunchKernelGGL(k_row_index<2>, g, t, 0, s, keys, n, top, bits, start.p); break;
    case 3: hipLaunchKernelGGL(k_row_index<3>, g, t, 0, s, keys, n, top, bits, start.p); break;
    default: hipLaunchKernelGGL(k_row_index<4>, g, t, 0, s, keys, n, top, bits, start.p); break;
  }
  HIP_TRY(hipGetLastError());
  ix->start = start.p;
  ix->bits = bits;
  return KH_OK;
}

// The masks cost one more pass over the keys (0.28 ms for 6.2e7 rows), which
// pays where many keys looked up are no rows: the lookups of 4e6 reads
// localised take 2.4 ms with masks, 3.1 without.  The traversal's and the
// merge's keys nearly all are rows.
int kh::masked_index_build(Pool* pool, const uint64_t* keys, int64_t n, uint32_t k,
                           Buf<uint32_t>& start, Buf<uint64_t>& entry, MaskedIndex* ix,
                           hipStream_t s) {
  RowIndex x{};
  entry.pool = pool;
  for (int most = 32;; most = x.bits > 4 ? x.bits - 3 : 1) {
    KH_TRY(row_index_build(pool, keys, n, k, start, &x, s, most));
    const int rc = entry.alloc((1ull << x.bits) + 1);
    if (rc == KH_OK) break;
    if (rc != KH_ENOMEM || x.bits == 1) return rc;
  }
  const int room = (2 * (int)k < 32 ? 2 * (int)k : 32) - x.bits;
  const int sub = room < 5 ? room : 5;
  uint2* e = reinterpret_cast<uint2*>(entry.p);
  const int W = (int)(k + 31) / 32, top = 2 * (int)k - 64 * (W - 1);
  const dim3 g((unsigned)(((1ull << x.bits) + kXB) / kXB)), t(kXB);
  switch (W) {
    case 1: hipLaunchKernelGGL(k_row_masks<1>, g, t, 0, s, keys, top, x, sub, e); break;
    case 2: hipLaunchKernelGGL(k_row_masks<2>, g, t, 0, s, keys, top, x, sub, e); break;
    case 3: hipLaunchKernelGGL(k_row_masks<3>, g, t, 0, s, keys, top, x, sub, e); break;
    default: hipLaunchKernelGGL(k_row_masks<4>, g, t, 0, s, keys, top, x, sub, e); break;
  }
  HIP_TRY(hipGetLastError());
  ix->entry = e;
  ix->bits = x.bits;
  ix->sub = sub;
  return KH_OK;
}
