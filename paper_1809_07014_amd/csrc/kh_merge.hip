// Merging the k-mers of earlier contigs into a k-mer table (paper Section
// II, Algorithm 1's Merge step, and the subsection on merging k-mer sets):
// contigs assembled with a smaller k contribute every one of their k-mers as
// an error-free k-mer with unique high-quality extensions; a k-mer already
// in the table keeps its row (the reads' k-mers are stored first), a new
// one becomes a row with count 0 whose code per side is the neighbouring
// contig base when all its occurrences have one and agree, 'X' when none
// has one, 'F' otherwise.
//
// Method.  Nearly every contig k-mer is a row of the table already, so the
// contigs' windows are first looked up in it (through an index of the sorted
// rows by their top bits), and only the windows that are not there are
// counted, as reads whose every base is of high quality with min_count 1:
// that gives each new k-mer its number of occurrences and its
// neighbouring-base tallies, from which the rule above follows (an occurrence
// lacks a left neighbour iff the count exceeds the left tallies' sum).  The
// new rows' places among the table's come from the same index; a table row
// moves up by the number of new rows placed at or before it.
#include <algorithm>
#include <vector>

#include "kh_device.hpp"
#include "kh_host.hpp"
#include "kh_rows.hpp"

using namespace kh;

namespace {

constexpr int kMB = 256;

// The contigs' windows that are no rows of the table: one bit per window
// start (64 per word, by position), and in ctr the valid windows and the
// absent ones.
//
// Bound by the lookups' random lines (an index entry and the rows of its
// bucket per window); the planes stream.  7.4e7 windows against 6.0e7 rows
// (k = 33): 4.0 ms; counting every window in a table of its own and sorting
// its 7e7 rows took 20 ms.
template <int W>
__global__ __launch_bounds__(kBlock) void k_absent(AbsentArgs a, RowIndex ix) {
  __shared__ uint64_t s_bases[kBaseWords];
  __shared__ uint64_t s_hq[kPlaneWords];
  __shared__ uint64_t s_bad[kPlaneWords];
  __shared__ uint64_t s_st[kPlaneWords];
  __shared__ uint64_t s_red[kBlock / 64];
  const int tid = threadIdx.x;
  const int top = 2 * (int)a.k - 64 * (W - 1);
  const int64_t n_tiles = (a.n + kTile - 1) / kTile;
  uint64_t win = 0, absent = 0;
  for (int64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
    const int64_t P0 = t * kTile, O = P0 - kHalo;
    __syncthreads();
    stage_tile(a.bases, a.hq, a.bad, a.st, a.base_words, a.plane_words, O, s_bases, s_hq, s_bad,
               s_st);
    __syncthreads();
#pragma unroll 1
    for (int j = 0; j < kTile / kBlock; ++j) {
      const int64_t p = P0 + j * kBlock + tid;
      const uint32_t lp = (uint32_t)(p - O);
      bool miss = false;
      if (p + (int64_t)a.k <= a.n && !any_bits(s_bad, lp, a.k) &&
          !any_bits(s_st, lp + 1, a.k - 1)) {
        uint64_t f[W], r[W];
        window_words<W>(s_bases, 2 * lp, a.k, f);
        revcomp_words<W>(f, a.k, r);
        const bool use_rc = words_less<W>(r, f);
#pragma unroll
        for (int w = 0; w < W; ++w) f[w] = use_rc ? r[w] : f[w];
        ++win;
        miss = find_row<W>(a.keys, ix, top, f) < 0;
        absent += miss ? 1 : 0;
      }
      const uint64_t m = __ballot(miss);
      if ((tid & 63) == 0) a.absent[p >> 6] = m;
    }
  }
  __syncthreads();
  block_add(&a.ctr[kCtrWindows], win, s_red);
  __syncthreads();
  block_add(&a.ctr[kCtrPassed], absent, s_red);
}

// New rows: the table rows before each (its place is that plus its own
// number; the places rise with the rows).
template <int W>
__global__ __launch_bounds__(kMB) void k_merge_probe(const uint64_t* tkeys, RowIndex ix, int top,
                                                     const uint64_t* ckeys, int64_t nc,
                                                     int64_t* cpos) {
  const int64_t j = (int64_t)blockIdx.x * kMB + threadIdx.x;
  if (j >= nc) return;
  const uint64_t* q = ckeys + j * W;
  const uint32_t p = row_prefix<W>(q, top, ix.bits);
  const int64_t lo = ix.start[p], hi = ix.start[(uint64_t)p + 1];
  cpos[j] = lo + lower_bound_rows<W>(tkeys + lo * W, hi - lo, q);
}

__device__ __forceinline__ uint8_t contig_side(const uint32_t* tallies, uint32_t count) {
  uint32_t sum = 0, nb = 0, which = 0;
  for (int b = 0; b < 4; ++b) {
    sum += tallies[b];
    if (tallies[b]) {
      ++nb;
      which = (uint32_t)b;
    }
  }
  if (nb == 0) return 'X';
  if (nb == 1 && sum == count) return (uint8_t)"ACGT"[which];
  return 'F';
}

// Entries of the ascending cpos[lo, hi) that are at most i, plus lo.
__device__ __forceinline__ int64_t places_up_to(const int64_t* cpos, int64_t lo, int64_t hi,
                                                int64_t i) {
  while (lo < hi) {
    const int64_t mid = lo + (hi - lo) / 2;
    if (cpos[mid] <= i)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

// Table rows keep their record; each moves up by the new rows before it.  A
// block's rows share a short stretch of the new rows, found by two searches
// per block.
//
// Bound by the rows themselves, read and written once: 6.0e7 rows of two-word
// keys (6.5 GB) in 1.93 ms (4.7 ms with a binary search over all contig rows
// per table row).
template <int W>
__global__ __launch_bounds__(kMB) void k_merge_place_table(
    const uint64_t* tkeys, const uint32_t* tcounts, const uint32_t* text, const uint8_t* tcodes,
    int64_t nt, const int64_t* cpos, int64_t nc, uint64_t* okeys, uint32_t* ocounts,
    uint32_t* oext, uint8_t* ocodes) {
  __shared__ int64_t s_range[2];
  const int64_t i0 = (int64_t)blockIdx.x * kMB, i = i0 + threadIdx.x;
  if (threadIdx.x < 2)  // new rows at or before the block's first row, its last one
    s_range[threadIdx.x] = places_up_to(cpos, 0, nc, threadIdx.x == 0 ? i0 : i0 + kMB - 1);
  __syncthreads();
  if (i >= nt) return;
  const int64_t o = i + places_up_to(cpos, s_range[0], s_range[1], i);
#pragma unroll
  for (int j = 0; j < W; ++j) okeys[o * W + j] = tkeys[i * W + j];
  ocounts[o] = tcounts[i];
  const uint4* e = reinterpret_cast<const uint4*>(text + i * 8);
  uint4* d = reinterpret_cast<uint4*>(oext + o * 8);
  d[0] = e[0];
  d[1] = e[1];
  reinterpret_cast<uint16_t*>(ocodes)[o] = reinterpret_cast<const uint16_t*>(tcodes)[i];
}

// New contig rows: count 0, no tallies, codes from the contig neighbours.
template <int W>
__global__ __launch_bounds__(kMB) void k_merge_place_contigs(
    const uint64_t* ckeys, const uint32_t* ccounts, const uint32_t* cext, int64_t nc,
    const int64_t* cpos, uint64_t* okeys, uint32_t* ocounts, uint32_t* oext, uint8_t* ocodes) {
  const int64_t j = (int64_t)blockIdx.x * kMB + threadIdx.x;
  if (j >= nc) return;
  const int64_t o = cpos[j] + j;
#pragma unroll
  for (int w = 0; w < W; ++w) okeys[o * W + w] = ckeys[j * W + w];
  ocounts[o] = 0;
#pragma unroll
  for (int x = 0; x < 8; ++x) oext[o * 8 + x] = 0;
  ocodes[2 * o] = contig_side(cext + j * 8, ccounts[j]);
  ocodes[2 * o + 1] = contig_side(cext + j * 8 + 4, ccounts[j]);
}

unsigned mgrid(int64_t n) { return (unsigned)((n + kMB - 1) / kMB); }

template <int W>
int merge_rows(kh_ctx* ctx, const kh_table* t, const RowIndex& ix, Buf<uint32_t>& start,
               const kh_table* c, hipStream_t s, kh_table* out) {
  Pool* pool = &ctx->pool;
  const int64_t nt = t->n_rows, nc = c->n_rows, n = nt + nc;
  Buf<int64_t> cpos(pool);
  Buf<uint64_t> keys(pool);
  Buf<uint32_t> counts(pool), ext(pool);
  Buf<uint8_t> codes(pool);
  KH_TRY(cpos.alloc(nc + 1));
  if (nc > 0) {
    hipLaunchKernelGGL((k_merge_probe<W>), dim3(mgrid(nc)), dim3(kMB), 0, s, t->keys, ix,
                       2 * (int)t->k - 64 * (W - 1), c->keys, nc, cpos.p);
    HIP_TRY(hipGetLastError());
  }
  start.reset();  // the index gives way to the merged rows
  KH_TRY(keys.alloc((uint64_t)n * W));
  KH_TRY(counts.alloc((uint64_t)n));
  KH_TRY(ext.alloc((uint64_t)n * 8));
  KH_TRY(codes.alloc((uint64_t)n * 2));
  if (nt > 0) {
    hipLaunchKernelGGL((k_merge_place_table<W>), dim3(mgrid(nt)), dim3(kMB), 0, s, t->keys,
                       t->counts, t->ext, t->codes, nt, cpos.p, nc, keys.p, counts.p, ext.p,
                       codes.p);
    HIP_TRY(hipGetLastError());
  }
  if (nc > 0) {
    hipLaunchKernelGGL((k_merge_place_contigs<W>), dim3(mgrid(nc)), dim3(kMB), 0, s, c->keys,
                       c->counts, c->ext, nc, cpos.p, keys.p, counts.p, ext.p, codes.p);
    HIP_TRY(hipGetLastError());
  }
  HIP_TRY(hipStreamSynchronize(s));
  out->n_rows = n;
  out->n_windows = t->n_windows;
  out->keys = keys.release();
  out->counts = counts.release();
  out->ext = ext.release();
  out->codes = codes.release();
  return KH_OK;
}

}  // namespace

void kh::launch_absent(const AbsentArgs& a, const RowIndex& ix, int blocks, hipStream_t s) {
  const dim3 g((unsigned)std::max<int64_t>(1, std::min<int64_t>(blocks, (a.n + kTile - 1) / kTile)));
  switch ((a.k + 31) / 32) {
    case 1: hipLaunchKernelGGL(k_absent<1>, g, dim3(kBlock), 0, s, a, ix); break;
    case 2: hipLaunchKernelGGL(k_absent<2>, g, dim3(kBlock), 0, s, a, ix); break;
    case 3: hipLaunchKernelGGL(k_absent<3>, g, dim3(kBlock), 0, s, a, ix); break;
    default: hipLaunchKernelGGL(k_absent<4>, g, dim3(kBlock), 0, s, a, ix); break;
  }
}

extern "C" int kh_merge_contigs(kh_ctx* ctx, const kh_table* t, const char* seq,
                                const int64_t* offsets, int64_t n_contigs, int on_device,
                                void* hip_stream, kh_table** out) {
  if (!ctx || !t || !out) return fail(KH_EINVAL, "NULL argument");
  *out = nullptr;
  if (!t->ctx) return fail(KH_EINVAL, "the table's context was destroyed");
  if (t->ctx->device != ctx->device)
    return fail(KH_EINVAL, "the table lives on device %d, the context on %d", t->ctx->device,
                ctx->device);
  if (n_contigs < 0 || (n_contigs > 0 && (!seq || !offsets)))
    return fail(KH_EINVAL, "bad contig arrays");
  if (t->k % 2 == 0) return fail(KH_EINVAL, "k must be odd");
  HIP_TRY(hipSetDevice(ctx->device));
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  // ---- the contigs' k-mers, counted as reads of high quality everywhere
  int64_t total = 0;
  if (n_contigs > 0) {
    if (on_device) {
      KH_TRY(fetch(ctx, s, {&total, offsets + n_contigs, 8}));
    } else {
      total = offsets[n_contigs];
    }
  }
  std::vector<uint8_t> hq;
  Buf<uint8_t> dq(&ctx->pool);
  kh_reads r{};
  r.seq = seq;
  r.offsets = offsets;
  r.n_reads = n_contigs;
  r.on_device = on_device ? 1 : 0;
  if (on_device) {
    const uint64_t words = ((uint64_t)std::max<int64_t>(total, 0) + 8) / 8;
    KH_TRY(dq.alloc(8 * words));
    launch_fill_u64(reinterpret_cast<uint64_t*>(dq.p), words, 0ull, s);
    r.qual = reinterpret_cast<const char*>(dq.p);
  } else {
    hq.assign((size_t)total + 1, 0);
    r.qual = reinterpret_cast<const char*>(hq.data());
  }
  kh_params p;
  kh_default_params(&p, t->k);
  p.min_count = 1;
  p.qual_offset = 0;  // every quality byte is 0 and the cutoff 0: all bases count
  p.qual_cutoff = 0;
  p.load_factor = 0.7f;  // contig k-mers are nearly all distinct: plan for their count
  if (t->n_rows > (int64_t)0xfffffffe) return fail(KH_EINVAL, "too many rows");
  Buf<uint32_t> start(&ctx->pool);
  RowIndex ix{};
  KH_TRY(row_index_build(&ctx->pool, t->keys, t->n_rows, t->k, start, &ix, s));
  kh_table* c = nullptr;
  KH_TRY(make_table(ctx, t->k, &c));
  if (const int crc = count_absent(ctx, &r, p, t->keys, ix, s, c)) {
    kh_table_free(c);
    return crc;
  }
  kh_table* m = nullptr;
  int rc = make_table(ctx, t->k, &m);
  if (rc == KH_OK) {
    switch ((t->k + 31) / 32) {
      case 1: rc = merge_rows<1>(ctx, t, ix, start, c, s, m); break;
      case 2: rc = merge_rows<2>(ctx, t, ix, start, c, s, m); break;
      case 3: rc = merge_rows<3>(ctx, t, ix, start, c, s, m); break;
      default: rc = merge_rows<4>(ctx, t, ix, start, c, s, m); break;
    }
  }
  kh_table_free(c);
  if (rc != KH_OK) {
    kh_table_free(m);
    return rc;
  }
  *out = m;
  return KH_OK;
}
