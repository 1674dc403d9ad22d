// Applying an ordering (rcm_apply.h): the permuted matrix B = P A P^T with
// sorted rows, and y = A x as a probe of the locality an ordering buys.
//
// Permutation: new row degrees are gathered and scanned into B's row
// pointer; every row of A is read once, its columns renamed by iperm and
// ranked against each other, and written to its sorted places: a row of up
// to 16 entries by eight lanes, one of up to 64 by a wave, a longer one by a
// work-group of its own (a bitonic sort of (column, position) pairs, in LDS
// or, for very long rows, in a scratch array).
// Product: a group of eight lanes per row (rows of meshes hold 5 to 13
// entries), each lane striding the row, then a reduction across the group;
// the rest of a long row by the whole wave.

#include "rcm_apply.h"

#include <hip/hip_runtime.h>

#include "rcm_common.hpp"

namespace rcm {
namespace {

constexpr int kThreads = 256;

inline size_t align_up(size_t x) { return (x + 255) / 256 * 256; }

inline int grid_for(int64_t work, int threads, int max_blocks = 8192) {
  int64_t b = (work + threads - 1) / threads;
  if (b < 1) b = 1;
  if (b > max_blocks) b = max_blocks;
  return static_cast<int>(b);
}

// Workspace regions of rcm_permute.
struct ApplyLayout {
  size_t deg, blk, counts, begin, sort, total;
  bool begins;  // there is room for the rows' begins
};

// The workspace's size is part of the interface: room for a copy of the
// columns and values, although rows are sorted where they are read.  The
// numbers of medium and long rows and the rows' begins lie there.  A matrix of
// so few entries that the begins do not fit goes without them.
ApplyLayout apply_layout(int32_t n, int64_t nnz, bool with_values) {
  ApplyLayout L{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off += align_up(bytes);
    return at;
  };
  const size_t N = static_cast<size_t>(n), M = static_cast<size_t>(nnz);
  L.deg = take(4 * N);
  L.blk = take(4 * (N / 4096 + 2));
  const size_t copies = align_up(4 * M) + (with_values ? align_up(8 * M) : 0);
  L.counts = take(copies);  // (nothing without an entry)
  L.begin = L.counts + align_up(8);
  L.begins = align_up(8) + 4 * N <= copies;
  L.sort = take(8 * M);  // (column, position) pairs of rows too long for LDS
  L.total = off;
  return L;
}

// Row k of B starts at begin[k] in A (begin null: not kept) and has deg[k]
// entries; counts (null without any entry) starts at 0.
__global__ void k_new_degrees(int32_t n, const int32_t* __restrict__ rowptr,
                              const int32_t* __restrict__ perm, int32_t* __restrict__ deg,
                              int32_t* __restrict__ begin, int32_t* __restrict__ counts) {
  const int32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (counts != nullptr && t < 2) counts[t] = 0;
  for (int32_t k = t; k < n; k += gridDim.x * blockDim.x) {
    const int32_t v = perm[k];
    const int32_t a = rowptr[v];
    deg[k] = rowptr[v + 1] - a;
    if (begin != nullptr) begin[k] = a;
  }
}

// Where row k of B begins in A: kept, or by way of the order.
template <bool kKept>
struct Begins {
  const int32_t* kept;
  const int32_t* rowptr;
  const int32_t* perm;
  __device__ __forceinline__ int32_t operator[](int32_t k) const {
    return kKept ? kept[k] : rowptr[perm[k]];
  }
};

// Row k of B: row perm[k] of A with its columns renamed by iperm, sorted
// (equal columns in input order).  Eight lanes take a row of at most
// kShortRow entries, an entry or two a lane, and rank them against each other
// by shuffles; a longer row goes to the list of medium rows (from the front
// of `list`) or of long ones (from its end), which later kernels sort.
//
// Bound by the random row reads and the gathers of iperm, so each group has
// kUnroll rows in flight, a row is read with one request per array whatever
// its length, the sorted entries go straight out (the rows of a wave are one
// contiguous range of the output), and a die's L2 sees consecutive rows
// (xcd_tile): the columns of rows near each other are the same few thousand,
// each read by about seven rows.  The 128^3 grid with values, whole call: 663 us
// with a thread per row and no order among the dies, 270 us so (1.4 TB/s of the
// matrix's and orders' own 384 MB; banded input 582 -> 122 us); 1,000,000
// vertices of mean degree 12 in banded order, a fifth of the rows longer than
// 16: 1,590 -> 235 us.
constexpr int kShortRow = 16;
constexpr int kMediumRow = 64;
constexpr int kUnroll = 4;
constexpr int kGroup = 8;  // lanes per row, here and in the product
constexpr int kGroups = kThreads / kGroup;
constexpr int kTileRows = kGroups * kUnroll;

// Rank of the group's entry c among its eight, equal ones in lane order.
__device__ __forceinline__ int group_rank(int32_t c, int sub) {
  int r = 0;
#pragma unroll
  for (int m = 1; m < kGroup; ++m) {
    const int32_t o = __shfl_xor(c, m, kGroup);
    r += o < c || (o == c && (sub ^ m) < sub) ? 1 : 0;
  }
  return r;
}

template <bool kVals, bool kKept>
__global__ void __launch_bounds__(kThreads)
k_move_rows(int32_t n, const int32_t* __restrict__ colidx,
            const double* __restrict__ vals, Begins<kKept> begin,
            const int32_t* __restrict__ iperm, const int32_t* __restrict__ rowptr_out,
            int32_t* __restrict__ colidx_out, double* __restrict__ vals_out,
            int32_t* __restrict__ list, int32_t* __restrict__ counts) {
  const int64_t k0 = xcd_tile() * kTileRows + threadIdx.x / kGroup;
  const int sub = threadIdx.x % kGroup;
  constexpr int32_t kPast = 0x7FFFFFFF;  // past the row: above every column
  // the tile's longer rows, listed with one atomic a block (an atomic a row
  // took 700 us on a graph with 180,000 such rows)
  __shared__ int32_t found[2], base[2], rows[2][kTileRows];
  if (threadIdx.x < 2) found[threadIdx.x] = 0;
  __syncthreads();
  int32_t a[kUnroll], len[kUnroll], o[kUnroll], c[kUnroll];
  double x[kUnroll];
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const int64_t k = k0 + u * kGroups;
    const int32_t kk = k < n ? static_cast<int32_t>(k) : n - 1;
    a[u] = begin[kk];
    o[u] = rowptr_out[kk];
    len[u] = k < n ? rowptr_out[kk + 1] - o[u] : 0;
  }
  // (indices clamped into the matrix's entries, behind which the arrays may hold
  // anything, so that all loads are issued at once)
  const int32_t last = rowptr_out[n] - 1;
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const uint32_t e = min(static_cast<uint32_t>(a[u] + min(sub, max(len[u] - 1, 0))),
                           static_cast<uint32_t>(last));
    c[u] = colidx[e];
    if (kVals) x[u] = vals[e];
  }
  if (last < 0) return;
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) c[u] = iperm[c[u]];
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    if (sub >= len[u]) c[u] = kPast;
    int rank = group_rank(c[u], sub);
    if (len[u] > kShortRow) {
      if (sub == 0) {
        const int l = len[u] <= kMediumRow ? 0 : 1;
        rows[l][atomicAdd(&found[l], 1)] = static_cast<int32_t>(k0 + u * kGroups);
      }
      continue;
    }
    if (len[u] > kGroup) {
      // a second entry per lane, later in the row than every first one
      const bool has = sub + kGroup < len[u];
      int32_t d = kPast;
      double y = 0.0;
      if (has) {
        d = iperm[colidx[a[u] + kGroup + sub]];
        if (kVals) y = vals[a[u] + kGroup + sub];
      }
      int rank2 = group_rank(d, sub);
#pragma unroll
      for (int m = 0; m < kGroup; ++m) {
        rank += __shfl_xor(d, m, kGroup) < c[u] ? 1 : 0;
        rank2 += __shfl_xor(c[u], m, kGroup) <= d ? 1 : 0;
      }
      if (has) {
        colidx_out[o[u] + rank2] = d;
        if (kVals) vals_out[o[u] + rank2] = y;
      }
    }
    if (sub < len[u]) {
      colidx_out[o[u] + rank] = c[u];
      if (kVals) vals_out[o[u] + rank] = x[u];
    }
  }
  __syncthreads();
  if (threadIdx.x < 2 && found[threadIdx.x] > 0)
    base[threadIdx.x] = atomicAdd(&counts[threadIdx.x], found[threadIdx.x]);
  __syncthreads();
  for (int i = threadIdx.x; i < found[0]; i += kThreads) list[base[0] + i] = rows[0][i];
  for (int i = threadIdx.x; i < found[1]; i += kThreads) list[n - 1 - base[1] - i] = rows[1][i];
}

// The medium rows: a wave each, an entry a lane, ranked against the others
// by broadcasts.
template <bool kKept>
__global__ void __launch_bounds__(kThreads)
k_sort_medium_rows(const int32_t* __restrict__ colidx, const double* __restrict__ vals,
                   Begins<kKept> begin, const int32_t* __restrict__ iperm,
                   const int32_t* __restrict__ rowptr_out, const int32_t* __restrict__ list,
                   const int32_t* __restrict__ counts, int32_t* __restrict__ colidx_out,
                   double* __restrict__ vals_out) {
  const int32_t count = counts[0];
  const int lane = threadIdx.x & 63;
  const int32_t waves = static_cast<int32_t>(gridDim.x) * (kThreads / 64);
  for (int32_t r = static_cast<int32_t>(blockIdx.x) * (kThreads / 64) +
                   static_cast<int32_t>(threadIdx.x >> 6);
       r < count; r += waves) {
    const int32_t k = list[r];
    const int32_t a = begin[k], o = rowptr_out[k], len = rowptr_out[k + 1] - o;
    int32_t c = 0;
    double x = 0.0;
    if (lane < len) {
      c = iperm[colidx[a + lane]];
      if (vals) x = vals[a + lane];
    }
    int rank = 0;
    for (int j = 0; j < len; ++j) {
      const int32_t y = __shfl(c, j, 64);
      rank += y < c || (y == c && j < lane) ? 1 : 0;
    }
    if (lane < len) {
      colidx_out[o + rank] = c;
      if (vals) vals_out[o + rank] = x;
    }
  }
}

// The long rows: one work-group per row (a grid-stride loop over the end of
// the list).  The row's entries become (column << 32 | position) pairs,
// distinct even if a column repeats, so the sort puts equal columns in input
// order as the short rows do, and the values follow their positions.  They
// are sorted by a bitonic network whose comparators all put the smaller pair
// first (each merge starts by comparing mirrored positions), so positions
// past the row can stand for pairs above every other without being stored: a
// comparator that would reach one is a no-op.  Rows of up to kLongLds entries
// sort in LDS, longer ones in place in the scratch array, with a barrier of
// the work-group between the steps.
constexpr int kLongThreads = 256;
constexpr int kLongLds = 8192;

__device__ __forceinline__ void bitonic_pairs(unsigned long long* a, int32_t len, int32_t pow2) {
  for (int32_t k = 2; k <= pow2; k <<= 1) {
    for (int32_t j = k >> 1; j > 0; j >>= 1) {
      for (int32_t i = threadIdx.x; i < pow2; i += kLongThreads) {
        const int32_t p = j == (k >> 1) ? (i ^ (k - 1)) : (i ^ j);
        if (p > i && p < len) {
          const unsigned long long x = a[i], y = a[p];
          if (y < x) {
            a[i] = y;
            a[p] = x;
          }
        }
      }
      __syncthreads();
    }
  }
}

template <bool kKept>
__global__ void __launch_bounds__(kLongThreads)
k_sort_long_rows(int32_t n, const int32_t* __restrict__ colidx, const double* __restrict__ vals,
                 Begins<kKept> begin, const int32_t* __restrict__ iperm,
                 const int32_t* __restrict__ rowptr_out, const int32_t* __restrict__ list,
                 const int32_t* __restrict__ counts, unsigned long long* __restrict__ pairs,
                 int32_t* __restrict__ colidx_out, double* __restrict__ vals_out) {
  __shared__ unsigned long long sp[kLongLds];
  const int32_t count = counts[1];
  for (int32_t r = blockIdx.x; r < count; r += gridDim.x) {
    const int32_t k = list[n - 1 - r];
    const int32_t first = begin[k];
    const int32_t o = rowptr_out[k];
    const int32_t len = rowptr_out[k + 1] - o;
    int32_t pow2 = 1;
    while (pow2 < len) pow2 <<= 1;
    unsigned long long* a = len <= kLongLds ? sp : pairs + o;
    for (int32_t i = threadIdx.x; i < len; i += kLongThreads)
      a[i] = (static_cast<unsigned long long>(static_cast<uint32_t>(iperm[colidx[first + i]]))
              << 32) |
             static_cast<uint32_t>(i);
    __syncthreads();
    bitonic_pairs(a, len, pow2);
    for (int32_t i = threadIdx.x; i < len; i += kLongThreads) {
      const unsigned long long x = a[i];
      colidx_out[o + i] = static_cast<int32_t>(x >> 32);
      if (vals) vals_out[o + i] = vals[first + static_cast<uint32_t>(x)];
    }
    __syncthreads();
  }
}

// One batch of the product: eight entries, from `off` on, of each of a group's
// kRows rows, whose entries left are [at, end) with `at` the lane's first one.
// (Unsigned throughout: the last rows of nearly 2^31 entries reach past that.)
//
// Near rows, none of them empty and all of at most two batches: branch-free,
// so that every load is issued before the first is waited for; past its end a
// row's last entry is read again, and not added.
template <bool kVals, int kRows>
__device__ __forceinline__ void near_load(const int32_t* __restrict__ colidx,
                                          const double* __restrict__ vals, const uint32_t* at,
                                          const uint32_t* end, uint32_t off, int32_t* c,
                                          double* w) {
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    const uint32_t e = min(at[u] + off, end[u] - 1u);
    c[u] = colidx[e];
    w[u] = kVals ? vals[e] : 1.0;
  }
}
template <int kRows>
__device__ __forceinline__ void near_add(const double* __restrict__ x, const uint32_t* at,
                                         const uint32_t* end, uint32_t off, const int32_t* c,
                                         const double* w, double* s) {
  double g[kRows];
#pragma unroll
  for (int u = 0; u < kRows; ++u) g[u] = x[c[u]];
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    const double t = fma(w[u], g[u], s[u]);
    s[u] = at[u] + off < end[u] ? t : s[u];
  }
}

// Other rows: through buffers over the wave's entries and over x, where a lane
// without an entry asks for a place past the end, which makes no request and
// gives 0.  Read again and again, the last entries of the shorter rows of a
// wave cost as many requests as the entries themselves (a random geometric
// graph of 1,000,000 vertices, rows of up to 30 entries, in random order with
// values: 172 us, 146 so).
constexpr uint32_t kNowhere = 0xFFFFFFF8u;
constexpr uint32_t kFarSpan = 1u << 28;  // entries a wave's buffers cover
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, static_cast<int>(bytes),
                                           0x00020000);  // 32-bit raw data
}
__device__ __forceinline__ double load_f64(__amdgpu_buffer_rsrc_t b, uint32_t byte) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(b, byte, 0, 0));
}
template <bool kVals, int kRows>
__device__ __forceinline__ void far_load(__amdgpu_buffer_rsrc_t colidx,
                                         __amdgpu_buffer_rsrc_t vals, const uint32_t* at,
                                         const uint32_t* end, uint32_t off, int32_t* c,
                                         double* w) {
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    const uint32_t e = at[u] + off;
    const bool has = e < end[u];
    c[u] = __builtin_amdgcn_raw_buffer_load_b32(colidx, has ? 4u * e : kNowhere, 0, 0);
    w[u] = kVals ? load_f64(vals, has ? 8u * e : kNowhere) : 1.0;
  }
}
template <int kRows>
__device__ __forceinline__ void far_add(__amdgpu_buffer_rsrc_t x, const uint32_t* at,
                                        const uint32_t* end, uint32_t off, const int32_t* c,
                                        const double* w, double* s) {
  double g[kRows];
#pragma unroll
  for (int u = 0; u < kRows; ++u)
    g[u] = load_f64(x, at[u] + off < end[u] ? 8u * static_cast<uint32_t>(c[u]) : kNowhere);
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    const double t = fma(w[u], g[u], s[u]);
    s[u] = at[u] + off < end[u] ? t : s[u];
  }
}

// y = A x.  Bound by the matrix's bytes where x's gathers hit the die's L2, by
// those gathers else, so each group of eight lanes keeps kRows rows in flight:
// the bounds of all of them, then eight entries of each, then the next eight
// with the first ones' gathers of x, and so on.  A die takes consecutive rows
// (xcd_tile).  Up to kMediumRow entries the sums are those of one row at a
// time: a lane's entries in order by fma, then halves of the group.  Past
// that the batches go on while half of a wave's rows have entries left; what
// is left of a row is then added by its lanes (up to 64 entries) or by the
// whole wave.
// On the 128^3 grid in banded order with values: 76 us with one row in
// flight, 51 us with four (4.2 TB/s of 217 MB; a copy reaches 5.05).  10,000
// rows of 1,000 entries with values: 62 us as a lane group a row with one in
// flight, 202 us with four, 58 us so.
template <bool kVals, int kRows>
__global__ void __launch_bounds__(kThreads)
k_spmv(int32_t n, const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
       const double* __restrict__ vals, const double* __restrict__ x, double* __restrict__ y) {
  const int64_t r0 = xcd_tile() * (kGroups * kRows) + threadIdx.x / kGroup;
  const uint32_t lane = threadIdx.x % kGroup;
  uint32_t at[kRows], end[kRows];
  double s[kRows];
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    const int64_t r = r0 + u * kGroups;
    const int32_t rr = r < n ? static_cast<int32_t>(r) : n - 1;
    at[u] = static_cast<uint32_t>(rowptr[rr]);
    end[u] = static_cast<uint32_t>(rowptr[rr + 1]);
  }
  // entries counted from the wave's first one
  const uint32_t first = __builtin_amdgcn_readfirstlane(at[0]);
  const uint32_t span = __builtin_amdgcn_readlane(end[kRows - 1], 63) - first;
  colidx += first;
  if (kVals) vals += first;
  uint32_t longest = 0, shortest = 1;
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    longest = max(longest, end[u] - at[u]);
    shortest = min(shortest, end[u] - at[u]);
    at[u] += lane - first;
    end[u] -= first;
    s[u] = 0.0;
  }
  uint32_t off = 0;  // entries of every row that are done
  int32_t c[kRows], c2[kRows];
  double w[kRows], w2[kRows];
  if (__all(shortest > 0 && longest <= 2 * kGroup)) {
    near_load<kVals, kRows>(colidx, vals, at, end, 0, c, w);
    const bool more = __any(longest > kGroup);
    if (more) near_load<kVals, kRows>(colidx, vals, at, end, kGroup, c2, w2);
    near_add<kRows>(x, at, end, 0, c, w, s);
    if (more) near_add<kRows>(x, at, end, kGroup, c2, w2, s);
    off = 2 * kGroup;
  } else if (span < kFarSpan && n < 1 << 29) {  // (32-bit byte offsets)
    const __amdgpu_buffer_rsrc_t bc = buffer_of(colidx, 4u * span);
    const __amdgpu_buffer_rsrc_t bv = buffer_of(vals, 8u * span);
    const __amdgpu_buffer_rsrc_t bx = buffer_of(x, 8u * static_cast<uint32_t>(n));
    auto worth = [&](uint32_t o) -> bool {
      if (o < kMediumRow) return __any(o < longest);
      if (kRows == 1) return false;
      int rows = 0;
#pragma unroll
      for (int u = 0; u < kRows; ++u) rows += __popcll(__ballot(at[u] - lane + o < end[u]));
      return rows >= 32 * kRows;
    };
    far_load<kVals, kRows>(bc, bv, at, end, 0, c, w);
    while (true) {
      const bool more = worth(off + kGroup);
      if (more) far_load<kVals, kRows>(bc, bv, at, end, off + kGroup, c2, w2);
      far_add<kRows>(bx, at, end, off, c, w, s);
      off += kGroup;
      if (!more) break;
      const bool more2 = worth(off + kGroup);
      if (more2) far_load<kVals, kRows>(bc, bv, at, end, off + kGroup, c, w);
      far_add<kRows>(bx, at, end, off, c2, w2, s);
      off += kGroup;
      if (!more2) break;
    }
  }
  if (__any(off < longest)) {
    const uint32_t wave_lane = threadIdx.x & 63;
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
      const uint32_t b = at[u] - lane + off;
      const uint32_t left = b < end[u] ? end[u] - b : 0u;
      if (left <= 64)
        for (uint32_t e = b + lane; e < end[u]; e += kGroup)
          s[u] = fma(kVals ? vals[e] : 1.0, x[colidx[e]], s[u]);
      unsigned long long rows = __ballot(lane == 0 && left > 64);
      while (rows != 0) {
        const int from = __builtin_ctzll(rows);
        rows &= rows - 1;
        uint32_t e = __builtin_amdgcn_readlane(b, from) + wave_lane;
        const uint32_t to = __builtin_amdgcn_readlane(end[u], from);
        double p = 0.0, q = 0.0;
        for (; e + 64 < to; e += 128) {
          const int32_t c0 = colidx[e], c1 = colidx[e + 64];
          const double w0 = kVals ? vals[e] : 1.0, w1 = kVals ? vals[e + 64] : 1.0;
          p = fma(w0, x[c0], p);
          q = fma(w1, x[c1], q);
        }
        if (e < to) p = fma(kVals ? vals[e] : 1.0, x[colidx[e]], p);
        p += q;
#pragma unroll
        for (int m = kGroup; m < 64; m <<= 1) p += __shfl_xor(p, m, 64);
        if (wave_lane / kGroup == static_cast<uint32_t>(from) / kGroup) s[u] += p;
      }
    }
  }
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
#pragma unroll
    for (int m = kGroup / 2; m > 0; m >>= 1) s[u] += __shfl_xor(s[u], m, kGroup);
    const int64_t r = r0 + u * kGroups;
    if (lane == 0 && r < n) y[r] = s[u];
  }
}

// Rows in flight per group: as many as leave the chip full.  With values, and
// 1, 2 and 4 in flight: 200,000 rows of 1 to 30 entries in random order 16.3,
// 17.4, 18.9 us; 450,000 rows, one in twenty of 150 entries and the others of
// 6, 60.5, 49.4, 59.2; the banded 128^3 grid 54, 39, 38.
template <bool kVals, int kRows>
void launch_spmv(int32_t n, const int32_t* rowptr, const int32_t* colidx, const double* vals,
                 const double* x, double* y, hipStream_t s) {
  constexpr int kTile = kGroups * kRows;
  k_spmv<kVals, kRows><<<xcd_grid((static_cast<int64_t>(n) + kTile - 1) / kTile), kThreads, 0,
                         s>>>(n, rowptr, colidx, vals, x, y);
}
template <bool kVals>
void launch_spmv(int32_t n, const int32_t* rowptr, const int32_t* colidx, const double* vals,
                 const double* x, double* y, hipStream_t s) {
  if (n < 1 << 18)
    launch_spmv<kVals, 1>(n, rowptr, colidx, vals, x, y, s);
  else if (n < 1 << 19)
    launch_spmv<kVals, 2>(n, rowptr, colidx, vals, x, y, s);
  else
    launch_spmv<kVals, 4>(n, rowptr, colidx, vals, x, y, s);
}

// The rows' kernels of rcm_permute.
template <bool kKept>
hipError_t launch_moves(int32_t n, int64_t nnz, const int32_t* colidx, const double* vals,
                        Begins<kKept> begin, const int32_t* iperm, const int32_t* rowptr_out,
                        int32_t* colidx_out, double* vals_out, int32_t* list, int32_t* counts,
                        unsigned long long* pairs, hipStream_t s) {
  const unsigned blocks = xcd_grid((static_cast<int64_t>(n) + kTileRows - 1) / kTileRows);
  if (vals)
    k_move_rows<true, kKept><<<blocks, kThreads, 0, s>>>(
        n, colidx, vals, begin, iperm, rowptr_out, colidx_out, vals_out, list, counts);
  else
    k_move_rows<false, kKept><<<blocks, kThreads, 0, s>>>(
        n, colidx, vals, begin, iperm, rowptr_out, colidx_out, vals_out, list, counts);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // (a row needs more than kShortRow of the nnz entries to be listed)
  const int64_t most = nnz / (kShortRow + 1);
  if (most > 0) {
    k_sort_medium_rows<<<grid_for(most, kThreads / 64, 2048), kThreads, 0, s>>>(
        colidx, vals, begin, iperm, rowptr_out, list, counts, colidx_out, vals_out);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (nnz > kMediumRow)
    k_sort_long_rows<<<grid_for(nnz / (kMediumRow + 1), 1, 1024), kLongThreads, 0, s>>>(
        n, colidx, vals, begin, iperm, rowptr_out, list, counts, pairs, colidx_out, vals_out);
  return hipGetLastError();
}

}  // namespace
}  // namespace rcm

using namespace rcm;

extern "C" {

size_t rcm_permute_workspace_bytes(int32_t n, int64_t nnz, int32_t with_values) {
  if (n <= 0 || nnz < 0 || nnz >= (1ll << 31) - 1) return 0;
  return apply_layout(n, nnz, with_values != 0).total;
}

rcm_status rcm_permute(int32_t n, int64_t nnz, const int32_t* rowptr, const int32_t* colidx,
                       const double* vals, const int32_t* perm, const int32_t* iperm,
                       int32_t* rowptr_out, int32_t* colidx_out, double* vals_out,
                       void* workspace, size_t workspace_bytes, void* stream) {
  if (n < 0 || nnz < 0 || nnz >= (1ll << 31) - 1) return RCM_ERR_INVALID_ARGUMENT;
  if (n == 0) return RCM_OK;
  if (!rowptr || !perm || !iperm || !rowptr_out || (nnz > 0 && (!colidx || !colidx_out)))
    return RCM_ERR_INVALID_ARGUMENT;
  if (vals && !vals_out) return RCM_ERR_INVALID_ARGUMENT;
  const ApplyLayout L = apply_layout(n, nnz, vals != nullptr);
  if (!workspace || workspace_bytes < L.total) return RCM_ERR_WORKSPACE_TOO_SMALL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  int32_t* deg = reinterpret_cast<int32_t*>(ws + L.deg);
  int32_t* begin = L.begins ? reinterpret_cast<int32_t*>(ws + L.begin) : nullptr;
  int32_t* blk = reinterpret_cast<int32_t*>(ws + L.blk);
  unsigned long long* pairs = reinterpret_cast<unsigned long long*>(ws + L.sort);
  // the degrees are scanned before the rows move: deg then takes the lists of
  // medium and long rows
  int32_t* list = deg;
  int32_t* counts = nnz > 0 ? reinterpret_cast<int32_t*>(ws + L.counts) : nullptr;
  k_new_degrees<<<grid_for(n, kThreads), kThreads, 0, s>>>(n, rowptr, perm, deg, begin, counts);
  if (hipGetLastError() != hipSuccess) return RCM_ERR_HIP;
  if (launch_exclusive_scan(deg, rowptr_out, n, blk, rowptr_out + n, s) != hipSuccess)
    return RCM_ERR_HIP;
  if (nnz == 0) return RCM_OK;
  auto move = [&](auto begin) {
    return launch_moves(n, nnz, colidx, vals, begin, iperm, rowptr_out, colidx_out, vals_out,
                        list, counts, pairs, s);
  };
  const hipError_t e = L.begins ? move(Begins<true>{begin, rowptr, perm})
                                : move(Begins<false>{nullptr, rowptr, perm});
  return e == hipSuccess ? RCM_OK : RCM_ERR_HIP;
}

rcm_status rcm_spmv(int32_t n, const int32_t* rowptr, const int32_t* colidx, const double* vals,
                    const double* x, double* y, void* stream) {
  if (n < 0) return RCM_ERR_INVALID_ARGUMENT;
  if (n == 0) return RCM_OK;
  if (!rowptr || !x || !y) return RCM_ERR_INVALID_ARGUMENT;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (vals)
    launch_spmv<true>(n, rowptr, colidx, vals, x, y, s);
  else
    launch_spmv<false>(n, rowptr, colidx, vals, x, y, s);
  return hipGetLastError() == hipSuccess ? RCM_OK : RCM_ERR_HIP;
}

}  // extern "C"
