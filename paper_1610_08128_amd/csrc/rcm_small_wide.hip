// The one-work-group engine for a whole small graph in LDS (rcm_small.hip),
// for graphs with long rows: 16 waves work on every phase, 16 lanes on a row.
//
// The one-wave engine walks a level's rows 64 at a time, one lane a row, so
// with a dozen entries or more in a row the time of a level is that of its
// longest row, and the row checks compare a row's entries pairwise in one
// lane.  Here the lanes of a row take its entries side by side, and a level
// is a fixed chain of LDS round trips: its vertices, their row records, the
// columns, the atomics on the neighbours' claim words, the places of the
// vertices found.
//
// The vertices are renumbered by (degree, id) as they are loaded, so that the
// new number alone is SortPerm's key among siblings and the minimum of a
// level the next root: neither degrees nor pairs of words are compared in a
// pass.  A labelled level claims with atomic minima of the parents' labels
// (the (select2nd, min) product), and the lane whose atomic finds the word
// free lists the child.  Up to kRanked children are then ranked by
// (parent, number) with all of them in every wave's registers: a wave takes
// every 16th child and counts the smaller keys with ballots.  More are
// grouped by parent with LDS counters and a scan, and ranked among their
// siblings.
//
// Measured on MI355X, a random geometric graph of 3,000 vertices with rows of
// 12 entries: 1,746 us a call on one wave, 251 here (load 4, checks and sort 30,
// a search level 0.7, a labelled one 1.8, statistics 9).  A work-group of 512
// threads took 331.

#include "rcm_common.hpp"

namespace rcm {

namespace {

constexpr int kWT = 1024;
constexpr int kWWaves = kWT / 64;
constexpr uint32_t kFree = 0xFFFFFFFFu;   // claim word: unclaimed, unstamped
constexpr uint32_t kStamp = 0x80000000u;  // words from here on: not labelled
constexpr int32_t kMaxN = 8192;
constexpr int kPer = kMaxN / kWT;         // vertices per thread
// Lanes of a row in a pass: 4 lanes of 4 entries took 1.12 times as long for a
// graph of mean row 12, 8 lanes of 2 1.06 times (one wave's share of a level
// then waits for more entries in turn).
constexpr int kRowLanes = 16;
constexpr int kRanked = 256;              // children ranked in registers
// Row record: where the row begins, its length, whether it holds its diagonal.
constexpr int kBeginBits = 17;
constexpr uint32_t kBeginMask = (1u << kBeginBits) - 1u;
constexpr uint32_t kLenMask = (1u << 13) - 1u;
constexpr int kDiagBit = 31;
static_assert(kMaxN <= static_cast<int32_t>(kLenMask) + 1, "a row's length fits its field");

inline __host__ __device__ size_t al8(size_t x) { return (x + 7) & ~static_cast<size_t>(7); }

inline __host__ __device__ size_t wide_bytes(int64_t n, int64_t nnz) {
  const size_t N = static_cast<size_t>(n);
  return 2 * al8(4 * N) + al8(2 * static_cast<size_t>(nnz)) + 2 * al8(2 * N) + al8(2 * N + 16) +
         al8(4 * ((N + 31) / 32));
}

struct WLds {
  uint32_t* rec;   // row records by number
  uint32_t* clm;   // claims and stamps; final label of an ordered vertex
  uint16_t* ci;    // columns
  uint16_t* ord;   // order of the component (search queue, labels)
  uint16_t* orig;  // caller's id by number
  uint16_t* lst;   // a labelled level's children as they were found
  uint32_t* todo;  // bitmap by caller's id: not ordered yet, isolated ones aside
};

struct WShared {
  int32_t cnt[3];
  int32_t bad;
  int32_t root;
  int32_t stop;
  int32_t named;  // a vertex without neighbours of its own was ordered with a component
  int32_t run;
  int32_t wsum[kWWaves];
  int32_t wcnt[16 * kWWaves];
  int32_t red[4][kWWaves];
  unsigned long long edges;
};
constexpr size_t kWideStatic = 2048;
static_assert(sizeof(WShared) <= kWideStatic, "the static LDS outgrew its reserve");

struct WPass {
  int32_t ecc, root, count;
};

__device__ __forceinline__ uint32_t wave_min(uint32_t x) {
  x = row_min(x);
  uint32_t r = kFree;
#pragma unroll
  for (int l = 0; l < 64; l += 16) {
    const uint32_t y = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(x), l));
    r = y < r ? y : r;
  }
  return r;
}

// Degrees, repeated columns, bandwidth and profile of the input order, from
// the caller's numbering (rows in clm): 16 lanes a row.  Rows of up to 32
// entries are compared in registers, longer ones through a bitmap per wave,
// a row at a time.  Returns whether a column repeats.
__device__ __forceinline__ bool check_rows(const WLds& L, int32_t n, int32_t nnz, uint16_t* deg,
                                           int32_t* bw, int32_t* prof) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, sub = tid & 15;
  const int wave = uniform(tid >> 6);
  const int32_t words = (n + 31) / 32;
  uint32_t* bits = reinterpret_cast<uint32_t*>(L.ord) + wave * words;
  bool dup = false;
  constexpr int kAhead = 2;  // four rows each
  for (int32_t i0 = wave * 4 * kAhead; i0 < n; i0 += kWWaves * 4 * kAhead) {
    const uint32_t s = static_cast<uint32_t>(sub);
    uint32_t a[kAhead], len[kAhead], x0[kAhead], x1[kAhead];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const int32_t i = i0 + 4 * j + (lane >> 4);
      a[j] = L.clm[i < n ? i : 0];
      const uint32_t b = L.clm[i + 1 < n ? i + 1 : 0];
      len[j] = i < n ? (i + 1 < n ? b : static_cast<uint32_t>(nnz)) - a[j] : 0u;
    }
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      x0[j] = L.ci[s < len[j] ? a[j] + s : 0u];
      x1[j] = L.ci[s + 16 < len[j] ? a[j] + s + 16 : 0u];
    }
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const int32_t i = i0 + 4 * j + (lane >> 4);
      const uint32_t me = static_cast<uint32_t>(i);
      x0[j] = s < len[j] ? x0[j] : kStamp | s;
      x1[j] = s + 16 < len[j] ? x1[j] : kStamp | 16u | s;
      bool self = x0[j] == me || x1[j] == me;
      uint32_t mn = x0[j] < x1[j] ? x0[j] : x1[j];
      mn = mn < me ? mn : me;
      // ascending rows repeat nothing (the lane before; a row's 16th entry
      // comes before its 17th)
      const uint32_t b0 = dpp<0x111>(x0[j]), b1 = dpp<0x111>(x1[j]), e0 = dpp<0x121>(x0[j]);
      const bool up = sub == 0 ? e0 < x1[j] : b0 < x0[j] && b1 < x1[j];
      if (!__all(up)) {
        const uint32_t same = same_in<1>(x0[j]) | same_in<1>(x1[j]) |
                              (x0[j] == x1[j] ? 1u : 0u) | same_between<1>(x0[j], x1[j]);
        dup |= same != 0;
      }
      if (__any(len[j] > 32)) {
        for (uint32_t k = s + 32; k < len[j]; k += 16) {
          const uint32_t x = L.ci[a[j] + k];
          self |= x == me;
          mn = x < mn ? x : mn;
        }
        for (int l = 0; l < 64; l += 16) {
          const uint32_t rl =
              static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(len[j]), l));
          const uint32_t ra =
              static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(a[j]), l));
          if (rl <= 32) continue;
          for (uint32_t k = lane; k < rl; k += 64) {
            const uint32_t x = L.ci[ra + k];
            const uint32_t bit = 1u << (x & 31u);
            dup |= (atomicOr(&bits[x >> 5], bit) & bit) != 0;
          }
          __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
          for (uint32_t k = lane; k < rl; k += 64) bits[L.ci[ra + k] >> 5] = 0;
          __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        }
      }
      const unsigned long long sm = __ballot(self);
      mn = row_min(mn);
      if (i < n && sub == 0) {
        const bool diag = ((sm >> (lane & 48)) & 0xffffu) != 0;
        deg[i] = static_cast<uint16_t>(len[j] - (diag ? 1u : 0u));
        const int32_t beta = i - static_cast<int32_t>(mn);
        *bw = beta > *bw ? beta : *bw;
        *prof += beta;
      }
    }
  }
  return dup;
}

// orig[] = the ids sorted by (degree, id): stable counting passes over four
// bits of the degree each, every wave on its own stretch of the list.
__device__ __forceinline__ void sort_by_degree(const WLds& L, WShared& S, int32_t n,
                                               const uint16_t* deg, int32_t maxdeg) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const int wave = uniform(tid >> 6);
  const int32_t chunk = ((n + kWWaves - 1) / kWWaves + 63) & ~63;
  const int32_t lo = wave * chunk, hi = lo + chunk < n ? lo + chunk : n;
  int passes = 1;
  while (maxdeg >> (4 * passes) != 0) ++passes;
  for (int t = 0; t < passes; ++t) {
    uint16_t* dst = ((passes - 1 - t) & 1) == 0 ? L.orig : L.ord;
    const uint16_t* src = dst == L.orig ? L.ord : L.orig;
    if (tid < 16 * kWWaves) S.wcnt[tid] = 0;
    __syncthreads();
    int32_t id[kPer], rank[kPer];
    uint32_t digit[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int32_t i = lo + j * 64 + lane;
      id[j] = -1;
      if (i < hi) id[j] = t == 0 ? i : static_cast<int32_t>(src[i]);
      digit[j] = 0;
      if (id[j] >= 0) digit[j] = (static_cast<uint32_t>(deg[id[j]]) >> (4 * t)) & 15u;
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      rank[j] = 0;
      if (lo + j * 64 >= hi) continue;
      unsigned long long peers = __ballot(id[j] >= 0);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool bit = (digit[j] >> q & 1u) != 0;
        const unsigned long long m = __ballot(bit);
        peers &= bit ? m : ~m;
      }
      const int below = __builtin_amdgcn_mbcnt_hi(
          static_cast<uint32_t>(peers >> 32),
          __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(peers), 0));
      if (id[j] >= 0) {
        // (a wave's own counters: read, then raised by the last of its peers)
        int32_t* c = &S.wcnt[static_cast<int>(digit[j]) * kWWaves + wave];
        rank[j] = *static_cast<volatile int32_t*>(c) + below;
        if (below + 1 == __popcll(peers)) *static_cast<volatile int32_t*>(c) = rank[j] + 1;
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
    __syncthreads();
    if (wave == 0) {
      int c[4], sum = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        c[q] = S.wcnt[4 * lane + q];
        sum += c[q];
      }
      int run = wave_scan(sum) - sum;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        S.wcnt[4 * lane + q] = run;
        run += c[q];
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if (id[j] >= 0)
        dst[S.wcnt[static_cast<int>(digit[j]) * kWWaves + wave] + rank[j]] =
            static_cast<uint16_t>(id[j]);
    __syncthreads();
  }
}

// The unvisited neighbours of the level ord[fb, fe): marked (search: with the
// pass's stamp) or claimed (labelled: with the parent's label), and listed in
// out[] in any order.  Stamps descend from pass to pass, so either is an
// atomic minimum, and a vertex is new where the word was above every mark of
// this pass.  kRowLanes lanes a row, an entry each.
template <bool kLabel>
__device__ __forceinline__ void reach(const WLds& L, int32_t fb, int32_t fe, uint32_t stamp,
                                      uint16_t* out, int32_t* cnt, uint32_t* lowest, int tid) {
  const int lane = tid & 63;
  const uint32_t top = kLabel ? kStamp - 1u : stamp;
  for (int32_t i = fb + tid / kRowLanes; i < fe; i += kWT / kRowLanes) {
    const uint32_t r = L.rec[L.ord[i]];
    const uint32_t a = r & kBeginMask, len = (r >> kBeginBits) & kLenMask;
    // (the diagonal's word is the row's own vertex's, which is marked)
    for (uint32_t k = static_cast<uint32_t>(tid % kRowLanes); k < len; k += kRowLanes) {
      const uint32_t x = L.ci[a + k];
      const uint32_t old = atomicMin(&L.clm[x], kLabel ? static_cast<uint32_t>(i) : stamp);
      *lowest = old < *lowest ? old : *lowest;
      const unsigned long long m = __ballot(old > top);
      if (m == 0) continue;
      const int first = __builtin_ctzll(m);
      int base = 0;
      if (lane == first) base = lds_add(cnt, __popcll(m));
      base = __builtin_amdgcn_readlane(base, first);
      const int at = base + __builtin_amdgcn_mbcnt_hi(
                                static_cast<uint32_t>(m >> 32),
                                __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0));
      if (old > top) out[at] = static_cast<uint16_t>(x);
    }
  }
}

// The m <= kRanked children in lst, to their labels: ranked by (parent,
// number), 64 keys to a register of every wave.
__device__ __forceinline__ void place_ranked(const WLds& L, int32_t fe, int32_t m, int tid) {
  constexpr int kRegs = kRanked / 64;
  const int lane = tid & 63;
  const int wave = uniform(tid >> 6);
  if (wave >= m) return;
  uint32_t key[kRegs];
#pragma unroll
  for (int q = 0; q < kRegs; ++q) {
    key[q] = kFree;
    if (q * 64 >= m) continue;
    const int32_t i = q * 64 + lane;
    const uint32_t x = L.lst[i < m ? i : 0];
    const uint32_t p = L.clm[x];
    if (i < m) key[q] = p << 16 | x;
  }
  int rank = 0, mine = 0;
#pragma unroll
  for (int q = 0; q < kRegs; ++q) {
#pragma unroll
    for (int t = 0; t < 64 / kWWaves; ++t) {
      const int from = wave + t * kWWaves;
      if (q * 64 + from >= m) continue;
      const uint32_t k = static_cast<uint32_t>(
          __builtin_amdgcn_readlane(static_cast<int>(key[q]), from));
      int r = 0;
#pragma unroll
      for (int y = 0; y < kRegs; ++y) {
        if (y * 64 >= m) continue;
        r += __popcll(__ballot(key[y] < k));
      }
      constexpr int kEach = 64 / kWWaves;
      if (lane == q * kEach + t) {
        rank = r;
        mine = static_cast<int>(k & 0xffffu);
      }
    }
  }
  // lane q * 64 / kWWaves + t holds child q * 64 + t * kWWaves + wave
  const int q = lane / (64 / kWWaves), t = lane % (64 / kWWaves);
  if (q < kRegs && q * 64 + t * kWWaves + wave < m) L.ord[fe + rank] = static_cast<uint16_t>(mine);
}

// The m children in lst of the w parents ord[fb, fe), to their labels:
// grouped by parent, then ranked among their siblings.  The parents' counters
// are 16-bit words behind the children (m + w <= n).
__device__ __forceinline__ void place_grouped(const WLds& L, WShared& S, int32_t fb, int32_t fe,
                                              int32_t m, int tid) {
  const int lane = tid & 63;
  const int wave = uniform(tid >> 6);
  const int32_t w = fe - fb;
  uint16_t* pc = L.lst + ((m + 1) & ~1);
  uint32_t* pw = reinterpret_cast<uint32_t*>(pc);
  for (int32_t i = tid; i < (w + 1) / 2; i += kWT) pw[i] = 0;
  __syncthreads();
  int32_t x[kPer], p[kPer], arr[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int32_t i = tid + j * kWT;
    x[j] = -1;
    if (i >= m) continue;
    x[j] = L.lst[i];
    p[j] = static_cast<int32_t>(L.clm[x[j]]) - fb;
    const int sh = 16 * (p[j] & 1);
    arr[j] = static_cast<int32_t>(atomicAdd(&pw[p[j] >> 1], 1u << sh) >> sh & 0xffffu);
  }
  __syncthreads();
  // exclusive prefix over the parents, consecutive ones to a thread
  const int32_t each = (w + kWT - 1) / kWT;
  int32_t c[kPer], sum = 0;
#pragma unroll
  for (int y = 0; y < kPer; ++y) {
    c[y] = 0;
    const int32_t i = tid * each + y;
    if (y < each && i < w) c[y] = pc[i];
    sum += c[y];
  }
  const int32_t incl = wave_scan(sum);
  if (lane == 63) S.wsum[wave] = incl;
  __syncthreads();
  int32_t run = incl - sum;
  for (int y = 0; y < wave; ++y) run += S.wsum[y];
#pragma unroll
  for (int y = 0; y < kPer; ++y) {
    const int32_t i = tid * each + y;
    if (y < each && i < w) pc[i] = static_cast<uint16_t>(run);
    run += c[y];
  }
  __syncthreads();
  int32_t first[kPer], rank[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    if (x[j] < 0) continue;
    first[j] = pc[p[j]];
    L.ord[fe + first[j] + arr[j]] = static_cast<uint16_t>(x[j]);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    if (x[j] < 0) continue;
    const int32_t end = p[j] + 1 < w ? pc[p[j] + 1] : m;
    rank[j] = 0;
#pragma unroll 4
    for (int32_t i = first[j]; i < end; ++i) rank[j] += L.ord[fe + i] < x[j] ? 1 : 0;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j)
    if (x[j] >= 0) L.ord[fe + first[j] + rank[j]] = static_cast<uint16_t>(x[j]);
}

// One breadth-first pass from root over the component whose order starts at
// o: a search (visits marked with stamp, below every earlier pass's) or the
// labelled BFS, which leaves every vertex's parent's label in its claim word.
// Either takes the words above its marks as unvisited; words below kStamp (a
// search) or below o (labelled) belong to ordered components.
template <bool kLabel>
__device__ __forceinline__ WPass wide_pass(const WLds& L, WShared& S, int32_t o, int32_t root,
                                           uint32_t stamp) {
  // (opaque, so that what a pass derives from it is computed there and takes
  // no registers elsewhere)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  if (tid == 0) {
    L.ord[o] = static_cast<uint16_t>(root);
    L.clm[root] = kLabel ? static_cast<uint32_t>(o) : stamp;
    S.cnt[0] = 0;
  }
  __syncthreads();
  int32_t fb = o, fe = o + 1, ecc = 0;
  int l3 = 0;
  uint32_t lowest = kFree;
  while (true) {
    int32_t* cnt = &S.cnt[l3];
    l3 = l3 == 2 ? 0 : l3 + 1;
    if (tid == 0) S.cnt[l3] = 0;
    // (every vertex is found once per pass: the list and the queue stay
    // within n)
    uint16_t* out = kLabel ? L.lst : L.ord + fe;
    reach<kLabel>(L, fb, fe, stamp, out, cnt, &lowest, tid);
    __syncthreads();
    const int32_t m = uniform(*cnt);
    if (m == 0) break;
    if (kLabel) {
      if (m <= kRanked)
        place_ranked(L, fe, m, tid);
      else
        place_grouped(L, S, fb, fe, m, tid);
      __syncthreads();
    }
    fb = fe;
    fe += m;
    ++ecc;
  }
  if (lowest < (kLabel ? static_cast<uint32_t>(o) : kStamp)) S.bad = 1;
  uint32_t k = kFree;
  for (int32_t i = fb + lane; i < fe; i += 64) {
    const uint32_t x = L.ord[i];
    k = x < k ? x : k;
  }
  WPass r;
  r.ecc = ecc;
  r.root = static_cast<int32_t>(wave_min(k));
  r.count = fe - o;
  __syncthreads();
  return r;
}

// Over the work-group, in every thread; red is free before the call.
__device__ __forceinline__ int32_t block_max(int32_t x, int32_t* red) {
  const int32_t w = static_cast<int32_t>(~wave_min(~static_cast<uint32_t>(x)));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = w;
  __syncthreads();
  return static_cast<int32_t>(
      ~wave_min(~static_cast<uint32_t>(red[threadIdx.x % kWWaves])));
}
__device__ __forceinline__ int32_t block_sum(int32_t x, int32_t* red) {
  const int32_t incl = wave_scan(x);
  if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6] = incl;
  __syncthreads();
  int32_t r = 0;
#pragma unroll
  for (int i = 0; i < kWWaves; ++i) r += red[i];
  return uniform(r);
}

// One graph: checks, statistics, every component, reversal, result.
__global__ void __launch_bounds__(kWT) k_small_wide(SmallJob J, SmallOpts O) {
  extern __shared__ __align__(16) char smem[];
  __shared__ WShared S;
  const int tid = threadIdx.x, lane = tid & 63;
  const int32_t n = J.n;
  const int32_t nnz = J.nnz >= 0 ? J.nnz : J.rowptr[n];
  SmallResult* R = J.res;
  if (tid == 0) R->nnz = nnz;
  if (nnz < 0) {
    if (tid == 0) R->status = RCM_ERR_BAD_CSR;
    return;
  }
  if (nnz >= 1 << kBeginBits || wide_bytes(n, nnz) > static_cast<size_t>(O.lds_bytes)) {
    if (tid == 0) R->status = kSmallDeclined;
    return;
  }
  long long tk[7];
  tk[0] = wall_clock64();
  WLds L;
  {
    const size_t N = static_cast<size_t>(n);
    char* p = smem;
    L.rec = reinterpret_cast<uint32_t*>(p);
    p += al8(4 * N);
    L.clm = reinterpret_cast<uint32_t*>(p);
    p += al8(4 * N);
    L.ci = reinterpret_cast<uint16_t*>(p);
    p += al8(2 * static_cast<size_t>(nnz));
    L.ord = reinterpret_cast<uint16_t*>(p);
    p += al8(2 * N);
    L.orig = reinterpret_cast<uint16_t*>(p);
    p += al8(2 * N);
    L.lst = reinterpret_cast<uint16_t*>(p);
    p += al8(2 * N + 16);
    L.todo = reinterpret_cast<uint32_t*>(p);
  }
  // 1. rows and columns into LDS, with the structural checks
  bool bad = false;
  if (tid == 0) {
    S.bad = 0;
    S.named = 0;
    S.edges = 0;
  }
  {
    int32_t r[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int32_t i = tid + j * kWT;
      r[j] = J.rowptr[i < n ? i : n];
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int32_t i = tid + j * kWT;
      if (i >= n) {
        bad |= r[j] != nnz;
        continue;
      }
      bad |= r[j] < 0 || r[j] > nnz || (i == 0 && r[j] != 0);
      L.clm[i] = static_cast<uint32_t>(r[j] < 0 ? 0 : (r[j] > nnz ? nnz : r[j]));
    }
    // (n can be a multiple of the threads' share)
    if (tid == 0 && J.rowptr[n] != nnz) bad = true;
  }
  constexpr int kLoad = 8;
  const bool al16 = (reinterpret_cast<uintptr_t>(J.colidx) & 15) == 0;
  const int32_t quads = al16 ? nnz >> 2 : 0;  // whole 16-byte groups
  const int4* c4 = reinterpret_cast<const int4*>(J.colidx);
  for (int32_t i0 = tid; i0 < quads; i0 += kWT * kLoad) {
    int4 v[kLoad];
#pragma unroll
    for (int j = 0; j < kLoad; ++j) {
      const int32_t i = i0 + j * kWT;
      v[j] = c4[i < quads ? i : i0];
    }
#pragma unroll
    for (int j = 0; j < kLoad; ++j) {
      const int32_t i = i0 + j * kWT;
      if (i >= quads) continue;
      const uint32_t c[4] = {static_cast<uint32_t>(v[j].x), static_cast<uint32_t>(v[j].y),
                             static_cast<uint32_t>(v[j].z), static_cast<uint32_t>(v[j].w)};
#pragma unroll
      for (int h = 0; h < 4; ++h) bad |= c[h] >= static_cast<uint32_t>(n);
      *reinterpret_cast<uint2*>(L.ci + 4 * i) =
          make_uint2((c[0] & 0xffffu) | c[1] << 16, (c[2] & 0xffffu) | c[3] << 16);
    }
  }
  for (int32_t k0 = 4 * quads + tid; k0 < nnz; k0 += kWT * kLoad) {
    int32_t v[kLoad];
#pragma unroll
    for (int j = 0; j < kLoad; ++j) {
      const int32_t k = k0 + j * kWT;
      v[j] = J.colidx[k < nnz ? k : k0];
    }
#pragma unroll
    for (int j = 0; j < kLoad; ++j) {
      const int32_t k = k0 + j * kWT;
      if (k >= nnz) continue;
      bad |= v[j] < 0 || v[j] >= n;
      L.ci[k] = static_cast<uint16_t>(v[j]);
    }
  }
  // (the waves' bitmaps of the duplicate check, in ord and orig)
  const int32_t words = (n + 31) / 32;
  for (int32_t i = tid; i < kWWaves * words; i += kWT) reinterpret_cast<uint32_t*>(L.ord)[i] = 0;
  for (int32_t i = tid; i < words; i += kWT) L.todo[i] = 0;
  __syncthreads();
  // rowptr must not decrease (checked once every entry is in LDS)
  for (int32_t i = tid; i + 1 < n; i += kWT) bad |= L.clm[i + 1] < L.clm[i];
  if (__syncthreads_or(bad)) {
    if (tid == 0) R->status = RCM_ERR_BAD_CSR;
    return;
  }
  tk[1] = wall_clock64();
  // 2. row checks and input statistics, then the vertices by (degree, id)
  uint16_t* deg = reinterpret_cast<uint16_t*>(L.rec);
  // (a profile is below n^2 / 2 < 2^31)
  int32_t bw = 0, prof = 0;
  if (__syncthreads_or(check_rows(L, n, nnz, deg, &bw, &prof))) {
    if (tid == 0) R->status = RCM_ERR_BAD_CSR;
    return;
  }
  bw = block_max(bw, S.red[0]);
  prof = block_sum(prof, S.red[1]);
  int32_t maxdeg = 0, isolated = 0;
  for (int32_t i = tid; i < n; i += kWT) {
    const int32_t d = deg[i];
    maxdeg = d > maxdeg ? d : maxdeg;
    isolated += d == 0 ? 1 : 0;
    if (d > 0) atomicOr(&L.todo[i >> 5], 1u << (i & 31));
  }
  maxdeg = block_max(maxdeg, S.red[2]);
  isolated = block_sum(isolated, S.red[3]);
  sort_by_degree(L, S, n, deg, uniform(maxdeg));
  {
    // (the records take the degrees' place)
    uint32_t rec[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int32_t r = tid + j * kWT;
      if (r >= n) continue;
      const uint32_t id = L.orig[r];
      const uint32_t a = L.clm[id];
      const uint32_t b =
          static_cast<int32_t>(id) + 1 < n ? L.clm[id + 1] : static_cast<uint32_t>(nnz);
      rec[j] = a | (b - a) << kBeginBits | (b - a - deg[id]) << kDiagBit;
      L.lst[id] = static_cast<uint16_t>(r);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPer; ++j)
      if (tid + j * kWT < n) L.rec[tid + j * kWT] = rec[j];
  }
  __syncthreads();
  {
    constexpr int kPairs = 4;
    uint32_t* pairs = reinterpret_cast<uint32_t*>(L.ci);
    for (int32_t q0 = tid; q0 < nnz >> 1; q0 += kWT * kPairs) {
      uint32_t c[kPairs], lo[kPairs], hi[kPairs];
#pragma unroll
      for (int j = 0; j < kPairs; ++j) {
        const int32_t q = q0 + j * kWT;
        c[j] = pairs[q < nnz >> 1 ? q : q0];
      }
#pragma unroll
      for (int j = 0; j < kPairs; ++j) {
        lo[j] = L.lst[c[j] & 0xffffu];
        hi[j] = L.lst[c[j] >> 16];
      }
#pragma unroll
      for (int j = 0; j < kPairs; ++j)
        if (q0 + j * kWT < nnz >> 1) pairs[q0 + j * kWT] = lo[j] | hi[j] << 16;
    }
    if ((nnz & 1) != 0 && tid == 0) L.ci[nnz - 1] = L.lst[L.ci[nnz - 1]];
  }
  for (int32_t r = tid; r < n; r += kWT) L.clm[r] = kFree;
  __syncthreads();
  if (O.check_full) {
    // (r, c) present needs (c, r) present
    bool miss = false;
    for (int32_t r = tid / 16; r < n; r += kWT / 16) {
      const uint32_t rr = L.rec[r], len = (rr >> kBeginBits) & kLenMask;
      for (uint32_t k = tid % 16; k < len; k += 16) {
        const uint32_t rc = L.rec[L.ci[(rr & kBeginMask) + k]];
        const uint32_t a = rc & kBeginMask, lc = (rc >> kBeginBits) & kLenMask;
        bool found = false;
#pragma unroll 4
        for (uint32_t q = 0; q < lc; ++q) found |= L.ci[a + q] == static_cast<uint32_t>(r);
        miss |= !found;
      }
    }
    if (__syncthreads_or(miss)) {
      if (tid == 0) R->status = RCM_ERR_NOT_SYMMETRIC;
      return;
    }
  }
  tk[2] = wall_clock64();
  long long t_search = 0, t_label = 0, t_rev = 0;
  // 3. components in increasing lowest-id order
  int32_t err = 0, ncomp = 0, diameter = 0, nbfs_all = 0, nlevels = 0;
  long long edges = 0;
  uint32_t stamp = kFree;
  int32_t o = 0, w_from = 0, alone = 0;
  // abort polls: one read of the caller's flag whenever 4096 units of work
  // have passed since the last (a level walked is one unit, a component
  // begun 64), checked between passes
  uint32_t since_poll = 0;
  auto abort_poll = [&](uint32_t units) -> bool {
    if (O.abort_flag == nullptr) return false;
    since_poll += units;
    if (since_poll < 4096) return false;
    since_poll = 0;
    if (tid == 0) S.stop = abort_requested(O.abort_flag) ? 1 : 0;
    __syncthreads();
    const bool hit = S.stop != 0;
    __syncthreads();
    return hit;
  };
  while (o < n) {
    if (abort_poll(64)) {
      err = RCM_ERR_ABORTED;
      break;
    }
    // the lowest id not ordered yet, isolated ones aside (every wave finds it)
    int32_t s = n;
    while (s == n && w_from < words) {
      const uint32_t word = w_from + lane < words ? L.todo[w_from + lane] : 0u;
      const unsigned long long m = __ballot(word != 0);
      if (m == 0) {
        w_from += 64;
        continue;
      }
      const int l = __builtin_ctzll(m);
      w_from += l;
      s = 32 * w_from + __builtin_ctz(static_cast<uint32_t>(
                            __builtin_amdgcn_readlane(static_cast<int>(word), l)));
    }
    // The isolated vertices have the lowest numbers, in the order of their
    // ids: those before s are components of their own, in one go (two level
    // structures and one level each).  Where other rows name one, which only
    // an asymmetric pattern does, it can have its place already.
    int32_t next = alone;
    for (int32_t hi = isolated; next < hi;) {
      const int32_t mid = (next + hi) >> 1;
      if (uniform(L.orig[mid]) < s) next = mid + 1;
      else hi = mid;
    }
    if (next > alone) {
      int32_t run = next - alone;
      auto put = [&](int32_t x, int32_t t) {
        const int32_t id = L.orig[x];
        const int32_t at = O.reverse_mode ? n - 1 - o - t : o + t;
        J.perm[at] = id + J.id_off;
        if (J.iperm) J.iperm[id] = at + J.pos_off;
        L.clm[x] = static_cast<uint32_t>(o + t);
      };
      if (uniform(S.named) == 0) {
        for (int32_t t = tid; t < run; t += kWT) put(alone + t, t);
      } else {
        // (the first wave, the open ones packed)
        if (tid < 64) {
          int32_t t = 0;
          for (int32_t x0 = alone; x0 < next; x0 += 64) {
            const int32_t x = x0 + lane;
            const bool open = x < next && L.clm[x] >= kStamp;
            const unsigned long long m = __ballot(open);
            if (open)
              put(x, t + __builtin_amdgcn_mbcnt_hi(
                             static_cast<uint32_t>(m >> 32),
                             __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0)));
            t += __popcll(m);
          }
          if (lane == 0) S.run = t;
        }
        __syncthreads();
        run = uniform(S.run);
      }
      alone = next;
      ncomp += run;
      nbfs_all += 2 * run;
      nlevels += run;
      o += run;
      since_poll += run > 0 ? 64u * static_cast<uint32_t>(run - 1) : 0u;
      __syncthreads();
      if (o >= n) break;
    }
    if (s == n) {  // fewer vertices reached than expected: cannot happen
      err = RCM_ERR_NOT_SYMMETRIC;
      break;
    }
    int32_t size = 1, nbfs = 2, levels = 1;
    {
      const long long ts0 = wall_clock64();
      for (int32_t r = tid; r < n; r += kWT)
        if (L.orig[r] == s) S.root = r;
      __syncthreads();
      int32_t root = uniform(S.root), nlvl = -1, asym = 0;
      bool label = false, labelled = false, last = false, aborted = false;
      WPass r;
      nbfs = 1;
      // (one place calls either kind of pass)
      while (true) {
        const long long tl0 = wall_clock64();
        if (label) {
          if (labelled) {
            for (int32_t i = o + tid; i < o + size; i += kWT) L.clm[L.ord[i]] = kFree;
            __syncthreads();
          }
          r = wide_pass<true>(L, S, o, root, 0u);
          labelled = true;
          t_label += wall_clock64() - tl0;
        } else {
          r = wide_pass<false>(L, S, o, root, --stamp);
        }
        asym = uniform(S.bad);
        if (nlvl < 0) {
          size = r.count;  // (its first search)
        } else {
          asym |= r.count != size ? 1 : 0;
        }
        if (asym != 0 || last) break;
        if (r.ecc > nlvl) {
          if (abort_poll(static_cast<uint32_t>(r.ecc) + 1u)) {
            aborted = true;
            break;
          }
          nlvl = r.ecc;
          root = r.root;
          ++nbfs;
          // Algorithm 2 would return this vertex if the search does not go
          // deeper, and Algorithm 3 starts there: run the search as the
          // labelled BFS
          label = O.pp_variant == 0 && nbfs >= 3;
        } else {
          if (labelled) break;
          if (O.pp_variant == 1) root = r.root;
          label = last = true;
        }
      }
      t_search += wall_clock64() - ts0;
      if (aborted) {
        err = RCM_ERR_ABORTED;
        break;
      }
      if (asym != 0) {
        err = RCM_ERR_NOT_SYMMETRIC;
        break;
      }
      levels = r.ecc + 1;
    }
    // reversal: Cuthill-McKee label o + t goes to position anchor - t.  The
    // claim word keeps a value below o + size: the position or the label.
    const long long tr0 = wall_clock64();
    const int32_t anchor = O.reverse_mode ? n - 1 - o : o + size - 1;
    for (int32_t t = tid; t < size; t += kWT) {
      const uint32_t x = L.ord[o + t], id = L.orig[x];
      const int32_t at = anchor - t;
      J.perm[at] = static_cast<int32_t>(id) + J.id_off;
      if (J.iperm) J.iperm[id] = at + J.pos_off;
      L.clm[x] = static_cast<uint32_t>(O.reverse_mode ? o + t : at);
      if (static_cast<int32_t>(x) < isolated) S.named = 1;
      const uint32_t rx = L.rec[x];
      edges += static_cast<long long>(nbfs + 1) *
               (((rx >> kBeginBits) & kLenMask) - (rx >> kDiagBit));
      atomicAnd(&L.todo[id >> 5], ~(1u << (id & 31u)));
    }
    __syncthreads();
    t_rev += wall_clock64() - tr0;
    ncomp += 1;
    nbfs_all += nbfs;
    nlevels += levels;
    diameter = levels - 1 > diameter ? levels - 1 : diameter;
    o += size;
  }
  if (err != 0) {
    if (tid == 0) R->status = err;
    return;
  }
  // 4. bandwidth and profile of the result: eight lanes a row
  tk[3] = wall_clock64();
  int32_t bw2 = 0, prof2 = 0;
  for (int32_t v = tid / 8; v < n; v += kWT / 8) {
    const uint32_t rv = L.rec[v], a = rv & kBeginMask, len = (rv >> kBeginBits) & kLenMask;
    const int32_t k = static_cast<int32_t>(L.clm[v]);
    // (reverse_mode keeps labels, whose order is the reverse of the positions')
    int32_t lo = k, hi = k;
    for (uint32_t q = tid % 8; q < len; q += 16) {
      const int32_t k0 = static_cast<int32_t>(L.clm[L.ci[a + q]]);
      const int32_t k1 = static_cast<int32_t>(L.clm[L.ci[a + (q + 8 < len ? q + 8 : q)]]);
      lo = k0 < lo ? k0 : lo;
      lo = k1 < lo ? k1 : lo;
      hi = k0 > hi ? k0 : hi;
      hi = k1 > hi ? k1 : hi;
    }
    int32_t beta = O.reverse_mode ? hi - k : k - lo;
    int32_t y = static_cast<int32_t>(dpp<0xB1>(static_cast<uint32_t>(beta)));
    beta = y > beta ? y : beta;
    y = static_cast<int32_t>(dpp<0x4E>(static_cast<uint32_t>(beta)));
    beta = y > beta ? y : beta;
    y = static_cast<int32_t>(dpp<0x141>(static_cast<uint32_t>(beta)));
    beta = y > beta ? y : beta;
    if (tid % 8 == 0) {
      bw2 = beta > bw2 ? beta : bw2;
      prof2 += beta;
    }
  }
  __syncthreads();
  bw2 = block_max(bw2, S.red[0]);
  prof2 = block_sum(prof2, S.red[1]);
  edges = wave_sum_i64(edges);
  if (lane == 0) atomicAdd(&S.edges, static_cast<unsigned long long>(edges));
  __syncthreads();
  if (tid == 0) {
    R->bw_before = static_cast<unsigned long long>(bw);
    R->prof_before = static_cast<unsigned long long>(prof);
    R->bw_after = static_cast<unsigned long long>(bw2);
    R->prof_after = static_cast<unsigned long long>(prof2);
    R->edges = S.edges;
    R->ncomp = ncomp;
    R->diameter = diameter;
    R->nbfs = nbfs_all;
    R->nlevels = nlevels;
    // the searches' time includes a labelled pass that served as a search
    R->ticks[0] = tk[1] - tk[0];
    R->ticks[1] = tk[2] - tk[1];
    R->ticks[2] = t_search;
    R->ticks[3] = t_label;
    R->ticks[4] = t_rev;
    R->ticks[5] = wall_clock64() - tk[3];
    R->status = RCM_OK;
  }
}

}  // namespace

// n from 64 (the waves' bitmaps of the duplicate check share 4 n bytes) to
// below kMaxN (a row of every vertex still fits its length's field).
size_t small_wide_lds_bytes(int64_t n, int64_t nnz) {
  if (n < 64 || n >= kMaxN || nnz >= 1 << kBeginBits) return ~static_cast<size_t>(0);
  return wide_bytes(n, nnz) + kWideStatic;
}

hipError_t launch_small_wide(const SmallJob& job, const SmallOpts& opts, hipStream_t s) {
  if (small_wide_lds_bytes(job.n, job.nnz < 0 ? 0 : job.nnz) >
      static_cast<size_t>(opts.lds_bytes))
    return hipErrorInvalidValue;
  SmallOpts o = opts;
  o.lds_bytes = job.nnz < 0 ? opts.lds_bytes - static_cast<int32_t>(kWideStatic)
                            : static_cast<int32_t>(wide_bytes(job.n, job.nnz));
  const hipError_t e =
      hipFuncSetAttribute(reinterpret_cast<const void*>(k_small_wide),
                          hipFuncAttributeMaxDynamicSharedMemorySize, o.lds_bytes);
  if (e != hipSuccess) return e;
  k_small_wide<<<1, kWT, static_cast<size_t>(o.lds_bytes), s>>>(job, o);
  return hipGetLastError();
}

}  // namespace rcm
