// The component engine: one work-group of 1,024 threads orders one connected
// component of moderate level width, with everything a level needs beyond
// the rows themselves in LDS.  It computes what the team kernel computes
// (rcm_bfs.hip): Algorithm 2's searches, Algorithm 3's labelled BFS in
// SortPerm's (parent label, degree, id) order, and the reversal.
//
// What bounds a level is a chain of dependent memory and LDS round trips,
// whatever the level's width up to the work-group's, so the chain is kept
// short:
//  - visited marks are a bitmap of the component's graph in LDS (at most
//    kComponentRange vertices), so a found vertex costs no global atomic and
//    a pass starts with a clear of range / 32 words;
//  - the frontier stays in LDS; a component with a level wider than that
//    holds is declined and the team kernel orders it;
//  - where every row of the component has at most kEllWidth entries, the
//    frontier holds the rows themselves (EllLevels): a found vertex's row is
//    loaded from the fixed-stride copy, at an address known from its number,
//    the moment it is found, so a level makes one memory round trip.  Other
//    components (CsrLevels) make two: the frontier's columns, then the found
//    vertices' records.  Several lanes share a row, so long rows spread over
//    the work-group (one longer than kHeavyRow takes all of it);
//  - a labelled level enters its unlabelled neighbours into an LDS hash
//    table, where an atomic minimum keeps the smallest parent (the
//    (select2nd, min) product).  The children are then grouped by parent
//    with LDS counters and a scan, and ranked by (degree, id) inside their
//    group by comparing against the siblings: no row is read a second time.
//
// Measured on MI355X (whole calls, the team kernel alone against this
// engine first): a random geometric graph of 100,003 vertices in 4 patches
// (mean degree 12, levels about 250 wide) 21.3 -> 2.7 ms, a labelled level
// 44 -> 8 us and a search level 6 -> 3.5 us (the team kernel ranked each
// child against its parent's whole row); the 223 x 227 grid 4.3 -> 2.2 ms; a
// 32 x 1,000 strip 8.2 -> 3.4 ms, a search level 0.7 us and a labelled one
// 1.9; 96 graphs of 1,000 to 200,000 vertices in a batch 36 -> 10.6 ms.

#include "rcm_common.hpp"

namespace rcm {

namespace {

// 16 waves: with 8 or 4 the levels of a random geometric graph took 1.4 and
// 2.2 times as long, a 32-wide strip's the same.
constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int32_t kHeavyRow = 512;  // longer rows take the whole work-group
constexpr int kHeavyCap = 32;
constexpr int kScanAll = 512;       // parents a single wave scans
constexpr int32_t kNone = -1;
constexpr uint32_t kSelf = 0x80000000u;  // the row holds its diagonal entry
// A bit of a level's count, raised (by or, as many lanes can find one) when a
// vertex of it has a row too long for the copy.  The count below it never
// reaches it: a vertex is counted once per pass.  (A word of its own, read
// with the count, made a level of the 223 x 227 grid 2 % slower.)
constexpr int32_t kLongRow = 1 << 24;
static_assert(kLongRow > kComponentRange && kLongRow > kLongRange, "above every count");

// The next level's table of a labelled level: vertex and smallest parent's
// index in the level, at most half full (see reach_label), the slot of each
// child found, and the children counted per parent.
template <int kCap, int kBits>
struct Table {
  static constexpr int kHash = 1 << kBits;
  static constexpr int kHashBits = kBits;
  static_assert(kHash >= 2 * kCap, "at most half full");
  int32_t hk[kHash];
  uint32_t hv[kHash];
  uint16_t slot[kCap];
  int32_t pcnt[kCap];
};

// A frontier record: vertex, row begin, row length with kSelf on top.
struct Rec {
  int32_t v;
  int32_t begin;
  uint32_t len;
};
struct CsrLds {
  static constexpr int kCap = kComponentCap;
  Table<kCap, 12> t;
  Rec fr[2][kCap];
};
// The frontier as rows: the row's entries, then the vertex itself.
struct EllLds {
  static constexpr int kCap = kComponentEllCap;
  Table<kCap, 11> t;
  int32_t v[2][kCap];
  int4 row[2][kCap][2];
};

struct Lds {
  uint32_t bits[kComponentRange / 32];
  union {
    CsrLds csr;
    EllLds ell;
  };
  int32_t wtot[kWaves];
  int2 cnt[3];                // level mod 3: size of the level being found (and kLongRow),
                              // long rows of its parents (CsrLevels)
  int32_t heavy[kHeavyCap];
  unsigned long long key;
  long long red[16];
  int32_t task;
  int32_t stop;
};
static_assert(sizeof(Lds) <= 160 * 1024, "one work-group's LDS");

// What the work-group knows about the component it orders.
struct Ctx {
  int32_t base;    // first vertex of its graph
  int32_t range;   // vertices of its graph
  int32_t size;    // vertices of the component (-1: not known yet)
  int32_t anchor;  // position of Cuthill-McKee label 0
  int32_t width;   // widest level taken on
  int32_t level;   // of the frontier
  int tid;         // this thread's number
  uint32_t polls;
  int32_t state;
  bool grows;      // declined for its growth
};
// a pass over a component: a level structure of the search, the first one of
// a component of unknown size, the labelled BFS
enum { kSearch = 0, kProbe, kLabelled };
// why an ordering stopped: the levels are too wide, a row is too long for the
// copy, the pattern is not symmetric, the caller wants it stopped
enum { kRun = 0, kDecline, kLong, kAsym, kAbort };

// A probed vertex's distance as the renumbering reads it: under the tag of
// component 0's first pass (BfsParams::dkey).
__device__ __forceinline__ unsigned long long distance_word(int32_t d) {
  return (static_cast<unsigned long long>(kProbeTag) << 32) |
         (0xFFFFFFFFu - static_cast<uint32_t>(d));
}

struct Pass {
  int32_t ecc;
  uint64_t key;     // minimum (degree, id) of the last level
  int32_t count;    // vertices reached
  long long m;      // their degrees (labelled passes)
};

__device__ __forceinline__ void flag_error(GlobalCtl* g, int32_t code) {
  int32_t expected = 0;
  __hip_atomic_compare_exchange_strong(&g->error, &expected, code, __ATOMIC_RELAXED,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Every 64th level: the caller's abort flag and the launch's error word.
// All threads call it at the same level; true when the work-group must stop.
__device__ __forceinline__ bool poll_abort(const ComponentParams& P, Lds& S, Ctx& c) {
  if (P.abort_flag == nullptr || (++c.polls & 63u) != 0) return false;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t stop = ld_relaxed(&P.gctl->error) != 0 ? 1 : 0;
    if (!stop && abort_requested(P.abort_flag)) {
      flag_error(P.gctl, RCM_ERR_ABORTED);
      stop = 1;
    }
    S.stop = stop;
  }
  __syncthreads();
  return uniform(S.stop) != 0;
}

__device__ __forceinline__ uint32_t bit_of(uint32_t x) { return 1u << (x & 31u); }

// Which of the wave's active lanes' kN entries are new in a search: their
// bits are set here, and *base is the first of the places reserved for them
// in the next level (one atomic for the wave); at[j] is entry j's.
template <int kN>
__device__ __forceinline__ void reserve(int32_t* cnt, const bool* fresh, int32_t* at) {
  int32_t total = 0;
#pragma unroll
  for (int j = 0; j < kN; ++j) {
    const unsigned long long m = __ballot(fresh[j]);
    at[j] = total + static_cast<int32_t>(__builtin_amdgcn_mbcnt_hi(
                        static_cast<uint32_t>(m >> 32),
                        __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0)));
    total += __popcll(m);
  }
  int32_t base = 0;
  if (total != 0) {
    const unsigned long long act = __ballot(true);
    if ((threadIdx.x & 63) == static_cast<unsigned>(__ffsll(static_cast<long long>(act)) - 1))
      base = lds_add(cnt, total);
    base = __builtin_amdgcn_readfirstlane(base);
  }
#pragma unroll
  for (int j = 0; j < kN; ++j) at[j] += base;
}

// Past kCap records a labelled level is given up: nothing more is entered, and
// the count says so however many calls meet it (added to by each of them, it
// took the value of another answer, and could wrap).  Returns whether this
// level is.
template <int kCap>
__device__ __forceinline__ bool given_up(int32_t* cnt) {
  const bool wide = *static_cast<volatile int32_t*>(cnt) >= kCap;
  if (wide) atomicMax(cnt, kCap + 1);
  return wide;
}

// Search: marks the open entries' bits; fresh[j] = this lane marked it.
template <int kN>
__device__ __forceinline__ void mark(Lds& S, const uint32_t* x, const bool* open, bool* fresh) {
  uint32_t old[kN];
#pragma unroll
  for (int j = 0; j < kN; ++j) {
    old[j] = 0xFFFFFFFFu;
    if (open[j]) old[j] = atomicOr(&S.bits[x[j] >> 5], bit_of(x[j]));
  }
#pragma unroll
  for (int j = 0; j < kN; ++j) fresh[j] = (old[j] & bit_of(x[j])) == 0;
}

// The table slot of v after its first place h held another vertex, entered
// if it was not there (*fresh); -1 when the table is full.
template <class T>
__device__ __forceinline__ int table_probe(T& t, int32_t v, uint32_t h, bool* fresh) {
  for (int i = 1; i < T::kHash; ++i) {
    h = (h + 1) & (T::kHash - 1);
    int32_t k = t.hk[h];
    if (k == kNone) {
      k = atomicCAS(&t.hk[h], kNone, v);
      if (k == kNone) {
        *fresh = true;
        return static_cast<int>(h);
      }
    }
    if (k == v) return static_cast<int>(h);
  }
  return -1;
}

// Labelled level: enters the open entries w into the table with their
// smallest parent, each step for all kN entries before the next one waits
// for it; fresh[j] = this lane entered w[j], at slot[j].
template <int kN, class T>
__device__ __forceinline__ void enter(T& t, const int32_t* w, const bool* open, int32_t parent,
                                      bool* fresh, int* slot) {
  int32_t k[kN];
#pragma unroll
  for (int j = 0; j < kN; ++j) {
    slot[j] = static_cast<int>((static_cast<uint32_t>(w[j]) * 2654435761u) >> (32 - T::kHashBits));
    fresh[j] = false;
    k[j] = w[j];
    if (open[j]) k[j] = t.hk[slot[j]];
  }
#pragma unroll
  for (int j = 0; j < kN; ++j)
    if (open[j] && k[j] == kNone) {
      k[j] = atomicCAS(&t.hk[slot[j]], kNone, w[j]);
      if (k[j] == kNone) {
        fresh[j] = true;
        k[j] = w[j];
      }
    }
#pragma unroll
  for (int j = 0; j < kN; ++j)
    if (k[j] != w[j]) slot[j] = table_probe(t, w[j], static_cast<uint32_t>(slot[j]), &fresh[j]);
#pragma unroll
  for (int j = 0; j < kN; ++j)
    if (open[j] && slot[j] >= 0) atomicMin(&t.hv[slot[j]], static_cast<uint32_t>(parent));
}

// Place of a key among the siblings keys[first, end): SortPerm's order inside
// the group.
__device__ __forceinline__ int32_t place(const unsigned long long* keys, int32_t first,
                                         int32_t end, uint64_t key) {
  int32_t to = first;
  for (int32_t x = first; x < end; x += 4) {
    uint64_t k4[4];
#pragma unroll
    for (int y = 0; y < 4; ++y) k4[y] = keys[x + y < end ? x + y : x];
#pragma unroll
    for (int y = 0; y < 4; ++y) to += x + y < end && k4[y] < key ? 1 : 0;
  }
  return to;
}

// ---------------------------------------------------------------------------
// Levels of any rows: records in LDS, columns and records from memory.
// ---------------------------------------------------------------------------
struct CsrLevels {
  using L = CsrLds;
  static constexpr int kCap = L::kCap;
  static constexpr bool kDirect = false;
  static constexpr int kRows = 0;
  __device__ static int32_t label_level(const ComponentParams&, Lds&, const Ctx&, int, int32_t,
                                        int32_t, int2*, long long*) {
    return 0;
  }
  struct Kept {
    Rec r;
  };
  __device__ static L& lds(Lds& S) { return S.csr; }
  __device__ static uint32_t row_len(const Rec& r) { return r.len & ~kSelf; }
  __device__ static Rec make(int32_t v, int4 inf) {
    const uint32_t len = static_cast<uint32_t>(inf.y - inf.x);
    return Rec{v, inf.x, len | (static_cast<int32_t>(len) != inf.z ? kSelf : 0u)};
  }
  __device__ static uint64_t key(const Rec& r) {
    return pack_key(static_cast<int32_t>(row_len(r) - (r.len >> 31)), r.v);
  }
  __device__ static void root(const ComponentParams& P, Lds& S, int32_t v) {
    S.csr.fr[0][0] = make(v, P.vinfo[v]);
  }
  __device__ static uint64_t level_key(Lds& S, int b, int32_t i) { return key(S.csr.fr[b][i]); }
  __device__ static Kept keep(Lds& S, int b, int32_t i) { return Kept{S.csr.fr[b][i]}; }
  __device__ static int32_t vertex(const Kept& k) { return k.r.v; }
  __device__ static uint64_t key(const Kept& k) { return key(k.r); }
  __device__ static void put(Lds& S, int b, int32_t i, const Kept& k) { S.csr.fr[b][i] = k.r; }
  // the old frontier's place, once its rows have been expanded
  __device__ static void* spare(Lds& S, int b) { return S.csr.fr[b]; }
  static constexpr size_t kSpare = sizeof(Rec) * kCap;

  template <int kMode, int kN>
  __device__ static __forceinline__ void reach(const ComponentParams& P, Lds& S, const Ctx& c,
                                               Rec* next, int32_t* cnt, const int32_t* w,
                                               int32_t parent) {
    constexpr bool kLabel = kMode == kLabelled;
    bool open[kN], fresh[kN];
    uint32_t x[kN];
#pragma unroll
    for (int j = 0; j < kN; ++j) {
      x[j] = static_cast<uint32_t>(w[j] - c.base);
      open[j] = false;
      if (w[j] >= 0) open[j] = (S.bits[x[j] >> 5] & bit_of(x[j])) == 0;
    }
    int slot[kN];
    if (kLabel) {
      const bool wide = given_up<kCap>(cnt);
#pragma unroll
      for (int j = 0; j < kN; ++j) open[j] = open[j] && !wide;
      enter<kN>(S.csr.t, w, open, parent, fresh, slot);
    } else {
      mark<kN>(S, x, open, fresh);
    }
    // the found vertices' records, on their way while their places are
    // reserved (branch-free, so that none waits for another: an entry that
    // is not new loads the first vertex's, unused)
    int4 inf[kN];
#pragma unroll
    for (int j = 0; j < kN; ++j) inf[j] = P.vinfo[fresh[j] ? w[j] : c.base];
    // (stored behind the loads, which would otherwise wait for it)
    if (kMode == kProbe && P.dkey) {
#pragma unroll
      for (int j = 0; j < kN; ++j)
        if (fresh[j]) P.dkey[w[j]] = distance_word(c.level + 1);
    }
    int32_t at[kN];
    reserve<kN>(cnt, fresh, at);
#pragma unroll
    for (int j = 0; j < kN; ++j) fresh[j] = fresh[j] && at[j] < kCap;
#pragma unroll
    for (int j = 0; j < kN; ++j)
      if (kLabel && fresh[j]) S.csr.t.slot[at[j]] = static_cast<uint16_t>(slot[j]);
#pragma unroll
    for (int j = 0; j < kN; ++j)
      if (fresh[j]) next[at[j]] = make(w[j], inf[j]);
  }

  template <int kMode, int kLanes, int kEntries>
  __device__ static __forceinline__ void rows(const ComponentParams& P, Lds& S, const Ctx& c,
                                              const Rec* cur, int32_t len, Rec* next,
                                              int2* cnt) {
    const int sub = c.tid % kLanes;
    for (int32_t i = c.tid / kLanes; i < len; i += kThreads / kLanes) {
      const Rec a = cur[i];
      int32_t la = static_cast<int32_t>(row_len(a));
      if (la > kHeavyRow) {
        int h = 0;
        if (sub == 0) h = atomicAdd(&cnt->y, 1);
        h = __shfl(h, 0, kLanes);
        // (past the list the lanes read the row, unless the level is known
        // to be too wide: the declined probe of a random graph of 4,000
        // vertices with rows of 1,570 takes 0.13 ms, 1.06 with all rows read)
        if (h < kHeavyCap) {
          if (sub == 0) S.heavy[h] = i;
          la = 0;
        } else if (*static_cast<volatile int32_t*>(&cnt->x) > c.width) {
          la = 0;
        }
      }
      for (int32_t k = sub; k < la; k += kLanes * kEntries) {
        int32_t w[kEntries];
#pragma unroll
        for (int j = 0; j < kEntries; ++j)
          w[j] = P.colidx[a.begin + (k + j * kLanes < la ? k + j * kLanes : k)];
#pragma unroll
        for (int j = 1; j < kEntries; ++j)
          if (k + j * kLanes >= la) w[j] = kNone;
        reach<kMode, kEntries>(P, S, c, next, &cnt->x, w, i);
      }
    }
  }

  // The rows of the `len` records of buffer b: eight lanes a row with two
  // entries each in flight (four lanes where rows hold at most 8 entries on
  // average, so that half the waves do it); long rows by the whole
  // work-group afterwards.  Ends with a barrier.
  template <int kMode>
  __device__ static __forceinline__ int32_t expand(const ComponentParams& P, Lds& S, const Ctx& c,
                                                   int b, int32_t len, int2* cnt) {
    const Rec* cur = S.csr.fr[b];
    Rec* next = S.csr.fr[b ^ 1];
    if (P.short_rows)
      rows<kMode, 4, 2>(P, S, c, cur, len, next, cnt);
    else
      rows<kMode, 8, 2>(P, S, c, cur, len, next, cnt);
    __syncthreads();
    const int2 n = make_int2(uniform(cnt->x), uniform(cnt->y));
    if (n.y == 0 || n.x > c.width) return n.x;
    const int32_t nh = n.y < kHeavyCap ? n.y : kHeavyCap;
    for (int32_t h = 0; h < nh; ++h) {
      const int32_t i = S.heavy[h];
      const Rec a = cur[i];
      const int32_t la = static_cast<int32_t>(row_len(a));
      for (int32_t k = c.tid; k < la; k += kThreads) {
        const int32_t w[1] = {P.colidx[a.begin + k]};
        reach<kMode, 1>(P, S, c, next, &cnt->x, w, i);
      }
    }
    __syncthreads();
    return cnt->x;
  }
};

// ---------------------------------------------------------------------------
// Levels of rows of at most kEllWidth entries: the rows themselves in LDS.
// ---------------------------------------------------------------------------
struct EllLevels {
  using L = EllLds;
  static constexpr int kCap = L::kCap;
  static constexpr bool kDirect = true;
  struct Kept {
    int32_t v;
    int4 a, b;
  };
  __device__ static L& lds(Lds& S) { return S.ell; }
  // off-diagonal entries: the places that do not hold the vertex itself
  __device__ static int32_t degree(int32_t v, int4 a, int4 b) {
    return (a.x != v) + (a.y != v) + (a.z != v) + (a.w != v) + (b.x != v) + (b.y != v) +
           (b.z != v) + (b.w != v);
  }
  __device__ static void root(const ComponentParams& P, Lds& S, int32_t v) {
    const int4 a = P.ell[2 * static_cast<size_t>(v)];
    S.ell.v[0][0] = v;
    S.ell.row[0][0][0] = a;
    S.ell.row[0][0][1] = P.ell[2 * static_cast<size_t>(v) + 1];
    if (a.x < 0) S.cnt[0].x = kLongRow;
  }
  __device__ static Kept keep(Lds& S, int b, int32_t i) {
    return Kept{S.ell.v[b][i], S.ell.row[b][i][0], S.ell.row[b][i][1]};
  }
  __device__ static int32_t vertex(const Kept& k) { return k.v; }
  __device__ static uint64_t key(const Kept& k) { return pack_key(degree(k.v, k.a, k.b), k.v); }
  __device__ static uint64_t level_key(Lds& S, int b, int32_t i) { return key(keep(S, b, i)); }
  __device__ static void put(Lds& S, int b, int32_t i, const Kept& k) {
    S.ell.v[b][i] = k.v;
    S.ell.row[b][i][0] = k.a;
    S.ell.row[b][i][1] = k.b;
  }
  __device__ static void* spare(Lds& S, int b) { return S.ell.row[b]; }
  static constexpr size_t kSpare = 2 * sizeof(int4) * kCap;

  // Up to kRows rows take eight lanes each, an entry a lane (the shortest
  // chain); more take four lanes with two entries each (half the waves).
  static constexpr int kRows = kThreads / kEllWidth;

  // This lane's kN entries of row i: which of them are not the vertex
  // itself (its diagonal and the padding).
  template <int kN>
  __device__ static __forceinline__ void entries(Lds& S, const Ctx& c, int b, int32_t i, int sub,
                                                 int32_t* w, uint32_t* x, bool* open) {
    const int32_t v = S.ell.v[b][i];
    const int32_t* row = reinterpret_cast<const int32_t*>(S.ell.row[b][i]) + kN * sub;
#pragma unroll
    for (int j = 0; j < kN; ++j) w[j] = row[j];
#pragma unroll
    for (int j = 0; j < kN; ++j) {
      x[j] = static_cast<uint32_t>(w[j] - c.base);
      open[j] = w[j] != v;
    }
  }
  // The rows of the found vertices.  Branch-free, so that no load waits for
  // another: an entry that is not new loads the first vertex's row, one line
  // for the wave, unused.  (Plain ints, which stay in registers.)
  template <int kN>
  __device__ static __forceinline__ void load_rows(const ComponentParams& P, const Ctx& c,
                                                   const int32_t* w, const bool* fresh,
                                                   int32_t (*r)[kEllWidth]) {
#pragma unroll
    for (int j = 0; j < kN; ++j) {
      const int4* row = P.ell + 2 * static_cast<size_t>(fresh[j] ? w[j] : c.base);
      const int4 lo = row[0], hi = row[1];
      r[j][0] = lo.x; r[j][1] = lo.y; r[j][2] = lo.z; r[j][3] = lo.w;
      r[j][4] = hi.x; r[j][5] = hi.y; r[j][6] = hi.z; r[j][7] = hi.w;
    }
  }
  __device__ static __forceinline__ void store(Lds& S, int b, int32_t at, int32_t v,
                                               const int32_t* r) {
    S.ell.v[b][at] = v;
    S.ell.row[b][at][0] = make_int4(r[0], r[1], r[2], r[3]);
    S.ell.row[b][at][1] = make_int4(r[4], r[5], r[6], r[7]);
  }

  template <int kMode, int kN>
  __device__ static __forceinline__ void expand_row(const ComponentParams& P, Lds& S,
                                                    const Ctx& c, int b, int32_t i, int sub,
                                                    int2* cnt) {
    constexpr bool kLabel = kMode == kLabelled;
    int32_t w[kN], r[kN][kEllWidth], at[kN];
    uint32_t x[kN];
    bool open[kN], fresh[kN];
    int slot[kN];
    entries<kN>(S, c, b, i, sub, w, x, open);
    if (kLabel) {
      const bool wide = given_up<kCap>(&cnt->x);
      uint32_t word[kN];
#pragma unroll
      for (int j = 0; j < kN; ++j) word[j] = S.bits[x[j] >> 5];
#pragma unroll
      for (int j = 0; j < kN; ++j) open[j] = !wide && (word[j] & bit_of(x[j])) == 0;
      enter<kN>(S.ell.t, w, open, i, fresh, slot);
    } else {
      mark<kN>(S, x, open, fresh);
    }
    // the rows are on their way while their places are reserved
    load_rows<kN>(P, c, w, fresh, r);
    // (stored behind the loads, which would otherwise wait for it)
    if (kMode == kProbe && P.dkey) {
#pragma unroll
      for (int j = 0; j < kN; ++j)
        if (fresh[j]) P.dkey[w[j]] = distance_word(c.level + 1);
    }
    reserve<kN>(&cnt->x, fresh, at);
#pragma unroll
    for (int j = 0; j < kN; ++j) {
      if (!fresh[j] || at[j] >= kCap) continue;
      if (kLabel) S.ell.t.slot[at[j]] = static_cast<uint16_t>(slot[j]);
      store(S, b ^ 1, at[j], w[j], r[j]);
      if (r[j][0] < 0) atomicOr(&cnt->x, kLongRow);
    }
  }

  // Ends with a barrier.
  template <int kMode>
  __device__ static __forceinline__ int32_t expand(const ComponentParams& P, Lds& S, const Ctx& c,
                                                   int b, int32_t len, int2* cnt) {
    if (len <= kRows) {
      const int32_t i = c.tid / kEllWidth;
      if (i < len) expand_row<kMode, 1>(P, S, c, b, i, c.tid % kEllWidth, cnt);
    } else {
      constexpr int kLanes = kEllWidth / 2;
      for (int32_t i = c.tid / kLanes; i < len; i += kThreads / kLanes)
        expand_row<kMode, 2>(P, S, c, b, i, c.tid % kLanes, cnt);
    }
    __syncthreads();
    return cnt->x;
  }

  // A labelled level of at most kRows parents: a lane keeps the child it
  // enters, row and all, in registers until its place is known, so nothing
  // is reserved, stored or read back in between.  Returns
  // the children found (their labels written, the level in buffer b ^ 1), or
  // having placed none, a number too large for c.width or c.size or kLongRow.
  __device__ static __forceinline__ int32_t label_level(const ComponentParams& P, Lds& S,
                                                        const Ctx& c, int b, int32_t len,
                                                        int32_t total, int2* cnt, long long* m) {
    constexpr int kN = 1;
    const int tid = c.tid, lane = tid & 63, sub = tid % kEllWidth;
    const int32_t i = tid / kEllWidth;
    auto& t = S.ell.t;
    int32_t w[kN], r[kN][kEllWidth], par[kN], arr[kN];
    uint32_t x[kN];
    bool open[kN], fresh[kN];
    int slot[kN];
#pragma unroll
    for (int j = 0; j < kN; ++j) fresh[j] = false;
    if (tid < len) t.pcnt[tid] = 0;
    if (i < len) {
      entries<kN>(S, c, b, i, sub, w, x, open);
      uint32_t word[kN];
#pragma unroll
      for (int j = 0; j < kN; ++j) word[j] = S.bits[x[j] >> 5];
#pragma unroll
      for (int j = 0; j < kN; ++j) open[j] = (word[j] & bit_of(x[j])) == 0;
      // (kRows rows of kEllWidth entries cannot fill the table)
      enter<kN>(t, w, open, i, fresh, slot);
      load_rows<kN>(P, c, w, fresh, r);
#pragma unroll
      for (int j = 0; j < kN; ++j)
        if (fresh[j] && r[j][0] < 0) cnt->x = kLongRow;  // (counts nothing)
    }
    __syncthreads();
    if (uniform(cnt->x) != 0) return kLongRow;
#pragma unroll
    for (int j = 0; j < kN; ++j)
      if (fresh[j]) {
        par[j] = static_cast<int32_t>(t.hv[slot[j]]);
        arr[j] = atomicAdd(&t.pcnt[par[j]], 1);
        t.hk[slot[j]] = kNone;
        t.hv[slot[j]] = kUnclaimed;
        atomicOr(&S.bits[x[j] >> 5], bit_of(x[j]));
      }
    __syncthreads();
    // every wave scans the counts by itself, two parents a lane at most
    constexpr int kEach = kRows / 64;
    unsigned long long* keys = static_cast<unsigned long long*>(spare(S, b));
    int32_t* pre = reinterpret_cast<int32_t*>(keys + kCap);
    const int each = (len + 63) >> 6;
    const int32_t p0 = lane * each;
    int32_t n[kEach], sum = 0;
#pragma unroll
    for (int y = 0; y < kEach; ++y) {
      n[y] = 0;
      if (y < each && p0 + y < len) n[y] = t.pcnt[p0 + y];
      sum += n[y];
    }
    const int32_t incl = wave_scan(sum);
    const int32_t found = __builtin_amdgcn_readlane(incl, 63);
    if (found == 0 || found > c.width || total + found > c.size) return found;
    int32_t run = incl - sum;
    const bool busy = __ballot(fresh[0]) != 0;
    if (busy) {
#pragma unroll
      for (int y = 0; y < kEach; ++y) {
        if (y < each && p0 + y < len) pre[p0 + y] = run;
        run += n[y];
      }
      if (lane == 63) pre[len] = found;
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
    int32_t first[kN], end[kN];
    uint64_t key[kN];
#pragma unroll
    for (int j = 0; j < kN; ++j)
      if (fresh[j]) {
        first[j] = pre[par[j]];
        end[j] = pre[par[j] + 1];
        key[j] = pack_key(degree(w[j], make_int4(r[j][0], r[j][1], r[j][2], r[j][3]),
                                 make_int4(r[j][4], r[j][5], r[j][6], r[j][7])), w[j]);
        keys[first[j] + arr[j]] = key[j];
      }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kN; ++j)
      if (fresh[j]) {
        const int32_t to = place(keys, first[j], end[j], key[j]);
        store(S, b ^ 1, to, w[j], r[j]);
        const int32_t pos = c.anchor - total - to;
        P.perm[pos] = w[j];
        P.iperm[w[j]] = pos;
        *m += static_cast<long long>(key[j] >> 32);
      }
    __syncthreads();
    return found;
  }
};

// One breadth-first pass from root.  A search only measures: eccentricity,
// the last level's minimum (degree, id), the vertices reached.  A labelled
// pass also writes perm and iperm: label t at position anchor - t.
template <class V, int kMode>
__device__ __forceinline__ Pass component_pass(const ComponentParams& P, Lds& S, Ctx& c,
                                               int32_t root) {
  constexpr bool kLabel = kMode == kLabelled;
  constexpr int kCap = V::kCap;
  constexpr int kPer = kCap / kThreads;      // children per thread after a level
  constexpr int kWavePar = kCap / kWaves;    // parents of one wave's share of a long scan
  static_assert(kCap % kThreads == 0 && kWavePar % 64 == 0, "even shares");
  static_assert(V::kSpare >= (sizeof(uint64_t) + sizeof(int32_t)) * kCap,
                "keys and prefix fit the old frontier");
  // Opaque to the compiler, so that what a pass derives from it is computed
  // there: hoisted to the start of the kernel, the lane constants of all the
  // passes together spilled to scratch, whose loads wait for the stores of
  // labels before them.
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  c.tid = tid;
  auto& L = V::lds(S);
  for (int32_t i = tid; i < (c.range + 31) / 32; i += kThreads) S.bits[i] = 0;
  if (kLabel)
    for (int i = tid; i < decltype(L.t)::kHash; i += kThreads) {
      L.t.hk[i] = kNone;
      L.t.hv[i] = kUnclaimed;
    }
  if (tid < 3) S.cnt[tid] = make_int2(0, 0);
  __syncthreads();
  long long m = 0;
  if (tid == 0) {
    V::root(P, S, root);
    S.bits[(root - c.base) >> 5] = bit_of(static_cast<uint32_t>(root - c.base));
    if (kMode == kProbe && P.dkey) P.dkey[root] = distance_word(0);
    if (kLabel) {
      P.perm[c.anchor] = root;
      P.iperm[root] = c.anchor;
      m = static_cast<long long>(V::level_key(S, 0, 0) >> 32);
    }
  }
  __syncthreads();
  int32_t len = 1, total = 1, level = 0, near = 0;
  int l3 = 0;
  if (uniform(S.cnt[0].x) != 0) c.state = kLong;  // the root's own row
  while (c.state == kRun) {
    const int b = level & 1;
    if (kMode == kProbe) c.level = level;
    int2* cnt = &S.cnt[l3];
    l3 = l3 == 2 ? 0 : l3 + 1;
    if (tid == 0) S.cnt[l3] = make_int2(0, 0);
    const bool direct = kLabel && V::kDirect && len <= V::kRows;
    int32_t found;
    if (direct) {
      found = V::label_level(P, S, c, b, len, total, cnt, &m);
    } else {
      if (kLabel)
        for (int32_t i = tid; i < len; i += kThreads) L.t.pcnt[i] = 0;
      found = V::template expand<kMode>(P, S, c, b, len, cnt);
    }
    found = uniform(found);
    if (found == 0) break;
    if (found > c.width) {
      c.state = V::kDirect && found >= kLongRow ? kLong : kDecline;
      break;
    }
    if (kMode == kProbe && P.growth > 0) {
      // a component of unknown size whose levels grow like a volume's
      // (distance 8 against distance 4) will be too wide further out
      if (level == 3) near = found;
      if (level == 7 && found * 10 >= near * P.growth) {
        c.state = kDecline;
        c.grows = true;
        break;
      }
    }
    if (c.size >= 0 && total + found > c.size) {
      c.state = kAsym;  // left the component: the pattern is not symmetric
      break;
    }
    if (kLabel && !direct) {
      // group the children by parent (their order of arrival in a group is
      // arbitrary), give the table's slots back, mark the children visited
      const int wave = tid >> 6, lane = tid & 63;
      typename V::Kept r[kPer];
      int32_t par[kPer], arr[kPer];
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        const int32_t i = tid + j * kThreads;
        par[j] = 0;
        if (i < found) {
          const int s = L.t.slot[i];
          r[j] = V::keep(S, b ^ 1, i);
          par[j] = static_cast<int32_t>(L.t.hv[s]);
          arr[j] = atomicAdd(&L.t.pcnt[par[j]], 1);
          L.t.hk[s] = kNone;
          L.t.hv[s] = kUnclaimed;
          const uint32_t x = static_cast<uint32_t>(V::vertex(r[j]) - c.base);
          atomicOr(&S.bits[x >> 5], bit_of(x));
        }
      }
      __syncthreads();
      unsigned long long* keys = static_cast<unsigned long long*>(V::spare(S, b));
      int32_t* pre = reinterpret_cast<int32_t*>(keys + kCap);
      // exclusive prefix of the counts over the parents.  Up to kScanAll
      // parents every wave with children scans them all by itself (and
      // stores what the others store), which saves a barrier and the sum
      // over the waves
      int32_t before = 0;
      const bool busy = wave * 64 < found;  // this wave holds children
      if (len <= kScanAll) {
        if (busy) {
          constexpr int kEach = kScanAll / 64;
          const int each = (len + 63) >> 6;  // parents per lane
          const int32_t p0 = lane * each;
          int32_t n[kEach], sum = 0;
#pragma unroll
          for (int x = 0; x < kEach; ++x) {
            if (x >= each) break;
            n[x] = p0 + x < len ? L.t.pcnt[p0 + x] : 0;
            sum += n[x];
          }
          int32_t run = wave_scan(sum) - sum;
#pragma unroll
          for (int x = 0; x < kEach; ++x) {
            if (x >= each) break;
            if (p0 + x < len) pre[p0 + x] = run;
            run += n[x];
          }
          __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        }
      } else {
        // kWavePar parents a wave, then the waves' totals, in every wave
        if (wave * kWavePar < len) {
          const int32_t p0 = wave * kWavePar + lane * (kWavePar / 64);
          int32_t n[kWavePar / 64], sum = 0;
#pragma unroll
          for (int x = 0; x < kWavePar / 64; ++x) {
            n[x] = p0 + x < len ? L.t.pcnt[p0 + x] : 0;
            sum += n[x];
          }
          const int32_t incl = wave_scan(sum);
          int32_t run = incl - sum;
#pragma unroll
          for (int x = 0; x < kWavePar / 64; ++x) {
            if (p0 + x < len) pre[p0 + x] = run;
            run += n[x];
          }
          if (lane == 63) S.wtot[wave] = incl;
        }
        __syncthreads();
        const int32_t t = lane < kWaves && lane * kWavePar < len ? S.wtot[lane] : 0;
        before = wave_scan(t) - t;
      }
      int32_t first[kPer], end[kPer];
      uint64_t key[kPer];
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        if (!busy) continue;
        const int32_t i = tid + j * kThreads;
        const int32_t p = par[j], q = p + 1 < len ? p + 1 : p;
        first[j] = pre[p];
        end[j] = p + 1 < len ? pre[q] : found;
        if (len > kScanAll) {
          // (both shuffles by the whole wave: a lane outside a branch has
          // no value to give)
          const int32_t off_p = __shfl(before, p / kWavePar, 64);
          const int32_t off_q = __shfl(before, q / kWavePar, 64);
          first[j] += off_p;
          end[j] += p + 1 < len ? off_q : 0;
        }
        if (i < found) {
          key[j] = V::key(r[j]);
          keys[first[j] + arr[j]] = key[j];
        }
      }
      __syncthreads();
      // rank inside the group: SortPerm's order among siblings
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        const int32_t i = tid + j * kThreads;
        if (i >= found) continue;
        const int32_t to = place(keys, first[j], end[j], key[j]);
        V::put(S, b ^ 1, to, r[j]);
        const int32_t v = V::vertex(r[j]), pos = c.anchor - total - to;
        P.perm[pos] = v;
        P.iperm[v] = pos;
        m += static_cast<long long>(key[j] >> 32);
      }
      __syncthreads();
    }
    total += found;
    len = found;
    ++level;
    if (poll_abort(P, S, c)) {
      c.state = kAbort;
      break;
    }
  }
  Pass r;
  r.ecc = level;
  r.count = total;
  r.key = kMaxKey;
  r.m = 0;
  if (c.state == kRun) {
    // the minimum (degree, id) of the last level
    uint64_t k = kMaxKey;
    for (int32_t i = tid; i < len; i += kThreads) {
      const uint64_t x = V::level_key(S, level & 1, i);
      k = x < k ? x : k;
    }
    if (tid == 0) S.key = kMaxKey;
    __syncthreads();
    k = wave_min_u64(k);
    if ((tid & 63) == 0 && k != kMaxKey) atomicMin(&S.key, static_cast<unsigned long long>(k));
    __syncthreads();
    r.key = uniform(static_cast<uint64_t>(S.key));
    if (kLabel) r.m = block_sum_i64(m, S.red);
    if (c.size >= 0 && total != c.size) c.state = kAsym;
  }
  __syncthreads();
  return r;
}

// One pass of the kind asked for, on the fixed-stride rows or on the CSR.
__device__ __forceinline__ Pass run_pass(const ComponentParams& P, Lds& S, Ctx& c, int kind,
                                         bool ell, int32_t root) {
  c.state = kRun;
  if (ell) {
    c.width = P.width_limit < EllLevels::kCap ? P.width_limit : EllLevels::kCap;
    if (kind == kLabelled) return component_pass<EllLevels, kLabelled>(P, S, c, root);
    if (kind == kProbe) return component_pass<EllLevels, kProbe>(P, S, c, root);
    return component_pass<EllLevels, kSearch>(P, S, c, root);
  }
  c.width = P.width_limit < CsrLevels::kCap ? P.width_limit : CsrLevels::kCap;
  if (kind == kLabelled) return component_pass<CsrLevels, kLabelled>(P, S, c, root);
  if (kind == kProbe) return component_pass<CsrLevels, kProbe>(P, S, c, root);
  return component_pass<CsrLevels, kSearch>(P, S, c, root);
}

// The whole ordering of a component, or why not (c.state).  A task of unknown
// size is only probed: its first level structure, reported in *P.probe (and,
// when it is not the whole graph, its vertices in P.visit).  resume: that
// probe's component, ordered from there.
__device__ __forceinline__ void order_component(const ComponentParams& P, Lds& S, Ctx& c,
                                                const CompTask& task, bool resume) {
  c.size = task.size;
  c.anchor = task.anchor;
  // Algorithm 2 from the component's lowest id; from the third search on the
  // search is the labelled BFS itself (Algorithm 3 starts at the root of the
  // last search), and stands if its eccentricity does not grow
  bool ell = P.ell != nullptr;
  int kind = task.size < 0 ? kProbe : kSearch;
  int32_t nbfs = 1, root = task.seed, nlvl = -2;
  while (true) {
    Pass r;
    if (resume && nbfs == 1) {
      r.ecc = uniform(P.probe->ecc);
      r.key = uniform(static_cast<uint64_t>(P.probe->key));
      r.count = task.size;
      r.m = 0;
      c.state = kRun;
    } else {
      r = run_pass(P, S, c, kind, ell, root);
    }
    if (ell && (c.state == kLong ||
                (c.state == kDecline && P.width_limit > EllLevels::kCap && !c.grows))) {
      // a row too long for the copy, or a level too wide for its rows: the
      // same pass on the CSR, and the others after it
      ell = false;
      continue;
    }
    if (c.state != kRun) {
      if (kind == kProbe && threadIdx.x == 0) P.probe->ecc = c.level;
      return;
    }
    if (kind == kProbe) {
      if (threadIdx.x == 0) {
        P.probe->ecc = r.ecc;
        P.probe->size = r.count;
        P.probe->key = r.key;
      }
      if (r.count != c.range)
        for (int32_t i = threadIdx.x; i < c.range; i += kThreads)
          P.visit[c.base + i] = static_cast<int32_t>(S.bits[i >> 5] >> (i & 31) & 1u);
      return;
    }
    if (nbfs == 1) nlvl = r.ecc - 1;
    const bool deeper = r.ecc > nlvl;
    if (kind == kLabelled && (P.pp_variant == 1 || !deeper)) {
      if (threadIdx.x == 0) {
        CompResult* res = P.results + task.index;
        res->root = root;
        res->nbfs = nbfs;
        res->levels = r.ecc + 1;
        res->size = task.size;
        res->m = r.m;
      }
      return;
    }
    const int32_t last = static_cast<int32_t>(r.key & 0xffffffffu);
    if (deeper) {
      nlvl = r.ecc;
      ++nbfs;
      root = last;
      kind = P.pp_variant == 0 && nbfs >= 3 ? kLabelled : kSearch;
    } else {
      // the searches ended before the third: the labelled BFS from the root
      // of the last one, or (Algorithm 4) from the vertex it returned
      if (P.pp_variant == 1) root = last;
      kind = kLabelled;
    }
  }
}

__global__ void __launch_bounds__(kThreads) k_component(ComponentParams P) {
  __shared__ Lds S;
  if (P.bad_csr != nullptr && ld_relaxed(P.bad_csr) != 0) return;
  Ctx c{};
  const int32_t tasks = P.n_head + P.n_big + P.n_small;
  uint32_t fetched = 0;
  while (true) {
    shuffle_delay(P.shuffle, blockIdx.x, fetched++);
    __syncthreads();
    if (threadIdx.x == 0) {
      int32_t ti = atomicAdd(P.queue, 1);
      if (ti < tasks && ld_relaxed(&P.gctl->error) != 0) ti = tasks;
      S.task = ti;
    }
    __syncthreads();
    const int32_t taken = uniform(S.task);
    if (taken >= tasks) return;
    const int32_t ti = shuffle_index(taken, tasks, P.shuffle);
    const int list = ti < P.n_head ? 0 : (ti < P.n_head + P.n_big ? 1 : 2);
    CompTask task = list == 0   ? P.head
                    : list == 1 ? P.big[ti - P.n_head]
                                : P.small[ti - P.n_head - P.n_big];
    task.seed = uniform(task.seed);
    task.size = uniform(task.size);
    task.index = uniform(task.index);
    task.anchor = uniform(task.anchor);
    const bool resume = list == 0 && P.head.size >= 0;
    const int seg = P.nseg > 1 ? find_segment(P.seg_off, P.nseg, task.seed) : 0;
    c.base = P.nseg > 1 ? uniform(P.seg_off[seg]) : 0;
    c.range = (P.nseg > 1 ? uniform(P.seg_off[seg + 1]) : P.n) - c.base;
    c.state = kDecline;
    if (c.range <= kComponentRange) {
      c.grows = false;
      order_component(P, S, c, task, resume);
    }
    if (threadIdx.x == 0) {
      // (whatever was neither ordered nor refused is left to the team kernel)
      const bool left = c.state == kDecline || c.state == kLong;
      P.declined[ti] = left ? 1 : 0;
      if (left) atomicAdd(&P.counts[list], 1);
      if (c.state == kAsym) flag_error(P.gctl, RCM_ERR_NOT_SYMMETRIC);
    }
    if (c.state == kAbort) return;
  }
}

// ---------------------------------------------------------------------------
// The first level structure of a long component of a graph too large for the
// engine above: levels of at most kLongCap vertices of bounded rows, visited
// marks of at most kLongRange vertices.  It only measures, so its LDS holds
// the marks and two levels of rows, and nothing else.  A level is one memory
// round trip, the rows of the vertices found (0.82 us for the strip of 32 x
// 31,250 vertices, whose rows no die's L2 holds; the team took 1.65).  Loads
// of the next level's rows ahead of the barrier made it 1.29 us: the loads
// behind them wait for them.
// ---------------------------------------------------------------------------
constexpr int kLongThreads = 512;
constexpr int kLongCap = 256;
struct LongLds {
  uint32_t bits[kLongRange / 32];
  int4 row[2][kLongCap][2];
  int32_t v[2][kLongCap];
  int32_t cnt[3];             // level mod 3: size of the level being found (and kLongRow)
  int32_t stop;
  unsigned long long key;
};
static_assert(sizeof(LongLds) <= 160 * 1024, "one work-group's LDS");

// kN entries a lane of the rows of the level's vertices: the new ones, with
// their rows, to the next level.  (A row's own vertex and its fillers are
// marked already.)
template <int kN>
__device__ __forceinline__ void long_reach(const ComponentParams& P, LongLds& S, int b,
                                           int32_t len, int32_t level, int32_t* cnt) {
  constexpr int kLanes = kEllWidth / kN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int32_t i = tid / kLanes;
  if (i >= len) return;
  const int32_t* mine = reinterpret_cast<const int32_t*>(S.row[b][i]) + kN * (tid % kLanes);
  int32_t w[kN], r[kN][kEllWidth];
  uint32_t old[kN];
  bool fresh[kN];
#pragma unroll
  for (int j = 0; j < kN; ++j) w[j] = mine[j];
#pragma unroll
  for (int j = 0; j < kN; ++j)
    old[j] = atomicOr(&S.bits[static_cast<uint32_t>(w[j]) >> 5],
                      bit_of(static_cast<uint32_t>(w[j])));
#pragma unroll
  for (int j = 0; j < kN; ++j) {
    fresh[j] = (old[j] & bit_of(static_cast<uint32_t>(w[j]))) == 0;
    const int4* row = P.ell + 2 * static_cast<size_t>(fresh[j] ? w[j] : 0);
    const int4 lo = row[0], hi = row[1];
    r[j][0] = lo.x; r[j][1] = lo.y; r[j][2] = lo.z; r[j][3] = lo.w;
    r[j][4] = hi.x; r[j][5] = hi.y; r[j][6] = hi.z; r[j][7] = hi.w;
  }
  // (behind the loads, which would otherwise wait for the stores)
#pragma unroll
  for (int j = 0; j < kN; ++j)
    if (fresh[j]) P.dkey[w[j]] = distance_word(level + 1);
  int total = 0;
  unsigned long long m[kN], all = 0;
#pragma unroll
  for (int j = 0; j < kN; ++j) {
    m[j] = __ballot(fresh[j]);
    total += __popcll(m[j]);
    all |= m[j];
  }
  if (all == 0) return;
  const int first = __builtin_ctzll(all);
  int base = 0;
  if (lane == first) base = lds_add(cnt, total);
  base = __builtin_amdgcn_readlane(base, first);
#pragma unroll
  for (int j = 0; j < kN; ++j) {
    const int at = base + __builtin_amdgcn_mbcnt_hi(
                              static_cast<uint32_t>(m[j] >> 32),
                              __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m[j]), 0));
    base += __popcll(m[j]);
    if (!fresh[j] || at >= kLongCap) continue;
    S.v[b ^ 1][at] = w[j];
    S.row[b ^ 1][at][0] = make_int4(r[j][0], r[j][1], r[j][2], r[j][3]);
    S.row[b ^ 1][at][1] = make_int4(r[j][4], r[j][5], r[j][6], r[j][7]);
    if (r[j][0] < 0) atomicOr(cnt, kLongRow);
  }
}

__global__ void __launch_bounds__(kLongThreads) k_long_probe(ComponentParams P) {
  __shared__ LongLds S;
  if (ld_relaxed(P.bad_csr) != 0) return;
  const int tid = threadIdx.x;
  for (int32_t i = tid; i < (P.n + 31) / 32; i += kLongThreads) S.bits[i] = 0;
  if (tid < 3) S.cnt[tid] = 0;
  __syncthreads();
  if (tid == 0) {
    const int4 lo = P.ell[0];
    S.v[0][0] = 0;
    S.row[0][0][0] = lo;
    S.row[0][0][1] = P.ell[1];
    S.bits[0] = 1;
    S.key = kMaxKey;
    P.dkey[0] = distance_word(0);
    S.stop = lo.x < 0 ? 1 : 0;
  }
  __syncthreads();
  bool decline = uniform(S.stop) != 0;
  int32_t len = 1, total = 1, level = 0, near = 0;
  int l3 = 0;
  while (!decline) {
    int32_t* cnt = &S.cnt[l3];
    l3 = l3 == 2 ? 0 : l3 + 1;
    if (tid == 0) S.cnt[l3] = 0;
    const int b = level & 1;
    if (len <= kLongThreads / 8)
      long_reach<1>(P, S, b, len, level, cnt);
    else if (len <= kLongThreads / 4)
      long_reach<2>(P, S, b, len, level, cnt);
    else
      long_reach<4>(P, S, b, len, level, cnt);
    __syncthreads();
    const int32_t found = uniform(*cnt);
    if (found == 0) break;
    // (a level that grows like a volume's: see component_pass)
    if (level == 3) near = found;
    decline = found > kLongCap || (level == 7 && found * 10 >= near * P.growth);
    total += found;
    len = found;
    ++level;
    if (P.abort_flag != nullptr && (level & 63) == 0) {
      if (tid == 0) {
        S.stop = abort_requested(P.abort_flag) ? 1 : 0;
        if (S.stop != 0) flag_error(P.gctl, RCM_ERR_ABORTED);
      }
      __syncthreads();
      if (uniform(S.stop) != 0) return;
      __syncthreads();
    }
  }
  if (decline) {
    if (tid == 0) {
      P.probe->ecc = level > 0 ? level - 1 : 0;
      atomicAdd(&P.counts[0], 1);
    }
    return;
  }
  // the minimum (degree, id) of the last level
  if (tid < len) {
    const int32_t v = S.v[level & 1][tid];
    const int4 lo = S.row[level & 1][tid][0], hi = S.row[level & 1][tid][1];
    atomicMin(&S.key, static_cast<unsigned long long>(
                          pack_key(EllLevels::degree(v, lo, hi), v)));
  }
  __syncthreads();
  if (tid == 0) {
    P.probe->ecc = level;
    P.probe->size = total;
    P.probe->key = S.key;
  }
  if (total != P.n)
    for (int32_t i = tid; i < P.n; i += kLongThreads)
      P.visit[i] = static_cast<int32_t>(S.bits[i >> 5] >> (i & 31) & 1u);
}

// The declined tasks, in list order (vertex 0's component and the large ones,
// then the small ones), for the team kernel: one work-group.
__global__ void __launch_bounds__(kThreads)
k_declined(ComponentParams P, CompTask* __restrict__ big_out, CompTask* __restrict__ small_out) {
  __shared__ int scratch[17];
  const int32_t n_first = P.n_head + P.n_big;
  for (int l = 0; l < 2; ++l) {
    const int32_t n = l == 0 ? n_first : P.n_small;
    const int32_t* d = l == 0 ? P.declined : P.declined + n_first;
    CompTask* out = l == 0 ? big_out : small_out;
    int32_t run = 0;
    for (int32_t i0 = 0; i0 < n; i0 += kThreads) {
      const int32_t i = i0 + threadIdx.x;
      const int take = i < n && d[i] != 0 ? 1 : 0;
      int total;
      const int at = block_excl_scan(take, scratch, &total);
      if (take)
        out[run + at] = l == 1 ? P.small[i] : (i < P.n_head ? P.head : P.big[i - P.n_head]);
      run += total;
    }
  }
}

// A declined probe's last level that was expanded completely: its vertices'
// records; what lies behind them is found again.
__global__ void __launch_bounds__(256)
k_front(ComponentParams P, int32_t level, int4* __restrict__ qi, int32_t* __restrict__ front) {
  const unsigned long long at = distance_word(level);
  for (int32_t v = blockIdx.x * 256 + threadIdx.x; v < P.n; v += gridDim.x * 256) {
    const unsigned long long w = P.dkey[v];
    if (w == 0 || w > at) continue;  // (a larger word is a shorter distance)
    if (w == at) {
      const int4 inf = P.vinfo[v];
      qi[atomicAdd(front, 1)] = make_int4(v, inf.x, inf.y, level);
    } else {
      P.dkey[v] = 0;
    }
  }
}

}  // namespace

hipError_t launch_component(const ComponentParams& p, hipStream_t s) {
  const int64_t tasks = static_cast<int64_t>(p.n_head) + p.n_big + p.n_small;
  if (tasks <= 0) return hipSuccess;
  // a work-group's LDS leaves room for one per CU; more would only queue
  const int blocks = static_cast<int>(tasks < 1024 ? tasks : 1024);
  k_component<<<blocks, kThreads, 0, s>>>(p);
  return hipGetLastError();
}

hipError_t launch_long_probe(const ComponentParams& p, hipStream_t s) {
  k_long_probe<<<1, kLongThreads, 0, s>>>(p);
  return hipGetLastError();
}

hipError_t launch_front(const ComponentParams& p, int32_t level, int4* qi, int32_t* front,
                        hipStream_t s) {
  k_front<<<static_cast<unsigned>((p.n + 1023) / 1024), 256, 0, s>>>(p, level, qi, front);
  return hipGetLastError();
}

hipError_t launch_declined(const ComponentParams& p, CompTask* big_out, CompTask* small_out,
                           hipStream_t s) {
  k_declined<<<1, kThreads, 0, s>>>(p, big_out, small_out);
  return hipGetLastError();
}

}  // namespace rcm
