// Types, kernel arguments and small device helpers shared by the attention kernels.
#pragma once
#include "svg_internal.h"

namespace svg {
namespace attn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;   // operand type of the transposing LDS read

enum Mode { kDense = 0, kSparse = 1, kProfile = 2, kSparseExact = 3, kSparseGather = 4 };

constexpr float kNegBig = -1.0e30f;     // finite stand-in for -inf as the initial row maximum
constexpr float kLazySum = 8192.0f;      // a lane's per-tile sum of exponentials above this forces a new reference maximum

constexpr int kNoTile = 0x7fffffff;
constexpr unsigned kRsrcFlags = 0x00020000u;   // raw buffer, 32-bit data format (gfx9 encoding)

typedef __attribute__((address_space(3))) unsigned char lds_byte;

// Raw buffer descriptor as four scalar words.
__device__ __forceinline__ u32x4 buffer_words(const void* base, unsigned bytes) {
  const uintptr_t p = reinterpret_cast<uintptr_t>(base);
  return u32x4{(unsigned)__builtin_amdgcn_readfirstlane((unsigned)p), (unsigned)__builtin_amdgcn_readfirstlane((unsigned)(p >> 32) & 0xffffu),
               (unsigned)__builtin_amdgcn_readfirstlane(bytes), kRsrcFlags};
}
// Two loads of 16 bytes per lane straight from memory into LDS, lane l at lds_address + 16 l and, for
// the second, `step` bytes behind; out of range reads give zeros.  Written as assembly because the compiler,
// which cannot tell the two staging buffers apart, puts a wait for every such load in front of the next
// LDS read; the one wait that is needed is wait_loads_to_lds() in front of the barrier that publishes the tile.
// A load must issue five wait states after a vector instruction (v_readfirstlane, v_readlane of a spilled
// register) that wrote a scalar register it reads.  The compiler keeps that distance for loads it knows of but
// not in front of this statement, so the statement holds all of it: one for s_mov, four for s_nop 3.  Two loads
// share it (a statement with the same wait for every load cost 0.0-0.4 % of the attention passes, this one
// nothing that could be measured).
// m0 holds a byte address anywhere in the 160 KB of LDS: the second team of svg_teams.hip stages above 64 KB.
// The statement overwrites m0 and says so; the compiler warns that it will not save a reserved register, once for
// every place the function is inlined.  Nothing has to be saved: no other instruction of these kernels uses
// m0 (a test looks through the compiler's output for one).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_to_lds(const u32x4 rsrc, int voffset0, int voffset1, int soffset0, int soffset1,
                                            unsigned lds_address, const int step) {
  asm volatile("s_mov_b32 m0, %5\n\ts_nop 3\n\tbuffer_load_dwordx4 %0, %2, %3 offen lds\n\t"
               "s_add_u32 m0, m0, %6\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %4 offen lds"
               :: "v"(voffset0), "v"(voffset1), "s"(rsrc), "s"(soffset0), "s"(soffset1), "s"(lds_address), "i"(step)
               : "memory", "m0", "scc");
}
#pragma clang diagnostic pop
// Waits until at most N of this wavefront's loads are outstanding (they complete in order).
template <int N>
__device__ __forceinline__ void wait_loads_to_lds() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// A bare workgroup barrier.  For loops in which LDS is written by such loads only and every read of the
// staging buffers was consumed before.
__device__ __forceinline__ void barrier_loads_done() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The tiles of a kept-tile list row, handed out in turn, from entry `start` on and around its end, then kNoTile:
// 64 entries at a time wait in a register (one per lane), the next 64 are in flight.  Every value taken
// is the same in all lanes.
struct TileList {
  const int32_t* row;
  int len, start, taken, now, ahead;
  int step, first;      // two teams: every second entry, from this one on

  __device__ __forceinline__ int load(int base) const {
    int i = (base + (int)(threadIdx.x & 63)) * step + first;
    if (i >= len) return kNoTile;
    i += start;
    return row[i >= len ? i - len : i];
  }
  __device__ __forceinline__ void open(const int32_t* row_, int len_, int start_, int step_ = 1, int first_ = 0) {
    row = row_;
    len = len_;
    start = start_;
    step = step_;
    first = first_;
    taken = 0;
    ahead = load(0);
  }
  // One rarely taken branch: a workgroup that has its compute unit to itself feels every instruction between two tiles.
  __device__ __forceinline__ int next() {
    const int lane = taken & 63;
    if (lane == 0) {
      now = ahead;
      asm volatile("" : "+v"(now));       // the copy first: the next 64 then go to the register they are waited for in
      ahead = load(taken + 64);
    }
    ++taken;
    return __builtin_amdgcn_readlane(now, lane);
  }
};

// --------------------------------------------------------------------------------------------
// Dispatch order of the block-sparse passes.
//
// Workgroups are dealt round-robin to the 8 XCDs (blockIdx.x % 8) and start in the order of
// blockIdx.x / 8, so what a workgroup works on decides both which L2 serves it and when it
// starts.  Two things make query tiles unequal: a tile that holds a text row keeps every key
// tile (its list is many times longer than the others'), and the lists of the two patterns
// differ in length while the labels, known on the device only, say which heads have which.
//  * Heavy tiles (those with a text row) start first on every XCD, a head's heavy tiles on
//    one XCD (they stream the same K and V), heads dealt to the XCDs in turn.  Started last
//    they would run on alone after every other workgroup of their XCD has finished.
//  * Where a heavy tile is much longer than an even share of the work it is the whole time of the pass (with few heads or
//    short lists: 18 heads of 1909 tokens 47 of 51 us).  Then four workgroups take it, 32 rows each, its keys
//    split over their wavefronts (svg_split.h), dealt to all XCDs.  That costs about 2.5 times the tile's work and takes 0.3 of
//    its time, so it needs places that would be empty (ratio: nk places / (light tiles + 4 heavy tiles)) and a heavy list that is long
//    beside the others, which then take the time of the pass.  Time whole over time in parts, 580 calls of 2 to 92 heads of 190 to 45000
//    tokens, both head dimensions, FP8 among them (8 heads of 18977 tokens 392 -> 265 us, FP8 257 -> 183):
//      ratio above 2.08, a heavy list 16 tiles and more longer than the mean other one: 0.96-2.05, median 1.44; in parts
//      ratio above 3.2, 12 key tiles and more: 0.94-1.65, median 1.23; in parts
//      ratio 2.08 to 3.2, lists closer than that: 0.76-1.37, median 0.98; whole, as below 12 key tiles (0.92-1.29)
//      ratio 1.82 to 2.08: 0.77-1.47, median 1.02; 1.3 to 1.82: 0.77-1.27, median 1.01; below: 0.62-1.04; whole
//  * The other tiles of all heads with the same label form one sequence (head after head,
//    ascending query tiles); every XCD takes one contiguous eighth of the spatial sequence
//    and one of the temporal sequence, the one with the longer lists first.  Each XCD so gets
//    the same share of both kinds of work whatever the labels are, and consecutive workgroups
//    of an XCD still are nearby query tiles of one head (overlapping key windows).  Where a compute unit holds one workgroup (two teams)
//    and the 32 of an XCD would not do for both eighths rounded up by themselves, what the second sequence has beyond a multiple of eight goes to the XCDs that
//    the first has left out (xcd_share): 138 and 115 tiles gave an XCD 33 (11 heads of 2910 rows 19.6 us with one team, 23.4 with two, so 17.4, exact
//    24.1, 28.1, 20.7; head dimension 128 29.0, 35.0, 26.1).  Not so elsewhere: the last tile of an eighth has a short list at the end of a sequence (6 heads of 21885 rows with the first-frame sink, 1026 tiles for 512 places, 478
//    -> 578 us), and text-row tiles decide how full an XCD is where there are any (0.88-1.07).
//  * Inside the part of a head that an XCD takes, the query tiles are dispatched with a stride:
//    0, r, 2r, ..., then 1, r+1, ...  A workgroup walks its list one key tile per tile time, the
//    window of query tile g + 1 lies BM / BN = 2 key tiles above that of g, and in steady state
//    a place on the XCD frees up every T / slots tile times (T: tiles per list, slots: resident
//    workgroups).  With r = T / (2 slots) the next workgroup starts exactly as much later as
//    its window lies higher, so all workgroups of the XCD read the same key tile at the same
//    time and L2 serves all but one of them.  r is rounded, at least 1, per label (the lists of
//    the two patterns differ in length).
// With more than 256 heads the labels are not looked at: one sequence in head order.
// --------------------------------------------------------------------------------------------
constexpr int kXcdUnits = 32;          // compute units of an XCD
constexpr int kWideLabelWords = 4;     // label classes are formed for up to 64 * kWideLabelWords heads

struct SparseOrder {
  int g_lo;    // a head's query tiles without a text row are [g_lo, g_lo + nl)
  int nl;
  int nh;      // tiles with a text row per head (the others, ascending)
  int hmax;    // workgroups per XCD reserved for them
  int slots;   // workgroups resident on one XCD (sets the stride, see above)
  int parts_log2;      // workgroups reserved per tile with a text row: 1 << parts_log2; 0: none is taken in parts
  int nk;              // key tiles, what a tile with a text row keeps
  int places;          // workgroups resident on the chip; two teams: as with one, the lines of sparse_slot were measured so, and all parts find a place (two_teams)
};

inline SparseOrder sparse_order(int BH, int nqt, int BM, int off, int video_end, int N, int slots, int places, int parts_log2, int nk) {
  SparseOrder so;
  const int lo = off > 0 ? (off + BM - 1) / BM : 0;
  int hi = video_end < N ? video_end / BM : nqt;
  so.g_lo = lo < nqt ? lo : nqt;
  if (hi < so.g_lo) hi = so.g_lo;
  so.nl = hi - so.g_lo;
  so.nh = nqt - so.nl;
  so.hmax = so.nh * ((BH + 7) / 8);
  so.slots = slots;
  // With so many heavy tiles that their parts alone are above the line (see above) whatever the labels say, no workgroups
  // are reserved for parts: idle, they took up to 6 % of the pass (4000 heads of 220 rows 131 -> 140 us, FP8 201 -> 213),
  // and from 2^22 heavy tiles on the grid was too large to launch.
  so.parts_log2 = nk >= 12 && 12ll * places > 100ll * BH * so.nh ? parts_log2 : 0;
  so.nk = nk;
  so.places = places;
  return so;
}

// grid size: an XCD's two eighths together hold at most floor(BH nl / 8) + 2 tiles
inline unsigned sparse_grid(const SparseOrder& so, int BH) {
  return 8u * (unsigned)(((long long)so.hmax << so.parts_log2) + (long long)BH * so.nl / 8 + 2);
}

// Where the share of XCD xcd of n things begins if the n % 8 left over go one each to the XCDs from first_extra on, XCD 0 behind XCD 7.
__host__ __device__ inline int xcd_share(long long n, int xcd, int first_extra) {
  const int extra = (int)(n & 7), wrapped = first_extra + extra - 8;
  const int behind = xcd - first_extra;
  const int given = (wrapped > 0 ? (xcd < wrapped ? xcd : wrapped) : 0) + (behind < 0 ? 0 : behind < extra ? behind : extra);
  return (int)(xcd * (n >> 3)) + given;
}

// Which (head, query tile, pattern) does this workgroup take?  false: none.  For a tile without
// text rows, cl is its index in its label's sequence and head_cl0 the index of its head's first
// tile there (cl = -1 for a heavy tile).  Every value returned is the same in all lanes.
// (LW: 64-head words of label bits; the kernels are built for 1 and for kWideLabelWords, and the
// launcher takes the wide form only when there are more than 64 heads)
template <int LW, int TEAMS = 1>
__device__ __forceinline__ bool sparse_slot(const SparseOrder so, const int BH, const uint8_t* labels,
                                            const int32_t* rp_s, const int32_t* rp_t, const int xcd, const int loc,
                                            int& bh, int& grp, int& pat, int& cl, int& head_cl0, int& part) {
  const int lane = threadIdx.x & 63;
  // The labels as bit masks, 64 heads per word (bit = temporal).  Words of their own, not an array: the
  // compiler put an array into LDS (8 KB of it) or scratch memory.
  static_assert(LW == 1 || LW == 4, "one variable per word");
  const bool classed = labels != nullptr && BH <= 64 * LW;
  auto label = [&](int w) -> int {
    const int h = 64 * w + lane;
    return classed && h < BH ? labels[h] : 0;
  };
  const int l0 = label(0), l1 = LW > 1 ? label(1) : 0, l2 = LW > 1 ? label(2) : 0, l3 = LW > 1 ? label(3) : 0;
  // List tiles of a head's light query tiles, per pattern, on their way together with the labels: one after the
  // other they cost the short passes 0.3 us (8-25 us, 1.2 % at the mean of 90 calls).
  const int nnz_s = rp_s[so.g_lo + so.nl] - rp_s[so.g_lo], nnz_t = rp_t[so.g_lo + so.nl] - rp_t[so.g_lo];
  const unsigned long long m0 = __builtin_amdgcn_ballot_w64(l0 != 0);
  const unsigned long long m1 = LW > 1 ? __builtin_amdgcn_ballot_w64(l1 != 0) : 0ull, m2 = LW > 1 ? __builtin_amdgcn_ballot_w64(l2 != 0) : 0ull,
                           m3 = LW > 1 ? __builtin_amdgcn_ballot_w64(l3 != 0) : 0ull;
  const int nT = __builtin_popcountll(m0) + __builtin_popcountll(m1) + __builtin_popcountll(m2) + __builtin_popcountll(m3);
  auto label_bit = [&](int h) -> int {
    const int w = h >> 6;
    const unsigned long long word = LW == 1 || w == 0 ? m0 : w == 1 ? m1 : w == 2 ? m2 : m3;
    return (int)((word >> (h & 63)) & 1);
  };
  cl = -1;
  head_cl0 = 0;
  part = -1;
  const int nS = BH - nT;
  const long long light = (long long)nS * nnz_s + (long long)nT * nnz_t;
  const long long longest = (long long)so.nk * so.places, even = light + 4ll * BH * so.nh * so.nk;
  const bool split = so.parts_log2 > 0 && (5 * longest > 16 * even || (12 * longest > 25 * even && (so.nk - 16ll) * BH * so.nl >= light));
  // (whole heavy tiles leave the workgroups of the other parts at the end of the grid, where they do not come between)
  const int front = split ? so.hmax << so.parts_log2 : so.hmax;
  if (loc < front) {
    int l = loc;
    if (split) {
      const int i = loc * 8 + xcd;      // all parts dealt to the XCDs in turn
      part = i & ((1 << so.parts_log2) - 1);
      l = i >> so.parts_log2;
      bh = l / so.nh;
    } else {
      bh = xcd + 8 * (loc / so.nh);
    }
    const int j = l % so.nh;
    if (bh >= BH) return false;
    grp = j < so.g_lo ? j : j + so.nl;
    pat = classed ? label_bit(bh) : (labels ? labels[bh] != 0 : 0);
    return true;
  }
  if (so.nl == 0) return false;
  int l = loc - front;
  int first = nS == 0;            // the label whose sequence comes first
  if (nT > 0 && nS > 0) first = nnz_t > nnz_s;
  const int nA = first ? nT : nS;
  const long long NA = (long long)nA * so.nl, NB = (long long)(BH - nA) * so.nl;
  int a0, a1, b0, b1;
  if (TEAMS > 1 && so.nh == 0 && BH * so.nl > 8 * kXcdUnits - 16) {
    const int left = (int)(NA & 7);
    a0 = xcd_share(NA, xcd, 0), a1 = xcd_share(NA, xcd + 1, 0);
    b0 = xcd_share(NB, xcd, left), b1 = xcd_share(NB, xcd + 1, left);
  } else {
    a0 = (int)((xcd * NA) >> 3), a1 = (int)(((xcd + 1) * NA) >> 3);
    b0 = (int)((xcd * NB) >> 3), b1 = (int)(((xcd + 1) * NB) >> 3);
  }
  int c = first;
  if (l < a1 - a0) {
    cl = a0 + l;
  } else {
    l -= a1 - a0;
    if (l >= b1 - b0) return false;
    cl = b0 + l;
    c = !first;
  }
  const int kth = cl / so.nl;
  head_cl0 = kth * so.nl;
  {
    // strided order inside the part [s0, s1) of this head that lies in the XCD's chunk
    const int c0 = c == first ? a0 : b0, c1 = c == first ? a1 : b1;
    const int s0 = max(c0, head_cl0), s1 = min(c1, head_cl0 + so.nl);
    const int len = s1 - s0;
    const int tiles_per_list = (c ? nnz_t : nnz_s) / so.nl;
    const int r = min(16, (tiles_per_list + so.slots) / (2 * so.slots));      // round(T / (2 slots))
    int idx = cl - s0;
    if (r > 1 && len > r) {
      int p = 0;
      for (; p < r; ++p) {        // which pass (p, p + r, p + 2r, ...) the idx-th workgroup belongs to
        const int in_pass = (len - p + r - 1) / r;
        if (idx < in_pass) break;
        idx -= in_pass;
      }
      idx = p + idx * r;
    }
    cl = s0 + idx;
  }
  grp = so.g_lo + (cl - head_cl0);
  if (classed) {
    // the kth head (from 0) with label c: find its word, then its bit
    bh = 0;
    int before = 0;
    bool found = false;
    auto look_in = [&](int w, unsigned long long word) {
      const int left = BH - 64 * w;
      const unsigned long long valid = left >= 64 ? ~0ull : left > 0 ? (1ull << left) - 1 : 0ull;
      const unsigned long long cm = c ? word : ~word & valid;
      const int cnt = __builtin_popcountll(cm);
      if (!found && kth < before + cnt) {
        const int rank = __builtin_popcountll(cm & ((1ull << lane) - 1));
        const unsigned long long hit = __builtin_amdgcn_ballot_w64(((cm >> lane) & 1) != 0 && rank == kth - before);
        bh = 64 * w + __builtin_ctzll(hit);
        found = true;
      }
      before += cnt;
    };
    look_in(0, m0);
    if (LW > 1) {
      look_in(1, m1);
      look_in(2, m2);
      look_in(3, m3);
    }
    pat = c;
  } else {
    bh = kth;
    pat = labels ? labels[bh] != 0 : 0;
  }
  return true;
}

// Quotient and remainder of v < 2^22 by d without a division; inv = floor((2^32 - 1) / d) (the quotient of the product is the true
// one or one less).
__device__ __forceinline__ unsigned divide(unsigned v, unsigned d, unsigned inv, unsigned& rest) {
  unsigned q = __umulhi(v, inv);
  rest = v - q * d;
  if (rest >= d) {
    rest -= d;
    ++q;
  }
  return q;
}

// transformed_to_token for kernels that are bound by latency and by fetching their own instructions: no division.
struct POuter {
  unsigned P, frames, inv_frames;      // frames of a position: F, or F - 1 behind the first frame
  int sink;
  // offset of the token at offset v of the P-outer order, and its position
  __device__ __forceinline__ int token(int v, int& pos) const {
    const bool first_frame = sink && v < (int)P;
    unsigned f;
    const unsigned p = divide(sink ? (unsigned)v - P : (unsigned)v, frames, inv_frames, f);
    pos = first_frame ? v : (int)p;
    return first_frame ? v : (int)((f + (sink ? 1u : 0u)) * P + p);
  }
  __device__ __forceinline__ int token(int v) const {
    int pos;
    return token(v, pos);
  }
};
inline POuter p_outer(const Geo& g) {
  POuter o;
  o.P = (unsigned)g.P;
  o.frames = g.sink ? (unsigned)(g.F > 1 ? g.F - 1 : 1) : (unsigned)g.F;
  o.inv_frames = 0xffffffffu / o.frames;
  o.sink = g.sink;
  return o;
}

struct AttnArgs {
  const __bf16* q;
  const __bf16* k;
  const __bf16* v;
  const __bf16* k_t;          // sparse: P-outer copies of k and v read by temporal heads instead of k, v; may be null
  const __bf16* v_t;
  void* o;                    // bf16 [B,H,N,D] (dense, sparse) or fp32 [slots][BH][t][D] (profile)
  const uint8_t* labels;      // sparse: per-head pattern, may be null
  const int32_t* row_table;   // gathering sparse form: token row of every P-outer row, nk * BN entries
  const int32_t* row_ptr[2];
  const int32_t* col_idx[2];
  const int32_t* rows;        // profile: sampled rows
  const int32_t* order_t;     // profile: indices into rows[], grouped by in-frame position (temporal variant); null: few rows, which the workgroups sort themselves
  int t;                      // profile: number of sampled rows
  ProfilePlan plan;           // profile: parts of the unmasked pass and of the masked passes
  int pieces;                 // profile: output slots of the unmasked pass where it runs in pieces and stands for the spatial pass too, or 0
  unsigned* tickets;          // profile: a word per head that this launch clears for the error pass; may be null
  float2* stats;              // profile: (reference maximum, row sum) per (output slot, head, row)
  int N, nk, BH;
  int nqt;                    // workgroups per head: query tiles (dense, sparse) or ceil(t / rows per workgroup) (profile)
  SparseOrder so;             // sparse: which workgroup takes which (head, query tile)
  int total;                  // logical workgroups
  int cohort;                 // dense: consecutive logical workgroups that go to one XCD
  int qo_token_order;         // sparse: q is read and o written in token order also for temporal heads
  float scale_log2;           // softmax scale * log2(e)
  int off, video_end, F, P, w_s, w_t, sink;
  int rows_per_group;         // profile: sampled rows per workgroup (the groups are balanced); 0: dealt in 32s
  // the split form
  int blocks_log2;            // workgroups per query tile: bm = 32 << blocks_log2
  int halves_log2;            // units of 32 keys per key tile: bn = 32 << halves_log2
  unsigned inv_P;             // floor((2^32 - 1) / P)
  POuter order;
};

// The form for calls with few rows (svg_split.hip).
bool split_form(const Geo& g, int mode, int t);      // does the split form take this call? (t: sampled rows of a profiling call)
bool split_sorts_rows(int t);                        // profiling: needs no row order from profile_order_kernel
int launch_split(const Geo& g, AttnArgs a, int mode, hipStream_t stream);

// Query tiles that go to one XCD in a row in a dense pass, `most` at the most.
int dense_cohort(int tiles, int most);

// The form for calls of at most one query tile to a compute unit (svg_teams.hip).
bool two_teams(const Geo& g);
int launch_teams(const Geo& g, const AttnArgs& a, int mode, hipStream_t stream);

// Profiling: the first workgroup clears the tickets of the error pass, which nothing reads in this launch.  (Its size is an argument of the template:
// blockDim.x brings 256 bytes of arguments: with those of gridDim.x in the error pass 0.7 % of 51 calls of 9-19 us)
template <int THREADS>
__device__ __forceinline__ void clear_tickets(const AttnArgs& a) {
  if (blockIdx.x == 0 && a.tickets != nullptr)
    for (int i = threadIdx.x; i < a.BH; i += THREADS) a.tickets[i] = 0;
}

// Coarse position bin of a sampled row for the temporal profiling pass (text rows first).
constexpr int kOrderBins = 2048;
__device__ __forceinline__ int order_bin(int n, int off, int video_end, int P) {
  if (n < off || n >= video_end) return 0;
  const int p = (n - off) % P;
  return 1 + (int)(((long long)p * (kOrderBins - 1)) / P);
}

// Lanes l and l^32 own the two halves of one query's keys.  v_permlane32_swap with
// both operands equal returns {x[l % 32], x[32 + l % 32]} in every lane, so the
// combined maximum / sum needs no LDS traffic.
__device__ __forceinline__ float both_halves_max(float x) {
  const unsigned u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float both_halves_sum(float x) {
  const unsigned u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Lanes l, l ^ 16, l ^ 32 and l ^ 48 own the quarters of one query's keys (the bf16 kernels);
// v_permlane16_swap exchanges neighbouring quarters the way v_permlane32_swap exchanges halves.
__device__ __forceinline__ float quarters_max(float x) {
  const unsigned u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return both_halves_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float quarters_sum(float x) {
  const unsigned u = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return both_halves_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// Minimum over the 16 lanes of a quarter wavefront (the rows of a 16-query block), the same in every lane.
__device__ __forceinline__ int quad_rows_min(int x) {
  x = min(x, __builtin_amdgcn_mov_dpp(x, 0x128, 0xf, 0xf, true));      // rotated by 8, 4, 2 and 1 lanes inside the quarter
  x = min(x, __builtin_amdgcn_mov_dpp(x, 0x124, 0xf, 0xf, true));
  x = min(x, __builtin_amdgcn_mov_dpp(x, 0x122, 0xf, 0xf, true));
  x = min(x, __builtin_amdgcn_mov_dpp(x, 0x121, 0xf, 0xf, true));
  return __builtin_amdgcn_readfirstlane(x);
}

// Minimum over the wavefront.
__device__ __forceinline__ int wave_min(int x) {
  x = min(x, __builtin_amdgcn_mov_dpp(x, 0x128, 0xf, 0xf, true));
  x = min(x, __builtin_amdgcn_mov_dpp(x, 0x124, 0xf, 0xf, true));
  x = min(x, __builtin_amdgcn_mov_dpp(x, 0x122, 0xf, 0xf, true));
  x = min(x, __builtin_amdgcn_mov_dpp(x, 0x121, 0xf, 0xf, true));
  return min(min(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
             min(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}

}  // namespace attn

}  // namespace svg
