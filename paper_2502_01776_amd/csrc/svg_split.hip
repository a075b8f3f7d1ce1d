// The attention passes for calls with few query rows (dense, block-sparse over a kept-tile list, exact masks, k and v
// gathered in place, and the passes of online profiling): the keys are split over the wavefronts of a workgroup.
//
// A call of a few hundred rows and heads gives attn_kernel (svg_attn.hip) fewer workgroups than the chip has places, and
// each of them walks its key tiles one after the other at 0.7-1.2 us a tile, most of it the latency of a lone
// workgroup: 13 tiles of 64 keys were 10 of the 15 us of the sparse pass over 8 heads of 787 rows.  Here a workgroup
// owns 32 query rows and each of its four wavefronts every fourth unit of 32 keys, with the products, layouts and softmax of
// attn_kernel, and at the end the four results (output, maximum, row sum) are merged through LDS.  Four times as many
// workgroups, a quarter of the chain in each: that pass takes 8 us, at 2 heads of 3290 rows 43.6 -> 20 us.
//
// A wavefront loads its K unit straight into the registers of the first product's A operand and stages its V unit through
// its own piece of LDS (rows in, transposing reads out), so there is no barrier before the merge.  Nothing
// is shared between wavefronts: a CU's loads move 8 KB (head dimension 64) or 16 KB for 32 x 32 scores, four times what
// attn_kernel's staged tiles need, and at 64 bytes a clock that is what bounds the kernel once all CUs are busy
// (0.4-0.6 of attn_kernel's rate with ten times the workgroups); it is taken only where split_form() says so.
// Eight wavefronts (one workgroup per CU at head dimension 128) measured 5-25 % slower throughout, two register sets
// for the loads at head dimension 64 up to 12 % (more instructions to fetch; a cold instruction cache is a
// good part of a short call).  With so few units per wavefront the row maximum is taken every time: attn_kernel's
// reference maximum would make the first unit, often a quarter of the work, take its exponentials twice.
#include "svg_split.h"

namespace svg {

namespace {

using namespace attn;

constexpr int kMaxFrames = 61; // profiling keeps one run of keys per frame in a lane, beside text prefix, sink and text suffix

template <int D, int MODE>
__global__ __launch_bounds__(64 * kWaves, 2) void split_kernel(AttnArgs a) {
  constexpr bool SPARSE = MODE == kSparse || MODE == kSparseExact || MODE == kSparseGather;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[split_lds_bytes(D)];
  // Which rows of which head?
  const int xcd = blockIdx.x & 7, loc = blockIdx.x >> 3;
  int bh = 0, grp = 0, pat = 0, variant = 0, chunk = 0, row0 = 0, list_begin = 0, list_end = 0;
  if (MODE == kProfile) {
    const int pairs = a.BH * a.nqt, pairs_per_xcd = (pairs + 7) >> 3, nm = a.plan.n_masked;
    const int unit = loc / pairs_per_xcd, pair = xcd * pairs_per_xcd + (loc - unit * pairs_per_xcd);
    clear_tickets<64 * kWaves>(a);
    if (unit >= a.plan.slots() || pair >= pairs) return;
    variant = unit < nm ? 1 : unit < 2 * nm ? 2 : 0;
    chunk = unit < nm ? unit : unit < 2 * nm ? unit - nm : unit - 2 * nm;
    bh = pair / a.nqt;
    grp = pair - bh * a.nqt;
  } else {
    // the row groups of a head, which stream the same K and V, on one XCD.  No look at the labels and lists to
    // order the work by: all workgroups start at once here, and reading them first would be one more trip to memory.
    const int per_xcd = (a.total + 7) >> 3, lid = xcd * per_xcd + loc;
    if (loc >= per_xcd || lid >= a.total) return;
    bh = lid / a.nqt;
    const int block = lid - bh * a.nqt;
    row0 = block * kRows;
    if (SPARSE) {
      grp = block >> a.blocks_log2;
      list_begin = a.row_ptr[0][grp];
      list_end = a.row_ptr[0][grp + 1];
      if (a.labels != nullptr) {
        const int t0 = a.row_ptr[1][grp], t1 = a.row_ptr[1][grp + 1];      // both patterns' lists while the label is on its way
        pat = __builtin_amdgcn_readfirstlane(a.labels[bh] != 0);
        list_begin = pat ? t0 : list_begin;
        list_end = pat ? t1 : list_end;
      }
    }
  }
  split_body<D, MODE>(a, lds, bh, row0, grp, pat, list_begin, list_end, variant, chunk);
}

template <int D, int MODE>
int launch_split_one(const AttnArgs& a, unsigned grid, hipStream_t stream) {
  (void)hipGetLastError();
  hipLaunchKernelGGL((split_kernel<D, MODE>), dim3(grid), dim3(64 * kWaves), 0, stream, a);
  return hip_status(hipGetLastError());
}

}  // namespace

namespace attn {

// Where the lines lie, by the number of workgroups (heads x groups of 32 rows), from 1100 calls of 1 to 48 heads and 192
// to 24000 rows, time of attn_kernel with whole text-row tiles over time here.  A CU holds three workgroups at head dimension 64 and two at 128;
// beyond one (256) or two (512) to a CU the last of them can cost as much as they save:
//   dense, exact masks: 1.03-3.0 up to 640 and 416 (0.98 once, at 589); dense 0.9 at 824 and 0.87 at 610
//   plain sparse:       64: 1.07-1.6 up to 512, 0.87-1.26 from there to 640.  128: 1.27-1.8 up to 256; to 416 0.96-1.40, 0.93-1.24 with fewer
//                       than 16 key tiles
//   gathering:          has the line of plain sparse, so that k and v gathered in place give the bits of the layout passes (beyond it 0.92-1.55 at 64
//                       and 1.03-1.24 at 128 with fewer than 16 key tiles)
//   32-row query tiles: a lone wavefront walks the list in attn_kernel, so its length decides.  Exact masks 1.0-2.1 up to 640 and 416.  With text rows or
//                       48 key tiles and more 0.96-2.2 up to 600 and 416.  Shorter ones: sparse at 128 1.08-1.8 up to 256, 0.87-1.01 beyond; at 64 1.0-1.5 up to 256, 0.97-1.02 beyond with
//                       fewer than 16 key tiles, 0.89-0.97 over 512; dense at 128 with fewer than 16 0.92-0.99 over 256, 1.02-1.13 with more
//   profiling:          1.0-3.0 up to 128 and 1.05-2.6 up to 72 workgroups per pass and part; 0.97 at 140, 0.91 at 168 and 96.  The K and V that
//                       they read between them count as well: at head dimension 64 64 x 118800 keys 1.16, but 77 x 34400 0.98, 90 x 29700 0.95,
//                       92 x 72500 0.81; at 128 48 x 118800 1.09 (28 x 54000 with 10 rows a head 0.97)
bool split_form(const Geo& g, int mode, int t) {
  const long long heads = (long long)g.B * g.H;
  const bool d64 = g.D == 64;
  if (mode != kProfile) {
    int most = d64 ? 640 : 416;
    if (g.bm == 128) {
      if (mode == kSparse || mode == kSparseGather) most = d64 ? 512 : g.nk < 16 ? 256 : 416;
    } else if (mode != kSparseExact) {
      const bool long_lists = g.T > 0 || g.nk >= 48, few_tiles = g.nk < 16;
      if (d64) most = long_lists ? 600 : mode == kSparse && few_tiles ? 256 : 512;
      else if (!long_lists && (mode == kSparse || few_tiles)) most = 256;
    }
    return heads * ((g.N + kRows - 1) / kRows) <= most;
  }
  const long long groups = heads * ((t + kRows - 1) / kRows);
  if (g.F > kMaxFrames || groups > (g.D == 64 ? 128 : 72)) return false;
  return groups <= (g.D == 64 ? 64 : 48) || groups * g.N <= (g.D == 64 ? 2400000 : 1600000);
}

bool split_sorts_rows(int t) { return t <= kSortRows; }

int launch_split(const Geo& g, AttnArgs a, int mode, hipStream_t stream) {
  unsigned grid;
  if (mode == kProfile) {
    a.nqt = (a.t + kRows - 1) / kRows;
    a.rows_per_group = (a.t + a.nqt - 1) / a.nqt;
    a.total = a.BH * a.nqt;
    grid = 8u * (unsigned)(a.plan.slots() * ((a.total + 7) / 8));
  } else {
    a.nqt = (a.N + kRows - 1) / kRows;
    a.total = a.BH * a.nqt;
    grid = 8u * (unsigned)((a.total + 7) / 8);
  }
  const bool wide = g.D == 128;
  switch (mode) {
    case kDense: return wide ? launch_split_one<128, kDense>(a, grid, stream) : launch_split_one<64, kDense>(a, grid, stream);
    case kSparse: return wide ? launch_split_one<128, kSparse>(a, grid, stream) : launch_split_one<64, kSparse>(a, grid, stream);
    case kSparseExact: return wide ? launch_split_one<128, kSparseExact>(a, grid, stream) : launch_split_one<64, kSparseExact>(a, grid, stream);
    case kSparseGather: return wide ? launch_split_one<128, kSparseGather>(a, grid, stream) : launch_split_one<64, kSparseGather>(a, grid, stream);
    default: return wide ? launch_split_one<128, kProfile>(a, grid, stream) : launch_split_one<64, kProfile>(a, grid, stream);
  }
}

}  // namespace attn

}  // namespace svg
