// Host side of the C ABI: argument validation, error strings, and the kept-tile
// list builder.  The tile list depends only on the geometry, so it is built on the
// host in closed form (interval arithmetic on frame / position groups) and the
// caller uploads it once per shape.
#include <algorithm>
#include <cmath>
#include <vector>

#include "svg_internal.h"

namespace svg {

static thread_local hipError_t g_last_hip_error = hipSuccess;
void note_hip_error(hipError_t e) { g_last_hip_error = e; }

// ---------------------------------------------------------------------------------------------
// Plan of the profiling passes (see ProfilePlan), from measurements on MI355X with 64 workgroups
// resident per XCD (96 at head dimension 64, where three fit a CU):
//  * Unmasked pass: four parts and two of half their length at the end, so that the workgroups
//    that finish last are short ones (1-3 % less time than eight equal parts; anything from
//    four to eight parts measured within 1 % of each other).  Fewer parts for short sequences,
//    and three when the sampled rows alone already give every XCD hundreds of workgroups.
//    Below 24 key tiles one part, except for few sampled rows at head dimension 128 where the masked
//    passes are cut: from 13 tiles and up to 64 rows three, and one part less of each masked pass (the same
//    workspace), because a workgroup walks its tiles one after the other and those of the unmasked pass are the
//    longest chain of the call.  Profiling of 2 to 24 heads, this cut against one part: 13 tiles 23.9 -> 22.1 us
//    (16 rows) and 28.0 -> 27.9 (64 rows), 15 tiles 26.8 -> 23.7 and 31.2 -> 29.9, 19 tiles 31.8 -> 28.1 and 36.4 -> 35.3,
//    23 tiles 36.1 -> 30.7 (16 rows); of all cases inside the line none more than 0.8 % slower.  Outside it the
//    shorter cut of the masked passes costs more than it gives: 128 rows 33.3 -> 35.5 us at 13 tiles and 42.5 -> 43.6
//    at 19; 8 tiles 26.3 -> 29.3 (100 rows); 11 tiles 25.8 -> 26.7 (64 rows); head dimension 64, with half the
//    products per tile, 12 tiles 22.6 -> 24.9 and 19 tiles 28.6 -> 32.3 (100 rows), 23.7 -> 24.3 (19 tiles, 16 rows).
//  * Masked passes: one part each, unless the (head, row group) pairs are so few that the two
//    masked workgroups per pair cannot fill an XCD; then as many parts (up to four) as keep
//    them within its resident places.  CogVideoX-v1 at 1 % (12 pairs per XCD): three parts,
//    -32 % time; 0.1 % of the rows at the 119k-token shape (3 pairs): four parts, 3.9 -> 1.3 ms;
//    with 15 or more pairs per XCD two parts of each of three passes are slower (566 -> 573 us at 40 heads of 32760 rows, 620 -> 639 at 48 of
//    45104, 2839 -> 2914 at 24 of 119056).
// ---------------------------------------------------------------------------------------------
namespace {

constexpr int kSlots = 64;            // workgroups resident on one XCD: 32 CUs x 2 (x 3 at D = 64)

void fill_bounds(ProfilePlan* p, int n_big, int n_small, int nk) {
  p->n_full = n_big + n_small;
  const int total = 2 * n_big + n_small;
  int cum = 0;
  for (int c = 0; c <= p->n_full; ++c) {
    p->full_bound[c] = (int)(((long long)nk * cum) / total);
    cum += c < n_big ? 2 : 1;
  }
  p->full_bound[p->n_full] = nk;
}

}  // namespace

ProfilePlan profile_plan(const Geo& g, int t) {
  const int groups = (t + g.bm - 1) / g.bm;
  const long long pairs = (long long)g.B * g.H * groups;
  const long long pairs_x = (pairs + 7) / 8;
  ProfilePlan plan = {};      // the error pass is built for 1, 3, 4 and 6 parts of the unmasked pass
  const int slots = g.D == 64 ? kSlots * 3 / 2 : kSlots;
  plan.n_masked = (int)std::max<long long>(1, std::min<long long>(kMaxMaskedParts, (slots - 8) / (2 * pairs_x)));
  if (g.nk >= 13 && g.nk < 24 && t <= 64 && plan.n_masked >= 3 && g.D == 128) {
    --plan.n_masked;
    fill_bounds(&plan, 3, 0, g.nk);
  } else if (g.nk < 24) fill_bounds(&plan, 1, 0, g.nk);
  else if (pairs_x >= 4 * kSlots) fill_bounds(&plan, 1, 2, g.nk);
  else if (g.nk < 96) fill_bounds(&plan, 2, 2, g.nk);
  else fill_bounds(&plan, 4, 2, g.nk);
  return plan;
}

// How a launch cuts the passes: as profile_plan says, which also sizes the workspace, or otherwise into no more parts in all.
//  * The split form (svg_split.hip) has four times the row groups, and a part that starts when another has ended lengthens the call by its
//    own time.  Where the plan's parts do not all find a place at once and four parts and three do, those are taken (from 96 groups on, at head
//    dimension 64, four and two); fewer than a tenth too many do no harm, the last parts are short ones.  Plan over cut, by groups of rows to an
//    XCD, 230 calls of 1-100 heads, 1600-55000 keys and 8-1200 rows: head dimension 128 three 1.00-1.31, four 0.80-1.03, five
//    0.81-1.08, six 0.88-1.26, median 1.06 (48 groups of 9086 rows 72.8 -> 61.4 us); 64 four to seven 0.80-1.07, median 0.93, nine 1.06-1.15,
//    ten 0.83-1.09, twelve 0.92-1.16.
//    Where the unmasked pass is not cut, three parts of each pass: 4 heads of 272 rows 9.5 -> 9.0, 24 of 820 12.9 -> 12.1.
// The general form keeps the plan's cut, or runs the unmasked pass in pieces (below).  (Three passes, eight parts of the unmasked pass and three of the masked ones for few heads with many
// groups of rows, whose windows are narrow only where the caller sorts the rows: 60 calls of 1-14 heads, 6200-120000 keys and 641-2400 rows
// ran at 0.76-1.08 of the plan's speed with rows in random order, median 0.80, and at 0.80-1.21 with sorted ones.)
ProfilePlan profile_cut(const Geo& g, int t, const ProfilePlan& plan, bool split) {
  if (!split || plan.n_masked != 4) return plan;
  ProfilePlan cut = plan;
  if (plan.n_full == 1) {
    cut.n_masked = 3;
    fill_bounds(&cut, 0, 3, g.nk);
    return cut;
  }
  const long long per_xcd = ((long long)g.B * g.H * ((t + 31) / 32) + 7) / 8;
  cut.n_masked = g.D == 64 && per_xcd >= 12 ? 2 : 3;
  fill_bounds(&cut, 0, 4, g.nk);
  auto helps = [&](int places) { return 10 * plan.slots() * per_xcd > 11 * places && cut.slots() * per_xcd <= places; };
  // all places of an XCD, or at head dimension 128, where two workgroups of a CU get in each other's way, one to a CU
  return helps(g.D == 64 ? kSlots * 3 / 2 : kSlots) || (g.D == 128 && helps(kSlots / 2)) ? cut : plan;
}

// The unmasked pass in pieces, for the general form.  What it saves is the spatial pass, about (2 w_s + 1 + frames of a group's rows) / F of
// an unmasked one, all of it where the caller's rows come in no order; what it costs is a visit of a few keys, and a piece's store, at every frame
// boundary where a window of the group ends.  Frames of at least four key tiles, and sequences from 24 tiles on, keep that small.  Profiling, three
// passes against pieces, rows in ascending and in random order: 48 heads of 17776 tokens at head dimension 64 186 -> 138 and 208 -> 139 us, 48 of
// 45104 636 -> 458 and 901 -> 462, at 128 40 of 32760 583 -> 427 and 856 -> 419, 24 of 119056 2865 -> 2558 and 4226 -> 2619, 3 of them
// 505 -> 450 and 762 -> 452.
//
// The parts of the two passes share the workspace of the plan, and an XCD's places.  Taken are as many temporal ones as make the estimated time the
// shortest: the longest chain of either pass, or the work of an XCD on all its places and, where the parts are more than the places, the last part behind
// it.  In units of the unmasked pass, whose last two parts have half the length of the others; a masked key tile counts 1.6, and a part more has to promise a tenth.
// 340 calls of 1-64 heads, 700-130000 keys and 16-1200 rows with one to four temporal parts: 0.7 % slower than with the best number at the mean, 13 % at the most (a tile of 1.2-1.8
// 0.8-1.5 %).  The plan's number, less one at head dimension 128 and one more at two numbers of groups, was 8-9 % and 60 % slower, and slower than three passes: up to 9 groups of rows
// to an XCD the temporal pass is the longest chain (30 heads of 9216 tokens and 92 rows with three, four parts 113 -> 90 us, 60 of 4914 and 49 97 -> 79; three
// passes 88 and 82).  239 calls in all, rows in order: the former numbers 0.62-1.39 times the time of three passes, 0.91 at the mean, these 0.57-1.07 and 0.83.
// Three passes where they are estimated 15 % shorter with the rows in order: where the workspace leaves the unmasked pass three parts or less (14 heads of 6000 tokens, 663 rows 1.12,
// 12 of 8100, 883 1.06; of the other calls five were 1-3 % slower in pieces than in three passes).
int profile_pieces(const Geo& g, int t, const ProfilePlan& plan, ProfilePlan* cut) {
  const int kept = g.T > 0 || g.sink ? 1 : 0;
  const int room = plan.slots() - 2 - kept;      // parts of both passes the workspace holds beside the two cuts and the kept keys
  if (g.nk < 24 || g.P < 4 * g.bn || room < 2) return 0;
  const int groups = (t + g.bm - 1) / g.bm;
  const double pairs_x = (double)(((long long)g.B * g.H * groups + 7) / 8), frames = g.F, positions = g.P;
  const double places = g.bm == 128 ? (g.D == 64 ? kSlots * 3 / 2 : kSlots) : (g.D == 64 ? 256 : 160);      // 32-row tiles: by LDS and registers
  const double kMaskedTile = 1.6;
  const int sides = std::min(2, groups - 1);      // of a group's rows on which other positions lie
  const double temporal = kMaskedTile * std::min(1.0, ((double)sides * g.w_t + g.bn + positions / groups) / positions);
  const double spatial = kMaskedTile * std::min(1.0, ((double)sides * g.w_s + 1 + frames / groups) / frames);
  auto small_parts = [](int n_full) { return n_full >= 3 ? 2 : 0; };
  auto longest_part = [&](int n_full) { return 2.0 / (2 * n_full - small_parts(n_full)); };
  *cut = plan;
  double shortest = 0;
  for (int nm = 1; nm <= kMaxMaskedParts && nm < room; ++nm) {
    const int nf = std::min(room - nm, kMaxPieces - 3);
    const double last = nf >= 3 ? longest_part(nf) / 2 : longest_part(nf);
    const double all = pairs_x * (1 + temporal) / places + (pairs_x * (nf + nm) > places ? last : 0);
    const double time = std::max({temporal / nm, longest_part(nf), all});
    if (nm > 1 && 1.1 * time >= shortest) continue;
    shortest = time;
    cut->n_masked = nm;
    fill_bounds(cut, nf - small_parts(nf), small_parts(nf), g.nk);
  }
  const double three = std::max({temporal / plan.n_masked, spatial / plan.n_masked, longest_part(plan.n_full),
                                 pairs_x * (1 + temporal + spatial) / places});
  return shortest > 1.15 * three ? 0 : cut->n_full + 2 + kept;
}

// A head's squared errors take one block per pass over its rows, and the sums of its blocks are added up in a fixed order: with up to
// kTicketBlocks blocks in all by the one that takes the last of the head's tickets, with more by a launch of its own.  A launch behind another costs
// a call 1-2 us.  A ticket costs an exchange with the memory behind the L2 caches, which slows the other blocks down: launch against tickets, whole calls,
// 4 blocks 18.6 -> 17.7 us and 17.1 -> 16.2, 24 blocks 21.9 -> 21.2, 40 25.2 -> 24.7, 60 78.7 -> 78.4; 76 349.8 -> 350.0, 82 70.3 -> 70.6 and 85.4 -> 85.8, 100 86.5 -> 87.1, 144
// 95.1 -> 96.4, 200 94.7 -> 96.8, 440 177.6 -> 184.8.
// Two passes in one block need neither.  The second costs what its rows and the parts to be merged cost, 0.5-2 us, and that is less than a ticket where it is three eighths full at most (24-58
// us, 46 calls: 0.4 us less, and 0-4 % of 1-32 heads with 2 rows in it; half full even, full 2-11 % more), with up to three
// parts of the unmasked pass (6 heads of 1200 rows 18.4 -> 17.8 us and 16.7 -> 16.0, 12 18.8 -> 18.6, 30 27.3 -> 26.9 and 21.9 -> 21.1; but four and four parts 12 heads 20.8 -> 21.9, 20
// 24.3 -> 25.7, six and four 29.5 -> 31.2), and less than a launch with all but the many outputs of pieces: 50 heads of 2400 rows 53.3 -> 52.0, 80 61.6 -> 58.9, 160 of 1200
// 52.7 -> 48.7, 180 of 4800 146.1 -> 142.9; in pieces 64 94.9 -> 95.6, 80 95.2 -> 96.3.
int error_blocks(const Geo& g, int t, const ProfilePlan& cut, int pieces) {
  const int passes = (t + err_rows(g.D) - 1) / err_rows(g.D);
  const bool nearly_one = 8 * (t - err_rows(g.D)) <= 3 * err_rows(g.D);
  const bool one_block = passes == 2 && !pieces && (cut.n_full <= 3 || nearly_one || 2ll * g.B * g.H > kTicketBlocks);
  return one_block ? 1 : passes;
}

int make_geo(const svg_shape_t* s, Geo* g) {
  if (!s) return SVG_ERR_INVALID_ARG;
  if (s->B <= 0 || s->H <= 0 || s->F <= 0 || s->P <= 0 || s->T < 0) return SVG_ERR_INVALID_ARG;
  if (s->w_s < 0 || s->w_t < 0) return SVG_ERR_INVALID_ARG;
  if (s->text_first != 0 && s->text_first != 1) return SVG_ERR_INVALID_ARG;
  if (s->sink_first_frame != 0 && s->sink_first_frame != 1) return SVG_ERR_INVALID_ARG;
  if (!(s->softmax_scale == s->softmax_scale) || std::isinf(s->softmax_scale)) return SVG_ERR_INVALID_ARG;
  if (s->D != 64 && s->D != 128) return SVG_ERR_UNSUPPORTED;
  const bool big = s->block_m == 128 && s->block_n == 64;
  const bool small = s->block_m == 32 && s->block_n == 32;
  if (!big && !small) return SVG_ERR_UNSUPPORTED;
  const int64_t n = (int64_t)s->F * s->P + s->T;
  // row indices, tile indices and B*H*nq must fit comfortably in int32
  if (n > (1 << 22)) return SVG_ERR_UNSUPPORTED;
  const int64_t nq = (n + s->block_m - 1) / s->block_m;
  if ((int64_t)s->B * s->H * nq > (int64_t)1 << 30) return SVG_ERR_UNSUPPORTED;
  g->B = s->B; g->H = s->H; g->F = s->F; g->P = s->P; g->T = s->T; g->D = s->D;
  g->N = (int)n;
  g->text_first = s->text_first;
  g->off = s->text_first ? s->T : 0;
  g->video_end = g->off + s->F * s->P;
  // (wider windows keep nothing more, and the kernels add a coordinate to the half-window in 32 bits)
  g->w_s = std::min(s->w_s, s->F); g->w_t = std::min(s->w_t, s->P); g->sink = s->sink_first_frame;
  g->bm = s->block_m; g->bn = s->block_n;
  g->nq = (int)nq;
  g->nk = (int)((n + s->block_n - 1) / s->block_n);
  g->scale = s->softmax_scale > 0.f ? s->softmax_scale : 1.0f / std::sqrt((float)s->D);
  return SVG_OK;
}

}  // namespace svg

using svg::Geo;

extern "C" {

const char* svg_strerror(int status) {
  switch (status) {
    case SVG_OK: return "ok";
    case SVG_ERR_INVALID_ARG: return "invalid argument";
    case SVG_ERR_UNSUPPORTED: return "unsupported head dimension, tile shape or size";
    case SVG_ERR_WORKSPACE: return "workspace missing or too small";
    case SVG_ERR_ALIAS: return "input and output overlap";
    case SVG_ERR_HIP: return "HIP runtime error";
    default: return "unknown status";
  }
}

const char* svg_version(void) { return "0.2"; }

const char* svg_last_hip_error(void) { return hipGetErrorString(svg::g_last_hip_error); }

size_t svg_workspace_bytes(const svg_shape_t* shape, int32_t t) {
  Geo g;
  if (svg::make_geo(shape, &g) != SVG_OK || t <= 0) return 0;
  const size_t a = svg::profile_workspace_bytes(g, t), b = svg::row_table_bytes(g);
  return a > b ? a : b;
}

int svg_profile_plan(const svg_shape_t* shape, int32_t t, int32_t* n_full, int32_t* n_masked,
                     int32_t* full_bound) {
  Geo g;
  int rc = svg::make_geo(shape, &g);
  if (rc != SVG_OK) return rc;
  if (t <= 0 || !n_full || !n_masked) return SVG_ERR_INVALID_ARG;
  const svg::ProfilePlan plan = svg::profile_plan(g, t);
  *n_full = plan.n_full;
  *n_masked = plan.n_masked;
  if (full_bound)
    for (int c = 0; c <= svg::kMaxProfileParts; ++c) full_bound[c] = plan.full_bound[c < plan.n_full ? c : plan.n_full];
  return SVG_OK;
}

int svg_tile_counts(const svg_shape_t* shape, int32_t* nq, int32_t* nk) {
  Geo g;
  int rc = svg::make_geo(shape, &g);
  if (rc != SVG_OK) return rc;
  if (!nq || !nk) return SVG_ERR_INVALID_ARG;
  *nq = g.nq;
  *nk = g.nk;
  return SVG_OK;
}

int svg_tile_list_build(const svg_shape_t* shape, int pattern, int32_t* row_ptr, int32_t* col_idx,
                        int64_t cap, int64_t* nnz_out) {
  Geo g;
  int rc = svg::make_geo(shape, &g);
  if (rc != SVG_OK) return rc;
  if (pattern != SVG_HEAD_SPATIAL && pattern != SVG_HEAD_TEMPORAL && pattern != SVG_LIST_TEMPORAL_FRAME_MAJOR)
    return SVG_ERR_INVALID_ARG;
  if (!row_ptr || !nnz_out || (col_idx && cap < 0)) return SVG_ERR_INVALID_ARG;
  const bool frame_major_temporal = pattern == SVG_LIST_TEMPORAL_FRAME_MAJOR;

  // In its own order a pattern groups `unit` consecutive video rows: a frame (P rows)
  // for spatial, a position (F rows) for temporal; `groups` of them; window w groups.
  const int unit = pattern == SVG_HEAD_SPATIAL ? g.P : g.F;
  const int groups = pattern == SVG_HEAD_SPATIAL ? g.F : g.P;
  const int w = pattern == SVG_HEAD_SPATIAL ? g.w_s : g.w_t;
  const int v0 = g.off, v1 = g.video_end;  // video rows [v0, v1)

  std::vector<uint8_t> keep(g.nk);
  // tiles kept by every video query: text keys, and frame-0 keys if the sink is on
  std::vector<uint8_t> always(g.nk, 0);
  auto mark = [&](std::vector<uint8_t>& m, int64_t lo, int64_t hi) {  // rows [lo, hi] inclusive
    if (lo > hi) return;
    for (int b = (int)(lo / g.bn); b <= (int)(hi / g.bn); ++b) m[b] = 1;
  };
  if (g.T > 0) {
    if (g.text_first) mark(always, 0, g.T - 1); else mark(always, v1, g.N - 1);
  }
  // first-frame sink: in every order frame 0 is the first P video rows (the transformed order of a
  // temporal head keeps it as a block in front, see transformed_to_token)
  if (g.sink) mark(always, v0, v0 + g.P - 1);
  const bool sink_temporal = g.sink && pattern == SVG_HEAD_TEMPORAL;

  int64_t nnz = 0;
  bool overflow = false;
  row_ptr[0] = 0;
  for (int a = 0; a < g.nq; ++a) {
    const int64_t r0 = (int64_t)a * g.bm;
    const int64_t r1 = std::min<int64_t>(r0 + g.bm, g.N) - 1;
    const bool has_text_query = g.T > 0 && (r0 < v0 || r1 >= v1);
    if (has_text_query) {
      std::fill(keep.begin(), keep.end(), (uint8_t)1);
    } else if (frame_major_temporal) {
      // Rows r0..r1 in F-outer order cover the in-frame positions [pa, pb] of one frame, or
      // wrap over a frame end ([pa, P) and [0, pb]), or every position; each position
      // interval keeps, in EVERY frame, the keys within w_t positions of it.
      keep = always;
      const int64_t pa = (r0 - v0) % g.P, pb = (r1 - v0) % g.P;
      const bool one_frame = (r0 - v0) / g.P == (r1 - v0) / g.P;
      auto keep_positions = [&](int64_t lo, int64_t hi) {
        lo = std::max<int64_t>(0, lo - g.w_t);
        hi = std::min<int64_t>(g.P - 1, hi + g.w_t);
        for (int f = 0; f < g.F; ++f) mark(keep, v0 + (int64_t)f * g.P + lo, v0 + (int64_t)f * g.P + hi);
      };
      if (one_frame) {
        keep_positions(pa, pb);
      } else if (r1 - r0 + 1 >= g.P) {
        keep_positions(0, g.P - 1);
      } else {
        keep_positions(pa, g.P - 1);
        keep_positions(0, pb);
      }
    } else if (sink_temporal) {
      // Transformed order with the sink: rows [v0, v0 + P) are frame 0 in position order, rows from
      // b0 = v0 + P on hold positions outer over the other F - 1 frames.  Frame-0 keys are kept
      // anyway; of the others a query at position p keeps the positions within w_t of it.  The
      // tile's rows may lie in either part or in both.
      keep = always;
      const int64_t b0 = v0 + g.P, rest = g.F - 1;
      auto keep_positions = [&](int64_t lo, int64_t hi) {
        if (rest <= 0) return;
        lo = std::max<int64_t>(0, lo - g.w_t);
        hi = std::min<int64_t>(g.P - 1, hi + g.w_t);
        mark(keep, b0 + lo * rest, b0 + (hi + 1) * rest - 1);
      };
      if (r0 < b0) keep_positions(r0 - v0, std::min<int64_t>(r1, b0 - 1) - v0);
      if (r1 >= b0 && rest > 0) keep_positions((std::max<int64_t>(r0, b0) - b0) / rest, (r1 - b0) / rest);
    } else {
      keep = always;
      const int64_t ga = (r0 - v0) / unit, gb = (r1 - v0) / unit;
      const int64_t lo = v0 + std::max<int64_t>(0, ga - w) * unit;
      const int64_t hi = v0 + std::min<int64_t>(groups, gb + w + 1) * unit - 1;
      mark(keep, lo, hi);
    }
    for (int b = 0; b < g.nk; ++b) {
      if (!keep[b]) continue;
      if (col_idx) {
        if (nnz < cap) col_idx[nnz] = b; else overflow = true;
      }
      ++nnz;
    }
    if (nnz > INT32_MAX) return SVG_ERR_UNSUPPORTED;
    row_ptr[a + 1] = (int32_t)nnz;
  }
  *nnz_out = nnz;
  return overflow ? SVG_ERR_INVALID_ARG : SVG_OK;
}

}  // extern "C"
