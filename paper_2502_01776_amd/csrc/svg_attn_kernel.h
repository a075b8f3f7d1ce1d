// FlashAttention-style forward kernels for gfx950 (MI355X): dense attention, the
// block-sparse pass over a kept-tile list (Sec. 4.3), and the masked passes of online
// profiling over sampled query rows (Alg. 1, Sec. 4.1).
//
// One workgroup owns one query tile of one head; each of its NW wavefronts owns 32
// query rows and all BN keys of the current key tile.  Both matrix products are
// computed TRANSPOSED with v_mfma_f32_16x16x32_bf16, every LDS operand feeding two products,
// one per 16-query block of the wavefront:
//     S^T = K Q^T      (A = K tile from LDS,  B = Q^T held in registers)
//     O^T += V^T P^T   (A = V^T from LDS,     B = P^T taken from S^T's registers)
// In the 16x16 accumulator layout a lane holds ONE query column (lane % 16) and the key rows
// 4 g + {0..3}, g = lane / 16, so the softmax row statistics are per-lane register reductions
// plus an exchange among lanes l, l ^ 16, l ^ 32, l ^ 48 where one is needed at all, the rescale
// factor is one scalar per lane and query block, and the exponentiated S^T registers of two
// 16-key blocks are, after bf16 packing, exactly the B operand of the second product: its
// k-slots 8 g + {0..7} hold keys {4 g + j} and {16 + 4 g + j}, j < 4, of a 32-key step, and the
// V^T operand is read in the same key order, so P never moves between lanes or through LDS.
//
// Why 16x16x32 and not 32x32x16: the chip is power-limited here, and the smaller form moves
// half the accumulator traffic per operation.  Loops of the kernel's instruction mix measured
// 2093 against 1788 TFLOP/s (products only) and 1419 against 1364 (with one 1 KB operand
// read per 32768 operations and the softmax).
//
// The loop is skewed by one tile: with the scores of tile j in registers a wavefront takes their
// exponentials, one run of VALU work, and then issues the products of tile j + 1's scores and of tile
// j's output as one batch, one run of matrix work.  The first operands of a batch are read from LDS before
// the exponentials, every other one behind the products, and no wavefront waits for the results of
// the products it has just issued.  (Taken tile by tile, scores, exponentials, output: dense 18.33 ms instead of
// 17.65 at 40 heads of 32760 tokens, profiling 2.99 instead of 2.84 at the 119k-token shape, the sparse
// pass 5.45 instead of 5.12 at head dimension 64 and 45k tokens, and no difference at head
// dimension 128.)  The masked passes still take their tiles one by one: see the main loop.
//
// Staging: K and V tiles go from memory straight into LDS (buffer_load_dwordx4 ... lds, bounds-checked
// descriptors, loop-invariant offsets), two buffers each, with the loads of K of tile j + 2 and V of j + 1
// in flight during trip j and one barrier per trip.  Such a load writes 64 x 16 consecutive
// bytes, so rows cannot be padded; the bank swizzles are applied on the memory side (a lane
// fetches the piece of its row that belongs at its place).  V stays row-major too: the transposing
// LDS read of gfx950 (ds_read_b64_tr_b16) hands a lane the same channel of four consecutive
// keys, so two of them are a whole A operand of the second product and nothing is
// transposed in registers.  (Loads that always hit L2 make the dense pass 1 % faster, no loads at all 12 %:
// it is the moving of the bytes into LDS that costs, not their latency.)
// (With the tiles staged through registers and ds_write_b128, and 32x32x16 products, the sparse pass
// took 24.5 ms instead of 22.3 at the 119k-token shape with 15 % of the tiles kept, 3.22
// instead of 2.89 ms at 40 heads of 32760 tokens, 4.08 instead of 3.69 ms at head dimension 64, and
// the dense pass 19.7 instead of 17.9 ms; the LDS writes alone occupied the LDS a quarter of the
// time, and the 32 staging registers now hold operands.)
//
// Softmax: fp32, base-2 exponentials with scale * log2 e folded into one FMA per
// element.  The exponentials are taken against the current reference maximum without
// looking at the tile's own maximum; only when a row sum shows that the reference is
// too small does the wave fall back to the classic update (tile maximum, rescale).
// P is rounded to bf16 for the second product; accumulation is fp32; the running sum
// uses the unrounded P at head dimension 128 and the rounded P at head dimension 64.
//
// Measured on MI355X:
//  * With 32 query rows per wavefront every 32768 operations need a fresh 1 KB operand from LDS.
//  * The chip is power-limited under this load: the shader clock sits near 1.9 GHz (2.4 GHz
//    nominal), and a loop of nothing but MFMAs on random operands is held there too.  A
//    variant that idles more runs at a higher clock and ends up at the same rate; what
//    pays is less work per tile (instructions, LDS and memory traffic), not fewer cycles.
//  * A lone wavefront hides few cycles of other instructions behind its own
//    MFMAs; two wavefronts on a SIMD overlap one's VALU work with the other's
//    products much better, and best when each runs long homogeneous phases (products /
//    softmax) and the one issuing products has the higher wave priority.  Interleaving
//    softmax slices between the products of the same wavefront was 10 % slower.
//  * 64 query rows per wavefront (every LDS operand feeding twice as many products) needs more than
//    the 256 registers a wavefront has at two per SIMD; with one wavefront per SIMD it
//    loses the overlap above and was 5 % slower.  A 256-row workgroup (two query tiles
//    sharing every staged tile, the two halves one phase apart) halved staging and L2
//    traffic per product and came out even: more cycles at a higher clock.
#pragma once
#include <type_traits>

#include "svg_split.h"

namespace svg {

namespace {

using namespace attn;

// Wave priority while a wavefront issues products (0 elsewhere).  The two
// wavefronts sharing a SIMD then settle into opposite phases: the products of one run
// back to back while the other's softmax and staging instructions fill the gaps.  Where a tile is
// taken in one go, its first product ranks above its second (1 % less time than equal ranks, 1 % more with the
// ranks swapped): a wavefront that starts a tile is not held up by one that finishes one.
constexpr int kPrioOutput = 1;
constexpr int prio_scores(bool sequential) { return sequential ? 2 : 1; }
// Dense: the most consecutive query tiles that share an XCD (and its L2) at a time.  Fewer where 64 would not deal the XCDs equal
// numbers of tiles (dense_cohort): 186 tiles in 64s use three of the eight XCDs.  Blocks of 64 against equal ones: 186 tiles of 6 heads
// 114.6 -> 78.9 us at head dimension 128 and 64.3 -> 51.0 at 64, 256 116.9 -> 84.8 and 67.0 -> 55.3, 384 169 -> 148 and 96.7 -> 93.1, 576
// 393 -> 360 and 244 -> 191, 768 650 -> 540 and 390 -> 300, 2112 1029 -> 1007 and 592 -> 552; multiples of 512 have blocks of 64 as before.
constexpr int kCohort = 64;
// LDS operands kept in flight ahead of the products: twelve where the registers allow it (the
// unmasked passes at head dimension 128; 1.2 % less time than eight, 0.9 % than six), eight in the
// forms with mask state or row numbers in registers, four at head dimension 64 (three to six measured within 1 %)
constexpr int prefetch_depth(int D, int NW, int MODE) {
  return D != 128 || NW != 4 ? 4 : MODE == kDense || MODE == kSparse ? 12 : 8;
}
// Wavefronts per SIMD the register budget is set for.  Head dimension 128 fills 256 registers
// (two wavefronts).  At head dimension 64 the accumulators are half as large and every form fits
// 168 registers: three workgroups per CU, whose wavefronts cover each other's softmax phases
// (the longer phase at this head dimension) better than two workgroups with twice the keys per
// barrier did (4-7 % less time in the dense and sparse passes, 14 % in profiling).
// The 32-row form is a single wavefront, and asking for two per SIMD keeps it inside 256 registers: with more
// allowed (one per SIMD, or LDS for four workgroups on the CU's four SIMDs) the compiler puts every accumulator
// into the second half of the register file and moves it to the first and back around the softmax, 144 of 480
// instructions of a tile at head dimension 64 and 240 of 679 at 128: 12 heads of 1410 rows dense 36.8 -> 28.1 and
// 53.7 -> 42.3 us, sparse 35.2 -> 28.3 and 53.0 -> 40.0.
constexpr int waves_per_simd(int D, int NW, int MODE) {
  return NW != 4 ? 2 : D == 64 ? 3 : 2;
}

// TEAMS: one, or two teams of NW wavefronts that share the query tile and take its key tiles in turn (svg_teams.hip)
// PIECED: profiling with the unmasked pass in pieces (PieceRule) and no spatial pass.  A kernel of its own: as a flag in the profiling kernel
// the pieces cost the calls that run three passes 24 more spilled scalars in all loops (20 in the 32-row form, which had none): 60 heads of 4800 rows in 32-row
// tiles 188 us as one kernel, 184 as two, 70 heads of 17500 rows 281 and 279, and calls in pieces, whose kernel has no spatial pass, 123 and 120 (cogvideox_v1), 426 and 418 (cogvideox_v15).
template <int D, int NW, int BN, int MODE, int LW, int TEAMS = 1, bool PIECED = false>
__global__ __launch_bounds__(64 * NW * TEAMS, TEAMS > 1 ? TEAMS : waves_per_simd(D, NW, MODE)) void attn_kernel(AttnArgs a) {
  constexpr int BM = 32 * NW;            // query rows per workgroup = rows of a query tile
  constexpr int THREADS = 64 * NW;       // of a team
  constexpr int CPR = D / 8;             // 16-byte pieces per row
  constexpr int QB = 2;                  // 16-query blocks per wavefront
  constexpr int KB = BN / 16;            // 16-key blocks per tile
  constexpr int KS = BN / 32;            // 32-key steps of the second product
  // kSparseExact is kSparse with the head's element mask applied inside every visited tile
  // kSparseGather is kSparse with k and v of the temporal heads left in token order: the rows of
  // a key tile are fetched from where the layout transformation would have taken them
  constexpr bool SPARSE = MODE == kSparse || MODE == kSparseExact || MODE == kSparseGather;
  constexpr bool GATHER = MODE == kSparseGather;
  static_assert(!GATHER || NW == 4, "the gathering form exists for 128-row query tiles");
  constexpr bool MASKABLE = MODE == kProfile || MODE == kSparseExact;
  constexpr int DS = D / 32;             // 32-channel steps of the first product
  constexpr int CB = D / 16;             // 16-channel blocks of O^T
  constexpr int PIECES = BN * CPR;       // 16-byte pieces of a K tile, and of a V tile
  // Staging work: every thread requests PER_THREAD pieces of K and of V,
  // so all wavefronts reach the barrier with the same amount of work behind them.
  constexpr int PER_THREAD = PIECES / THREADS;
  static_assert(PER_THREAD % 2 == 0, "the direct loads come in pairs");
  static_assert(PIECES % THREADS == 0 && THREADS % CPR == 0, "every thread stages the same piece of whole rows");
  // K staging: row-major, the 16-byte pieces of a row XOR-swizzled with the row number (k_swizzle),
  // which puts the same piece of 16 consecutive keys, what 16 lanes of an A operand read, on
  // different banks.
  constexpr int K_ROW = D * 2;
  constexpr int K_BYTES = BN * K_ROW;
  // V staging: row-major as well, not transposed.  The A operand of the second product is V^T,
  // which the transposing LDS read of gfx950 (ds_read_b64_tr_b16) delivers directly: the 16
  // lanes of a quarter wavefront read 4 rows x 16 channels (lane s: 8 bytes of row s / 4 at
  // channel 4 (s % 4)) and lane i receives channel i of the four rows.  Two such reads (rows
  // 4 q + {0..3} and 16 + 4 q + {0..3} of a 32-key step, q = lane / 16) are one operand in the key
  // order the weights are held in.  The 32-byte slots of a row are XOR-swizzled with the row number
  // (v_swizzle), so that the same slot of the eight rows a half wavefront reads falls on different
  // banks.
  constexpr int V_ROW = D * 2;
  constexpr int V_BYTES = BN * V_ROW;
  constexpr int STAGE_BYTES = K_BYTES + V_BYTES;

  // Two K tiles and two V tiles per team, and nothing else: with 8 bytes
  // more the 32-row form at head dimension 128 fits a CU four times, not five (see waves_per_simd).
  static_assert(2 * STAGE_BYTES <= 65536, "two workgroups, or the two teams of one, fit a CU");
  static_assert(!SPARSE || NW != 4 || split_lds_bytes(D) <= 2 * STAGE_BYTES, "text-row tiles in parts merge in the same LDS");
  static_assert(TEAMS == 1 || (TEAMS == 2 && NW == 4 && MODE != kProfile), "two teams take the general passes over 128-row query tiles");
  __shared__ __attribute__((aligned(1024))) unsigned char all_lds[TEAMS * 2 * STAGE_BYTES];
  // A loop of four- and eight-byte instructions runs at a rate of its own from each of the two places it can begin at in a group of eight bytes: which of them are cut by the
  // lines the instructions come in.  Most forms do not notice, these lose up to 8 % where it begins on a multiple of eight, with few workgroups to a CU above all (gathering at head
  // dimension 64, one head of 42210 rows 132.9 us and 122.9, 24 of 1960 37.2 and 35.7; exact masks 18 of 6960 98.5 and 96.5; 32-row tiles, 8 heads of 16842 502 and 494), so four
  // bytes are put in front of theirs.  Where it begins is in a test: more or less code in front turns it round.
  if constexpr (TEAMS == 1 && LW == 1 && ((D == 64 && NW == 4 && (MODE == kSparseGather || MODE == kSparseExact)) || (D == 128 && NW == 1 && MODE == kSparse)))
    asm volatile("s_nop 0");
  const int team = TEAMS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / THREADS);
  unsigned char* const lds = all_lds + team * 2 * STAGE_BYTES;

  // ======================================================================================
  // Which (head, row group) is this workgroup?  Consecutive logical ids are placed on the
  // same XCD (workgroups are dealt round-robin over the 8 XCDs), so the query tiles that
  // stream the same K/V share one L2.
  // ======================================================================================
  const int xcd = blockIdx.x & 7, loc = blockIdx.x >> 3;
  int bh = 0, grp = 0, variant = 0, chunk = 0;
  if (MODE == kProfile) {
    // (head, row group) pairs are split into 8 contiguous chunks, one per XCD.  Each pair
    // has 2 n_masked + n_full units, or n_masked + n_full in pieces: the parts of the spatial pass, of the temporal pass (both
    // skip most key tiles) and of the unmasked pass.  Units are the outer index inside an
    // XCD's chunk, so neighbouring workgroups stream the same keys for neighbouring row
    // groups of one head.
    const int pairs = a.BH * a.nqt;
    const int pairs_per_xcd = (pairs + 7) >> 3;
    const int unit = loc / pairs_per_xcd;
    const int pair = xcd * pairs_per_xcd + (loc - unit * pairs_per_xcd);
    const int nm = a.plan.n_masked, ns = PIECED ? 0 : nm;      // parts of the temporal and of the spatial pass
    clear_tickets<THREADS * TEAMS>(a);
    if (unit >= ns + nm + a.plan.n_full || pair >= pairs) return;
    // the masked passes first: their workgroups are the longest ones (mask work on top of
    // about as many tiles), so they should not be the last to start
    variant = !PIECED && unit < ns ? 1 : unit < ns + nm ? 2 : 0;         // 0 unmasked, 1 spatial, 2 temporal
    chunk = unit < ns ? unit : unit < ns + nm ? unit - ns : unit - ns - nm;    // which part of its pass
    bh = pair / a.nqt;
    grp = pair - bh * a.nqt;
  } else if (MODE == kDense) {
    // Dense: blocks of up to kCohort consecutive logical ids go to one XCD, consecutive blocks to
    // consecutive XCDs.  An XCD's L2 serves neighbouring query tiles of one head, and at
    // any time all XCDs work on the same one or two heads, whose K/V (61 MB per head at
    // the 120k-token shape) then stay in the memory-side cache in front of HBM; with one
    // head per XCD the dense pass runs into the HBM bandwidth (-11 % time).
    const int lid = ((loc / a.cohort) * 8 + xcd) * a.cohort + (loc % a.cohort);
    if (lid >= a.total) return;
    bh = lid / a.nqt;
    grp = lid - bh * a.nqt;
  }
  // sparse: heavy tiles first, then an eighth of each label's sequence of tiles
  int pat = 0, cl = -1, head_cl0 = 0;
  if (SPARSE) {
    int part;
    if (!sparse_slot<LW, TEAMS>(a.so, a.BH, a.labels, a.row_ptr[0], a.row_ptr[1], xcd, loc, bh, grp, pat, cl, head_cl0, part)) return;
    bh = __builtin_amdgcn_readfirstlane(bh);
    grp = __builtin_amdgcn_readfirstlane(grp);
    pat = __builtin_amdgcn_readfirstlane(pat);
    if constexpr (NW == 4) {
      if (__builtin_amdgcn_readfirstlane(part) >= 0) {
        const int row0 = grp * BM + __builtin_amdgcn_readfirstlane(part) * 32;
        if (row0 >= a.N || team > 0) return;
        const int32_t* rp = a.row_ptr[pat];
        split_body<D, MODE>(a, lds, bh, row0, grp, pat, __builtin_amdgcn_readfirstlane(rp[grp]), __builtin_amdgcn_readfirstlane(rp[grp + 1]), 0, 0);
        return;
      }
    }
  }

  // profile: the unmasked pass needs no key codes, tile summaries or element masks (only the
  // ragged end of the sequence, handled like in the dense pass)
  const bool masked = MODE == kSparseExact || (MODE == kProfile && __builtin_amdgcn_readfirstlane(variant) != 0);

  const int tid = TEAMS == 1 ? threadIdx.x : threadIdx.x & (THREADS - 1);      // in the team
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int g = lane >> 4;       // which quarter of the wavefront
  const int r = lane & 15;       // query column within a 16-query block / row of the A operand

  const size_t head = (size_t)bh * a.N;

  // ======================================================================================
  // This lane's query rows (one per 16-query block), their mask windows, and Q^T as the B operand.
  // ======================================================================================
  int qslot[QB], qrow[QB];       // row (profile: index into rows[])
  // Profile: the sampled rows are dealt evenly to the row groups, rows_per_group each or (0) in 32s.  A wavefront without rows stages its
  // share of the tiles and computes nothing; in pieces which of a workgroup's it is changes from one to the next, so that no SIMD has them
  // all (in three passes 0.5-2 % slower).  A lane without a row of its own shadows the group's first row and writes nothing.
  const int n32 = (a.t + 31) / 32, per_group = MODE == kProfile ? n32 / a.nqt : 0, one_more = n32 - per_group * a.nqt;
  const int row0 = a.rows_per_group ? min(grp * a.rows_per_group, a.t - 1) : 32 * (grp * per_group + min(grp, one_more));
  const int row1 = min(row0 + (a.rows_per_group ? a.rows_per_group : 32 * (per_group + (grp < one_more ? 1 : 0))), a.t);
  const int own32 = PIECED ? (wave + loc) & (NW - 1) : wave;
  const bool active = MODE != kProfile || __builtin_amdgcn_readfirstlane(row0 + own32 * 32) < row1;
  if (MODE == kProfile) {
    int slot[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      qslot[qb] = row0 + own32 * 32 + qb * 16 + r;
      qslot[qb] = qslot[qb] < row1 ? qslot[qb] : a.t;
      slot[qb] = qslot[qb] < a.t ? qslot[qb] : row0;
    }
    // The temporal variant takes the sampled rows grouped by in-frame position, so that
    // a workgroup's rows share a narrow position range and most key tiles can be
    // skipped; results are still written at the row's own slot.
    if (variant == 2) {
      const int32_t* order = a.order_t;
      if (order == nullptr) {
        // as many rows as threads at most: the workgroup sorts them itself, each row counting
        // the rows in front of it, in the order profile_order_kernel would give them.  With 130 to 256 rows that takes 7-9 us
        // of the workgroups of this pass and saves a launch of 6-7 us in front of all of them: 26 calls of 12-200 heads (the
        // 32-row form with 40-64 rows) 0.99-1.07 times as fast as with the launch, 22 of them faster (48 heads of 17776 tokens
        // and 178 rows at head dimension 64 184.8 -> 178.3 us)
        int* const bin = reinterpret_cast<int*>(lds);
        int* const sorted = bin + THREADS;
        if (tid < a.t) bin[tid] = order_bin(a.rows[tid], a.off, a.video_end, a.P);
        __syncthreads();
        if (tid < a.t) {
          const int own = bin[tid];
          int rank = 0;
#pragma unroll 8
          for (int j = 0; j < a.t; ++j) rank += bin[j] < own || (bin[j] == own && j < tid);
          sorted[rank] = tid;
        }
        __syncthreads();
        slot[0] = sorted[slot[0]];
        slot[1] = sorted[slot[1]];
        // The first tile is staged over the list.  In the one-wavefront form the barrier is nothing, and a direct
        // load is not ordered behind LDS reads: the statement has them answered.
        asm volatile("" ::"v"(slot[0]), "v"(slot[1]) : "memory");
        __syncthreads();
      } else {
        slot[0] = order[slot[0]];
        slot[1] = order[slot[1]];
      }
    }
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      if (qslot[qb] < a.t) qslot[qb] = slot[qb];
      qrow[qb] = a.rows[slot[qb]];
    }
  } else {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      qslot[qb] = grp * BM + wave * 32 + qb * 16 + r;
      qrow[qb] = min(qslot[qb], a.N - 1);
    }
  }

  // Element masks.  In the order the keys are read in, a row keeps one run of keys beside those every
  // row keeps (rows below keep_head: text prefix and first-frame sink; rows from video_end on:
  // text suffix): [win_lo, win_hi) in key rows, because both patterns group consecutive rows, frames
  // (P rows) for a spatial head, positions (F rows, F - 1 behind the sink block) for a temporal
  // head in P-outer order.  Only the temporal profiling pass, which reads the keys in F-outer order,
  // has such a run in every frame: there the window is in in-frame positions.
  const int keep_head = a.sink ? a.off + a.P : a.off;
  const bool by_position = MODE == kProfile && variant == 2;
  int win_lo[QB], win_hi[QB];
  auto row_window = [&](int c, int groups, int w, int base, int unit, int& lo, int& hi) {
    w = min(w, groups);
    lo = base + max(0, c - w) * unit;
    hi = base + min(groups, c + w + 1) * unit;
  };
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {      // a text query keeps everything
    win_lo[qb] = 0;
    win_hi[qb] = by_position ? a.P : a.N;
  }
  // Unmasked pass in pieces (PieceRule): the frames of a lane's rows, and of two of the workgroup's rows per lane, from which every
  // wavefront finds the next key at which a piece of any of them ends.  Two to a register (P is at least 128, so frame numbers stay below 2^15), as the
  // register budget is full; -1: a text row, which has no part in the errors.
  const bool pieces = PIECED && variant == 0;
  const PieceRule rule = {a.off, a.video_end, keep_head, a.F, a.P, a.w_s};
  int own_frames = -1, cut_frames = -1;
  if (pieces) {
    auto frame = [&](int n) { return n >= a.off && n < a.video_end ? (n - a.off) / a.P : -1; };
    auto group_row = [&](int i) { return a.rows[min(row0 + i, row1 - 1)]; };
    own_frames = (frame(qrow[0]) & 0xffff) | (frame(qrow[1]) << 16);
    cut_frames = (frame(group_row(lane)) & 0xffff) | (frame(group_row(lane + 64)) << 16);
  }
  // keeps what is worked out from the value at the rare place that needs it, out of the registers of the loop
  auto opaque = [](int x) -> int {
    asm volatile("" : "+v"(x));
    return x;
  };
  auto frame_of = [](int frames, int i) { return i ? frames >> 16 : (int)(short)frames; };
  int c_lo = 0x7fffffff, c_hi = -1;      // profile: smallest and largest coordinate of the workgroup's rows
  if (MODE == kProfile && masked) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
      if (qrow[qb] >= a.off && qrow[qb] < a.video_end) {
        const int vq = qrow[qb] - a.off;
        const int fq = vq / a.P;
        const int c = variant == 1 ? fq : vq - fq * a.P;
        if (variant == 1) row_window(c, a.F, a.w_s, a.off, a.P, win_lo[qb], win_hi[qb]);
        else row_window(c, a.P, a.w_t, 0, 1, win_lo[qb], win_hi[qb]);
        c_lo = min(c_lo, c);
        c_hi = max(c_hi, c);
      }
    // (a text query attends to everything under both masks, so its masked outputs equal
    // the unmasked one by definition: it adds nothing to either error, the error kernel
    // skips it, and it need not widen this workgroup's key range)
    // reduced inside the wavefronts first: LDS atomics of all 64 lanes on one address are expanded into
    // a loop over the lanes, 1 us per atomic at the start of every workgroup
    int* const wave_range = reinterpret_cast<int*>(lds);      // smallest and largest coordinate of each wavefront's rows
    wave_range[2 * wave] = quad_rows_min(c_lo);
    wave_range[2 * wave + 1] = -quad_rows_min(-c_hi);
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      c_lo = min(c_lo, wave_range[2 * w]);
      c_hi = max(c_hi, wave_range[2 * w + 1]);
    }
    c_lo = __builtin_amdgcn_readfirstlane(c_lo);
    c_hi = __builtin_amdgcn_readfirstlane(c_hi);
    asm volatile("" ::"s"(c_lo), "s"(c_hi) : "memory");      // the reads are answered: the first tile is staged over them
    __syncthreads();
  }

  // sparse: this head's pattern; with q and o kept in token order, the row of a temporal
  // head that this lane reads and writes is the token whose transformed position is qrow
  // (Sec. 4.2: position off + p F + f holds token off + f P + p; with the first-frame sink,
  // frame 0 leads as a block)
  // a temporal head reads the P-outer copies of k and v when the caller keeps them apart from
  // the originals (which the spatial heads read in place)
  const bool kv_copy = SPARSE && __builtin_amdgcn_readfirstlane(pat) != 0 && a.k_t != nullptr;
  const __bf16* kh = (kv_copy ? a.k_t : a.k) + head * D;
  const __bf16* vh = (kv_copy ? a.v_t : a.v) + head * D;
  int io_row[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const int n = qrow[qb];
    const bool video = n >= a.off && n < a.video_end;
    io_row[qb] = n;
    if (SPARSE && a.qo_token_order && pat && video)
      io_row[qb] = a.off + (int)transformed_to_token((unsigned)(n - a.off), (unsigned)a.F, (unsigned)a.P, a.sink);
    if (MODE == kSparseExact && video) {
      // the window of the head's pattern in the order its tile list refers to
      if (pat) {
        unsigned pq;
        transformed_to_token((unsigned)(n - a.off), (unsigned)a.F, (unsigned)a.P, a.sink, &pq);
        row_window((int)pq, a.P, a.w_t, keep_head, a.sink ? a.F - 1 : a.F, win_lo[qb], win_hi[qb]);
      } else {
        row_window((n - a.off) / a.P, a.F, a.w_s, a.off, a.P, win_lo[qb], win_hi[qb]);
      }
    }
  }

  // smallest and largest window bounds over the video rows of the wavefront: most tiles lie inside every
  // such row's window or outside all of them, which these decide without a look at the rows
  int lo_min = 0, lo_max = 0, hi_min = 0, hi_max = 0;
  bool video[QB] = {}, has_text = false;
  if (MASKABLE) {
    int lo[2] = {0x7fffffff, 0x7fffffff}, hi[2] = {0x7fffffff, 0x7fffffff};      // smallest, smallest negative
    bool text = false;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      video[qb] = qrow[qb] >= a.off && qrow[qb] < a.video_end;
      text = text || !video[qb];
      if (video[qb]) {
        lo[0] = min(lo[0], win_lo[qb]);
        lo[1] = min(lo[1], -win_lo[qb]);
        hi[0] = min(hi[0], win_hi[qb]);
        hi[1] = min(hi[1], -win_hi[qb]);
      }
    }
    lo_min = quad_rows_min(lo[0]);
    lo_max = -quad_rows_min(lo[1]);
    hi_min = quad_rows_min(hi[0]);
    hi_max = -quad_rows_min(hi[1]);
    has_text = __builtin_amdgcn_ballot_w64(text) != 0;
  }

  bf16x8 qreg[QB][DS];     // lane (g, r) holds Q[row 16 qb + r][32 s + 8 g .. +8]
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const __bf16* qp = a.q + (head + io_row[qb]) * D + g * 8;
#pragma unroll
    for (int s = 0; s < DS; ++s) qreg[qb][s] = *reinterpret_cast<const bf16x8*>(qp + s * 32);
  }

  // ======================================================================================
  // Tile cursor: the next key tile of this workgroup, or kNoTile.
  //   dense   : 0 .. nk-1
  //   sparse  : the query tile's row of the head's CSR list
  //   profile : tiles of the key intervals that can hold a kept key for ANY row of the
  //             workgroup, ascending: text prefix | frame 0 (sink) | the window around the
  //             rows' frames (spatial) or, per frame, the window around the rows' positions
  //             (temporal) | text suffix; the unmasked pass walks its key range.  A superset
  //             is enough: the element mask is still applied inside every visited tile.
  // ======================================================================================
  TileList list = {};                // sparse
  int lj = team, l_end = 0;          // dense: counter; profile, unmasked pass: counter and end of the tiles of part chunk
  if (MODE == kProfile && !PIECED && variant == 0) {
    lj = a.plan.full_bound[chunk];
    l_end = a.plan.full_bound[chunk + 1];
  }
  int n_tiles = a.nk;                // two teams: tiles of the workgroup
  if (SPARSE) {
    const int32_t* rp = a.row_ptr[pat];
    const int lbeg = __builtin_amdgcn_readfirstlane(rp[grp]), lend = __builtin_amdgcn_readfirstlane(rp[grp + 1]);
    n_tiles = lend - lbeg;
    list.open(a.col_idx[pat] + lbeg, n_tiles, 0, TEAMS, team);
    // The list is walked from its first entry.  Neighbouring query tiles run at the same time on
    // one XCD with key windows shifted by BM / BN tiles against each other, so each finds in L2
    // what its neighbour fetched a moment ago.  (An earlier form started all query tiles of a
    // cohort of up to 64 at one common key tile and walked the lists cyclically; with whole heads
    // dealt to the XCDs that saved a third of the traffic past L2, with the dispatch order used
    // now it cost 1-2 % time and nearly doubled that traffic: 47.9 against 27.5 GB per launch at
    // the 119k-token shape.)
  }
  int pseg = 0, pj = 0, pjb = -1;
  auto profile_segment = [&](int sidx, int& k0, int& k1) -> bool {   // false: no more segments
    const int nv = variant == 1 ? 1 : a.F;
    if (sidx == 0) {            // text prefix
      k0 = 0;
      k1 = a.off - 1;
    } else if (sidx == 1) {     // first-frame sink
      k0 = a.off;
      k1 = a.sink ? a.off + a.P - 1 : a.off - 1;
    } else if (sidx < 2 + nv) {
      if (c_hi < 0) {           // every row of the workgroup is a text row: nothing to do
        k0 = 0;
        k1 = -1;
      } else if (variant == 1) {
        k0 = a.off + max(0, c_lo - a.w_s) * a.P;
        k1 = a.off + min(a.F, c_hi + a.w_s + 1) * a.P - 1;
      } else {
        const int f = sidx - 2;
        k0 = a.off + f * a.P + max(0, c_lo - a.w_t);
        k1 = a.off + f * a.P + min(a.P - 1, c_hi + a.w_t);
      }
    } else if (sidx == 2 + nv) {  // text suffix
      k0 = a.video_end;
      k1 = a.N - 1;
    } else {
      return false;
    }
    return true;
  };
  int pleft = 0x7fffffff;    // profile: tiles this workgroup may still take
  // profile: makes [pj, pjb] the next non-empty run of tiles of the pass (intervals may overlap
  // or touch; a tile is handed out once); false when the pass is exhausted
  auto profile_interval = [&]() -> bool {
    while (pj > pjb) {
      int k0, k1;
      if (!profile_segment(pseg, k0, k1)) return false;
      ++pseg;
      if (k1 < k0) continue;
      const int ja = k0 / BN, jb = k1 / BN;
      if (jb < pj) continue;
      pj = max(pj, ja);
      pjb = jb;
    }
    return true;
  };
  // In pieces a tile is a visit of up to BN keys from any key on.  Packed: first key << 8, bit 7 where a piece may end (kCut), number
  // of keys.  They are the part's video keys, cut where a piece of any row ends, and behind the last part's the keys every row keeps.
  constexpr int kCut = 128;
  int v_key = 0, v_end = 0, v_last = 0, v_region = 2;      // next key, end of the piece and of the part's (video) keys
  bool v_cut = pieces;
  if (pieces) {
    v_key = v_end = rule.bound(a.plan, chunk, BN);
    v_last = rule.bound(a.plan, chunk + 1, BN);
    if (chunk == a.plan.n_full - 1) v_region = 0;
  }
  auto next_cut = [&](int key) -> int {
    int c = v_last;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int f = frame_of(opaque(cut_frames), i);
      int lo, hi;
      rule.window(f, lo, hi);
      if (f >= 0 && lo > key) c = min(c, lo);
      if (f >= 0 && hi > key) c = min(c, hi);
    }
    return wave_min(c);
  };
  auto next_visit = [&]() -> int {
    while (v_key >= v_end) {
      if (v_end < v_last) {
        v_end = next_cut(v_key);
        v_cut = true;
      } else if (v_region == 0) {
        v_region = 1;
        v_cut = true;
        v_key = 0;
        v_end = v_last = keep_head;
      } else if (v_region == 1) {
        v_region = 2;
        v_cut = v_cut || keep_head == 0;
        v_key = a.video_end;
        v_end = v_last = a.N;
      } else {
        return kNoTile;
      }
    }
    const int n = min(BN, v_end - v_key);
    const int visit = (v_key << 8) | (v_cut ? kCut : 0) | n;
    v_cut = false;
    v_key += n;
    return visit;
  };
  auto visit_key = [](int visit) { return visit >> 8; };
  // masks: is it asked by the loop of the masked passes?  Each loop then holds the state of its own walk only.  In three passes no scalar is spilled (14 and 10 were in 128-row tiles) and a tenth of
  // the code is gone: 187 calls 1.02-1.05 times as fast as with one walk for both loops, whose code was 1-6 % slower in 32-row tiles at head dimension 128 once it had no pieces in it (97 heads of 850 rows
  // 41.9 us, now 39.4).  In pieces 32 spilled scalars become 14,
  // a tile of the temporal pass at head dimension 64 996 instructions 827, and 124 calls take 0.94-1.01 of the time, 0.983 at the mean (48 heads of 17776 rows 119 -> 115 us).
  auto next_tile = [&](auto masks) -> int {
    if (SPARSE) return list.next();
    if (MODE == kDense) {
      const int j = lj;
      if (j >= a.nk) return kNoTile;
      lj = j + TEAMS;
      return j;
    }
    if constexpr (!decltype(masks)::value) {      // profile
      if constexpr (PIECED) return next_visit();
      return lj < l_end ? lj++ : kNoTile;
    }
    if (pleft <= 0) return kNoTile;
    if (!profile_interval()) return kNoTile;
    --pleft;
    return PIECED ? (pj++ * BN) << 8 : pj++;
  };
  if (MODE == kProfile && variant != 0 && a.plan.n_masked > 1) {
    // a masked pass in parts: count the tiles of the whole pass, then take the part's share
    int total = 0;
    while (profile_interval()) {
      total += pjb - pj + 1;
      pj = pjb + 1;
    }
    const int first = (int)(((long long)total * chunk) / a.plan.n_masked);
    pleft = (int)(((long long)total * (chunk + 1)) / a.plan.n_masked) - first;
    pseg = 0; pj = 0; pjb = -1;
    int skip = first;
    while (skip > 0 && profile_interval()) {
      const int n = min(skip, pjb - pj + 1);
      pj += n;
      skip -= n;
    }
  }
  // ======================================================================================
  // Staging of one K/V tile.
  // ======================================================================================
  // The copy is done by the load unit (buffer_load_dwordx4 ... lds): lane l of a wavefront's load
  // lands at the load's LDS address + 16 l, so piece u = tid + THREADS i of the LDS image is thread
  // tid's i-th load, and the swizzles below are applied on the memory side: the lane fetches the
  // piece of its row that belongs at that place.  No staging registers, no LDS write instructions.
  //
  // The descriptor of a tile starts at the tile's first key row and covers the rows up to
  // N, so the per-thread offsets are loop invariant, no clamping arithmetic is needed, and
  // rows beyond N (ragged last tile) read as zero.
  constexpr int ROW_STEP = THREADS / CPR;
  const int stage_row = tid / CPR, stage_piece = tid % CPR;      // row stage_row + ROW_STEP i of the tile
  // In LDS, 16-byte piece p of K row n sits at piece p ^ k_swizzle(n) of the row and 32-byte slot s
  // of V row n at slot s ^ v_swizzle(n) (head dimension 64: two rows share the 64 banks)
  auto k_swizzle = [](int n) { return D == 128 ? n & 15 : (n >> 1) & 7; };
  auto v_swizzle = [](int n) { return D == 128 ? n & 7 : (n >> 1) & 3; };
  auto k_piece = [&](int i) { return stage_piece ^ k_swizzle(stage_row + i * ROW_STEP); };
  auto v_piece = [&](int i) { return stage_piece ^ (v_swizzle(stage_row + i * ROW_STEP) << 1); };
  // 128-row query tiles: ROW_STEP is a multiple of the swizzles' period, every i has the same piece
  constexpr bool SAME_PIECE = NW == 4;
  static_assert(!SAME_PIECE || ROW_STEP % 16 == 0, "the swizzles repeat every 16 rows");
  const unsigned lds_wave = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_byte*)lds + wave * 1024);

  // Gathering form: every K/V row is fetched through a table of source rows.  For a temporal
  // head row v of the P-outer order is token row_table[entries + v] (Sec. 4.2; text rows map to
  // themselves); a spatial head uses the identity half row_table[v], so that both kinds run the
  // same instructions.  Rows beyond N map to a row outside the tensor, which the bounds-checked
  // loads return as zero.  The entries of a tile are loaded one tile ahead of its K rows and kept for its V rows, a
  // thread's PER_THREAD entries in one load (the table keeps them together, row_table_kernel); a
  // row is 2 D contiguous bytes, so the loads stay whole cache lines.
  const int tab_base = GATHER && pat != 0 ? a.nk * BN * 4 : 0;
  struct Rows { int row[GATHER ? PER_THREAD : 1]; };
  auto load_table = [&](int col_any) -> Rows {
    Rows rows = {};
    const int key0 = __builtin_amdgcn_readfirstlane(col_any) * BN;
    const __amdgpu_buffer_rsrc_t rt = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<int32_t*>(a.row_table), 0, 2u * (unsigned)a.nk * BN * 4u, kRsrcFlags);
    if constexpr (GATHER && PER_THREAD == 4) {
      const u32x4 e = __builtin_amdgcn_raw_buffer_load_b128(rt, stage_row * 16, tab_base + key0 * 4, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) rows.row[i] = (int)e[i];
    } else if constexpr (GATHER) {
      static_assert(!GATHER || PER_THREAD == 4 || PER_THREAD == 2, "one load fetches a thread's row numbers");
      const u32x2 e = __builtin_amdgcn_raw_buffer_load_b64(rt, stage_row * 8, tab_base + key0 * 4, 0);
      rows.row[0] = (int)e[0];
      rows.row[1] = (int)e[1];
    }
    return rows;
  };

  // one tensor's rows of a tile into the LDS image at dst; piece(i): the piece of its row a thread's
  // i-th load fetches
  auto load_rows = [&](const __bf16* src, int col_any, const Rows& rows, auto piece, unsigned dst) {
    if constexpr (GATHER) {
      const u32x4 rsrc = buffer_words(src, (unsigned)a.N * (D * 2));
#pragma unroll
      for (int i = 0; i < PER_THREAD; i += 2)
        load_to_lds(rsrc, rows.row[i] * (D * 2) + piece(i) * 16, rows.row[i + 1] * (D * 2) + piece(i + 1) * 16, 0, 0,
                    dst + i * THREADS * 16, THREADS * 16);
    } else {
      // the tile index is the same in every lane; saying so keeps the descriptors scalar
      const int col_one = __builtin_amdgcn_readfirstlane(col_any);
      const int key0 = PIECED ? visit_key(col_one) : col_one * BN;
      const u32x4 rsrc = buffer_words(src + (size_t)key0 * D, (unsigned)(a.N - key0) * (D * 2));
#pragma unroll
      for (int i = 0; i < PER_THREAD; i += 2) {
        auto lane_offset = [&](int n) { return stage_row * (D * 2) + piece(n) * 16 + (SAME_PIECE ? 0 : n * ROW_STEP * (D * 2)); };
        auto tile_offset = [&](int n) { return SAME_PIECE ? n * ROW_STEP * (D * 2) : 0; };
        load_to_lds(rsrc, lane_offset(i), lane_offset(i + 1), tile_offset(i), tile_offset(i + 1), dst + i * THREADS * 16, THREADS * 16);
      }
    }
  };
  auto load_k = [&](int col, const Rows& rows, int buf) { load_rows(kh, col, rows, k_piece, lds_wave + buf * K_BYTES); };
  auto load_v = [&](int col, const Rows& rows, int buf) { load_rows(vh, col, rows, v_piece, lds_wave + 2 * K_BYTES + buf * V_BYTES); };

  // ======================================================================================
  // The parts of a trip.
  // ======================================================================================
  f32x4 oacc[CB][QB], sacc[KB][QB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) oacc[cb][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run[QB], l_run[QB];      // reference maximum (raw logits, before scaling), this lane's share of the running row sum
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    m_run[qb] = kNegBig;
    l_run[qb] = 0.f;
  }

  // Operand reads.  K: lane (g, r) reads piece 4 s + g of row r of a 16-key block.  V^T: as a source
  // lane of the transposing read, lane 16 g + s supplies the 8 bytes of row 4 g + s / 4 of a 16-key
  // half step at channel 16 cb + 4 (s % 4).
  int k_off[DS], v_off[CB];
  {
#pragma unroll
    for (int s = 0; s < DS; ++s) k_off[s] = r * K_ROW + (((4 * s + g) ^ k_swizzle(r)) << 4);
    const int row = 4 * g + (r >> 2);
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) v_off[cb] = row * V_ROW + ((cb ^ v_swizzle(row)) << 5) + ((r & 3) << 3);
  }
  constexpr int PF = prefetch_depth(D, NW, MODE), PRIO_SCORES = prio_scores(MODE == kSparseExact);
  constexpr int NS = KB * DS;          // operands of the first product, order (pair of kb, s, kb in the pair)
  constexpr int NV = KS * CB;          // operands of the second product, order (ks, cb)
  static_assert(PF <= NS && PF <= NV, "the window of operands in flight spans at most two products");
  auto k_block = [](int i) { return (i / (2 * DS)) * 2 + (i & 1); };
  auto k_step = [](int i) { return (i >> 1) % DS; };
  auto k_operand = [&](int buf, int i) -> bf16x8 {
    return *reinterpret_cast<const bf16x8*>(lds + buf * K_BYTES + k_block(i) * 16 * K_ROW + k_off[k_step(i)]);
  };
  auto v_operand = [&](int buf, int i) -> bf16x8 {
    const unsigned char* src = lds + 2 * K_BYTES + buf * V_BYTES + (i / CB) * 32 * V_ROW + v_off[i % CB];
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)src);
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(src + 16 * V_ROW));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  const bool ragged = (a.N % BN) != 0;
  // What a masked pass knows of a tile: does this wavefront need it at all, and does it need
  // per-element masks?  (a row that keeps none of the tile's keys while others do needs no element
  // masks either: it takes its exponentials against +inf, i.e. all weights zero)
  struct TileMask {
    bool skip, need_masks, drop[QB];
    unsigned long long keep[QB];       // mixed tiles: bit n = the row keeps the tile's n-th key
  };
  int pos_tile = 0, pos_first = -a.off;      // temporal profiling pass: a tile and its first key's in-frame position
  auto tile_mask = [&](int tile) -> TileMask {
    TileMask t = {};
    if (!(MASKABLE && masked)) return t;
    const int k0 = __builtin_amdgcn_readfirstlane(tile) * BN, k1 = k0 + BN;
    const bool special = k0 < keep_head || k1 > a.video_end;   // some key is kept by every row, or lies beyond N
    int first = k0;              // the tile's first key in the coordinate of the windows
    if (by_position) {
      // its in-frame position: the tiles of a pass ascend, by less than a frame except at its start
      pos_first += (tile - pos_tile) * BN;
      pos_tile = tile;
      if (pos_first >= a.P) pos_first -= a.P;
      if (pos_first >= a.P) pos_first = (int)((unsigned)pos_first % (unsigned)a.P);
      first = pos_first;
    }
    bool all = false, none = false;
    if (special) {
      all = k1 <= keep_head || (k0 >= a.video_end && k1 <= a.N);
    } else if (!by_position || first + BN <= a.P) {
      all = first >= lo_max && first + BN <= hi_min;
      none = first + BN <= lo_min || first >= hi_max;
    } else if (first + BN <= 2 * a.P) {        // the end of one frame and the start of the next
      none = first >= hi_max && first + BN - a.P <= lo_min;
    }
    // (a text row keeps everything: beside video rows that keep nothing it needs the tile, but no bits)
    t.skip = none && !has_text;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) t.drop[qb] = none && video[qb];
    if (!all && !none) {
      auto ones = [](int n) -> unsigned long long {      // the n lowest bits
        n = min(max(n, 0), 64);
        return n == 0 ? 0ull : ~0ull >> (64 - n);
      };
      const unsigned long long full = ones(BN), in_range = ones(a.N - k0) & full;
      const unsigned long long always = (ones(keep_head - k0) | ~ones(a.video_end - k0)) & in_range;
      bool any_kept = false, any_part = false;
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        unsigned long long m = 0;
        // (by position: one window in every frame the tile touches)
        int f = first;
#pragma unroll 1
        do {
          m |= ones(win_hi[qb] - f) & ~ones(win_lo[qb] - f);
          f -= a.P;
        } while (by_position && f + BN > 0);
        t.keep[qb] = (m & in_range) | always;
        any_kept = any_kept || t.keep[qb] != 0;
        any_part = any_part || (t.keep[qb] != 0 && t.keep[qb] != full);
      }
      t.skip = __builtin_amdgcn_ballot_w64(any_kept) == 0;         // no row of this wave keeps any key
      t.need_masks = __builtin_amdgcn_ballot_w64(any_part) != 0;   // some row keeps a part of them
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        t.drop[qb] = !t.need_masks && t.keep[qb] == 0;
        t.keep[qb] >>= 4 * g;        // this lane's keys are 16 kb + 4 g + i
      }
    }
    return t;
  };
  // sacc[kb][qb][i] belongs to key  tile * BN + 16 kb + 4 g + i
  auto mask_scores = [&](int tile, const TileMask& t) {
    if (MASKABLE && masked) {
      if (t.need_masks) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
          const unsigned word[2] = {(unsigned)t.keep[qb], (unsigned)(t.keep[qb] >> 32)};
#pragma unroll
          for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              // the score or -inf by bits: two instructions and no condition register per score, where a
              // compare and a select took three and a register pair each
              const unsigned kept = (unsigned)__builtin_amdgcn_sbfe((int)word[kb >> 1], 16 * (kb & 1) + i, 1);
              sacc[kb][qb][i] = __uint_as_float((__float_as_uint(sacc[kb][qb][i]) & kept) | (0xff800000u & ~kept));
            }
        }
      }
    } else if (PIECED ? (tile & (kCut - 1)) != BN : ragged && tile == a.nk - 1) {
      int lim = (PIECED ? tile & (kCut - 1) : a.N - tile * BN) - 4 * g;     // keys with 16 kb + i >= lim are out of range
      // opaque to the optimiser: keeps this rarely taken masking code inside the
      // branch instead of being speculated into every tile
      asm volatile("" : "+v"(lim));
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (kb * 16 + i >= lim) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) sacc[kb][qb][i] = -INFINITY;
          }
    }
  };

  // Online softmax, two queries per lane.
  // Fast path: exponentials are taken against the current reference m_run without
  // looking at the tile's maximum.  That is the same softmax as long as nothing
  // overflows, which the row sum reveals: if any lane's partial sum exceeds
  // kLazySum (or is inf / NaN) the whole wave takes the slow path, which finds the
  // tile maximum, raises the reference, rescales O^T and the running sum, and redoes
  // the tile's exponentials.  With a reference within 2^13 of the true maximum the
  // fp32 sums and bf16 weights lose nothing, and almost every tile after the first
  // few stays on the fast path (no max reduction, no rescale).
  bf16x8 pb[KS][QB];
  auto exponentiate = [&](int qb, float mc) -> float {
    float l_loc = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      f32x8 p;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[2 * ks + (e >> 2)][qb][e & 3], a.scale_log2, -mc));
        if (D != 64) l_loc += p[e];
      }
      pb[ks][qb] = __builtin_convertvector(p, bf16x8);
      if (D == 64) {
        // Head dimension 64 is bound by the softmax's VALU work, so the row sum is taken two
        // weights per instruction: dot products of the packed pairs with (1, 1), i.e. over
        // the ROUNDED weights.  (At D = 128 this was slower: the dot products run on the
        // matrix pipeline and compete with the MFMAs there.)  The pairs are taken by vector
        // shuffles: extracted as 32-bit words of the bit-cast vector, the compiler fed all
        // four dot products the same register.
        const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
        const bf16x8 pv = pb[ks][qb];
        l_loc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pv, pv, 0, 1), ones, l_loc, false);
        l_loc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pv, pv, 2, 3), ones, l_loc, false);
        l_loc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pv, pv, 4, 5), ones, l_loc, false);
        l_loc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pv, pv, 6, 7), ones, l_loc, false);
      }
    }
    return l_loc;
  };
  auto softmax = [&](const bool (&drop)[QB]) {
    float l_loc[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
      l_loc[qb] = exponentiate(qb, MASKABLE && drop[qb] ? INFINITY : m_run[qb] * a.scale_log2);
    if (__builtin_amdgcn_ballot_w64(!(l_loc[0] <= kLazySum && l_loc[1] <= kLazySum)) != 0) {
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        float m_loc = sacc[0][qb][0];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int e = 0; e < 4; ++e) m_loc = fmaxf(m_loc, sacc[kb][qb][e]);
        m_loc = quarters_max(m_loc);
        if (MASKABLE && drop[qb]) m_loc = -INFINITY;
        const float m_new = fmaxf(m_run[qb], m_loc);
        const float alpha = __builtin_amdgcn_exp2f((m_run[qb] - m_new) * a.scale_log2);
        m_run[qb] = m_new;
        l_run[qb] *= alpha;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
          for (int e = 0; e < 4; ++e) oacc[cb][qb][e] *= alpha;
        l_loc[qb] = exponentiate(qb, MASKABLE && drop[qb] ? INFINITY : m_new * a.scale_log2);
      }
    }
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) l_run[qb] += l_loc[qb];
  };

  // Profiling: one pass's or piece's output of a row (normalised), reference maximum and row sum, to an output slot.
  auto put = [&](int qb, int slot, float l_tot) {
    const size_t at = ((size_t)slot * a.BH + bh) * a.t + opaque(qslot[qb]);
    float* op = static_cast<float*>(a.o) + at * D;
    if (g == 0) a.stats[at] = make_float2(m_run[qb], l_tot);
    const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) *reinterpret_cast<f32x4*>(op + cb * 16 + 4 * g) = oacc[cb][qb] * inv;
  };
  auto start_again = [&](int qb) {      // a piece owes nothing to the ones before it, the reference maximum neither
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) oacc[cb][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
    m_run[qb] = kNegBig;
    l_run[qb] = 0.f;
  };
  auto cuts_before = [&](int qb, int key) -> int {
    const int f = frame_of(opaque(own_frames), qb);
    int lo, hi;
    rule.window(f, lo, hi);
    return f < 0 ? 0 : (lo < key) + (hi < key);
  };
  // Ends of pieces in front of a key (see PieceRule).  `close`: of all pieces of the video keys.
  auto end_pieces = [&](int key, bool close) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      int at = cuts_before(qb, key);
      const int to = close ? 3 : cuts_before(qb, key + 1);
      float l_tot = quarters_sum(l_run[qb]);
      if (at < to) {
        for (; at < to; ++at) {
          if (qslot[qb] < a.t) put(qb, chunk + at, l_tot);
          start_again(qb);
          l_tot = 0.f;
        }
      }
    }
  };
  auto cut_before = [&](int visit) {
    if (PIECED && (visit & kCut) != 0) {
      const int key = visit_key(visit);
      const bool kept = key < keep_head || key >= a.video_end;
      end_pieces(kept ? a.video_end : key, kept);
    }
  };

  // The products.  Operand reads run PF operands ahead of their use (a rolling window of PF operand
  // registers, through both products of a batch); the scheduling barriers pin the read / product interleave.
  bf16x8 opnd[PF];
  auto read_k_ahead = [&](int buf) {
#pragma unroll
    for (int i = 0; i < PF; ++i) opnd[i] = k_operand(buf, i);
    __builtin_amdgcn_sched_barrier(0);
  };
  // S^T = K Q^T of the tile in K buffer kbuf; v_follows: the window goes on with the V^T operands of V buffer vbuf
  auto scores = [&](int kbuf, auto v_follows, int vbuf) {
    __builtin_amdgcn_s_setprio(PRIO_SCORES);
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      const int kb = k_block(i), s = k_step(i);
      const bf16x8 ka = opnd[i % PF];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        if (s == 0) sacc[kb][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
        sacc[kb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qreg[qb][s], sacc[kb][qb], 0, 0, 0);
      }
      if (i + PF < NS) opnd[i % PF] = k_operand(kbuf, i + PF);
      else if (decltype(v_follows)::value) opnd[i % PF] = v_operand(vbuf, i + PF - NS);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // O^T += V^T P^T; at: window slot of the first operand
  auto output = [&](int vbuf, auto at_c) {
    constexpr int AT = decltype(at_c)::value;
    __builtin_amdgcn_s_setprio(kPrioOutput);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int ks = i / CB, cb = i % CB;
      const bf16x8 va = opnd[(AT + i) % PF];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
        oacc[cb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, pb[ks][qb], oacc[cb][qb], 0, 0, 0);
      if (i + PF < NV) opnd[(AT + i) % PF] = v_operand(vbuf, i + PF);
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_setprio(0);
  };
  const std::true_type yes;
  const std::false_type no;
  const std::integral_constant<int, 0> first_slot;
  const std::integral_constant<int, NS> after_scores;

  // ======================================================================================
  // Main loop, skewed by one tile: trip j holds the scores of tile j.  LDS holds K of tile j + 1 and V of
  // j; K of j + 2 and V of j + 1 are on their way into it.  The forms with mask state take one tile
  // after the other under masks (K and V of j in LDS, of j + 1 on their way): which wavefronts need a tile
  // differs, and the registers do not hold the masks of two tiles beside the rest.
  // ======================================================================================
  const bool sequential = MASKABLE && masked;
  int col, col1, col2 = kNoTile;
  if (MODE == kProfile && sequential) {
    col = next_tile(yes);
    col1 = next_tile(yes);
  } else {
    col = next_tile(no);
    col1 = next_tile(no);
    if (!sequential) col2 = next_tile(no);
  }
  Rows rows_v = {}, rows_k = {};        // gathering form: rows of the tiles whose V and K are fetched next
  if (col != kNoTile) {
    if (GATHER) rows_k = load_table(col);
    load_k(col, rows_k, 0);
    load_v(col, rows_k, 0);
  }
  if (!sequential && col1 != kNoTile) {
    if (GATHER) rows_v = load_table(col1);
    load_k(col1, rows_v, 1);
  }
  if (GATHER && col2 != kNoTile) rows_k = load_table(col2);
  wait_loads_to_lds<0>();
  __syncthreads();

  // Touch Q here so that its loads are known to have completed before the loop.  Without
  // this the compiler's wait-count bookkeeping still sees them pending at the loop head
  // and emits vmcnt waits in front of the first products of every iteration, which then
  // wait for the NEXT tile's freshly issued global loads instead.
#pragma unroll
  for (int s = 0; s < DS; ++s) asm volatile("" ::"v"(qreg[0][s]), "v"(qreg[1][s]));

  int buf = 0;
  if (sequential) {
    while (col != kNoTile) {
      if (col1 != kNoTile) {
        load_k(col1, rows_k, buf ^ 1);
        load_v(col1, rows_k, buf ^ 1);
      }
      col2 = next_tile(yes);
      const TileMask t = tile_mask(PIECED ? visit_key(col) / BN : col);
      if (active && !t.skip) {
        read_k_ahead(buf);
        scores(buf, yes, buf);
        __builtin_amdgcn_s_setprio(0);
        mask_scores(col, t);
        softmax(t.drop);
        output(buf, after_scores);
      }
      wait_loads_to_lds<0>();
      barrier_loads_done();
      buf ^= 1;
      col = col1;
      col1 = col2;
    }
    if (TEAMS > 1 && team == 1 && (n_tiles & 1)) barrier_loads_done();      // the other team's last tile
  } else if constexpr (MODE != kSparseExact) {
    const bool no_drop[QB] = {false, false};
    if (active && col != kNoTile) {
      read_k_ahead(0);
      scores(0, no, 0);
      __builtin_amdgcn_s_setprio(0);
      mask_scores(col, TileMask{});
    }
    __syncthreads();                      // the first trip stages tile 2 over tile 0's keys
    while (col1 != kNoTile) {
      const int col3 = next_tile(no);
      if (col2 != kNoTile) load_k(col2, rows_k, buf);
      load_v(col1, rows_v, buf ^ 1);
      if (GATHER) {
        rows_v = rows_k;
        if (col3 != kNoTile) rows_k = load_table(col3);
      }
      if (active) {
        cut_before(col);
        read_k_ahead(buf ^ 1);
        softmax(no_drop);
        scores(buf ^ 1, yes, buf);
        output(buf, after_scores);
        mask_scores(col1, TileMask{});
      }
      wait_loads_to_lds<0>();
      barrier_loads_done();
      buf ^= 1;
      col = col1;
      col1 = col2;
      col2 = col3;
    }
    if (TEAMS > 1 && team == 1 && (n_tiles & 1) && n_tiles > 1) barrier_loads_done();      // the other team's last trip
    if (active && col != kNoTile) {
      cut_before(col);
#pragma unroll
      for (int i = 0; i < PF; ++i) opnd[i] = v_operand(buf, i);
      softmax(no_drop);
      output(buf, first_slot);
    }
  }

  // Two teams: each finishes one 16-query block of every wavefront with what the other has of it (output, maximum, row
  // sum), handed over through LDS.
  if constexpr (TEAMS > 1) {
    constexpr int PART = CB * 1024;
    static_assert(2 * NW * (PART + 512) <= TEAMS * 2 * STAGE_BYTES, "the halves fit the LDS of the tiles");
    unsigned char* const outs = all_lds + lane * 16;
    unsigned char* const stats = all_lds + 2 * NW * PART + lane * 8;
    const int slot = team * NW + wave, other = (team ^ 1) * NW + wave;
    __syncthreads();      // the last operands are read
    const float l_sum[QB] = {quarters_sum(l_run[0]), quarters_sum(l_run[1])};
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) *reinterpret_cast<f32x4*>(outs + slot * PART + cb * 1024) = team ? oacc[cb][0] : oacc[cb][1];
    *reinterpret_cast<float2*>(stats + slot * 512) = team ? make_float2(m_run[0], l_sum[0]) : make_float2(m_run[1], l_sum[1]);
    __syncthreads();
    const float2 st = *reinterpret_cast<const float2*>(stats + other * 512);
    const float m_own = team ? m_run[1] : m_run[0], l_own = team ? l_sum[1] : l_sum[0];
    const float m_all = fmaxf(m_own, st.x);
    const float w_own = __builtin_amdgcn_exp2f((m_own - m_all) * a.scale_log2), w_other = __builtin_amdgcn_exp2f((st.x - m_all) * a.scale_log2);
    const float l_tot = l_own * w_own + st.y * w_other;
    const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    const int row = team ? qslot[1] : qslot[0];
    if (row < a.N) {
      __bf16* op = static_cast<__bf16*>(a.o) + (head + (team ? io_row[1] : io_row[0])) * D;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        const f32x4 own = team ? oacc[cb][1] : oacc[cb][0];
        const f32x4 theirs = *reinterpret_cast<const f32x4*>(outs + other * PART + cb * 1024);
        *reinterpret_cast<bf16x4*>(op + cb * 16 + 4 * g) = __builtin_convertvector(own * (w_own * inv) + theirs * (w_other * inv), bf16x4);
      }
    }
    return;
  }

  // ======================================================================================
  // Epilogue: normalise and store.  oacc[cb][qb][i] = O[query 16 qb + r][16 cb + 4 g + i]
  // ======================================================================================
  if (PIECED && pieces && chunk == a.plan.n_full - 1 && a.pieces == a.plan.n_full + 2) {
    end_pieces(a.video_end, true);      // no keys that every row keeps: the video keys were the last
    return;
  }
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const float l_tot = quarters_sum(l_run[qb]);
    const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    if (MODE == kProfile) {
      // output slots: the parts or pieces of the unmasked pass, the parts of the spatial pass, of the temporal pass
      int slot = variant == 0 ? chunk : a.plan.n_full + (variant - 1) * a.plan.n_masked + chunk;
      if (PIECED) {
        if (variant != 0) slot = a.pieces + chunk;
        else if (chunk == a.plan.n_full - 1) slot = a.pieces - 1;
        else slot += cuts_before(qb, v_last);
      }
      if (qslot[qb] < a.t) put(qb, slot, l_tot);
    } else if (qslot[qb] < a.N) {
      __bf16* op = static_cast<__bf16*>(a.o) + (head + io_row[qb]) * D;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
        *reinterpret_cast<bf16x4*>(op + cb * 16 + 4 * g) = __builtin_convertvector(oacc[cb][qb] * inv, bf16x4);
    }
  }
}

// rows_total: N for dense / sparse, t for profiling
template <int D, int NW, int BN, int MODE, int TEAMS = 1, bool PIECED = false>
int launch_one(AttnArgs a, int rows_total, hipStream_t stream) {
  constexpr int BM = 32 * NW;
  a.nqt = (rows_total + BM - 1) / BM;
  a.total = a.BH * a.nqt;
  constexpr int COHORT = kCohort / TEAMS;
  const int blocks = (a.total + 8 * COHORT - 1) / (8 * COHORT);      // dense: blocks of consecutive tiles per XCD
  a.cohort = dense_cohort(a.total, COHORT);
  const unsigned per_xcd = (unsigned)blocks * (unsigned)a.cohort;
  if (MODE == kSparse || MODE == kSparseExact || MODE == kSparseGather) {
    const int per_cu = NW == 4 ? waves_per_simd(D, NW, MODE) : 2;
    a.so = sparse_order(a.BH, a.nqt, BM, a.off, a.video_end, a.N, TEAMS > 1 ? 32 : 32 * per_cu, 256 * per_cu, NW == 4 ? 2 : 0, a.nk);
  }
  const unsigned grid = MODE == kProfile ? (unsigned)(8 * (a.plan.slots() - (PIECED ? a.plan.n_masked : 0)) * ((a.total + 7) / 8))
                        : MODE == kDense ? 8u * per_xcd : sparse_grid(a.so, a.BH);
  (void)hipGetLastError();   // drop any stale error left by earlier runtime calls of the process
  constexpr bool SPARSE_MODE = MODE == kSparse || MODE == kSparseExact || MODE == kSparseGather;
  if constexpr (SPARSE_MODE && TEAMS == 1) {      // (two teams: 21 heads at most, see two_teams)
    if (a.BH > 64) {      // label classes over more than one 64-head word
      hipLaunchKernelGGL((attn_kernel<D, NW, BN, MODE, kWideLabelWords>), dim3(grid), dim3(64 * NW), 0, stream, a);
      return hip_status(hipGetLastError());
    }
  }
  hipLaunchKernelGGL((attn_kernel<D, NW, BN, MODE, 1, TEAMS, PIECED>), dim3(grid), dim3(64 * NW * TEAMS), 0, stream, a);
  return hip_status(hipGetLastError());
}

}  // namespace

}  // namespace svg
