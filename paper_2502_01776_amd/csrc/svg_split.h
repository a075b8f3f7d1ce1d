// The body of a workgroup that splits the keys of 32 query rows over its wavefronts: see svg_split.hip, and the text-row query
// tiles in svg_attn.hip.
#pragma once
#include "svg_attn_common.h"

namespace svg {
namespace attn {

constexpr int kWaves = 4;
constexpr int kRows = 32;      // query rows of a workgroup
constexpr int kKeys = 32;      // keys a wavefront takes at a time: one unit
constexpr int kSortRows = 64 * kWaves;      // sampled rows a workgroup sorts by itself
constexpr int split_lds_bytes(int D) { return kWaves * kRows * D * 4; }

// lds: split_lds_bytes(D).  Sparse and dense: rows row0 .. row0 + 31 of head bh, entries [list_begin, list_end) of pattern
// pat's list; profiling: group grp of the sampled rows, part chunk of pass variant.
template <int D, int MODE>
__device__ __forceinline__ void split_body(const AttnArgs& a, unsigned char* const lds, const int bh, const int row0, const int grp, const int pat,
                                           const int list_begin, const int list_end, const int variant, const int chunk) {
  constexpr int W = kWaves;
  constexpr bool SPARSE = MODE == kSparse || MODE == kSparseExact || MODE == kSparseGather;
  constexpr bool GATHER = MODE == kSparseGather, MASKABLE = MODE == kProfile || MODE == kSparseExact;
  constexpr int QB = 2, KB = 2;            // 16-query blocks, 16-key blocks of a unit
  constexpr int DS = D / 32, CB = D / 16;  // 32-channel steps of the first product, 16-channel blocks of O^T
  constexpr int ROW = D * 2, CPR = D / 8;  // bytes and 16-byte pieces of a row
  constexpr int V_LOADS = kKeys * CPR / 64;
  constexpr int PART = CB * QB * 1024;     // bytes of a wavefront's O^T; its V unit is staged in the first half of them
  static_assert(kKeys * ROW <= PART, "a wavefront's V unit lies in its own part");
  static_assert((CB * QB) % W == 0, "the merge deals blocks of O^T to the wavefronts");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r = lane & 15;
  const size_t head = (size_t)bh * a.N;

  // ---- this lane's query rows (profiling: as in attn_kernel, in groups of up to 32)
  int qslot[QB], qrow[QB];
  if (MODE == kProfile) {
    int slot[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      const int in_group = qb * 16 + r;
      qslot[qb] = in_group < a.rows_per_group ? grp * a.rows_per_group + in_group : a.t;
      slot[qb] = qslot[qb] < a.t ? qslot[qb] : min(grp * a.rows_per_group, a.t - 1);
    }
    if (variant == 2 && a.nqt > 1) {      // (one group holds the same rows in any order)
      if (a.order_t == nullptr) {
        int* const bin = reinterpret_cast<int*>(lds);
        int* const sorted = bin + kSortRows;
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
        __syncthreads();
      } else {
        slot[0] = a.order_t[slot[0]];
        slot[1] = a.order_t[slot[1]];
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
      qslot[qb] = row0 + qb * 16 + r;
      qrow[qb] = min(qslot[qb], a.N - 1);
    }
  }

  // ---- mask windows: the run of keys (temporal profiling pass: of in-frame positions) a row keeps, see attn_kernel
  const bool masked = MODE == kSparseExact || (MODE == kProfile && variant != 0);
  const int keep_head = a.sink ? a.off + a.P : a.off;
  const bool by_position = MODE == kProfile && variant == 2;
  int win_lo[QB], win_hi[QB], io_row[QB];
  bool video[QB];
  int c_lo = 0x7fffffff, c_hi = 0x7fffffff;      // smallest and smallest negative coordinate
  auto row_window = [&](int c, int groups, int w, int base, int unit, int& lo, int& hi) {
    w = min(w, groups);
    lo = base + max(0, c - w) * unit;
    hi = base + min(groups, c + w + 1) * unit;
  };
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    win_lo[qb] = 0;
    win_hi[qb] = by_position ? a.P : a.N;
    const int n = qrow[qb];
    io_row[qb] = n;
    video[qb] = n >= a.off && n < a.video_end;
    if (!video[qb]) continue;
    const int v = n - a.off;
    int pos = 0;
    if (SPARSE && pat) {
      const int token = a.off + a.order.token(v, pos);
      if (a.qo_token_order) io_row[qb] = token;
    }
    if (MASKABLE && masked) {
      unsigned in_frame;
      const int fq = (int)divide((unsigned)v, (unsigned)a.P, a.inv_P, in_frame);
      if (MODE == kSparseExact) {
        if (pat) row_window(pos, a.P, a.w_t, keep_head, a.sink ? a.F - 1 : a.F, win_lo[qb], win_hi[qb]);
        else row_window(fq, a.F, a.w_s, a.off, a.P, win_lo[qb], win_hi[qb]);
      } else {
        const int c = variant == 1 ? fq : (int)in_frame;
        if (variant == 1) row_window(c, a.F, a.w_s, a.off, a.P, win_lo[qb], win_hi[qb]);
        else row_window(c, a.P, a.w_t, 0, 1, win_lo[qb], win_hi[qb]);
        c_lo = min(c_lo, c);
        c_hi = min(c_hi, -c);
      }
    }
  }
  int lo_min = 0, lo_max = 0, hi_min = 0, hi_max = 0;
  bool has_text = false;
  if (MASKABLE) {
    int lo[2] = {0x7fffffff, 0x7fffffff}, hi[2] = {0x7fffffff, 0x7fffffff};
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
      if (video[qb]) {
        lo[0] = min(lo[0], win_lo[qb]);
        lo[1] = min(lo[1], -win_lo[qb]);
        hi[0] = min(hi[0], win_hi[qb]);
        hi[1] = min(hi[1], -win_hi[qb]);
      }
    lo_min = quad_rows_min(lo[0]);
    lo_max = -quad_rows_min(lo[1]);
    hi_min = quad_rows_min(hi[0]);
    hi_max = -quad_rows_min(hi[1]);
    has_text = __builtin_amdgcn_ballot_w64(!(video[0] && video[1])) != 0;
    if (MODE == kProfile) {
      c_lo = quad_rows_min(c_lo);
      c_hi = -quad_rows_min(c_hi);
    }
  }

  bf16x8 qreg[QB][DS];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const __bf16* qp = a.q + (head + io_row[qb]) * D + g * 8;
#pragma unroll
    for (int st = 0; st < DS; ++st) qreg[qb][st] = *reinterpret_cast<const bf16x8*>(qp + st * 32);
  }
  const bool kv_copy = SPARSE && pat != 0 && a.k_t != nullptr;
  const __bf16* kh = (kv_copy ? a.k_t : a.k) + head * D;
  const __bf16* vh = (kv_copy ? a.v_t : a.v) + head * D;

  // ---- the wavefront's units: every W-th of the workgroup's
  const int n_all = (a.N + kKeys - 1) / kKeys;
  const int32_t* cols = nullptr;
  int base = 0, now = 0, u = wave, u_end = n_all;
  int seg_first = 0, seg_before = 0x7fffffff;      // profile: this lane's run of units and the number of units in front of it
  auto load_cols = [&](int at) -> int {
    const int i = at + lane;
    return i < list_end - list_begin ? cols[i] : 0;
  };
  if (SPARSE) {
    cols = (pat ? a.col_idx[1] : a.col_idx[0]) + list_begin;
    u_end = (list_end - list_begin) << a.halves_log2;
    now = load_cols(0);
  } else if (MODE == kProfile && variant == 0) {
    u += a.plan.full_bound[chunk] << a.halves_log2;
    u_end = min(n_all, a.plan.full_bound[chunk + 1] << a.halves_log2);
  } else if (MODE == kProfile) {
    // The runs of units that can hold a kept key for any row of the workgroup, one to a lane: text prefix, first-frame
    // sink, the window around the rows' frames (spatial) or, per frame, around their positions (temporal), text suffix.
    const int nv = variant == 1 ? 1 : a.F, f = lane - 2;
    int k0 = 0, k1 = -1;
    if (lane == 0) k1 = a.off - 1;
    else if (lane == 1) {
      k0 = a.off;
      k1 = a.sink ? a.off + a.P - 1 : -1;
    } else if (f < nv) {
      if (c_lo <= c_hi) {
        k0 = variant == 1 ? a.off + max(0, c_lo - a.w_s) * a.P : a.off + f * a.P + max(0, c_lo - a.w_t);
        k1 = variant == 1 ? a.off + min(a.F, c_hi + a.w_s + 1) * a.P - 1 : a.off + f * a.P + min(a.P - 1, c_hi + a.w_t);
      }
    } else if (f == nv) {
      k0 = a.video_end;
      k1 = a.N - 1;
    }
    // runs ascend; a unit that two of them touch belongs to the first
    int last = k1 < k0 ? -1 : k1 / kKeys;
    const int own_last = last;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int x = __shfl_up(last, d, 64);
      if (lane >= d) last = max(last, x);
    }
    const int before = __shfl_up(last, 1, 64);
    seg_first = max(k0 / kKeys, lane == 0 ? 0 : before + 1);
    const int n = max(0, own_last - seg_first + 1);
    int sum = n;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int x = __shfl_up(sum, d, 64);
      if (lane >= d) sum += x;
    }
    const int total = __builtin_amdgcn_readlane(sum, 63);
    seg_before = n > 0 ? sum - n : 0x7fffffff;
    u += (int)(((long long)total * chunk) / a.plan.n_masked);
    u_end = (int)(((long long)total * (chunk + 1)) / a.plan.n_masked);
  }
  auto next_unit = [&]() -> int {      // first key of the next unit or kNoTile
    const int n = u;
    if (n >= u_end) return kNoTile;
    u += W;
    if (SPARSE) {
      const int e = n >> a.halves_log2, half = n & ((1 << a.halves_log2) - 1);
      if (e >= base + 64) {
        base += 64;
        now = load_cols(base);
      }
      return ((__builtin_amdgcn_readlane(now, e - base) << a.halves_log2) + half) * kKeys;
    }
    if (MODE == kProfile && variant != 0) {
      const int at = 63 - __builtin_clzll(__builtin_amdgcn_ballot_w64(seg_before <= n));      // the last run that starts at n or before
      return (__builtin_amdgcn_readlane(seg_first, at) + n - __builtin_amdgcn_readlane(seg_before, at)) * kKeys;
    }
    return n * kKeys;
  };

  // ---- loads.  K: the A operand of the first product as it is; V: rows, staged through LDS
  struct Rows { int k[KB], v[V_LOADS]; };
  auto key_rows = [&](int key0) -> Rows {       // byte offsets of the rows
    Rows x;
    if constexpr (GATHER) {
      const int key = key0 + (lane & 31);
      int row = key;
      if (pat && key >= a.off && key < a.video_end) row = a.off + a.order.token(key - a.off);
      if (key >= a.N) row = 0x00ffffff;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) x.k[kb] = __shfl(row, 16 * kb + r, 64) * ROW;
#pragma unroll
      for (int i = 0; i < V_LOADS; ++i) x.v[i] = __shfl(row, (lane + 64 * i) / CPR, 64) * ROW;
    } else {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) x.k[kb] = (16 * kb + r) * ROW;
#pragma unroll
      for (int i = 0; i < V_LOADS; ++i) x.v[i] = (lane + 64 * i) / CPR * ROW;
    }
    return x;
  };
  auto rsrc = [&](const __bf16* p, int key0) {
    const int first = GATHER ? 0 : key0;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16*>(p + (size_t)first * D), 0, (unsigned)max(0, a.N - first) * ROW, kRsrcFlags);
  };
  bf16x8 kreg[KB][DS];
  u32x4 vreg[V_LOADS];
  auto load_k = [&](int key0, const Rows& x) {
    const auto rs = rsrc(kh, key0);
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int st = 0; st < DS; ++st)
        kreg[kb][st] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs, x.k[kb] + 16 * g + 64 * st, 0, 0));
  };
  auto load_v = [&](int key0, const Rows& x) {
    const auto rs = rsrc(vh, key0);
#pragma unroll
    for (int i = 0; i < V_LOADS; ++i)
      vreg[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, x.v[i] + (lane & (CPR - 1)) * 16, 0, 0);
  };
  unsigned char* const own = lds + wave * PART;
  auto v_swizzle = [](int n) { return D == 128 ? n & 7 : (n >> 1) & 3; };
  auto stage_v = [&]() {
#pragma unroll
    for (int i = 0; i < V_LOADS; ++i) {
      const int row = (lane + 64 * i) / CPR, p = lane & (CPR - 1);
      *reinterpret_cast<u32x4*>(own + row * ROW + ((p ^ (v_swizzle(row) << 1)) << 4)) = vreg[i];
    }
  };
  int v_off[CB];
  {
    const int row = 4 * g + (r >> 2);
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) v_off[cb] = row * ROW + ((cb ^ v_swizzle(row)) << 5) + ((r & 3) << 3);
  }
  auto v_operand = [&](int cb) -> bf16x8 {
    const unsigned char* src = own + v_off[cb];
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)src);
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(src + 16 * ROW));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  f32x4 oacc[CB][QB], sacc[KB][QB];
  float m_run[QB], l_run[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    m_run[qb] = kNegBig;
    l_run[qb] = 0.f;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) oacc[cb][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // ---- masks of a unit
  struct UnitMask { bool skip, bits, drop[QB]; unsigned keep[QB]; };      // as attn_kernel's TileMask, for 32 keys
  auto unit_mask = [&](int k0) -> UnitMask {
    UnitMask t = {};
    if (!(MASKABLE && masked)) return t;
    const int k1 = k0 + kKeys;
    int first = k0;
    if (by_position) {
      first = k0 - a.off;
      if (first >= a.P) {
        unsigned rest;
        divide((unsigned)first, (unsigned)a.P, a.inv_P, rest);
        first = (int)rest;
      }
    }
    bool all = false, none = false;
    if (k0 < keep_head || k1 > a.video_end) {
      all = k1 <= keep_head || (k0 >= a.video_end && k1 <= a.N);
    } else if (!by_position || first + kKeys <= a.P) {
      all = first >= lo_max && first + kKeys <= hi_min;
      none = first + kKeys <= lo_min || first >= hi_max;
    } else if (first + kKeys <= 2 * a.P) {
      none = first >= hi_max && first + kKeys - a.P <= lo_min;
    }
    t.skip = none && !has_text;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) t.drop[qb] = none && video[qb];
    if (!all && !none) {
      auto ones = [](int n) -> unsigned { return n <= 0 ? 0u : ~0u >> (32 - min(n, 32)); };
      const unsigned in_range = ones(a.N - k0);
      const unsigned always = (ones(keep_head - k0) | ~ones(a.video_end - k0)) & in_range;
      bool any_kept = false, any_part = false;
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        unsigned m = 0;
        int f = first;
#pragma unroll 1
        do {
          m |= ones(win_hi[qb] - f) & ~ones(win_lo[qb] - f);
          f -= a.P;
        } while (by_position && f + kKeys > 0);
        t.keep[qb] = (m & in_range) | always;
        any_kept = any_kept || t.keep[qb] != 0;
        any_part = any_part || (t.keep[qb] != 0 && t.keep[qb] != ~0u);
      }
      t.skip = __builtin_amdgcn_ballot_w64(any_kept) == 0;
      t.bits = __builtin_amdgcn_ballot_w64(any_part) != 0;
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        t.drop[qb] = !t.bits && t.keep[qb] == 0;
        t.keep[qb] >>= 4 * g;
      }
    }
    return t;
  };
  auto mask_scores = [&](int k0, const UnitMask& t) {
    if (MASKABLE && masked) {
      if (t.bits) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
          for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const unsigned kept = (unsigned)__builtin_amdgcn_sbfe((int)t.keep[qb], 16 * kb + i, 1);
              sacc[kb][qb][i] = __uint_as_float((__float_as_uint(sacc[kb][qb][i]) & kept) | (0xff800000u & ~kept));
            }
      }
    } else if (k0 + kKeys > a.N) {
      int lim = a.N - k0 - 4 * g;
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

  // ---- softmax of a unit.  The row sum is over the weights as in attn_kernel: rounded at head dimension 64
  bf16x8 pb[QB];
  auto exponentiate = [&](int qb, float mc) -> float {
    float l_loc = 0.f;
    f32x8 p;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[e >> 2][qb][e & 3], a.scale_log2, -mc));
      if (D != 64) l_loc += p[e];
    }
    pb[qb] = __builtin_convertvector(p, bf16x8);
    if (D == 64) {
      const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
      const bf16x8 pv = pb[qb];
      l_loc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pv, pv, 0, 1), ones, l_loc, false);
      l_loc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pv, pv, 2, 3), ones, l_loc, false);
      l_loc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pv, pv, 4, 5), ones, l_loc, false);
      l_loc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pv, pv, 6, 7), ones, l_loc, false);
    }
    return l_loc;
  };
  auto softmax = [&](const bool (&drop)[QB]) {
    float m_new[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      float m_loc = sacc[0][qb][0];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e) m_loc = fmaxf(m_loc, sacc[kb][qb][e]);
      m_loc = quarters_max(m_loc);
      m_new[qb] = MASKABLE && drop[qb] ? m_run[qb] : fmaxf(m_run[qb], m_loc);
    }
    if (__builtin_amdgcn_ballot_w64(m_new[0] > m_run[0] || m_new[1] > m_run[1]) != 0) {
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        const float alpha = __builtin_amdgcn_exp2f((m_run[qb] - m_new[qb]) * a.scale_log2);
        m_run[qb] = m_new[qb];
        l_run[qb] *= alpha;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
          for (int e = 0; e < 4; ++e) oacc[cb][qb][e] *= alpha;
      }
    }
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) l_run[qb] += exponentiate(qb, MASKABLE && drop[qb] ? INFINITY : m_run[qb] * a.scale_log2);
  };

  // ---- main loop: the next unit is requested as soon as the present one's registers are free
  auto request = [&](int key0) {
    if (key0 == kNoTile) return;
    const Rows x = key_rows(key0);
    load_k(key0, x);
    load_v(key0, x);
  };
  int key = next_unit();
  request(key);
  while (key != kNoTile) {
    const int next = next_unit();
    const UnitMask t = unit_mask(key);
    if (!t.skip) {
#pragma unroll
      for (int st = 0; st < DS; ++st)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) {
            if (st == 0) sacc[kb][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
            sacc[kb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kreg[kb][st], qreg[qb][st], sacc[kb][qb], 0, 0, 0);
          }
      stage_v();
    }
    request(next);
    if (!t.skip) {
      mask_scores(key, t);
      softmax(t.drop);
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        const bf16x8 va = v_operand(cb);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) oacc[cb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, pb[qb], oacc[cb][qb], 0, 0, 0);
      }
    }
    key = next;
  }

  // ---- merge: every wavefront scales its part with its share of the row, then finishes some 16 x 16 blocks of O^T
  float l_tot[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    l_tot[qb] = quarters_sum(l_run[qb]);
    if (g == 0) *reinterpret_cast<float2*>(own + (16 * qb + r) * 8) = make_float2(m_run[qb], l_tot[qb]);
  }
  __syncthreads();
  float2 part_stats[QB][W];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb)
#pragma unroll
    for (int w = 0; w < W; ++w) part_stats[qb][w] = *reinterpret_cast<const float2*>(lds + w * PART + (16 * qb + r) * 8);
  __syncthreads();      // (read by all before the parts are written over them)
  float m_all[QB], l_all[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const float2* const st = part_stats[qb];
    m_all[qb] = kNegBig;
#pragma unroll
    for (int w = 0; w < W; ++w) m_all[qb] = fmaxf(m_all[qb], st[w].y > 0.f ? st[w].x : kNegBig);
    l_all[qb] = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const float x = st[w].y * __builtin_amdgcn_exp2f((st[w].x - m_all[qb]) * a.scale_log2);
      l_all[qb] += st[w].y > 0.f ? x : 0.f;
    }
    const float weight = __builtin_amdgcn_exp2f((m_run[qb] - m_all[qb]) * a.scale_log2) / l_all[qb];
    const float mine = l_tot[qb] > 0.f ? weight : 0.f;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
      *reinterpret_cast<f32x4*>(own + (cb * QB + qb) * 1024 + lane * 16) = oacc[cb][qb] * mine;
  }
  __syncthreads();
  constexpr int BLOCKS = CB * QB / W;      // 16 x 16 blocks of O^T a wavefront finishes
#pragma unroll
  for (int i = 0; i < BLOCKS; ++i) {
    const int block = wave * BLOCKS + i, cb = block / QB;
    const bool second = block % QB != 0;
    f32x4 sum = *reinterpret_cast<const f32x4*>(lds + block * 1024 + lane * 16);
#pragma unroll
    for (int w = 1; w < W; ++w) sum += *reinterpret_cast<const f32x4*>(lds + w * PART + block * 1024 + lane * 16);
    const int slot = second ? qslot[1] : qslot[0];
    if (MODE == kProfile) {
      if (slot < a.t) {
        const int out = variant == 0 ? chunk : a.plan.n_full + (variant - 1) * a.plan.n_masked + chunk;
        const size_t at = ((size_t)out * a.BH + bh) * a.t + slot;
        *reinterpret_cast<f32x4*>(static_cast<float*>(a.o) + at * D + cb * 16 + 4 * g) = sum;
        if (cb == 0 && g == 0) a.stats[at] = second ? make_float2(m_all[1], l_all[1]) : make_float2(m_all[0], l_all[0]);
      }
    } else if (slot < a.N) {
      *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(a.o) + (head + (second ? io_row[1] : io_row[0])) * D + cb * 16 + 4 * g) =
          __builtin_convertvector(sum, bf16x4);
    }
  }
}

}  // namespace attn

}  // namespace svg
