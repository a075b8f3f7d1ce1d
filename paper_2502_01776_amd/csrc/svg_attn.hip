// Launches of the attention kernel (svg_attn_kernel.h), the order, error and label kernels of online profiling
// (Alg. 1, Sec. 4.1) and the row table of the gathering form.
#include "svg_attn_kernel.h"

namespace svg {

namespace {

// Groups the sampled rows by in-frame position for the temporal profiling variant:
// order[] receives the indices 0..t-1 sorted by a coarse position bin (text rows
// first), ascending inside a bin.  One workgroup, counting sort with LDS atomics; the
// atomics leave the order inside a bin to chance, and which rows share a wavefront
// decides where that wavefront renews its reference maximum, i.e. the rounding of the
// results, so every bin is sorted afterwards to make the grouping, and with it every
// output bit, the same on every run.
__global__ __launch_bounds__(1024) void profile_order_kernel(const int32_t* rows, int t, int off,
                                                             int video_end, int P, int32_t* order) {
  __shared__ int hist[kOrderBins];
  __shared__ int part[1024];
  const int tid = threadIdx.x;
  auto bin_of = [&](int n) -> int { return order_bin(n, off, video_end, P); };
  for (int i = tid; i < kOrderBins; i += 1024) hist[i] = 0;
  __syncthreads();
  for (int i = tid; i < t; i += 1024) atomicAdd(&hist[bin_of(rows[i])], 1);
  __syncthreads();
  // exclusive scan of the 2048 bins: two per thread, then Hillis-Steele over the pair sums
  const int h0 = hist[2 * tid], h1 = hist[2 * tid + 1];
  part[tid] = h0 + h1;
  __syncthreads();
  for (int step = 1; step < 1024; step <<= 1) {
    const int add = tid >= step ? part[tid - step] : 0;
    __syncthreads();
    part[tid] += add;
    __syncthreads();
  }
  const int base = part[tid] - (h0 + h1);
  hist[2 * tid] = base;
  hist[2 * tid + 1] = base + h0;
  __syncthreads();
  for (int i = tid; i < t; i += 1024) order[atomicAdd(&hist[bin_of(rows[i])], 1)] = i;
  __syncthreads();
  // hist[b] is now the end of bin b; insertion sort of each (short) bin by row index
  for (int b = 2 * tid; b < 2 * tid + 2; ++b) {
    const int s = b == 0 ? 0 : hist[b - 1], e = hist[b];
    for (int i = s + 1; i < e; ++i) {
      const int x = order[i];
      int j = i - 1;
      while (j >= s && order[j] > x) {
        order[j + 1] = order[j];
        --j;
      }
      order[j + 1] = x;
    }
  }
}

// Squared errors of the two masked outputs against the unmasked one (Alg. 1, last
// block): block (x, bh) sums PASSES times err_rows(D) sampled rows of head bh.  Each of the three outputs of
// a row is first reassembled from the parts its pass was cut into: part r holds its normalised
// output O_r, its reference maximum m_r and its row sum l_r, and O = sum_r w_r O_r / sum_r w_r with
// w_r = l_r * 2^((m_r - max_r m_r) * scale_log2); a part that kept no key of the row has
// l_r = 0.  Text query rows are skipped (both masks keep every key for them, so they
// contribute exactly zero).
//
// Bound by latency for few rows and by memory for many.  A thread owns four channels of a row, so a
// row takes D / 4 lanes and a block 1024 / (D / 4) rows at a time; every thread works the
// weights of its row out itself (the lanes of a row read the same words) and all its loads, of the
// statistics and of every part, are independent of each other.  The numbers of parts are template arguments
// for that reason: NF is exact but for pieces, parts beyond n_full and n_masked (at most NM) are read as the last one with weight zero.
// (An earlier form, 16 rows per block, worked the weights out on 48 threads and walked the parts in
// a loop of dependent loads: 24.6 us at 24 rows of 6 heads, 31 at 91 rows of 16, 29 at 328 of 40, 39 at
// 1191 of 24; then 4.7, 6.4, 12.1 and 23.7.)
// How many blocks a head has, and how their sums come together (the launch before this one cleared the tickets): error_blocks in svg_host.cpp.

__device__ __forceinline__ void store_label(float sum_s, float sum_t, int bh, int t, int D, uint8_t* labels, float* mse) {
  const float per = (float)t * (float)D;
  const float ms = sum_s / per, mt = sum_t / per;
  if (mse) {
    mse[2 * bh + 0] = ms;
    mse[2 * bh + 1] = mt;
  }
  labels[bh] = ms < mt ? SVG_HEAD_SPATIAL : SVG_HEAD_TEMPORAL;      // Alg. 1
}

__device__ __forceinline__ float wave_sum(float x) {      // fixed order: deterministic
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) x += __shfl_xor(x, m, 64);
  return x;
}

// With the unmasked pass in pieces (a.pieces = n_full of them, at most NF) the spatial output is merged from those of the row's window and
// of the keys that every row keeps.
struct PieceArgs {
  ProfilePlan plan;
  PieceRule rule;
  int bn;
};
struct NoPieces {};
template <bool PIECES>
using PieceArgsIf = std::conditional_t<PIECES, PieceArgs, NoPieces>;      // (100 bytes of arguments; and gridDim.x brings 256, see clear_tickets)

template <int D, int NF, int NM, bool PIECES, int PASSES>
__global__ __launch_bounds__(kErrThreads) void profile_error_kernel(const float* ws, const float2* stats, const int32_t* rows,
                                                                    int BH, int t, int n_full, int n_masked, float scale_log2, int off,
                                                                    int video_end, float2* partial, unsigned* tickets,
                                                                    uint8_t* labels, float* mse, unsigned n_blocks, PieceArgsIf<PIECES> pieces) {
  constexpr int LANES = D / 4, ROWS = err_rows(D);
  const int bh = blockIdx.y;
  const int c = threadIdx.x % LANES;
  // The parts of a pass: loads of all of them, and the pass reassembled from those that `of` names.
  auto load = [&](auto parts_c, int slot0, int parts, int row, float2* st, f32x4* x) {
    constexpr int PARTS = decltype(parts_c)::value;
#pragma unroll
    for (int r = 0; r < PARTS; ++r) {
      const size_t at = ((size_t)(slot0 + min(r, parts - 1)) * BH + bh) * t + row;
      st[r] = stats[at];
      x[r] = *reinterpret_cast<const f32x4*>(ws + at * D + 4 * c);
      if (r >= parts) st[r].y = 0.f;
    }
  };
  auto merged = [&](auto parts_c, const float2* st, const f32x4* x, auto of) -> f32x4 {
    constexpr int PARTS = decltype(parts_c)::value;
    float m_max = -3.0e38f;
#pragma unroll
    for (int r = 0; r < PARTS; ++r)
      if (of(r) && st[r].y > 0.f) m_max = fmaxf(m_max, st[r].x);
    float w[PARTS], den = 0.f;
#pragma unroll
    for (int r = 0; r < PARTS; ++r) {
      w[r] = of(r) && st[r].y > 0.f ? st[r].y * __builtin_amdgcn_exp2f((st[r].x - m_max) * scale_log2) : 0.f;
      den += w[r];
    }
    const float inv = den > 0.f ? 1.0f / den : 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < PARTS; ++r)
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = __builtin_fmaf(w[r] * inv, x[r][e], o[e]);
    return o;
  };
  const std::integral_constant<int, NF> full_parts;
  const std::integral_constant<int, NM> masked_parts;
  auto all = [](int) { return true; };
  float acc_s = 0.f, acc_t = 0.f;
#pragma unroll 1
  for (int pass = 0; pass < PASSES; ++pass) {
    const int own = (blockIdx.x * PASSES + pass) * ROWS + (int)threadIdx.x / LANES, row = min(own, t - 1);
    const int n = rows[row];
    const bool video = n >= off && n < video_end;
    float2 st[NF], st_m[NM];
    f32x4 x[NF], x_m[NM];
    f32x4 f, os;
    load(full_parts, 0, n_full, row, st, x);
    if constexpr (PIECES) {
      load(masked_parts, n_full, n_masked, row, st_m, x_m);
      int first = 0, last = 0;
      pieces.rule.window_slots(pieces.plan, video ? (n - off) / pieces.rule.P : 0, pieces.bn, first, last);
      const int kept = n_full > pieces.plan.n_full + 2 ? n_full - 1 : -1;
      f = merged(full_parts, st, x, all);
      os = merged(full_parts, st, x, [&](int r) { return (r >= first && r <= last) || r == kept; });
    } else {
      f = merged(full_parts, st, x, all);
      load(masked_parts, n_full, n_masked, row, st_m, x_m);
      os = merged(masked_parts, st_m, x_m, all);
      load(masked_parts, n_full + n_masked, n_masked, row, st_m, x_m);
    }
    const f32x4 ot = merged(masked_parts, st_m, x_m, all);
    if (own < t && video) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float ds = f[e] - os[e], dt = f[e] - ot[e];
        acc_s = __builtin_fmaf(ds, ds, acc_s);
        acc_t = __builtin_fmaf(dt, dt, acc_t);
      }
    }
  }
  __shared__ float2 wave_part[kErrThreads / 64];
  acc_s = wave_sum(acc_s);
  acc_t = wave_sum(acc_t);
  if ((threadIdx.x & 63) == 0) wave_part[threadIdx.x >> 6] = make_float2(acc_s, acc_t);
  __syncthreads();
  if (threadIdx.x >= 64) return;
  float sum_s = 0.f, sum_t = 0.f;
  for (int w = 0; w < kErrThreads / 64; ++w) {
    sum_s += wave_part[w].x;
    sum_t += wave_part[w].y;
  }
  if (n_blocks > 1 && tickets == nullptr) {
    if (threadIdx.x == 0) partial[(size_t)bh * n_blocks + blockIdx.x] = make_float2(sum_s, sum_t);
    return;
  }
  if (n_blocks > 1) {
    float* const mine = reinterpret_cast<float*>(partial + (size_t)bh * n_blocks);
    unsigned ticket = 0;
    if (threadIdx.x == 0) {
      __hip_atomic_store(mine + 2 * blockIdx.x, sum_s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(mine + 2 * blockIdx.x + 1, sum_t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      ticket = __hip_atomic_fetch_add(tickets + bh, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (__builtin_amdgcn_readfirstlane(ticket) != n_blocks - 1) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");      // for the lanes that took no ticket
    sum_s = sum_t = 0.f;
    for (unsigned i = threadIdx.x; i < n_blocks; i += 64) {
      sum_s += __hip_atomic_load(mine + 2 * i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      sum_t += __hip_atomic_load(mine + 2 * i + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    sum_s = wave_sum(sum_s);
    sum_t = wave_sum(sum_t);
  }
  if (threadIdx.x == 0) store_label(sum_s, sum_t, bh, t, D, labels, mse);
}

// MSE_s, MSE_t and the label from the partial sums of many blocks.
__global__ __launch_bounds__(64) void profile_label_kernel(const float2* partial, int n_partial, int t, int D,
                                                           uint8_t* labels, float* mse) {
  const int bh = blockIdx.x;
  float sum_s = 0.f, sum_t = 0.f;
  for (int i = threadIdx.x; i < n_partial; i += 64) {
    const float2 p = partial[(size_t)bh * n_partial + i];
    sum_s += p.x;
    sum_t += p.y;
  }
  sum_s = wave_sum(sum_s);
  sum_t = wave_sum(sum_t);
  if (threadIdx.x == 0) store_label(sum_s, sum_t, bh, t, D, labels, mse);
}

template <int D, int NF, bool PIECES>
void launch_error(const AttnArgs& a, int blocks, const PieceArgsIf<PIECES>& pieces, const float2* stats, float2* partial, uint8_t* labels, float* mse, hipStream_t stream) {
  auto kernel = a.plan.n_masked == 1 ? profile_error_kernel<D, NF, 1, PIECES, 1> : profile_error_kernel<D, NF, kMaxMaskedParts, PIECES, 1>;
  if constexpr (!PIECES)
    if (blocks == 1 && a.t > err_rows(D)) kernel = a.plan.n_masked == 1 ? profile_error_kernel<D, NF, 1, false, 2> : profile_error_kernel<D, NF, kMaxMaskedParts, false, 2>;
  hipLaunchKernelGGL(kernel, dim3(blocks, a.BH), dim3(kErrThreads), 0, stream, static_cast<const float*>(a.o), stats, a.rows,
                     a.BH, a.t, PIECES ? a.pieces : NF, a.plan.n_masked, a.scale_log2, a.off, a.video_end, partial, a.tickets, labels, mse, (unsigned)blocks, pieces);
}

template <int D>
int launch_error_parts(const Geo& g, const AttnArgs& a, int blocks, const float2* stats, float2* partial, uint8_t* labels, float* mse, hipStream_t stream) {
  (void)hipGetLastError();
  const PieceArgs pieces = {a.plan, piece_rule(g), g.bn};
  if (a.pieces > kMaxPieces) return SVG_ERR_UNSUPPORTED;
  if (a.pieces > 7) launch_error<D, kMaxPieces, true>(a, blocks, pieces, stats, partial, labels, mse, stream);
  else if (a.pieces) launch_error<D, 7, true>(a, blocks, pieces, stats, partial, labels, mse, stream);
  else switch (a.plan.n_full) {      // the numbers of parts profile_plan and profile_cut give the unmasked pass
    case 1: launch_error<D, 1, false>(a, blocks, {}, stats, partial, labels, mse, stream); break;
    case 3: launch_error<D, 3, false>(a, blocks, {}, stats, partial, labels, mse, stream); break;
    case 4: launch_error<D, 4, false>(a, blocks, {}, stats, partial, labels, mse, stream); break;
    case 6: launch_error<D, 6, false>(a, blocks, {}, stats, partial, labels, mse, stream); break;
    default: return SVG_ERR_UNSUPPORTED;
  }
  const int rc = hip_status(hipGetLastError());
  if (rc != SVG_OK || blocks == 1 || a.tickets != nullptr) return rc;
  hipLaunchKernelGGL(profile_label_kernel, dim3(a.BH), dim3(64), 0, stream, partial, blocks, a.t, D, labels, mse);
  return hip_status(hipGetLastError());
}

template <int MODE, bool PIECED = false>
int dispatch(const Geo& g, const AttnArgs& a, int rows_total, hipStream_t stream) {
  if (split_form(g, MODE, a.t)) return launch_split(g, a, MODE, stream);
  if (g.bm == 128) {
    if (MODE != kProfile && two_teams(g)) return launch_teams(g, a, MODE, stream);
    return g.D == 128 ? launch_one<128, 4, 64, MODE, 1, PIECED>(a, rows_total, stream)
                      : launch_one<64, 4, 64, MODE, 1, PIECED>(a, rows_total, stream);
  }
  if constexpr (MODE == kSparseGather) return SVG_ERR_UNSUPPORTED;
  else return g.D == 128 ? launch_one<128, 1, 32, MODE, 1, PIECED>(a, rows_total, stream)
                         : launch_one<64, 1, 32, MODE, 1, PIECED>(a, rows_total, stream);
}

// Source rows for the gathering form: table[v] = v (spatial heads), table[entries + v] = token
// row of row v of the P-outer order (text rows: themselves); padding: a row outside the tensor.
// Inside a 64-key tile the entries are kept in the order in which the threads take them: the rows
// s, s + 64 / per_thread, ... that one thread of the attention kernel stages stand together.
__global__ void row_table_kernel(int32_t* table, int entries, int per_thread_log2, int N, int off, int video_end,
                                 int F, int P, int sink) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= entries) return;
  const int place = e & 63;
  const int v = (e & ~63) + (place >> per_thread_log2) + ((place & ((1 << per_thread_log2) - 1)) << (6 - per_thread_log2));
  int same = 0x00ffffff, moved = 0x00ffffff;
  if (v < N) {
    same = v;
    moved = v >= off && v < video_end ? off + (int)transformed_to_token((unsigned)(v - off), (unsigned)F, (unsigned)P, sink) : v;
  }
  table[e] = same;
  table[entries + e] = moved;
}

AttnArgs base_args(const Geo& g, const void* q, const void* k, const void* v, void* o) {
  AttnArgs a = {};
  a.q = static_cast<const __bf16*>(q);
  a.k = static_cast<const __bf16*>(k);
  a.v = static_cast<const __bf16*>(v);
  a.o = o;
  a.N = g.N; a.nk = g.nk; a.BH = g.B * g.H;
  a.scale_log2 = g.scale * 1.4426950408889634f;
  a.off = g.off; a.video_end = g.video_end; a.F = g.F; a.P = g.P;
  a.w_s = g.w_s; a.w_t = g.w_t; a.sink = g.sink;
  a.blocks_log2 = g.bm == 128 ? 2 : 0;
  a.halves_log2 = g.bn == 64 ? 1 : 0;
  a.inv_P = 0xffffffffu / (unsigned)g.P;
  a.order = p_outer(g);
  return a;
}

}  // namespace

// Equal blocks, one more or less to an XCD, except where whole blocks to all XCDs leave no more tiles than an XCD has compute units: one XCD then
// has a tile to each of its compute units behind the others, and its neighbours in L2 stay 64.  512 k + r tiles, blocks of 64 against equal ones: r = 1-32
// 109.6 -> 114.2 us (27 heads of 19 tiles, head dimension 128; 58.5 -> 61.4 at 64), 1511 -> 1610 (60 of 60), 0.94-1.00 in 40 calls; r = 40-128 146.2 -> 136.1 (24 of 23; 92.3 -> 73.6),
// 187.1 -> 182.2 (56 of 19; 110.8 -> 97.3), 1.01-1.32 in 19.  With 32-row tiles 0.98-1.00 and 0.98-1.25.
namespace attn {
int dense_cohort(int tiles, int most) {
  const int blocks = (tiles + 8 * most - 1) / (8 * most);
  return blocks > 1 && tiles - (blocks - 1) * 8 * most <= kXcdUnits ? most : (tiles + 8 * blocks - 1) / (8 * blocks);
}
}  // namespace attn

int launch_attention(const Geo& g, const void* q, const void* k, const void* v, const void* k_t, const void* v_t,
                     void* o, const uint8_t* labels, const int32_t* row_ptr_s, const int32_t* col_idx_s,
                     const int32_t* row_ptr_t, const int32_t* col_idx_t, bool sparse,
                     bool qo_token_order, bool element_mask, int32_t* row_table, hipStream_t stream) {
  AttnArgs a = base_args(g, q, k, v, o);
  a.k_t = static_cast<const __bf16*>(k_t);
  a.v_t = static_cast<const __bf16*>(v_t);
  a.labels = labels;
  a.qo_token_order = sparse && qo_token_order ? 1 : 0;
  a.row_ptr[0] = row_ptr_s; a.col_idx[0] = col_idx_s;
  a.row_ptr[1] = labels ? row_ptr_t : row_ptr_s; a.col_idx[1] = labels ? col_idx_t : col_idx_s;      // (read beside the others, without labels not used)
  if (sparse && row_table) {
    // k and v in token order: build the row table, then the gathering form (the split form needs no table)
    if (element_mask || g.bm != 128) return SVG_ERR_UNSUPPORTED;
    if (split_form(g, kSparseGather, 0)) return launch_split(g, a, kSparseGather, stream);
    const int entries = g.nk * g.bn;
    (void)hipGetLastError();
    hipLaunchKernelGGL(row_table_kernel, dim3((entries + 255) / 256), dim3(256), 0, stream, row_table, entries,
                       g.D == 128 ? 2 : 1, g.N, g.off, g.video_end, g.F, g.P, g.sink);
    const int rc = hip_status(hipGetLastError());
    if (rc != SVG_OK) return rc;
    a.row_table = row_table;
    return dispatch<kSparseGather>(g, a, g.N, stream);
  }
  if (sparse && element_mask) return dispatch<kSparseExact>(g, a, g.N, stream);
  return sparse ? dispatch<kSparse>(g, a, g.N, stream) : dispatch<kDense>(g, a, g.N, stream);
}

int launch_profile(const Geo& g, const void* q, const void* k, const void* v, const int32_t* rows,
                   int t, uint8_t* labels, float* mse, float* workspace, hipStream_t stream) {
  AttnArgs a = base_args(g, q, k, v, workspace);
  a.rows = rows;
  a.t = t;
  // workspace: fp32 outputs [slots][BH][t][D] (parts of the unmasked, the spatial and the
  // temporal pass, or pieces of the unmasked and parts of the temporal one), statistics float2 [slots][BH][t], partial error sums float2
  // [BH][ceil(t/16)], row order int32 [t]
  const bool split = split_form(g, kProfile, t);
  a.plan = profile_cut(g, t, profile_plan(g, t), split);
  int ns = a.plan.slots();
  ProfilePlan cut;
  if (!split && (a.pieces = profile_pieces(g, t, a.plan, &cut)) != 0) {
    a.plan = cut;
    ns = a.pieces + cut.n_masked;
  }
  // Rows in equal numbers, or in whole wavefronts of 32 where that makes no group more than a tenth larger: the temporal pass of the largest is
  // the longest chain.  Equal numbers against 32s: 1191 rows 2567 -> 2495 us at 24 heads of 119056 tokens, but 140 rows in two groups (70, or 96
  // and 44) 97 -> 107 us at 30 heads of 6300; 328 rows in three and 451 in four (17 and 13 % larger) the same.
  const int groups = (t + g.bm - 1) / g.bm, even = (t + groups - 1) / groups, largest = 32 * (((t + 31) / 32 + groups - 1) / groups);
  a.rows_per_group = 10ll * largest <= 11ll * even ? 0 : even;
  const size_t out_floats = (size_t)ns * a.BH * t * g.D;
  float2* stats = reinterpret_cast<float2*>(workspace + out_floats);
  float2* partial = stats + (size_t)ns * a.BH * t;
  a.stats = stats;
  // profile_workspace_bytes keeps room for ceil(t / 16) partial sums per head, which is more than the blocks wherever there are several: the tickets lie behind them
  const int blocks = error_blocks(g, t, a.plan, a.pieces);
  if (error_tickets(g, blocks)) a.tickets = reinterpret_cast<unsigned*>(partial + (size_t)a.BH * blocks);
  if (split ? !split_sorts_rows(t) : t > 2 * g.bm) {
    // (a workgroup sorts as many rows as it has threads)
    int32_t* order = reinterpret_cast<int32_t*>(partial + (size_t)a.BH * ((t + 15) / 16));
    a.order_t = order;
    (void)hipGetLastError();
    hipLaunchKernelGGL(profile_order_kernel, dim3(1), dim3(1024), 0, stream, rows, t, g.off, g.video_end,
                       g.P, order);
    const int rc = hip_status(hipGetLastError());
    if (rc != SVG_OK) return rc;
  }
  const int rc = a.pieces ? dispatch<kProfile, true>(g, a, t, stream) : dispatch<kProfile>(g, a, t, stream);
  if (rc != SVG_OK) return rc;
  return g.D == 128 ? launch_error_parts<128>(g, a, blocks, stats, partial, labels, mse, stream)
                    : launch_error_parts<64>(g, a, blocks, stats, partial, labels, mse, stream);
}

}  // namespace svg
