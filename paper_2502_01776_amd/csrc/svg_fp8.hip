// FP8 variant of the block-sparse attention pass (Sec. 4.3 "Quantization", Sec. 5.2) for
// gfx950 (MI355X): q, k, v quantised to 8-bit floating point (OCP E4M3, one scale per head
// and tensor, scale = max|x| / 448), both matrix products on the FP8 matrix instruction
// v_mfma_f32_16x16x128_f8f6f4 (twice the bf16 rate, half the operand bytes), fp32
// accumulation and softmax, bf16 output.  Head dimension 128 and 128 x 64 tiles only (the
// paper applies FP8 only there: with head dimension 64 it gains nothing, Sec. 5.2).
//
// Two steps:
//   svg_fp8_quantize         one pass for the per-head maxima, one pass that converts and, for
//                            temporal heads, applies the layout transformation of Sec. 4.2 to
//                            k and v on the way (so the bf16 layout passes are not needed);
//                            v is written as ready-made LDS images of its 64-key tiles.
//   svg_sparse_attn_fp8_fwd  the attention kernel.  Same decomposition as the bf16 kernel
//                            (one workgroup per query tile, 32 query rows per wavefront, both
//                            products transposed so that a lane owns one query of each 16-query block).  A
//                            trip of the loop takes TWO 64-key tiles: their 128 keys are one k-step of the
//                            second product, as the 128 channels are of the first.  The
//                            attention weights are packed four to a register (E4M3 after scaling by
//                            2^8, which puts weights down to 2^-17 of the row maximum inside the
//                            format's range), and the row sums come out of the matrix unit too: one more
//                            product per 16 queries multiplies the weights with a block of
//                            ones, so the denominator is the sum of the ROUNDED weights, the
//                            result is an exact weighted mean of v rows, and 64 additions per
//                            lane and trip leave the VALU, which is the busiest unit here.
//
// The loop is skewed by one trip: with the scores of pair j in registers, a wavefront takes their
// exponentials (one long run of VALU work) and then issues the products of pair j + 1's scores
// and of pair j's output back to back (one long run of matrix work).  The operands of the first products are
// read from LDS before the exponentials, the others behind the products, and the K and V images
// come from memory straight into LDS a trip ahead, so nothing in a trip waits for LDS or memory.
//
// What bounds it (per trip and wavefront, from counters and from loops of the same instructions without
// memory): 1088 clocks of products and 242 VALU instructions; a product of this form keeps the VALU
// from issuing for about 20 of its 32 clocks, so two wavefronts per SIMD cannot do better than
// about 2260 clocks, and the kernel takes 2400.  At 119k tokens and 15 % of the tiles 13.4 ms against
// 14.8 ms on one box: 0.6 ms from the skewed loop (with 32x32x64 products and single tiles), the rest from the
// 16x16x128 form, which moves half the accumulator bytes per operation.  Taking the exponentials against a
// maximum looked at in every eighth trip only saved 15 % of the VALU work but lost 1.5 % of
// accuracy (the largest weight no longer is a power of two) and was no faster.
#include <type_traits>

#include "svg_attn_common.h"

namespace svg {

namespace {

using namespace attn;

typedef int i32x8 __attribute__((ext_vector_type(8)));

constexpr int kD = 128;                    // head dimension = bytes of a quantised row
constexpr int kBM = 128, kBN = 64;
constexpr int kCohort = 64;
constexpr float kE4M3Max = 448.0f;
constexpr float kWeightShift = 8.0f;       // attention weights are stored as 2^8 * exp(s - reference)

// LDS image of a key tile.  K: 64 rows of 128 bytes; 16-byte piece p of row n sits at piece
// p ^ k_swizzle(n) (two rows share the 64 banks).  A ds_read_b128 serves lanes 0-3, 12-15 and 20-27
// together (and the others in groups of the same form), here rows m .. m + 7 and m + 32 .. m + 39, half of them
// at one channel piece and half two pieces on; with this swizzle they fall on different banks.
__device__ constexpr int k_swizzle(int n) { return (((n >> 1) & 1) | (n & 4)) ^ ((n & 32) ? 6 : 0); }
// V^T: [half-wave g][channel d][32 key slots]; slot i = 4 j + c of half-wave g is key
// 32 (j / 4) + 8 (j % 4) + 4 g + c, the key whose weight sits in byte c of register j of
// the packed weights.  The two 16-byte halves of a channel's 32 bytes are swapped for
// channels with bit 3 set, which makes the operand reads conflict-free.
constexpr int kTileBytes = kBN * kD;       // bytes of one tile in k8, in v8t and of each image (8192)
constexpr int kPairBytes = 2 * kTileBytes; // a trip of the attention kernel takes two tiles

__host__ __device__ constexpr int v_slot_key(int g, int i) {
  return 32 * ((i >> 2) >> 2) + 8 * ((i >> 2) & 3) + 4 * g + (i & 3);
}

// --------------------------------------------------------------------------------------------
// Quantisation
// --------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void fp8_zero_kernel(unsigned* p, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0u;
}

constexpr int kAmaxPieces = 16;            // 16-byte pieces per thread

// Largest magnitude of each (tensor, head): bf16 magnitudes compare like their bit patterns.
// Heads of up to 1024 rows take one block of 1024 threads, which writes the maximum itself; longer ones
// several blocks of 256 that meet in an atomic maximum, for which the words are cleared first (a launch that
// is nothing beside a pass over a long head; without it a whole layer of 960 rows and 6 heads takes 61.9
// instead of 62.5 us).
template <int THREADS>
__global__ __launch_bounds__(THREADS) void fp8_amax_kernel(const u32x4* q, const u32x4* k, const u32x4* v,
                                                           unsigned long long pieces_per_head, unsigned* amax,
                                                           int BH) {
  const int bh = blockIdx.y, tensor = blockIdx.z;
  const u32x4* src = (tensor == 0 ? q : tensor == 1 ? k : v) + (size_t)bh * pieces_per_head;
  const unsigned long long base = (unsigned long long)blockIdx.x * (THREADS * kAmaxPieces) + threadIdx.x;
  unsigned m = 0;
#pragma unroll 4
  for (int i = 0; i < kAmaxPieces; ++i) {
    const unsigned long long u = base + (unsigned long long)i * THREADS;
    if (u < pieces_per_head) {
      const u32x4 x = __builtin_nontemporal_load(&src[u]);
#pragma unroll
      for (int w = 0; w < 4; ++w) m = max(m, max(x[w] & 0x7fffu, (x[w] >> 16) & 0x7fffu));
    }
  }
  __shared__ unsigned red[THREADS];
  red[threadIdx.x] = m;
  __syncthreads();
  for (unsigned step = THREADS / 2; step > 0; step >>= 1) {
    if (threadIdx.x < step) red[threadIdx.x] = max(red[threadIdx.x], red[threadIdx.x + step]);
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  if (gridDim.x == 1) amax[tensor * BH + bh] = red[0] << 16;      // as fp32 bits
  else atomicMax(&amax[tensor * BH + bh], red[0] << 16);
}

struct QuantArgs {
  const u32x4* in[3];          // q, k, v: bf16 [B,H,N,128] in token order
  unsigned char* q8;           // [B,H,N,128]
  unsigned char* k8;           // [B,H,nk*64,128], rows beyond N zero
  unsigned char* v8t;          // [B,H,nk][8192]: LDS images
  float* scales;               // [3][BH]
  const unsigned* amax;        // [3][BH] fp32 bits
  const uint8_t* labels;
  int N, BH, off, video_end, F, P, sink;
};

// One workgroup converts one 64-row tile of one head of one tensor.
__global__ __launch_bounds__(256) void fp8_quantize_kernel(QuantArgs a) {
  const int tile = blockIdx.x, bh = blockIdx.y, tensor = blockIdx.z;
  const int tid = threadIdx.x;
  const float amax = __uint_as_float(a.amax[tensor * a.BH + bh]);
  const float scale = amax > 0.f ? amax / kE4M3Max : 1.0f;
  if (tile == 0 && tid == 0) a.scales[tensor * a.BH + bh] = scale;
  const float inv_scale = 1.0f / scale;      // codes = nearest even of x * (1 / scale), both in fp32
  // k and v of temporal heads are written in P-outer order: row m holds token off + f P + p
  // with m = off + p F + f (Sec. 4.2); q stays in token order (the attention kernel gathers it)
  const bool permute = tensor != 0 && a.labels != nullptr && a.labels[bh] == SVG_HEAD_TEMPORAL;
  const u32x4* src = a.in[tensor] + (size_t)bh * a.N * (kD / 8);

  __shared__ __attribute__((aligned(16))) unsigned char tile_bytes[kBN * (kD + 4)];   // v only: [key][d], rows padded
  uint2 packed[4];
  int row_of[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int u = tid + 256 * i;                 // piece: row u / 16, channels 8 (u % 16) ..
    const int rr = u >> 4, c = u & 15;
    const int m = tile * kBN + rr;
    row_of[i] = m;
    u32x4 x = {0u, 0u, 0u, 0u};
    if (m < a.N) {
      int s = m;
      if (permute && m >= a.off && m < a.video_end) {
        s = a.off + (int)transformed_to_token((unsigned)(m - a.off), (unsigned)a.F, (unsigned)a.P, a.sink);
      }
      x = __builtin_nontemporal_load(&src[(size_t)s * (kD / 8) + c]);
    }
    unsigned out[2];
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      float y[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const unsigned word = x[2 * w + (e >> 1)];
        const float val = __uint_as_float((e & 1) ? (word & 0xffff0000u) : (word << 16));
        y[e] = fminf(fmaxf(val * inv_scale, -kE4M3Max), kE4M3Max);
      }
      int pk = __builtin_amdgcn_cvt_pk_fp8_f32(y[0], y[1], 0, false);
      pk = __builtin_amdgcn_cvt_pk_fp8_f32(y[2], y[3], pk, true);
      out[w] = (unsigned)pk;
    }
    packed[i] = make_uint2(out[0], out[1]);
  }
  if (tensor != 2) {
    unsigned char* dst = tensor == 0 ? a.q8 + (size_t)bh * a.N * kD
                                     : a.k8 + ((size_t)bh * gridDim.x) * kTileBytes;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int u = tid + 256 * i;
      if (tensor == 1 || row_of[i] < a.N)
        *reinterpret_cast<uint2*>(dst + (size_t)row_of[i] * kD + (u & 15) * 8) = packed[i];
    }
    return;
  }
  // v: transpose through LDS into the tile's image
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int u = tid + 256 * i;
    unsigned char* p = tile_bytes + (u >> 4) * (kD + 4) + (u & 15) * 8;
    *reinterpret_cast<unsigned*>(p) = packed[i].x;
    *reinterpret_cast<unsigned*>(p + 4) = packed[i].y;
  }
  __syncthreads();
  const int g = tid >> 7, d = tid & 127;
  unsigned img[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    unsigned w = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) w |= (unsigned)tile_bytes[v_slot_key(g, 4 * j + c) * (kD + 4) + d] << (8 * c);
    img[j] = w;
  }
  unsigned char* dst = a.v8t + ((size_t)bh * gridDim.x + tile) * kTileBytes + g * (kD * 32) + d * 32;
  const int sw = (d >> 3) & 1;
  *reinterpret_cast<u32x4*>(dst + 16 * sw) = u32x4{img[0], img[1], img[2], img[3]};
  *reinterpret_cast<u32x4*>(dst + 16 * (1 - sw)) = u32x4{img[4], img[5], img[6], img[7]};
}

// --------------------------------------------------------------------------------------------
// Attention
// --------------------------------------------------------------------------------------------
struct Fp8Args {
  const unsigned char* q8;
  const unsigned char* k8;
  const unsigned char* v8t;
  const float* scales;         // [3][BH]: q, k, v
  __bf16* o;                   // [B,H,N,128] bf16, token order
  const uint8_t* labels;
  const int32_t* row_ptr[2];
  const int32_t* col_idx[2];
  int N, nk, BH, nqt;
  SparseOrder so;              // which workgroup takes which (head, query tile)
  float scale_log2;            // softmax scale * log2(e), before the quantisation scales
  int off, video_end, F, P, sink, w_s, w_t;
};

template <int LW>
__global__ __launch_bounds__(256, 2) void attn_fp8_kernel(Fp8Args a) {
  constexpr int QB = 2;          // 16-query blocks per wavefront
  constexpr int KB = 8;          // 16-key blocks per pair of tiles
  constexpr int CB = kD / 16;    // 16-channel blocks of O^T
  constexpr int PF = 4;          // operands in flight ahead of the products
  __shared__ __attribute__((aligned(1024))) unsigned char lds[4 * kPairBytes];      // two pairs of K images, two of V images
  static_assert(sizeof(lds) <= 65536, "the direct loads take a 16-bit LDS address");

  // heavy query tiles first, then an eighth of each label's sequence of tiles (the same
  // dispatch order as the bf16 kernel)
  int bh = 0, grp = 0, pat = 0, cl = -1, head_cl0 = 0;
  if (!sparse_slot<LW>(a.so, a.BH, a.labels, a.row_ptr[0], a.row_ptr[1], bh, grp, pat, cl, head_cl0)) return;
  bh = __builtin_amdgcn_readfirstlane(bh);
  grp = __builtin_amdgcn_readfirstlane(grp);
  pat = __builtin_amdgcn_readfirstlane(pat);
  cl = __builtin_amdgcn_readfirstlane(cl);
  head_cl0 = __builtin_amdgcn_readfirstlane(head_cl0);

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, r = lane & 15;

  const size_t tiles_head = (size_t)bh * a.nk;
  const unsigned char* kh = a.k8 + tiles_head * kTileBytes;
  const unsigned char* vh = a.v8t + tiles_head * kTileBytes;

  // this lane's queries, one per 16-query block: position qslot in the order the tile list refers to; for a
  // temporal head that is token off + f P + p with qslot = off + p F + f (q and o stay in token order)
  int qslot[QB], io_row[QB];
  i32x8 qreg[QB];      // lane (g, r) holds channels 32 g .. + 32 of its query
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    qslot[qb] = grp * kBM + wave * 32 + qb * 16 + r;
    const int qrow = min(qslot[qb], a.N - 1);
    io_row[qb] = qrow;
    if (pat && qrow >= a.off && qrow < a.video_end)
      io_row[qb] = a.off + (int)transformed_to_token((unsigned)(qrow - a.off), (unsigned)a.F, (unsigned)a.P, a.sink);
    const unsigned char* qp = a.q8 + ((size_t)bh * a.N + io_row[qb]) * kD + g * 32;
    const i32x4 lo = *reinterpret_cast<const i32x4*>(qp), hi = *reinterpret_cast<const i32x4*>(qp + 16);
    qreg[qb] = i32x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  }
  // logits in units of log2: s_raw * c with the two quantisation scales folded in.  The product of tiny scales
  // underflows to zero; the smallest normal number in its place leaves the logits zero as well, but a masked
  // score times it stays -inf, where times zero it would be NaN.
  const float c_product = a.scale_log2 * a.scales[bh] * a.scales[a.BH + bh];
  const float c_log2 = c_product == 0.f ? 0x1p-126f : c_product;
  const float v_scale = a.scales[2 * a.BH + bh];

  // ---- tile cursor: the query tile's list row, walked cyclically from the cohort's common
  // starting tile
  const int32_t* rp = a.row_ptr[pat];
  const int32_t* cols = a.col_idx[pat];
  const int lbeg = __builtin_amdgcn_readfirstlane(rp[grp]);
  const int lend = __builtin_amdgcn_readfirstlane(rp[grp + 1]);
  const int entries = lend - lbeg;
  int start = 0;
  // cohort size by geometry: the largest power of two for which the anchor lies inside every
  // member's key window; short windows start at their own first tile
  const int win_tiles = (int)min((pat ? (2LL * a.w_t + 1) * a.F : (2LL * a.w_s + 1) * a.P) / kBN, 1LL << 20);
  int cs = kCohort;
  while (cs > 1 && (cs - 1) * (kBM / kBN) >= win_tiles) cs >>= 1;
  if (entries > 1 && cl >= 0 && cs >= 8) {
    const int first_video_tile = (a.off + kBN - 1) / kBN;
    const int top = a.so.g_lo + min(cl | (cs - 1), head_cl0 + a.so.nl - 1) - head_cl0;
    const int c_first = cols[lbeg], c_last = cols[lend - 1];
    int anchor = -1;
    for (int j = rp[top], e = min(rp[top + 1], rp[top] + 8); j < e; ++j)
      if (cols[j] >= first_video_tile) { anchor = cols[j]; break; }
    if (anchor >= c_first && anchor <= c_last) {
      int lo = 0, hi = entries;
      const int from_front = anchor - c_first;
      if (from_front < entries && cols[lbeg + from_front] == anchor) {
        lo = from_front;
      } else {
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (cols[lbeg + mid] < anchor) lo = mid + 1; else hi = mid;
        }
      }
      if (lo < entries && cols[lbeg + lo] == anchor) start = lo;
    }
    start = __builtin_amdgcn_readfirstlane(start);
  }
  TileList list;
  list.open(cols + lbeg, entries, start);

  // ---- staging: both tile images are 8 KB, two 16-byte pieces per thread each, copied by the load
  // unit: piece u = tid + 256 i of an image is thread tid's i-th load, K's swizzle is applied on
  // the memory side
  const unsigned lds_wave = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_byte*)lds + wave * 1024);
  const int k_src = (tid >> 3) * kD + (((tid & 7) ^ k_swizzle(tid >> 3)) << 4), v_src = tid * 16;
  auto load_image = [&](const unsigned char* images, int tile, int voffset0, int voffset1, unsigned dst) {
    const u32x4 rsrc = buffer_words(images + (size_t)__builtin_amdgcn_readfirstlane(tile) * kTileBytes, kTileBytes);
    load_to_lds(rsrc, voffset0, voffset1, 0, 4096, dst, 4096);
  };
  // (a list of odd length ends with a pair whose second half repeats the first and is masked)
  struct Pair { int a, b; };
  auto load_k = [&](Pair t, int j) {
    const unsigned dst = lds_wave + (j & 1) * kPairBytes;
    load_image(kh, t.a, k_src, k_src ^ 96, dst);            // the swizzles of rows n and n + 32 differ by 6
    load_image(kh, t.b == kNoTile ? t.a : t.b, k_src, k_src ^ 96, dst + kTileBytes);
  };
  auto load_v = [&](Pair t, int j) {
    const unsigned dst = lds_wave + (2 + (j & 1)) * kPairBytes;
    load_image(vh, t.a, v_src, v_src, dst);
    load_image(vh, t.b == kNoTile ? t.a : t.b, v_src, v_src, dst + kTileBytes);
  };
  auto next_pair = [&]() -> Pair {
    const int first = list.next();
    return Pair{first, first == kNoTile ? kNoTile : list.next()};
  };

  // ---- operand reads.  A lane's keys have to be those of 16 consecutive bytes of the V image, so
  // row m of the kb-th 16-key block of a tile is key 8 kb + m % 8 + 32 (m / 8): lane (g, r) then gets the
  // scores of keys 8 kb + 4 (g % 2) + {0..3} + 32 (g / 2), which is what half g % 2, piece g / 2 of the image holds.
  const int k_row = (r & 7) + 32 * (r >> 3);
  const int k_rd = k_row * kD + (((2 * g) ^ k_swizzle(k_row)) << 4);       // the second piece differs in bit 4
  const int v_rd = (g & 1) * (kD * 32) + r * 32 + 16 * ((g >> 1) ^ ((r >> 3) & 1));
  auto read32 = [](const unsigned char* lo, const unsigned char* hi) -> i32x8 {
    const i32x4 x = *reinterpret_cast<const i32x4*>(lo);
    const i32x4 y = *reinterpret_cast<const i32x4*>(hi);
    return i32x8{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
  };
  auto k_operand = [&](int j, int kb) -> i32x8 {
    const unsigned char* p = lds + (j & 1) * kPairBytes + (kb >> 2) * kTileBytes + (kb & 3) * 8 * kD;
    return read32(p + k_rd, p + (k_rd ^ 16));
  };
  auto v_operand = [&](int j, int cb) -> i32x8 {
    const unsigned char* p = lds + (2 + (j & 1)) * kPairBytes + cb * 512 + v_rd;
    return read32(p, p + kTileBytes);
  };

  f32x4 oacc[CB][QB], lacc[QB], sacc[KB][QB];
  float m_run[QB];           // running row maximum, raw logits
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    m_run[qb] = kNegBig;
    lacc[qb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) oacc[cb][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  i32x8 ones;          // 32 x E4M3 1.0
#pragma unroll
  for (int j = 0; j < 8; ++j) ones[j] = 0x38383838;
  asm volatile("" : "+v"(ones));
  const bool ragged = (a.N % kBN) != 0;

  auto product = [](const i32x8& x, const i32x8& y, const f32x4& z) -> f32x4 {
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(x, y, z, 0, 0, 0, 0, 0, 0);
  };
  // S^T of one 16-key block: all 128 channels are one step
  auto score_block = [&](const i32x8& k_op, int kb) {
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) sacc[kb][qb] = product(k_op, qreg[qb], f32x4{0.f, 0.f, 0.f, 0.f});
  };
  // keys beyond N in the last tile, and all keys of a missing second tile
  auto mask_pair = [&](Pair t) {
    if (t.b != kNoTile && !(ragged && (t.a == a.nk - 1 || t.b == a.nk - 1))) return;
    int lim[2] = {a.N - t.a * kBN - 32 * (g >> 1) - 4 * (g & 1), t.b == kNoTile ? -kBN : a.N - t.b * kBN - 32 * (g >> 1) - 4 * (g & 1)};
    asm volatile("" : "+v"(lim[0]), "+v"(lim[1]));      // keeps this rarely taken code out of every trip
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (8 * (kb & 3) + i >= lim[kb >> 2]) {
#pragma unroll
          for (int qb = 0; qb < QB; ++qb) sacc[kb][qb][i] = -INFINITY;
        }
  };

  // ---- main loop.  Trip j holds the scores of pair j; it takes their exponentials, and then issues the
  // products of pair j + 1's scores and of pair j's output as one batch (see the top of the file).
  // LDS holds K of pair j + 1 and V of pair j, with K of j + 2 and V of j + 1 in flight.
  auto trip = [&](auto more_c, int j, Pair following) {
    constexpr bool MORE = decltype(more_c)::value;
    i32x8 opnd[PF];
#pragma unroll
    for (int i = 0; i < PF; ++i) opnd[i] = MORE ? k_operand(j + 1, i) : v_operand(j, i);
    // softmax, two queries per lane: weights 2^8 exp(s - maximum), four keys to a register
    i32x8 pb[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      float tmax = sacc[0][qb][0];
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int i = 0; i < 4; ++i) tmax = fmaxf(tmax, sacc[kb][qb][i]);
      tmax = quarters_max(tmax);
      if (__builtin_amdgcn_ballot_w64(tmax > m_run[qb]) != 0) {      // some row of the block has a new maximum
        const float m_new = fmaxf(m_run[qb], tmax);
        const float alpha = __builtin_amdgcn_exp2f((m_run[qb] - m_new) * c_log2);
        m_run[qb] = m_new;
        lacc[qb][0] *= alpha;                  // (only this element is ever read)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
          for (int i = 0; i < 4; ++i) oacc[cb][qb][i] *= alpha;
      }
      const float mc = m_run[qb] * c_log2 - kWeightShift;
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        float p[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[kb][qb][i], c_log2, -mc));
        // (the first conversion writes the low half of its destination and keeps the rest: giving it
        // a value that dies here as the "rest" saves a register clear; the second one fills the high half)
        const int w = __builtin_amdgcn_cvt_pk_fp8_f32(p[0], p[1], (int)__float_as_uint(p[0]), false);
        pb[qb][kb] = __builtin_amdgcn_cvt_pk_fp8_f32(p[2], p[3], w, true);
      }
    }
    __builtin_amdgcn_s_setprio(1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) lacc[qb] = product(ones, pb[qb], lacc[qb]);
    __builtin_amdgcn_sched_barrier(0);
    if (MORE) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) {
        const i32x8 k_op = opnd[kb % PF];
        score_block(k_op, kb);
        opnd[kb % PF] = kb + PF < KB ? k_operand(j + 1, kb + PF) : v_operand(j, kb + PF - KB);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const i32x8 v_op = opnd[cb % PF];
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) oacc[cb][qb] = product(v_op, pb[qb], oacc[cb][qb]);
      if (cb + PF < CB) opnd[cb % PF] = v_operand(j, cb + PF);
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_setprio(0);
    if (MORE) mask_pair(following);
  };

  Pair now = next_pair(), next1 = next_pair();
  if (now.a != kNoTile) {
    load_k(now, 0);
    load_v(now, 0);
  }
  if (next1.a != kNoTile) load_k(next1, 1);
  wait_loads_to_lds<0>();
  __syncthreads();
  asm volatile("" ::"v"(qreg[0]), "v"(qreg[1]));
  if (now.a != kNoTile) {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) score_block(k_operand(0, kb), kb);
    mask_pair(now);
  }
  __syncthreads();         // the first trip stages pair 2 over pair 0's keys
  int j = 0;
  for (; next1.a != kNoTile; ++j) {
    const Pair next2 = next_pair();
    if (next2.a != kNoTile) load_k(next2, j + 2);
    load_v(next1, j + 1);
    trip(std::true_type{}, j, next1);
    wait_loads_to_lds<0>();
    barrier_loads_done();
    now = next1;
    next1 = next2;
  }
  if (now.a != kNoTile) trip(std::false_type{}, j, now);

  // ---- epilogue: oacc[cb][qb][i] = O[query 16 qb + r][16 cb + 4 g + i]; lacc[qb][0] = row sum
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const float l_tot = lacc[qb][0];
    const float inv = l_tot > 0.f ? v_scale / l_tot : 0.f;
    if (qslot[qb] < a.N) {
      __bf16* op = a.o + ((size_t)bh * a.N + io_row[qb]) * kD;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
        *reinterpret_cast<bf16x4*>(op + cb * 16 + 4 * g) = __builtin_convertvector(oacc[cb][qb] * inv, bf16x4);
    }
  }
}

}  // namespace

int launch_fp8_quantize(const Geo& g, const void* q, const void* k, const void* v, const uint8_t* labels,
                        void* q8, void* k8, void* v8t, float* scales, hipStream_t stream) {
  const int BH = g.B * g.H;
  if (BH > 65535) return SVG_ERR_UNSUPPORTED;
  unsigned* amax = reinterpret_cast<unsigned*>(scales + 3 * BH);
  (void)hipGetLastError();
  const unsigned long long pieces = (unsigned long long)g.N * (kD / 8);
  const u32x4 *qp = static_cast<const u32x4*>(q), *kp = static_cast<const u32x4*>(k), *vp = static_cast<const u32x4*>(v);
  if (pieces <= 1024 * kAmaxPieces) {
    hipLaunchKernelGGL(fp8_amax_kernel<1024>, dim3(1, BH, 3), dim3(1024), 0, stream, qp, kp, vp, pieces, amax, BH);
  } else {
    hipLaunchKernelGGL(fp8_zero_kernel, dim3((3 * BH + 255) / 256), dim3(256), 0, stream, amax, 3 * BH);
    const int rc = hip_status(hipGetLastError());
    if (rc != SVG_OK) return rc;
    const unsigned chunks = (unsigned)((pieces + 256 * kAmaxPieces - 1) / (256 * kAmaxPieces));
    hipLaunchKernelGGL(fp8_amax_kernel<256>, dim3(chunks, BH, 3), dim3(256), 0, stream, qp, kp, vp, pieces, amax, BH);
  }
  const int rc = hip_status(hipGetLastError());
  if (rc != SVG_OK) return rc;
  QuantArgs a;
  a.in[0] = static_cast<const u32x4*>(q);
  a.in[1] = static_cast<const u32x4*>(k);
  a.in[2] = static_cast<const u32x4*>(v);
  a.q8 = static_cast<unsigned char*>(q8);
  a.k8 = static_cast<unsigned char*>(k8);
  a.v8t = static_cast<unsigned char*>(v8t);
  a.scales = scales;
  a.amax = amax;
  a.labels = labels;
  a.N = g.N; a.BH = BH; a.off = g.off; a.video_end = g.video_end; a.F = g.F; a.P = g.P; a.sink = g.sink;
  hipLaunchKernelGGL(fp8_quantize_kernel, dim3(g.nk, BH, 3), dim3(256), 0, stream, a);
  return hip_status(hipGetLastError());
}

int launch_fp8_attention(const Geo& g, const void* q8, const void* k8, const void* v8t, const float* scales,
                         void* o, const uint8_t* labels, const int32_t* row_ptr_s, const int32_t* col_idx_s,
                         const int32_t* row_ptr_t, const int32_t* col_idx_t, hipStream_t stream) {
  Fp8Args a = {};
  a.q8 = static_cast<const unsigned char*>(q8);
  a.k8 = static_cast<const unsigned char*>(k8);
  a.v8t = static_cast<const unsigned char*>(v8t);
  a.scales = scales;
  a.o = static_cast<__bf16*>(o);
  a.labels = labels;
  a.row_ptr[0] = row_ptr_s; a.col_idx[0] = col_idx_s;
  a.row_ptr[1] = row_ptr_t; a.col_idx[1] = col_idx_t;
  a.N = g.N; a.nk = g.nk; a.BH = g.B * g.H;
  a.nqt = g.nq;
  // (no stride in the dispatch order: this kernel starts the query tiles of a cohort at a common key tile
  // instead, which measured 0.6-1.8 % faster here than the stride with or without that start)
  a.so = sparse_order(a.BH, a.nqt, kBM, g.off, g.video_end, g.N, 1 << 24);
  a.scale_log2 = g.scale * 1.4426950408889634f;
  a.off = g.off; a.video_end = g.video_end; a.F = g.F; a.P = g.P; a.sink = g.sink;
  a.w_s = g.w_s; a.w_t = g.w_t;
  const unsigned grid = sparse_grid(a.so, a.BH);
  (void)hipGetLastError();
  if (a.BH > 64) hipLaunchKernelGGL(attn_fp8_kernel<kWideLabelWords>, dim3(grid), dim3(256), 0, stream, a);
  else hipLaunchKernelGGL(attn_fp8_kernel<1>, dim3(grid), dim3(256), 0, stream, a);
  return hip_status(hipGetLastError());
}

}  // namespace svg
