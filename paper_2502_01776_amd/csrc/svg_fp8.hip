// FP8 variant of the block-sparse attention pass (Sec. 4.3 "Quantization", Sec. 5.2) for
// gfx950 (MI355X): q, k, v quantised to 8-bit floating point (OCP E4M3, one scale per head
// and tensor, scale = max|x| / 448), both matrix products on the FP8 matrix instruction
// v_mfma_f32_32x32x64_f8f6f4 (twice the bf16 rate, half the operand bytes), fp32
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
//                            products transposed so that a lane owns one query), but a whole
//                            64-key tile is ONE k-step of the second product, the attention
//                            weights are packed four to a register (E4M3 after scaling by 2^8,
//                            which puts weights down to 2^-17 of the row maximum inside the
//                            format's range), and the row sums come out of the matrix unit too:
//                            a ninth, smaller product per tile multiplies the weights with
//                            ones, so the denominator is the sum of the ROUNDED weights, the
//                            result is an exact weighted mean of v rows, and 32 additions per
//                            lane and tile leave the VALU, which is the busiest unit here.
//
// The loop holds the scores of tile j and the weights of tile j - 1: the products of tile j + 1's scores and of tile j - 1's row sums and
// output are issued one by one with the exponentials of tile j in between, four keys behind each, so that a wavefront covers its
// own VALU work and two to a SIMD seldom want the same unit.  K and V images come from memory straight into LDS, two tiles to a
// barrier.  At 119k tokens and 15 % of the tiles 12.81 ms where the form before, exponentials and products in phases of their own, took 13.51, and one
// barrier a tile 12.95; 7 heads of 8187 rows 119.9 -> 100.4 us, 9 of 3335 43.7 -> 36.0.  Tiles go in pairs.  An odd list was rounded up by a tile of zeros behind it, and the one of zeros
// in front of every list cost it products too, so short lists lost to the form before (61 calls of 184-18676 rows 1.05 times its time, up to 1.16); now the first tile
// of an odd list is weighted by itself before the pairs: 0.998 of the form before, 81 heads of 539 rows 16.9 -> 15.1 us, 20 of 4000 54.1 -> 51.8, 119k tokens 13.65 -> 13.57 ms.  Leaving
// the loop between the two tiles of the last pair instead made the loop worse (119k 13.90 -> 14.41).  Even lists of two to four tiles remain up to 1.13 times the form before.  In counters 2.89e7 cycles at 2.04 GHz became
// 2.64e7 at 1.92: the clock falls as the units fill, matrix unit 49 -> 51 % of the cycles, VALU 64 -> 70 %; waiting for data and barriers a wavefront spends 17 % of its
// time, waiting for issue 31 %.  A raised wave priority from the first product to the last: 12.93 ms, and text-row
// tiles taken in parts, which run beside other workgroups, late (2 heads of 51074 rows 311 -> 334 us).  The maximum of the next tile
// taken behind its products instead of in front of the exponentials: no difference.
//
// The weights of a tile are rounded against the row maximum up to and including that tile, so that the
// largest weight of a tile that brings a new maximum is a power of two, i.e. exact.  Two tiles to a trip on
// v_mfma_f32_16x16x128_f8f6f4 (half the accumulator bytes per operation) took 0.90 of the time of the tile-by-tile
// kernel where this takes 0.93, but give two tiles one maximum and half of those weights a rounding error: 0.4-7 % more
// error against exact weights in spatial heads.  With the first of two tiles added by itself wherever the second
// exceeds its maximum the error was the same as here and the time that of the tile-by-tile kernel.  Looking at the
// maximum in every eighth trip only saved 15 % of the VALU work, lost 1.5 % of accuracy and was no faster.
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
// p ^ k_swizzle(n) (two rows share the 64 banks), so that the 16 lanes a ds_read_b128 serves
// together (consecutive keys, same channel piece) fall on different banks.
__device__ constexpr int k_swizzle(int n) { return (n >> 1) & 7; }
// V^T: [half-wave g][channel d][32 key slots]; slot i = 4 j + c of half-wave g is key
// 32 (j / 4) + 8 (j % 4) + 4 g + c, the key whose weight sits in byte c of register j of
// the packed weights.  The two 16-byte halves of a channel's 32 bytes are swapped for
// channels with bit 3 set, which makes the operand reads conflict-free.
constexpr int kTileBytes = kBN * kD;       // bytes of one tile in k8, in v8t and of each image (8192)
constexpr int kStages = 4;                 // K and V images held in LDS (a power of two)

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
// instead of 62.5 us).  The lanes of a wavefront exchange their maxima in registers, where ten rounds through LDS with a barrier each took
// 4-5 us of a short block: the whole quantisation of 24 heads of 960 rows 16.5 -> 12.5 us, 20 of 1442 19.5 -> 14.1, 8 of 3910 20.1 -> 15.2, 12 of 8000
// 39.6 -> 37.0, 24 of 119056 1000 -> 998; 40 of 32760 441 -> 445 on one
// card, 435 -> 437 on another (24 of them 268 -> 269, 263 -> 263).  Four or sixteen loads at a time, four in a loop, and tiles converted in the reverse order, those read last
// first, are no faster there (443-445 and 438-440); four in a loop cost short heads 6 %.
template <int THREADS>
__global__ __launch_bounds__(THREADS, THREADS == 1024 ? 8 : 4) void fp8_amax_kernel(const u32x4* q, const u32x4* k, const u32x4* v,
                                                           unsigned long long pieces_per_head, unsigned* amax,
                                                           int BH) {
  const int bh = blockIdx.y, tensor = blockIdx.z;
  const u32x4* src = (tensor == 0 ? q : tensor == 1 ? k : v) + (size_t)bh * pieces_per_head;
  const unsigned long long base = (unsigned long long)blockIdx.x * (THREADS * kAmaxPieces) + threadIdx.x;
  unsigned m = 0;
  // loads on their way at once: with 1024 threads what two blocks to a compute unit leave registers for (16 were one block: 97 heads of 101 rows 9.6 -> 11.4 us, now 8.9; 145 of
  // 194 13.5 -> 15.5, now 12.6; 102 of 740 28.5 -> 30.1, now 29.0; eight 9.5, 13.4 and 29.4), and none of a batch that lies behind the head
  constexpr int BATCH = THREADS == 1024 ? 4 : 8, UNROLL = THREADS == 1024 ? 1 : kAmaxPieces / BATCH;
#pragma unroll UNROLL
  for (int i0 = 0; i0 < kAmaxPieces; i0 += BATCH) {
    if (THREADS == 1024 && base - threadIdx.x + i0 * THREADS >= pieces_per_head) break;
    u32x4 x[BATCH];
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const unsigned long long u = base + (unsigned long long)(i0 + i) * THREADS;
      x[i] = u32x4{0u, 0u, 0u, 0u};
      if (u < pieces_per_head) x[i] = __builtin_nontemporal_load(&src[u]);
    }
#pragma unroll
    for (int i = 0; i < BATCH; ++i)
#pragma unroll
      for (int w = 0; w < 4; ++w) m = max(m, max(x[i][w] & 0x7fffu, (x[i][w] >> 16) & 0x7fffu));
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, d, 64));
  __shared__ unsigned red[THREADS / 64];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x != 0) return;
#pragma unroll
  for (int w = 1; w < THREADS / 64; ++w) m = max(m, red[w]);
  if (gridDim.x == 1) amax[tensor * BH + bh] = m << 16;      // as fp32 bits
  else atomicMax(&amax[tensor * BH + bh], m << 16);
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
  POuter order;                // attn_fp8_split_kernel
};

__device__ __forceinline__ f32x16 product(const i32x8& x, const i32x8& y, const f32x16& z) {
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(x, y, z, 0, 0, 0, 0, 0, 0);
}
// Row sums of the rounded weights by a 16x16x128 product: half the time and a quarter of the accumulators of a 32x32x64 product
// with ones.  Its B operand has query lane % 16 in the quarter wavefronts 0 and 2 and query 16 + lane % 16 in 1 and 3; the A
// operand has ones where the quarter of the column's keys and the quarter that receives the row agree in that, and every
// lane gets the sum over both halves of its own query's keys, in all four elements.
__device__ __forceinline__ i32x8 row_sum_operand(int lane) {
  const int x = ((lane >> 4) & 1) == ((lane >> 2) & 1) ? 0x38383838 : 0;      // E4M3 1.0
  i32x8 select;
#pragma unroll
  for (int j = 0; j < 8; ++j) select[j] = x;
  asm volatile("" : "+v"(select));
  return select;
}
__device__ __forceinline__ f32x4 row_sum(const i32x8& select, const i32x8& weights, const f32x4& z) {
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(select, weights, z, 0, 0, 0, 0, 0, 0);
}

// --------------------------------------------------------------------------------------------
// Attention of calls with few rows: as split_kernel (svg_split.hip), 32 query rows per workgroup, every fourth key tile per
// wavefront, merged through LDS.  The tiles of k8 and v8t hold whole operands in 16-byte pieces, so both go from
// memory straight to registers and nothing is staged.  6 heads of 960 rows 18.2 -> 9.9 us, 2 of 3290 rows 52.6 -> 21.8.  Two
// workgroups fit a CU: time of attn_fp8_kernel without parts of text-row tiles over time here, 1 to 48 heads of 200 to 19000 rows, 1.07-2.7 up
// to 512 groups of 32 rows.  Up to 600, where some CUs take a third, it depends on the lists: 0.98-1.5 from 4096 rows a head on, 0.77-1.03 below
// (0.73-1.33 with text rows, whose tiles attn_fp8_kernel now takes in parts).
// --------------------------------------------------------------------------------------------
constexpr int kSplitWaves = 4, kSplitRows = 32;

// lds: 64 KB.  Rows row0 .. row0 + 31 of head bh, entries [list_begin, list_end) of pattern pat's list.
__device__ __forceinline__ void fp8_split_body(const Fp8Args& a, unsigned char* const lds, const int bh, const int row0, const int pat,
                                               const int list_begin, const int list_end) {
  constexpr int PART = kSplitRows * kD * 4;      // bytes of a wavefront's O^T
  float* const tile_max = reinterpret_cast<float*>(lds);      // [2][wavefront][row]; the parts come after the last use
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, r = lane & 31;
  const int32_t* cols = (pat ? a.col_idx[1] : a.col_idx[0]) + list_begin;
  const int entries = list_end - list_begin;
  int base = 0, now = lane < entries ? cols[lane] : 0, u = wave;
  auto next_tile = [&]() -> int {
    const int n = u;
    if (n >= entries) return kNoTile;
    u += kSplitWaves;
    if (n >= base + 64) {
      base += 64;
      now = base + lane < entries ? cols[base + lane] : 0;
    }
    return __builtin_amdgcn_readlane(now, n - base);
  };

  const int qslot = row0 + r, qrow = min(qslot, a.N - 1);
  int io_row = qrow;
  if (pat && qrow >= a.off && qrow < a.video_end)
    io_row = a.off + a.order.token(qrow - a.off);
  auto read32 = [](const unsigned char* lo, const unsigned char* hi) -> i32x8 {
    const i32x4 x = *reinterpret_cast<const i32x4*>(lo);
    const i32x4 y = *reinterpret_cast<const i32x4*>(hi);
    return i32x8{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
  };
  i32x8 qreg[2];
  {
    const unsigned char* qp = a.q8 + ((size_t)bh * a.N + io_row) * kD + g * 32;
#pragma unroll
    for (int s = 0; s < 2; ++s) qreg[s] = read32(qp + s * 64, qp + s * 64 + 16);
  }
  const float c_product = a.scale_log2 * a.scales[bh] * a.scales[a.BH + bh];
  const float c_log2 = c_product == 0.f ? 0x1p-126f : c_product;      // (see attn_fp8_kernel)
  const float v_scale = a.scales[2 * a.BH + bh];
  const unsigned char* kh = a.k8 + (size_t)bh * a.nk * kTileBytes + r * kD + g * 32;
  const int sw = (r >> 3) & 1;
  const unsigned char* vh = a.v8t + (size_t)bh * a.nk * kTileBytes + g * (kD * 32) + r * 32;
  i32x8 kreg[4], vreg[4];
  auto request_k = [&](int tile) {
    const unsigned char* p = kh + (size_t)tile * kTileBytes;
#pragma unroll
    for (int i = 0; i < 4; ++i) kreg[i] = read32(p + (i >> 1) * 32 * kD + (i & 1) * 64, p + (i >> 1) * 32 * kD + (i & 1) * 64 + 16);
  };
  auto request_v = [&](int tile) {
    const unsigned char* p = vh + (size_t)tile * kTileBytes;
#pragma unroll
    for (int db = 0; db < 4; ++db) vreg[db] = read32(p + db * 1024 + 16 * sw, p + db * 1024 + 16 * (1 - sw));
  };

  f32x16 oacc[4], sacc[2];
  f32x4 lacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int e = 0; e < 16; ++e)
#pragma unroll
    for (int db = 0; db < 4; ++db) oacc[db][e] = 0.f;
  const i32x8 select = row_sum_operand(lane);
  float m_run = kNegBig;
  int tile = next_tile();
  if (tile != kNoTile) {
    request_k(tile);
    request_v(tile);
  }
  // A round takes one tile per wavefront.  A weight is rounded against the row maximum up to and including its own tile in
  // list order, as in attn_fp8_kernel (see the top of the file): the wavefronts tell each other their tiles' maxima.
  float m_round = kNegBig;      // row maximum over the tiles of all earlier rounds
  for (int round = 0; round * kSplitWaves < entries; ++round) {
    const int next = next_tile();
    const bool own_tile = tile != kNoTile;
    float tmax = kNegBig;
    if (own_tile) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
        for (int e = 0; e < 16; ++e) sacc[kb][e] = 0.f;
#pragma unroll
        for (int s = 0; s < 2; ++s) sacc[kb] = product(kreg[2 * kb + s], qreg[s], sacc[kb]);
      }
      if (next != kNoTile) request_k(next);
      if (tile * kBN + kBN > a.N) {
        int lim = a.N - tile * kBN - 4 * g;
        asm volatile("" : "+v"(lim));
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (32 * kb + 8 * (e >> 2) + (e & 3) >= lim) sacc[kb][e] = -INFINITY;
      }
      tmax = sacc[0][0];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 16; ++e) tmax = fmaxf(tmax, sacc[kb][e]);
      tmax = both_halves_max(tmax);
    }
    if (g == 0) tile_max[(round & 1) * kSplitWaves * kSplitRows + wave * kSplitRows + r] = tmax;
    __syncthreads();
    float m_new = m_round;
#pragma unroll
    for (int w = 0; w < kSplitWaves; ++w) {
      const float x = tile_max[(round & 1) * kSplitWaves * kSplitRows + w * kSplitRows + r];
      m_round = fmaxf(m_round, x);
      if (w <= wave) m_new = m_round;
    }
    if (own_tile) {
      if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {
        const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * c_log2);
        m_run = m_new;
        lacc[0] *= alpha;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
          for (int e = 0; e < 16; ++e) oacc[db][e] *= alpha;
      }
      const float mc = m_run * c_log2 - kWeightShift;
      i32x8 pb;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        float p[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) p[c] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[j >> 2][4 * (j & 3) + c], c_log2, -mc));
        const int w = __builtin_amdgcn_cvt_pk_fp8_f32(p[0], p[1], (int)__float_as_uint(p[0]), false);
        pb[j] = __builtin_amdgcn_cvt_pk_fp8_f32(p[2], p[3], w, true);
      }
      lacc = row_sum(select, pb, lacc);
#pragma unroll
      for (int db = 0; db < 4; ++db) oacc[db] = product(vreg[db], pb, oacc[db]);
      if (next != kNoTile) request_v(next);
    }
    tile = next;
  }

  // ---- merge (see split_kernel); v's scale and the row sum go into a wavefront's share
  unsigned char* const own = lds + wave * PART;
  if (entries > 0) __syncthreads();      // the last tile maxima are read
  if (g == 0) *reinterpret_cast<float2*>(own + r * 8) = make_float2(m_run, lacc[0]);
  __syncthreads();
  float2 st[kSplitWaves];
  float m_all = kNegBig, l_all = 0.f;
#pragma unroll
  for (int w = 0; w < kSplitWaves; ++w) st[w] = *reinterpret_cast<const float2*>(lds + w * PART + r * 8);
  __syncthreads();      // (read by all before the parts are written over them)
#pragma unroll
  for (int w = 0; w < kSplitWaves; ++w) m_all = fmaxf(m_all, st[w].y > 0.f ? st[w].x : kNegBig);
#pragma unroll
  for (int w = 0; w < kSplitWaves; ++w) {
    const float x = st[w].y * __builtin_amdgcn_exp2f((st[w].x - m_all) * c_log2);
    l_all += st[w].y > 0.f ? x : 0.f;
  }
  const float share = __builtin_amdgcn_exp2f((m_run - m_all) * c_log2) * v_scale / l_all;
  const float mine = lacc[0] > 0.f ? share : 0.f;
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f32x4 x;
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) x[jj] = oacc[db][4 * i + jj] * mine;
      *reinterpret_cast<f32x4*>(own + (4 * db + i) * 1024 + lane * 16) = x;
    }
  __syncthreads();
  if (qslot >= a.N) return;
  __bf16* op = a.o + ((size_t)bh * a.N + io_row) * kD + 32 * wave + 4 * g;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const unsigned char* src = lds + (4 * wave + i) * 1024 + lane * 16;
    f32x4 sum = *reinterpret_cast<const f32x4*>(src);
#pragma unroll
    for (int w = 1; w < kSplitWaves; ++w) sum += *reinterpret_cast<const f32x4*>(src + w * PART);
    *reinterpret_cast<bf16x4*>(op + 8 * i) = __builtin_convertvector(sum, bf16x4);
  }
}

__global__ __launch_bounds__(64 * kSplitWaves, 2) void attn_fp8_split_kernel(Fp8Args a) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[kSplitWaves * kSplitRows * kD * 4];
  const int total = a.BH * a.nqt, per_xcd = (total + 7) >> 3, loc = blockIdx.x >> 3, lid = (blockIdx.x & 7) * per_xcd + loc;
  if (loc >= per_xcd || lid >= total) return;
  const int bh = lid / a.nqt, row0 = (lid - bh * a.nqt) * kSplitRows, grp = row0 / kBM;
  int list_begin = a.row_ptr[0][grp], list_end = a.row_ptr[0][grp + 1], pat = 0;
  if (a.labels != nullptr) {
    const int t0 = a.row_ptr[1][grp], t1 = a.row_ptr[1][grp + 1];
    pat = __builtin_amdgcn_readfirstlane(a.labels[bh] != 0);
    list_begin = pat ? t0 : list_begin;
    list_end = pat ? t1 : list_end;
  }
  fp8_split_body(a, lds, bh, row0, pat, list_begin, list_end);
}

template <int LW>
__global__ __launch_bounds__(256, 2) void attn_fp8_kernel(Fp8Args a) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * kStages * kTileBytes];      // K images, then V images
  static_assert(sizeof(lds) <= 81920, "two workgroups fit a CU");

  // heavy query tiles first, then an eighth of each label's sequence of tiles (the same
  // dispatch order as the bf16 kernel)
  int bh = 0, grp = 0, pat = 0, cl = -1, head_cl0 = 0, part;
  if (!sparse_slot<LW>(a.so, a.BH, a.labels, a.row_ptr[0], a.row_ptr[1], blockIdx.x & 7, blockIdx.x >> 3, bh, grp, pat, cl, head_cl0, part)) return;
  bh = __builtin_amdgcn_readfirstlane(bh);
  grp = __builtin_amdgcn_readfirstlane(grp);
  pat = __builtin_amdgcn_readfirstlane(pat);
  cl = __builtin_amdgcn_readfirstlane(cl);
  head_cl0 = __builtin_amdgcn_readfirstlane(head_cl0);
  part = __builtin_amdgcn_readfirstlane(part);
  if (part >= 0) {      // a query tile with text rows that is taken in parts
    const int row0 = grp * kBM + part * kSplitRows;
    if (row0 >= a.N) return;
    const int32_t* rp = a.row_ptr[pat];
    fp8_split_body(a, lds, bh, row0, pat, __builtin_amdgcn_readfirstlane(rp[grp]), __builtin_amdgcn_readfirstlane(rp[grp + 1]));
    return;
  }

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 5, r = lane & 31;

  const size_t tiles_head = (size_t)bh * a.nk;
  const unsigned char* kh = a.k8 + tiles_head * kTileBytes;
  const unsigned char* vh = a.v8t + tiles_head * kTileBytes;

  // this lane's query: position qslot in the order the tile list refers to; for a temporal
  // head that is token off + f P + p with qslot = off + p F + f (q and o stay in token order)
  const int qslot = grp * kBM + wave * 32 + r;
  const int qrow = min(qslot, a.N - 1);
  int io_row = qrow;
  if (pat && qrow >= a.off && qrow < a.video_end)
    io_row = a.off + (int)transformed_to_token((unsigned)(qrow - a.off), (unsigned)a.F, (unsigned)a.P, a.sink);
  i32x8 qreg[2];       // lane (g, r) holds channels 64 s + 32 g .. + 32 of its query
  {
    const unsigned char* qp = a.q8 + ((size_t)bh * a.N + io_row) * kD + g * 32;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const i32x4 lo = *reinterpret_cast<const i32x4*>(qp + s * 64);
      const i32x4 hi = *reinterpret_cast<const i32x4*>(qp + s * 64 + 16);
      qreg[s] = i32x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    }
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
  // (no tile: every address is out of range, nothing is fetched and the unused image reads as zero; a branch around the loads
  // would cut the trip into blocks, between which the compiler moves the products and exponentials as it likes)
  auto load_image = [&](const unsigned char* images, int tile_any, int voffset, unsigned dst) {
    const int tile = __builtin_amdgcn_readfirstlane(tile_any);
    const u32x4 rsrc = buffer_words(images + (size_t)(tile == kNoTile ? 0 : tile) * kTileBytes, tile == kNoTile ? 0 : kTileBytes);
    load_to_lds(rsrc, voffset, voffset, 0, 4096, dst, 4096);
  };
  auto load_k = [&](int tile, int j) { load_image(kh, tile, k_src, lds_wave + (j & (kStages - 1)) * kTileBytes); };
  auto load_v = [&](int tile, int j) { load_image(vh, tile, v_src, lds_wave + (kStages + (j & (kStages - 1))) * kTileBytes); };

  // ---- operand reads.  K: lane (g, r) reads pieces 4 s + 2 g and 4 s + 2 g + 1 of row r of a
  // 32-key block; V^T: 32 bytes of channel r of a 32-channel block.
  const int k_row = r * kD, k_sw = k_swizzle(r);
  const int k_lo = k_row + (((2 * g) ^ k_sw) << 4);          // the other pieces differ from it in bits 4 and 6
  const int sw = (r >> 3) & 1;
  const int v_rd_lo = g * (kD * 32) + r * 32 + 16 * sw;
  const int v_rd_hi = g * (kD * 32) + r * 32 + 16 * (1 - sw);
  auto read32 = [](const unsigned char* lo, const unsigned char* hi) -> i32x8 {
    const i32x4 x = *reinterpret_cast<const i32x4*>(lo);
    const i32x4 y = *reinterpret_cast<const i32x4*>(hi);
    return i32x8{x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
  };
  auto k_operand = [&](int j, int i) -> i32x8 {              // i = 2 kb + s
    const unsigned char* p = lds + (j & (kStages - 1)) * kTileBytes + (i >> 1) * 32 * kD;
    const int at = (i & 1) ? k_lo ^ 64 : k_lo;
    return read32(p + at, p + (at ^ 16));
  };
  auto v_operand = [&](int j, int db) -> i32x8 {
    const unsigned char* p = lds + (kStages + (j & (kStages - 1))) * kTileBytes + db * 1024;
    return read32(p + v_rd_lo, p + v_rd_hi);
  };

  f32x16 oacc[4], sacc[2][2];      // two sets of scores: a tile's and the next one's
  f32x4 lacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int e = 0; e < 16; ++e)
#pragma unroll
    for (int db = 0; db < 4; ++db) oacc[db][e] = 0.f;
  const i32x8 select = row_sum_operand(lane);
  float m_run = kNegBig;     // reference maximum of the row, raw logits
  const bool ragged = (a.N % kBN) != 0;

  // i-th of the four products of S^T = K Q^T: two 32-key blocks x two 64-channel steps
  auto first_product = [&](f32x16 (&sc)[2], const i32x8& k_op, int i) {
    if ((i & 1) == 0) {
#pragma unroll
      for (int e = 0; e < 16; ++e) sc[i >> 1][e] = 0.f;
    }
    sc[i >> 1] = product(k_op, qreg[i & 1], sc[i >> 1]);
  };
  auto mask_tail = [&](f32x16 (&sc)[2], int tile) {       // keys beyond N in the last tile
    if (!(ragged && tile == a.nk - 1)) return;
    int lim = a.N - tile * kBN - 4 * g;
    asm volatile("" : "+v"(lim));        // keeps this rarely taken code out of every tile
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (32 * kb + 8 * (e >> 2) + (e & 3) >= lim) sc[kb][e] = -INFINITY;
  };
  i32x8 pb[2];
  float mc = 0.f;
  auto weights4 = [&](const f32x16 (&sc)[2], i32x8& out, int j) {      // 2^8 exp(s - reference) of four keys
    float p[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
      p[c] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[j >> 2][4 * (j & 3) + c], c_log2, -mc));
    // (the first conversion writes the low half of its destination and keeps the rest: giving it
    // a value that dies here as the "rest" saves a register clear; the second one fills the high half)
    const int w = __builtin_amdgcn_cvt_pk_fp8_f32(p[0], p[1], (int)__float_as_uint(p[0]), false);
    int packed = __builtin_amdgcn_cvt_pk_fp8_f32(p[2], p[3], w, true);
    asm volatile("" : "+v"(packed));      // here and not where it is used, a trip later
    out[j] = packed;
  };
  auto tile_maximum = [&](const f32x16 (&sc)[2]) -> float {
    float tmax = sc[0][0];
#pragma unroll
    for (int e = 1; e < 16; ++e) tmax = fmaxf(tmax, sc[0][e]);
#pragma unroll
    for (int e = 0; e < 16; ++e) tmax = fmaxf(tmax, sc[1][e]);
    return both_halves_max(tmax);
  };

  // ---- main loop.  Trip j holds the scores of tile j and the weights of tile j - 1: it takes the exponentials of the former
  // between the products of tile j + 1's scores and of tile j - 1's row sums and output, a product and four keys at a time.
  // Trips come in pairs, so that both sets of scores stay in their registers, with one barrier a pair: at its start LDS holds K of tiles
  // j + 1 and j + 2 and V of j - 1 and j, and the two tiles behind them are on their way into the places of those before.
  // The first tile of an odd list is weighted before them; with an even one a tile of zeros without weight lies in front.
  const int odd = entries & 1;
  const int col0 = odd ? list.next() : kNoTile;
  int col = list.next(), col1 = list.next(), col2 = list.next();
  if (entries > 0) {
    int j = odd, col3 = kNoTile, col4 = kNoTile;
    load_v(col0, j - 1);
    load_k(col, j);
    load_v(col, j);
    load_k(col1, j + 1);
    load_k(col2, j + 2);
    if (odd) load_k(col0, 0);
    wait_loads_to_lds<0>();
    __syncthreads();
    asm volatile("" ::"v"(qreg[0]), "v"(qreg[1]));
    auto scores = [&](f32x16 (&sc)[2], int at, int tile) {
      i32x8 op[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) op[i] = k_operand(at, i);
#pragma unroll
      for (int i = 0; i < 4; ++i) first_product(sc, op[i], i);
      mask_tail(sc, tile);
    };
    pb[1] = i32x8{0, 0, 0, 0, 0, 0, 0, 0};
    if (odd) {
      scores(sacc[1], 0, col0);
      m_run = fmaxf(m_run, tile_maximum(sacc[1]));
      mc = m_run * c_log2 - kWeightShift;
#pragma unroll
      for (int i = 0; i < 8; ++i) weights4(sacc[1], pb[1], i);
    }
    scores(sacc[0], j, col);
    __syncthreads();      // the first pair stages K of its fourth tile over the first one's
    auto trip = [&](auto set) {
      constexpr int CUR = decltype(set)::value;      // which set of scores is tile j's
      f32x16(&now)[2] = sacc[CUR];
      f32x16(&next)[2] = sacc[CUR ^ 1];
      i32x8 opnd[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) opnd[i] = k_operand(j + 1, i);
      const float tmax = tile_maximum(now);
      const bool raise = __builtin_amdgcn_ballot_w64(tmax > m_run) != 0;      // some row of the wavefront has a new maximum
      const float m_new = fmaxf(m_run, tmax);
      const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * c_log2);
      m_run = m_new;
      mc = m_run * c_log2 - kWeightShift;
      __builtin_amdgcn_sched_barrier(0);
      lacc = row_sum(select, pb[CUR ^ 1], lacc);
      if (CUR == 0) {      // behind a product: in front of it a workgroup alone on its compute unit waited for all their scalar instructions
        load_k(col3, j + 3);
        load_v(col1, j + 1);
        load_k(col4, j + 4);
        load_v(col2, j + 2);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        const int i = (n >> 1) + 2 * (n & 1);      // the two 32-key blocks in turn
        first_product(next, opnd[i], i);
        __builtin_amdgcn_sched_barrier(0);
        opnd[i] = v_operand(j - 1, i);
        weights4(now, pb[CUR], n);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        const int db = (n >> 1) + 2 * (n & 1);
        oacc[db] = product(opnd[db], pb[CUR ^ 1], oacc[db]);
        __builtin_amdgcn_sched_barrier(0);
        weights4(now, pb[CUR], 4 + n);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (raise) {
        lacc[0] *= alpha;                  // (only this element is ever read)
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
          for (int e = 0; e < 16; ++e) oacc[db][e] *= alpha;
      }
      mask_tail(next, CUR == 0 ? col1 : col2);
      ++j;
    };
    while (col != kNoTile) {
      col3 = list.next();
      col4 = list.next();
      trip(std::integral_constant<int, 0>{});
      trip(std::integral_constant<int, 1>{});
      wait_loads_to_lds<0>();
      barrier_loads_done();
      col = col2;
      col1 = col3;
      col2 = col4;
    }
    lacc = row_sum(select, pb[1], lacc);
#pragma unroll
    for (int db = 0; db < 4; ++db) oacc[db] = product(v_operand(j - 1, db), pb[1], oacc[db]);
  }

  // ---- epilogue: oacc[db][4 i + jj] = O[query r][32 db + 8 i + 4 g + jj]; lacc[0] = row sum
  const float l_tot = lacc[0];
  const float inv = l_tot > 0.f ? v_scale / l_tot : 0.f;
  if (qslot < a.N) {
    __bf16* op = a.o + ((size_t)bh * a.N + io_row) * kD;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        f32x4 x;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) x[jj] = oacc[db][4 * i + jj] * inv;
        *reinterpret_cast<bf16x4*>(op + db * 32 + 8 * i + 4 * g) = __builtin_convertvector(x, bf16x4);
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

bool fp8_split_form(const Geo& g) {
  const long long groups = (long long)g.B * g.H * ((g.N + kSplitRows - 1) / kSplitRows);
  return groups <= (g.N >= 4096 ? 600 : 512);
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
  a.row_ptr[1] = labels ? row_ptr_t : row_ptr_s; a.col_idx[1] = labels ? col_idx_t : col_idx_s;      // (read beside the others, without labels not used)
  a.N = g.N; a.nk = g.nk; a.BH = g.B * g.H;
  a.nqt = g.nq;
  // (no stride in the dispatch order: this kernel starts the query tiles of a cohort at a common key tile
  // instead, which measured 0.6-1.8 % faster here than the stride with or without that start)
  a.so = sparse_order(a.BH, a.nqt, kBM, g.off, g.video_end, g.N, 1 << 24, 512, 2, g.nk);
  a.scale_log2 = g.scale * 1.4426950408889634f;
  a.off = g.off; a.video_end = g.video_end; a.F = g.F; a.P = g.P; a.sink = g.sink;
  a.w_s = g.w_s; a.w_t = g.w_t;
  a.order = p_outer(g);
  (void)hipGetLastError();
  if (fp8_split_form(g)) {
    const long long groups = (long long)a.BH * ((a.N + kSplitRows - 1) / kSplitRows);
    a.nqt = (a.N + kSplitRows - 1) / kSplitRows;
    hipLaunchKernelGGL(attn_fp8_split_kernel, dim3(8u * (unsigned)((groups + 7) / 8)), dim3(64 * kSplitWaves), 0, stream, a);
    return hip_status(hipGetLastError());
  }
  const unsigned grid = sparse_grid(a.so, a.BH);
  if (a.BH > 64) hipLaunchKernelGGL(attn_fp8_kernel<kWideLabelWords>, dim3(grid), dim3(256), 0, stream, a);
  else hipLaunchKernelGGL(attn_fp8_kernel<1>, dim3(grid), dim3(256), 0, stream, a);
  return hip_status(hipGetLastError());
}

}  // namespace svg
