// Per-sample gradients g_i = delta_i^T a_i tile by tile in registers for the linear layers that the 16-bit tile
// kernel does not take: fp32 activations, and 16-bit ones whose rows are not 16-byte aligned.  Three uses:
//   MODE 0 (inner products): every finished sample tile is multiplied with the tile of G;
//   MODE 1 (statistics): it is squared (its share of ||g_i||^2) and added to the running sum that becomes G.
//   MODE 3 (norms of blocks whose gradient sum is supplied): it is squared.
// sum_tile_kernel (MODE 2) forms the gradient sum alone, all token rows as one sample, by fp32 MFMA: the same chain of fused multiply-adds, in row order,
// as wgrad_f32_kernel's, so the result is the same bit for bit (AdamW, next in a training step, divides by sqrt(v) and
// would blow up a last bit where gradient and second moment are both near zero).
#include <algorithm>
#include <type_traits>
#include <utility>

#include "common.h"

namespace adloco {

typedef __attribute__((ext_vector_type(4))) float pt_f32x4;
typedef __attribute__((ext_vector_type(16))) float pt_f32x16;

__device__ __forceinline__ double pt_wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// ---------------------------------------------------------------------------------------
// Workgroup = one square tile of 64 * W rows (d_out) and columns (d_in) of one layer for a run of consecutive samples;
// four waves as 2 x 2, wave tile 32W x 32W, 16x16x32 MFMA of 16-bit values, two (W = 2) or four (W = 1) workgroups to a
// compute unit.  16-bit elements are staged as they are.  An fp32 value is cut into three bf16 values that add up to it
// exactly (8 significand bits each), and six of the nine products of two such values are summed; the three left out are
// below 2^-24 of the product together (2^-28 in the mean square).  Six bf16 MFMAs take 96 cycles where the fp32 MFMA takes 256.
// Error against fp64: the MFMA rounds its sum of 32 products about once, not to nearest; a product that stands alone comes
// out within 2.4 x 2^-24 (0.56 in the mean square) where a rounding to nearest gives 1 (0.42), but the fp32 MFMA rounds
// every product's addition.  Normal values, T rows, of the fp32 MFMA's mean square error: T 1 1.36, 2 1.12, 3 0.91, 8 0.58,
// 32 0.37, 256 0.80, 1024 0.84; positive ones T 256 0.78, 2048 0.64 (and 5e-8 too small on average).  So up to four rows the
// tile is formed by fp32 MFMA (form_f32); with the two larger of the products left out (eight MFMAs) a single product is off
// by 0.55 in the mean square, and the kernel takes 14 % longer.  Still less exact than the fp32 MFMA: an entry that one
// token of a longer sequence makes up alone.  Sums of fp16 products, the same way: T 2 1.15, 3 0.97, 8 0.67, 32 0.48, 2048 0.36.
// Before it is cut a value is multiplied by 2^24, so that all its parts are normal numbers whatever it is.  Where a part or
// a sum overflows (values from 2^103, sums from 2^79, infinities, NaN) the finished tile is not finite, and each wave whose
// part of it is not forms that part again by fp32 MFMA straight from memory (form_f32): statistics of {768 -> 3072}, B 8,
// T 256 of values around 1e32, or of NaN alone, 0.28 ms; of ordinary values 0.104 (fp32 MFMA throughout: 0.157).
// Bound by issue: beside a 16x16x32 MFMA two other instructions find room in its 16 cycles, here there are three (matrix
// cores 52 % busy, one workgroup cutting and storing while the other's MFMAs run).  Not faster, measured on the statistics
// below: 32x32x16 MFMAs (0.71 ms); residuals by v_dot2c (fewer instructions, more wait states: 0.75); 256 x 128 tiles with
// the cutting between the MFMAs of eight waves (0.75 ms), of four (0.89).
// Statistics of 4 x {768 -> 2304, 768 -> 768, 768 -> 3072, 3072 -> 768}, B 8, T 256: 0.72 ms, 161 TFLOP/s (fp32 MFMA: 1.20
// ms); inner products of one such block, B 4, T 250: 0.09 ms (0.155).
// A chunk is 32 token rows; a thread fetches 2 W columns of eight of them, so that the eight values of a column that an
// MFMA operand holds are in one thread.  Rows past T and columns past the layer are staged as zeros, so any width, stride,
// alignment and sequence length runs here.  One stage of LDS: while one workgroup cuts and stores, the other's MFMAs run.
// Column kC * l + j of the tile (kC = 2 W) lies in LDS row 32 * j + l, pieces of eight tokens permuted so that neither the
// writes (16 rows at a time) nor the reads (rows 0-3 and 12-15 of one piece with 4-11 of the next) meet in the banks.
// ---------------------------------------------------------------------------------------
constexpr int kPtThreads = 256;
constexpr int kPtK = 32;                                     // token rows of a chunk
constexpr int kPtFew = 4;                                    // up to so many token rows, fp32 tiles are those of form_f32

struct PtArgs {
  const LayerDev* layers;
  const int4* tiles;      // entries of a tile list, of which `used` slots per XCD are launched
  const int2* part;       // the list's (tile, first partial tile)
  double* out;            // MODE 0: [tile][B][2]: <tile_i, G tile>, sum of squares of tile_i; MODE 1 and 3, [tile][B]: the latter
  int slots, used, T, B, group, whole;
  float* partials;        // MODE 1: [pieces][64W][64W]
  int accumulate;         // MODE 1 and 2: G += sum instead of G = sum
};

typedef __attribute__((ext_vector_type(4))) unsigned pt_u32x4;
typedef __attribute__((ext_vector_type(2))) float pt_f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 pt_bf16x2;
__device__ __forceinline__ int pt_piece(int row, int piece) { return piece ^ (-(row >> 2) & 3); }
__device__ __forceinline__ unsigned pt_pack(float x, float y) {
  const pt_f32x2 v = {x, y};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, pt_bf16x2));
}

template <typename E, int MODE, int W>
__global__ __launch_bounds__(kPtThreads, W == 2 ? 2 : 4) void plain_tile_kernel(PtArgs g) {
  constexpr bool kF32 = std::is_same<E, float>::value, kF16 = std::is_same<E, _Float16>::value;
  constexpr int kEdge = 64 * W, kC = 2 * W, kP = kF32 ? 3 : 1;
  __shared__ pt_u32x4 lds[2][kP][kEdge][4];                  // [delta, a][part][row][eight tokens]
  __shared__ double red[2][4][2];                            // sums of the four waves, samples in turn
  typedef __attribute__((ext_vector_type(kC))) E EV;
  const int seq = blockIdx.x / kNumXcd, entry = blockIdx.x % kNumXcd * g.slots + seq % g.used;
  const int4 tile = g.tiles[entry];
  if (tile.x < 0) return;
  const SampleRun S = MODE == 1 ? list_piece(tile.w, g.B, g.whole != 0) : list_run(tile.w, g.B, g.group, seq / g.used);
  const int s0 = S.first, cnt = S.count;
  if (cnt == 0) return;
  const int2 part = g.part[entry];
  const LayerDev L = g.layers[tile.x];
  const int e0 = tile.y, c0 = tile.z, T = g.T;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const bool edge = e0 + kEdge > L.d_out || c0 + kEdge > L.d_in;

  // ---- staging: waves 0 and 1 delta, 2 and 3 a; this thread's kC columns of tokens tok .. tok + 7 of the chunk
  const int sl = lane & 31, tg = (wave & 1) * 2 + (lane >> 5), tok = tg * 8;
  // (addresses on the scalar unit but for one pointer per lane, and no masks where a chunk lies within T and the layer:
  // with masks and products of 64 bits for every row, the vector unit was busier with addresses than with the splits)
  typedef const __attribute__((address_space(1))) E* mem_ptr;
  typedef EV EVu __attribute__((aligned(sizeof(E))));        // (vector loads need no more than the element's alignment)
  typedef const __attribute__((address_space(1))) EVu* mem_vec;
  const long long stride = wave < 2 ? L.delta_stride : L.a_stride;
  const int width = wave < 2 ? L.d_out - e0 : L.d_in - c0, left = width - sl * kC;      // valid columns: of the tile, from this thread's on
  const mem_ptr src = (mem_ptr)(reinterpret_cast<const E*>(wave < 2 ? L.delta : L.a) + ((long long)s0 * T + tok) * stride +
                                (wave < 2 ? e0 : c0) + sl * kC);
  const bool inside = width >= kEdge;
  E raw[8][kC];
  // token rows t0 .. t0 + 31 of the sample whose rows start at `base` rows from the entry's first
  auto load = [&](long long base, int t0) {
    const mem_ptr p = src + (base + t0) * stride;
    if (inside && t0 + kPtK <= T) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const EV x = *(mem_vec)(p + i * stride);
#pragma unroll
        for (int j = 0; j < kC; ++j) raw[i][j] = x[j];
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
#pragma unroll
        for (int j = 0; j < kC; ++j) raw[i][j] = E(0);
        if (t0 + tok + i < T && left >= kC) {
          const EV x = *(mem_vec)(p + i * stride);
#pragma unroll
          for (int j = 0; j < kC; ++j) raw[i][j] = x[j];
        } else if (t0 + tok + i < T) {
#pragma unroll
          for (int j = 0; j < kC - 1; ++j)
            if (j < left) raw[i][j] = p[i * stride + j];
        }
      }
    }
  };
  constexpr float kScale = 16777216.f, kUnscale = 1.f / kScale / kScale;
  auto store = [&]() {
    pt_u32x4* to = &lds[wave >> 1][0][sl][pt_piece(sl, tg)];
#pragma unroll
    for (int j = 0; j < kC; ++j) {
      pt_u32x4 v[kP];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if constexpr (kF32) {
          const float x = raw[2 * i][j], y = raw[2 * i + 1][j];
          const unsigned h = pt_pack(x * kScale, y * kScale);
          const float xm = fmaf(x, kScale, -__uint_as_float(h << 16)), ym = fmaf(y, kScale, -__uint_as_float(h & 0xffff0000u));
          const unsigned m = pt_pack(xm, ym);
          v[0][i] = h;
          v[1][i] = m;
          v[2][i] = pt_pack(xm - __uint_as_float(m << 16), ym - __uint_as_float(m & 0xffff0000u));
        } else {
          v[0][i] = unsigned(__builtin_bit_cast(unsigned short, raw[2 * i][j])) |
                    unsigned(__builtin_bit_cast(unsigned short, raw[2 * i + 1][j])) << 16;
        }
      }
#pragma unroll
      for (int p = 0; p < kP; ++p) to[(p * kEdge + 32 * j) * 4] = v[p];
    }
  };

  // ---- accumulators; element j of block (m, n): row kC * (wm * 16 + (lane/16)*4 + j) + m, column kC * (wn * 16 +
  // lane%16) + n of the tile.  gt: the tile of G (MODE 0) or the running sum of the sample tiles (MODE 1).
  const int r16 = lane & 15, kg = lane >> 4;
  const int out_r0 = kC * (wm * 16 + kg * 4), out_c = kC * (wn * 16 + r16);
  mfma_f32x4 acc[kC][kC], gt[kC][kC];             // (only MODE 1 has the second set)
#pragma unroll
  for (int m = 0; m < kC; ++m)
#pragma unroll
    for (int n = 0; n < kC; ++n)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[m][n][j] = gt[m][n][j] = 0.f;

  const int rd_piece = pt_piece(r16, kg);
  auto frag = [&](int op, int p, int m) {
    return __builtin_bit_cast(mfma_bf16x8, lds[op][p][32 * m + 16 * (op ? wn : wm) + r16][rd_piece]);
  };
  auto compute = [&]() {
    mfma_bf16x8 fc[kP][kC];
#pragma unroll
    for (int p = kP - 1; p >= 0; --p)
#pragma unroll
      for (int n = 0; n < kC; ++n) fc[p][n] = frag(1, p, n);
#pragma unroll
    for (int m = 0; m < kC; ++m) {
      mfma_bf16x8 fe[kP];
#pragma unroll
      for (int p = 0; p < kP; ++p) fe[p] = frag(0, p, m);
      if constexpr (kF32) {
        // smallest products first
        constexpr int pe[6] = {2, 0, 1, 1, 0, 0}, pc[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int q = 0; q < 6; ++q)
#pragma unroll
          for (int n = 0; n < kC; ++n) acc[m][n] = mfma_16x16x32_v<false>(fe[pe[q]], fc[pc[q]][n], acc[m][n]);
      } else {
#pragma unroll
        for (int n = 0; n < kC; ++n) acc[m][n] = mfma_16x16x32_v<kF16>(fe[0], fc[0][n], acc[m][n]);
      }
    }
  };
  // on a tile that reaches past the layer, an infinite input times a column of zeros is NaN: those entries are left out
  auto clear_edge = [&]() __attribute__((always_inline)) {
    int rows = L.d_out - e0 - out_r0, cols = L.d_in - c0 - out_c;
    asm volatile("" : "+v"(rows), "+v"(cols));    // (or the comparisons would be kept in registers across the loop)
#pragma unroll
    for (int m = 0; m < kC; ++m)
#pragma unroll
      for (int n = 0; n < kC; ++n)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (kC * j + m >= rows || n >= cols) acc[m][n][j] = 0.f;
  };
  // This wave's part of a sample's tile by fp32 MFMA (16x16x4, the accumulator layout of the 16-bit ones), from memory.
  auto form_f32 = [&](long long row) __attribute__((always_inline)) {
    int r = e0 + kC * (wm * 16 + r16), c = c0 + kC * (wn * 16 + r16), tk = kg;
    asm volatile("" : "+v"(r), "+v"(c), "+v"(tk));              // (as in clear_edge)
    const float* pd = reinterpret_cast<const float*>(L.delta) + (row + tk) * L.delta_stride + r;
    const float* pa = reinterpret_cast<const float*>(L.a) + (row + tk) * L.a_stride + c;
    r = L.d_out - r;
    c = L.d_in - c;
#pragma unroll
    for (int m = 0; m < kC; ++m)
#pragma unroll
      for (int n = 0; n < kC; ++n)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[m][n][j] = 0.f;
    for (int t = 0; t < T; t += 4, pd += 4 * L.delta_stride, pa += 4 * L.a_stride) {
      const int rows = t + tk < T ? r : 0, cols = t + tk < T ? c : 0;       // valid columns from pd and pa on
      float x[kC], y[kC];
#pragma unroll
      for (int j = 0; j < kC; ++j) {
        x[j] = j < rows ? pd[j] : 0.f;
        y[j] = j < cols ? pa[j] : 0.f;
      }
#pragma unroll
      for (int m = 0; m < kC; ++m)
#pragma unroll
        for (int n = 0; n < kC; ++n) acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[m], y[n], acc[m][n], 0, 0, 0);
    }
  };
  auto squares = [&]() __attribute__((always_inline)) {
    double sq = 0.0;
#pragma unroll
    for (int m = 0; m < kC; ++m)
#pragma unroll
      for (int n = 0; n < kC; ++n)
#pragma unroll
        for (int j = 0; j < 4; ++j) sq = fma(double(acc[m][n][j]), double(acc[m][n][j]), sq);
    return sq;
  };

  const int nk = (T + kPtK - 1) / kPtK;
  const long long n_chunks = (long long)cnt * nk;
  int k = 0, sample = 0;                          // chunk within the sample, sample within the entry
  auto put = [&](int i) {                         // the sums of the entry's i-th sample, behind a barrier
    const double (*r)[2] = red[i & 1];
    double* const d = g.out + ((size_t)part.x * g.B + s0 + i) * (MODE == 0 ? 2 : 1);
    if (MODE == 0) d[0] = (r[0][0] + r[1][0]) + (r[2][0] + r[3][0]);
    d[MODE == 0 ? 1 : 0] = (r[0][1] + r[1][1]) + (r[2][1] + r[3][1]);
  };
  load(0, 0);
  for (long long c = 0; c < n_chunks; ++c) {
    __syncthreads();                              // the last chunk has been read, the sums of a sample are there
    if (k == 0 && sample > 0 && threadIdx.x == 0) put(sample - 1);
    store();
    const bool last = k + 1 == nk;
    if (c + 1 < n_chunks) load((long long)(sample + (last ? 1 : 0)) * T, last ? 0 : (k + 1) * kPtK);
    __syncthreads();
    compute();
    if (!last) {
      ++k;
      continue;
    }
    if constexpr (kF32) {
      float unscale = kUnscale;
      asm volatile("" : "+v"(unscale));           // (or all entries would be multiplied in every chunk)
#pragma unroll
      for (int m = 0; m < kC; ++m)
#pragma unroll
        for (int n = 0; n < kC; ++n)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[m][n][j] *= unscale;
    }
    if (edge) clear_edge();
    double dot = 0.0, sq = squares();
    double limit = T <= kPtFew ? 0.0 : __builtin_inf();
    asm volatile("" : "+s"(limit));               // (or a second loop is made for few rows, and both are slower)
    if constexpr (kF32) if (__builtin_expect(__any(!(sq < limit)), 0)) {
      form_f32((long long)(s0 + sample) * T);
      if (edge) clear_edge();
      sq = squares();
    }
#pragma unroll
    for (int m = 0; m < kC; ++m) {
      float G[4][kC];                             // MODE 0: read again for every sample, to keep it took scratch memory
      if (MODE == 0) {
        typedef __attribute__((ext_vector_type(kC), aligned(sizeof(float)))) float FVu;
        int rows = L.d_out - e0 - out_r0, cols = L.d_in - c0 - out_c;
        asm volatile("" : "+v"(rows), "+v"(cols));            // (as in clear_edge)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float* const p = L.grad_sum + (size_t)(e0 + out_r0 + kC * j + m) * L.d_in + c0 + out_c;
          if (!edge) {
            const FVu v = *reinterpret_cast<const FVu*>(p);
#pragma unroll
            for (int n = 0; n < kC; ++n) G[j][n] = v[n];
          } else {
#pragma unroll
            for (int n = 0; n < kC; ++n) G[j][n] = kC * j + m < rows && n < cols ? p[n] : 0.f;
          }
        }
      }
#pragma unroll
      for (int n = 0; n < kC; ++n)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float v = acc[m][n][j];
          if (MODE == 0) dot = fma(double(v), double(G[j][n]), dot);
          if (MODE == 1) gt[m][n][j] += v;
          acc[m][n][j] = 0.f;
        }
    }
    if (MODE == 0) dot = pt_wave_sum(dot);
    sq = pt_wave_sum(sq);
    if (lane == 0) {
      red[sample & 1][wave][0] = dot;
      red[sample & 1][wave][1] = sq;
    }
    ++sample;
    k = 0;
  }
  __syncthreads();
  if (threadIdx.x == 0) put(cnt - 1);
  if (MODE == 1) {
    float* pt = cnt < g.B ? g.partials + (size_t)(part.y + (tile.w & 0xffff)) * (kEdge * kEdge) : nullptr;
#pragma unroll
    for (int m = 0; m < kC; ++m)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int n = 0; n < kC; ++n) {
          const int r = out_r0 + kC * j + m, c = out_c + n;
          const float v = gt[m][n][j];
          if (pt) {
            pt[r * kEdge + c] = v;
          } else if (e0 + r < L.d_out && c0 + c < L.d_in) {
            float* d = L.grad_sum + (size_t)(e0 + r) * L.d_in + c0 + c;
            *d = g.accumulate ? *d + v : v;
          }
        }
  }
}

// ---------------------------------------------------------------------------------------
// MODE 2.  fp32 MFMA (32x32x2: exact products, fp32 sums, 157 TFLOP/s over the chip); a chunk is 32 / W token rows, two
// LDS stages: one MFMA lasts 64 cycles and needs two LDS reads at most, so plain register staging keeps it fed.  W columns
// next to each other go to the W MFMA blocks of a wave (block m holds rows W * r + m): one LDS read of W floats feeds W
// blocks, and a lane owns W consecutive columns of G.
// ---------------------------------------------------------------------------------------
template <int W>
__global__ __launch_bounds__(kPtThreads, W == 2 ? 2 : 4) void sum_tile_kernel(PtArgs g) {
  constexpr int kEdge = 64 * W, kK = 32 / W;
  constexpr int kPieces = kEdge / 4;                         // pieces of four columns in a staged row
  constexpr int kLd = kK * kPieces / kPtThreads;             // pieces a thread stages per operand and chunk: 2
  __shared__ __attribute__((aligned(16))) float lds[2][2][kK][kEdge];
  typedef __attribute__((ext_vector_type(W))) float FV;
  const int4 tile = g.tiles[blockIdx.x % kNumXcd * g.slots + blockIdx.x / kNumXcd];
  if (tile.x < 0 || (tile.w & 0xffff) != 0) return;          // (no tile, or a further piece of one)
  const LayerDev L = g.layers[tile.x];
  const int e0 = tile.y, c0 = tile.z, T = g.T;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const bool fast = L.fast != 0;                  // 16-byte aligned rows, widths that are multiples of 8

  // ---- staging: thread's piece q of operand op is row row0 + q * kRowStep of the chunk, columns col .. col + 3
  const int col = (threadIdx.x % kPieces) * 4, row0 = threadIdx.x / kPieces;
  constexpr int kRowStep = kPtThreads / kPieces;
  const float* const pd = static_cast<const float*>(L.delta) + e0 + col;
  const float* const pa = static_cast<const float*>(L.a) + c0 + col;
  const int left_d = L.d_out - e0 - col, left_a = L.d_in - c0 - col;     // valid columns from here on
  auto fetch = [&](const float* p, int left) -> pt_f32x4 {
    pt_f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (fast) {
      if (left > 0) v = *reinterpret_cast<const pt_f32x4*>(p);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (j < left) v[j] = p[j];
    }
    return v;
  };
  pt_f32x4 rd[kLd], ra[kLd];
  auto load = [&](int t0) {
#pragma unroll
    for (int q = 0; q < kLd; ++q) {
      const int t = t0 + row0 + q * kRowStep;
      const bool ok = t < T;
      rd[q] = fetch(pd + (long long)t * L.delta_stride, ok ? left_d : 0);
      ra[q] = fetch(pa + (long long)t * L.a_stride, ok ? left_a : 0);
    }
  };
  auto store = [&](int st) {
#pragma unroll
    for (int q = 0; q < kLd; ++q) {
      *reinterpret_cast<pt_f32x4*>(&lds[st][0][row0 + q * kRowStep][col]) = rd[q];
      *reinterpret_cast<pt_f32x4*>(&lds[st][1][row0 + q * kRowStep][col]) = ra[q];
    }
  };

  // element j of block (m, n): tile row wm * 32W + W * ((j/4)*8 + (lane/32)*4 + j%4) + m, column wn * 32W + W * (lane%32) + n
  pt_f32x16 acc[W][W];
#pragma unroll
  for (int m = 0; m < W; ++m)
#pragma unroll
    for (int n = 0; n < W; ++n)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[m][n][j] = 0.f;
  const int nk = (T + kK - 1) / kK;
  load(0);
  store(0);
  __syncthreads();
  for (int c = 0; c < nk; ++c) {
    const int st = c & 1;
    const bool more = c + 1 < nk;
    if (more) load((c + 1) * kK);
#pragma unroll
    for (int ks = 0; ks < kK / 2; ++ks) {
      const FV fe = *reinterpret_cast<const FV*>(&lds[st][0][ks * 2 + (lane >> 5)][wm * 32 * W + W * (lane & 31)]);
      const FV fc = *reinterpret_cast<const FV*>(&lds[st][1][ks * 2 + (lane >> 5)][wn * 32 * W + W * (lane & 31)]);
#pragma unroll
      for (int m = 0; m < W; ++m)
#pragma unroll
        for (int n = 0; n < W; ++n)
          acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x2f32(fe[m], fc[n], acc[m][n], 0, 0, 0);
    }
    if (more) store(st ^ 1);                      // (read last in the chunk before: everybody is past its barrier)
    __syncthreads();
  }
#pragma unroll
  for (int m = 0; m < W; ++m)
#pragma unroll
    for (int n = 0; n < W; ++n)
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int r = e0 + wm * 32 * W + W * ((j >> 2) * 8 + (lane >> 5) * 4 + (j & 3)) + m;
        const int c = c0 + wn * 32 * W + W * (lane & 31) + n;
        if (r < L.d_out && c < L.d_in) {
          float* d = L.grad_sum + (size_t)r * L.d_in + c;
          *d = g.accumulate ? *d + acc[m][n][j] : acc[m][n][j];
        }
      }
}

// Partial tiles of the entries that were split along the samples -> grad_sum, in piece order (repeatable).  One
// workgroup per 4 rows of a split tile, one thread per column;  split[t] = (layer, e0, c0, pieces << 16 | first piece).
constexpr int kPtRedRows = 4;
template <int EDGE>
__global__ __launch_bounds__(EDGE) void plain_tile_reduce_kernel(const LayerDev* layers, const int4* split, int B,
                                                                const float* partials, int accumulate) {
  const int t = blockIdx.x / (EDGE / kPtRedRows), r0 = (blockIdx.x % (EDGE / kPtRedRows)) * kPtRedRows;
  const int4 S = split[t];
  const LayerDev L = layers[S.x];
  const int pieces = min(S.w >> 16, B);
  const float* base = partials + (size_t)(S.w & 0xffff) * (EDGE * EDGE) + threadIdx.x;
  const int col = S.z + threadIdx.x;
  float v[kPtRedRows];
#pragma unroll
  for (int r = 0; r < kPtRedRows; ++r) v[r] = 0.f;
  for (int p = 0; p < pieces; ++p)
#pragma unroll
    for (int r = 0; r < kPtRedRows; ++r) v[r] += base[(size_t)p * (EDGE * EDGE) + (r0 + r) * EDGE];
#pragma unroll
  for (int r = 0; r < kPtRedRows; ++r) {
    const int row = S.y + r0 + r;
    if (row >= L.d_out || col >= L.d_in) continue;
    float* d = L.grad_sum + (size_t)row * L.d_in + col;
    *d = accumulate ? *d + v[r] : v[r];
  }
}

// One workgroup per (listed layer, sample): the sums of the layer's tiles ranges[q], .., ranges[q + 1] - 1.
// dot (may be NULL; then `out` holds the sums of squares alone) and sq receive one float per (layer, sample), those of sq
// `sq_stride` floats apart.
__global__ __launch_bounds__(64) void plain_tile_finalize_kernel(const double* out, const int* lay, const int* ranges, int B,
                                                                float* dot, float* sq, int sq_stride) {
  const int q = blockIdx.x / B, i = blockIdx.x % B, width = dot ? 2 : 1;
  double d = 0.0, s = 0.0;
  for (int t = ranges[q] + threadIdx.x; t < ranges[q + 1]; t += 64) {
    const double* o = out + ((size_t)t * B + i) * width;
    if (dot) d += o[0];
    s += o[width - 1];
  }
  d = pt_wave_sum(d);
  s = pt_wave_sum(s);
  if (threadIdx.x == 0) {
    const size_t at = size_t(lay[q]) * B + i;
    if (dot) dot[at] = float(d);
    sq[at * sq_stride] = float(s);
  }
}

// ---- host side ------------------------------------------------------------------------------

// Time model of plain_tile_kernel<float, ..>: cycles of 2.1 GHz that `wgs` workgroups on a compute unit take for `samples`
// samples each.  A workgroup on its own needs the second figure of a pair per chunk (from load to load) and per finished
// tile; several share the SIMDs, each taking the first figure of them.  Fitted, like the 16 us of a split, to 300 lists
// (1 to 48 layers, widths 32 to 8192, B 1 to 48, T 1 to 2048, four forms each): the choice is within 1.3 % of the best form
// on average; worst, 1.5 times, on five tiles of 130 x 390 that are mostly edge.
static double plain_run(int W, double wgs, double samples, int T) {
  const double chunks = double((T + kPtK - 1) / kPtK);
  if (W == 2) return 17700.0 + samples * (chunks * std::max(3110.0 * wgs, 5320.0) + std::max(740.0 * wgs, 2160.0));
  return 6300.0 + samples * (chunks * std::max(1105.0 * wgs, 2740.0) + std::max(310.0 * wgs, 1240.0));
}

// Inner products and norms alone, whose runs of samples fill the last round.
int plain_tile_width(const std::vector<LayerDev>& layers, const std::vector<char>& use, int B, int T) {
  double best = 0.0;
  int pick = 0;
  for (int W = 2; W >= 1; --W) {
    const TileGeom geom = plain_tile_geom(W);
    long long n = 0;
    for (size_t l = 0; l < layers.size(); ++l)
      if (use[l]) n += (long long)((layers[l].d_out + geom.e - 1) / geom.e) * ((layers[l].d_in + geom.c - 1) / geom.c);
    const int group = run_length(n, B, T, geom);
    const long long wgs = n * ((B + group - 1) / group), room = (long long)geom.room * kNumXcd, left = wgs % room;
    double cost = double(wgs / room) * plain_run(W, geom.room / 32.0, group, T);
    if (left) cost += plain_run(W, double((left + kNumCu - 1) / kNumCu), group, T);
    if (!pick || cost < best) {
      best = cost;
      pick = W;
    }
  }
  return pick;
}

// Gradient sums alone, whose kernel is another.  128-wide tiles need a quarter fewer LDS bytes per product and half the
// loads; 64-wide ones fill the chip on small layers.  Time model in MFMA cycles per token row: w workgroups on a compute
// unit share its four SIMDs, a row costs a wave 128 (W = 2) or 32 cycles (W = 1) of its SIMD, and no less than 64 for the
// loop around the MFMAs.
int sum_tile_width(const std::vector<LayerDev>& layers, const std::vector<char>& use) {
  double best = 0.0;
  int pick = 2;
  for (int W = 2; W >= 1; --W) {
    const int edge = 64 * W, room = plain_tile_room(W);
    long long n = 0;
    for (size_t l = 0; l < layers.size(); ++l)
      if (use[l]) n += (long long)((layers[l].d_out + edge - 1) / edge) * ((layers[l].d_in + edge - 1) / edge);
    const long long nx = (n + kNumXcd - 1) / kNumXcd, left = nx % room;
    const double row = W == 2 ? 128.0 : 32.0;
    double cost = double(nx / room) * std::max(row * room / 32, 64.0);
    if (left) cost += std::max(row * double((left + 31) / 32), 64.0);
    if (W == 2 || cost < best * 0.98) {
      best = cost;
      pick = W;
    }
  }
  return pick;
}

// Statistics (mode 1): tile width, and whether the tiles of the incomplete last round are split along the samples.  A split
// costs one more launch and its partial tiles a trip through memory at 3 TB/s; a call of this size waits for the host's
// launches anyway, behind which a longer kernel hides.
PlainChoice plain_tile_choice(const TileList* lists, int B, int T) {
  PlainChoice pick{2, false};
  double best = 0.0;
  for (int W = 1; W <= 2; ++W)
    for (int whole = 1; whole >= 0; --whole) {
      const TileList& p = lists[W - 1];
      if (!p.built) continue;
      const int room = plain_tile_room(W);
      double t = 0.0;
      bool cut = false;
      double bytes = 0.0;
      for (int x = 0; x < kNumXcd; ++x) {
        const int full = p.n[x] / room, left = p.n[x] % room, S = whole ? 1 : std::max(1, std::min(p.pieces[x], B));
        double tx = full * plain_run(W, room / 32.0, B, T);
        if (left) tx += plain_run(W, double((left * S + 31) / 32), double((B + S - 1) / S), T);
        if (S > 1) bytes += double(left) * S * p.edge * p.edge * sizeof(float);
        cut = cut || S > 1;
        t = std::max(t, tx);
      }
      if (cut) t += 16.0 * 2100.0 + bytes / 3e6 * 2100.0;
      if (!whole && !cut) continue;               // (the same form again)
      if (best == 0.0 || t < best) {
        best = t;
        pick = PlainChoice{W, whole != 0};
      }
    }
  return pick;
}

hipError_t launch_plain_tiles(const LayerDev* layers, const TileList& list, int mode, int B, int T, int dtype, int accumulate,
                              bool whole, int group, double* out, float* dot, float* sq, int sq_stride, hipStream_t st) {
  const int used = mode == 1 && !whole ? list.used(B) : list.used(1);
  const PtArgs a{layers, list.tiles(), list.part(), out, list.slots, used, T, B, group, whole ? 1 : 0,
                 static_cast<float*>(list.ptiles.ptr), accumulate};
  const int runs = mode == 0 || mode == 3 ? (B + group - 1) / group : 1;
  const dim3 grid(unsigned(used) * unsigned(runs) * kNumXcd), block(kPtThreads);
#define PT_LAUNCH(E, MODE)                                                                              \
  do {                                                                                                  \
    if (list.edge == 128) hipLaunchKernelGGL((plain_tile_kernel<E, MODE, 2>), grid, block, 0, st, a);   \
    else hipLaunchKernelGGL((plain_tile_kernel<E, MODE, 1>), grid, block, 0, st, a);                    \
  } while (0)
  if (mode == 2 && list.edge == 128) hipLaunchKernelGGL(sum_tile_kernel<2>, grid, block, 0, st, a);
  else if (mode == 2) hipLaunchKernelGGL(sum_tile_kernel<1>, grid, block, 0, st, a);
  else if (mode == 1) PT_LAUNCH(float, 1);             // (16-bit statistics have kernels of their own)
  else if (mode == 3) PT_LAUNCH(float, 3);
  else if (dtype == ADLOCO_BF16) PT_LAUNCH(unsigned short, 0);
  else if (dtype == ADLOCO_F16) PT_LAUNCH(_Float16, 0);
  else PT_LAUNCH(float, 0);
#undef PT_LAUNCH
  if (mode == 1 && !whole && B > 1 && list.n_split > 0) {
    if (list.edge == 128)
      hipLaunchKernelGGL(plain_tile_reduce_kernel<128>, dim3(unsigned(list.n_split) * (128 / kPtRedRows)), dim3(128), 0,
                         st, layers, list.split(), B, a.partials, accumulate);
    else
      hipLaunchKernelGGL(plain_tile_reduce_kernel<64>, dim3(unsigned(list.n_split) * (64 / kPtRedRows)), dim3(64), 0,
                         st, layers, list.split(), B, a.partials, accumulate);
  }
  if (sq)
    hipLaunchKernelGGL(plain_tile_finalize_kernel, dim3(unsigned(list.n_listed) * B), dim3(64), 0, st, out, list.layers(),
                       list.ranges(), B, dot, sq, sq_stride);
  return hipGetLastError();
}

}  // namespace adloco
