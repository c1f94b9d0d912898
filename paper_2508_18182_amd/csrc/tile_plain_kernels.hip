// Per-sample gradients g_i = delta_i^T a_i tile by tile in registers for the linear layers that the 16-bit tile
// kernel does not take: fp32 activations, and 16-bit ones whose rows are not 16-byte aligned.  Two uses, as there:
//   MODE 0 (inner products): every finished sample tile is multiplied with the tile of G;
//   MODE 1 (statistics): it is squared (its share of ||g_i||^2) and added to the running sum that becomes G.
//   MODE 3 (norms of blocks whose gradient sum is supplied): it is squared.
// MODE 2 is the gradient sum alone, all token rows as one sample: the same chain of fused multiply-adds, in row order,
// as wgrad_f32_kernel's, so the result is the same bit for bit (AdamW, next in a training step, divides by sqrt(v) and
// would blow up a last bit where gradient and second moment are both near zero).
#include <algorithm>

#include "common.h"

namespace adloco {

typedef __attribute__((ext_vector_type(4))) float pt_f32x4;
typedef __attribute__((ext_vector_type(16))) float pt_f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned short pt_u16x4;
typedef __attribute__((ext_vector_type(4))) _Float16 pt_h16x4;

__device__ __forceinline__ float pt_elem(float v) { return v; }
__device__ __forceinline__ float pt_elem(unsigned short h) { return __uint_as_float(unsigned(h) << 16); }
__device__ __forceinline__ float pt_elem(_Float16 h) { return float(h); }
template <typename E> struct PtVec;
template <> struct PtVec<float> { typedef pt_f32x4 type; };
template <> struct PtVec<unsigned short> { typedef pt_u16x4 type; };
template <> struct PtVec<_Float16> { typedef pt_h16x4 type; };

__device__ __forceinline__ double pt_wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// ---------------------------------------------------------------------------------------
// Workgroup = one square tile of 64 * W rows (d_out) and columns (d_in) of one layer for a run of consecutive samples;
// four waves as 2 x 2, wave tile 32W x 32W, fp32 MFMA (32x32x2: exact products, fp32 sums, 157 TFLOP/s over the chip).
// Bound by the matrix cores: one MFMA lasts 64 cycles and needs two LDS reads at most, so plain register staging with
// two LDS stages and two (W = 2) to four (W = 1) workgroups per compute unit keep them fed; rows past T and columns
// past the layer are staged as zeros, so any width, stride, alignment and sequence length runs here.  A chunk is
// 32 / W token rows: 16 KiB of LDS and the same 1024 * W MFMA cycles in either form.
// Statistics of 4 x {768 -> 2304, 768 -> 768, 768 -> 3072, 3072 -> 768}, B 8, T 256: 1.25 ms, 93 TFLOP/s (Gram and
// gradient-sum kernels on the vector unit: 5.02 ms); inner products of one such block, B 4, T 250: 0.18 ms (runs of
// samples dealt to the XCDs layer by layer: 0.41 ms; one thread per gradient row: 145 ms).
// W columns next to each other go to the W MFMA blocks of a wave (block m holds rows W * r + m): one LDS read of
// W floats feeds W blocks, and a lane owns W consecutive columns of G.
// ---------------------------------------------------------------------------------------
constexpr int kPtThreads = 256;

struct PtArgs {
  const LayerDev* layers;
  const int4* tiles;      // entries of a tile list, of which `used` slots per XCD are launched
  const int2* part;       // the list's (tile, first partial tile)
  double* out;            // MODE 0: [tile][B][2]: <tile_i, G tile>, sum of squares of tile_i; MODE 1 and 3, [tile][B]: the latter
  int slots, used, T, B, group, whole;
  float* partials;        // MODE 1: [pieces][64W][64W]
  int accumulate;         // MODE 1 and 2: G += sum instead of G = sum
};

template <typename E, int MODE, int W>
__global__ __launch_bounds__(kPtThreads, W == 2 ? 2 : 4) void plain_tile_kernel(PtArgs g) {
  constexpr int kEdge = 64 * W, kK = 32 / W;
  constexpr int kPieces = kEdge / 4;                         // pieces of four columns in a staged row
  constexpr int kLd = kK * kPieces / kPtThreads;             // pieces a thread stages per operand and chunk: 2
  __shared__ __attribute__((aligned(16))) float lds[2][2][kK][kEdge];
  __shared__ double red[2][4][2];                            // sums of the four waves, samples in turn
  typedef typename PtVec<E>::type EV;
  typedef __attribute__((ext_vector_type(W))) float FV;
  const int seq = blockIdx.x / kNumXcd, entry = blockIdx.x % kNumXcd * g.slots + seq % g.used;
  const int4 tile = g.tiles[entry];
  if (tile.x < 0) return;
  const SampleRun S = MODE == 1 || MODE == 2 ? list_piece(tile.w, g.B, g.whole != 0) : list_run(tile.w, g.B, g.group, seq / g.used);
  const int s0 = S.first, cnt = S.count;
  if (cnt == 0) return;
  const int2 part = g.part[entry];
  const LayerDev L = g.layers[tile.x];
  const int e0 = tile.y, c0 = tile.z, T = g.T;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const bool edge = e0 + kEdge > L.d_out || c0 + kEdge > L.d_in;
  const bool fast = L.fast != 0;                  // 16-byte aligned rows, widths that are multiples of 8

  // ---- staging: thread's piece q of operand op is row row[q] of the chunk, columns col .. col + 3
  const int col = (threadIdx.x % kPieces) * 4, row0 = threadIdx.x / kPieces;
  constexpr int kRowStep = kPtThreads / kPieces;
  const E* const pd = reinterpret_cast<const E*>(L.delta) + (long long)s0 * T * L.delta_stride + e0 + col;
  const E* const pa = reinterpret_cast<const E*>(L.a) + (long long)s0 * T * L.a_stride + c0 + col;
  const int left_d = L.d_out - e0 - col, left_a = L.d_in - c0 - col;     // valid columns from here on
  auto fetch = [&](const E* p, int left) -> pt_f32x4 {
    pt_f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (fast) {
      if (left > 0) {
        const EV x = *reinterpret_cast<const EV*>(p);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = pt_elem(E(x[j]));
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (j < left) v[j] = pt_elem(p[j]);
    }
    return v;
  };
  pt_f32x4 rd[kLd], ra[kLd];
  // token rows t0 .. t0 + kK - 1 of the sample whose rows start at `base` rows from the entry's first
  auto load = [&](long long base, int t0) {
#pragma unroll
    for (int q = 0; q < kLd; ++q) {
      const int t = t0 + row0 + q * kRowStep;
      const bool ok = t < T;
      rd[q] = fetch(pd + (base + t) * L.delta_stride, ok ? left_d : 0);
      ra[q] = fetch(pa + (base + t) * L.a_stride, ok ? left_a : 0);
    }
  };
  auto store = [&](int st) {
#pragma unroll
    for (int q = 0; q < kLd; ++q) {
      *reinterpret_cast<pt_f32x4*>(&lds[st][0][row0 + q * kRowStep][col]) = rd[q];
      *reinterpret_cast<pt_f32x4*>(&lds[st][1][row0 + q * kRowStep][col]) = ra[q];
    }
  };

  // ---- accumulators; element j of block (m, n): tile row wm * 32W + W * ((j/4)*8 + (lane/32)*4 + j%4) + m, column
  // wn * 32W + W * (lane%32) + n.  gt: the tile of G (MODE 0) or the running sum of the sample tiles (MODE 1).
  const int out_c = wn * 32 * W + W * (lane & 31);
  auto out_r = [&](int m, int j) { return wm * 32 * W + W * ((j >> 2) * 8 + (lane >> 5) * 4 + (j & 3)) + m; };
  pt_f32x16 acc[W][W], gt[W][W];                  // (MODE 2 and 3 have no second set)
#pragma unroll
  for (int m = 0; m < W; ++m)
#pragma unroll
    for (int n = 0; n < W; ++n)
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        acc[m][n][j] = 0.f;
        float v = 0.f;
        if (MODE == 0) {
          const int r = e0 + out_r(m, j), c = c0 + out_c + n;
          if (r < L.d_out && c < L.d_in) v = L.grad_sum[(size_t)r * L.d_in + c];
        }
        gt[m][n][j] = v;
      }

  const int nk = (T + kK - 1) / kK;
  const long long n_chunks = (long long)cnt * nk;
  load(0, 0);
  store(0);
  __syncthreads();
  int k = 0, sample = 0;                          // chunk within the sample, sample within the entry
  for (long long c = 0; c < n_chunks; ++c) {
    const int st = int(c & 1);
    const bool more = c + 1 < n_chunks;
    const bool last = k + 1 == nk;
    if (more) load((long long)(sample + (last ? 1 : 0)) * T, last ? 0 : (k + 1) * kK);
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
    if (MODE == 2) {
      ++k;                                        // (one sample)
    } else if (last) {
      // on a tile that reaches past the layer, an infinite input times a column of zeros is NaN: those entries are left out
      if (edge) {
        int rows = L.d_out - e0 - out_r(0, 0), cols = L.d_in - c0 - out_c;
        asm volatile("" : "+v"(rows), "+v"(cols));  // (or the comparisons would be kept in registers across the loop)
#pragma unroll
        for (int m = 0; m < W; ++m)
#pragma unroll
          for (int n = 0; n < W; ++n)
#pragma unroll
            for (int j = 0; j < 16; ++j)
              if (W * ((j >> 2) * 8 + (j & 3)) + m >= rows || n >= cols) acc[m][n][j] = 0.f;
      }
      double dot = 0.0, sq = 0.0;
#pragma unroll
      for (int m = 0; m < W; ++m)
#pragma unroll
        for (int n = 0; n < W; ++n)
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const float v = acc[m][n][j];
            if (MODE == 0) dot = fma(double(v), double(gt[m][n][j]), dot);
            else if (MODE == 1) gt[m][n][j] += v;
            sq = fma(double(v), double(v), sq);
            acc[m][n][j] = 0.f;
          }
      if (MODE == 0) dot = pt_wave_sum(dot);
      sq = pt_wave_sum(sq);
      if (lane == 0) {
        red[sample & 1][wave][0] = dot;
        red[sample & 1][wave][1] = sq;
      }
      ++sample;
      k = 0;
    } else {
      ++k;
    }
    if (more) store(st ^ 1);                      // (read last in the chunk before: everybody is past its barrier)
    __syncthreads();
    if (MODE != 2 && last && threadIdx.x == 0) {  // (written again two samples, and so two barriers, later)
      const double (*r)[2] = red[(sample - 1) & 1];
      double* const d = g.out + ((size_t)part.x * g.B + s0 + sample - 1) * (MODE == 0 ? 2 : 1);
      if (MODE == 0) d[0] = (r[0][0] + r[1][0]) + (r[2][0] + r[3][0]);
      d[MODE == 0 ? 1 : 0] = (r[0][1] + r[1][1]) + (r[2][1] + r[3][1]);
    }
  }
  if (MODE == 1 || MODE == 2) {
    float* pt = MODE == 1 && cnt < g.B ? g.partials + (size_t)(part.y + (tile.w & 0xffff)) * (kEdge * kEdge) : nullptr;
#pragma unroll
    for (int m = 0; m < W; ++m)
#pragma unroll
      for (int n = 0; n < W; ++n)
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int r = out_r(m, j), c = out_c + n;
          const float v = MODE == 1 ? gt[m][n][j] : acc[m][n][j];
          if (pt) {
            pt[r * kEdge + c] = v;
          } else if (e0 + r < L.d_out && c0 + c < L.d_in) {
            float* d = L.grad_sum + (size_t)(e0 + r) * L.d_in + c0 + c;
            *d = g.accumulate ? *d + v : v;
          }
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

// 128-wide tiles need a quarter fewer LDS bytes per product and half the loads; 64-wide ones fill the chip on small
// layers.  Gradient sums, inner products and norms alone (runs of samples fill the last round).  Time model in MFMA cycles per token row: w workgroups on a compute unit share its four SIMDs, a row costs a
// wave 128 (W = 2) or 32 cycles (W = 1) of its SIMD, and no less than 64 for the loop around the MFMAs.
int plain_tile_width(const std::vector<LayerDev>& layers, const std::vector<char>& use, int B) {
  double best = 0.0;
  int pick = 2;
  for (int W = 2; W >= 1; --W) {
    const int edge = 64 * W, room = plain_tile_room(W);
    long long n = 0;
    for (size_t l = 0; l < layers.size(); ++l)
      if (use[l]) n += (long long)((layers[l].d_out + edge - 1) / edge) * ((layers[l].d_in + edge - 1) / edge);
    const long long nx = (n + kNumXcd - 1) / kNumXcd, left = nx % room;
    const double row = W == 2 ? 128.0 : 32.0;
    double cost = double(nx / room) * B * std::max(row * room / 32, 64.0);
    if (left) {
      const long long S = std::min<long long>(std::max<long long>(room / left, 1), B);
      const double wgs = double((left * S + 31) / 32);
      cost += double((B + S - 1) / S) * std::max(row * wgs, 64.0);
    }
    if (W == 2 || cost < best * 0.98) {
      best = cost;
      pick = W;
    }
  }
  return pick;
}

// Statistics (mode 1): tile width, and whether the tiles of the incomplete last round are split along the samples, by a
// time model in cycles of 2.1 GHz.  A workgroup on its own needs 2400 cycles (64-wide tiles; 128-wide: 2800) per chunk, from
// load to load, and 2000 per finished tile; w workgroups on a compute unit no less than 1126 w (2048 w) and 300 w
// (1200 w) of its SIMDs.  Split tiles cost one more launch, 8 us, and their partial tiles a trip through memory at 3 TB/s;
// 8 us more are asked of them because a call of this size waits for the host's launches, behind which a longer kernel
// hides (statistics, norm test and outer step of one layer 64 -> 32, B 8, T 16: 85 us whole, 89 us split).
// Of 270 calls on 1 to 16 layers with 32 to 2048 token rows, the choice is within 2.3 % of the best of the four forms on
// average, within 20 % at worst; a fixed line at 512 rows (and 128-wide tiles as if always split) missed it by 12 % on
// average and was 2.6 times slower at worst: one layer 768 -> 768, B 8, T 64 69 us instead of 34.
PlainChoice plain_tile_choice(const TileList* lists, int B, int T) {
  PlainChoice pick{2, false};
  double best = 0.0;
  for (int W = 1; W <= 2; ++W)
    for (int whole = 1; whole >= 0; --whole) {
      const TileList& p = lists[W - 1];
      if (!p.built) continue;
      const int room = plain_tile_room(W);
      const double chunks = double((T + 32 / W - 1) / (32 / W));
      auto run = [&](double wgs, double samples) {
        return samples * (chunks * std::max((W == 2 ? 2048.0 : 1126.0) * wgs, W == 2 ? 2800.0 : 2400.0) +
                          std::max((W == 2 ? 1200.0 : 300.0) * wgs, 2000.0));
      };
      double t = 0.0;
      bool cut = false;
      double bytes = 0.0;
      for (int x = 0; x < kNumXcd; ++x) {
        const int full = p.n[x] / room, left = p.n[x] % room, S = whole ? 1 : std::max(1, std::min(p.pieces[x], B));
        double tx = full * run(room / 32.0, B);
        if (left) tx += run(double((left * S + 31) / 32), double((B + S - 1) / S));
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
  if (mode == 2) PT_LAUNCH(float, 2);
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
