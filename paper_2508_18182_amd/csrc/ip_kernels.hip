// Kernels that form the per-sample gradients g_i = delta_i^T a_i of the linear layers tile by tile
// in registers (never in memory) and reduce each tile on the spot:
//   * inner products c_i = <g_i, G> with the batch gradient sum G, whose variance the
//     inner-product test and the augmented inner-product test of Section 3.3.2 need;
//   * the statistics of the norm test (eq. 4, Section 3.3.1): ||g_i||^2 from the squares of the
//     tiles while they are being added up to G -- the route of adloco_grad_stats where G is
//     formed by the library.
// Aligned 16-bit layers take the MFMA tile kernels (ip_tile_kernel, and short_tile_kernel for short sequences); every
// other layer the plain tile kernel (tile_plain_kernels.hip).  The dot kernels of the vector / table blocks and the reductions
// follow.  The inner-product paths also return the explicit ||g_i||^2, a second
// route to the Gram kernel's result.
#include <type_traits>

#include "common.h"

namespace adloco {

constexpr int kIpThreads = 256;

__device__ __forceinline__ float ip_elem(unsigned short h) { return __uint_as_float(unsigned(h) << 16); }
__device__ __forceinline__ float ip_elem(_Float16 h) { return float(h); }
__device__ __forceinline__ float ip_elem(float f) { return f; }

__device__ __forceinline__ double ip_wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double ip_block_sum(double v, double* lds4) {
  v = ip_wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) lds4[threadIdx.x >> 6] = v;
  __syncthreads();
  return (lds4[0] + lds4[1]) + (lds4[2] + lds4[3]);
}

// ---------------------------------------------------------------------------------------
// Tile path (aligned 16-bit linear layers).
// Work item = one 256 (d_out) x 128 (d_in) tile of one layer for a run of consecutive samples.
// The workgroup (four waves as 2 x 2, one per SIMD, wave tile 128 x 64, 16x16x32 MFMA) streams the token rows of its
// samples in chunks of 32 through one uninterrupted load pipeline.  After the last chunk of a sample the accumulators
// hold that sample's gradient tile.  A second set of 128 registers per lane, in the MFMA accumulator layout, holds
//   MODE 0 (inner products): the tile of G; the finished sample tile is multiplied element-wise
//     with it and summed over the wave; two floats per (tile, sample, wave) leave the chip;
//   MODE 1 (statistics): the running sum of the sample tiles; each finished tile is squared and
//     summed (its share of ||g_i||^2) and added to the running sum, which is stored as the tile of G at the end;
//   MODE 2 (norms of blocks whose gradient sum is supplied): nothing, each finished tile is squared and summed.
// That work on a finished tile is spread between the MFMAs of the next sample's first chunk, which start from zero
// instead of the old accumulators: each block is read just before its first MFMA of the new sample.
// A 256 x 256 tile would need 256 accumulators + 256 registers of the second set per lane: the whole register file.
//   Staging: global -> LDS directly, six stages of 32 token rows x (256 + 128) columns, loads five chunks ahead.  A
//   load instruction moves 1 KiB: two token rows of delta (2 x 512 B) or four of a (4 x 256 B); the 1 KiB blocks are
//   1056 bytes apart and the rows are dealt to them so that the eight rows that 32 lanes of a transpose read touch
//   start in eight different groups of banks.  LDS reads go out one by one behind the MFMAs, loads in pairs from one
//   scalar base (the rows are in the lane offsets: a scalar instruction counts here, with one wave per SIMD), one barrier
//   per chunk.  Columns of a past the edge of the layer re-read the last valid 16-byte piece and are left out of every
//   sum.  Columns of delta past the edge are never loaded: their lanes are switched off and the LDS is cleared
//   beforehand; check_rows() takes care of what an infinite a makes of those zeros.  RAGGED (T not a multiple of 32):
//   token rows past T come from a line of zeros.
// What bounds it: the instruction slots of one wave per SIMD (about 115 instructions and 32 MFMAs of 16 cycles per chunk;
// 380 vector instructions per finished tile) and the chip's power: matrix cores 53 to 59 % busy at 1.75 of 2.4 GHz, LDS
// 21 %, no bank conflicts, 12 % of the wave cycles waiting.  48 GPT-2-small linears, B 32, T 512 (2.78 TFLOP): 2.73 ms for statistics, 2.85 ms for the inner
// products with norms (eight waves of 64 x 64 with 32x32x16 MFMAs: 2.90 and 3.05 ms on the same card); without loads, with
// loads that all hit the L2, or without the work on finished tiles each is 0.2 to 0.5 ms less.  The same linears in fp16
// with B 5, T 1001, added to a gradient sum: 1.07 ms (Gram kernel and 128 x 128 gradient-sum kernel: 2.37 ms).
// ---------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(4))) short ip_s16x4;
typedef __attribute__((ext_vector_type(8))) short ip_s16x8;
typedef __attribute__((ext_vector_type(4))) unsigned ip_u32x4;

constexpr int kIpE = 256;                         // tile rows (d_out side)
constexpr int kIpC = 128;                         // tile columns (d_in side)
constexpr int kIpK = 32;                          // token rows per stage
constexpr int kIpBlk = 1024 + 32;                 // one load instruction + 32 B skew
constexpr int kIpOpE = 16 * kIpBlk;               // delta side of a stage
constexpr int kIpOpC = 8 * kIpBlk;                // a side of a stage
constexpr int kIpStage = kIpOpE + kIpOpC;         // 24.75 KiB
constexpr int kIpWaves = 4;
constexpr int kIpFM = 8, kIpFN = 4;               // 16x16 MFMA blocks per wave along d_out and d_in
constexpr int kIpLd = 6;                          // loads per wave and chunk: four of delta, two of a
constexpr int kIpStages = 6;
constexpr int kIpLds = kIpStages * kIpStage;      // 148.5 KiB

struct IpTileArgs {
  const LayerDev* layers;
  const int4* tiles;      // MODE 0, [8][slots]: (layer, e0, c0, first sample | samples << 16); layer < 0: none; else the
                          // entries of a tile list, of which `used` slots per XCD are launched
  float* out;             // MODE 0, [8 * slots][group][waves][2]: <tile_i, G tile>, sum of squares of tile_i;
                          // else [tile][B][waves]: sum of squares
  int slots, used, T, B, group;
  const int2* part;       // MODE 1 and 2: the list's (tile, first partial tile)
  float* partials;        // MODE 1: [pieces][256][128] fp32
  int accumulate;         // MODE 1: G += sum instead of G = sum
};

__device__ __attribute__((aligned(16))) const unsigned ip_zero_line[4] = {0, 0, 0, 0};

// Sum over the 64 lanes without the LDS round trips of a shuffle chain: four DPP steps leave the
// total of each row of 16 lanes in all of its lanes, the four row totals are then read as scalars.
__device__ __forceinline__ float ip_wave_sum_f32(float v) {
#define IP_DPP(x, ctrl) \
  __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, (x)), (ctrl), 0xf, 0xf, true))
  v += IP_DPP(v, 0xB1);    // quad_perm [1,0,3,2]
  v += IP_DPP(v, 0x4E);    // quad_perm [2,3,0,1]
  v += IP_DPP(v, 0x141);   // row_half_mirror
  v += IP_DPP(v, 0x140);   // row_mirror
#undef IP_DPP
  const int b = __builtin_bit_cast(int, v);
  return (__builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 0)) +
          __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 16))) +
         (__builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 32)) +
          __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 48)));
}

template <int N> __device__ __forceinline__ void ip_wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 0xf) | ((N >> 4) << 14));
}

// MODE 1 is the explicit form of the per-sample norms: when G has to be formed here anyway, its
// per-sample terms pass through the registers and the Gram contraction is not needed.
// SQ: also return the tile's sum of squares (always in MODE 1).  ODD: a sample has an odd number of chunks (the two
// fragment sets take turns, so that the loop over the samples is written for one parity).
template <int MODE, bool SQ, bool F16, bool RAGGED, bool ODD>
__global__ __launch_bounds__(64 * kIpWaves, 1) void ip_tile_kernel(IpTileArgs g) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int xcd = blockIdx.x % kNumXcd, seq = blockIdx.x / kNumXcd, slot = MODE == 2 ? seq % g.used : seq;
  const int entry = xcd * g.slots + slot;
  const int4 tile = g.tiles[entry];
  if (tile.x < 0) return;
  const SampleRun S = MODE == 0   ? SampleRun{tile.w & 0xffff, tile.w >> 16}
                      : MODE == 1 ? list_piece(tile.w, g.B, false)
                                  : list_run(tile.w, g.B, g.group, seq / g.used);
  if (S.count == 0) return;
  const int2 part = MODE == 0 ? int2{0, 0} : g.part[entry];
  const LayerDev L = g.layers[tile.x];
  const int e0 = tile.y, c0 = tile.z;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;        // 2 x 2 waves
  const int i16 = lane & 15, grp = lane >> 4;
  const int nk_sample = (g.T + kIpK - 1) / kIpK;  // chunks per sample
  const int nk = S.count * nk_sample;             // chunks of this entry: the host keeps it below 2^31
  const unsigned lds_base = lds_address(lds);     // LDS byte addresses are handled as integers

  // ---- second register set.  Accumulator element j of a 16x16 block: row grp * 4 + j, column i16.  MODE 0: this
  // lane's entries of the G tile (past the edge: the last ones, which meet nothing); MODE 1: running sum of the sample tiles.
  const int rows_in = L.d_out - e0 - wm * 128;    // rows of this wave's part that the layer has
  float gt[kIpFM][kIpFN][4];
  if constexpr (MODE != 2)
#pragma unroll
  for (int m = 0; m < kIpFM; ++m) {
    const bool in = m * 16 + grp * 4 < rows_in;   // (widths are multiples of 8: the four rows are in or out together)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int tr = e0 + wm * 128 + m * 16 + grp * 4 + j;
      const float* const row = MODE == 0 ? L.grad_sum + (size_t)(in ? tr : 0) * L.d_in : nullptr;
#pragma unroll
      for (int n = 0; n < kIpFN; ++n) {
        const float v = MODE == 0 ? row[std::min(c0 + wn * 64 + n * 16 + i16, L.d_in - 1)] : 0.f;
        gt[m][n][j] = in ? v : 0.f;
      }
    }
  }
  if (e0 + kIpE > L.d_out) {                      // the columns of delta past the edge stay zero throughout
    for (int o = threadIdx.x * 16; o < kIpLds; o += 64 * kIpWaves * 16)
      *reinterpret_cast<ip_u32x4*>(lds + o) = ip_u32x4{0, 0, 0, 0};
    __syncthreads();
  }

  // ---- direct loads.  Delta: block b = wave + 4 * i (i = 0..3) holds rows r and r + 16 (lanes 0-31, 32-63) with
  // r = (b & 3) | (b & 4) << 1 | (b & 8) >> 1, i.e. wave + {0, 8, 4, 12}[i].  a: block b = wave + 4 * i (i = 0, 1)
  // holds rows r, r + 4, r + 16, r + 20 (16 lanes each) with r = wave + 8 * i.  Address = first row of the chunk (scalar
  // registers) + a byte offset per lane, computed once (the host keeps row strides below 2^25).
  constexpr int kRowsE[4] = {0, 8, 4, 12};
  const int row_e = wave + 16 * (lane >> 5), row_c = wave + 4 * (grp & 1) + 16 * (grp >> 1);
  const int col_e = e0 + (lane & 31) * 8, col_c = std::min(c0 + i16 * 8, L.d_in - 8);
  unsigned off_e[4], off_c[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) off_e[i] = unsigned((row_e + kRowsE[i]) * L.delta_stride + col_e) * 2u;
#pragma unroll
  for (int i = 0; i < 2; ++i) off_c[i] = unsigned((row_c + 8 * i) * L.a_stride + col_c) * 2u;
  const unsigned long long all = __builtin_amdgcn_ballot_w64(lane < 64);   // (kept in scalar registers)
  const unsigned long long ok_e = __builtin_amdgcn_ballot_w64(col_e < L.d_out);
  const long long first = (long long)S.first * g.T;
  const unsigned short* pe = uniform_ptr(reinterpret_cast<const unsigned short*>(L.delta) + first * L.delta_stride);
  const unsigned short* pc = uniform_ptr(reinterpret_cast<const unsigned short*>(L.a) + first * L.a_stride);
  const unsigned ld_base = lds_base + wave * kIpBlk;
  int ld_left = g.T;                              // RAGGED: rows of the sample from the next chunk to load on
  auto issue_loads = [&](int i, unsigned st, unsigned long long on) {   // loads 2 * i and 2 * i + 1
    const unsigned to = ld_base + st + (i < 2 ? 2 * i * 4 * kIpBlk : kIpOpE);
    if (i < 2)
      direct_load_lds16_masked2(pe, off_e[2 * i], to, off_e[2 * i + 1], to + 4 * kIpBlk, ok_e & on);
    else
      direct_load_lds16_masked2(pc, off_c[0], to, off_c[1], to + 4 * kIpBlk, all & on);
  };
  auto next_chunk = [&]() {
    int step = kIpK;
    if (RAGGED) {
      step = ld_left < kIpK ? ld_left : kIpK;
      ld_left -= step;
      if (ld_left == 0) ld_left = g.T;
    }
    pe += step * L.delta_stride;
    pc += step * L.a_stride;
  };
  // all loads of a chunk with fewer than 32 rows
  auto issue_short_chunk = [&](unsigned st) {
    const unsigned char* z = reinterpret_cast<const unsigned char*>(ip_zero_line);
#pragma unroll
    for (int i = 0; i < kIpLd; ++i) {
      const bool e = i < 4;
      const unsigned char* p = reinterpret_cast<const unsigned char*>(e ? pe : pc) + (e ? off_e[i & 3] : off_c[i & 1]);
      const bool in = e ? row_e + kRowsE[i & 3] < ld_left && col_e < L.d_out : row_c + 8 * (i & 1) < ld_left;
      direct_load_lds16(in ? p : z, ld_base + st + (e ? i * 4 * kIpBlk : kIpOpE + (i - 4) * 4 * kIpBlk));
    }
  };

  // ---- fragments by LDS transpose reads.  Within a group of 16 lanes, lane s points at the 4 columns 4*(s%4).. of
  // token row 8*grp + s/4 (+ 4 for the second read); the read hands lane i column i of the group's 16 at the four
  // token rows: lane l ends up with column m0 + l%16, token rows (l/16)*8 + 0..7, the operand of a 16x16x32 MFMA.
  typedef __attribute__((address_space(3))) ip_s16x4* lds_ptr;
  const unsigned lane_rd = unsigned(((i16 >> 2) | (grp & 1) << 2) * kIpBlk + (grp >> 1) * 512 + (i16 & 3) * 8);
  const unsigned lane_e = lds_base + lane_rd + wm * 256, lane_c = lds_base + lane_rd + kIpOpE + wn * 128;
  struct Frags { ip_s16x4 v[kIpFN + kIpFM][2]; };  // a side, then delta side; first and last four token rows
  auto read1 = [&](int r, unsigned be, unsigned bc, Frags& f) {
    const int i = r >> 1, h = r & 1;
    if (i < kIpFN)
      f.v[i][h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(size_t)bc + (i * 32 + h * 256) / 8);
    else
      f.v[i][h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(size_t)be + ((i - kIpFN) * 32 + h * 8 * kIpBlk) / 8);
  };
  auto frag = [&](const Frags& f, int i) -> mfma_bf16x8 {
    ip_s16x8 v = {f.v[i][0][0], f.v[i][0][1], f.v[i][0][2], f.v[i][0][3], f.v[i][1][0], f.v[i][1][1], f.v[i][1][2], f.v[i][1][3]};
    return __builtin_bit_cast(mfma_bf16x8, v);
  };

  mfma_f32x4 acc[kIpFM][kIpFN];
#pragma unroll
  for (int m = 0; m < kIpFM; ++m)
#pragma unroll
    for (int n = 0; n < kIpFN; ++n)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[m][n][j] = 0.f;
  mfma_fence(acc);

  // Sums of a finished sample tile, by block column n: what a lane holds there lies in one column of the layer, so that
  // columns past the edge are left out once per sample (put_sample).
  float dot[kIpFN] = {0.f, 0.f, 0.f, 0.f}, sq[kIpFN] = {0.f, 0.f, 0.f, 0.f};
  const int cols_in = L.d_in - c0 - wn * 64 - i16;
  auto take_block = [&](int m, int n) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float v = mfma_acc(acc[m][n], j);
      if constexpr (MODE == 0) dot[n] = fmaf(v, gt[m][n][j], dot[n]);
      else if constexpr (MODE == 1) asm volatile("v_add_f32 %0, %0, %1" : "+v"(gt[m][n][j]) : "v"(v));   // (in place: no register to spare)
      if (SQ) sq[n] = fmaf(v, v, sq[n]);
    }
  };
  // (Before the first sample ends there is no finished tile: the cleared accumulators, which give NaN on an infinite
  // entry of G, are taken and not stored.)
  constexpr int kDst = MODE == 0 ? 2 : 1;         // floats per sample and wave
  float* const dst0 = g.out + ((MODE == 0 ? (size_t)entry * g.group : (size_t)part.x * g.B + S.first) * kIpWaves + wave) * kDst;
  float* dst = dst0 - kDst * kIpWaves;
  // Rows past the edge are sums of zeros times a: zero, or NaN where a column of a has an infinite entry or a NaN.  The
  // last eight rows of the wave's part, past the edge if any are, tell which.  In the second case the finished tile is
  // summed here row by row, before the fresh MFMAs overwrite it, and put_sample takes these sums.
  bool again = false;
  float dot_again = 0.f, sq_again = 0.f;
  auto check_rows = [&]() {
    again = false;
    if (rows_in >= kIpFM * 16) return;
    asm volatile("s_nop 15\n\ts_nop 15");         // (behind the last MFMA)
    bool bad = false;
#pragma unroll
    for (int n = 0; n < kIpFN; ++n) bad = bad || !(mfma_acc(acc[kIpFM - 1][n], 3) == 0.f);
    again = __builtin_amdgcn_ballot_w64(bad) >> 32 != 0;
    if (!again) return;
    float d[kIpFN] = {0.f, 0.f, 0.f, 0.f}, q[kIpFN] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int m = 0; m < kIpFM; ++m)
      if (m * 16 + grp * 4 < rows_in)
#pragma unroll
        for (int n = 0; n < kIpFN; ++n)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float v = mfma_acc(acc[m][n], j);
            if (MODE == 0) d[n] = fmaf(v, gt[m][n][j], d[n]);
            if (SQ) q[n] = fmaf(v, v, q[n]);
          }
    dot_again = sq_again = 0.f;
#pragma unroll
    for (int n = 0; n < kIpFN; ++n)
      if (n * 16 < cols_in) {
        dot_again += d[n];
        sq_again += q[n];
      }
  };
  auto put_sample = [&]() {
#pragma unroll
    for (int n = 0; n < kIpFN; ++n) {
      if (MODE == 0) dot[n] = n * 16 < cols_in ? dot[n] : 0.f;
      if (SQ) sq[n] = n * 16 < cols_in ? sq[n] : 0.f;
    }
    const float d = MODE == 0 ? ip_wave_sum_f32(again ? dot_again : (dot[0] + dot[1]) + (dot[2] + dot[3])) : 0.f;
    const float s = SQ ? ip_wave_sum_f32(again ? sq_again : (sq[0] + sq[1]) + (sq[2] + sq[3])) : 0.f;
    if (lane == 0 && dst >= dst0) {
      if (MODE == 0) {
        dst[0] = d;
        dst[1] = s;
      } else {
        dst[0] = s;
      }
    }
    dst += kDst * kIpWaves;
#pragma unroll
    for (int n = 0; n < kIpFN; ++n) dot[n] = sq[n] = 0.f;
  };

  // Chunk c's fragments are read during the MFMAs of chunk c-1, so that the stage of chunk c is free when its MFMAs
  // begin and takes chunk c + kIpStages there.
  const unsigned st_end = kIpStages * kIpStage;
  unsigned st = 0;                                // byte offset of the stage of chunk c
  // fresh: first chunk of a sample; on: all ones, or 0 where no whole chunk is left to load: the loads are then issued
  // with no lane taking part, so that the number of loads behind a chunk is always the same
  auto period = [&](auto fresh_tag, unsigned long long on, const Frags& cur, Frags& nxt) {
    constexpr bool fresh = decltype(fresh_tag)::value;
    const unsigned stn = st + kIpStage == st_end ? 0u : st + kIpStage;
    const unsigned be = lane_e + stn, bc = lane_c + stn;
#pragma unroll
    for (int i = 0; i < kIpFM * kIpFN; ++i) {
      const int m = i / kIpFN, n = m & 1 ? kIpFN - 1 - i % kIpFN : i % kIpFN;
      if (fresh) {
        take_block(m, n);
        mfma_16x16x32_fresh<F16>(acc[m][n], frag(cur, kIpFN + m), frag(cur, n));
      } else {
        mfma_16x16x32<F16>(acc[m][n], frag(cur, kIpFN + m), frag(cur, n));
      }
      if (i == 1) {
        // chunk c+1 has landed for me (the ones behind it may be in flight), then for everybody; everybody has
        // read all of chunk c
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        ip_wait_vmcnt<kIpLd * (kIpStages - 2)>();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      }
      if (i >= 2 && i < 2 + 2 * (kIpFM + kIpFN)) read1(i - 2, be, bc, nxt);   // (after the last chunk: in bounds)
      if (i % 8 == 7 && i / 8 < kIpLd / 2) issue_loads(i / 8, st, on);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (fresh)                                    // (or the compiler moves sums to where they are stored, 128 values with them)
#pragma unroll
      for (int n = 0; n < kIpFN; ++n) asm volatile("" : "+v"(dot[n]), "+v"(sq[n]));
    st = stn;
  };

  // prologue: kIpStages chunks in flight, chunk 0 landed
#pragma unroll
  for (int s = 0; s < kIpStages; ++s)
    if (s < nk) {
      if (RAGGED && ld_left < kIpK) {
        issue_short_chunk(s * kIpStage);
      } else {
#pragma unroll
        for (int i = 0; i < kIpLd / 2; ++i) issue_loads(i, s * kIpStage, ~0ull);
      }
      next_chunk();
    }
  // The G registers are needed only at the end of the first sample, but a wait placed there by the
  // compiler would drain the load pipeline at every sample; pin them down here, once.
  if constexpr (MODE != 2)
#pragma unroll
  for (int m = 0; m < kIpFM; ++m)
#pragma unroll
    for (int n = 0; n < kIpFN; ++n)
#pragma unroll
      for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(gt[m][n][j]));
  if (nk >= kIpStages) ip_wait_vmcnt<kIpLd * (kIpStages - 1)>(); else ip_wait_vmcnt<0>();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  Frags f0, f1;
#pragma unroll
  for (int r = 0; r < 2 * (kIpFM + kIpFN); ++r) read1(r, lane_e, lane_c, f0);

  int c = 0;                                      // chunk of the entry
  auto chunk = [&](auto fresh_tag, const Frags& cur, Frags& nxt) {
    const unsigned st_now = st;
    const bool more = c + kIpStages < nk;
    const bool whole = more && !(RAGGED && ld_left < kIpK);
    period(fresh_tag, whole ? ~0ull : 0ull, cur, nxt);
    if (RAGGED && more && !whole) issue_short_chunk(st_now);   // (the barrier inside the period has freed the stage)
    if (more) next_chunk();
    ++c;
  };
  const std::true_type fresh{};
  const std::false_type rest{};
  const int pairs = (nk_sample - 1) / 2;
  // One straight chain of definitions for the accumulators (no two code paths that join): the register allocator would
  // otherwise copy them from one set of registers to another in every chunk.
  for (;;) {
    chunk(fresh, f0, f1);
    put_sample();
    for (int p = 0; p < pairs; ++p) {
      chunk(rest, f1, f0);
      chunk(rest, f0, f1);
    }
    if (!ODD) chunk(rest, f1, f0);
    if (c >= nk) break;
    check_rows();
    if (ODD) {
      chunk(fresh, f1, f0);
      put_sample();
      for (int p = 0; p < pairs; ++p) {
        chunk(rest, f0, f1);
        chunk(rest, f1, f0);
      }
      if (c >= nk) break;
      check_rows();
    }
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  mfma_fence(acc);
  check_rows();
#pragma unroll
  for (int m = 0; m < kIpFM; ++m)
#pragma unroll
    for (int n = 0; n < kIpFN; ++n) take_block(m, n);
  put_sample();

  if constexpr (MODE == 1) {
    if (S.count < g.B) {
      float* pt = g.partials + (size_t)(part.y + (tile.w & 0xffff)) * (kIpE * kIpC);
#pragma unroll
      for (int m = 0; m < kIpFM; ++m)
#pragma unroll
        for (int n = 0; n < kIpFN; ++n)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            pt[(wm * 128 + m * 16 + grp * 4 + j) * kIpC + wn * 64 + n * 16 + i16] = gt[m][n][j];
    } else {
      put_grad_tile<kIpFM, kIpFN, 4>(L.grad_sum, L.d_out, L.d_in, e0 + wm * 128 + grp * 4, c0 + wn * 64 + i16,
                                     g.accumulate != 0, e0 + kIpE <= L.d_out && c0 + kIpC <= L.d_in,
                                     [&](int m, int n, int j) { return gt[m][n][j]; });
    }
  }
}

// ---------------------------------------------------------------------------------------
// The same tiles for short sequences (whole chunks): eight waves as 4 x 2, two per SIMD, wave tile 64 x 64, 32x32x16
// MFMA.  What a sample costs beyond its MFMAs -- the work on its finished tile, and the start and end of an entry -- runs
// next to the MFMAs of the SIMD's other wave here, while the four waves above have nothing to hide it behind; their
// cheaper chunks outweigh that on longer sequences (short_sequences()).
//   Staging: four stages of 32 token rows, loads two chunks ahead.  A load instruction moves token rows j, j + 16 of delta
//   (2 x 512 B) or rows j, j + 8, j + 16, j + 24 of a (4 x 256 B); the 1 KiB blocks are 1088 bytes apart so that the four
//   consecutive rows of a transpose read fall into different banks.  Columns past the edge re-read the last valid piece.
// ---------------------------------------------------------------------------------------
constexpr int kStBlk = 1024 + 64;                 // one load instruction + 64 B skew
constexpr int kStOpE = 16 * kStBlk;               // delta side of a stage
constexpr int kStOpC = 8 * kStBlk;                // a side of a stage
constexpr int kStStage = kStOpE + kStOpC;         // 25.5 KiB
constexpr int kStWM = 4, kStWN = 2;               // waves along d_out and d_in
constexpr int kStWaves = kStWM * kStWN;
constexpr int kStFM = kIpE / (32 * kStWM);        // 32x32 MFMA blocks per wave along d_out
constexpr int kStFN = kIpC / (32 * kStWN);        // ... along d_in
constexpr int kStLdE = 16 / kStWaves, kStLdC = 8 / kStWaves, kStLd = kStLdE + kStLdC;   // loads per wave
constexpr int kStStages = 4;
constexpr int kStLds = kStStages * kStStage;      // 102 KiB

__device__ __forceinline__ int st_row_off_e(int row) { return (row & 15) * kStBlk + (row >> 4) * 512; }
__device__ __forceinline__ int st_row_off_c(int row) { return (row & 7) * kStBlk + (row >> 3) * 256; }

template <int MODE, bool SQ, bool F16>
__global__ __launch_bounds__(64 * kStWaves, 1) void short_tile_kernel(IpTileArgs g) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int entry = blockIdx.x % kNumXcd * g.slots + blockIdx.x / kNumXcd;
  const int4 tile = g.tiles[entry];
  if (tile.x < 0) return;
  const SampleRun S = MODE == 0 ? SampleRun{tile.w & 0xffff, tile.w >> 16} : list_piece(tile.w, g.B, false);
  if (S.count == 0) return;
  const int2 part = MODE == 0 ? int2{0, 0} : g.part[entry];
  const LayerDev L = g.layers[tile.x];
  const int e0 = tile.y, c0 = tile.z;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / kStWN, wn = wave % kStWN;  // kStWM x kStWN waves
  const int nk_sample = g.T / kIpK;               // chunks per sample
  const long long ck0 = (long long)S.first * nk_sample;
  const int nk = S.count * nk_sample;              // chunks of this entry: the host keeps it below 2^31

  // ---- second register set.  Accumulator element j of a 32x32 block: row
  // (j/4)*8 + (lane/32)*4 + j%4, column lane%32.  MODE 0: this lane's entries of the G tile
  // (zero past the edge); MODE 1: running sum of the sample tiles.
  float gt[kStFM][kStFN][16];
#pragma unroll
  for (int m = 0; m < kStFM; ++m)
#pragma unroll
    for (int n = 0; n < kStFN; ++n) {
      const int tc = c0 + wn * (32 * kStFN) + n * 32 + (lane & 31);
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int tr = e0 + wm * (32 * kStFM) + m * 32 + (j >> 2) * 8 + (lane >> 5) * 4 + (j & 3);
        gt[m][n][j] = MODE == 0 ? L.grad_sum[(size_t)std::min(tr, L.d_out - 1) * L.d_in + std::min(tc, L.d_in - 1)] : 0.f;
      }
    }
  const bool edge = e0 + kIpE > L.d_out || c0 + kIpC > L.d_in;
  auto for_past_edge = [&](auto&& f) {
    int rows = L.d_out - e0 - wm * (32 * kStFM) - (lane >> 5) * 4, cols = L.d_in - c0 - wn * (32 * kStFN) - (lane & 31);
    asm volatile("" : "+v"(rows), "+v"(cols));     // (or the comparisons would be kept in registers across the loop)
#pragma unroll
    for (int m = 0; m < kStFM; ++m)
#pragma unroll
      for (int n = 0; n < kStFN; ++n)
#pragma unroll
        for (int j = 0; j < 16; ++j)
          if (n * 32 >= cols || m * 32 + (j >> 2) * 8 + (j & 3) >= rows) f(m, n, j);
  };
  if (MODE == 0 && edge) for_past_edge([&](int m, int n, int j) { gt[m][n][j] = 0.f; });

  // ---- direct loads, kStLd per wave and chunk: delta instructions j = wave, wave + kStWaves, ..
  // (rows j and j + 16, 16-byte piece lane % 32), then a instructions j = wave, .. (rows
  // j + 8 * (lane / 16), piece lane % 16).  Columns past the edge re-read the last valid piece.
  // Address = (first row of the chunk: wave-uniform, scalar registers) + (row within the chunk and
  // column: a 32-bit byte offset per lane, computed once; the host keeps row strides below 2^25).
  unsigned lane_off[kStLd];
  int lds_off[kStLd];
#pragma unroll
  for (int i = 0; i < kStLd; ++i) {
    const bool is_a = i >= kStLdE;
    const int j = wave + kStWaves * (is_a ? i - kStLdE : i);
    const int row = is_a ? j + 8 * (lane >> 4) : j + 16 * (lane >> 5);
    const int piece = is_a ? (lane & 15) : (lane & 31);
    const int d = is_a ? L.d_in : L.d_out;
    int col = (is_a ? c0 : e0) + piece * 8;
    col = col < d ? col : d - 8;
    lane_off[i] = unsigned(row * (is_a ? L.a_stride : L.delta_stride) + col) * 2u;
    lds_off[i] = (is_a ? kStOpE : 0) + j * kStBlk;
  }
  const unsigned short* const run_e = reinterpret_cast<const unsigned short*>(L.delta) + ck0 * kIpK * L.delta_stride;
  const unsigned short* const run_c = reinterpret_cast<const unsigned short*>(L.a) + ck0 * kIpK * L.a_stride;
  const unsigned lds_base = lds_address(lds);       // LDS byte addresses are handled as integers
  // stage indices are carried along (no modulo in the loop: kStStages need not be a power of two)
  auto issue_loads = [&](int c, int st) {
    const unsigned stage = lds_base + unsigned(st) * kStStage;
    const unsigned short* const pe = run_e + (long long)c * kIpK * L.delta_stride;
    const unsigned short* const pc = run_c + (long long)c * kIpK * L.a_stride;
#pragma unroll
    for (int i = 0; i < kStLd; ++i)
      direct_load_lds16_s(lane_off[i], i >= kStLdE ? pc : pe, stage + lds_off[i]);
  };

  // ---- fragments by LDS transpose reads.  Within a group of 16 lanes, lane s points at the 4
  // columns 4*(s%4).. of token row kbase + s/4; the read hands lane i column i of the group's
  // 16 at the four token rows.  Lane l ends up with column m0 + l%32, token rows
  // ks*16 + (l/32)*8 + 0..7.
  const int i16 = lane & 15;
  const int krow = (lane >> 5) * 8 + (i16 >> 2);              // + ks*16 (+4 for the upper half)
  const int ccol = ((lane >> 4) & 1) * 16 + (i16 & 3) * 4;    // column within a 32-wide block
  // Every read address of a k-step is stage + (a part that depends on the lane) + (a constant of the
  // fragment): three lane parts -- delta side; a side, rows r and r + 4, which wrap differently in
  // its 8-row blocks -- are kept in registers, the constants ride in the offset field of the read.
  typedef __attribute__((address_space(3))) ip_s16x4* lds_ptr;
  const unsigned lane_e = unsigned(st_row_off_e(krow) + (wm * (32 * kStFM) + ccol) * 2);
  const unsigned lane_c0 = unsigned(kStOpE + st_row_off_c(krow) + (wn * (32 * kStFN) + ccol) * 2);
  const unsigned lane_c1 = unsigned(kStOpE + st_row_off_c(krow + 4) + (wn * (32 * kStFN) + ccol) * 2);
  auto frag = [&](lds_ptr p0, lds_ptr p1) -> mfma_bf16x8 {
    ip_s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(p0);
    ip_s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(p1);
    ip_s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(mfma_bf16x8, v);
  };
  // token rows ks*16 + krow (+4) of the stage: row blocks of 16 (delta) and 8 (a) rows make ks * 512
  // bytes on both sides; 32 columns are 64 bytes; offsets in units of the 8-byte read
  auto read_frags = [&](int st, int ks, mfma_bf16x8 (&fa)[kStFM], mfma_bf16x8 (&fb)[kStFN]) {
    const unsigned stage = lds_base + unsigned(st) * kStStage;
    const lds_ptr be = (lds_ptr)(size_t)(stage + lane_e);
    const lds_ptr bc0 = (lds_ptr)(size_t)(stage + lane_c0), bc1 = (lds_ptr)(size_t)(stage + lane_c1);
#pragma unroll
    for (int m = 0; m < kStFM; ++m)
      fa[m] = frag(be + (ks * 512 + m * 64) / 8, be + (ks * 512 + m * 64 + 4 * kStBlk) / 8);
#pragma unroll
    for (int n = 0; n < kStFN; ++n)
      fb[n] = frag(bc0 + (ks * 512 + n * 64) / 8, bc1 + (ks * 512 + n * 64) / 8);
  };

  mfma_f32x16 acc[kStFM][kStFN];
#pragma unroll
  for (int m = 0; m < kStFM; ++m)
#pragma unroll
    for (int n = 0; n < kStFN; ++n)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[m][n][j] = 0.f;

  auto mfma4 = [&](const mfma_bf16x8 (&a)[kStFM], const mfma_bf16x8 (&b)[kStFN]) {
#pragma unroll
    for (int m = 0; m < kStFM; ++m)
#pragma unroll
      for (int n = 0; n < kStFN; ++n)
        acc[m][n] = mfma_32x32x16<F16>(a[m], b[n], acc[m][n]);
    // the LDS reads of the next k-step go out two at a time behind the first MFMAs
#pragma unroll
    for (int i = 0; i < kStFM + kStFN; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
    if (kStFM * kStFN > kStFM + kStFN)
      __builtin_amdgcn_sched_group_barrier(0x008, kStFM * kStFN - kStFM - kStFN, 0);
  };

  // prologue: chunks 0 .. kStStages-2 in flight
#pragma unroll
  for (int s = 0; s < kStStages - 1; ++s)
    if (s < nk) issue_loads(s, s);
  // The G registers are needed only at the end of the first sample, but a wait placed there by the
  // compiler would drain the load pipeline at every sample; pin them down here, once.
  if (MODE == 0) {
#pragma unroll
    for (int m = 0; m < kStFM; ++m)
#pragma unroll
      for (int n = 0; n < kStFN; ++n)
#pragma unroll
        for (int j = 0; j < 16; ++j) asm volatile("" : "+v"(gt[m][n][j]));
  }
  if (nk >= kStStages - 1) ip_wait_vmcnt<kStLd * (kStStages - 2)>(); else ip_wait_vmcnt<0>();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");

  int left = nk_sample, sample_out = 0;
  constexpr int kDst = MODE == 0 ? 2 : 1;         // floats per sample and wave
  float* dst = g.out + ((MODE == 0 ? (size_t)entry * g.group : (size_t)part.x * g.B + S.first) * kStWaves + wave) * kDst;
  mfma_bf16x8 fa[2][kStFM], fb[2][kStFN];
  read_frags(0, 0, fa[0], fb[0]);
  int st_cur = 0, st_load = kStStages - 1;        // stage of chunk c; stage that chunk c-1 frees
  for (int c = 0; c < nk; ++c) {
    const int st_next = st_cur + 1 == kStStages ? 0 : st_cur + 1;
    read_frags(st_cur, 1, fa[1], fb[1]);
    mfma4(fa[0], fb[0]);
    if (c + 1 < nk) {
      // chunk c+1 has landed for me (the chunks behind it may still be in flight), then for
      // everybody; every wave is done with chunk c-1, whose stage takes chunk c-1+kStStages
      if (c + kStStages - 2 < nk) ip_wait_vmcnt<kStLd * (kStStages - 3)>(); else ip_wait_vmcnt<0>();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      if (c + kStStages - 1 < nk) issue_loads(c + kStStages - 1, st_load);
    }
    read_frags(c + 1 < nk ? st_next : st_cur, 0, fa[0], fb[0]);
    mfma4(fa[1], fb[1]);
    st_load = st_cur;
    st_cur = st_next;
    if (--left == 0) {
      // the sample's tile is complete: reduce it against the G tile, clear it
      float dot = 0.f, sq = 0.f;
      if (edge) {
        // entries past the edge of the layer hold products of re-read columns, which must not enter a sum
        for_past_edge([&](int m, int n, int j) { acc[m][n][j] = 0.f; });
      }
#pragma unroll
      for (int m = 0; m < kStFM; ++m)
#pragma unroll
        for (int n = 0; n < kStFN; ++n)
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const float v = acc[m][n][j];
            if (MODE == 0) dot = fmaf(v, gt[m][n][j], dot);
            else gt[m][n][j] += v;
            if (SQ) sq = fmaf(v, v, sq);
            acc[m][n][j] = 0.f;
          }
      if (MODE == 0) dot = ip_wave_sum_f32(dot);
      if (SQ) sq = ip_wave_sum_f32(sq);
      if (lane == 0) {
        if (MODE == 0) {
          dst[size_t(sample_out) * (kDst * kStWaves)] = dot;
          dst[size_t(sample_out) * (kDst * kStWaves) + 1] = sq;
        } else {
          dst[size_t(sample_out) * (kDst * kStWaves)] = sq;
        }
      }
      ++sample_out;
      left = nk_sample;
    }
  }
  if constexpr (MODE == 1) {
    float* const pt = S.count < g.B ? g.partials + (size_t)(part.y + (tile.w & 0xffff)) * (kIpE * kIpC) : nullptr;
#pragma unroll
    for (int m = 0; m < kStFM; ++m)
#pragma unroll
      for (int n = 0; n < kStFN; ++n) {
        const int tc = wn * (32 * kStFN) + n * 32 + (lane & 31), tr0 = wm * (32 * kStFM) + m * 32 + (lane >> 5) * 4;
        if (pt) {
#pragma unroll
          for (int j = 0; j < 16; ++j) pt[(tr0 + (j >> 2) * 8 + (j & 3)) * kIpC + tc] = gt[m][n][j];
          continue;
        }
        // (the old entries are requested together, at addresses clamped to the layer; widths are multiples of 8: four
        // rows are in or out together)
        float was[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) was[j] = 0.f;
        if (g.accumulate) {
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const int r = std::min(e0 + tr0 + (j >> 2) * 8 + (j & 3), L.d_out - 1), c = std::min(c0 + tc, L.d_in - 1);
            was[j] = L.grad_sum[(size_t)r * L.d_in + c];
          }
        }
        if (c0 + tc < L.d_in)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (e0 + tr0 + q * 8 < L.d_out)
#pragma unroll
              for (int j = q * 4; j < q * 4 + 4; ++j) {
                float* const d = L.grad_sum + (size_t)(e0 + tr0 + q * 8 + (j & 3)) * L.d_in + c0 + tc;
                *d = g.accumulate ? was[j] + gt[m][n][j] : gt[m][n][j];
              }
      }
  }
}

// Statistics form: sums the partial tiles of the entries that were split along the samples, in
// piece order (fixed order: repeatable), into grad_sum.  One workgroup per 4 rows of a split tile,
// one thread per column, rows unrolled so that their loads are in flight together;
// split[t] = (layer, e0, c0, pieces << 16 | first partial tile).
constexpr int kIpRedRows = 4;
__global__ __launch_bounds__(kIpC) void stats_tile_reduce_kernel(const LayerDev* layers, const int4* split, int B,
                                                                const float* partials, int accumulate) {
  const int t = blockIdx.x / (kIpE / kIpRedRows), r0 = (blockIdx.x % (kIpE / kIpRedRows)) * kIpRedRows;
  const int4 S = split[t];
  const LayerDev L = layers[S.x];
  const int pieces = min(S.w >> 16, B);
  const float* base = partials + (size_t)(S.w & 0xffff) * (kIpE * kIpC) + threadIdx.x;
  const int col = S.z + threadIdx.x;
  float v[kIpRedRows];
#pragma unroll
  for (int r = 0; r < kIpRedRows; ++r) v[r] = 0.f;
  for (int p = 0; p < pieces; ++p)
#pragma unroll
    for (int r = 0; r < kIpRedRows; ++r) v[r] += base[(size_t)p * (kIpE * kIpC) + (r0 + r) * kIpC];
#pragma unroll
  for (int r = 0; r < kIpRedRows; ++r) {
    const int row = S.y + r0 + r;
    if (row >= L.d_out || col >= L.d_in) continue;
    float* d = L.grad_sum + (size_t)row * L.d_in + col;
    *d = accumulate ? *d + v[r] : v[r];
  }
}

// Statistics form: ||g_i^l||^2 = sum over the layer's tiles and waves of the tile's sum of squares, to where the common
// reduction picks it up.  One workgroup per (listed layer, sample); the tiles of the q-th listed layer lay[q] are
// ranges[q], .., ranges[q + 1] - 1.
__global__ __launch_bounds__(64) void stats_tile_finalize_kernel(const float* out, int waves, const int* lay,
                                                                const int* ranges, int B, float* partials) {
  const int q = blockIdx.x / B, i = blockIdx.x % B;
  double s = 0.0;
  for (int t = ranges[q] + threadIdx.x; t < ranges[q + 1]; t += 64) {
    const float* o = out + ((size_t)t * B + i) * waves;
    for (int w = 0; w < waves; w += 4)
#pragma unroll
      for (int v = 0; v < 4; ++v) s += double(o[w + v]);
  }
  s = ip_wave_sum(s);
  if (threadIdx.x == 0) partials[size_t(lay[q]) * B + i] = float(s);
}

// Tile table.  All tiles of one (layer, run of samples) stream the same rows, so such a set
// goes to one XCD (one L2); sets are dealt to the least loaded XCD, largest first.  The run
// length trades the once-per-entry costs (G tile, pipeline fill) against the balance of the last
// round of workgroups.
TileGeom ip_tile_geom() { return TileGeom{kIpE, kIpC, kIpK, kNumCu / kNumXcd}; }

// Cost in chunks: a run of s samples costs s * T/k + 8; `room` workgroups run at a time on each of the 8 XCDs.
int run_length(long long tiles, int B, int T, TileGeom geom) {
  const double per_sample = double((T + geom.k - 1) / geom.k), fixed = 8.0;
  double best = 0.0;
  int group = 1;
  for (int gsz = 1; gsz <= std::min(B, 0x7fff); ++gsz) {
    const long long runs = (B + gsz - 1) / gsz;
    const double rounds = std::ceil(double(tiles * runs) / (double(geom.room) * kNumXcd));
    const double cost = rounds * (gsz * per_sample + fixed);
    if (gsz == 1 || cost < best * 0.999) {
      best = cost;
      group = gsz;
    }
  }
  return group;
}

int make_ip_tiles(const std::vector<LayerDev>& layers, const std::vector<char>& use, int B, int T, TileGeom geom,
                  int forced_group, std::vector<int4>& out, int& group) {
  auto tiles_of = [&](const LayerDev& L) {
    return (long long)((L.d_out + geom.e - 1) / geom.e) * ((L.d_in + geom.c - 1) / geom.c);
  };
  long long tiles_all = 0;
  for (size_t l = 0; l < layers.size(); ++l)
    if (use[l]) tiles_all += tiles_of(layers[l]);
  group = run_length(tiles_all, B, T, geom);
  if (forced_group > 0) group = std::min(std::min(forced_group, B), 0x7fff);
  struct Set { int layer, s0, cnt; long long n; };
  std::vector<Set> sets;
  for (size_t l = 0; l < layers.size(); ++l) {
    if (!use[l]) continue;
    for (int s0 = 0; s0 < B; s0 += group)
      sets.push_back({int(l), s0, std::min(group, B - s0), tiles_of(layers[l])});
  }
  std::stable_sort(sets.begin(), sets.end(), [](const Set& x, const Set& y) {
    return x.n * x.cnt > y.n * y.cnt;
  });
  std::vector<std::vector<int4>> per(kNumXcd);
  std::vector<long long> load(kNumXcd, 0);
  for (const Set& S : sets) {
    int bx = 0;
    for (int x = 1; x < kNumXcd; ++x)
      if (load[x] < load[bx]) bx = x;
    load[bx] += S.n * S.cnt;
    const LayerDev& L = layers[S.layer];
    for_tiles_blocked((L.d_out + geom.e - 1) / geom.e, (L.d_in + geom.c - 1) / geom.c, geom.e / geom.c, [&](int e, int c) {
      per[bx].push_back(int4{S.layer, e * geom.e, c * geom.c, S.s0 | (S.cnt << 16)});
    });
  }
  size_t slots = 0;
  for (auto& v : per) slots = std::max(slots, v.size());
  out.assign(size_t(kNumXcd) * slots, int4{-1, 0, 0, 0});
  for (int x = 0; x < kNumXcd; ++x)
    for (size_t i = 0; i < per[x].size(); ++i) out[x * slots + i] = per[x][i];
  return int(slots);
}

template <int MODE, bool SQ, bool F16> static auto ip_tile_variant_t(int T) {
  const bool odd = (T + kIpK - 1) / kIpK % 2 != 0;
  if (T % kIpK != 0)
    return odd ? ip_tile_kernel<MODE, SQ, F16, true, true> : ip_tile_kernel<MODE, SQ, F16, true, false>;
  return odd ? ip_tile_kernel<MODE, SQ, F16, false, true> : ip_tile_kernel<MODE, SQ, F16, false, false>;
}
template <int MODE, bool SQ> static auto ip_tile_variant(int dtype, int T) {
  return dtype == ADLOCO_F16 ? ip_tile_variant_t<MODE, SQ, true>(T) : ip_tile_variant_t<MODE, SQ, false>(T);
}

template <typename K> static hipError_t launch_tiles(K kern, int waves, int lds, const IpTileArgs& a, hipStream_t st) {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  const unsigned runs = a.group > 0 && a.part ? unsigned((a.B + a.group - 1) / a.group) : 1u;
  hipLaunchKernelGGL(kern, dim3(unsigned(a.used) * runs * kNumXcd), dim3(64 * waves), lds, st, a);
  return hipGetLastError();
}

// True where the eight-wave kernel takes less time: T, and chunks of 32 token rows per compute unit (a small call does
// not reach the power limit, under which the four waves gain).  Measured, eight against four waves, gpt blocks of width
// d, us: statistics {d 1024, 6 blocks, B 5}: T 64 165 / 182, T 128 218 / 217, T 256 307 / 294; {768, 1 block, B 16}: T 128
// 57.8 / 62.4, T 256 83 / 87, T 512 140 / 138; {1024, 6, 16}: T 96 391 / 402, T 128 472 / 455; {1024, 1, 32}: T 160 182 /
// 189, T 256 259 / 258.  Inner products {1024, 6, 5}: T 64 171 / 202, T 128 214 / 242, T 256 307 / 313, T 512 514 / 480;
// {1024, 6, 16}: T 256 772 / 760; {1024, 1, 2}: T 512 72 / 78; {1024, 1, 5}: T 512 127 / 128, T 1024 216 / 203.
bool short_sequences(const std::vector<LayerDev>& layers, const std::vector<char>& use, int B, int T, bool inner_products) {
  if (T % kIpK != 0) return false;                // (whole chunks only)
  double tiles = 0.0;
  for (size_t l = 0; l < layers.size(); ++l)
    if (use[l]) tiles += double((layers[l].d_out + kIpE - 1) / kIpE) * double((layers[l].d_in + kIpC - 1) / kIpC);
  const double chunks = tiles * B * (T / kIpK) / kNumCu;
  if (inner_products) return T <= 128 || (T <= 256 && chunks < 600.0) || (T <= 512 && chunks < 100.0);
  return T <= 96 || (T <= 192 && chunks < 200.0) || (T <= 256 && tiles <= kNumCu);
}

int tile_waves(bool short_form) { return short_form ? kStWaves : kIpWaves; }

hipError_t launch_ip_tiles(const LayerDev* layers, const void* tiles, int slots, int T, int group,
                           int dtype, bool want_sq, bool short_form, float* ip_out, hipStream_t st) {
  if (slots <= 0) return hipSuccess;
  const IpTileArgs a{layers, static_cast<const int4*>(tiles), ip_out, slots, slots, T, 0, group, nullptr, nullptr, 0};
  if (short_form) {
    const bool h = dtype == ADLOCO_F16;
    auto kern = want_sq ? (h ? short_tile_kernel<0, true, true> : short_tile_kernel<0, true, false>)
                        : (h ? short_tile_kernel<0, false, true> : short_tile_kernel<0, false, false>);
    return launch_tiles(kern, kStWaves, kStLds, a, st);
  }
  return launch_tiles(want_sq ? ip_tile_variant<0, true>(dtype, T) : ip_tile_variant<0, false>(dtype, T), kIpWaves, kIpLds, a,
                      st);
}

hipError_t launch_square_tiles(const LayerDev* layers, const TileList& list, int B, int T, int dtype, float* out,
                               float* partials, hipStream_t st) {
  const IpTileArgs a{layers, list.tiles(), out, list.slots, list.used(1), T, B, run_length(list.n_tiles, B, T, ip_tile_geom()),
                     list.part(), nullptr, 0};
  hipError_t e = launch_tiles(ip_tile_variant<2, true>(dtype, T), kIpWaves, kIpLds, a, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(stats_tile_finalize_kernel, dim3(unsigned(list.n_listed) * B), dim3(64), 0, st, out, kIpWaves, list.layers(),
                     list.ranges(), B, partials);
  return hipGetLastError();
}

// The tiles of a layer go to one XCD where possible (they stream the same rows): all tiles in layer order (within a
// layer: blocks of tiles that share rows) are cut into eight equal runs, so that a layer stays on one XCD unless it
// straddles a cut, and the XCDs get the same number of tiles.  The tiles of an XCD's incomplete last round of workgroups
// can be split along the samples into as many pieces as fill the round, whose partial sums a small kernel adds up in
// piece order; all first pieces come first, then all second ones.
void make_tile_list(const std::vector<LayerDev>& layers, const std::vector<char>& use, TileGeom geom, bool split, TileList& list,
                    std::vector<int4>& tiles, std::vector<int2>& part, std::vector<int4>& split_tiles, std::vector<int>& csr,
                    int& n_pieces) {
  std::vector<int4> all;
  std::vector<int> lay, ranges(1, 0);
  for (size_t l = 0; l < layers.size(); ++l) {
    if (!use[l]) continue;
    for_tiles_blocked((layers[l].d_out + geom.e - 1) / geom.e, (layers[l].d_in + geom.c - 1) / geom.c, geom.e / geom.c,
                      [&](int e, int c) { all.push_back(int4{int(l), e * geom.e, c * geom.c, 1 << 16}); });
    lay.push_back(int(l));
    ranges.push_back(int(all.size()));
  }
  split_tiles.clear();
  n_pieces = 0;
  std::vector<std::vector<int4>> fin(kNumXcd);
  std::vector<std::vector<int2>> finp(kNumXcd);
  for (int x = 0; x < kNumXcd; ++x) {
    const size_t first = all.size() * x / kNumXcd;
    const int n = int(all.size() * (x + 1) / kNumXcd - first), full = n / geom.room * geom.room;
    int left = n - full, S = split && left > 0 ? geom.room / left : 1;
    if (S < 2 || n_pieces + left * S > 0xffff) left = 0, S = 1;
    list.n[x] = n;
    list.left[x] = left;
    list.pieces[x] = S;
    for (int p = 0; p < S; ++p)
      for (int i = p == 0 ? 0 : n - left; i < n; ++i) {
        int4 e = all[first + i];
        const int at = i < n - left ? 0 : n_pieces + (i - (n - left)) * S;
        e.w = i < n - left ? 1 << 16 : p | (S << 16);
        fin[x].push_back(e);
        finp[x].push_back(int2{int(first) + i, at});
        if (p == 0 && S > 1 && i >= n - left) split_tiles.push_back(int4{e.x, e.y, e.z, (S << 16) | at});
      }
    if (S > 1) n_pieces += left * S;
  }
  size_t slots = 0;
  for (auto& v : fin) slots = std::max(slots, v.size());
  tiles.assign(size_t(kNumXcd) * slots, int4{-1, 0, 0, 0});
  part.assign(size_t(kNumXcd) * slots, int2{0, 0});
  for (int x = 0; x < kNumXcd; ++x)
    for (size_t i = 0; i < fin[x].size(); ++i) {
      tiles[x * slots + i] = fin[x][i];
      part[x * slots + i] = finp[x][i];
    }
  list.edge = geom.e;
  list.slots = int(slots);
  list.n_tiles = int(all.size());
  list.n_split = int(split_tiles.size());
  list.n_listed = int(lay.size());
  csr = lay;
  csr.insert(csr.end(), ranges.begin(), ranges.end());
}

hipError_t launch_stats_tiles(const LayerDev* layers, const TileList& list, int B, int T, int dtype, int accumulate,
                              bool short_form, float* out, float* partials, hipStream_t st) {
  const IpTileArgs a{layers, list.tiles(), out, list.slots, list.used(B), T, B, B, list.part(),
                     static_cast<float*>(list.ptiles.ptr), accumulate};
  hipError_t e;
  if (short_form)
    e = launch_tiles(dtype == ADLOCO_F16 ? short_tile_kernel<1, true, true> : short_tile_kernel<1, true, false>, kStWaves,
                     kStLds, a, st);
  else
    e = launch_tiles(ip_tile_variant<1, true>(dtype, T), kIpWaves, kIpLds, a, st);
  if (e != hipSuccess) return e;
  if (list.n_split > 0 && B > 1)
    hipLaunchKernelGGL(stats_tile_reduce_kernel, dim3(unsigned(list.n_split) * (kIpE / kIpRedRows)), dim3(kIpC), 0, st,
                       layers, list.split(), B, a.partials, accumulate);
  hipLaunchKernelGGL(stats_tile_finalize_kernel, dim3(unsigned(list.n_listed) * B), dim3(64), 0, st, out,
                     tile_waves(short_form), list.layers(), list.ranges(), B, partials);
  return hipGetLastError();
}

// Vector blocks: v_i [d] is in `vec` (vector_rowsum_kernel); <v_i, G> -> dot[layer, sample].
__global__ __launch_bounds__(kIpThreads) void vector_ip_kernel(const LayerDev* layers, const AuxDesc* tab,
                                                              int B, const float* vec, float* dot) {
  __shared__ double lds4[4];
  const AuxDesc A = tab[blockIdx.x / B];
  const int sample = blockIdx.x % B;
  const LayerDev L = layers[A.layer];
  const float* v = vec + A.vec_off + (long long)sample * L.d_out;
  double acc = 0.0;
  for (int c = threadIdx.x; c < L.d_out; c += kIpThreads) acc += double(v[c]) * double(L.grad_sum[c]);
  const double s = ip_block_sum(acc, lds4);
  if (threadIdx.x == 0) dot[size_t(A.layer) * B + sample] = float(s);
}

// Embedding tables: <g_i, G> = sum_t <delta_t, G[id_t, :]>; ids outside [0, V) own no row of the
// table and contribute nothing.
template <typename E>
__global__ __launch_bounds__(kIpThreads) void embed_ip_kernel(const LayerDev* layers, const AuxDesc* tab,
                                                             int B, int T, float* dot) {
  __shared__ double lds4[4];
  const AuxDesc A = tab[blockIdx.x / B];
  const int sample = blockIdx.x % B;
  const LayerDev L = layers[A.layer];
  const int* ids = reinterpret_cast<const int*>(L.a) + (long long)sample * T;
  const E* D = reinterpret_cast<const E*>(L.delta) + (long long)sample * T * L.delta_stride;
  double acc = 0.0;
  for (int t = 0; t < T; ++t) {
    const int id = ids[t];
    if (id < 0 || id >= L.d_in) continue;
    const float* row = L.grad_sum + (size_t)id * L.d_out;
    float s = 0.f;
    for (int c = threadIdx.x; c < L.d_out; c += kIpThreads)
      s = fmaf(ip_elem(D[(long long)t * L.delta_stride + c]), row[c], s);
    acc += double(s);
  }
  const double s = ip_block_sum(acc, lds4);
  if (threadIdx.x == 0) dot[size_t(A.layer) * B + sample] = float(s);
}

// One workgroup per sample i: c_i = sum of its tile results + sum over the other blocks;
// likewise the explicit ||g_i||^2.  A tile entry covers samples [w & 0xffff, + (w >> 16)) and
// leaves, per sample and wave, a pair at tile_out[((k * group + sample - first) * waves + wave) * 2].
__global__ __launch_bounds__(kIpThreads) void ip_finalize_samples_kernel(
    const int4* tiles, const float* tile_out, long long n_tiles, int group, int waves, const float* dot, const float* sq,
    const unsigned char* in_tiles, int n_layers, int B, float* per_sample_ip, float* per_sample_sq,
    double* sample_f64) {
  __shared__ double lds4[4];
  const int i = blockIdx.x;
  double c = 0.0, q = 0.0;
  for (long long k = threadIdx.x; k < n_tiles; k += kIpThreads) {
    const int4 t = tiles[k];
    const int s0 = t.w & 0xffff, cnt = t.w >> 16;
    if (t.x >= 0 && i >= s0 && i < s0 + cnt) {
      const float* o = tile_out + ((size_t)k * group + (i - s0)) * (2 * waves);
      for (int w = 0; w < waves; w += 4)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          c += double(o[2 * (w + v)]);
          q += double(o[2 * (w + v) + 1]);
        }
    }
  }
  for (int l = threadIdx.x; l < n_layers; l += kIpThreads)
    if (!in_tiles[l]) {
      c += double(dot[size_t(l) * B + i]);
      q += double(sq[size_t(l) * B + i]);
    }
  const double cs = ip_block_sum(c, lds4);
  const double qs = ip_block_sum(q, lds4);
  if (threadIdx.x == 0) {
    per_sample_ip[i] = float(cs);
    if (per_sample_sq) per_sample_sq[i] = float(qs);
    sample_f64[i] = cs;
  }
}

// One workgroup: sum_ip (+)= sum_i c_i, sum_ip_sq (+)= sum_i c_i^2, n_samples (+)= B.
__global__ __launch_bounds__(1024) void ip_finalize_batch_kernel(const double* sample_f64, int B,
                                                                 adloco_ip_acc* acc, int accumulate) {
  __shared__ double lds[16];
  double a = 0.0, b = 0.0;
  for (int i = threadIdx.x; i < B; i += blockDim.x) {
    a += sample_f64[i];
    b += sample_f64[i] * sample_f64[i];
  }
  a = ip_wave_sum(a);
  b = ip_wave_sum(b);
  if ((threadIdx.x & 63) == 0) { lds[threadIdx.x >> 6] = a; }
  __syncthreads();
  double sa = 0.0;
  if (threadIdx.x == 0) for (int w = 0; w < 16; ++w) sa += lds[w];
  __syncthreads();
  if ((threadIdx.x & 63) == 0) { lds[threadIdx.x >> 6] = b; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double sb = 0.0;
    for (int w = 0; w < 16; ++w) sb += lds[w];
    if (accumulate) {
      acc->sum_ip += sa;
      acc->sum_ip_sq += sb;
      acc->n_samples += B;
    } else {
      acc->sum_ip = sa;
      acc->sum_ip_sq = sb;
      acc->n_samples = B;
    }
    acc->reserved = 0;
  }
}

hipError_t launch_ip_vector_table(const LayerDev* layers, const AuxDesc* vec_tab, int n_vec,
                                  const AuxDesc* emb_tab, int n_emb, int B, int T, int dtype,
                                  const float* vec, float* dot, hipStream_t st) {
  if (n_vec > 0)
    hipLaunchKernelGGL(vector_ip_kernel, dim3(unsigned(n_vec) * B), dim3(kIpThreads), 0, st, layers,
                       vec_tab, B, vec, dot);
  if (n_emb > 0) {
    if (dtype == ADLOCO_BF16)
      hipLaunchKernelGGL(embed_ip_kernel<unsigned short>, dim3(unsigned(n_emb) * B), dim3(kIpThreads), 0,
                         st, layers, emb_tab, B, T, dot);
    else if (dtype == ADLOCO_F16)
      hipLaunchKernelGGL(embed_ip_kernel<_Float16>, dim3(unsigned(n_emb) * B), dim3(kIpThreads), 0,
                         st, layers, emb_tab, B, T, dot);
    else
      hipLaunchKernelGGL(embed_ip_kernel<float>, dim3(unsigned(n_emb) * B), dim3(kIpThreads), 0, st,
                         layers, emb_tab, B, T, dot);
  }
  return hipGetLastError();
}

hipError_t launch_ip_finalize(const void* tiles, const float* tile_out, long long n_tiles, int group, int waves,
                              const float* dot, const float* sq, const unsigned char* in_tiles,
                              int n_layers, int B, float* per_sample_ip, float* per_sample_sq,
                              double* sample_f64, adloco_ip_acc* acc, int accumulate, hipStream_t st) {
  hipLaunchKernelGGL(ip_finalize_samples_kernel, dim3(B), dim3(kIpThreads), 0, st,
                     static_cast<const int4*>(tiles), tile_out, n_tiles, group, waves, dot, sq, in_tiles, n_layers, B,
                     per_sample_ip, per_sample_sq, sample_f64);
  hipLaunchKernelGGL(ip_finalize_batch_kernel, dim3(1), dim3(1024), 0, st, sample_f64, B, acc,
                     accumulate);
  return hipGetLastError();
}

}  // namespace adloco
