// Gradient sum of a linear layer over the batch: G^l (+)= sum_i delta_i^T a_i, i.e. B times
// the mini-batch gradient of eq. 1 (and Algorithm 3's "g <- g + grad L" across micro-batches).
// A GEMM [d_out, d_in] with the contraction over all B*T token rows.  Both operands are stored
// token-major (the contraction index is the slow one), so tiles are staged in LDS as they are
// and handed to the MFMA through the LDS transpose read of gfx950.
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace adloco {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef mfma_f32x4 f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;

struct WgradArgs {
  const LayerDev* layers;
  int n_layers;
  long long rows;      // B*T
  int accumulate;
};

__device__ __forceinline__ int find_layer_wg(const LayerDev* layers, int n_layers, int b) {
  int lo = 0, hi = n_layers - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (layers[mid].wg_blk_start <= b) lo = mid; else hi = mid - 1;
  }
  // layers with ADLOCO_GRAD_PROVIDED own no workgroup and share a start with their successor;
  // the search lands on the last layer with that start, which is the one that owns workgroups.
  return lo;
}

// ---------------------------------------------------------------------------------------
// bf16: 128 (d_out) x 128 (d_in) output tile per workgroup, 4 waves 2x2, MFMA 32x32x16.
// LDS stage: 32 token rows of delta[.,128] and of a[.,128], row pitch 144 elements.
// ---------------------------------------------------------------------------------------
constexpr int kWt = 128;
constexpr int kWk = 32;
constexpr int kWpitch = 144;                      // elements; 288 bytes
constexpr int kWopBytes = kWk * kWpitch * 2;      // one operand of one stage
constexpr int kWstage = 2 * kWopBytes;
constexpr int kWlds = 2 * kWstage;

struct WChunk { u32x4 v[4]; };

__device__ __forceinline__ void wgrad_load(const LayerDev& L, long long rows, long long k0, int e0,
                                           int c0, WChunk& r) {
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int e = threadIdx.x + 256 * it;
    const int op = e >> 9;                 // 0: delta (d_out side), 1: a (d_in side)
    const int row = (e & 511) >> 4;
    const int ch = e & 15;
    const unsigned short* base = reinterpret_cast<const unsigned short*>(op ? L.a : L.delta);
    const long long stride = op ? L.a_stride : L.delta_stride;
    const int d = op ? L.d_in : L.d_out;
    const int col = (op ? c0 : e0) + ch * 8;
    const long long k = k0 + row;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (k < rows && col < d) {
      const unsigned short* src = base + k * stride + col;
      if (L.fast) {
        v = *reinterpret_cast<const u32x4*>(src);
      } else {
        unsigned short h[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) h[j] = (col + j < d) ? src[j] : (unsigned short)0;
        v[0] = h[0] | (unsigned(h[1]) << 16);
        v[1] = h[2] | (unsigned(h[3]) << 16);
        v[2] = h[4] | (unsigned(h[5]) << 16);
        v[3] = h[6] | (unsigned(h[7]) << 16);
      }
    }
    r.v[it] = v;
  }
}

__device__ __forceinline__ void wgrad_store(unsigned char* stage, const WChunk& r) {
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int e = threadIdx.x + 256 * it;
    const int op = e >> 9;
    const int row = (e & 511) >> 4;
    const int ch = e & 15;
    *reinterpret_cast<u32x4*>(stage + op * kWopBytes + row * (kWpitch * 2) + ch * 16) = r.v[it];
  }
}

// Fragment of the MFMA operand for output rows/cols m0..m0+31 and k-step ks (16 token rows):
// lane l holds column m0 + l%32 at the eight token rows ks*16 + (l/32)*8 + 0..7.
template <int VARIANT>
__device__ __forceinline__ bf16x8 wgrad_frag(const unsigned char* op_base, int m0, int ks,
                                             int lane) {
  const int kbase = ks * 16 + (lane >> 5) * 8;
  if (VARIANT == 0) {
    // gather: eight 2-byte reads down one column
    const unsigned short* p =
        reinterpret_cast<const unsigned short*>(op_base) + kbase * kWpitch + m0 + (lane & 31);
    s16x8 v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = (short)p[j * kWpitch];
    return __builtin_bit_cast(bf16x8, v);
  } else {
    // LDS transpose read: within each group of 16 lanes, lane s points at 4 consecutive columns
    // of token row kbase + s/4 (columns 4*(s%4)..+3 of the group's 16); the instruction hands
    // lane i the four token rows of column i.
    const int i = lane & 15;
    const int colbase = m0 + ((lane >> 4) & 1) * 16 + (i & 3) * 4;
    const unsigned short* p =
        reinterpret_cast<const unsigned short*>(op_base) + (kbase + (i >> 2)) * kWpitch + colbase;
    typedef __attribute__((address_space(3))) s16x4* lds_ptr;
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p));
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + 4 * kWpitch));
    s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  }
}

template <int VARIANT, bool F16>
__device__ __forceinline__ void wgrad_mma(const unsigned char* stage, int wm, int wn, int lane,
                                          f32x16 (&acc)[2][2]) {
  const unsigned char* dt = stage;               // delta tile: rows = tokens, cols = d_out
  const unsigned char* at = stage + kWopBytes;   // a tile
#pragma unroll
  for (int ks = 0; ks < kWk / 16; ++ks) {
    bf16x8 fa[2], fb[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) fa[m] = wgrad_frag<VARIANT>(dt, wm * 64 + m * 32, ks, lane);
#pragma unroll
    for (int n = 0; n < 2; ++n) fb[n] = wgrad_frag<VARIANT>(at, wn * 64 + n * 32, ks, lane);
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int n = 0; n < 2; ++n)
        acc[m][n] = mfma_32x32x16<F16>(fa[m], fb[n], acc[m][n]);
  }
}

template <int VARIANT, bool F16>
__global__ __launch_bounds__(256, 2) void wgrad_bf16_kernel(WgradArgs g) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[kWlds];
  const int layer = find_layer_wg(g.layers, g.n_layers, blockIdx.x);
  const LayerDev L = g.layers[layer];
  const int tiles_c = (L.d_in + kWt - 1) / kWt;
  const int tile = blockIdx.x - L.wg_blk_start;
  const int e0 = (tile / tiles_c) * kWt;
  const int c0 = (tile % tiles_c) * kWt;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 1, wn = wave & 1;

  f32x16 acc[2][2];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[m][n][j] = 0.f;

  const long long nk = (g.rows + kWk - 1) / kWk;
  WChunk regs;
  wgrad_load(L, g.rows, 0, e0, c0, regs);
  wgrad_store(lds, regs);
  __syncthreads();
  for (long long c = 0; c < nk; ++c) {
    unsigned char* cur = lds + (c & 1) * kWstage;
    unsigned char* nxt = lds + ((c + 1) & 1) * kWstage;
    const bool more = c + 1 < nk;
    if (more) wgrad_load(L, g.rows, (c + 1) * kWk, e0, c0, regs);
    wgrad_mma<VARIANT, F16>(cur, wm, wn, lane, acc);
    if (more) wgrad_store(nxt, regs);
    __syncthreads();
  }

  // accumulator element j of a 32x32 block: row (j/4)*8 + (lane/32)*4 + j%4, column lane%32
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const int col = c0 + wn * 64 + n * 32 + (lane & 31);
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int row = e0 + wm * 64 + m * 32 + (j >> 2) * 8 + (lane >> 5) * 4 + (j & 3);
        if (row < L.d_out && col < L.d_in) {
          float* dst = L.grad_sum + (size_t)row * L.d_in + col;
          *dst = g.accumulate ? *dst + acc[m][n][j] : acc[m][n][j];
        }
      }
    }
}

// ---------------------------------------------------------------------------------------
// bf16 fast path: 256 (d_out) x 256 (d_in) output tile per workgroup of four waves (2 x 2, each 128 x 128, one per
// SIMD), used when every row is 16-byte aligned and widths are multiples of 8.  What bounds it is power: at 84 % busy matrix cores the chip holds 1.57 of its 2.4 GHz, so the kernel is laid
// out for little energy per product -- the 16x16x32 MFMA, and wave tiles of 128 x 128, which read a third less from LDS
// than eight waves of 128 x 64.  Sum over the 96 linears of the 350M model, 32 x 1024 tokens: 13.9 ms, 1.42 PFLOP/s,
// also where it is added to a sum (15.4 ms with every old entry of G loaded and waited for by itself)
// (eight waves with the 32x32x16 MFMA: 15.8 ms; four waves with it: 15.3 ms); without its global loads 11.4 ms, with
// loads that all hit the L2 12.9 ms.
//   Staging: global -> LDS directly, four stages of 32 token rows x (256 + 256) columns; one wave instruction moves
//   two token rows of one operand (2 x 512 contiguous bytes).
//   The operands of a chunk are read from LDS during the MFMAs of the chunk before, one read behind each MFMA, and
//   the direct loads go out one behind every other MFMA: with a single wave per SIMD anything issued in a burst would
//   leave the matrix core idle.  One barrier per chunk; loads run three chunks ahead.
//   Tiles are dealt to the XCDs layer by layer (table built on the host): the tiles of one layer run next to each
//   other on one XCD and stream the same columns out of that XCD's L2.
//   Columns beyond d_out / d_in re-read the last valid 16-byte piece; those accumulators are never stored.  Token rows
//   past the last one (in the last chunk) come from a line of zeros: 2 blocks of 1024 -> {3 x 1024, 1024, 4 x 1024},
//   16 x 77 tokens take 0.24 ms (128 x 128 kernel with register staging: 0.49 ms).
// ---------------------------------------------------------------------------------------
constexpr int kXt = 256;                          // tile edge
constexpr int kXk = 32;                           // token rows per stage
constexpr int kXrowB = kXt * 2;                   // bytes per staged row of one operand
constexpr int kXblk = 2 * kXrowB + 32;            // one load instruction: two rows, + 32 B pad
constexpr int kXop = 16 * kXblk;                  // 17 KiB
constexpr int kXstage = 2 * kXop;                 // 34 KiB
constexpr int kXstages = 4;
constexpr int kXthreads = 256;
constexpr int kXlds = kXstages * kXstage;         // 136 KiB

__device__ __attribute__((aligned(16))) const unsigned wgx_zero_line[4] = {0, 0, 0, 0};

struct WgradXArgs {
  const LayerDev* layers;
  const int4* tiles;      // [8][slots]: (layer, e0, c0, split); layer < 0 = no tile.
                          // split = 0: whole contraction, result goes to grad_sum;
                          // else (S << 24) | (piece << 16) | slot: piece of S equal parts of
                          // the contraction, result goes to partial tile `slot` of `partials`
  float* partials;        // [pieces][256][256] fp32
  int slots;
  long long rows;
  int accumulate;
};

template <int N> __device__ __forceinline__ void wgx_wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 0xf) | ((N >> 4) << 14));
}

// Token row of a chunk that half h of LDS block b holds.  Blocks are 1056 bytes apart, i.e. block b starts
// 32 * (b % 8) bytes into the 256 bytes of the banks; a transpose read touches, per 32 lanes, 32 bytes of the rows
// 0..3 and 8..11 (or another such octet), which this order puts into blocks of all eight residues: no conflicts.
__device__ __forceinline__ int wgx_row(int b, int h) { return (b & 3) | (b & 8) >> 1 | (b & 4) << 1 | h << 4; }

template <bool F16>
__global__ __launch_bounds__(kXthreads, 1) void wgrad_bf16_x_kernel(WgradXArgs g) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int xcd = blockIdx.x % kNumXcd, slot = blockIdx.x / kNumXcd;
  const int4 tile = g.tiles[xcd * g.slots + slot];
  if (tile.x < 0) return;
  const LayerDev L = g.layers[tile.x];
  const int e0 = tile.y, c0 = tile.z;
  const int split_s = (tile.w >> 24) & 0xff, split_p = (tile.w >> 16) & 0xff, split_id = tile.w & 0xffff;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;        // 2 x 2 waves; wave tile 128 (e) x 128 (c)
  // chunk range of this workgroup: everything, or piece split_p of split_s equal parts
  // (32-bit counters keep the loop's compares on the scalar unit; the host keeps rows / 32 < 2^31)
  const long long nk_all = (g.rows + kXk - 1) / kXk;
  const long long ck0 = split_s ? nk_all * split_p / split_s : 0;
  const int nk = int((split_s ? nk_all * (split_p + 1) / split_s : nk_all) - ck0);
  // rows of the last chunk of this workgroup
  const long long rest = g.rows - (ck0 + nk - 1) * kXk;
  const int last_rows = rest < kXk ? int(rest) : kXk;

  // ---- direct loads: block b = wave + 4 * q (q = 0..3) of each operand, 16-byte piece lane % 32 of row
  // wgx_row(b, lane / 32).  Address = (first row of the chunk: scalar registers) + (row within the chunk and
  // column: a 32-bit byte offset per lane, computed once; the host keeps row strides below 2^25).
  unsigned lane_off[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int op = i >> 2;                        // 0: delta (d_out side), 1: a (d_in side)
    const int row = wgx_row(wave + 4 * (i & 3), lane >> 5);
    const int d = op ? L.d_in : L.d_out;
    int col = (op ? c0 : e0) + (lane & 31) * 8;
    col = col < d ? col : d - 8;
    lane_off[i] = unsigned(row * (op ? L.a_stride : L.delta_stride) + col) * 2u;
  }
  const unsigned short* pe = uniform_ptr(reinterpret_cast<const unsigned short*>(L.delta) + ck0 * kXk * L.delta_stride);
  const unsigned short* pc = uniform_ptr(reinterpret_cast<const unsigned short*>(L.a) + ck0 * kXk * L.a_stride);
  const unsigned lds_base = lds_address(lds);       // LDS byte addresses are handled as integers
  const unsigned ld_base = lds_base + wave * kXblk;
  // load i of this wave for the chunk at pe / pc, into stage st
  auto issue_load = [&](int i, unsigned st) {
    direct_load_lds16_s(lane_off[i], i >= 4 ? pc : pe,
                        ld_base + st + (i >> 2) * kXop + (i & 3) * 4 * kXblk);
  };
  // all loads of chunk c at once; the last chunk may be short
  auto issue_chunk = [&](int c, unsigned st) {
    if (c == nk - 1 && last_rows < kXk) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const unsigned char* p = reinterpret_cast<const unsigned char*>(i >= 4 ? pc : pe) + lane_off[i];
        const bool ok = wgx_row(wave + 4 * (i & 3), lane >> 5) < last_rows;
        direct_load_lds16(ok ? p : reinterpret_cast<const unsigned char*>(wgx_zero_line),
                          ld_base + st + (i >> 2) * kXop + (i & 3) * 4 * kXblk);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) issue_load(i, st);
    }
  };
  auto next_chunk = [&]() {
    pe += kXk * L.delta_stride;
    pc += kXk * L.a_stride;
  };

  // ---- fragments by LDS transpose reads.  Within a group of 16 lanes, lane s points at the 4 columns 4*(s%4).. of
  // token row 8*(lane/16) + s/4 (+ 4 for the second read); the read hands lane i column i of the group's 16 at the
  // four token rows.  Lane l ends up with column m0 + l%16, token rows (l/16)*8 + 0..7: the operand of a 16x16x32
  // MFMA.  Every read address is stage + (a part that depends on the lane) + (a constant of the fragment).
  const int i16 = lane & 15, grp = lane >> 4;
  typedef __attribute__((address_space(3))) s16x4* lds_ptr;
  const unsigned lane_rd = unsigned(((i16 >> 2) | (grp & 1) << 2) * kXblk + (grp >> 1) * kXrowB + (i16 & 3) * 8);
  const unsigned lane_e = lds_base + lane_rd + wm * 256, lane_c = lds_base + lane_rd + kXop + wn * 256;
  struct Frags { s16x4 v[16][2]; };                // [0..7] a side, [8..15] delta side; first and last four token rows
  auto read1 = [&](int r, unsigned be, unsigned bc, Frags& f) {
    const int i = r >> 1, h = r & 1;
    const lds_ptr p = (lds_ptr)(size_t)(i < 8 ? bc : be);
    f.v[i][h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(p + ((i & 7) * 32 + h * 8 * kXblk) / 8);
  };
  auto frag = [&](const Frags& f, int i) -> bf16x8 {
    s16x8 v = {f.v[i][0][0], f.v[i][0][1], f.v[i][0][2], f.v[i][0][3], f.v[i][1][0], f.v[i][1][1], f.v[i][1][2], f.v[i][1][3]};
    return __builtin_bit_cast(bf16x8, v);
  };

  f32x4 acc[8][8];
#pragma unroll
  for (int m = 0; m < 8; ++m)
#pragma unroll
    for (int n = 0; n < 8; ++n)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[m][n][j] = 0.f;
  mfma_fence(acc);

  // Chunk c's fragments are read during the MFMAs of chunk c-1, so that stage c mod 4 is free when chunk c's MFMAs
  // begin and takes chunk c+4 there.
  const unsigned st_end = kXstages * kXstage;
  unsigned st = 0;                                 // byte offset of the stage of chunk c
  auto period = [&](auto tail_tag, int c, const Frags& cur, Frags& nxt) {
    constexpr bool tail = decltype(tail_tag)::value;
    const unsigned stn = st + kXstage == st_end ? 0u : st + kXstage;
    const unsigned be = lane_e + stn, bc = lane_c + stn;
    #pragma unroll
    for (int i = 0; i < 64; ++i) {
      const int m = i >> 3, n = m & 1 ? 7 - (i & 7) : i & 7;
      mfma_16x16x32<F16>(acc[m][n], frag(cur, 8 + m), frag(cur, n));
      if (i == 1 && (!tail || c + 1 < nk)) {
        // chunk c+1 has landed for me (the two behind it may be in flight), then for everybody; everybody has
        // read all of chunk c
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (!tail || c + 3 < nk) wgx_wait_vmcnt<16>(); else if (c + 2 < nk) wgx_wait_vmcnt<8>(); else wgx_wait_vmcnt<0>();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      }
      if (i >= 2 && i < 34) read1(i - 2, be, bc, nxt);   // (after the last chunk: of no use, but in bounds)
      if (!tail && i >= 36 && i < 52 && (i & 1)) issue_load((i - 36) >> 1, st);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (tail && c + kXstages < nk) {
      issue_chunk(c + kXstages, st);
      next_chunk();
    }
    if (!tail) next_chunk();
    st = stn;
  };

  // prologue: chunks 0 .. 3 in flight, chunk 0 landed
#pragma unroll
  for (int s = 0; s < kXstages; ++s)
    if (s < nk) {
      issue_chunk(s, s * kXstage);
      next_chunk();
    }
  if (nk >= kXstages) wgx_wait_vmcnt<24>(); else wgx_wait_vmcnt<0>();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  Frags f0, f1;
#pragma unroll
  for (int r = 0; r < 32; ++r) read1(r, lane_e, lane_c, f0);
  int c = 0;
  for (; c + 2 + kXstages < nk; c += 2) {          // (the last chunk is loaded in the loop below)
    period(std::false_type{}, c, f0, f1);
    period(std::false_type{}, c + 1, f1, f0);
  }
  for (; c < nk; c += 2) {
    period(std::true_type{}, c, f0, f1);
    if (c + 1 < nk) period(std::true_type{}, c + 1, f1, f0);
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  mfma_fence(acc);

  // accumulator element j of a 16x16 block: row (lane/16)*4 + j, column lane%16
  if (split_s) {
    float* part = g.partials + (size_t)split_id * (kXt * kXt);
#pragma unroll
    for (int m = 0; m < 8; ++m)
#pragma unroll
      for (int n = 0; n < 8; ++n)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          part[(wm * 128 + m * 16 + grp * 4 + j) * kXt + wn * 128 + n * 16 + i16] = acc[m][n][j];
  } else {
    put_grad_tile<8, 8, 4>(L.grad_sum, L.d_out, L.d_in, e0 + wm * 128 + grp * 4, c0 + wn * 128 + i16,
                           g.accumulate != 0, e0 + kXt <= L.d_out && c0 + kXt <= L.d_in,
                           [&](int m, int n, int j) { return acc[m][n][j]; });
  }
}

// Sums the partial tiles of a split contraction in piece order (fixed order: repeatable) and adds them to / stores
// them in grad_sum.  One workgroup per 4 rows of one split tile, one thread per column; bound by the latency of its
// loads, so the old entries of G and those of four pieces are requested together (48 tiles of 256 x 256 in five
// pieces: piece by piece, G last, 14 us).
struct WgradSplitTile { int layer, e0, c0, w; };   // w = (pieces << 16) | first partial tile
constexpr int kXredRows = 4;
__global__ __launch_bounds__(kXt) void wgrad_reduce_kernel(const LayerDev* layers, const WgradSplitTile* tiles,
                                                           const float* partials, int accumulate) {
  const int t = blockIdx.x / (kXt / kXredRows), r0 = (blockIdx.x % (kXt / kXredRows)) * kXredRows;
  const WgradSplitTile S = tiles[t];
  const LayerDev L = layers[S.layer];
  const int pieces = S.w >> 16;
  const float* base = partials + (size_t)(S.w & 0xffff) * (kXt * kXt) + r0 * kXt + threadIdx.x;
  const int col = S.c0 + threadIdx.x;
  float old[kXredRows], v[kXredRows];
#pragma unroll
  for (int r = 0; r < kXredRows; ++r) {
    const int row = S.e0 + r0 + r;
    old[r] = accumulate && row < L.d_out && col < L.d_in ? L.grad_sum[(size_t)row * L.d_in + col] : 0.f;
    v[r] = 0.f;
  }
  constexpr int kAhead = 4;
  for (int p = 0; p < pieces; p += kAhead) {
    float x[kAhead][kXredRows];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      const int pp = p + q < pieces ? p + q : pieces - 1;
#pragma unroll
      for (int r = 0; r < kXredRows; ++r) x[q][r] = base[(size_t)pp * (kXt * kXt) + r * kXt];
    }
#pragma unroll
    for (int q = 0; q < kAhead; ++q)
#pragma unroll
      for (int r = 0; r < kXredRows; ++r) v[r] += p + q < pieces ? x[q][r] : 0.f;
  }
#pragma unroll
  for (int r = 0; r < kXredRows; ++r) {
    const int row = S.e0 + r0 + r;
    if (row < L.d_out && col < L.d_in)
      L.grad_sum[(size_t)row * L.d_in + col] = accumulate ? old[r] + v[r] : v[r];
  }
}

// ---------------------------------------------------------------------------------------
// fp32 inputs: plain FMA path, 32x32 output tile, 2x2 entries per thread.
// ---------------------------------------------------------------------------------------
constexpr int kWtF = 32;
constexpr int kWkF = 16;

__global__ __launch_bounds__(256) void wgrad_f32_kernel(WgradArgs g) {
  __shared__ float sd[kWkF][kWtF + 1];
  __shared__ float sa[kWkF][kWtF + 1];
  const int layer = find_layer_wg(g.layers, g.n_layers, blockIdx.x);
  const LayerDev L = g.layers[layer];
  const int tiles_c = (L.d_in + kWtF - 1) / kWtF;
  const int tile = blockIdx.x - L.wg_blk_start;
  const int e0 = (tile / tiles_c) * kWtF;
  const int c0 = (tile % tiles_c) * kWtF;
  const float* D = reinterpret_cast<const float*>(L.delta);
  const float* A = reinterpret_cast<const float*>(L.a);
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  float acc[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
  for (long long k0 = 0; k0 < g.rows; k0 += kWkF) {
    for (int e = threadIdx.x; e < kWkF * kWtF; e += 256) {
      const int row = e / kWtF, col = e % kWtF;
      const long long k = k0 + row;
      sd[row][col] = (k < g.rows && e0 + col < L.d_out) ? D[k * L.delta_stride + e0 + col] : 0.f;
      sa[row][col] = (k < g.rows && c0 + col < L.d_in) ? A[k * L.a_stride + c0 + col] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kWkF; ++k) {
      const float d0 = sd[k][ty * 2], d1 = sd[k][ty * 2 + 1];
      const float a0 = sa[k][tx * 2], a1 = sa[k][tx * 2 + 1];
      acc[0][0] = fmaf(d0, a0, acc[0][0]);
      acc[0][1] = fmaf(d0, a1, acc[0][1]);
      acc[1][0] = fmaf(d1, a0, acc[1][0]);
      acc[1][1] = fmaf(d1, a1, acc[1][1]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int row = e0 + ty * 2 + i, col = c0 + tx * 2 + j;
      if (row < L.d_out && col < L.d_in) {
        float* dst = L.grad_sum + (size_t)row * L.d_in + col;
        *dst = g.accumulate ? *dst + acc[i][j] : acc[i][j];
      }
    }
}

int wgrad_tile_edge(int dtype) { return is_16bit(dtype) ? kWt : kWtF; }

// Tile table of the fast kernel: [8 XCDs][slots] entries (layer, e0, c0, split).  The tiles of
// all layers, in layer order, are cut into eight equal runs, one per XCD: the tiles of a layer
// stream the same rows out of one L2 (a layer that straddles a cut out of two), and no XCD has
// more work than another.
// All tiles cost the same, so an XCD's 32 CUs work in rounds; the tiles of an incomplete last
// round are split along the contraction into as many pieces as fill the round, written to
// partial tiles and summed afterwards by wgrad_reduce_kernel.
int make_wgrad_x_tiles(const std::vector<LayerDev>& layers, std::vector<int4>& out,
                       std::vector<int4>& split_tiles, int& n_pieces) {
  constexpr int kCuPerXcd = kNumCu / kNumXcd;
  // all tiles in layer order (within a layer: blocks of tiles that share rows), cut into eight
  // equal runs: a layer stays on one XCD unless it straddles a cut, and the XCDs get the same
  // number of tiles
  std::vector<int4> all;
  for (size_t l = 0; l < layers.size(); ++l) {
    if (layers[l].provided || layers[l].kind != ADLOCO_KIND_LINEAR) continue;
    for_tiles_blocked((layers[l].d_out + kXt - 1) / kXt, (layers[l].d_in + kXt - 1) / kXt, 1,
                      [&](int e, int c) { all.push_back(int4{int(l), e * kXt, c * kXt, 0}); });
  }
  std::vector<std::vector<int4>> per(kNumXcd);
  for (int x = 0; x < kNumXcd; ++x)
    for (size_t i = all.size() * x / kNumXcd; i < all.size() * (x + 1) / kNumXcd; ++i)
      per[x].push_back(all[i]);
  split_tiles.clear();
  n_pieces = 0;
  std::vector<std::vector<int4>> fin(kNumXcd);
  for (int x = 0; x < kNumXcd; ++x) {
    const int n = int(per[x].size());
    const int full = n / kCuPerXcd * kCuPerXcd, left = n - full;
    const int S = left > 0 ? kCuPerXcd / left : 1;
    for (int i = 0; i < full; ++i) fin[x].push_back(per[x][i]);
    for (int i = full; i < n; ++i) {
      if (S < 2 || n_pieces + S > 0xffff) {
        fin[x].push_back(per[x][i]);
        continue;
      }
      split_tiles.push_back(int4{per[x][i].x, per[x][i].y, per[x][i].z, (S << 16) | n_pieces});
      for (int p = 0; p < S; ++p) {
        int4 e = per[x][i];
        e.w = (S << 24) | (p << 16) | (n_pieces + p);
        fin[x].push_back(e);
      }
      n_pieces += S;
    }
  }
  size_t slots = 0;
  for (auto& v : fin) slots = std::max(slots, v.size());
  out.assign(size_t(kNumXcd) * slots, int4{-1, 0, 0, 0});
  for (int x = 0; x < kNumXcd; ++x)
    for (size_t i = 0; i < fin[x].size(); ++i) out[x * slots + i] = fin[x][i];
  return int(slots);
}

hipError_t launch_wgrad_x(const LayerDev* layers, const void* tiles, int slots,
                          const void* split_tiles, int n_split, float* partials, long long rows,
                          int accumulate, int dtype, hipStream_t st) {
  if (slots <= 0) return hipSuccess;
  auto kern = dtype == ADLOCO_F16 ? wgrad_bf16_x_kernel<true> : wgrad_bf16_x_kernel<false>;
  {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kXlds);
    if (e != hipSuccess) return e;
  }
  WgradXArgs a{layers, static_cast<const int4*>(tiles), partials, slots, rows, accumulate};
  hipLaunchKernelGGL(kern, dim3(unsigned(slots * kNumXcd)), dim3(kXthreads), kXlds, st, a);
  if (n_split > 0)
    hipLaunchKernelGGL(wgrad_reduce_kernel, dim3(unsigned(n_split) * (kXt / kXredRows)), dim3(256), 0, st, layers,
                       static_cast<const WgradSplitTile*>(split_tiles), partials, accumulate);
  return hipGetLastError();
}

hipError_t launch_wgrad(const LayerDev* layers, int n_layers, int n_blocks, long long rows,
                        int dtype, int accumulate, int variant, hipStream_t st) {
  if (n_blocks <= 0) return hipSuccess;
  WgradArgs a{layers, n_layers, rows, accumulate};
  if (is_16bit(dtype)) {
    const bool h = dtype == ADLOCO_F16;
    auto kern = variant == 0 ? (h ? wgrad_bf16_kernel<0, true> : wgrad_bf16_kernel<0, false>)
                             : (h ? wgrad_bf16_kernel<1, true> : wgrad_bf16_kernel<1, false>);
    hipLaunchKernelGGL(kern, dim3(n_blocks), dim3(256), 0, st, a);
  } else {
    hipLaunchKernelGGL(wgrad_f32_kernel, dim3(n_blocks), dim3(256), 0, st, a);
  }
  return hipGetLastError();
}

}  // namespace adloco
