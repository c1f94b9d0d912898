// Internal definitions shared by the translation units of libadloco (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "adloco.h"
#include "adloco_internal.h"

namespace adloco {

// 16-bit element types: bf16 and IEEE half share every data path (they are moved as 16-bit lanes);
// only the MFMA instruction and the conversion to fp32 differ.
inline bool is_16bit(int dtype) { return dtype == ADLOCO_BF16 || dtype == ADLOCO_F16; }
typedef __attribute__((ext_vector_type(8))) __bf16 mfma_bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 mfma_f16x8;
typedef __attribute__((ext_vector_type(16))) float mfma_f32x16;
// One 32x32x16 MFMA on fragments held as bf16x8 bit patterns; F16 reinterprets them as halves.
template <bool F16>
__device__ __forceinline__ mfma_f32x16 mfma_32x32x16(mfma_bf16x8 a, mfma_bf16x8 b, mfma_f32x16 c) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(mfma_f16x8, a),
                                                  __builtin_bit_cast(mfma_f16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

typedef __attribute__((ext_vector_type(4))) float mfma_f32x4;
// One 16x16x32 MFMA with the accumulator pinned to the accumulation registers.  Under the chip's power limit this form
// is worth about 15 % over 32x32x16: a loop of MFMAs fed from LDS with Gaussian bf16 data, four waves of 128 x 128 per
// compute unit, runs at 1917 TFLOP/s against 1672 (1.83 against 1.67 PFLOP/s with eight waves of 128 x 64); on zeros,
// where power does not limit, both reach 2.41.  Inline assembly because the compiler otherwise parks operand registers
// in the accumulation half of the register file inside the loop.  It does not see the hazards of an MFMA in assembly:
// call mfma_fence() on the accumulators between their last MFMA and the first ordinary instruction that reads them, and
// between ordinary writes and the first MFMA.
template <bool F16>
__device__ __forceinline__ void mfma_16x16x32(mfma_f32x4& c, mfma_bf16x8 a, mfma_bf16x8 b) {
  if constexpr (F16)
    asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
  else
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
// The same instruction with its scheduling and registers left to the compiler.
template <bool F16>
__device__ __forceinline__ mfma_f32x4 mfma_16x16x32_v(mfma_bf16x8 a, mfma_bf16x8 b, mfma_f32x4 c) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(mfma_f16x8, a), __builtin_bit_cast(mfma_f16x8, b), c,
                                                  0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// The same with the accumulator in vector registers.
template <bool F16>
__device__ __forceinline__ void mfma_16x16x32_vgpr(mfma_f32x4& c, mfma_bf16x8 a, mfma_bf16x8 b) {
  if constexpr (F16)
    asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
  else
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
// The same from zero: the old accumulators are only overwritten.  A reader of the old values in between needs no fence
// if many MFMAs lie between the one that wrote them and itself.
template <bool F16>
__device__ __forceinline__ void mfma_16x16x32_fresh(mfma_f32x4& c, mfma_bf16x8 a, mfma_bf16x8 b) {
  if constexpr (F16)
    asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, 0" : "+a"(c) : "v"(a), "v"(b));
  else
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "+a"(c) : "v"(a), "v"(b));
}
// Element j of an accumulator block, read in place.
__device__ __forceinline__ float mfma_acc(const mfma_f32x4& c, int j) {
  float v;
  asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(c[j]));
  return v;
}
template <int M, int N> __device__ __forceinline__ void mfma_fence(mfma_f32x4 (&acc)[M][N]) {
  asm volatile("s_nop 15\n\ts_nop 15");
#pragma unroll
  for (int m = 0; m < M; ++m)
#pragma unroll
    for (int n = 0; n < N; ++n) asm volatile("" : "+a"(acc[m][n]));   // ordered behind the wait states
}
template <int M, int N> __device__ __forceinline__ void mfma_fence_v(mfma_f32x4 (&acc)[M][N]) {     // ... in vector registers
  asm volatile("s_nop 15\n\ts_nop 15");
#pragma unroll
  for (int m = 0; m < M; ++m)
#pragma unroll
    for (int n = 0; n < N; ++n) asm volatile("" : "+v"(acc[m][n]));
}

// MI355X: 256 compute units in 8 XCDs; consecutive workgroup ids are dealt round-robin to
// the XCDs, each of which has its own L2.
constexpr int kNumXcd = 8;
constexpr int kNumCu = 256;

// Order of the ne x nc output tiles of one layer for the tile tables of the MFMA kernels: blocks of
// about 32 tiles (one round of an XCD's workgroups, which share that XCD's L2) whose shape streams
// the fewest distinct rows of a and delta -- as many tile columns as tile rows for square tiles,
// `aspect` times as many when a tile is `aspect` times as high as wide.  f(e, c) is called once per
// tile, e = tile row (d_out side), c = tile column (d_in side).
template <typename F>
inline void for_tiles_blocked(int ne, int nc, int aspect, F f) {
  const int per_round = kNumCu / kNumXcd;
  int nc_blk = 1;
  while (nc_blk * nc_blk < per_round * aspect) ++nc_blk;            // ~ sqrt(32 * aspect)
  nc_blk = nc_blk < nc ? nc_blk : nc;
  const int ne_blk = per_round / nc_blk > 1 ? per_round / nc_blk : 1;
  for (int eb = 0; eb < ne; eb += ne_blk)
    for (int cb = 0; cb < nc; cb += nc_blk)
      for (int e = eb; e < eb + ne_blk && e < ne; ++e)
        for (int c = cb; c < cb + nc_blk && c < nc; ++c) f(e, c);
}

// Device-side view of one linear layer (built on the host, uploaded once per change).
struct LayerDev {
  const void* a;
  const void* delta;
  float* grad_sum;
  long long a_stride;      // elements between token rows
  long long delta_stride;
  int d_in;
  int d_out;
  int fast;                // 1: rows 16-byte aligned and d % 8 == 0 for both operands
  int provided;            // 1: caller maintains grad_sum (no wgrad for this layer)
  int wg_blk_start;        // first workgroup of this layer in the wgrad launch
  int sq_blk_start;        // first workgroup of this layer in the squared-norm launch
  int kind;                // ADLOCO_KIND_* (0: linear weight)
  int delta_twin;          // vector blocks: first earlier vector block reading the same delta rows, or -1
  int a_twin;              // linear blocks: first earlier linear block reading the same activation rows
                           // (same a, stride, d_in) with the same d_out and delta stride, or -1
};

// One vector (bias / gain) or embedding-table block in the launches of its kernels.
struct AuxDesc {
  int layer;               // index into the layer table
  int slabs;               // column slabs of d_out (256 wide for vectors, 64 for tables)
  int blk_start;           // first workgroup in the (sample, slab) launch: B * slabs per block
  int blk_start2;          // first workgroup in the per-slab launch (vectors: column sums)
  long long vec_off;       // vectors: offset (floats) of this block's [B, d_out] sums
  long long vec_off_bias;  // vectors: >= 0: this gain block also forms the row sums of the bias block that
                           // reads the same delta, stored at this offset (that block has no workgroups of its own)
  long long perm_off;      // tables: offset (ints) of this block's [B, T] token order
  long long part_off;      // tables: offset (doubles) of this block's [B, slabs] slab totals
};

// One wave-wide direct load global -> LDS: lane l's 16 bytes at `src` land at LDS byte address
// `lds_addr` + 16*l (`lds_addr` is wave-uniform and travels in M0).  Written as inline assembly
// on purpose: the compiler orders the builtin form against every later LDS read with a full
// `s_waitcnt vmcnt(0)`, which would expose the whole memory latency in each pipeline step.  The
// caller therefore owns the ordering: its own s_waitcnt vmcnt(N) + workgroup barrier before any
// wave reads the bytes, and vmcnt(0) before compiler-visible memory traffic that must see them.
__device__ __forceinline__ void direct_load_lds16(const void* src, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :: "v"(src), "s"(lds_addr) : "m0");
}
// The same with the address split into a wave-uniform 64-bit base (scalar registers) and a 32-bit
// byte offset per lane: a kernel that walks along its rows bumps the base on the scalar unit and
// keeps the lane offsets constant, so that no vector instruction is spent on addresses.
// The base goes through a scalar copy: a load needs five wait states behind a vector instruction that wrote its scalar
// base (v_readfirstlane, or v_readlane where the compiler reloads a spilled register), and the compiler does not count
// them for inline assembly; the copy is interlocked by the hardware, and stands where M0 needs a wait state anyway.
__device__ __forceinline__ void direct_load_lds16_s(unsigned lane_off, const void* base, unsigned lds_addr) {
  unsigned long long b;
  asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0"
               : "=&s"(b) : "v"(lane_off), "s"(base), "s"(lds_addr) : "m0");
}
// Two such loads from one base with only the lanes of `mask` taking part: the 16 bytes of the others stay as they are in
// LDS.  All 64 lanes have to be active at the call.
__device__ __forceinline__ void direct_load_lds16_masked2(const void* base, unsigned off0, unsigned lds_addr0, unsigned off1,
                                                          unsigned lds_addr1, unsigned long long mask) {
  unsigned long long b;
  asm volatile("s_mov_b32 m0, %4\n\ts_mov_b64 %0, %3\n\ts_mov_b64 exec, %6\n\tglobal_load_lds_dwordx4 %1, %0\n\t"
               "s_mov_b32 m0, %5\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %0\n\ts_mov_b64 exec, -1"
               : "=&s"(b) : "v"(off0), "v"(off1), "s"(base), "s"(lds_addr0), "s"(lds_addr1), "s"(mask) : "m0");
}
// A wave-uniform pointer that the compiler may hold in vector registers, moved to scalar registers
// (the direct loads above take their base address there).
template <typename P> __device__ __forceinline__ const P* uniform_ptr(const P* p) {
  const unsigned long long v = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane(unsigned(v));
  const unsigned hi = __builtin_amdgcn_readfirstlane(unsigned(v >> 32));
  return reinterpret_cast<const P*>((unsigned long long)hi << 32 | lo);
}
// LDS byte address of a pointer into the workgroup's dynamic shared memory, as a scalar.
__device__ __forceinline__ unsigned lds_address(const void* p) {
  return __builtin_amdgcn_readfirstlane(
      (unsigned)(size_t)(const __attribute__((address_space(3))) unsigned char*)p);
}

// A wave's M x N accumulator blocks of 16 x 16 -> G [d_out, d_in]: this lane's element j of block (m, n) is entry
// (r + 16 * m + j, c + 16 * n).  The old entries of `MB` block rows are requested together (addresses past the edge are
// clamped): one by one, each load would be waited for on its own, about 1 us apiece at the end of every tile.  whole
// (the same for all lanes): no entry lies past the edge, and none is checked.
template <int M, int N, int MB, typename F>
__device__ __forceinline__ void put_grad_tile(float* G, int d_out, int d_in, int r, int c, bool accumulate, bool whole, F value) {
  static_assert(M % MB == 0, "whole batches");
#pragma unroll
  for (int m0 = 0; m0 < M; m0 += MB) {
    float old[MB][N][4];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int n = 0; n < N; ++n)
#pragma unroll
        for (int j = 0; j < 4; ++j) old[m][n][j] = 0.f;
    if (accumulate) {
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int rr = r + (m0 + m) * 16 + j, cc = c + n * 16;
            old[m][n][j] = G[(size_t)(rr < d_out ? rr : d_out - 1) * d_in + (cc < d_in ? cc : d_in - 1)];
          }
    }
    if (whole) {
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float* row = G + (size_t)(r + (m0 + m) * 16 + j) * d_in + c;
#pragma unroll
          for (int n = 0; n < N; ++n) {
            const float v = value(m0 + m, n, j);
            row[n * 16] = accumulate ? old[m][n][j] + v : v;
          }
        }
      continue;
    }
    // (widths are multiples of 8: the four rows of a lane's part of a block are in or out together)
#pragma unroll
    for (int n = 0; n < N; ++n)
      if (c + n * 16 < d_in)
#pragma unroll
        for (int m = 0; m < MB; ++m)
          if (r + (m0 + m) * 16 < d_out)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const float v = value(m0 + m, n, j);
              G[(size_t)(r + (m0 + m) * 16 + j) * d_in + c + n * 16] = accumulate ? old[m][n][j] + v : v;
            }
  }
}

// What the Gram contraction of a layer table contracts, for the choice between its kernels.
struct GramLoad {
  int count = 0;                 // groups of linear layers that are contracted together
  double chunks = 0, longest = 0;  // elements of all of them and of the longest, in chunks of 64
};

struct Scratch {
  void* ptr = nullptr;
  size_t bytes = 0;
};

// Tiles of the per-sample gradients of one layer table, for any batch size and sequence length: the same list serves
// every call on these shapes, in whatever order batches come, and a captured call replays with it.
struct TileList {
  Scratch tab;              // int4 [8][slots] entries (layer, first row, first column, piece | pieces << 16), layer < 0: none;
                            // int2 [8][slots]: (tile, first partial tile); int4 split tiles; int listed layers | tile ranges
  Scratch ptiles;           // partial tiles of the entries that can be split along the samples
  size_t off_part = 0, off_split = 0, off_csr = 0;
  int edge = 0;             // tile rows
  int slots = 0, n_tiles = 0, n_split = 0, n_listed = 0;
  int n[kNumXcd] = {}, left[kNumXcd] = {}, pieces[kNumXcd] = {};   // per XCD: tiles; of them in the incomplete last round
  std::vector<char> use;    // per block of the table: 1 = in the list
  bool built = false;
  // slots in use when a tile is split into at most `cap` pieces (first pieces come first on every XCD)
  int used(int cap) const {
    int u = 0;
    for (int x = 0; x < kNumXcd; ++x) {
      const int s = pieces[x] < cap ? pieces[x] : cap;
      u = u > n[x] + left[x] * (s - 1) ? u : n[x] + left[x] * (s - 1);
    }
    return u;
  }
  template <typename T> const T* at(size_t off) const {
    return reinterpret_cast<const T*>(static_cast<const char*>(tab.ptr) + off);
  }
  const int4* tiles() const { return at<int4>(0); }
  const int2* part() const { return at<int2>(off_part); }
  const int4* split() const { return at<int4>(off_split); }
  const int* layers() const { return at<int>(off_csr); }
  const int* ranges() const { return at<int>(off_csr) + n_listed; }   // tiles [q], .. of the q-th listed layer
};
// Samples that an entry covers: its piece of the batch (no more pieces than samples), or run `run` of `group` samples.
struct SampleRun { int first, count; };
__device__ __forceinline__ SampleRun list_piece(int w, int B, bool whole) {
  const int S = whole ? 1 : min(w >> 16, B), p = w & 0xffff;
  if (p >= S) return SampleRun{0, 0};
  const int s0 = B * p / S;
  return SampleRun{s0, B * (p + 1) / S - s0};
}
__device__ __forceinline__ SampleRun list_run(int w, int B, int group, int run) {
  return (w & 0xffff) ? SampleRun{0, 0} : SampleRun{run * group, min(group, B - run * group)};
}

}  // namespace adloco

struct adloco_ctx {
  int device = 0;
  std::string err;
  // scratch
  adloco::Scratch partials;    // float  [n_units * pairs] Gram partial sums
  adloco::Scratch layer_tab;   // LayerDev[n_layers]
  adloco::Scratch red_f64;     // double partial sums of the streaming reductions
  adloco::Scratch sample_f64;  // double [B] per-sample totals
  adloco::Scratch order_tab;   // int [n_layers] launch order (heaviest first)
  adloco::Scratch group_tab;   // GramGroup[n_groups], int[n_groups] launch order of the groups; then, at
                               // single_off, the same with every linear layer in a group of its own
  int n_groups = 0;
  size_t single_off = 0;
  adloco::GramLoad gram_load[2];   // with every linear layer by itself; in groups
  std::vector<adloco::LayerDev> layer_tab_host;  // last uploaded copy
  std::vector<int> order_host;
  adloco::Scratch job_tab;     // GramJob[] of the dual-tile Gram kernel
  int job_tab_nt = -1;         // number of row blocks the uploaded job table was built for
  int job_tab_n = 0;
  int gram_job_order = -1;     // where the jobs of two diagonal tile pairs go among a unit's jobs: 0 first,
                               // 1 last, 2 spread; -1: first for long sequences (T >= 768), last for short
                               // ones (measured: +9 % at T = 1024, -1.5 % at T = 512 for `first`)
  bool all_fast64 = false;     // every layer: aligned rows and widths that are multiples of 64
  int min_width = 0;           // smallest width of a linear block
  adloco::Scratch wgx_tab;     // tile table of the fast gradient-sum kernel
  int wgx_slots = 0;           // tiles per XCD in that table (0: not built for this layer table)
  adloco::Scratch wgx_split;   // split tiles (layer, e0, c0, pieces) for the reduction
  adloco::Scratch wgx_part;    // partial tiles of the split contraction, 256 KiB each
  int wgx_n_split = 0;
  bool all_fast = false;       // every layer without a provided gradient: aligned, widths % 8 == 0
  int n_linear = 0;            // linear-weight blocks in the table (= entries of order_tab)
  // vector (bias / gain) and embedding-table blocks
  std::vector<adloco::AuxDesc> vec_host, emb_host;
  adloco::Scratch vec_tab, emb_tab;   // device copies of the two descriptor lists
  adloco::Scratch aux_vec;     // float  per vector block [B, d_out]
  adloco::Scratch aux_perm;    // int    per table block  [B, T]
  adloco::Scratch aux_part;    // double per table block  [B, slabs]
  int aux_B = -1, aux_T = -1;  // batch shape the descriptor lists were built for
  int vec_blocks = 0, vec_blocks2 = 0, emb_blocks = 0;
  // inner products (Section 3.3.2)
  adloco::Scratch ip_tab;      // int4 tile table of the inner-product form of the tile GEMM
  adloco::Scratch ip_tile_out; // float [tiles][ip_group][waves][2]
  bool ip_short = false;       // the tile kernel for short sequences
  adloco::Scratch ip_dot, ip_sq;   // float [n_layers][B] of the blocks outside the tile table
  adloco::Scratch ip_flags;    // unsigned char [n_layers]: 1 = block is in the tile table
  int ip_slots = 0, ip_group = 1, ip_B = -1, ip_T = -1;
  adloco::TileList ip_rest[2]; // linear blocks outside that table: 64- and 128-wide tiles
  int ip_rest_W = 1;           // which of them the batch takes
  bool ip_any_rest = false;
  int ip_rest_group = 1;
  int ip_group_tuning = 0;     // 0: cost model; else samples per tile entry
  // statistics by per-sample gradient tiles: of the blocks whose gradient sum is formed here, or of all if none is.
  // Built with the layer table; a list for which there is no memory is missing, and its routes with it.
  adloco::TileList tiles16;    // aligned 16-bit blocks
  adloco::TileList tiles32[2]; // fp32 blocks: 64- and 128-wide tiles
  adloco::Scratch tile_out;    // results per (tile, sample)
  bool lin_fast = false;       // every linear block: 16-byte aligned rows, widths % 8 == 0, strides below 2^25
  int n_formed = 0;            // linear blocks whose gradient sum is formed here
  int stats_variant = 1;       // 1: tile form when eligible; 0: Gram + gradient-sum kernels
  // the vector / table kernels (HBM-bound) can run next to the kernels of the linear blocks (MFMA /
  // L2-bound) on a second stream, forked from and joined to the caller's stream by events; measured,
  // that buys nothing (both go through the same L2), so it is off unless "overlap_aux" asks for it
  hipStream_t side_stream = nullptr;
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;
  int overlap_aux = 0;
  int wgrad_blocks = 0;        // workgroups of the wgrad launch for the uploaded table
  int table_dtype = -1;        // dtype the uploaded table was built for
  int table_inputs = -1;       // 1: the table was built by a call that reads a and delta
  int plain_tiles_tuning = 0;  // plain tiles: 0: time model; 1, 2: 64- or 128-wide; + 4 (fp32 statistics): none split
  size_t scratch_limit = 0;    // largest scratch allocation, bytes (0: no limit); for tests of the calls' behaviour without memory
  int table_builds = 0;        // how often a shape-dependent table has been (re)built
  long long max_lin_stride = 0;  // widest row stride (elements) among the linear blocks of the table
  double* pinned = nullptr;    // 8 doubles of pinned host memory (read-back of the tests' sums)
  // optional per-kernel event timing ("profile" knob)
  struct ProfRec { int kernel; hipEvent_t start, stop; };
  std::vector<ProfRec> prof;
  std::vector<hipEvent_t> prof_free;
  int profile = 0;
  // tuning
  int gram_variant = 1;        // 1: region or dual-tile kernel when eligible; 2, 3: the latter, the former; 0: always the generic one
  int gram_kernel = 0;         // of the last statistics call: 0 none, 1 general, 2 dual-tile, 3 region
  int wgrad_variant = 2;       // 2: 256x256 fast kernel when eligible; 1/0: 128x128 kernel (LDS transpose reads / gathers)
  int stream_blocks_per_cu = 0;   // resident workgroups per CU of the streaming kernels; 0: automatic
  int stream_variant = 0;
};

namespace adloco {

inline int fail(adloco_ctx* ctx, int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (ctx) ctx->err = buf;
  return code;
}

#define ADLOCO_HIP_CHECK(ctx, expr)                                                      \
  do {                                                                                   \
    hipError_t e_ = (expr);                                                              \
    if (e_ != hipSuccess)                                                                \
      return adloco::fail((ctx), ADLOCO_EHIP, "%s failed: %s (%s:%d)", #expr,            \
                          hipGetErrorString(e_), __FILE__, __LINE__);                    \
  } while (0)

// Event timing of one kernel launch when ctx->profile is set (no-ops otherwise).
enum ProfKernel { kProfGram = 0, kProfWgrad, kProfFinalize, kProfSqnorm, kProfOuter, kProfMerge,
                  kProfVecTab, kProfInner, kProfIp, kProfTileStats, kProfCount };
hipEvent_t prof_begin(adloco_ctx* ctx, hipStream_t st);
void prof_end(adloco_ctx* ctx, int kernel, hipEvent_t start, hipStream_t st);

// Grow-only scratch buffer.  Growing frees the old block, which waits for the device.
int ensure_scratch(adloco_ctx* ctx, Scratch& s, size_t bytes);
// The same for a route that a call can do without: false if the memory cannot be had, or not without an allocation while
// the stream is being captured.
bool obtain_scratch(adloco_ctx* ctx, Scratch& s, size_t bytes, hipStream_t st);

// Kernel launchers (defined next to their kernels).  All return a hipError_t from the launch.
struct GramLaunch {
  const LayerDev* layers;   // device table
  const int* order;         // device: launch order of layer indices, heaviest first
  int n_layers, B, T;
  float* partials;          // [n_layers][B][n_pairs]
  int n_pairs;              // tile pairs per (layer, sample)
  int tile;                 // T-tile edge used by the kernel
  int dtype = ADLOCO_BF16;  // element type of a and delta
};
// Linear layers that read the same activation tensor (q / k / v, gate / up of a transformer block):
// their A A^T is one and the same, so the dual-tile Gram kernel forms it once per group and runs the
// members' delta delta^T contractions against it one after the other.
constexpr int kGramGroupMax = 4;
struct GramGroup {
  int n;                      // members, 1 .. kGramGroupMax
  int layer[kGramGroupMax];   // indices into the layer table; all share a, d_in, d_out and the strides
};
// One workgroup of the dual-tile Gram kernel: up to two 128x128 tile pairs (A-block, B-block)
// drawn from at most three distinct 128-row blocks.
struct GramJob {
  int blk[3];      // distinct row blocks to stage (unused entries repeat blk[0])
  int nblk;        // 2 or 3 (1 when T fits one block)
  int sa[2], sb[2];  // per tile pair: which staged block supplies the rows / the columns
  float w[2];      // 1 on the diagonal, 2 off it (symmetry), 0 for an absent second pair
};
std::vector<GramJob> make_gram_jobs(int nt, int order);
int gram_tile_edge(int dtype, int variant);
// g.order: launch order of GROUP indices; g.n_layers: number of groups; g.n_pairs: partial sums per
// (layer, sample) = gram_dual_parts(n_jobs)
hipError_t launch_gram_bf16_dual(const GramLaunch& g, const GramGroup* groups, const GramJob* jobs,
                                 int n_jobs, int variant, hipStream_t st);
int gram_dual_parts(int n_jobs);
// The same on 256 x 256 regions of the Gram matrices, for sequences that fill them: widths of at least 128 and
// (T + 256) * row stride below 2^31 elements; g.n_pairs = 4 * gram_region_jobs(T) partial sums per (layer, sample).
int gram_region_jobs(int T);
hipError_t launch_gram_region(const GramLaunch& g, const GramGroup* groups, hipStream_t st);
hipError_t launch_gram_bf16(const GramLaunch& g, int variant, hipStream_t st);
hipError_t launch_gram_f32(const GramLaunch& g, hipStream_t st);
int wgrad_tile_edge(int dtype);
int make_wgrad_x_tiles(const std::vector<LayerDev>& layers, std::vector<int4>& out,
                       std::vector<int4>& split_tiles, int& n_pieces);
hipError_t launch_wgrad_x(const LayerDev* layers, const void* tiles, int slots,
                          const void* split_tiles, int n_split, float* partials, long long rows,
                          int accumulate, int dtype, hipStream_t st);
hipError_t launch_wgrad(const LayerDev* layers, int n_layers, int n_blocks, long long rows,
                        int dtype, int accumulate, int variant, hipStream_t st);
hipError_t launch_finalize_stats(const float* partials, int n_layers, int B, int n_pairs,
                                 float* per_sample, float* per_layer_sample, double* sample_f64,
                                 adloco_stats_acc* acc, int accumulate, hipStream_t st);
int vector_table_slab();
int embed_table_slab();
hipError_t launch_vector_stats(const LayerDev* layers, const AuxDesc* tab, int n_tab,
                               int blocks_rowsum, int blocks_colsum, int B, int T, int dtype,
                               float* vec, float* partials, int n_pairs, int accumulate,
                               bool write_grad_sum, hipStream_t st);
// Tiles of a tile kernel: e rows (d_out side) x c columns, chunks of k token rows, `room` workgroups resident per XCD.
struct TileGeom { int e, c, k, room; };
int make_ip_tiles(const std::vector<LayerDev>& layers, const std::vector<char>& use, int B, int T, TileGeom geom,
                  int forced_group, std::vector<int4>& out, int& group);
TileGeom ip_tile_geom();
hipError_t launch_ip_tiles(const LayerDev* layers, const void* tiles, int slots, int T, int group,
                           int dtype, bool want_sq, bool short_form, float* ip_out, hipStream_t st);
// Which of the two 16-bit tile kernels: the one for short sequences (short_form), and the wave sums per tile and sample.
bool short_sequences(const std::vector<LayerDev>& layers, const std::vector<char>& use, int B, int T, bool inner_products);
int tile_waves(bool short_form);
// Tile list of the blocks of `use`; split: the tiles of an XCD's incomplete last round can be cut along the samples.
void make_tile_list(const std::vector<LayerDev>& layers, const std::vector<char>& use, TileGeom geom, bool split, TileList& list,
                    std::vector<int4>& tiles, std::vector<int2>& part, std::vector<int4>& split_tiles, std::vector<int>& csr,
                    int& n_pieces);
// Samples per run that take the least time for `tiles` tiles.
int run_length(long long tiles, int B, int T, TileGeom geom);
// ||g_i||^2 of aligned 16-bit blocks, and (launch_stats_tiles) their gradient sums -> one partial sum per (layer, sample).
// out: tile_waves() floats per (tile, sample).
hipError_t launch_square_tiles(const LayerDev* layers, const TileList& list, int B, int T, int dtype, float* out,
                               float* partials, hipStream_t st);
hipError_t launch_stats_tiles(const LayerDev* layers, const TileList& list, int B, int T, int dtype, int accumulate,
                              bool short_form, float* out, float* partials, hipStream_t st);
// Resident workgroups per XCD of the plain tile kernel: two (128-wide tiles) or four per compute unit.
constexpr int plain_tile_room(int W) { return kNumCu / kNumXcd * (W == 2 ? 2 : 4); }
inline TileGeom plain_tile_geom(int W) { return TileGeom{64 * W, 64 * W, 32, plain_tile_room(W)}; }
int plain_tile_width(const std::vector<LayerDev>& layers, const std::vector<char>& use, int B, int T);
int sum_tile_width(const std::vector<LayerDev>& layers, const std::vector<char>& use);
struct PlainChoice { int W; bool whole; };       // tile width 64 * W; whole: no tile is split
PlainChoice plain_tile_choice(const TileList* lists, int B, int T);
// mode 0: <g_i, G> -> dot and ||g_i||^2 -> sq; fp32 only: mode 1: G and ||g_i||^2 -> sq (whole: no tile is split); mode 2: G
// (B = 1, T = all token rows, sq = NULL); mode 3: ||g_i||^2 -> sq.  group: samples per run (modes 0 and 3).  out: one
// double per (tile, sample), two in mode 0.
hipError_t launch_plain_tiles(const LayerDev* layers, const TileList& list, int mode, int B, int T, int dtype, int accumulate,
                              bool whole, int group, double* out, float* dot, float* sq, int sq_stride, hipStream_t st);
hipError_t launch_ip_vector_table(const LayerDev* layers, const AuxDesc* vec_tab, int n_vec,
                                  const AuxDesc* emb_tab, int n_emb, int B, int T, int dtype,
                                  const float* vec, float* dot, hipStream_t st);
hipError_t launch_ip_finalize(const void* tiles, const float* tile_out, long long n_tiles, int group, int waves,
                              const float* dot, const float* sq, const unsigned char* in_tiles,
                              int n_layers, int B, float* per_sample_ip, float* per_sample_sq,
                              double* sample_f64, adloco_ip_acc* acc, int accumulate, hipStream_t st);
hipError_t launch_embed_stats(const LayerDev* layers, const AuxDesc* tab, int n_tab, int blocks_rows,
                              int B, int T, int dtype, int* perm, double* part, float* partials,
                              int n_pairs, hipStream_t st);
// sum_l ||grad_sum_l||^2 of the n_layers blocks of a device table, whose sq_blk_start fields add up to nblk workgroups
// (sqnorm_partials()); partial holds nblk doubles.  The sum, *acc and *ip (each unless NULL) go to host[0], host[2..3]
// and host[4..7] of pinned host memory, valid once the stream has been waited for.
int sqnorm_chunk();
size_t sqnorm_partials(const std::vector<LayerDev>& host_layers);
hipError_t launch_sqnorm(const LayerDev* layers, int n_layers, size_t nblk, double* partial,
                         const adloco_stats_acc* acc, const adloco_ip_acc* ip, double* host, hipStream_t st);
// Whether a kernel on `device` may read `p`: memory of that device (another one's need not be mapped here), 8-byte
// aligned.  The read-back copies from any other address.
inline bool is_memory_of(const hipPointerAttribute_t& a, int device) {
  return a.type == hipMemoryTypeDevice && a.device == device;
}
bool kernel_can_read(const adloco_ctx* ctx, const void* p);
// adloco_grad_stats.  pinned_order (adloco_round): gradient sums of fp32 blocks and of token rows that are no multiple
// of 32 are added up in the order of the kernels for whole contractions, not sample by sample or piece by piece.  A
// round returns parameters after several AdamW steps, which divide by sqrt(v): where gradient and second moment are
// both near zero, the last bit of a gradient sum becomes up to 4e-4 of the outer momentum's norm.
int grad_stats(adloco_ctx* ctx, const adloco_linear_desc* layers, int n_layers, int B, int T, int dtype,
               float* per_sample_sqnorm, float* per_layer_sample_sqnorm, adloco_stats_acc* acc, uint32_t flags,
               bool pinned_order, void* stream);
// Looks up, for the context's device, the address of the file-scope device array that serves
// adloco_norm_test_noalloc (called once per context by adloco_create, with the device current).
int no_alloc_init(adloco_ctx* ctx);

}  // namespace adloco
