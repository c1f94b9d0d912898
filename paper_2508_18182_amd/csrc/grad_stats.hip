// Entry points of the statistics half: adloco_grad_stats (per-sample norms by the Gram
// identity, gradient sum, S1 accumulation) and adloco_norm_test (S2 on the device, then the
// decision on the host).
#include <algorithm>
#include <numeric>

#include "common.h"

using namespace adloco;

namespace {

constexpr int kMaxLayers = 4096;

// The device copy of the layer table keeps its shapes, strides and launch positions from call to
// call; only the three pointers of every block change when the caller hands in other tensors (fresh
// activations of the next micro-batch, another worker's gradient buffers).  They travel in the
// argument of a small kernel, so that a call on a known list of shapes uploads nothing, waits for
// nothing, and can be captured into a graph with its pointers in it.
constexpr int kPtrChunk = 120;
struct PtrChunk {
  int first, count, which;            // which: 1 = a and delta, 2 = grad_sum, 3 = all
  int pad;
  const void* a[kPtrChunk];
  const void* delta[kPtrChunk];
  float* grad_sum[kPtrChunk];
};
__global__ void set_layer_pointers_kernel(LayerDev* tab, PtrChunk c) {
  const int i = threadIdx.x;
  if (i >= c.count) return;
  LayerDev& L = tab[c.first + i];
  if (c.which & 1) {
    L.a = c.a[i];
    L.delta = c.delta[i];
  }
  if (c.which & 2) L.grad_sum = c.grad_sum[i];
}

int upload_pointers(adloco_ctx* ctx, const std::vector<LayerDev>& tab, int which, hipStream_t st) {
  PtrChunk c;
  for (size_t first = 0; first < tab.size(); first += kPtrChunk) {
    c.first = int(first);
    c.count = int(std::min<size_t>(kPtrChunk, tab.size() - first));
    c.which = which;
    c.pad = 0;
    for (int i = 0; i < c.count; ++i) {
      c.a[i] = tab[first + i].a;
      c.delta[i] = tab[first + i].delta;
      c.grad_sum[i] = tab[first + i].grad_sum;
    }
    hipLaunchKernelGGL(set_layer_pointers_kernel, dim3(1), dim3(128), 0, st,
                       static_cast<LayerDev*>(ctx->layer_tab.ptr), c);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
      return fail(ctx, ADLOCO_EHIP, "pointer table launch failed: %s", hipGetErrorString(e));
  }
  return ADLOCO_OK;
}

// Everything of a block that the tables, tile lists and kernel choices depend on: all of LayerDev
// but the addresses themselves (their alignment class is in `fast`, whether they are there at all
// is compared).
bool same_shape(const LayerDev& x, const LayerDev& y) {
  return x.a_stride == y.a_stride && x.delta_stride == y.delta_stride && x.d_in == y.d_in &&
         x.d_out == y.d_out && x.fast == y.fast && x.provided == y.provided && x.kind == y.kind &&
         x.wg_blk_start == y.wg_blk_start && x.sq_blk_start == y.sq_blk_start && x.delta_twin == y.delta_twin && x.a_twin == y.a_twin &&
         (x.a == nullptr) == (y.a == nullptr) && (x.delta == nullptr) == (y.delta == nullptr) &&
         (x.grad_sum == nullptr) == (y.grad_sum == nullptr);
}

// Uploads a tile list.  One for which there is no memory stays missing: its routes are not taken.
void build_tile_list(adloco_ctx* ctx, TileList& p, const std::vector<LayerDev>& tab, const std::vector<char>& use, TileGeom geom,
                     bool split, hipStream_t st) {
  ++ctx->table_builds;
  p.built = false;
  std::vector<int4> tiles, split_tiles;
  std::vector<int2> part;
  std::vector<int> csr;
  int n_pieces = 0;
  make_tile_list(tab, use, geom, split, p, tiles, part, split_tiles, csr, n_pieces);
  p.use = use;
  if ((long long)p.slots * kNumXcd > 0x7fffffffLL) return;
  std::vector<char> blob;
  auto append = [&](const void* src, size_t n) {
    const size_t at = blob.size();
    blob.insert(blob.end(), static_cast<const char*>(src), static_cast<const char*>(src) + n);
    return at;
  };
  append(tiles.data(), tiles.size() * sizeof(int4));
  p.off_split = append(split_tiles.data(), split_tiles.size() * sizeof(int4));
  p.off_part = append(part.data(), part.size() * sizeof(int2));
  p.off_csr = append(csr.data(), csr.size() * sizeof(int));
  if (!obtain_scratch(ctx, p.tab, blob.size(), st)) return;
  if (!obtain_scratch(ctx, p.ptiles, size_t(n_pieces) * geom.e * geom.c * sizeof(float), st)) return;
  p.built = hipMemcpyAsync(p.tab.ptr, blob.data(), blob.size(), hipMemcpyHostToDevice, st) == hipSuccess &&
            hipStreamSynchronize(st) == hipSuccess;
}

// Build the device view of the layer list.  A list whose shapes (widths, strides, kinds, flags,
// alignment classes) equal those of the previous call only has its pointers refreshed, by a kernel on
// the caller's stream; any other list rebuilds every table that depends on it, which allocates,
// copies from pageable memory and waits for the stream.
int prepare_tables(adloco_ctx* ctx, const adloco_linear_desc* layers, int n_layers, int dtype,
                   bool need_inputs, hipStream_t st) {
  const size_t esize = is_16bit(dtype) ? 2 : 4;
  std::vector<LayerDev> tab(n_layers);
  const int wt = wgrad_tile_edge(dtype);
  const int chunk = sqnorm_chunk();
  long long wg = 0, sq = 0;
  for (int l = 0; l < n_layers; ++l) {
    const adloco_linear_desc& d = layers[l];
    if (d.d_in < 1 || d.d_out < 1)
      return fail(ctx, ADLOCO_EINVAL, "layer %d: d_in = %d, d_out = %d must be >= 1", l, d.d_in, d.d_out);
    if (d.reserved != 0 || (d.flags & ~(ADLOCO_GRAD_PROVIDED | ADLOCO_KIND_MASK)))
      return fail(ctx, ADLOCO_EINVAL, "layer %d: unknown flags or non-zero reserved field", l);
    const bool provided = d.flags & ADLOCO_GRAD_PROVIDED;
    const int kind = int(d.flags & ADLOCO_KIND_MASK);
    if (kind != ADLOCO_KIND_LINEAR && kind != ADLOCO_KIND_VECTOR && kind != ADLOCO_KIND_EMBED)
      return fail(ctx, ADLOCO_EINVAL, "layer %d: unknown kind 0x%x", l, kind);
    if (kind == ADLOCO_KIND_VECTOR && d.d_in != 1)
      return fail(ctx, ADLOCO_EINVAL, "layer %d: a vector block needs d_in = 1", l);
    if (kind == ADLOCO_KIND_EMBED && !provided)
      return fail(ctx, ADLOCO_EINVAL, "layer %d: an embedding block needs ADLOCO_GRAD_PROVIDED", l);
    LayerDev L{};
    L.a = d.a;
    L.delta = d.delta;
    L.grad_sum = d.grad_sum;
    L.a_stride = d.a_row_stride ? d.a_row_stride : (kind == ADLOCO_KIND_VECTOR ? d.d_out : d.d_in);
    L.delta_stride = d.delta_row_stride ? d.delta_row_stride : d.d_out;
    L.d_in = d.d_in;
    L.d_out = d.d_out;
    L.provided = provided ? 1 : 0;
    L.kind = kind;
    if (need_inputs) {
      if (!d.delta || (!d.a && kind != ADLOCO_KIND_VECTOR))
        return fail(ctx, ADLOCO_EINVAL, "layer %d: a or delta is NULL", l);
      const long long a_width = kind == ADLOCO_KIND_LINEAR ? d.d_in : d.d_out;
      if ((kind != ADLOCO_KIND_EMBED && d.a && L.a_stride < a_width) || L.delta_stride < d.d_out)
        return fail(ctx, ADLOCO_EINVAL, "layer %d: row stride smaller than the row", l);
      const size_t a_esize = kind == ADLOCO_KIND_EMBED ? 4 : esize;
      if ((reinterpret_cast<uintptr_t>(d.a) % a_esize) || (reinterpret_cast<uintptr_t>(d.delta) % esize))
        return fail(ctx, ADLOCO_EINVAL, "layer %d: a or delta not aligned to its element size", l);
      if (!provided && !d.grad_sum)
        return fail(ctx, ADLOCO_EINVAL, "layer %d: grad_sum is NULL without ADLOCO_GRAD_PROVIDED", l);
      const bool d_fast = (reinterpret_cast<uintptr_t>(d.delta) % 16 == 0) && (d.d_out % 8 == 0) &&
                          (L.delta_stride % 8 == 0);
      if (kind == ADLOCO_KIND_LINEAR)
        L.fast = d_fast && (reinterpret_cast<uintptr_t>(d.a) % 16 == 0) && (d.d_in % 8 == 0) &&
                 (L.a_stride % 8 == 0);
      else if (kind == ADLOCO_KIND_VECTOR)
        L.fast = d_fast && (!d.a || ((reinterpret_cast<uintptr_t>(d.a) % 16 == 0) &&
                                     (L.a_stride % 8 == 0)));
      else
        L.fast = 0;
    } else if (!d.grad_sum) {
      return fail(ctx, ADLOCO_EINVAL, "layer %d: grad_sum is NULL", l);
    }
    if (d.grad_sum && (reinterpret_cast<uintptr_t>(d.grad_sum) % 4))
      return fail(ctx, ADLOCO_EINVAL, "layer %d: grad_sum not 4-byte aligned", l);
    L.a_twin = -1;
    if (need_inputs && kind == ADLOCO_KIND_LINEAR && d.a)
      for (int j = 0; j < l; ++j)
        if (tab[j].kind == ADLOCO_KIND_LINEAR && tab[j].a == L.a && tab[j].a_stride == L.a_stride &&
            tab[j].d_in == L.d_in && tab[j].d_out == L.d_out && tab[j].delta_stride == L.delta_stride) {
          L.a_twin = j;
          break;
        }
    L.delta_twin = -1;
    if (need_inputs && kind == ADLOCO_KIND_VECTOR)
      for (int j = 0; j < l; ++j)
        if (tab[j].kind == ADLOCO_KIND_VECTOR && tab[j].delta == L.delta && tab[j].d_out == L.d_out &&
            tab[j].delta_stride == L.delta_stride) {
          L.delta_twin = j;
          break;
        }
    L.wg_blk_start = int(wg);
    L.sq_blk_start = int(sq);
    if (!provided && kind == ADLOCO_KIND_LINEAR)
      wg += (long long)((d.d_out + wt - 1) / wt) * ((d.d_in + wt - 1) / wt);
    sq += ((long long)d.d_in * d.d_out + chunk - 1) / chunk;
    if (wg > 0x7fffffffLL || sq > 0x7fffffffLL)
      return fail(ctx, ADLOCO_EUNSUPPORTED, "layer list too large for one launch");
    tab[l] = L;
  }
  bool same = ctx->table_dtype == dtype && ctx->table_inputs == int(need_inputs) &&
              tab.size() == ctx->layer_tab_host.size();
  for (size_t l = 0; same && l < tab.size(); ++l) same = same_shape(tab[l], ctx->layer_tab_host[l]);
  if (same) {
    int rc = upload_pointers(ctx, tab, 3, st);
    if (rc) return rc;
    ctx->layer_tab_host = std::move(tab);
    return ADLOCO_OK;
  }
  ++ctx->table_builds;
  // linear layers, heaviest first, so that the tail of the Gram launch is made of cheap workgroups
  std::vector<int> order;
  for (int l = 0; l < n_layers; ++l)
    if (tab[l].kind == ADLOCO_KIND_LINEAR) order.push_back(l);
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) {
    return (long long)tab[x].d_in + tab[x].d_out > (long long)tab[y].d_in + tab[y].d_out;
  });
  int rc = ensure_scratch(ctx, ctx->layer_tab, tab.size() * sizeof(LayerDev));
  if (rc) return rc;
  rc = ensure_scratch(ctx, ctx->order_tab, std::max<size_t>(order.size(), 1) * sizeof(int));
  if (rc) return rc;
  ctx->layer_tab_host.clear();          // invalid until both copies are enqueued
  ctx->table_dtype = -1;
  ADLOCO_HIP_CHECK(ctx, hipMemcpyAsync(ctx->layer_tab.ptr, tab.data(), tab.size() * sizeof(LayerDev),
                                       hipMemcpyHostToDevice, st));
  if (!order.empty())
    ADLOCO_HIP_CHECK(ctx, hipMemcpyAsync(ctx->order_tab.ptr, order.data(), order.size() * sizeof(int),
                                         hipMemcpyHostToDevice, st));
  // pageable sources: make sure the runtime has consumed them before they go out of scope
  ADLOCO_HIP_CHECK(ctx, hipStreamSynchronize(st));
  bool f64 = need_inputs;
  for (const LayerDev& L : tab)
    if (L.kind == ADLOCO_KIND_LINEAR) f64 = f64 && L.fast && L.d_in % 64 == 0 && L.d_out % 64 == 0;
  ctx->all_fast64 = f64;
  ctx->min_width = 0x7fffffff;
  for (const LayerDev& L : tab)
    if (L.kind == ADLOCO_KIND_LINEAR) ctx->min_width = std::min(ctx->min_width, std::min(L.d_in, L.d_out));
  long long widest = 0;
  for (const LayerDev& L : tab)
    if (L.kind == ADLOCO_KIND_LINEAR) widest = std::max(widest, std::max(L.a_stride, L.delta_stride));
  ctx->max_lin_stride = widest;
  bool fast = need_inputs;
  for (const LayerDev& L : tab)
    if (L.kind == ADLOCO_KIND_LINEAR) fast = fast && (L.provided || L.fast);
  ctx->all_fast = fast;
  ctx->n_linear = int(order.size());
  {
    // groups of linear layers that read the same activation tensor, for the dual-tile Gram kernel
    std::vector<GramGroup> groups;
    std::vector<int> group_of(tab.size(), -1);
    for (int l = 0; l < n_layers; ++l) {
      if (tab[l].kind != ADLOCO_KIND_LINEAR) continue;
      const int t = tab[l].a_twin;
      if (t >= 0 && group_of[t] >= 0 && groups[group_of[t]].n < kGramGroupMax && tab[t].fast == tab[l].fast) {
        GramGroup& G = groups[group_of[t]];
        G.layer[G.n++] = l;
        group_of[l] = group_of[t];
      } else {
        GramGroup G{};
        G.n = 1;
        G.layer[0] = l;
        group_of[l] = int(groups.size());
        groups.push_back(G);
      }
    }
    // a second table with every layer in a group of its own, for sequences with a ragged last tile
    std::vector<GramGroup> single;
    for (int l : order) {
      GramGroup G{};
      G.n = 1;
      G.layer[0] = l;
      single.push_back(G);
    }
    std::vector<int> gorder(groups.size()), sorder(single.size());
    std::iota(gorder.begin(), gorder.end(), 0);
    std::iota(sorder.begin(), sorder.end(), 0);       // `order` is sorted already
    auto weight = [&](int gi) {
      const GramGroup& G = groups[gi];
      return (long long)tab[G.layer[0]].d_in + (long long)G.n * tab[G.layer[0]].d_out;
    };
    std::stable_sort(gorder.begin(), gorder.end(), [&](int x, int y) { return weight(x) > weight(y); });
    // layout: groups | their order | singleton groups | their order
    std::vector<char> blob;
    auto append = [&](const void* p, size_t n) {
      const char* c = static_cast<const char*>(p);
      blob.insert(blob.end(), c, c + n);
    };
    append(groups.data(), groups.size() * sizeof(GramGroup));
    append(gorder.data(), gorder.size() * sizeof(int));
    ctx->single_off = blob.size();
    append(single.data(), single.size() * sizeof(GramGroup));
    append(sorder.data(), sorder.size() * sizeof(int));
    rc = ensure_scratch(ctx, ctx->group_tab, std::max<size_t>(blob.size(), 16));
    if (rc) return rc;
    if (!blob.empty()) {
      ADLOCO_HIP_CHECK(ctx, hipMemcpyAsync(ctx->group_tab.ptr, blob.data(), blob.size(), hipMemcpyHostToDevice, st));
      ADLOCO_HIP_CHECK(ctx, hipStreamSynchronize(st));
    }
    ctx->n_groups = int(groups.size());
    for (int g = 0; g < 2; ++g) {
      GramLoad& load = ctx->gram_load[g];
      load = GramLoad{};
      for (const GramGroup& G : g ? groups : single) {
        const LayerDev& L = tab[G.layer[0]];
        const double chunks = (L.d_in + double(G.n) * L.d_out) / 64;
        ++load.count;
        load.chunks += chunks;
        load.longest = std::max(load.longest, chunks);
      }
    }
  }
  ctx->aux_B = ctx->aux_T = -1;         // the vector / table descriptor lists follow the table
  ctx->ip_B = ctx->ip_T = -1;           // and so does the inner-product tile table
  ctx->lin_fast = need_inputs && widest < (1 << 25);
  for (const LayerDev& L : tab)
    if (L.kind == ADLOCO_KIND_LINEAR) ctx->lin_fast = ctx->lin_fast && L.fast;
  ctx->n_formed = 0;
  for (const LayerDev& L : tab) ctx->n_formed += L.kind == ADLOCO_KIND_LINEAR && !L.provided;
  {
    // tile lists of every route that a call on this table can take, whatever its batch: of the blocks whose gradient sum is
    // formed here, or of all linear blocks if none is (the 16-bit kernels take either all blocks or none)
    for (TileList* p : {&ctx->tiles16, &ctx->tiles32[0], &ctx->tiles32[1], &ctx->ip_rest[0], &ctx->ip_rest[1]}) p->built = false;
    std::vector<char> use(n_layers, 0);
    for (int l = 0; l < n_layers; ++l) use[l] = tab[l].kind == ADLOCO_KIND_LINEAR && !(ctx->n_formed && tab[l].provided);
    const bool all = ctx->n_formed == 0 || ctx->n_formed == ctx->n_linear;
    if (need_inputs && ctx->n_linear > 0 && is_16bit(dtype) && ctx->lin_fast && all)
      build_tile_list(ctx, ctx->tiles16, tab, use, ip_tile_geom(), ctx->n_formed > 0, st);
    if (need_inputs && ctx->n_linear > 0 && dtype == ADLOCO_F32)
      for (int W = 1; W <= 2; ++W) build_tile_list(ctx, ctx->tiles32[W - 1], tab, use, plain_tile_geom(W), ctx->n_formed > 0, st);
  }
  ctx->wgx_slots = 0;
  if (fast && is_16bit(dtype) && wg > 0 && widest < (1 << 25)) {
    std::vector<int4> tiles, split;
    int n_pieces = 0;
    const int slots = make_wgrad_x_tiles(tab, tiles, split, n_pieces);
    rc = ensure_scratch(ctx, ctx->wgx_tab, tiles.size() * sizeof(int4));
    if (rc) return rc;
    rc = ensure_scratch(ctx, ctx->wgx_split, std::max<size_t>(split.size(), 1) * sizeof(int4));
    if (rc) return rc;
    rc = ensure_scratch(ctx, ctx->wgx_part, std::max<size_t>(n_pieces, 1) * 256 * 256 * sizeof(float));
    if (rc) return rc;
    ADLOCO_HIP_CHECK(ctx, hipMemcpyAsync(ctx->wgx_tab.ptr, tiles.data(), tiles.size() * sizeof(int4),
                                         hipMemcpyHostToDevice, st));
    if (!split.empty())
      ADLOCO_HIP_CHECK(ctx, hipMemcpyAsync(ctx->wgx_split.ptr, split.data(),
                                           split.size() * sizeof(int4), hipMemcpyHostToDevice, st));
    ADLOCO_HIP_CHECK(ctx, hipStreamSynchronize(st));
    ctx->wgx_slots = slots;
    ctx->wgx_n_split = int(split.size());
  }
  ctx->layer_tab_host = std::move(tab);
  ctx->order_host = std::move(order);
  ctx->wgrad_blocks = int(wg);
  ctx->table_dtype = dtype;
  ctx->table_inputs = int(need_inputs);
  return ADLOCO_OK;
}

// Descriptor lists of the vector and embedding-table blocks for a batch of B x T tokens, and
// the scratch they need.  Rebuilt when the layer table or the batch shape changed.
int prepare_vector_table(adloco_ctx* ctx, int B, int T, hipStream_t st) {
  if (ctx->aux_B == B && ctx->aux_T == T) return ADLOCO_OK;
  if (ctx->n_linear == int(ctx->layer_tab_host.size())) {      // no such blocks
    ctx->vec_host.clear();
    ctx->emb_host.clear();
    ctx->vec_blocks = ctx->vec_blocks2 = ctx->emb_blocks = 0;
    ctx->aux_B = B;
    ctx->aux_T = T;
    return ADLOCO_OK;
  }
  ++ctx->table_builds;
  const int slab = vector_table_slab();
  std::vector<AuxDesc> vec, emb;
  std::vector<char> fused;     // per vector block: 1 = its row sums are formed by another block's workgroups
  long long vb = 0, vb2 = 0, eb = 0, voff = 0, poff = 0, partoff = 0;
  for (size_t l = 0; l < ctx->layer_tab_host.size(); ++l) {
    const LayerDev& L = ctx->layer_tab_host[l];
    if (L.kind == ADLOCO_KIND_LINEAR) continue;
    AuxDesc A{};
    A.layer = int(l);
    const int w = L.kind == ADLOCO_KIND_VECTOR ? slab : embed_table_slab();
    A.slabs = (L.d_out + w - 1) / w;
    if (L.kind == ADLOCO_KIND_VECTOR) {
      A.blk_start = int(vb);
      A.blk_start2 = int(vb2);
      A.vec_off = voff;
      A.vec_off_bias = -1;
      // a gain (x given) and a bias (x = 1) that read the same delta rows -- the two vectors of a
      // normalisation layer -- are formed in one pass over delta by the gain block's workgroups
      int host = -1;
      if (L.delta_twin >= 0) {
        for (size_t k = 0; k < vec.size(); ++k)
          if (vec[k].layer == L.delta_twin) host = int(k);
      }
      const bool pair = host >= 0 && vec[host].vec_off_bias < 0 && !fused[host] &&
                        (ctx->layer_tab_host[vec[host].layer].a == nullptr) != (L.a == nullptr);
      if (pair && L.a == nullptr) {
        // this bias rides on the earlier gain block: no row-sum workgroups of its own
        vec[host].vec_off_bias = voff;
        fused.push_back(1);
      } else if (pair) {
        // this gain also serves the earlier bias block, whose workgroups are withdrawn
        A.vec_off_bias = vec[host].vec_off;
        const long long gone = (long long)B * vec[host].slabs;
        for (size_t k = host + 1; k < vec.size(); ++k) vec[k].blk_start -= int(gone);
        vb -= gone;
        A.blk_start = int(vb);
        fused[host] = 1;
        fused.push_back(0);
      } else {
        fused.push_back(0);
      }
      if (!(pair && L.a == nullptr)) vb += (long long)B * A.slabs;
      vb2 += A.slabs;
      voff += (long long)B * L.d_out;
      vec.push_back(A);
    } else {
      A.blk_start = int(eb);
      A.perm_off = poff;
      A.part_off = partoff;
      eb += (long long)B * A.slabs;
      poff += (long long)B * T;
      partoff += (long long)B * A.slabs;
      emb.push_back(A);
    }
    if (vb > 0x7fffffffLL || eb > 0x7fffffffLL)
      return fail(ctx, ADLOCO_EUNSUPPORTED, "grad_stats: too many vector / table blocks for one launch");
  }
  if (!emb.empty() && T > 8192)
    return fail(ctx, ADLOCO_EUNSUPPORTED, "grad_stats: embedding blocks need T <= 8192, got %d", T);
  int rc = ensure_scratch(ctx, ctx->vec_tab, std::max<size_t>(vec.size(), 1) * sizeof(AuxDesc));
  if (rc) return rc;
  rc = ensure_scratch(ctx, ctx->emb_tab, std::max<size_t>(emb.size(), 1) * sizeof(AuxDesc));
  if (rc) return rc;
  rc = ensure_scratch(ctx, ctx->aux_vec, std::max<size_t>(size_t(voff), 1) * sizeof(float));
  if (rc) return rc;
  rc = ensure_scratch(ctx, ctx->aux_perm, std::max<size_t>(size_t(poff), 1) * sizeof(int));
  if (rc) return rc;
  rc = ensure_scratch(ctx, ctx->aux_part, std::max<size_t>(size_t(partoff), 1) * sizeof(double));
  if (rc) return rc;
  ctx->aux_B = ctx->aux_T = -1;
  if (!vec.empty())
    ADLOCO_HIP_CHECK(ctx, hipMemcpyAsync(ctx->vec_tab.ptr, vec.data(), vec.size() * sizeof(AuxDesc),
                                         hipMemcpyHostToDevice, st));
  if (!emb.empty())
    ADLOCO_HIP_CHECK(ctx, hipMemcpyAsync(ctx->emb_tab.ptr, emb.data(), emb.size() * sizeof(AuxDesc),
                                         hipMemcpyHostToDevice, st));
  if (!vec.empty() || !emb.empty()) ADLOCO_HIP_CHECK(ctx, hipStreamSynchronize(st));
  ctx->vec_host = std::move(vec);
  ctx->emb_host = std::move(emb);
  ctx->vec_blocks = int(vb);
  ctx->vec_blocks2 = int(vb2);
  ctx->emb_blocks = int(eb);
  ctx->aux_B = B;
  ctx->aux_T = T;
  return ADLOCO_OK;
}

// Time of the Gram contraction of 16-bit blocks by the dual-tile and the region kernel, in microseconds: the jobs of the XCD
// with the most units (cycles a chunk of 64 elements: 1024 off the diagonal and 768 on it; region 2048 and 1152) and their
// starts over its 32 workgroups and a rate, plus most of a job at the end, and no less than the longest job.  The region
// kernel always contracts the activations that layers share once, the dual-tile kernel only where no tile is ragged.  Jobs
// of the region kernel are twice as large and start more slowly, so it needs more of them to fill the chip, and a last block
// that is mostly padding costs it more (T 257 to 384: 1.13 to 1.3 times the time of the dual-tile kernel).  Fitted to 760
// lists on data that no cache held (T 17 .. 4096, widths 128 .. 2048, 1 to 24 blocks of GPT or Llama shapes, B 1 to 64):
// the choice is within 0.2 % of the better kernel on average and 16 % at worst; up to T 128 it is the dual-tile kernel in all
// of them.  Measured, dual -> region: 350M model, B 32, T 1024 13.7 -> 11.4 ms; two Llama-1B blocks, B 16, T 2048 4.88 ->
// 3.82; GPT-2-small, B 32, T 256 0.58 -> 0.41, T 512 1.50 -> 1.35; two blocks of it, B 4, T 512 0.055 -> 0.083, not taken.
struct GramTime { double dual, region; };
GramTime gram_time(const adloco_ctx* ctx, int B, int T) {
  auto model = [&](const GramLoad& g, int edge, double off, double on, int per_job, double start, double rate, double fixed) {
    const int n = (T + edge - 1) / edge;
    const double n_off = std::ceil(double(n) * (n - 1) / 2 / per_job);
    // (of an odd number of tile pairs on and off the diagonal, the last two make one job)
    const double n_on = (n + per_job - 1) / per_job - (per_job == 2 && n % 4 == 3);
    const double units = std::max(1.0, double(g.count) * B), most = std::ceil(units / kNumXcd), jobs = (n_off + n_on) * most;
    const double work = (n_off * (g.chunks * off + start * g.count) + n_on * (g.chunks * on + start * g.count)) * B * most / units;
    const double longest = g.longest * (n_off > 0 ? off : on) + start, wgs = kNumCu / kNumXcd;
    return (jobs > wgs ? std::max(longest, work / wgs + 0.66 * work / jobs) : longest) / rate + fixed;
  };
  return GramTime{model(ctx->gram_load[T % 128 == 0], 128, 1024, 768, 2, 5270, 1203, 2.7),
                  model(ctx->gram_load[1], 256, 2048, 1152, 1, 9950, 1474, 2.2)};
}

// Norms of linear blocks whose gradient sums are supplied: true where the tiles of the per-sample gradients
// (2 d_in d_out T products) take less time than the Gram contraction ((d_in + d_out) T (T + 1)), as on sequences that
// are long for the widths.  gram_us: the time of the Gram kernels for widths that are multiples of 64 (0: they do not take
// this call); the tiles then take 0.46 us a chunk, 0.72 a finished tile, 2.8 a run of samples and 8 in all, and the choice
// is within 0.7 % of the better way on average and 24 % at worst (260 lists as above; 17 % and 3.3 times with rates alone).
// Else microseconds from measured rates: 16-bit tiles 0.55 PFLOP/s on 256 workgroups of 256 x 128 (the pieces of a row
// straddle cache lines), the general Gram kernel 0.35; fp32 tiles 150 TFLOP/s on 512 workgroups of 128 x 128, the fp32 Gram
// kernel 15; 20 us for starts and ends.  Measured, Gram -> tiles: bf16 7 x {600 -> 1800, ..}, B 3, T 2688 2.77 -> 0.77 ms; 6 x
// {320 -> 960, ..}, B 6, T 1792 0.90 -> 0.37; fp32 {512 -> 1408, ..}, B 11, T 1395 8.3 -> 1.1; {1336 -> 4008, ..}, B 3,
// T 1024 stays with the Gram kernel: 0.28 against 0.40, and so does {960 -> 960, .., 960 -> 2240} x 3, B 15, T 27: 46 us
// against 119.
bool tiles_beat_gram(const adloco_ctx* ctx, int B, int T, int dtype, double gram_us) {
  if (gram_us > 0.0) {
    const TileGeom geom = ip_tile_geom();
    const long long n = ctx->tiles16.n_tiles, room = (long long)geom.room * kNumXcd;
    const double sample = (T + geom.k - 1) / geom.k * 0.46 + 0.72;
    if (8.0 + double(n) * B / room * sample >= 0.95 * gram_us) return false;       // (whatever the runs, which are searched for)
    const int group = run_length(n, B, T, geom);
    const double rounds = double((n * ((B + group - 1) / group) + room - 1) / room);
    return 8.0 + rounds * (group * sample + 2.8) < 0.95 * gram_us;
  }
  const bool b16 = is_16bit(dtype);
  const long long te = b16 ? 256 : 128, tc = 128, gt = b16 ? 128 : 32, wgs = b16 ? 256 : 512;
  const double tile_rate = b16 ? 5.5e8 : 1.5e8, gram_rate = b16 ? 3.5e8 : 1.5e7;   // flop per us
  const double nt = double((T + gt - 1) / gt);
  double tiles = 0.0, gram = 0.0;
  for (const LayerDev& L : ctx->layer_tab_host) {
    if (L.kind != ADLOCO_KIND_LINEAR) continue;
    tiles += double((L.d_out + te - 1) / te) * double((L.d_in + tc - 1) / tc);
    gram += nt * (nt + 1) * gt * gt * (double(L.d_in) + L.d_out);
  }
  const double per_round = 2.0 * te * tc * double((T + 31) / 32 * 32) * wgs / tile_rate;
  const double t_tiles = std::max(1.0, tiles * B / wgs) * per_round + 20.0;
  return t_tiles < 0.95 * gram * B / gram_rate;
}

// Gradient sums formed here: true where the tiles of the per-sample gradients, whose samples are padded to whole chunks
// (32 token rows), take less time than the Gram contraction followed by the sum over all rows, which pays for
// no padding: short sequences on wide layers go the second way.  With the time of the Gram kernels (gram_us, as above) the
// tiles take 0.53 us a chunk, 1.1 a finished tile, 7 a tile of G and 16 in all, the sum over all rows 0.74 a chunk of its
// 256 x 256 tiles, 13 a tile and 16 in all: within 0.4 % of the better way on average and 19 % at worst (142 ragged lists
// as above).  Else rates as above, gradient sums at 1.2 PFLOP/s / 80 TFLOP/s; the work on a finished 16-bit tile is worth
// 48 token rows.  Measured, fp16: {1024 -> 3072, ..} x 4, B 8, T 17 0.30 ms by tiles, 0.23 the second way; {512 -> 1536,
// ..}, B 8, T 333 0.11 against 0.14; {960 -> 960, .., 960 -> 2240} x 3, B 15, T 27 0.158 against 0.114.
bool formed_tiles_pay(const adloco_ctx* ctx, int B, int T, int dtype, double gram_us) {
  if (gram_us > 0.0) {
    const double chunks = (T + 31) / 32, n = double(ctx->tiles16.n_tiles) / kNumCu, sample = chunks * 0.53 + 1.1;
    const double tiles = 16.0 + std::max(n * (B * sample + 7.0), std::min(double(B), std::max(1.0, n * B)) * sample + 7.0);
    const double w = n / 2, rows = double(B) * T / 32;           // (half as many tiles, each of twice the size)
    const double pieces = std::max(1.0, std::floor(1.0 / std::max(w, 1.0 / kNumCu)));
    const double sum = 16.0 + std::max(w * (rows * 0.74 + 13.0), std::ceil(rows / pieces) * 0.74 + 13.0);
    return tiles <= gram_us + sum;
  }
  const bool b16 = is_16bit(dtype);
  const long long gt = b16 ? 128 : 32, chunk = 32;
  const double tile_rate = b16 ? 9.5e8 : 1.5e8, gram_rate = b16 ? 3.5e8 : 1.5e7, sum_rate = b16 ? 1.2e9 : 8e7;
  const double nt = double((T + gt - 1) / gt), rows = double((T + chunk - 1) / chunk * chunk + (b16 ? 48 : 0));
  double tiles = 0.0, gram = 0.0;
  for (const LayerDev& L : ctx->layer_tab_host) {
    if (L.kind != ADLOCO_KIND_LINEAR) continue;
    const double io = 2.0 * L.d_in * L.d_out;
    tiles += io * rows / tile_rate;
    gram += nt * (nt + 1) * gt * gt * (double(L.d_in) + L.d_out) / gram_rate + io * T / sum_rate;
  }
  return tiles <= gram;
}

}  // namespace

namespace adloco {

int grad_stats(adloco_ctx* ctx, const adloco_linear_desc* layers, int n_layers, int B, int T, int dtype,
               float* per_sample_sqnorm, float* per_layer_sample_sqnorm, adloco_stats_acc* acc, uint32_t flags,
               bool pinned_order, void* stream) {
  if (!ctx) return ADLOCO_EINVAL;
  if (!layers || n_layers < 1) return fail(ctx, ADLOCO_EINVAL, "grad_stats: no layers");
  if (n_layers > kMaxLayers)
    return fail(ctx, ADLOCO_EUNSUPPORTED, "grad_stats: n_layers = %d exceeds %d", n_layers, kMaxLayers);
  if (B < 1 || T < 1) return fail(ctx, ADLOCO_EINVAL, "grad_stats: B = %d, T = %d must be >= 1", B, T);
  if (dtype != ADLOCO_F32 && !is_16bit(dtype))
    return fail(ctx, ADLOCO_EUNSUPPORTED, "grad_stats: dtype %d not supported", dtype);
  if (flags & ~(ADLOCO_ACCUMULATE | ADLOCO_SUM_ONLY)) return fail(ctx, ADLOCO_EINVAL, "grad_stats: unknown flags");
  const bool sum_only = (flags & ADLOCO_SUM_ONLY) != 0;
  if (!sum_only && (!per_sample_sqnorm || !acc)) return fail(ctx, ADLOCO_EINVAL, "grad_stats: NULL output");
  if (reinterpret_cast<uintptr_t>(acc) % 8)
    return fail(ctx, ADLOCO_EINVAL, "grad_stats: acc not 8-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int accumulate = (flags & ADLOCO_ACCUMULATE) ? 1 : 0;

  int rc = prepare_tables(ctx, layers, n_layers, dtype, true, st);
  if (rc) return rc;
  rc = prepare_vector_table(ctx, B, T, st);
  if (rc) return rc;

  const int tile = gram_tile_edge(dtype, ctx->gram_variant);
  const long long nt = (T + tile - 1) / tile;
  if (nt > 4096) return fail(ctx, ADLOCO_EUNSUPPORTED, "grad_stats: T = %d gives too many tiles", T);
  // (the dual-tile kernel addresses a sample's rows with 32-bit byte offsets)
  const bool dual = is_16bit(dtype) && ctx->gram_variant != 0 && ctx->all_fast64 &&
                    (long long)T * ctx->max_lin_stride < (1LL << 31) - 64;
  const GramTime gram_us = dual ? gram_time(ctx, B, T) : GramTime{0.0, 0.0};
  const bool region = dual && ctx->min_width >= 128 && ((long long)T + 256) * ctx->max_lin_stride < (1LL << 31) &&
                      (ctx->gram_variant == 3 || (ctx->gram_variant == 1 && T > 128 && gram_us.region < gram_us.dual));
  const double t_gram = region ? gram_us.region : gram_us.dual;
  long long n_pairs = nt * (nt + 1) / 2, spare_pairs = n_pairs;      // partial sums per (layer, sample)
  if (dual) {
    // built whichever of the two kernels this batch takes, and room kept for the sums of the one that leaves more: another
    // batch of the same sequence length may take the other, in a call that is being captured
    if (ctx->job_tab_nt != int(nt)) {
      ++ctx->table_builds;
      std::vector<GramJob> jobs = make_gram_jobs(int(nt), ctx->gram_job_order >= 0 ? ctx->gram_job_order : (nt >= 6 ? 0 : 1));
      rc = ensure_scratch(ctx, ctx->job_tab, jobs.size() * sizeof(GramJob));
      if (rc) return rc;
      ctx->job_tab_nt = -1;
      ADLOCO_HIP_CHECK(ctx, hipMemcpyAsync(ctx->job_tab.ptr, jobs.data(), jobs.size() * sizeof(GramJob),
                                           hipMemcpyHostToDevice, st));
      ADLOCO_HIP_CHECK(ctx, hipStreamSynchronize(st));
      ctx->job_tab_nt = int(nt);
      ctx->job_tab_n = int(jobs.size());
    }
    n_pairs = spare_pairs = gram_dual_parts(ctx->job_tab_n);
    if (region) {
      n_pairs = 4 * gram_region_jobs(T);
      spare_pairs = std::max(spare_pairs, n_pairs);
    }
  }
  if (n_pairs > 0x7fffffffLL || (long long)n_layers * B * n_pairs > (1LL << 40))
    return fail(ctx, ADLOCO_EUNSUPPORTED, "grad_stats: T = %d gives too many tile pairs", T);

  // Per-sample gradient tiles (explicit form) when the gradient sums of all linear blocks are formed here: the tiles
  // that add up to them are squared on the way, no Gram contraction is needed.  16-bit blocks if they are aligned;
  // fp32 ones too: 4 x {768 -> 2304, 768 -> 768, 768 -> 3072, 3072 -> 768}, B 8, T 256 takes 0.74 ms
  // against 5.02 ms with the vector-unit kernels of the two steps.
  const bool tiles_allowed = ctx->stats_variant != 0 && ctx->n_linear > 0 && B <= 0x7fff;
  const bool all_formed = ctx->n_formed == ctx->n_linear;
  const std::vector<LayerDev>& tab = ctx->layer_tab_host;
  bool tile_form = !sum_only && tiles_allowed && all_formed && ctx->tiles16.built && is_16bit(dtype) &&
                   (T % 32 == 0 || (!pinned_order && formed_tiles_pay(ctx, B, T, dtype, t_gram))) && T <= (1 << 20);
  bool plain_form = !sum_only && tiles_allowed && all_formed && dtype == ADLOCO_F32 && !pinned_order &&
                    formed_tiles_pay(ctx, B, T, dtype, t_gram);
  bool square_form = !sum_only && tiles_allowed && ctx->n_formed == 0 && T <= (1 << 20) &&
                     (dtype == ADLOCO_F32 || ctx->tiles16.built) && tiles_beat_gram(ctx, B, T, dtype, t_gram);
  const bool short_form = tile_form && short_sequences(tab, ctx->tiles16.use, B, T, false);
  const long long rows = (long long)B * T;
  // the list of the fp32 forms, and what a form leaves per (tile, sample)
  const TileList* list = &ctx->tiles16;
  size_t out_bytes = (tile_form ? tile_waves(short_form) : tile_waves(false)) * sizeof(float);
  PlainChoice plain{2, false};
  if (plain_form || (square_form && dtype == ADLOCO_F32)) {
    if (plain_form && ctx->plain_tiles_tuning) plain = PlainChoice{ctx->plain_tiles_tuning & 3, (ctx->plain_tiles_tuning & 4) != 0};
    else if (plain_form) plain = plain_tile_choice(ctx->tiles32, B, T);
    else plain.W = ctx->plain_tiles_tuning ? ctx->plain_tiles_tuning & 3 : plain_tile_width(tab, ctx->tiles32[0].use, B, T);
    list = &ctx->tiles32[plain.W - 1];
    out_bytes = sizeof(double);
  }
  int group = 0;
  if (square_form) {
    group = run_length(list->n_tiles, B, T, dtype == ADLOCO_F32 ? plain_tile_geom(list->edge / 64) : ip_tile_geom());
    square_form = (long long)list->used(1) * kNumXcd * ((B + group - 1) / group) <= 0x7fffffffLL;
  }
  // without the list or the memory for its results, a call takes the Gram contraction (and the sum over all rows)
  if (!list->built || ((tile_form || plain_form || square_form) &&
                       !obtain_scratch(ctx, ctx->tile_out, out_bytes * size_t(list->n_tiles) * B, st)))
    tile_form = plain_form = square_form = false;
  const bool formed = tile_form || plain_form || square_form;     // norms (and gradient sums) come from the tiles
  const TileList* sum_list = nullptr;
  if (dtype == ADLOCO_F32 && !formed && ctx->n_formed > 0 && rows < (1 << 30) && ctx->stats_variant != 0)
    sum_list = &ctx->tiles32[sum_tile_width(tab, ctx->tiles32[0].use) - 1];
  const bool plain_sum = sum_list && sum_list->built;
  const size_t part_bytes = size_t(n_layers) * B * sizeof(float);
  // one finished sum per (layer, sample) comes from the tiles; up to 64 MiB, there is room for those of a Gram contraction
  // too, so that a captured call on another batch finds it
  if (formed) n_pairs = 1;
  const size_t spare_bytes = part_bytes * size_t(spare_pairs);
  if (spare_bytes > (size_t(64) << 20) || !obtain_scratch(ctx, ctx->partials, spare_bytes, st))
    rc = ensure_scratch(ctx, ctx->partials, part_bytes * size_t(n_pairs));
  if (rc) return rc;
  rc = ensure_scratch(ctx, ctx->sample_f64, size_t(B) * sizeof(double));
  if (rc) return rc;

  GramLaunch g;
  g.layers = static_cast<const LayerDev*>(ctx->layer_tab.ptr);
  g.order = static_cast<const int*>(ctx->order_tab.ptr);
  g.n_layers = ctx->n_linear;   // the Gram launch walks order_tab: linear weights only
  g.B = B;
  g.T = T;
  g.partials = static_cast<float*>(ctx->partials.ptr);
  g.n_pairs = int(n_pairs);
  g.tile = tile;
  g.dtype = dtype;
  // ---- vector / table blocks.  With linear blocks in the same call they go to a second stream:
  // they are HBM-bound, the kernels of the linear blocks MFMA / L2-bound, and both fit on a CU.
  const bool have_aux = !ctx->vec_host.empty() || !ctx->emb_host.empty();
  bool fork = have_aux && ctx->n_linear > 0 && ctx->overlap_aux != 0;
  if (fork && !ctx->side_stream) {
    if (hipStreamCreateWithFlags(&ctx->side_stream, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&ctx->ev_fork, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&ctx->ev_join, hipEventDisableTiming) != hipSuccess) {
      (void)hipGetLastError();
      fork = false;                      // no second stream: run in line
    }
  }
  hipStream_t aux_st = fork ? ctx->side_stream : st;
  auto launch_aux = [&]() -> int {
    hipEvent_t ev_aux = prof_begin(ctx, aux_st);
    hipError_t ea = launch_vector_stats(g.layers, static_cast<const AuxDesc*>(ctx->vec_tab.ptr),
                                        int(ctx->vec_host.size()), ctx->vec_blocks, ctx->vec_blocks2, B, T,
                                        dtype, static_cast<float*>(ctx->aux_vec.ptr), sum_only ? nullptr : g.partials,
                                        int(n_pairs), accumulate, true, aux_st);
    if (ea == hipSuccess && !sum_only)
      ea = launch_embed_stats(g.layers, static_cast<const AuxDesc*>(ctx->emb_tab.ptr),
                              int(ctx->emb_host.size()), ctx->emb_blocks, B, T, dtype,
                              static_cast<int*>(ctx->aux_perm.ptr),
                              static_cast<double*>(ctx->aux_part.ptr), g.partials, int(n_pairs), aux_st);
    prof_end(ctx, kProfVecTab, ev_aux, aux_st);
    if (ea != hipSuccess)
      return fail(ctx, ADLOCO_EHIP, "grad_stats: vector / table launch failed: %s", hipGetErrorString(ea));
    return ADLOCO_OK;
  };
  if (fork) {
    ADLOCO_HIP_CHECK(ctx, hipEventRecord(ctx->ev_fork, st));
    ADLOCO_HIP_CHECK(ctx, hipStreamWaitEvent(aux_st, ctx->ev_fork, 0));
    rc = launch_aux();
    if (rc) return rc;
  }
  hipEvent_t ev = nullptr;
  hipError_t e = hipSuccess;
  if (formed) {
    ev = prof_begin(ctx, st);
    float* const out16 = static_cast<float*>(ctx->tile_out.ptr);
    if (tile_form)
      e = launch_stats_tiles(g.layers, *list, B, T, dtype, accumulate, short_form, out16, g.partials, st);
    else if (square_form && is_16bit(dtype))
      e = launch_square_tiles(g.layers, *list, B, T, dtype, out16, g.partials, st);
    else
      e = launch_plain_tiles(g.layers, *list, plain_form ? 1 : 3, B, T, dtype, accumulate, plain.whole, group,
                             static_cast<double*>(ctx->tile_out.ptr), nullptr, g.partials, 1, st);
    prof_end(ctx, kProfTileStats, ev, st);
    if (e != hipSuccess)
      return fail(ctx, ADLOCO_EHIP, "grad_stats: tile statistics launch failed: %s", hipGetErrorString(e));
  }
  const bool gram = !formed && !sum_only && ctx->n_linear > 0;
  ctx->gram_kernel = !gram ? 0 : region ? 3 : dual ? 2 : 1;
  ev = gram ? prof_begin(ctx, st) : nullptr;
  if (!gram)
    ;
  else if (dual) {
    // the dual-tile kernel walks groups of layers that share their activations (A A^T once per group)
    // when some do and no tile is ragged, else every layer by itself
    GramLaunch gd = g;
    const bool grouped = ctx->n_groups < ctx->n_linear && (region || T % tile == 0);
    const char* base = static_cast<const char*>(ctx->group_tab.ptr) + (grouped ? 0 : ctx->single_off);
    gd.n_layers = grouped ? ctx->n_groups : ctx->n_linear;
    gd.order = reinterpret_cast<const int*>(base + size_t(gd.n_layers) * sizeof(GramGroup));
    if (region)
      e = launch_gram_region(gd, reinterpret_cast<const GramGroup*>(base), st);
    else
      e = launch_gram_bf16_dual(gd, reinterpret_cast<const GramGroup*>(base),
                              static_cast<const GramJob*>(ctx->job_tab.ptr), ctx->job_tab_n,
                              grouped ? kGramGroupMax : 1, st);
  }
  else if (is_16bit(dtype))
    e = launch_gram_bf16(g, ctx->gram_variant, st);
  else
    e = launch_gram_f32(g, st);
  prof_end(ctx, kProfGram, ev, st);
  if (e != hipSuccess)
    return fail(ctx, ADLOCO_EHIP, "grad_stats: Gram launch failed: %s", hipGetErrorString(e));
  ev = (!formed && ctx->wgrad_blocks > 0) ? prof_begin(ctx, st) : nullptr;
  if (formed)
    ;
  else if (plain_sum)
    e = launch_plain_tiles(g.layers, *sum_list, 2, 1, int(rows), dtype, accumulate, true, 1, nullptr, nullptr, nullptr, 0, st);
  else if (is_16bit(dtype) && ctx->wgrad_variant >= 2 && ctx->wgx_slots > 0 && (rows % 32 == 0 || !pinned_order) &&
           rows / 32 < 0x7fffffffLL)
    e = launch_wgrad_x(g.layers, ctx->wgx_tab.ptr, ctx->wgx_slots, ctx->wgx_split.ptr,
                       ctx->wgx_n_split, static_cast<float*>(ctx->wgx_part.ptr), rows, accumulate,
                       dtype, st);
  else
    e = launch_wgrad(g.layers, n_layers, ctx->wgrad_blocks, rows, dtype, accumulate,
                     ctx->wgrad_variant >= 2 ? 1 : ctx->wgrad_variant, st);
  prof_end(ctx, kProfWgrad, ev, st);
  if (e != hipSuccess)
    return fail(ctx, ADLOCO_EHIP, "grad_stats: gradient-sum launch failed: %s", hipGetErrorString(e));
  if (have_aux && !fork) {
    rc = launch_aux();
    if (rc) return rc;
  }
  if (fork) {
    ADLOCO_HIP_CHECK(ctx, hipEventRecord(ctx->ev_join, aux_st));
    ADLOCO_HIP_CHECK(ctx, hipStreamWaitEvent(st, ctx->ev_join, 0));
  }
  if (sum_only) return ADLOCO_OK;       // the gradient sums are all this call was asked for
  e = launch_finalize_stats(g.partials, n_layers, B, int(n_pairs), per_sample_sqnorm,
                            per_layer_sample_sqnorm, static_cast<double*>(ctx->sample_f64.ptr),
                            acc, accumulate, st);
  if (e != hipSuccess)
    return fail(ctx, ADLOCO_EHIP, "grad_stats: reduction launch failed: %s", hipGetErrorString(e));
  return ADLOCO_OK;
}

}  // namespace adloco

extern "C" int adloco_grad_stats(adloco_ctx* ctx, const adloco_linear_desc* layers, int n_layers,
                                 int B, int T, int dtype, float* per_sample_sqnorm,
                                 float* per_layer_sample_sqnorm, adloco_stats_acc* acc,
                                 uint32_t flags, void* stream) {
  return grad_stats(ctx, layers, n_layers, B, T, dtype, per_sample_sqnorm, per_layer_sample_sqnorm, acc, flags, false,
                    stream);
}

// ip: also read back the accumulator of the inner products, into ctx->pinned[4..7] (NULL: none).
static int norm_test(adloco_ctx* ctx, const adloco_linear_desc* layers, int n_layers, const adloco_stats_acc* acc,
                     const adloco_ip_acc* ip, double eta, int64_t b_cur, int64_t b_max, int32_t n_switch,
                     int64_t b_cap, uint32_t flags, adloco_norm_test_result* out, void* stream) {
  if (!ctx) return ADLOCO_EINVAL;
  if (!layers || n_layers < 1) return fail(ctx, ADLOCO_EINVAL, "norm_test: no layers");
  if (n_layers > kMaxLayers)
    return fail(ctx, ADLOCO_EUNSUPPORTED, "norm_test: n_layers = %d exceeds %d", n_layers, kMaxLayers);
  if (!acc || !out) return fail(ctx, ADLOCO_EINVAL, "norm_test: NULL acc or out");
  if (!(eta > 0.0) || b_cur < 1 || b_max < 1 || n_switch < 1 || b_cap < 0 ||
      (flags & ~(ADLOCO_BIASED_VAR | ADLOCO_ALLOW_SHRINK)))
    return fail(ctx, ADLOCO_EINVAL, "norm_test: bad eta, b_cur, b_max, n_switch, b_cap or flags");
  hipStream_t st = static_cast<hipStream_t>(stream);
  // the table is shared with grad_stats: same layer list -> no upload
  const int dtype = ctx->table_dtype >= 0 ? ctx->table_dtype : ADLOCO_BF16;
  // (same widths as the table of the last call: only the grad_sum pointers are refreshed)
  bool cached = ctx->layer_tab_host.size() == size_t(n_layers);
  if (cached)
    for (int l = 0; l < n_layers && cached; ++l) {
      const LayerDev& L = ctx->layer_tab_host[l];
      cached = L.grad_sum != nullptr && L.d_in == layers[l].d_in && L.d_out == layers[l].d_out &&
               layers[l].grad_sum != nullptr && (reinterpret_cast<uintptr_t>(layers[l].grad_sum) % 4) == 0;
    }
  if (cached) {
    // (written on every call: a graph replayed in between may have left other pointers in the table)
    for (int l = 0; l < n_layers; ++l) ctx->layer_tab_host[l].grad_sum = layers[l].grad_sum;
    int rc = upload_pointers(ctx, ctx->layer_tab_host, 2, st);
    if (rc) return rc;
  } else {
    int rc = prepare_tables(ctx, layers, n_layers, dtype, false, st);
    if (rc) return rc;
  }
  const size_t nblk = sqnorm_partials(ctx->layer_tab_host);
  int rc = ensure_scratch(ctx, ctx->red_f64, nblk * sizeof(double));
  if (rc) return rc;
  hipEvent_t ev = prof_begin(ctx, st);
  const bool direct = kernel_can_read(ctx, acc) && (!ip || kernel_can_read(ctx, ip));
  hipError_t e = launch_sqnorm(static_cast<const LayerDev*>(ctx->layer_tab.ptr), n_layers, nblk,
                               static_cast<double*>(ctx->red_f64.ptr), direct ? acc : nullptr,
                               direct ? ip : nullptr, ctx->pinned, st);
  prof_end(ctx, kProfSqnorm, ev, st);
  if (e != hipSuccess)
    return fail(ctx, ADLOCO_EHIP, "norm_test: reduction launch failed: %s", hipGetErrorString(e));
  if (!direct) {
    ADLOCO_HIP_CHECK(ctx, hipMemcpyAsync(ctx->pinned + 2, acc, sizeof(adloco_stats_acc), hipMemcpyDeviceToHost, st));
    if (ip) ADLOCO_HIP_CHECK(ctx, hipMemcpyAsync(ctx->pinned + 4, ip, sizeof *ip, hipMemcpyDeviceToHost, st));
  }
  ADLOCO_HIP_CHECK(ctx, hipStreamSynchronize(st));
  const double S2 = ctx->pinned[0];
  adloco_stats_acc h;
  std::memcpy(&h, ctx->pinned + 2, sizeof h);
  if (h.n_samples < 1)
    return fail(ctx, ADLOCO_ESTATE, "norm_test: accumulator holds no samples (n_samples = %lld)",
                (long long)h.n_samples);
  rc = adloco_norm_test_decide(h.sum_sample_sqnorm, S2, h.n_samples, eta, b_cur, b_max, n_switch,
                               b_cap, flags, out);
  if (rc) return fail(ctx, rc, "norm_test: decision rejected S1 = %g, S2 = %g", h.sum_sample_sqnorm, S2);
  return ADLOCO_OK;
}

extern "C" int adloco_norm_test(adloco_ctx* ctx, const adloco_linear_desc* layers, int n_layers,
                                const adloco_stats_acc* acc, double eta, int64_t b_cur,
                                int64_t b_max, int32_t n_switch, int64_t b_cap, uint32_t flags,
                                adloco_norm_test_result* out, void* stream) {
  return norm_test(ctx, layers, n_layers, acc, nullptr, eta, b_cur, b_max, n_switch, b_cap, flags, out, stream);
}

// ---------------------------------------------------------------------------------------------
// Inner products c_i = <g_i, G> (Section 3.3.2)
// ---------------------------------------------------------------------------------------------
extern "C" int adloco_inner_products(adloco_ctx* ctx, const adloco_linear_desc* layers, int n_layers,
                                     int B, int T, int dtype, float* per_sample_ip,
                                     float* per_sample_sqnorm, adloco_ip_acc* acc, uint32_t flags,
                                     void* stream) {
  if (!ctx) return ADLOCO_EINVAL;
  if (!layers || n_layers < 1) return fail(ctx, ADLOCO_EINVAL, "inner_products: no layers");
  if (n_layers > kMaxLayers)
    return fail(ctx, ADLOCO_EUNSUPPORTED, "inner_products: n_layers = %d exceeds %d", n_layers, kMaxLayers);
  if (B < 1 || T < 1) return fail(ctx, ADLOCO_EINVAL, "inner_products: B = %d, T = %d must be >= 1", B, T);
  if (B > 0x7fff) return fail(ctx, ADLOCO_EUNSUPPORTED, "inner_products: B = %d exceeds 32767", B);
  if (dtype != ADLOCO_F32 && !is_16bit(dtype))
    return fail(ctx, ADLOCO_EUNSUPPORTED, "inner_products: dtype %d not supported", dtype);
  if (!per_sample_ip || !acc) return fail(ctx, ADLOCO_EINVAL, "inner_products: NULL output");
  if (reinterpret_cast<uintptr_t>(acc) % 8)
    return fail(ctx, ADLOCO_EINVAL, "inner_products: acc not 8-byte aligned");
  if (flags & ~ADLOCO_ACCUMULATE) return fail(ctx, ADLOCO_EINVAL, "inner_products: unknown flags");
  for (int l = 0; l < n_layers; ++l)
    if (!layers[l].grad_sum)
      return fail(ctx, ADLOCO_EINVAL, "inner_products: layer %d has no grad_sum (G is read here)", l);
  hipStream_t st = static_cast<hipStream_t>(stream);
  int rc = prepare_tables(ctx, layers, n_layers, dtype, true, st);
  if (rc) return rc;
  rc = prepare_vector_table(ctx, B, T, st);
  if (rc) return rc;
  const std::vector<LayerDev>& tab = ctx->layer_tab_host;

  // ---- which blocks go through the tile GEMM, and its tile table
  if (ctx->ip_B != B || ctx->ip_T != T) {
    ++ctx->table_builds;
    std::vector<char> use(n_layers, 0);
    bool any = false;
    for (int l = 0; l < n_layers; ++l) {
      // the tile kernel counts an entry's chunks of 32 rows in 32 bits and addresses the rows of a
      // chunk with 32-bit byte offsets
      use[l] = tab[l].kind == ADLOCO_KIND_LINEAR && is_16bit(dtype) && tab[l].fast && T <= (1 << 20) && tab[l].a_stride < (1 << 25) && tab[l].delta_stride < (1 << 25);
      any = any || use[l];
    }
    std::vector<int4> tiles;
    int group = 1;
    const int slots = any ? make_ip_tiles(tab, use, B, T, ip_tile_geom(), ctx->ip_group_tuning, tiles, group) : 0;
    const bool short_form = short_sequences(tab, use, B, T, true);
    if ((long long)slots * kNumXcd > 0x7fffffffLL)
      return fail(ctx, ADLOCO_EUNSUPPORTED, "inner_products: too many tiles for one launch");
    rc = ensure_scratch(ctx, ctx->ip_tab, std::max<size_t>(tiles.size(), 1) * sizeof(int4));
    if (rc) return rc;
    rc = ensure_scratch(ctx, ctx->ip_tile_out,
                        std::max<size_t>(tiles.size(), 1) * group * 2 * tile_waves(short_form) * sizeof(float));
    if (rc) return rc;
    rc = ensure_scratch(ctx, ctx->ip_flags, size_t(n_layers));
    if (rc) return rc;
    ctx->ip_B = ctx->ip_T = -1;
    if (!tiles.empty())
      ADLOCO_HIP_CHECK(ctx, hipMemcpyAsync(ctx->ip_tab.ptr, tiles.data(), tiles.size() * sizeof(int4),
                                           hipMemcpyHostToDevice, st));
    ADLOCO_HIP_CHECK(ctx, hipMemcpyAsync(ctx->ip_flags.ptr, use.data(), size_t(n_layers),
                                         hipMemcpyHostToDevice, st));
    ADLOCO_HIP_CHECK(ctx, hipStreamSynchronize(st));
    std::vector<char> rest(n_layers, 0);
    bool any_rest = false;
    for (int l = 0; l < n_layers; ++l) {
      rest[l] = tab[l].kind == ADLOCO_KIND_LINEAR && !use[l];
      any_rest = any_rest || rest[l];
    }
    if (any_rest) {
      ctx->ip_rest_W = ctx->plain_tiles_tuning ? ctx->plain_tiles_tuning & 3 : plain_tile_width(tab, rest, B, T);
      const TileGeom geom = plain_tile_geom(ctx->ip_rest_W);
      TileList& p = ctx->ip_rest[ctx->ip_rest_W - 1];          // (one per width, which changes from batch to batch)
      if (!p.built || p.use != rest) build_tile_list(ctx, p, tab, rest, geom, false, st);
      if (!p.built) return fail(ctx, ADLOCO_ENOMEM, "inner_products: no memory for the tile list");
      ctx->ip_rest_group = ctx->ip_group_tuning > 0 ? std::min(ctx->ip_group_tuning, B) : run_length(p.n_tiles, B, T, geom);
      if ((long long)p.used(1) * kNumXcd * ((B + ctx->ip_rest_group - 1) / ctx->ip_rest_group) > 0x7fffffffLL)
        return fail(ctx, ADLOCO_EUNSUPPORTED, "inner_products: too many tiles for one launch");
    }
    ctx->ip_any_rest = any_rest;
    ctx->ip_slots = slots;
    ctx->ip_group = group;
    ctx->ip_short = short_form;
    ctx->ip_B = B;
    ctx->ip_T = T;
  }
  const TileList& ip_rest = ctx->ip_rest[ctx->ip_rest_W - 1];
  if (ctx->ip_any_rest) {
    rc = ensure_scratch(ctx, ctx->tile_out, size_t(ip_rest.n_tiles) * B * 2 * sizeof(double));
    if (rc) return rc;
  }
  rc = ensure_scratch(ctx, ctx->ip_dot, size_t(n_layers) * B * sizeof(float));
  if (rc) return rc;
  rc = ensure_scratch(ctx, ctx->ip_sq, size_t(n_layers) * B * sizeof(float));
  if (rc) return rc;
  rc = ensure_scratch(ctx, ctx->sample_f64, size_t(B) * sizeof(double));
  if (rc) return rc;
  const LayerDev* dl = static_cast<const LayerDev*>(ctx->layer_tab.ptr);
  float* dot = static_cast<float*>(ctx->ip_dot.ptr);
  float* sq = static_cast<float*>(ctx->ip_sq.ptr);
  hipEvent_t ev = prof_begin(ctx, st);
  hipError_t e = launch_ip_tiles(dl, ctx->ip_tab.ptr, ctx->ip_slots, T, ctx->ip_group, dtype,
                                 per_sample_sqnorm != nullptr, ctx->ip_short,
                                 static_cast<float*>(ctx->ip_tile_out.ptr), st);
  if (e == hipSuccess && ctx->ip_any_rest)
    e = launch_plain_tiles(dl, ip_rest, 0, B, T, dtype, 0, true, ctx->ip_rest_group,
                           static_cast<double*>(ctx->tile_out.ptr), dot, sq, 1, st);
  if (e == hipSuccess && !ctx->vec_host.empty())
    e = launch_vector_stats(dl, static_cast<const AuxDesc*>(ctx->vec_tab.ptr), int(ctx->vec_host.size()),
                            ctx->vec_blocks, ctx->vec_blocks2, B, T, dtype,
                            static_cast<float*>(ctx->aux_vec.ptr), sq, 1, 0, false, st);
  if (e == hipSuccess && !ctx->emb_host.empty())
    e = launch_embed_stats(dl, static_cast<const AuxDesc*>(ctx->emb_tab.ptr), int(ctx->emb_host.size()),
                           ctx->emb_blocks, B, T, dtype, static_cast<int*>(ctx->aux_perm.ptr),
                           static_cast<double*>(ctx->aux_part.ptr), sq, 1, st);
  if (e == hipSuccess)
    e = launch_ip_vector_table(dl, static_cast<const AuxDesc*>(ctx->vec_tab.ptr), int(ctx->vec_host.size()),
                               static_cast<const AuxDesc*>(ctx->emb_tab.ptr), int(ctx->emb_host.size()),
                               B, T, dtype, static_cast<const float*>(ctx->aux_vec.ptr), dot, st);
  if (e == hipSuccess)
    e = launch_ip_finalize(ctx->ip_tab.ptr, static_cast<const float*>(ctx->ip_tile_out.ptr),
                           (long long)ctx->ip_slots * kNumXcd, ctx->ip_group, tile_waves(ctx->ip_short), dot, sq,
                           static_cast<const unsigned char*>(ctx->ip_flags.ptr), n_layers, B,
                           per_sample_ip, per_sample_sqnorm, static_cast<double*>(ctx->sample_f64.ptr),
                           acc, (flags & ADLOCO_ACCUMULATE) ? 1 : 0, st);
  prof_end(ctx, kProfIp, ev, st);
  if (e != hipSuccess)
    return fail(ctx, ADLOCO_EHIP, "inner_products: launch failed: %s", hipGetErrorString(e));
  return ADLOCO_OK;
}

extern "C" int adloco_inner_product_test(adloco_ctx* ctx, const adloco_linear_desc* layers, int n_layers,
                                         const adloco_stats_acc* acc, const adloco_ip_acc* ip,
                                         double vartheta, double nu, int64_t b_cur, int64_t b_max,
                                         int32_t n_switch, int64_t b_cap, adloco_ip_test_result* out,
                                         void* stream) {
  if (!ctx) return ADLOCO_EINVAL;
  if (!acc || !ip || !out) return fail(ctx, ADLOCO_EINVAL, "inner_product_test: NULL acc, ip or out");
  // S2 exactly as the norm test forms it (also validates the layer list)
  adloco_norm_test_result nt;
  int rc = norm_test(ctx, layers, n_layers, acc, ip, 1.0, b_cur, b_max, n_switch, b_cap, 0, &nt, stream);
  if (rc) return rc;
  adloco_ip_acc h;
  std::memcpy(&h, ctx->pinned + 4, sizeof h);
  if (h.n_samples != nt.n_samples)
    return fail(ctx, ADLOCO_ESTATE, "inner_product_test: the inner products cover %lld samples, the "
                "statistics %lld", (long long)h.n_samples, (long long)nt.n_samples);
  rc = adloco_inner_product_decide(nt.S1, nt.S2, h.sum_ip, h.sum_ip_sq, nt.n_samples, vartheta, nu,
                                   b_cur, b_max, n_switch, b_cap, out);
  if (rc) return fail(ctx, rc, "inner_product_test: decision rejected its arguments");
  return ADLOCO_OK;
}
