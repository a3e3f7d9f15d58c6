// Checks the attention work list of ragged batches (plan.cpp, host code only):
// the items of every row block cover its key tiles exactly once, in order, each
// split with a partial of its own inside its merge group.
// Usage: work_split <iterations> <seed>; prints "ok <plans> cut <n> whole <m> unmerged <k>"
// (cut: plans with a row block in pieces of lengths that differ by more than a tile, which
// equal splits never do; whole: cut plans whose row blocks equal splits would all leave
// whole; unmerged: plans, with extraction plans, that merge nothing, and so run the kernels
// without a merge).
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include <set>
#include <tuple>
#include <vector>
#include "plan.hpp"
using namespace c2kv;
#define CHECK(c) do { if (!(c)) { std::printf("FAIL %s line %d iter %d\n", #c, __LINE__, it); return 1; } } while (0)
// Whether the plan of `batch` requests of 4096 tokens, 4 query heads a kv-head, has row
// blocks merged in the attention kernel.
static bool in_kernel(int batch, int kv_heads, int suffix, int splits, c2kv_dtype dtype) {
  c2kv_attn_cfg cfg{};
  cfg.n_kv_heads = kv_heads;
  cfg.n_q_heads = 4 * kv_heads;
  cfg.head_dim = 128;
  cfg.act_dtype = dtype;
  cfg.rope_base = 1e4;
  c2kv_plan_opts o{};
  o.kv_splits = splits;
  std::vector<int32_t> off, zero(batch, 0), span(batch, 4096), koff, kept;
  std::vector<int64_t> row0(batch, 0);
  for (int b = 0; b <= batch; ++b) { off.push_back(b); koff.push_back(4096 * b); }
  for (int i = 0; i < 4096 * batch; ++i) kept.push_back(i % 4096);
  c2kv_compose_desc d{};
  d.batch = d.n_segments = batch; d.req_seg_off = off.data();
  d.seg_row0 = row0.data(); d.seg_span = span.data(); d.seg_orig_pos0 = zero.data();
  d.seg_kept_off = koff.data(); d.kept_idx = kept.data();
  Plan p;
  std::string err;
  if (build_plan(cfg, d, suffix, &o, p, err) != C2KV_OK) std::abort();
  return p.merge_in_kernel;
}
int main(int argc, char** argv) {
  const int iters = argc > 1 ? atoi(argv[1]) : 300;
  std::mt19937_64 rng(argc > 2 ? atoll(argv[2]) : 1);
  auto U = [&](int lo, int hi) { return std::uniform_int_distribution<int>(lo, hi)(rng); };
  int cut = 0, whole = 0, unmerged = 0, it = -1;
  // few bytes, more bytes, fp32; more than one round in few and in more splits, one round
  CHECK(in_kernel(2, 8, 1, 5, C2KV_BF16) && in_kernel(6, 8, 4, 4, C2KV_BF16));
  CHECK(!in_kernel(5, 8, 4, 5, C2KV_BF16) && !in_kernel(2, 8, 1, 8, C2KV_BF16));
  CHECK(!in_kernel(2, 8, 1, 4, C2KV_F32));
  CHECK(in_kernel(12, 8, 64, 3, C2KV_BF16) && !in_kernel(12, 8, 64, 4, C2KV_BF16));
  CHECK(!in_kernel(8, 8, 64, 3, C2KV_BF16));
  for (it = 0; it < iters; ++it) {
    c2kv_attn_cfg cfg{};
    const int hk[] = {1, 2, 4, 8}, G[] = {1, 3, 4, 8};
    cfg.n_kv_heads = hk[U(0, 3)];
    cfg.n_q_heads = cfg.n_kv_heads * G[U(0, 3)];
    cfg.head_dim = U(0, 1) ? 64 : 128;
    cfg.act_dtype = U(0, 3) == 0 ? C2KV_F32 : C2KV_BF16;
    cfg.rope_base = 1e4;
    c2kv_plan_opts o{};
    const int cus[] = {0, 8, 20, 256};
    o.num_cus = cus[U(0, 3)];
    int B = U(1, 12), S = U(0, 1) ? U(1, 4) : U(5, 300), most = U(0, 3) ? U(1, 6000) : 0;
    // one long request among short ones: more pieces of it than a row block may have
    const bool giant = it % 100 == 99;
    if (giant) { B = 401; S = 1; cfg.n_q_heads = cfg.n_kv_heads = 1; o.num_cus = 256; }
    std::vector<int32_t> req_off(B + 1, 0), span, orig, koff{0}, kept;
    std::vector<int64_t> row0;
    for (int b = 0; b < B; ++b) {
      const int n = giant ? (b ? 100 : 200000) : most ? U(most / 3, most) : 0;
      if (n > 0) {
        row0.push_back(0);
        span.push_back(n);
        orig.push_back(0);
        for (int i = 0; i < n; ++i) kept.push_back(i);
        koff.push_back(int32_t(kept.size()));
      }
      req_off[b + 1] = int32_t(span.size());
    }
    c2kv_compose_desc d{};
    d.batch = B; d.n_segments = int32_t(span.size()); d.req_seg_off = req_off.data();
    d.seg_row0 = row0.data(); d.seg_span = span.data(); d.seg_orig_pos0 = orig.data();
    d.seg_kept_off = koff.data(); d.kept_idx = kept.data();
    Plan p;
    std::string err;
    CHECK(build_plan(cfg, d, S, &o, p, err) == C2KV_OK);

    if (p.merges.empty()) CHECK(!p.merge_in_kernel);
    o.merge_mode = U(0, 2);
    Plan asked;
    CHECK(build_plan(cfg, d, S, &o, asked, err) == C2KV_OK);
    CHECK(asked.merges.size() == p.merges.size());
    if (o.merge_mode > 0)
      CHECK(asked.merge_in_kernel == (o.merge_mode == 1 && !p.merges.empty()));
    // extraction: one item a row block, nothing to merge unless the grid is nearly empty
    const int n_tok = U(64, 700);
    Plan sif;
    CHECK(build_sif_plan(cfg, B, n_tok, U(1, 16), U(0, 20), &o, sif, err) == C2KV_OK);
    CHECK(!(sif.merges.empty() && sif.merge_in_kernel));
    unmerged += p.merges.empty() + sif.merges.empty();

    const int g = cfg.n_q_heads / cfg.n_kv_heads, R = g * S, RB = p.rows_per_block;
    std::map<std::tuple<int, int, int>, std::vector<WorkItem>> blocks;
    for (const auto& w : p.items) blocks[{w.b, w.g, w.row0}].push_back(w);
    CHECK(int64_t(blocks.size()) == int64_t(B) * cfg.n_kv_heads * ((R + RB - 1) / RB));
    std::set<int> partials;
    int shortest = 1 << 30;
    bool uneven = false;
    for (auto& kv : blocks) {
      auto& v = kv.second;
      std::sort(v.begin(), v.end(), [](const WorkItem& x, const WorkItem& y) { return x.tile0 < y.tile0; });
      const int n = p.req_slot0[v[0].b + 1] - p.req_slot0[v[0].b];
      const int rows = std::min(RB, R - v[0].row0), tmax = (v[0].row0 + rows - 1) / g;
      CHECK(v.front().tile0 == 0 && v.back().tile1 == (n + 63) / 64 + (tmax + 64) / 64);
      int lo = 1 << 30, hi = 0;
      for (size_t i = 0; i < v.size(); ++i) {
        CHECK(v[i].nrows == rows && v[i].tile0 < v[i].tile1);
        lo = std::min(lo, v[i].tile1 - v[i].tile0);
        hi = std::max(hi, v[i].tile1 - v[i].tile0);
        if (i) CHECK(v[i].tile0 == v[i - 1].tile1);
        if (v.size() == 1) { CHECK(v[i].partial == -1 && v[i].merge == -1); continue; }
        CHECK(v[i].merge >= 0 && v[i].merge < int(p.merges.size()));
        const MergeGroup& m = p.merges[v[i].merge];
        CHECK(m.b == v[i].b && m.g == v[i].g && m.row0 == v[i].row0 && m.nrows == rows);
        CHECK(m.nsplit == int(v.size()) && m.nsplit <= p.max_splits && m.nsplit <= kMaxSplits);
        CHECK(v[i].partial == m.part0 + (int(i) << m.f32) && v[i].part_f32 == m.f32);
        for (int k = 0; k <= m.f32; ++k) CHECK(partials.insert(v[i].partial + k).second);
      }
      uneven |= hi - lo > 1;
      if (v.size() > 1) shortest = std::min(shortest, lo);
    }
    CHECK(int(partials.size()) == p.n_partials);
    // with at least one row block per slot, equal splits leave all of them whole
    const int cu = o.num_cus > 0 ? o.num_cus : 256;
    if (int(blocks.size()) >= cu * (RB == 64 ? 2 : 1) && !p.merges.empty()) {
      for (const MergeGroup& m : p.merges) CHECK(m.f32 || cfg.act_dtype == C2KV_F32);
      ++whole;
    }
    CHECK(p.part_rows % 16 == 0 && p.part_rows <= RB && p.part_rows >= std::min(R, RB));
    CHECK(p.ws.part_o + size_t(cfg.act_dtype == C2KV_F32 ? 4 : 2) * p.n_partials * p.part_rows *
              cfg.head_dim <= p.ws.part_lse);
    CHECK(p.ws.part_lse + sizeof(float) * size_t(p.n_partials) * p.part_rows <= p.ws.total);
    if (uneven) { CHECK(shortest >= 2); ++cut; }
  }
  std::printf("ok %d cut %d whole %d unmerged %d\n", iters, cut, whole, unmerged);
  return 0;
}
