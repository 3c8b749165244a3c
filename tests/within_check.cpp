// Host-only check of plans in a limited workspace (tests/test_planner.py builds
// and runs it; no GPU is touched): of a launch whose free choice does not fit,
// the list that is planned fits, and none of the lists cut to a longest piece,
// and none of the balance cuts, that fit is estimated more than 5 % faster (the
// planner prefers piece slots of 32 MB at up to 4 %); it takes one entry of the
// plan cache and is served from there, for any workspace that holds it up to the
// one it was planned for.  Prints "ok <launches limited>".
#include "../paper_2609_04774_amd/csrc/cp_attn.cpp"

#include <cstdio>

namespace cpattn {
int launch_partial(const PartialParams&, void*) { return 1; }
int launch_merge(const MergeParams&, void*) { return 1; }
int launch_upload(void*, const void*, size_t, void*) { return 1; }
}  // namespace cpattn

namespace {

int failures = 0;

struct Launch {
  int64_t P, R;
  int C, rank, Hq, Hkv;
};

void expect(bool ok, const Launch& l, size_t bytes, const char* what, double a = 0, double b = 0) {
  if (!ok && failures++ < 5)
    std::printf("FAIL P %lld R %lld C %d rank %d heads %d/%d in %zu bytes: %s (%.1f, %.1f)\n", (long long)l.P,
                (long long)l.R, l.C, l.rank, l.Hq, l.Hkv, bytes, what, a, b);
}

cp_partial_desc desc(const Launch& l) {
  cp_partial_desc d;
  std::memset(&d, 0, sizeof(d));
  make_plan(l.P, l.R, l.C, l.rank, &d.plan);
  void* f = reinterpret_cast<void*>(0x100000);
  d.q = d.k_new = d.v_new = d.k_cache = d.v_cache = f;
  d.o = d.lse = static_cast<float*>(f);
  d.block_table = static_cast<const int32_t*>(f);
  d.n_blocks = 1 << 20;
  d.include_prefix = 1;
  d.kv_rank = CP_KV_ALL;
  return d;
}

// The fastest estimate among the lists that fit (infinity: none does).
double fastest_within(const Launch& l, const Plan& launch, size_t bytes) {
  double best = INFINITY;
  for (int rows : {kRowsSmall, kRowsLarge}) {
    const Blocks b = list_blocks(launch.descs, l.Hq, l.Hkv, rows);
    auto consider = [&](int64_t cap) {
      Plan p;
      p.descs = launch.descs;
      plan_items(b, kTargetPieces, false, cap, &p);
      int64_t shortest = kMinPieceTiles;
      for (const WorkItem& w : p.items)
        if (w.piece >= 0) shortest = std::min<int64_t>(shortest, w.t_end - w.t_begin);
      if (shortest < kMinPieceTiles || (cap > 0 && p.n_pieces > kTargetPieces) || layout_of(p).total > bytes) return;
      best = std::min(best, estimate_us(p));
    };
    consider(0);
    for (int64_t k = 1; k <= kMaxPieces && b.max_tiles > 0; ++k) consider((b.max_tiles + k - 1) / k);
  }
  return best;
}

// Whether the limit bound the choice.
bool check(const Launch& l, size_t bytes) {
  const cp_partial_desc d = desc(l);
  Plan plan, again;
  Layout lay;
  size_t wanted = 0;
  g_plan_cache.clear();
  if (build_plan_within(&d, 1, l.Hq, l.Hkv, bytes, &plan, &lay, &wanted) != CP_OK) {
    expect(false, l, bytes, "build_plan_within");
    return false;
  }
  const double best = fastest_within(l, plan, bytes);
  if (lay.total > bytes) {
    expect(best == INFINITY, l, bytes, "refused, but a list fits", (double)lay.total, best);
    return true;
  }
  const double us = estimate_us(plan);
  if (wanted > bytes) expect(us <= 1.05 * best, l, bytes, "estimate, and the fastest that fits", us, best);
  expect(g_plan_cache.size() == 1, l, bytes, "plan cache entries", (double)g_plan_cache.size());
  const size_t hits = g_plan_cache_hits;
  for (size_t same : {bytes, (bytes + lay.total) / 2, lay.total}) {
    build_plan_within(&d, 1, l.Hq, l.Hkv, same, &again, &lay, &wanted);
    expect(again.items.size() == plan.items.size() &&
               std::memcmp(again.items.data(), plan.items.data(), plan.items.size() * sizeof(WorkItem)) == 0,
           l, same, "another list from the cache");
  }
  expect(g_plan_cache_hits == hits + 3, l, bytes, "not served from the plan cache", (double)(g_plan_cache_hits - hits));
  return wanted > bytes;
}

}  // namespace

int main() {
  const size_t scratch = CP_NOALLOC_SCRATCH_BYTES;
  int limited = 0;
  // Launches whose free choice needs more than the scratch of
  // cp_attn_partial_noalloc.
  for (const Launch& l : {Launch{50080, 2414, 4, 2, 32, 8}, Launch{0, 35958, 8, 0, 8, 2}, Launch{126976, 417, 8, 0, 32, 8},
                          Launch{0, 32768, 4, 0, 32, 8}}) {
    expect(check(l, scratch), l, scratch, "a limited plan");
    // A byte less than the free choice needs.
    const cp_partial_desc d = desc(l);
    const size_t full = cp_attn_partial_workspace_size(&d, 1, l.Hq, l.Hkv);
    expect(check(l, full - 1), l, full - 1, "a limited plan");
    expect(!check(l, full), l, full, "the free choice");
  }
  uint64_t rng = 0x9e3779b97f4a7c15ULL;
  auto next = [&](uint64_t n) {
    rng ^= rng << 13;
    rng ^= rng >> 7;
    rng ^= rng << 17;
    return (int64_t)(rng % n);
  };
  const int heads[][2] = {{32, 8}, {64, 8}, {8, 1}, {16, 16}, {8, 2}, {24, 3}};
  for (int i = 0; i < 60; ++i) {
    const int C = 1 << next(4);
    const int* h = heads[next(6)];
    const bool prefix = next(2);
    const Launch l{prefix ? 16 * (int64_t)std::pow(2.0, next(1200) / 100.0) : 0,
                   (int64_t)std::pow(2.0, prefix ? 5 + next(800) / 100.0 : 9 + next(800) / 100.0), C, (int)next(C), h[0], h[1]};
    limited += check(l, scratch);
    limited += check(l, (size_t)std::pow(2.0, 12 + next(1500) / 100.0));
  }
  if (failures) return 1;
  std::printf("ok %d\n", limited);
  return 0;
}
