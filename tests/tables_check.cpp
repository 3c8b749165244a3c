// Host-only check of the launch tables' argument form (tests/test_tables.py
// builds and runs it; no GPU is touched): every item and split item of a plan
// that fits comes back from its 64-bit word unchanged, the largest value of
// each field included, and a plan with a larger value, more descriptors or
// more words than the form holds is refused (it then goes through the
// workspace).  And of plans in a given workspace: any that holds the tables of
// the uncut 384-row list gets a plan that fits it, with fewer pieces than the
// free choice.  Prints "ok <plans that fit>" on success.
#include "../paper_2609_04774_amd/csrc/cp_attn.cpp"

#include <cstdio>

namespace cpattn {
int launch_partial(const PartialParams&, void*) { return 1; }
int launch_merge(const MergeParams&, void*) { return 1; }
int launch_upload(void*, const void*, size_t, void*) { return 1; }
}  // namespace cpattn

namespace {

int failures = 0;

void expect(bool ok, const char* what) {
  if (!ok && failures++ == 0) std::printf("FAIL %s\n", what);
}

bool same_item(const WorkItem& a, const WorkItem& b) {
  return a.desc == b.desc && a.chunk == b.chunk && a.q_block == b.q_block && a.head_group == b.head_group &&
         (a.t_end < 0) == (b.t_end < 0) && (a.t_end < 0 || (a.t_begin == b.t_begin && a.t_end == b.t_end)) &&
         a.piece == b.piece;
}

// Whether the plan fits; if it does, every word is compared.
bool check(const Plan& plan) {
  InlineTables t;
  const size_t need = plan.descs.size() * sizeof(DevDesc) + 8 * (plan.items.size() + plan.splits.size());
  if (!pack_inline(plan, &t)) return false;
  expect(need <= kInlineBytes && plan.descs.size() <= 32, "a plan beyond the space was taken");
  expect(std::memcmp(t.bytes, plan.descs.data(), plan.descs.size() * sizeof(DevDesc)) == 0, "descriptors");
  const unsigned char* at = t.bytes + plan.descs.size() * sizeof(DevDesc);
  uint64_t x;
  for (const WorkItem& w : plan.items) {
    std::memcpy(&x, at, 8);
    at += 8;
    expect(same_item(item_of_inline(x), w), "work item");
  }
  for (const SplitItem& s : plan.splits) {
    std::memcpy(&x, at, 8);
    at += 8;
    const SplitItem y = split_of_inline(x);
    expect(std::memcmp(&y, &s, sizeof(s)) == 0, "split item");
  }
  return true;
}

}  // namespace

int main() {
  int fit = 0, beyond = 0;
  for (int64_t R : {1, 70, 300, 1024, 3000, 11003})
    for (int64_t P : {0, 16, 4096, 65536})
      for (int C : {1, 2, 4, 8})
        for (int n_descs : {1, 2, 9, 33}) {
          std::vector<cp_partial_desc> d((size_t)n_descs);
          for (auto& x : d) {
            std::memset(&x, 0, sizeof(x));
            make_plan(P, R, C, C - 1, &x.plan);
            void* f = reinterpret_cast<void*>(0x100000);
            x.q = x.k_new = x.v_new = x.k_cache = x.v_cache = f;
            x.o = x.lse = static_cast<float*>(f);
            x.block_table = static_cast<const int32_t*>(f);
            x.n_blocks = 1 << 20;
            x.include_prefix = 1;
            x.kv_rank = CP_KV_ALL;
          }
          Plan plan;
          expect(build_plan(d.data(), n_descs, 8, 2, kTargetPieces, &plan) == CP_OK, "build_plan");
          const size_t need = (size_t)n_descs * sizeof(DevDesc) + 8 * (plan.items.size() + plan.splits.size());
          const bool in = check(plan);
          // No field of these plans is beyond its bits: the space decides.
          expect(in == (n_descs <= 32 && need <= kInlineBytes), "fits by its size");
          ++(in ? fit : beyond);
          const size_t total = layout_of(plan).total;
          Plan least;
          least.descs = plan.descs;
          plan_uncached(8, 2, 0, kRowsLarge, &least);
          const size_t floor = layout_of(least).total;
          for (size_t bytes : {total, total - 1, (total + floor) / 2, floor}) {
            if (bytes < floor) continue;
            Plan part;
            Layout lay;
            size_t wanted = 0;
            expect(build_plan_within(d.data(), n_descs, 8, 2, bytes, &part, &lay, &wanted) == CP_OK, "plan within");
            expect(wanted == total && lay.total <= bytes, "a plan that fits the workspace");
            expect(bytes == total ? part.n_pieces == plan.n_pieces : part.n_pieces <= plan.n_pieces, "fewer pieces");
            check(part);
          }
        }
  expect(fit > 50 && beyond > 50, "both sides of the limit met");
  // The largest value of each field, and one more.
  Plan one;
  one.descs.resize(1);
  std::memset(&one.descs[0], 0, sizeof(DevDesc));
  const WorkItem top{0, 1, kInlineQBlocks - 1, kInlineGroups - 1, kInlineTile - 1, kInlineTile - 1, kInlinePiece - 1, 0};
  const SplitItem stop{0, 1, kInlineQBlocks - 1, kInlineGroups - 1, kInlinePiece - 1, kInlinePieces - 1};
  one.items = {top, WorkItem{0, 0, 0, 0, 0, -1, -1, 0}};
  one.splits = {stop};
  expect(check(one), "largest values");
  for (int f = 0; f < 7; ++f) {
    Plan more = one;
    WorkItem& w = more.items[0];
    SplitItem& s = more.splits[0];
    int32_t* field[] = {&w.q_block, &w.head_group, &w.t_begin, &w.t_end, &w.piece, &s.first_piece, &s.n_pieces};
    ++*field[f];
    expect(!check(more), "a value beyond its bits was taken");
  }
  static_assert((size_t)kMaxPieces < (size_t)kInlinePieces, "pieces of a split item");
  if (failures) return 1;
  std::printf("ok %d\n", fit);
  return 0;
}
