// Host check of attention launches whose keys are split over workgroups,
// compiled against the kernel source.  The map: every (query head or packed
// group, query block, split) is served by exactly one workgroup, and no XCD has
// more than one workgroup more than another.  The rule: windows and prefixes
// short of twice the new tokens are not split under whole query blocks, no split
// is empty, and the partials fit their buffer.  Prints "ok <cases>" or the first
// failure.
#include "../../paper_2609_30884_amd/csrc/attn_bf16.hip"

#include <cstdio>
#include <vector>

namespace crf {
namespace {

int fail(const char *what, int nq, int nkv, int a, int b) {
  std::printf("FAIL %s (nq=%d nkv=%d %d %d)\n", what, nq, nkv, a, b);
  return 1;
}

int check_map(int nq, int nkv, int nqb, int n_splits, int packed) {
  const int group = nq / nkv, heads = packed ? nkv : nq;
  std::vector<int> cover((size_t)heads * nqb * n_splits, 0);
  int on_xcd[8] = {};
  const int grid = attn_split_grid(nq, nkv, nqb, n_splits, packed);
  for (int bid = 0; bid < grid; ++bid) {
    int head = -1, qblk = -1, split = -1;
    if (!attn_split_block(bid, nq, nkv, nqb, n_splits, packed, head, qblk, split)) continue;
    if (head < 0 || head >= nq || (packed && head % group) || qblk < 0 || qblk >= nqb || split < 0 || split >= n_splits)
      return fail("out of range", nq, nkv, nqb, n_splits);
    ++cover[((size_t)(packed ? head / group : head) * nqb + qblk) * n_splits + split];
    ++on_xcd[bid % 8];
  }
  for (int c : cover)
    if (c != 1) return fail("part not served exactly once", nq, nkv, nqb, n_splits);
  for (int c : on_xcd)
    if (c > on_xcd[7] + 1 || c < on_xcd[7]) return fail("XCDs unevenly loaded", nq, nkv, nqb, n_splits);
  return 0;
}

int check_rule(int nq, int nkv, int Mq, int q_off, int64_t max_splits, int &hits) {
  int packed = -1;
  const int st = attn_split(Mq, q_off, nq, nkv, max_splits, packed);
  if (st == 0) return 0;
  const int ntiles = (q_off + Mq + BKV - 1) / BKV, n = (ntiles + st - 1) / st;
  if (Mq > 16 && (packed || q_off < 2 * Mq)) return fail("whole blocks split without a long prefix", nq, nkv, Mq, q_off);
  if (packed && nq / nkv * Mq > BQ) return fail("packed rows past the block", nq, nkv, Mq, q_off);
  if (n > max_splits || (n - 1) * st >= ntiles) return fail("splits", nq, nkv, Mq, q_off);
  hits += Mq > 16;
  return 0;
}

}  // namespace
}  // namespace crf

int main() {
  using namespace crf;
  const int layouts[][2] = {{12, 2}, {28, 4}, {7, 1}, {8, 8}, {16, 2}, {16, 8}, {12, 6}};
  int cases = 0, hits = 0;
  for (const auto &l : layouts) {
    for (int n_splits : {1, 2, 3, 5, 8, 16, 33})
      for (int nqb = 1; nqb <= 24; ++nqb) {
        if (check_map(l[0], l[1], nqb, n_splits, 0) || (nqb == 1 && check_map(l[0], l[1], 1, n_splits, 1))) return 1;
        ++cases;
      }
    for (int Mq = 1; Mq <= 3000; Mq += Mq < 20 ? 1 : 53)
      for (int q_off : {0, 1, 100, 2031, 4096, 8003, 16384})
        for (int64_t max_splits : {0, 1, 2, 7, 1000}) {
          if (check_rule(l[0], l[1], Mq, q_off, max_splits, hits)) return 1;
          ++cases;
        }
  }
  if (hits < 50) return fail("rule hardly taken", 0, 0, hits, 0);
  std::printf("ok %d\n", cases);
  return 0;
}
