// Host check of attention windows whose long query blocks take their keys in two
// parts, compiled against the kernel source.  The map: every short block of every
// query head is served by exactly one workgroup, every long one by one workgroup
// per part, each XCD serves only the query heads of its KV head.  The rule: it
// names a block only when both parts of every block from there on hold keys, and
// the partials of those rows fit the buffer.  Prints "ok <cases>" or the first
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

int check_map(int nq, int nkv, int nqb, int long0) {
  int xcd_r = 0;
  attn_window_grid(nq, nkv, nqb, xcd_r);
  std::vector<int> cover((size_t)nq * nqb * 2, 0);
  const int grid = attn_halves_grid(nq, nkv, nqb, xcd_r, long0);
  for (int bid = 0; bid < grid; ++bid) {
    int head = -1, qblk = -1, split = -1;
    if (!attn_halves_block(bid, nq, nkv, nqb, xcd_r, long0, head, qblk, split)) continue;
    if (head < 0 || head >= nq || qblk < 0 || qblk >= nqb || split < 0 || split > 1)
      return fail("out of range", nq, nkv, nqb, long0);
    if (head / (nq / nkv) != bid % 8 / xcd_r) return fail("XCD serves another KV head", nq, nkv, nqb, long0);
    ++cover[((size_t)head * nqb + qblk) * 2 + split];
  }
  for (int h = 0; h < nq; ++h)
    for (int b = 0; b < nqb; ++b)
      for (int sp = 0; sp < 2; ++sp)
        if (cover[((size_t)h * nqb + b) * 2 + sp] != (sp == 0 || b >= long0 ? 1 : 0))
          return fail("part not served exactly once", nq, nkv, nqb, long0);
  return 0;
}

int check_rule(int nq, int nkv, int hd, int Mq, int q_off, int64_t cap, int &hits) {
  const int nqb = (Mq + BQ - 1) / BQ;
  int st = 0;
  const int long0 = attn_halves(Mq, q_off, nq, nqb, hd, cap, st);
  if (long0 < 0) return 0;
  ++hits;
  if (long0 >= nqb || st < 16) return fail("rule range", nq, nkv, Mq, q_off);
  if (2 * (int64_t)nq * (Mq - long0 * BQ) * (hd + 4) > cap) return fail("partials exceed their buffer", nq, nkv, Mq, q_off);
  for (int b = long0; b < nqb; ++b) {
    const int last_key = q_off + std::min((b + 1) * BQ, Mq) - 1;
    if (last_key / BKV + 1 <= st) return fail("second part empty", nq, nkv, Mq, q_off);
  }
  return 0;
}

}  // namespace
}  // namespace crf

int main() {
  using namespace crf;
  const int layouts[][2] = {{28, 4}, {12, 2}, {4, 2}, {8, 8}, {16, 8}, {6, 1}, {32, 8}, {7, 1}};
  int cases = 0, hits = 0;
  for (const auto &l : layouts) {
    for (int nqb = 1; nqb <= 70; ++nqb)
      for (int long0 = 0; long0 < nqb; long0 += 1 + nqb / 9) {
        if (check_map(l[0], l[1], nqb, long0)) return 1;
        ++cases;
      }
    for (int hd : {64, 128})
      for (int Mq = 1; Mq <= 20000; Mq += 61)
        for (int q_off : {0, 1, 640, 9001})
          for (int64_t cap : {(int64_t)512 * 128 * (hd + 4), (int64_t)1 << 20, (int64_t)0}) {
            if (check_rule(l[0], l[1], hd, Mq, q_off, cap, hits)) return 1;
            ++cases;
          }
  }
  if (hits < 100) return fail("rule never taken", 0, 0, hits, 0);
  std::printf("ok %d\n", cases);
  return 0;
}
