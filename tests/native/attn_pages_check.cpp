// Host check of the page bases that an attention workgroup stages, compiled
// against the kernel source: for query blocks of new tokens over a prefix that
// need not end on a tile, whole or with their keys in parts, every row that the
// workgroup's tiles load (all keys of a tile that exist, whether the block's
// queries see them or not) lies on a page whose base is staged when the load
// is issued, the refills of a long prefix among them.  Prints "ok <cases>" or
// the first failure.
#include "../../paper_2609_30884_amd/csrc/attn_bf16.hip"

#include <cstdio>

namespace crf {
namespace {

int check(int q_off, int Mq, int ps, int n_splits) {
  const int M = q_off + Mq, nqb = (Mq + BQ - 1) / BQ, all = (M + BKV - 1) / BKV;
  const int split_tiles = (all + n_splits - 1) / n_splits;
  for (int qblk = 0; qblk < nqb; ++qblk) {
    const int last_key = std::min(q_off + (qblk + 1) * BQ, M) - 1, ntiles = last_key / BKV + 1;
    const int needed = attn_pages(last_key, M, ps);
    if (needed > (M - 1) / ps + 1) {
      std::printf("FAIL page past the keys (q_off=%d Mq=%d ps=%d block %d)\n", q_off, Mq, ps, qblk);
      return 1;
    }
    for (int sp = 0; sp < n_splits; ++sp) {
      const int t0 = sp * split_tiles, t1 = std::min(ntiles, t0 + split_tiles);
      int first = t0 * BKV / ps;
      for (int t = t0; t < t1; ++t) {
        // the refill that the load of tile t follows (the first tile's pages are always staged afresh)
        if (t > t0 && (std::min((t + 1) * BKV, M) - 1) / ps >= first + PGCAP) first = t * BKV / ps;
        const int staged = first + std::min(PGCAP, needed - first);
        for (int key = t * BKV; key < std::min((t + 1) * BKV, M); ++key)
          if (key / ps < first || key / ps >= staged) {
            std::printf("FAIL key %d of tile %d not staged (q_off=%d Mq=%d ps=%d splits=%d block %d)\n", key, t, q_off,
                        Mq, ps, n_splits, qblk);
            return 1;
          }
      }
    }
  }
  return 0;
}

}  // namespace
}  // namespace crf

int main() {
  int cases = 0;
  for (int q_off : {0, 1, 63, 64, 300, 2031, 2300, 8003, 9001})
    for (int Mq : {1, 17, 128, 129, 200, 257, 1500})
      for (int ps : {1, 8, 16, 32, 100})
        for (int n_splits : {1, 2, 5, 20}) {
          if (crf::check(q_off, Mq, ps, n_splits)) return 1;
          ++cases;
        }
  std::printf("ok %d\n", cases);
  return 0;
}
