// Pivot blocks of the long-row refactorization (analyze.h: long_row_blocks) on
// the host analysis of random matrices: for every row and every place its run
// could start, the blocks cover the row's pivots in order, hold consecutive
// rows with nested U patterns, and none goes past the row before the run.
// And rows_per_chunk: independent rows share a workgroup where there are more of
// them than workgroups run at once, and only there.
// Prints "ok <blocks of several rows> <blocks that end with the link>".
#include <cstdint>
#include <cstdio>
#include <string>
#include <vector>

#include "../paper_2306_14337_amd/csrc/analyze.h"

namespace {

uint64_t g_state = 0x9E3779B97F4A7C15ull;
double uniform() {
  g_state ^= g_state << 13;
  g_state ^= g_state >> 7;
  g_state ^= g_state << 17;
  return (double)(g_state >> 11) * (1.0 / 9007199254740992.0);
}

int fail(const char* what, int32_t n, int32_t i, int32_t run) {
  std::printf("FAIL %s (n=%d row %d run %d)\n", what, n, i, run);
  return 1;
}

}  // namespace

int main() {
  constexpr int32_t MOST = 8;
  long multi = 0, with_link = 0;
  for (int32_t n : {1, 2, 9, 30, 70}) {
    for (double density : {0.03, 0.1, 0.9}) {
      std::vector<int64_t> rp = {0};
      std::vector<int32_t> ci;
      std::vector<double> v;
      for (int32_t i = 0; i < n; i++) {
        for (int32_t j = 0; j < n; j++)
          if (i == j || uniform() < density) {
            ci.push_back(j);
            v.push_back(uniform() + (i == j ? 4.0 : 0.0));
          }
        rp.push_back((int64_t)ci.size());
      }
      kktlu::AnalyzeOptions opt;
      opt.tau = 1e-10;
      kktlu::Analysis an;
      std::string msg;
      if (kktlu::analyze(n, (int64_t)ci.size(), rp.data(), ci.data(), v.data(), nullptr, opt, an,
                         &msg) < 0)
        return fail(msg.c_str(), n, -1, -1);
      const std::vector<uint8_t> nested = kktlu::nested_rows(an);
      std::vector<kktlu::LongBlock> blocks;
      for (int32_t i = 0; i < n; i++) {
        const int32_t rs = an.lu_rowptr[i], dl = an.diag[i] - rs;
        for (int32_t run = 0; run <= i; run++) {
          kktlu::long_row_blocks(an, nested, i, dl, run, MOST, blocks);
          const int32_t link = run - 1;
          int32_t t = 0;
          for (const kktlu::LongBlock& b : blocks) {
            if (b.t != t || b.p < 1 || b.p > MOST) return fail("not in order", n, i, run);
            t += b.p;
            const int32_t c = an.lu_col[rs + b.t], last = c + b.p - 1;
            if (b.p == 1) continue;
            multi++;
            if (last > link) return fail("a block goes past the link", n, i, run);
            with_link += last == link;
            if (c >= link - MOST && b.p > MOST / 2) return fail("not halved", n, i, run);
            for (int32_t k = c; k < last; k++) {  // row k's U part without k + 1 is row k + 1's
              if (an.lu_col[rs + b.t + (k - c) + 1] != k + 1)
                return fail("rows not consecutive", n, i, run);
              const std::vector<int32_t> up(an.lu_col.begin() + an.diag[k] + 2,
                                            an.lu_col.begin() + an.lu_rowptr[k + 1]);
              const std::vector<int32_t> next(an.lu_col.begin() + an.diag[k + 1] + 1,
                                              an.lu_col.begin() + an.lu_rowptr[k + 2]);
              if (an.lu_col[an.diag[k] + 1] != k + 1 || up != next)
                return fail("patterns not nested", n, i, run);
            }
          }
          if (t != dl) return fail("pivots missing", n, i, run);
        }
      }
    }
  }
  // row_heights against its definition, rows in any order
  {
    std::vector<int64_t> rp = {0};
    std::vector<int32_t> ci;
    std::vector<double> v;
    const int32_t n = 60;
    for (int32_t i = 0; i < n; i++) {
      for (int32_t j = 0; j < n; j++)
        if (i == j || uniform() < 0.04) {
          ci.push_back(j);
          v.push_back(uniform() + (i == j ? 4.0 : 0.0));
        }
      rp.push_back((int64_t)ci.size());
    }
    kktlu::AnalyzeOptions opt;
    opt.tau = 1e-10;
    kktlu::Analysis an;
    std::string msg;
    if (kktlu::analyze(n, (int64_t)ci.size(), rp.data(), ci.data(), v.data(), nullptr, opt, an,
                       &msg) < 0)
      return fail(msg.c_str(), n, -1, -1);
    for (int32_t c0 : {0, 17, 40, n}) {
      std::vector<int32_t> want(n, 0);
      for (int32_t pass = 0; pass < n; pass++)
        for (int32_t i = 0; i < n; i++)
          for (int32_t q = an.lu_rowptr[i]; q < an.diag[i]; q++) {
            const int32_t k = an.lu_col[q];
            if ((k < c0 || i < c0) && want[k] < want[i] + 1) want[k] = want[i] + 1;
          }
      if (kktlu::row_heights(an, c0) != want) return fail("heights", n, c0, 0);
    }
  }
  for (int64_t rows : {1, 7, 255, 256, 257, 672, 1472, 4000, 8192})
    for (int64_t count : {1, 2, 64})
      for (int waves : {1, 4, 8})
        for (int64_t slots : {1, 16, 256, 512, 1280}) {
          const int64_t per = kktlu::rows_per_chunk(rows, count, waves, slots, true);
          if (per < 1 || per > waves) return fail("rows per chunk", (int32_t)rows, waves, 0);
          if (rows * count <= slots && per != 1) return fail("not spread", (int32_t)rows, waves, 0);
          // chunks beyond the workgroups that run at once only if those are full
          if ((rows + per - 1) / per * count > slots + count && per < waves)
            return fail("chunks in turn", (int32_t)rows, waves, (int32_t)slots);
          if (kktlu::rows_per_chunk(rows, count, waves, slots, false) != waves)
            return fail("a row per wave", (int32_t)rows, waves, 0);
        }
  if (kktlu::rows_per_chunk(100000, 1, 4, 256, false) != 4 * 12)
    return fail("wide level", 100000, 4, 0);
  std::printf("ok %ld %ld\n", multi, with_link);
  return 0;
}
