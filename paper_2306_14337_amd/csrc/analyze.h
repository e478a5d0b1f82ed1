// Host-side analysis of the first matrix of a same-pattern sequence:
// ordering, pivot sequence, factor patterns, value maps and schedules.
// (Sections 4 and 5.1: symbolic phase plus the first numeric factorization on
// the CPU; its permutations and L/U structures are reused for every later
// system.)
#pragma once
#include <cstdint>
#include <string>
#include <vector>

namespace kktlu {

struct AnalyzeOptions {
  int ordering = 0;       // 0 minimum degree on A+A^T, 1 natural, 2 user-supplied
  double tau = 1e-10;     // threshold partial pivoting
  int matching = 0;       // 1: maximum-product matching and scaling first (match_scale)
};

struct Analysis {
  int32_t n = 0;
  int64_t nnz = 0;
  std::vector<int32_t> Q, Qinv;  // Q[k] = original index of step k
  std::vector<int32_t> P, Pinv;  // P[k] = A'-row pivoted at step k
  // combined factors, CSR in pivot order: L strict part, diagonal, U strict part
  std::vector<int32_t> lu_rowptr;  // n+1
  std::vector<int32_t> lu_col;     // f
  std::vector<int32_t> diag;       // n, position of (i,i)
  std::vector<double> lu_val0;     // values from the pivoting pass
  std::vector<int32_t> lu_src;     // f, index into A's values or -1 (fill)
  // row dependency schedule (refactorization and L solve): rows by level
  std::vector<int32_t> lev_ptr, lev_rows;
  std::vector<int32_t> lev_maxlen;  // longest LU row of each level
  // U-solve schedule
  std::vector<int32_t> ulev_ptr, ulev_rows;
  // transposed views: column-major order of the strict L part and of U, as
  // positions into the CSR arrays (for the transposed solve)
  std::vector<int32_t> ut_ptr, ut_pos;   // column j of U: rows i<=j (diag last)
  std::vector<int32_t> lt_ptr, lt_pos;   // column j of strict L: rows i>j
  std::vector<int32_t> ltlev_ptr, ltlev_rows;  // L^T solve (descending) schedule
  std::vector<int32_t> utlev_ptr, utlev_rows;  // U^T solve (ascending) schedule
  int64_t nnz_l = 0, nnz_u = 0;
  int warn_singular = 0;
  // matching and scaling (empty without): the analysed matrix is
  // Ahat = Pm Dr A Dc, row j of Ahat being row match[j] of A scaled by
  // dr[match[j]] and column c by dc[c]; lu_src and the pivoting pass refer to
  // Ahat's values through A's positions; ascale[p] = dr[i] dc[j] for A's
  // stored entry p = (i, j) (powers of two: the scaled values are exact)
  std::vector<int32_t> match;
  std::vector<double> dr, dc, ascale;
};

// Maximum-product perfect matching of A's nonzero entries and power-of-two
// scaling from the canonical dual potentials (Section 5.2.1's MC64-style
// preprocessing): costs c_ij = log(cmax_j) - log|a_ij|, the minimum-cost
// perfect matching by successive shortest augmenting paths (Dijkstra over
// reduced costs with a binary heap), the largest column potentials v <= 0
// feasible with that matching (shortest distances from a source joined to
// every column, by a queue-based Bellman-Ford), u_i = c_{i,s(i)} - v_{s(i)},
// dr_i = 2^round(u_i / ln 2), dc_j = 2^round((v_j - log cmax_j) / ln 2).
// match[j] = row matched to column j.  Returns KKT_OK or
// KKT_ERR_STRUCTURALLY_SINGULAR (no perfect matching of nonzeros).
int match_scale(int32_t n, const int64_t* rowptr, const int32_t* colind, const double* val,
                std::vector<int32_t>& match, std::vector<double>& dr, std::vector<double>& dc);

// Status codes use the public enum's values.
int validate_csr(int32_t n, int64_t nnz, const int64_t* rowptr, const int32_t* colind,
                 std::string* msg);

// Exact minimum degree on pattern(A + A^T), ties -> smallest index.
void order_minimum_degree(int32_t n, const int64_t* rowptr, const int32_t* colind,
                          std::vector<int32_t>& Q);

// Full analysis.  Returns a kkt_status value; msg gets details on failure.
int analyze(int32_t n, int64_t nnz, const int64_t* rowptr, const int32_t* colind,
            const double* values0, const int32_t* user_q, const AnalyzeOptions& opt,
            Analysis& out, std::string* msg);

// The analysis of Ahat = Pm Dr A Dc for a given matching and scaling (used by
// analyze with opt.matching = 1 and by re-analysis, which keeps them): the
// result describes Ahat's factors with lu_src referring to A's positions and
// match, dr, dc, ascale set.
int analyze_scaled(int32_t n, int64_t nnz, const int64_t* rowptr, const int32_t* colind,
                   const double* values, const std::vector<int32_t>& match,
                   const std::vector<double>& dr, const std::vector<double>& dc,
                   const int32_t* user_q, const AnalyzeOptions& opt, Analysis& out,
                   std::string* msg);

// Batch of independent instances as one block-diagonal system: pattern p
// (n[p], nnz[p], rowptr[p], colind[p], values0[p]) is analysed once (patterns
// in parallel threads) and instance t is a copy of the analysis of pattern
// inst_pattern[t] with its rows and A positions offset; the level schedules
// are merged level by level.  row_off / nnz_off get the instance offsets
// (count + 1 entries).
int analyze_batch(int32_t npat, const int32_t* n, const int64_t* nnz,
                  const int64_t* const* rowptr, const int32_t* const* colind,
                  const double* const* values0, int32_t count, const int32_t* inst_pattern,
                  const AnalyzeOptions& opt, Analysis& out, std::vector<int64_t>& row_off,
                  std::vector<int64_t>& nnz_off, std::string* msg);

// nested[k]: row k + 1's U pattern is row k's without column k + 1.
std::vector<uint8_t> nested_rows(const Analysis& an);

// Per row the longest chain of rows that wait for each other behind it (rows of
// the dense block, c0 and up, do not wait for each other).
std::vector<int32_t> row_heights(const Analysis& an, int32_t c0);

// Rows of one level that do not wait for each other, `rows` of them in each of
// `count` instances, as chunks for workgroups of `waves` waves, of which `slots`
// run at once: the rows per chunk.  spread: the band's rows fit the chip's waves.
// Then a row gets a workgroup (and with it a CU's caches and LDS) for itself, as
// long as the chunks fit the workgroups that run at once; a workgroup of long
// rows may have a CU for itself, and chunks beyond that would come in turn while
// its other waves have nothing to do (refactorization, us, a row a chunk / this
// rule: dense matrices of 700 and 1500 rows 623 / 584 and 1687 / 1374, random ones
// with dense blocks of 1504 and 1888 rows 1108 / 1066 and 1511 / 1437).
// Else a row per wave; wide levels take up to 16 rows per wave and chunk, as a
// ticket counter serializes at about 10 ns per chunk.
int64_t rows_per_chunk(int64_t rows, int64_t count, int waves, int64_t slots, bool spread);

// Row i's first dl pivots as the long-row refactorization takes them: blocks
// (t, p) of pivots t .. t + p - 1 of the row, consecutive rows with nested U
// patterns, at most `most` of them.  run: the first row of the run that row i
// belongs to; the row before it (the run's link) ends a block, if it does not
// form one by itself, and the run's own rows, which their waves hand over in
// LDS, are blocks of one.
// Blocks that start within `most` rows of the link take at most half as many:
// those rows are published one after the other while this row waits.
// Refactorization, us, halves / whole blocks there: 3k buses 382 / 389, 10k 657
// / 670, 30k 1187 / 1208, 70k 2388 / 2403, 32 grids of 500 to 5,000 buses 1272
// / 1276, 128 x 2k 2735 / 2723.  With blocks that stop before the link, which
// then always goes by itself: 400, 669, 1202, 2433, 1300, 2742; with blocks that
// run across it into the run: 419, 664, 1189, 2394, 1327, 2731.
struct LongBlock {
  int32_t t, p;
};
void long_row_blocks(const Analysis& an, const std::vector<uint8_t>& nested, int32_t i, int32_t dl,
                     int32_t run, int32_t most, std::vector<LongBlock>& out);

}  // namespace kktlu
