// LOGIT-mode QER scores of bf16 heads (Sec. 3.3, Eqs. 6-7 up to the frame
// mean): qer_strm_kernel, which streams the keys through LDS by DMA, launched
// by the QER driver.
#pragma once

#include "common.h"

namespace cofie {

// One key sequence of a launch over several (cofie_qer_rank_streams) and the
// stacked query rows that read it: its tiles sit at [tile0, tile0 + ntiles)
// of the launch's tile space, side by side with the other sequences'.
struct QerStreamDesc {
  int64_t key0;    // first key row
  int32_t n_keys;  // key rows
  int32_t tile0;   // first tile
  int32_t ntiles;  // ceil(n_keys / 16)
  int32_t q0;      // first stacked query row (of each query term)
  int32_t n_rows;  // query rows (whole queries where there are several)
  int32_t pad;
};

struct StrmArgs {
  const uint8_t* K;          // key rows of row_bytes
  const uint8_t* Q;          // [P][nq_total] query rows of row_bytes
  int64_t row_bytes;         // a multiple of 128 NS
  int32_t nq_total;
  int32_t nseg;              // 128-byte segments per row and contraction slice
  const QerStreamDesc* seq;  // device [n_seq]; null: `one`
  QerStreamDesc one;
  int32_t n_seq;
  int32_t tiles;             // 16-key tiles over all sequences
  int32_t nwg;
  int32_t xcd_order;         // 1: consecutive shares to the workgroups of one XCD (nwg a multiple of 8)
  float scale;
  float* m;                  // m[g * m_stride + key] = scale * max over the rows of query g
  int64_t m_stride;
  int32_t group_rows;        // rows per query (a multiple of 16); 0: one query, row 0 of m
  int32_t accumulate;        // one query: take the max with what m holds
  int32_t* clear;            // workgroup 0 zeroes clear[0, nclear)
  int32_t nclear;
};

// Work split: NS contraction slices, query rows of one launch (a query chunk)
// at most, workgroups.  NS = 0: not this kernel.
struct StrmPlan {
  int NS, max_rows, nwg;
};
// P query terms (1, or 3 for folded grouped heads) of Lc elements, whole
// 128-byte segments, at least two; rows that one launch must take (0: a
// launch may take any part of them -- the plan then depends on the keys only,
// so that queries ranked together or alone add in the same order).
StrmPlan plan_strm(int64_t tiles, int64_t Lc, int P, int rows, int cus);
// Scores of one query chunk per sequence (rows: the widest chunk's).  In a
// dry run, the address model instead.
int launch_strm(const StrmArgs& a, const StrmPlan& p, int P, int rows, hipStream_t s);

}  // namespace cofie
