// Where the inner-product scan kernel keeps what in LDS.  The kernel forms its addresses and the
// launcher sizes the allocation from this one description.
#pragma once

#include <stddef.h>

#include "ivfpq.h"

#if defined(__HIPCC__)
#define IVFPQ_HD __host__ __device__
#else
#define IVFPQ_HD
#endif

constexpr int IP_META = 64;       // probed lists whose metadata is held at a time
constexpr int IP_TOP = 128;       // keys of a wavefront's sorted list

struct IpCarve {   // byte offsets; the table starts at 0 and shares its place with the merge's staging
  int query;       // float [D]
  int queue_id;    // int64 [NW][64]
  int queue_d;     // uint32 [NW][64]
  int bounds;      // uint32: bound, then a rank per wavefront
  int row0;        // int64 [IP_META] first row of a list
  int block0;      // int64 [IP_META] its first code block
  int len;         // int32 [IP_META]
  int start;       // float [IP_META] its term of the scores
  int lower;       // float [IP_META] lower bound on the score of any of its points
  int thr;         // float [IVFPQ_MAX_M] thresholds
  int thr_in;      // float [IVFPQ_MAX_M] ... of the inner sphere
  int row_min;     // float [IVFPQ_MAX_M] smallest value of each table row
  int row_abs;     // float [IVFPQ_MAX_M] largest magnitude of each table row
  int suffix;      // float [IVFPQ_MAX_M / 8 + 2] sums of row_min from every eighth row on, then the sum of row_abs
  int end;
};

IVFPQ_HD constexpr int ip_query_at(int M, int nw) { return M * 1024 > nw * IP_TOP * 12 ? M * 1024 : nw * IP_TOP * 12; }
IVFPQ_HD constexpr int ip_query_bytes(int D) { return (D * 4 + 15) & ~15; }

IVFPQ_HD constexpr IpCarve ip_carve(int M, int D, int nw) {
  IpCarve c = {};
  c.query = ip_query_at(M, nw);
  c.queue_id = c.query + ip_query_bytes(D);
  c.queue_d = c.queue_id + nw * 64 * 8;
  c.bounds = c.queue_d + nw * 64 * 4;
  c.row0 = c.bounds + ((4 * (nw + 1) + 15) & ~15);
  c.block0 = c.row0 + IP_META * 8;
  c.len = c.block0 + IP_META * 8;
  c.start = c.len + IP_META * 4;
  c.lower = c.start + IP_META * 4;
  c.thr = c.lower + IP_META * 4;
  c.thr_in = c.thr + IVFPQ_MAX_M * 4;
  c.row_min = c.thr_in + IVFPQ_MAX_M * 4;
  c.row_abs = c.row_min + IVFPQ_MAX_M * 4;
  c.suffix = c.row_abs + IVFPQ_MAX_M * 4;
  c.end = c.suffix + (IVFPQ_MAX_M / 8 + 2) * 4;
  return c;
}
