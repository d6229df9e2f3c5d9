// The LDS regions of the inner-product scan for every shape and number of wavefronts: each holds what
// the kernel indexes in it, none reaches into the next, and the last ends within the allocation.
#include <stdio.h>
#include <stdlib.h>

#include "scan_ip_carve.h"

static void need(bool ok, const char *what, int M, int D, int nw) {
  if (ok) return;
  printf("M = %d, D = %d, %d wavefronts: %s\n", M, D, nw, what);
  exit(1);
}

int main() {
  int shapes = 0;
  for (int M = 1; M <= IVFPQ_MAX_M; ++M)
    for (int dsub = 1; dsub <= 100; ++dsub)
      for (int nw = 8; nw <= 16; nw += 8, ++shapes) {
        const int D = M * dsub;
        const IpCarve c = ip_carve(M, D, nw);
        need(c.query >= M * 1024 && c.query >= nw * IP_TOP * 12, "table and staging", M, D, nw);
        need(c.query + D * 4 <= c.queue_id, "query", M, D, nw);
        need(c.queue_id % 8 == 0 && c.queue_id + nw * 64 * 8 <= c.queue_d, "queued ids", M, D, nw);
        need(c.queue_d + nw * 64 * 4 <= c.bounds, "queued distances", M, D, nw);
        need(c.bounds + (1 + nw) * 4 <= c.row0, "bound and ranks", M, D, nw);
        need(c.row0 % 8 == 0 && c.row0 + IP_META * 8 <= c.block0, "first rows", M, D, nw);
        need(c.block0 + IP_META * 8 <= c.len, "first blocks", M, D, nw);
        need(c.len + IP_META * 4 <= c.start && c.start + IP_META * 4 <= c.lower && c.lower + IP_META * 4 <= c.thr, "list metadata", M, D, nw);
        need(c.thr + M * 4 <= c.thr_in && c.thr_in + M * 4 <= c.row_min, "thresholds", M, D, nw);
        need(c.row_min + M * 4 <= c.row_abs && c.row_abs + M * 4 <= c.suffix, "row minima", M, D, nw);
        need(c.suffix + ((M + 7) / 8 + 1) * 4 <= c.end, "suffix sums and the magnitude behind them", M, D, nw);
      }
  printf("ip_carve_driver: %d shapes clean\n", shapes);
  return 0;
}
