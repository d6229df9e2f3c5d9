// The query-major scan for shapes without a specialised kernel: scan_kernel with DSUB = 0, one
// instance per number of 16-byte code chunks (1 to 8: up to 128 subspaces).

#include "scan_kernel.h"

namespace ivfpq {

int launch_scan_rt(const ScanArgs &a, const RadiiSq &r2, int64_t grid, bool dump, hipStream_t s) {
  // Tables of at most 32 KiB: four workgroups of 4 wavefronts per CU, as for the specialised shapes,
  // unless the bound on a large k needs the lists of 8.
  const bool four = !(a.wide_cap > 0 && 4 * KP < a.k_out);
  switch ((a.Mp + 15) / 16) {
    case 1: return four ? launch_scan_t<16, 0, 4>(a, r2, grid, dump, s) : launch_scan_t<16, 0, 8>(a, r2, grid, dump, s);
    case 2: return four ? launch_scan_t<32, 0, 4>(a, r2, grid, dump, s) : launch_scan_t<32, 0, 8>(a, r2, grid, dump, s);
    case 3: return launch_scan_t<48, 0, 8>(a, r2, grid, dump, s);
    case 4: return launch_scan_t<64, 0, 8>(a, r2, grid, dump, s);
    case 5: return launch_scan_t<80, 0, 8>(a, r2, grid, dump, s);
    case 6: return launch_scan_t<96, 0, 8>(a, r2, grid, dump, s);
    case 7: return launch_scan_t<112, 0, 8>(a, r2, grid, dump, s);
    default: return launch_scan_t<128, 0, 8>(a, r2, grid, dump, s);
  }
}

}  // namespace ivfpq
