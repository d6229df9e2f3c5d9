// C ABI of the library: argument validation, index construction, workspace
// planning and the entry points declared in include/ivfpq.h.  No kernel lives
// here; every step of the search path runs in coarse.hip / scan.hip.

#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <atomic>
#include <new>
#include <vector>

#include "ivfpq_internal.h"

namespace ivfpq {

static thread_local char g_err[512] = "";

void set_error(const char *fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof g_err, fmt, ap);
  va_end(ap);
}

int hip_fail(hipError_t e, const char *what) {
  set_error("HIP error %d (%s) in %s", (int)e, hipGetErrorString(e), what);
  return IVFPQ_ERR_HIP;
}

static size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// budget == 0: the proposal matrix of the filtering stage takes up to 1 GiB (queries are
// processed in chunks of q_chunk).  budget > 0: everything must fit in `budget` bytes; the
// chunk shrinks (in steps of 128 queries) to make it fit, and total = SIZE_MAX says that not
// even the smallest chunk does.
Workspace plan_workspace(const ivfpq_index *ix, int64_t Q, int32_t nprobe, int32_t k, size_t budget) {
  (void)k;
  Workspace w;
  memset(&w, 0, sizeof w);
  w.nlist_pad = (ix->nlist + 63) & ~63;
  // enough workgroups to fill 256 CUs a few times over when the batch is small
  int64_t ns = Q > 0 ? (2048 + Q - 1) / Q : 1;
  if (ns > nprobe) ns = nprobe;
  if (ns > 64) ns = 64;
  if (ns < 1) ns = 1;
  w.nsplit = (int32_t)ns;
  size_t fixed = 2 * align256((size_t)Q * nprobe * 4) + align256((size_t)Q * 4);
  if (w.nsplit > 1) fixed += align256((size_t)Q * w.nsplit * 128 * 4) + align256((size_t)Q * w.nsplit * 128 * 8);
  // scratch of the filtering stage per query: a row of the product, or (many lists) the keys
  // the product keeps plus a sixteenth of a row for the queries that need every distance
  const int32_t nkeys = coarse_fused_keys(ix->nlist, nprobe, ix->D);
  const size_t row_bytes = nkeys > 0 ? (size_t)nkeys * 4 + (size_t)w.nlist_pad / 4 + 1 : (size_t)w.nlist_pad * 4;
  int64_t qc = ((int64_t)1 << 30) / (int64_t)row_bytes;
  qc &= ~(int64_t)127;
  if (qc < 128) qc = 128;
  if (budget > 0) {
    const size_t spare = 256 + (nkeys > 0 ? (size_t)(FB_SLOTS + 1) * w.nlist_pad * 4 + 1024 : 0);   // fixed part and rounding of the scratch size
    const int64_t fit = fixed + spare <= budget ? (int64_t)((budget - fixed - spare) / row_bytes) : 0;
    if (fit < qc) qc = fit >= Q ? fit : (fit & ~(int64_t)127);
    if (qc < 1 || (qc < 128 && qc < Q)) {
      w.total = SIZE_MAX;
      return w;
    }
  }
  if (qc > Q) qc = Q;
  w.q_chunk = qc < 1 ? 1 : qc;
  size_t off = 0;
  w.coarse_dist = off; off += align256(coarse_scratch_floats(w.nlist_pad, nkeys, w.q_chunk) * 4);
  w.probe_ids = off;   off += align256((size_t)Q * nprobe * 4);
  w.probe_dist = off;  off += align256((size_t)Q * nprobe * 4);
  w.coarse_flags = off; off += align256((size_t)Q * 4);
  if (w.nsplit > 1) {
    w.part_d = off;    off += align256((size_t)Q * w.nsplit * 128 * 4);
    w.part_id = off;   off += align256((size_t)Q * w.nsplit * 128 * 8);
  }
  w.total = off;
  return w;
}

static std::atomic<int> g_wide_cap{8192};  // slots per query of the wide selection

void set_wide_cap(int v) { g_wide_cap.store(v, std::memory_order_relaxed); }

WideWorkspace plan_wide(const ivfpq_index *ix, int64_t Q, int32_t k, int32_t mode) {
  WideWorkspace w = {};
  if (ix->metric != IVFPQ_METRIC_L2 || mode != 0 || k <= 128 || k > 8 * 128 || Q < 1) return w;
  w.cap = g_wide_cap.load(std::memory_order_relaxed);
  if (w.cap == 0) return w;  // switched off: pass by pass
  // the slot arrays take at most 1 GiB: larger batches go through them in chunks
  int64_t qc = ((int64_t)1 << 30) / ((int64_t)w.cap * 12);
  if (qc < 1024) qc = 1024;
  w.q_chunk = qc < Q ? qc : Q;
  auto a256 = [](size_t v) { return (v + 255) & ~(size_t)255; };
  size_t off = 0;
  w.d = off;     off += a256((size_t)w.q_chunk * w.cap * 4);
  w.id = off;    off += a256((size_t)w.q_chunk * w.cap * 8);
  w.n = off;     off += a256((size_t)w.q_chunk * 4);
  w.bound = off; off += a256((size_t)w.q_chunk * 4);
  w.qmap = off;  off += a256((size_t)w.q_chunk * 4);
  w.total = off;
  return w;
}

// Lists of the list-major wide selection's first stage: as many as hold 2 k points on average.  0 where it does not
// serve: shapes without list-major kernels, few pairs or long lists (the lines of the list-major scan), slots that
// do not hold twice the first lists (those near a query are longer than the mean) or so few that the stages crawl,
// and batches too small for the stages' twenty launches against clustered data, whose k neighbours the query-major scan
// finds in a part of the nearest list.  us of a search, query-major / in stages, clustered data and data without structure:
//   points a list, k, queries     48 subspaces                  64 subspaces                  16 subspaces
//   977    129     512            97 / 135,   339 / 247         92 / 124,   391 / 258         75 / 124,   274 / 204
//          129    1024           135 / 148,   586 / 326        143 / 142,   672 / 347         99 / 140,   337 / 259
//          129    2048           222 / 187,  1102 / 493        228 / 188,  1283 / 542        165 / 180,   618 / 379
//          129    8192           707 / 498,  4128 / 1511       739 / 518,  4785 / 1727       520 / 471,  2138 / 1118
//          300     512           140 / 151,   371 / 273        106 / 130,   393 / 278         83 / 131,   300 / 233
//          300    1024           193 / 170,   655 / 357        159 / 149,   715 / 371        111 / 150,   381 / 294
//         1000     512           496 / 336,   527 / 382        555 / 370,   575 / 388        402 / 285,   451 / 339
//   3906   129    2048           283 / 309,  2620 / 788        303 / 336,  3348 / 938        215 / 254,  1138 / 515
//          129    4096           512 / 534,  5115 / 1442       560 / 596,  6496 / 1743       367 / 438,  2137 / 955
//          300    2048           325 / 342,  2677 / 824        340 / 352,  3407 / 951        252 / 270,  1232 / 552
//         1000     512           201 / 245,   845 / 465        193 / 213,  1016 / 489        177 / 192,   543 / 376
//         1000    2048           512 / 441,  2940 / 1020       507 / 436,  3500 / 1116       452 / 350,  1765 / 742
//   244    129     512           765 / 155,   855 / 270        798 / 148,   946 / 287        214 / 138,   251 / 239
//          300    8192          1145 / 1101                   1234 / 1224                    833 / 976,  4364 / -
// (32 probes.)  The line is where clustered data pays a tenth at most; without structure the stages take a half to a quarter.
static int32_t wide_first(const ivfpq_index *ix, const WideWorkspace &w, int32_t nprobe, int32_t k, int32_t strategy) {
  const int64_t Q = w.q_chunk;
  if (strategy == IVFPQ_SCAN_QUERY_MAJOR || !byte_table_shape(ix)) return 0;
  if (Q * (int64_t)nprobe < 16384 || ix->N > (int64_t)4096 * ix->nlist || ix->N < (int64_t)ix->nlist * 128) return 0;
  if (ix->max_list_len >= (1 << 20) || Q * (int64_t)nprobe > 0x3FFFFFFFll) return 0;
  const bool few = 2 * (int64_t)k * ix->nlist < ix->N;   // neighbours against the points of a list
  const double share = (double)Q * k * ix->nlist / (double)ix->N;
  if (share < (few && ix->M > 16 ? 128.0 : 240.0)) return 0;
  if (few && (Q < (ix->M > 16 ? 1024 : 2048) || (ix->M == 16 && 8 * (int64_t)k * ix->nlist < ix->N))) return 0;
  const int64_t first = (2 * (int64_t)k * ix->nlist + ix->N - 1) / ix->N;
  if (first * 2 > nprobe || first * 2 * ix->N > (int64_t)w.cap * ix->nlist) return 0;
  int stages = 1;
  for (int32_t p = (int32_t)first; p < nprobe; ++stages) {
    const int32_t next = wide_next(w, k, p, nprobe);
    if (next == p || stages == LM_STAGES) return 0;
    p = next;
  }
  return (int32_t)first;
}

WideWorkspace plan_wide(const ivfpq_index *ix, int64_t Q, int32_t nprobe, int32_t k, int32_t mode, int32_t strategy) {
  WideWorkspace w = plan_wide(ix, Q, k, mode);
  if (w.total == 0) return w;
  w.first = wide_first(ix, w, nprobe, k, strategy);
  w.lm_off = w.total;
  if (w.first > 0) {
    w.lm.first = w.first;
    w.lm.cap = w.cap;
    plan_list_major_tables(w.lm, ix->nlist, w.q_chunk, nprobe);
    w.total += w.lm.total;
  }
  return w;
}

static int check_common(const ivfpq_index *ix, const void *q, int64_t Q, int32_t nprobe, const char *fn) {
  if (!ix) { set_error("%s: index is NULL", fn); return IVFPQ_ERR_INVALID_ARGUMENT; }
  if (Q < 0) { set_error("%s: Q = %lld is negative", fn, (long long)Q); return IVFPQ_ERR_INVALID_ARGUMENT; }
  if (Q > 0 && !q) { set_error("%s: queries pointer is NULL", fn); return IVFPQ_ERR_INVALID_ARGUMENT; }
  if ((uintptr_t)q % 16) { set_error("%s: queries pointer must be 16-byte aligned", fn); return IVFPQ_ERR_INVALID_ARGUMENT; }
  if (Q > 0) {  // the index lives on one device; the kernels would fault on another one's pointers
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) (void)hipGetLastError();
    else if (dev != ix->device) {
      set_error("%s: the index was created on device %d, the current device is %d", fn, ix->device, dev);
      return IVFPQ_ERR_INVALID_ARGUMENT;
    }
  }
  if (nprobe < 1 || nprobe > ix->nlist) {
    set_error("%s: nprobe = %d outside [1, nlist = %d]", fn, nprobe, ix->nlist);
    return IVFPQ_ERR_INVALID_ARGUMENT;
  }
  if (nprobe > IVFPQ_MAX_NPROBE) {
    set_error("%s: nprobe = %d above the limit %d", fn, nprobe, IVFPQ_MAX_NPROBE);
    return IVFPQ_ERR_UNSUPPORTED;
  }
  return IVFPQ_OK;
}

// nearest bf16, ties to even; infinities and NaN keep their upper half (a NaN its payload's top bit)
static uint16_t bf16_bits(float x) {
  uint32_t u;
  memcpy(&u, &x, 4);
  if ((u & 0x7F800000u) == 0x7F800000u) return (uint16_t)((u >> 16) | ((u & 0x7FFFFFu) ? 0x40u : 0u));
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

static int check_k(int32_t k, const char *fn) {
  if (k < 1) { set_error("%s: k = %d must be positive", fn, k); return IVFPQ_ERR_INVALID_ARGUMENT; }
  if (k > IVFPQ_MAX_K) { set_error("%s: k = %d above the limit %d", fn, k, IVFPQ_MAX_K); return IVFPQ_ERR_UNSUPPORTED; }
  return IVFPQ_OK;
}

static int make_radii(const ivfpq_index *ix, const float *radii, RadiiSq *out, const char *fn) {
  if (!radii) { set_error("%s: radii pointer is NULL", fn); return IVFPQ_ERR_INVALID_ARGUMENT; }
  memset(out, 0, sizeof *out);
  for (int m = 0; m < ix->M; ++m) {
    const float r = radii[m];
    if (!(r >= 0.0f)) {  // catches NaN and negatives
      set_error("%s: radii[%d] = %g must be >= 0 (or +inf)", fn, m, (double)r);
      return IVFPQ_ERR_INVALID_ARGUMENT;
    }
    out->v[m] = r * r;  // fp32 product; +inf stays +inf
  }
  return IVFPQ_OK;
}

static int check_workspace(const Workspace &w, const void *ws, size_t bytes, const char *fn) {
  if (w.total == 0) return IVFPQ_OK;
  if (!ws) { set_error("%s: workspace pointer is NULL (%zu bytes needed)", fn, w.total); return IVFPQ_ERR_WORKSPACE; }
  if ((uintptr_t)ws % 256) { set_error("%s: workspace must be 256-byte aligned", fn); return IVFPQ_ERR_WORKSPACE; }
  if (bytes < w.total) { set_error("%s: workspace has %zu bytes, %zu needed", fn, bytes, w.total); return IVFPQ_ERR_WORKSPACE; }
  return IVFPQ_OK;
}

// Queries that go through the list-major scan together.  Where AUTO takes it on long lists, and on shapes without byte tables
// whichever way it is asked for, it serves calls that the query-major scan serves with a few KiB of workspace a query: there
// the candidates' slots (up to 128 KiB a query) take 1 GiB at most, 2 GiB on those shapes (16 384 queries of 64 probes), or
// what 4096 queries want of them; larger batches go through them in pieces.  Anywhere else all queries of the call.
static int64_t lm_together(const ivfpq_index *ix, int64_t Q, int32_t nprobe, int32_t requested) {
  if (byte_table_shape(ix) && (requested == IVFPQ_SCAN_LIST_MAJOR || ix->N <= (int64_t)4096 * ix->nlist)) return Q;
  const int64_t room = (int64_t)1 << (byte_table_shape(ix) ? 30 : 31);
  int64_t fit = room / ((int64_t)plan_list_major(ix, 1, nprobe).cap * 8) & ~(int64_t)63;
  if (fit < 4096) fit = 4096;
  return Q < fit ? Q : fit;
}

constexpr int64_t LM_ALWAYS = 16384;   // (query, list) pairs

// Which way stages 2-4 run.  A request for the list-major scan is honoured where that scan is
// built (L2, k <= 128, the specialised shapes), anything else runs query-major.  Left to the
// library (AUTO), the list-major scan serves batches with enough (query, list) pairs to group,
// over indexes whose lists are short: there the per-query fixed costs of the query-major
// kernel dominate, while long lists (the 100M-point configuration) gain more from its
// per-block pruning.  Measured: faster on every 1M-point workload and on the 10M-point one,
// four times slower on the 100M-point one.
static bool use_list_major(const ivfpq_index *ix, int64_t Q, int32_t nprobe, int32_t k, int32_t mode,
                           int32_t requested) {
  if (requested == IVFPQ_SCAN_QUERY_MAJOR || !list_major_supported(ix, nprobe, k)) return false;
  if (!byte_table_shape(ix) && mode != IVFPQ_SCORE_DISTANCE) return false;   // (the hit counts' byte tables serve them query-major)
  if (requested == IVFPQ_SCAN_LIST_MAJOR) return true;
  const int64_t pairs = Q * (int64_t)nprobe;
  if (pairs < LM_ALWAYS) {
    // Fewer pairs pay where all lists fit the head pass: a query whose nearest list does not has a workgroup to itself for
    // all of its lists (two components a list, 64 queries, 64 subspaces 156 / 528 us, 100 subspaces 400 / 1436).  us of a search of 32
    // probes, query-major / list-major, otherwise:
    //   queries                               64           128           200           300           450
    //   64 subspaces, clustered          86 / 53       87 / 54       91 / 55      102 / 65      100 / 72
    //   48, clustered                    77 / 49       79 / 50       82 / 50       95 / 58       95 / 64
    //   48, without structure          153 / 160     182 / 196     229 / 216     296 / 238     382 / 275
    //   48, hit counts                 171 / 148     215 / 177     266 / 187     332 / 211     411 / 237
    //   16, clustered                    87 / 44       76 / 45       75 / 47       74 / 48       76 / 58
    //   100, clustered                   78 / 76      86 / 105      93 / 106     123 / 111     133 / 113
    // So it does from 8 probes on (16 subspaces, 1000 queries of 4: 51 / 55) and while the k nearest and a few more fit the head
    // pass' 128 keys: beyond, ties of the histogram's bins leave queries over, which are redone (64 subspaces, 300 queries, k = 128:
    // 104 / 112, k = 100 104 / 66; of random calls with k = 112 and radii that hold nine tenths of the entries, half lose).
    // With 16 subspaces the query-major scan is cheap, and calls whose bound lets many of a list's points through pay for their
    // candidates (without structure, 128, 256 and 510 queries, lists of 976, k = 10 107 / 80, 125 / 91, 190 / 123; k = 100 122 / 136,
    // 145 / 173, 216 / 218; lists of 390, k = 100 106 / 125, 121 / 162, 178 / 210; lists of 2000 gain), and so do hit counts of few
    // queries, which the query-major scan splits over workgroups (162 queries, k = 100 286 / 617).
    // With 48 and 64 subspaces lists of 8 k points are asked for: on shorter ones the k-th distance over the nearest list rules
    // out little (64 subspaces, k = 100, 166 queries of 57 probes, lists of 330 without structure 234 / 486, 473 of 16, clustered lists
    // of 688 97 / 144; 48, 470 of 16, lists of 510 223 / 296; of 30 random calls on such lists with 64 subspaces a quarter lose).
    // Over 5600 random calls between the lines and LM_ALWAYS, query-major over list-major as a geometric mean, least, and how many of 100
    // are below 0.95, radii that hold a tenth to half of the entries: 16 subspaces 1.38, 0.89, 1; its hit counts 1.47, 0.91, none; 48
    // 1.64, 0.79, 1, hit counts 1.64, 0.92, 1; 64 1.61, 0.54 (lists of a few hundred points, k = 100), 3, hit counts 1.74, 0.87, 1; 73
    // and more 1.96, 0.61 (clustered data, 64 probes), 2.  Radii that hold nine tenths: distances 1.3 to 1.6, 0.40, 2 to 11; hit counts
    // 16 subspaces 1.16, 0.42, 27, 48 and 64 1.6, 0.82, 1.  (Taken before 8 k was asked for.)
    if (nprobe < 8 || k > 100) return false;
    if (pairs < (ix->M == 16 ? 4096 : byte_table_shape(ix) ? 6144 : 9600)) return false;
    if (mode == IVFPQ_SCORE_DISTANCE && !head_pass_holds_all(ix)) return false;
    if (ix->M == 16 && !(mode == IVFPQ_SCORE_DISTANCE ? ix->N >= (int64_t)16 * k * ix->nlist : (k <= 64 && Q >= 256 && pairs >= 6144))) return false;
    if (ix->M != 16 && byte_table_shape(ix) && mode == IVFPQ_SCORE_DISTANCE && ix->N < (int64_t)8 * k * ix->nlist) return false;
    return ix->N <= (int64_t)4096 * ix->nlist;
  }
  // 73 subspaces and more: no byte tables for the head pass on long lists, and lists that it does not hold pay where they are
  // short on average and the queries many, or the queries very many.  100 subspaces, two components a list, query-major / list-major: 617
  // queries, lists of 2113 2674 / 3527 us, 1000, 977 5022 / 4114, 4000, 977 19 661 / 10 471; such lists of 1024 points on average at
  // most, random calls of fewer than 1024 queries: 0.94 times as fast, two thirds of them lose (75 x 3, 800 queries of 43
  // probes 1799 / 2268; 121 x 2, 392 of 80 629 / 1152), 1024 to 4096 1.3 times, one in 40.  k <= 112: the head pass ranks 128 keys, and beyond 112
  // the ties of the histogram's bins leave queries over on any kind of data, which are redone (k = 128, 69 random calls: 0.89 times as
  // fast, two thirds lose, 100 subspaces, 205 queries of 82 probes 107 / 218; k = 112, 76 calls: 1.62 times, one in nine loses; up
  // to 100 1.8 times, 4 of 100).  Of 760 random calls that these lines let through 4 of 100 lose, the least 0.68, nearly all of them where
  // the radii hold nine tenths of the entries; 1.8 times as fast as a geometric mean.
  if (!byte_table_shape(ix)) {
    if (k > 112) return false;
    return ix->N <= (int64_t)4096 * ix->nlist && (head_pass_holds_all(ix) || Q >= (ix->N <= (int64_t)1024 * ix->nlist ? 1024 : 4096));
  }
  if (ix->N <= (int64_t)4096 * ix->nlist) return true;
  // Longer lists: the query-major scan prunes block by block, the list-major one shares each pass over a list among the
  // queries that probe it.  Distances only (the hit counts' first lists are ranked query-major either way).  Query-major /
  // list-major, us, k = 100, 64 probes, 64 subspaces of clustered data unless said:
  //   queries                          512         1024         2048         4096          8192
  //   lists of 5000              149 / 271    257 / 295    315 / 351    590 / 492    1145 / 791
  //   7812                       358 / 550    540 / 706    898 / 810   1272 / 1052   2123 / 1570
  //   15 625 (32 probes)         776 / 994  1241 / 1156  1860 / 1577   3567 / 2305   6247 / 3728
  //   5000, two components a list
  //                             1301 / 858  2509 / 1425  5184 / 2370   9609 / 4285  18753 / 8297
  //   5000, 48 subspaces without structure
  //                             2210 / 883  4209 / 1281  7886 / 1905  15441 / 3312  30708 / 6035
  // and by shape and by the share of the entries that the radii hold, lists of 7812, k = 100 (another index: 512 lists):
  //   queries                                       2048              4096              8192
  //   64 subspaces, clustered, 0.25            381 / 415         721 / 581        1437 / 978
  //   64, clustered, 0.9                       382 / 578         724 / 814        1439 / 1343
  //   48, clustered, 0.25                      330 / 336         627 / 497        1220 / 772
  //   48, clustered, 0.9                       330 / 495         625 / 672        1220 / 1000
  //   16, clustered, 0.25                      245 / 370         448 / 505         856 / 774
  //   16, clustered, 0.9                       245 / 357         448 / 501         856 / 763
  //   16, components that touch, 0.25         3441 / 884        6421 / 1562      12199 / 2937
  //   64, without structure, 0.25            11512 / 2223      22336 / 4117      44167 / 7953
  //   48, without structure, 0.25             9529 / 1877      18205 / 3384      35900 / 6408
  //   16, without structure, 0.25             3472 / 1001       6726 / 1700      13090 / 3098
  // The line is where clustered data whose radii hold a part of the entries breaks even with 48 and 64 subspaces; with 16,
  // and with radii that hold nearly everything, such data pays up to half there and gains from 8192 queries on, and any
  // other data takes a third to a fifth of the time all the way (which a caller knows, and can ask for either way).
  // Two queries a list at least.  (100M points in 16 384 lists, fewer than one
  // query a list, the nearest ones eight times the mean: query-major.)  What counts are the queries that go together.
  const int64_t together = lm_together(ix, Q, nprobe, requested);
  return mode == IVFPQ_SCORE_DISTANCE && ix->N <= (int64_t)16384 * ix->nlist && together >= (int64_t)2 * ix->nlist &&
         (double)together * (double)ix->N / ix->nlist >= 1.6e7 && ix->max_list_len < (1 << 20);
}

}  // namespace ivfpq

using namespace ivfpq;

extern "C" {

const char *ivfpq_last_error(void) { return g_err; }

int ivfpq_set_option(const char *name, int value) {
  if (name && !strcmp(name, "scan_waves")) {
    if (value != 0 && value != 4 && value != 8 && value != 16) {
      set_error("set_option: scan_waves must be 0, 4, 8 or 16");
      return IVFPQ_ERR_INVALID_ARGUMENT;
    }
    set_scan_waves(value);
    return IVFPQ_OK;
  }
  if (name && !strcmp(name, "scan_ablate")) {
    if (value & ~(8 | 16 | 32 | 64 | 128)) {
      set_error("set_option: scan_ablate accepts the bits 8, 16, 32, 64 and 128 only");
      return IVFPQ_ERR_INVALID_ARGUMENT;
    }
    set_scan_ablate(value);
    return IVFPQ_OK;
  }
  if (name && !strcmp(name, "scan_loads")) {
    if (value < 0 || value > 3) { set_error("set_option: scan_loads must be 0, 1, 2 or 3"); return IVFPQ_ERR_INVALID_ARGUMENT; }
    set_scan_variant(value);
    return IVFPQ_OK;
  }
  if (name && !strcmp(name, "lm_first")) {
    if (value < 1 || value > 64) { set_error("set_option: lm_first must be in [1, 64]"); return IVFPQ_ERR_INVALID_ARGUMENT; }
    set_lm_first(value);
    return IVFPQ_OK;
  }
  if (name && !strcmp(name, "lm_cap")) {
    if (value != 0 && (value < 64 || value > 65536)) { set_error("set_option: lm_cap must be 0 or in [64, 65536]"); return IVFPQ_ERR_INVALID_ARGUMENT; }
    set_lm_cap(value);
    return IVFPQ_OK;
  }
  if (name && !strcmp(name, "bound_grid")) {
    if (value < 0 || value > 2) { set_error("set_option: bound_grid must be 0, 1 or 2"); return IVFPQ_ERR_INVALID_ARGUMENT; }
    set_bound_grid(value);
    return IVFPQ_OK;
  }
  if (name && !strcmp(name, "wide_cap")) {
    if (value != 0 && (value < 1024 || value > 65536)) { set_error("set_option: wide_cap must be 0 or in [1024, 65536]"); return IVFPQ_ERR_INVALID_ARGUMENT; }
    set_wide_cap(value);
    return IVFPQ_OK;
  }
  set_error("set_option: unknown option");
  return IVFPQ_ERR_INVALID_ARGUMENT;
}

int64_t ivfpq_coarse_fallbacks(int reset) {
  unsigned int n = 0;
  const int rc = coarse_fallbacks(reset, &n);
  return rc == IVFPQ_OK ? (int64_t)n : (int64_t)rc;
}

void ivfpq_index_destroy(ivfpq_index *ix) {
  if (!ix) return;
  (void)hipFree(ix->d_centroids);
  (void)hipFree(ix->d_cnorm);
  (void)hipFree(ix->d_csplit);
  (void)hipFree(ix->d_box);
  (void)hipFree(ix->d_cb_split);
  (void)hipFree(ix->d_grid);
  (void)hipFree(ix->d_grid_par);
  (void)hipFree(ix->d_codebooks);
  (void)hipFree(ix->d_list_offsets);
  (void)hipFree(ix->d_list_blocks);
  (void)hipFree(ix->d_codes);
  (void)hipFree(ix->d_ids);
  delete ix;
}

int ivfpq_index_create(const ivfpq_index_desc *d, ivfpq_index **out) {
  const char *fn = "index_create";
  if (!d || !out) { set_error("%s: NULL argument", fn); return IVFPQ_ERR_INVALID_ARGUMENT; }
  *out = nullptr;
  if (d->ksub != IVFPQ_KSUB) { set_error("%s: ksub = %d, only 256 is supported", fn, d->ksub); return IVFPQ_ERR_UNSUPPORTED; }
  if (d->N < 0 || d->D < 1 || d->nlist < 1 || d->M < 1) {
    set_error("%s: N, D, nlist, M must be positive (N may be 0)", fn);
    return IVFPQ_ERR_INVALID_ARGUMENT;
  }
  if (d->D % d->M) { set_error("%s: D = %d is not a multiple of M = %d", fn, d->D, d->M); return IVFPQ_ERR_INVALID_ARGUMENT; }
  if (d->metric != IVFPQ_METRIC_L2 && d->metric != IVFPQ_METRIC_IP) {
    set_error("%s: metric = %d unknown", fn, d->metric);
    return IVFPQ_ERR_INVALID_ARGUMENT;
  }
  if (d->M > IVFPQ_MAX_M) { set_error("%s: M = %d above the limit %d", fn, d->M, IVFPQ_MAX_M); return IVFPQ_ERR_UNSUPPORTED; }
  if (d->N >= ((int64_t)1 << 32)) { set_error("%s: N = %lld must be below 2^32", fn, (long long)d->N); return IVFPQ_ERR_UNSUPPORTED; }
  if (!d->centroids || !d->codebooks || !d->list_offsets || (d->N > 0 && !d->codes)) {
    set_error("%s: NULL array in the description", fn);
    return IVFPQ_ERR_INVALID_ARGUMENT;
  }
  // list offsets: host copy (works for host and device sources once a device exists;
  // a plain host pointer is read directly so that bad input is caught without a GPU)
  std::vector<int64_t> offs((size_t)d->nlist + 1);
  hipPointerAttribute_t attr;
  bool on_device = false;
  if (hipPointerGetAttributes(&attr, d->list_offsets) == hipSuccess)
    on_device = attr.type == hipMemoryTypeDevice;
  else
    (void)hipGetLastError();
  if (on_device) {
    IVFPQ_HIP_TRY(hipMemcpy(offs.data(), d->list_offsets, offs.size() * 8, hipMemcpyDeviceToHost));
  } else {
    memcpy(offs.data(), d->list_offsets, offs.size() * 8);
  }
  if (offs[0] != 0 || offs[d->nlist] != d->N) {
    set_error("%s: list_offsets must start at 0 and end at N", fn);
    return IVFPQ_ERR_INVALID_ARGUMENT;
  }
  std::vector<int64_t> blocks((size_t)d->nlist + 1);
  blocks[0] = 0;
  int64_t max_len = 0;
  for (int c = 0; c < d->nlist; ++c) {
    const int64_t len = offs[c + 1] - offs[c];
    if (len < 0) { set_error("%s: list_offsets decrease at list %d", fn, c); return IVFPQ_ERR_INVALID_ARGUMENT; }
    if (len > 0x7FFFFFC0ll) { set_error("%s: list %d longer than 2^31 points", fn, c); return IVFPQ_ERR_UNSUPPORTED; }
    if (len > max_len) max_len = len;
    blocks[c + 1] = blocks[c] + (len + 63) / 64;
  }

  ivfpq_index *ix = new (std::nothrow) ivfpq_index;
  if (!ix) { set_error("%s: out of host memory", fn); return IVFPQ_ERR_NO_MEMORY; }
  memset(ix, 0, sizeof *ix);
  ix->N = d->N; ix->D = d->D; ix->nlist = d->nlist; ix->M = d->M; ix->dsub = d->D / d->M;
  ix->metric = d->metric;
  ix->Mp = (d->M + 3) & ~3;
  ix->total_blocks = blocks[d->nlist];
  ix->code_bytes = ix->total_blocks * ivfpq_block_bytes(ix->Mp);
  ix->max_list_len = max_len;

  int rc = IVFPQ_OK;
  uint8_t *d_rows = nullptr;
  bool rows_owned = false;
  std::vector<float> cent_h, cnorm;
#define TRY_OR_FAIL(expr)                                   \
  do {                                                      \
    hipError_t _e = (expr);                                 \
    if (_e != hipSuccess) {                                 \
      rc = _e == hipErrorOutOfMemory ? IVFPQ_ERR_NO_MEMORY : IVFPQ_ERR_HIP; \
      set_error("%s: HIP error %d (%s) in %s", fn, (int)_e, hipGetErrorString(_e), #expr); \
      goto fail;                                            \
    }                                                       \
  } while (0)
  TRY_OR_FAIL(hipGetDevice(&ix->device));
  {
    const size_t cb = (size_t)d->nlist * d->D * 4, kb = (size_t)d->M * 256 * ix->dsub * 4;
    TRY_OR_FAIL(hipMalloc(&ix->d_centroids, cb));
    TRY_OR_FAIL(hipMalloc(&ix->d_cnorm, (size_t)d->nlist * 4));
    TRY_OR_FAIL(hipMalloc(&ix->d_codebooks, kb));
    TRY_OR_FAIL(hipMalloc(&ix->d_list_offsets, offs.size() * 8));
    TRY_OR_FAIL(hipMalloc(&ix->d_list_blocks, blocks.size() * 8));
    // padding behind the last list: for an empty list the scan reads (and ignores) one
    // 1 KiB chunk at the list's base
    TRY_OR_FAIL(hipMalloc(&ix->d_codes, (size_t)ix->code_bytes + 4096));
    TRY_OR_FAIL(hipMemset(ix->d_codes + ix->code_bytes, 0, 4096));
    TRY_OR_FAIL(hipMalloc(&ix->d_ids, d->N > 0 ? (size_t)d->N * 8 : 256));
    TRY_OR_FAIL(hipMemcpy(ix->d_centroids, d->centroids, cb, hipMemcpyDefault));
    TRY_OR_FAIL(hipMemcpy(ix->d_codebooks, d->codebooks, kb, hipMemcpyDefault));
    TRY_OR_FAIL(hipMemcpy(ix->d_list_offsets, offs.data(), offs.size() * 8, hipMemcpyHostToDevice));
    TRY_OR_FAIL(hipMemcpy(ix->d_list_blocks, blocks.data(), blocks.size() * 8, hipMemcpyHostToDevice));
    // squared centroid norms: only rank proposals in the filtering stage
    cent_h.resize((size_t)d->nlist * d->D);
    TRY_OR_FAIL(hipMemcpy(cent_h.data(), ix->d_centroids, cb, hipMemcpyDeviceToHost));
    cnorm.resize(d->nlist);
    float mx = 0.0f;
    for (int c = 0; c < d->nlist; ++c) {
      double s = 0.0;
      for (int i = 0; i < d->D; ++i) s += (double)cent_h[(size_t)c * d->D + i] * cent_h[(size_t)c * d->D + i];
      cnorm[c] = (float)s;
      if (cnorm[c] > mx) mx = cnorm[c];
    }
    ix->max_cnorm = mx;
    TRY_OR_FAIL(hipMemcpy(ix->d_cnorm, cnorm.data(), (size_t)d->nlist * 4, hipMemcpyHostToDevice));
    // many lists (for some nprobe): the product that proposes lists takes the centroids as two bf16
    // parts each (coarse_gemm_top_kernel)
    ix->ksplit = (d->D + 31) & ~31;
    if (coarse_fused_keys(d->nlist, 1, d->D) > 0) {
      const size_t part = (size_t)d->nlist * ix->ksplit;
      std::vector<uint16_t> split(2 * part, 0);
      for (int c = 0; c < d->nlist; ++c)
        for (int i = 0; i < d->D; ++i) {
          const float x = cent_h[(size_t)c * d->D + i];
          const uint16_t hi = bf16_bits(x);
          const uint32_t hb = (uint32_t)hi << 16;
          float hf;
          memcpy(&hf, &hb, 4);
          split[(size_t)c * ix->ksplit + i] = hi;
          split[part + (size_t)c * ix->ksplit + i] = bf16_bits(x - hf);
        }
      TRY_OR_FAIL(hipMalloc(&ix->d_csplit, split.size() * 2));
      TRY_OR_FAIL(hipMemcpy(ix->d_csplit, split.data(), split.size() * 2, hipMemcpyHostToDevice));
    }
    // list-major byte tables (lm_part_kernel): per entry (high part, rest) of both coordinates and of |entry|^2 as bf16, two
    // zeros.  Nothing in it is infinite or not a number: the products would spread that to other rows by way of the zeros
    // they multiply it with.  (The kernel looks at the entries themselves for what is not held here.)
    if (part_table_shape(ix)) {
      const size_t n = (size_t)d->M * 256;
      std::vector<float> cb_h(2 * n);
      TRY_OR_FAIL(hipMemcpy(cb_h.data(), ix->d_codebooks, kb, hipMemcpyDeviceToHost));
      std::vector<uint16_t> split(8 * n, 0);
      for (size_t i = 0; i < n; ++i) {
        float v[3] = {cb_h[2 * i], cb_h[2 * i + 1], 0.0f};
        v[2] = fmaf(v[1], v[1], v[0] * v[0]);
        if (!(v[2] < SPLIT_FAR)) {
          v[0] = v[1] = 0.0f;
          v[2] = SPLIT_FAR;
        }
        for (int j = 0; j < 3; ++j) {
          const uint16_t hi = bf16_bits(v[j]);
          const uint32_t hb = (uint32_t)hi << 16;
          float hf;
          memcpy(&hf, &hb, 4);
          split[8 * i + 2 * j] = hi;
          split[8 * i + 2 * j + 1] = bf16_bits(v[j] - hf);
        }
      }
      TRY_OR_FAIL(hipMalloc(&ix->d_cb_split, split.size() * 2));
      TRY_OR_FAIL(hipMemcpy(ix->d_cb_split, split.data(), split.size() * 2, hipMemcpyHostToDevice));
    }
    // per list and subspace, the bounding box of the entries the list's points use (filled
    // below from the codes; an empty list keeps the all-zero box)
    TRY_OR_FAIL(hipMalloc(&ix->d_box, (size_t)d->nlist * d->D * 2 * 4));
    TRY_OR_FAIL(hipMemset(ix->d_box, 0, (size_t)d->nlist * d->D * 2 * 4));
    // two-dimensional subspaces, L2: a grid per subspace with, for every cell, a lower bound on
    // the squared distance from any point of the cell to the nearest entry (the second
    // ingredient of the list-level bound, see probe_bound_kernel)
    if (ix->dsub == 2 && d->metric == IVFPQ_METRIC_L2) {
      TRY_OR_FAIL(hipMalloc(&ix->d_grid, (size_t)d->M * GRID_G * GRID_G * 4));
      TRY_OR_FAIL(hipMalloc(&ix->d_grid_par, (size_t)d->M * 8 * 4));
      rc = launch_codebook_grid(ix, nullptr);
      if (rc != IVFPQ_OK) goto fail;
      TRY_OR_FAIL(hipDeviceSynchronize());
    }
    if (d->N > 0) {
      bool codes_dev = false;
      if (hipPointerGetAttributes(&attr, d->codes) == hipSuccess) codes_dev = attr.type == hipMemoryTypeDevice;
      else (void)hipGetLastError();
      if (codes_dev) {
        d_rows = const_cast<uint8_t *>(d->codes);
      } else {
        TRY_OR_FAIL(hipMalloc(&d_rows, (size_t)d->N * d->M));
        rows_owned = true;
        TRY_OR_FAIL(hipMemcpy(d_rows, d->codes, (size_t)d->N * d->M, hipMemcpyHostToDevice));
      }
      rc = launch_relayout(ix, d_rows, nullptr);
      if (rc != IVFPQ_OK) goto fail;
      rc = launch_list_boxes(ix, d_rows, nullptr);
      if (rc != IVFPQ_OK) goto fail;
      if (d->ids) TRY_OR_FAIL(hipMemcpy(ix->d_ids, d->ids, (size_t)d->N * 8, hipMemcpyDefault));
      else {
        rc = launch_iota(ix->d_ids, d->N, nullptr);
        if (rc != IVFPQ_OK) goto fail;
      }
      TRY_OR_FAIL(hipDeviceSynchronize());
    }
  }
  if (rows_owned) (void)hipFree(d_rows);
  *out = ix;
  return IVFPQ_OK;
fail:
  if (rows_owned) (void)hipFree(d_rows);
  ivfpq_index_destroy(ix);
  return rc;
#undef TRY_OR_FAIL
}

int ivfpq_index_get_info(const ivfpq_index *ix, ivfpq_index_info *info) {
  if (!ix || !info) { set_error("index_get_info: NULL argument"); return IVFPQ_ERR_INVALID_ARGUMENT; }
  info->N = ix->N; info->D = ix->D; info->nlist = ix->nlist; info->M = ix->M; info->dsub = ix->dsub;
  info->code_bytes = ix->code_bytes; info->max_list_len = ix->max_list_len;
  info->metric = ix->metric;
  return IVFPQ_OK;
}

void ivfpq_radius_model_destroy(ivfpq_radius_model *md) {
  if (!md) return;
  (void)hipFree(md->d_block);
  delete md;
}

int ivfpq_radius_model_create(const ivfpq_index *ix, const ivfpq_radius_model_desc *d,
                              ivfpq_radius_model **out) {
  const char *fn = "radius_model_create";
  if (!ix || !d || !out) { set_error("%s: NULL argument", fn); return IVFPQ_ERR_INVALID_ARGUMENT; }
  *out = nullptr;
  if (!d->lo || !d->cells_per_unit || !d->map || !d->coef || !d->fallback) {
    set_error("%s: NULL array in the description", fn);
    return IVFPQ_ERR_INVALID_ARGUMENT;
  }
  if (d->M != ix->M) {
    set_error("%s: M = %d differs from the index's %d", fn, d->M, ix->M);
    return IVFPQ_ERR_INVALID_ARGUMENT;
  }
  if (ix->dsub != 2) {
    set_error("%s: the density map is two-dimensional; the index has dsub = %d", fn, ix->dsub);
    return IVFPQ_ERR_UNSUPPORTED;
  }
  if (d->grid < 1 || d->grid > 1024 || d->degree < 0 || d->degree > 8) {
    set_error("%s: grid = %d outside [1, 1024] or degree = %d outside [0, 8]", fn, d->grid, d->degree);
    return IVFPQ_ERR_INVALID_ARGUMENT;
  }
  const int M = d->M, G = d->grid, nc = d->degree + 1;
  for (int i = 0; i < 2 * M; ++i) {
    if (!isfinite(d->lo[i]) || !isfinite(d->cells_per_unit[i]) || !(d->cells_per_unit[i] > 0.0f)) {
      set_error("%s: lo / cells_per_unit of subspace %d not finite or not positive", fn, i / 2);
      return IVFPQ_ERR_INVALID_ARGUMENT;
    }
  }
  for (int m = 0; m < M; ++m) {
    if (!isfinite(d->fallback[m]) || d->fallback[m] < 0.0f) {
      set_error("%s: fallback[%d] must be finite and >= 0", fn, m);
      return IVFPQ_ERR_INVALID_ARGUMENT;
    }
  }
  ivfpq_radius_model *md = new (std::nothrow) ivfpq_radius_model;
  if (!md) { set_error("%s: out of host memory", fn); return IVFPQ_ERR_NO_MEMORY; }
  memset(md, 0, sizeof *md);
  md->M = M; md->grid = G; md->degree = d->degree;
  // lo | cells_per_unit | coef | fallback | map; every part starts on a multiple of 8 bytes
  const size_t n_lo = 2 * (size_t)M, n_coef = ((size_t)M * nc + 1) & ~(size_t)1, n_fb = ((size_t)M + 1) & ~(size_t)1;
  const size_t n_map = (size_t)M * G * G;
  std::vector<float> host(2 * n_lo + n_coef + n_fb + n_map, 0.0f);
  memcpy(host.data(), d->lo, n_lo * 4);
  memcpy(host.data() + n_lo, d->cells_per_unit, n_lo * 4);
  memcpy(host.data() + 2 * n_lo, d->coef, (size_t)M * nc * 4);
  memcpy(host.data() + 2 * n_lo + n_coef, d->fallback, (size_t)M * 4);
  memcpy(host.data() + 2 * n_lo + n_coef + n_fb, d->map, n_map * 4);
  hipError_t e = hipGetDevice(&md->device);
  if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void **>(&md->d_block), host.size() * 4);
  if (e == hipSuccess) e = hipMemcpy(md->d_block, host.data(), host.size() * 4, hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    ivfpq_radius_model_destroy(md);
    if (e == hipErrorOutOfMemory) { set_error("%s: out of device memory", fn); return IVFPQ_ERR_NO_MEMORY; }
    return hip_fail(e, fn);
  }
  md->d_lo = md->d_block;
  md->d_cpu = md->d_lo + n_lo;
  md->d_coef = md->d_cpu + n_lo;
  md->d_fallback = md->d_coef + n_coef;
  md->d_map = md->d_fallback + n_fb;
  *out = md;
  return IVFPQ_OK;
}

int ivfpq_query_radii(const ivfpq_index *ix, const ivfpq_radius_model *md, const float *d_queries,
                      int64_t Q, const int32_t *d_probe_ids, int32_t nprobe, float scale,
                      float *d_radii, void *stream) {
  const char *fn = "query_radii";
  int rc = check_common(ix, d_queries, Q, nprobe, fn);
  if (rc) return rc;
  if (!md) { set_error("%s: model is NULL", fn); return IVFPQ_ERR_INVALID_ARGUMENT; }
  if (md->M != ix->M || ix->dsub != 2) {
    set_error("%s: the model was made for another index shape", fn);
    return IVFPQ_ERR_INVALID_ARGUMENT;
  }
  if (!isfinite(scale) || scale < 0.0f) {
    set_error("%s: scale must be finite and >= 0", fn);
    return IVFPQ_ERR_INVALID_ARGUMENT;
  }
  if (Q == 0) return IVFPQ_OK;
  if (!d_probe_ids || !d_radii) { set_error("%s: NULL pointer", fn); return IVFPQ_ERR_INVALID_ARGUMENT; }
  return launch_query_radii(ix, md, d_queries, Q, d_probe_ids, nprobe, scale, d_radii,
                            static_cast<hipStream_t>(stream));
}

size_t ivfpq_search_workspace_bytes(const ivfpq_index *ix, int64_t Q, int32_t nprobe, int32_t k) {
  return ivfpq_search_workspace_bytes_ex(ix, Q, nprobe, k, nullptr);
}

size_t ivfpq_search_workspace_bytes_ex(const ivfpq_index *ix, int64_t Q, int32_t nprobe, int32_t k,
                                       const ivfpq_scoring *sc) {
  if (!ix || Q < 0 || nprobe < 1 || nprobe > ix->nlist || k < 1) return 0;
  const Workspace w = plan_workspace(ix, Q, nprobe, k);
  size_t n = w.total;
  if (use_list_major(ix, Q, nprobe, k, sc ? sc->mode : IVFPQ_SCORE_DISTANCE, sc ? sc->strategy : IVFPQ_SCAN_AUTO))
    n = align256(w.total) + plan_list_major(ix, lm_together(ix, Q, nprobe, sc ? sc->strategy : IVFPQ_SCAN_AUTO), nprobe).total;
  else if (const size_t wide = plan_wide(ix, Q, nprobe, k, sc ? sc->mode : IVFPQ_SCORE_DISTANCE, sc ? sc->strategy : IVFPQ_SCAN_AUTO).total)
    n = align256(w.total) + wide;
  return n < 256 ? 256 : n;
}

int ivfpq_resolve_strategy(const ivfpq_index *ix, int64_t Q, int32_t nprobe, int32_t k, const ivfpq_scoring *sc) {
  if (!ix || Q < 0 || nprobe < 1 || nprobe > ix->nlist || k < 1) {
    set_error("resolve_strategy: invalid argument");
    return IVFPQ_ERR_INVALID_ARGUMENT;
  }
  if (sc && (sc->strategy < IVFPQ_SCAN_AUTO || sc->strategy > IVFPQ_SCAN_LIST_MAJOR)) {
    set_error("resolve_strategy: scan strategy %d unknown", sc->strategy);
    return IVFPQ_ERR_INVALID_ARGUMENT;
  }
  return use_list_major(ix, Q, nprobe, k, sc ? sc->mode : IVFPQ_SCORE_DISTANCE, sc ? sc->strategy : IVFPQ_SCAN_AUTO)
             ? IVFPQ_SCAN_LIST_MAJOR : IVFPQ_SCAN_QUERY_MAJOR;
}

int ivfpq_coarse(const ivfpq_index *ix, const float *d_queries, int64_t Q, int32_t nprobe,
                 int32_t *d_probe_ids, float *d_probe_dist, void *ws, size_t ws_bytes, void *stream) {
  const char *fn = "coarse";
  int rc = check_common(ix, d_queries, Q, nprobe, fn);
  if (rc) return rc;
  if (Q == 0) return IVFPQ_OK;
  if (!d_probe_ids) { set_error("%s: output pointer is NULL", fn); return IVFPQ_ERR_INVALID_ARGUMENT; }
  const Workspace w = plan_workspace(ix, Q, nprobe, 1);
  if ((rc = check_workspace(w, ws, ws_bytes, fn))) return rc;
  char *base = static_cast<char *>(ws);
  return launch_coarse(ix, d_queries, Q, nprobe, d_probe_ids, d_probe_dist,
                       reinterpret_cast<float *>(base + w.coarse_dist), w.q_chunk, w.nlist_pad,
                       reinterpret_cast<int32_t *>(base + w.coarse_flags), static_cast<hipStream_t>(stream));
}

// scoring defaults (distances, shared radii) when the caller passes none
static int unpack_scoring(const ivfpq_index *ix, const ivfpq_scoring *sc, const float *radii, RadiiSq *r2,
                          int32_t *mode, const float **d_query_radii, const char *fn,
                          int32_t *strategy = nullptr) {
  *mode = IVFPQ_SCORE_DISTANCE;
  *d_query_radii = nullptr;
  if (strategy) *strategy = IVFPQ_SCAN_AUTO;
  if (sc) {
    if (sc->mode < IVFPQ_SCORE_DISTANCE || sc->mode > IVFPQ_SCORE_HIT_REWARD) {
      set_error("%s: scoring mode %d unknown", fn, sc->mode);
      return IVFPQ_ERR_INVALID_ARGUMENT;
    }
    if (sc->strategy < IVFPQ_SCAN_AUTO || sc->strategy > IVFPQ_SCAN_LIST_MAJOR) {
      set_error("%s: scan strategy %d unknown", fn, sc->strategy);
      return IVFPQ_ERR_INVALID_ARGUMENT;
    }
    *mode = sc->mode;
    *d_query_radii = sc->d_query_radii;
    if (strategy) *strategy = sc->strategy;
  }
  if (*d_query_radii) {  // per-query radii replace the shared ones
    memset(r2, 0, sizeof *r2);
    return IVFPQ_OK;
  }
  return make_radii(ix, radii, r2, fn);
}

// Stages 2-4 query-major.  For k above 128 the slots of the wide selection lie behind the usual
// workspace; a workspace without room for them still serves the call, pass by pass.
static int scan_query_major(const ivfpq_index *ix, const float *d_queries, int64_t Q, int32_t nprobe,
                            const int32_t *d_probe_ids, int32_t k, const RadiiSq &r2, int32_t mode, const float *qr,
                            int64_t *d_out_ids, float *d_out_dist, const Workspace &w, char *base, size_t ws_bytes,
                            hipStream_t s, int32_t strategy) {
  WideWorkspace ww = plan_wide(ix, Q, nprobe, k, mode, strategy);
  if (ww.first > 0 && ws_bytes < align256(w.total) + ww.total) {   // room for the slots alone
    ww.total = ww.lm_off;
    ww.first = 0;
  }
  // (the flags of the filtering stage have been read when the scan starts: their place holds the
  // bounds that the workgroups of a query share)
  ScanView view = {0, nullptr, false, nullptr, nullptr, reinterpret_cast<uint32_t *>(base + w.coarse_flags)};
  if (ww.total > 0 && ws_bytes >= align256(w.total) + ww.total) {
    view.wide = &ww;
    view.wide_base = base + align256(w.total);
  }
  return launch_scan(ix, d_queries, Q, nprobe, d_probe_ids, k, r2, w.nsplit,
                     reinterpret_cast<uint32_t *>(base + w.part_d), reinterpret_cast<int64_t *>(base + w.part_id),
                     d_out_ids, d_out_dist, nullptr, nullptr, nullptr, nullptr, mode, qr,
                     reinterpret_cast<float *>(base + w.probe_dist), s, &view);
}

// Whether a call goes list-major with the workspace it has: AUTO on long lists and below LM_ALWAYS pairs, and every call on shapes
// without byte tables, is served query-major where the workspace only has room for that.
static bool goes_list_major(const ivfpq_index *ix, int64_t Q, int32_t nprobe, int32_t k, int32_t mode, int32_t strategy,
                            const Workspace &w, size_t ws_bytes) {
  if (!use_list_major(ix, Q, nprobe, k, mode, strategy)) return false;
  if (byte_table_shape(ix) &&
      (strategy == IVFPQ_SCAN_LIST_MAJOR || (ix->N <= (int64_t)4096 * ix->nlist && Q * (int64_t)nprobe >= LM_ALWAYS))) return true;
  return ws_bytes >= align256(w.total) + plan_list_major(ix, lm_together(ix, Q, nprobe, strategy), nprobe).total;
}

// Stages 2-4 list-major: the usual workspace, then the list-major part behind it.
static int scan_list_major(const ivfpq_index *ix, const float *d_queries, int64_t Q, int32_t nprobe,
                           const int32_t *d_probe_ids, int32_t k, const RadiiSq &r2, int32_t mode, const float *qr,
                           int64_t *d_out_ids, float *d_out_dist, const Workspace &w, void *ws, size_t ws_bytes,
                           hipStream_t s, int32_t strategy, const char *fn) {
  const int64_t step = lm_together(ix, Q, nprobe, strategy);
  const LmWorkspace lw = plan_list_major(ix, step, nprobe);
  Workspace both = w;
  both.total = align256(w.total) + lw.total;
  if (int rc = check_workspace(both, ws, ws_bytes, fn)) return rc;
  char *base = static_cast<char *>(ws);
  float *probe_lb = reinterpret_cast<float *>(base + w.probe_dist);
  for (int64_t q0 = 0; q0 < Q; q0 += step) {
    const int64_t n = Q - q0 < step ? Q - q0 : step;
    if (int rc = launch_scan_list_major(ix, d_queries + q0 * ix->D, n, nprobe, d_probe_ids + q0 * nprobe, k, r2, mode,
                                        qr ? qr + q0 * ix->M : nullptr, probe_lb + q0 * nprobe, d_out_ids + q0 * k,
                                        d_out_dist + q0 * k, lw, base + align256(w.total), s))
      return rc;
  }
  return IVFPQ_OK;
}

int ivfpq_build_lut_ex(const ivfpq_index *ix, const float *d_queries, int64_t Q, int32_t nprobe,
                       const int32_t *d_probe_ids, const float *radii, const ivfpq_scoring *scoring,
                       float *d_lut, uint64_t *d_mask, void *stream) {
  const char *fn = "build_lut";
  int rc = check_common(ix, d_queries, Q, nprobe, fn);
  if (rc) return rc;
  RadiiSq r2;
  int32_t mode;
  const float *qr;
  if ((rc = unpack_scoring(ix, scoring, radii, &r2, &mode, &qr, fn))) return rc;
  if (Q == 0) return IVFPQ_OK;
  if (!d_probe_ids || !d_lut) { set_error("%s: NULL pointer", fn); return IVFPQ_ERR_INVALID_ARGUMENT; }
  return launch_build_lut(ix, d_queries, Q, nprobe, d_probe_ids, r2, d_lut, d_mask, mode, qr,
                          static_cast<hipStream_t>(stream));
}

int ivfpq_build_lut(const ivfpq_index *ix, const float *d_queries, int64_t Q, int32_t nprobe,
                    const int32_t *d_probe_ids, const float *radii, float *d_lut, uint64_t *d_mask,
                    void *stream) {
  return ivfpq_build_lut_ex(ix, d_queries, Q, nprobe, d_probe_ids, radii, nullptr, d_lut, d_mask, stream);
}

int ivfpq_scan_topk_ex(const ivfpq_index *ix, const float *d_queries, int64_t Q, int32_t nprobe,
                       const int32_t *d_probe_ids, int32_t k, const float *radii,
                       const ivfpq_scoring *scoring, int64_t *d_out_ids, float *d_out_dist, void *ws,
                       size_t ws_bytes, void *stream) {
  const char *fn = "scan_topk";
  int rc = check_common(ix, d_queries, Q, nprobe, fn);
  if (rc) return rc;
  if ((rc = check_k(k, fn))) return rc;
  RadiiSq r2;
  int32_t mode, strategy;
  const float *qr;
  if ((rc = unpack_scoring(ix, scoring, radii, &r2, &mode, &qr, fn, &strategy))) return rc;
  if (Q == 0) return IVFPQ_OK;
  if (!d_probe_ids || !d_out_ids || !d_out_dist) { set_error("%s: NULL pointer", fn); return IVFPQ_ERR_INVALID_ARGUMENT; }
  const Workspace w = plan_workspace(ix, Q, nprobe, k);
  char *base = static_cast<char *>(ws);
  if (goes_list_major(ix, Q, nprobe, k, mode, strategy, w, ws_bytes))
    return scan_list_major(ix, d_queries, Q, nprobe, d_probe_ids, k, r2, mode, qr, d_out_ids, d_out_dist, w, ws,
                           ws_bytes, static_cast<hipStream_t>(stream), strategy, fn);
  if ((rc = check_workspace(w, ws, ws_bytes, fn))) return rc;
  return scan_query_major(ix, d_queries, Q, nprobe, d_probe_ids, k, r2, mode, qr, d_out_ids, d_out_dist, w, base,
                          ws_bytes, static_cast<hipStream_t>(stream), strategy);
}

int ivfpq_scan_topk(const ivfpq_index *ix, const float *d_queries, int64_t Q, int32_t nprobe,
                    const int32_t *d_probe_ids, int32_t k, const float *radii, int64_t *d_out_ids,
                    float *d_out_dist, void *ws, size_t ws_bytes, void *stream) {
  return ivfpq_scan_topk_ex(ix, d_queries, Q, nprobe, d_probe_ids, k, radii, nullptr, d_out_ids, d_out_dist,
                            ws, ws_bytes, stream);
}

// ---- the search that allocates nothing and takes no workspace -----------------------------
// Its workspace is this array: one copy per GPU, held from the moment the library is loaded
// on that GPU until the process ends.  The name is a host-side stand-in, not a device
// address: host code only ever uses the pointer that hipGetSymbolAddress returns for the
// current device (scratch_address), and the kernels receive that pointer as an argument,
// exactly as they receive a caller's workspace.
static __device__ __align__(256) __attribute__((used)) unsigned char scratch[IVFPQ_NOALLOC_SCRATCH_BYTES];

static constexpr int MAX_DEVICES = 64;
static std::atomic<void *> g_scratch_ptr[MAX_DEVICES];

// Device address of `scratch` on the current device, looked up once per device.
static int scratch_address(void **out, const char *fn) {
  int dev = -1;
  IVFPQ_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= MAX_DEVICES) {
    set_error("%s: device ordinal %d outside [0, %d)", fn, dev, MAX_DEVICES);
    return IVFPQ_ERR_UNSUPPORTED;
  }
  void *p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!p) {
    IVFPQ_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p || (uintptr_t)p % 256) {
      set_error("%s: the static scratch array has no usable device address", fn);
      return IVFPQ_ERR_HIP;
    }
    g_scratch_ptr[dev].store(p, std::memory_order_release);  // two threads racing here store the same address
  }
  *out = p;
  return IVFPQ_OK;
}

// Stages 1-4 with the workspace `base` carved as `w` says.
static int search_in_workspace(const ivfpq_index *ix, const float *d_queries, int64_t Q, int32_t nprobe,
                               int32_t k, const RadiiSq &r2, int32_t mode, const float *qr, int64_t *d_out_ids,
                               float *d_out_dist, const Workspace &w, char *base, size_t ws_bytes, hipStream_t s,
                               int32_t strategy) {
  int32_t *probe_ids = reinterpret_cast<int32_t *>(base + w.probe_ids);
  int rc = launch_coarse(ix, d_queries, Q, nprobe, probe_ids, nullptr,
                         reinterpret_cast<float *>(base + w.coarse_dist), w.q_chunk, w.nlist_pad,
                         reinterpret_cast<int32_t *>(base + w.coarse_flags), s);
  if (rc) return rc;
  return scan_query_major(ix, d_queries, Q, nprobe, probe_ids, k, r2, mode, qr, d_out_ids, d_out_dist, w, base,
                          ws_bytes, s, strategy);
}

int ivfpq_search_noalloc(const ivfpq_index *ix, const float *d_queries, int64_t Q, int32_t nprobe, int32_t k,
                         const float *radii, int64_t *d_out_ids, float *d_out_dist, void *stream) {
  const char *fn = "search_noalloc";
  int rc = check_common(ix, d_queries, Q, nprobe, fn);
  if (rc) return rc;
  if ((rc = check_k(k, fn))) return rc;
  RadiiSq r2;
  if ((rc = make_radii(ix, radii, &r2, fn))) return rc;
  if (Q == 0) return IVFPQ_OK;
  if (!d_out_ids || !d_out_dist) { set_error("%s: NULL pointer", fn); return IVFPQ_ERR_INVALID_ARGUMENT; }
  const Workspace w = plan_workspace(ix, Q, nprobe, k, IVFPQ_NOALLOC_SCRATCH_BYTES);
  if (w.total == SIZE_MAX || w.total > IVFPQ_NOALLOC_SCRATCH_BYTES) {
    set_error("%s: Q = %lld, nprobe = %d with nlist = %d need more than the %u bytes of built-in scratch; "
              "use ivfpq_search with a workspace, or smaller batches", fn, (long long)Q, nprobe, ix->nlist,
              (unsigned)IVFPQ_NOALLOC_SCRATCH_BYTES);
    return IVFPQ_ERR_WORKSPACE;
  }
  void *base = nullptr;
  if ((rc = scratch_address(&base, fn))) return rc;
  // Nothing in the workspace has to start at zero: every region is written in full (for the
  // rows and probes of this call) before it is read, so the previous call's contents do not matter.
  return search_in_workspace(ix, d_queries, Q, nprobe, k, r2, IVFPQ_SCORE_DISTANCE, nullptr, d_out_ids,
                             d_out_dist, w, static_cast<char *>(base), IVFPQ_NOALLOC_SCRATCH_BYTES,
                             static_cast<hipStream_t>(stream), IVFPQ_SCAN_QUERY_MAJOR);
}

int ivfpq_search_ex(const ivfpq_index *ix, const float *d_queries, int64_t Q, int32_t nprobe, int32_t k,
                    const float *radii, const ivfpq_scoring *scoring, int64_t *d_out_ids,
                    float *d_out_dist, void *ws, size_t ws_bytes, void *stream) {
  const char *fn = "search";
  int rc = check_common(ix, d_queries, Q, nprobe, fn);
  if (rc) return rc;
  if ((rc = check_k(k, fn))) return rc;
  RadiiSq r2;
  int32_t mode, strategy;
  const float *qr;
  if ((rc = unpack_scoring(ix, scoring, radii, &r2, &mode, &qr, fn, &strategy))) return rc;
  if (Q == 0) return IVFPQ_OK;
  if (!d_out_ids || !d_out_dist) { set_error("%s: NULL pointer", fn); return IVFPQ_ERR_INVALID_ARGUMENT; }
  const Workspace w = plan_workspace(ix, Q, nprobe, k);
  if (goes_list_major(ix, Q, nprobe, k, mode, strategy, w, ws_bytes)) {
    Workspace both = w;
    both.total = align256(w.total) + plan_list_major(ix, lm_together(ix, Q, nprobe, strategy), nprobe).total;
    if ((rc = check_workspace(both, ws, ws_bytes, fn))) return rc;   // before anything is enqueued
    char *base = static_cast<char *>(ws);
    int32_t *probe_ids = reinterpret_cast<int32_t *>(base + w.probe_ids);
    rc = launch_coarse(ix, d_queries, Q, nprobe, probe_ids, nullptr, reinterpret_cast<float *>(base + w.coarse_dist),
                       w.q_chunk, w.nlist_pad, reinterpret_cast<int32_t *>(base + w.coarse_flags),
                       static_cast<hipStream_t>(stream));
    if (rc) return rc;
    return scan_list_major(ix, d_queries, Q, nprobe, probe_ids, k, r2, mode, qr, d_out_ids, d_out_dist, w, ws,
                           ws_bytes, static_cast<hipStream_t>(stream), strategy, fn);
  }
  if ((rc = check_workspace(w, ws, ws_bytes, fn))) return rc;
  return search_in_workspace(ix, d_queries, Q, nprobe, k, r2, mode, qr, d_out_ids, d_out_dist, w,
                             static_cast<char *>(ws), ws_bytes, static_cast<hipStream_t>(stream), strategy);
}

int ivfpq_search(const ivfpq_index *ix, const float *d_queries, int64_t Q, int32_t nprobe, int32_t k,
                 const float *radii, int64_t *d_out_ids, float *d_out_dist, void *ws, size_t ws_bytes,
                 void *stream) {
  return ivfpq_search_ex(ix, d_queries, Q, nprobe, k, radii, nullptr, d_out_ids, d_out_dist, ws, ws_bytes,
                         stream);
}

int ivfpq_scan_all_ex(const ivfpq_index *ix, const float *d_queries, int64_t Q, int32_t nprobe,
                      const int32_t *d_probe_ids, const float *radii, const ivfpq_scoring *scoring,
                      const int64_t *d_cand_offsets, float *d_all_dist, int64_t *d_all_ids,
                      int32_t *d_errors, void *stream) {
  const char *fn = "scan_all";
  int rc = check_common(ix, d_queries, Q, nprobe, fn);
  if (rc) return rc;
  RadiiSq r2;
  int32_t mode;
  const float *qr;
  if ((rc = unpack_scoring(ix, scoring, radii, &r2, &mode, &qr, fn))) return rc;
  if (!d_errors) { set_error("%s: NULL pointer", fn); return IVFPQ_ERR_INVALID_ARGUMENT; }
  if (Q > 0 && (!d_probe_ids || !d_cand_offsets || !d_all_dist || !d_all_ids)) {
    set_error("%s: NULL pointer", fn);
    return IVFPQ_ERR_INVALID_ARGUMENT;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  rc = launch_fill_i32(d_errors, 1, 0, s);
  if (rc || Q == 0) return rc;
  // the dump variant of the scan kernel keeps no top-k, so k and the result pointers are unused
  return launch_scan(ix, d_queries, Q, nprobe, d_probe_ids, 0, r2, 1, nullptr, nullptr, nullptr, nullptr,
                     d_cand_offsets, d_all_dist, d_all_ids, d_errors, mode, qr, nullptr, s);
}

int ivfpq_scan_all(const ivfpq_index *ix, const float *d_queries, int64_t Q, int32_t nprobe,
                   const int32_t *d_probe_ids, const float *radii, const int64_t *d_cand_offsets,
                   float *d_all_dist, int64_t *d_all_ids, int32_t *d_errors, void *stream) {
  return ivfpq_scan_all_ex(ix, d_queries, Q, nprobe, d_probe_ids, radii, nullptr, d_cand_offsets, d_all_dist,
                           d_all_ids, d_errors, stream);
}

}  // extern "C"
