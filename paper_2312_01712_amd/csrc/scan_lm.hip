// List-major batched scan: the queries that probe the same inverted list are served
// together, eight at a time (two where fp32 tables serve), from ONE pass over the list's codes.
//
// Paper Sec. 5.2 / Algorithm 1 builds an inverted entry -> points map per list so that the
// distance calculation (Sec. 5.3) touches a list's points once per hit entry.  On CDNA4 the
// dense code stream is the better carrier, and what the map buys -- work shared inside a list
// -- is had by turning the loop nest around: the outer loop runs over lists, the queries that
// selected a list (Sec. 2.1 step A) are grouped, and the group shares the list's code stream
// and ONE table look-up per (point, subspace): the tables of the two queries of a group are
// interleaved entry by entry, so a single 8-byte LDS read returns both queries' values for a
// point's code.  The LDS gather rate, which bounds the query-major scan on data where
// nothing can be pruned, is per lane-address and not per byte, so two queries cost what one
// did (lm_scan_kernel); with a byte per query the same read serves eight (lm_byte_kernel).  Sums keep the
// subspace order of the plain loop: results are bit for bit those of the query-major scan.
//
// A query's lists are now scanned by different workgroups at different times, so the running
// k-th distance is not at hand.  Instead:
//   A  the nearest list of every query (with hit counts, or several first lists, the first few) is
//      ranked first and leaves each query's top-k of it; tau_q = its k-th distance bounds the
//      final k-th distance from above.  Three ways: list-major with fp32 tables (the head pass:
//      lm_scan_kernel<HEAD>), on long lists with byte tables (lm_byte_kernel<HEAD>, whose candidates
//      lm_settle_kernel ranks; some queries only get a bound from it), else the query-major kernel;
//   B  (query, list) pairs of the remaining probes whose list-level lower bound exceeds tau_q
//      are dropped; the others are bucketed by list (count, offsets, fill);
//   C  the list-major scan appends to the query's candidate buffer what may lie within tau_q (anything
//      above cannot be in the result): from fp32 tables every point with distance <= tau_q as (distance,
//      row), with hit counts from byte tables every point with score <= tau_q likewise; from byte tables
//      of distances every point whose byte sum is within the query's limit, as (list, row);
//   D  one wavefront per query merges its buffer into the top-k of phase A by (distance, id):
//      lm_merge_kernel, or, behind byte tables of distances, lm_settle_kernel, which forms the
//      candidates' distances first (its wavefronts together; behind a head pass with byte tables and in the
//      largest batches a wavefront by itself, the queries sorted out by lm_sort_out_kernel).
// B to D run twice where a query has many probes.  A query whose buffer overflows is redone by the
// query-major kernel, so the result is always that of the plain loop.

#include "scan_device.h"

namespace {

constexpr int LM_G = 2;        // queries per group (interleaved tables, 8-byte look-ups)
constexpr int LMB_G = 8;       // ... with byte tables (lm_byte_kernel)
constexpr int LM_NW = 8;       // wavefronts per workgroup: one workgroup per CU (the table fills most of its LDS), 2 per SIMD, 256 registers each
constexpr int LM_STAGE1 = 7;   // probes of the first of two main passes (behind the lists ranked first)
constexpr int LM_QUEUE = 64;   // accepted candidates a wavefront holds per query before it appends them
constexpr int LM_SEL_WORDS = 16;     // head pass: small LDS block of selection state
constexpr int32_t LM_SEEDED = -2;
constexpr int LM_BINS = 1024;        // head pass: bins of the selection histogram
constexpr int LM_COLLECT = 128;      // head pass: candidates a query may collect (the sorted list of a wavefront)

typedef float floatx2 __attribute__((ext_vector_type(2)));

struct LmArgs {
  const float *queries;         // [Q][D]
  const int32_t *probe_ids;     // [Q][nprobe]
  const float *probe_lb;        // [Q][nprobe] list-level lower bounds, or NULL
  const float *centroids;       // [nlist][D]
  const float *codebooks;       // [M][256][dsub]
  const uint16_t *cb_split;     // [M][256][8] its entries as pairs of bf16 (lm_part_kernel), or NULL
  const int64_t *list_offsets;  // [nlist+1]
  const int64_t *list_blocks;   // [nlist+1]
  const uint8_t *codes;         // interleaved blocks
  const int64_t *ids;           // [N]
  int64_t *out_ids;             // [Q][k]: phase A's top-k on entry to the merge, the result after it
  float *out_dist;              // [Q][k]
  int32_t *cnt;                 // [nlist] pairs per list; then [2]: queries to be redone, and those of them taken up; then per stage [2]: queries with candidates, and those of them taken up by lm_settle_kernel
  int32_t *rank;                // [max(Q, Q*(nprobe-first))] position of a pair among its list's pairs, -1: no pair
  int32_t *base;                // [nlist+1] first pair slot of a list (ranges padded to whole groups); [nlist] = slots in use
  int2 *pairs;                  // [Q*(nprobe-first) + (LMB_G - 1) nlist] (query, list); query -1 pads a list's range
  uint32_t *gcnt;               // [Q] candidates appended (may run past cap: the query then counts as overflowed)
  uint2 *cand;                  // [Q][cap] (distance bits, row in the index); from byte tables of distances (list, row)
  int32_t *qmap;                // [Q] q for a query to be redone query-major, -1 otherwise
  int32_t *redo;                // [Q] those queries, in any order (the place of rank)
  int32_t *qmap_head;           // [Q] head pass: q for a query whose nearest list is left to the query-major kernel, else -1, or
                                // LM_SEEDED: its result holds any k points of that list, which bound its k-th distance
  int32_t head_max;             // head pass: longest list (points) whose distances fit the workgroup's LDS
  const float *query_radii;     // [Q][M] or NULL
  float rmax;                   // largest r_m^2 of the shared radii
  int64_t Q;
  int32_t D, M, dsub, Mp, nlist, nprobe, first, k, cap, mode;
  int32_t p0, p1;               // the probes [p0, p1) of every query that the current main pass serves
  int32_t later;                // this is not the first main pass: qmap already names queries to be redone
  int32_t stage;                // which of the passes of a call with candidates to settle
  int32_t fresh;                // byte tables in the head pass: the queries have no result yet
  int32_t list_redo;            // lm_settle_kernel in place: this is the last pass, queries to be redone are listed too
  int32_t parts;                // byte tables of distances go by in parts (lm_part_kernel)
  int32_t seeded;               // behind that pass: qmap_head may be LM_SEEDED
  int32_t group;                // queries per group of the pass the pairs are bucketed for
  int32_t head_done;            // the head pass has run: queries it left out (qmap_head) have no first-list result yet
  const float *tau;             // [Q] x tau_stride: the k-th distance that filters the main pass (NaN: none yet)
  int32_t tau_stride;
  // Behind the wide selection's first lists (k above KP; NULL otherwise) the slots are its own: cand is [Q][cap] row,
  // as 64 bits, once settled, with the distances beside; cap the slots of a query
  int32_t *wide_n;              // [Q] slots in use, -1: a query that is left out
  uint32_t *wide_d;             // [Q][cap] distance keys
};

// One thread per (query, probe >= first).  fill == 0: count the surviving pairs of every list
// (and clear the query's candidate count); the value the count returns is the pair's position
// among its list's pairs and is kept (rank, -1 for a pair that takes no part), so that
// fill == 1 only has to write the pair to that position of the list's slot range: no second
// evaluation of the predicate and no second atomic operation on the per-list words.
// head == 1 (the head pass): one thread per query, the pair is (query, its nearest list); a
// query whose nearest list is missing, empty or too long for the head pass is handed to the
// query-major kernel through qmap_head instead.
__global__ __launch_bounds__(256) void lm_pairs_kernel(LmArgs a, int fill, int head) {
  const int np2 = head ? 1 : a.p1 - a.p0;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= a.Q * np2) return;
  const int64_t q = idx / np2;
  const int p = head ? 0 : a.p0 + (int)(idx % np2);
  const int32_t c = a.probe_ids[q * a.nprobe + p];
  if (fill) {
    const int32_t r = a.rank[idx];
    if (r >= 0) a.pairs[a.base[c] + r] = make_int2((int)q, c);
    return;
  }
  if (head) a.gcnt[q] = 0u;
  if (!head && p == a.p0) a.gcnt[q] = a.wide_n && a.wide_n[q] > 0 ? (uint32_t)a.wide_n[q] : 0u;
  bool take = true;
  // a query the head pass left out has no bound yet: it takes no part here and is redone query-major
  // over all of its lists (lm_sort_out_kernel or, where that does not run, name_query names it)
  if (!head && a.head_done && a.qmap_head[q] >= 0) take = false;
  if (!head && a.later && a.qmap[q] >= 0) take = false;   // nor does one whose slots have overflowed
  if (!head && a.seeded && p == 0 && a.qmap_head[q] != LM_SEEDED) take = false;   // the head pass has ranked this list
  if (a.wide_n && a.wide_n[q] < 0) take = false;
  const bool exists = (uint32_t)c < (uint32_t)a.nlist;
  const int64_t len = exists ? a.list_offsets[c + 1] - a.list_offsets[c] : 0;
  if (head) {
    const bool ok = len > 0 && len <= a.head_max;
    a.qmap_head[q] = ok ? -1 : (int32_t)q;
    take = ok;
  }
  if (len <= 0) take = false;
  if (take && !head && a.probe_lb) {
    // no point of the list can reach the k-th distance that phase A already guarantees
    if (a.probe_lb[q * a.nprobe + p] > a.tau[q * a.tau_stride]) take = false;
  }
  a.rank[idx] = take ? atomicAdd(&a.cnt[c], 1) : -1;
}

template <int J>
__device__ __forceinline__ float xor_f32(float v) { return __uint_as_float(xor_u32<J, true>(__float_as_uint(v))); }

// The list-level bounds of a main pass behind the head pass, and the count of its pairs (lm_pairs_kernel's, fill == 0): the
// bounds of probe_bound_kernel, two-dimensional subspaces and distances, a quarter of a wavefront per pair and 16 subspaces at
// a time, ended where they pass the query's k-th distance so far: the terms are not negative, so what is summed by then is
// a lower bound too.  A list that is too far is so by half of its subspaces or a few more, and what the bounds cost is their
// way from the L2 (24 bytes per pair and subspace).  Queries that are left to the query-major scan get theirs in full.
// 10 000 queries, clustered data, bounds up front and count / so: 64 subspaces of 32 probes 64 + 5 / 38 us, 100 of 64 184 + 5 / 102;
// 48 of 64 without structure, where none ends early, 117 + 118 / 155.
// The pairs of a workgroup are counted by one instruction: atomics on a line are served one after the other, those of an
// instruction together (four lanes at a time, 30 000 pairs on few lists took 70 us, the whole of probe_bound_kernel and lm_pairs_kernel 37).
constexpr int LM_BOUND_SETS = 2;   // pairs of a quarter of a wavefront, whose loads are issued together
constexpr int LM_BOUND_NW = 64 / (4 * LM_BOUND_SETS);   // wavefronts: 64 pairs
template <bool GRID>
__global__ __launch_bounds__(LM_BOUND_NW * 64) void lm_bound_kernel(LmArgs a, RadiiSq r2, const float *__restrict__ box, const float *__restrict__ grid,
                                                       const float *__restrict__ grid_par, float *__restrict__ lb) {
  const int lane = threadIdx.x & 63, l = lane & 15;
  const uint32_t np2 = (uint32_t)(a.p1 - a.p0), total = (uint32_t)a.Q * np2;   // (below 2^31)
  __shared__ int32_t counted[64];   // list of a pair that is counted, or -1
  const uint32_t slot0 = (threadIdx.x >> 6) * (4 * LM_BOUND_SETS) + (lane >> 4), idx0 = blockIdx.x * 64 + slot0;
  uint32_t q[LM_BOUND_SETS];
  int32_t c[LM_BOUND_SETS];
  bool want[LM_BOUND_SETS], named[LM_BOUND_SETS], exists[LM_BOUND_SETS], alive[LM_BOUND_SETS];
  float tau[LM_BOUND_SETS], acc[LM_BOUND_SETS], sum[LM_BOUND_SETS];
#pragma unroll
  for (int s = 0; s < LM_BOUND_SETS; ++s) {
    const uint32_t idx = idx0 + 4 * s, in = idx < total ? idx : total - 1;   // (a pair past the end is computed and not stored)
    q[s] = in / np2;
    const int p = a.p0 + (int)(in % np2);
    c[s] = a.probe_ids[(int64_t)q[s] * a.nprobe + p];
    exists[s] = (uint32_t)c[s] < (uint32_t)a.nlist;
    if (!exists[s]) c[s] = 0;
    const int32_t left = a.qmap_head[q[s]];
    // left out by the head pass or out of slots in the pass before: redone over all lists
    named[s] = left >= 0 || (a.later && a.qmap[q[s]] >= 0);
    want[s] = exists[s] && a.list_offsets[c[s] + 1] > a.list_offsets[c[s]] && !(a.seeded && p == 0 && left != LM_SEEDED);   // (else the head pass has ranked this list)
    tau[s] = named[s] ? __builtin_inff() : a.tau[(int64_t)q[s] * a.tau_stride];
    acc[s] = sum[s] = 0.0f;
    alive[s] = want[s];
  }
#pragma unroll 1
  for (int m0 = 0; m0 < a.M; m0 += 16) {
    const int m = m0 + l;
    const bool on = m < a.M;
#pragma unroll
    for (int s = 0; s < LM_BOUND_SETS; ++s) {
      if (!on || !alive[s]) continue;
      const float2 qv = *reinterpret_cast<const float2 *>(a.queries + (int64_t)q[s] * a.D + 2 * m);
      const float2 cv = *reinterpret_cast<const float2 *>(a.centroids + (int64_t)c[s] * a.D + 2 * m);
      const float4 v = reinterpret_cast<const float4 *>(box + (int64_t)c[s] * a.D * 2)[m];
      const float x0 = qv.x - cv.x, x1 = qv.y - cv.y;
      const float t0 = fmaxf(fmaxf(v.x - x0, x0 - v.z), 0.0f);
      const float t1 = fmaxf(fmaxf(v.y - x1, x1 - v.w), 0.0f);
      float best = fmaf(t1, t1, t0 * t0);
      if constexpr (GRID) {   // see probe_bound_kernel
        const float4 gp0 = reinterpret_cast<const float4 *>(grid_par)[2 * m];
        const float2 gp1 = reinterpret_cast<const float2 *>(grid_par)[4 * m + 2];
        const float fx = fminf(fmaxf((x0 - gp0.x) * gp1.x, 0.0f), (float)(ivfpq::GRID_G - 1));
        const float fy = fminf(fmaxf((x1 - gp0.y) * gp1.y, 0.0f), (float)(ivfpq::GRID_G - 1));
        const float cell = grid[(int64_t)m * (ivfpq::GRID_G * ivfpq::GRID_G) + (int)fy * ivfpq::GRID_G + (int)fx];
        const float o0 = fmaxf(fmaxf(gp0.x - x0, x0 - gp0.z), 0.0f);
        const float o1 = fmaxf(fmaxf(gp0.y - x1, x1 - gp0.w), 0.0f);
        best = fmaxf(best, cell + fmaf(o1, o1, o0 * o0));
      }
      float rm2 = r2.v[m];
      if (a.query_radii) {
        const float r = a.query_radii[(int64_t)q[s] * a.M + m];
        rm2 = r * r;
      }
      acc[s] += fminf(best, rm2);
    }
    bool any = false;
#pragma unroll
    for (int s = 0; s < LM_BOUND_SETS; ++s) {
      float v = acc[s];
      v += xor_f32<1>(v);
      v += xor_f32<2>(v);
      v += xor_f32<4>(v);
      v += xor_f32<8>(v);
      sum[s] = v * 0.999755859375f;   // (the roundings of this evaluation against the table's)
      alive[s] = alive[s] && !(sum[s] > tau[s]);
      any = any || alive[s];
    }
    if (__ballot(any) == 0ull) break;
  }
#pragma unroll
  for (int s = 0; s < LM_BOUND_SETS; ++s) {
    const uint32_t idx = idx0 + 4 * s;
    if (l == 0) counted[slot0 + 4 * s] = idx < total && alive[s] && !named[s] ? c[s] : -1;
    if (l != 0 || idx >= total) continue;
    const int p = a.p0 + (int)(idx % np2);
    float *row = lb + (int64_t)q[s] * a.nprobe;
    row[p] = exists[s] ? sum[s] : 0.0f;
    if (p == a.p0) {
      a.gcnt[q[s]] = 0u;
      if (!a.later)
        for (int x = 0; x < a.p0; ++x) row[x] = 0.0f;   // (lists ranked by the head pass: no bound, wherever they are scanned again)
    }
  }
  __syncthreads();
  const uint32_t idx = blockIdx.x * 64 + threadIdx.x;
  if (threadIdx.x >= 64 || idx >= total) return;
  const int32_t list = counted[threadIdx.x];
  a.rank[idx] = list >= 0 ? atomicAdd(&a.cnt[list], 1) : -1;
}

// Slot ranges of the lists: base[c] = sum over c' < c of cnt[c'] rounded up to a.group.  The
// padding slots of a range are marked (query -1), the counts are cleared.
// One workgroup.
__global__ __launch_bounds__(1024) void lm_offsets_kernel(LmArgs a) {
  __shared__ int part[1024];
  const int tid = threadIdx.x;
  const int chunk = (a.nlist + 1023) / 1024;
  const int lo = tid * chunk < a.nlist ? tid * chunk : a.nlist;
  const int hi = lo + chunk < a.nlist ? lo + chunk : a.nlist;
  int sum = 0;
  for (int c = lo; c < hi; ++c) sum += (a.cnt[c] + a.group - 1) / a.group * a.group;
  part[tid] = sum;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const int v = tid >= off ? part[tid - off] : 0;
    __syncthreads();
    part[tid] += v;
    __syncthreads();
  }
  int run = part[tid] - sum;
  for (int c = lo; c < hi; ++c) {
    const int n = a.cnt[c], padded = (n + a.group - 1) / a.group * a.group;
    a.base[c] = run;
    for (int j = n; j < padded; ++j) a.pairs[run + j] = make_int2(-1, c);
    run += padded;
    a.cnt[c] = 0;   // left clear for the next pass over this workspace
  }
  if (tid == 1023) a.base[a.nlist] = part[1023];
}

// Head pass of a batch that one workgroup can sort: what lm_pairs_kernel, lm_offsets_kernel and lm_pairs_kernel do, the counts
// in LDS, and the clearing of zero_n counters, which would be a launch each (4.7 us, nearly all of it the launch).  us of a
// search, 64 subspaces, 32 probes, four launches / so: 512 queries 76.5 / 71.4, 1000 93.5 / 90.0, 2000 125.9 / 124.3, 3000
// 159.8 / 160.2, 4096 189.9 / 193.7, 10 000 344 / 353 (one CU waits for a line of the probes per query): up to 2048.
constexpr int LMH_THREADS = 1024, LMH_QUERIES = 2, LMH_LISTS = 16384;   // queries of a thread
__global__ __launch_bounds__(LMH_THREADS) void lm_head_pairs_kernel(LmArgs a, int64_t zero_n) {
  extern __shared__ __align__(16) unsigned char smem[];
  LDS uint32_t *cnt = (LDS uint32_t *)smem, *part = cnt + a.nlist;   // [nlist] pairs of a list, then where they begin; [LMH_THREADS]
  const int tid = threadIdx.x;
  for (int64_t i = tid; i < zero_n; i += LMH_THREADS) a.cnt[i] = 0;
  for (int i = tid; i < a.nlist; i += LMH_THREADS) cnt[i] = 0u;
  int32_t c[LMH_QUERIES], rank[LMH_QUERIES];
#pragma unroll
  for (int j = 0; j < LMH_QUERIES; ++j) {
    const int64_t q = tid + j * LMH_THREADS;
    c[j] = q < a.Q ? a.probe_ids[q * a.nprobe] : -1;
  }
#pragma unroll
  for (int j = 0; j < LMH_QUERIES; ++j) {
    const bool exists = (uint32_t)c[j] < (uint32_t)a.nlist;
    const int64_t len = exists ? a.list_offsets[c[j] + 1] - a.list_offsets[c[j]] : 0;
    rank[j] = len > 0 && len <= a.head_max ? 0 : -1;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < LMH_QUERIES; ++j) {
    const int64_t q = tid + j * LMH_THREADS;
    if (q >= a.Q) break;
    a.gcnt[q] = 0u;
    a.qmap_head[q] = rank[j] >= 0 ? -1 : (int32_t)q;
    if (rank[j] >= 0) rank[j] = (int32_t)__hip_atomic_fetch_add(&cnt[c[j]], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __syncthreads();
  const uint32_t g = (uint32_t)a.group;
  const int chunk = (a.nlist + LMH_THREADS - 1) / LMH_THREADS;
  const int lo = tid * chunk < a.nlist ? tid * chunk : a.nlist, hi = lo + chunk < a.nlist ? lo + chunk : a.nlist;
  uint32_t sum = 0;
  for (int x = lo; x < hi; ++x) sum += (cnt[x] + g - 1) / g * g;
  part[tid] = sum;
  __syncthreads();
  for (int off = 1; off < LMH_THREADS; off <<= 1) {
    const uint32_t v = tid >= off ? part[tid - off] : 0u;
    __syncthreads();
    part[tid] += v;
    __syncthreads();
  }
  uint32_t run = part[tid] - sum;
  for (int x = lo; x < hi; ++x) {
    const uint32_t n = cnt[x], padded = (n + g - 1) / g * g;
    for (uint32_t j = n; j < padded; ++j) a.pairs[run + j] = make_int2(-1, x);
    cnt[x] = run;
    run += padded;
  }
  if (tid == LMH_THREADS - 1) a.base[a.nlist] = (int32_t)part[tid];   // (all that is read of it behind this)
  __syncthreads();
#pragma unroll
  for (int j = 0; j < LMH_QUERIES; ++j) {
    const int64_t q = tid + j * LMH_THREADS;
    if (q >= a.Q) break;
    if (rank[j] >= 0) a.pairs[cnt[c[j]] + (uint32_t)rank[j]] = make_int2((int)q, c[j]);
  }
}

// 8-byte look-up of a point's code in an interleaved table row (2 KiB per row): the byte
// select of the sub-dword addressing form extracts the code and scales it by 8.
__device__ __forceinline__ uint32_t code_offset8(uint32_t w, int j) {
  uint32_t a;
  const uint32_t three = 3u;
  switch (j) {
    case 0: asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0" : "=v"(a) : "s"(three), "v"(w)); break;
    case 1: asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1" : "=v"(a) : "s"(three), "v"(w)); break;
    case 2: asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2" : "=v"(a) : "s"(three), "v"(w)); break;
    default: asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_3" : "=v"(a) : "s"(three), "v"(w)); break;
  }
  return a;
}

// d0 += table value of query 0, d1 += that of query 1, for subspaces [h, h1) in subspace order;
// the look-ups of a group are issued together and added afterwards (see lookup_group).
template <int MT>
__device__ __forceinline__ void lookup_group2(const CodeRegs<((MT + 3) / 4 * 4) / 4> &r, int h, int h1, float &d0,
                                              float &d1) {
  floatx2 t[LOOKUP_GROUP];
#pragma unroll
  for (int j = 0; j < LOOKUP_GROUP; ++j) {
    const int m = h + j;
    if (m < h1) {
      // the table starts at LDS address 0 (no static LDS: checked when the kernel is prepared)
      const uint32_t off = code_offset8(r.w[m >> 2], m & 3);
      t[j] = *(const LDS floatx2 *)(uintptr_t)(uint32_t)(m * 2048 + off);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < LOOKUP_GROUP; ++j)
    if (h + j < h1) {
      d0 += t[j][0];
      d1 += t[j][1];
    }
  __builtin_amdgcn_sched_barrier(0);
}

// Append a wavefront's queued candidates of one query to the query's buffer: `slot` is where
// the buffer's counter stood when the wavefront reserved its n entries.
__device__ __forceinline__ void lm_store(const LmArgs &a, int64_t q, uint32_t slot, LDS uint32_t *qd,
                                         LDS uint32_t *qrow, int n, int lane) {
  // past the capacity nothing is stored; the counter has grown all the same, which marks the
  // query as overflowed
  if (slot + (uint32_t)n <= (uint32_t)a.cap && lane < n)
    a.cand[q * a.cap + slot + lane] = make_uint2(qd[lane], qrow[lane]);
}

__device__ __forceinline__ void lm_flush(const LmArgs &a, int64_t q, LDS uint32_t *qd, LDS uint32_t *qrow, int n,
                                         int lane) {
  uint32_t slot = 0;
  if (lane == 0) slot = atomicAdd(&a.gcnt[q], (uint32_t)n);
  slot = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot);
  lm_store(a, q, slot, qd, qrow, n, lane);
}

// Offer a block's distances for one query: every valid point with distance <= tau is queued.
__device__ __forceinline__ void lm_offer(const LmArgs &a, int64_t q, float dist, bool valid, uint32_t tau,
                                         uint32_t row, LDS uint32_t *qd, LDS uint32_t *qrow, int &qcount, int lane) {
  const uint32_t bits = __float_as_uint(dist);
  const bool pass = valid && bits <= tau;
  const unsigned long long bal = __ballot(pass);
  if (bal == 0) return;
  const int n = __popcll(bal);
  if (qcount + n > LM_QUEUE) {
    lm_flush(a, q, qd, qrow, qcount, lane);
    qcount = 0;
  }
  if (pass) {
    const int slot = qcount + __popcll(bal & ((1ull << lane) - 1ull));
    qd[slot] = bits;
    qrow[slot] = row;
  }
  qcount += n;
}

// ---- head pass: exact top-k of ONE list per query, without a bound to filter by ----------
// The nearest list of a query has to be ranked in full.  Its distances (bit patterns of
// non-negative floats, which order like the values) are kept in LDS; a histogram of 1024 bins
// of equal width finds the bin of the k-th smallest, everything up to that bin is collected (k keys plus the few that share the last bin) and one wavefront per query
// sorts the collected keys by (distance, id).  More than LM_COLLECT collected keys (masses of
// equal distances) hand the query to the query-major kernel.

// bin b of a histogram lives at word (b % 16) * 64 + b / 16, so that lane l, which owns the 16
// consecutive bins 16 l .. 16 l + 15, reads them without bank conflicts
__device__ __forceinline__ uint32_t lds_add(LDS uint32_t *p) {   // LDS atomic increment, returns the old value
  return __hip_atomic_fetch_add(p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
constexpr int LM_BPL = LM_BINS / 64;   // bins per lane
__device__ __forceinline__ int lm_hidx(uint32_t bin) { return (int)(((bin % LM_BPL) << 6) | (bin / LM_BPL)); }

// One wavefront: the bin that holds the need-th smallest key (need >= 1, at most the number
// of keys counted) and the number of keys in the bins below it.
__device__ inline void lm_find_bin(const LDS uint32_t *hist, uint32_t need, int lane, uint32_t &bin, uint32_t &below) {
  uint32_t sum = 0;
  for (int j = 0; j < LM_BPL; ++j) sum += hist[j * 64 + lane];
  uint32_t incl = sum;
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t v = (uint32_t)__shfl_up((int)incl, off);
    if (lane >= off) incl += v;
  }
  const uint32_t excl = incl - sum;
  const bool mine = excl < need && need <= incl;   // exactly one lane
  uint32_t b = 0, bl = 0, run = excl;
  if (mine) {
    for (int j = 0; j < LM_BPL; ++j) {
      const uint32_t c = hist[j * 64 + lane];
      if (run < need && need <= run + c) {
        b = (uint32_t)LM_BPL * lane + j;
        bl = run;
      }
      run += c;
    }
  }
  const unsigned long long bal = __ballot(mine);
  const int src = bal ? __ffsll((long long)bal) - 1 : 0;
  bin = (uint32_t)__shfl((int)b, src);
  below = (uint32_t)__shfl((int)bl, src);
}

// One task: a list and the (up to) LM_G queries of a group that probe it.
struct LmTask {
  int32_t c;
  int64_t q0, q1;      // q1 == q0 when the group is half empty (has1 false): its copy is dropped
  bool has1;
  int64_t row0;
  int32_t len, nb;
  const uint8_t *base;
  float tauv;          // main pass: lane 0 holds tau of q0, the other lanes tau of q1 (a vector load, like the metadata)
};

// Head pass: the histogram's window.  No table entry exceeds its row's r_m^2, so a distance lies in [0, sum of the r_m^2]: with
// finite radii the window is known before the scan and every distance is counted as it is produced.  Otherwise (infinite
// radii) the window is the range the distances turn out to span, and they are counted in a pass of their own.  Bins have
// equal width in value; bin_of is monotone in the distance, which is all the selection needs.
struct LmWindow {
  float lo[2], scale[2];
  bool known;
  __device__ __forceinline__ uint32_t bin_of(int g, uint32_t key) const {
    const float x = (__uint_as_float(key) - (g ? lo[1] : lo[0])) * (g ? scale[1] : scale[0]);   // (selected: indexed, they would be in scratch)
    return x >= (float)(LM_BINS - 1) ? (uint32_t)(LM_BINS - 1) : (x > 0.0f ? (uint32_t)x : 0u);
  }
};
__device__ __forceinline__ LmWindow lm_window(const LDS float *sr2, int M, int lane) {
  float s0 = lane < M ? sr2[lane] : 0.0f, s1 = lane < M ? sr2[IVFPQ_MAX_M + lane] : 0.0f;
  if (lane + 64 < M) {   // (at most 128)
    s0 += sr2[lane + 64];
    s1 += sr2[IVFPQ_MAX_M + lane + 64];
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    s0 += __shfl_xor(s0, off);
    s1 += __shfl_xor(s1, off);
  }
  LmWindow w;
  w.known = s0 > 0.0f && s0 < __builtin_inff() && s1 > 0.0f && s1 < __builtin_inff();   // same in every wavefront
  w.lo[0] = w.lo[1] = 0.0f;
  w.scale[0] = (float)LM_BINS / s0;
  w.scale[1] = (float)LM_BINS / s1;
  return w;
}

// Head pass: the k nearest of a scanned list, for the queries of its task, from the distances in LDS.  The collected keys
// are held where the table was (`coll`).  AHEAD: LDS reads of the rank sort in flight.
template <int AHEAD>
__device__ __forceinline__ void lm_select_head(const LmArgs &a, const LmTask &done, LmWindow &w, uint32_t mn0, uint32_t mn1, uint32_t mx0, uint32_t mx1,
                                               LDS unsigned char *coll, LDS uint32_t *ssel, LDS uint32_t *hist, const LDS uint32_t *sdist,
                                               int tid, int lane, int wave) {
  LDS uint32_t *coll_d = (LDS uint32_t *)coll;             // [2][LM_COLLECT] collected keys: distance bits ...
  LDS uint32_t *coll_pos = coll_d + LM_G * LM_COLLECT;     // ... their positions in the list ...
  LDS uint32_t *coll_rank = coll_pos + LM_G * LM_COLLECT;  // ... and in sorted order
  const int L = done.len, k = a.k;
  const int ng = done.has1 ? 2 : 1;
  // window not known: smallest and largest key of each query's list (this wavefront's share first)
  if (!w.known)
    for (int g = 0; g < ng; ++g) {
      uint32_t lo = g ? mn1 : mn0, hi = g ? mx1 : mx0;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
        const uint32_t ol = (uint32_t)__shfl_xor((int)lo, off), oh = (uint32_t)__shfl_xor((int)hi, off);
        lo = ol < lo ? ol : lo;
        hi = oh > hi ? oh : hi;
      }
      if (lane == 0) {
        __hip_atomic_fetch_min(&ssel[4 + g], lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_fetch_max(&ssel[6 + g], hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
  __syncthreads();   // the list is scanned: every distance is in LDS and the table's LDS is free
  uint32_t top[2] = {LM_BINS, LM_BINS};   // collect keys whose bin is <= top (everything when the list is short)
  if (tid < LM_G * LM_COLLECT) {           // empty slots: the sentinel, and rank 0
    coll_d[tid] = SENT_D;
    coll_rank[tid] = 0u;
  }
  if (L <= LM_COLLECT) __syncthreads();    // (else the barriers of the histogram come before the slots are filled)
  if (L > LM_COLLECT) {                    // uniform; then k <= LM_COLLECT < L: the k-th smallest exists
    if (!w.known) {
      for (int g = 0; g < 2; ++g) {
        w.lo[g] = __uint_as_float(ssel[4 + g]);
        w.scale[g] = (float)LM_BINS / (__uint_as_float(ssel[6 + g]) - w.lo[g]);   // one value only: every key in bin 0
      }
      for (int i = tid; i < L; i += LM_NW * 64)
        for (int g = 0; g < ng; ++g) lds_add(&hist[g * LM_BINS + lm_hidx(w.bin_of(g, sdist[g * a.head_max + i]))]);
      __syncthreads();
    }
    if (wave < ng) {                       // wavefront g ranks query g's histogram
      uint32_t bin, below;
      lm_find_bin(hist + wave * LM_BINS, (uint32_t)k, lane, bin, below);
      if (lane == 0) ssel[2 + wave] = bin;
    }
    __syncthreads();
    top[0] = ssel[2];
    top[1] = ssel[3];
  }
  // collect (distance, position in the list) of the keys up to that bin; a wavefront reserves
  // the slots of its keys with one atomic operation
  for (int i0 = wave * 64; i0 < L; i0 += LM_NW * 64) {
    const int i = i0 + lane;
    for (int g = 0; g < ng; ++g) {
      const uint32_t key = i < L ? sdist[g * a.head_max + i] : 0u;
      const bool take = i < L && w.bin_of(g, key) <= top[g];
      const unsigned long long bal = __ballot(take);
      if (bal == 0ull) continue;
      uint32_t first = 0;
      if (lane == 0) first = __hip_atomic_fetch_add(&ssel[g], (uint32_t)__popcll(bal), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      first = (uint32_t)__builtin_amdgcn_readfirstlane((int)first);
      const uint32_t slot = first + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
      if (take && slot < (uint32_t)LM_COLLECT) {
        coll_d[g * LM_COLLECT + slot] = key;
        coll_pos[g * LM_COLLECT + slot] = (uint32_t)i;
      }
    }
  }
  __syncthreads();
  // Rank sort, all wavefronts: thread (query g, key i, half h) counts the keys of half h of
  // query g's collected keys that precede key i in (distance, id) order; the two halves add
  // up to the key's position in the sorted order.  Unused slots hold the sentinel, which
  // precedes nothing, so the count runs over a fixed 64 slots, four per LDS read.  The id of
  // a key is requested before the count and only needed after it; where distances tie (rare)
  // the ids of the tying keys are fetched on the spot.
  {
    const int g = tid >> 8, i = tid & (LM_COLLECT - 1), h = (tid >> 7) & 1;
    const uint32_t n = ssel[g];
    const bool live = g < ng && n <= (uint32_t)LM_COLLECT && (uint32_t)i < n;
    const uint32_t md = live ? coll_d[g * LM_COLLECT + i] : SENT_D;
    const uint32_t mpos = live ? coll_pos[g * LM_COLLECT + i] : 0u;
    int64_t mid = SENT_ID;
    if (live) mid = a.ids[done.row0 + mpos];
    uint32_t before = 0, ties = 0;
    const LDS uintx4 *half = (const LDS uintx4 *)(coll_d + g * LM_COLLECT + h * (LM_COLLECT / 2));
#pragma unroll AHEAD
    for (int j = 0; j < LM_COLLECT / 8; ++j) {
      const uintx4 od = half[j];
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        before += od[x] < md ? 1u : 0u;
        ties += od[x] == md ? 1u : 0u;
      }
    }
    if (live) {
      if (ties > ((i >> 6) == h ? 1u : 0u)) {
        const int j0 = h * (LM_COLLECT / 2);
        for (int j = j0; j < j0 + LM_COLLECT / 2 && j < (int)n; ++j)
          if (coll_d[g * LM_COLLECT + j] == md && a.ids[done.row0 + coll_pos[g * LM_COLLECT + j]] < mid) ++before;
      }
      if (before) __hip_atomic_fetch_add(&coll_rank[g * LM_COLLECT + i], before, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();
    const int64_t q = g ? done.q1 : done.q0;
    if (g < ng && h == 0) {
      if (n > (uint32_t)LM_COLLECT) {
        if (i == 0) a.qmap_head[q] = (int32_t)q;   // too many equal distances: left to the query-major kernel
      } else if ((uint32_t)i < n) {
        const uint32_t r = coll_rank[g * LM_COLLECT + i];
        if (r < (uint32_t)k) {
          a.out_ids[q * k + r] = mid;
          a.out_dist[q * k + r] = __uint_as_float(md);
        }
      } else if (i < k) {                           // fewer than k points in the list
        a.out_ids[q * k + i] = -1;
        a.out_dist[q * k + i] = __builtin_inff();
      }
    }
  }
}

// Persistent workgroups, one per CU.  Tasks are sorted by list; in every round the grid takes
// the next gridDim.x tasks, and within a round the workgroups of one XCD (workgroup b runs on
// XCD b % 8) take a run of consecutive tasks, so that the tasks which stream the same list's
// codes share an L2.  Everything a task needs from global memory -- its pair entries, the
// list's metadata, the two query rows, the centroid, the first code block -- is requested
// while the task before it is still being scanned, so that a workgroup (the only one on its
// CU: the interleaved table fills most of the LDS) does not sit idle through a chain of
// dependent loads at every task boundary.
// HEAD: the head pass -- a task's list is the nearest list of its queries; no bound exists yet,
// every distance is kept (in LDS) and the exact top-k of the list is selected per query and
// written to the query's output row, where the main pass and the merge find it.
template <int MT, int DSUB, bool HEAD>
__global__ __launch_bounds__(LM_NW * 64) __attribute__((amdgpu_waves_per_eu(LM_NW / 4))) void lm_scan_kernel(LmArgs a, RadiiSq r2) {
  constexpr int NW = LM_NW;
  constexpr int MPT = (MT + 3) / 4 * 4;
  constexpr int ITER = (MT + NW - 1) / NW;
  constexpr int NCH = MPT / 16 + (MPT % 16) / 4;
  extern __shared__ __align__(16) unsigned char smem[];
  LDS unsigned char *smem3 = (LDS unsigned char *)smem;
  const int D = a.D;   // LM_G * D <= NT and LM_G * MT <= NT: one element per thread (checked by the launcher)
  const int dpad = (D + 3) & ~3;
  // LDS carve: interleaved table [MT][256][2] | residuals [2][dpad] | r_m^2 [2][MAX_M] | queues
  LDS float *lut = (LDS float *)smem3;
  LDS float *sres = (LDS float *)(smem3 + MT * 2048);
  LDS float *sr2 = sres + LM_G * dpad;
  LDS uint32_t *queue = (LDS uint32_t *)(sr2 + LM_G * IVFPQ_MAX_M);  // main pass: [NW][G][2][LM_QUEUE]
  // head pass: selection state, the histograms, then the distances [2][head_max]; the
  // collected keys use the table's LDS once the list has been scanned
  LDS uint32_t *ssel = queue;                      // [LM_SEL_WORDS]
  LDS uint32_t *hist = queue + LM_SEL_WORDS;       // [2][LM_BINS]
  LDS uint32_t *sdist = hist + LM_G * LM_BINS;     // [2][head_max]

  int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  LDS uint32_t *qd0 = queue + (wave * LM_G + 0) * 2 * LM_QUEUE, *qrow0 = qd0 + LM_QUEUE;
  LDS uint32_t *qd1 = queue + (wave * LM_G + 1) * 2 * LM_QUEUE, *qrow1 = qd1 + LM_QUEUE;

  // this wavefront's codebook rows (rows wave, wave + NW, ...) stay in registers for the whole
  // kernel; the head pass at 64 subspaces has registers for six of its eight rows and fetches
  // the others (from the L2) when a task's table is built
  constexpr int RES = (HEAD && ITER > 6) ? 6 : ITER;
  float4 cbr[RES][DSUB];
  auto load_row = [&](int it, float4 (&row)[DSUB]) __attribute__((always_inline)) {
    const int m = wave + it * NW;
    const int mc = m < MT ? m : MT - 1;
    const GLOBAL uint8_t *cb = uniform_ptr(a.codebooks + (int64_t)mc * 256 * DSUB);
#pragma unroll
    for (int x = 0; x < DSUB; ++x)
      row[x] = load_f4(cb, (uint32_t)(lane * 16 * DSUB + 16 * x));
  };
#pragma unroll
  for (int it = 0; it < RES; ++it) load_row(it, cbr[it]);

  const int ntasks = a.base[a.nlist] / LM_G;
  const int nwg = gridDim.x, b = blockIdx.x;
  const int in_round = (nwg & 7) == 0 ? (b & 7) * (nwg >> 3) + (b >> 3) : b;

  // what this thread contributes to a task's residuals and radii: element tid of [2][D] / [2][MT]
  const int rg = tid >= D ? 1 : 0, rd = tid - rg * D;
  const bool r_on = tid < LM_G * D;
  const int mg = tid >= MT ? 1 : 0, mm = tid - mg * MT;
  const bool m_on = tid < LM_G * MT;

  // A task's pair entries and its list's metadata are requested with VECTOR loads (a lane each:
  // even lanes the first pair entry, odd lanes the second; lanes 0 and 1 the list's row range,
  // the others its first block), although every lane of the wavefront wants the same values:
  // scalar loads share their counter with the LDS, so a scalar load in flight makes the next
  // LDS read of the scan wait for it, whereas vector loads complete in order behind the code
  // stream and cost nothing when they are consumed a scan later.
  auto fetch_pairs = [&](int t) __attribute__((always_inline)) { return a.pairs[(int64_t)t * LM_G + (lane & 1)]; };
  auto fetch_meta = [&](const int2 &pv) __attribute__((always_inline)) {
    const int c = __builtin_amdgcn_readlane(pv.y, 0);
    const int64_t *src = lane < 2 ? a.list_offsets + c + lane : a.list_blocks + c;
    return *src;
  };
  auto lane64 = [&](int64_t v, int l) __attribute__((always_inline)) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
    return (int64_t)(((uint64_t)hi << 32) | lo);
  };
  // everything else a task needs, requested together: bounds, this thread's residual and radius
  // element, the wavefront's first code block
  auto fetch_task = [&](const int2 &pv, int64_t mv, LmTask &tk, float &qv, float &cv, float &rv,
                        CodeRegs<MPT / 4> &first) __attribute__((always_inline)) {
    tk.c = __builtin_amdgcn_readlane(pv.y, 0);
    tk.q0 = __builtin_amdgcn_readlane(pv.x, 0);
    tk.has1 = __builtin_amdgcn_readlane(pv.x, 1) >= 0;
    tk.q1 = tk.has1 ? __builtin_amdgcn_readlane(pv.x, 1) : tk.q0;
    tk.row0 = lane64(mv, 0);
    tk.len = (int)(lane64(mv, 1) - tk.row0);
    tk.nb = (tk.len + 63) >> 6;
    tk.base = a.codes + lane64(mv, 2) * ivfpq_block_bytes(MPT);
    tk.tauv = 0.0f;
    if constexpr (!HEAD) tk.tauv = a.out_dist[(lane == 0 ? tk.q0 : tk.q1) * a.k + a.k - 1];
    qv = cv = 0.0f;
    if (r_on) {
      qv = a.queries[(rg ? tk.q1 : tk.q0) * D + rd];
      cv = a.centroids[(int64_t)tk.c * D + rd];
    }
    rv = 0.0f;
    if (m_on) {
      rv = r2.v[mm];
      if (a.query_radii) {
        const float r = a.query_radii[(mg ? tk.q1 : tk.q0) * MT + mm];
        rv = r * r;
      }
    }
    const int b0 = wave < tk.nb ? wave : tk.nb - 1;   // nb >= 1: only non-empty lists have tasks
    load_chunks<MPT, 0, NCH>(tk.base, tk.nb, b0, lane, first);
  };

  LmTask tk;
  float qv, cv, rv;
  CodeRegs<MPT / 4> nxt;
  int t = in_round;
  if (t >= ntasks) return;
  int2 npv = make_int2(0, 0);   // pair entries of the next task
  {
    const int2 pv = fetch_pairs(t);
    if (t + nwg < ntasks) npv = fetch_pairs(t + nwg);
    fetch_task(pv, fetch_meta(pv), tk, qv, cv, rv, nxt);
  }
  // main pass: the candidates of the task before, queued in LDS, and where they go
  uint32_t pend_slot = 0;
  int64_t pend_q0 = 0, pend_q1 = 0;
  int pend_c0 = 0, pend_c1 = 0;
  auto drain_pending = [&]() __attribute__((always_inline)) {
    const uint32_t s0 = (uint32_t)__builtin_amdgcn_readlane((int)pend_slot, 0);
    const uint32_t s1 = (uint32_t)__builtin_amdgcn_readlane((int)pend_slot, 1);
    if (pend_c0 > 0) lm_store(a, pend_q0, s0, qd0, qrow0, pend_c0, lane);
    if (pend_c1 > 0) lm_store(a, pend_q1, s1, qd1, qrow1, pend_c1, lane);
    pend_c0 = pend_c1 = 0;
  };
  for (;;) {
    asm volatile("" : "+v"(tid), "+v"(lane));   // (addresses formed anew for every task: kept across tasks they spill)
    if (r_on) sres[rg * dpad + rd] = qv - cv;
    if (m_on) sr2[mg * IVFPQ_MAX_M + mm] = rv;
    if (HEAD && tid < LM_SEL_WORDS)   // [0..1] keys collected, [2..3] bin of the k-th key, [4..5] smallest key, [6..7] largest key
      ssel[tid] = (tid == 4 || tid == 5) ? 0xFFFFFFFFu : 0u;
    if constexpr (HEAD)
      for (int i = tid; i < LM_G * LM_BINS; i += NW * 64) hist[i] = 0u;
    __syncthreads();
    // ---- the two tables, interleaved: row m holds (query 0, query 1) of entry 0, of entry 1, ... ----
    auto build_rows = [&](auto mode_tag) __attribute__((always_inline)) {
      constexpr int MODE = decltype(mode_tag)::value;
      float4 cbs[ITER > RES ? ITER - RES : 1][DSUB];   // streamed rows, requested together
#pragma unroll
      for (int it = RES; it < ITER; ++it) load_row(it, cbs[it - RES]);
#pragma unroll
      for (int it = 0; it < ITER; ++it) {
        const int m = wave + it * NW;
        if (m < MT) {
          const float4 *row = it < RES ? cbr[it < RES ? it : 0] : cbs[it >= RES ? it - RES : 0];
          float res0[DSUB], res1[DSUB];
#pragma unroll
          for (int j = 0; j < DSUB; ++j) {
            res0[j] = sres[m * DSUB + j];
            res1[j] = sres[dpad + m * DSUB + j];
          }
          const float4 v0 = lut_entry4<DSUB, MODE>(res0, row, sr2[m]);
          const float4 v1 = lut_entry4<DSUB, MODE>(res1, row, sr2[IVFPQ_MAX_M + m]);
          LDS floatx4 *dst = (LDS floatx4 *)(lut + m * 512 + 8 * lane);
          dst[0] = floatx4{v0.x, v1.x, v0.y, v1.y};
          dst[1] = floatx4{v0.z, v1.z, v0.w, v1.w};
        }
      }
    };
    if (a.mode == 0) build_rows(std::integral_constant<int, 0>{});
    else if (a.mode == 1) build_rows(std::integral_constant<int, 1>{});
    else build_rows(std::integral_constant<int, 2>{});
    // on their way while this task is scanned: the next task's list metadata, the pair
    // entries of the task after it
    const int tn = t + nwg;
    const bool more = tn < ntasks;
    int64_t nmv = 0;
    int2 nnv = make_int2(0, 0);
    if (more) nmv = fetch_meta(npv);
    if (tn + nwg < ntasks) nnv = fetch_pairs(tn + nwg);
    if constexpr (!HEAD) drain_pending();   // the queues are free again before this task fills them
    __syncthreads();
    // ---- one pass over the list's codes serves both queries ----
    int qc0 = 0, qc1 = 0;
    uint32_t mn0 = 0xFFFFFFFFu, mn1 = 0xFFFFFFFFu, mx0 = 0u, mx1 = 0u;   // head pass: key range of this wavefront's points
    LmWindow win;
    if constexpr (HEAD) win = lm_window(sr2, MT, lane);
    // tau_q as the bit pattern of a non-negative float (orders like the value; +inf when the
    // first lists held fewer than k points)
    const uint32_t tau0 = (uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(tk.tauv), 0);
    const uint32_t tau1 = (uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(tk.tauv), 1);
    const int last = tk.nb - 1;
    for (int blk = wave; blk < tk.nb; blk += NW) {
      CodeRegs<MPT / 4> cur = nxt;
      const int bn = blk + NW < last ? blk + NW : last;
      load_chunks<MPT, 0, NCH>(tk.base, tk.nb, bn, lane, nxt);   // past the end: re-reads the last block, in bounds
      float d0 = 0.0f, d1 = 0.0f;
#pragma unroll
      for (int h = 0; h < MT; h += LOOKUP_GROUP) lookup_group2<MT>(cur, h, cmin(h + LOOKUP_GROUP, MT), d0, d1);
      const int i = blk * 64 + lane;
      const bool valid = i < tk.len;
      const uint32_t row = (uint32_t)(tk.row0 + i);
      if constexpr (HEAD) {
        if (valid) {
          const uint32_t k0 = __float_as_uint(d0), k1 = __float_as_uint(d1);
          sdist[i] = k0;
          sdist[a.head_max + i] = k1;
          if (win.known) {
            lds_add(&hist[lm_hidx(win.bin_of(0, k0))]);
            lds_add(&hist[LM_BINS + lm_hidx(win.bin_of(1, k1))]);
          } else {
            mn0 = k0 < mn0 ? k0 : mn0;
            mx0 = k0 > mx0 ? k0 : mx0;
            mn1 = k1 < mn1 ? k1 : mn1;
            mx1 = k1 > mx1 ? k1 : mx1;
          }
        }
      } else {
        lm_offer(a, tk.q0, d0, valid, tau0, row, qd0, qrow0, qc0, lane);
        if (tk.has1) lm_offer(a, tk.q1, d1, valid, tau1, row, qd1, qrow1, qc1, lane);
      }
    }
    // the rest of the next task's inputs is requested before this task's candidates are
    // appended: both wait on the memory system at the same time
    const LmTask done = tk;
    if (more) {
      fetch_task(npv, nmv, tk, qv, cv, rv, nxt);
      npv = nnv;
    }
    if constexpr (HEAD) {
      lm_select_head<16>(a, done, win, mn0, mn1, mx0, mx1, smem3, ssel, hist, sdist, tid, lane, wave);
    } else {
      // One atomic instruction reserves the space of both queues: lane g for query g.  Its
      // result is not waited for here: the queued candidates are written to the reserved slots
      // after the next task's table is built (drain_pending), so the round trip of the atomic
      // is hidden behind that work.
      pend_slot = 0;
      const int n_mine = lane == 0 ? qc0 : (lane == 1 ? qc1 : 0);
      if (n_mine > 0) pend_slot = atomicAdd(&a.gcnt[lane == 0 ? done.q0 : done.q1], (uint32_t)n_mine);
      pend_q0 = done.q0;
      pend_q1 = done.q1;
      pend_c0 = qc0;
      pend_c1 = qc1;
    }
    if (!more) {
      if constexpr (!HEAD) drain_pending();
      break;
    }
    t = tn;
    __syncthreads();  // every wavefront is done with the table and the residuals before the next task rewrites them
  }
}

// ---- main pass with byte tables -----------------------------------------------------------------
// What bounds the pass over the lists is the LDS: a wavefront's gather of 8 bytes per lane costs
// what one of 4 does (measured: 10.0 and 10.4 lanes per clock and CU), so the values that fit 8
// bytes decide.  With fp32 tables that is two queries' values; here it is EIGHT: a table entry
// holds one byte per query of the group.
//
// Distances: the byte is a LOWER BOUND on the fp32 table value in units of 1/s_q, floor(s_q v) (up
// to a known offset per row) cut off at LMB_TOP, so the sum of a point's bytes bounds its distance
// from below.  A point whose
// sum, in those units, lies above the query's k-th distance so far cannot enter the result and
// is dropped; every other point (a fraction of a percent) gets its distance in fp32 from the
// codebook itself (lm_settle_kernel), with the operations and in the order of the reference, and only that distance
// is compared, stored and ranked.  So the result is bit for bit that of the fp32 tables; the bytes
// only decide which sums need not be formed.  LMB_TOP = 63: four bytes add up within a byte, so
// a group of four subspaces costs two adds per four queries before the bytes are spread to
// 16-bit sums (64 x 63 < 2^16).
// Hit counts (Sec. 5.4): the penalties 0, 1, 2 ARE bytes, their sums (at most 2 MT <= 128) too:
// the byte sums are the result and nothing has to be recomputed.
//
// 1M x 96, 64 probes, 10 000 queries (every (query, list) pair scanned): 7.1 ms with two queries
// per fp32 table, 3.6 ms with byte tables and every task settling its candidates, 2.6 and 0.45 ms with
// lm_settle_kernel behind (0.2 of which the merge took before); hit counts, 5000 queries: 3.6, 1.4, 1.2 ms.
constexpr int LMB_NW = 16;      // wavefronts: one workgroup per CU (the table takes 2 KiB per subspace), 4 per SIMD
constexpr int LMB_QUEUE = 3072; // candidates a task holds; more go to the queries' slots one by one
constexpr int LMB_TOP = 63;
constexpr float LMB_RANGE = 9.0e4f;   // a value below it, and what is added to it, stay below 3 x 2^15

typedef uint16_t ushortx2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));

// What is wanted of a task, kept between its request and its use.
template <int DSUB>
struct LmbFetch {
  float q[DSUB], c[DSUB];   // lane m: subspace m of the query and of the list's centroid
  float r2, tau;
  uint32_t n;               // its candidates so far
  int32_t qid;              // the query (-1: the group has fewer)
};

// Floats of a (subspace, query) record, padded to whole 16-byte reads.
constexpr int lmb_rec(int dsub) { return dsub == 2 ? 4 : 8; }
constexpr int LMB_SMALL = 64;   // words: two sets of a task's limits and queries, the two queue counters, the head pass's counts
constexpr int LMB_BINS = 256;   // head pass: bins of a query's byte sums
constexpr int LMB_SPARE = 64;   // head pass: points of the k-th sum's bin offered beyond k
constexpr int lmb_shift(int mt) { return mt > 16 ? 4 : 2; }   // 63 mt >> shift < LMB_BINS
constexpr size_t lmb_lds(int mt, int dsub, bool head) {
  return (head ? (size_t)LMB_G * LMB_BINS * 4 + (size_t)mt * 4 : 0) + (size_t)mt * 2048 + (size_t)LMB_G * mt * (4 * lmb_rec(dsub) + 4 + 2) + (size_t)mt * 4 + (size_t)LMB_QUEUE * 4 + LMB_SMALL * 4;
}

// Candidates that a task's queue has no room for go straight to their queries' slots, with one atomic for all lanes: radii that
// hold next to nothing make most points of a list candidates, and an atomic for each took 20 ms of a search of 5.
// (A function of its own, so that the pass's registers are not shaped by it.)
__device__ __attribute__((noinline)) void lmb_spill(uint32_t *gcnt, uint2 *cand, uint32_t cap, const LDS int32_t *sq, bool over,
                                                    uint32_t g, uint32_t x, uint32_t row, int lane) {
  uint32_t mine = 0, before = 0;
  for (int y = 0; y < LMB_G; ++y) {
    const unsigned long long b = __ballot(over && g == (uint32_t)y);
    if (lane == y) mine = (uint32_t)__popcll(b);
    if (g == (uint32_t)y) before = (uint32_t)__popcll(b & ((1ull << lane) - 1ull));
  }
  uint32_t slot = 0;
  if (lane < LMB_G && mine > 0) slot = atomicAdd(&gcnt[sq[lane]], mine);
  slot = (uint32_t)__shfl((int)slot, (int)g) + before;
  if (over && slot < cap) cand[(int64_t)sq[g] * cap + slot] = make_uint2(x, row);
}

__device__ __forceinline__ uint32_t pick(uint32_t c, uint32_t a, uint32_t b) { return c ? a : b; }

// A task has two phases and a barrier behind each: the table (vector ALU and matrix units) and the pass
// over the codes (LDS).  What else a task needs is out of their way.  The next task's parameters are
// formed by wavefronts 8 to 15 behind their share of the blocks, while the others, which have one block
// more, still scan.  The candidates leave the LDS for the queries' slots in the shadow of the next
// table, and their fp32 distances are formed by lm_settle_kernel, query by query: settled here they cost
// 8.5 of a task's 30 thousand clocks, since every task had to put the codebook where the table was and had
// candidates (125) for half of the lanes.
//
// HEAD: the pass over every query's nearest list, without a k-th distance to compare with.  The list is passed over
// twice: the first pass counts the byte sums in a histogram per query (256 bins in LDS), the second one offers points up
// to a limit that the histogram gives:
//  - every point up to the bin of the k-th smallest sum and as much beyond as the bytes can have lost.  Where the units
//    are those of the largest radius, nothing but what lies outside its radius is cut off, at that radius' own value: a
//    byte is less than 1 below s v + offset and at most twice the raise above it, so k points have
//    s distance + offsets < sum_k + MT, and one as near has a sum of at most sum_k + MT + the raises.
//  - or, where that is more points than are worth settling (radii that hold next to nothing or, with units of their own,
//    nearly everything), the points below the bin of the k-th smallest sum and of that bin as many as make k and
//    LMB_SPARE.  Any k points will do: the k-th of their distances bounds the query's k-th distance, and the main pass starts over
//    from that with this list among the others (LM_SEEDED).  Nothing is asked of the bytes then but a good order.
// A point to settle costs about what 8 to 16 byte sums do, a table about a thousand.
// 8192 queries of 64 probes, k = 100, us with the fp32 head pass / with byte tables, every point the bytes cannot rule out offered /
// so: 64 subspaces, clustered, lists of 3906, radii that hold 0.25 of the entries 1253 / 983 / 1011, 0.5 1081 / 1789 / 994, 0.9
// 1076 / 4331 / 990; 16 subspaces, lists of 7812, infinite radii (query-major before) 889 / 3895 / 877.
// (With 64 subspaces eight registers spill, all of them once a task and outside of the passes over the list.)
template <int MT, int DSUB, int MODE, bool HEAD = false>
__global__ __launch_bounds__(LMB_NW * 64) __attribute__((amdgpu_waves_per_eu(4))) void lm_byte_kernel(LmArgs a, RadiiSq r2) {
  constexpr int NW = LMB_NW;
  constexpr int ITER = (MT + NW - 1) / NW;
  constexpr int NCH = MT / 16;
  constexpr int PW = lmb_rec(DSUB);
  static_assert(MT % 16 == 0 && MT <= 64, "whole chunks, one lane per subspace");
  extern __shared__ __align__(16) unsigned char smem[];
  LDS unsigned char *smem3 = (LDS unsigned char *)smem;
  // LDS carve: table [MT][256][8 bytes] | records [MT][8][PW]: distances -2 s residual, s; hit counts
  // residual, r_m^2 | constants [MT][8] | highest bytes [MT][8], 16 bits each | largest |entry|^2 of a subspace [MT] |
  // queue | small words
  LDS float *srec = (LDS float *)(smem3 + (size_t)MT * 2048);
  LDS float *scon = srec + MT * LMB_G * PW;
  LDS uint16_t *stop = (LDS uint16_t *)(scon + MT * LMB_G);
  LDS float *semax = (LDS float *)(stop + MT * LMB_G);
  LDS uint32_t *queue = (LDS uint32_t *)(semax + MT);
  LDS uint32_t *small = queue + LMB_QUEUE;
  // two sets: a task's are read until its candidates have left, when the next one's are already there
  LDS uint32_t *sT = small;                        // [2][8] sums below this are candidates
  LDS int32_t *sq = (LDS int32_t *)(small + 16);   // [2][8] queries
  LDS uint32_t *qn = small + 32;                   // [2] candidates offered to the queue
  LDS int32_t *room = (LDS int32_t *)(small + 40); // head pass: [8] points of the last bin below the limit that may still be offered
  LDS uint32_t *wraps = small + 48;                // [2][8] values of the query's table may wrap
  LDS uint32_t *hist = small + LMB_SMALL;          // head pass: [8][LMB_BINS], then the mean |entry|^2 of a subspace [MT]
  LDS float *semean = (LDS float *)(hist + LMB_G * LMB_BINS);

  int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  const int ntasks = a.base[a.nlist] / LMB_G;
  const int nwg = gridDim.x, b = blockIdx.x;
  int t = (nwg & 7) == 0 ? (b & 7) * (nwg >> 3) + (b >> 3) : b;   // runs of tasks per XCD, as in lm_scan_kernel
  if (t >= ntasks) return;

  // This wavefront's codebook rows, resident: lane l holds entries l, 64 + l, 128 + l, 192 + l of
  // each.
  float ent[ITER][4][DSUB];
#pragma unroll
  for (int it = 0; it < ITER; ++it) {
    const int m = wave + it * NW;   // < MT or not: MT is a multiple of NW
    float emax = 0.0f, esum = 0.0f;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const float *src = a.codebooks + ((int64_t)m * 256 + x * 64 + lane) * DSUB;
      float n2 = 0.0f;
#pragma unroll
      for (int j = 0; j < DSUB; ++j) {
        ent[it][x][j] = src[j];
        n2 = fmaf(src[j], src[j], n2);
      }
      emax = fmaxf(emax, n2);
      esum += n2;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) emax = fmaxf(emax, __shfl_xor(emax, off));
    if (lane == 0) semax[m] = emax;
    if constexpr (HEAD) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) esum += __shfl_xor(esum, off);
      if (lane == 0) semean[m] = esum * (1.0f / 256.0f);
    }
  }

  // (vector loads for what all lanes want alike: see lm_scan_kernel)
  auto fetch_pairs = [&](int t) __attribute__((always_inline)) { return a.pairs[(int64_t)t * LMB_G + (lane & (LMB_G - 1))]; };
  auto fetch_meta = [&](const int2 &pv) __attribute__((always_inline)) {
    const int c = __builtin_amdgcn_readlane(pv.y, 0);
    const int64_t *src = lane < 2 ? a.list_offsets + c + lane : a.list_blocks + c;
    return *src;
  };
  auto lane64 = [&](int64_t v, int l) __attribute__((always_inline)) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
    return (int64_t)(((uint64_t)hi << 32) | lo);
  };
  // wavefront 8 + g brings the parameters of query g: a lane per subspace
  constexpr int W0 = NW - LMB_G;
  auto fetch_params = [&](const int2 &pv, LmbFetch<DSUB> &f) __attribute__((always_inline)) {
    f.qid = -1;
    f.r2 = f.tau = 0.0f;
    f.n = 0u;
#pragma unroll
    for (int j = 0; j < DSUB; ++j) f.q[j] = f.c[j] = 0.0f;
    if (wave < W0) return;
    const int c = __builtin_amdgcn_readlane(pv.y, 0);
    const int q0 = __builtin_amdgcn_readlane(pv.x, 0);   // a task's first query exists
    f.qid = __builtin_amdgcn_readlane(pv.x, wave - W0);
    if (lane < MT) {
      const int64_t q = f.qid >= 0 ? f.qid : q0;
      if constexpr (DSUB == 2) {
        const float2 qv = *reinterpret_cast<const float2 *>(a.queries + q * a.D + 2 * lane);
        const float2 cv = *reinterpret_cast<const float2 *>(a.centroids + (int64_t)c * a.D + 2 * lane);
        f.q[0] = qv.x; f.q[1] = qv.y; f.c[0] = cv.x; f.c[1] = cv.y;
      } else {
        const float4 qv = *reinterpret_cast<const float4 *>(a.queries + q * a.D + 4 * lane);
        const float4 cv = *reinterpret_cast<const float4 *>(a.centroids + (int64_t)c * a.D + 4 * lane);
        f.q[0] = qv.x; f.q[1] = qv.y; f.q[2] = qv.z; f.q[3] = qv.w;
        f.c[0] = cv.x; f.c[1] = cv.y; f.c[2] = cv.z; f.c[3] = cv.w;
      }
      f.r2 = r2.v[lane];
      if (a.query_radii) {
        const float r = a.query_radii[q * MT + lane];
        f.r2 = fminf(r * r, __builtin_inff());   // (a NaN cuts nothing off, like an infinite radius)
      }
      if constexpr (!HEAD) {
        f.tau = a.tau[q * a.tau_stride];
        f.n = a.gcnt[q];
      }
    }
  };
  // ... and writes them to the records and to set `par` of the small words
  auto put_params = [&](const LmbFetch<DSUB> &f, int par) __attribute__((always_inline)) {
    if (wave < W0) return;
    const int g = wave - W0;
    const bool on = lane < MT;
    float res[DSUB];
#pragma unroll
    for (int j = 0; j < DSUB; ++j) res[j] = f.q[j] - f.c[j];
    const float tau = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(f.tau)));
    LDS float *rec = srec + (lane * LMB_G + g) * PW;
    uint32_t T, wrap = 0u;
    if constexpr (MODE == 0) {
      // Units: the largest r_m^2 (no table value exceeds it), or, where that is wider, four times
      // the mean value of a point within tau, maps to LMB_TOP; values beyond are cut off, which
      // keeps the sum a lower bound.  (Head pass: of a point at the mean distance, |r|^2 + the mean |e|^2.)
      float rr = 0.0f;
#pragma unroll
      for (int j = 0; j < DSUB; ++j) rr = fmaf(res[j], res[j], rr);
      const float far = on ? sqrtf(rr) + sqrtf(semax[lane]) : 0.0f;
      float rmax = a.rmax, mean = HEAD && on ? rr + semean[lane] : 0.0f;
      auto over_lanes = [&](auto fold) __attribute__((always_inline)) {
        fold([](float v) __attribute__((always_inline)) { return __shfl_xor(v, 32); });
        fold([](float v) __attribute__((always_inline)) { return __shfl_xor(v, 16); });
        fold([](float v) __attribute__((always_inline)) { return xor_f32<8>(v); });
        fold([](float v) __attribute__((always_inline)) { return xor_f32<4>(v); });
        fold([](float v) __attribute__((always_inline)) { return xor_f32<2>(v); });
        fold([](float v) __attribute__((always_inline)) { return xor_f32<1>(v); });
      };
      if (a.query_radii) {
        rmax = on ? f.r2 : 0.0f;
        over_lanes([&](auto other) __attribute__((always_inline)) { rmax = fmaxf(rmax, other(rmax)); });
      }
      if constexpr (HEAD) over_lanes([&](auto other) __attribute__((always_inline)) { mean += other(mean); });
      const float cap = fmaxf(fminf(rmax, (HEAD ? mean : tau) * (4.0f / (float)MT)), 1e-30f);
      const float s = ((float)LMB_TOP - 0.01f) / cap;   // infinite radii and no k-th distance: 0
      wrap = __ballot(on && !(s * far * far < LMB_RANGE)) != 0ull ? 1u : 0u;
      // Offset of a row: up to the next integer at the row's cap, so that entries outside the
      // radius (most of them) lose nothing to the floor; what the offsets add is known.
      const float x = fminf(f.r2, cap) * s, top = ceilf(x), off = top - x;
      // A byte is taken from the bits of 2^15 + value, whose last place is 2^-8: the DSUB + 2 roundings at
      // that magnitude move a value by 2^-9 each (RAISE counts one more), those of |r|^2 - 2 r.e + |e|^2 in place
      // of |r - e|^2 by 2^-24 of s (|r| + |e|)^2 each: fewer than 3 DSUB + 4 of them (REL counts four more).
      // The values are raised by that much, so that none is below 0.
      constexpr float RAISE = (DSUB + 3) / 512.0f, REL = (3 * DSUB + 8) / 16777216.0f;
      float add = 0.0f;
      if (on) {
        const float err = fmaf(s * far, far * REL, RAISE);
#pragma unroll
        for (int j = 0; j < DSUB; ++j) rec[j] = -2.0f * s * res[j];
        rec[DSUB] = s;
        scon[lane * LMB_G + g] = fmaf(rr, s, off + err) + 32768.0f;
        stop[lane * LMB_G + g] = (uint16_t)top;   // NaN (0 x inf): 0
        add = HEAD ? 2.0f * err : off + 2.0f * err;
      }
      // Limit on the byte sum of a point with distance <= tau: s tau, relative roundings (the fp32
      // sum, the scaling: 2^-23 each, at most 70 of them), the offsets, the raise and the roundings again.
      over_lanes([&](auto other) __attribute__((always_inline)) { add += other(add); });
      // (Head pass: what lies between the k-th smallest sum and the limit.)
      const float lim = HEAD ? add + (float)MT + 2.0f : fmaf(tau * s, 1.00001f, add) + 0.25f;
      T = lim < 60000.0f ? (uint32_t)lim : 60000u;   // NaN (0 x inf, or no k-th distance): every point
      if (HEAD && !(rmax <= cap)) T = 0u;            // values inside a radius are cut off
    } else {
      if (on) {
#pragma unroll
        for (int j = 0; j < DSUB; ++j) rec[j] = res[j];
        rec[DSUB] = f.r2;
      }
      T = tau < 60000.0f ? (uint32_t)tau : 60000u;
    }
    if (lane == 0) {
      wraps[par * 8 + g] = wrap;
      sT[par * 8 + g] = f.qid >= 0 && f.n <= (uint32_t)a.cap ? T + 1u : 0u;   // (a query out of slots is redone, and offers no more)
      sq[par * 8 + g] = f.qid;
      if (g == 0) qn[par] = 0u;
    }
  };

  int2 npv = make_int2(0, 0);   // pair entries of the next task
  LmbFetch<DSUB> fx;
  CodeRegs<MT / 4> nxt;
  int64_t row0;
  int list, len, nb;
  const uint8_t *base;
  auto take_meta = [&](const int2 &pv, int64_t mv) __attribute__((always_inline)) {
    list = __builtin_amdgcn_readlane(pv.y, 0);
    row0 = lane64(mv, 0);
    len = (int)(lane64(mv, 1) - row0);
    nb = (len + 63) >> 6;   // >= 1: only non-empty lists have tasks
    base = a.codes + lane64(mv, 2) * ivfpq_block_bytes(MT);
    load_chunks<MT, 0, NCH>(base, nb, wave < nb ? wave : nb - 1, lane, nxt);
  };
  // A task's candidates: their room is reserved when the list has been scanned, and they are
  // written once the next task's table is built, so that nothing waits for the atomic's way.
  uint32_t p_slot = 0, p_x = 0, p_row = 0;
  int32_t p_q = 0;
  bool p_has = false;
  uint32_t p_where = 0;   // lane that holds the first slot of the candidate's query, and the candidate's place behind it
  auto drain = [&]() __attribute__((always_inline)) {
    const uint32_t slot = (uint32_t)__shfl((int)p_slot, (int)(p_where & 7u)) + (p_where >> 3);
    if (p_has && slot < (uint32_t)a.cap) a.cand[(int64_t)p_q * a.cap + slot] = make_uint2(p_x, p_row);
    p_has = false;
  };
  if constexpr (HEAD)
    for (int i = tid; i < LMB_G * LMB_BINS; i += NW * 64) hist[i] = 0u;
  __syncthreads();   // semax
  {
    const int2 pv = fetch_pairs(t);
    if (t + nwg < ntasks) npv = fetch_pairs(t + nwg);
    const int64_t mv = fetch_meta(pv);
    fetch_params(pv, fx);
    take_meta(pv, mv);
    put_params(fx, 0);
  }
  __syncthreads();
  for (int par = 0;; par ^= 1) {
    // (the addresses of all phases are formed anew for every task: kept across tasks, they took 60
    // registers that are not there)
    asm volatile("" : "+v"(tid), "+v"(lane));
    // ---- the table: row m holds, entry by entry, one byte per query ----
    // Distances: s |r - e|^2 + offset as a product of depth DSUB + 1 on the matrix units, four
    // queries (rows) by 64 entries (columns, a lane each) at a time.  The sums carry 2^15, so bits 8
    // to 23 are a value's whole part, or 2^15 and more where it does not fit.  From 3 x 2^15 on they wrap: where entries lie that
    // far out (the largest radius is 1/38 of the way to them or less) the sums are cut off there.  Per four
    // values two permutations that pair those bits, two minima with the rows' highest bytes and
    // one permutation that collects the bytes.  This phase is bound by what a SIMD's four wavefronts issue (9.2
    // thousand clocks for 48 subspaces): a median and a conversion to a byte per value, conversions to normalised
    // 16 bits, or half of the products on the vector ALU all took as long to 3 %.
    const bool five = sq[par * 8 + 4] >= 0;   // uniform
    auto build_table = [&](auto cut) __attribute__((always_inline)) {
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
      const int m = wave + it * NW;
      float nrm[4];   // |entry|^2, formed anew for every task like the addresses
#pragma unroll
      for (int x = 0; x < 4 && MODE == 0; ++x) {
        float e0 = ent[it][x][0];
        asm volatile("" : "+v"(e0));
        nrm[x] = e0 * e0;
#pragma unroll
        for (int j = 1; j < DSUB; ++j) nrm[x] = fmaf(ent[it][x][j], ent[it][x][j], nrm[x]);
      }
      uint32_t w[2][4];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int x = 0; x < 4; ++x) w[h][x] = 0u;
        if (h == 1 && !five) break;
        if constexpr (MODE == 0) {
          const floatx4 con = *(const LDS floatx4 *)(scon + m * LMB_G + 4 * h);
          const LDS ushortx2 *top = (const LDS ushortx2 *)(stop + m * LMB_G + 4 * h);
          const ushortx2 top01 = top[0], top23 = top[1];
          auto bytes_of = [&](const floatx4 &acc) __attribute__((always_inline)) {
            uint32_t b[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              b[g] = __float_as_uint(acc[g]);
              if constexpr (decltype(cut)::value) b[g] = umin32(b[g], 0x47C00000u);   // 3 x 2^15 (bits of positive numbers order like them)
            }
            const uint32_t v01 = __builtin_amdgcn_perm(b[1], b[0], 0x06050201u);
            const uint32_t v23 = __builtin_amdgcn_perm(b[3], b[2], 0x06050201u);
            const ushortx2 lo = __builtin_elementwise_min(__builtin_bit_cast(ushortx2, v01), top01);
            const ushortx2 hi = __builtin_elementwise_min(__builtin_bit_cast(ushortx2, v23), top23);
            return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, hi), __builtin_bit_cast(uint32_t, lo), 0x06040200u);
          };
          const LDS float *fac = srec + (m * LMB_G + 4 * h + (lane & 3)) * PW;   // row lane % 4 of every 4 x 4 block
          float f[DSUB + 1];
          const floatx4 f0 = *(const LDS floatx4 *)fac;
#pragma unroll
          for (int j = 0; j < DSUB; ++j) f[j] = f0[j];
          f[DSUB] = DSUB == 2 ? f0[2] : fac[4];
#pragma unroll
          for (int y = 0; y < 4; y += 2) {   // two chains of products side by side
            floatx4 acc[2] = {con, con};
#pragma unroll
            for (int j = 0; j < DSUB; ++j)
#pragma unroll
              for (int x = 0; x < 2; ++x) acc[x] = __builtin_amdgcn_mfma_f32_4x4x1f32(f[j], ent[it][y + x][j], acc[x], 0, 0, 0);
#pragma unroll
            for (int x = 0; x < 2; ++x) acc[x] = __builtin_amdgcn_mfma_f32_4x4x1f32(f[DSUB], nrm[y + x], acc[x], 0, 0, 0);
#pragma unroll
            for (int x = 0; x < 2; ++x) w[h][y + x] = bytes_of(acc[x]);
          }
        } else {
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const LDS float *rec = srec + (m * LMB_G + 4 * h + g) * PW;
            const floatx4 p0 = *(const LDS floatx4 *)rec;
            const float rm2 = DSUB == 2 ? p0[2] : rec[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
              const float t0 = p0[0] - ent[it][x][0];
              float d2 = t0 * t0;
#pragma unroll
              for (int j = 1; j < DSUB; ++j) {
                const float tj = p0[j] - ent[it][x][j];
                d2 = fmaf(tj, tj, d2);
              }
              if constexpr (MODE == 1) w[h][x] |= d2 <= rm2 ? 0u : (1u << (8 * g));
              else w[h][x] |= d2 <= 0.25f * rm2 ? 0u : (d2 <= rm2 ? (1u << (8 * g)) : (2u << (8 * g)));
            }
          }
        }
      }
#pragma unroll
      for (int x = 0; x < 4; ++x) *(LDS uintx2 *)(smem3 + m * 2048 + (x * 64 + lane) * 8) = uintx2{w[0][x], w[1][x]};
      __builtin_amdgcn_sched_barrier(0);   // a row at a time: their temporaries together do not fit the registers
    }
    };
    if (MODE == 0 && __ballot(wraps[par * 8 + (lane & 7)] != 0u) != 0ull) build_table(std::true_type{});
    else build_table(std::false_type{});
    const int tn = t + nwg;
    const bool more = tn < ntasks;
    int64_t nmv = 0;
    int2 nnv = make_int2(0, 0);
    if (more) {
      nmv = fetch_meta(npv);
      fetch_params(npv, fx);
    }
    if (tn + nwg < ntasks) nnv = fetch_pairs(tn + nwg);
    if (__ballot(p_has) != 0) drain();
    __syncthreads();   // the table is complete; the queue has been read
    // ---- one pass over the list's codes serves all queries of the group ----
    // sums of queries (0, 2), (1, 3), (4, 6), (5, 7) as 16-bit halves
    const int last = nb - 1;
    auto each_block = [&](auto use) __attribute__((always_inline)) {
    for (int blk = wave; blk < nb; blk += NW) {
      CodeRegs<MT / 4> cur = nxt;
      load_chunks<MT, 0, NCH>(base, nb, blk + NW < last ? blk + NW : last, lane, nxt);   // past the end: the last block again
      uint32_t s[4] = {0u, 0u, 0u, 0u}, raw0 = 0u, raw1 = 0u;
      auto high_bytes = [](uint32_t x) __attribute__((always_inline)) {   // both halves shifted at once
        return __builtin_bit_cast(uint32_t, (ushortx2)(__builtin_bit_cast(ushortx2, x) >> (ushortx2){8, 8}));
      };
#pragma unroll
      for (int h = 0; h < MT; h += 8) {
        uintx2 v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const uint32_t off = code_offset8(cur.w[(h + j) >> 2], j & 3);   // the table starts at LDS address 0
          v[j] = *(const LDS uintx2 *)(uintptr_t)(uint32_t)((h + j) * 2048 + off);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 8; j += 4) {   // four bytes below 64 add up within a byte
          const uint32_t x0 = (v[j][0] + v[j + 1][0] + v[j + 2][0]) + v[j + 3][0];
          const uint32_t x1 = (v[j][1] + v[j + 1][1] + v[j + 2][1]) + v[j + 3][1];
          if constexpr (MODE == 0) {
            s[0] += x0 & 0x00FF00FFu;
            s[1] += high_bytes(x0);
            s[2] += x1 & 0x00FF00FFu;
            s[3] += high_bytes(x1);
          } else {
            raw0 += x0;
            raw1 += x1;
          }
        }
        if constexpr (MODE != 0) asm volatile("" : "+v"(raw0), "+v"(raw1));   // (nor are these left for the end)
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (MODE != 0) {
        s[0] = raw0 & 0x00FF00FFu;
        s[1] = high_bytes(raw0);
        s[2] = raw1 & 0x00FF00FFu;
        s[3] = high_bytes(raw1);
      }
      if constexpr (HEAD)   // (the sums of queries 4 to 7 are formed here, not where they are first wanted, with every look-up kept until then)
        asm volatile("" : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]), "+v"(s[3]));
      use(blk * 64 + lane, s);
    }
    };
    if constexpr (HEAD) {
      each_block([&](int i, const uint32_t (&s)[4]) __attribute__((always_inline)) {
        if (i >= len) return;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const int g0 = (x >> 1) * 4 + (x & 1);
          if (x < 2 || five) {
            lds_add(&hist[g0 * LMB_BINS + ((s[x] & 0xFFFFu) >> lmb_shift(MT))]);
            lds_add(&hist[(g0 + 2) * LMB_BINS + (s[x] >> (16 + lmb_shift(MT)))]);
          }
        }
      });
      __syncthreads();
      if (wave < LMB_G) {   // wavefront g: the bin of query g's k-th smallest sum, four bins a lane
        const uintx4 c = *(const LDS uintx4 *)(hist + wave * LMB_BINS + 4 * lane);
        const uint32_t sum = c[0] + c[1] + c[2] + c[3];
        uint32_t incl = sum;
        for (int off = 1; off < 64; off <<= 1) {
          const uint32_t v = (uint32_t)__shfl_up((int)incl, off);
          if (lane >= off) incl += v;
        }
        uint32_t run = incl - sum, need = (uint32_t)a.k, bin = LMB_BINS, below = 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (run < need && need <= run + c[j]) {
            bin = (uint32_t)(4 * lane + j);
            below = run;
          }
          run += c[j];
        }
        const unsigned long long bal = __ballot(bin != (uint32_t)LMB_BINS);   // at most one lane
        const uint32_t has = sT[par * 8 + wave];                              // 0: no query
        int32_t spare = INT_MAX;
        if (has != 0u) {
          uint32_t limit = 60001u;   // fewer than k points: all of them
          if (bal != 0ull) {
            const int at = (int)__builtin_ctzll(bal);
            bin = (uint32_t)__builtin_amdgcn_readlane((int)bin, at);
            below = (uint32_t)__builtin_amdgcn_readlane((int)below, at);
            limit = umin32(((bin + 1u) << lmb_shift(MT)) - 1u + has, 60001u);
            const uint32_t last = (limit - 1u) >> lmb_shift(MT);
            uint32_t n = 0;   // points in the bins up to the limit's
#pragma unroll
            for (int j = 0; j < 4; ++j) n += (uint32_t)(4 * lane + j) <= last ? c[j] : 0u;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) n += (uint32_t)__shfl_xor((int)n, off);
            if (has == 1u || n > (uint32_t)a.cap || 8u * n > (uint32_t)len + 1024u + 8u * (need + 2u * LMB_SPARE)) {
              limit = (bin + 1u) << lmb_shift(MT);
              spare = (int32_t)(need - below + LMB_SPARE);
            }
          }
          if (lane == 0) {
            sT[par * 8 + wave] = limit;
            if (spare != INT_MAX) a.qmap_head[sq[par * 8 + wave]] = LM_SEEDED;
          }
        }
        if (lane == 0) room[wave] = spare;
      }
      __syncthreads();
      asm volatile("" : "+v"(tid), "+v"(lane));
      for (int i = tid; i < LMB_G * LMB_BINS; i += NW * 64) hist[i] = 0u;   // for the next task
      load_chunks<MT, 0, NCH>(base, nb, wave < nb ? wave : nb - 1, lane, nxt);   // the second pass starts over
    }
    // the limits to compare with
    uint32_t lim[4], seeds = 0u;   // head pass: bit g: query g is offered just enough points
    if constexpr (HEAD) seeds = (uint32_t)(__ballot(room[lane & (LMB_G - 1)] != INT_MAX) & 0xFFull);
    {
      const LDS uint32_t *T = sT + par * 8;
      lim[0] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(T[0] | (T[2] << 16)));
      lim[1] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(T[1] | (T[3] << 16)));
      lim[2] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(T[4] | (T[6] << 16)));
      lim[3] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(T[5] | (T[7] << 16)));
    }
    each_block([&](int i, const uint32_t (&s)[4]) __attribute__((always_inline)) {
      uint32_t z[4], any = 0u;   // limit - sum, saturated at 0: non-zero halves are candidates
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        z[x] = __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(ushortx2, lim[x]), __builtin_bit_cast(ushortx2, s[x])));
        any |= z[x];
      }
      if (__ballot(i < len && any != 0u) == 0) return;
      uint32_t mask = 0u;   // bit g: the point is a candidate of query g
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int g0 = (x >> 1) * 4 + (x & 1);
        mask |= (z[x] & 0xFFFFu) ? 1u << g0 : 0u;
        mask |= (z[x] >> 16) ? 4u << g0 : 0u;
      }
      if (i >= len) mask = 0u;
      for (unsigned long long bal = __ballot(mask != 0u); bal != 0; bal = __ballot(mask != 0u)) {
        bool take = mask != 0u, over = false;   // (over: no room in the queue)
        uint32_t g = 0u, word = 0u;
        if (take) {
          g = (uint32_t)__ffs((int)mask) - 1u;
          mask &= mask - 1u;
        }
        if constexpr (HEAD) {   // of the last bin no more than there is room for
          if (take && ((seeds >> g) & 1u)) {
            const uint32_t zz = (g & 4u) ? ((g & 1u) ? z[3] : z[2]) : ((g & 1u) ? z[1] : z[0]);
            if (((g & 2u) ? zz >> 16 : zz & 0xFFFFu) <= (1u << lmb_shift(MT)))
              take = room[g] > 0 && __hip_atomic_fetch_sub(&room[g], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > 0;
          }
          bal = __ballot(take);
          if (bal == 0ull) continue;
        }
        uint32_t first = 0;
        if (lane == 0) first = __hip_atomic_fetch_add(&qn[par], (uint32_t)__popcll(bal), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        first = (uint32_t)__builtin_amdgcn_readfirstlane((int)first);
        if (take) {
          const uint32_t pos = first + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
          word = ((uint32_t)i << 3) | g;
          if constexpr (MODE != 0) {   // the score travels with the point (at most 2 MT <= 128)
            const uint32_t s0 = s[0], s1 = s[1], s2 = s[2], s3 = s[3];   // (picked by value: by place, every block's sums went to scratch memory)
            const uint32_t lo = pick(g & 1u, s1, s0), hi = pick(g & 1u, s3, s2), zz = pick(g & 4u, hi, lo);
            word = ((uint32_t)i << 11) | (((g & 2u) ? zz >> 16 : zz & 0xFFFFu) << 3) | g;
          }
          if (pos < (uint32_t)LMB_QUEUE) queue[pos] = word;
          else over = true;
        }
        // straight to the queries' slots (the head pass offers no query more than it has slots)
        if constexpr (HEAD) {
          if (over) {
            const int64_t q = sq[par * 8 + g];
            const uint32_t slot = atomicAdd(&a.gcnt[q], 1u);
            if (slot < (uint32_t)a.cap) a.cand[q * a.cap + slot] = make_uint2((uint32_t)list, (uint32_t)(row0 + i));
          }
        } else if (__ballot(over) != 0) {
          lmb_spill(a.gcnt, a.cand, (uint32_t)a.cap, sq + par * 8, over, g,
                    MODE == 0 ? (uint32_t)list : __float_as_uint((float)((word >> 3) & 255u)), (uint32_t)(row0 + i), lane);
        }
      }
    });
    if (more) put_params(fx, par ^ 1);
    __syncthreads();   // the list is scanned: the queue is complete, the next task's records are there
    const int n = (int)umin32(qn[par], (uint32_t)LMB_QUEUE);
    const int64_t drow0 = row0;
    const int dlist = list;
    if (more) {
      take_meta(npv, nmv);
      npv = nnv;
    }
    for (int e0 = wave * 64; e0 < n; e0 += NW * 64) {
      if (__ballot(p_has) != 0) drain();
      const bool live = e0 + lane < n;
      const uint32_t word = live ? queue[e0 + lane] : 0u;
      const uint32_t g = word & 7u, i = word >> (MODE == 0 ? 3 : 11);
      // one atomic instruction reserves the room of all queries: lane g for query g
      uint32_t mine = 0, before = 0;
#pragma unroll
      for (int x = 0; x < LMB_G; ++x) {
        const unsigned long long bal = __ballot(live && g == (uint32_t)x);
        if (lane == x) mine = (uint32_t)__popcll(bal);
        if (g == (uint32_t)x) before = (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
      }
      p_slot = 0;
      if (lane < LMB_G && mine > 0) p_slot = atomicAdd(&a.gcnt[sq[par * 8 + lane]], mine);
      p_where = (before << 3) | g;
      p_x = MODE == 0 ? (uint32_t)dlist : __float_as_uint((float)((word >> 3) & 255u));
      p_row = (uint32_t)(drow0 + i);
      p_q = sq[par * 8 + g];
      p_has = live;
    }
    if (!more) {
      if (__ballot(p_has) != 0) drain();
      break;
    }
    t = tn;
  }
}

#include "scan_lm_parts.h"
#include "scan_lm_pairs.h"

// What follows a pass with byte tables of distances: the queries that have candidates are listed (in the place of
// the pairs, whose groups have all been served), the queries to be redone marked and, behind the last pass of a
// large batch (list_redo), listed too.  (One atomic per list and wavefront of 64 queries.)
__global__ __launch_bounds__(256) void lm_sort_out_kernel(LmArgs a, int list_redo) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int lane = threadIdx.x & 63;
  bool named = false, active = false;
  if (q < a.Q && a.wide_n) {
    const uint32_t n = a.gcnt[q];
    const int32_t n0 = a.wide_n[q];
    active = n0 >= 0 && n > (uint32_t)n0 && n <= (uint32_t)a.cap;
    a.qmap[q] = n0;                                            // from here on lm_settle_kernel settles
    if (n > (uint32_t)a.cap) a.wide_n[q] = -1;                 // its slots did not suffice
    else if (active) a.wide_n[q] = (int32_t)n;
  } else if (q < a.Q) {
    const uint32_t n = a.gcnt[q];
    named = n > (uint32_t)a.cap || ((a.head_done || a.fresh) && a.qmap_head[q] >= 0) || (a.later && a.qmap[q] >= 0);
    active = !named && n > 0u;
    if (!a.fresh) a.qmap[q] = named ? (int32_t)q : -1;
    else if (named) a.qmap_head[q] = (int32_t)q;
  }
  auto put = [&](bool on, int32_t *count, int32_t *list) __attribute__((always_inline)) {
    const unsigned long long bal = __ballot(on);
    if (bal == 0ull) return;
    int first = 0;
    if (lane == 0) first = atomicAdd(count, __popcll(bal));
    first = __builtin_amdgcn_readfirstlane(first);
    if (on) list[first + __popcll(bal & ((1ull << lane) - 1ull))] = (int32_t)q;
  };
  put(active, a.cnt + a.nlist + 2 + 2 * a.stage, (int32_t *)a.pairs);
  if (list_redo) put(named, a.cnt + a.nlist, a.redo);
}

// One wavefront per query: the candidates of the list-major scan are merged into the top-k of
// the first lists by (distance, id).  Queries whose buffer overflowed are handed to the
// query-major kernel through qmap.  What may enter is queued in LDS and folded in 64 at a time, the next 64 slots on
// their way meanwhile (a sort and a fetch of ids for every 64 slots of which one may enter, each after its loads:
// hit counts of 5000 queries, 1M x 96, both rounds: 227 us, 88 so).
constexpr int LMQ_WORDS = 128;   // of a queue: fewer than 64 waiting and the 64 of a group

// Names a query that is to be redone; whether it is.
__device__ __forceinline__ bool name_query(const LmArgs &a, int64_t q, bool write) {
  const bool overflow = a.gcnt[q] > (uint32_t)a.cap || (a.head_done && a.qmap_head[q] >= 0) || (a.later && a.qmap[q] >= 0);
  if (write) a.qmap[q] = overflow ? (int32_t)q : -1;
  return overflow;
}

__device__ __forceinline__ void merge_query(const LmArgs &a, int64_t q, int lane, LDS uint32_t *qd, LDS uint32_t *qrow) {
  const uint32_t n = a.gcnt[q];
  if (name_query(a, q, lane == 0) || n == 0) return;   // redone elsewhere / phase A's result stands
  const int k = a.k;
  Key L0, L1;
  {
    const int64_t o = q * k;
    const bool in0 = lane < k, in1 = 64 + lane < k;
    const int64_t id0 = in0 ? a.out_ids[o + lane] : -1, id1 = in1 ? a.out_ids[o + 64 + lane] : -1;
    L0.d = id0 >= 0 ? __float_as_uint(a.out_dist[o + lane]) : SENT_D;
    L0.id = id0 >= 0 ? id0 : SENT_ID;
    L1.d = id1 >= 0 ? __float_as_uint(a.out_dist[o + 64 + lane]) : SENT_D;
    L1.id = id1 >= 0 ? id1 : SENT_ID;
  }
  Key tau;
  {
    const Key t0 = bcast_key(L0, (k - 1) & 63), t1 = bcast_key(L1, (k - 1) & 63);
    tau = (k - 1) < 64 ? t0 : t1;
  }
  const uint2 *slots = a.cand + q * a.cap;
  auto slot_of = [&](uint32_t u) __attribute__((always_inline)) { return slots[u + lane < n ? u + lane : n - 1]; };
  int waiting = 0;
  uint2 e = slot_of(0);
  for (uint32_t off = 0; off < n; off += 64) {
    const uint2 next = slot_of(off + 64);
    const bool in = off + lane < n && e.x <= tau.d;   // a larger distance fails whatever its id
    const unsigned long long bal = __ballot(in);
    if (in) {
      const int pos = waiting + __popcll(bal & ((1ull << lane) - 1ull));
      qd[pos] = e.x;
      qrow[pos] = e.y;
    }
    waiting += __popcll(bal);
    while (waiting >= 64 || (waiting > 0 && off + 64 >= n)) {   // the last 64, at the end all
      const int m = waiting < 64 ? waiting : 64;
      waiting -= m;
      Key c;
      c.d = SENT_D;
      c.id = SENT_ID;
      if (lane < m) {
        c.d = qd[waiting + lane];
        if (c.d <= tau.d) c.id = a.ids[qrow[waiting + lane]];
      }
      const bool pass = kless(c, tau);
      if (__ballot(pass) == 0) continue;
      if (!pass) {
        c.d = SENT_D;
        c.id = SENT_ID;
      }
      wave_sort_desc<true>(c, lane);
      wave_merge<true>(L0, L1, c, lane);
      const Key t0 = bcast_key(L0, (k - 1) & 63), t1 = bcast_key(L1, (k - 1) & 63);
      tau = (k - 1) < 64 ? t0 : t1;
    }
    e = next;
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const Key e = h ? L1 : L0;
    const int i = h * 64 + lane;
    if (i < k) {
      const bool real = e.d != SENT_D;
      a.out_ids[q * k + i] = real ? e.id : -1;
      a.out_dist[q * k + i] = real ? __uint_as_float(e.d) : __builtin_inff();
    }
  }
}

// ---- the candidates of the byte tables: distances in fp32, merged into the queries' results --------
// One wavefront per query at a time, a lane per candidate: the entries come from the codebook, which the
// workgroup keeps in its LDS (one workgroup of 16 wavefronts per CU; the queries that have candidates are taken up one by one), the
// query's row and radii through scalar registers, the centroid's row from the L2 (a query's candidates
// stand in its slots in runs of the same list, so few lines serve a wavefront).  The operations and their order are those of the reference.
// A candidate within the k-th distance so far is queued, and 64 at a time are folded into the query's
// sorted list.  Three requests are in flight while a group of 64 is summed: the next group's codes, its lists'
// ranges before them, and the slots of the group after it.
constexpr int LMS_NW = 16;
// Slots a wavefront settles at a time for the wide selection, where a query's are independent.  1M x 128, 2000 queries
// of 32 probes, k = 1000: 581 us with a query a wavefront, 224 so.
constexpr int LMS_PIECE = 512;
constexpr int LMS_QUEUE = LMQ_WORDS;
// Rows of the codebook in LDS.  200 KiB of 100 rows do not fit: the last 36 are looked up in the L2.
constexpr int lms_rows(int mt) { return mt <= 64 ? mt : 64; }
constexpr size_t lms_lds(int mt, int dsub) { return (size_t)lms_rows(mt) * 1024 * dsub + (size_t)LMS_NW * (LMS_QUEUE * 8 + mt * 4) + 16; }
#define CONSTANT __attribute__((address_space(4)))

// WIDE: behind the wide selection's first lists.  A candidate's distance and row take its slot; those beyond the bound
// are left to wide_select_kernel, which picks the k nearest of a query's slots.
// PLACE: the wavefronts of a workgroup share its queries' slots piece by piece; a candidate's distance and row take its
// slot, and when all are settled a wavefront each ranks the queries, as lm_merge_kernel does.  With a wavefront a query (MERGE)
// few queries leave most wavefronts idle, and one that has many candidates keeps its workgroup waiting.  1M points, 32
// probes, without structure, us of a search with every task settling its own candidates / MERGE / PLACE: 512 queries,
// 16 subspaces, k = 10 129 / 166 / 122, k = 100 201 / 222 / 149, 48, k = 100 200 / 225 / 176; 2048, 16, k = 100 409 / 376 / 310;
// 8192, 16, k = 100 1255 / 1026 / 959, 48 1695 / 1384 / 1325; clustered, 512 queries, 16, k = 10 69 / 73 / 68 (a launch less than MERGE).
enum { LMS_MERGE, LMS_WIDE, LMS_PLACE };
constexpr int LMS_SHARE = 128;   // slots of such a piece
template <int MT, int DSUB, int HOW>
__global__ __launch_bounds__(LMS_NW * 64) __attribute__((amdgpu_waves_per_eu(4))) void lm_settle_kernel(LmArgs a, RadiiSq r2) {
  constexpr int NCH = MT / 16, TAIL = MT % 16, ROWS = lms_rows(MT);
  constexpr bool AT_ONCE = MT <= 64;
  static_assert(AT_ONCE ? TAIL == 0 : TAIL == 4, "16-byte chunks, and one of 4 bytes");
  constexpr bool WIDE = HOW == LMS_WIDE, PLACE = HOW == LMS_PLACE;
  extern __shared__ __align__(16) unsigned char smem[];
  LDS unsigned char *smem3 = (LDS unsigned char *)smem;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t *active = (const int32_t *)a.pairs;   // queries with candidates, listed by lm_sort_out_kernel
  const int pieces = WIDE ? (a.cap + LMS_PIECE - 1) / LMS_PIECE : 1;   // of a query
  const int nwg = gridDim.x;
  LDS uint32_t *taken = (LDS uint32_t *)(smem3 + lms_lds(MT, DSUB) - 16);
  int nqueries, nactive;
  int32_t own = 0, upto = 0;   // PLACE, lane i: candidates of the workgroup's query i, pieces up to and with it
  auto list_named = [&](bool named, int32_t q) __attribute__((always_inline)) {
    const unsigned long long bal = __ballot(named);
    if (!a.list_redo || bal == 0ull) return;
    int first = 0;
    if (lane == 0) first = atomicAdd(a.cnt + a.nlist, __popcll(bal));
    first = __builtin_amdgcn_readfirstlane(first);
    if (named) a.redo[first + __popcll(bal & ((1ull << lane) - 1ull))] = q;
  };
  const int32_t lane_q = (int32_t)blockIdx.x + lane * nwg;
  if constexpr (PLACE) {   // the queries blockIdx.x, blockIdx.x + nwg, ..., at most 64
    nqueries = ((int)a.Q - (int)blockIdx.x + nwg - 1) / nwg;
    if (lane < nqueries) own = (int32_t)a.gcnt[lane_q];
    if ((uint32_t)own > (uint32_t)a.cap) own = 0;   // (redone)
    upto = (own + LMS_SHARE - 1) / LMS_SHARE;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int32_t v = __shfl_up(upto, off);
      if (lane >= off) upto += v;
    }
    nactive = __builtin_amdgcn_readlane(upto, 63);
    if (nactive == 0) {
      if (wave == 0) list_named(lane < nqueries && name_query(a, lane_q, true), lane_q);
      return;
    }
  } else {
    nqueries = a.cnt[a.nlist + 2 + 2 * a.stage];
    nactive = nqueries * pieces;
    if ((int)blockIdx.x >= nactive) return;
  }
  for (int i = tid; i < ROWS * 256 * DSUB / 4; i += LMS_NW * 64)
    ((LDS floatx4 *)smem3)[i] = ((const floatx4 *)a.codebooks)[i];
  LDS uint32_t *qd = (LDS uint32_t *)(smem3 + (size_t)ROWS * 1024 * DSUB) + wave * LMS_QUEUE * 2, *qrow = qd + LMS_QUEUE;
  LDS float *sr2 = (LDS float *)(smem3 + (size_t)ROWS * 1024 * DSUB + (size_t)LMS_NW * LMS_QUEUE * 8) + wave * MT;   // r_m^2 of the wavefront's query
  if (tid == 0) *taken = 0u;
  __syncthreads();   // from here on every wavefront is by itself, until PLACE has settled all
  const int k = a.k;
  int32_t *ticket = a.cnt + a.nlist + 3 + 2 * a.stage;
  // Three quarters of the queries are dealt to the workgroups, whose wavefronts take them up by a counter in LDS; the
  // others are taken up by whoever is free.  (All of them so, an atomic on one word of global memory for each: 454 us
  // instead of 322 for the two passes of 10 000 queries of the 1M x 96 configuration.)  The wide selection's
  // pieces are dealt out altogether, the first pieces of all queries first.
  const int dealt = WIDE || PLACE ? nactive : nactive - nactive / 4;
  for (;;) {
    uint32_t turn = 0;
    if (lane == 0) turn = lds_add(taken);
    int x = PLACE ? __builtin_amdgcn_readfirstlane((int)turn) : (int)blockIdx.x + nwg * __builtin_amdgcn_readfirstlane((int)turn);
    if (x >= dealt) {
      if (WIDE || PLACE) break;
      int32_t next = 0;
      if (lane == 0) next = atomicAdd(ticket, 1);
      x = dealt + __builtin_amdgcn_readfirstlane(next);
      if (x >= nactive) break;
    }
    const int i = PLACE ? __popcll(__ballot(upto <= x)) : WIDE ? x % nqueries : x;   // (pieces of the queries before it: at most x)
    const int64_t q = PLACE ? (int)blockIdx.x + i * nwg : __builtin_amdgcn_readfirstlane(active[i]);
    int n = PLACE ? __builtin_amdgcn_readlane(own, i) : __builtin_amdgcn_readfirstlane((int)a.gcnt[q]), n0 = 0;   // 1 .. cap
    if constexpr (PLACE) {
      n0 = (x - (i > 0 ? __builtin_amdgcn_readlane(upto, i - 1) : 0)) * LMS_SHARE;
      n = n < n0 + LMS_SHARE ? n : n0 + LMS_SHARE;
    }
    if constexpr (WIDE) {
      n0 = __builtin_amdgcn_readfirstlane(a.qmap[q]) + x / nqueries * LMS_PIECE;
      n = n < n0 + LMS_PIECE ? n : n0 + LMS_PIECE;
    }
    if (n > n0) {
      uint2 *slots = a.cand + q * a.cap;
      Key L0, L1, tau;
      uint32_t bound = SENT_D;   // on the k-th distance, besides the list's
      const bool none = !PLACE && (a.fresh || (a.seeded && a.qmap_head[q] == LM_SEEDED));   // no result to merge into
      auto take_tau = [&]() __attribute__((always_inline)) {
        const Key t0 = bcast_key(L0, (k - 1) & 63), t1 = bcast_key(L1, (k - 1) & 63);
        tau = (k - 1) < 64 ? t0 : t1;
        if (tau.d > bound) {
          tau.d = bound;
          tau.id = SENT_ID;
        }
      };
      if constexpr (HOW == LMS_MERGE) {
        const int64_t o = q * k;
        const bool in0 = !none && lane < k, in1 = !none && 64 + lane < k;
        if (none && !a.fresh) bound = (uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(a.out_dist[o + k - 1]));
        const int64_t id0 = in0 ? a.out_ids[o + lane] : -1, id1 = in1 ? a.out_ids[o + 64 + lane] : -1;
        L0.d = id0 >= 0 ? __float_as_uint(a.out_dist[o + lane]) : SENT_D;
        L0.id = id0 >= 0 ? id0 : SENT_ID;
        L1.d = id1 >= 0 ? __float_as_uint(a.out_dist[o + 64 + lane]) : SENT_D;
        L1.id = id1 >= 0 ? id1 : SENT_ID;
        take_tau();
      }
      int waiting = 0;
      bool changed = none;
      auto fold = [&](int from, int count) __attribute__((always_inline)) {   // at most 64 of the queue
        Key c;
        c.d = SENT_D;
        c.id = SENT_ID;
        if (lane < count) {
          c.d = qd[from + lane];
          if (c.d <= tau.d) c.id = a.ids[qrow[from + lane]];   // (the bound may have tightened since: no id fetched)
        }
        const bool pass = kless(c, tau);
        if (__ballot(pass) == 0) return;
        if (!pass) {
          c.d = SENT_D;
          c.id = SENT_ID;
        }
        wave_sort_desc<true>(c, lane);
        wave_merge<true>(L0, L1, c, lane);
        take_tau();
        changed = true;
      };
      // a lane past the end repeats the query's last candidate; it is not offered
      auto slot_of = [&](int u) __attribute__((always_inline)) { return slots[u + lane < n ? u + lane : n - 1]; };
      struct Where { int64_t o0, o1, blk; };
      auto where_of = [&](uint32_t c) __attribute__((always_inline)) {
        return Where{a.list_offsets[c], a.list_offsets[c + 1], a.list_blocks[c]};
      };
      auto codes_of = [&](const uint2 &e, const Where &w, uint32_t (&cw)[MT / 4]) __attribute__((always_inline)) {
        const uint32_t i = e.y - (uint32_t)w.o0;   // (rows are below 2^32)
        const int64_t nb = (w.o1 - w.o0 + 63) >> 6;
        const uint8_t *src = a.codes + w.blk * ivfpq_block_bytes(MT) + (int64_t)(i >> 6) * 1024 + (i & 63u) * 16;
#pragma unroll
        for (int j = 0; j < NCH; ++j) {
          const uintx4 v = *(const GLOBAL uintx4 *)(src + j * nb * 1024);
#pragma unroll
          for (int x = 0; x < 4; ++x) cw[4 * j + x] = v[x];
        }
      };
      uintptr_t qaddr = (uintptr_t)(a.queries + q * a.D);
      for (int m = lane; m < MT; m += 64) {
        float r = r2.v[m];
        if (a.query_radii) {
          r = a.query_radii[q * MT + m];
          r = r * r;
        }
        sr2[m] = r;
      }
      uint2 e = slot_of(n0), en = slot_of(n0 + 64);
      // One word per four subspaces: a candidate's codes all at once, or, where their registers spill, 16 at a time.
      uint32_t cw[AT_ONCE ? MT / 4 : 4];
      const uint8_t *here = nullptr;
      uint32_t chunk = 0;   // from a candidate's 16 codes to the next
      int32_t last = 0;     // from its last 16 to those behind them
      auto load_chunk = [&](const uint8_t *src, uint32_t *w) __attribute__((always_inline)) {
        const uintx4 v = *(const GLOBAL uintx4 *)src;
#pragma unroll
        for (int x = 0; x < 4; ++x) w[x] = v[x];
      };
      auto go_to = [&](const uint2 &e, const Where &w) __attribute__((always_inline)) {
        const uint32_t i = e.y - (uint32_t)w.o0;
        here = a.codes + w.blk * ivfpq_block_bytes(MT) + (int64_t)(i >> 6) * 1024 + (i & 63u) * 16;
        chunk = (uint32_t)((w.o1 - w.o0 + 63) >> 6) << 10;
        last = (int32_t)chunk - (int32_t)(i >> 6) * 768 - (int32_t)(i & 63u) * 12;
      };
      if constexpr (AT_ONCE) {
        codes_of(e, where_of(e.x), cw);
      } else {
        go_to(e, where_of(e.x));
        load_chunk(here, cw);
      }
      for (int u = n0; u < n; u += 64) {
        asm volatile("" : "+s"(qaddr) : : "memory");   // (the query's row and radii are read anew: kept across groups they spill)
        const CONSTANT float *qp = (const CONSTANT float *)qaddr;
        const Where wn = where_of(en.x);
        const uint2 enn = slot_of(u + 128);
        const float *cp = a.centroids + (int64_t)e.x * (MT * DSUB);
        float dist = 0.0f;
        uint32_t cwn[AT_ONCE ? MT / 4 : 1];
        // (one piece of code for all steps: with the loads of all hoisted to the front the registers spill)
        constexpr int STEP = DSUB == 2 ? 16 : 4;   // subspaces whose part of the centroid's row is requested together
        constexpr int LK = MT == 48 ? 8 : 4;       // look-ups in flight (more spill)
        typedef float entry __attribute__((ext_vector_type(DSUB)));
        // `count` subspaces from m0 on, their codes in w; behind the centroid's rows, which are wanted sooner, `then` is requested
        auto add_up = [&](int m0, auto count, const uint32_t *w, auto then) __attribute__((always_inline)) {
          constexpr int N = decltype(count)::value;
          floatx4 cv[N * DSUB / 4];
#pragma unroll
          for (int x = 0; x < N * DSUB / 4; ++x) cv[x] = *(const GLOBAL floatx4 *)(cp + m0 * DSUB + 4 * x);
          then();
          const LDS unsigned char *rows = smem3 + m0 * 1024 * DSUB;
#pragma unroll
          for (int h = 0; h < N; h += LK) {
            entry ev[LK];
            floatx4 rm2[LK / 4];
            if (ROWS == MT || m0 < ROWS) {
#pragma unroll
              for (int x = 0; x < LK; ++x) {
                const uint32_t code = (w[(h + x) >> 2] >> (8 * (x & 3))) & 0xFFu;
                ev[x] = *(const LDS entry *)(rows + (h + x) * 1024 * DSUB + code * (4 * DSUB));
              }
            } else {
#pragma unroll
              for (int x = 0; x < LK; ++x) {
                const uint32_t code = (w[(h + x) >> 2] >> (8 * (x & 3))) & 0xFFu;
                ev[x] = *(const GLOBAL entry *)(uniform_ptr(a.codebooks + (m0 + h + x) * 256 * DSUB) + code * (4 * DSUB));
              }
            }
#pragma unroll
            for (int x = 0; x < LK / 4; ++x) rm2[x] = *(const LDS floatx4 *)(sr2 + m0 + h + 4 * x);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int x = 0; x < LK; ++x) {
              float d2 = 0.0f;
#pragma unroll
              for (int y = 0; y < DSUB; ++y) {
                const int z = (h + x) * DSUB + y;
                const float t = (qp[m0 * DSUB + z] - cv[z >> 2][z & 3]) - ev[x][y];
                d2 = y == 0 ? t * t : fmaf(t, t, d2);
              }
              dist += table_value<0>(d2, rm2[x >> 2][x & 3]);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        };
        std::integral_constant<int, STEP> whole;
        if constexpr (AT_ONCE) {
#pragma unroll 1
          for (int m0 = 0; m0 < MT; m0 += STEP) {
            uint32_t w[STEP / 4];
#pragma unroll
            for (int x = 0; x < STEP / 4; ++x) w[x] = cw[x];
            add_up(m0, whole, w, [&]() __attribute__((always_inline)) {
              if (m0 + STEP == MT) codes_of(en, wn, cwn);
#pragma unroll
              for (int x = STEP / 4; x < MT / 4; ++x) cw[x - STEP / 4] = cw[x];
            });
          }
        } else {
#pragma unroll 1
          for (int m0 = 0; m0 < MT - TAIL; m0 += STEP) {
            uint32_t w[STEP / 4];
#pragma unroll
            for (int x = 0; x < STEP / 4; ++x) w[x] = cw[x];
            add_up(m0, whole, w, [&]() __attribute__((always_inline)) {
              if (m0 + STEP < MT - TAIL) {
                here += chunk;
                load_chunk(here, cw);
              } else {
                cw[0] = *(const GLOBAL uint32_t *)(here + last);
              }
            });
          }
          const uint32_t w = cw[0];
          add_up(MT - TAIL, std::integral_constant<int, TAIL == 0 ? STEP : TAIL>{}, &w, [&]() __attribute__((always_inline)) {
            go_to(en, wn);
            load_chunk(here, cw);
          });
        }
        const uint32_t bits = __float_as_uint(dist);
        if constexpr (WIDE) {
          if (u + lane < n) {
            a.wide_d[q * a.cap + u + lane] = bits;
            slots[u + lane] = make_uint2(e.y, 0u);
          }
        } else if constexpr (PLACE) {
          if (u + lane < n) slots[u + lane] = make_uint2(bits, e.y);
        } else {
          const bool pass = u + lane < n && bits <= tau.d;
          const unsigned long long bal = __ballot(pass);
          if (bal != 0ull) {
            if (pass) {
              const int pos = waiting + __popcll(bal & ((1ull << lane) - 1ull));
              qd[pos] = bits;
              qrow[pos] = e.y;
            }
            waiting += __popcll(bal);
          }
          while (waiting >= 64 || (waiting > 0 && u + 64 >= n)) {   // the last 64, at the end all
            const int m = waiting < 64 ? waiting : 64;
            waiting -= m;
            fold(waiting, m);
          }
        }
        e = en;
        en = enn;
        if constexpr (AT_ONCE) {
#pragma unroll
          for (int x = 0; x < MT / 4; ++x) cw[x] = cwn[x];
        }
      }
      if (HOW == LMS_MERGE && changed) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const Key x = h ? L1 : L0;
          const int i = h * 64 + lane;
          if (i < k) {
            const bool real = x.d != SENT_D;
            a.out_ids[q * k + i] = real ? x.id : -1;
            a.out_dist[q * k + i] = real ? __uint_as_float(x.d) : __builtin_inff();
          }
        }
      }
    }
  }
  if constexpr (PLACE) {
    __syncthreads();   // all slots are settled
    for (int i = wave; i < nqueries; i += LMS_NW) merge_query(a, (int)blockIdx.x + i * nwg, lane, qd, qrow);
    if (a.list_redo) {
      __syncthreads();   // all queries are named
      if (wave == 0) list_named(lane < nqueries && a.qmap[lane_q] >= 0, lane_q);
    }
  }
}

__global__ __launch_bounds__(256) void lm_merge_kernel(LmArgs a) {
  __shared__ uint32_t sqd[4][LMQ_WORDS], sqrow[4][LMQ_WORDS];
  const int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (q >= a.Q) return;
  merge_query(a, q, threadIdx.x & 63, (LDS uint32_t *)sqd[threadIdx.x >> 6], (LDS uint32_t *)sqrow[threadIdx.x >> 6]);
}

std::atomic<int> g_lm_first{1};     // lists per query that are ranked first (their k-th distance filters the rest)
std::atomic<int> g_lm_cap{0};       // candidate slots per query; 0: by the number of probes (lm_auto_cap)

constexpr size_t lm_fixed_lds(int M, int D) {   // table, residuals, radii
  const int dpad = (D + 3) & ~3;
  return (size_t)M * 2048 + (size_t)LM_G * dpad * 4 + (size_t)LM_G * IVFPQ_MAX_M * 4;
}
size_t lm_scan_lds(int M, int D) { return lm_fixed_lds(M, D) + (size_t)LM_NW * LM_G * 2 * LM_QUEUE * 4; }
// head pass: the distances of the list's points for both queries live in LDS next to the table
constexpr int lm_head_max(int M, int D) {
  const int64_t spare = (int64_t)LDS_PER_CU - (int64_t)lm_fixed_lds(M, D) - LM_SEL_WORDS * 4 - LM_G * LM_BINS * 4;
  int64_t n = spare / (LM_G * 4);
  n &= ~(int64_t)63;
  return (int)(n > 8192 ? 8192 : (n < 0 ? 0 : n));
}
static_assert(lm_head_max(64, 128) >= ivfpq::lm_head_fits(64) && lm_head_max(48, 96) >= ivfpq::lm_head_fits(48) && lm_head_max(16, 64) >= ivfpq::lm_head_fits(16) &&
              lpp_head_max(256) >= ivfpq::LPP_HEAD_FITS, "the longest lists that AUTO counts on");
size_t lm_head_lds(int M, int D) { return lm_fixed_lds(M, D) + (size_t)LM_G * lm_head_max(M, D) * 4 + LM_SEL_WORDS * 4 + LM_G * LM_BINS * 4; }

// The queries that qmap names, as a list.  (One atomic per wavefront of 64 queries: one per query, from
// lm_merge_kernel, took 110 us where all of 10 000 are named.)
__global__ __launch_bounds__(256) void lm_redo_kernel(LmArgs a) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int lane = threadIdx.x & 63;
  const bool named = q < a.Q && a.qmap[q] >= 0;
  const unsigned long long bal = __ballot(named);
  if (bal == 0ull) return;
  int first = 0;
  if (lane == 0) first = atomicAdd(&a.cnt[a.nlist], __popcll(bal));
  first = __builtin_amdgcn_readfirstlane(first);
  if (named) a.redo[first + __popcll(bal & ((1ull << lane) - 1ull))] = (int32_t)q;
}

template <int MT, int DSUB, bool HEAD>
int launch_lm_scan_t(const LmArgs &a, const RadiiSq &r2, int grid, hipStream_t s) {
  auto kern = lm_scan_kernel<MT, DSUB, HEAD>;
  static std::atomic<uint64_t> prepared;
  if (int rc = prepare_kernel(kern, prepared)) return rc;
  const size_t lds = HEAD ? lm_head_lds(MT, a.D) : lm_scan_lds(MT, a.D);
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(LM_NW * 64), lds, s, a, r2);
  return IVFPQ_OK;
}

template <int MT, int DSUB, int MODE, bool HEAD = false>
int launch_lm_byte_t(const LmArgs &a, const RadiiSq &r2, int grid, hipStream_t s) {
  auto kern = lm_byte_kernel<MT, DSUB, MODE, HEAD>;
  static std::atomic<uint64_t> prepared;
  if (int rc = prepare_kernel(kern, prepared)) return rc;
  static_assert(lmb_lds(MT, DSUB, HEAD) <= (size_t)LDS_PER_CU, "byte tables, records and queue fit a CU");
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(LMB_NW * 64), lmb_lds(MT, DSUB, HEAD), s, a, r2);
  return IVFPQ_OK;
}

template <int MT, int DSUB>
int launch_lm_part_t(const LmArgs &a, const RadiiSq &r2, int cus, hipStream_t s) {
  auto kern = lm_part_kernel<MT, DSUB>;
  static std::atomic<uint64_t> prepared;
  if (int rc = prepare_kernel(kern, prepared)) return rc;
  static_assert(LMP_WG * lmp_lds(MT, DSUB) <= (size_t)LDS_PER_CU, "the workgroups fit a CU");
  hipLaunchKernelGGL(kern, dim3((unsigned)(LMP_WG * cus)), dim3(LMP_NW * 64), lmp_lds(MT, DSUB), s, a, r2);
  return IVFPQ_OK;
}

template <int MT, int DSUB, bool HEAD>
int launch_lm_pair_t(const LmArgs &a, const RadiiSq &r2, int cus, hipStream_t s) {
  auto kern = lm_pair_kernel<MT, DSUB, HEAD>;
  static std::atomic<uint64_t> prepared;
  if (int rc = prepare_kernel(kern, prepared)) return rc;
  hipLaunchKernelGGL(kern, dim3((unsigned)(LPP_WG * cus)), dim3(LPP_NW * 64), HEAD ? lpp_head_lds(a.D) : lpp_main_lds(a.D), s, a, r2);
  return IVFPQ_OK;
}

template <bool HEAD>
int launch_lm_pair(const LmArgs &a, const RadiiSq &r2, int cus, hipStream_t s) {
  if constexpr (HEAD) {   // (the further lists of these shapes: lm_scan_kernel)
    if (a.M == 48 && a.dsub == 2) return launch_lm_pair_t<48, 2, true>(a, r2, cus, s);
    if (a.M == 64 && a.dsub == 2) return launch_lm_pair_t<64, 2, true>(a, r2, cus, s);
  }
  if (a.M == 100 && a.dsub == 2) return launch_lm_pair_t<100, 2, HEAD>(a, r2, cus, s);
  switch (a.dsub) {
    case 1: return launch_lm_pair_t<0, 1, HEAD>(a, r2, cus, s);
    case 2: return launch_lm_pair_t<0, 2, HEAD>(a, r2, cus, s);
    default: return launch_lm_pair_t<0, 3, HEAD>(a, r2, cus, s);
  }
}

template <int MT, int DSUB, int HOW>
int launch_lm_settle_t(const LmArgs &a, const RadiiSq &r2, int grid, hipStream_t s) {
  auto kern = lm_settle_kernel<MT, DSUB, HOW>;
  static std::atomic<uint64_t> prepared;
  if (int rc = prepare_kernel(kern, prepared)) return rc;
  static_assert(lms_lds(MT, DSUB) <= (size_t)LDS_PER_CU, "codebook and queues fit a CU");
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(LMS_NW * 64), lms_lds(MT, DSUB), s, a, r2);
  return IVFPQ_OK;
}

template <int HOW>
int launch_lm_settle(const LmArgs &a, const RadiiSq &r2, int cus, hipStream_t s) {
  const int grid = a.Q < cus ? (int)a.Q : cus;   // (a workgroup without a query of its own leaves at once)
  if (a.M == 48) return launch_lm_settle_t<48, 2, HOW>(a, r2, grid, s);
  if (a.M == 64) return launch_lm_settle_t<64, 2, HOW>(a, r2, grid, s);
  if constexpr (HOW != LMS_WIDE)
    if (a.M == 100) return launch_lm_settle_t<100, 2, HOW>(a, r2, grid, s);
  return launch_lm_settle_t<16, 4, HOW>(a, r2, grid, s);
}

template <int MODE>
int launch_lm_byte_m(const LmArgs &a, const RadiiSq &r2, int grid, hipStream_t s) {
  if (a.M == 48) return launch_lm_byte_t<48, 2, MODE>(a, r2, grid, s);
  if (a.M == 64) return launch_lm_byte_t<64, 2, MODE>(a, r2, grid, s);
  return launch_lm_byte_t<16, 4, MODE>(a, r2, grid, s);
}

int launch_lm_byte(const LmArgs &a, const RadiiSq &r2, int grid, hipStream_t s) {
  if (a.M == 100) return launch_lm_part_t<100, 2>(a, r2, grid, s);
  if (a.parts && a.mode == 0) return a.M == 48 ? launch_lm_part_t<48, 2>(a, r2, grid, s) : launch_lm_part_t<64, 2>(a, r2, grid, s);
  if (a.mode == 0) return launch_lm_byte_m<0>(a, r2, grid, s);
  if (a.mode == 1) return launch_lm_byte_m<1>(a, r2, grid, s);
  return launch_lm_byte_m<2>(a, r2, grid, s);
}

int launch_lm_byte_head(const LmArgs &a, const RadiiSq &r2, int grid, hipStream_t s) {
  if (a.M == 48) return launch_lm_byte_t<48, 2, 0, true>(a, r2, grid, s);
  if (a.M == 64) return launch_lm_byte_t<64, 2, 0, true>(a, r2, grid, s);
  return launch_lm_byte_t<16, 4, 0, true>(a, r2, grid, s);
}

template <bool HEAD>
int launch_lm_scan(const ivfpq_index *ix, const LmArgs &a, const RadiiSq &r2, int grid, hipStream_t s) {
  if (ix->M == 48) return launch_lm_scan_t<48, 2, HEAD>(a, r2, grid, s);
  if (ix->M == 64) return launch_lm_scan_t<64, 2, HEAD>(a, r2, grid, s);
  return launch_lm_scan_t<16, 4, HEAD>(a, r2, grid, s);
}

}  // namespace

namespace ivfpq {

void set_lm_first(int v) { g_lm_first.store(v, std::memory_order_relaxed); }
void set_lm_cap(int v) { g_lm_cap.store(v, std::memory_order_relaxed); }

bool list_major_supported(const ivfpq_index *ix, int32_t nprobe, int32_t k) {
  if (ix->metric != IVFPQ_METRIC_L2 || k > KP) return false;
  if (!list_major_shape(ix) || LM_G * ix->D > LM_NW * 64 || LM_G * ix->M > LM_NW * 64) return false;
  if (byte_table_shape(ix) && lm_scan_lds(ix->M, ix->D) > (size_t)LDS_PER_CU) return false;
  return nprobe > g_lm_first.load(std::memory_order_relaxed);
}

// Indexes on which the head pass may run with byte tables: lists that are long, or do not fit the fp32 form's LDS.
static bool byte_head_lists(const ivfpq_index *ix) {
  return byte_table_shape(ix) && ix->max_list_len < (1 << 20) &&
         (ix->N > (int64_t)4096 * ix->nlist || (ix->max_list_len > lm_head_max(ix->M, ix->D) && ix->N >= (int64_t)2800 * ix->nlist));
}

LmWorkspace plan_list_major(const ivfpq_index *ix, int64_t Q, int32_t nprobe) {
  LmWorkspace w;
  w.first = g_lm_first.load(std::memory_order_relaxed);
  // Candidates that pass the first lists' bound grow with the number of lists probed; a query
  // that runs out of slots costs a query-major pass over all of its lists.  Measured on the
  // 1M x 96 configuration (64 probes): 4096 slots 11.39 ms per batch, 8192 10.88, 16384 10.71.
  w.cap = g_lm_cap.load(std::memory_order_relaxed);
  if (w.cap == 0) w.cap = nprobe >= 64 ? 16384 : (nprobe * 256 > 4096 ? nprobe * 256 : 4096);
  // (a main pass that starts over behind a head pass with byte tables has the first lists among its pairs)
  plan_list_major_tables(w, ix->nlist, Q, byte_head_lists(ix) ? nprobe + w.first : nprobe);
  w.cand = w.total;
  w.total += lm_align((size_t)Q * w.cap * 8);
  return w;
}

static LmArgs lm_args(const ivfpq_index *ix, const float *d_queries, int64_t Q, int32_t nprobe, const int32_t *d_probe_ids,
                      const RadiiSq &r2, const float *d_query_radii, const float *d_probe_lb, const LmWorkspace &w, char *lm_base) {
  LmArgs a = {};
  a.queries = d_queries;
  a.probe_ids = d_probe_ids;
  a.probe_lb = d_probe_lb;
  a.centroids = ix->d_centroids;
  a.codebooks = ix->d_codebooks;
  a.cb_split = ix->d_cb_split;
  a.list_offsets = ix->d_list_offsets;
  a.list_blocks = ix->d_list_blocks;
  a.codes = ix->d_codes;
  a.ids = ix->d_ids;
  a.cnt = reinterpret_cast<int32_t *>(lm_base + w.cnt);
  a.rank = reinterpret_cast<int32_t *>(lm_base + w.rank);
  a.redo = a.rank;
  a.base = reinterpret_cast<int32_t *>(lm_base + w.base);
  a.pairs = reinterpret_cast<int2 *>(lm_base + w.pairs);
  a.gcnt = reinterpret_cast<uint32_t *>(lm_base + w.gcnt);
  a.cand = reinterpret_cast<uint2 *>(lm_base + w.cand);
  a.qmap = reinterpret_cast<int32_t *>(lm_base + w.qmap);
  a.qmap_head = reinterpret_cast<int32_t *>(lm_base + w.qmap_head);
  a.query_radii = d_query_radii;
  a.Q = Q;
  a.D = ix->D; a.M = ix->M; a.dsub = ix->dsub; a.Mp = ix->Mp; a.nlist = ix->nlist;
  a.nprobe = nprobe; a.first = w.first; a.cap = w.cap;
  a.p0 = w.first;
  a.p1 = nprobe;
  a.group = LM_G;
  for (int m = 0; m < ix->M; ++m) a.rmax = r2.v[m] > a.rmax ? r2.v[m] : a.rmax;
  // A table in parts serves LMP_SEG points of a list, and with a longer one it is made again.  us of a search with whole byte
  // tables / in parts, 64 probes (48 subspaces, 10 000 queries, without structure), 32 probes (64, 8192, without structure), k = 100,
  // by the mean list: 48: 500 2421 / 2105, 977 3439 / 3073, 1515 3982 / 3895, 1953 3573 / 3690, 2500 3994 / 4349, 3906 5212 / 5996;
  // 64: 977 2203 / 1996, 1515 2308 / 2040, 1953 2498 / 2184, 2941 2812 / 2907, 3906 3090 / 3146.  The line is where both gain.
  // Lists of very different lengths: the long ones are probed the most, and the mean says nothing about them (48 subspaces, lists of
  // 1108, the longest of 95 742, 2567 queries of 12 probes 1484 / 1841; random calls with a list above 8192 points 1.00 times as fast, one
  // in seven loses a twentieth and more; with shorter ones and 512 queries 1.12 times, one in 60).  Small batches have a task or
  // two for a workgroup, which then waits for every part's rows (a search: 64 subspaces, clustered, 185 queries of 100 probes 88 / 104,
  // 296 of 72 99 / 115, 300 of 32, radii per query 82 / 90, 451 of 64 118 / 123; 48, 217 of 83 238 / 254; without structure 450 of 64
  // 281 / 249, 511 of 32 140 / 131, 300 of 32 137 / 138): whole below 512 queries.
  a.parts = ix->d_cb_split && ix->N <= (int64_t)1536 * ix->nlist && ix->max_list_len <= 4 * LMP_SEG && Q >= 512 ? 1 : 0;
  return a;
}

// One wavefront per query: every point of its first lists becomes a candidate of the wide selection.
__global__ __launch_bounds__(256) void wide_seed_kernel(LmArgs a, uint32_t *__restrict__ bound) {
  const int lane = threadIdx.x & 63;
  const int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (q >= a.Q) return;
  int64_t n = 0;
  for (int p = 0; p < a.first && n <= a.cap; ++p) {
    const int32_t c = a.probe_ids[q * a.nprobe + p];
    if ((uint32_t)c >= (uint32_t)a.nlist) continue;
    const int64_t o0 = a.list_offsets[c], len = a.list_offsets[c + 1] - o0;
    if (n + len <= a.cap)
      for (int64_t i = lane; i < len; i += 64) a.cand[q * a.cap + n + i] = make_uint2((uint32_t)c, (uint32_t)(o0 + i));
    n += len;
  }
  if (lane == 0) {
    a.gcnt[q] = n <= a.cap ? (uint32_t)n : (uint32_t)a.cap + 1u;
    a.wide_n[q] = 0;
    bound[q] = SENT_D;
  }
}

// The wide selection's candidates (k above KP).  stage 0: all points of the first w.first lists.  Later ones: what lies
// within the query's bound so far in the probes [p0, p1), from byte tables; it takes the slots behind those in use.
// Either way the candidates' distances are formed.  (The per-list counts and the words behind them are zero at first.)
int launch_wide_stage(const ivfpq_index *ix, const float *d_queries, int64_t Q, int32_t nprobe, const int32_t *d_probe_ids,
                      const RadiiSq &r2, const float *d_query_radii, const float *d_probe_lb, uint32_t *wide_d, int64_t *wide_id,
                      int32_t *wide_n, uint32_t *wide_bound, int32_t cap, const LmWorkspace &w, char *lm_base, int stage,
                      int32_t p0, int32_t p1, hipStream_t s) {
  LmArgs a = lm_args(ix, d_queries, Q, nprobe, d_probe_ids, r2, d_query_radii, d_probe_lb, w, lm_base);
  a.cand = reinterpret_cast<uint2 *>(wide_id);
  a.cap = cap;
  a.tau = reinterpret_cast<const float *>(wide_bound);   // (keys of distances are their bits; none yet: a NaN)
  a.tau_stride = 1;
  a.wide_n = wide_n;
  a.wide_d = wide_d;
  a.group = LMB_G;
  a.stage = stage;
  a.p0 = p0;
  a.p1 = p1;
  int dev = 0, cus = 0;
  IVFPQ_HIP_TRY(hipGetDevice(&dev));
  IVFPQ_HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  if (cus < 1) cus = 1;
  if (stage == 0) {
    hipLaunchKernelGGL(wide_seed_kernel, dim3((unsigned)((Q + 3) / 4)), dim3(256), 0, s, a, wide_bound);
  } else {
    const unsigned pair_grid = (unsigned)((Q * (p1 - p0) + 255) / 256);
    hipLaunchKernelGGL(lm_pairs_kernel, dim3(pair_grid), dim3(256), 0, s, a, 0, 0);
    hipLaunchKernelGGL(lm_offsets_kernel, dim3(1), dim3(1024), 0, s, a);
    hipLaunchKernelGGL(lm_pairs_kernel, dim3(pair_grid), dim3(256), 0, s, a, 1, 0);
    if (int rc = launch_lm_byte(a, r2, cus, s)) return rc;
  }
  hipLaunchKernelGGL(lm_sort_out_kernel, dim3((unsigned)((Q + 255) / 256)), dim3(256), 0, s, a, 0);
  return launch_lm_settle<LMS_WIDE>(a, r2, cus, s);
}

int launch_scan_list_major(const ivfpq_index *ix, const float *d_queries, int64_t Q, int32_t nprobe,
                           const int32_t *d_probe_ids, int32_t k, const RadiiSq &r2, int32_t mode,
                           const float *d_query_radii, float *d_probe_lb, int64_t *d_out_ids, float *d_out_dist,
                           const LmWorkspace &w, char *lm_base, hipStream_t s) {
  if (Q * (int64_t)nprobe > 0x7FFFFFFFll || w.pairs_cap > 0x7FFFFFFFll) {
    set_error("scan (list-major): %lld (query, probe) pairs exceed 2^31", (long long)(Q * (int64_t)nprobe));
    return IVFPQ_ERR_UNSUPPORTED;
  }

  LmArgs a = lm_args(ix, d_queries, Q, nprobe, d_probe_ids, r2, d_query_radii, (get_scan_ablate() & 64) ? nullptr : d_probe_lb, w, lm_base);
  a.out_ids = d_out_ids;
  a.out_dist = d_out_dist;
  a.tau = d_out_dist + k - 1;
  a.tau_stride = k;
  // The tables of two queries in parts (lm_pair_kernel), two workgroups per CU, or whole (lm_scan_kernel).  us of a search of 32
  // probes, clustered data, k = 100, whole / in parts, by the mean list:
  //   queries                      600         1000         1500         2200         4000         6000        10 000
  //   64 subspaces, 400                    133 / 129                 188 / 185                 357 / 336
  //   64, 500                                                                                               467 / 430
  //   64, 977                   83 / 79     97 / 102    117 / 109    152 / 138    213 / 203                 413 / 364
  //   64, 1430                              98 / 100                 142 / 139                 311 / 271
  //   64, 1953                                                                                              485 / 411
  //   64, 2700                                                                                              655 / 499
  //   64, 3906                             172 / 142                (byte tables from 8 million points on)
  //   48, 977                   93 / 93    108 / 112    130 / 125    163 / 154    238 / 232
  // The line is where the kernel in parts is faster for good: below it most workgroups have one task, and nothing to hide the
  // codebook's way from the L2 behind.
  int dev = 0, cus = 0;
  IVFPQ_HIP_TRY(hipGetDevice(&dev));
  IVFPQ_HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  if (cus < 1) cus = 1;
  // (48 subspaces: whole tables leave room for longer lists, and every query whose list has none is redone.  Radii per query, two
  // components a list, 7312 queries, lists of 2035: 3362 us, in parts 4046.)
  const bool longer_whole = byte_table_shape(ix) && lm_head_max(ix->M, ix->D) > lpp_head_max(ix->D) && ix->max_list_len > lpp_head_max(ix->D);
  const bool table_parts = !byte_table_shape(ix) || (ix->dsub == 2 && !longer_whole && (Q > (int64_t)4 * cus || ix->N >= (int64_t)2048 * ix->nlist));
  a.head_max = table_parts ? lpp_head_max(ix->D) : lm_head_max(ix->M, ix->D);
  a.k = k;
  a.mode = mode;

  // ---- the first lists of every query: they give the bound tau_q that filters the rest ----
  // One list per query under distance scoring: the head pass ranks it list-major (queries that
  // share a nearest list share its table pass); what the head pass leaves out (qmap_head) skips
  // the list-major scan and is redone query-major at the end.  Otherwise (several first lists, or the hit-count scorings,
  // whose masses of equal scores the head pass's selection is not made for): query-major.
  // The head pass with byte tables where lists are long: those that do not fit the fp32 form's LDS cost a query-major
  // pass each, and the longer a list the more the eight queries of a look-up save against settling the candidates.
  // us of a search with the fp32 head pass / with byte tables (64 probes, k = 100):
  //   queries                                      1024         2048         4096         8192
  //   64 subspaces, clustered, lists of 977 (10 000 queries)                             418 / 488
  //   64, clustered, 2441 (10 000 queries, 2.4 a list; the scan alone)                   666 / 820
  //   64, clustered, 1953                     129 / 228    176 / 276    267 / 339    492 / 542
  //   64, clustered, 4000                     253 / 361    406 / 408    684 / 590   1248 / 881
  //   64, clustered, 7812                     590 / 706    943 / 810   1310 / 1052  2162 / 1570
  //   48, without structure, 3906            2558 / 1038  3141 / 1621  5021 / 2766  7402 / 5093
  // and lists of 3636, the longest of 10 000, 64 probes, k = 100, the radii holding 0.25 / 0.9 of the entries (where they hold
  // much, the pass only finds bounds and the nearest lists are scanned again):
  //   queries                                  2200                       4096                       8192
  //   64 subspaces, clustered       896 / 830,  408 / 672    1645 / 1222,  677 / 822    2744 / 2138, 1234 / 1169
  //   48, clustered                1447 / 1018, 446 / 569    2072 / 1606,  724 / 728    3415 / 2857, 1143 / 1037
  //   16, clustered                 321 / 361,  341 / 417     424 / 458,   478 / 536     688 / 712,   817 / 800
  //   64, without structure        9121 / 2106, 7446 / 2184 16022 / 3507, 13098 / 3531 31495 / 6311, 25446 / 6448
  //   48, without structure        3073 / 1720, 2933 / 1734  4200 / 2667, 4019 / 2680   6536 / 4800, 6286 / 4843
  //   16, without structure        1690 / 984,  1599 / 982   2323 / 1477, 2196 / 1445   3617 / 2515, 3429 / 2485
  // The line is where data without structure, and clustered data whose radii hold a part of the entries, gains; clustered
  // data with wide radii pays for it in the smaller batches.
  int rc = IVFPQ_OK;
  const int64_t head_points = (int64_t)((double)Q * (double)ix->N / ix->nlist);
  const bool head_bytes = byte_head_lists(ix) && w.first == 1 && mode == IVFPQ_SCORE_DISTANCE && !(get_scan_ablate() & 8) &&
                          head_points >= 8000000;
  const bool head_pass = w.first == 1 && mode == IVFPQ_SCORE_DISTANCE && (head_bytes || a.head_max >= 64);
  if (head_bytes) {
    a.head_max = INT_MAX;
    a.group = LMB_G;
    a.fresh = 1;
  }
  // List-level lower bounds of every (query, probe): behind the head pass, where its k-th distances end most of them early
  // (lm_bound_kernel), or up front.  Either way the per-list counts are cleared (lm_offsets_kernel leaves them clear for the pass after it).
  const bool late_bounds = head_pass && a.probe_lb && ix->dsub == 2;
  const bool head_sorted = head_pass && Q <= LMH_THREADS * LMH_QUERIES && ix->nlist <= LMH_LISTS;
  if (late_bounds && !head_sorted) rc = launch_fill_i32(a.cnt, lm_counters(ix->nlist), 0, s);
  else if (!late_bounds) rc = launch_probe_bounds(ix, d_queries, Q, nprobe, d_probe_ids, r2, mode, d_query_radii, d_probe_lb, s, a.cnt, lm_counters(ix->nlist));
  if (rc) return rc;
  if (head_pass) {
    if (head_sorted) {
      static std::atomic<uint64_t> prepared;
      if (int e = prepare_kernel(lm_head_pairs_kernel, prepared)) return e;
      hipLaunchKernelGGL(lm_head_pairs_kernel, dim3(1), dim3(LMH_THREADS), (size_t)(ix->nlist + LMH_THREADS) * 4, s, a,
                         late_bounds ? lm_counters(ix->nlist) : 0);
    } else {
      const unsigned qgrid = (unsigned)((Q + 255) / 256);
      hipLaunchKernelGGL(lm_pairs_kernel, dim3(qgrid), dim3(256), 0, s, a, 0, 1);
      hipLaunchKernelGGL(lm_offsets_kernel, dim3(1), dim3(1024), 0, s, a);
      hipLaunchKernelGGL(lm_pairs_kernel, dim3(qgrid), dim3(256), 0, s, a, 1, 1);
    }
    rc = head_bytes ? launch_lm_byte_head(a, r2, cus, s) : (table_parts ? launch_lm_pair<true>(a, r2, cus, s) : launch_lm_scan<true>(ix, a, r2, cus, s));
    if (rc) return rc;
    if (head_bytes) {
      hipLaunchKernelGGL(lm_sort_out_kernel, dim3((unsigned)((Q + 255) / 256)), dim3(256), 0, s, a, 0);
      rc = launch_lm_settle<LMS_MERGE>(a, r2, cus, s);
      if (rc) return rc;
    }
  }
  a.head_done = head_pass ? 1 : 0;
  a.fresh = 0;
  const int32_t main_first = head_bytes ? 0 : w.first;   // (the nearest list of queries that are only seeded)
  if (!head_pass) {
    ScanView head = {nprobe, nullptr, true};
    rc = launch_scan(ix, d_queries, Q, w.first, d_probe_ids, k, r2, 1, nullptr, nullptr, d_out_ids, d_out_dist,
                     nullptr, nullptr, nullptr, nullptr, mode, d_query_radii, d_probe_lb, s, &head);
    if (rc) return rc;
  }

  // ---- the other lists, list-major: pairs bucketed by list, scan, merge ----
  // With byte tables unless most queries may have no k-th distance to compare with yet (lists
  // shorter than k on average leave them without one after their first list, and then every point
  // is a candidate), a position does not fit the queue's words, or the early exit of the sums is
  // switched off (a plain scan forms every sum).  A candidate costs about what 16 byte sums do, and the shorter
  // the lists against k, the more of their points are candidates.  10 000 queries, 32 probes, us with fp32 pairs
  // / with byte tables at a mean list of so many k: data with cluster structure, 48 subspaces 2.9 2363 / 1887,
  // 6.8 2929 / 1992, 9.8 3275 / 2064; data without, 48 subspaces 2.9 3008 / 3809, 4.9 3405 / 3819, 6.8 3666 /
  // 3903, 8.9 2581 / 2460, 9.8 4057 / 3984, 64 subspaces 2.9 3436 / 3962, 4.9 3902 / 3903, 6.8 4248 / 3936;
  // 16 subspaces 2.9 2343 / 2276, 9.8 2742 / 2302; 100 (2000 queries, 64 probes) without 9.8 4768 / 3810, k = 10 4623 / 2768.  So from 6 on, with 16 subspaces from 2 on, and with the
  // hit counts, whose byte sums are the result.
  const bool bytes = (byte_table_shape(ix) || part_table_shape(ix)) && ix->N >= (int64_t)(mode == 0 && ix->M > 16 ? 6 : 2) * k * ix->nlist && ix->max_list_len < (1 << 20) && !(get_scan_ablate() & 8);
  a.group = bytes ? LMB_G : LM_G;
  // Many probes: the nearest few lists first, merged, so that the rest is filtered by a k-th distance
  // over eight lists instead of one.  That costs five launches (14 us of 10 000 queries) where the bounds rule
  // everything out, and pays where they do not.  10 000 queries, k = 100, lists of 976, us in one round / two:
  //   probes                          16           32           47           64          128
  //   48 subspaces, clustered    1177 / 1222  2070 / 2091  2885 / 2899  3810 / 3810  7302 / 7256
  //   48, without structure      2172 / 1772  4001 / 2734  5630 / 3638  7387 / 4650  14618 / 8511
  //   64, clustered               381 / 395    416 / 431    453 / 467    496 / 510    730 / 745
  //   64, without structure      2239 / 1930  3994 / 3062  5584 / 4126  7298 / 5318  13494 / 9868
  //   16, clustered               315 / 330    389 / 403    460 / 474    541 / 555    965 / 980
  // (2000 queries, 64 clustered: 131 / 143 at 32 probes, 143 / 156 at 64).  The line is where the two rounds cost
  // clustered data 3 % or less of a large batch.  With 100 subspaces, whose filtering and bounds are dearer, they don't pay where
  // lists have a structure at all: 10 000 queries of clustered data 666 / 700, 1000 165 / 202, two components a list, 4000
  // 10456 / 11065, radii per query 1150 / 1231; without structure, 2000, k = 10 2768 / 2774, k = 100 3809 / 3096 (7619 query-major).
  // The candidates of byte tables of distances are settled where they stand by the wavefronts that share a workgroup's
  // queries, and ranked behind that; up to 64 queries a workgroup.  Queries without a result of the head pass (LM_SEEDED), and
  // larger batches, take a wavefront a query (lm_sort_out_kernel, lm_settle_kernel<LMS_MERGE>).
  const bool in_place = bytes && mode == 0 && !head_bytes && Q <= (int64_t)64 * cus;
  const int split = bytes && ix->M != 100 && nprobe - w.first >= 2 * LM_STAGE1 + 32 ? w.first + LM_STAGE1 : nprobe;
  for (int p0 = main_first, p1 = split; p0 < nprobe; p0 = p1, p1 = nprobe) {
    a.p0 = p0;
    a.p1 = p1;
    a.later = p0 > main_first ? 1 : 0;
    a.seeded = head_bytes && !a.later ? 1 : 0;
    a.stage = a.later + 1;
    const int64_t npairs = Q * (p1 - p0);
    const unsigned pair_grid = (unsigned)((npairs + 255) / 256);
    if (late_bounds) {
      const unsigned bound_grid = (unsigned)((npairs + 63) / 64);
      if (bounds_use_grid(ix)) hipLaunchKernelGGL(lm_bound_kernel<true>, dim3(bound_grid), dim3(LM_BOUND_NW * 64), 0, s, a, r2, ix->d_box, ix->d_grid, ix->d_grid_par, d_probe_lb);
      else hipLaunchKernelGGL(lm_bound_kernel<false>, dim3(bound_grid), dim3(LM_BOUND_NW * 64), 0, s, a, r2, ix->d_box, nullptr, nullptr, d_probe_lb);
    } else {
      hipLaunchKernelGGL(lm_pairs_kernel, dim3(pair_grid), dim3(256), 0, s, a, 0, 0);
    }
    hipLaunchKernelGGL(lm_offsets_kernel, dim3(1), dim3(1024), 0, s, a);
    hipLaunchKernelGGL(lm_pairs_kernel, dim3(pair_grid), dim3(256), 0, s, a, 1, 0);
    rc = bytes ? launch_lm_byte(a, r2, cus, s) : (byte_table_shape(ix) ? launch_lm_scan<false>(ix, a, r2, cus, s) : launch_lm_pair<false>(a, r2, cus, s));
    if (rc) return rc;
    if (in_place) {
      a.list_redo = p1 == nprobe && Q > 4096 ? 1 : 0;
      rc = launch_lm_settle<LMS_PLACE>(a, r2, cus, s);
      if (rc) return rc;
    } else if (bytes && mode == 0) {
      hipLaunchKernelGGL(lm_sort_out_kernel, dim3((unsigned)((Q + 255) / 256)), dim3(256), 0, s, a, p1 == nprobe && Q > 4096 ? 1 : 0);
      rc = launch_lm_settle<LMS_MERGE>(a, r2, cus, s);
      if (rc) return rc;
    } else {
      hipLaunchKernelGGL(lm_merge_kernel, dim3((unsigned)((Q + 3) / 4)), dim3(256), 0, s, a);
    }
  }
  IVFPQ_HIP_TRY(hipGetLastError());
  // queries whose candidate buffer overflowed: the query-major kernel over all of their probes
  // (and those the head pass left out).  A large batch lists them first; up to 4096 queries a workgroup per query
  // that looks whether it is named takes as long where none is, and where all are (lists too long for the head
  // pass: 2771 queries, 64 subspaces, 48 probes) 562 us against 625, since every query starts with fresh registers.
  ScanView redo = {0, a.qmap, true};
  if (Q > 4096 && (byte_table_shape(ix) || part_table_shape(ix))) {   // (shapes whose query-major kernel takes a list)
    redo.qmap = nullptr;
    redo.qlist = a.redo;
    redo.qlist_n = a.cnt + ix->nlist;
    if (!bytes || mode != 0) hipLaunchKernelGGL(lm_redo_kernel, dim3((unsigned)((Q + 255) / 256)), dim3(256), 0, s, a);   // (lm_sort_out_kernel has listed them)
  }
  return launch_scan(ix, d_queries, Q, nprobe, d_probe_ids, k, r2, 1, nullptr, nullptr, d_out_ids, d_out_dist,
                     nullptr, nullptr, nullptr, nullptr, mode, d_query_radii, d_probe_lb, s, &redo);
}

}  // namespace ivfpq
