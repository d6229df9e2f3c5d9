// Selective L2-LUT construction, distance calculation and top-k, fused
// (paper Sec. 4.1 and Algorithm 2 for the table; Sec. 2.1 step D and Sec. 5.3
// for the accumulation; Sec. 2.1 for the final selection).
//
// One workgroup serves one (query, probe group).  For each probed list it
//   1. builds the thresholded table for (query, list) in LDS: entry e of
//      subspace m stores d2 = ||res_m - codebook[m][e]||^2 if d2 <= r_m^2 and
//      the clamp r_m^2 otherwise (res = query - list centroid);
//   2. streams the list's codes from HBM, one point per lane, 16 bytes per load,
//      and sums the table values of the point's codes in subspace order (fp32,
//      the same order as a plain loop, so sums are reproducible bit for bit).
//      A block of 64 points is dropped as soon as partial sum + (sum of the row
//      minima of the remaining subspaces) exceeds the current k-th distance for
//      all of its points, and code bytes that were not needed are never requested:
//      exact, i.e. the result is that of the plain loop;
//   3. keeps, per wavefront, the 128 best (distance, id) pairs seen so far as a
//      sorted list spread over the lanes' registers; candidates that beat the
//      current k-th best are queued in LDS and folded in 64 at a time with a
//      bitonic merge.
// At the end the wavefronts' lists are merged and the first k written out.
//
// The paper builds the table on RT cores (a ray per (query, list, subspace)
// against one sphere per entry) and accumulates on tensor cores.  CDNA4 has
// neither RT cores nor a reason to turn a byte-indexed gather into a matrix
// product: the radius test is a compare on the vector ALU and the accumulation
// is bound by HBM and LDS gather rates.
#pragma once

#include "scan_device.h"

namespace {

// BYTE: the hit-count scorings with a byte table (one byte per entry, 256 bytes per row,
// integer sums) instead of the float table; the sums are the same small integers either way.
// DSUB == 0: the form for shapes without a kernel of their own.  MT is the number of subspaces rounded
// up to whole 16-byte chunks of codes; M (any number in the last chunk) and dsub are run-time values.
// It shares everything with the others -- chunked loads, eight look-ups in flight, row minima, early
// exits, the list-level bound -- but streams its codebook rows per list.  (500k x 120, 30 subspaces of 4:
// the form it replaces built its table entry by entry from scalar loads, pruned nothing and had one
// look-up in flight: 1205 us of scan for 999 queries, 335 us so.)
// KIND: SCAN_ALL writes every candidate's distance instead of a top-k; SCAN_SPLIT is the form in
// which several workgroups share a query's probes (its exchange of bounds costs registers that the
// plain form spills for: 7 % on lists of 8000 points).
// SCAN_LISTED serves the queries of a list that a kernel before it made (usually none): as many workgroups as
// the chip holds at once, each of which takes the next entry when it is done with one.  10 000 queries of 16
// subspaces, nearly all of them named: 4820 us a batch; 5118 where every workgroup serves the named ones among
// a fixed share of the batch, 6590 with half as many workgroups.  None named: a workgroup per query of the batch
// that looks whether it is takes 16 us, this form and the kernel that makes the list 10.
enum { SCAN_TOPK = 0, SCAN_ALL = 1, SCAN_SPLIT = 2, SCAN_LISTED = 3 };
template <int MT, int DSUB, int NW, int KIND, bool BYTE>
__device__ __forceinline__ void scan_query(const ScanArgs &a, const RadiiSq &r2, int64_t q, int split) {
  constexpr bool DUMP = KIND == SCAN_ALL, SPLIT = KIND == SCAN_SPLIT;
  constexpr int NT = NW * 64;
  using Acc = std::conditional_t<BYTE, uint32_t, float>;
  constexpr int MPT = (MT + 3) / 4 * 4;
  constexpr bool RT = DSUB == 0;   // any M with MT / 16 chunks, any dsub
  extern __shared__ __align__(16) unsigned char smem[];
  const int M = RT ? a.M : MT;
  const int Mp = RT ? a.Mp : MPT;
  const int D = a.D;
  // LDS carve: table | merge staging (aliases the table) | query | queues | tau
  const int lut_bytes = M * (BYTE ? 256 : 1024);
  const int stage_bytes = NW * KP * 12;
  const int region0 = lut_bytes > stage_bytes ? lut_bytes : stage_bytes;
  LDS unsigned char *smem3 = (LDS unsigned char *)smem;
  LDS float *lut = (LDS float *)smem3;
  LDS float *sq = (LDS float *)(smem3 + region0);
  const int sq_bytes = 2 * ((D * 4 + 15) & ~15);  // the query, then the residual of the current list
  LDS float *sres = sq + (sq_bytes >> 3);
  LDS int64_t *queue_id = (LDS int64_t *)(smem3 + region0 + sq_bytes);
  LDS uint32_t *queue_d = (LDS uint32_t *)(smem3 + region0 + sq_bytes + NW * 64 * 8);
  LDS uint32_t *tau_words = (LDS uint32_t *)(smem3 + region0 + sq_bytes + NW * 64 * 12);
  // per-probe list metadata of up to META probes, staged once per chunk of probes so
  // that a probe does not start with a chain of dependent scalar loads
  constexpr int META = 64;
  const int tau_bytes = (4 * (2 * NW + 4) + 15) & ~15;  // bound | ranks [NW] | wide: slots taken, overflow | wide: counts [NW]
  LDS int64_t *meta_row0 = (LDS int64_t *)(smem3 + region0 + sq_bytes + NW * 64 * 12 + tau_bytes);
  LDS int64_t *meta_blk = meta_row0 + META;
  LDS int32_t *meta_len = (LDS int32_t *)(meta_blk + META);
  LDS int32_t *meta_c = meta_len + META;
  LDS float *meta_lb = (LDS float *)(meta_c + META);
  LDS float *sr2 = meta_lb + META;  // [M] r_m^2 of this query
  LDS uint32_t *srmin = (LDS uint32_t *)(sr2 + IVFPQ_MAX_M);  // [M][4] partial minima (bit patterns) of each row of the current table

  int tid = threadIdx.x;
  if (KIND == SCAN_LISTED) asm volatile("" : "+v"(tid));   // (addresses formed anew for every query: kept across queries, they spill)
  int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform, kept in a scalar register
  LDS float *ssuf = (LDS float *)(srmin + 4 * IVFPQ_MAX_M) + wave * SUF_SLOTS;  // this wavefront's suffix sums of srmin, per 8 subspaces
  LDS uint32_t *stat = (LDS uint32_t *)((LDS float *)(srmin + 4 * IVFPQ_MAX_M) + NW * SUF_SLOTS);  // blocks scanned / scanned to the end
  const int p_begin = SPLIT ? (int)((int64_t)a.nprobe * split / a.nsplit) : 0;
  const int p_end = SPLIT ? (int)((int64_t)a.nprobe * (split + 1) / a.nsplit) : a.nprobe;
  const int32_t *probes = a.probe_ids + q * a.probe_stride;
  // with a query map only the queries it names are served (uniform over the workgroup)
  if (a.qmap && a.qmap[q] < 0) return;
  // Bound on the query's k-th distance from the workgroups that serve its other probe groups, as
  // its complement (0: none yet).  Any workgroup's own bound is an upper bound on the final k-th
  // distance, so the smallest of them is one too, and a late value is only looser.
  uint32_t *const gb = SPLIT && a.gbound ? a.gbound + q : nullptr;
  uint32_t gseen = gb ? __hip_atomic_load(gb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
  if (SPLIT && gb && a.probe_lb) {
    // a group whose lists are all ruled out needs neither codebook nor metadata: its list is empty
    // (one wavefront decides for all: the bound may change between two reads of it)
    LDS uint32_t *alive = (LDS uint32_t *)lut;   // free until the first table is built, two barriers on
    if (wave == 0) {
      const float b = __uint_as_float(~gseen);
      bool in = gseen == 0u;
      for (int p = p_begin + lane; p < p_end; p += 64) in = in || a.probe_lb[q * a.probe_stride + p] <= b;
      if (lane == 0) *alive = 0u;
      if (__ballot(in) != 0 && lane == 0) *alive = 1u;
    }
    __syncthreads();
    if (*(volatile LDS uint32_t *)alive == 0u) {
      if (tid < KP) a.part_d[(q * a.nsplit + split) * KP + tid] = SENT_D;
      return;
    }
  }

  int64_t dump_pos = 0;
  if (DUMP) {
    int64_t total = 0;
    for (int p = 0; p < a.nprobe; ++p) {
      const int32_t c = probes[p];
      if ((uint32_t)c < (uint32_t)a.nlist) total += a.list_offsets[c + 1] - a.list_offsets[c];
    }
    if (total != a.cand_offsets[q + 1] - a.cand_offsets[q]) {
      if (tid == 0) atomicAdd(a.errors, 1);
      return;
    }
    dump_pos = a.cand_offsets[q];
  }

  // What a chunk of probes needs of its lists, a thread per probe: two trips to memory, one behind the
  // other.  The first chunk's first trip goes out before anything else, its second behind the
  // codebook's.
  struct ProbeMeta {
    int32_t c;
    int64_t r0, r1, blk;
    float lb;
  };
  auto fetch_probe = [&](int p0) __attribute__((always_inline)) { return tid < META && p0 + tid < p_end ? probes[p0 + tid] : -1; };
  auto fetch_meta = [&](int p0, int32_t cc) __attribute__((always_inline)) {
    ProbeMeta f = {0, 0, 0, 0, 0.0f};
    {
      if ((uint32_t)cc < (uint32_t)a.nlist) {   // a probe id outside [0, nlist) becomes an empty list
        f.c = cc;
        f.r0 = a.list_offsets[cc];
        f.r1 = a.list_offsets[cc + 1];
        f.blk = a.list_blocks[cc];
        if (a.probe_lb) f.lb = a.probe_lb[q * a.probe_stride + p0 + tid];
      }
    }
    return f;
  };
  auto put_meta = [&](const ProbeMeta &f, int p0) __attribute__((always_inline)) {
    if (tid < META && p0 + tid < p_end) {
      meta_c[tid] = f.c;
      meta_row0[tid] = f.r0;
      meta_len[tid] = (int)(f.r1 - f.r0);
      meta_blk[tid] = f.blk;
      meta_lb[tid] = f.lb;
    }
  };
  const int32_t first_probe = fetch_probe(p_begin);
  for (int i = tid; i < D; i += NT) sq[i] = a.queries[q * D + i];
  for (int m = tid; m < MT; m += NT) {
    float v = r2.v[m];
    if (a.query_radii && m < M) {
      const float r = a.query_radii[q * M + m];
      v = r * r;
    }
    sr2[m] = v;
    srmin[4 * m] = srmin[4 * m + 1] = srmin[4 * m + 2] = srmin[4 * m + 3] = 0u;
  }
  const int mode = a.mode;
  if (tid <= NW) tau_words[tid] = tid == 0 ? ~gseen : SENT_D;
  if (tid < 2) stat[tid] = 0u;
  const bool wide = !DUMP && a.wide_cap > 0;
  if (tid < 2) tau_words[NW + 1 + tid] = 0u;
  SharedTau sh;
  sh.bound = tau_words;
  sh.rank = tau_words + 1;
  sh.nw = NW;
  sh.wave = wave;
  // wide selection: the bound is on the k_out-th distance, from ceil(k_out / NW) keys per wavefront
  sh.jrank = ((wide ? a.k_out : a.k) + NW - 1) / NW;
  sh.wide = wide ? tau_words + NW + 1 : nullptr;
  sh.wide_d = wide ? a.wide_d + q * a.wide_cap : nullptr;
  sh.wide_id = wide ? a.wide_id + q * a.wide_cap : nullptr;
  sh.wide_cap = a.wide_cap;

  WaveTop st;
  init_wave_top<false, DUMP>(st, a, q);
  LDS uint32_t *qd = queue_d + wave * 64;
  LDS int64_t *qid = queue_id + wave * 64;

  // Codebook rows of this wavefront (rows wave, wave + NW, ...): the first RES of them
  // stay in registers for the whole kernel -- the codebook is the same for every list
  // and re-reading all of it per list costs a quarter of the kernel on short lists --
  // the remaining STR are streamed per list.  RES is what fits beside the scan's
  // registers at 4 wavefronts per SIMD.
  constexpr bool VEC = DSUB == 2 || DSUB == 4;
  constexpr int ITER = (MT + NW - 1) / NW;
  constexpr int DS4 = VEC ? DSUB : 1;
  constexpr int WPE = scan_wpe(BYTE ? (MT + 3) / 4 : MT, NW);
  // (a dsub = 4 row takes 16 registers and its table arithmetic more temporaries: with resident
  // rows the kernel spilled up to 198 registers, so those rows are all streamed)
  constexpr int RES_REGS = DS4 == 4 ? 0 : res_regs(WPE), RES_MAX_TOTAL = res_max_total(WPE);
  constexpr int RES_BUDGET = RES_REGS < RES_MAX_TOTAL - 2 * (MPT / 4) ? RES_REGS : RES_MAX_TOTAL - 2 * (MPT / 4);
  constexpr int RES_CAP = (RES_BUDGET > 0 ? RES_BUDGET : 0) / (4 * DS4);
  constexpr int RES = !VEC ? 0 : (ITER < RES_CAP ? ITER : RES_CAP);
  constexpr int STR = VEC ? ITER - RES : 0;
  float4 cbr[RES > 0 ? RES : 1][DS4];
  if constexpr (VEC) {
#pragma unroll
    for (int it = 0; it < RES; ++it) {
      const int m = wave + it * NW;
      const int mc = m < MT ? m : MT - 1;
      const GLOBAL uint8_t *cb = uniform_ptr(a.codebooks + (int64_t)mc * 256 * DSUB);
#pragma unroll
      for (int x = 0; x < DSUB; ++x)
        cbr[it][x] = load_f4(cb, (uint32_t)(lane * 16 * DSUB + 16 * x));
    }
  }
  const ProbeMeta first_meta = fetch_meta(p_begin, first_probe);
  // Code chunks per point (16-byte chunks, then 4-byte chunks) and how many of them
  // the "first half" loading mode fetches ahead; that mode exists when it splits the
  // chunks in two non-empty parts.
  constexpr int NCH = MPT / 16 + (MPT % 16) / 4;
  constexpr int HCH = (MPT / 16 + 1) / 2;
  constexpr int MH = 16 * HCH;  // subspaces covered by the first HCH chunks
  constexpr bool HALF_OK = HCH >= 1 && HCH < NCH && MH < MT;
  constexpr bool QUARTER_OK = HALF_OK && HCH >= 2;  // the first chunk alone (16 subspaces) is a proper part
  // How much of a block is fetched ahead: 0 all chunks, 1 the first half, 2 the first chunk;
  // the rest is fetched when a block turns out to need it.  While pruning, most blocks end
  // within their first chunk.
  int depth = 0, depth_later = 0;
  if (HALF_OK && !DUMP && a.load_mode != 1) depth_later = (QUARTER_OK && a.load_mode != 2) ? 2 : 1;
  // the first list of a query is scanned without any bound, so every block of it is needed
  // whole: it is fetched whole (in the default mode), the lists after it by parts
  if (a.load_mode != 0) depth = depth_later;
  auto load_part = [&](auto j0, auto j1, const uint8_t *lb, int nblk, int blk, CodeRegs<MPT / 4> &r) __attribute__((always_inline)) {
    constexpr int J0 = decltype(j0)::value, J1 = decltype(j1)::value;
    if constexpr (RT) load_chunks_rt<MPT, J0, J1>(lb, nblk, blk, lane, Mp, r);
    else load_chunks<MPT, J0, J1>(lb, nblk, blk, lane, r);
  };
  std::integral_constant<int, 0> c0;
  std::integral_constant<int, 1> c1;
  std::integral_constant<int, HALF_OK ? 1 : NCH> cA;   // what is always fetched ahead ends here
  std::integral_constant<int, HCH> cH;
  std::integral_constant<int, NCH> cE;
  auto load_ahead = [&](const uint8_t *lb, int nblk, int blk, CodeRegs<MPT / 4> &r) __attribute__((always_inline)) {
    load_part(c0, cA, lb, nblk, blk, r);
    if constexpr (HALF_OK) {
      if (depth < 2) load_part(c1, cH, lb, nblk, blk, r);
      if (depth < 1) load_part(cH, cE, lb, nblk, blk, r);
    }
  };
  bool sres_ready = false;
  // Pruning (row minima, checks of the partial sums, partial loads) pays only where blocks
  // do end early.  The workgroup counts, over the first PROBE_LISTS lists of its query, how
  // many blocks were scanned and how many of them to the end; if nearly all were, the rest
  // of the lists are scanned plainly.  Results do not depend on it.
  constexpr int PROBE_LISTS = 4;
  bool prune = !DUMP && !(a.ablate & 16);
  uint32_t tot_blocks = 0, tot_full = 0;
  bool pushed = false, decided = (a.ablate & 16) != 0;
  auto push_counts = [&](int last_list) __attribute__((always_inline)) {
    if (!DUMP && !pushed && last_list - p_begin >= PROBE_LISTS - 1) {
      pushed = true;
      if (lane == 0) {
        __hip_atomic_fetch_add(stat, tot_blocks, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_fetch_add(stat + 1, tot_full, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
  };
  put_meta(first_meta, p_begin);
  __syncthreads();
  for (int p = p_begin; p < p_end; ++p) {
    // (addresses formed anew for every list: kept across lists, they spill)
    asm volatile("" : "+v"(tid), "+v"(lane));
    const int pm = (p - p_begin) & (META - 1);
    if (pm == 0) {
      // (every wavefront has passed the second barrier of the previous probe, so nobody still
      // reads the old entries; the first chunk is there already)
      if (p > p_begin) {
        put_meta(fetch_meta(p, fetch_probe(p)), p);
        __syncthreads();
      }
    }
    const int32_t c = __builtin_amdgcn_readfirstlane(meta_c[pm]);
    const int64_t row0 = meta_row0[pm];
    const int len = __builtin_amdgcn_readfirstlane(meta_len[pm]);
    const int nb = (len + 63) >> 6;
    const uint8_t *base = a.codes + meta_blk[pm] * ivfpq_block_bytes(Mp);
    const float *cen = a.centroids + (int64_t)c * D;
    // Loads that do not depend on LDS go out before the barrier, so that their
    // latency overlaps the tail of the previous list: the streamed part of this
    // wavefront's codebook rows and the first code block of the new list.
    float4 cbs[STR > 0 ? STR : 1][DS4];
    CodeRegs<MPT / 4> nxt;
    // The residual q - centroid of a list is formed once, in LDS.  For the list after
    // this one the centroid is requested now and the residual written after this
    // list's table is finished, so the next table does not wait for it.
    const bool next_known = D <= NT && pm + 1 < META && p + 1 < p_end;
    float cen_next = 0.0f;
    if (!sres_ready)
      for (int i = tid; i < D; i += NT) sres[i] = sq[i] - cen[i];
    if (next_known && tid < D)
        cen_next = *reinterpret_cast<const GLOBAL float *>(
            uniform_ptr(a.centroids + (int64_t)__builtin_amdgcn_readfirstlane(meta_c[pm + 1]) * D) + (uint32_t)(tid * 4));
    if constexpr (VEC) {
#pragma unroll
      for (int it = 0; it < STR; ++it) {
        const int m = wave + (RES + it) * NW;
        const int mc = m < MT ? m : MT - 1;
        const GLOBAL uint8_t *cb = uniform_ptr(a.codebooks + (int64_t)mc * 256 * DSUB);
#pragma unroll
        for (int x = 0; x < DSUB; ++x)
          cbs[it][x] = load_f4(cb, (uint32_t)(lane * 16 * DSUB + 16 * x));
      }
    }
    {
      // an empty list still has readable padding behind its base
      // (with 128 registers only the first chunk goes out here, whatever the depth: the
      // registers of the other chunks stay free while the table is built)
      const int b0 = wave < nb ? wave : (nb > 0 ? nb - 1 : 0);
      if constexpr (WPE == 2) load_ahead(base, nb, b0, nxt);
      else load_part(c0, cA, base, nb, b0, nxt);
    }
    __syncthreads();  // previous list fully scanned (and sq written) before the table changes
    if (!DUMP && wide && sh.wide[0] > (uint32_t)(a.wide_cap >> 2) && sh.wide[1] == 0u)
      wide_compact<NW>(sh, tau_words + NW + 3, tid, lane, wave);
    if (!DUMP && !decided && p - p_begin >= PROBE_LISTS) {  // every wavefront has pushed its counts
      decided = true;
      if (!(a.ablate & 32)) {
        const uint32_t nblk = stat[0], nfull = stat[1];
        prune = 8 * (uint64_t)nfull < 7 * (uint64_t)nblk;
      }
    }
    // List-level bound (probe_bound_kernel): if not even the lower bound on any point of
    // this list is within the workgroup's bound on the k-th distance, neither table nor scan
    // is needed.  Between the two barriers nobody scans, so every wavefront reads the same
    // shared bound and the decision is uniform over the workgroup.
    bool skip_list = false;
    if (!DUMP) {
      const uint32_t bnd = *(volatile LDS uint32_t *)sh.bound;
      skip_list = bnd != SENT_D && meta_lb[pm] > __uint_as_float(bnd);
    }
    if (skip_list) {
      // Ruled out.  The bound cannot change while nobody scans, so the following probes of
      // this metadata chunk are checked right here and the workgroup goes on with the first
      // one that is not ruled out: a run of skipped lists costs one barrier.
      // A lane per probe of the chunk finds its end at once (probe by probe, each with its own trip
      // to the LDS, 60 ruled-out lists took 20 of the 100 thousand clocks of a query of the
      // 1M x 200 configuration).
      const float bound_f = __uint_as_float(*(volatile LDS uint32_t *)sh.bound);
      const int left = p_end - (p - pm) < META ? p_end - (p - pm) : META;   // probes of this chunk
      const bool mine = lane >= pm && lane < left;
      const unsigned long long dead = __ballot(mine && meta_lb[mine ? lane : pm] > bound_f) >> pm;
      const int run = ~dead == 0ull ? 64 : __ffsll((long long)~dead) - 1;   // >= 1: this probe is ruled out
      const int pn = p + run;
      if (!pushed) {   // all pruned: counts for the switch
        const int nbn = mine && lane < pm + run ? (meta_len[lane] + 63) >> 6 : 0;
        uint32_t c = wave < nbn ? (uint32_t)((nbn - 1 - wave) / NW + 1) : 0u;
        c += xor_u32<1, true>(c);
        c += xor_u32<2, true>(c);
        c += xor_u32<4, true>(c);
        c += xor_u32<8, true>(c);
        c += xor_u32<16, true>(c);
        c += xor_u32<32, true>(c);
        tot_blocks += (uint32_t)__builtin_amdgcn_readfirstlane((int)c);
      }
      push_counts(pn - 1);
      __syncthreads();  // nobody still reads the metadata when the next chunk is staged
      sres_ready = false;
      p = pn - 1;
      continue;
    }
    // ---- selective table for (query, list c) ----
    {
      // one subspace per wavefront and pass, four consecutive entries per lane; the
      // scoring mode is resolved once per list, outside the unrolled passes
      [[maybe_unused]] auto build_rows = [&](auto mode_tag) __attribute__((always_inline)) {
        constexpr int MODE = decltype(mode_tag)::value;
        constexpr int NBATCH = (ITER + 7) / 8;
        uint32_t lo[NBATCH][8];  // this lane's minimum over its entries of each row (for the early exit)
#pragma unroll
        for (int it = 0; it < NBATCH * 8; ++it) lo[it >> 3][it & 7] = 0xFFFFFFFFu;
        // With 256 registers (WPE == 2) the passes form straight-line code (the validity of
        // a row is known at compile time for every pass but the last) and the compiler
        // overlaps their LDS reads.  With 128 registers that form spills, so each row stays
        // a block of its own.
        constexpr bool STRAIGHT = WPE == 2;
#pragma unroll
        for (int it = 0; it < ITER; ++it) {
          const int m = wave + it * NW;
          if ((STRAIGHT && (it + 1) * NW <= MT) || m < MT) {
            float res[DS4];
#pragma unroll
            for (int j = 0; j < DS4; ++j) res[j] = sres[m * DSUB + j];
            const float4 v = lut_entry4<DSUB, MODE>(res, it < RES ? cbr[it < RES ? it : 0] : cbs[it >= RES ? it - RES : 0], sr2[m]);
            if constexpr (BYTE)   // penalties 0, 1, 2: four entries in one dword
              *((LDS uint32_t *)lut + m * 64 + lane) = (uint32_t)v.x | ((uint32_t)v.y << 8) | ((uint32_t)v.z << 16) | ((uint32_t)v.w << 24);
            else
              *(LDS floatx4 *)(lut + m * 256 + 4 * lane) = floatx4{v.x, v.y, v.z, v.w};
            if (!DUMP)
              lo[it >> 3][it & 7] = umin32(umin32(__float_as_uint(v.x), __float_as_uint(v.y)),
                                           umin32(__float_as_uint(v.z), __float_as_uint(v.w)));
          }
        }
        if (!DUMP && prune) {
          // one partial minimum per row and 16 lanes goes to LDS; the reader takes the
          // smallest of the four
#pragma unroll
          for (int bt = 0; bt < NBATCH; ++bt) {
            const uint32_t d = rows8_min16(lo[bt], lane);
            const int it = bt * 8 + (lane & 7);
            const int m = wave + it * NW;
            if ((lane & 15) < 8 && it < ITER && m < MT) srmin[4 * m + (lane >> 4)] = d;
          }
        }
      };
      // run-time shapes: a row at a time, its minima over 16 lanes straight to LDS
      [[maybe_unused]] auto build_rows_rt = [&](auto mode_tag) __attribute__((always_inline)) {
        lut_rows_rt<decltype(mode_tag)::value>(sres, sr2, a.codebooks, wave, M, NW, a.dsub, lane, [&](int m, float4 v, auto strided) __attribute__((always_inline)) {
          if constexpr (decltype(strided)::value) {
            lut[m * 256 + lane] = v.x;
            lut[m * 256 + 64 + lane] = v.y;
            lut[m * 256 + 128 + lane] = v.z;
            lut[m * 256 + 192 + lane] = v.w;
          } else {
            *(LDS floatx4 *)(lut + m * 256 + 4 * lane) = floatx4{v.x, v.y, v.z, v.w};
          }
          if (!DUMP && prune) {
            uint32_t lo = umin32(umin32(__float_as_uint(v.x), __float_as_uint(v.y)), umin32(__float_as_uint(v.z), __float_as_uint(v.w)));
            lo = umin32(lo, xor_u32<1, true>(lo));
            lo = umin32(lo, xor_u32<2, true>(lo));
            lo = umin32(lo, xor_u32<4, true>(lo));
            lo = umin32(lo, xor_u32<8, true>(lo));
            if ((lane & 15) == 0) srmin[4 * m + (lane >> 4)] = lo;
          }
        });
      };
      auto build = [&](auto mode_tag) __attribute__((always_inline)) {
        if constexpr (RT) build_rows_rt(mode_tag);
        else build_rows(mode_tag);
      };
      if (mode == 0) build(std::integral_constant<int, 0>{});
      else if (mode == 1) build(std::integral_constant<int, 1>{});
      else build(std::integral_constant<int, 2>{});
    }
    __syncthreads();
    if (next_known && tid < D) sres[tid] = sq[tid] - cen_next;  // this list's table is complete
    sres_ready = next_known;
    if (SPLIT && gb) gseen = __hip_atomic_load(gb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // arrives during the scan
    // ---- distance calculation over list c ----
    {
      // Two register sets: `nxt` receives the loads of the next block while `cur` is
      // looked up.  Loads are issued for every iteration (past the end they re-read the
      // list's last block, which is in bounds), so the block in flight never has to
      // complete before the current one can be used.
      // Suffix sums of the row minima at the check points (every 8 subspaces), per wavefront:
      // lane l holds rows l and 64 + l, groups of 8 lanes are summed in place, then the
      // groups are accumulated from the last one down.
      float suf0 = 0.0f;
      if (!DUMP && prune) {
        constexpr int NG = (MT + 7) / 8;
        auto row_min = [&](int m) {
          const uintx4 p = *(const LDS uintx4 *)(srmin + 4 * m);
          return __uint_as_float(umin32(umin32(p[0], p[1]), umin32(p[2], p[3])));
        };
        float v0 = lane < MT ? row_min(lane) : 0.0f;
        float v1 = (MT > 64 && lane + 64 < MT) ? row_min((MT > 64 ? 64 : 0) + lane) : 0.0f;
        v0 = group8_sum(v0);
        v1 = group8_sum(v1);
        float acc = 0.0f;
#pragma unroll
        for (int j = NG - 1; j >= 0; --j) {
          const int gl = __builtin_amdgcn_readlane((int)__float_as_uint(j < 8 ? v0 : v1), (j & 7) * 8);
          acc += __uint_as_float((uint32_t)gl);
          if (lane == 0) ssuf[j] = acc;
        }
        if (lane == 0) ssuf[NG] = 0.0f;
        suf0 = acc;
      }
      if (wave < nb) {
        const int last = nb - 1;
        int blocks = 0, full = 0;
        if constexpr (HALF_OK && WPE != 2) {  // the rest of what is fetched ahead of the first block
          if (depth < 2) load_part(c1, cH, base, nb, wave, nxt);
          if (depth < 1) load_part(cH, cE, base, nb, wave, nxt);
        }
        for (int b = wave; b < nb; b += NW) {
          CodeRegs<MPT / 4> cur = nxt;
          const int bn = b + NW < last ? b + NW : last;
          load_ahead(base, nb, bn, nxt);
          const int i = b * 64 + lane;
          const bool valid = i < len;
          if (DUMP) {
            const float dist = BYTE ? adc_sum_bytes<MT>(lut, cur) : adc_sum<MT, RT>(lut, cur, 0.0f, M);
            if (valid) {
              a.all_dist[dump_pos + i] = dist;
              a.all_ids[dump_pos + i] = a.ids[row0 + i];
            }
          } else {
            const uint32_t shared = *(volatile LDS uint32_t *)sh.bound;
            const uint32_t pref = (a.ablate & 8) ? SENT_D : ((wide || shared < st.tau.d) ? shared : st.tau.d);
            // bound on the k-th smallest distance, enlarged as adc_part_exit needs it
            const float tauf = pref == SENT_D ? __builtin_inff() : __uint_as_float(pref) * 1.0001220703125f;
            Acc dist = 0;
            ++blocks;
            // no point of this list can reach the bound any more (it only tightens): the
            // wavefront is done with the list, and requests no further blocks of it
            if (prune && !(suf0 <= tauf)) {
              blocks += (nb - 1 - b) / NW;
              break;
            }
            // The block in up to three parts (first chunk, rest of the first half, second
            // half); most blocks end in an early part, and a part that was not fetched ahead
            // is fetched when a block turns out to need it.
            if constexpr (QUARTER_OK) {
              if (!adc_part_exit<MT, 0, 16, RT>(lut, cur, ssuf, tauf, prune, valid, dist, M)) continue;
              if (depth == 2) load_part(c1, cH, base, nb, b, cur);
              if (!adc_part_exit<MT, 16, MH, RT>(lut, cur, ssuf, tauf, prune, valid, dist, M)) continue;
            } else if constexpr (HALF_OK) {
              if (!adc_part_exit<MT, 0, MH, RT>(lut, cur, ssuf, tauf, prune, valid, dist, M)) continue;
            }
            if constexpr (HALF_OK) {
              if (depth >= 1) load_part(cH, cE, base, nb, b, cur);
            }
            if (!adc_part_exit<MT, HALF_OK ? MH : 0, MT, RT>(lut, cur, ssuf, tauf, prune, valid, dist, M)) continue;
            ++full;
            wave_offer(st, acc_value(dist), valid, row0 + i, a.ids, qd, qid, lane, a.k, sh);
          }
        }
        tot_blocks += blocks;
        tot_full += full;
      }
      // without pruning every block is needed whole; the list during which pruning was
      // switched off still had its blocks fetched by halves
      depth = (!prune && a.load_mode < 2) ? 0 : depth_later;
      push_counts(p);
    }
    if (DUMP) dump_pos += len;
    if (SPLIT && gb && tid == 0) {   // exchange bounds with the query's other workgroups
      const uint32_t own = *(volatile LDS uint32_t *)sh.bound;
      if (own < ~gseen) __hip_atomic_fetch_max(gb, ~own, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else __hip_atomic_fetch_min(sh.bound, ~gseen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  }
  if (DUMP) return;
  if (wide) finish_wide(st, qd, qid, lane, tid, sh, a, q);
  else finish_topk<NW>(st, qd, qid, lane, wave, sh, smem3, a, q, split, gb);
}

template <int MT, int DSUB, int NW, int KIND, bool BYTE = false>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(scan_wpe(BYTE ? (MT + 3) / 4 : MT, NW)))) void scan_kernel(ScanArgs a, RadiiSq r2) {
  if constexpr (KIND == SCAN_SPLIT) {
    // Probe groups in the order of their lists: the workgroups with the nearest lists of all queries
    // come first, so that the bounds they publish (a.gbound) are there when most of the others start.
    const int nq = gridDim.x / a.nsplit;
    scan_query<MT, DSUB, NW, KIND, BYTE>(a, r2, blockIdx.x % nq, blockIdx.x / nq);
  } else if constexpr (KIND == SCAN_LISTED) {
    extern __shared__ __align__(16) unsigned char smem[];
    LDS int *shared_next = (LDS int *)smem;   // the table's first word: free between two queries
    const int n = a.qlist_n[0];
    for (int i = blockIdx.x; i < n;) {
      int next = n;
      if (threadIdx.x == 0 && n > (int)gridDim.x) next = (int)gridDim.x + atomicAdd(a.qlist_n + 1, 1);   // arrives during the query
      scan_query<MT, DSUB, NW, KIND, BYTE>(a, r2, a.qlist[i], 0);
      __syncthreads();
      if (threadIdx.x == 0) *shared_next = next;
      __syncthreads();
      i = __builtin_amdgcn_readfirstlane(*shared_next);
    }
  } else {
    scan_query<MT, DSUB, NW, KIND, BYTE>(a, r2, blockIdx.x, 0);
  }
}

template <int MT, int DSUB, int NW, bool BYTE = false>
int launch_scan_t(const ScanArgs &a, const RadiiSq &r2, int64_t grid, bool dump, hipStream_t s) {
  const int lut_bytes = a.M * (BYTE ? 256 : 1024), stage = NW * KP * 12;
  const size_t lds = (size_t)(lut_bytes > stage ? lut_bytes : stage) + 2 * ((a.D * 4 + 15) & ~15) +
                     (size_t)NW * 64 * 12 + ((4 * (2 * NW + 4) + 15) & ~15) + 64 * 28 + 5 * IVFPQ_MAX_M * 4 +
                     (size_t)NW * SUF_SLOTS * 4 + 16;
  static_assert(NW * 64 * 12 + 64 * 28 + 5 * IVFPQ_MAX_M * 4 >= 7 * 1024, "lookup_tail reads at most seven rows behind the table");
  if (lds > (size_t)LDS_PER_CU) {
    ivfpq::set_error("scan: %zu bytes of LDS needed, 163840 available", lds);
    return IVFPQ_ERR_UNSUPPORTED;
  }
  const int kind = dump ? SCAN_ALL : (a.nsplit > 1 ? SCAN_SPLIT : (a.qlist ? SCAN_LISTED : SCAN_TOPK));
  auto kern = kind == SCAN_ALL ? scan_kernel<MT, DSUB, NW, SCAN_ALL, BYTE>
                               : (kind == SCAN_SPLIT ? scan_kernel<MT, DSUB, NW, SCAN_SPLIT, BYTE> : scan_kernel<MT, DSUB, NW, SCAN_TOPK, BYTE>);
  if constexpr (DSUB != 0)   // (the shapes the list-major scan hands queries over for)
    if (kind == SCAN_LISTED) {
      kern = scan_kernel<MT, DSUB, NW, SCAN_LISTED, BYTE>;
      // as many as the chip holds at once: what a CU's LDS and its SIMDs' registers allow
      const int64_t waves = 4 * scan_wpe(BYTE ? (MT + 3) / 4 : MT, NW) / NW, fit = LDS_PER_CU / (int64_t)lds;
      const int64_t room = 256 * (waves < 1 ? 1 : (waves < fit ? waves : fit));
      if (grid > room) grid = room;
    }
  static std::atomic<uint64_t> prepared[4];
  if (int rc = prepare_kernel(kern, prepared[kind])) return rc;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(NW * 64), lds, s, a, r2);
  return IVFPQ_OK;
}

}  // namespace
