// List-major scan with fp32 tables of two queries, a table in parts of 16 subspaces (included by scan_lm.hip, which says what
// a group, the head pass and the main pass are).  Distances.
//
// lm_scan_kernel holds a whole table in LDS, 2 KiB a subspace: one workgroup per CU whose table, scan and selection follow
// one another (23, 36 and 33 of a hundred clocks of the head pass with 64 subspaces), and nothing at all beyond 78
// subspaces.  Here a part of the table goes by at a time, the sums of the points staying in registers in between, so that
// two workgroups share a CU and one's selection hides behind the other's look-ups.  The codebook comes from the L2 for
// every task instead of standing in registers.  Sums are formed in subspace order, as anywhere.
// A list is scanned LPP_SEG points at a time, and a longer one costs another table for each.
// Head pass of 10 000 queries over 1M points in 1024 lists, k = 100: 64 subspaces 242 us with lm_scan_kernel, 197 so; 100
// subspaces, which went query-major (1174 us), 299 (67 of the LDS' gathers alone, 10 lanes a clock and CU).

constexpr int LPP_NW = LM_NW;    // wavefronts of a workgroup
constexpr int LPP_WG = 2;        // workgroups per CU: 4 wavefronts per SIMD, 128 vector registers each
constexpr int LPP_PART = 16;     // subspaces of a part: a 16-byte chunk of the lists' layout
constexpr int LPP_NB = 4;        // blocks of 64 points whose sums a wavefront holds
constexpr int LPP_SEG = LPP_NW * LPP_NB * 64;   // points of a list that are scanned with one table
constexpr int LPP_BUF = LPP_PART * 2048;

constexpr size_t lpp_fixed_lds(int D) { return LPP_BUF + (size_t)LM_G * ((D + 3) & ~3) * 4 + (size_t)LM_G * IVFPQ_MAX_M * 4 + 16; }
size_t lpp_main_lds(int D) { return lpp_fixed_lds(D) + (size_t)LPP_NW * LM_G * 2 * LM_QUEUE * 4; }
// head pass: the distances of the list's points for both queries
constexpr int lpp_head_max(int D) {
  const int64_t spare = (int64_t)(LDS_PER_CU / LPP_WG) - (int64_t)lpp_fixed_lds(D) - LM_SEL_WORDS * 4 - LM_G * LM_BINS * 4;
  const int64_t n = spare / (LM_G * 4) & ~(int64_t)63;
  return n < 0 ? 0 : (int)n;
}
size_t lpp_head_lds(int D) { return lpp_fixed_lds(D) + (size_t)LM_G * lpp_head_max(D) * 4 + LM_SEL_WORDS * 4 + LM_G * LM_BINS * 4; }

template <int MT, int DSUB, bool HEAD>
__global__ __launch_bounds__(LPP_NW * 64) __attribute__((amdgpu_waves_per_eu(LPP_WG * LPP_NW / 4))) void lm_pair_kernel(LmArgs a, RadiiSq r2) {
  constexpr int NW = LPP_NW, NB = LPP_NB;
  constexpr bool RT = MT == 0;   // any number of subspaces, up to 128
  const int M = RT ? a.M : MT, Mp = RT ? a.Mp : (MT + 3) / 4 * 4;
  const int P = (M + LPP_PART - 1) / LPP_PART;
  constexpr int TAIL = MT % LPP_PART;   // subspaces of the last part where it is short
  constexpr int ROWS = LPP_PART / NW;   // rows of a part that a wavefront makes
  static_assert(TAIL == 0 || TAIL == 4, "16-byte chunks and one of 4 bytes");
  extern __shared__ __align__(16) unsigned char smem[];
  LDS unsigned char *smem3 = (LDS unsigned char *)smem;
  const int D = a.D;   // LM_G * D <= NT and LM_G * M <= NT: one element per thread (checked by the launcher)
  const int dpad = (D + 3) & ~3;
  // LDS carve: table [16][256][2] | residuals [2][dpad] | r_m^2 [2][MAX_M] | the task after the next | head pass: selection
  // state, histograms, distances [2][head_max]; main pass: queues
  LDS float *sres = (LDS float *)(smem3 + LPP_BUF);
  LDS float *sr2 = sres + LM_G * dpad;
  LDS int32_t *t_after = (LDS int32_t *)(sr2 + LM_G * IVFPQ_MAX_M);
  LDS uint32_t *queue = (LDS uint32_t *)(t_after + 4);   // main pass: [NW][G][2][LM_QUEUE]
  LDS uint32_t *ssel = queue;                            // head pass: [LM_SEL_WORDS]
  LDS uint32_t *hist = queue + LM_SEL_WORDS;             // [2][LM_BINS]
  LDS uint32_t *sdist = hist + LM_G * LM_BINS;           // [2][head_max]

  int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  LDS uint32_t *qd0 = queue + (wave * LM_G + 0) * 2 * LM_QUEUE, *qrow0 = qd0 + LM_QUEUE;
  LDS uint32_t *qd1 = queue + (wave * LM_G + 1) * 2 * LM_QUEUE, *qrow1 = qd1 + LM_QUEUE;

  // Tasks as in lm_part_kernel: the first two of a workgroup are given, further ones are drawn.
  const int ntasks = a.base[a.nlist] / LM_G;
  const int nwg = gridDim.x, b = blockIdx.x;
  const int xcds = (nwg & 7) == 0 ? 8 : 1, run = nwg / xcds, xcd = b % xcds;
  auto task_of = [&](int n) __attribute__((always_inline)) { return n / run * nwg + xcd * run + n % run; };
  const int t = task_of(b / xcds);
  int t_next = task_of(b / xcds + run);
  int32_t *ticket = a.cnt + ivfpq::lm_tickets(a.nlist, a.stage) + xcd * ivfpq::LM_TICKET_STEP;
  if (t >= ntasks) return;

  // what this thread contributes to a task's residuals and radii: element tid of [2][D] / [2][MT]
  const int rg = tid >= D ? 1 : 0, rd = tid - rg * D;
  const bool r_on = tid < LM_G * D;
  const int mg = tid >= M ? 1 : 0, mm = tid - mg * M;
  const bool m_on = tid < LM_G * M;

  // this wavefront's rows of a part: 16 part + wave, and 8 further on
  float4 row[ROWS][DSUB];
  auto load_rows = [&](int part) __attribute__((always_inline)) {
#pragma unroll
    for (int it = 0; it < ROWS; ++it) {
      const int m = part * LPP_PART + it * NW + wave;
      const GLOBAL uint8_t *cb = uniform_ptr(a.codebooks + (int64_t)(m < M ? m : M - 1) * 256 * DSUB);
#pragma unroll
      for (int x = 0; x < DSUB; ++x) row[it][x] = load_f4(cb, (uint32_t)(lane * 16 * DSUB + 16 * x));
    }
  };
  uintx4 code[NB];   // a part's codes of the wavefront's blocks
  auto load_codes = [&](const uint8_t *base, int nb, int seg, int part, int i) __attribute__((always_inline)) {
    const int at = seg + wave + i * NW, blk = at < nb ? at : nb - 1;   // no such block: the last one
    if (RT ? part < (Mp >> 4) : (TAIL == 0 || part < P - 1)) {
      const GLOBAL uint8_t *sp = uniform_ptr(base + ((int64_t)part * nb + blk) * 1024);
      code[i] = *(const GLOBAL uintx4 *)(sp + (uint32_t)(lane * 16));
    } else if constexpr (RT) {
      code[i] = uintx4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int t = 0; t < 3; ++t)
        if (t < ((Mp >> 2) & 3)) {
          const GLOBAL uint8_t *sp = uniform_ptr(base + (int64_t)(Mp >> 4) * nb * 1024 + ((int64_t)t * nb + blk) * 256);
          code[i][t] = *(const GLOBAL uint32_t *)(sp + (uint32_t)(lane * 4));
        }
    } else {
      const GLOBAL uint8_t *sp = uniform_ptr(base + (int64_t)(MT / 16) * nb * 1024 + (int64_t)blk * 256);
      code[i] = uintx4{*(const GLOBAL uint32_t *)(sp + (uint32_t)(lane * 4)), 0u, 0u, 0u};
    }
  };

  // (vector loads for what all lanes want alike: see lm_scan_kernel)
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
  float qv = 0.0f, cv = 0.0f, rv = 0.0f;
  auto fetch_task = [&](const int2 &pv, int64_t mv, LmTask &tk) __attribute__((always_inline)) {
    tk.c = __builtin_amdgcn_readlane(pv.y, 0);
    tk.q0 = __builtin_amdgcn_readlane(pv.x, 0);
    tk.has1 = __builtin_amdgcn_readlane(pv.x, 1) >= 0;
    tk.q1 = tk.has1 ? __builtin_amdgcn_readlane(pv.x, 1) : tk.q0;
    tk.row0 = lane64(mv, 0);
    tk.len = (int)(lane64(mv, 1) - tk.row0);
    tk.nb = (tk.len + 63) >> 6;   // >= 1: only non-empty lists have tasks
    tk.base = a.codes + lane64(mv, 2) * ivfpq_block_bytes(Mp);
    tk.tauv = 0.0f;
    if constexpr (!HEAD) tk.tauv = a.tau[(lane == 0 ? tk.q0 : tk.q1) * a.tau_stride];
    if (r_on) {
      qv = a.queries[(rg ? tk.q1 : tk.q0) * D + rd];
      cv = a.centroids[(int64_t)tk.c * D + rd];
    }
    if (m_on) {
      rv = r2.v[mm];
      if (a.query_radii) {
        const float r = a.query_radii[(mg ? tk.q1 : tk.q0) * M + mm];
        rv = r * r;
      }
    }
  };
  auto put_task = [&]() __attribute__((always_inline)) {
    if (r_on) sres[rg * dpad + rd] = qv - cv;
    if (m_on) sr2[mg * IVFPQ_MAX_M + mm] = rv;
    if constexpr (HEAD) {
      if (tid < LM_SEL_WORDS) ssel[tid] = (tid == 4 || tid == 5) ? 0xFFFFFFFFu : 0u;   // see lm_scan_kernel
      for (int i = tid; i < LM_G * LM_BINS; i += NW * 64) hist[i] = 0u;
    }
  };

  LmTask tk;
  int2 npv = make_int2(0, 0);   // pair entries of the next task
  int64_t nmv = 0;              // ... and its list's metadata
  {
    const int2 pv = fetch_pairs(t);
    if (t_next < ntasks) npv = fetch_pairs(t_next);
    load_rows(0);
    fetch_task(pv, fetch_meta(pv), tk);
    put_task();
#pragma unroll
    for (int i = 0; i < NB; ++i) load_codes(tk.base, tk.nb, 0, 0, i);
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

  int part = 0, seg = 0;   // the part of the table; the first block of the points that are scanned with it
  bool behind = false;     // this is not the first task
  int32_t drawn = 0;
  int qc0 = 0, qc1 = 0;
  uint32_t mn0 = 0xFFFFFFFFu, mn1 = 0xFFFFFFFFu, mx0 = 0u, mx1 = 0u;   // head pass: key range of this wavefront's points
  float sum[NB][LM_G];
  for (;;) {
    asm volatile("" : "+v"(tid), "+v"(lane));   // (addresses formed anew for every part: kept across parts they spill)
    __syncthreads();   // the task's residuals and radii are there, and nobody reads the part before any more
    if (part == 0 && seg == 0 && behind) {   // the task after this one is known by now
      t_next = __builtin_amdgcn_readfirstlane(*t_after);
      if (t_next < ntasks) npv = fetch_pairs(t_next);
    }
    const bool last_part = part == P - 1, last_seg = seg + NB * NW >= tk.nb, more = t_next < ntasks;
    const bool new_task = last_part && last_seg;
    // ---- the part's rows, interleaved: (query 0, query 1) of entry 0, of entry 1, ... ----
#pragma unroll
    for (int it = 0; it < ROWS; ++it) {
      const int m = part * LPP_PART + it * NW + wave;
      if ((!RT && TAIL == 0) || m < M) {
        float res0[DSUB], res1[DSUB];
#pragma unroll
        for (int j = 0; j < DSUB; ++j) {
          res0[j] = sres[m * DSUB + j];
          res1[j] = sres[dpad + m * DSUB + j];
        }
        const float4 v0 = lut_entry4<DSUB, 0>(res0, row[it], sr2[m]);
        const float4 v1 = lut_entry4<DSUB, 0>(res1, row[it], sr2[IVFPQ_MAX_M + m]);
        LDS floatx4 *dst = (LDS floatx4 *)(smem3 + (it * NW + wave) * 2048 + lane * 32);
        dst[0] = floatx4{v0.x, v1.x, v0.y, v1.y};
        dst[1] = floatx4{v0.z, v1.z, v0.w, v1.w};
      }
    }
    if constexpr (!HEAD)
      if (part == 0) drain_pending();   // the queues are free again before this task fills them
    __syncthreads();   // the part's rows are complete
    // ---- on their way while the part is scanned: the next part's rows, what the next task wants; and a block's next
    // codes from where its look-ups are made, in the registers of the ones looked up ----
    LmTask ntk = tk;
    if (part == 0 && last_seg && more) {
      nmv = fetch_meta(npv);
      if (tid == 0) drawn = atomicAdd(ticket, 1);
    }
    if (new_task && more) fetch_task(npv, nmv, ntk);
    load_rows(last_part ? 0 : part + 1);
    const bool to_next = new_task && more;   // (behind the last task: codes that are not looked at)
    const uint8_t *next_base = to_next ? ntk.base : tk.base;
    const int next_nb = to_next ? ntk.nb : tk.nb, next_seg = new_task ? 0 : (last_part ? seg + NB * NW : seg), next_part = last_part ? 0 : part + 1;
    // ---- look-ups ----
    if (part == 0) {
#pragma unroll
      for (int i = 0; i < NB; ++i) sum[i][0] = sum[i][1] = 0.0f;
    }
    auto look_up = [&](auto count) __attribute__((always_inline)) {   // so many subspaces of the part
      constexpr int N = decltype(count)::value, G = N < 8 ? N : 8;
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        if (seg + wave + i * NW < tk.nb) {
#pragma unroll
          for (int h = 0; h < N; h += G) {
            floatx2 v[G];
#pragma unroll
            for (int j = 0; j < G; ++j) {
              const uint32_t off = code_offset8(code[i][(h + j) >> 2], j & 3);   // the table starts at LDS address 0
              v[j] = *(const LDS floatx2 *)(uintptr_t)(uint32_t)((h + j) * 2048 + off);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < G; ++j) {
              sum[i][0] += v[j][0];
              sum[i][1] += v[j][1];
            }
            asm volatile("" : "+v"(sum[i][0]), "+v"(sum[i][1]));   // (the additions stay here: moved to where the block's loop is left, they keep all look-ups in registers)
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        load_codes(next_base, next_nb, next_seg, next_part, i);
      }
    };
    if constexpr (RT) {
      const int left = M - part * LPP_PART;
      if (left >= LPP_PART) {
        look_up(std::integral_constant<int, LPP_PART>{});
      } else {   // four at a time; what is behind the last subspace adds nothing (no sum is below zero: + 0 leaves it)
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          uintx4 w = code[i];
          load_codes(next_base, next_nb, next_seg, next_part, i);
          if (seg + wave + i * NW >= tk.nb) continue;
#pragma unroll 1
          for (int h = 0; h < left; h += 4) {
            floatx2 v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
              v[j] = *(const LDS floatx2 *)(uintptr_t)(uint32_t)((h + j) * 2048 + code_offset8(w[0], j));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              sum[i][0] += h + j < left ? v[j][0] : 0.0f;
              sum[i][1] += h + j < left ? v[j][1] : 0.0f;
            }
            w = uintx4{w[1], w[2], w[3], 0u};
          }
        }
      }
    } else if (TAIL == 0 || !last_part) {
      look_up(std::integral_constant<int, LPP_PART>{});
    } else {
      look_up(std::integral_constant<int, TAIL == 0 ? LPP_PART : TAIL>{});
    }
    // ---- these points are summed ----
    if (last_part) {
      if constexpr (HEAD) {
        LmWindow win = lm_window(sr2, M, lane);
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          if (seg + wave + i * NW >= tk.nb) break;
          const int at = (seg + wave + i * NW) * 64 + lane;
          if (at < tk.len) {
            const uint32_t k0 = __float_as_uint(sum[i][0]), k1 = __float_as_uint(sum[i][1]);
            sdist[at] = k0;
            sdist[a.head_max + at] = k1;
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
        }
        if (last_seg) {
          lm_select_head<4>(a, tk, win, mn0, mn1, mx0, mx1, smem3, ssel, hist, sdist, tid, lane, wave);
          mn0 = mn1 = 0xFFFFFFFFu;
          mx0 = mx1 = 0u;
        }
      } else {
        const uint32_t tau0 = (uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(tk.tauv), 0);
        const uint32_t tau1 = (uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(tk.tauv), 1);
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          if (seg + wave + i * NW >= tk.nb) break;
          const int at = (seg + wave + i * NW) * 64 + lane;
          const bool valid = at < tk.len;
          lm_offer(a, tk.q0, sum[i][0], valid, tau0, (uint32_t)(tk.row0 + at), qd0, qrow0, qc0, lane);
          if (tk.has1) lm_offer(a, tk.q1, sum[i][1], valid, tau1, (uint32_t)(tk.row0 + at), qd1, qrow1, qc1, lane);
        }
        if (last_seg) {
          // one atomic instruction reserves the space of both queues, which are written once a part of the next table is built
          pend_slot = 0;
          const int n_mine = lane == 0 ? qc0 : (lane == 1 ? qc1 : 0);
          if (n_mine > 0) pend_slot = atomicAdd(&a.gcnt[lane == 0 ? tk.q0 : tk.q1], (uint32_t)n_mine);
          pend_q0 = tk.q0;
          pend_q1 = tk.q1;
          pend_c0 = qc0;
          pend_c1 = qc1;
          qc0 = qc1 = 0;
        }
      }
    }
    if (new_task && !more) break;
    // ---- what is up next ----
    if (new_task) {
      put_task();
      if (tid == 0) *t_after = task_of(2 * run + drawn);
      behind = true;
      tk = ntk;
      seg = 0;
    } else if (last_part) {
      seg += NB * NW;
    }
    part = last_part ? 0 : part + 1;
  }
  if constexpr (!HEAD) drain_pending();
}
