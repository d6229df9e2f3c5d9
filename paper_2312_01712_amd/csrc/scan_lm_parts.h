// Main pass of the list-major scan under distances, two-dimensional subspaces: byte tables that hold gains, a table in parts
// of 16 subspaces (included by scan_lm.hip, which says what a group of eight queries is, and where candidates go).
//
// lm_byte_kernel holds a whole table in LDS: one workgroup per CU, whose 16 wavefronts build it together, wait, gather from it
// together and wait again (9.2 and 9.6 of 20 thousand clocks a task with 48 subspaces).  What that costs is instructions: a
// wavefront issues one in 8 clocks at best, and four to a SIMD do not hide that.  Here
//  - a value is made by the matrix units from split factors (two products of depth 32 for four queries and 64 entries,
//    beside which the vector ALU is free) and becomes a byte by one conversion, which rounds, cuts off at 0 and packs; in
//    lm_byte_kernel by three products of depth 1, during which nothing else issues, and 5/4 instructions and what cuts off;
//  - look-ups are added up by the matrix units: one addition and half a product each instead of three and a half additions;
//  - a table goes by in parts, so that a workgroup takes 32 KiB for it whatever the number of subspaces, and two of them,
//    8 wavefronts each, share a CU: the start and end of one's task hide behind the other's work.
// The points of a list are scanned LMP_SEG at a time, their sums in registers; a longer list costs another table for each.
// A part's codes are one 16-byte chunk of the lists' layout.
// 1M x 96, 64 probes, 10 000 queries, both passes: 2.59 ms with lm_byte_kernel, 2.21 so; 1M x 128, 2000 queries of 32 probes,
// the stages of k = 1000: 270 and 254 us.  100 subspaces, for which whole tables do not fit a CU: 2000 queries of 64 probes,
// without structure, a search with fp32 tables of two queries (lm_pair_kernel) 4768 us, so 3810 (k = 10: 4623, 2768).

constexpr int LMP_NW = 8;        // wavefronts of a workgroup
constexpr int LMP_WG = 2;        // workgroups per CU: 4 wavefronts per SIMD, 128 vector registers each
constexpr int LMP_PART = 16;     // subspaces of a part
constexpr int LMP_NB = 4;        // blocks of 64 points whose sums a wavefront holds
constexpr int LMP_SEG = LMP_NW * LMP_NB * 64;   // points of a list that are scanned with one table
constexpr int LMP_BUF = LMP_PART * 2048;
constexpr int LMP_QUEUE = 4096;  // candidates a task holds; more go to the queries' slots one by one
constexpr int LMP_SMALL = 56;    // words: two sets of a task's starting sums, queries and scales, then the queue's counter and a task
constexpr size_t lmp_lds(int mt, int dsub) {
  return LMP_BUF + (size_t)LMB_G * mt * (4 * dsub + 4) + (size_t)mt * 4 + LMP_QUEUE * 4 + LMP_SMALL * 4;
}

// What is wanted of a task, kept between its request and its use: lane m holds subspaces m and, of H = 2, 64 + m.
template <int DSUB, int H>
struct LmpFetch {
  float q[H][DSUB], c[H][DSUB], r2[H], tau;
  uint32_t n;
  int32_t qid;
};

typedef int intx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Errors of a table value, in units of a byte: LMP_REL of s (|r| + |e|)^2 for the split factors (either is within 2^-17 of
// its value, and so is |e|^2: half of it; what the products' sums lose is 2^-20 of the largest of them), LMP_RAISE for the constant.
// A value is raised by as much, so that it is no less than what an entry gains, and may be above that by twice as much.
constexpr float LMP_RAISE = 1.0f / 1024.0f, LMP_REL = 1.0f / 32768.0f;

// A value as a pair of bf16: the rest in the low half.
__device__ __forceinline__ uint32_t split_bf16(float v) {
  const __bf16 hi = (__bf16)v, lo = (__bf16)(v - (float)hi);
  return ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16) | __builtin_bit_cast(uint16_t, lo);
}

// Which of its row's entries (of half a row) lane `lane` holds in step x: the quarters of a wavefront are a step apart, so
// that the four rows they write to are met at four places of the LDS' banks.
__device__ __forceinline__ int lmp_entry(int x, int lane) { return (((x + (lane >> 4)) & 7) << 4) | (lane & 15); }

// lmb_spill in a loop, part of the kernel: around a call the sums and the next part's codes would have to be saved.
__device__ __forceinline__ void lmp_spill(const LmArgs &a, const LDS int32_t *sq, bool over, uint32_t g, uint32_t x, uint32_t row, int lane) {
#pragma unroll 1
  for (uint32_t y = 0; y < (uint32_t)LMB_G; ++y) {
    const unsigned long long b = __ballot(over && g == y);
    if (b == 0ull) continue;
    const int64_t q = sq[y];
    uint32_t slot = 0;
    if (lane == 0) slot = atomicAdd(&a.gcnt[q], (uint32_t)__popcll(b));
    slot = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot) + (uint32_t)__popcll(b & ((1ull << lane) - 1ull));
    if (over && g == y && slot < (uint32_t)a.cap) a.cand[q * a.cap + slot] = make_uint2(x, row);
  }
}

template <int MT, int DSUB>
__global__ __launch_bounds__(LMP_NW * 64) __attribute__((amdgpu_waves_per_eu(LMP_WG * LMP_NW / 4))) void lm_part_kernel(LmArgs a, RadiiSq r2) {
  constexpr int NW = LMP_NW, NB = LMP_NB;
  constexpr int P = (MT + LMP_PART - 1) / LMP_PART, TAIL = MT % LMP_PART;   // parts; subspaces of the last one where it is short
  constexpr int H = (MT + 63) / 64;   // subspaces of a lane
  static_assert((TAIL == 0 || TAIL == 4) && MT <= 128 && P >= 3 && DSUB == 2, "16-byte chunks and one of 4 bytes; the queue is read, cleared and filled again in three parts");
  static_assert(MT * LMB_TOP < 1 << 16, "sums");
  static_assert(NW == LMB_G, "a wavefront per query of a group forms its parameters");
  extern __shared__ __align__(16) unsigned char smem[];
  LDS unsigned char *smem3 = (LDS unsigned char *)smem;
  // LDS carve: table [16][256][8 bytes] | records [MT][8][DSUB]: 2 s residual, split | constants [MT][8] | largest |entry|^2
  // of a subspace [MT] | queue | small words
  LDS uint32_t *srec = (LDS uint32_t *)(smem3 + LMP_BUF);
  LDS float *scon = (LDS float *)(srec + MT * LMB_G * DSUB);
  LDS float *semax = scon + MT * LMB_G;
  LDS uint32_t *queue = (LDS uint32_t *)(semax + MT);
  LDS uint32_t *small = queue + LMP_QUEUE;
  LDS int32_t *sT = (LDS int32_t *)small;          // [2][8] what a point's sum starts from: negative ends are candidates
  LDS int32_t *sq = (LDS int32_t *)(small + 16);   // [2][8] queries
  LDS uint32_t *ss = small + 32;                   // [2][8] -s, split (s: units of a byte per squared distance)
  LDS uint32_t *qn = small + 48;                   // candidates offered to the queue
  LDS int32_t *t_after = (LDS int32_t *)(small + 49);   // the task after the next

  int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ntasks = a.base[a.nlist] / LMB_G;
  const int nwg = gridDim.x, b = blockIdx.x;
  // Runs of tasks per XCD, as in lm_scan_kernel.  Behind their first two the workgroups of an XCD take them up one by one:
  // dealt out, the ones whose wavefronts a SIMD prefers end early and leave the others a CU of 8 wavefronts (an eighth of
  // the pass over 10 000 queries of the 1M x 96 configuration).
  const int xcds = (nwg & 7) == 0 ? 8 : 1, run = nwg / xcds, xcd = b % xcds;
  auto task_of = [&](int n) __attribute__((always_inline)) { return n / run * nwg + xcd * run + n % run; };
  const int t = task_of(b / xcds);
  int t_next = task_of(b / xcds + run);
  int32_t *ticket = a.cnt + ivfpq::lm_tickets(a.nlist, a.stage) + xcd * ivfpq::LM_TICKET_STEP;
  if (t >= ntasks) return;

  // What this wavefront needs of the codebook for its share of a part: of the four rows 4 (wave / 2) .. + 3 the entries of half
  // wave % 2, split into pairs of bf16 (made with the index), a quarter of the wavefront per row and 16 entries at a time.
  constexpr int STEPS = 8;
  uintx4 ent[STEPS];
  auto load_rows = [&](int part) __attribute__((always_inline)) {
    const int m0 = part * LMP_PART + (wave >> 1) * 4;
    const GLOBAL uint8_t *rows = uniform_ptr(a.cb_split + (int64_t)(TAIL == 0 || m0 < MT ? m0 : MT - 4) * (256 * 8));   // no such rows: the last ones
#pragma unroll
    for (int x = 0; x < STEPS; ++x)
      ent[x] = *(const GLOBAL uintx4 *)(rows + (uint32_t)((lane >> 4) * 4096 + (wave & 1) * 2048 + lmp_entry(x, lane) * 16));
  };
  // largest |entry|^2 of every subspace (infinite entries gain nothing on the clamp)
#pragma unroll 1
  for (int m = wave; m < MT; m += NW) {
    float emax = 0.0f;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const float2 e = *reinterpret_cast<const float2 *>(a.codebooks + ((int64_t)m * 256 + x * 64 + lane) * DSUB);
      const float n2 = fmaf(e.y, e.y, e.x * e.x);
      if (n2 < __builtin_inff()) emax = fmaxf(emax, n2 < ivfpq::SPLIT_FAR ? n2 : __builtin_inff());   // (finite, yet not what the split holds: no bound then)
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) emax = fmaxf(emax, __shfl_xor(emax, off));
    if (lane == 0) semax[m] = emax;
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
  // wavefront g brings the parameters of query g: a lane per subspace
  LmpFetch<DSUB, H> fx;
  auto fetch_params = [&](const int2 &pv) __attribute__((always_inline)) {
    const int c = __builtin_amdgcn_readlane(pv.y, 0);
    const int q0 = __builtin_amdgcn_readlane(pv.x, 0);   // a task's first query exists
    fx.qid = __builtin_amdgcn_readlane(pv.x, wave);
    const int64_t q = fx.qid >= 0 ? fx.qid : q0;
#pragma unroll
    for (int x = 0; x < H; ++x) {
      const int m = lane + 64 * x < MT ? lane + 64 * x : MT - 1;
      const float2 qv = *reinterpret_cast<const float2 *>(a.queries + q * a.D + 2 * m);
      const float2 cv = *reinterpret_cast<const float2 *>(a.centroids + (int64_t)c * a.D + 2 * m);
      fx.q[x][0] = qv.x; fx.q[x][1] = qv.y; fx.c[x][0] = cv.x; fx.c[x][1] = cv.y;
      fx.r2[x] = a.query_radii ? a.query_radii[q * MT + m] : r2.v[m];   // (squared where it is used)
    }
    fx.tau = a.tau[q * a.tau_stride];
    fx.n = a.gcnt[q];
  };
  // ... and writes them to the records and to set `par` of the small words.  LOST: every rounding of the fp32 sums of a point's
  // distance and of what is formed here, 2^-23 each, at most MT + 6.
  constexpr float LOST = MT <= 64 ? 1.0e-5f : 1.6e-5f;
  static_assert((MT + 6) * 1.1920929e-7f < LOST, "roundings");
  auto put_params = [&](int par) __attribute__((always_inline)) {
    bool on[H];
    float rm2[H], res[H][DSUB], rr[H], far[H];
    const float tau = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(fx.tau)));
    // A byte holds what an entry GAINS on the clamp: s (cap_m - |r - e|^2), cap_m being r_m^2 or, where that is smaller,
    // the unit's end: the largest r_m^2 (no table value exceeds it), or, where that is wider, four times the mean value of
    // a point within tau.  Rounded up, so that the sum of a point's bytes is no less than what it gains in all, and
    // cut off at 0 by the conversion itself: entries outside the radius (most of them), infinitely far ones and those
    // that are not a number lose nothing.  A point within tau gains at least s (sum of cap_m - tau).
    float farthest = 0.0f, widest = 0.0f;
#pragma unroll
    for (int x = 0; x < H; ++x) {
      on[x] = lane + 64 * x < MT;
      rm2[x] = fx.r2[x];
      if (a.query_radii) rm2[x] = fminf(rm2[x] * rm2[x], __builtin_inff());   // (a NaN cuts nothing off, like an infinite radius)
      rr[x] = 0.0f;
#pragma unroll
      for (int j = 0; j < DSUB; ++j) {
        res[x][j] = fx.q[x][j] - fx.c[x][j];
        rr[x] = fmaf(res[x][j], res[x][j], rr[x]);
      }
      far[x] = on[x] ? sqrtf(rr[x]) + sqrtf(semax[lane + 64 * x]) : 0.0f;
      far[x] *= far[x];
      farthest = fmaxf(farthest, far[x]);
      widest = fmaxf(widest, on[x] ? rm2[x] : 0.0f);
    }
    auto over_lanes = [&](auto fold) __attribute__((always_inline)) {
      fold([](float v) __attribute__((always_inline)) { return xor_f32<32>(v); });
      fold([](float v) __attribute__((always_inline)) { return xor_f32<16>(v); });
      fold([](float v) __attribute__((always_inline)) { return xor_f32<8>(v); });
      fold([](float v) __attribute__((always_inline)) { return xor_f32<4>(v); });
      fold([](float v) __attribute__((always_inline)) { return xor_f32<2>(v); });
      fold([](float v) __attribute__((always_inline)) { return xor_f32<1>(v); });
    };
    float rmax = a.rmax;
    over_lanes([&](auto other) __attribute__((always_inline)) { farthest = fmaxf(farthest, other(farthest)); });
    if (a.query_radii) {
      rmax = widest;
      over_lanes([&](auto other) __attribute__((always_inline)) { rmax = fmaxf(rmax, other(rmax)); });
    }
    const float cap = fmaxf(fminf(rmax, tau * (4.0f / (float)MT)), 1e-30f);
    // No byte is above LMB_TOP, which the sum of two as a signed byte needs and the conversion does not see to (it cuts off at
    // 255): a value is at most s (cap + 2 LMP_REL farthest) + 2 LMP_RAISE + 0.5 < LMB_TOP + 0.5.  (Room for the raise alone let
    // bytes of 70 and more through where cap is small, and points on their query were missed.)
    const float s = ((float)LMB_TOP - 0.6f) / fmaf(farthest, 2.0f * LMP_REL, cap);   // (infinite radii and no k-th distance: 0)
    float least = 0.0f;
#pragma unroll
    for (int x = 0; x < H; ++x) {
      const float most = fminf(rm2[x], cap) * s, err = fmaf(s * far[x], LMP_REL, LMP_RAISE);
      if (on[x]) {
        const int at = (lane + 64 * x) * LMB_G + wave;
#pragma unroll
        for (int j = 0; j < DSUB; ++j) srec[at * DSUB + j] = split_bf16(2.0f * s * res[x][j]);
        scon[at] = most - s * rr[x] + (0.5f + err);   // (rounded to nearest: half a unit up)
        least += most - LOST * (most + 1.0f);
      }
    }
    over_lanes([&](auto other) __attribute__((always_inline)) { least += other(least); });
    least -= tau * s * (1.0f + LOST);
    const int32_t start = least > 1.0f ? (int32_t)least - 1 : -1;   // NaN (0 x inf, or no k-th distance): every point
    if (lane == 0) {
      sT[par * 8 + wave] = fx.qid >= 0 && fx.n <= (uint32_t)a.cap ? start : 0x40000000;   // (a query out of slots is redone, and offers no more)
      sq[par * 8 + wave] = fx.qid;
      ss[par * 8 + wave] = split_bf16(-s);
    }
  };

  // ---- this wavefront's share of part `part` (set `par` of the small words) ----
  // A quarter of the wavefront (lanes 16 h .. 16 h + 15) holds 16 entries of its own row, split in eight
  // 16-bit values: the high parts and rests of both coordinates and of |entry|^2.  One product of depth 32 serves the four
  // rows: its 16 rows are four queries for each of them, and what does not belong together is multiplied by zero.  A
  // second one with the rests of the queries' factors, and the constant as its third operand, make the gains of four
  // queries for the lane's entry.
  // (Products of depth 1, exact in fp32, take 9 clocks of a SIMD for four values, and nothing else issues meanwhile:
  // v_mfma_f32_4x4x1 with an addition beside each takes the sum of both times and more, v_mfma_f32_16x16x32_bf16 takes 16
  // for as many with the vector ALU free.)
  auto build = [&](int part, int par) __attribute__((always_inline)) {
    if (TAIL != 0 && part == P - 1 && wave >= TAIL / 2) return;
    const bool five = sq[par * 8 + 4] >= 0;   // uniform
    const int h = lane >> 4, m = part * LMP_PART + (wave >> 1) * 4 + h;
    const bool mine = ((lane & 15) >> 2) == h;   // the lanes that hold the factors of their own quarter's rows
    bf16x8 fh[2], fl[2];
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      const uintx2 f = *(const LDS uintx2 *)(srec + (m * LMB_G + 4 * y + (lane & 3)) * DSUB);
      const uint32_t sc = ss[par * 8 + 4 * y + (lane & 3)];
      const uint32_t f0 = mine ? f[0] : 0u, f1 = mine ? f[1] : 0u, f2 = mine ? sc : 0u;
      constexpr uint32_t HI = 0x03020302u, LO = 0x01000100u;   // either half twice
      fh[y] = __builtin_bit_cast(bf16x8, uintx4{__builtin_amdgcn_perm(f0, f0, HI), __builtin_amdgcn_perm(f1, f1, HI), __builtin_amdgcn_perm(f2, f2, HI), 0u});
      fl[y] = __builtin_bit_cast(bf16x8, uintx4{__builtin_amdgcn_perm(f0, f0, LO), __builtin_amdgcn_perm(f1, f1, LO), __builtin_amdgcn_perm(f2, f2, LO), 0u});
    }
    floatx4 con[2];
#pragma unroll
    for (int y = 0; y < 2; ++y) con[y] = *(const LDS floatx4 *)(scon + m * LMB_G + 4 * y);
    LDS unsigned char *dst = smem3 + ((wave >> 1) * 4 + h) * 2048 + (wave & 1) * 1024;
    auto all_steps = [&](auto halves) __attribute__((always_inline)) {   // 2: a group of five queries and more
      constexpr int Y = decltype(halves)::value, X = 2;   // chains of products side by side: X Y
#pragma unroll
      for (int x = 0; x < STEPS; x += X) {
        floatx4 acc[X][Y];
#pragma unroll
        for (int z = 0; z < X; ++z)
#pragma unroll
          for (int y = 0; y < Y; ++y) acc[z][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fl[y], __builtin_bit_cast(bf16x8, ent[x + z]), con[y], 0, 0, 0);
#pragma unroll
        for (int z = 0; z < X; ++z)
#pragma unroll
          for (int y = 0; y < Y; ++y) acc[z][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fh[y], __builtin_bit_cast(bf16x8, ent[x + z]), acc[z][y], 0, 0, 0);
        uint32_t w[X][2] = {};
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
          for (int z = 0; z < X; ++z)
#pragma unroll
            for (int y = 0; y < Y; ++y) w[z][y] = __builtin_amdgcn_cvt_pk_u8_f32(acc[z][y][g], g, w[z][y]);
#pragma unroll
        for (int z = 0; z < X; ++z) *(LDS uintx2 *)(dst + lmp_entry(x + z, lane) * 8) = uintx2{w[z][0], w[z][1]};
      }
    };
    if (five) all_steps(std::integral_constant<int, 2>{});
    else all_steps(std::integral_constant<int, 1>{});
  };

  // the task being scanned: list, rows, blocks; the part of it; its first block of this segment
  int list = 0, len = 0, nb = 0, part = 0, seg = 0, par = 0;
  int64_t row0 = 0;
  const uint8_t *base = nullptr;
  // A task's candidates: their room is reserved when the list has been scanned, and they are written once a part of the
  // next table is built, so that nothing waits for the atomic's way.  The queue holds them until then.
  int q_list = 0, q_par = 0;   // list, rows and small words of the candidates in the queue
  int64_t q_row0 = 0;
  uint32_t p_slot = 0;         // lane g: the first slot reserved for query g
  bool p_has = false;          // (uniform)
  auto queued = [&](int e0, uint32_t &word) __attribute__((always_inline)) {
    const bool live = e0 + lane < (int)umin32(*qn, (uint32_t)LMP_QUEUE);
    word = live ? queue[e0 + lane] : 0u;
    return live;
  };
  auto reserve = [&](int e0) __attribute__((always_inline)) {
    uint32_t word, mine = 0;
    const bool live = queued(e0, word);
    // one atomic instruction reserves the room of all queries: lane g for query g
#pragma unroll
    for (int x = 0; x < LMB_G; ++x) {
      const unsigned long long bal = __ballot(live && (word & 7u) == (uint32_t)x);
      if (lane == x) mine = (uint32_t)__popcll(bal);
    }
    p_slot = 0;
    if (lane < LMB_G && mine > 0) p_slot = atomicAdd(&a.gcnt[sq[q_par * 8 + lane]], mine);
  };
  auto drain = [&](int e0) __attribute__((always_inline)) {
    uint32_t word, before = 0;
    const bool live = queued(e0, word);
    const uint32_t g = word & 7u, i = word >> 3;
#pragma unroll
    for (int x = 0; x < LMB_G; ++x) {
      const unsigned long long bal = __ballot(live && g == (uint32_t)x);
      if (g == (uint32_t)x) before = (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
    }
    const uint32_t slot = (uint32_t)__shfl((int)p_slot, (int)g) + before;
    if (live && slot < (uint32_t)a.cap)
      a.cand[(int64_t)sq[q_par * 8 + g] * a.cap + slot] = make_uint2((uint32_t)q_list, (uint32_t)(q_row0 + i));
  };
  auto take_queue = [&]() __attribute__((always_inline)) {
    const int n = __builtin_amdgcn_readfirstlane((int)umin32(*qn, (uint32_t)LMP_QUEUE));
    for (int e0 = (NW + wave) * 64; e0 < n; e0 += NW * 64) {   // (few tasks have more than 512)
      reserve(e0);
      drain(e0);
    }
    p_has = wave * 64 < n;
    if (p_has) reserve(wave * 64);
  };

  // the first task's first part
  int2 npv = make_int2(0, 0);   // pair entries of the next task
  int64_t nmv;                  // ... and its list's metadata
  {
    const int2 pv = fetch_pairs(t);
    nmv = fetch_meta(pv);
    fetch_params(pv);
    load_rows(0);
    if (t_next < ntasks) npv = fetch_pairs(t_next);
    list = __builtin_amdgcn_readlane(pv.y, 0);
    row0 = lane64(nmv, 0);
    len = (int)(lane64(nmv, 1) - row0);
    nb = (len + 63) >> 6;   // >= 1: only non-empty lists have tasks
    base = a.codes + lane64(nmv, 2) * ivfpq_block_bytes(MT);
    if (tid == 0) *qn = 0u;
    __syncthreads();   // semax
    put_params(0);
  }
  intx4 sums[NB][2];   // of the wavefront's blocks, less what their queries need: negative ends are candidates
  int32_t drawn = 0;

  for (;;) {
    asm volatile("" : "+v"(tid), "+v"(lane));   // (addresses formed anew: kept across intervals they spill)
    __syncthreads();   // the records are there, and nobody reads the part before any more
    const bool last_part = part == P - 1, last_seg = seg + NB * NW >= nb, more = t_next < ntasks;
    const bool new_task = last_part && last_seg;
    build(part, par);
    if (part == 0) take_queue();   // (its atomics behind the wait for the codebook's rows)
    // The part's codes.  (Lists are shorter than 2^20 points: an offset has 32 bits.)
    uintx4 code[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int blk = seg + wave + i * NW;
      const uint32_t in = (uint32_t)(blk < nb ? blk : nb - 1);   // no such block: the last one
      if (TAIL == 0 || !last_part)
        code[i] = *(const GLOBAL uintx4 *)((const GLOBAL uint8_t *)(uintptr_t)base + ((((uint32_t)(part * nb) + in) << 10) + (uint32_t)(lane * 16)));
      else
        code[i] = uintx4{*(const GLOBAL uint32_t *)((const GLOBAL uint8_t *)(uintptr_t)base + (((uint32_t)((P - 1) * nb) << 10) + (in << 8) + (uint32_t)(lane * 4))), 0u, 0u, 0u};
    }
    __syncthreads();   // the part's rows are complete
    if (new_task && more) {
      nmv = fetch_meta(npv);
      fetch_params(npv);
    }
    if (part == 0 && last_seg && more && tid == 0) drawn = atomicAdd(ticket, 1);
    if (part == 1 && tid == 0) {
      *qn = 0u;
      *t_after = task_of(2 * run + drawn);
    }
    // ---- scan ----
    const int end = seg + NB * NW < nb ? seg + NB * NW : nb;   // of this segment's blocks
    const bool five = sq[par * 8 + 4] >= 0;   // uniform
    if (part == 0) {
      const LDS intx4 *T = (const LDS intx4 *)(sT + par * 8);
      const intx4 t0 = T[0], t1 = T[1];
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        sums[i][0] = t0;
        sums[i][1] = t1;
      }
    }
    // The matrix that adds up bytes: row 4 h + g takes byte g (and 4 + g in the second form) of the lanes of quarter h, so
    // that lane l ends up with the sums of its own point, queries 0 .. 3 (4 .. 7).
    const int pick_byte = ((lane & 15) >> 2) == (lane >> 4) ? 0xFF << (8 * (lane & 3)) : 0;   // (-1: gains are taken off)
    const intx4 low_four = {pick_byte, 0, pick_byte, 0}, high_four = {0, pick_byte, 0, pick_byte};
    // Two bytes below 64 add up within a byte; the matrix units spread four look-ups' to the sums of eight queries.  (On
    // the vector ALU -- four bytes added up, spread to 16 bits and accumulated -- 10 clocks a look-up, 5 so.)
    auto look_up = [&](auto count) __attribute__((always_inline)) {   // so many subspaces of the part
      constexpr int N = decltype(count)::value, G = N < 8 ? N : 8;
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        if (seg + wave + i * NW >= end) break;
#pragma unroll
        for (int h = 0; h < N; h += G) {
          uintx2 v[G];
#pragma unroll
          for (int j = 0; j < G; ++j) {
            const uint32_t off = code_offset8(code[i][(h + j) >> 2], j & 3);   // the table starts at LDS address 0
            v[j] = *(const LDS uintx2 *)(uintptr_t)(uint32_t)((h + j) * 2048 + off);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int j = 0; j < G; j += 4) {
            const intx4 b = {(int)(v[j][0] + v[j + 1][0]), (int)(v[j][1] + v[j + 1][1]), (int)(v[j + 2][0] + v[j + 3][0]), (int)(v[j + 2][1] + v[j + 3][1])};
            sums[i][0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(low_four, b, sums[i][0], 0, 0, 0);
            if (five) sums[i][1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(high_four, b, sums[i][1], 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    if (TAIL == 0 || !last_part) look_up(std::integral_constant<int, LMP_PART>{});
    else look_up(std::integral_constant<int, TAIL == 0 ? LMP_PART : TAIL>{});
    // ---- the list's points are summed: those that may gain what their queries need are candidates ----
    if (last_part) {
      const int first = (seg + wave) * 64 + lane;
      auto any_of = [&](int z) __attribute__((always_inline)) {
        const intx4 &s0 = sums[z][0], &s1 = sums[z][1];
        const int any = ((s0[0] | s0[1]) | (s0[2] | s0[3])) | ((s1[0] | s1[1]) | (s1[2] | s1[3]));
        return any < 0 && first + z * NW * 64 < len;
      };
      auto mask_of = [&](int z) __attribute__((always_inline)) {
        uint32_t mask = 0u;
#pragma unroll
        for (int g = 0; g < LMB_G; ++g) mask |= ((uint32_t)sums[z][g >> 2][g & 3] >> 31) << g;
        return first + z * NW * 64 < len ? mask : 0u;
      };
      static_assert(NB * LMB_G <= 32, "a bit for every sum");
      uint32_t mask = 0u;   // bit 8 z + g: the lane's point of block z is a candidate of query g
#pragma unroll
      for (int z = 0; z < NB; ++z)
        if (__ballot(any_of(z)) != 0) mask |= mask_of(z) << (LMB_G * z);
#pragma unroll 1
      for (unsigned long long bal = __ballot(mask != 0u); bal != 0; bal = __ballot(mask != 0u)) {
        const bool take = mask != 0u;
        const uint32_t bit = (uint32_t)__ffs((int)mask) - 1u, g = bit & 7u;
        mask &= mask - 1u;
        const int i = first + (int)(bit >> 3) * NW * 64;
        uint32_t to = 0;
        if (lane == 0) to = __hip_atomic_fetch_add(qn, (uint32_t)__popcll(bal), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        to = (uint32_t)__builtin_amdgcn_readfirstlane((int)to) + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
        const bool over = take && to >= (uint32_t)LMP_QUEUE;   // no room in the queue
        if (take && !over) queue[to] = ((uint32_t)i << 3) | g;
        if (__ballot(over) != 0) lmp_spill(a, sq + par * 8, over, g, (uint32_t)list, (uint32_t)(row0 + i), lane);   // straight to the queries' slots
      }
      q_list = list;
      q_row0 = row0;
      q_par = par;
    }
    if (new_task && more) put_params(par ^ 1);
    if (p_has) drain(wave * 64);
    p_has = false;
    if (new_task && !more) break;
    load_rows(last_part ? 0 : part + 1);
    // ---- what is up next ----
    part = last_part ? 0 : part + 1;
    if (new_task) {
      list = __builtin_amdgcn_readlane(npv.y, 0);
      row0 = lane64(nmv, 0);
      len = (int)(lane64(nmv, 1) - row0);
      nb = (len + 63) >> 6;
      base = a.codes + lane64(nmv, 2) * ivfpq_block_bytes(MT);
      seg = 0;
      par ^= 1;
      t_next = __builtin_amdgcn_readfirstlane(*t_after);
      if (t_next < ntasks) npv = fetch_pairs(t_next);
    } else if (last_part) {
      seg += NB * NW;
    }
  }
  __syncthreads();
  take_queue();
  if (p_has) drain(wave * 64);
}
