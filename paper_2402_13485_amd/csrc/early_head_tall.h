// Early-head scoring, many score rows (see head_plan): tiles of 32*MI rows x 256 vocabulary entries.
// Included by early_prune.hip inside namespace propd, after the helpers it uses.
//
// The scoring GEMM has few rows (the nodes that have children: 704 at B = 16, T = 128) against a
// wide vocabulary.  A round of workgroups costs about 10 + 4 * MI (head_plan), so the shape
// is the one whose row tiles hold the rows with little padding in the fewest rounds:
// 704 rows are two tiles of 352 and 250 workgroups, ONE round of the 256 compute units; 832 rows
// are four tiles of 224 in two rounds (three of 352 would need as many rounds of larger tiles).
// With 256-row tiles of the 32x32x16 instruction and one shape for rows like 704 only, the
// pruning calls at 264, 352, 528, 832 and 1056 rows x 4096 took 181, 181, 212, 293 and 395 us; now
// 142, 155, 186, 265 and 329.
//   - 8 waves as 2 (rows) x 4 (columns), a wave owns 16*MI x 64 as MI x 4 tiles of the
//     16x16x32 bf16 MFMA: up to 176 accumulator registers (MI = 11) of the 256 a wave may have at
//     two waves per SIMD, which leaves room for operands only if they are streamed;
//   - K advances 32 per step through a ring of four LDS stages (64-byte rows, 38 KB for MI = 11),
//     filled by direct global->LDS loads three steps ahead.  The 16-byte chunks of a
//     row are XOR-swizzled with key(row) = (row >> 1) & 3: a fragment read of this MFMA has
//     lane -> (row lane % 16, chunk lane / 16), and with the key (row >> 2) & 3
//     every such read took twice its time in bank conflicts (measured: 64 against 38 ticks);
//   - per step a wave reads its B fragments and then streams the A fragments
//     through a four-deep register ring: the read of fragment i + 3 is issued behind the
//     MFMAs of fragment i, waits are placed by hand (LDS reads return in order).  Meeting in the
//     middle of a step and reading the next step's first fragments behind the last products of
//     this one, so that no wave waits after a barrier, changed nothing at 224 x 256 and cost 3 % at
//     352 x 256: loads and products compete, not reads (704 x 5120: 279 us whole, 211 without loads,
//     210 without products, 270 without fragment reads);
//   - epilogues: rank counts or log-sum-exp partials on this accumulator layout: a
//     row of the tile lives in the 16 lanes of a quarter wave (column = lane % 16 + 16 j), a
//     lane holds rows 16 i + 4 (lane / 16) + r.
#pragma once

constexpr int kTallStages = 4;
constexpr int kTallEpiChildren = 12;  // children of a row per epilogue pass

constexpr int kTallNJ = 4;  // matrix tiles of a wave side by side in the vocabulary

// What depends on the wave tile of MI x kTallNJ matrix tiles.
template <int MI>
struct Tall {
  static constexpr int kWaveRows = 16 * MI, kWaveCols = 16 * kTallNJ;
  static constexpr int kBM = 2 * kWaveRows, kBN = 4 * kWaveCols;
  static constexpr int kRows = kBM + kBN;                       // LDS rows of a stage
  static constexpr int kStageBytes = kRows * kGemmRowBytes;     // 38912 for MI = 11
  static constexpr int kGroups = kRows / 16, kAGroups = kBM / 16;  // 16-row groups, one load instruction each
  static constexpr int kLoads = (kGroups + 7) / 8;              // of a wave per K step, at most
  static constexpr int kIssueAt = MI / 2 - 1;  // the loads of a later step are issued behind this fragment's products
  static_assert(kTallStages * kStageBytes <= kHeadLdsBytes, "ring of stages");
};

template <int N>
__device__ __forceinline__ void tall_wait_lds(u32x4 &a) {
  asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(a) : "n"(N));
}
template <int N>
__device__ __forceinline__ void tall_wait_lds2(u32x4 &a, u32x4 &b) {
  asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(a), "+v"(b) : "n"(N));
}

template <int MI>
using TallAcc = f32x4[MI][kTallNJ];

// LDS accesses with the row's offset as an immediate of the instruction: one address register
// serves all rows of a lane.  (Left to itself the compiler materialises an address per row,
// keeps all of them across the passes and spills the accumulators for it.)
template <int OFFSET>
__device__ __forceinline__ uint32_t tall_lds_read4(uint32_t addr) {
  uint32_t r;
  asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFFSET));
  return r;
}
template <int OFFSET>
__device__ __forceinline__ void tall_lds_write4(uint32_t addr, uint32_t v) {
  asm volatile("ds_write_b32 %0, %1 offset:%2" ::"v"(addr), "v"(v), "n"(OFFSET) : "memory");
}
__device__ __forceinline__ void tall_wait_row(uint32_t &meta, u32x4 &thr) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(meta), "+v"(thr));
}
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Sum over the 16 lanes of each quarter wave, left in lanes 15, 31, 47 and 63.
__device__ __forceinline__ int quarter_wave_sum_to_last(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);  // row_shr:8
  return v;
}

// Top-k membership by counting (Section 4.1, "Pruning Criterion"): for every child c of the
// row's node, the scores of the row that beat the child's own score (a higher score, or the
// same score at a lower id) are counted; the count of this column tile goes to the child's
// slot of the tile in cnt_part, and the decision kernel adds the tiles up.
//
// The children of the tile's rows are staged in LDS (the ring is free by now), kTallEpiChildren
// per row and pass.  "Beats" is turned into one comparison per score: for the columns of a
// wave that all lie above the child's token the threshold is the own score (z > own), for
// columns that all lie below it the next smaller float (z > pred(own), i.e. z >= own); only
// the one wave whose columns contain the token compares per lane, on a side path marked by
// a NaN threshold, which the main comparison counts as nothing.  A lane counts its own columns
// in a byte per child, and one cross-lane sum per row and four children (DPP) leaves the row's
// counts in the last lane of each quarter wave.
template <int MI>
__device__ __forceinline__ void tall_epilogue_count(TallAcc<MI> &acc, int m0, int v0, int n_tile, int vocab,
                                                    int tid_in, int my_pos, int my_cc,
                                                    const HeadTables &tb, unsigned char *smem) {
  using G = Tall<MI>;
  constexpr int NJ = kTallNJ;
  constexpr int BM = G::kBM, WN = G::kWaveCols, E = kTallEpiChildren, NW = 4;
  static_assert(E % 4 == 0 && WN < 256, "four byte-sized counts per word");
  // everything below is derived from this copy of the thread id, which the compiler cannot see
  // through: otherwise it computes the dozens of LDS addresses of this epilogue before the K loop
  int tid = tid_in;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, c16 = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 2, wn = wave & 3;
  int *s_max = reinterpret_cast<int *>(smem);
  int *s_cc = s_max + 64;                                // [BM] children in this pass | flags << 8
  int *s_pos = s_cc + BM;                                // [BM]
  float *s_thr = reinterpret_cast<float *>(s_pos + BM);  // [NW][BM][E]
  float *s_own = s_thr + NW * BM * E;                    // [BM][E]
  int *s_tok = reinterpret_cast<int *>(s_own + BM * E);  // [BM][E]
  int *s_node = s_tok + BM * E;                          // [BM][E]
  int *s_count = s_node + BM * E;                        // [NW][BM][E/4]
  static_assert((64 + 2 * BM + (NW + 3) * BM * E + NW * BM * (E / 4)) * 4 <= kHeadLdsBytes, "epilogue tables");
  if (v0 + G::kBN > vocab) {  // columns past the vocabulary can beat nothing
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const bool out = v0 + wn * WN + 16 * j + c16 >= vocab;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] = out ? -INFINITY : acc[i][j][r];
    }
  }
  __syncthreads();  // every wave is done with the ring
  if (tid == 0) *s_max = 0;
  __syncthreads();
  {
    const int wave_max = wave_reduce_max(tid < BM ? my_cc : 0);
    if (lane == 0 && wave_max > 0) atomicMax(s_max, wave_max);
  }
  __syncthreads();
  const int max_cc = *s_max;
  const int row0 = wm * G::kWaveRows + 4 * q;  // this lane's rows: row0 + 16 i + r
  for (int e0 = 0; e0 < max_cc; e0 += E) {
    if (tid < BM) {
      int n = my_cc - e0;
      s_cc[tid] = n < 0 ? 0 : (n > E ? E : n);
      s_pos[tid] = my_pos + e0;
    }
    __syncthreads();
    {
      // The slots of a thread in two goes, all reads of one in flight together: a go is two dependent
      // reads long whatever its size, and the operand registers of the K loop are free by now.
      constexpr int kSlots = (BM * E + kGemmThreads - 1) / kGemmThreads, kChunk = (kSlots + 1) / 2;
#pragma unroll 1
      for (int j0 = 0; j0 < kSlots; j0 += kChunk) {
        int c[kChunk], t[kChunk];
        float o[kChunk];
#pragma unroll
        for (int j = 0; j < kChunk; ++j) {
          const int slot = tid + kGemmThreads * (j0 + j), row = slot / E, e = slot - row * E;
          c[j] = (slot < BM * E && e < (s_cc[row] & 255)) ? tb.child_list[s_pos[row] + e] : -1;
        }
#pragma unroll
        for (int j = 0; j < kChunk; ++j) {
          t[j] = c[j] >= 0 ? tb.token[c[j]] : -1;
          o[j] = c[j] >= 0 ? tb.own[c[j]] : INFINITY;
        }
#pragma unroll
        for (int j = 0; j < kChunk; ++j) {
          const int slot = tid + kGemmThreads * (j0 + j), row = slot / E;
          if (slot < BM * E) {
            const bool ok = t[j] >= 0 && t[j] < vocab;
            s_own[slot] = ok ? o[j] : INFINITY;
            s_tok[slot] = ok ? t[j] : -1;
            s_node[slot] = c[j];
#pragma unroll
            for (int w4 = 0; w4 < NW; ++w4) {
              const int c0 = v0 + w4 * WN;
              float thr = INFINITY;
              if (ok) {
                const bool inside = t[j] >= c0 && t[j] < c0 + WN;
                thr = t[j] < c0 ? o[j] : (inside ? __uint_as_float(0x7fc00000u) : float_pred(o[j]));
                if (inside) atomicOr(&s_cc[row], 256 << w4);
              }
              s_thr[w4 * BM * E + slot] = thr;
            }
          }
        }
      }
    }
    __syncthreads();
    // this lane's rows in the order (i, r)
    typedef __attribute__((address_space(3))) void lds_void;
    const uint32_t cc_addr = (uint32_t)(uintptr_t)(lds_void *)(s_cc + row0);
    const uint32_t thr_addr = (uint32_t)(uintptr_t)(lds_void *)(s_thr + wn * BM * E + row0 * E);
    const uint32_t count_addr = (uint32_t)(uintptr_t)(lds_void *)(s_count + wn * BM * (E / 4) + row0 * (E / 4));
    static_for<MI * 4>([&](auto idx_c) {
      constexpr int idx = decltype(idx_c)::value;
      constexpr int i = idx >> 2, r = idx & 3, off = 16 * i + r;
      uint32_t meta = tall_lds_read4<off * 4>(cc_addr);
      u32x4 thr_u = gemm_lds_read16<off * E * 4>(thr_addr);
      tall_wait_row(meta, thr_u);
      f32x4 thr4 = __builtin_bit_cast(f32x4, thr_u);
      const int m0q = __builtin_amdgcn_readlane((int)meta, 0), m1q = __builtin_amdgcn_readlane((int)meta, 16);
      const int m2q = __builtin_amdgcn_readlane((int)meta, 32), m3q = __builtin_amdgcn_readlane((int)meta, 48);
      int n_all = m0q & 255;
      n_all = (m1q & 255) > n_all ? (m1q & 255) : n_all;
      n_all = (m2q & 255) > n_all ? (m2q & 255) : n_all;
      n_all = (m3q & 255) > n_all ? (m3q & 255) : n_all;
      const bool side_path = (((m0q | m1q | m2q | m3q) >> (8 + wn)) & 1) != 0;
      // This body stands in the code once per row of a lane, so it is kept short: unrolled over e4, with
      // the side path's reads per child, the epilogue of one shape was 300 KB of instructions, fetched
      // once per tile (the pruning call at 704 rows x 5120: 288 us then, 266 now).
#pragma unroll 1
      for (int e4 = 0; e4 < n_all; e4 += 4) {
        const int ent0 = (row0 + opaque(off)) * E + e4;
        if (e4 > 0) thr4 = *reinterpret_cast<const f32x4 *>(s_thr + wn * BM * E + ent0);
        int packed = 0;
#pragma unroll
        for (int j4 = 0; j4 < 4; ++j4) {
          int cnt = 0;
#pragma unroll
          for (int j = 0; j < NJ; ++j) cnt += acc[i][j][r] > thr4[j4] ? 1 : 0;
          packed += cnt << (8 * j4);
        }
        if (side_path) {
          const f32x4 own4 = *reinterpret_cast<const f32x4 *>(s_own + ent0);
          const i32x4 tok4 = *reinterpret_cast<const i32x4 *>(s_tok + ent0);
#pragma unroll
          for (int j4 = 0; j4 < 4; ++j4) {
            const bool mine = thr4[j4] != thr4[j4];
            if (__ballot(mine) == 0) continue;  // uniform; one child of four rows as a rule
            const float own = mine ? own4[j4] : INFINITY;
            int cnt = 0;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
              const int before_tok = tok4[j4] - (v0 + wn * WN + 16 * j + c16);  // > 0: the column lies below the token
              const float z = acc[i][j][r];
              cnt += ((z > own || (z == own && before_tok > 0 && mine)) && before_tok != 0) ? 1 : 0;
            }
            packed += cnt << (8 * j4);
          }
        }
        packed = quarter_wave_sum_to_last(packed);
        if (c16 == 15) {
          if (e4 == 0) tall_lds_write4<off * (E / 4) * 4>(count_addr, (uint32_t)packed);
          else s_count[wn * BM * (E / 4) + (row0 + opaque(off)) * (E / 4) + (e4 >> 2)] = packed;
        }
      }
    });
    __syncthreads();
    for (int slot = tid; slot < BM * E; slot += kGemmThreads) {
      const int c = s_node[slot];
      if (c >= 0) {
        const int word = slot >> 2, sh = 8 * (slot & 3);
        int cnt = 0;
#pragma unroll
        for (int w4 = 0; w4 < NW; ++w4) cnt += (s_count[w4 * BM * (E / 4) + word] >> sh) & 255;
        tb.cnt_part[(size_t)n_tile * tb.cnt_stride + c] = cnt;
      }
    }
    __syncthreads();  // the next pass, or the next tile's loads, reuse this memory
  }
}

// (max, sum of exponentials) per row: every wave its columns, the four wave columns merged through
// LDS, one pair per row and tile.
template <int MI>
__device__ __forceinline__ void tall_epilogue_lse(const TallAcc<MI> &acc, int m0, int v0, int m_total, int vocab,
                                                  int n_tile, int tid, const HeadTables &tb, unsigned char *smem) {
  using G = Tall<MI>;
  constexpr int NJ = kTallNJ;
  const int lane = tid & 63, c16 = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 2, wn = wave & 3;
  float *s_part = reinterpret_cast<float *>(smem);  // [BM][4][2]
  __syncthreads();                                  // every wave is done with the ring
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float mx = -INFINITY;
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        if (v0 + wn * G::kWaveCols + 16 * j + c16 < vocab) mx = fmaxf(mx, acc[i][j][r]);
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, kWave));
      float sum = 0.f;
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        if (v0 + wn * G::kWaveCols + 16 * j + c16 < vocab && mx != -INFINITY) sum += expf(acc[i][j][r] - mx);
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) sum += __shfl_xor(sum, o, kWave);
      if (c16 == 0) {
        float *dst = s_part + ((wm * G::kWaveRows + 16 * i + 4 * q + r) * 4 + wn) * 2;
        dst[0] = mx;
        dst[1] = sum;
      }
    }
  __syncthreads();
  if (tid < G::kBM && m0 + tid < m_total) {
    float mx = s_part[8 * tid], sum = s_part[8 * tid + 1];
#pragma unroll
    for (int w = 1; w < 4; ++w) lse_merge(mx, sum, s_part[8 * tid + 2 * w], s_part[8 * tid + 2 * w + 1]);
    float *dst = tb.lse_part + ((size_t)(m0 + tid) * tb.parts + n_tile) * 2;
    dst[0] = mx;
    dst[1] = sum;
  }
}

template <int MI, int KIND>
__device__ __forceinline__ void early_head_tall_tile(
    int hidden, int vocab, int m_total, int m0, int v0, int n_tile,
    const uint16_t *__restrict__ hidden_states, const uint16_t *__restrict__ head_weight,
    const HeadTables &tb, unsigned char *smem) {
  using G = Tall<MI>;
  constexpr int NJ = kTallNJ;
  typedef __attribute__((address_space(3))) void lds_void;
  typedef const __attribute__((address_space(1))) void global_void;
  const uint32_t smem_base = (uint32_t)(uintptr_t)(lds_void *)smem;
  int tid = threadIdx.x;  // opaque: see early_head_small_tile
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  int my_pos = 0, my_cc = 0;
  if (KIND == 0 && tid < G::kBM && m0 + tid < m_total) {
    my_pos = tb.row_info[2 * (m0 + tid)];
    my_cc = tb.row_info[2 * (m0 + tid) + 1];
  }

  // ---- loader: group gi = wave + 8 j (16 rows, 1 KB) for j = 0 .. n_groups - 1
  const int ld_row = lane >> 2;
  const int ld_chunk = ((lane & 3) ^ ((lane >> 3) & 3)) << 4;  // byte offset in the global row: chunk ^ key(row)
  const bool all_groups = wave + 8 * (G::kLoads - 1) < G::kGroups;  // kLoads groups, else one fewer
  const unsigned char *src[G::kLoads];
#pragma unroll
  for (int j = 0; j < G::kLoads; ++j) {
    const int gi = wave + 8 * j;
    if (gi < G::kAGroups) {
      int m = m0 + 16 * gi + ld_row;
      m = m < m_total ? m : m_total - 1;
      src[j] = reinterpret_cast<const unsigned char *>(hidden_states + (size_t)tb.row_src[m] * hidden) + ld_chunk;
    } else {
      int v = v0 + 16 * (gi - G::kAGroups) + ld_row;
      v = v < vocab ? v : vocab - 1;
      src[j] = reinterpret_cast<const unsigned char *>(head_weight + (size_t)v * hidden) + ld_chunk;
    }
  }
  int k_off = 0;  // bytes into the rows of the next step to issue
  auto issue = [&](int slot) {
    unsigned char *dst = smem + slot * G::kStageBytes + wave * 1024;
#pragma unroll
    for (int j = 0; j < G::kLoads; ++j)
      if (j + 1 < G::kLoads || all_groups)
        __builtin_amdgcn_global_load_lds((global_void *)(src[j] + k_off), (lds_void *)(dst + j * 8192), 16, 0, 0);
    k_off += kGemmRowBytes;
  };
  // until at most STEPS steps' loads of this wave are outstanding
  auto wait_steps = [&](auto steps) {
    constexpr int N = decltype(steps)::value;
    if (all_groups) gemm_wait_vmem<N * G::kLoads>();
    else gemm_wait_vmem<N * (G::kLoads - 1)>();
  };
  using none = std::integral_constant<int, 0>;
  using one_step = std::integral_constant<int, 1>;
  using two_steps = std::integral_constant<int, 2>;

  // ---- per-lane LDS read addresses: row lane % 16 of a 16-row block, chunk lane / 16 (swizzled)
  const int c16 = lane & 15, kq = lane >> 4;
  const uint32_t frag_off = c16 * kGemmRowBytes + ((kq ^ ((c16 >> 1) & 3)) << 4);
  const uint32_t a_rd = smem_base + wm * G::kWaveRows * kGemmRowBytes + frag_off;
  const uint32_t b_rd = smem_base + (G::kBM + wn * G::kWaveCols) * kGemmRowBytes + frag_off;

  TallAcc<MI> acc;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int n_steps = hidden / kBK;
  const int n_pro = n_steps < kTallStages - 1 ? n_steps : kTallStages - 1;
  int slot_ld = 0;
  for (int i = 0; i < n_pro; ++i) {
    issue(slot_ld);
    slot_ld = slot_ld + 1 == kTallStages ? 0 : slot_ld + 1;
  }
  if (n_pro == 3) wait_steps(two_steps{});
  else if (n_pro == 2) wait_steps(one_step{});
  else wait_steps(none{});
  __builtin_amdgcn_s_barrier();
  uint32_t so = 0;  // byte offset of the stage being multiplied
  for (int step = 0; step < n_steps; ++step) {
    const uint32_t pa = a_rd + so, pb = b_rd + so;
    u32x4 bf[NJ], af[4];
    // the first product needs only A0 and B0: they are read first
    af[0] = gemm_lds_read16<0>(pa);
    static_for<NJ>([&](auto j) { bf[j] = gemm_lds_read16<j * 1024>(pb); });
    af[1] = gemm_lds_read16<1024>(pa);
    af[2] = gemm_lds_read16<2048>(pa);
    static_for<MI>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      constexpr int allowed = MI - 1 - i < 2 ? MI - 1 - i : 2;  // younger A reads in flight
      if constexpr (i == 0) {
        tall_wait_lds2<NJ + 1>(af[0], bf[0]);
        acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, af[0]),
                                                            __builtin_bit_cast(bf16x8, bf[0]), acc[0][0], 0, 0, 0);
        static_for<NJ>([&](auto j) { tall_wait_lds2<2>(af[0], bf[j]); });
      } else {
        tall_wait_lds<allowed>(af[i & 3]);
      }
#pragma unroll
      for (int j = (i == 0 ? 1 : 0); j < NJ; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, af[i & 3]),
                                                            __builtin_bit_cast(bf16x8, bf[j]), acc[i][j], 0, 0, 0);
      if constexpr (i + 3 < MI) af[(i + 3) & 3] = gemm_lds_read16<(i + 3) * 1024>(pa);
      if (i == G::kIssueAt && step + kTallStages - 1 < n_steps) {
        issue(slot_ld);  // step + 3, into the slot of step - 1
        slot_ld = slot_ld + 1 == kTallStages ? 0 : slot_ld + 1;
      }
    });
    if (step + 1 < n_steps) {
      // this wave has read everything of this step's slot; the next step has landed once at
      // most the steps after it that were issued (up to two) are outstanding
      if (step + 3 < n_steps) wait_steps(two_steps{});
      else if (step + 2 < n_steps) wait_steps(one_step{});
      else wait_steps(none{});
      __builtin_amdgcn_s_barrier();  // it is visible; every wave is done with this step's slot
      so = so + G::kStageBytes == kTallStages * G::kStageBytes ? 0 : so + G::kStageBytes;
    }
  }
  mfma_settle();
  if (KIND == 0) tall_epilogue_count<MI>(acc, m0, v0, n_tile, vocab, tid, my_pos, my_cc, tb, smem);
  else tall_epilogue_lse<MI>(acc, m0, v0, m_total, vocab, n_tile, tid, tb, smem);
}
