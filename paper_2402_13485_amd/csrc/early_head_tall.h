// Early-head scoring, many score rows (see head_plan): tiles of 32*MI rows x 256 vocabulary entries.
// Included by early_prune.hip inside namespace propd, after the helpers it uses.
//
// The scoring GEMM has few rows (the nodes that have children: 704 at B = 16, T = 128) against a
// wide vocabulary.  A round of workgroups costs about 7 + 4 * MI (head_plan), so the shape
// is the one whose row tiles hold the rows with little padding in the fewest rounds:
// 704 rows are two tiles of 352 and 250 workgroups, ONE round of the 256 compute units; 832 rows
// are four tiles of 224 in two rounds (three of 352 would need as many rounds of larger tiles).
//   - 8 waves as 2 (rows) x 4 (columns), a wave owns 16*MI x 64 as MI x 4 tiles of the
//     16x16x32 bf16 MFMA: up to 176 accumulator registers (MI = 11) of the 256 a wave may have at
//     two waves per SIMD, which leaves room for operands only if they are streamed;
//   - K advances 64 per step, through a ring of LDS slots for each operand (128-byte rows), filled by
//     direct global->LDS loads.  Every load takes whole 128-byte lines: the load path charges per line
//     touched, and steps of 32 (half a line of a row per load, every line fetched twice) could not keep
//     up with the products.  What a load has left to land matters as much: B, which comes from
//     HBM, is requested two steps ahead; up to MI = 8 it has three slots for that, beyond it two,
//     and its slot is handed back in the middle of a step, when every wave has its fragments in
//     registers.  A, which comes from the L2, is requested one step ahead, two for MI = 5.
//     Pruning call, us, steps of 32 in four stages / of 64 in two / as it is: 704 rows x 5120 x 32000
//     250 / 235 / 235, 440 x 4096 159 / 155 / 146, 308 x 4096 139 / 142 / 122, 836 x 4096 276 / 266 / 258, 352 x 4096 x
//     128256 446 / 451 / 417, 132 x 4096 x 128256 305 / 327 / 300, 176 x 1600 x 50257 90 / 90 / 82.  With B in two slots
//     up to MI = 8 too: 176 x 4096 x 128256 344 instead of 321.
//     704 x 5120 multiplies at 1.2 PFLOP/s, as fast as a large product of the library here (1.06 for the
//     kernel with its epilogue); in two stages a
//     call took 221 us without loads, 240 without products, without fragment reads and as it was;
//   - the 16-byte chunks of a row are XOR-swizzled with key(row) = (row >> 1) & 7, so that the fragment
//     reads of this MFMA (lane -> row lane % 16, chunk lane / 16) are free of bank conflicts;
//   - per step a wave streams 2*MI fragments of A through a four-deep register ring: the read of
//     fragment g + 3 is issued behind the MFMAs of fragment g, waits are placed by hand (LDS reads return in
//     order).  Of the four B fragments of a step's second half two are read ahead into registers
//     of their own; there is no room for more;
//   - a row of an odd number of 32s ends in a step whose second half is zeros;
//   - epilogues: rank counts or log-sum-exp partials on this accumulator layout: a
//     row of the tile lives in the 16 lanes of a quarter wave (column = lane % 16 + 16 j), a
//     lane holds rows 16 i + 4 (lane / 16) + r.
#pragma once

constexpr int kTallBK = 64, kTallRowBytes = 2 * kTallBK;  // depth of a step; bytes of a row in it
constexpr int kTallEpiChildren = 12;  // children of a row per epilogue pass

constexpr int kTallNJ = 4;  // matrix tiles of a wave side by side in the vocabulary

// What depends on the wave tile of MI x kTallNJ matrix tiles.
template <int MI>
struct Tall {
  static constexpr int kWaveRows = 16 * MI, kWaveCols = 16 * kTallNJ;
  static constexpr int kBM = 2 * kWaveRows, kBN = 4 * kWaveCols;
  static constexpr int kABytes = kBM * kTallRowBytes, kBBytes = kBN * kTallRowBytes;  // of a step: 44 KB (MI = 11), 32 KB
  // Slots of the two rings.  With three a load has two steps to land; where B has only two, its slot
  // is handed back in the middle of a step, when its fragments are in registers.
  static constexpr int kASlots = 3 * (kABytes + kBBytes) <= kHeadLdsBytes ? 3 : 2;           // 3: MI = 5
  static constexpr int kBSlots = 2 * kABytes + 3 * kBBytes <= kHeadLdsBytes ? 3 : 2;         // 3: MI <= 8
  static_assert(kASlots * kABytes + kBSlots * kBBytes <= kHeadLdsBytes, "rings");
  static constexpr int kAGroups = kBM / 8;                      // 8-row groups, one load instruction each
  static constexpr int kALoads = (kAGroups + 7) / 8, kBLoads = kBN / 64;  // of a wave per step (A: at most)
  static constexpr bool kNarrow = MI > kTallWideMI;             // row addresses as 32-bit offsets
  // fragment of A behind whose products fragment j of B of a step's second half is read: two of them
  // early, into registers of their own, the others when their registers are free
  static constexpr int b_at(int j) { return j < 2 ? MI - 5 + j : MI - 1; }
  // such reads behind fragment g
  static constexpr int b_behind(int g) {
    int count = 0;
    for (int j = 0; j < kTallNJ; ++j) count += b_at(j) == g ? 1 : 0;
    return count;
  }
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
  // first position in child_list (24 bits) and children (at most 127) of the thread's row, in one
  // register; where these are short it waits for the epilogue in LDS, behind the rings
  int my_row = 0;
  constexpr bool kParked = KIND == 0 && G::kNarrow;
  static_assert(!kParked || G::kASlots * G::kABytes + G::kBSlots * G::kBBytes + 4 * kGemmThreads <= kHeadLdsBytes, "parked");
  int *parked = reinterpret_cast<int *>(smem + G::kASlots * G::kABytes + G::kBSlots * G::kBBytes);
  if (KIND == 0 && tid < G::kBM && m0 + tid < m_total)
    my_row = tb.row_info[2 * (m0 + tid)] | tb.row_info[2 * (m0 + tid) + 1] << 24;
  if constexpr (kParked) parked[tid] = my_row;

  // ---- loader: a load instruction fills 8 rows of 128 bytes (1 KB); wave w takes groups w + 8 j of
  //      both operands
  const int ld_row = 8 * wave + (lane >> 3);
  // byte offset in the global row: chunk ^ key(row); a wave's groups are all even or all odd
  const int ld_chunk = ((lane & 7) ^ ((4 * wave + (lane >> 4)) & 7)) << 4;
  const bool all_a = wave + 8 * (G::kALoads - 1) < G::kAGroups;  // kALoads groups of A, else one fewer
  // Where registers are short the rows are addressed by 32-bit offsets from the operand's first byte of
  // this tile (head_plan takes such shapes only where all score rows, and the 256 weight rows of a tile,
  // lie within 4 GiB), and those of B, at constant distances up to the tile's last row in the vocabulary,
  // from the first.
  using Src = std::conditional_t<G::kNarrow, uint32_t, const unsigned char *>;
  constexpr int kBOwn = G::kNarrow ? 1 : G::kBLoads;
  Src a_src[G::kALoads], b_src[kBOwn];
  const unsigned char *a_base = reinterpret_cast<const unsigned char *>(hidden_states);
  const unsigned char *b_base = reinterpret_cast<const unsigned char *>(head_weight + (size_t)v0 * hidden);
  // (within the tile: the distance to the last row of the vocabulary itself may pass 32 bits)
  const uint32_t b_last = (uint32_t)min(vocab - 1 - v0, G::kBN - 1) * (uint32_t)(2 * hidden);
#pragma unroll
  for (int j = 0; j < G::kALoads; ++j) {
    const int m = m0 + ld_row + 64 * j, row = tb.row_src[m < m_total ? m : m_total - 1];
    if constexpr (G::kNarrow) a_src[j] = (uint32_t)row * (uint32_t)(2 * hidden);
    else a_src[j] = a_base + (size_t)row * (2 * (size_t)hidden);
  }
#pragma unroll
  for (int j = 0; j < kBOwn; ++j) {
    const int v = ld_row + 64 * j;
    if constexpr (G::kNarrow) b_src[j] = (uint32_t)v * (uint32_t)(2 * hidden);
    else b_src[j] = b_base + (size_t)(v0 + v < vocab ? v : vocab - 1 - v0) * (2 * (size_t)hidden);
  }
  unsigned char *a_smem = smem + wave * 1024, *b_smem = smem + G::kASlots * G::kABytes + wave * 1024;
  // The last step of a row of an odd number of 32s: the lanes of its second half fetch the first again,
  // and put zeros in its place once it has landed (products of zeros leave a sum as it is).
  const int n_steps = (hidden + kTallBK - 1) / kTallBK;
  const bool half_end = hidden % kTallBK != 0;
  auto load_a = [&](int step, int slot, auto jc) {
    constexpr int j = decltype(jc)::value;
    if (j + 1 < G::kALoads || all_a) {
      const int chunk = ld_chunk & (half_end && step + 1 == n_steps ? ~64 : ~0);
      lds_void *dst = (lds_void *)(a_smem + slot * G::kABytes + j * 8192);
      if constexpr (G::kNarrow)
        __builtin_amdgcn_global_load_lds((global_void *)(a_base + (size_t)step * kTallRowBytes + (a_src[j] + chunk)), dst, 16, 0, 0);
      else
        __builtin_amdgcn_global_load_lds((global_void *)(a_src[j] + ((size_t)step * kTallRowBytes + chunk)), dst, 16, 0, 0);
    }
  };
  auto load_b = [&](int step, int slot, auto jc) {
    constexpr int j = decltype(jc)::value;
    const int chunk = ld_chunk & (half_end && step + 1 == n_steps ? ~64 : ~0);
    lds_void *dst = (lds_void *)(b_smem + slot * G::kBBytes + j * 8192);
    if constexpr (G::kNarrow) {
      uint32_t off = b_src[0] + (uint32_t)(j * 128) * (uint32_t)hidden;  // 64 rows each
      off = off < b_last ? off : b_last;
      __builtin_amdgcn_global_load_lds((global_void *)(b_base + (size_t)step * kTallRowBytes + (off + chunk)), dst, 16, 0, 0);
    } else {
      __builtin_amdgcn_global_load_lds((global_void *)(b_src[j] + ((size_t)step * kTallRowBytes + chunk)), dst, 16, 0, 0);
    }
  };
  // Step `step`, in the given slots, is there for all waves.  Of this wave's loads those of B of the
  // step after it (and of A where that has three slots) may be outstanding, if there is one.
  auto landed = [&](int step, int slot_a, int slot_b) {
    if (step + 1 >= n_steps) gemm_wait_vmem<0>();
    else if (G::kASlots == 2) gemm_wait_vmem<G::kBLoads>();
    else if (all_a) gemm_wait_vmem<G::kBLoads + G::kALoads>();
    else gemm_wait_vmem<G::kBLoads + G::kALoads - 1>();
    if (half_end && step + 1 == n_steps) {
      if (ld_chunk & 64) {
        // (opaque, so that no register holds it, or the lane, outside this branch)
        const uint32_t zero = (uint32_t)opaque(0);
        const u32x4 zeros = {zero, zero, zero, zero};
        const int lane = opaque(threadIdx.x) & 63;
#pragma unroll
        for (int j = 0; j < G::kALoads; ++j)
          if (j + 1 < G::kALoads || all_a)
            *reinterpret_cast<u32x4 *>(a_smem + slot_a * G::kABytes + j * 8192 + 16 * lane) = zeros;
#pragma unroll
        for (int j = 0; j < G::kBLoads; ++j)
          *reinterpret_cast<u32x4 *>(b_smem + slot_b * G::kBBytes + j * 8192 + 16 * lane) = zeros;
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    __builtin_amdgcn_s_barrier();
  };

  // ---- per-lane LDS read addresses: row lane % 16 of a 16-row block, chunk lane / 16 (swizzled);
  //      the second 32 of K lie 64 bytes away, up or down
  const int c16 = lane & 15, kq = lane >> 4;
  const uint32_t frag_off = c16 * kTallRowBytes + ((kq ^ ((c16 >> 1) & 7)) << 4);
  const uint32_t a_rd = smem_base + wm * G::kWaveRows * kTallRowBytes + frag_off;
  const uint32_t b_rd = smem_base + G::kASlots * G::kABytes + wn * G::kWaveCols * kTallRowBytes + frag_off;

  TallAcc<MI> acc;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  constexpr int SA = G::kASlots, SB = G::kBSlots;
  auto next_slot = [](int slot, int n) { return slot + 1 == n ? 0 : slot + 1; };
  static_for<2>([&](auto i) {
    if (i < n_steps) {
      if constexpr (i < SA - 1) static_for<G::kALoads>([&](auto j) { load_a(i, i, j); });
      static_for<G::kBLoads>([&](auto j) { load_b(i, i, j); });
    }
  });
  landed(0, 0, 0);
  // slots being multiplied and being filled
  int slot_a = 0, slot_b = 0, fill_a = SA - 1, fill_b = SB - 1;
  for (int step = 0;; ++step) {
    const bool more_a = step + SA - 1 < n_steps, more_b = step + 2 < n_steps;
    if constexpr (SB == 2) fill_b = slot_b;
    constexpr int N = 2 * MI;  // fragments of A in a step
    const uint32_t so_a = a_rd + slot_a * G::kABytes, so_b = b_rd + slot_b * G::kBBytes;
    const uint32_t pa[2] = {so_a, so_a ^ 64u}, pb[2] = {so_b, so_b ^ 64u};
    u32x4 bf[NJ + 2], af[4];
    auto read_a = [&](auto gc) {
      constexpr int g = decltype(gc)::value;
      if constexpr (g < N) af[g & 3] = gemm_lds_read16<(g % MI) * 16 * kTallRowBytes>(pa[g / MI]);
    };
    // the first product needs only A0 and B0: they are read first
    read_a(std::integral_constant<int, 0>{});
    static_for<NJ>([&](auto j) { bf[j] = gemm_lds_read16<j * 16 * kTallRowBytes>(pb[0]); });
    read_a(std::integral_constant<int, 1>{});
    read_a(std::integral_constant<int, 2>{});
    static_for<N>([&](auto gc) {
      constexpr int g = decltype(gc)::value, i = g % MI, ks = g / MI;
      // reads younger than fragment g of A
      constexpr int allowed = (g + 1 < N) + (g + 2 < N) + G::b_behind(g - 2) + G::b_behind(g - 1);
      if constexpr (g == 0) {
        tall_wait_lds2<NJ + 1>(af[0], bf[0]);
        acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, af[0]),
                                                            __builtin_bit_cast(bf16x8, bf[0]), acc[0][0], 0, 0, 0);
        static_for<NJ>([&](auto j) { tall_wait_lds2<2>(af[0], bf[j]); });
      } else {
        tall_wait_lds<allowed>(af[g & 3]);
        if constexpr (g == MI) tall_wait_lds2<allowed>(bf[NJ], bf[NJ + 1]);
      }
      static_for<NJ>([&](auto j) {
        if constexpr (g == MI && j == 2) tall_wait_lds2<1>(bf[2], bf[3]);
        if constexpr (g > 0 || j > 0)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(bf16x8, af[g & 3]), __builtin_bit_cast(bf16x8, bf[ks == 1 && j < 2 ? NJ + j : j]),
              acc[i][j], 0, 0, 0);
      });
      static_for<NJ>([&](auto j) {
        if constexpr (G::b_at(j) == g) bf[j < 2 ? NJ + j : j] = gemm_lds_read16<j * 16 * kTallRowBytes>(pb[1]);
      });
      read_a(std::integral_constant<int, g + 3>{});
      // the loads: A first, then B, whose slot is free here
      if constexpr (SB == 2 && g == MI) {
        if (more_b) __builtin_amdgcn_s_barrier();
      }
      if constexpr (g < G::kALoads) {
        if (more_a) load_a(step + SA - 1, fill_a, gc);
      }
      constexpr int jb = g - (SB == 2 ? MI + 1 : G::kALoads);
      if constexpr (jb >= 0 && jb < G::kBLoads) {
        if (more_b) load_b(step + 2, fill_b, std::integral_constant<int, jb>{});
      }
    });
    // this wave has read all of its slots
    slot_a = next_slot(slot_a, SA);
    fill_a = next_slot(fill_a, SA);
    slot_b = next_slot(slot_b, SB);
    fill_b = next_slot(fill_b, SB);
    if (step + 1 >= n_steps) break;
    landed(step + 1, slot_a, slot_b);
  }
  mfma_settle();
  tid = opaque(threadIdx.x);
  if constexpr (kParked) my_row = parked[tid];
  if (KIND == 0) tall_epilogue_count<MI>(acc, m0, v0, n_tile, vocab, tid, my_row & 0xffffff, my_row >> 24, tb, smem);
  else tall_epilogue_lse<MI>(acc, m0, v0, m_total, vocab, n_tile, tid, tb, smem);
}
