// Early-head scoring, fp32 operands.  Included by early_prune.hip inside namespace propd.
//
// Few score rows (the nodes that have children) against the whole vocabulary: for small batches
// the kernel is a stream of the weight matrix from HBM, for large ones the fp32 matrix cores
// bound it (157 TFLOP/s).  One wave owns 16 vocabulary entries x 16*MT score rows as
// v_mfma_f32_16x16x4_f32 tiles, eight waves (side by side in the vocabulary) make a workgroup.
//   - The instruction wants one float per lane, row lane % 16, k = lane / 16, and the order of k
//     is free as long as both operands and every kernel use the same one.  A lane takes the 16
//     bytes of k = 16 c + 4 (lane / 16) .. + 3 of its row and four instructions use one of the
//     four floats each, so no operand is ever transposed.
//   - Weight rows go straight from memory to the registers that multiply them: a load is 64
//     contiguous bytes of 16 rows, and up to three blocks of 128 floats are in flight behind the
//     one being multiplied (8 waves x 24 KB per compute unit).  Score rows, which all eight
//     waves need, pass through LDS, one block ahead: read by every wave for itself they took
//     twice the load path of the weights (51 us instead of 37 at the size below).  Rows need 4-byte
//     alignment only and may have any length.
//   - Every element is ONE chain over k in rising chunks, starting from zero; a row's tail is
//     filled with zeros, which leave the sum as it is.  own_scores in prune_prepare_kernel runs
//     the same chain, so a child's own score is the same bits as its element here.
//   - The scores pass through LDS once, see rows_epilogue.
// Against one thread per score (every lane walking a weight row of its own, each row fetched
// once per score row): 22 rows x 1024 x 32000, 4186 -> 37 us (131 MB of weights,
// 3.6 TB/s); 704 rows x 2048 x 32000 runs at 95 TFLOP/s.
#pragma once

struct F32Plan {
  int mt;                // wave tile: 16*mt score rows x 16 vocabulary entries
  int m_tiles, n_tiles;  // column tiles are 128 wide
};

// The fewest row tiles first, then the fewest padded rows: padding costs matrix instructions
// (32000 entries x 1024, pruning call: 11 rows 57.9 us at mt 1, 61.5 at 2; 22 rows 65 us at 2, 78.6
// at 4), a second row tile costs a second pass over the weights (44 rows: 84 us at 4, 89 at 2).
// A tile of twice the width (half the reads of the score rows per product) was no faster at 88
// rows (121 against 126 us) and slower at 704 x 2048 (1064 against 990 us).
__host__ __device__ inline F32Plan f32_plan(int m_total, int vocab) {
  F32Plan pl;
  pl.mt = m_total <= 16 ? 1 : (m_total <= 32 ? 2 : 4);
  pl.m_tiles = (m_total + 16 * pl.mt - 1) / (16 * pl.mt);
  pl.n_tiles = (vocab + 127) / 128;
  return pl;
}

constexpr int kF32Threads = kGemmThreads, kF32Waves = kF32Threads / kWave;
constexpr int kF32MaxRows = 64, kF32Cols = kRowsCols;
constexpr int kF32Block = 128, kF32Chunks = kF32Block / 16;  // floats of a row per block, chunks of 16
constexpr int kF32RowBytes = kF32Block * 4 + 16;             // padded: 16 rows start 4 banks apart
// two blocks of the score rows, then (the operands are done with it) the tile's scores
constexpr int kF32LdsBytes = 2 * kF32MaxRows * kF32RowBytes;
static_assert(kF32LdsBytes >= kF32MaxRows * kF32Cols * 4, "scores");

typedef f32x4 f32x4_a4 __attribute__((aligned(4)));  // 16 bytes at a 4-byte aligned address

// 16 bytes of a row with `left` floats from p on (any number, also none), filled with zeros.
__device__ __forceinline__ f32x4 f32_piece(const float *p, int left) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (left >= 4) return *reinterpret_cast<const f32x4_a4 *>(p);
#pragma unroll
  for (int j = 0; j < 3; ++j)
    if (j < left) v[j] = p[j];
  return v;
}

template <int MT, int KIND>
__device__ __forceinline__ void early_head_f32_tile(int hidden, int vocab, int m_total, int m0, int v0, int n_tile,
                                                    const float *__restrict__ hidden_states,
                                                    const float *__restrict__ head_weight, const HeadTables &tb,
                                                    unsigned char *smem) {
  constexpr int BM = 16 * MT, BN = kF32Cols;
  constexpr int R = 4;  // blocks of weight rows in registers
  constexpr int kBufBytes = BM * kF32RowBytes;
  static_assert(2 * kBufBytes <= kF32LdsBytes && BM * BN * 4 <= kF32LdsBytes, "LDS");
  // opaque, so that no shape's address arithmetic is hoisted out of the loop over tiles into
  // registers that stay occupied while another shape runs
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, kq = lane >> 4;
  const int col = 16 * wave + c16;
  const float *wp = head_weight + (size_t)(v0 + col < vocab ? v0 + col : vocab - 1) * hidden + 4 * kq;
  // score rows: thread -> row tid / 32 (+ 16 i), 16-byte piece tid % 32 of a block; rows past the
  // last re-read it, nobody looks at their scores
  const float *ap[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    int m = m0 + 16 * i + (tid >> 5);
    m = m < m_total ? m : m_total - 1;
    ap[i] = hidden_states + (size_t)tb.row_src[m] * hidden + 4 * (tid & 31);
  }
  unsigned char *a_wr = smem + (tid >> 5) * kF32RowBytes + (tid & 31) * 16;
  const unsigned char *a_rd = smem + c16 * kF32RowBytes + kq * 16;

  f32x4 acc[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 w[R][kF32Chunks], ra[MT];
  const int n_blocks = hidden / kF32Block;  // whole blocks; the rest of a row is one more, guarded
  auto load_w = [&](auto slot, int block) {
    constexpr int s = decltype(slot)::value;
#pragma unroll
    for (int k = 0; k < kF32Chunks; ++k)
      w[s][k] = *reinterpret_cast<const f32x4_a4 *>(wp + block * kF32Block + 16 * k);
  };
  auto load_a = [&](int block) {
#pragma unroll
    for (int i = 0; i < MT; ++i) ra[i] = *reinterpret_cast<const f32x4_a4 *>(ap[i] + block * kF32Block);
  };
  auto store_a = [&](int block) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
      *reinterpret_cast<f32x4 *>(a_wr + (block & 1) * kBufBytes + i * 16 * kF32RowBytes) = ra[i];
  };
  // the block is in LDS for every wave, and every wave is done with the block two before it; the
  // loads in flight are not waited for
  auto meet = [&]() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto chunk = [&](int block, int k, const f32x4 &wk) {
    f32x4 a[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
      a[i] = *reinterpret_cast<const f32x4 *>(a_rd + (block & 1) * kBufBytes + i * 16 * kF32RowBytes + k * 64);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < MT; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][j], wk[j], acc[i], 0, 0, 0);
  };
  if (n_blocks > 0) load_a(0);
  static_for<R - 1>([&](auto i) {
    if (i < n_blocks) load_w(i, i);
  });

  const int m1 = m0 + BM < m_total ? m0 + BM : m_total;
  NodeChunk nodes = {0, -1, 0, 0.f};
  NodeRange range = {0, 0, 1, false};
  if (KIND == 0) {  // while the first blocks are on their way
    range = nodes_of_rows(m0, m1, m_total, tb);
    nodes.node = chunk_node(range, range.first, wave, lane, tb);
    if (__builtin_expect(!range.listed, 1)) load_values(nodes, tb);
  }

  meet();  // the tile before this one has been read
  for (int b0 = 0; b0 < n_blocks; b0 += R)
    static_for<R>([&](auto i) {
      const int b = b0 + i;
      if (b >= n_blocks) return;  // uniform
      constexpr int s = decltype(i)::value;
      store_a(b);
      if (b + 1 < n_blocks) load_a(b + 1);
      if (b + R - 1 < n_blocks) load_w(std::integral_constant<int, (s + R - 1) % R>{}, b + R - 1);
      meet();
#pragma unroll
      for (int k = 0; k < kF32Chunks; ++k) chunk(b, k, w[s][k]);
    });
  if (n_blocks * kF32Block < hidden) {  // the rest of the rows, zeros after it
    const int x0 = n_blocks * kF32Block;
#pragma unroll
    for (int i = 0; i < MT; ++i) ra[i] = f32_piece(ap[i] + x0, hidden - x0 - 4 * (tid & 31));
    store_a(n_blocks);
    meet();
    for (int k = 0; x0 + 16 * k < hidden; ++k)
      chunk(n_blocks, k, f32_piece(wp + x0 + 16 * k, hidden - x0 - 16 * k - 4 * kq));
  }
  mfma_settle();
  if (KIND == 0 && __builtin_expect(range.listed, 0)) load_values(nodes, tb);

  float *s_z = reinterpret_cast<float *>(smem);
  __syncthreads();  // the score rows have been read
  // element (row, col) of a 16 x 16 tile: lane col + 16 * (row / 4), register row % 4
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) s_z[(16 * i + 4 * kq + r) * BN + col] = acc[i][r];
  __syncthreads();
  rows_epilogue<KIND>(nodes, range, s_z, wave, lane, m0, m1, v0, vocab, n_tile, tb);
}

// Persistent over the tiles, XCD-aware like the bf16 kernel: the row tiles of one column tile are
// adjacent in time on one XCD, so its weight rows come from HBM once.
template <int KIND>
__global__ __launch_bounds__(kF32Threads) void early_head_f32_kernel(int hidden, int vocab, int B,
                                                                    const float *__restrict__ hidden_states,
                                                                    const float *__restrict__ head_weight,
                                                                    HeadTables tb) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[kF32LdsBytes];
  const int m_total = tb.row_base[B];
  if (m_total <= 0) return;
  const F32Plan pl = f32_plan(m_total, vocab);
  const long long total = (long long)kXcds * ((pl.n_tiles + kXcds - 1) / kXcds) * pl.m_tiles;
  for (long long tile = blockIdx.x; tile < total; tile += gridDim.x) {
    const int xcd = (int)(tile % kXcds);
    const long long slot = tile / kXcds;
    const int n_tile = (int)(slot / pl.m_tiles) * kXcds + xcd;
    if (n_tile >= pl.n_tiles) continue;
    const int m0 = (int)(slot % pl.m_tiles) * 16 * pl.mt, v0 = n_tile * kF32Cols;
    if (pl.mt == 1)
      early_head_f32_tile<1, KIND>(hidden, vocab, m_total, m0, v0, n_tile, hidden_states, head_weight, tb, smem);
    else if (pl.mt == 2)
      early_head_f32_tile<2, KIND>(hidden, vocab, m_total, m0, v0, n_tile, hidden_states, head_weight, tb, smem);
    else
      early_head_f32_tile<4, KIND>(hidden, vocab, m_total, m0, v0, n_tile, hidden_states, head_weight, tb, smem);
  }
}
