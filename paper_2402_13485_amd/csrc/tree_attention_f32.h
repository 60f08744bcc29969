// Tree-masked attention, fp32 operands, fp32 throughout.  Included by tree_attention.hip inside
// namespace propd.
//
// The fp32 matrix instructions are slow (157 TFLOP/s on the chip), so the kernel needs few bytes
// per cycle (under 16 per compute unit) and no LDS on the operand path; what has to be found is
// enough waves.  One wave owns 16*QG queries of a (sequence, head) unit and walks 16-row tiles
// of K/V; the four waves of a workgroup take the tiles of its key range in turn, and a unit's
// keys are split over further workgroups while the chip is not full.
//   - v_mfma_f32_16x16x4_f32 wants one float per lane: row lane % 16, k = lane / 16, and the
//     order of k is free.  S^T = K . Q^T: a lane loads 16 bytes k = 16 c + 4 (lane / 16) .. + 3 of its
//     K row and of its query row, four instructions use one float each.
//   - A lane then holds the scores of query lane % 16 and keys 4 (lane / 16) + r: the softmax
//     statistics are per lane (halves meet by two lane exchanges), and the weights in register r
//     are the B operand of O^T += V^T . P^T for the four keys {4 (lane / 16) + r}.
//   - The order of d in O^T is free as well: block (h, e), row i stands for d = 64 h + 4 i + e, so
//     that the V operand of four blocks is one 16-byte load (4 rows x 256 contiguous bytes per
//     instruction), and a lane's results are 16 contiguous floats.
//   - The next tile's K is requested behind the scores of this one, V behind the weighted sum.
//   - The waves' results are merged through LDS; a unit split over workgroups leaves (O, max, sum)
//     per workgroup for tree_attn_f32_combine_kernel.
// Against one wave per query with every lane walking K rows of its own (2 x 16 units, 48 queries,
// up to 1024 keys, d = 128): 868 -> 21 us, merge kernel 4 us.
#pragma once

constexpr int kF32AttnWaves = 4, kF32AttnThreads = kF32AttnWaves * kWave;
constexpr int kF32MaxSplits = 16;

typedef f32x4 f32x4_a4 __attribute__((aligned(4)));  // 16 bytes at a 4-byte aligned address

struct AttnParamsF32 : AttnParamsPlain<float> {
  int units, splits;
  float scale_log2e;
  float *part;  // [units][query pairs][splits] records of (O [32][D], max [32], sum [32])
};

__host__ __device__ constexpr size_t f32_part_floats(int D) { return (size_t)32 * (D + 2); }

// A result to be merged with factor f: left out where the factor is zero (an infinity would be NaN).
__device__ __forceinline__ float f32_part(float o, float f) { return f == 0.f ? 0.f : o; }

// QG groups of 16 queries of one key range of one unit; s_o, s_ml: the workgroup's LDS.
template <int D, int QG>
__device__ __forceinline__ void f32_attn_range(const AttnParamsF32 &p, int unit, int pair, int split, int b, int q0,
                                               int L, int T, float *s_o, float *s_ml) {
  constexpr int kC = D / 16, kH = D / 64, kRow = D + 4;  // chunks of 16 floats; LDS row, padded
  constexpr int kRows = 16 * QG;
  float *s_m = s_ml, *s_l = s_ml + kF32AttnWaves * 32;  // [wave][32]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15, kq = lane >> 4;
  const int n_cache = (L + 15) / 16, n_tiles = n_cache + (T + 15) / 16;
  const int lo = (int)((long long)n_tiles * split / p.splits), hi = (int)((long long)n_tiles * (split + 1) / p.splits);
  const float *kc = p.k_cache + (size_t)unit * p.L_max * D, *vc = p.v_cache + (size_t)unit * p.L_max * D;
  const float *kt = p.k_tree + (size_t)unit * p.T_max * D, *vt = p.v_tree + (size_t)unit * p.T_max * D;

  f32x4 kf[kC], vf[4][kH];
  auto load_k = [&](int tile) {
    const bool tree = tile >= n_cache;
    const int j0 = 16 * (tree ? tile - n_cache : tile), last = (tree ? T : L) - 1;
    const int row = j0 + c16 < last ? j0 + c16 : last;  // rows past the end: the last one, masked
    const float *src = (tree ? kt : kc) + (size_t)row * D + 4 * kq;
#pragma unroll
    for (int c = 0; c < kC; ++c) kf[c] = *reinterpret_cast<const f32x4_a4 *>(src + 16 * c);
  };
  auto load_v = [&](int tile) {
    const bool tree = tile >= n_cache;
    const int j0 = 16 * (tree ? tile - n_cache : tile), last = (tree ? T : L) - 1;
    const float *src = (tree ? vt : vc) + 4 * c16;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = j0 + 4 * kq + r < last ? j0 + 4 * kq + r : last;
#pragma unroll
      for (int h = 0; h < kH; ++h) vf[r][h] = *reinterpret_cast<const f32x4_a4 *>(src + (size_t)row * D + 64 * h);
    }
  };
  int tile = lo + wave;
  if (tile < hi) {
    load_k(tile);
    load_v(tile);
  }
  // queries (lanes past the tree take its last node: valid memory, never stored)
  f32x4 qf[QG][kC];
  uint64_t a_lo[QG], a_hi[QG];
#pragma unroll
  for (int g = 0; g < QG; ++g) {
    const int t = q0 + 16 * g + c16 < T ? q0 + 16 * g + c16 : T - 1;
    const float *src = p.q + ((size_t)unit * p.T_max + t) * D + 4 * kq;
#pragma unroll
    for (int c = 0; c < kC; ++c) qf[g][c] = *reinterpret_cast<const f32x4_a4 *>(src + 16 * c);
    a_lo[g] = p.anc[((size_t)b * p.T_max + t) * 2];
    a_hi[g] = p.anc[((size_t)b * p.T_max + t) * 2 + 1];
  }
  float m_run[QG], l_run[QG];
  f32x4 o[QG][kH][4];
#pragma unroll
  for (int g = 0; g < QG; ++g) {
    m_run[g] = -INFINITY;
    l_run[g] = 0.f;
#pragma unroll
    for (int h = 0; h < kH; ++h)
#pragma unroll
      for (int e = 0; e < 4; ++e) o[g][h][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  for (; tile < hi; tile += kF32AttnWaves) {
    f32x4 sc[QG];
#pragma unroll
    for (int g = 0; g < QG; ++g) sc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < kC; ++c)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int g = 0; g < QG; ++g) sc[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][j], qf[g][c][j], sc[g], 0, 0, 0);
    mfma_settle();
    if (tile + kF32AttnWaves < hi) load_k(tile + kF32AttnWaves);
    const bool tree = tile >= n_cache;
    const int j0 = 16 * (tree ? tile - n_cache : tile), n_valid = (tree ? T : L) - j0;
    float least = INFINITY;
#pragma unroll
    for (int g = 0; g < QG; ++g) {
#pragma unroll
      for (int r = 0; r < 4; ++r) sc[g][r] *= p.scale_log2e;
      if (tree || n_valid < 16) {  // uniform
        // rows of the tile that exist and (tree rows) that the query's root path holds
        uint32_t vis = n_valid >= 16 ? 0xffffu : (1u << n_valid) - 1u;
        if (tree) vis &= (uint32_t)((j0 < 64 ? a_lo[g] : a_hi[g]) >> (j0 & 63));
        vis >>= 4 * kq;
#pragma unroll
        for (int r = 0; r < 4; ++r) sc[g][r] = ((vis >> r) & 1u) ? sc[g][r] : -INFINITY;
      }
      float m_new = fmaxf(fmaxf(sc[g][0], sc[g][1]), fmaxf(sc[g][2], sc[g][3]));
      m_new = fmaxf(m_new, __shfl_xor(m_new, 16, kWave));
      m_new = fmaxf(m_new, __shfl_xor(m_new, 32, kWave));
      m_new = fmaxf(m_new, m_run[g]);
      const float m_safe = m_new == -INFINITY ? 0.f : m_new;  // nothing visible so far: weights 0
      const float alpha = fast_exp2(m_run[g] - m_safe);
      m_run[g] = m_new;
      float sum = 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        sc[g][r] = fast_exp2(sc[g][r] - m_safe);
        sum += sc[g][r];
        least = fminf(least, sc[g][r]);
      }
      l_run[g] = l_run[g] * alpha + sum;
#pragma unroll
      for (int h = 0; h < kH; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int r = 0; r < 4; ++r) o[g][h][e][r] *= alpha;
    }
    if (__ballot(least < 0x1p-126f) != 0) {  // weights of zero: V is looked through, see not_finite_sum
      uint32_t top = 0;  // of the bits without their signs, shifted (a masked copy would be kept for the use below)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int h = 0; h < kH; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t twice = __float_as_uint(vf[r][h][e]) << 1;
            top = twice > top ? twice : top;
          }
      if (__ballot(top >= 0xff000000u) != 0) {
#pragma unroll
        for (int h = 0; h < kH; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
#pragma unroll
            for (int g = 0; g < QG; ++g) {
              f32x4 codes = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
              for (int r = 0; r < 4; ++r)
                codes = __builtin_amdgcn_mfma_f32_16x16x4f32(not_finite_code(__float_as_uint(vf[r][h][e])),
                                                             sc[g][r] != 0.f ? 1.f : 0.f, codes, 0, 0, 0);
              mfma_settle();
#pragma unroll
              for (int r = 0; r < 4; ++r) o[g][h][e][r] += not_finite_sum(codes[r]);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
              vf[r][h][e] = not_finite_code(__float_as_uint(vf[r][h][e])) != 0.f ? 0.f : vf[r][h][e];
          }
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int h = 0; h < kH; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int g = 0; g < QG; ++g)
            o[g][h][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][h][e], sc[g][r], o[g][h][e], 0, 0, 0);
    mfma_settle();
    if (tile + kF32AttnWaves < hi) load_v(tile + kF32AttnWaves);
  }

  // ---- merge the four waves: O[query][d = 64 h + 16 kq + 4 r + e]
#pragma unroll
  for (int g = 0; g < QG; ++g) {
#pragma unroll
    for (int h = 0; h < kH; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const f32x4 v = {o[g][h][0][r], o[g][h][1][r], o[g][h][2][r], o[g][h][3][r]};
        *reinterpret_cast<f32x4 *>(s_o + (wave * kRows + 16 * g + c16) * kRow + 64 * h + 16 * kq + 4 * r) = v;
      }
    float l = l_run[g];
    l += __shfl_xor(l, 16, kWave);
    l += __shfl_xor(l, 32, kWave);
    if (kq == 0) {
      s_m[wave * 32 + 16 * g + c16] = m_run[g];
      s_l[wave * 32 + 16 * g + c16] = l;
    }
  }
  __syncthreads();
  // thread -> query tid / LPQ, every LPQ-th 16-byte piece of its row
  constexpr int LPQ = kF32AttnThreads / (16 * QG), kPieces = D / 4 / LPQ;
  const int row = threadIdx.x / LPQ, part = threadIdx.x % LPQ, t = q0 + row;
  float M = -INFINITY, lsum = 0.f, f[kF32AttnWaves];
#pragma unroll
  for (int w = 0; w < kF32AttnWaves; ++w) M = fmaxf(M, s_m[w * 32 + row]);
  const float m_safe = M == -INFINITY ? 0.f : M;
#pragma unroll
  for (int w = 0; w < kF32AttnWaves; ++w) {
    f[w] = fast_exp2(s_m[w * 32 + row] - m_safe);
    lsum += s_l[w * 32 + row] * f[w];
  }
  f32x4 acc[kPieces];
#pragma unroll
  for (int x = 0; x < kPieces; ++x) {
    acc[x] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kF32AttnWaves; ++w) {
      const f32x4 v = *reinterpret_cast<const f32x4 *>(s_o + (w * kRows + row) * kRow + 4 * (part + LPQ * x));
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[x][j] += f32_part(v[j], f[w]) * f[w];
    }
  }
  if (p.splits == 1) {
    if (t >= T) return;
    float *dst = p.out + ((size_t)unit * p.T_max + t) * D;
#pragma unroll
    for (int x = 0; x < kPieces; ++x) {
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[x][j] /= lsum;
      *reinterpret_cast<f32x4_a4 *>(dst + 4 * (part + LPQ * x)) = acc[x];
    }
    return;
  }
  float *rec = p.part + (((size_t)unit * ((p.T_max + 31) / 32) + pair) * p.splits + split) * f32_part_floats(D);
#pragma unroll
  for (int x = 0; x < kPieces; ++x) *reinterpret_cast<f32x4 *>(rec + row * D + 4 * (part + LPQ * x)) = acc[x];
  if (part == 0) {
    rec[32 * D + row] = M;
    rec[32 * D + 32 + row] = lsum;
  }
}

// One workgroup per (unit, 32 queries, split).  MQ: groups of 16 queries it may find (1 when T_max <= 16).
template <int D, int MQ>
__global__ __launch_bounds__(kF32AttnThreads, 2) void tree_attn_f32_kernel(AttnParamsF32 p) {
  __shared__ __attribute__((aligned(16))) float s_o[kF32AttnWaves * 16 * MQ * (D + 4)];
  __shared__ float s_ml[2 * kF32AttnWaves * 32];
  // the query groups of one key range run on one XCD where the counts allow (its L2 holds the rows)
  const unsigned per_pair = (unsigned)p.units * (unsigned)p.splits;
  const unsigned block = blockIdx.y * gridDim.x + blockIdx.x;
  const int pair = (int)(block / per_pair);
  const unsigned us = block - (unsigned)pair * per_pair;
  const int unit = (int)(us / (unsigned)p.splits), split = (int)(us - (unsigned)unit * (unsigned)p.splits);
  const int b = unit / p.H, q0 = 32 * pair;
  int T = p.n_nodes[b], L = p.seq_lens[b];
  T = T < 1 ? 1 : (T > p.T_max ? p.T_max : T);
  L = L < 0 ? 0 : (L > p.L_max ? p.L_max : L);
  if (q0 >= T) return;  // also where the last row of the grid is not full
  if (MQ == 1 || q0 + 16 >= T) f32_attn_range<D, 1>(p, unit, pair, split, b, q0, L, T, s_o, s_ml);
  else f32_attn_range<D, MQ>(p, unit, pair, split, b, q0, L, T, s_o, s_ml);
}

// Units split over workgroups: out = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s, always in
// the order of the splits, all of a thread's pieces requested before the first is used.  One
// thread per 16 bytes of the result.
template <int D>
__global__ __launch_bounds__(kF32AttnThreads) void tree_attn_f32_combine_kernel(AttnParamsF32 p) {
  constexpr int LPQ = D / 4, kRows = kF32AttnThreads / LPQ, kBlocks = 32 / kRows;
  const int n_pairs = (p.T_max + 31) / 32;
  const unsigned up = blockIdx.x / kBlocks;
  const int unit = (int)(up / (unsigned)n_pairs), pair = (int)(up - (unsigned)unit * (unsigned)n_pairs);
  int T = p.n_nodes[unit / p.H];
  T = T < 1 ? 1 : (T > p.T_max ? p.T_max : T);
  const int row = (blockIdx.x % kBlocks) * kRows + threadIdx.x / LPQ, part = threadIdx.x % LPQ, t = 32 * pair + row;
  if (32 * pair + (int)(blockIdx.x % kBlocks) * kRows >= T) return;  // uniform
  const float *rec = p.part + (size_t)up * p.splits * f32_part_floats(D);
  f32x4 v[kF32MaxSplits];
  float m[kF32MaxSplits], l[kF32MaxSplits];
#pragma unroll
  for (int s = 0; s < kF32MaxSplits; ++s) {
    const float *q = rec + (s < p.splits ? s : 0) * f32_part_floats(D);
    v[s] = *reinterpret_cast<const f32x4 *>(q + row * D + 4 * part);
    m[s] = q[32 * D + row];
    l[s] = q[32 * D + 32 + row];
  }
  float M = -INFINITY;
#pragma unroll
  for (int s = 0; s < kF32MaxSplits; ++s) M = fmaxf(M, m[s]);  // past the last split: the first once more
  const float m_safe = M == -INFINITY ? 0.f : M;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  float lsum = 0.f;
#pragma unroll
  for (int s = 0; s < kF32MaxSplits; ++s) {
    if (s < p.splits) {  // uniform
      const float f = fast_exp2(m[s] - m_safe);
      lsum += l[s] * f;
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] += f32_part(v[s][j], f) * f;
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] /= lsum;
  if (t < T) *reinterpret_cast<f32x4_a4 *>(p.out + ((size_t)unit * p.T_max + t) * D + 4 * part) = acc;
}

// Workgroups per unit and 32 queries.  `full`, two workgroups for every compute unit with at least kF32MinTiles tiles each, unless
// another number makes the longest chain shorter.  A chain is counted in rounds of 16-row tiles that a wave takes (about
// 2.1 us each at d = 128); a second workgroup on a compute unit costs about two rounds, its loads and matrix
// instructions being in the way of the first one's (one round at d = 64, and where sequences may be shorter than the
// longest), and the merge kernel two (three of the short ones at d = 64 and at most 16 queries).  Considered are all
// numbers that leave one workgroup per compute unit, and those beyond `full` that leave two; of equal cost `full`, then the least.
// Where `full` leaves two already and the last of several groups of 32 queries has 16 or fewer, so that its workgroups end
// early, more of them pay now and then only: `full` then.  Splits also shorten the chains of the sums: no less than three quarters
// of `full` are taken, and the mean error against 64 bits over 40 calls of random sizes is what it was (0.997 of it).
// Calls, us, with `full` / this rule: 16 units of 115 x 561 25.2 / 19.2 (320 / 256 workgroups), 16 x 63 x 1082 22.7 / 19.6 (288 /
// 256), 8 x 115 x 198 18.0 / 13.4 (64 / 160), 12 x 86 x 1063 (d = 64) 16.6 / 14.1, 40 x 20 x 1279 (d = 64) 17.1 / 15.9 (400 / 440).
// With `full` / the other number where `full` is kept: 40 x 108 x 158 23.4 / 26.1 (320 / 480), 16 x 65 x 980 (d = 64) 14.6 / 15.7
// (384 / 432), 32 x 78 x 484 23.8 / 25.1 (384 / 480), 64 x 12 x 211 (d = 64) 8.0 / 8.6 (64 / 256).  308 calls of random sizes for
// which another number is taken: geometric mean 1.157, and none more than 2 % slower but four ragged batches, whose lengths
// the host does not know (36 x 51 x up to 623 0.89 to 1.12, 96 x 29 x up to 551 0.91 to 1.04).
constexpr int kF32MinTiles = 8;
static int f32_splits(long long base, int tiles, int cus, size_t workspace_bytes, int D, int T_max, bool one_sequence) {
  long long most = (long long)(workspace_bytes / (f32_part_floats(D) * 4)) / base;  // room for the partial results
  if (most > kF32MaxSplits) most = kF32MaxSplits;
  long long full = (2ll * cus + base - 1) / base;
  if (full > tiles / kF32MinTiles) full = tiles / kF32MinTiles;
  if (full > most) full = most;
  if (full < 1) full = 1;
  const bool short_last = T_max > 32 && (T_max - 1) % 32 < 16;
  auto cost = [&](long long s) {
    const long long rounds = ((tiles + s - 1) / s + kF32AttnWaves - 1) / kF32AttnWaves;
    return rounds + (s > 1 ? (D == 64 && T_max <= 16 ? 3 : 2) : 0) + (base * s > cus ? (D == 128 && one_sequence ? 2 : 1) : 0);
  };
  long long best = full;
  for (long long s = (3 * full + 3) / 4; s <= most && base * s <= 2ll * cus; ++s) {
    if (base * s > cus && (s < full || (short_last && base * full > cus))) continue;
    if (cost(s) < cost(best)) best = s;
  }
  return (int)best;
}

template <int D>
static bool launch_f32(AttnParamsF32 p, int cus, void *workspace, size_t workspace_bytes, hipStream_t st) {
  const int pairs = (p.T_max + 31) / 32;
  // records are read and written 16 bytes at a time
  if (!workspace || reinterpret_cast<uintptr_t>(workspace) % 16 != 0) workspace_bytes = 0;
  p.part = reinterpret_cast<float *>(workspace);
  p.splits = f32_splits((long long)p.units * pairs, (p.L_max + 15) / 16 + (p.T_max + 15) / 16, cus, workspace_bytes, D,
                        p.T_max, p.units == p.H);
  // a dimension of the grid holds fewer than 2^32 threads, and there may be 2^28 units
  constexpr unsigned kGridX = 1u << 22;
  const unsigned blocks = (unsigned)p.units * (unsigned)pairs * (unsigned)p.splits;
  const dim3 grid(blocks < kGridX ? blocks : kGridX, (blocks + kGridX - 1) / kGridX);
  if (p.T_max <= 16)
    hipLaunchKernelGGL((tree_attn_f32_kernel<D, 1>), grid, dim3(kF32AttnThreads), 0, st, p);
  else
    hipLaunchKernelGGL((tree_attn_f32_kernel<D, 2>), grid, dim3(kF32AttnThreads), 0, st, p);
  if (!launch_ok()) return false;
  if (p.splits == 1) return true;
  constexpr unsigned kBlocks = 32 / (kF32AttnThreads / (D / 4));
  hipLaunchKernelGGL(tree_attn_f32_combine_kernel<D>, dim3((unsigned)p.units * (unsigned)pairs * kBlocks),
                     dim3(kF32AttnThreads), 0, st, p);
  return launch_ok();
}
