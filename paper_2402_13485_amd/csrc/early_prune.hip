// Early pruning of the token tree (Section 4.1: "Pruning Process", "Pruning Criterion" and
// "Implementation Optimization").
//
// Kernel chain, all on the caller's stream, no host round trip:
//   prune_prepare_kernel  one launch, two kinds of workgroups.  Workgroup 0: which nodes have
//                         children (only those need early-head scores), the table of score
//                         rows, and every node's children grouped by parent.  The others:
//                         each child's OWN score z_p[tok_c], 8 children per workgroup, by the
//                         same chain of matrix instructions that the scoring kernel runs for
//                         that element, so the two values are the same bits
//   early_head_bf16_kernel  scores z = hidden[parent rows] . head_weight^T as a bf16 MFMA
//                         GEMM with fp32 accumulation (M = parent rows, N = vocabulary,
//                         K = hidden).  The scores never leave the registers: the epilogue
//                         compares every score of a row with the own scores of that row's
//                         children and leaves, per child and column tile, the count of scores
//                         that beat it (the top-k membership test; plain stores, every slot
//                         written exactly once, so the sums do not depend on any order), or, for the
//                         probability criterion, leaves (max, sum of exponentials) per row
//                         and column tile
//   early_head_f32_kernel the same on the fp32 matrix instructions (early_head_f32.h)
//   prune_finish_kernel   per sequence: the criterion's decision per node (rank against k, or
//                         path marginal against the threshold / the keep count; for the latter the
//                         log-sum-exp of every row from the tile partials first), fail bits by
//                         ballot, branch elimination by testing the cached ancestor bitset
//                         against the fail bits, order-preserving compaction by prefix
//                         popcount, mask subsampling by bit extraction; then the survivor rows of
//                         the listed payload tensors, shared among the workgroups of the sequence;
//                         the last sequence to arrive leaves the prefix sum of the survivor counts
//   cu_nodes_kernel       that prefix sum where nothing was scored
#include <atomic>
#include <cstdlib>
#include <type_traits>
#include <utility>

#include "common.h"

namespace propd {

// ------------------------------------------------------------------------------------
// scratch layout
// ------------------------------------------------------------------------------------
constexpr int kNoteTiles = 0;    // column tiles of the scoring kernel's plan
constexpr int kNoteArrived = 1;  // sequences, or lines of them, whose survivor counts are written (prune_finish_kernel)
constexpr int kNoteLine = 32;    // words of a line; in the lines behind the first one arrive some of the sequences each

// Lines on which the sequences of a batch arrive (a power of two; 0: all on the first).  Arrivals on one line pass one by
// one, about 8 ns each: prune_finish_kernel at 1000 sequences of 16 nodes 26.7 us with one line, 21.7 with 32.  The notes
// have room for one word per node slot.
__host__ __device__ inline int arrival_lines(int B, int T_max) {
  int lines = 0;
  if (B > 64)
    for (lines = 32; lines > 0 && (long long)(lines + 1) * kNoteLine > (long long)B * T_max; lines >>= 1) {
    }
  return lines;
}

struct PruneScratch {
  int32_t *row_src;     // [B*T_max]  score row -> b*T_max + node
  int32_t *row_base;    // [B+1]      score rows of the sequences before b; [B] = total rows
  int32_t *row_info;    // [B*T_max][2] score row -> (first position in child_list, children)
  int32_t *child_list;  // [B*T_max]  b*T_max + child, grouped by parent, in the order of the score rows; as many places
                        //            for a sequence as it has nodes, -1 in those left over
  float *own;           // [B*T_max]  z_parent[token] of every non-root node
  int32_t *notes;       // what the kernels leave each other, see kNote*
  float *lse_part;      // [row_cap * parts][2]  probability criterion: (max, sum exp) per tile
  int32_t *node_row;    // [B*T_max]  top-k criterion: node -> score row of its parent, or -1 (in the place of lse_part)
  int32_t *cnt_part;    // [vocab / 128][B*T_max]  top-k criterion: per column tile, the scores of the
                        //                       parent's row that beat the node's token
  size_t row_cap, parts, total_bytes;
};

static PruneScratch carve_scratch(void *base, int B, int T_max, int vocab) {
  PruneScratch s;
  char *p = reinterpret_cast<char *>(base);
  size_t off = 0;
  const size_t nt = (size_t)B * T_max;
  auto take = [&](size_t bytes) {
    char *q = p ? p + off : nullptr;
    off += align_up(bytes, 256);
    return q;
  };
  s.row_src = reinterpret_cast<int32_t *>(take(nt * 4));
  s.row_base = reinterpret_cast<int32_t *>(take((size_t)(B + 1) * 4));
  s.row_info = reinterpret_cast<int32_t *>(take(nt * 8));
  s.child_list = reinterpret_cast<int32_t *>(take(nt * 4));
  s.own = reinterpret_cast<float *>(take(nt * 4));
  s.notes = reinterpret_cast<int32_t *>(take(nt * 4));  // (at least 64 words)
  s.row_cap = (size_t)B * (T_max > 1 ? T_max - 1 : 1);  // a node with children is not a leaf
  s.parts = ((size_t)vocab + 127) / 128;  // column parts of a row: one per tile, of at least 128 columns
  s.lse_part = reinterpret_cast<float *>(take(s.row_cap * s.parts * 8));
  s.node_row = reinterpret_cast<int32_t *>(s.lse_part);  // row_cap * 8 bytes are never less than B*T_max * 4
  s.cnt_part = reinterpret_cast<int32_t *>(take(s.parts * nt * 4));
  s.total_bytes = off;
  return s;
}

size_t early_prune_workspace_bytes(int B, int T_max, int vocab) {
  return carve_scratch(nullptr, B, T_max, vocab).total_bytes;
}

__device__ __forceinline__ int clamp_tree(int T, int T_max) { return T < 1 ? 1 : (T > T_max ? T_max : T); }

constexpr int kScanThreads = 256;

// Exclusive prefix sum of in[0..n) into out[0..n], out[n] = total.  One workgroup.
__device__ void block_exclusive_scan(const int32_t *__restrict__ in, int32_t *__restrict__ out,
                                     int n) {
  const int tid = threadIdx.x;
  const int per = (n + kScanThreads - 1) / kScanThreads;
  const int lo = tid * per, hi = (lo + per < n) ? lo + per : n;
  int sum = 0;
  for (int x = lo; x < hi; ++x) sum += in[x];
  // exclusive scan of the per-thread sums: within each wave by shuffles, then across waves
  const int lane = tid & 63, wv = tid >> 6;
  int incl = sum;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int up = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += up;
  }
  __shared__ int s_wave[kScanThreads / kWave];
  if (lane == kWave - 1) s_wave[wv] = incl;
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kScanThreads / kWave; ++w) {
    if (w < wv) before += s_wave[w];
    total += s_wave[w];
  }
  if (tid == 0) out[n] = total;
  int run = before + incl - sum;
  for (int x = lo; x < hi; ++x) {
    const int v = in[x];
    out[x] = run;
    run += v;
  }
}

__global__ __launch_bounds__(kScanThreads) void cu_nodes_kernel(int B,
                                                                const int32_t *__restrict__ n_kept,
                                                                int32_t *__restrict__ cu_nodes) {
  block_exclusive_scan(n_kept, cu_nodes, B);
}

// ------------------------------------------------------------------------------------
// preparation: tables (the first workgroups) and the children's own scores (the others)
// ------------------------------------------------------------------------------------
struct PrepareArgs {
  int B, T_max, hidden, vocab;
  const int32_t *n_nodes, *parent, *token;
  const void *hidden_states, *head_weight;
  int32_t *row_src, *row_base, *row_info, *child_list, *notes;
  int32_t *node_row;  // top-k criterion, otherwise NULL
  float *own;
};

constexpr int kTableWaves = kScanThreads / kWave;  // sequences per table workgroup, one per wave

// Everything a wave needs from other lanes goes through a 128-entry array of its own in LDS,
// ordered by the wave's own program order (LDS operations of a wave complete in order).
__device__ __forceinline__ void wave_lds_fence() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// The valid parent of node `nd` of a tree with T nodes as loaded (-1: none; a parent that is no
// earlier node makes no edge).
__device__ __forceinline__ int valid_parent(int nd, int T, int p) {
  return (nd > 0 && nd < T && p >= 0 && p < nd) ? p : -1;
}

// Table workgroup g, wave wv: the tables of sequence b = kTableWaves * g + wv, two nodes per lane
// (lane and lane + 64).  A sequence's score rows, and its places in the list of children, follow those of all sequences
// before it, so the wave needs the numbers of nodes with children, and of nodes, of every earlier sequence: the waves of the
// workgroup count them together (sequence x by wave x % kTableWaves, a mark per parent in LDS,
// all loads of a wave's sequences in flight before the first is used) and exchange the counts
// through LDS.  No workgroup waits for another: each one counts for itself what it needs.
__device__ void prepare_tables(const PrepareArgs &a, int g) {
  constexpr int kBatch = 8;  // sequences a wave counts per round
  __shared__ int s_cnt[kTableWaves][PROPD_MAX_TREE];
  __shared__ int s_rows[kTableWaves], s_nodes[kTableWaves];  // rows and nodes before this workgroup's sequences, per counting wave
  __shared__ int s_own[kTableWaves], s_own_nodes[kTableWaves];  // of the workgroup's own sequences
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int *cnt = s_cnt[wv];
  const int b = kTableWaves * g + wv;
  const int node[2] = {lane, lane + 64};

  // ---- nodes with children of the earlier sequences this wave counts: x = wv, wv + 4, ... < 4 g
  int rows_before = 0, nodes_before = 0;
  for (int x0 = wv; x0 < kTableWaves * g; x0 += kTableWaves * kBatch) {
    int Tx[kBatch], px[kBatch][2];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int x = x0 + kTableWaves * i;
      const bool in = x < kTableWaves * g;
      const size_t base = (size_t)(in ? x : 0) * a.T_max;
      Tx[i] = in ? clamp_tree(a.n_nodes[x], a.T_max) : 0;
#pragma unroll
      for (int h = 0; h < 2; ++h) px[i][h] = node[h] < a.T_max ? a.parent[base + node[h]] : -1;
    }
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      if (x0 + kTableWaves * i >= kTableWaves * g) break;  // uniform
      nodes_before += Tx[i];
      cnt[node[0]] = 0;
      cnt[node[1]] = 0;
      wave_lds_fence();
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int p = valid_parent(node[h], Tx[i], px[i][h]);
        if (p >= 0) cnt[p] = 1;
      }
      wave_lds_fence();
      rows_before += __popcll(__ballot(cnt[node[0]] != 0)) + __popcll(__ballot(cnt[node[1]] != 0));
      wave_lds_fence();
    }
  }

  // ---- this wave's own sequence
  int T = 0, par[2] = {-1, -1}, slot[2] = {0, 0}, mine[2] = {0, 0}, incl[2] = {0, 0}, par_before[2] = {0, 0};
  int run_par = 0, run_kids = 0;
  const size_t base = (size_t)(b < a.B ? b : 0) * a.T_max;
  if (b < a.B) {  // uniform over the wave
    T = clamp_tree(a.n_nodes[b], a.T_max);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      par[h] = valid_parent(node[h], T, node[h] < a.T_max ? a.parent[base + node[h]] : -1);
      cnt[node[h]] = 0;
    }
    wave_lds_fence();
    // children per parent; the value before the addition numbers a child among its siblings
#pragma unroll
    for (int h = 0; h < 2; ++h) slot[h] = par[h] >= 0 ? atomicAdd(&cnt[par[h]], 1) : 0;
    wave_lds_fence();
    mine[0] = cnt[node[0]];
    mine[1] = cnt[node[1]];
    wave_lds_fence();
    // exclusive prefix of the child counts over the nodes, and of "has children"
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      incl[h] = mine[h];
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const int up = __shfl_up(incl[h], o, kWave);
        if (lane >= o) incl[h] += up;
      }
      const int total = __shfl(incl[h], 63, kWave);
      incl[h] += run_kids;
      run_kids += total;
      const uint64_t has = __ballot(mine[h] > 0);
      par_before[h] = run_par + __popcll(has & ((1ull << lane) - 1ull));
      run_par += __popcll(has);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) cnt[node[h]] = incl[h] - mine[h];  // first position of this node's children
  }
  if (lane == 0) {
    s_rows[wv] = rows_before;
    s_nodes[wv] = nodes_before;
    s_own[wv] = run_par;
    s_own_nodes[wv] = T;
  }
  __syncthreads();
  if (b >= a.B) return;
  int first = 0, place = 0;
#pragma unroll
  for (int w = 0; w < kTableWaves; ++w) {
    first += s_rows[w] + (w < wv ? s_own[w] : 0);
    place += s_nodes[w] + (w < wv ? s_own_nodes[w] : 0);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (par[h] >= 0) a.child_list[place + cnt[par[h]] + slot[h]] = (int)base + node[h];
    if (node[h] >= run_kids && node[h] < T) a.child_list[place + node[h]] = -1;
    if (mine[h] > 0) {
      const int r = first + par_before[h];
      a.row_src[r] = (int)base + node[h];
      a.row_info[2 * r] = place + incl[h] - mine[h];
      a.row_info[2 * r + 1] = mine[h];
    }
  }
  if (a.node_row) {
    // the score row of every node's parent, -1 for nodes (and padding) without one
    wave_lds_fence();
    cnt[node[0]] = par_before[0];
    cnt[node[1]] = par_before[1];
    wave_lds_fence();
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (node[h] < a.T_max) a.node_row[base + node[h]] = par[h] >= 0 ? first + cnt[par[h]] : -1;
  }
  if (lane == 0) {
    a.row_base[b] = first;
    if (b == a.B - 1) a.row_base[a.B] = first + run_par;
  }
}

// The children's own scores: workgroup (b, group) takes nodes 8*group .. +7 of
// sequence b (few nodes per workgroup: the rows are fetched once, from all over the weight
// matrix, and it is the number of workgroups that brings the bytes in flight).  Tile rows:
// A row j = hidden state of the parent of node j, B row j = weight row of node j's token; the
// diagonal of A . B^T holds the scores wanted (rows 8..15 of the 16-row tile repeat rows
// 0..7).  All four waves fetch (coalesced, eight 512-byte steps ahead, through registers into
// a padded double buffer in LDS); wave 0 runs the chain of matrix instructions over
// K in rising order, starting from zero.
//   bf16: the chain of 16x16x32 instructions that the tiles of many rows of the scoring kernel run
//     for every element (the 32x32x16 chain of the tile of few rows, two instructions per 32 of K,
//     gives the same bits: measured, and held to it by the test of equal scores on both).
//   fp32: the chain of 16x16x4 instructions of the fp32 scoring kernel: the four floats of a
//     lane's 16-byte piece one after the other.  (One lane per node walking its two rows took
//     78 us for 62 nodes of 1024 floats, a chain of 1024 dependent loads.)
constexpr int kOwnNodes = 8;                      // children per workgroup
constexpr int kOwnStepBytes = 512;                // bytes of a row per fetch step
constexpr int kOwnRowBytes = kOwnStepBytes + 16;  // padded: the 8 rows start 4 banks apart
constexpr int kOwnAhead = 8;

typedef u32x4 u32x4_a4 __attribute__((aligned(4)));  // 16 bytes at a 4-byte aligned address

template <bool kBf16>
__device__ void own_scores(const PrepareArgs &a, int b, int group) {
  constexpr int kElem = kBf16 ? 2 : 4, kPiece = 16 / kElem;  // bytes per element, elements per 16-byte piece
  constexpr int kOwnStep = kOwnStepBytes / kElem;
  __shared__ __attribute__((aligned(16))) unsigned char s_tile[2][2][kOwnNodes * kOwnRowBytes];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int T = clamp_tree(a.n_nodes[b], a.T_max);
  if (kOwnNodes * group >= T) return;  // uniform over the workgroup
  const size_t base = (size_t)b * a.T_max;
  // loader: thread -> (row, 16-byte piece of the step's 512 bytes)
  const int ld_row = tid >> 5, ld_piece = tid & 31;
  int nd = kOwnNodes * group + ld_row;
  nd = nd < T ? nd : T - 1;
  int p = nd > 0 ? a.parent[base + nd] : 0;
  p = (p >= 0 && p < T) ? p : 0;
  int tk = a.token[base + nd];
  tk = (tk >= 0 && tk < a.vocab) ? tk : 0;
  const char *a_src = reinterpret_cast<const char *>(a.hidden_states) + (base + p) * (size_t)a.hidden * kElem;
  const char *b_src = reinterpret_cast<const char *>(a.head_weight) + (size_t)tk * a.hidden * kElem;
  const int n_steps = (a.hidden + kOwnStep - 1) / kOwnStep;
  // 64-byte groups of a row (bf16: whole, the row length is a multiple of 32; fp32: the last
  // one is filled with zeros, as in the scoring kernel)
  const int n_groups = (a.hidden * kElem + 63) / 64;
  u32x4 ra[kOwnAhead], rb[kOwnAhead];
  auto fetch = [&](int slot, int step) {
    const int x = step * kOwnStep + ld_piece * kPiece;  // the piece's first element
    if (kBf16) {
      const int off = (step < n_steps && x < a.hidden ? x : ld_piece * kPiece < a.hidden ? ld_piece * kPiece : 0) * kElem;
      ra[slot] = *reinterpret_cast<const u32x4 *>(a_src + off);
      rb[slot] = *reinterpret_cast<const u32x4 *>(b_src + off);
    } else if (x + kPiece <= a.hidden) {
      ra[slot] = *reinterpret_cast<const u32x4_a4 *>(a_src + (size_t)x * kElem);
      rb[slot] = *reinterpret_cast<const u32x4_a4 *>(b_src + (size_t)x * kElem);
    } else {
      ra[slot] = rb[slot] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int j = 0; j < kPiece; ++j)
        if (x + j < a.hidden) {
          ra[slot][j] = reinterpret_cast<const uint32_t *>(a_src)[x + j];
          rb[slot][j] = reinterpret_cast<const uint32_t *>(b_src)[x + j];
        }
    }
  };
#pragma unroll
  for (int i = 0; i < kOwnAhead; ++i) fetch(i, i);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  // fragment of one 64-byte group: lane -> row lane % 16 (rows 8..15 repeat rows 0..7), 16-byte
  // piece lane / 16
  const int c16 = lane & 15, kq = lane >> 4;
  const int frag_off = (c16 & (kOwnNodes - 1)) * kOwnRowBytes + kq * 16;
  // Wave 0 reads a step's fragments while it multiplies those of the step before, so that the chain of
  // products does not wait for LDS once per step: pruning call 75.2 -> 73.8 us at 1 x 64 nodes x 4096, 239.3 ->
  // 237.4 at 16 x 128 x 5120; nothing in fp32.  (The barrier of the next step waits for these reads,
  // and the buffer is written again only behind it.)
  constexpr int kGroups = kOwnStepBytes / 64;
  u32x4 fa[2][kGroups], fb[2][kGroups];
  auto read = [&](int set, const unsigned char *pa, const unsigned char *pb) {
#pragma unroll
    for (int ks = 0; ks < kGroups; ++ks) {
      fa[set][ks] = *reinterpret_cast<const u32x4 *>(pa + frag_off + ks * 64);
      fb[set][ks] = *reinterpret_cast<const u32x4 *>(pb + frag_off + ks * 64);
    }
  };
  auto product = [&](const u32x4 &x, const u32x4 &y) {
    if constexpr (kBf16) {
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), acc, 0, 0, 0);
    } else {
      const f32x4 xf = __builtin_bit_cast(f32x4, x), yf = __builtin_bit_cast(f32x4, y);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(xf[j], yf[j], acc, 0, 0, 0);
    }
  };
  auto last_step = [&](int set) {  // may end inside
    const int left = n_groups - (n_steps - 1) * kGroups;
#pragma unroll
    for (int ks = 0; ks < kGroups; ++ks)
      if (ks < left) product(fa[set][ks], fb[set][ks]);
  };
  static_assert(kOwnAhead % 2 == 0, "the fragment set of a step is its number's parity");
  for (int s0 = 0; s0 < n_steps; s0 += kOwnAhead) {
#pragma unroll
    for (int i = 0; i < kOwnAhead; ++i) {
      const int step = s0 + i;
      if (step >= n_steps) break;  // uniform
      unsigned char *buf_a = s_tile[step & 1][0], *buf_b = s_tile[step & 1][1];
      *reinterpret_cast<u32x4 *>(buf_a + ld_row * kOwnRowBytes + ld_piece * 16) = ra[i];
      *reinterpret_cast<u32x4 *>(buf_b + ld_row * kOwnRowBytes + ld_piece * 16) = rb[i];
      fetch(i, step + kOwnAhead);
      __syncthreads();  // the step is in LDS; wave 0 has read the other buffer
      if (wave == 0) {
        read(i & 1, buf_a, buf_b);
        if (step > 0) {
#pragma unroll
          for (int ks = 0; ks < kGroups; ++ks) product(fa[1 - (i & 1)][ks], fb[1 - (i & 1)][ks]);
        }
      }
    }
  }
  if (wave != 0) return;
  if (n_steps & 1) last_step(0);
  else last_step(1);
  mfma_settle();
  // element (row, col) of the tile sits in lane col + 16 * (row / 4), register row % 4: the
  // diagonal element of column j < 8 is in the lane quarter j >> 2, register j & 3
  float diag = 0.f;
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (r == (c16 & 3)) diag = acc[r];
  const int my_node = kOwnNodes * group + c16;
  if (c16 < kOwnNodes && kq == (c16 >> 2) && my_node > 0 && my_node < T) a.own[base + my_node] = diag;
}

template <bool kBf16>
__global__ __launch_bounds__(kScanThreads) void prune_prepare_kernel(PrepareArgs a) {
  const int table_groups = (a.B + kTableWaves - 1) / kTableWaves;
  if ((int)blockIdx.x < table_groups) {
    if (blockIdx.x == 0) {
      if (threadIdx.x == 0) a.notes[kNoteArrived] = 0;
      if (threadIdx.x >= 1 && (int)threadIdx.x <= arrival_lines(a.B, a.T_max)) a.notes[threadIdx.x * kNoteLine] = 0;
    }
    prepare_tables(a, blockIdx.x);
    return;
  }
  const int groups = (a.T_max + kOwnNodes - 1) / kOwnNodes;
  const int ob = blockIdx.x - table_groups;
  const int b = ob / groups, group = ob - b * groups;
  own_scores<kBf16>(a, b, group);
}

// What the scoring kernels need besides the operands.
struct HeadTables {
  const int32_t *row_src, *row_base, *row_info, *child_list, *token, *node_row;
  const float *own;
  int32_t *cnt_part;  // [column tile][cnt_stride]
  int cnt_stride;     // B * T_max
  int T_max;
  float *lse_part;
  int parts;  // column parts per row in lse_part
  int32_t *n_tiles;  // bf16: the column tiles of the plan, left for prune_finish_kernel
};

// ------------------------------------------------------------------------------------
// early head, bf16 MFMA
// ------------------------------------------------------------------------------------
// C[m][v] = sum_x A[m][x] * W[v][x].  Both operands are contiguous along x, which is the layout the
// matrix instructions want (8 consecutive x per lane), so tiles go global -> LDS -> operands
// without any transpose.  Two kinds of tiles, chosen on the device from the row count (head_plan):
//   - few (at most 128, or 192 in one round): early_head_small_tile, a stream of the weights;
//   - more: the tiles of early_head_tall.h, 32*MI rows x 256 vocabulary entries in several
//     shapes.  They are bound by operand delivery and the matrix cores together.
// Common to all:
//   - K advances through a ring of LDS stages filled by direct global->LDS loads (no staging
//     registers, no LDS stores), whose 16-byte chunks are XOR-swizzled on the global side so that
//     fragment reads are free of bank conflicts;
//   - the A rows are gathered through the row table by the loads themselves; rows past
//     the last one and vocabulary entries past the last re-read the last valid one and
//     are left out by the epilogue;
//   - every element is one chain of products in rising K, started from zero, the same bits
//     whatever the tile (two 32x32x16 products sum 32 of K as one 16x16x32 does: measured, and held
//     to it by the test of equal scores), so that a child's own score can be compared with any;
//   - the scores stay in the accumulators: the epilogue turns them into rank counts (or
//     log-sum-exp partials) and nothing of size rows x vocabulary ever reaches memory;
//   - the grid is one-dimensional, persistent and XCD-aware.  Workgroups are handed to the 8
//     XCDs round-robin, each XCD has its own L2: tile id -> (xcd, slot), and an XCD walks
//     its own vocabulary tiles with all row tiles of one vocabulary tile adjacent in time,
//     so a weight tile is fetched from HBM once and hits in that XCD's L2 for the other
//     row tiles.
constexpr int kBK = 32;
constexpr int kGemmThreads = 512, kGemmWaves = kGemmThreads / kWave;
constexpr int kTallWideMI = 8;  // the tallest tile whose registers have room for row addresses of 64 bits
constexpr int kXcds = 8;
constexpr int kHeadLdsBytes = 163840;  // dynamic LDS of the scoring kernel: the largest ring of its tile shapes

template <int N>
__device__ __forceinline__ void gemm_wait_vmem() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

template <int N>
__device__ __forceinline__ void gemm_wait_at_most(int n) {
  if constexpr (N == 0) {
    gemm_wait_vmem<0>();
  } else {
    if (n >= N) gemm_wait_vmem<N>();
    else gemm_wait_at_most<N - 1>(n);
  }
}
// Waits until at most n <= MAXN of this wave's loads are outstanding (n = whole steps of 1 to 4 loads).
template <int MAXN>
__device__ __forceinline__ void gemm_wait_outstanding(int n) { gemm_wait_at_most<MAXN>(n); }

// LDS read issued as inline assembly so that the wait for it can be placed by hand: the
// compiler's own placement waits for every outstanding LDS read, also the ones issued ahead
// for the next half step.  The result is valid only after gemm_wait_frag<>().
template <int OFFSET>
__device__ __forceinline__ u32x4 gemm_lds_read16(uint32_t addr) {
  u32x4 r;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFFSET));
  return r;
}

typedef __attribute__((ext_vector_type(4))) int i32x4;

// A loop whose index is a compile-time constant in every iteration: accumulator registers can
// only be named by constants, and an ordinary loop this large is not always unrolled.
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// the largest float below x (x itself for -inf and NaN): z > float_pred(x)  <=>  z >= x
__device__ __forceinline__ float float_pred(float x) {
  const uint32_t u = __float_as_uint(x);
  if (x > 0.f) return __uint_as_float(u - 1u);
  if (x == 0.f) return __uint_as_float(0x80000001u);
  if (x < 0.f && x > -INFINITY) return __uint_as_float(u + 1u);
  return x;
}

// (max, sum of exp(z - max)) of two parts of a row, merged
__device__ __forceinline__ void lse_merge(float &m, float &s, float m2, float s2) {
  const float mm = m > m2 ? m : m2;
  s = (m == -INFINITY ? 0.f : s * expf(m - mm)) + (m2 == -INFINITY ? 0.f : s2 * expf(m2 - mm));
  m = mm;
}

// ---- epilogues over whole rows, for the tiles of few score rows (the fp32 tiles and the bf16 tile
//      of few rows): the scores of the tile, rows x 128 columns, pass through LDS.
//   top-k: a wave takes a child (every eighth node) against the 128 scores of its parent's row, four
//     children's scores in flight.  The nodes' rows, tokens and own scores, one node per lane, are fetched
//     while the first operands are on their way (of listed nodes, see NodeRange, behind the products).
//   probability: a wave takes a row (every eighth).
// The loops are not unrolled over the rows: this code runs once per tile, and instructions cost their
// fetch.  As an unrolled loop over up to 16 rows per wave, with the children of each in registers of its own, it
// took 8 us at 88 rows with 248 children, and its tables 4 us in front of the first load.  Pruning call, us: 5 ragged
// trees of up to 70 nodes x 2304 x 8192 52.4 -> 45.9, 9 x 31 x 3232 x 16001 72.1 -> 64.4, 1 x 64 x 4096 x 32000 71.7 ->
// 69.0, fp32 2 x 32 x 1024 x 32000 58.3 -> 56.8.
constexpr int kRowsCols = 128;

// Where the nodes come from: the slots of the sequences that the tile's rows belong to, if these are one chunk; else
// the list of the rows' children, whose entries are fetched in front, and what they name behind the products (in
// slots that are mostly empty most chunks held nothing: a call of 128 trees of 2 nodes in slots of 128, x 1024 x 8192, took
// 71 us, 39 from the list).
constexpr int kChunkNodes = kGemmWaves * kWave;
struct NodeChunk {  // one node per lane
  int node, row, tok;
  float own;
};
struct NodeRange {  // slots, or positions in child_list
  int first, end, T;  // T: entries of a sequence (list: as if there were eight)
  bool listed;
};

__device__ __forceinline__ void load_values(NodeChunk &c, const HeadTables &tb) {
  const int at = c.node < 0 ? 0 : c.node;  // no node: as the first root, which has no parent either
  c.row = tb.node_row[at];
  c.tok = tb.token[at];
  c.own = tb.own[at];
}

// The lane's place in a chunk: eight neighbours go to eight waves, node i of sequence b to wave i + b + b / 8 (for the sequence
// of the first of the eight), so that the nodes of a tree and the same nodes of many trees are spread evenly: 64 trees of 2
// nodes in slots of 8, x 256 x 16384, 35 us for the call with wave i + 8 b, 25 so.
__device__ __forceinline__ int chunk_place(int T, int wave, int lane) {
  static_assert(kGemmWaves == 8, "eight neighbours, eight waves");
  const int b = (int)(((float)(8 * lane) + .5f) * __builtin_amdgcn_rcpf((float)T));
  return 8 * lane + ((wave - b * (1 - T) - (b >> 3)) & 7);
}

// the lane's node of the chunk that starts at x0; past the end the first one of the range
__device__ __forceinline__ int chunk_node(const NodeRange &r, int x0, int wave, int lane, const HeadTables &tb) {
  const int x = x0 + chunk_place(r.T, wave, lane), at = x < r.end ? x : r.first;
  return r.listed ? tb.child_list[at] : at;
}

// the nodes whose parents have (slots: may have) score rows of m0 .. m1 - 1
__device__ __forceinline__ NodeRange nodes_of_rows(int m0, int m1, int m_total, const HeadTables &tb) {
  NodeRange r = {0, tb.cnt_stride, tb.T_max, false};
  if (r.end > kChunkNodes) {
    if (m0 > 0) r.first = tb.row_src[m0] / tb.T_max * tb.T_max;
    if (m1 < m_total) r.end = tb.row_src[m1 - 1] / tb.T_max * tb.T_max + tb.T_max;
    r.listed = r.end - r.first > kChunkNodes;
  }
  if (r.listed) {
    r.T = 8;
    r.first = tb.row_info[2 * m0];
    r.end = tb.row_info[2 * m1 - 2] + tb.row_info[2 * m1 - 1];
  }
  return r;
}

// rows m0 .. m1 - 1 of the tile lie in s_z from its start
template <int KIND>
__device__ __forceinline__ void rows_epilogue(NodeChunk nodes, const NodeRange &range, const float *s_z, int wave, int lane,
                                              int m0, int m1, int v0, int vocab, int n_tile, const HeadTables &tb) {
  constexpr int kX = kRowsCols / kWave;
  if (KIND == 0) {
    int32_t *dst = tb.cnt_part + (size_t)n_tile * tb.cnt_stride;
    for (int x0 = range.first;;) {
      const bool mine = x0 + chunk_place(range.T, wave, lane) < range.end && nodes.row >= m0 && nodes.row < m1;
      uint64_t rest = __builtin_amdgcn_ballot_w64(mine);
      int count = 0;
      constexpr int N = 4;  // children at a time; past the last one the same once more
      while (rest) {
        int src[N], t[N];
        float zo[N], z[N][kX];
        uint64_t cur = rest;
#pragma unroll
        for (int j = 0; j < N; ++j) {
          src[j] = __builtin_ctzll(cur);
          rest = cur & (cur - 1);
          cur = rest ? rest : cur;
          const int row = __builtin_amdgcn_readlane(nodes.row, src[j]) - m0;
          t[j] = __builtin_amdgcn_readlane(nodes.tok, src[j]);
          zo[j] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(nodes.own), src[j]));
#pragma unroll
          for (int x = 0; x < kX; ++x) z[j][x] = s_z[row * kRowsCols + kWave * x + lane];
        }
#pragma unroll
        for (int j = 0; j < N; ++j) {
          int c = 0;
#pragma unroll
          for (int x = 0; x < kX; ++x) {
            const int v = v0 + kWave * x + lane;  // the token's own column and columns past the vocabulary never count
            c += __popcll(__builtin_amdgcn_ballot_w64(v < vocab && v != t[j] && (z[j][x] > zo[j] || (z[j][x] == zo[j] && v < t[j]))));
          }
          count = lane == src[j] ? c : count;
        }
      }
      if (mine) dst[nodes.node] = count;
      x0 += kChunkNodes;
      if (__builtin_expect(x0 >= range.end, 1)) break;
      nodes.node = chunk_node(range, x0, wave, lane, tb);
      load_values(nodes, tb);
    }
  } else {
#pragma unroll 1
    for (int m = m0 + wave; m < m1; m += kGemmWaves) {
      // columns past the vocabulary add nothing to a sum of exponentials
      float z[kX], mx = -INFINITY;
#pragma unroll
      for (int x = 0; x < kX; ++x) {
        z[x] = v0 + kWave * x + lane < vocab ? s_z[(m - m0) * kRowsCols + kWave * x + lane] : -INFINITY;
        mx = fmaxf(mx, z[x]);
      }
      mx = wave_reduce_max(mx);
      float sum = 0.f;
#pragma unroll
      for (int x = 0; x < kX; ++x) sum += (v0 + kWave * x + lane < vocab && mx != -INFINITY) ? expf(z[x] - mx) : 0.f;
      sum = wave_reduce_sum(sum);
      if (lane == 0) {
        float *dst = tb.lse_part + ((size_t)m * tb.parts + n_tile) * 2;
        dst[0] = mx;
        dst[1] = sum;
      }
    }
  }
}

// ------------------------------------------------------------------------------------
// Few score rows (at most 192 in the whole batch, see head_plan: a small batch or small trees).  The
// scoring kernel is then a stream of the weight matrix through the compute units, and a step
// (a barrier, fragment reads whose latency a handful of matrix instructions cannot hide)
// costs more than its bytes.  This tile takes 64-deep steps: half as many steps for the same
// bytes, whole 128-byte lines from every row (the last step of a row of an odd number of 32s fetches
// its half twice and multiplies it once).  128 vocabulary entries x RA rows per workgroup, eight
// waves as 4 (rows) x 2 (columns) blocks of 64 x 64 where the rows exist, 32x32x16 instructions; LDS
// rows are 128 bytes, their eight 16-byte chunks XOR-swizzled with key(row) = (row >> 1) & 7 (a
// fragment read takes rows r .. r + 15 of one chunk column in one pass: two rows share a 256-byte
// bank line, eight keys spread the eight pairs).
// RA = 32, 128 or 192 rows have room.  RA = 32: a wave then has one 32-row block to multiply instead of two (pruning
// call at 22 rows x 4096 x 32000: 80 us, 83 with RA = 128; a shape for 64 rows gained nothing at 44).  RA = 192: four
// stages instead of three are 1 to 2 us slower.  Call with room for 256 rows / 192, us: 130 rows x 4096 x
// 8192 83.0 / 78.7, 160 x 4096 x 8192 84.1 / 86.0.
// The K loop runs at 5.8 TB/s of weights, read once and non-temporally (without that 6 us more); a
// ring of seven stages instead of four changes nothing, and neither does requesting 256 or 512
// bytes of a row together.  Kernel at that size: 72.8 -> 55.6 us with the row epilogue, the
// children fetched before the K loop and a tile plan without 64-bit divisions (14 -> 10 us
// outside the K loop; 72 rows: 83 -> 71 us).
// ------------------------------------------------------------------------------------
struct GemmFrag {
  u32x4 a[2], b[2];
};
// Waits until at most N LDS reads of this wave are outstanding (they return in order); the
// fragment named is the one waited for, so that its uses stay below the wait.
template <int N>
__device__ __forceinline__ void gemm_wait_frag(GemmFrag &f) {
  asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(f.a[0]), "+v"(f.a[1]), "+v"(f.b[0]), "+v"(f.b[1]) : "n"(N));
}

constexpr int kSmallBK = 64;
constexpr int kSmallMaxRows = 192;  // rows that this tile is used for at most, see head_plan
constexpr int kSmallRowBytes = kSmallBK * 2;                          // 128
constexpr int kSmallWBytes = 128 * kSmallRowBytes;                    // 16 KB of weight rows per stage

template <int KIND, int RA>
__device__ __forceinline__ void early_head_small_tile(
    int hidden, int vocab, int m_total, int v0, int n_tile,
    const uint16_t *__restrict__ hidden_states, const uint16_t *__restrict__ head_weight,
    const HeadTables &tb, unsigned char *gemm_smem) {
  constexpr int FN = 2;
  constexpr int kStages = RA == 192 ? 3 : 4, kWOffset = RA * kSmallRowBytes, kStageBytes = kWOffset + kSmallWBytes;
  static_assert(kStages * kStageBytes <= kHeadLdsBytes, "ring");
  constexpr int kALoads = RA > 64 ? RA / 64 : 1;  // 8-row groups of score rows a wave may have to fetch
  constexpr int kX = RA == 32 ? 1 : 2;         // 32-row blocks of a wave's 64 rows that exist
  typedef __attribute__((address_space(3))) void lds_void;
  typedef const __attribute__((address_space(1))) void global_void;
  const uint32_t smem_base = (uint32_t)(uintptr_t)(lds_void *)gemm_smem;
  // The thread id is made opaque: what is derived from it (addresses, row and chunk numbers)
  // is then computed here, inside the loop over tiles, and not hoisted out of that loop into
  // registers that stay occupied while the other tile shapes run.
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int l32 = lane & 31, g = lane >> 5;
  // ---- loader: a load instruction fills 8 rows of 128 bytes (1 KB).  A stage has RA / 8 such
  //      groups of score rows, fetched by wave g / kALoads, and 16 of weight rows; wave w takes
  //      groups 2w and 2w + 1 of those.  Groups of score rows wholly past the last are not fetched.
  const int ld_row = lane >> 3, ld_pos = lane & 7;
  const unsigned char *a_src[kALoads], *b_src[2];
  bool a_on[kALoads];
  // the lane's chunk lies in the second half of the 128 bytes: a half step fetches the first instead
  int a_back[kALoads], b_back[2];
  int per_step = 2;  // loads of this wave per K step
#pragma unroll
  for (int j = 0; j < kALoads; ++j) {
    const int r = 8 * (kALoads * wave + j) + ld_row;  // row of the tile = LDS row
    a_on[j] = kALoads * wave + j < RA / 8 && 8 * (kALoads * wave + j) < m_total;
    per_step += a_on[j] ? 1 : 0;
    const int m = r < m_total ? r : m_total - 1;
    const int chunk = ld_pos ^ ((r >> 1) & 7);
    a_back[j] = chunk & 4 ? 64 : 0;
    a_src[j] = reinterpret_cast<const unsigned char *>(hidden_states + (size_t)tb.row_src[m] * hidden) + (chunk << 4);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int r = 8 * (2 * wave + j) + ld_row;
    const int v = v0 + r < vocab ? v0 + r : vocab - 1;
    const int chunk = ld_pos ^ ((r >> 1) & 7);
    b_back[j] = chunk & 4 ? 64 : 0;
    b_src[j] = reinterpret_cast<const unsigned char *>(head_weight + (size_t)v * hidden) + (chunk << 4);
  }
  const bool w_on = wm * 64 < m_total;  // this wave's 64 rows hold score rows
  const int n_steps = (hidden + kSmallBK - 1) / kSmallBK;
  const bool half_end = hidden % kSmallBK != 0;  // the last step is 32 deep
  auto issue = [&](int slot, int step) {
    if (half_end && step + 1 == n_steps) {
#pragma unroll
      for (int j = 0; j < kALoads; ++j) a_src[j] -= a_back[j];
#pragma unroll
      for (int j = 0; j < 2; ++j) b_src[j] -= b_back[j];
    }
    unsigned char *dst = gemm_smem + slot * kStageBytes;
#pragma unroll
    for (int j = 0; j < kALoads; ++j) {
      if (a_on[j])
        __builtin_amdgcn_global_load_lds((global_void *)a_src[j], (lds_void *)(dst + (kALoads * wave + j) * 1024), 16, 0, 0);
      a_src[j] += kSmallRowBytes;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      __builtin_amdgcn_global_load_lds((global_void *)b_src[j], (lds_void *)(dst + kWOffset + (2 * wave + j) * 1024), 16, 0, 2 /* nt */);
      b_src[j] += kSmallRowBytes;
    }
  };

  // ---- per-lane LDS read addresses: operand row l32 of a 32-row block (the key of row + 32 is
  //      the key of the row), chunk 2 * ks + g for the K sub-step ks of 16
  uint32_t a_rd[4], b_rd[4];
  {
    const int key = (l32 >> 1) & 7;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int off = l32 * kSmallRowBytes + (((2 * ks + g) ^ key) << 4);
      a_rd[ks] = smem_base + wm * 64 * kSmallRowBytes + off;
      b_rd[ks] = smem_base + kWOffset + wn * 64 * kSmallRowBytes + off;
    }
  }
  typedef GemmFrag Frag;
  auto read = [&](Frag &f, uint32_t so, int ks) {
    const uint32_t pa = a_rd[ks] + so, pb = b_rd[ks] + so;
    f.a[0] = gemm_lds_read16<0>(pa);
    if constexpr (kX == 2) f.a[1] = gemm_lds_read16<32 * kSmallRowBytes>(pa);
    else f.a[1] = u32x4{0u, 0u, 0u, 0u};
    f.b[0] = gemm_lds_read16<0>(pb);
    f.b[1] = gemm_lds_read16<32 * kSmallRowBytes>(pb);
  };
  f32x16 acc[2][FN];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < FN; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;
  auto mma = [&](const Frag &f) {
#pragma unroll
    for (int x = 0; x < kX; ++x)
#pragma unroll
      for (int y = 0; y < FN; ++y)
        acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            __builtin_bit_cast(bf16x8, f.a[x]), __builtin_bit_cast(bf16x8, f.b[y]), acc[x][y], 0, 0, 0);
  };

  const int n_pro = n_steps < kStages ? n_steps : kStages;
  constexpr int kMaxOutstanding = (kStages - 1) * (kALoads + 2);
  int slot_ld = 0;
  NodeChunk nodes = {0, -1, 0, 0.f};
  NodeRange range = {0, tb.cnt_stride, tb.T_max, false};
  if (KIND == 0 && __builtin_expect(range.end > kChunkNodes, 0)) {
    range = nodes_of_rows(0, m_total, m_total, tb);
    nodes.node = chunk_node(range, range.first, wave, lane, tb);
  }
  for (int i = 0; i < n_pro; ++i) {
    issue(slot_ld, i);
    slot_ld = slot_ld + 1 == kStages ? 0 : slot_ld + 1;
  }
  // (loads younger than the ring's only make the counted waits below stricter)
  if (KIND == 0 && __builtin_expect(!range.listed, 1)) {
    nodes.node = chunk_node(range, 0, wave, lane, tb);
    load_values(nodes, tb);
  }
  gemm_wait_outstanding<kMaxOutstanding>((n_pro - 1) * per_step);
  __builtin_amdgcn_s_barrier();
  constexpr int kReads = kX + FN;  // LDS reads of one K sub-step
  Frag f0, f1;
  if (w_on) read(f0, 0, 0);
  uint32_t so = 0;  // byte offset of the stage being multiplied
  for (int step = 0; step < n_steps; ++step) {
    if (w_on) {
      read(f1, so, 1);
      gemm_wait_frag<kReads>(f0);  // the reads just issued fly while the MFMAs below run
      mma(f0);
      if (!half_end || step + 1 < n_steps) {
        read(f0, so, 2);
        gemm_wait_frag<kReads>(f1);
        mma(f1);
        read(f1, so, 3);
        gemm_wait_frag<kReads>(f0);
        mma(f0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (w_on) gemm_wait_frag<0>(f1);  // this wave is done with the slot of this step
    if (step + 1 < n_steps) {
      const int issued_after = n_steps - 2 - step;  // steps after the next that have been issued, if not more than fit
      if (issued_after >= kStages - 2) {
        static_for<kALoads + 1>([&](auto a) {  // 2 .. kALoads + 2 loads per step
          if (per_step == 2 + a) gemm_wait_vmem<(2 + a) * (kStages - 2)>();
        });
      } else {
        gemm_wait_outstanding<kMaxOutstanding>(issued_after * per_step);
      }
      __builtin_amdgcn_s_barrier();  // it is visible; every wave is done with this step's slot
      if (step + kStages < n_steps) {
        issue(slot_ld, step + kStages);  // into the slot of this step
        slot_ld = slot_ld + 1 == kStages ? 0 : slot_ld + 1;
      }
      so = so + kStageBytes == kStages * kStageBytes ? 0 : so + kStageBytes;
      if (w_on) read(f0, so, 0);
    }
    if (w_on) mma(f1);
    __builtin_amdgcn_sched_barrier(0);
  }
  mfma_settle();
  if (KIND == 0 && __builtin_expect(range.listed, 0)) load_values(nodes, tb);
  // element (row, col) of a 32 x 32 tile: lane col + 32 * (row / 4 % 2), register 4 * (row / 8) + row % 4
  float *s_z = reinterpret_cast<float *>(gemm_smem);
  __syncthreads();  // every wave is done with the ring
  if (w_on) {
#pragma unroll
    for (int x = 0; x < kX; ++x)
#pragma unroll
      for (int y = 0; y < FN; ++y)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          s_z[(wm * 64 + 32 * x + 8 * (r >> 2) + 4 * g + (r & 3)) * kRowsCols + wn * 64 + 32 * y + l32] = acc[x][y][r];
  }
  __syncthreads();
  rows_epilogue<KIND>(nodes, range, s_z, wave, lane, 0, m_total, v0, vocab, n_tile, tb);
  __syncthreads();  // the next tile's loads reuse this memory
}


#include "early_head_tall.h"

// Which tile a call uses: decided on the device by every workgroup (and by the kernels
// that read the per-tile results) from the row count, which the host never sees.
//   - At most 128 rows: the tile of few rows, one row tile, 128 entries wide (32000 entries: 250
//     workgroups).
//   - 129 to 192 rows: the same where one round of it covers the vocabulary and rows have 64 elements
//     for each score row beyond 112.  Pruning call, us, few rows / best other, at 8192 and 32000 entries on the
//     two sides of that line: 130 rows x 2048 53.8 / 60.2, 59.8 / 60.3, x 1024 40.6 / 41.9, 43.1 / 45.1; 144 x 2048 56.3 / 60.1, 61.5 /
//     61.2, x 1024 42.6 / 42.4, 45.1 / 46.4; 160 x 3072 72.1 / 76.1, 75.3 / 76.4, x 2048 58.2 / 61.2, 64.0 / 61.6; 176 x 4096
//     86.7 / 90.2, 95.3 / 97.8, x 2048 59.0 / 60.9, 64.8 / 64.5; 192 x 5120 102.6 / 105.4, 108.3 / 117.6, x 4096 (24000 entries) 94.0 /
//     90.9; in two rounds 176 x 4096 x 64000 205 / 176, 132 x 3584 x 152064 391 / 294.
//   - More: the shape of the least cost = rounds of workgroups over the compute units x
//     (7 + 4 * mi).  Pruning call, us, one round at 4096 x 32000 (43 of it beside the kernel): 122 for 160 x 256,
//     134 for 192, 146 for 224, 158 for 256, 170 for 288, 183 for 320, 200 for 352 x 256.  Tiles of 192 columns
//     were no better, of 128 columns worse.
struct HeadPlan {
  int mi;  // tile of 32*mi x 256; 0: the tile of few rows
  int m_tiles, n_tiles;
};

constexpr int kTallMaxMI = 11;
#define PROPD_TALL_SHAPES(X) X(11) X(10) X(9) X(8) X(7) X(6) X(5)  // the larger first: of equal cost the first is taken

__host__ __device__ inline HeadPlan head_plan(int m_total, int hidden, int vocab, int cus, int force, int max_mi) {
  const HeadPlan few = {0, 1, (vocab - 1) / 128 + 1};
  if (force == 0 && (m_total <= 128 || (m_total <= kSmallMaxRows && few.n_tiles <= cus && hidden >= 64 * (m_total - 112))))
    return few;
  const int rows = m_total > 0 ? m_total : 1, nt = (vocab - 1) / 256 + 1;
  const float inv = 1.f / (float)cus;  // instead of a 64-bit division per shape in front of the first load
  auto rounds = [&](long long tiles) -> long long {
    if (tiles >= (1ll << 24)) return (tiles + cus - 1) / cus;
    const int t = (int)tiles;  // by the reciprocal, off by one at most
    int q = (int)((float)t * inv);
    q -= q * cus > t ? 1 : 0;
    q += (q + 1) * cus <= t ? 1 : 0;  // q = t / cus
    return q * cus < t ? q + 1 : q;
  };
  HeadPlan pl = {};
  long long best = -1;
  auto take = [&](int mi) {
    const int mt = (rows - 1) / (32 * mi) + 1;
    const long long cost = rounds((long long)mt * nt) * (7 + 4 * mi);
    if (best >= 0 && cost >= best) return;
    best = cost;
    pl = HeadPlan{mi, mt, nt};
  };
#define X(MI) \
  if (MI <= max_mi && (force == 0 || (force == 1 && MI == 8) || (force == 2 && MI == (max_mi < 11 ? max_mi : 11)))) take(MI);
  PROPD_TALL_SHAPES(X)
#undef X
  return pl;
}

// Persistent over the tiles: tile -> (xcd, slot) as described above, a workgroup takes tiles
// blockIdx.x, blockIdx.x + gridDim.x, ... (the grid is a multiple of the XCD count).
template <int KIND>
__global__ __launch_bounds__(kGemmThreads, 1) void early_head_bf16_kernel(
    int hidden, int vocab, int B, int cus, int force, int max_mi, const uint16_t *__restrict__ hidden_states,
    const uint16_t *__restrict__ head_weight, HeadTables tb) {
  const int m_total = tb.row_base[B];
  if (m_total <= 0) return;
  const HeadPlan pl = head_plan(m_total, hidden, vocab, cus, force, max_mi);
  const int m_tiles = pl.m_tiles, n_tiles = pl.n_tiles;
  if (blockIdx.x == 0 && threadIdx.x == 0) *tb.n_tiles = n_tiles;
  const long long total = (long long)kXcds * ((n_tiles + kXcds - 1) / kXcds) * m_tiles;
  extern __shared__ __attribute__((aligned(1024))) unsigned char gemm_smem[];
  for (long long tile = blockIdx.x; tile < total; tile += gridDim.x) {
    const int xcd = (int)(tile % kXcds);
    const long long slot = tile / kXcds;
    const int group = slot < (1ll << 31) ? (int)((uint32_t)slot / (uint32_t)m_tiles) : (int)(slot / m_tiles);
    const int n_tile = group * kXcds + xcd;
    if (n_tile >= n_tiles) continue;
    const int m_tile = (int)(slot - (long long)group * m_tiles);
    // a wave may be here while another still reads the last stage of the tile before this one
    if (tile != blockIdx.x) __syncthreads();
    if (pl.mi == 0) {
      const int v0 = n_tile * 128;
      if (m_total <= 32)
        early_head_small_tile<KIND, 32>(hidden, vocab, m_total, v0, n_tile, hidden_states, head_weight, tb, gemm_smem);
      else if (m_total <= 128)
        early_head_small_tile<KIND, 128>(hidden, vocab, m_total, v0, n_tile, hidden_states, head_weight, tb, gemm_smem);
      else
        early_head_small_tile<KIND, 192>(hidden, vocab, m_total, v0, n_tile, hidden_states, head_weight, tb, gemm_smem);
      continue;
    }
#define X(MI)                                                                                              \
  if (pl.mi == MI)                                                                                         \
    early_head_tall_tile<MI, KIND>(hidden, vocab, m_total, m_tile * 32 * MI, n_tile * 256, n_tile,          \
                                   hidden_states, head_weight, tb, gemm_smem);
    PROPD_TALL_SHAPES(X)
#undef X
  }
}

#include "early_head_f32.h"

// which criterion decides (Section 4.1, "Pruning Criterion")
struct Criterion {
  int kind;             // 0 top-k, 1 probability threshold, 2 probability rank
  int top_k;            // kind 0
  float log_threshold;  // kind 1
  int keep_count;       // kind 2
  float *log_marginal;  // kinds 1, 2: optional output
};

// ------------------------------------------------------------------------------------
// the decision, branch elimination, compaction, mask subsampling, payload rows of survivors
// ------------------------------------------------------------------------------------
struct PayloadArgs {
  const char *src[PROPD_MAX_PAYLOADS];
  char *dst[PROPD_MAX_PAYLOADS];
  unsigned long long per_row[PROPD_MAX_PAYLOADS];  // pieces of a row: of 16 bytes (vec16), or bytes
  unsigned outer[PROPD_MAX_PAYLOADS];
  long long stride_b[PROPD_MAX_PAYLOADS], stride_outer[PROPD_MAX_PAYLOADS], stride_t[PROPD_MAX_PAYLOADS];
  int vec16[PROPD_MAX_PAYLOADS];  // rows, strides and bases are all 16-byte multiples
  int n;
};

struct FinishArgs {
  int B, T_max, vocab, bf16, scored, parts, lines, slices;  // slices: workgroups per sequence, in x if there are several
  unsigned long long inv_slices;  // 2^64 / slices
  Criterion crit;
  const int32_t *n_nodes, *parent, *token, *depth;
  const uint64_t *anc;
  const int32_t *row_base, *row_info, *child_list, *cnt_part;
  const float *own, *lse_part;
  int32_t *notes;
  uint64_t *keep_bits;
  int32_t *new_index, *orig_index, *n_kept, *cu_nodes, *out_n_nodes, *out_parent, *out_token, *out_depth;
  uint64_t *out_anc;
  int32_t *rank_out;
  PayloadArgs pa;
};

constexpr int kFinishSplit = 4;  // threads that add up one node's per-tile counts
constexpr int kFinishThreads = PROPD_MAX_TREE * kFinishSplit;
constexpr int kRowLanes = 8;     // threads that take the partial sums of one score row
constexpr int kGatherItems = 4;  // pieces a thread has in flight

// Workgroups per sequence: at most one for 2048 pieces of payload (of which typically a quarter
// to a half survive) and one per compute unit in the whole batch, since each works out its sequence's decision; two
// per compute unit for large payloads, and no fewer than three for two units.  Pruning call, us, at one / two per compute
// unit: 5 sequences x 32 heads x 70 nodes (545 blocks of 2048) 52.5 / 54.1 (four: 58.0), 32 x 128 nodes, hidden only (1024)
// 232.6 / 235.0, 27 x 16 x 128 (1863) 144.8 / 143.1, 16 x 40 x 128 (2560) 235.0 / 232.4.  Rows of 41 KB per node, by
// workgroups in the batch: 129 sequences of 128 nodes 258 163, 387 143, 516 155; 65 260 87, 455 81, 520 86; 257 of 64 257 171, 514
// 143.
static int finish_slices(int B, long long blocks, int cus) {
  const bool large = blocks >= 6ll * cus;
  long long slices = (large ? 2ll * cus : cus) / B;
  if (large && 2 * slices * B < 3ll * cus) ++slices;
  if (slices > (blocks + B - 1) / B) slices = (blocks + B - 1) / B;
  return (int)(slices < 1 ? 1 : (slices > 1024 ? 1024 : slices));
}

// The pieces [lo, hi) of one payload of one sequence, counted as (outer, survivor, piece of its row), in
// chunks of kGatherItems per thread, all loads of a chunk in flight before its first store.  A thread divides
// once; from piece to piece it adds the (outer, survivor, piece) that the distance comes to.
template <typename N, typename V>
__device__ __forceinline__ void gather_pieces(const char *src, char *dst, long long stride_outer, long long stride_t,
                                              N lo, N hi, N kept, N per_row, const int *s_orig) {
  const N per_outer = kept * per_row;
  const N step_o = (N)kFinishThreads / per_outer, step_r = (N)kFinishThreads - step_o * per_outer;
  const N step_j = step_r / per_row, step_c = step_r - step_j * per_row;
  const N first = lo + (N)threadIdx.x;
  N o = first / per_outer, j, c;
  {
    const N r = first - o * per_outer;
    j = r / per_row;
    c = r - j * per_row;
  }
  for (N x0 = first; x0 < hi; x0 += (N)(kGatherItems * kFinishThreads)) {
    V v[kGatherItems];
    long long to[kGatherItems];
#pragma unroll
    for (int k = 0; k < kGatherItems; ++k) {
      const bool in = x0 + (N)(k * kFinishThreads) < hi;  // past the end: the first piece of the chunk once more, not stored
      const long long at = (long long)o * stride_outer + (long long)c * (long long)sizeof(V);
      to[k] = k == 0 || in ? at + (long long)j * stride_t : to[0];
      const char *from = src + at + (long long)s_orig[(int)j] * stride_t;
      from = k == 0 || in ? from : src + (long long)s_orig[0] * stride_t;
      v[k] = *reinterpret_cast<const V *>(from);
      c += step_c;
      N carry = c >= per_row ? 1 : 0;
      c -= carry ? per_row : 0;
      j += step_j + carry;
      carry = j >= kept ? 1 : 0;
      j -= carry ? kept : 0;
      o += step_o + carry;
    }
#pragma unroll
    for (int k = 0; k < kGatherItems; ++k)
      if (x0 + (N)(k * kFinishThreads) < hi) *reinterpret_cast<V *>(dst + to[k]) = v[k];
  }
}

// Every workgroup of a sequence works out its decision for itself, four threads per node for the counts and
// one for the rest; the first one writes it down, and all share the payload rows.
//   top-k: a node fails when `top_k` or more scores of its parent's row beat its token's, or
//     its token id lies outside the vocabulary.
//   probability: the log marginal of a node's sequence is the sum of log q over its root path
//     (the cached ancestor set, root excluded, in root-to-node order), log q = own score - log sum exp of
//     the parent's row; it fails when the marginal is below the threshold, or when `keep_count` or
//     more sequences of the tree are more probable (equal marginals: the lower node index counts
//     as more probable); a marginal of zero probability always fails.
// The kernel is a chain of dependent reads (counts, rows), not bytes: as two kernels, three for the probability
// criterion, it had a launch and a first read more each, and the origins of the rows went through memory.  Pruning
// call, us: 16 sequences x 40 heads x 128 nodes 236 -> 232, probability criterion at 32 ragged trees 240 -> 233, 31 x 40 x 52
// 118.5 -> 112, 1 x 64 nodes x 4096 76.1 -> 75.0, fp32 1 x 32 x 389 x 1011 28.2 -> 25.0.
__global__ __launch_bounds__(kFinishThreads) void prune_finish_kernel(FinishArgs a) {
  const int b = (int)(a.slices > 1 ? blockIdx.y : blockIdx.x), slice = (int)(a.slices > 1 ? blockIdx.x : 0);
  const int i = threadIdx.x & (PROPD_MAX_TREE - 1), q = threadIdx.x / PROPD_MAX_TREE;
  const int T_max = a.T_max;
  const size_t base = (size_t)b * T_max;
  // Everything this thread reads is requested before the first value is used: the tree size,
  // the tile count and the node's own words do not wait for each other.  Slots past the tree
  // are read too (they exist) and dropped.
  const bool slot = i < T_max, worker = q == 0;
  const int T_raw = a.n_nodes[b];
  uint64_t a_lo = 0, a_hi = 0;
  int my_token = -1, my_depth = -1, my_parent = -1;
  if (worker && slot) {
    a_lo = a.anc[(base + i) * 2];
    a_hi = a.anc[(base + i) * 2 + 1];
    my_token = a.token[base + i];
    my_depth = a.depth[base + i];
    my_parent = a.parent[base + i];
  }
  __shared__ uint64_t s_fail[2], s_keep[2];
  __shared__ float s_q[PROPD_MAX_TREE], s_lm[PROPD_MAX_TREE];
  __shared__ int s_sum[kFinishSplit][PROPD_MAX_TREE], s_orig[PROPD_MAX_TREE], s_last;

  int m_total = 0, n_tiles = 0;
  if (a.scored) {
    m_total = a.row_base[a.B];
    // left by the scoring kernel (which has nothing to do without rows): worked out here it stood
    // 2 us in front of the first count
    const int left = a.notes[kNoteTiles];
    if (m_total > 0) n_tiles = a.bf16 ? left : f32_plan(m_total, a.vocab).n_tiles;
  }
  if (a.crit.kind == 0) {
    // rank = the counts of all column tiles (none where nothing was scored)
    int sum = 0;
    if (slot && i > 0) {
      const int32_t *src = a.cnt_part + base + i;
      const size_t stride = (size_t)a.B * T_max;
      constexpr int kInFlight = 32;
      for (int t0 = q; t0 < n_tiles; t0 += kFinishSplit * kInFlight) {
        int v[kInFlight];
#pragma unroll
        for (int k = 0; k < kInFlight; ++k) {
          const int t = t0 + kFinishSplit * k;
          v[k] = t < n_tiles ? src[(size_t)t * stride] : 0;
        }
#pragma unroll
        for (int k = 0; k < kInFlight; ++k) sum += v[k];
      }
    }
    s_sum[q][i] = sum;
  } else {
    // log q of the children of every score row: the log-sum-exp of the row from its tile partials, eight
    // threads per row (the largest maximum first, then one exponential per partial)
    if (worker) s_q[i] = 0.f;
    const int m0 = a.row_base[b], m1 = a.row_base[b + 1];
    const int part = threadIdx.x & (kRowLanes - 1);
    __syncthreads();
    for (int mb = m0; mb < m1; mb += kFinishThreads / kRowLanes) {
      const int m = mb + (int)threadIdx.x / kRowLanes;
      const bool row = m < m1;
      const float *src = a.lse_part + (size_t)(row ? m : m0) * a.parts * 2;
      const int pos = a.row_info[2 * (row ? m : m0)], cc = row ? a.row_info[2 * m + 1] : 0;
      float mx = -INFINITY, sum = 0.f;
      constexpr int kInFlight = 16;
      for (int t0 = part; t0 < n_tiles; t0 += kRowLanes * kInFlight) {
        float pm[kInFlight], ps[kInFlight], top = mx;
#pragma unroll
        for (int k = 0; k < kInFlight; ++k) {
          const int t = t0 + kRowLanes * k, tt = t < n_tiles ? t : t0;
          pm[k] = src[2 * tt];
          ps[k] = src[2 * tt + 1];
        }
#pragma unroll
        for (int k = 0; k < kInFlight; ++k) top = fmaxf(top, pm[k]);  // past the end: the first once more
        sum = mx == -INFINITY ? 0.f : sum * expf(mx - top);
#pragma unroll
        for (int k = 0; k < kInFlight; ++k)
          if (t0 + kRowLanes * k < n_tiles && pm[k] != -INFINITY) sum += ps[k] * expf(pm[k] - top);
        mx = top;
      }
#pragma unroll
      for (int o = kRowLanes / 2; o > 0; o >>= 1) {
        const float m2 = __shfl_xor(mx, o, kWave), s2 = __shfl_xor(sum, o, kWave);
        lse_merge(mx, sum, m2, s2);
      }
      const float lse = mx + logf(sum);
      for (int e = part; e < cc; e += kRowLanes) {
        const int c = a.child_list[pos + e];
        const int t = a.token[c], nd = c - (int)base;
        // a token id outside the vocabulary has probability 0
        if (nd >= 0 && nd < T_max) s_q[nd] = (t >= 0 && t < a.vocab) ? a.own[c] - lse : -INFINITY;
      }
    }
  }
  const int T = clamp_tree(T_raw, T_max);
  const bool valid = i < T;
  if (!valid) {
    a_lo = a_hi = 0;
    my_token = -1;
  }
  __syncthreads();
  // one thread per node does the work; the others only meet it at the barriers
  bool fail = false;
  if (a.crit.kind == 0) {
    if (worker) {
      int my_rank = -1;
      if (valid) {
        my_rank = 0;
#pragma unroll
        for (int k = 0; k < kFinishSplit; ++k) my_rank += s_sum[k][i];
        // a token id outside the vocabulary can be in no top-k list
        if (i > 0 && (my_token < 0 || my_token >= a.vocab)) my_rank = a.vocab;
      }
      if (a.rank_out && slot && slice == 0) a.rank_out[base + i] = my_rank;
      fail = valid && i > 0 && my_rank >= a.crit.top_k;
    }
  } else {
    float lm = 0.f;
    if (worker && valid && i > 0) {
      uint64_t lo = a_lo & ~1ull, hi = a_hi;
      while (lo) {
        lm += s_q[__ffsll((long long)lo) - 1];
        lo &= lo - 1;
      }
      while (hi) {
        lm += s_q[64 + __ffsll((long long)hi) - 1];
        hi &= hi - 1;
      }
    }
    if (worker) s_lm[i] = valid ? lm : -INFINITY;
    __syncthreads();
    if (worker && valid && i > 0) {
      if (a.crit.kind == 1) {
        fail = !(lm >= a.crit.log_threshold);
      } else {
        int ahead = 0;
        for (int j = 0; j < T; ++j) ahead += (s_lm[j] > lm) || (s_lm[j] == lm && j < i);
        fail = ahead >= a.crit.keep_count;
      }
      fail = fail || !(lm > -INFINITY);
    }
    if (worker && a.crit.log_marginal && slot && slice == 0) a.crit.log_marginal[base + i] = valid ? lm : 0.f;
  }
  if (worker) {
    const uint64_t fb = __ballot(fail);
    if ((i & 63) == 0) s_fail[i >> 6] = fb;
  }
  __syncthreads();
  // a node goes as soon as any node of its root path failed
  const bool keep = worker && valid && ((a_lo & s_fail[0]) | (a_hi & s_fail[1])) == 0;
  if (worker) {
    const uint64_t kb = __ballot(keep);
    if ((i & 63) == 0) s_keep[i >> 6] = kb;
  }
  __syncthreads();
  const uint64_t k_lo = s_keep[0], k_hi = s_keep[1];
  const int kept = __popcll(k_lo) + __popcll(k_hi);
  const int ni = keep ? popc128_below(k_lo, k_hi, i) : -1;
  if (keep) s_orig[ni] = i;
  if (worker && slice == 0) {
    if (slot) a.new_index[base + i] = ni;
    if (keep) {
      a.orig_index[base + ni] = i;
      a.out_token[base + ni] = my_token;
      a.out_depth[base + ni] = my_depth;
      const int p = i == 0 ? -1 : my_parent;
      a.out_parent[base + ni] = (p >= 0 && p < T) ? popc128_below(k_lo, k_hi, p) : -1;
      // subsample the cached mask: keep the columns of survivors, renumbered
      uint64_t r_lo = 0, r_hi = 0;
      uint64_t w = a_lo & k_lo;
      while (w) {
        const int j = __ffsll((long long)w) - 1;
        w &= w - 1;
        const int pos = popc128_below(k_lo, k_hi, j);
        if (pos < 64) r_lo |= 1ull << pos; else r_hi |= 1ull << (pos - 64);
      }
      w = a_hi & k_hi;
      while (w) {
        const int j = 64 + __ffsll((long long)w) - 1;
        w &= w - 1;
        const int pos = popc128_below(k_lo, k_hi, j);
        if (pos < 64) r_lo |= 1ull << pos; else r_hi |= 1ull << (pos - 64);
      }
      a.out_anc[(base + ni) * 2] = r_lo;
      a.out_anc[(base + ni) * 2 + 1] = r_hi;
    }
    if (i >= kept && slot) {
      a.orig_index[base + i] = -1;
      a.out_token[base + i] = -1;
      a.out_depth[base + i] = -1;
      a.out_parent[base + i] = -1;
      a.out_anc[(base + i) * 2] = 0;
      a.out_anc[(base + i) * 2 + 1] = 0;
    }
    if (i == 0) {
      a.keep_bits[2 * b] = k_lo;
      a.keep_bits[2 * b + 1] = k_hi;
      __hip_atomic_store(a.n_kept + b, kept, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (a.B > 1 && a.scored) {
        // The prefix sum of the survivor counts is left to the workgroup that finds all other sequences arrived;
        // nobody waits, and the counter was cleared by the preparation.  Count and arrival go through to
        // where all workgroups see them, in this order (a fence would also write the caches back).
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        auto arrive = [&](int word, int all) {
          return __hip_atomic_fetch_add(a.notes + word, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == all - 1;
        };
        if (a.lines == 0) {
          s_last = arrive(kNoteArrived, a.B);
        } else {  // the last one on a line arrives for it on the first
          const int l = b & (a.lines - 1);
          s_last = arrive((l + 1) * kNoteLine, (a.B - l + a.lines - 1) >> __builtin_ctz(a.lines)) && arrive(kNoteArrived, a.lines);
        }
      }
      if (a.out_n_nodes) a.out_n_nodes[b] = kept;
      if (a.B == 1) {
        a.cu_nodes[0] = 0;
        a.cu_nodes[1] = kept;
      }
    }
  }
  __syncthreads();  // s_orig
  // ---- payload rows.  The counted pieces of all payloads are one list, of which a slice takes an equal part.
  {
    unsigned long long total = 0, start = 0;
    for (int p = 0; p < a.pa.n; ++p) total += (unsigned long long)a.pa.outer[p] * (unsigned)kept * a.pa.per_row[p];
    const unsigned long long share = a.slices > 1 ? __umul64hi(total, a.inv_slices) + 1 : total;  // no less than total / slices
    const unsigned long long lo = share * (unsigned)slice, hi = lo + share < total ? lo + share : total;
    for (int p = 0; p < a.pa.n; ++p) {
      const unsigned long long items = (unsigned long long)a.pa.outer[p] * (unsigned)kept * a.pa.per_row[p];
      const unsigned long long from = lo > start ? lo - start : 0, to = hi > start ? (hi - start < items ? hi - start : items) : 0;
      start += items;
      if (from >= to) continue;  // uniform
      const char *src = a.pa.src[p] + b * a.pa.stride_b[p];
      char *dst = a.pa.dst[p] + b * a.pa.stride_b[p];
      const long long so = a.pa.stride_outer[p], st = a.pa.stride_t[p];
      if (items < (1ull << 31)) {
        if (a.pa.vec16[p])
          gather_pieces<uint32_t, u32x4>(src, dst, so, st, (uint32_t)from, (uint32_t)to, (uint32_t)kept, (uint32_t)a.pa.per_row[p], s_orig);
        else
          gather_pieces<uint32_t, uint8_t>(src, dst, so, st, (uint32_t)from, (uint32_t)to, (uint32_t)kept, (uint32_t)a.pa.per_row[p], s_orig);
      } else {
        if (a.pa.vec16[p])
          gather_pieces<uint64_t, u32x4>(src, dst, so, st, from, to, (uint64_t)kept, (uint64_t)a.pa.per_row[p], s_orig);
        else
          gather_pieces<uint64_t, uint8_t>(src, dst, so, st, from, to, (uint64_t)kept, (uint64_t)a.pa.per_row[p], s_orig);
      }
    }
  }
  if (slice != 0 || a.B == 1 || !a.scored || !s_last) return;  // uniform
  // exclusive scan, a run of sequences per thread
  __shared__ int s_wave[kFinishThreads / kWave];
  const int per = (a.B + kFinishThreads - 1) / kFinishThreads, x_lo = (int)threadIdx.x * per;
  const int x_hi = x_lo + per < a.B ? x_lo + per : a.B;
  int sum = 0;
  for (int x = x_lo; x < x_hi; ++x) sum += __hip_atomic_load(a.n_kept + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  int incl = sum;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int up = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += up;
  }
  if (lane == kWave - 1) s_wave[wv] = incl;
  __syncthreads();
  int run = incl - sum;
  for (int w = 0; w < wv; ++w) run += s_wave[w];
  for (int x = x_lo; x < x_hi; ++x) {
    a.cu_nodes[x] = run;
    run += __hip_atomic_load(a.n_kept + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (threadIdx.x == kFinishThreads - 1) a.cu_nodes[a.B] = run;  // its run of sequences is the last, or empty
}

}  // namespace propd

static int prune_compute_units() {
  static const int cus = [] {
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0)
      return prop.multiProcessorCount;
    return 256;
  }();
  return cus;
}

static propd_status prune_impl(
    const propd::Criterion &crit, const propd_tree *tree, propd_dtype dt, int32_t hidden, int32_t vocab,
    const void *hidden_states, const void *head_weight, uint64_t *keep_bits, int32_t *new_index,
    int32_t *orig_index, int32_t *n_kept, int32_t *cu_nodes, const propd_tree_out *tree_out,
    int32_t *rank_out, int32_t n_payloads, const propd_payload *payloads, void *workspace,
    size_t workspace_bytes, void *hip_stream) {
  using namespace propd;
  if (!tree || tree->B < 1 || tree->T_max < 1 || tree->T_max > PROPD_MAX_TREE || hidden < 1 ||
      vocab < 1 || (crit.kind == 0 && crit.top_k < 1))
    return PROPD_ERR_INVALID_ARG;
  if (!tree->n_nodes || !tree->parent || !tree->token || !tree->depth || !tree->anc ||
      !hidden_states || !head_weight || !keep_bits || !new_index || !orig_index || !n_kept ||
      !cu_nodes || !tree_out || !tree_out->parent || !tree_out->token || !tree_out->depth ||
      !tree_out->anc)
    return PROPD_ERR_INVALID_ARG;
  if (dt != PROPD_BF16 && dt != PROPD_F32) return PROPD_ERR_INVALID_ARG;
  if (n_payloads < 0 || n_payloads > PROPD_MAX_PAYLOADS || (n_payloads > 0 && !payloads))
    return PROPD_ERR_INVALID_ARG;
  if (dt == PROPD_BF16 && hidden % kBK != 0) return PROPD_ERR_UNSUPPORTED;
  // operand rows are fetched 16 bytes per lane (bf16) or 4 (fp32); the scratch holds 8-byte records
  const uintptr_t op_align = dt == PROPD_BF16 ? 16 : 4;
  if (reinterpret_cast<uintptr_t>(hidden_states) % op_align != 0 ||
      reinterpret_cast<uintptr_t>(head_weight) % op_align != 0 ||
      reinterpret_cast<uintptr_t>(workspace) % 16 != 0 || reinterpret_cast<uintptr_t>(tree->anc) % 8 != 0)
    return PROPD_ERR_INVALID_ARG;
  const int B = tree->B, T_max = tree->T_max;
  if ((long long)B * T_max > (1ll << 24)) return PROPD_ERR_UNSUPPORTED;
  long long total_blocks = 0;  // of 2048 pieces
  PayloadArgs pa = {};
  for (int p = 0; p < n_payloads; ++p) {
    const propd_payload &pl = payloads[p];
    if (!pl.src || !pl.dst || pl.outer < 1 || pl.row_bytes == 0 || pl.stride_t < 0 ||
        pl.stride_b < 0 || pl.stride_outer < 0 || pl.src == pl.dst)
      return PROPD_ERR_INVALID_ARG;
    pa.src[p] = reinterpret_cast<const char *>(pl.src);
    pa.dst[p] = reinterpret_cast<char *>(pl.dst);
    pa.outer[p] = (unsigned)pl.outer;
    pa.stride_b[p] = pl.stride_b;
    pa.stride_outer[p] = pl.stride_outer;
    pa.stride_t[p] = pl.stride_t;
    const uintptr_t any = reinterpret_cast<uintptr_t>(pl.src) | reinterpret_cast<uintptr_t>(pl.dst) |
                          (uintptr_t)pl.row_bytes | (uintptr_t)pl.stride_b |
                          (uintptr_t)pl.stride_outer | (uintptr_t)pl.stride_t;
    pa.vec16[p] = (any & 15) == 0;
    pa.per_row[p] = pl.row_bytes / (pa.vec16[p] ? 16 : 1);
    const long long rows = (long long)B * pl.outer;
    if (rows > (1ll << 31) - 1) return PROPD_ERR_UNSUPPORTED;
    const long long pieces = (long long)T_max * (long long)pa.per_row[p];
    const long long slices = (pieces + 2047) / 2048;
    if (slices > (1 << 24)) return PROPD_ERR_UNSUPPORTED;
    total_blocks += rows * slices;
    if (total_blocks > (1ll << 31) - 2) return PROPD_ERR_UNSUPPORTED;
  }
  const size_t need = early_prune_workspace_bytes(B, T_max, vocab);
  if (!workspace || workspace_bytes < need) return PROPD_ERR_WORKSPACE;
  PruneScratch ws = carve_scratch(workspace, B, T_max, vocab);
  hipStream_t st = as_stream(hip_stream);

  // tile-shape override for tuning runs: 2 = 352-row tiles, 1 (and whatever else is no 0) = 256-row tiles
  static const int force = [] {
    const char *e = getenv("PROPD_HEAD_PLAN");
    const int v = e ? atoi(e) : 0;
    return v == 0 || v == 2 ? v : 1;
  }();
  const bool scored = !(crit.kind == 0 && crit.top_k >= vocab);
  // top_k >= vocab: every id of the vocabulary is inside the list, no scores are needed (ids
  // outside the vocabulary still fail, in the decision kernel)
  const int cus = prune_compute_units();
  // the tallest tiles address their operand rows by 32-bit offsets
  const int max_mi = (unsigned long long)hidden * 2 * ((unsigned long long)B * T_max > 256 ? (unsigned long long)B * T_max : 256) <
                             (1ull << 32) ? kTallMaxMI : kTallWideMI;
  if (scored) {
    PrepareArgs pr;
    pr.B = B;
    pr.T_max = T_max;
    pr.hidden = hidden;
    pr.vocab = vocab;
    pr.n_nodes = tree->n_nodes;
    pr.parent = tree->parent;
    pr.token = tree->token;
    pr.hidden_states = hidden_states;
    pr.head_weight = head_weight;
    pr.row_src = ws.row_src;
    pr.row_base = ws.row_base;
    pr.row_info = ws.row_info;
    pr.child_list = ws.child_list;
    pr.notes = ws.notes;
    pr.node_row = crit.kind == 0 ? ws.node_row : nullptr;
    pr.own = ws.own;
    const unsigned prep_grid = (unsigned)((B + kTableWaves - 1) / kTableWaves) +
                               (unsigned)B * (unsigned)((T_max + kOwnNodes - 1) / kOwnNodes);
    if (dt == PROPD_BF16)
      hipLaunchKernelGGL(prune_prepare_kernel<true>, dim3(prep_grid), dim3(kScanThreads), 0, st, pr);
    else
      hipLaunchKernelGGL(prune_prepare_kernel<false>, dim3(prep_grid), dim3(kScanThreads), 0, st, pr);
    if (!launch_ok()) return PROPD_ERR_DEVICE;
    HeadTables tb;
    tb.row_src = ws.row_src;
    tb.row_base = ws.row_base;
    tb.row_info = ws.row_info;
    tb.child_list = ws.child_list;
    tb.token = tree->token;
    tb.own = ws.own;
    tb.node_row = ws.node_row;
    tb.T_max = T_max;
    tb.cnt_part = ws.cnt_part;
    tb.cnt_stride = B * T_max;
    tb.lse_part = ws.lse_part;
    tb.parts = (int)ws.parts;
    tb.n_tiles = ws.notes + kNoteTiles;
    if (dt == PROPD_BF16) {
      static std::atomic<bool> attr_set{false};  // calls may come from several threads
      if (!attr_set) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(&early_head_bf16_kernel<0>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kHeadLdsBytes) != hipSuccess ||
            hipFuncSetAttribute(reinterpret_cast<const void *>(&early_head_bf16_kernel<1>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kHeadLdsBytes) != hipSuccess)
          return PROPD_ERR_DEVICE;
        attr_set = true;
      }
      // one workgroup per compute unit and round, two rounds resident in the queue; fewer when
      // even the largest row count has fewer tiles
      const long long m_tiles_cap = (ws.row_cap + 159) / 160;  // no tile is smaller than 160 x 256
      const long long n_groups = ((vocab + 127) / 128 + kXcds - 1) / kXcds;          // or narrower than 128
      long long grid = kXcds * n_groups * m_tiles_cap;
      const long long persistent = (2ll * cus + kXcds - 1) / kXcds * kXcds;
      grid = grid < persistent ? grid : persistent;
      if (crit.kind == 0)
        hipLaunchKernelGGL(early_head_bf16_kernel<0>, dim3((unsigned)grid), dim3(kGemmThreads), kHeadLdsBytes, st,
                           hidden, vocab, B, cus, force, max_mi, reinterpret_cast<const uint16_t *>(hidden_states),
                           reinterpret_cast<const uint16_t *>(head_weight), tb);
      else
        hipLaunchKernelGGL(early_head_bf16_kernel<1>, dim3((unsigned)grid), dim3(kGemmThreads), kHeadLdsBytes, st,
                           hidden, vocab, B, cus, force, max_mi, reinterpret_cast<const uint16_t *>(hidden_states),
                           reinterpret_cast<const uint16_t *>(head_weight), tb);
    } else {
      // two workgroups per compute unit (their LDS), fewer when even the largest row count has
      // fewer tiles
      const long long n_groups = ((vocab + 127) / 128 + kXcds - 1) / kXcds;
      const long long most = kXcds * n_groups * (((long long)ws.row_cap + kF32MaxRows - 1) / kF32MaxRows);
      const long long persistent = (2ll * cus + kXcds - 1) / kXcds * kXcds;
      const unsigned grid = (unsigned)(most < persistent ? most : persistent);
      if (crit.kind == 0)
        hipLaunchKernelGGL(early_head_f32_kernel<0>, dim3(grid), dim3(kF32Threads), 0, st, hidden, vocab, B,
                           reinterpret_cast<const float *>(hidden_states),
                           reinterpret_cast<const float *>(head_weight), tb);
      else
        hipLaunchKernelGGL(early_head_f32_kernel<1>, dim3(grid), dim3(kF32Threads), 0, st, hidden, vocab, B,
                           reinterpret_cast<const float *>(hidden_states),
                           reinterpret_cast<const float *>(head_weight), tb);
    }
  }
  if (!launch_ok()) return PROPD_ERR_DEVICE;
  FinishArgs fa;
  fa.B = B;
  fa.T_max = T_max;
  fa.vocab = vocab;
  fa.bf16 = dt == PROPD_BF16 ? 1 : 0;
  fa.scored = scored ? 1 : 0;
  fa.crit = crit;
  fa.n_nodes = tree->n_nodes;
  fa.parent = tree->parent;
  fa.token = tree->token;
  fa.depth = tree->depth;
  fa.anc = tree->anc;
  fa.row_base = ws.row_base;
  fa.row_info = ws.row_info;
  fa.child_list = ws.child_list;
  fa.cnt_part = ws.cnt_part;
  fa.own = ws.own;
  fa.lse_part = ws.lse_part;
  fa.parts = (int)ws.parts;
  fa.notes = ws.notes;
  fa.keep_bits = keep_bits;
  fa.new_index = new_index;
  fa.orig_index = orig_index;
  fa.n_kept = n_kept;
  fa.cu_nodes = cu_nodes;
  fa.out_n_nodes = tree_out->n_nodes;
  fa.out_parent = tree_out->parent;
  fa.out_token = tree_out->token;
  fa.out_depth = tree_out->depth;
  fa.out_anc = tree_out->anc;
  fa.rank_out = rank_out;
  pa.n = n_payloads;
  fa.pa = pa;
  fa.lines = arrival_lines(B, T_max);
  fa.slices = finish_slices(B, total_blocks, cus);
  fa.inv_slices = ~0ull / (unsigned)fa.slices;
  hipLaunchKernelGGL(prune_finish_kernel, fa.slices > 1 ? dim3((unsigned)fa.slices, (unsigned)B) : dim3((unsigned)B),
                     dim3(kFinishThreads), 0, st, fa);
  if (!scored && B > 1) hipLaunchKernelGGL(cu_nodes_kernel, dim3(1), dim3(kScanThreads), 0, st, B, n_kept, cu_nodes);
  return launch_ok() ? PROPD_OK : PROPD_ERR_DEVICE;
}

extern "C" propd_status propd_early_prune(
    const propd_tree *tree, propd_dtype dt, int32_t hidden, int32_t vocab, int32_t top_k,
    const void *hidden_states, const void *head_weight, uint64_t *keep_bits, int32_t *new_index,
    int32_t *orig_index, int32_t *n_kept, int32_t *cu_nodes, const propd_tree_out *tree_out,
    int32_t *rank_out, int32_t n_payloads, const propd_payload *payloads, void *workspace,
    size_t workspace_bytes, void *hip_stream) {
  if (top_k < 1) return PROPD_ERR_INVALID_ARG;
  const propd::Criterion crit = {0, top_k, 0.f, 0, nullptr};
  return prune_impl(crit, tree, dt, hidden, vocab, hidden_states, head_weight, keep_bits, new_index,
                    orig_index, n_kept, cu_nodes, tree_out, rank_out, n_payloads, payloads,
                    workspace, workspace_bytes, hip_stream);
}

extern "C" propd_status propd_early_prune_prob(
    const propd_tree *tree, propd_dtype dt, int32_t hidden, int32_t vocab, propd_prob_mode mode,
    float threshold, int32_t keep_count, const void *hidden_states, const void *head_weight,
    uint64_t *keep_bits, int32_t *new_index, int32_t *orig_index, int32_t *n_kept,
    int32_t *cu_nodes, const propd_tree_out *tree_out, float *log_marginal, int32_t n_payloads,
    const propd_payload *payloads, void *workspace, size_t workspace_bytes, void *hip_stream) {
  propd::Criterion crit = {1, 1, 0.f, 0, log_marginal};
  if (mode == PROPD_PROB_THRESHOLD) {
    if (!(threshold >= 0.f) || threshold > 1.f) return PROPD_ERR_INVALID_ARG;
    crit.log_threshold = threshold > 0.f ? logf(threshold) : -INFINITY;
  } else if (mode == PROPD_PROB_RANK) {
    if (keep_count < 1) return PROPD_ERR_INVALID_ARG;
    crit.kind = 2;
    crit.keep_count = keep_count;
  } else {
    return PROPD_ERR_INVALID_ARG;
  }
  return prune_impl(crit, tree, dt, hidden, vocab, hidden_states, head_weight, keep_bits, new_index,
                    orig_index, n_kept, cu_nodes, tree_out, nullptr, n_payloads, payloads,
                    workspace, workspace_bytes, hip_stream);
}
