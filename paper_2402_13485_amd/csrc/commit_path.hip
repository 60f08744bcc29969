// Commit of the accepted path: the step that follows acceptance in a decoding loop
// (Section 2, "Verification": the longest verified sequence is kept; Section 5.1: greedy
// decoding).  The K/V rows of the accepted nodes move from the tree tensors to the end of
// the cache, the sequence grows by the acceptance length, and the step's tokens (the
// accepted candidates, then the model's own choice after the last of them) are written out.
#include "common.h"

namespace propd {

constexpr int kCommitThreads = 256;

// The new length and the step's tokens of sequence b, by the threads tid, tid + threads, ...
__device__ __forceinline__ void commit_tokens(int b, int tid, int threads, int T, int L, int a, int L_max, int T_max,
                                              const int32_t *__restrict__ token, const int32_t *__restrict__ accept_path,
                                              int path_stride, const int32_t *__restrict__ next_token,
                                              int32_t *__restrict__ seq_lens, int32_t *__restrict__ out_tokens,
                                              int out_stride) {
  const int kept = a > L_max - L ? L_max - L : a;
  if (tid == 0) seq_lens[b] = L + kept;
  if (!out_tokens) return;
  for (int j = tid; j < out_stride; j += threads) {
    int v = -1;
    if (j + 1 < a) {
      const int node = accept_path[(size_t)b * path_stride + j + 1];
      if (node >= 0 && node < T) v = token[(size_t)b * T_max + node];
    } else if (j + 1 == a) {
      v = next_token[b];
    }
    out_tokens[(size_t)b * out_stride + j] = v;
  }
}

// Short paths: one workgroup does all heads of a sequence, and then its length and tokens, so that the
// call is one launch instead of two (see commit_one_threads).
constexpr int kCommitOneThreads = 1024, kCommitOneItems = 4;  // pieces of K and of V of a thread requested together

__global__ __launch_bounds__(kCommitOneThreads) void commit_one_kernel(
    int H, int T_max, int L_max, int row_bytes, const int32_t *__restrict__ n_nodes, const int32_t *__restrict__ token,
    const int32_t *__restrict__ accept_len, const int32_t *__restrict__ accept_path, int path_stride,
    const int32_t *__restrict__ next_token, int32_t *__restrict__ seq_lens, const unsigned char *__restrict__ k_tree,
    const unsigned char *__restrict__ v_tree, unsigned char *__restrict__ k_cache,
    unsigned char *__restrict__ v_cache, int32_t *__restrict__ out_tokens, int out_stride) {
  const int b = blockIdx.x;
  int T = n_nodes[b], L = seq_lens[b], a = accept_len[b];
  T = T < 1 ? 1 : (T > T_max ? T_max : T);
  L = L < 0 ? 0 : (L > L_max ? L_max : L);
  a = a < 0 ? 0 : (a > path_stride ? path_stride : a);
  const int rows = a > L_max - L ? L_max - L : a, pieces = row_bytes / 16;
  const int items = rows * H * pieces, threads = blockDim.x;
  for (int item0 = threadIdx.x; item0 < items; item0 += kCommitOneItems * threads) {
    u32x4 kv[kCommitOneItems][2];
    size_t dst[kCommitOneItems];
    bool on[kCommitOneItems];
#pragma unroll
    for (int x = 0; x < kCommitOneItems; ++x) {
      const int wanted = item0 + x * threads, item = wanted < items ? wanted : item0;
      const int row = item / pieces, c = item - row * pieces, h = row / rows, j = row - h * rows;
      int node = accept_path[(size_t)b * path_stride + j];
      on[x] = wanted < items && node >= 0 && node < T;
      node = node >= 0 && node < T ? node : 0;
      const size_t unit = (size_t)b * H + h, src = (unit * T_max + node) * row_bytes + 16 * c;
      dst[x] = (unit * L_max + L + j) * row_bytes + 16 * c;
      kv[x][0] = *reinterpret_cast<const u32x4 *>(k_tree + src);
      kv[x][1] = *reinterpret_cast<const u32x4 *>(v_tree + src);
    }
#pragma unroll
    for (int x = 0; x < kCommitOneItems; ++x)
      if (on[x]) {
        *reinterpret_cast<u32x4 *>(k_cache + dst[x]) = kv[x][0];
        *reinterpret_cast<u32x4 *>(v_cache + dst[x]) = kv[x][1];
      }
  }
  __syncthreads();  // every thread has read the old length
  commit_tokens(b, threadIdx.x, threads, T, L, a, L_max, T_max, token, accept_path, path_stride, next_token,
                seq_lens, out_tokens, out_stride);
}

// One workgroup per (sequence, head): 16 lanes move the 16-byte pieces of one row.  Indices
// read from device arrays are range-checked; rows that would pass the end of the cache are
// dropped.
__global__ __launch_bounds__(kCommitThreads) void commit_rows_kernel(
    int H, int T_max, int L_max, int row_bytes, const int32_t *__restrict__ n_nodes,
    const int32_t *__restrict__ accept_len, const int32_t *__restrict__ accept_path,
    int path_stride, const int32_t *__restrict__ seq_lens, const unsigned char *__restrict__ k_tree,
    const unsigned char *__restrict__ v_tree, unsigned char *__restrict__ k_cache,
    unsigned char *__restrict__ v_cache) {
  const int unit = blockIdx.x, b = unit / H;
  int T = n_nodes[b];
  T = T < 1 ? 1 : (T > T_max ? T_max : T);
  int L = seq_lens[b];
  L = L < 0 ? 0 : (L > L_max ? L_max : L);
  int a = accept_len[b];
  a = a < 0 ? 0 : (a > path_stride ? path_stride : a);
  a = a > L_max - L ? L_max - L : a;
  const int pieces = row_bytes / 16;
  const size_t tree_base = (size_t)unit * T_max * row_bytes, cache_base = (size_t)unit * L_max * row_bytes;
  for (int item = threadIdx.x; item < a * pieces; item += kCommitThreads) {
    const int j = item / pieces, c = item - j * pieces;
    const int node = accept_path[(size_t)b * path_stride + j];
    if (node < 0 || node >= T) continue;
    const size_t src = tree_base + (size_t)node * row_bytes + 16 * c;
    const size_t dst = cache_base + (size_t)(L + j) * row_bytes + 16 * c;
    *reinterpret_cast<u32x4 *>(k_cache + dst) = *reinterpret_cast<const u32x4 *>(k_tree + src);
    *reinterpret_cast<u32x4 *>(v_cache + dst) = *reinterpret_cast<const u32x4 *>(v_tree + src);
  }
}

// One lane per sequence: the new length and the step's tokens.  Runs after the row copy,
// which reads the old lengths.
__global__ __launch_bounds__(kCommitThreads) void commit_tokens_kernel(
    int B, int T_max, int L_max, const int32_t *__restrict__ n_nodes,
    const int32_t *__restrict__ token, const int32_t *__restrict__ accept_len,
    const int32_t *__restrict__ accept_path, int path_stride,
    const int32_t *__restrict__ next_token, int32_t *__restrict__ seq_lens,
    int32_t *__restrict__ out_tokens, int out_stride) {
  const int b = blockIdx.x * kCommitThreads + threadIdx.x;
  if (b >= B) return;
  int T = n_nodes[b];
  T = T < 1 ? 1 : (T > T_max ? T_max : T);
  int L = seq_lens[b];
  L = L < 0 ? 0 : (L > L_max ? L_max : L);
  int a = accept_len[b];
  a = a < 0 ? 0 : (a > path_stride ? path_stride : a);
  commit_tokens(b, 0, 1, T, L, a, L_max, T_max, token, accept_path, path_stride, next_token, seq_lens, out_tokens,
                out_stride);
}

// Threads per sequence of the one-launch form, 0 where the call takes two launches.
//   - The line.  One workgroup moves 4096 pieces of K and of V in a round of its threads, a launch less
//     outweighs that.  What is left of a full buffer beyond a round costs more than the launch, unless
//     the other form is slow too: its second kernel writes a sequence's tokens one by one (from 32 of
//     them on), or its workgroups of a (sequence, head) each fill the chip more than twice.  Call, us, two launches / one,
//     with 3 nodes accepted and with a full buffer:
//       1 x 32 heads, 8 nodes of 256 bytes (4096 pieces)   7.1 / 6.5   7.6 / 7.3
//       1 x 40, 8 (5120, within the third of a round)      7.2 / 6.6   7.5 / 9.1 (5 accepted: 7.4 / 6.9)
//       1 x 64, 8 (8192)                                   7.2 / 6.9   7.7 / 10.0
//       64 x 64, 8                                         9.8 / 8.7  12.3 / 13.0
//       256 x 64, 8                                       17.6 / 12.1 28.0 / 23.1
//       1 x 16, 32 (8192)                                  9.6 / 6.1  11.8 / 10.0
//       1 x 4, 128 (8192)                                 17.5 / 5.1  31.5 / 9.9
//     The host saves a launch besides.
//   - The threads: one per piece, as long as those of all sequences fit the chip at once (2^19).  Beyond
//     that each takes several: 4096 x 1 head, 1 node of 128 bytes 8.7 / 7.5 (26.2 with 1024 threads), 4096 x 8, 8
//     of 256 bytes 59 / 49 (89), 1024 x 8, 8 19.0 / 16.0 (20.7).  It also keeps the threads of a
//     launch, which may be fewer than 2^32, from bounding the batch: 64 of them from 8192 sequences on.
static int commit_one_threads(int B, int H, int pieces, int path_stride) {
  const long long full = (long long)path_stride * H * pieces, round = (long long)kCommitOneThreads * kCommitOneItems;
  const bool others_slow = path_stride >= 32 || (long long)B * H > 4096;
  if (full > (others_slow ? 2 * round : round + round / 3)) return 0;
  int threads = kWave;
  while (threads < full && threads < kCommitOneThreads && 2ll * B * threads <= (1 << 19)) threads *= 2;
  return threads;
}

}  // namespace propd

extern "C" propd_status propd_commit_path(const propd_tree *tree, propd_dtype dt, int32_t H,
                                          int32_t d, const int32_t *accept_len,
                                          const int32_t *accept_path, int32_t path_stride,
                                          const int32_t *next_token, const void *k_tree,
                                          const void *v_tree, void *k_cache, void *v_cache,
                                          int32_t L_max, int32_t *seq_lens, int32_t *out_tokens,
                                          int32_t out_stride, void *hip_stream) {
  using namespace propd;
  if (!tree || tree->B < 1 || tree->T_max < 1 || tree->T_max > PROPD_MAX_TREE || H < 1 || d < 1 ||
      L_max < 1 || path_stride < 1 || !tree->n_nodes || !accept_len || !accept_path || !k_tree ||
      !v_tree || !k_cache || !v_cache || !seq_lens)
    return PROPD_ERR_INVALID_ARG;
  if (dt != PROPD_BF16 && dt != PROPD_F32) return PROPD_ERR_INVALID_ARG;
  if (out_tokens && (out_stride < 1 || !tree->token || !next_token)) return PROPD_ERR_INVALID_ARG;
  const long long row_bytes = (long long)d * (dt == PROPD_BF16 ? 2 : 4);
  if (row_bytes % 16 != 0 || row_bytes > (1 << 20)) return PROPD_ERR_UNSUPPORTED;
  for (const void *ptr : {k_tree, v_tree, (const void *)k_cache, (const void *)v_cache})
    if (reinterpret_cast<uintptr_t>(ptr) % 16 != 0) return PROPD_ERR_INVALID_ARG;
  const long long units = (long long)tree->B * H;
  if (units > (1ll << 30)) return PROPD_ERR_UNSUPPORTED;
  hipStream_t st = as_stream(hip_stream);
  const int one = commit_one_threads(tree->B, H, (int)(row_bytes / 16), path_stride);
  if (one > 0) {
    hipLaunchKernelGGL(commit_one_kernel, dim3((unsigned)tree->B), dim3((unsigned)one), 0, st, H, tree->T_max,
                       L_max, (int)row_bytes, tree->n_nodes, tree->token, accept_len, accept_path, path_stride,
                       next_token, seq_lens, reinterpret_cast<const unsigned char *>(k_tree),
                       reinterpret_cast<const unsigned char *>(v_tree), reinterpret_cast<unsigned char *>(k_cache),
                       reinterpret_cast<unsigned char *>(v_cache), out_tokens, out_stride);
    return launch_ok() ? PROPD_OK : PROPD_ERR_DEVICE;
  }
  hipLaunchKernelGGL(commit_rows_kernel, dim3((unsigned)units), dim3(kCommitThreads), 0, st, H,
                     tree->T_max, L_max, (int)row_bytes, tree->n_nodes, accept_len, accept_path,
                     path_stride, seq_lens, reinterpret_cast<const unsigned char *>(k_tree),
                     reinterpret_cast<const unsigned char *>(v_tree),
                     reinterpret_cast<unsigned char *>(k_cache),
                     reinterpret_cast<unsigned char *>(v_cache));
  if (!launch_ok()) return PROPD_ERR_DEVICE;
  hipLaunchKernelGGL(commit_tokens_kernel, dim3((unsigned)((tree->B + kCommitThreads - 1) / kCommitThreads)),
                     dim3(kCommitThreads), 0, st, tree->B, tree->T_max, L_max, tree->n_nodes,
                     tree->token, accept_len, accept_path, path_stride, next_token, seq_lens,
                     out_tokens, out_stride);
  return launch_ok() ? PROPD_OK : PROPD_ERR_DEVICE;
}
