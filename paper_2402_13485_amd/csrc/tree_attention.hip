// Tree-masked attention over the cached prefix plus each node's own root path
// (Section 2, "Verification"; Figure 2(b,c)).
//
// bf16 path (d = 64 and 128).  The work is a stream of K/V rows from HBM that all T
// tree queries of a (sequence, head) pair share, so the kernel is organised
// around reading every K and V row exactly once, as fast as HBM delivers them:
//   - the work of a call is the list of 32-row K/V stages of all (sequence, head)
//     units in order (cached rows, then tree rows); a persistent grid of two
//     workgroups per compute unit cuts that list into equal contiguous ranges, so
//     ragged sequence lengths balance by construction;
//   - a workgroup streams its range through a ring of LDS stages with direct
//     global->LDS loads (no registers, no LDS store instructions), issued NS-1
//     stages ahead of the math and running straight across unit boundaries; rows
//     are unpadded in LDS and their 16-byte chunks are XOR-swizzled by the load
//     addresses so that both MFMA operand read patterns are bank-conflict free;
//   - scores are computed transposed, S^T = K . Q^T, with the 32x32x16 bf16 MFMA,
//     so that a lane owns one query column: the running max / sum of the online
//     softmax are per-lane scalars, and the fp32 score registers, once
//     exponentiated and rounded to bf16, ARE the B operand of the second MFMA
//     O^T += V^T . P^T, with no shuffle or LDS round trip; V^T is read from
//     row-major V in LDS with the transposing LDS read;
//   - the cached prefix needs no mask; tree stages keep a score only where the
//     node's 128-bit ancestor set has the bit;
//   - the four waves of a workgroup split the query columns (32 each); a wave whose
//     columns lie beyond the tree only helps with the loads.  Trees of at most 64 nodes have two
//     waves per 32 columns, each with half of a stage's rows (see KS);
//   - a unit cut by a range boundary leaves fp32 partials (O, max, sum), at most
//     two per workgroup, and the workgroup holding its first piece leaves a record of the
//     cut; a second kernel merges the pieces of every recorded cut, in their order.
// Both head sizes run the same kernel.  d = 64 came from one wave per query (each lane walking K rows
// of its own): 8 x 16 units of 64 queries x 2048 keys, 4150 -> 31 us + 5 us merge (67 MB of K/V).
// Without a workspace or 16-byte alignment d = 64 runs a plain one-wave-per-query kernel.
// fp32 path: tree_attention_f32.h.
#include <atomic>
#include <type_traits>
#include <utility>

#include "common.h"

namespace propd {

constexpr int kAttnThreads = 256;
constexpr int kMaxGrid = 1024;   // workgroups of the persistent kernel, at most
constexpr int kStageRows = 32;   // K/V rows per ring stage
constexpr int kRingStages = 5;

// What depends on the head size D.
template <int D>
struct Geo {
  static constexpr int kRowBytes = D * 2;                     // one bf16 row
  static constexpr int kHalfStage = kStageRows * kRowBytes;   // K part of a stage; the V part follows
  static constexpr int kStageBytes = 2 * kHalfStage;          // 16 KB (D = 128) or 8 KB
  static constexpr int kChunks = kRowBytes / 16;              // 16-byte chunks of a row
  static constexpr int kLdRows = 1024 / kRowBytes;            // rows that one direct load of a wave fills
  static constexpr int kLoads = kHalfStage / 4096;            // direct loads of a wave per half stage
  static constexpr int kMb = D / 32;                          // 32-wide blocks of d of PV
  // Workgroups resident on a compute unit: what LDS (two rings of 80 KB) and registers (one wave per 32 queries 253
  // or, with kAnew, all 256; two 215 to 218) allow at D = 128, and registers at D = 64 with one wave (208).  With two it
  // takes 165 and 41 KB of LDS, and a third workgroup would fit (not measured).  A bound of four spilled at D = 64, which this
  // kernel must not: loads that it waits for by hand would land in registers given away meanwhile.
  static constexpr int kPerCu = 2;
  // Chunk c of row r of a stage lies at chunk position c ^ key(r).
  //   K: the 16 rows x 16 bytes that one pass of a fragment read takes (one chunk column) fall
  //      into 16 different bank groups (rows of 128 bytes: two rows share a 256-byte bank line)
  //   V: so do the 4 rows x 64 bytes of one transposing read
  static __device__ __forceinline__ int k_key(int r) { return D == 128 ? r & 15 : (r >> 1) & 7; }
  static __device__ __forceinline__ int v_key(int r) {
    return D == 128 ? ((r & 3) << 2) | ((r >> 2) & 3) : ((r >> 1) & 1) << 2;
  }
};

struct AttnParams {
  const uint16_t *q, *k_cache, *v_cache, *k_tree, *v_tree;
  uint16_t *out;
  const int32_t *seq_lens, *n_nodes;
  const uint64_t *anc;
  int B, H, T_max, L_max;
  float scale, scale_log2e;
  float *part_o;   // [2 * grid][4 waves][16 blocks][64 lanes][4]
  float *part_ml;  // [2 * grid][4 waves][m | l][64 lanes]
  int32_t *cuts;   // CutRecords: [units] by unit, or [grid] by the workgroup that holds the first piece
  int by_unit;     // see merge_by_unit
  int one_pass;    // see begin_one_pass
  int cus;         // compute units
};

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((address_space(3))) void lds_void;
typedef const __attribute__((address_space(1))) void global_void;

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// two floats -> packed bf16 pair (round to nearest even), one v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t cvt_pk_bf16(float lo, float hi) {
  const f32x2 f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}

// Transposing LDS read (ds_read_b64_tr_b16), issued as assembly so that the compiler does
// not fence it against the ring's direct loads in flight (the builtin counts as a possible
// LDS write, which would drain them).  The result is valid only after wait_lds<>().
template <int OFFSET>
__device__ __forceinline__ u32x2 lds_read_tr16(uint32_t addr) {
  u32x2 r;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFFSET));
  return r;
}

// LDS traffic between the waves of a workgroup, for the same reason as assembly.
template <int OFFSET>
__device__ __forceinline__ void lds_write16(uint32_t addr, f32x4 v) {
  asm volatile("ds_write_b128 %0, %1 offset:%2" ::"v"(addr), "v"(v), "n"(OFFSET) : "memory");
}
__device__ __forceinline__ void lds_write8(uint32_t addr, u32x2 v) {
  asm volatile("ds_write_b64 %0, %1" ::"v"(addr), "v"(v) : "memory");
}
template <class F, int... I>
__device__ __forceinline__ void static_for_i_impl(F &&f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for_i(F &&f) {
  static_for_i_impl(f, std::make_integer_sequence<int, N>{});
}

// wait until at most N LDS operations of this wave are outstanding; the registers named
// are the results being waited for, so that their uses cannot be scheduled above the wait
template <int N>
__device__ __forceinline__ void wait_lds(u32x2 (&a)[4]) {
  asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]) : "n"(N));
}
template <int N>
__device__ __forceinline__ void wait_lds(u32x2 (&a)[8]) {
  asm volatile("s_waitcnt lgkmcnt(%8)"
               : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]),
                 "+v"(a[7])
               : "n"(N));
}

// wait until at most N of this wave's vector memory operations are outstanding
template <int N>
__device__ __forceinline__ void wait_vmem() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Global loads and stores issued as assembly.  The main kernel waits for its vector memory
// operations itself, with explicit counts; the compiler's own bookkeeping would fence the
// ring's loads in flight at every use of a loaded register.  The compiler's hazard
// recognizer does not look inside assembly either: the stores carry their own wait states
// for data registers written just before by vector or cross-lane instructions, and after
// themselves, because a store wider than 8 bytes still reads its data registers when the
// next instruction issues.
__device__ __forceinline__ u32x4 global_load16_untracked(const void *ptr) {
  u32x4 r;
  asm volatile("s_nop 3\n\tglobal_load_dwordx4 %0, %1, off" : "=v"(r) : "v"(ptr) : "memory");
  return r;
}
__device__ __forceinline__ void global_store16_untracked(void *ptr, u32x4 v) {
  asm volatile("s_nop 7\n\tglobal_store_dwordx4 %0, %1, off sc1\n\ts_nop 3" ::"v"(ptr), "v"(v) : "memory");
}
__device__ __forceinline__ void global_store4_untracked(void *ptr, float v) {
  asm volatile("s_nop 7\n\tglobal_store_dword %0, %1, off sc1\n\ts_nop 3" ::"v"(ptr), "v"(v) : "memory");
}

// Exchange between the two 32-lane halves of a wave (v_permlane32_swap): afterwards lane
// l < 32 holds (a[l], a[l+32]) and lane l >= 32 holds (b[l-32], b[l]) in (a, b).
__device__ __forceinline__ void swap_halves(uint32_t &a, uint32_t &b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}

// A lane of the main kernel holds, for its query t = 32*wave + lane%32, the 64 values
// d = 32*mb + 8*q4 + 4*(lane/32) + j of O^T in o_acc[mb][4*q4 + j].
// Output rows: neighbouring q4 of the two lane halves are exchanged so that every lane
// writes 8 consecutive bf16 values (16 bytes) per store.
template <bool kUntracked>
__device__ __forceinline__ void store_out_block(uint16_t *orow, const f32x16 &o, float inv, int g, int mb) {
#pragma unroll
  for (int jp = 0; jp < 2; ++jp) {
    const int e = 8 * jp, od = 8 * jp + 4;  // first register of the even / odd q4 of the pair
    uint32_t a0 = cvt_pk_bf16(o[e] * inv, o[e + 1] * inv);
    uint32_t a1 = cvt_pk_bf16(o[e + 2] * inv, o[e + 3] * inv);
    uint32_t b0 = cvt_pk_bf16(o[od] * inv, o[od + 1] * inv);
    uint32_t b1 = cvt_pk_bf16(o[od + 2] * inv, o[od + 3] * inv);
    swap_halves(a0, b0);
    swap_halves(a1, b1);
    // lower half: d = 32*mb + 16*jp + 0..7, upper half: the 8 values after those
    const u32x4 w4 = {a0, a1, b0, b1};
    if (kUntracked) global_store16_untracked(orow + mb * 32 + 16 * jp + 8 * g, w4);
    else *reinterpret_cast<u32x4 *>(orow + mb * 32 + 16 * jp + 8 * g) = w4;
  }
}

// Partial results keep the register layout, so that a wave writes and reads them as
// contiguous 1 KB blocks: part_o[slot][wave][4*mb + q4][lane][j], part_ml[slot][wave][m|l][lane].
constexpr size_t kPartOFloats = 4 * 16 * 64 * 4;  // floats of part_o per slot
constexpr size_t kPartMlFloats = 4 * 2 * 64;     // floats of part_ml per slot
__device__ __forceinline__ size_t part_o_index(size_t slot, int wave, int blk, int lane) {
  return (((slot * 4 + wave) * 16 + blk) * 64 + lane) * 4;
}
__device__ __forceinline__ size_t part_ml_index(size_t slot, int wave, int which, int lane) {
  return ((slot * 4 + wave) * 2 + which) * 64 + lane;
}

// Work decomposition shared by the main kernel and the merge kernel.  The work of one
// call is made of K/V stages; a (sequence, head) unit is its cached stages followed by its
// tree stages.  Workgroup w of G does, in this order,
//   - k whole units w, w+G, ..., when all sequences have the same lengths (k = units / G):
//     no partial results, and all workgroups write their outputs at the same moments, which
//     the memory system takes far better than a trickle of stores into the read stream;
//   - the contiguous range [w*N/G, (w+1)*N/G) of the list of the N stages of the remaining
//     units (all units when lengths differ, so that every workgroup streams the same number
//     of rows whatever the mix); a unit cut by a range boundary is finished by the merge
//     kernel from per-workgroup partial results.
// With no more units than workgroups the ranges are cut so that none crosses a unit, where that
// costs little (begin_one_pass).
// A wave-uniform 32-bit load on the scalar path.  Issued as assembly: the compiler would
// use a vector load here and wait for it with vmcnt(0), which drains the ring.  The
// scalar cache is invalidated when a kernel starts, like the vector caches, so values
// that an earlier kernel or the caller rewrote in place are seen.
__device__ __forceinline__ int32_t uniform_load_i32(const int32_t *ptr) {
  const uint64_t a = (uint64_t)(uintptr_t)ptr;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  const uint64_t sa = ((uint64_t)hi << 32) | lo;  // in scalar registers
  int32_t v;
  asm volatile("s_load_dword %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(v) : "s"(sa) : "memory");
  return v;
}

struct StageMap {
  int B, H;
  const int32_t *seq_lens, *n_nodes;
  int L_max, T_max, cus;
  __device__ __forceinline__ int len(int b) const {
    const int L = uniform_load_i32(seq_lens + b);
    return L < 0 ? 0 : (L > L_max ? L_max : L);
  }
  __device__ __forceinline__ int nodes(int b) const {
    const int T = uniform_load_i32(n_nodes + b);
    return T < 1 ? 1 : (T > T_max ? T_max : T);
  }
  __device__ __forceinline__ int cache_stages(int b) const {
    return (len(b) + kStageRows - 1) / kStageRows;
  }
  __device__ __forceinline__ int tree_stages(int b) const {
    return (nodes(b) + kStageRows - 1) / kStageRows;
  }
  __device__ __forceinline__ int unit_stages(int b) const { return cache_stages(b) + tree_stages(b); }
  // the same for a sequence index that differs between lanes (plain loads); 0 past the batch
  __device__ __forceinline__ int unit_stages_lane(int b) const {
    if (b >= B) return 0;
    int L = seq_lens[b], T = n_nodes[b];
    L = L < 0 ? 0 : (L > L_max ? L_max : L);
    T = T < 1 ? 1 : (T > T_max ? T_max : T);
    return (L + kStageRows - 1) / kStageRows + (T + kStageRows - 1) / kStageRows;
  }
  // Sequence that holds stage x of the list of all units, and the stages before that
  // sequence; the last sequence if x lies past the end.  Every lane of the wave takes part:
  // 64 sequences are sized per pass, with a wave prefix sum.
  __device__ void locate(long long x, int &b_out, long long &b_start_out) const {
    const int lane = threadIdx.x & 63;
    long long base = 0;
    int b_found = B - 1;
    long long start_found = 0;
    bool found = false;
    for (int b0 = 0; b0 < B && !found; b0 += 64) {
      const long long mine = (long long)H * unit_stages_lane(b0 + lane);
      long long incl = mine;  // inclusive prefix over the lanes
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const long long up = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += up;
      }
      const long long excl = base + incl - mine;
      // the holder is the last sequence that starts at or before x
      const uint64_t le = __ballot(b0 + lane < B && excl <= x);
      const int n_le = __popcll(le);
      const long long total = __shfl(incl, 63, kWave);
      if (x < base + total || b0 + 64 >= B) {
        const int src = n_le > 0 ? n_le - 1 : 0;
        b_found = b0 + src;
        start_found = __shfl(excl, src, kWave);
        found = true;
      }
      base += total;
    }
    b_out = __builtin_amdgcn_readfirstlane(b_found);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)start_found);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)start_found >> 32));
    b_start_out = (long long)(((uint64_t)hi << 32) | lo);
  }
  // stages of all units before unit (b, h) in the list of all units
  __device__ long long stages_before(int b, int h) const {
    const int lane = threadIdx.x & 63;
    long long n = 0;
    for (int b0 = 0; b0 < b; b0 += 64)
      n += wave_reduce_sum(b0 + lane < b ? (long long)H * unit_stages_lane(b0 + lane) : 0ll);
    n += (long long)h * unit_stages(b);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)n);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)n >> 32));
    return (long long)(((uint64_t)hi << 32) | lo);
  }
};


struct Schedule {
  int k;                  // whole units per workgroup, done first
  long long first_split;  // first unit of the split list (= k * G)
  long long split_base;   // stages of the units before it
  long long n_split;      // stages of the split list
  // The split list is cut into G contiguous ranges: the first `rem` workgroups take
  // `quot` + 1 stages, the others `quot` (one division per kernel, none per range).
  long long quot, rem;
  int pieces = 0;  // > 0: no range crosses a unit, and this workgroup's unit is cut into so many
  // The softmax reference is set anew every so many stages (kernels with kAnew; the check alone costs 0.5 % of a long
  // call).  The largest weight of such a stage is exactly 1 and rounds to bf16 without error, like that of
  // a piece's first stage: with ranges that cross no unit there would be fewer of these, and the error against
  // 64 bits up to 4 % larger than with ranges that do (6 x 8 ragged units of 107 queries: 1.887e-3, 1.965e-3 without
  // this).  Set often enough that it is no larger; once per stage costs 1.1 us of 14.  A stage whose scores lie more than
  // 2^8 in the exponent below the highest one of the piece gets no such weight: see m_top.
  int anew = 1 << 30;
  __device__ __forceinline__ long long range_start(long long w) const {
    return w * quot + (w < rem ? w : rem);
  }
  // workgroup whose range holds stage x of the split list
  __device__ __forceinline__ long long range_owner(long long x) const {
    const long long big = rem * (quot + 1);  // stages held by the larger ranges
    if (n_split < (1ll << 31)) {             // the usual case: 32-bit divisions
      const uint32_t xx = (uint32_t)x, bb = (uint32_t)big, qq = (uint32_t)quot;
      return xx < bb ? xx / (qq + 1u) : (uint32_t)rem + (xx - bb) / qq;
    }
    return x < big ? x / (quot + 1) : rem + (x - big) / quot;
  }
};

// What the workgroup that holds the FIRST piece of a unit leaves for the merge kernel.  With few
// units (merge_by_unit) the records go by unit, and every unit gets one in every call;
// otherwise by workgroup (a workgroup holds the first piece of at most one cut unit), and every
// workgroup of the grid writes its own in every call (unit < 0: none).  The pieces of the unit
// lie in workgroups w_first .. w_last: the first in the second partial slot of w_first, the others in
// the first slot of theirs.
struct CutRecord {
  int32_t unit;
  int32_t w_last_and_nodes;  // w_last | (tree nodes of the unit's sequence << 16)
  int32_t w_first;
  int32_t pad;
};

__device__ __forceinline__ Schedule make_schedule(const StageMap &m, long long G) {
  Schedule sc;
  const int lane = threadIdx.x & 63;
  int us_min = 1 << 30, us_max = 0;
  long long n_all = 0;
  for (int b0 = 0; b0 < m.B; b0 += 64) {  // 64 sequences per pass, one per lane
    const bool in = b0 + lane < m.B;
    const int us = m.unit_stages_lane(b0 + lane);
    us_min = min(us_min, -wave_reduce_max(in ? -us : -(1 << 30)));
    us_max = max(us_max, wave_reduce_max(in ? us : 0));
    n_all += wave_reduce_sum((long long)m.H * us);
  }
  us_min = __builtin_amdgcn_readfirstlane(us_min);
  us_max = __builtin_amdgcn_readfirstlane(us_max);
  {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)n_all);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)n_all >> 32));
    n_all = (long long)(((uint64_t)hi << 32) | lo);
  }
  // whole units first only where they are (nearly) equally long: a workgroup's k of them
  // then differ by at most a few percent between workgroups
  const long long U = (long long)m.B * m.H;
  sc.k = (us_max - us_min) * 32 <= us_max ? (int)(U / G) : 0;
  sc.first_split = (long long)sc.k * G;
  sc.split_base = sc.k > 0 ? m.stages_before((int)(sc.first_split / m.H), (int)(sc.first_split % m.H)) : 0;
  sc.n_split = n_all - sc.split_base;
  sc.quot = sc.n_split / G;
  sc.rem = sc.n_split - sc.quot * G;
  return sc;
}

// Sums and extremes over the lanes by data-parallel moves between registers (a few cycles per step, a
// tenth of what a step through LDS takes).  `idle` fills the lanes that a step does not reach.
template <class F>
__device__ __forceinline__ int wave_scan_i32(int v, int idle, F &&join) {
  v = join(v, __builtin_amdgcn_update_dpp(idle, v, 0x111, 0xf, 0xf, false));  // row_shr:1
  v = join(v, __builtin_amdgcn_update_dpp(idle, v, 0x112, 0xf, 0xf, false));  // row_shr:2
  v = join(v, __builtin_amdgcn_update_dpp(idle, v, 0x114, 0xf, 0xf, false));  // row_shr:4
  v = join(v, __builtin_amdgcn_update_dpp(idle, v, 0x118, 0xf, 0xf, false));  // row_shr:8
  v = join(v, __builtin_amdgcn_update_dpp(idle, v, 0x142, 0xa, 0xf, false));  // row_bcast:15 into rows 1 and 3
  v = join(v, __builtin_amdgcn_update_dpp(idle, v, 0x143, 0xc, 0xf, false));  // row_bcast:31 into rows 2 and 3
  return v;
}

// Position of a workgroup in its own sequence of stages: stage s of unit (b, h).
struct Walk {
  long long unit;  // b * H + h
  int b, s;
  int L, T, cs, ts;         // cached rows, tree nodes, cached stages, tree stages of sequence b
  int whole_left;           // whole units still to do, this one included; 0 = in the split range
  long long split_unit;     // where this workgroup's split range starts
  int split_s;
  long long x_end;          // end of this workgroup's range in the split list
  __device__ __forceinline__ void load_sizes(const StageMap &m) {
    L = m.len(b);
    T = m.nodes(b);
    cs = (L + kStageRows - 1) / kStageRows;
    ts = (T + kStageRows - 1) / kStageRows;
  }
  __device__ __forceinline__ void set_unit(const StageMap &m, long long u) {
    unit = u;
    const int nb = (int)(u / m.H);
    if (nb != b) {
      b = nb;
      load_sizes(m);
    }
  }
  // the workgroup's first stage; returns the number of stages it will do
  __device__ int start(const StageMap &m, const Schedule &sc, long long w, long long G) {
    const long long U = (long long)m.B * m.H;
    const long long x0 = sc.range_start(w);
    int n_my = (int)(sc.range_start(w + 1) - x0);
    x_end = x0 + n_my;
    // locate stage split_base + x0 of the list of all units
    const long long x = sc.split_base + x0;
    long long b_start;
    m.locate(x, b, b_start);
    load_sizes(m);
    {
      const int us = cs + ts;
      const long long hh = (x - b_start) / us;
      split_unit = (long long)b * m.H + hh;
      split_s = (int)((x - b_start) - hh * us);
    }
    if (split_unit >= U) {  // an empty range at the very end: stay on valid memory
      split_unit = U - 1;
      split_s = 0;
    }
    whole_left = sc.k;
    if (sc.k > 0) {
      for (int j = 0; j < sc.k; ++j) n_my += m.unit_stages((int)((w + j * G) / m.H));
      b = -1;
      set_unit(m, w);
      s = 0;
    } else {
      b = -1;
      set_unit(m, split_unit);
      s = split_s;
    }
    return n_my;
  }
  // n / d rounded down, for whole n below 2^20 and inv = 1 / d to one unit in the last place: n + 1/2 is half a
  // d-th away from the next whole quotient, the error of the product at most n / d / 2^22
  static __device__ __forceinline__ float floor_quotient(float n, float inv) { return floorf((n + .5f) * inv); }
  // n / d rounded up, up = (d - 1/2) / d
  static __device__ __forceinline__ float ceil_quotient(float n, float inv, float up) { return floorf(fmaf(n, inv, up)); }
  // The schedule and the first stage at once, for at most 64 sequences and fewer than 2^31 stages:
  // every sequence's sizes are read once, into a lane, and what follows from them is 32-bit
  // arithmetic on registers.  It stands in front of a workgroup's first load, and a small call is
  // little else: 1 x 32 units of 64 queries x 1024 keys 19.8 -> 18.2 us for the call, 8 x 16 x 64 x 2048 (d =
  // 64) 35.0 -> 33.1, against loads per question, sums through LDS and 64-bit divisions.  (With ranges
  // that cross no unit and two waves per 32 queries these calls take 14.2 and 26.4 us now.)
  template <int D, int KS>
  __device__ __forceinline__ int begin_one_pass(const StageMap &m, Schedule &sc, int w, int G) {
    const int lane = threadIdx.x & 63, H = m.H;
    int len_l = m.seq_lens[lane < m.B ? lane : 0], nodes_l = m.n_nodes[lane < m.B ? lane : 0];
    len_l = len_l < 0 ? 0 : (len_l > m.L_max ? m.L_max : len_l);
    nodes_l = nodes_l < 1 ? 1 : (nodes_l > m.T_max ? m.T_max : nodes_l);
    const int us_l = lane < m.B ? (len_l + kStageRows - 1) / kStageRows + (nodes_l + kStageRows - 1) / kStageRows : 0;
    const int incl = wave_scan_i32(us_l, 0, [](int x, int y) { return x + y; });
    const uint32_t n_all = (uint32_t)(H * __builtin_amdgcn_readlane(incl, 63)), U = (uint32_t)(m.B * H);
    auto take_sizes = [&](int at) {
      b = at;
      L = __builtin_amdgcn_readlane(len_l, at);
      T = __builtin_amdgcn_readlane(nodes_l, at);
      cs = (L + kStageRows - 1) / kStageRows;
      ts = (T + kStageRows - 1) / kStageRows;
    };
    // ---- Ranges that cross no unit, where that makes the longest of them not much longer: a range of two
    //      units waits for queries and stores partials twice, 3 to 4 us after the others are done, and a
    //      unit in one piece needs no merge.  The longest range q is the least for which the pieces of
    //      all units, ceil(stages / q) each, fit the grid (a candidate per lane).
    if (U <= (uint32_t)G) {
      const float mean = (float)n_all * __builtin_amdgcn_rcpf((float)G);
      const uint32_t least_q = (n_all + (uint32_t)G - 1u) / (uint32_t)G, q = least_q + (uint32_t)lane;
      const float inv = __builtin_amdgcn_rcpf((float)q), up = ((float)q - .5f) * inv;
      float total = 0.f;  // beyond 2^24 not exact, and far beyond any grid
      const float us_f = (float)us_l;
      for (int i = 0; i < m.B; ++i)
        total += ceil_quotient(__uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(us_f), i)), inv, up);
      total *= (float)H;
      const uint64_t fit = __ballot(total <= (float)G), fit_cus = __ballot(total <= (float)m.cus);
      int pick = -1;
      if (fit != 0) {
        pick = __builtin_ctzll(fit);
        const float pieces = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(total), pick));
        const float longest = (float)(least_q + (uint32_t)pick);
        // How much longer: the more units there are for each workgroup, the more of them a range crosses, at a cost that does not grow
        // with its length.  Whole calls, us, at mean / longest stages, crossing / not: ragged lengths, 496 units 9.0 / 17 35.5 / 30.4,
        // 352 11.9 / 19 38.9 / 31.1, 280 22.9 / 32 57.8 / 48.5, 336 48.2 / 66 96.0 / 90.1, 256 32.8 / 46 64.3 / 60.0, 320 37.3 / 63
        // 73.7 / 86.5, 160 44 / 60 70.3 / 73.9; equal ones, 80 7.3 / 8 29.8 / 26.8, 200 (two waves per 32 queries) 84.8 / 109 134.1 /
        // 126.1, 200 (one) 67 / 86 120.3 / 126.2, 176 6.2 / 9 22.1 / 23.6.  In one piece each: 312 units of 57 queries 28.6 / 47 59.5 /
        // 53.7, 320 of 61 34.4 / 55 66.3 / 61.3, 352 of 15 105 / 153 150.9 / 156.2, 320 of 89 4.4 / 7 26.9 / 21.5, 320 of 104 86 / 137
        // 153.8 / 165.4.
        const float share = (float)U * __builtin_amdgcn_rcpf((float)G);
        const float one_each = KS == 2 ? 1.3f * mean + 11.f : 1.2f * mean + 8.f;
        const float several = fminf((1.f + (share < .5f ? .8f : 1.1f) * share) * mean + 1.f, (KS == 2 ? 1.25f : 1.15f) * mean + 17.f * share);
        // And by how many stages at most: a stage more costs 0.5 us and up where stages are bound by their chain (d = 64) and where
        // the trees are so small that rows come faster (T_max <= 8), against the 3 to 5 us that a crossing costs.  Whole calls, us, at
        // mean / longest stages, crossing / not: d = 64, equal lengths, 432 units 34.6 / 41 48.7 / 47.2, 372 27.6 / 38 37.8 / 40.1,
        // 336 40 / 61 47.2 / 57.5, two pieces each (one wave per 32 queries) 120 34 / 37 67.9 / 64.5, 152 29.4 / 33 52.5 / 54.3, 208 50 / 62 77.0
        // / 84.5; ragged, 416 19.1 / 30 34.3 / 28.9, 264 47.7 / 61 58.0 / 61.2.  d = 128, 1 to 8 queries, 416 27.6 / 34 45.2 / 43.9, 264 8.2 / 16
        // 19.1 / 21.0, 304 24.3 / 41 40.1 / 43.6, 444 51 / 59 79.4 / 72.8; several pieces each, 480 15.9 / 30 41.8 / 37.2, 208 61.8 / 76 91.1 /
        // 93.2, 296 48.1 / 68 78.7 / 83.0 (one each: 376 63.9 / 87 101.5 / 93.0).
        const bool same = __ballot(lane < m.B && us_l != __builtin_amdgcn_readfirstlane(us_l)) == 0;
        const bool one = pieces <= (float)U;
        const float more = D == 64 ? (same ? (KS == 1 && !one ? 3.3f : 6.5f) : 11.f) : (m.T_max <= 8 ? 14.f * share : one ? 1e9f : 14.15f);
        const float limit = fminf(one ? one_each : several, mean + more);
        // One wave per 32 queries and fewer workgroups left than half the chip: ranges that cross units stay, since which side is
        // faster depends on the number of stages.  Whole calls, us, crossing / not: 9 to 21 stages per unit 12.8 / 14.1 (1 x 8 units of 92 x 362), 14.2 / 14.9 (5 x 4 of 68 x 384), 12.5 /
        // 13.1 (d = 64, 3 of 85 x 180), 12.5 / 13.9 (d = 64, 16 of 127 x 136); 5 to 7 13.1 / 12.0 (3 of 74 x 100), 13.9 / 14.5 (2 x 16 of
        // 113 x up to 31); 27 and more 13.3 / 12.3 (2 x 2 of 69 x 754).  24 of random sizes: not crossing 0.89 to 1.10 of the time, 0.96 on average.
        if (longest > limit || (KS == 1 && pieces < .5f * (float)m.cus && pick > 0)) pick = -1;
        // Fewer, longer pieces, one workgroup per compute unit, where a unit would be cut into many: 32 units of 34 stages in 12 / 7
        // pieces 15.5 / 14.2, 8 of 247 in 62 / 31 22.7 / 18.6; 64 units in 8 / 4 20.8 / 21.4.  24 calls of random sizes to which it
        // applies: 1.10 times as fast on average, 0.94 to 1.35 (1 x 2 units of 33 x 2065 13.2 / 14.0, 5 x 4 of 114 x up to 1482 23.0 / 17.1).
        if (pick >= 0 && pieces > 8.f * (float)U && fit_cus != 0 && least_q + (uint32_t)__builtin_ctzll(fit_cus) <= 8u)
          pick = __builtin_ctzll(fit_cus);
      }
      if (pick >= 0) {
        const float inv_q = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(inv), pick));
        const float up_q = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(up), pick));
        const int mine = lane < m.B ? (int)ceil_quotient(us_f, inv_q, up_q) : 0;
        const int wgs_before = H * (wave_scan_i32(mine, 0, [](int x, int y) { return x + y; }) - mine);
        whole_left = 0;
        take_sizes(__popcll(__ballot(lane < m.B && wgs_before <= w)) - 1);
        const uint32_t at = (uint32_t)(w - __builtin_amdgcn_readlane(wgs_before, b)), P = (uint32_t)__builtin_amdgcn_readlane(mine, b);
        const float inv_p = __builtin_amdgcn_rcpf((float)P);
        const uint32_t head = (uint32_t)floor_quotient((float)at, inv_p), piece = at - head * P;
        sc.pieces = (int)P;
        sc.anew = (int)fminf((KS == 1 ? (mean < 5.f ? .67f : .5f) : mean < 6.f ? 1.f : .6f) * mean, 32.f);
        sc.anew = sc.anew > 1 ? sc.anew : 1;
        unit = split_unit = (long long)(b * H) + (head < (uint32_t)H ? head : 0);
        const uint32_t quot = (uint32_t)floor_quotient((float)(cs + ts), inv_p), rem = (uint32_t)(cs + ts) - quot * P;
        s = split_s = (int)(piece * quot + (piece < rem ? piece : rem));
        return head < (uint32_t)H ? (int)(quot + (piece < rem ? 1u : 0u)) : 0;  // 0: past the last unit
      }
    }
    const int most = wave_scan_i32(us_l, 0, [](int x, int y) { return x > y ? x : y; });
    const int least = wave_scan_i32(lane < m.B ? us_l : 1 << 30, 1 << 30, [](int x, int y) { return x < y ? x : y; });
    const int us_max = __builtin_amdgcn_readlane(most, 63), us_min = __builtin_amdgcn_readlane(least, 63);
    const int before_l = H * (incl - us_l);  // stages of the units of the sequences before
    sc.k = (us_max - us_min) * 32 <= us_max ? (int)(U / (uint32_t)G) : 0;
    sc.first_split = sc.k * G;
    uint32_t split_base = 0;
    if (sc.k > 0) {
      const int bs = sc.k * G / H;
      split_base = bs < m.B ? (uint32_t)(__builtin_amdgcn_readlane(before_l, bs) +
                                         (sc.k * G - bs * H) * __builtin_amdgcn_readlane(us_l, bs))
                            : n_all;
    }
    const uint32_t n_split = n_all - split_base, quot = n_split / (uint32_t)G, rem = n_split - quot * (uint32_t)G;
    sc.split_base = split_base;
    sc.n_split = n_split;
    sc.quot = quot;
    sc.rem = rem;
    const uint32_t x0 = (uint32_t)w * quot + ((uint32_t)w < rem ? (uint32_t)w : rem);
    int n_my = (int)(quot + ((uint32_t)w < rem ? 1u : 0u));
    x_end = x0 + (uint32_t)n_my;
    // the sequence that holds stage split_base + x0 is the last one that starts at or before it
    const uint32_t x = split_base + x0;
    const uint64_t starts = __ballot(lane < m.B && (uint32_t)before_l <= x);
    take_sizes(__popcll(starts) - 1);
    const uint32_t in_seq = x - (uint32_t)__builtin_amdgcn_readlane(before_l, b), hh = in_seq / (uint32_t)(cs + ts);
    split_unit = (long long)((uint32_t)(b * H) + hh);
    split_s = (int)(in_seq - hh * (uint32_t)(cs + ts));
    if (split_unit >= (long long)U) {  // an empty range at the very end: stay on valid memory
      split_unit = U - 1;
      split_s = 0;
    }
    whole_left = sc.k;
    unit = split_unit;
    s = split_s;
    if (sc.k > 0) {
      for (int j = 0; j < sc.k; ++j) n_my += __builtin_amdgcn_readlane(us_l, (w + j * G) / H);
      unit = w;
      s = 0;
      take_sizes(w / H);
    }
    return n_my;
  }
  __device__ __forceinline__ void advance(const StageMap &m, long long G, int n) {
    s += n;  // n <= stages left in the unit
    if (s < cs + ts) return;
    s = 0;
    if (whole_left > 0) {
      if (--whole_left > 0) {
        set_unit(m, unit + G);
      } else {
        set_unit(m, split_unit);
        s = split_s;
      }
    } else if (unit + 1 < (long long)m.B * m.H) {
      set_unit(m, unit + 1);
    }
  }
};

// Values of V that are not finite.  The tiled kernels multiply every row of a tile by a weight,
// zero for the rows that a query does not see (or that weigh less than the smallest number), and zero
// times such a value is NaN.  D = 64 and fp32 operands keep these values to the queries that give them
// weight: a tile is multiplied with zeros in the place of such values, and with a code in their place and
// zero for all others by weights of 0 and 1.  The sum of the codes tells how many +inf, -inf and NaN
// (at most 32 of each) the query sees in that column, and what to add to its result.
//   fp32: tiles that have weights of zero (tree rows; hardly any other) and such a value.  With a NaN in
//     every unit 2 x 16 units of 48 queries x 1024 keys take 31 us instead of 28, by HIP events.
//   D = 64: a weight of three parts has zeros among them in any tile, and looking through every
//     tile costs 1 us of 34, so a piece whose results hold a NaN is done once more: 83 us instead
//     of 38 where every unit of 8 x 16 has one (64 queries x 2048 keys; 0.6 us for the question).
constexpr float kCodePlus = 1.f, kCodeMinus = 64.f, kCodeNan = 4096.f;  // exact in bf16, sums exact in fp32
__device__ __forceinline__ float not_finite_sum(float codes) {
  const int n = (int)codes;
  float x = (n & 63) != 0 ? INFINITY : 0.f;
  x -= ((n >> 6) & 63) != 0 ? INFINITY : 0.f;
  return (n >> 12) != 0 ? __uint_as_float(0x7fc00000u) : x;
}
// the code of a value, 0 for a finite one
__device__ __forceinline__ float not_finite_code(uint32_t bits) {
  const uint32_t mag = bits & 0x7fffffffu;
  return mag < 0x7f800000u ? 0.f : mag > 0x7f800000u ? kCodeNan : bits >> 31 ? kCodeMinus : kCodePlus;
}
// both halves of a bf16 pair: their codes as a pair; the halves that have one become zero
__device__ __forceinline__ uint32_t take_not_finite(uint32_t &pair) {
  const uint32_t lo = __float_as_uint(not_finite_code(pair << 16)) >> 16;
  const uint32_t hi = __float_as_uint(not_finite_code(pair & 0xffff0000u)) & 0xffff0000u;
  pair &= (lo ? 0u : 0xffffu) | (hi ? 0u : 0xffff0000u);
  return lo | hi;
}

template <int MB>
__device__ __forceinline__ bool has_nan(const f32x16 (&o)[MB]) {
  float sum = 0.f;  // NaN as soon as a term is (and for +inf - inf)
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int r = 0; r < 16; ++r) sum += o[mb][r];
  return sum != sum;
}

// x * a + y * b; D = 64: an infinity in a piece that counts for nothing is left out
template <int D>
__device__ __forceinline__ float merge_add(float x, float a, float y, float b) {
  if constexpr (D == 64) {
    x = a == 0.f ? 0.f : x;
    y = b == 0.f ? 0.f : y;
  }
  return x * a + y * b;
}

// KS: waves per 32 queries.  1: the four waves split up to 128 queries.  2 (trees of at most 64 nodes, where
// half of the waves would only load): a wave takes 16 of a stage's 32 rows, with 16x16x32 products for the
// scores and 32x32x16, 16 keys deep, for the weighted sum, and the two waves of a query group merge
// their results through LDS at the end of a piece.  That halves the chain of a stage, which bounds
// the kernel at D = 64 (8 x 16 units, 64 queries, 2048 keys: 29.2 -> 26.4 us for the call; 96 x 50 x 2135 26.4 ->
// 23.4), pays at D = 128 where a workgroup has one piece (372 units x 49 x 5383 187 -> 178) and costs where it has
// many short ones (800 ragged units of up to 834 keys 37.2 -> 37.9, see propd_tree_attention).
// kAnew: see Schedule::anew.
// D = 128 multiplies bf16 weights with V.  D = 64 keeps them in fp32: a weight is the sum of three
// bf16 values, 8 of its 24 bits each, all of which are multiplied.  (With two of them a weight
// is off by up to 2^-17.  8 x 16 units of 64 queries x 2048 keys, whole call: 33.8 us, 30.7 with two.)
template <int NS, int D, int KS, bool kAnew>
__global__ __launch_bounds__(kAttnThreads, Geo<D>::kPerCu) void tree_attn_bf16_kernel(AttnParams p) {
  using G_ = Geo<D>;
  constexpr int kRowBytes = G_::kRowBytes, kHalfStage = G_::kHalfStage, kStageBytes = G_::kStageBytes;
  constexpr int kMb = G_::kMb, kLoads = G_::kLoads;
  constexpr int kQf = D / 16, kKs = kQf / KS;    // registers of 16 bytes of a lane's queries; MFMA steps over d of QK^T
  constexpr int kRegs = 16 / KS, kVSteps = 2 / KS;  // scores of a lane per stage; MFMA steps over the keys of PV
  constexpr bool kExact = D == 64;  // weights of fp32 precision, in several bf16 values
  constexpr int kParts = kExact ? 3 : 1;
  static_assert(NS >= 4, "three stages are in use by the math, the rest is in flight");
  constexpr int kAhead = NS - 3;  // stages in flight beyond the newest one the math uses
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const uint32_t smem_base = (uint32_t)(uintptr_t)(lds_void *)smem;  // LDS byte address of the ring

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, g = lane >> 5;
  const int q_group = KS == 1 ? wave : wave & 1, k_part = KS == 1 ? 0 : wave >> 1;
  const int t = q_group * 32 + l32;  // this lane's query column

  const StageMap map = {p.B, p.H, p.seq_lens, p.n_nodes, p.L_max, p.T_max, p.cus};
  const long long G = gridDim.x, w = blockIdx.x;
  Schedule sch;
  Walk cp;
  int n_my;
  if (p.one_pass) {
    n_my = cp.template begin_one_pass<D, KS>(map, sch, (int)w, (int)G);
  } else {
    sch = make_schedule(map, G);
    n_my = cp.start(map, sch, w, G);
  }
  CutRecord cut = {-1, 0, (int32_t)w, 0};
  auto leave_record = [&](long long at) {
    if (tid == 0) *reinterpret_cast<CutRecord *>(p.cuts + 4 * at) = cut;
  };
  if (n_my <= 0) {
    if (!p.by_unit) leave_record(w);
    return;
  }

  // ---- loader.  It walks the same stage list ahead of the math, one segment (the cached
  //      rows or the tree rows of a unit) at a time.  One direct load moves 64 lanes x 16
  //      bytes = 4 rows into 1 KB of LDS that is contiguous in lane order, so the swizzle is
  //      applied on the global side: the lane that fills chunk c of LDS row r fetches chunk
  //      c ^ key(r) of the global row.  A wave fills kLdRows consecutive rows per load, of each
  //      block of 4 * kLdRows rows; its keys do not depend on the block.  Rows past the last
  //      valid one of a segment re-read that last row: finite data that the mask discards (K) or
  //      that meets a zero weight (V); padding is never touched.
  constexpr int kLdRows = G_::kLdRows;
  const int ld_row = kLdRows * wave + lane / G_::kChunks;
  const int k_lane_chunk = ((lane % G_::kChunks) ^ G_::k_key(ld_row)) << 4;
  const int v_lane_chunk = ((lane % G_::kChunks) ^ G_::v_key(ld_row)) << 4;
  Walk lw = cp;  // the next stage to issue
  int ld_rows;                       // rows left in the segment, from the next stage to issue
  const unsigned char *ld_k, *ld_v;  // first row of the next stage to issue
  auto ld_segment = [&]() {          // the segment (cached or tree rows) that stage lw.s starts
    const bool tree = lw.s >= lw.cs;
    const int first_row = (tree ? lw.s - lw.cs : lw.s) * kStageRows;
    ld_rows = (tree ? lw.T : lw.L) - first_row;
    const size_t row0 = (size_t)lw.unit * (tree ? p.T_max : p.L_max) + first_row;
    ld_k = reinterpret_cast<const unsigned char *>(tree ? p.k_tree : p.k_cache) + row0 * kRowBytes;
    ld_v = reinterpret_cast<const unsigned char *>(tree ? p.v_tree : p.v_cache) + row0 * kRowBytes;
  };
  ld_segment();
  auto dma16 = [&](const unsigned char *src, unsigned char *dst) {
    __builtin_amdgcn_global_load_lds((global_void *)src, (lds_void *)dst, 16, 0, 2 /* nt */);
  };
  auto issue = [&](int slot) {
    unsigned char *dst = smem + slot * kStageBytes + wave * 1024;
    if (ld_rows >= kStageRows) {
#pragma unroll
      for (int i = 0; i < kLoads; ++i) {
        const int ro = (4 * kLdRows * i + ld_row) * kRowBytes;
        dma16(ld_k + (ro + k_lane_chunk), dst + i * 4096);
        dma16(ld_v + (ro + v_lane_chunk), dst + kHalfStage + i * 4096);
      }
    } else {
#pragma unroll
      for (int i = 0; i < kLoads; ++i) {
        int row = 4 * kLdRows * i + ld_row;
        row = row < ld_rows ? row : ld_rows - 1;
        dma16(ld_k + (row * kRowBytes + k_lane_chunk), dst + i * 4096);
        dma16(ld_v + (row * kRowBytes + v_lane_chunk), dst + kHalfStage + i * 4096);
      }
    }
    lw.advance(map, G, 1);
    if (ld_rows > kStageRows) {
      ld_rows -= kStageRows;
      ld_k += kHalfStage;
      ld_v += kHalfStage;
    } else {
      ld_segment();  // the tree rows of the unit, or another unit
    }
  };

  // ---- per-lane LDS read offsets within a stage
  // K as the A operand of S^T: lane = row l32, 8 consecutive d from 16*ks + 8*g (chunk 2*ks + g)
  uint32_t k_rd[kKs];
#pragma unroll
  for (int ks = 0; ks < kKs; ++ks) {
    const int r = KS == 1 ? l32 : 16 * k_part + (lane & 15), chunk = KS == 1 ? 2 * ks + g : 4 * ks + (lane >> 4);
    k_rd[ks] = smem_base + r * kRowBytes + ((chunk ^ G_::k_key(r)) << 4);
  }
  // V^T as the A operand of O^T: transposing read; in each group of 16 lanes, lane i points at
  // row i/4, 4 columns from 4*(i%4), and receives column i of those 4 rows.  Per MFMA k-step
  // (16 rows): slots 0..3 = rows 4g + 0..3, slots 4..7 = those rows + 8.
  uint32_t v_rd[kMb][2];
#pragma unroll
  for (int mb = 0; mb < kMb; ++mb)
#pragma unroll
    for (int hi = 0; hi < 2; ++hi) {
      const int r = (KS == 1 ? 4 * g + 8 * hi : 16 * k_part + 8 * g + 4 * hi) + ((lane & 15) >> 2);
      const int chunk = mb * 4 + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
      v_rd[mb][hi] = smem_base + kHalfStage + r * kRowBytes + ((chunk ^ G_::v_key(r)) << 4) + 8 * (lane & 1);
    }

  // ---- ring bookkeeping.  acquire() is called once per stage of the range, in order, by
  //      every wave: it waits for the stage's loads, meets the other waves, and refills the
  //      slot whose stage every wave finished two acquires ago.  Vector memory loads of a
  //      wave complete in issue order, so "stage x has landed" is "at most one stage's operations
  //      outstanding": the loads of stage x+1.  Query loads and output stores that the wave
  //      issued since then are waited for as well (loads and stores are not ordered against
  //      each other, so the stores cannot be counted off).
  static_assert(kAhead == 2, "the wait below allows exactly one younger stage in flight");
  int n_acq = 0;              // stages acquired so far
  int slot_acq = 0;           // slot of the next stage to acquire
  int slot_ld = 0;            // slot of the next stage to issue
  auto next_slot = [](int sl) { return sl + 1 == NS ? 0 : sl + 1; };
  auto fill_ring = [&]() {
#pragma unroll
    for (int i = 0; i < kAhead; ++i)
      if (n_acq + i < n_my) {
        issue(slot_ld);
        slot_ld = next_slot(slot_ld);
      }
  };
  auto acquire = [&]() -> int {
    if (n_acq + 1 < n_my) wait_vmem<2 * kLoads>(); else wait_vmem<0>();
    __builtin_amdgcn_s_barrier();
    if (n_acq + kAhead < n_my) {
      issue(slot_ld);
      slot_ld = next_slot(slot_ld);
    }
    const int sl = slot_acq;
    slot_acq = next_slot(slot_acq);
    ++n_acq;
    return sl;
  };

  // ---- a piece: the part of one unit that lies in this range
  struct Piece {
    int L, T, n_cache, s0, n_st, unit, b, n_cmp;
    bool whole;
  };
  auto piece_at = [&](const Walk &c, int n_done) {
    Piece pc;
    pc.L = c.L;
    pc.T = c.T;
    pc.n_cache = c.cs;
    pc.s0 = c.s;
    const int us = c.cs + c.ts;
    pc.n_st = us - c.s < n_my - n_done ? us - c.s : n_my - n_done;
    pc.whole = c.s == 0 && pc.n_st == us;
    pc.unit = (int)c.unit;
    pc.b = c.b;
    // Stages this wave has math for: none if its 32 query columns lie beyond the tree; tree
    // rows after its last query are descendants or strangers of all its queries, and those
    // stages are the last of the unit.
    pc.n_cmp = 0;
    if (q_group * 32 < c.T) {
      pc.n_cmp = c.cs + q_group + 1 - c.s;
      pc.n_cmp = pc.n_cmp > pc.n_st ? pc.n_st : (pc.n_cmp < 0 ? 0 : pc.n_cmp);
    }
    return pc;
  };

  // Q^T fragments (B operand: lane = query column, 8 consecutive d per K step) and the
  // ancestor set of this lane's node.  Lanes past the tree take node 0: valid memory, and
  // their columns are never stored.
  u32x4 qf[kQf], ancv;
  // D = 64: left to the compiler, whose waits come where wait_queries() waits for everything anyway
  auto load16 = [](const void *ptr) {
    if constexpr (kExact) return *reinterpret_cast<const u32x4 *>(ptr);
    else return global_load16_untracked(ptr);
  };
  auto load_queries = [&](const Piece &pc) {
    const int tq = t < pc.T ? t : 0;
    if constexpr (KS == 1) {
      const uint16_t *qrow = p.q + ((size_t)pc.unit * p.T_max + tq) * D + g * 8;
#pragma unroll
      for (int ks = 0; ks < kKs; ++ks) qf[ks] = load16(qrow + ks * 16);
    } else {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int t16 = 32 * q_group + 16 * j + (lane & 15);
        const uint16_t *qrow = p.q + ((size_t)pc.unit * p.T_max + (t16 < pc.T ? t16 : 0)) * D + (lane >> 4) * 8;
#pragma unroll
        for (int ks = 0; ks < kKs; ++ks) qf[j * kKs + ks] = load16(qrow + ks * 32);
      }
    }
    ancv = load16(p.anc + ((size_t)pc.b * p.T_max + tq) * 2);
  };
  auto wait_queries = [&]() {
    // the registers are named so that their uses cannot be scheduled above the wait
    auto tie = [&]() {
#pragma unroll
      for (int ks = 0; ks < kQf; ++ks) asm volatile("" : "+v"(qf[ks]));
      asm volatile("" : "+v"(ancv));
    };
    tie();
    // the first piece's were requested before the ring's loads, the first stage of which has landed
    if (kExact || n_acq != 1) wait_vmem<0>();
    tie();
  };

  float m_run, l_run, m_top;  // the softmax reference, the sum of the weights, the piece's highest score so far (kAnew)
  f32x16 o_acc[kMb];
  u32x2 vt[kVSteps][2 * kMb];
  // S^T = K . Q^T of one stage
  struct Scores {
    f32x16 all;      // KS = 1
    f32x4 half[2];   // KS = 2: 16 keys x 16 queries, twice
  };
  auto scores = [&](int sl) -> Scores {
    const uint32_t so = (uint32_t)sl * kStageBytes;
    Scores acc;
    if constexpr (KS == 1) {
#pragma unroll
      for (int r = 0; r < 16; ++r) acc.all[r] = 0.f;
    } else {
      acc.half[0] = acc.half[1] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int ks = 0; ks < kKs; ++ks) {
      const bf16x8 a = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8 *>(
          (uintptr_t)(k_rd[ks] + so));
      if constexpr (KS == 1) {
        acc.all = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8, qf[ks]), acc.all, 0, 0, 0);
      } else {
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc.half[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, qf[j * kKs + ks]), acc.half[j], 0, 0, 0);
      }
    }
    return acc;
  };
  // The scores of this lane's query, once they are there.  KS = 1: register r is key row 8 * (r / 4) + 4 * g +
  // r % 4 of the stage.  KS = 2: half j of a lane holds query 16 * j + lane % 16 and keys 4 * (lane / 16) + r; the
  // odd rows of 16 lanes of half 0 and the even ones of half 1 are exchanged, after which register r is
  // query t and key row 16 * k_part + 8 * g + r.
  auto take_scores = [&](const Scores &acc, float (&sc)[kRegs]) {
    if constexpr (KS == 1) {
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[r] = acc.all[r];
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc.half[0][r]), __float_as_uint(acc.half[1][r]), false, false);
        sc[r] = __uint_as_float(x[0]);
        sc[4 + r] = __uint_as_float(x[1]);
      }
    }
  };
  // start the transposing reads of a whole V stage: vt[ks2][2*mb + hi]
  auto read_v = [&](int sl) {
    const uint32_t so = (uint32_t)sl * kStageBytes;
#pragma unroll
    for (int mb = 0; mb < kMb; ++mb) {
      vt[0][2 * mb] = lds_read_tr16<0>(v_rd[mb][0] + so);
      vt[0][2 * mb + 1] = lds_read_tr16<0>(v_rd[mb][1] + so);
    }
    if constexpr (KS == 1) {
#pragma unroll
      for (int mb = 0; mb < kMb; ++mb) {
        vt[1][2 * mb] = lds_read_tr16<16 * kRowBytes>(v_rd[mb][0] + so);
        vt[1][2 * mb + 1] = lds_read_tr16<16 * kRowBytes>(v_rd[mb][1] + so);
      }
    }
  };
  // D = 64, a piece done for the second time: V values that are not finite are taken out of the V
  // registers read last, and what they add to O is added
  bool careful = false;
  auto take_out = [&](const uint32_t (&pw)[kParts][kRegs / 2]) __attribute__((always_inline)) {
    if (!kExact || !careful) return;
    wait_lds<0>(vt[0]);
    if constexpr (KS == 1) wait_lds<0>(vt[1]);
#pragma unroll
    for (int mb = 0; mb < kMb; ++mb) {
      f32x16 codes;
#pragma unroll
      for (int r = 0; r < 16; ++r) codes[r] = 0.f;
#pragma unroll
      for (int ks2 = 0; ks2 < kVSteps; ++ks2) {
        uint32_t v4[4] = {vt[ks2][2 * mb].x, vt[ks2][2 * mb].y, vt[ks2][2 * mb + 1].x, vt[ks2][2 * mb + 1].y};
        u32x4 code, seen;  // seen: 1 for a weight
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const uint32_t w2 = pw[0][4 * ks2 + x];
          seen[x] = (w2 & 0xffffu ? 0x3f80u : 0u) | (w2 >> 16 ? 0x3f800000u : 0u);
          code[x] = take_not_finite(v4[x]);
        }
        vt[ks2][2 * mb] = u32x2{v4[0], v4[1]};
        vt[ks2][2 * mb + 1] = u32x2{v4[2], v4[3]};
        codes = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, code),
                                                        __builtin_bit_cast(bf16x8, seen), codes, 0, 0, 0);
      }
      mfma_settle();  // O too: its last products came before
#pragma unroll
      for (int r = 0; r < 16; ++r) o_acc[mb][r] += not_finite_sum(codes[r]);
    }
  };
  // O^T += V^T . P^T with the V registers read last and the given weights
  auto weighted_sum = [&](const uint32_t (&pw)[kParts][kRegs / 2]) {
    wait_lds<0>(vt[0]);
    if constexpr (KS == 1) wait_lds<0>(vt[1]);
#pragma unroll
    for (int ks2 = 0; ks2 < kVSteps; ++ks2) {
#pragma unroll
      for (int part = kParts - 1; part >= 0; --part) {  // the small parts first
        const u32x4 pv = {pw[part][4 * ks2], pw[part][4 * ks2 + 1], pw[part][4 * ks2 + 2], pw[part][4 * ks2 + 3]};
        const bf16x8 pf = __builtin_bit_cast(bf16x8, pv);
#pragma unroll
        for (int mb = 0; mb < kMb; ++mb) {
          const u32x4 aw = {vt[ks2][2 * mb].x, vt[ks2][2 * mb].y, vt[ks2][2 * mb + 1].x,
                            vt[ks2][2 * mb + 1].y};
          o_acc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, aw), pf,
                                                              o_acc[mb], 0, 0, 0);
        }
      }
    }
  };

  // whether `mine` holds in any wave of the workgroup (which all come here)
  __shared__ int s_any[2];
  int n_any = 0;  // calls so far: a call leaves its number, the one before it is then no longer looked at
  if constexpr (kExact) {
    if (tid < 2) s_any[tid] = 0;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // seen by all after the first stage's barrier
  }
  auto any_wave = [&](bool mine) {
    ++n_any;
    int *word = s_any + (n_any & 1);
    if (mine) *word = n_any;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    return __builtin_amdgcn_readfirstlane(*word) == n_any;
  };

  auto put_blocks = [&](uint32_t at, auto from) __attribute__((always_inline)) {
    static_for_i<kMb / KS * 4>([&](auto x) __attribute__((always_inline)) {
      constexpr int X = decltype(x)::value, mb = decltype(from)::value + X / 4, q4 = X % 4;
      lds_write16<1024 * X>(at, f32x4{o_acc[mb][4 * q4], o_acc[mb][4 * q4 + 1], o_acc[mb][4 * q4 + 2], o_acc[mb][4 * q4 + 3]});
    });
  };
  const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3f803f80u);
  // a new running maximum is adopted only when it exceeds the reference by 2^8 in the
  // exponent; below that the weights simply exceed 1, by a factor fp32 sums and bf16 hold
  // D = 64: the reference is put 2^4 above the maximum instead, and adopted anew when that is
  // exceeded, so that weights are at most 1 and no product leaves the range of its V value
  // (finite, also where the scale is next to nothing)
  const float tau = fminf((kExact ? 4.f : 8.f) / p.scale_log2e, 1e38f);

  Piece pc = piece_at(cp, 0);
  // D = 128: the first piece's queries in front of the ring's loads, which they then need not be waited for behind
  // (15.8 -> 14.5 us at 32 units of 64 x 1024).  D = 64, where the compiler waits for them, the other way.
  if (kExact) fill_ring();
  if (pc.n_cmp > 0) load_queries(pc);
  if (!kExact) fill_ring();
  while (n_acq < n_my) {
    const int L = pc.L, T = pc.T, n_cache = pc.n_cache, s0 = pc.s0;
    m_run = m_top = -INFINITY;
    l_run = 0.f;
#pragma unroll
    for (int mb = 0; mb < kMb; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) o_acc[mb][r] = 0.f;

    if (pc.n_cmp > 0) {
      // The loop is software-pipelined over stages so that matrix and vector work of
      // different stages sit in one basic block: iteration i computes the scores of stage
      // i+1 (MFMA), the softmax weights of stage i (VALU), and adds stage i-1 to O (MFMA).
      int sl_cur = acquire();
      wait_queries();
      const uint64_t anc_lo = ((uint64_t)ancv.y << 32) | ancv.x, anc_hi = ((uint64_t)ancv.w << 32) | ancv.z;
      Scores raw = scores(sl_cur);
      uint32_t pw_prev[kParts][kRegs / 2];
      auto clear_prev = [&]() {
#pragma unroll
        for (int part = 0; part < kParts; ++part)
#pragma unroll
          for (int r = 0; r < kRegs / 2; ++r) pw_prev[part][r] = 0u;
      };
      clear_prev();
      int next_anew = sch.anew;

      auto stage = [&](int i, auto has_next, auto has_prev) {
        constexpr bool kNext = decltype(has_next)::value, kPrev = decltype(has_prev)::value;
        int sl_next = 0;
        if (kNext) sl_next = acquire();
        mfma_settle();  // raw was written by MFMAs of the previous iteration or the prologue
        float sc[kRegs];
        take_scores(raw, sc);

        const int s = s0 + i;
        const bool is_tree = s >= n_cache;
        const int j0 = (is_tree ? s - n_cache : s) * kStageRows;
        int n_valid = (is_tree ? T : L) - j0;
        n_valid = n_valid > kStageRows ? kStageRows : n_valid;
        // ---- mask (the softmax scale is positive, so it commutes with max and is applied
        //      inside the exponent).  Register r holds K/V row j0 + 8*(r/4) + 4*g + r%4 (KS = 1) or
        //      j0 + 16*k_part + 8*g + r (KS = 2), see take_scores.
        if (is_tree || n_valid < kStageRows) {  // uniform over the workgroup
          // visibility of the stage's rows to this lane's query: cached rows below L for
          // every query, tree rows only where the node's ancestor set has the bit
          uint32_t vis = n_valid >= 32 ? ~0u : ((1u << n_valid) - 1u);
          const uint64_t word = j0 >= 64 ? anc_hi : anc_lo;  // tree stages start at 0, 32, 64, 96
          vis &= is_tree ? (uint32_t)(word >> (j0 & 32)) : ~0u;
          vis >>= KS == 1 ? 4 * g : 16 * k_part + 8 * g;
#pragma unroll
          for (int r = 0; r < kRegs; ++r)
            sc[r] = ((vis >> (KS == 1 ? 8 * (r >> 2) + (r & 3) : r)) & 1u) ? sc[r] : -INFINITY;
        }
        // ---- running maximum
        float m_blk = -INFINITY;
#pragma unroll
        for (int r = 0; r < kRegs; ++r) m_blk = fmaxf(m_blk, sc[r]);
        {  // the other half of the stage's rows is in the lane 32 away
          uint32_t lo = __float_as_uint(m_blk), hi = lo;
          swap_halves(lo, hi);
          m_blk = fmaxf(__uint_as_float(lo), __uint_as_float(hi));
        }
        if constexpr (kAnew) m_top = fmaxf(m_top, m_blk);
        const bool anew = kAnew && i == next_anew;  // uniform
        if (anew) next_anew += sch.anew;
        if (anew || __builtin_amdgcn_ballot_w64(m_blk > (kExact ? m_run : m_run + tau)) != 0) {
          // rare: move the reference.  O must first receive the stage still pending, whose
          // weights are relative to the old reference.
          if (kPrev) {
            take_out(pw_prev);
            weighted_sum(pw_prev);
            clear_prev();
            mfma_settle();
          }
          // Set anew it may come down, but to no less than the highest score so far - tau: no weight exceeds
          // 2^8 then, however many stages of low scores follow a high one.
          const float m_new = fmaxf(anew ? m_top - tau : m_run, kExact ? m_blk + tau : m_blk);
          const float m_safe = m_new == -INFINITY ? 0.f : m_new;
          const float alpha = fast_exp2((m_run - m_safe) * p.scale_log2e);
          l_run *= alpha;
#pragma unroll
          for (int mb = 0; mb < kMb; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r) o_acc[mb][r] *= alpha;
          m_run = m_new;
        }
        const float neg_m = -(m_run == -INFINITY ? 0.f : m_run) * p.scale_log2e;

        if (kPrev) take_out(pw_prev);

        // ---- one block: scores of the next stage, weights of this one, O update of the last
        Scores raw_next;
        if (kNext) raw_next = scores(sl_next);
        uint32_t pw[kParts][kRegs / 2];
#pragma unroll
        for (int r = 0; r < kRegs; r += 2) {
          const float p0 = fast_exp2(fmaf(sc[r], p.scale_log2e, neg_m));
          const float p1 = fast_exp2(fmaf(sc[r + 1], p.scale_log2e, neg_m));
          if constexpr (kExact) {
            uint32_t rest0 = __float_as_uint(p0), rest1 = __float_as_uint(p1);
#pragma unroll
            for (int part = 0; part < kParts; ++part) {  // upper halves, and what they leave (without rounding)
              pw[part][r >> 1] = __builtin_amdgcn_perm(rest1, rest0, 0x07060302u);
              rest0 = __float_as_uint(__uint_as_float(rest0) - __uint_as_float(rest0 & 0xffff0000u));
              rest1 = __float_as_uint(__uint_as_float(rest1) - __uint_as_float(rest1 & 0xffff0000u));
            }
            l_run += p0 + p1;
          } else {
            pw[0][r >> 1] = cvt_pk_bf16(p0, p1);
            // the row sums are taken over the rounded bf16 weights, the values the MFMA multiplies
            l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pw[0][r >> 1]), ones,
                                                    l_run, false);
          }
        }
        if (kPrev) weighted_sum(pw_prev);
        read_v(sl_cur);  // V of this stage, used by the next iteration or the drain
#pragma unroll
        for (int part = 0; part < kParts; ++part)
#pragma unroll
          for (int r = 0; r < kRegs / 2; ++r) pw_prev[part][r] = pw[part][r];
        if (kNext) {
          raw = raw_next;
          sl_cur = sl_next;
        }
      };
      using yes = std::true_type;
      using no = std::false_type;
      if (pc.n_cmp == 1) {
        stage(0, no{}, no{});
      } else {
        stage(0, yes{}, no{});
        for (int i = 1; i < pc.n_cmp - 1; ++i) stage(i, yes{}, yes{});
        stage(pc.n_cmp - 1, no{}, yes{});
      }
      take_out(pw_prev);
      weighted_sum(pw_prev);  // drain
      mfma_settle();
    }
    // stages of the piece without math for this wave: keep the ring and the barriers going
    for (int i = pc.n_cmp; i < pc.n_st; ++i) acquire();

    if constexpr (kExact) {
      // a NaN in any wave's results: the piece once more, from its first stage, for all waves.
      // (No loads but the ring's are in flight here, and none of it is left behind.)
      const bool again = !careful && any_wave(__builtin_amdgcn_ballot_w64(has_nan(o_acc)) != 0);
      careful = again;
      if (again) {
        wait_vmem<0>();
        __builtin_amdgcn_s_barrier();
        lw = cp;
        ld_segment();
        n_acq -= pc.n_st;
        slot_acq = slot_ld = 0;
        fill_ring();
        continue;
      }
    }

    // ---- the next piece's queries are requested before this piece's results are stored:
    //      waiting for them later then does not wait for the stores
    const Piece done = pc;
    cp.advance(map, G, done.n_st);
    if (n_acq < n_my) {
      pc = piece_at(cp, n_acq);
      if (pc.n_cmp > 0) load_queries(pc);
    }

    if (s0 == 0 && !done.whole) {
      // the unit starts here and runs past the end of this range, which is the end of
      // this workgroup's work: its last stage lies us - n_st stages further
      const int us = n_cache + (T + kStageRows - 1) / kStageRows;
      cut.unit = done.unit;
      const long long w_last = sch.pieces > 0 ? w + sch.pieces - 1 : sch.range_owner(cp.x_end - 1 + (us - done.n_st));
      cut.w_last_and_nodes = (int32_t)w_last | (T << 16);
    }
    if (s0 == 0 && p.by_unit) leave_record(done.unit);

    // ---- write: lane holds d = mb*32 + 8*(r/4) + 4*g + r%4 for its query t
    l_run += __shfl_xor(l_run, 32, kWave);
    m_run *= p.scale_log2e;  // from here on the maximum is in the exponent's (log2) domain
    constexpr int kMyMb = kMb / KS;  // blocks of d this wave writes
    if constexpr (KS == 2) {
      // The two waves of a query group exchange halves of O and the statistics through the three ring slots of
      // the stages acquired last: none of them is in flight, behind a barrier nobody reads them any
      // more, and the next load into one is issued behind the next stage's barrier.
      static_assert(NS == 5 && kAhead == 2, "two stages in flight, three slots free");
      auto slot_before = [](int sl) { return sl == 0 ? NS - 1 : sl - 1; };
      const int last = slot_before(slot_acq), last2 = slot_before(last), last3 = slot_before(last2);
      const uint32_t o_at = smem_base + (uint32_t)(k_part == 0 ? last : last2) * kStageBytes + q_group * (kStageBytes / 2) + lane * 16;
      const uint32_t o_from = smem_base + (uint32_t)(k_part == 0 ? last2 : last) * kStageBytes + q_group * (kStageBytes / 2) + lane * 16;
      const uint32_t ml_at = smem_base + (uint32_t)last3 * kStageBytes + wave * 512 + lane * 8;
      const uint32_t ml_from = smem_base + (uint32_t)last3 * kStageBytes + (wave ^ 2) * 512 + lane * 8;
      __builtin_amdgcn_s_barrier();
      if (q_group * 32 < T) {
        if (k_part == 0) {
          // part 0 keeps the lower half of d, part 1 the upper
          put_blocks(o_at, std::integral_constant<int, kMyMb>{});
        } else {
          put_blocks(o_at, std::integral_constant<int, 0>{});
#pragma unroll
          for (int mb = 0; mb < kMyMb; ++mb) o_acc[mb] = o_acc[kMyMb + mb];
        }
        lds_write8(ml_at, u32x2{__float_as_uint(m_run), __float_as_uint(l_run)});
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");  // the reads below stay below
      if (q_group * 32 < T) {
        f32x4 other[kMyMb * 4];
#pragma unroll
        for (int x = 0; x < kMyMb * 4; ++x)
          other[x] = *reinterpret_cast<const __attribute__((address_space(3))) f32x4 *>((uintptr_t)(o_from + 1024 * x));
        const u32x2 ml = *reinterpret_cast<const __attribute__((address_space(3))) u32x2 *>((uintptr_t)ml_from);
        const float m2 = __uint_as_float(ml.x), l2 = __uint_as_float(ml.y);
        const float M = fmaxf(m_run, m2), M_safe = M == -INFINITY ? 0.f : M;
        const float a1 = fast_exp2(m_run - M_safe), a2 = fast_exp2(m2 - M_safe);
        l_run = l_run * a1 + l2 * a2;
        m_run = M;
#pragma unroll
        for (int mb = 0; mb < kMyMb; ++mb)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            o_acc[mb][r] = merge_add<D>(o_acc[mb][r], a1, other[4 * mb + r / 4][r % 4], a2);
          }
      }
    }
    if (q_group * 32 < T) {
      if (done.whole) {
        if (t < T) {
          uint16_t *orow = p.out + ((size_t)done.unit * p.T_max + t) * D;
#pragma unroll
          for (int mb = 0; mb < kMyMb; ++mb) store_out_block<true>(orow, o_acc[mb], 1.f / l_run, g, k_part * kMyMb + mb);
        }
      } else {
        // a range starts inside at most one unit and ends inside at most one
        const size_t ps = 2 * (size_t)w + (s0 > 0 ? 0 : 1);
        if (t < T) {
#pragma unroll
          for (int mb = 0; mb < kMyMb; ++mb)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
              const f32x4 w4 = {o_acc[mb][4 * q4], o_acc[mb][4 * q4 + 1], o_acc[mb][4 * q4 + 2],
                                o_acc[mb][4 * q4 + 3]};
              global_store16_untracked(p.part_o + part_o_index(ps, q_group, 4 * (k_part * kMyMb + mb) + q4, lane),
                                       __builtin_bit_cast(u32x4, w4));
            }
          if (k_part == 0) {
            global_store4_untracked(p.part_ml + part_ml_index(ps, q_group, 0, lane), m_run);
            global_store4_untracked(p.part_ml + part_ml_index(ps, q_group, 1, lane), l_run);
          }
        }
      }
    }
  }
  if (!p.by_unit) leave_record(w);
}

// Finish the units that a range boundary cut: out = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s
// over the pieces s of the unit, always in the order of the pieces.  Lanes map to (query, d) exactly
// as in the main kernel: register block 4 mb + q4 of a wave's 32 queries.
// What it costs is waves that find nothing to do and the chain of dependent reads (record,
// partials: written by other XCDs, so each comes from beyond the L2), not bytes.  Two kernels:
//   by unit (few units, each in many pieces): one workgroup per (unit, 32 queries, 32-wide block mb
//     of d), one wave per q4, up to 16 pieces requested together.
//   by workgroup (many units in a few pieces each): one wave per (workgroup of the main kernel, 32
//     queries, block mb), four pieces of the whole block together.  640 units of 4224 rows on 512
//     workgroups: 12 us; four such waves to a workgroup, or one wave per q4, cost 14 to 18 us.
// The steps of both are the same, one piece after the other, and so are the bits of the result.
// Where the line lies (merge_by_unit): at four pieces per unit.  Whole calls by unit / by workgroup,
// us, d = 128, equal lengths, on 512 workgroups: 32 units of 64 queries x 1024 keys 19.7 / 24.4, 40 x
// 128 x 3000 36.4 / 39.4, 64 x 128 x 2000 38.1 / 39.1, 96 x 32 x 700 20.6 / 21.9, 128 x 64 x 2048 42.0 / 42.5 (d =
// 64: 34.2 / 35.0), 160 x 128 x 1500 50.4 / 50.2, 256 x 64 x 1000 38.6 / 38.4, 256 x 128 x 4000 126.8 / 124.9, 480
// x 70 x 300 41.1 / 38.4.
static bool merge_by_unit(long long units, int grid) { return 4 * units <= grid; }
constexpr int kCombinePieces = 4, kCombineManyPieces = 16;

template <int D>
__global__ __launch_bounds__(kWave) void tree_attn_combine_kernel(AttnParams p) {
  constexpr int kMb = Geo<D>::kMb;
  const int groups = (p.T_max + 31) / 32;
  const int mb = blockIdx.x % kMb, item = blockIdx.x / kMb, w = item / groups, dw = item - w * groups;
  const CutRecord cut = *reinterpret_cast<const CutRecord *>(p.cuts + 4 * w);
  if (cut.unit < 0) return;
  const int T = cut.w_last_and_nodes >> 16, w_last = cut.w_last_and_nodes & 0xffff;
  if (dw * 32 >= T) return;
  const int lane = threadIdx.x;
  const int t = dw * 32 + (lane & 31), g = lane >> 5;
  // lanes beyond the tree read lane 0's data (valid memory) and store nothing
  const int ln = t < T ? lane : 0;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  float M = -INFINITY, lsum = 0.f;
  for (int w0 = w; w0 <= w_last; w0 += kCombinePieces) {
    f32x4 o[kCombinePieces][4];
    float m[kCombinePieces], l[kCombinePieces];
#pragma unroll
    for (int k = 0; k < kCombinePieces; ++k) {
      const int wg = w0 + k <= w_last ? w0 + k : w_last;  // past the last piece: re-read it, weight 0
      const size_t ps = 2 * (size_t)wg + (wg == w ? 1 : 0);
      m[k] = p.part_ml[part_ml_index(ps, dw, 0, ln)];
      l[k] = p.part_ml[part_ml_index(ps, dw, 1, ln)];
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        o[k][q4] = *reinterpret_cast<const f32x4 *>(p.part_o + part_o_index(ps, dw, 4 * mb + q4, ln));
    }
#pragma unroll
    for (int k = 0; k < kCombinePieces; ++k) {
      if (w0 + k > w_last) break;  // uniform
      const float M_new = fmaxf(M, m[k]);
      const float M_safe = M_new == -INFINITY ? 0.f : M_new;
      const float a_old = fast_exp2(M - M_safe), a_new = fast_exp2(m[k] - M_safe);
      lsum = lsum * a_old + l[k] * a_new;
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[4 * q4 + j] = merge_add<D>(acc[4 * q4 + j], a_old, o[k][q4][j], a_new);
      M = M_new;
    }
  }
  // the two lanes of an exchange pair hold the same query, so they are active together
  if (t < T) store_out_block<false>(p.out + ((size_t)cut.unit * p.T_max + t) * D, acc, 1.f / lsum, g, mb);
}

template <int D>
__global__ __launch_bounds__(4 * kWave) void tree_attn_combine_unit_kernel(AttnParams p) {
  constexpr int kMb = Geo<D>::kMb, N = kCombineManyPieces;
  const int groups = (p.T_max + 31) / 32;
  const int mb = blockIdx.x % kMb, item = blockIdx.x / kMb, unit = item / groups, dw = item - unit * groups;
  const CutRecord cut = *reinterpret_cast<const CutRecord *>(p.cuts + 4 * (size_t)unit);
  if (cut.unit < 0) return;
  const int T = cut.w_last_and_nodes >> 16, w_last = cut.w_last_and_nodes & 0xffff, w = cut.w_first;
  if (dw * 32 >= T) return;
  const int lane = threadIdx.x & 63, q4 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t = dw * 32 + (lane & 31), g = lane >> 5;
  const int ln = t < T ? lane : 0;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  float M = -INFINITY, lsum = 0.f;
  for (int w0 = w; w0 <= w_last; w0 += N) {
    f32x4 o[N];
    float m[N], l[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
      if (w0 + k <= w_last) {  // uniform
        const int wg = w0 + k;
        const size_t ps = 2 * (size_t)wg + (wg == w ? 1 : 0);
        m[k] = p.part_ml[part_ml_index(ps, dw, 0, ln)];
        l[k] = p.part_ml[part_ml_index(ps, dw, 1, ln)];
        o[k] = *reinterpret_cast<const f32x4 *>(p.part_o + part_o_index(ps, dw, 4 * mb + q4, ln));
      }
    }
#pragma unroll
    for (int k = 0; k < N; ++k)
      if (w0 + k <= w_last) {  // uniform
        const float M_new = fmaxf(M, m[k]);
        const float M_safe = M_new == -INFINITY ? 0.f : M_new;
        const float a_old = fast_exp2(M - M_safe), a_new = fast_exp2(m[k] - M_safe);
        lsum = lsum * a_old + l[k] * a_new;
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = merge_add<D>(acc[j], a_old, o[k][j], a_new);
        M = M_new;
      }
  }
  const float inv = 1.f / lsum;
  const int d0 = 32 * mb + 8 * q4;  // the wave's 8 columns; the lane's four start at d0 + 4 g
  if (t < T)
    *reinterpret_cast<u32x2 *>(p.out + ((size_t)cut.unit * p.T_max + t) * D + d0 + 4 * g) =
        u32x2{cvt_pk_bf16(acc[0] * inv, acc[1] * inv), cvt_pk_bf16(acc[2] * inv, acc[3] * inv)};
}

// ------------------------------------------------------------------------------------
// Plain path: one wave per (sequence, head, node); products, softmax and output sums in fp32.
// Serves bf16 operands with d = 64 that come without the workspace or the alignment of the tiled
// kernel.  Rows of V with weight zero are not looked at, so a value that is not finite reaches the
// queries that see it and no others.
// ------------------------------------------------------------------------------------
template <typename E>
struct AttnParamsPlain {
  const E *q, *k_cache, *v_cache, *k_tree, *v_tree;
  E *out;
  const int32_t *seq_lens, *n_nodes;
  const uint64_t *anc;
  int H, T_max, L_max;
  float scale;
};

__global__ __launch_bounds__(kWave) void tree_attn_plain_kernel(AttnParamsPlain<uint16_t> p) {
  constexpr int d = kWave;  // a lane owns a column of the result
  const int unit = blockIdx.x / p.T_max, i = blockIdx.x - unit * p.T_max;
  const int b = unit / p.H;
  int L = p.seq_lens[b];
  L = L < 0 ? 0 : (L > p.L_max ? p.L_max : L);
  int T = p.n_nodes[b];
  T = T < 1 ? 1 : (T > p.T_max ? p.T_max : T);
  if (i >= T) return;
  const int lane = threadIdx.x;
  const uint64_t a_lo = p.anc[((size_t)b * p.T_max + i) * 2];
  const uint64_t a_hi = p.anc[((size_t)b * p.T_max + i) * 2 + 1];
  const uint16_t *q = p.q + ((size_t)unit * p.T_max + i) * d;
  const uint16_t *kc = p.k_cache + (size_t)unit * p.L_max * d;
  const uint16_t *vc = p.v_cache + (size_t)unit * p.L_max * d;
  const uint16_t *kt = p.k_tree + (size_t)unit * p.T_max * d;
  const uint16_t *vt = p.v_tree + (size_t)unit * p.T_max * d;

  float m_run = -INFINITY, l_run = 0.f, o = 0.f;
  const int total = L + T;
  for (int j0 = 0; j0 < total; j0 += kWave) {
    const int j = j0 + lane;
    const bool in_cache = j < L;
    const int jt = j - L;
    const bool ok = in_cache || (j < total && test_bit128(a_lo, a_hi, jt));
    float s = -INFINITY;
    if (ok) {
      const uint16_t *kr = in_cache ? kc + (size_t)j * d : kt + (size_t)jt * d;
      float acc = 0.f;
      for (int x = 0; x < d; ++x) acc = fmaf(bf16_bits_to_f32(q[x]), bf16_bits_to_f32(kr[x]), acc);
      s = acc * p.scale;
    }
    const float m_new = fmaxf(m_run, wave_reduce_max(s));
    if (m_new == -INFINITY) continue;  // nothing visible in this chunk (uniform across the wave)
    const float alpha = expf(m_run - m_new);
    const float w = ok ? expf(s - m_new) : 0.f;
    l_run = l_run * alpha + wave_reduce_sum(w);
    o *= alpha;
    m_run = m_new;
    const uint64_t live = __ballot(w != 0.f);
    for (uint64_t rest = live; rest; rest &= rest - 1) {
      const int src = __ffsll((long long)rest) - 1;
      const float wj = __shfl(w, src, kWave);
      const int jj = j0 + src;
      const uint16_t *vr = jj < L ? vc + (size_t)jj * d : vt + (size_t)(jj - L) * d;
      o = fmaf(wj, bf16_bits_to_f32(vr[lane]), o);
    }
  }
  p.out[((size_t)unit * p.T_max + i) * d + lane] = (uint16_t)f32_to_bf16_bits(o / l_run);
}

#include "tree_attention_f32.h"

template <typename E>
static void fill_plain(AttnParamsPlain<E> &p, const propd_tree *tree, int H, float scale, const void *q,
                       const void *k_cache, const void *v_cache, const void *k_tree, const void *v_tree,
                       const int32_t *seq_lens, int L_max, void *out) {
  p.q = reinterpret_cast<const E *>(q);
  p.k_cache = reinterpret_cast<const E *>(k_cache);
  p.v_cache = reinterpret_cast<const E *>(v_cache);
  p.k_tree = reinterpret_cast<const E *>(k_tree);
  p.v_tree = reinterpret_cast<const E *>(v_tree);
  p.out = reinterpret_cast<E *>(out);
  p.seq_lens = seq_lens;
  p.n_nodes = tree->n_nodes;
  p.anc = tree->anc;
  p.H = H;
  p.T_max = tree->T_max;
  p.L_max = L_max;
  p.scale = scale;
}

// ------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------
static int compute_units() {
  static const int cus = [] {
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0)
      return prop.multiProcessorCount;
    return 256;
  }();
  return cus;
}

// Workgroups of the persistent kernel: at most one per two stages of the call, a bound the
// host can compute without a device (the workspace is sized by it) ...
static int grid_bound(int B, int H, int L_max, int T_max) {
  const long long per_unit = (L_max + kStageRows - 1) / kStageRows + (T_max + kStageRows - 1) / kStageRows;
  const long long stages = (long long)B * H * per_unit;
  long long grid = kMaxGrid;
  if (grid > (stages + 1) / 2) grid = (stages + 1) / 2;
  return (int)(grid < 1 ? 1 : grid);
}

// ... and as many as are resident on the chip.  (Ranges of three stages or more take 1 us less at 1 x 32
// units of 1088 rows, but a piece's largest weight is exactly 1 and rounds without error: with fewer
// pieces the error against 64 bits goes from 2.20e-3 to 2.24e-3.)
static int pick_grid(int per_cu, int B, int H, int L_max, int T_max) {
  const int bound = grid_bound(B, H, L_max, T_max), resident = per_cu * compute_units();
  return bound < resident ? bound : resident;
}

// Partial slots (two per workgroup) and cut records (one per workgroup) of the largest grid
// a call with these dimensions can use.
size_t tree_attention_workspace_bytes(int B, int H, int L_max, int T_max) {
  const size_t grid = (size_t)grid_bound(B, H, L_max, T_max), slots = 2 * grid;
  return align_up(slots * kPartOFloats * 4, 256) + align_up(slots * kPartMlFloats * 4, 256) +
         align_up(grid * sizeof(CutRecord), 256);
}

template <int D, int KS, bool kAnew>
static bool launch_bf16(const AttnParams &p, int grid, hipStream_t st) {
  constexpr int lds_bytes = kRingStages * Geo<D>::kStageBytes;
  static std::atomic<bool> attr_set{false};  // calls may come from several threads
  if (!attr_set) {
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(&tree_attn_bf16_kernel<kRingStages, D, KS, kAnew>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes) != hipSuccess)
      return false;
    attr_set = true;
  }
  hipLaunchKernelGGL((tree_attn_bf16_kernel<kRingStages, D, KS, kAnew>), dim3((unsigned)grid), dim3(kAttnThreads),
                     lds_bytes, st, p);
  if (!launch_ok()) return false;
  const unsigned blocks = (unsigned)(p.T_max + 31) / 32 * Geo<D>::kMb;
  if (p.by_unit)
    hipLaunchKernelGGL(tree_attn_combine_unit_kernel<D>, dim3((unsigned)(p.B * p.H) * blocks), dim3(4 * kWave), 0, st, p);
  else
    hipLaunchKernelGGL(tree_attn_combine_kernel<D>, dim3((unsigned)grid * blocks), dim3(kWave), 0, st, p);
  return launch_ok();
}

}  // namespace propd

extern "C" propd_status propd_tree_attention(const propd_tree *tree, propd_dtype dt, int32_t H,
                                             int32_t d, float scale, const void *q,
                                             const void *k_cache, const void *v_cache,
                                             const void *k_tree, const void *v_tree,
                                             const int32_t *seq_lens, int32_t L_max, void *out,
                                             void *workspace, size_t workspace_bytes,
                                             void *hip_stream) {
  using namespace propd;
  if (!tree || tree->B < 1 || tree->T_max < 1 || tree->T_max > PROPD_MAX_TREE || H < 1 ||
      L_max < 0 || !tree->n_nodes || !tree->anc || !q || !k_tree || !v_tree || !seq_lens || !out ||
      (L_max > 0 && (!k_cache || !v_cache)))
    return PROPD_ERR_INVALID_ARG;
  if (dt != PROPD_BF16 && dt != PROPD_F32) return PROPD_ERR_INVALID_ARG;
  if (!(scale > 0.f)) return PROPD_ERR_INVALID_ARG;  // the kernels take max before scaling
  const long long units = (long long)tree->B * H;
  if (units * tree->T_max > (1ll << 30) || units > (1ll << 28)) return PROPD_ERR_UNSUPPORTED;
  hipStream_t st = as_stream(hip_stream);

  if (dt == PROPD_F32) {
    if (d != 64 && d != 128) return PROPD_ERR_UNSUPPORTED;
    AttnParamsF32 p;
    fill_plain<float>(p, tree, H, scale, q, k_cache, v_cache, k_tree, v_tree, seq_lens, L_max, out);
    p.units = (int)units;
    p.scale_log2e = scale * 1.4426950408889634f;
    return (d == 64 ? launch_f32<64>(p, compute_units(), workspace, workspace_bytes, st)
                    : launch_f32<128>(p, compute_units(), workspace, workspace_bytes, st))
               ? PROPD_OK
               : PROPD_ERR_DEVICE;
  }
  if (d != 64 && d != 128) return PROPD_ERR_UNSUPPORTED;
  // rows are moved 16 bytes per lane, by direct loads to LDS and four-dword loads and stores
  bool aligned = true;
  for (const void *ptr : {q, k_cache, v_cache, k_tree, v_tree, (const void *)out, (const void *)tree->anc,
                          (const void *)workspace})
    aligned = aligned && reinterpret_cast<uintptr_t>(ptr) % 16 == 0;
  const size_t need = tree_attention_workspace_bytes(tree->B, H, L_max, tree->T_max);
  const bool scratch = workspace && workspace_bytes >= need;
  if (d == 64 && !(aligned && scratch)) {  // the smaller head may come without either: one wave per query
    AttnParamsPlain<uint16_t> p;
    fill_plain<uint16_t>(p, tree, H, scale, q, k_cache, v_cache, k_tree, v_tree, seq_lens, L_max, out);
    hipLaunchKernelGGL(tree_attn_plain_kernel, dim3((unsigned)(units * tree->T_max)), dim3(kWave), 0, st, p);
    return launch_ok() ? PROPD_OK : PROPD_ERR_DEVICE;
  }
  if (!aligned) return PROPD_ERR_INVALID_ARG;
  if (!scratch) return PROPD_ERR_WORKSPACE;
  AttnParams p;
  p.q = reinterpret_cast<const uint16_t *>(q);
  p.k_cache = reinterpret_cast<const uint16_t *>(k_cache);
  p.v_cache = reinterpret_cast<const uint16_t *>(v_cache);
  p.k_tree = reinterpret_cast<const uint16_t *>(k_tree);
  p.v_tree = reinterpret_cast<const uint16_t *>(v_tree);
  p.out = reinterpret_cast<uint16_t *>(out);
  p.seq_lens = seq_lens;
  p.n_nodes = tree->n_nodes;
  p.anc = tree->anc;
  p.H = H;
  p.T_max = tree->T_max;
  p.L_max = L_max;
  p.B = tree->B;
  p.scale = scale;
  p.scale_log2e = scale * 1.4426950408889634f;
  const int grid = pick_grid(d == 64 ? Geo<64>::kPerCu : Geo<128>::kPerCu, tree->B, H, L_max, tree->T_max);
  const size_t slots = 2 * (size_t)grid_bound(tree->B, H, L_max, tree->T_max);
  char *ws = reinterpret_cast<char *>(workspace);
  p.part_o = reinterpret_cast<float *>(ws);
  ws += align_up(slots * kPartOFloats * 4, 256);
  p.part_ml = reinterpret_cast<float *>(ws);
  ws += align_up(slots * kPartMlFloats * 4, 256);
  p.cuts = reinterpret_cast<int32_t *>(ws);
  p.by_unit = merge_by_unit(units, grid) ? 1 : 0;
  const long long unit_stages = (L_max + kStageRows - 1) / kStageRows + (tree->T_max + kStageRows - 1) / kStageRows;
  p.cus = compute_units();
  p.one_pass = tree->B <= kWave && units * unit_stages < (1ll << 31) && unit_stages < (1 << 20) ? 1 : 0;
  // Two waves per 32 queries, see KS.  By sizes alone: the lengths are not known here.  d = 128 with more units than
  // workgroups keeps one, whatever L_max (the slot's size): over 46 calls of 540 to 2048 units it takes 0.99 to 1.02 of two
  // waves' time where units have 8 stages and more on average (64 x 32 units of 64 x up to 776 101.9 / 100.3 us, 128 x 16 of 32 x up to
  // 3380 245.2 / 240.1), and 0.92 to 1.00 with fewer (17 x 32 of 64 x up to 32 16.2 / 17.6, 128 x 16 of 16 x up to 75 30.9 / 32.8).
  // d = 64 gains more than it loses: 40 such calls 0.95 (27 x 20 units of 33 x up to 101 15.2 / 16.0) to 1.27 (20 x 40 of 64 x 1985 140.1 /
  // 110.5), mean 1.03.  No more units than workgroups, both head sizes: 50 calls 0.96 to 1.25, mean 1.02.
  const bool split = tree->T_max <= 64 && (d == 64 || units <= grid);
  const bool anew = p.one_pass && units <= grid;
  if (!(d == 64 ? (split ? launch_bf16<64, 2, false>(p, grid, st) : launch_bf16<64, 1, false>(p, grid, st))
        : anew  ? (split ? launch_bf16<128, 2, true>(p, grid, st) : launch_bf16<128, 1, true>(p, grid, st))
                : (split ? launch_bf16<128, 2, false>(p, grid, st) : launch_bf16<128, 1, false>(p, grid, st))))
    return PROPD_ERR_DEVICE;
  return PROPD_OK;
}

extern "C" size_t propd_workspace_bytes(propd_ws_kind which, int32_t B, int32_t T_max, int32_t H,
                                        int32_t d, int32_t L_max, int32_t hidden, int32_t vocab) {
  (void)d;
  (void)hidden;
  if (B < 1 || T_max < 1 || T_max > PROPD_MAX_TREE) return 0;
  switch (which) {
    case PROPD_WS_TREE_ATTENTION:
      if (H < 1 || L_max < 0) return 0;
      return propd::tree_attention_workspace_bytes(B, H, L_max, T_max);
    case PROPD_WS_EARLY_PRUNE:
      if (vocab < 1) return 0;
      return propd::early_prune_workspace_bytes(B, T_max, vocab);
    case PROPD_WS_ACCEPT_PATH:
      return propd::accept_path_workspace_bytes(B, T_max);
  }
  return 0;
}
