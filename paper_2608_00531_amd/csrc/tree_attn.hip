// cure_tree_attn: tree-masked verification attention (Sec. 3.2 phase 3,
// Sec. 3.4, Sec. 3.5) as a split-KV ("flash-decoding") pass plus a
// log-sum-exp merge of the split partials.
//
// Every node of a sequence's candidate tree attends to the whole cached
// context and to the nodes on its own root path. The context is shared by all
// nodes, so the work is organised around the key/value stream: one workgroup
// owns (sequence, kv-head, row block, context split) and reads each K/V tile
// from HBM exactly once for all query rows of that kv-head -- the G query heads
// of every tree node, packed node-major. Only tiles that reach the tree rows
// at the tail of the sequence apply the ancestor bitmask.
//
// Five kernels compute a split:
//  * tree_attn_m16: bf16, scale > 0, head dim 128 (any row count, in
//    balanced row blocks of up to 256 rows) or 64 (up to 128 rows). Scores
//    are formed transposed, S^T = K Q^T, and the output as O^T = V^T P^T with
//    16x16x32 bf16 MFMAs, 16 query rows per wave. K/V tiles arrive in LDS by
//    DMA; V is read back transposed by the LDS transpose-read instruction in
//    exactly the token order the score MFMA leaves P in registers.
//  * tree_attn_rg: the same with two or three 16-row groups per wave, for head dim
//    128 with 257 - 384 rows and head dim 64 beyond 128 rows, in blocks of up to 192.
//  * tree_attn_mfma: the same with 32x32x16 MFMAs and 32 rows per wave, for head dim 64
//    beyond 192 rows, in blocks of up to 256.
//  * tree_attn_f32: fp32 on the fp32 matrix instructions, the same scheme with
//    the rows and the tokens of a block dealt over four waves.
//  * tree_attn_valu: fp32 or bf16, any supported shape, scale and alignment;
//    plain vector ALU code.
// A split writes normalised partial O and its log-sum-exp; attn_merge combines
// the splits of each row (skipped when a sequence has a single split, in which
// case the split kernel writes the final output itself).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "common.hpp"
#include "host_util.hpp"

namespace cure {
namespace {

constexpr int kTile = 64;            // tokens per K/V tile
constexpr int kStages = 2;           // K/V tile buffers in tree_attn_mfma's LDS ring
constexpr int kMaxGridY = 65535;     // largest grid y (the split index)
constexpr int kMinTps = 256;         // tokens per split, at least
constexpr int kMaxUnits = 512;       // entries of a compact launch's table
constexpr int kAncWords = CURE_MAX_TREE_NODES / 64;

struct Args {
  const void* q;
  const void* k;
  const void* v;
  void* o;
  float* lse;
  int32_t out_bf16;
  int32_t hq, hkv, group, n_max;
  float scale_log2;                  // scale * log2(e): scores live in the log2 domain
  const int64_t* kv_off;
  const int32_t* ctx_len;
  const int32_t* n_nodes;
  const int32_t* parent;
  int32_t tps, max_splits, rows_per_wg;
  int32_t* tree_status;
  float* part_o;                     // [batch][hq][n_max][max_splits][d]
  float* part_lse;                   // [batch][hq][n_max][max_splits]
};

// Arguments of a compact launch (see locate()).
struct CompactArgs : Args {
  int32_t row_blocks;
  uint32_t unit[kMaxUnits / 2];      // unit u in half u % 2 of word u / 2: sequence | split << 6
  int32_t seq_splits[64];            // splits each sequence may have
};

// Where a workgroup works: kv-head hk, row block rb and split s of sequence b,
// and the most splits that sequence may have.
struct Place {
  int b, hk, rb, s, max_splits;
};

// Full launches are a 3-D grid, (kv-heads x row blocks, splits, batch), in which a
// ragged batch leaves workgroups without work. Each of those still takes its turn
// when the dispatcher deals workgroups to the shader engines, so some engines are
// dealt more real ones than they have CUs for, and those start when the first
// have finished: on 16 sequences of 1k to 4k tokens (48 nodes, 256 of 384
// workgroups real) the longest workgroup ran 44 us and the kernel 58. A compact
// launch holds (kv-heads x row blocks) x the units the host counted, from a table
// in the kernel arguments: read by the scalar unit with the other arguments.
CURE_DEV Place locate(const Args& a) {
  return Place{(int)blockIdx.z, (int)(blockIdx.x % a.hkv), (int)(blockIdx.x / a.hkv), (int)blockIdx.y, a.max_splits};
}
CURE_DEV Place locate(const CompactArgs& a) {
  const int blocks = a.hkv * a.row_blocks;
  const int u = blockIdx.x / blocks, x = blockIdx.x - u * blocks;
  const int e = (a.unit[u >> 1] >> (16 * (u & 1))) & 0xffff;
  const int b = e & 63;
  return Place{b, x % a.hkv, x / a.hkv, e >> 6, a.seq_splits[b]};
}

// The most splits sequence b may have, for the merge.
CURE_DEV int max_splits_of(const Args& a, int) { return a.max_splits; }
CURE_DEV int max_splits_of(const CompactArgs& a, int b) { return a.seq_splits[b]; }

// Number of context splits of a sequence with T = ctx + nodes rows. The last
// split runs to T, so a clamp never drops rows.
CURE_DEV int split_count(int T, int N, int tps, int max_splits) {
  if (N <= 0 || T <= 0) return 0;
  return min((T + tps - 1) / tps, max_splits);
}

CURE_DEV int64_t part_index(const Args& a, int b, int head, int n, int s) {
  return (((int64_t)b * a.hq + head) * a.n_max + n) * a.max_splits + s;
}

// Loads sequence b's parent array, validates it and builds every node's
// ancestor bitmask (its root path, itself included). Returns true if valid.
CURE_DEV bool build_tree(const Args& a, int b, int N, int* s_parent,
                         unsigned long long (*s_anc)[kAncWords], int* s_bad) {
  if (threadIdx.x == 0) *s_bad = 0;
  __syncthreads();
  for (int n = threadIdx.x; n < N; n += blockDim.x) {
    const int p = a.parent[(int64_t)b * a.n_max + n];
    s_parent[n] = p;
    if (p < -1 || p >= n) *s_bad = 1;
  }
  __syncthreads();
  if (*s_bad) return false;
  for (int n = threadIdx.x; n < N; n += blockDim.x) {
    unsigned long long w[kAncWords] = {};
    for (int j = n; j >= 0; j = s_parent[j]) w[j >> 6] |= 1ull << (j & 63);
#pragma unroll
    for (int i = 0; i < kAncWords; ++i) s_anc[n][i] = w[i];
  }
  __syncthreads();
  return true;
}

// As build_tree, for a workgroup of at least N threads where thread n has
// already loaded parent[n] (the load is issued early, off the critical path).
CURE_DEV bool build_tree_loaded(int N, int my_parent, int* s_parent,
                                unsigned long long (*s_anc)[kAncWords], int* s_bad) {
  const int n = threadIdx.x;
  if (n == 0) *s_bad = 0;
  __syncthreads();
  if (n < N) {
    s_parent[n] = my_parent;
    if (my_parent < -1 || my_parent >= n) *s_bad = 1;
  }
  __syncthreads();
  if (*s_bad) return false;
  if (n < N) {
    unsigned long long w[kAncWords] = {};
    for (int j = n; j >= 0; j = s_parent[j]) w[j >> 6] |= 1ull << (j & 63);
#pragma unroll
    for (int i = 0; i < kAncWords; ++i) s_anc[n][i] = w[i];
  }
  __syncthreads();
  return true;
}

CURE_DEV void report_tree(const Args& a, int b, bool ok, bool reporter) {
  if (reporter && threadIdx.x == 0 && a.tree_status) a.tree_status[b] = ok ? CURE_OK : CURE_ERR_BAD_TREE;
}

// Visibility of cache row tok (relative to the sequence) for node n.
CURE_DEV bool visible(int tok, int L, int N, int n, const unsigned long long (*s_anc)[kAncWords]) {
  if (tok < L) return true;
  const int j = tok - L;
  if (j >= N) return false;
  return (s_anc[n][j >> 6] >> (j & 63)) & 1ull;
}

// Additive mask of token tok for node n inside a split that ends at `end`:
// +0 when visible() holds, -inf otherwise. Computed without branches (the
// ancestor word is read for a clamped row index and context rows ignore it;
// tok < end implies tok < ctx + nodes, so a row past the context is a tree
// row), so that adding it to a score leaves no divergent write to a register
// of an MFMA result vector.
CURE_DEV float mask_bias(int tok, int L, int end, int n,
                         const unsigned long long (*s_anc)[kAncWords]) {
  const int j = min(max(tok - L, 0), CURE_MAX_TREE_NODES - 1);
  const uint32_t bit = (uint32_t)(s_anc[n][j >> 6] >> (j & 63)) & 1u;
  const uint32_t vis = (uint32_t)(tok < L) | ((uint32_t)(tok < end) & bit);
  return __uint_as_float((vis ^ 1u) * 0xff800000u);
}

template <typename T>
CURE_DEV float ld_elem(const T* p);
template <>
CURE_DEV float ld_elem<float>(const float* p) { return *p; }
template <>
CURE_DEV float ld_elem<uint16_t>(const uint16_t* p) { return bf16_to_f32(*p); }

CURE_DEV void store_out(const Args& a, int64_t idx, float val) {
  if (a.out_bf16) reinterpret_cast<uint16_t*>(a.o)[idx] = f32_to_bf16(val);
  else reinterpret_cast<float*>(a.o)[idx] = val;
}

// ---------------------------------------------------------------------------
// Vector-ALU split kernel: 4 waves, 8 query rows per wave, one token per lane
// for the scores and D/64 output columns per lane for P V.
constexpr int kValuRowsPerWave = 8;
constexpr int kValuWaves = 4;
constexpr int kValuRows = kValuRowsPerWave * kValuWaves;

template <typename E, int D>
__global__ __launch_bounds__(256) void tree_attn_valu(Args a) {
  __shared__ int s_parent[CURE_MAX_TREE_NODES];
  __shared__ unsigned long long s_anc[CURE_MAX_TREE_NODES][kAncWords];
  __shared__ int s_bad;
  __shared__ float s_q[kValuRows][D];
  __shared__ float s_k[kTile][D + 1];
  __shared__ float s_v[kTile][D];
  __shared__ float s_p[kValuWaves][kValuRowsPerWave][kTile];

  const int b = blockIdx.z;
  const int hk = blockIdx.x % a.hkv;
  const int rb = blockIdx.x / a.hkv;
  const int s = blockIdx.y;
  const int N = min(a.n_nodes[b], a.n_max);
  const int L = a.ctx_len[b];
  const int T = L + N;
  const int S = split_count(T, N, a.tps, a.max_splits);
  const int rows = N * a.group;
  if (S == 0) {                         // no nodes: nothing to compute; the empty tree is valid
    report_tree(a, b, true, s == 0 && hk == 0 && rb == 0);
    return;
  }
  if (s >= S || rb * kValuRows >= rows) return;
  const bool reporter = s == 0 && hk == 0 && rb == 0;
  const bool ok = build_tree(a, b, N, s_parent, s_anc, &s_bad);
  report_tree(a, b, ok, reporter);
  if (!ok) return;

  const int begin = s * a.tps;
  const int end = (s == S - 1) ? T : begin + a.tps;
  const int64_t off = a.kv_off[b];
  const E* qp = reinterpret_cast<const E*>(a.q);
  const E* kp = reinterpret_cast<const E*>(a.k);
  const E* vp = reinterpret_cast<const E*>(a.v);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  for (int i = tid; i < kValuRows * D; i += 256) {
    const int r = i / D, d = i - r * D;
    const int R = rb * kValuRows + r;
    float val = 0.f;
    if (R < rows) {
      const int n = R / a.group, head = hk * a.group + R % a.group;
      val = ld_elem<E>(qp + (((int64_t)b * a.n_max + n) * a.hq + head) * D + d);
    }
    s_q[r][d] = val;
  }

  float m_run[kValuRowsPerWave], l_run[kValuRowsPerWave], acc[kValuRowsPerWave][D / 64];
#pragma unroll
  for (int i = 0; i < kValuRowsPerWave; ++i) {
    m_run[i] = -INFINITY;
    l_run[i] = 0.f;
#pragma unroll
    for (int c = 0; c < D / 64; ++c) acc[i][c] = 0.f;
  }

  for (int t0 = begin; t0 < end; t0 += kTile) {
    __syncthreads();
    for (int i = tid; i < kTile * D; i += 256) {
      const int t = i / D, d = i - t * D;
      const int tok = t0 + t;
      float kv = 0.f, vv = 0.f;
      if (tok < end) {
        const int64_t e = ((off + tok) * a.hkv + hk) * D + d;
        kv = ld_elem<E>(kp + e);
        vv = ld_elem<E>(vp + e);
      }
      s_k[t][d] = kv;
      s_v[t][d] = vv;
    }
    __syncthreads();

    // Scores for this wave's rows: lane = token.
    float sc[kValuRowsPerWave];
#pragma unroll
    for (int i = 0; i < kValuRowsPerWave; ++i) sc[i] = 0.f;
    for (int d = 0; d < D; ++d) {
      const float kd = s_k[lane][d];
#pragma unroll
      for (int i = 0; i < kValuRowsPerWave; ++i)
        sc[i] = fmaf(s_q[wave * kValuRowsPerWave + i][d], kd, sc[i]);
    }
    const int tok = t0 + lane;
#pragma unroll
    for (int i = 0; i < kValuRowsPerWave; ++i) {
      const int R = rb * kValuRows + wave * kValuRowsPerWave + i;
      const int n = min(R / a.group, N - 1);
      const bool vis = tok < end && visible(tok, L, N, n, s_anc);
      const float x = vis ? sc[i] * a.scale_log2 : -INFINITY;
      float mt = x;
      mt = wave_max(mt);
      const float m_new = fmaxf(m_run[i], mt);
      const float m_use = m_new == -INFINITY ? 0.f : m_new;
      const float p = exp2f(x - m_use);
      float ps = p;
      ps = wave_sum(ps);
      const float alpha = exp2f(m_run[i] - m_use);
      l_run[i] = l_run[i] * alpha + ps;
      m_run[i] = m_new;
#pragma unroll
      for (int c = 0; c < D / 64; ++c) acc[i][c] *= alpha;
      s_p[wave][i][lane] = p;
    }
    // P V: lane = output column(s).
    for (int t = 0; t < kTile; ++t) {
      float vv[D / 64];
#pragma unroll
      for (int c = 0; c < D / 64; ++c) vv[c] = s_v[t][lane + 64 * c];
#pragma unroll
      for (int i = 0; i < kValuRowsPerWave; ++i) {
        const float p = s_p[wave][i][t];
#pragma unroll
        for (int c = 0; c < D / 64; ++c) acc[i][c] = fmaf(p, vv[c], acc[i][c]);
      }
    }
  }

#pragma unroll
  for (int i = 0; i < kValuRowsPerWave; ++i) {
    const int R = rb * kValuRows + wave * kValuRowsPerWave + i;
    if (R >= rows) continue;
    const int n = R / a.group, head = hk * a.group + R % a.group;
    const float inv = l_run[i] > 0.f ? 1.f / l_run[i] : 0.f;
    const float lse2 = l_run[i] > 0.f ? m_run[i] + log2f(l_run[i]) : -INFINITY;
    if (S == 1) {
      const int64_t base = (((int64_t)b * a.n_max + n) * a.hq + head) * D;
#pragma unroll
      for (int c = 0; c < D / 64; ++c) store_out(a, base + lane + 64 * c, acc[i][c] * inv);
      if (lane == 0 && a.lse) a.lse[((int64_t)b * a.n_max + n) * a.hq + head] = lse2 * kLn2;
    } else {
      const int64_t pi = part_index(a, b, head, n, s);
#pragma unroll
      for (int c = 0; c < D / 64; ++c) a.part_o[pi * D + lane + 64 * c] = acc[i][c] * inv;
      if (lane == 0) a.part_lse[pi] = lse2 * kLn2;
    }
  }
}

// ---------------------------------------------------------------------------
// MFMA split kernels (bf16 in, fp32 accumulate): what they share.
//
// Per 64-token tile:
//   S^T = K Q^T, online softmax in the log2 domain, rescaling O only when a row's
//   maximum rises by more than 2^8 (values then stay below 2^8, safe in bf16 and
//   fp32), O^T += V^T P^T
// K and V tiles move HBM -> LDS by DMA (buffer loads that write LDS directly)
// through a ring of tile buffers: while one tile is computed, the next ones stream
// in. The per-sequence buffer resource bounds every read: rows past the sequence
// end read as zeros, and ring slots past the split's end are filled by reads at an
// offset past the resource, which touch no memory. LDS rows are 16-byte-chunk
// XOR-swizzled so that both the K reads (one row per lane) and the transposed V
// reads (4 rows x 16 columns per 16 lanes, ds_read_b64_tr_b16) spread over the
// banks: without conflicts at head dim 128, with 2.3 conflict cycles per LDS
// instruction counted at 64. The DMA is issued from inline assembly on purpose: written through the
// compiler builtin, every later LDS read of the current tile gets a wait on the
// next tile's DMA (the compiler cannot tell the buffers apart), which serialises
// the pipeline. Ordering is explicit instead: each loop iteration starts with
// s_waitcnt + barrier before any LDS read of the tile it uses.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

typedef int i32x4 __attribute__((ext_vector_type(4)));
constexpr int kRsrcWord3 = 0x00020000;     // raw (untyped) 32-bit access, gfx9 family

// A raw buffer resource over `bytes` bytes at `base`, as four wave-uniform
// dwords (SGPRs): base address (48 bits, stride 0), record count in bytes,
// and the gfx9-family word for untyped 32-bit access. Built from integer
// words rather than converted from the opaque resource type, which the
// compiler would spill through a per-thread memory copy.
CURE_DEV i32x4 raw_rsrc(const void* base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  return i32x4{__builtin_amdgcn_readfirstlane((int)(uint32_t)a),
               __builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu)),
               __builtin_amdgcn_readfirstlane((int)bytes),
               __builtin_amdgcn_readfirstlane(kRsrcWord3)};
}

CURE_DEV uint32_t lds_addr(const void* p) {
  return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(const lds_void*)p);
}

// LDS reads at a 32-bit LDS address: with a per-lane base and a compile-time
// constant the constant travels in the instruction's 16-bit offset field.
CURE_DEV bf16x8 lds_read16(uint32_t addr) {
  return *(const __attribute__((address_space(3))) bf16x8*)(uintptr_t)addr;
}
CURE_DEV i16x4 lds_read_tr8(uint32_t addr) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(uintptr_t)addr);
}

// 64 lanes x 16 bytes from a buffer resource straight into LDS: lane i's bytes
// land at lds_base + 16 * i (lds_base travels in M0). Out-of-range offsets
// read as zero.
CURE_DEV void dma16(uint32_t lds_base, uint32_t voff, i32x4 rsrc) {
  asm volatile("buffer_load_dwordx4 %0, %1, 0 offen nt lds"
               :
               : "v"(voff), "s"(rsrc), "{m0}"(lds_base)
               : "memory");
}

union Pack8 {
  uint4 u;
  bf16x8 v;
  i16x4 h[2];
};


// Three-input maximum as one v_max3_f32. Written as assembly because fmaxf
// first canonicalises every operand that may be a signalling NaN (an extra
// instruction per score); scores here are finite dot products or -inf.
CURE_DEV float max3_raw(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
constexpr float kRescaleLog2 = 8.f;       // lazy rescale threshold (log2 units)

template <int D>
struct TileGeo {
  static constexpr int kChunks = D / 8;             // 16-byte chunks per row
  static constexpr int kRowBytes = D * 2;
  static constexpr int kTileBytes = kTile * kRowBytes;
  static constexpr int kBlocks = kTileBytes / 1024;  // 1 KB DMA blocks per tile
  // Swizzle: the chunk index is XORed with a row-dependent value. Any value
  // keeps the layout correct (the DMA and every reader apply the same XOR); it
  // only decides which LDS banks one instruction touches. At head dim 128 the
  // chunk bits are (r1^r2, r1, r2, r0) of the row bits r0..r2: with it neither
  // the K operand reads (16 bytes per lane, 16 rows) nor the transposed V reads
  // (8 bytes per lane, 4 rows per 16 lanes) have bank conflicts, as measured
  // with SQ_LDS_BANK_CONFLICT on gfx950 (the earlier permutation of the row
  // bits cost 4 stall cycles per K read and 2 per V read).
  static CURE_DEV int swz(int row) {
    if (kChunks == 16) {
      const int r0 = row & 1, r1 = (row >> 1) & 1, r2 = (row >> 2) & 1;
      return (r1 ^ r2) | (r1 << 1) | (r2 << 2) | (r0 << 3);
    }
    return ((row & 3) << 1) | ((row >> 2) & 1);
  }
  static CURE_DEV int offset(int row, int chunk) {   // byte offset inside a tile
    return row * kRowBytes + ((chunk ^ swz(row)) << 4);
  }
};

// s_waitcnt immediate: at most `vm` vector-memory operations outstanding, no
// wait on export, all LDS/scalar-memory operations complete (gfx9 encoding:
// vmcnt[3:0] in bits 3:0, vmcnt[5:4] in bits 15:14, expcnt in 6:4).
constexpr int waitcnt_vm(int vm) { return (vm & 15) | ((vm >> 4) << 14) | (7 << 4); }
constexpr uint32_t kOobOffset = 0x80000000u;   // past any sequence's buffer resource

// ---------------------------------------------------------------------------
// MFMA split kernel with 32 query rows per wave (v_mfma_f32_32x32x16_bf16), for
// head dim 64 in blocks of up to 256 rows.
//
// Each of the NW waves owns 32 query rows; lane = query row in S^T, whose tile is 2
// token blocks x D/16 k-steps, and O^T takes D/32 column blocks x 4 k-steps. Bound by
// LDS reads, MFMA and softmax issue, so by the waves there are to overlap them: in 119
// VGPRs two workgroups, sixteen waves, share a CU, which two 16-row groups per wave
// (tree_attn_rg) need too many registers for. With the same splits, 8 sequences of 8k
// tokens and 256 rows take 59.6 us here, 70.0 in eight waves of two groups and 73.5 in
// two blocks of four waves; 16 of 2k - 8k and 400 rows 143.9, and 157.7 in four-wave
// blocks.
template <int D, int NW, int NBUF, class A>
__global__ __launch_bounds__(64 * NW, NBUF > 2 ? 1 : 2) void tree_attn_mfma(A a) {
  using G = TileGeo<D>;
  constexpr int kKSteps = D / 16;                  // MFMA k-steps for Q K^T
  constexpr int kDBlk = D / 32;                    // 32-column blocks of O^T
  constexpr int kDmaPerWave = G::kBlocks / NW;     // DMA blocks per wave per tensor
  // Each loop iteration waits until its tile has landed while the NBUF - 2
  // tiles issued after it may still be in flight (2 instructions per block).
  constexpr int kVmWait = waitcnt_vm((NBUF - 2) * 2 * kDmaPerWave);
  static_assert((NBUF - 2) * 2 * kDmaPerWave < 64, "vmcnt holds 6 bits");
  static_assert(G::kBlocks % NW == 0, "tile must split evenly across waves");

  __shared__ int s_parent[CURE_MAX_TREE_NODES];
  __shared__ unsigned long long s_anc[CURE_MAX_TREE_NODES][kAncWords];
  __shared__ int s_bad;
  __shared__ __attribute__((aligned(1024))) unsigned char s_k[NBUF][G::kTileBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char s_v[NBUF][G::kTileBytes];

  const Place at = locate(a);
  const int b = at.b, hk = at.hk, rb = at.rb, s = at.s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, col = lane & 31;

  // This lane's query row, and its query loads: they need only the launch
  // shape (rows past the sequence's nodes still lie inside q and are zeroed
  // below), so they go out together with the loads of the sequence's sizes,
  // as does each thread's parent entry for the tree.
  const int R = rb * a.rows_per_wg + wave * 32 + col;
  const bool r_in = R < a.n_max * a.group;
  bf16x8 qreg[kKSteps];
  {
    const int qn = r_in ? R / a.group : 0;
    const int qh = hk * a.group + (r_in ? R % a.group : 0);
    const uint16_t* qrow = reinterpret_cast<const uint16_t*>(a.q) +
                           (((int64_t)b * a.n_max + qn) * a.hq + qh) * D;
#pragma unroll
    for (int kk = 0; kk < kKSteps; ++kk) {
      Pack8 p;
      p.u = r_in ? *reinterpret_cast<const uint4*>(qrow + kk * 16 + half * 8)
                 : make_uint4(0, 0, 0, 0);
      qreg[kk] = p.v;
    }
  }
  const int my_parent = tid < a.n_max ? a.parent[(int64_t)b * a.n_max + tid] : -1;

  // The sequence's sizes and cache offset are independent loads: one round
  // trip. The empty asm keeps the compiler from sinking the offset's load
  // below the early exits (a second round trip).
  const int n_raw = a.n_nodes[b];
  const int L = a.ctx_len[b];
  const int64_t off = a.kv_off[b];
  asm volatile("" : : "s"(n_raw), "s"(L), "s"(off));
  const int N = min(n_raw, a.n_max);
  const int T = L + N;
  const int S = split_count(T, N, a.tps, at.max_splits);
  const int rows = N * a.group;
  if (S == 0) {                         // no nodes: nothing to compute; the empty tree is valid
    report_tree(a, b, true, s == 0 && hk == 0 && rb == 0);
    return;
  }
  if (s >= S || rb * a.rows_per_wg >= rows) return;

  const int begin = s * a.tps;
  const int end = (s == S - 1) ? T : begin + a.tps;

  // Buffer resources over this sequence's K and V rows (all kv-heads).
  const uint32_t seq_bytes = (uint32_t)T * (uint32_t)(a.hkv * G::kRowBytes);
  // Per lane and DMA block: byte offset of the source chunk for tile start 0.
  uint32_t src_off[kDmaPerWave];
#pragma unroll
  for (int j = 0; j < kDmaPerWave; ++j) {
    const int byte = (wave * kDmaPerWave + j) * 1024 + lane * 16;   // destination in tile
    const int row = byte / G::kRowBytes;
    const int pchunk = (byte % G::kRowBytes) >> 4;
    const int lchunk = pchunk ^ G::swz(row);
    src_off[j] = (uint32_t)((row * a.hkv + hk) * G::kRowBytes + (lchunk << 4));
  }
  const uint32_t tok_bytes = (uint32_t)(a.hkv * G::kRowBytes);
  // A tile at or past the split's end is still issued (at an out-of-range
  // offset) so that every iteration has the same number of DMAs in flight.
  const i32x4 rk4 = raw_rsrc(reinterpret_cast<const uint16_t*>(a.k) + off * a.hkv * D, seq_bytes);
  const i32x4 rv4 = raw_rsrc(reinterpret_cast<const uint16_t*>(a.v) + off * a.hkv * D, seq_bytes);
  auto dma_tile = [&](int buf, int t0) {
    const bool live = t0 < end;
#pragma unroll
    for (int j = 0; j < kDmaPerWave; ++j) {
      const uint32_t voff = live ? src_off[j] + (uint32_t)t0 * tok_bytes : kOobOffset;
      const int blk = (wave * kDmaPerWave + j) * 1024;
      dma16(lds_addr(&s_k[buf][blk]), voff, rk4);
      dma16(lds_addr(&s_v[buf][blk]), voff, rv4);
    }
  };

  // The first tiles' DMA goes out before anything else this workgroup loads.
#pragma unroll
  for (int i = 0; i < NBUF - 1; ++i) dma_tile(i, begin + i * kTile);

  const bool row_ok = R < rows;
  const int n = row_ok ? R / a.group : 0;
  const int head = hk * a.group + (row_ok ? R % a.group : 0);
  const bool wave_active = rb * a.rows_per_wg + wave * 32 < rows;

  // LDS byte offsets used by this lane, independent of the tile.
  // K rows blk*32 + col, logical chunk 2*kk + half.
  int k_row_base[2], k_swz[2];
#pragma unroll
  for (int blk = 0; blk < 2; ++blk) {
    const int row = blk * 32 + col;
    k_row_base[blk] = row * G::kRowBytes;
    k_swz[blk] = G::swz(row) ^ half;
  }
  // V transposed reads: lane j of each 16-lane group reads 8 bytes at row
  // (4*half + j/4) of a 4-row group, columns 4*(j%4) of a 16-column block.
  const int j16 = lane & 15, g16 = (lane >> 4) & 1;
  const int v_row_lane = 4 * half + (j16 >> 2);          // + 16*ks + 8*r
  const int v_chunk_lane = 2 * g16 + ((j16 & 3) >> 1);   // + 4*i
  const int v_byte_lane = (j16 & 1) * 8;

  // Only a split that reaches the tree's own rows needs the ancestor masks
  // (built while the first tile and the queries are in flight). The last
  // split always does, and it reports the tree's status. With a malformed
  // tree the other splits still run; the sequence's output is unspecified.
  if (end > L) {
    const bool ok = build_tree_loaded(N, my_parent, s_parent, s_anc, &s_bad);
    report_tree(a, b, ok, s == S - 1 && hk == 0 && rb == 0);
    if (!ok) {
      __builtin_amdgcn_s_waitcnt(0);      // no DMA may land after the workgroup ends
      return;
    }
  }

  f32x16 oacc[kDBlk];
#pragma unroll
  for (int i = 0; i < kDBlk; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[i][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const float c = a.scale_log2;
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};

  // Queries and the first tiles have landed. (This also tells the compiler
  // that no load it issued is pending, so it adds no waits inside the loop.)
  __builtin_amdgcn_s_waitcnt(0);
  if (!row_ok) {
#pragma unroll
    for (int kk = 0; kk < kKSteps; ++kk) qreg[kk] = bf16x8{};
  }
  for (int t0 = begin, buf = 0; t0 < end; t0 += kTile, buf = buf + 1 == NBUF ? 0 : buf + 1) {
    __builtin_amdgcn_s_waitcnt(kVmWait);  // this wave's DMA into `buf` has landed
    __syncthreads();                      // everyone's has; the previous buffer is free
    dma_tile(buf == 0 ? NBUF - 1 : buf - 1, t0 + (NBUF - 1) * kTile);
    if (!wave_active) continue;
    const unsigned char* kt = s_k[buf];
    const unsigned char* vt = s_v[buf];

    // S^T (tokens x query rows), raw dot products; two independent chains.
    f32x16 sacc[2];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
      for (int r = 0; r < 16; ++r) sacc[blk][r] = 0.f;
    // K operands are read one k-step ahead of the MFMAs that consume them.
    Pack8 ka[2][2];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
      ka[0][blk].u = *reinterpret_cast<const uint4*>(kt + k_row_base[blk] + (k_swz[blk] << 4));
#pragma unroll
    for (int kk = 0; kk < kKSteps; ++kk) {
      if (kk + 1 < kKSteps) {
#pragma unroll
        for (int blk = 0; blk < 2; ++blk)
          ka[(kk + 1) & 1][blk].u = *reinterpret_cast<const uint4*>(
              kt + k_row_base[blk] + (((2 * (kk + 1)) ^ k_swz[blk]) << 4));
      }
#pragma unroll
      for (int blk = 0; blk < 2; ++blk)
        sacc[blk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[kk & 1][blk].v, qreg[kk], sacc[blk], 0, 0, 0);
    }
    // Mask the tail, then the tile's row maximum (raw units; the scale is > 0).
    if (t0 + kTile > L) {
#pragma unroll
      for (int blk = 0; blk < 2; ++blk)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          sacc[blk][r] += mask_bias(t0 + blk * 32 + 8 * (r >> 2) + 4 * half + (r & 3), L, end, n, s_anc);
    }
    // Row maximum: one three-input max per two scores, in two chains.
    float mb[2] = {-INFINITY, -INFINITY};
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
      for (int r = 0; r < 16; r += 2) mb[blk] = max3_raw(mb[blk], sacc[blk][r], sacc[blk][r + 1]);
    const float m_tile = max_halves(max3_raw(mb[0], mb[1], mb[1])) * c;
    // Lazy rescale: move the reference only when the maximum rises by > 2^8.
    const bool grow = m_tile > m_run + kRescaleLog2;
    if (__builtin_expect(__ballot(grow) != 0, 0)) {
      if (grow) {
        const float alpha = fast_exp2(m_run - m_tile);
        l_run *= alpha;
#pragma unroll
        for (int i = 0; i < kDBlk; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[i][r] *= alpha;
        m_run = m_tile;
      }
    }
    const float nm = m_run == -INFINITY ? 0.f : -m_run;
    bf16x8 pb[4];
    float l0 = 0.f, l1 = 0.f;
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        bf16x8 v8;
#pragma unroll
        for (int e = 0; e < 8; ++e) v8[e] = (__bf16)fast_exp2(fmaf(sacc[blk][8 * j + e], c, nm));
        pb[blk * 2 + j] = v8;
        // Row sums of the probabilities as rounded for the MFMA (bf16 pairs).
#pragma unroll
        for (int e = 0; e < 8; e += 4) {
          l0 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v8[e], v8[e + 1]}, ones, l0, false);
          l1 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v8[e + 2], v8[e + 3]}, ones, l1, false);
        }
      }
    l_run += l0 + l1;

    // O^T += V^T P^T; the D/32 column blocks are independent chains.
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
      for (int i = 0; i < kDBlk; ++i) {
        Pack8 va;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          const int row = 16 * ks + 8 * r + v_row_lane;
          const int byte = G::offset(row, 4 * i + v_chunk_lane) + v_byte_lane;
          va.h[r] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(vt + byte));
        }
        oacc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va.v, pb[ks], oacc[i], 0, 0, 0);
      }
    }
  }

  __builtin_amdgcn_s_waitcnt(0);          // the ring's trailing DMAs land before exit
  if (!row_ok) return;
  const float l_tot = sum_halves(l_run);
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  const float lse_nat = l_tot > 0.f ? (m_run + log2f(l_tot)) * kLn2 : -INFINITY;
  if (S == 1) {
    const int64_t obase = (((int64_t)b * a.n_max + n) * a.hq + head) * D;
#pragma unroll
    for (int i = 0; i < kDBlk; ++i)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const int d0 = i * 32 + 8 * g4 + 4 * half;
        const float x0 = oacc[i][4 * g4] * inv, x1 = oacc[i][4 * g4 + 1] * inv;
        const float x2 = oacc[i][4 * g4 + 2] * inv, x3 = oacc[i][4 * g4 + 3] * inv;
        if (a.out_bf16) {
          uint2 pk;
          pk.x = pack_bf16x2(x0, x1);
          pk.y = pack_bf16x2(x2, x3);
          *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.o) + obase + d0) = pk;
        } else {
          *reinterpret_cast<float4*>(reinterpret_cast<float*>(a.o) + obase + d0) =
              make_float4(x0, x1, x2, x3);
        }
      }
    if (half == 0 && a.lse) a.lse[((int64_t)b * a.n_max + n) * a.hq + head] = lse_nat;
  } else {
    const int64_t pi = part_index(a, b, head, n, s);
#pragma unroll
    for (int i = 0; i < kDBlk; ++i)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const int d0 = i * 32 + 8 * g4 + 4 * half;
        *reinterpret_cast<float4*>(a.part_o + pi * D + d0) =
            make_float4(oacc[i][4 * g4] * inv, oacc[i][4 * g4 + 1] * inv,
                        oacc[i][4 * g4 + 2] * inv, oacc[i][4 * g4 + 3] * inv);
      }
    if (half == 0) a.part_lse[pi] = lse_nat;
  }
}

// ---------------------------------------------------------------------------
// MFMA split kernel with 16 query rows per wave (v_mfma_f32_16x16x32_bf16).
//
// A tile's row maxima are reduced only when a rescale could be due. Few registers
// per wave, so that two 8-wave workgroups (four waves per SIMD) share a CU, and row
// blocks of up to 256 rows fit one 16-wave workgroup with the rows spread evenly over
// the SIMDs.
// Wider trees take several row blocks of equal size (a multiple of 16 rows).
// The row blocks of one kv-head and split are hkv workgroup ids apart: with
// hkv a multiple of 8 the dispatcher, which deals workgroups to the 8 XCDs in
// turn, puts them on the same XCD, where they share its L2 for the K/V stream.
//
// Lane l = 16 g + c (c = l % 16, g = l / 16) owns query row c of its wave.
//   S^T = K Q^T, per 16-token block tb and 32-wide k-step ks:
//     A = K rows tb*16 + c, columns 32 ks + 8 g .. +7   (one 16-byte LDS read)
//     B = Q row c, columns 32 ks + 8 g .. +7             (registers)
//     D register r = score of token tb*16 + 4 g + r for row c
//   so a row's 64 scores sit in the four lanes c, c+16, c+32, c+48 and its
//   statistics reduce over lane xor 16 and xor 32.
//   O^T += V^T P^T, per 16-wide column block db and 32-token k-step kt, with
//   the k index 8 g + j standing for token 32 kt + 4 g + j (j < 4) or
//   32 kt + 16 + 4 g + (j - 4) (j >= 4): exactly the probabilities lane l
//   already holds from blocks 2 kt and 2 kt + 1, so P needs no exchange.
//     A = V^T: two transposed reads of 4 tokens x 16 columns per 16 lanes
//     D register r = O column 16 db + 4 g + r of row c
// At most 128 VGPRs (four waves per SIMD): two 8-wave workgroups share a CU
// whenever a launch has more workgroups than CUs.
template <int D, int NW, class A>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(4))) void tree_attn_m16(A a) {
  using G = TileGeo<D>;
  constexpr int kKSteps = D / 32;                  // k-steps for Q K^T
  constexpr int kDBlk = D / 16;                    // 16-column blocks of O^T
  constexpr int kDmaPerWave = G::kBlocks / NW;     // DMA blocks per wave per tensor
  constexpr int kKFrags = 4 * kKSteps;             // K operand fragments per tile
  constexpr int kVFrags = 2 * kDBlk;               // V^T operand fragments per tile
  constexpr int kAheadK = 4;                       // K reads in flight ahead of their MFMA
  constexpr int kAheadV = 4;                       // V^T reads in flight ahead of their MFMA
  static_assert(G::kBlocks % NW == 0, "tile must split evenly across waves");

  __shared__ int s_parent[CURE_MAX_TREE_NODES];
  __shared__ unsigned long long s_anc[CURE_MAX_TREE_NODES][kAncWords];
  __shared__ int s_bad;
  // K tiles 0 and 1, then V tiles 0 and 1.
  __shared__ __attribute__((aligned(1024))) unsigned char s_kv[4 * G::kTileBytes];

  const Place at = locate(a);
  const int b = at.b, hk = at.hk, rb = at.rb, s = at.s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 15, g = lane >> 4;

  // Query loads (need only the launch shape) and the parent entry go out with
  // the loads of the sequence's sizes.
  const int R = rb * a.rows_per_wg + wave * 16 + c;
  const bool r_in = R < a.n_max * a.group;
  bf16x8 qreg[kKSteps];
  {
    const int qn = r_in ? R / a.group : 0;
    const int qh = hk * a.group + (r_in ? R % a.group : 0);
    const uint16_t* qrow = reinterpret_cast<const uint16_t*>(a.q) +
                           (((int64_t)b * a.n_max + qn) * a.hq + qh) * D;
#pragma unroll
    for (int ks = 0; ks < kKSteps; ++ks) {
      Pack8 p;
      p.u = r_in ? *reinterpret_cast<const uint4*>(qrow + ks * 32 + g * 8)
                 : make_uint4(0, 0, 0, 0);
      qreg[ks] = p.v;
    }
  }
  const int my_parent = tid < a.n_max ? a.parent[(int64_t)b * a.n_max + tid] : -1;

  const int n_raw = a.n_nodes[b];
  const int L = a.ctx_len[b];
  const int64_t off = a.kv_off[b];
  asm volatile("" : : "s"(n_raw), "s"(L), "s"(off));
  const int N = min(n_raw, a.n_max);
  const int T = L + N;
  const int S = split_count(T, N, a.tps, at.max_splits);
  const int rows = N * a.group;
  if (S == 0) {                         // no nodes: nothing to compute; the empty tree is valid
    report_tree(a, b, true, s == 0 && hk == 0 && rb == 0);
    return;
  }
  if (s >= S || rb * a.rows_per_wg >= rows) return;

  const int begin = s * a.tps;
  const int end = (s == S - 1) ? T : begin + a.tps;

  const uint32_t seq_bytes = (uint32_t)T * (uint32_t)(a.hkv * G::kRowBytes);
  const uint32_t tok_bytes = (uint32_t)(a.hkv * G::kRowBytes);
  // Per lane and DMA block: byte offset of the source chunk, moving on by a tile
  // with each call. A split's tiles go to buffers 0, 1, 0, ...
  uint32_t src_off[kDmaPerWave];
#pragma unroll
  for (int j = 0; j < kDmaPerWave; ++j) {
    const int byte = (wave * kDmaPerWave + j) * 1024 + lane * 16;
    const int row = byte / G::kRowBytes;
    const int lchunk = ((byte % G::kRowBytes) >> 4) ^ G::swz(row);
    src_off[j] = (uint32_t)(begin + row) * tok_bytes + (uint32_t)(hk * G::kRowBytes + (lchunk << 4));
  }
  const i32x4 rk4 = raw_rsrc(reinterpret_cast<const uint16_t*>(a.k) + off * a.hkv * D, seq_bytes);
  const i32x4 rv4 = raw_rsrc(reinterpret_cast<const uint16_t*>(a.v) + off * a.hkv * D, seq_bytes);
  const uint32_t lds0 = lds_addr(s_kv);
  const uint32_t dma0 = __builtin_amdgcn_readfirstlane(lds0 + wave * kDmaPerWave * 1024);
  auto dma_tile = [&](int buf) {
#pragma unroll
    for (int j = 0; j < kDmaPerWave; ++j) {
      dma16(dma0 + buf * G::kTileBytes + j * 1024, src_off[j], rk4);
      dma16(dma0 + (2 + buf) * G::kTileBytes + j * 1024, src_off[j], rv4);
      src_off[j] += kTile * tok_bytes;
    }
  };
  dma_tile(0);

  // A row block may hold fewer rows than the workgroup has row waves.
  const bool own = wave * 16 < a.rows_per_wg;
  const bool row_ok = own && R < rows;
  const int n = row_ok ? R / a.group : 0;
  const int head = hk * a.group + (row_ok ? R % a.group : 0);
  const bool wave_active = own && rb * a.rows_per_wg + wave * 16 < rows;

  // LDS addresses of this lane's operands in tile buffer 0. The swizzle takes
  // only a row's low three bits, so the next 16-row block, the next 32-token
  // step and the other buffer are constants away: the loop over the tiles, a
  // buffer at a time, does no address arithmetic (46 -> 15 vector instructions
  // a tile beside the 48 of the softmax). Longest workgroup 97.2k -> 92.9k cycles
  // on the ragged batch and 164k -> 148k at 32k context; calls 58.0 -> 57.6 and
  // 102.6 -> 100.8 us, the clock being lower the busier the loop is.
  uint32_t k_at[kKSteps];                          // K: row c, chunk 4 ks + g
#pragma unroll
  for (int ks = 0; ks < kKSteps; ++ks) k_at[ks] = lds0 + G::offset(c, 4 * ks + g);
  // V: within a 16-lane group, lane j = c addresses row 4 g + j / 4 (+16) of
  // the k-step's 32 tokens, columns 16 db + 4 (j % 4) .. +3.
  uint32_t v_at[kDBlk];
#pragma unroll
  for (int db = 0; db < kDBlk; ++db)
    v_at[db] = lds0 + G::offset(4 * g + (c >> 2), 2 * db + ((c & 3) >> 1)) + (c & 1) * 8;

  if (end > L) {
    const bool ok = build_tree_loaded(N, my_parent, s_parent, s_anc, &s_bad);
    report_tree(a, b, ok, s == S - 1 && hk == 0 && rb == 0);
    if (!ok) {
      __builtin_amdgcn_s_waitcnt(0);
      return;
    }
  }

  f32x4 oacc[kDBlk];
#pragma unroll
  for (int i = 0; i < kDBlk; ++i) oacc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;            // l_run: this lane's share of the row sum
  const float cs = a.scale_log2;
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};

  __builtin_amdgcn_s_waitcnt(0);
  if (!row_ok) {
#pragma unroll
    for (int ks = 0; ks < kKSteps; ++ks) qreg[ks] = bf16x8{};
  }
  auto tile_step = [&](auto buf_c, int t0) {
    constexpr int buf = decltype(buf_c)::value;
    constexpr int kt = buf * G::kTileBytes, vt = (2 + buf) * G::kTileBytes;
    __builtin_amdgcn_s_waitcnt(0);        // this wave's DMA into `buf` has landed
    __syncthreads();                      // everyone's has; the other buffer is free
    if (t0 + kTile < end) dma_tile(buf ^ 1);
    if (!wave_active) return;

    // Scores: four 16-token blocks, each a chain of kKSteps MFMAs. The K
    // operand reads run kAheadK fragments ahead of the MFMA that takes them,
    // so LDS latency overlaps the matrix core instead of stalling each MFMA.
    f32x4 sacc[4];
#pragma unroll
    for (int tb = 0; tb < 4; ++tb) sacc[tb] = f32x4{0.f, 0.f, 0.f, 0.f};
    Pack8 kf[kKFrags];
#pragma unroll
    for (int i = 0; i < kAheadK; ++i) kf[i].v = lds_read16(k_at[i >> 2] + kt + (i & 3) * 16 * G::kRowBytes);
#pragma unroll
    for (int i = 0; i < kKFrags; ++i) {
      if (i + kAheadK < kKFrags) {
        const int j = i + kAheadK;
        kf[j].v = lds_read16(k_at[j >> 2] + kt + (j & 3) * 16 * G::kRowBytes);
      }
      sacc[i & 3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[i].v, qreg[i >> 2], sacc[i & 3], 0, 0, 0);
    }
    // Left alone, the scheduler sinks each read back next to its MFMA; pin the
    // order: kAheadK reads, then alternate one MFMA (0x008) and one LDS read
    // (0x100), then the last kAheadK MFMAs.
    __builtin_amdgcn_sched_group_barrier(0x100, kAheadK, 0);
#pragma unroll
    for (int i = 0; i < kKFrags - kAheadK; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, kAheadK, 0);
    if (t0 + kTile > L) {
#pragma unroll
      for (int tb = 0; tb < 4; ++tb)
#pragma unroll
        for (int r = 0; r < 4; ++r) sacc[tb][r] += mask_bias(t0 + tb * 16 + 4 * g + r, L, end, n, s_anc);
    }
    // V^T fragment i: k-step i / kDBlk, column block i % kDBlk. The first
    // kAheadV go out before the exponentials, which then hide their latency.
    Pack8 vf[kVFrags];
    auto load_v = [&](Pack8& f, int i) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        f.h[h] = lds_read_tr8(v_at[i % kDBlk] + vt + (32 * (i / kDBlk) + 16 * h) * G::kRowBytes);
    };
#pragma unroll
    for (int i = 0; i < kAheadV; ++i) load_v(vf[i], i);
    // Probabilities against the running reference m_run, bf16 for the P V
    // product, and the lane's share of the row sums from the same bf16 values.
    bf16x8 pb[2];                                  // k-steps kt = 0, 1 (blocks 2 kt, 2 kt + 1)
    float l0 = 0.f, l1 = 0.f;
    auto exps = [&](float nm) {
      l0 = 0.f;
      l1 = 0.f;
#pragma unroll
      for (int kt2 = 0; kt2 < 2; ++kt2) {
        bf16x8 v8;
#pragma unroll
        for (int j = 0; j < 8; ++j)
          v8[j] = (__bf16)fast_exp2(fmaf(sacc[2 * kt2 + (j >> 2)][j & 3], cs, nm));
        pb[kt2] = v8;
        l0 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v8[0], v8[1]}, ones, l0, false);
        l1 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v8[2], v8[3]}, ones, l1, false);
        l0 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v8[4], v8[5]}, ones, l0, false);
        l1 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v8[6], v8[7]}, ones, l1, false);
      }
    };
    // The reference moves lazily, when a row's maximum rises by more than 2^8.
    // The tile's row maxima are reduced only when that can happen: when a row
    // has no reference yet, or when some lane's probabilities sum to more than
    // 2^8 (otherwise none of them exceeds 2^8, so no row's maximum rose that
    // far). Up to rounding at the threshold the probabilities are those of
    // reducing the maximum on every tile.
    bool have = false, check = true;
    if (__ballot(m_run == -INFINITY) == 0) {
      exps(-m_run);
      have = true;
      check = __ballot(!(l0 + l1 <= 256.f)) != 0;
    }
    if (__builtin_expect(check, 0)) {
      // Row maximum over the lane's 16 scores (eight v_max3), then its 3 partners.
      float mb = max3_raw(sacc[0][0], sacc[0][1], sacc[0][2]);
#pragma unroll
      for (int i = 3; i < 15; i += 2)
        mb = max3_raw(mb, sacc[i >> 2][i & 3], sacc[(i + 1) >> 2][(i + 1) & 3]);
      mb = max3_raw(mb, sacc[3][3], sacc[3][3]);
      mb = max3_raw(mb, partner<16>(mb), mb);
      const float m_tile = max_halves(mb) * cs;
      const bool grow = m_tile > m_run + kRescaleLog2;
      const bool grew = __ballot(grow) != 0;
      if (grow) {
        const float alpha = fast_exp2(m_run - m_tile);
        l_run *= alpha;
#pragma unroll
        for (int i = 0; i < kDBlk; ++i) oacc[i] *= alpha;
        m_run = m_tile;
      }
      if (!have || grew) exps(m_run == -INFINITY ? 0.f : -m_run);
    }
    l_run += l0 + l1;

#pragma unroll
    for (int i = 0; i < kVFrags; ++i) {
      if (i + kAheadV < kVFrags) load_v(vf[i + kAheadV], i + kAheadV);
      oacc[i % kDBlk] =
          __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[i].v, pb[i / kDBlk], oacc[i % kDBlk], 0, 0, 0);
    }
  };
  // (No DMA is in flight after the last tile: none is issued past it.)
  for (int t0 = begin; t0 < end; t0 += 2 * kTile) {
    tile_step(std::integral_constant<int, 0>{}, t0);
    if (t0 + kTile < end) tile_step(std::integral_constant<int, 1>{}, t0 + kTile);
  }

  if (!row_ok) return;
  float l_tot = l_run + partner<16>(l_run);
  l_tot = sum_halves(l_tot);
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  const float lse_nat = l_tot > 0.f ? (m_run + log2f(l_tot)) * kLn2 : -INFINITY;
  if (S == 1) {
    const int64_t obase = (((int64_t)b * a.n_max + n) * a.hq + head) * D;
#pragma unroll
    for (int db = 0; db < kDBlk; ++db) {
      const int d0 = db * 16 + 4 * g;
      const float x0 = oacc[db][0] * inv, x1 = oacc[db][1] * inv;
      const float x2 = oacc[db][2] * inv, x3 = oacc[db][3] * inv;
      if (a.out_bf16) {
        uint2 pk;
        pk.x = pack_bf16x2(x0, x1);
        pk.y = pack_bf16x2(x2, x3);
        *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.o) + obase + d0) = pk;
      } else {
        *reinterpret_cast<float4*>(reinterpret_cast<float*>(a.o) + obase + d0) =
            make_float4(x0, x1, x2, x3);
      }
    }
    if (g == 0 && a.lse) a.lse[((int64_t)b * a.n_max + n) * a.hq + head] = lse_nat;
  } else {
    const int64_t pi = part_index(a, b, head, n, s);
#pragma unroll
    for (int db = 0; db < kDBlk; ++db)
      *reinterpret_cast<float4*>(a.part_o + pi * D + db * 16 + 4 * g) =
          make_float4(oacc[db][0] * inv, oacc[db][1] * inv, oacc[db][2] * inv, oacc[db][3] * inv);
    if (g == 0) a.part_lse[pi] = lse_nat;
  }
}

// ---------------------------------------------------------------------------
// MFMA split kernel with RG 16-row groups per wave (v_mfma_f32_16x16x32_bf16).
//
// The 16-row kernel's operand layout, tile stream, tree mask and online
// softmax, with two changes:
//  * each wave owns RG groups of 16 query rows, and every K fragment and V^T
//    fragment it reads from LDS feeds the MFMAs of all RG groups, so a tile's
//    LDS reads serve 16 RG rows per wave instead of 16 (LDS read bandwidth
//    co-bounds the K/V stream once a kv-head has more than ~128 rows);
//  * the K/V ring holds NBUF tiles, so NBUF - 1 tiles (32 KB each at head dim
//    128) are in flight while one is computed; only the first NDMA waves
//    issue the tile DMA (G::kBlocks / NDMA blocks per tensor each), and the
//    barrier after their wait releases the others.
// The block's ceil(rows_per_wg / 16) row groups are dealt so that the first
// n_full waves own RG groups each and the others RG - 1: waves w and w + 4
// share a SIMD, so with 8 waves every SIMD carries the same number of groups
// whenever the count allows (320 rows: 3 + 2 groups on each SIMD, where seven
// 3-group waves put 6 groups on three SIMDs and 3 on the fourth). A wave
// runs the tile loop's body instantiated for its own group count. Row r of a
// wave's group rg is query row rb * rows_per_wg + 16 (first + rg) + c, with
// first the wave's first group (lane l = 16 g + c as in the 16-row kernel).
template <int D, int NW, int RG, int NBUF, int NDMA, int HT, int WPE, class A>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
void tree_attn_rg(A a) {
  using G = TileGeo<D>;
  constexpr int kKSteps = D / 32;                  // k-steps for Q K^T
  constexpr int kDBlk = D / 16;                    // 16-column blocks of O^T
  constexpr int kDmaBlocks = G::kBlocks / NDMA;    // DMA blocks per DMA wave per tensor
  // The tile's 64 tokens are taken in HT steps of online softmax, each of
  // kTB 16-token blocks (scores) and kPV 32-token k-steps (P V). Head dim 128
  // takes two, for its registers. Head dim 64 takes one, as the 16-row kernel: a
  // row's probabilities are rounded to bf16 against the maximum of the first
  // step, so the more tokens that covers, the more often the largest one is
  // exactly 1. In two steps the error against 64 bits was 1.2 % larger (192 rows,
  // 8 sequences of 1k - 4k tokens: 2.323e-3 of the output and 2.295e-3) and the
  // calls were 0 - 10 % slower.
  constexpr int kTB = 4 / HT;
  constexpr int kPV = 2 / HT;
  constexpr int kKFrags = kTB * kKSteps;           // K operand fragments per step
  constexpr int kVFrags = kPV * kDBlk;             // V^T operand fragments per step
  constexpr int kAheadK = 4;                       // K reads in flight ahead of their MFMAs
  constexpr int kAheadV = 4;                       // V^T reads in flight ahead of their MFMAs
  // Each iteration waits until its tile has landed while the NBUF - 2 tiles
  // issued after it may still be in flight (2 instructions per block).
  constexpr int kVmWait = waitcnt_vm((NBUF - 2) * 2 * kDmaBlocks);
  static_assert(G::kBlocks % NDMA == 0 && NDMA <= NW, "DMA blocks split evenly over DMA waves");
  static_assert((NBUF - 2) * 2 * kDmaBlocks < 64, "vmcnt holds 6 bits");
  static_assert(NBUF >= 2, "a ring of at least two tiles");
  static_assert(HT == 1 || HT == 2, "one or two softmax steps per tile");

  __shared__ int s_parent[CURE_MAX_TREE_NODES];
  __shared__ unsigned long long s_anc[CURE_MAX_TREE_NODES][kAncWords];
  __shared__ int s_bad;
  __shared__ __attribute__((aligned(1024))) unsigned char s_k[NBUF][G::kTileBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char s_v[NBUF][G::kTileBytes];

  const Place at = locate(a);
  const int b = at.b, hk = at.hk, rb = at.rb, s = at.s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 15, g = lane >> 4;
  const int groups_wg = (a.rows_per_wg + 15) / 16;
  const int n_full = min(NW, max(0, groups_wg - (RG - 1) * NW));
  const int my_groups = wave < n_full ? RG : RG - 1;
  const int first = wave < n_full ? RG * wave : RG * n_full + (RG - 1) * (wave - n_full);
  const int wrow = rb * a.rows_per_wg + 16 * first;        // this wave's first row

  // Query loads (they need only the launch shape) and the parent entry go out
  // with the loads of the sequence's sizes.
  bf16x8 qreg[RG][kKSteps];
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    const int R = wrow + 16 * rg + c;
    const bool r_in = rg < my_groups && R < a.n_max * a.group;
    const int qn = r_in ? R / a.group : 0;
    const int qh = hk * a.group + (r_in ? R % a.group : 0);
    const uint16_t* qrow = reinterpret_cast<const uint16_t*>(a.q) +
                           (((int64_t)b * a.n_max + qn) * a.hq + qh) * D;
#pragma unroll
    for (int ks = 0; ks < kKSteps; ++ks) {
      Pack8 p;
      p.u = r_in ? *reinterpret_cast<const uint4*>(qrow + ks * 32 + g * 8)
                 : make_uint4(0, 0, 0, 0);
      qreg[rg][ks] = p.v;
    }
  }
  const int my_parent = tid < a.n_max ? a.parent[(int64_t)b * a.n_max + tid] : -1;

  const int n_raw = a.n_nodes[b];
  const int L = a.ctx_len[b];
  const int64_t off = a.kv_off[b];
  asm volatile("" : : "s"(n_raw), "s"(L), "s"(off));
  const int N = min(n_raw, a.n_max);
  const int T = L + N;
  const int S = split_count(T, N, a.tps, at.max_splits);
  const int rows = N * a.group;
  if (S == 0) {                         // no nodes: nothing to compute; the empty tree is valid
    report_tree(a, b, true, s == 0 && hk == 0 && rb == 0);
    return;
  }
  if (s >= S || rb * a.rows_per_wg >= rows) return;

  const int begin = s * a.tps;
  const int end = (s == S - 1) ? T : begin + a.tps;

  const uint32_t seq_bytes = (uint32_t)T * (uint32_t)(a.hkv * G::kRowBytes);
  const bool dma_wave = wave < NDMA;
  uint32_t src_off[kDmaBlocks];
#pragma unroll
  for (int j = 0; j < kDmaBlocks; ++j) {
    const int byte = ((dma_wave ? wave : 0) * kDmaBlocks + j) * 1024 + lane * 16;
    const int row = byte / G::kRowBytes;
    const int pchunk = (byte % G::kRowBytes) >> 4;
    const int lchunk = pchunk ^ G::swz(row);
    src_off[j] = (uint32_t)((row * a.hkv + hk) * G::kRowBytes + (lchunk << 4));
  }
  const uint32_t tok_bytes = (uint32_t)(a.hkv * G::kRowBytes);
  const i32x4 rk4 = raw_rsrc(reinterpret_cast<const uint16_t*>(a.k) + off * a.hkv * D, seq_bytes);
  const i32x4 rv4 = raw_rsrc(reinterpret_cast<const uint16_t*>(a.v) + off * a.hkv * D, seq_bytes);
  // Tiles at or past the split's end are still issued (at an out-of-range
  // offset, which reads nothing) so that every iteration of a DMA wave has
  // the same number of DMAs in flight.
  auto dma_tile = [&](int buf, int t0) {
    if (!dma_wave) return;
    const bool live = t0 < end;
#pragma unroll
    for (int j = 0; j < kDmaBlocks; ++j) {
      const uint32_t voff = live ? src_off[j] + (uint32_t)t0 * tok_bytes : kOobOffset;
      const int blk = (wave * kDmaBlocks + j) * 1024;
      dma16(lds_addr(&s_k[buf][blk]), voff, rk4);
      dma16(lds_addr(&s_v[buf][blk]), voff, rv4);
    }
  };
#pragma unroll
  for (int i = 0; i < NBUF - 1; ++i) dma_tile(i, begin + i * kTile);

  // A row block may hold fewer rows than the workgroup has row waves.
  bool row_ok[RG];
  int n_of[RG], head_of[RG];
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    const int R = wrow + 16 * rg + c;
    row_ok[rg] = rg < my_groups && 16 * (first + rg) < a.rows_per_wg && R < rows;
    n_of[rg] = row_ok[rg] ? R / a.group : 0;
    head_of[rg] = hk * a.group + (row_ok[rg] ? R % a.group : 0);
  }
  const bool wave_active = my_groups > 0 && 16 * first < a.rows_per_wg && wrow < rows;

  // LDS byte offsets of this lane's operands inside a tile. The swizzle takes
  // only the row's low three bits, so a 16-row block's offset is a constant
  // (an instruction immediate) away from the first block's.
  int k_off[kKSteps];                              // K: row tb*16 + c, chunk 4 ks + g
#pragma unroll
  for (int ks = 0; ks < kKSteps; ++ks) k_off[ks] = G::offset(c, 4 * ks + g);
  const int v_row = 4 * g + (c >> 2);
  int v_off[kDBlk];                                // V^T: rows v_row (+16 h, +32 kt), 16-col block db
#pragma unroll
  for (int db = 0; db < kDBlk; ++db) v_off[db] = G::offset(v_row, 2 * db + ((c & 3) >> 1)) + (c & 1) * 8;

  if (end > L) {
    const bool ok = build_tree_loaded(N, my_parent, s_parent, s_anc, &s_bad);
    report_tree(a, b, ok, s == S - 1 && hk == 0 && rb == 0);
    if (!ok) {
      __builtin_amdgcn_s_waitcnt(0);
      return;
    }
  }

  f32x4 oacc[RG][kDBlk];
#pragma unroll
  for (int rg = 0; rg < RG; ++rg)
#pragma unroll
    for (int i = 0; i < kDBlk; ++i) oacc[rg][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run[RG], l_run[RG];
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    m_run[rg] = -INFINITY;
    l_run[rg] = 0.f;
  }
  const float cs = a.scale_log2;
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};

  // Queries and the first tiles have landed. (This also tells the compiler
  // that no load it issued is pending, so it adds no waits inside the loop.)
  __builtin_amdgcn_s_waitcnt(0);
#pragma unroll
  for (int rg = 0; rg < RG; ++rg)
    if (!row_ok[rg]) {
#pragma unroll
      for (int ks = 0; ks < kKSteps; ++ks) qreg[rg][ks] = bf16x8{};
    }
  for (int t0 = begin, buf = 0; t0 < end; t0 += kTile, buf = buf + 1 == NBUF ? 0 : buf + 1) {
    __builtin_amdgcn_s_waitcnt(kVmWait);  // this wave's DMA into `buf` has landed
    __syncthreads();                      // everyone's has; the previous buffer is free
    dma_tile(buf == 0 ? NBUF - 1 : buf - 1, t0 + (NBUF - 1) * kTile);
    if (!wave_active) continue;
    const unsigned char* kt = s_k[buf];
    const unsigned char* vt = s_v[buf];
    // The tile's work for NG row groups (NG = RG or RG - 1, this wave's count).
    auto tile_body = [&](auto ng) {
      constexpr int NG = decltype(ng)::value;
#pragma unroll
      for (int hs = 0; hs < HT; ++hs) {
        // Scores of this step's kTB 16-token blocks x NG row groups, each a
        // chain of kKSteps MFMAs; every K fragment feeds all NG groups.
        f32x4 sacc[NG][kTB];
#pragma unroll
        for (int rg = 0; rg < NG; ++rg)
#pragma unroll
          for (int tb = 0; tb < kTB; ++tb) sacc[rg][tb] = f32x4{0.f, 0.f, 0.f, 0.f};
        Pack8 kf[kKFrags];
        auto load_k = [&](Pack8& f, int i) {
          f.u = *reinterpret_cast<const uint4*>(kt + (hs * kTB + i % kTB) * 16 * G::kRowBytes +
                                                k_off[i / kTB]);
        };
#pragma unroll
        for (int i = 0; i < kAheadK; ++i) load_k(kf[i], i);
#pragma unroll
        for (int i = 0; i < kKFrags; ++i) {
          if (i + kAheadK < kKFrags) load_k(kf[i + kAheadK], i + kAheadK);
#pragma unroll
          for (int rg = 0; rg < NG; ++rg)
            sacc[rg][i % kTB] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[i].v, qreg[rg][i / kTB],
                                                                       sacc[rg][i % kTB], 0, 0, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x100, kAheadK, 0);
#pragma unroll
        for (int i = 0; i < kKFrags - kAheadK; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, NG, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, NG * kAheadK, 0);
        const int s0 = t0 + hs * 16 * kTB;             // first token of this step
        if (s0 + 16 * kTB > L) {
#pragma unroll
          for (int rg = 0; rg < NG; ++rg)
#pragma unroll
            for (int tb = 0; tb < kTB; ++tb)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const int tok = s0 + tb * 16 + 4 * g + r;
                sacc[rg][tb][r] += mask_bias(tok, L, end, n_of[rg], s_anc);
              }
        }
        // V^T fragment i: k-step hs * kPV + i / kDBlk, column block i % kDBlk.
        Pack8 vf[kVFrags];
        auto load_v = [&](Pack8& f, int i) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int rows0 = 32 * (hs * kPV + i / kDBlk) + 16 * h;   // multiple of 8: swizzle-free
            f.h[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (lds_i16x4*)(vt + rows0 * G::kRowBytes + v_off[i % kDBlk]));
          }
        };
#pragma unroll
        for (int i = 0; i < kAheadV; ++i) load_v(vf[i], i);
        // Probabilities of group rg against its running reference, bf16 for
        // the P V product, and the lane's share of the row sum from them.
        bf16x8 pb[NG][kPV];
        float lsum[NG];
        auto exps = [&](int rg, float nm) {
          float l0 = 0.f, l1 = 0.f;
#pragma unroll
          for (int kt2 = 0; kt2 < kPV; ++kt2) {
            bf16x8 v8;
#pragma unroll
            for (int j = 0; j < 8; ++j)
              v8[j] = (__bf16)fast_exp2(fmaf(sacc[rg][2 * kt2 + (j >> 2)][j & 3], cs, nm));
            pb[rg][kt2] = v8;
            l0 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v8[0], v8[1]}, ones, l0, false);
            l1 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v8[2], v8[3]}, ones, l1, false);
            l0 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v8[4], v8[5]}, ones, l0, false);
            l1 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v8[6], v8[7]}, ones, l1, false);
          }
          lsum[rg] = l0 + l1;
        };
        // The lazy rescale of the 16-row kernel: each group's reference moves
        // when its row maximum rises by more than 2^8, and the maxima are
        // reduced only when that can happen (a row without a reference, or a
        // lane whose probabilities sum to more than 2^8).
        bool no_ref = false;
#pragma unroll
        for (int rg = 0; rg < NG; ++rg) no_ref |= m_run[rg] == -INFINITY;
        bool have = false, check = true;
        if (__ballot(no_ref) == 0) {
          bool big = false;
#pragma unroll
          for (int rg = 0; rg < NG; ++rg) {
            exps(rg, -m_run[rg]);
            big |= !(lsum[rg] <= 256.f);
          }
          have = true;
          check = __ballot(big) != 0;
        }
        if (__builtin_expect(check, 0)) {
          // Row maxima (the lane's 4 kTB scores, then its 3 partners).
          float m_tile[NG];
          bool grow_any = false;
#pragma unroll
          for (int rg = 0; rg < NG; ++rg) {
            float mb = max3_raw(sacc[rg][0][0], sacc[rg][0][1], sacc[rg][0][2]);
#pragma unroll
            for (int i = 3; i + 1 < 4 * kTB; i += 2)
              mb = max3_raw(mb, sacc[rg][i >> 2][i & 3], sacc[rg][(i + 1) >> 2][(i + 1) & 3]);
            mb = max3_raw(mb, sacc[rg][kTB - 1][3], sacc[rg][kTB - 1][3]);
            mb = max3_raw(mb, partner<16>(mb), mb);
            m_tile[rg] = max_halves(mb) * cs;
            grow_any |= m_tile[rg] > m_run[rg] + kRescaleLog2;
          }
          const bool grew = __ballot(grow_any) != 0;
          if (grew) {
#pragma unroll
            for (int rg = 0; rg < NG; ++rg) {
              if (m_tile[rg] > m_run[rg] + kRescaleLog2) {
                const float alpha = fast_exp2(m_run[rg] - m_tile[rg]);
                l_run[rg] *= alpha;
#pragma unroll
                for (int i = 0; i < kDBlk; ++i) oacc[rg][i] *= alpha;
                m_run[rg] = m_tile[rg];
              }
            }
          }
          if (!have || grew) {
#pragma unroll
            for (int rg = 0; rg < NG; ++rg) exps(rg, m_run[rg] == -INFINITY ? 0.f : -m_run[rg]);
          }
        }
#pragma unroll
        for (int rg = 0; rg < NG; ++rg) l_run[rg] += lsum[rg];
#pragma unroll
        for (int i = 0; i < kVFrags; ++i) {
          if (i + kAheadV < kVFrags) load_v(vf[i + kAheadV], i + kAheadV);
#pragma unroll
          for (int rg = 0; rg < NG; ++rg)
            oacc[rg][i % kDBlk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                vf[i].v, pb[rg][i / kDBlk], oacc[rg][i % kDBlk], 0, 0, 0);
        }
      }
    };
    if (my_groups == RG) tile_body(std::integral_constant<int, RG>{});
    else tile_body(std::integral_constant<int, (RG > 1 ? RG - 1 : 1)>{});
  }

  __builtin_amdgcn_s_waitcnt(0);          // the ring's trailing DMAs land before exit
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    if (!row_ok[rg]) continue;
    const int n = n_of[rg], head = head_of[rg];
    float l_tot = l_run[rg] + partner<16>(l_run[rg]);
    l_tot = sum_halves(l_tot);
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    const float lse_nat = l_tot > 0.f ? (m_run[rg] + log2f(l_tot)) * kLn2 : -INFINITY;
    if (S == 1) {
      const int64_t obase = (((int64_t)b * a.n_max + n) * a.hq + head) * D;
#pragma unroll
      for (int db = 0; db < kDBlk; ++db) {
        const int d0 = db * 16 + 4 * g;
        const float x0 = oacc[rg][db][0] * inv, x1 = oacc[rg][db][1] * inv;
        const float x2 = oacc[rg][db][2] * inv, x3 = oacc[rg][db][3] * inv;
        if (a.out_bf16) {
          uint2 pk;
          pk.x = pack_bf16x2(x0, x1);
          pk.y = pack_bf16x2(x2, x3);
          *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.o) + obase + d0) = pk;
        } else {
          *reinterpret_cast<float4*>(reinterpret_cast<float*>(a.o) + obase + d0) =
              make_float4(x0, x1, x2, x3);
        }
      }
      if (g == 0 && a.lse) a.lse[((int64_t)b * a.n_max + n) * a.hq + head] = lse_nat;
    } else {
      const int64_t pi = part_index(a, b, head, n, s);
#pragma unroll
      for (int db = 0; db < kDBlk; ++db)
        *reinterpret_cast<float4*>(a.part_o + pi * D + db * 16 + 4 * g) =
            make_float4(oacc[rg][db][0] * inv, oacc[rg][db][1] * inv, oacc[rg][db][2] * inv,
                        oacc[rg][db][3] * inv);
      if (g == 0) a.part_lse[pi] = lse_nat;
    }
  }
}

// ---------------------------------------------------------------------------
// fp32 split kernel on the matrix cores (v_mfma_f32_16x16x4_f32, fp32 products
// and sums: the same precision as the vector-ALU kernel).
//
// Bound by the fp32 matrix rate (256 flop per clock and CU; a large fp32 GEMM
// reaches 137 TFLOP/s on this card) and by what the matrix unit waits for: on the
// first batch below it is busy for 64 % of the cycles in which a SIMD holds its two
// waves, these wait for 22 % of theirs, and an LDS instruction has 1.7 conflict
// cycles. A workgroup is four waves over a block of
// 32 rows (or 16, when a kv-head has no more), each wave owning 16 query rows
// and 1 / WT of every tile's tokens (WT = 2 or 4), so no wave idles; the token
// shares are combined through LDS at the end. Small blocks fill two workgroups
// per CU evenly, which counts for more than reading K/V once per 64 rows (the
// row blocks of a kv-head share an XCD's L2): blocks of 64 rows (WT = 1) took
// 46.9 us against 40.3 on the first batch below, 1095 against 948 for 8
// sequences of 8k tokens and 80 nodes, and only a single 32k sequence gained
// (158 against 169). Measured per call against the vector-ALU kernel, which it
// replaces for aligned operands (its LDS broadcast of every query element per
// multiply bound it to 11 TFLOP/s): 4 sequences of 850 - 1780 tokens, 32 nodes,
// 32/8 heads of 128: 257 -> 40.3 us, 69 TFLOP/s with the merge; one sequence of
// 128 tokens, 12 nodes, 4 heads of 64: 29.2 -> 7.7 us in the kernel.
//
// Lane l = 16 g + c owns query row c of its wave's 16.
//   S^T = K Q^T, 16 tokens at a time: MFMA i of column group j (16 columns)
//     takes k index g for column 16 j + 4 g + i, so that one 16-byte read of K
//     (row c, columns 16 j + 4 g .. +3) feeds four MFMAs
//     D register r = score of token 4 g + r for row c
//   O^T += V^T P^T: MFMA r takes k index g for token 4 g + r, the probability
//     the lane already holds in register r; output row c' of block 4 h + i
//     stands for column 64 h + 4 c' + i, so that one 16-byte read of V (row
//     4 g + r, columns 64 h + 4 c .. +3) feeds four MFMAs
//     D register r of block 4 h + i = O column 64 h + 16 g + 4 r + i of row c
// LDS rows are XOR-swizzled by 16-byte chunk, so that the 16 lanes of a group cover
// all banks in the K reads (16 rows, one chunk column) and in the V reads (one row,
// 16 chunks).
// Hidden and out-of-range scores are replaced, not added to: an infinite or NaN
// K row that a node does not see leaves its result alone.
template <int D, int WT>
struct F32Geo {
  static_assert(WT == 2 || WT == 4, "two or four token shares");
  static constexpr int kTok = WT == 4 ? 64 : 32;         // tokens per K/V tile
  static constexpr int kTB = kTok / 16 / WT;             // 16-token blocks per wave and tile
  static constexpr int kRows = 64 / WT;                  // query rows per workgroup
  static constexpr int kRowBytes = D * 4;
  static constexpr int kTileBytes = kTok * kRowBytes;
  static constexpr int kDmaPerWave = kTileBytes / 1024 / 4;
  static constexpr int kWgsPerCu = kTileBytes > 16384 ? 1 : 2;   // LDS: two tiles of K and of V
  static CURE_DEV int offset(int row, int chunk) { return row * kRowBytes + ((chunk ^ (row & 15)) << 4); }
};

template <int D, int WT, class A>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu((F32Geo<D, WT>::kWgsPerCu))))
void tree_attn_f32(A a) {
  using G = F32Geo<D, WT>;
  constexpr int kTB = G::kTB;
  constexpr int kKGroups = D / 16;                 // 16-column groups of Q K^T
  constexpr int kDBlk = D / 16;                    // output blocks of 16 columns
  constexpr int kH = D / 64;

  __shared__ int s_parent[CURE_MAX_TREE_NODES];
  __shared__ unsigned long long s_anc[CURE_MAX_TREE_NODES][kAncWords];
  __shared__ int s_bad;
  __shared__ __attribute__((aligned(1024))) unsigned char s_kv[2][2][G::kTileBytes];  // [buffer][K, V]

  const Place at = locate(a);
  const int b = at.b, hk = at.hk, rb = at.rb, s = at.s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane & 15, g = lane >> 4;
  const int wt = wave % WT, wr = wave / WT;        // this wave's share of the tokens and its rows

  // Query loads (they need only the launch shape) and the parent entry go out
  // with the loads of the sequence's sizes.
  const int R = rb * G::kRows + wr * 16 + c;
  const bool r_in = R < a.n_max * a.group;
  f32x4 qreg[kKGroups];
  {
    const int qn = r_in ? R / a.group : 0;
    const int qh = hk * a.group + (r_in ? R % a.group : 0);
    const float* qrow = reinterpret_cast<const float*>(a.q) + (((int64_t)b * a.n_max + qn) * a.hq + qh) * D;
#pragma unroll
    for (int j = 0; j < kKGroups; ++j)
      qreg[j] = r_in ? *reinterpret_cast<const f32x4*>(qrow + 16 * j + 4 * g) : f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const int my_parent = tid < a.n_max ? a.parent[(int64_t)b * a.n_max + tid] : -1;

  const int n_raw = a.n_nodes[b];
  const int L = a.ctx_len[b];
  const int64_t off = a.kv_off[b];
  asm volatile("" : : "s"(n_raw), "s"(L), "s"(off));
  const int N = min(n_raw, a.n_max);
  const int T = L + N;
  const int S = split_count(T, N, a.tps, at.max_splits);
  const int rows = N * a.group;
  if (S == 0) {                         // no nodes: nothing to compute; the empty tree is valid
    report_tree(a, b, true, s == 0 && hk == 0 && rb == 0);
    return;
  }
  if (s >= S || rb * G::kRows >= rows) return;

  const int begin = s * a.tps;
  const int end = (s == S - 1) ? T : begin + a.tps;

  // The tile DMA of the bf16 kernels, with the tile's own rows as the buffer
  // resource, whose base moves on by a tile with each call: the device's lengths
  // may exceed the host's copies, and fp32 rows soon pass what 32-bit offsets
  // from the start of a sequence reach. Rows past the sequence read as zeros, and
  // a tile at or past the split's end has none.
  const uint32_t tok_bytes = (uint32_t)(a.hkv * G::kRowBytes);
  uint32_t src_off[G::kDmaPerWave];                // per lane and 1 KB block
#pragma unroll
  for (int j = 0; j < G::kDmaPerWave; ++j) {
    const int byte = (wave * G::kDmaPerWave + j) * 1024 + lane * 16;
    const int row = byte / G::kRowBytes;
    const int pchunk = (byte % G::kRowBytes) >> 4;
    src_off[j] = (uint32_t)row * tok_bytes + (uint32_t)(hk * G::kRowBytes + ((pchunk ^ (row & 15)) << 4));
  }
  const char* k_tile = reinterpret_cast<const char*>(a.k) + (off + begin) * (int64_t)tok_bytes;
  const char* v_tile = reinterpret_cast<const char*>(a.v) + (off + begin) * (int64_t)tok_bytes;
  auto dma_tile = [&](int buf, int t0) {
    const uint32_t bytes = t0 < end ? (uint32_t)min(T - t0, G::kTok) * tok_bytes : 0u;
    const i32x4 rk4 = raw_rsrc(k_tile, bytes), rv4 = raw_rsrc(v_tile, bytes);
    k_tile += (int64_t)G::kTok * tok_bytes;
    v_tile += (int64_t)G::kTok * tok_bytes;
#pragma unroll
    for (int j = 0; j < G::kDmaPerWave; ++j) {
      const int blk = (wave * G::kDmaPerWave + j) * 1024;
      dma16(lds_addr(&s_kv[buf][0][blk]), src_off[j], rk4);
      dma16(lds_addr(&s_kv[buf][1][blk]), src_off[j], rv4);
    }
  };
  dma_tile(0, begin);

  const bool row_ok = R < rows;
  const int n = row_ok ? R / a.group : 0;
  const int head = hk * a.group + (row_ok ? R % a.group : 0);
  const bool wave_active = rb * G::kRows + wr * 16 < rows;

  int k_off[kKGroups];                             // K: row 16 (kTB wt + tb) + c, chunk 4 j + g
#pragma unroll
  for (int j = 0; j < kKGroups; ++j) k_off[j] = G::offset(kTB * wt * 16 + c, 4 * j + g);
  int v_off[4];                                    // V: row 16 (kTB wt + tb) + 4 g + r, chunk 16 h + c
#pragma unroll
  for (int r = 0; r < 4; ++r) v_off[r] = G::offset(kTB * wt * 16 + 4 * g + r, c);

  // Only a split that reaches the tree's own rows needs the ancestor masks.
  if (end > L) {
    const bool ok = build_tree_loaded(N, my_parent, s_parent, s_anc, &s_bad);
    report_tree(a, b, ok, s == S - 1 && hk == 0 && rb == 0);
    if (!ok) {
      __builtin_amdgcn_s_waitcnt(0);               // no DMA may land after the workgroup ends
      return;
    }
  }

  f32x4 oacc[kDBlk];
#pragma unroll
  for (int i = 0; i < kDBlk; ++i) oacc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;            // l_run: this lane's share of the row sum
  const float cs = a.scale_log2;

  __builtin_amdgcn_s_waitcnt(0);
  if (!row_ok) {
#pragma unroll
    for (int j = 0; j < kKGroups; ++j) qreg[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  for (int t0 = begin, buf = 0; t0 < end; t0 += G::kTok, buf ^= 1) {
    __builtin_amdgcn_s_waitcnt(0);                 // this wave's DMA into `buf` has landed
    __syncthreads();                               // everyone's has; the other buffer is free
    dma_tile(buf ^ 1, t0 + G::kTok);
    if (!wave_active) continue;
    const unsigned char* kt = s_kv[buf][0];
    const unsigned char* vt = s_kv[buf][1];

    f32x4 sacc[kTB];
#pragma unroll
    for (int tb = 0; tb < kTB; ++tb) sacc[tb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < kKGroups; ++j) {
      f32x4 kf[kTB];
#pragma unroll
      for (int tb = 0; tb < kTB; ++tb)
        kf[tb] = *reinterpret_cast<const f32x4*>(kt + tb * 16 * G::kRowBytes + k_off[j]);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int tb = 0; tb < kTB; ++tb)
          sacc[tb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[tb][i], qreg[j][i], sacc[tb], 0, 0, 0);
    }
    // Scores in the log2 domain; hidden ones become -inf.
    float x[kTB][4];
    const bool tail = t0 + G::kTok > L;
#pragma unroll
    for (int tb = 0; tb < kTB; ++tb)
#pragma unroll
      for (int r = 0; r < 4; ++r) x[tb][r] = sacc[tb][r] * cs;
    if (tail) {
#pragma unroll
      for (int tb = 0; tb < kTB; ++tb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int tok = t0 + (kTB * wt + tb) * 16 + 4 * g + r;
          x[tb][r] = mask_bias(tok, L, end, n, s_anc) == 0.f ? x[tb][r] : -INFINITY;
        }
    }
    float mt = -INFINITY;
#pragma unroll
    for (int tb = 0; tb < kTB; ++tb)
#pragma unroll
      for (int r = 0; r < 4; ++r) mt = fmaxf(mt, x[tb][r]);
    mt = max_halves(fmaxf(mt, partner<16>(mt)));   // the row's tokens sit in lanes c + 16 k
    const float m_new = fmaxf(m_run, mt);
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    if (__ballot(m_new > m_run)) {                 // a maximum rose: rescale (factor 1 for the others)
      const float alpha = fast_exp2(m_run - m_use);
      l_run *= alpha;
#pragma unroll
      for (int i = 0; i < kDBlk; ++i) oacc[i] *= alpha;
    }
    m_run = m_new;
    float p[kTB][4], ps = 0.f;
#pragma unroll
    for (int tb = 0; tb < kTB; ++tb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p[tb][r] = fast_exp2(x[tb][r] - m_use);
        ps += p[tb][r];
      }
    l_run += ps;
#pragma unroll
    for (int tb = 0; tb < kTB; ++tb)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int h = 0; h < kH; ++h) {
          const f32x4 vf = *reinterpret_cast<const f32x4*>(vt + tb * 16 * G::kRowBytes + h * 256 + v_off[r]);
#pragma unroll
          for (int i = 0; i < 4; ++i)
            oacc[4 * h + i] =
                __builtin_amdgcn_mfma_f32_16x16x4f32(vf[i], p[tb][r], oacc[4 * h + i], 0, 0, 0);
        }
  }

  __builtin_amdgcn_s_waitcnt(0);                   // the trailing out-of-range DMA lands before LDS is reused
  float l_tot = l_run + partner<16>(l_run);
  l_tot = sum_halves(l_tot);
  {
    // The other token shares of these rows, a record of D + 2 floats per row
    // and share in the tile buffers, once every wave is done with those.
    __syncthreads();
    float* s_o = reinterpret_cast<float*>(&s_kv[0][0][0]);
    constexpr int kRec = 64 * (4 * kDBlk + 2);     // floats per wave
    static_assert(4 * kRec * 4 <= (int)sizeof(s_kv), "the token shares fit the tile buffers");
    if (wt > 0) {
      float* d = s_o + wave * kRec + lane;
#pragma unroll
      for (int i = 0; i < kDBlk; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) d[64 * (4 * i + r)] = oacc[i][r];
      d[64 * 4 * kDBlk] = m_run;
      d[64 * (4 * kDBlk + 1)] = l_tot;
    }
    __syncthreads();
    if (wt > 0) return;
#pragma unroll
    for (int w = 1; w < WT; ++w) {
      const float* d = s_o + (wave + w) * kRec + lane;
      const float m2 = d[64 * 4 * kDBlk], l2 = d[64 * (4 * kDBlk + 1)];
      const float m_new = fmaxf(m_run, m2);
      const float m_use = m_new == -INFINITY ? 0.f : m_new;
      const float a1 = fast_exp2(m_run - m_use), a2 = fast_exp2(m2 - m_use);
      l_tot = l_tot * a1 + l2 * a2;
#pragma unroll
      for (int i = 0; i < kDBlk; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) oacc[i][r] = oacc[i][r] * a1 + d[64 * (4 * i + r)] * a2;
      m_run = m_new;
    }
  }
  if (!row_ok) return;
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  const float lse_nat = l_tot > 0.f ? (m_run + log2f(l_tot)) * kLn2 : -INFINITY;
  const int64_t orow = ((int64_t)b * a.n_max + n) * a.hq + head;
  const int64_t pi = S == 1 ? 0 : part_index(a, b, head, n, s);
#pragma unroll
  for (int h = 0; h < kH; ++h)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int d0 = 64 * h + 16 * g + 4 * r;
      const float4 x = make_float4(oacc[4 * h][r] * inv, oacc[4 * h + 1][r] * inv,
                                   oacc[4 * h + 2][r] * inv, oacc[4 * h + 3][r] * inv);
      if (S > 1) {
        *reinterpret_cast<float4*>(a.part_o + pi * D + d0) = x;
      } else if (a.out_bf16) {
        uint2 pk;
        pk.x = pack_bf16x2(x.x, x.y);
        pk.y = pack_bf16x2(x.z, x.w);
        *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.o) + orow * D + d0) = pk;
      } else {
        *reinterpret_cast<float4*>(reinterpret_cast<float*>(a.o) + orow * D + d0) = x;
      }
    }
  if (g == 0) {
    if (S > 1) a.part_lse[pi] = lse_nat;
    else if (a.lse) a.lse[orow] = lse_nat;
  }
}

// ---------------------------------------------------------------------------
// LSE merge: one wave per output row (b, n, head).
//
// A split's partial row is D floats = D/4 lanes of float4, so one load
// instruction covers 64/(D/4) splits (2 at D=128, 4 at D=64). A batch of NB
// such loads, with each split's LSE alongside, is issued before anything is
// reduced, and NB is the smallest of 2, 4, 8 that covers the launch's largest
// split count when it can: the partials then take one memory round trip,
// with no more registers held than that needs. When every sequence has the
// launch's largest split count that batch goes out with the loads of the
// sequence's sizes; otherwise (kOwnSplits, a ragged batch) the sizes come
// first and each row reads only its own splits' slots, instead of fetching
// slots it would discard. The lane groups holding different splits are
// combined with xor shuffles at the end.
template <int D, int NB, bool kOwnSplits, class A>
__global__ __launch_bounds__(256) void attn_merge(A a) {
  constexpr int kLanesPerSplit = D / 4;
  constexpr int kSplitsPerLoad = kWave / kLanesPerSplit;
  constexpr int kSplitsPerBatch = kSplitsPerLoad * NB;
  // Grid (heads / 4, n_max, batch): the row's coordinates come straight from
  // the block index (no 64-bit divisions).
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int head = blockIdx.x * 4 + wave;
  const int n = blockIdx.y;
  const int b = blockIdx.z;
  if (head >= a.hq) return;
  const int64_t p0 = part_index(a, b, head, n, 0);
  const int sub = lane / kLanesPerSplit;            // which split of a load this lane holds
  const int col = (lane % kLanesPerSplit) * 4;      // its four output columns

  // The first batch of partials is loaded together with the sequence's sizes
  // (its addresses need neither): one memory round trip. Slots past the
  // sequence's own split count hold stale data and are masked out below.
  float4 v[NB];
  float l[NB];
  auto load_batch = [&](int s0, int limit) {
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int sp = s0 + u * kSplitsPerLoad + sub;
      const bool ok = sp < limit;
      v[u] = ok ? *reinterpret_cast<const float4*>(a.part_o + (p0 + sp) * D + col)
                : make_float4(0.f, 0.f, 0.f, 0.f);
      l[u] = ok ? a.part_lse[p0 + sp] : -INFINITY;
    }
  };
  if (!kOwnSplits) load_batch(0, a.max_splits);
  const int n_raw = a.n_nodes[b];
  const int L = a.ctx_len[b];
  const int N = min(n_raw, a.n_max);
  if (n >= N) return;
  const int S = split_count(L + N, N, a.tps, max_splits_of(a, b));
  if (S <= 1) return;
  if (kOwnSplits) {
    load_batch(0, S);
  } else {
    // Slots past this sequence's own split count get zero weight (the plan
    // comes from host copies of the sizes, so this cannot be taken for granted).
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      if (u * kSplitsPerLoad + sub >= S) {
        v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        l[u] = -INFINITY;
      }
    }
  }
  // Reference maximum: from the loaded batch when it holds every split, else
  // from all of the row's LSEs.
  float m = -INFINITY;
  if (S <= kSplitsPerBatch) {
#pragma unroll
    for (int u = 0; u < NB; ++u) m = fmaxf(m, l[u]);
  } else {
    for (int sp = lane; sp < S; sp += kWave) m = fmaxf(m, a.part_lse[p0 + sp]);
  }
  m = wave_max(m);
  const float ms = m == -INFINITY ? 0.f : m;     // empty splits (lse = -inf) weigh 0

  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  float wsum = 0.f;
  for (int s0 = 0;;) {
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const float w = fast_exp2((l[u] - ms) * kLog2e);
      wsum += w;
      acc.x = fmaf(w, v[u].x, acc.x);
      acc.y = fmaf(w, v[u].y, acc.y);
      acc.z = fmaf(w, v[u].z, acc.z);
      acc.w = fmaf(w, v[u].w, acc.w);
    }
    s0 += kSplitsPerBatch;
    if (s0 >= S) break;
    load_batch(s0, S);
  }
  if (kLanesPerSplit == 16) {                       // lane groups 16 apart
    acc.x += partner<16>(acc.x);
    acc.y += partner<16>(acc.y);
    acc.z += partner<16>(acc.z);
    acc.w += partner<16>(acc.w);
    wsum += partner<16>(wsum);
  }
  acc.x = sum_halves(acc.x);                        // and 32 apart
  acc.y = sum_halves(acc.y);
  acc.z = sum_halves(acc.z);
  acc.w = sum_halves(acc.w);
  wsum = sum_halves(wsum);
  if (sub != 0) return;
  const float inv = wsum > 0.f ? 1.f / wsum : 0.f;
  const int64_t obase = (((int64_t)b * a.n_max + n) * a.hq + head) * D + col;
  store_out(a, obase, acc.x * inv);
  store_out(a, obase + 1, acc.y * inv);
  store_out(a, obase + 2, acc.z * inv);
  store_out(a, obase + 3, acc.w * inv);
  if (lane == 0 && a.lse) a.lse[((int64_t)b * a.n_max + n) * a.hq + head] =
      wsum > 0.f ? m + logf(wsum) : -INFINITY;
}

// ---------------------------------------------------------------------------
// LSE merge of launches with at most four splits: D / 4 lanes per output row (b, n,
// head), each holding four columns of every split's partial row, so a wave covers
// two rows at head dim 128 and four at 64 and combines them without any exchange
// between lanes. Every split's loads are issued before the sequence's sizes have
// arrived (the launch says how many splits the sequence may have; slots past its
// own count on the device are masked out).
//
// Bound by the partials' round trips, so by how many waves of them there are: a
// wave per row takes several rounds once a launch has more rows than the chip
// holds waves (8192), which is what large launches with few splits have. Per
// call, wave per row and here: ragged batch (3 splits, 24.6k rows) 61.2 and
// 58.8 us; 80-node trees of 8 sequences (4 splits, 20.5k rows) 105.9 and 103.2,
// where the runs of one side differ by 2.8 %; head dim 64 (2 splits, 24.6k rows)
// 33.3 and 32.3, (16.4k rows) 35.8 and 35.1.
// With fewer rows or more splits the wave per row is ahead, as it spreads a row's
// loads over more lanes: fp32 (8.2k rows) 46.4 and 47.1, 2 sequences (2k rows)
// 11.3 and 12.7; 32k context (8 splits) 105.5 and 106.8, head dim 64 (11
// splits) 30.3 and 34.2.
constexpr int kFewSplits = 4;
constexpr int64_t kManyRows = 16384;
static_assert(kFewSplits == 4, "instantiated for two and four splits");

template <int D, int NB, class A>
__global__ __launch_bounds__(256) void attn_merge_few(A a) {
  constexpr int kLanes = D / 4;
  constexpr int kRows = 256 / kLanes;
  // Grid (heads / kRows, n_max, batch): the row's coordinates come straight from
  // the block index (no 64-bit divisions).
  const int head = blockIdx.x * kRows + threadIdx.x / kLanes;
  const int col = (threadIdx.x % kLanes) * 4;
  const int n = blockIdx.y;
  const int b = blockIdx.z;
  if (head >= a.hq) return;
  const int64_t p0 = part_index(a, b, head, n, 0);
  const int slots = max_splits_of(a, b);
  float4 v[NB];
  float l[NB];
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const bool ok = u < slots;
    v[u] = ok ? *reinterpret_cast<const float4*>(a.part_o + (p0 + u) * D + col)
              : make_float4(0.f, 0.f, 0.f, 0.f);
    l[u] = ok ? a.part_lse[p0 + u] : -INFINITY;
  }
  const int n_raw = a.n_nodes[b];
  const int L = a.ctx_len[b];
  const int N = min(n_raw, a.n_max);
  if (n >= N) return;
  const int S = split_count(L + N, N, a.tps, slots);
  if (S <= 1) return;
  // Slots past the count hold stale data (the plan comes from host copies of the
  // sizes): no weight, and no value that could turn one into a NaN.
  float m = -INFINITY;
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    if (u >= S) {
      v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      l[u] = -INFINITY;
    }
    m = fmaxf(m, l[u]);
  }
  const float ms = m == -INFINITY ? 0.f : m;               // empty splits (lse = -inf) weigh 0
  float wsum = 0.f;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const float w = fast_exp2((l[u] - ms) * kLog2e);
    wsum += w;
    acc.x = fmaf(w, v[u].x, acc.x);
    acc.y = fmaf(w, v[u].y, acc.y);
    acc.z = fmaf(w, v[u].z, acc.z);
    acc.w = fmaf(w, v[u].w, acc.w);
  }
  const float inv = wsum > 0.f ? 1.f / wsum : 0.f;
  const int64_t orow = ((int64_t)b * a.n_max + n) * a.hq + head;
  const int64_t obase = orow * D + col;
  store_out(a, obase, acc.x * inv);
  store_out(a, obase + 1, acc.y * inv);
  store_out(a, obase + 2, acc.z * inv);
  store_out(a, obase + 3, acc.w * inv);
  if (col == 0 && a.lse) a.lse[orow] = wsum > 0.f ? m + logf(wsum) : -INFINITY;
}

// Status of a launch with no tree nodes at all: every sequence's (empty)
// tree is valid. A fill kernel rather than a memset, so that the call stays
// capturable in a graph.
__global__ __launch_bounds__(256) void tree_status_ok(int32_t* status, int batch) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < batch) status[i] = CURE_OK;
}

// ---------------------------------------------------------------------------
// Host-side plan: tokens per split and the launch shape.
enum class Path { kValu, kF32, kBf16 };   // kernel family: vector ALU, fp32 or bf16 matrix cores

struct Plan {
  Path path;
  bool rows16;        // MFMA kernel with 16 query rows per wave
  bool rows64;        // head dim 64 beyond 128 rows: tree_attn_rg with two or three row groups,
  bool rows32;        // or the MFMA kernel with 32 query rows per wave
  bool rows48;        // MFMA kernel with three 16-row groups per wave (tree_attn_rg)
  int nw;             // waves per workgroup
  int rows_per_wg;
  int row_blocks;
  int tps;
  int max_splits;
  bool uniform_splits;  // every sequence with nodes has max_splits splits (host sizes)
  int wgs_per_cu;       // workgroups of the kernel that a CU holds at once, by LDS and registers
};

// The three-row-group kernel as instantiated: 8 waves of up to 48 query rows
// (one workgroup per CU, a two-tile ring), two 32-token softmax steps per
// tile; planned for 257 - 384 rows.
constexpr int kRg3Waves = 8;
constexpr int kRg3Rows = kRg3Waves * 48;
// Head dim 64 beyond 128 rows: the most rows of a workgroup of tree_attn_rg.
constexpr int kRg64Rows4 = 4 * 48;

Plan make_plan(int32_t batch, int32_t hq, int32_t hkv, int32_t d, int32_t n_max,
               const int32_t* host_ctx_len, const int32_t* host_n_nodes, int32_t kv_split,
               Path path) {
  Plan p{};
  p.path = path;
  const bool mfma = path == Path::kBf16;
  const int group = hq / hkv;
  const int rows = n_max * group;
  // Head dim 128: the 16-row kernel, in balanced row blocks of at most 256
  // rows (8 waves up to 128 rows, else 16), except for 257 - 384 rows, which
  // one workgroup of the three-row-group kernel covers. Per call at 8k
  // context x 8 sequences: 320 rows 126 µs against 144 for two 160-row
  // blocks of the 16-row kernel, 352 rows 139 against 151; at 224 and 256
  // rows the 16-row kernel's single block is ahead (103 vs 106, 109 vs 113).
  // Head dim 64: the 16-row kernel up to 128 rows, else two or three row groups
  // per wave or 32 rows per wave.
  p.rows48 = mfma && d == 128 && rows > 256 && rows <= kRg3Rows;
  p.rows64 = mfma && d == 64 && rows > 128;
  p.rows16 = mfma && !p.rows48 && !p.rows64;
  // Row blocks of at most `most` rows, balanced, in multiples of 16.
  const auto balance_rows = [&](int most) {
    p.row_blocks = (rows + most - 1) / most;
    p.rows_per_wg = ((rows + p.row_blocks - 1) / p.row_blocks + 15) / 16 * 16;
  };
  if (p.rows48) {
    // 257 - 384 rows: one block of eight waves of two or three 16-row groups,
    // so each K/V tile is streamed once per kv-head (two 16-row blocks would
    // stream it twice) and every LDS operand read feeds two or three row
    // groups. The block holds exactly the launch's row groups, so the kernel
    // deals them evenly over the SIMDs.
    p.row_blocks = 1;
    p.rows_per_wg = (rows + 15) / 16 * 16;
    p.nw = kRg3Waves;
  } else if (p.rows16) {
    balance_rows(256);
    p.nw = p.rows_per_wg > 128 ? 16 : 8;
  } else if (p.rows64) {
    // Blocks of at most 256 rows at first; the waves come with the splits, below.
    balance_rows(256);
  } else {
    if (path == Path::kF32) {
      // Four waves over 32 rows, two to a row group (F32Geo's WT = 2): the
      // vector-ALU kernel's blocks, and with two workgroups per CU its splits,
      // so no call needs more workspace. Up to 16 rows share the tokens four ways.
      p.nw = 4;
      p.rows_per_wg = rows <= 16 ? 16 : 32;
    } else {
      p.nw = kValuWaves;
      p.rows_per_wg = kValuRows;
    }
    p.row_blocks = std::max(1, (rows + p.rows_per_wg - 1) / p.rows_per_wg);
  }
  int64_t t_max = 0, t_sum = 0;
  for (int b = 0; b < batch; ++b) {
    const int N = std::min(host_n_nodes[b], n_max);
    if (N <= 0) continue;
    const int64_t T = (int64_t)host_ctx_len[b] + N;
    t_max = std::max(t_max, T);
    t_sum += T;
  }
  const auto round_tile = [](int64_t t) {
    return std::max<int64_t>(kTile, (t + kTile - 1) / kTile * kTile);
  };
  // Workgroups of one launch: splits of every sequence x kv-heads x row blocks.
  const auto workgroups = [&](int64_t tps) {
    int64_t c = 0;
    for (int b = 0; b < batch; ++b) {
      const int N = std::min(host_n_nodes[b], n_max);
      if (N > 0) c += ((int64_t)host_ctx_len[b] + N + tps - 1) / tps;
    }
    return c * hkv * p.row_blocks;
  };
  // Workgroups planned per CU. Two 8-wave 16-row workgroups fit one, but the
  // longer splits of one halve the partial rows the merge reads, and a second
  // workgroup measured no faster.
  int wgs_per_cu = 2;
  if (p.rows16 || p.rows48) wgs_per_cu = 1;
  else if (path == Path::kF32 && d == 128 && p.rows_per_wg == 16) wgs_per_cu = F32Geo<128, 4>::kWgsPerCu;
  const int64_t cus = device_cu_count();
  int64_t slots = wgs_per_cu * cus;
  // The shortest split (at least kMinTps tokens) whose workgroups are all
  // resident at once, so no workgroup waits for a second round. A batch with
  // more sequence x head pairs than that gets a single split per sequence.
  const auto shortest_resident_split = [&]() {
    const int64_t hi = round_tile(t_max);
    const int64_t lo = round_tile(std::max<int64_t>(
        kMinTps, (t_sum * hkv * p.row_blocks + slots - 1) / std::max<int64_t>(1, slots)));
    if (lo >= hi || workgroups(hi) > slots) return hi;
    // workgroups() falls as tps grows: bisect over multiples of the tile.
    int64_t a = lo / kTile, z = hi / kTile;         // workgroups(z * kTile) <= slots
    while (a < z) {
      const int64_t m = (a + z) / 2;
      if (workgroups(m * kTile) <= slots) z = m;
      else a = m + 1;
    }
    return z * kTile;
  };
  int64_t tps;
  // fp32 blocks that overfill the chip in single splits may leave much of a last round
  // idle (640 blocks of 512 slots: 62 % used). Then the bf16 plan's splits are taken, which
  // spread that round thinner; the workspace covers them. Single splits and these, us a
  // call at 80 nodes: 8 sequences of 8k tokens 935 and 815, 10 of 4k (78 % used) 626 and
  // 559, 9 of 0.7k - 4k (70 %) 407 and 354, 8 of 0.4k - 1.4k 181 and 161, though 9 of 2.5k
  // 320 and 335. At 0.7k - 1.2k tokens the merge costs what the round gains (8 of 700 119
  // and 145, 9 of 1.2k 181 and 197), and 88 % used and more leave nothing to gain (11 of 700
  // 146 and 153 in two splits). At head dim 64 a CU holds three of these workgroups, so the
  // round is not idle (16 sequences of 500 tokens, 768 blocks: 41 in single splits, 64 split).
  const auto fp32_tail_idle = [&]() {
    const int64_t wgs = workgroups(round_tile(t_max));
    return path == Path::kF32 && d == 128 && t_max > 1280 && wgs > slots &&
           5 * wgs < 4 * ((wgs + slots - 1) / slots * slots);
  };
  if (kv_split > 0) {
    tps = round_tile((t_max + kv_split - 1) / kv_split);
  } else if (fp32_tail_idle()) {
    tps = make_plan(batch, hq, hkv, d, n_max, host_ctx_len, host_n_nodes, 0, Path::kBf16).tps;
  } else {
    tps = shortest_resident_split();
    // A small launch (even the shortest splits leave most CUs idle, as for one
    // sequence) cuts the 16-row kernel's rows into more blocks, of at least 32
    // rows: the blocks of one kv-head and split are hkv workgroup ids apart,
    // so they share an XCD's L2 for the K/V stream, and more CUs stream it
    // (one sequence at 128 rows: 72 -> 216 workgroups).
    const int64_t fits = slots / std::max<int64_t>(1, workgroups(tps));
    if (p.rows16 && fits >= 2 && rows >= 64) {
      const int blocks = (int)std::min<int64_t>((int64_t)p.row_blocks * fits, rows / 32);
      if (blocks > p.row_blocks) {
        p.rows_per_wg = ((rows + blocks - 1) / blocks + 15) / 16 * 16;
        p.row_blocks = (rows + p.rows_per_wg - 1) / p.rows_per_wg;
        p.nw = p.rows_per_wg > 128 ? 16 : 8;
        tps = shortest_resident_split();
      }
    }
  }
  // Head dim 64 beyond 128 rows. Blocks of at most 192 rows: tree_attn_rg with eight
  // waves of two row groups when one workgroup per CU holds the launch, and with four
  // waves of three, two workgroups per CU, otherwise: with equal splits eight waves
  // start faster (4 sequences of 0.5k - 2k tokens, 192 rows: 17.6 us a call against
  // 19.2), and two four-wave workgroups fill a CU better (16 of 8k: 79.3 against 84.5).
  // Rows that balance to larger blocks are cut that small when the launch stays within
  // one workgroup per CU (one sequence of 2k, 256 rows: 16.6 against 18.4), and are left
  // to tree_attn_mfma otherwise. Neither changes the splits: longer ones, for one
  // workgroup per CU, were 0 - 25 % faster on short contexts, but the error against 64
  // bits grew by up to 2.9 %: a row's probabilities are rounded to bf16 against the
  // maximum over its split's first tile, and the largest one is exact when it is that
  // maximum, which is rarer the longer a split is.
  if (p.rows64 && p.rows_per_wg > kRg64Rows4) {
    balance_rows(kRg64Rows4);
    if (workgroups(tps) > cus) {
      p.rows64 = false;
      p.rows32 = true;
      p.rows_per_wg = 256;
      p.row_blocks = (rows + 255) / 256;
      p.nw = 8;
    }
  }
  if (p.rows64) p.nw = workgroups(tps) > cus ? 4 : 8;
  if (p.rows16 || p.rows64) p.wgs_per_cu = p.nw == (p.rows64 ? 4 : 8) ? 2 : 1;
  else p.wgs_per_cu = p.rows48 || (path == Path::kF32 && wgs_per_cu == 1) ? 1 : 2;
  // Splits index the grid's y dimension (at most kMaxGridY).
  tps = std::max<int64_t>(tps, round_tile((t_max + kMaxGridY - 1) / kMaxGridY));
  p.tps = (int)std::min<int64_t>(tps, INT32_MAX / 2);
  p.max_splits = t_max > 0 ? (int)((t_max + p.tps - 1) / p.tps) : 0;
  p.uniform_splits = true;
  for (int b = 0; b < batch; ++b) {
    const int N = std::min(host_n_nodes[b], n_max);
    if (N <= 0) continue;
    const int64_t T = (int64_t)host_ctx_len[b] + N;
    if ((T + p.tps - 1) / p.tps < p.max_splits) p.uniform_splits = false;
  }
  return p;
}

size_t plan_workspace(const Plan& p, int32_t batch, int32_t hq, int32_t d, int32_t n_max) {
  if (p.max_splits <= 1) return 0;
  const size_t parts = (size_t)batch * hq * n_max * p.max_splits;
  return align_up(parts * d * sizeof(float), 256) + align_up(parts * sizeof(float), 256);
}

// The kernel family of a call, from its types, sizes and alignment.
//  * bf16: addresses a sequence's K/V rows with 32-bit byte offsets and takes the
//    row maximum on raw scores, so scale > 0; operands that are not 16-byte
//    aligned are refused later on.
//  * fp32: any finite scale; operands that are not 16-byte aligned (o: 8 bytes
//    for a bf16 output) stay on the vector-ALU kernel, which takes them all.
Path choose_path(int32_t dtype, int32_t out_dtype, int32_t d, int32_t hkv, float scale,
                 uint32_t flags, int64_t t_max, const void* q, const void* k, const void* v,
                 const void* o) {
  if ((flags & CURE_ATTN_FORCE_VALU) || !std::isfinite(scale)) return Path::kValu;
  if (dtype == CURE_BF16) {
    const bool reach = (t_max + kTile) * hkv * d * 2 < (int64_t(1) << 31);
    return scale > 0.f && reach ? Path::kBf16 : Path::kValu;
  }
  const uintptr_t in = reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(k) |
                       reinterpret_cast<uintptr_t>(v);
  const uintptr_t out = reinterpret_cast<uintptr_t>(o) % (out_dtype == CURE_BF16 ? 8 : 16);
  return in % 16 == 0 && out == 0 ? Path::kF32 : Path::kValu;
}

}  // namespace
}  // namespace cure

using namespace cure;

extern "C" size_t cure_tree_attn_workspace_size(int32_t batch, int32_t hq, int32_t hkv,
                                                int32_t d, int32_t n_max,
                                                const int32_t* host_ctx_len,
                                                const int32_t* host_n_nodes,
                                                int32_t kv_split) {
  if (batch <= 0 || hq <= 0 || hkv <= 0 || hq % hkv || n_max <= 0 || !host_ctx_len ||
      !host_n_nodes)
    return 0;
  // The kernel families' plans may differ in row blocking; report the largest need.
  size_t need = 0;
  for (const Path path : {Path::kValu, Path::kF32, Path::kBf16}) {
    const Plan p = make_plan(batch, hq, hkv, d, n_max, host_ctx_len, host_n_nodes, kv_split, path);
    need = std::max(need, plan_workspace(p, batch, hq, d, n_max));
  }
  return need;
}

extern "C" cure_status cure_tree_attn(const void* q, const void* k, const void* v, void* o,
                                      float* lse, int32_t dtype, int32_t out_dtype,
                                      int32_t batch, int32_t hq, int32_t hkv, int32_t d,
                                      float scale, const int64_t* kv_off,
                                      const int32_t* ctx_len, const int32_t* n_nodes,
                                      const int32_t* parent, int32_t n_max,
                                      const int32_t* host_ctx_len,
                                      const int32_t* host_n_nodes, int32_t kv_split,
                                      uint32_t flags, int32_t* tree_status, void* workspace,
                                      size_t workspace_bytes, void* stream) {
  if (dtype != CURE_F32 && dtype != CURE_BF16) return CURE_ERR_INVALID_ARG;
  if (out_dtype != CURE_F32 && out_dtype != CURE_BF16) return CURE_ERR_INVALID_ARG;
  if (batch < 0 || hq <= 0 || hkv <= 0 || n_max < 0 || kv_split < 0) return CURE_ERR_INVALID_ARG;
  if (hq % hkv != 0) return CURE_ERR_INVALID_ARG;
  if (d != 64 && d != 128) return CURE_ERR_UNSUPPORTED;
  if (n_max > CURE_MAX_TREE_NODES) return CURE_ERR_UNSUPPORTED;
  if (batch == 0) return CURE_OK;
  if (n_max == 0) {                     // no sequence can have nodes
    if (tree_status) {
      hipLaunchKernelGGL(tree_status_ok, dim3((unsigned)((batch + 255) / 256)), dim3(256), 0,
                         as_stream(stream), tree_status, batch);
      return launch_status();
    }
    return CURE_OK;
  }
  if (!q || !k || !v || !o || !kv_off || !ctx_len || !n_nodes || !parent || !host_ctx_len ||
      !host_n_nodes)
    return CURE_ERR_INVALID_ARG;
  for (int b = 0; b < batch; ++b)
    if (host_ctx_len[b] < 0 || host_n_nodes[b] < 0 || host_n_nodes[b] > n_max)
      return CURE_ERR_INVALID_ARG;
  int64_t t_max = 0;
  for (int b = 0; b < batch; ++b)
    t_max = std::max<int64_t>(t_max, (int64_t)host_ctx_len[b] + host_n_nodes[b]);
  const Path path = choose_path(dtype, out_dtype, d, hkv, scale, flags, t_max, q, k, v, o);
  const bool mfma = path == Path::kBf16;
  const Plan p = make_plan(batch, hq, hkv, d, n_max, host_ctx_len, host_n_nodes, kv_split, path);
  if (p.max_splits == 0) {              // no sequence has tree nodes
    if (tree_status) {
      hipLaunchKernelGGL(tree_status_ok, dim3((unsigned)((batch + 255) / 256)), dim3(256), 0,
                         as_stream(stream), tree_status, batch);
      return launch_status();
    }
    return CURE_OK;
  }
  const size_t need = plan_workspace(p, batch, hq, d, n_max);
  if (need > 0 && (!workspace || workspace_bytes < need)) return CURE_ERR_WORKSPACE;
  if ((size_t)p.row_blocks * hkv > 65535 || batch > 65535) return CURE_ERR_UNSUPPORTED;

  CompactArgs a{};                      // its Args part serves full launches
  a.q = q;
  a.k = k;
  a.v = v;
  a.o = o;
  a.lse = lse;
  a.out_bf16 = out_dtype == CURE_BF16;
  a.hq = hq;
  a.hkv = hkv;
  a.group = hq / hkv;
  a.n_max = n_max;
  a.scale_log2 = scale * kLog2e;
  a.kv_off = kv_off;
  a.ctx_len = ctx_len;
  a.n_nodes = n_nodes;
  a.parent = parent;
  a.tps = p.tps;
  a.max_splits = p.max_splits;
  a.rows_per_wg = p.rows_per_wg;
  a.tree_status = tree_status;
  if (need > 0) {
    const size_t parts = (size_t)batch * hq * n_max * p.max_splits;
    a.part_o = reinterpret_cast<float*>(workspace);
    a.part_lse = reinterpret_cast<float*>(reinterpret_cast<char*>(workspace) +
                                          align_up(parts * d * sizeof(float), 256));
  }
  if (mfma) {
    // The MFMA kernel reads q, k and v as 16-byte vectors.
    const uintptr_t mis = reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(k) |
                          reinterpret_cast<uintptr_t>(v);
    if (mis % 16 != 0) return CURE_ERR_INVALID_ARG;
    if (a.out_bf16 ? reinterpret_cast<uintptr_t>(o) % 8 : reinterpret_cast<uintptr_t>(o) % 16)
      return CURE_ERR_INVALID_ARG;
  }
  // Split partials are written and read as 16-byte vectors.
  if (need > 0 && reinterpret_cast<uintptr_t>(workspace) % 16 != 0) return CURE_ERR_INVALID_ARG;

  hipStream_t st = as_stream(stream);
  // KV heads (and row blocks) vary fastest: consecutive workgroups, which the
  // dispatcher spreads over the XCDs and starts together, read the heads of
  // the same token range, so concurrent reads cover whole cache rows.
  dim3 grid(hkv * p.row_blocks, p.max_splits, batch);
  // A ragged batch of up to 64 sequences may be launched compactly (locate()), where
  // workgroups without work would delay others or put two on one CU beside an idle one.
  // They do neither when the CUs hold the full grid one each, nor when they hold it all at
  // once and have to take two each anyway, and two small ones on a CU (few rows, shortest
  // splits) cost little; the compact form's look-ups then cost 0.3 - 0.7 us, and with two
  // each it starts less evenly. Full and compact, us a call: 2 sequences of 2k - 3k tokens,
  // 6 nodes, head dim 64, 9.0 and 9.4; 4 of 0.9k - 1.8k, 100 nodes, 29.3 and 32.3; 8 of
  // 0.4k - 2.8k, 16 nodes, 32 rows a block, 11.7 and 12.4; but 3 of 1k - 2.6k, 32 nodes,
  // head dim 128, 21.3 and 19.4, 5 of 1k - 6.9k, 6 nodes, 16 heads in long splits, 39.8 and
  // 34.3, and fp32, 8 of 0.4k - 2.8k, 16 nodes, 32.0 and 23.5.
  // A launch that is being captured may be replayed when other sequences are the long
  // ones, so there every sequence may take max_splits, and the splits that the host's sizes
  // leave empty are listed behind the others. Replays of 16 sequences captured at 1k -
  // 4k tokens, 48 nodes, with these lengths, these permuted, random ones: 67, 76 and 83
  // us; with the splits in use alone 64, 92 and 93, as a full grid 77, 75 and 83 (8 of
  // 2k - 8k, 80 nodes: 84, 136, 121; 83, 187, 185; 114, 121, 124).
  bool compact = path != Path::kValu && !p.uniform_splits && batch <= 64;
  if (compact) {
    int used[64];
    int64_t units = 0;
    for (int b = 0; b < batch; ++b) {
      const int N = std::min(host_n_nodes[b], n_max);
      const int64_t T = (int64_t)host_ctx_len[b] + N;
      // A sequence without nodes has one unit, which reports its status.
      used[b] = N > 0 ? (int)((T + p.tps - 1) / p.tps) : 1;
      units += used[b];
    }
    const int64_t blocks = (int64_t)hkv * p.row_blocks, wgs = units * blocks, all = blocks * p.max_splits * batch;
    const int64_t cus = device_cu_count();
    const bool small = path == Path::kBf16 && p.rows_per_wg <= 64 && p.tps <= kMinTps;
    compact = all > (small ? p.wgs_per_cu : 1) * cus && (wgs <= cus || all > p.wgs_per_cu * cus);
    const bool captured = compact && is_capturing(st);
    if (captured) units = (int64_t)p.max_splits * batch;
    // The runtime takes fewer than 2^32 threads in a grid dimension.
    compact = compact && units <= kMaxUnits && units * blocks * 64 * p.nw < (int64_t(1) << 32);
    if (compact) {
      int u = 0;
      const auto list = [&](int b, int i) {
        a.unit[u >> 1] |= (uint32_t)(b | i << 6) << (16 * (u & 1));
        ++u;
      };
      for (int b = 0; b < batch; ++b) {
        for (int i = 0; i < used[b]; ++i) list(b, i);
        a.seq_splits[b] = captured ? p.max_splits : used[b];
      }
      for (int b = 0; b < batch && captured; ++b)
        for (int i = used[b]; i < p.max_splits; ++i) list(b, i);
      a.row_blocks = p.row_blocks;
      grid = dim3((unsigned)(units * blocks));
    }
  }
  const Args& full = a;
#define CURE_ATTN(threads, kernel, ...)                                                                    \
  do {                                                                                                     \
    if (compact) hipLaunchKernelGGL((kernel<__VA_ARGS__, CompactArgs>), grid, dim3(threads), 0, st, a);    \
    else hipLaunchKernelGGL((kernel<__VA_ARGS__, Args>), grid, dim3(threads), 0, st, full);                \
  } while (0)
  if (p.rows48) {
    CURE_ATTN(64 * kRg3Waves, tree_attn_rg, 128, kRg3Waves, 3, 2, 4, 2, 2);
  } else if (p.rows16) {
    if (d == 128 && p.nw == 8) CURE_ATTN(512, tree_attn_m16, 128, 8);
    else if (d == 128) CURE_ATTN(1024, tree_attn_m16, 128, 16);
    else CURE_ATTN(512, tree_attn_m16, 64, 8);
  } else if (p.rows32) {
    CURE_ATTN(512, tree_attn_mfma, 64, 8, kStages);
  } else if (p.rows64) {
    if (p.nw == 4) CURE_ATTN(256, tree_attn_rg, 64, 4, 3, 2, 4, 1, 2);
    else CURE_ATTN(512, tree_attn_rg, 64, 8, 2, 2, 8, 1, 3);
  } else if (path == Path::kF32) {
    if (d == 128 && p.rows_per_wg == 16) CURE_ATTN(256, tree_attn_f32, 128, 4);
    else if (d == 128) CURE_ATTN(256, tree_attn_f32, 128, 2);
    else if (p.rows_per_wg == 16) CURE_ATTN(256, tree_attn_f32, 64, 4);
    else CURE_ATTN(256, tree_attn_f32, 64, 2);
  } else if (dtype == CURE_BF16) {
    if (d == 128) hipLaunchKernelGGL((tree_attn_valu<uint16_t, 128>), grid, dim3(256), 0, st, full);
    else hipLaunchKernelGGL((tree_attn_valu<uint16_t, 64>), grid, dim3(256), 0, st, full);
  } else {
    if (d == 128) hipLaunchKernelGGL((tree_attn_valu<float, 128>), grid, dim3(256), 0, st, full);
    else hipLaunchKernelGGL((tree_attn_valu<float, 64>), grid, dim3(256), 0, st, full);
  }
#undef CURE_ATTN
  if (hipGetLastError() != hipSuccess) return CURE_ERR_HIP;
  if (p.max_splits > 1 && p.max_splits <= kFewSplits && (int64_t)batch * n_max * hq >= kManyRows) {
    const int rows = 1024 / d;                          // output rows per workgroup
    const dim3 mgrid((unsigned)((hq + rows - 1) / rows), (unsigned)n_max, (unsigned)batch);
#define CURE_MERGE(DD, NN)                                                                                \
    do {                                                                                                  \
      if (compact) hipLaunchKernelGGL((attn_merge_few<DD, NN, CompactArgs>), mgrid, dim3(256), 0, st, a); \
      else hipLaunchKernelGGL((attn_merge_few<DD, NN, Args>), mgrid, dim3(256), 0, st, full);             \
    } while (0)
    if (d == 128 && p.max_splits == 2) CURE_MERGE(128, 2);
    else if (d == 128) CURE_MERGE(128, kFewSplits);
    else if (p.max_splits == 2) CURE_MERGE(64, 2);
    else CURE_MERGE(64, kFewSplits);
#undef CURE_MERGE
  } else if (p.max_splits > 1) {
    const dim3 mgrid((unsigned)((hq + 3) / 4), (unsigned)n_max, (unsigned)batch);
    const int per_load = 256 / d;                       // splits per merge load
    const int nb = p.max_splits <= 2 * per_load ? 2 : p.max_splits <= 4 * per_load ? 4 : 8;
    const bool own = !p.uniform_splits;
#define CURE_MERGE(DD, NN)                                                                                   \
    do {                                                                                                     \
      if (compact) hipLaunchKernelGGL((attn_merge<DD, NN, true, CompactArgs>), mgrid, dim3(256), 0, st, a);  \
      else if (own) hipLaunchKernelGGL((attn_merge<DD, NN, true, Args>), mgrid, dim3(256), 0, st, full);     \
      else hipLaunchKernelGGL((attn_merge<DD, NN, false, Args>), mgrid, dim3(256), 0, st, full);             \
    } while (0)
    if (d == 128) {
      if (nb == 2) CURE_MERGE(128, 2);
      else if (nb == 4) CURE_MERGE(128, 4);
      else CURE_MERGE(128, 8);
    } else {
      if (nb == 2) CURE_MERGE(64, 2);
      else if (nb == 4) CURE_MERGE(64, 4);
      else CURE_MERGE(64, 8);
    }
#undef CURE_MERGE
  }
  return launch_status();
}
