// Block-sparse attention with un-permutation (Eq. (2), Sec. 3.1).
//
// For query block u the key stream is the concatenation of the rows of its
// selected key blocks (ascending block id); the softmax of each query is
// taken over that stream (renormalised), flash-attention style with an
// online maximum, and row i of Q' is written to O[q_perm[i]].  Only the
// last 32-key tile of a stream is partial, whatever the block sizes.
#include <math.h>

#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace park {

constexpr int AT_MAXC = 2048;

// exclusive prefix of the selected block sizes into cum[0..n] and the first
// row of each selected block into kst[0..n), NT threads (ids outside
// [0, nblk) count as empty)
template <int NT>
__device__ void prefix_sizes(const int* __restrict__ sel, int n, int nblk,
                             const int* __restrict__ koff, int* cum, int* kst, int* tmp) {
  constexpr int PT = AT_MAXC / NT;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  int x[PT];
  int s = 0;
#pragma unroll
  for (int k = 0; k < PT; ++k) {
    const int i = tid * PT + k;
    x[k] = 0;
    if (i < n) {
      const int v = sel[i];
      int start = -1;
      if ((unsigned)v < (unsigned)nblk) {
        start = koff[v];
        x[k] = max(0, koff[v + 1] - start);
      }
      kst[i] = start;
    }
    s += x[k];
  }
  int inc = s;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(inc, o, 64);
    if (lane >= o) inc += y;
  }
  if (lane == 63) tmp[wid] = inc;
  __syncthreads();
  int pre = 0;
  for (int w = 0; w < wid; ++w) pre += tmp[w];
  int run = pre + inc - s;
#pragma unroll
  for (int k = 0; k < PT; ++k) {
    const int i = tid * PT + k;
    if (i < n) cum[i] = run;
    run += x[k];
    if (i == n - 1) cum[n] = run;
  }
  if (n == 0 && tid == 0) cum[0] = 0;
  __syncthreads();
}

// row of stream position p: binary search of the last m with cum[m] <= p
// (LDS only; -1 past the end of the stream)
__device__ __forceinline__ int stream_row(int p, const int* cum, const int* kst, int n) {
  if (p >= cum[n]) return -1;
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (cum[mid] <= p) lo = mid;
    else hi = mid - 1;
  }
  return kst[lo] < 0 ? -1 : kst[lo] + (p - cum[lo]);
}

typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

// maximum of v over lanes l and l ^ 32 (a cross-half lane swap, no LDS traffic)
__device__ __forceinline__ float max_xor32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(v, fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
// two floats to bf16 (round to nearest even, v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{a, b}, bf16x2_t));
}

template <typename OT>
__device__ __forceinline__ void store_out2(OT* p, float a, float b);
template <>
__device__ __forceinline__ void store_out2<float>(float* p, float a, float b) {
  *(float2*)p = make_float2(a, b);
}
template <>
__device__ __forceinline__ void store_out2<bf16_t>(bf16_t* p, float a, float b) {
  *(uint32_t*)p = pack_bf(a, b);
}

// fp32 inputs: both contractions on v_mfma_f32_32x32x2_f32 (fp32 products and
// sums), a workgroup per 32 rows of a query block.
//
// What bounds it: a small float32 layer has few query blocks (64 at 1 x 4096
// tokens), so the chip is idle unless the key stream of one block is split as
// well: the eight wavefronts of a workgroup take the stream's 32-key tiles in
// turn, each with its own online softmax, and their partial results are added
// in wavefront order at the end.  Operands go straight from global memory to
// registers (no LDS, no barrier in the tile loop): with
// S^T = K Q^T in C layout a lane holds the scores of query l % 32 and keys
// 8 b + 4 (l / 32) + r, which is the B operand of O^T += V^T P^T when step
// (b, r) of the product takes those two keys, so the probabilities stay where
// they are.  The previous kernel (one workgroup per query block, dot products
// and P V on the vector ALU through LDS) took 2314 us at 1 x 4096 tokens,
// d = 64, top 25%; this one 86 us (1.07 GFLOP: 0.5 -> 12 TFLOP/s).
template <typename OT, int D>
__global__ __launch_bounds__(512, 2) void k_attn_f32(
    const float* __restrict__ Qp, const float* __restrict__ Kp, const float* __restrict__ Vp,
    const int* __restrict__ q_offsets, const int* __restrict__ k_offsets,
    const int* __restrict__ kv_count, const int* __restrict__ kv_index,
    const int* __restrict__ q_perm, int N, int CQ, int CK, float scale, float scale_log2,
    OT* __restrict__ O, float* __restrict__ lse) {
  constexpr int NW = 8, RT = 32, KT = 32, DB = D / 32, PS = 36;
  constexpr bool PRE = D == 64;  // next tile's keys loaded during P V (registers allow it)
  __shared__ int cum[AT_MAXC + 1];
  __shared__ int kst[AT_MAXC];
  __shared__ int tmp[NW];
  __shared__ float ml[2][NW][RT];     // running maximum and sum of each wavefront's share
  __shared__ float part[NW][RT][PS];  // 32 dimensions of each wavefront's O (4 pad columns)
  const int u = blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
  const int* qo = q_offsets + (size_t)h * (CQ + 1);
  const int q0 = min(max(qo[u], 0), N), q1 = min(max(qo[u + 1], q0), N);
  if (q0 + RT * (int)blockIdx.z >= q1) return;
  const size_t row = (size_t)h * CQ + u;
  const int nsel = min(max(kv_count[row], 0), CK);
  prefix_sizes<64 * NW>(kv_index + row * CK, nsel, CK, k_offsets + (size_t)h * (CK + 1), cum, kst,
                        tmp);
  const int nk = cum[nsel];
  const float* Qh = Qp + (size_t)h * N * D;
  const float* Kh = Kp + (size_t)h * N * D;
  const float* Vh = Vp + (size_t)h * N * D;
  const int w = tid >> 6, l = tid & 63, hf = l >> 5, c32 = l & 31;
  const int ntiles = (nk + KT - 1) / KT;
  for (int r0 = q0 + RT * (int)blockIdx.z; r0 < q1; r0 += RT * (int)gridDim.z) {
    const int nr = min(RT, q1 - r0);
    // operand k-index: step 4 j + e of the score product takes dimensions
    // 8 j + e (lanes 0..31) and 8 j + 4 + e (lanes 32..63) of both operands
    float4 qf[D / 8];
#pragma unroll
    for (int j = 0; j < D / 8; ++j)
      qf[j] = c32 < nr ? *(const float4*)(Qh + (size_t)(r0 + c32) * D + 8 * j + 4 * hf)
                       : make_float4(0.f, 0.f, 0.f, 0.f);
    float m = -INFINITY, lsum = 0.0f;
    f32x16_t acc[DB];
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[b][q] = 0.0f;
    float4 kf[D / 8];
    int src = 0;
    auto load_k = [&](int t) {
      src = min(max(stream_row(t * KT + c32, cum, kst, nsel), 0), N - 1);
#pragma unroll
      for (int j = 0; j < D / 8; ++j)
        kf[j] = *(const float4*)(Kh + (size_t)src * D + 8 * j + 4 * hf);
    };
    if (PRE && w < ntiles) load_k(w);
    for (int t = w; t < ntiles; t += NW) {
      if (!PRE) load_k(t);
      // V row of key 8 b + 4 hf + r, dimension 32 db + c32
      float vf[16][DB];
      auto load_v = [&](int b) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int s = __shfl(src, 8 * b + 4 * hf + r, 64);
#pragma unroll
          for (int db = 0; db < DB; ++db) vf[4 * b + r][db] = Vh[(size_t)s * D + 32 * db + c32];
        }
      };
      const int left = nk - t * KT;  // keys of the tile; those past the stream's end count for nothing
      auto key_in = [&](int q) { return 8 * (q >> 2) + 4 * hf + (q & 3) < left; };
      if (PRE) {
#pragma unroll
        for (int b = 0; b < 4; ++b) load_v(b);
      }
      f32x16_t st;
#pragma unroll
      for (int q = 0; q < 16; ++q) st[q] = 0.0f;
#pragma unroll
      for (int j = 0; j < D / 8; ++j) {
        st = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j].x, qf[j].x, st, 0, 0, 0);
        st = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j].y, qf[j].y, st, 0, 0, 0);
        st = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j].z, qf[j].z, st, 0, 0, 0);
        st = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j].w, qf[j].w, st, 0, 0, 0);
      }
      if (PRE && t + NW < ntiles) load_k(t + NW);
      if (left < KT) {
#pragma unroll
        for (int q = 0; q < 16; ++q) st[q] = key_in(q) ? st[q] : -INFINITY;
      }
      float tmax = st[0];
#pragma unroll
      for (int q = 1; q < 16; ++q) tmax = fmaxf(tmax, st[q]);
      const float mnew = fmaxf(m, max_xor32(tmax));
      const float alpha = mnew == m ? 1.0f : __builtin_amdgcn_exp2f((m - mnew) * scale_log2);
      const float mref = mnew == -INFINITY ? 0.0f : mnew;
      m = mnew;
      lsum *= alpha;
#pragma unroll
      for (int b = 0; b < DB; ++b) acc[b] *= alpha;
      // the difference to the maximum is taken before the scaling, so that the
      // exponent's rounding is relative to that difference
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        st[q] = __builtin_amdgcn_exp2f((st[q] - mref) * scale_log2);
        lsum += st[q];
      }
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        if (!PRE) load_v(b);
        if (left < KT) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int db = 0; db < DB; ++db) vf[4 * b + r][db] = key_in(4 * b + r) ? vf[4 * b + r][db] : 0.0f;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int db = 0; db < DB; ++db)
            acc[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[4 * b + r][db], st[4 * b + r],
                                                           acc[db], 0, 0, 0);
      }
    }
    lsum += __shfl_xor(lsum, 32, 64);
    if (hf == 0) {
      ml[0][w][c32] = m;
      ml[1][w][c32] = lsum;
    }
    __syncthreads();
    // the eight shares of a row: common maximum, this wavefront's factor
    {
      float mall = ml[0][0][c32];
#pragma unroll
      for (int i = 1; i < NW; ++i) mall = fmaxf(mall, ml[0][i][c32]);
      const float fac = m == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((m - mall) * scale_log2);
#pragma unroll
      for (int b = 0; b < DB; ++b) acc[b] *= fac;
    }
    // output row qr and two dimensions of each 32 per thread
    const int qr = tid >> 4, dc = 2 * (tid & 15);
    float mall = ml[0][0][qr], lall = 0.0f;
#pragma unroll
    for (int i = 1; i < NW; ++i) mall = fmaxf(mall, ml[0][i][qr]);
#pragma unroll
    for (int i = 0; i < NW; ++i)
      if (ml[0][i][qr] != -INFINITY)
        lall += ml[1][i][qr] * __builtin_amdgcn_exp2f((ml[0][i][qr] - mall) * scale_log2);
    const float inv = lall > 0.0f ? 1.0f / lall : 0.0f;
    const int dst = qr < nr ? q_perm[(size_t)h * N + r0 + qr] : -1;
    const bool ok = (unsigned)dst < (unsigned)N;
    // natural-log normaliser of the row: mall is its largest raw score
    if (lse && ok && dc == 0)
      lse[(size_t)h * N + dst] = lall > 0.0f ? mall * scale + logf(lall) : -INFINITY;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
#pragma unroll
      for (int b = 0; b < 4; ++b)
        *(float4*)&part[w][c32][8 * b + 4 * hf] = make_float4(
            acc[db][4 * b], acc[db][4 * b + 1], acc[db][4 * b + 2], acc[db][4 * b + 3]);
      __syncthreads();
      float a = 0.0f, c = 0.0f;
#pragma unroll
      for (int i = 0; i < NW; ++i) {
        const float2 y = *(const float2*)&part[i][qr][dc];
        a += y.x;
        c += y.y;
      }
      if (ok) store_out2<OT>(O + ((size_t)h * N + dst) * D + 32 * db + dc, a * inv, c * inv);
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------------------
// bf16 MFMA path: operand and accumulator vector types, output stores.
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;
typedef const __attribute__((address_space(3))) bf16x8_t lds_bf16x8_t;
typedef const __attribute__((address_space(3))) f32x4_t lds_f32x4_t;

template <typename OT>
__device__ __forceinline__ void store_out4(OT* p, float a, float b, float c, float d);
template <>
__device__ __forceinline__ void store_out4<float>(float* p, float a, float b, float c, float d) {
  *(float4*)p = make_float4(a, b, c, d);
}
template <>
__device__ __forceinline__ void store_out4<bf16_t>(bf16_t* p, float a, float b, float c, float d) {
  *(uint2*)p = make_uint2(pack_bf(a, b), pack_bf(c, d));
}

// MinHash of a selected key-block set: min over the selected ids of a fixed
// integer hash (an avalanche mixer), used to order query blocks so that blocks
// selecting nearly the same key blocks are neighbours.
__device__ __forceinline__ uint32_t attn_hash(uint32_t v) {
  v ^= v >> 16;
  v *= 0x7feb352du;
  v ^= v >> 15;
  v *= 0x846ca68bu;
  v ^= v >> 16;
  return v;
}

// XOR swizzle of the 16-byte chunk index within a K row (an involution): the
// 16 rows one S^T MFMA reads land in 16 different bank groups.
template <int D>
__device__ __forceinline__ int swz_k(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }

// One wave-wide LDS DMA: lane l's 16 bytes at base + off land at LDS byte
// address lds + 16 l (base and lds wave-uniform).  Written as inline assembly
// so that the compiler does not treat the transfer as a pending LDS store: it
// would otherwise wait for every DMA in flight before each LDS read.
// Completion is tracked explicitly with wait_vmcnt() and a barrier.
__device__ __forceinline__ void lds_dma16(const void* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base),
               "s"(lds)
               : "memory", "m0");
}

__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(size_t)(const __attribute__((address_space(3))) void*)p;
}

// waits until at most N vector-memory operations of this wavefront are outstanding
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// ------------------------------------------------------------------------
// Grouped block-sparse attention.
//
// Query blocks that select nearly the same key blocks share one key/value
// stream: the plan orders the query blocks of a head by two MinHash values of
// their selected key-block sets and cuts the concatenated rows into groups of
// at most ATTN_R rows and ATTN_LB query blocks.  A workgroup streams the
// union of its blocks' selections once (ascending key-block id) and each row
// keeps only the keys of the key blocks its own query block selected, so the
// result per row is the same renormalised softmax over its own selection.
//
// What bounds it and why it is built this way (measured with timing-only
// copies at 24 x 119056 tokens, d = 128, top 10%, 24.3 TFLOP issued):
//  * A 32 x 32 tile of a wavefront is 17 MFMAs (257 ns at the 2.1 GHz the chip
//    holds under them) and about 90 vector operations with 16 exponentials
//    (160 ns); on one SIMD the two overlap only in part, so the compute alone
//    takes 18 ms, 21.7 ms with its LDS reads.  A single wavefront per SIMD
//    issues vector operations at half rate: two wavefronts of 64 rows instead
//    of four of 32 save a third of the LDS reads but take 31.6 ms.
//  * So every LDS read is issued half a step before its use, vector work sits
//    between the MFMAs, and what else a step did is taken out of it: the
//    stream rows come from a table (the cursors they replace were a divergent
//    loop of dependent LDS reads in every step), the selection bias from one
//    more MFMA (bias rows x one-hot block) instead of 16 LDS floats per lane.
//    30.5 -> 27.3 ms.
//  * d = 64 runs three wavefronts per SIMD (168 registers, 48 KB of LDS per
//    workgroup): 1730 -> 1290 us at 16 x 32227 tokens, top 15%.  d = 128 needs
//    80 KB for its rings, two workgroups per CU.
//  * Short streams (40 x 75600 tokens, top-p 0.9: 24 tiles per group) are bound
//    by the chain of loads before the first tile: selections from the plan's
//    bit rows (one load per block, no LDS atomics), Q and the output row loaded
//    beside them, and one table segment expanded before the first tile:
//    1970 -> 1670 us.

// neighbouring groups that run on one XCD at a time; 4 loses nowhere much (1, 2,
// 4, 8: 1806, 1786, 1723, 1778 us at 40 x 75600, top-p; 28.6, 29.0, 28.7, 28.9 ms
// at 24 x 119056; 9.69, 9.82, 9.71, 9.92 at 8 x 119056; 1386, 1375, 1353, 1371 us
// at 16 x 32227, d = 64; 491, 503, 509, 503 at 8 x 16384; equal at 40 x 75600 in
// blocks of 128 and 3 x 6000)
constexpr int ATTN_BUN = 4;
constexpr int ATTN_R = 128;  // rows per group (32 per wavefront)
constexpr int ATTN_KSLOTS = 3;  // K tiles in LDS (V: one more)
constexpr int ATTN_UCAP = 1024;  // key blocks of the union per stream chunk
constexpr int ATTN_LB = 16;          // query blocks per group (bits of a selection word)
constexpr int ATTN_SEG = 512;        // stream positions expanded to rows at a time

static int attn_windows(int N) { return (N + ATTN_R - 1) / ATTN_R; }
// groups per head: every window of ATTN_R rows, split further when it holds
// more than ATTN_LB query blocks (a window boundary cuts at most one block)
int attn_groups_per_head(int N, int CQ) {
  const int W = attn_windows(N);
  return W + (CQ + W + ATTN_LB - 1) / ATTN_LB + 1;
}

// Selection families.  fam[h][u] = the smallest query block v (u itself
// included) whose selected key-block set overlaps u's with Jaccard index above
// 1/2 (3 |S_u & S_v| > |S_u| + |S_v|).  Blocks whose selections are nearly the
// same (on video latents: query clusters of the same content) then share one
// value, and sorting by fam[fam[u]] makes the blocks of a family neighbours in
// the group plan.
//
// k_attn_selbits: the selection of every (head, query block) as a 64-word bit
// row (CK <= 2048), one wavefront per row, fam = u, and the parts of the
// plan's sort key that come from the selection (MinHash values, key tiles).
__global__ __launch_bounds__(256) void k_attn_selbits(const int* __restrict__ kv_count,
                                                      const int* __restrict__ kv_index,
                                                      const int* __restrict__ q_offsets,
                                                      const int* __restrict__ k_offsets, int H,
                                                      int N, int CQ, int CK,
                                                      uint32_t* __restrict__ bits,
                                                      int* __restrict__ fam,
                                                      uint4* __restrict__ rkey) {
  __shared__ uint32_t rowb[4][64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const size_t row = (size_t)blockIdx.x * 4 + wid;
  const bool valid = row < (size_t)H * CQ;
  rowb[wid][lane] = 0u;
  __syncthreads();
  uint32_t m1 = 0xffffffffu, m2 = 0xffffffffu;
  int nkey = 0;
  if (valid) {
    const int h = (int)(row / (size_t)CQ);
    const int* koff = k_offsets + (size_t)h * (CK + 1);
    const int n = min(max(kv_count[row], 0), CK);
    const int* sel = kv_index + row * CK;
    for (int j = lane; j < n; j += 64) {
      const int v = sel[j];
      m1 = min(m1, attn_hash((uint32_t)v));
      m2 = min(m2, attn_hash((uint32_t)v + 7919u));
      if ((unsigned)v < (unsigned)CK) {
        atomicOr(&rowb[wid][v >> 5], 1u << (v & 31));
        nkey += max(0, koff[v + 1] - koff[v]);
      }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    m1 = min(m1, (uint32_t)__shfl_xor((int)m1, o, 64));
    m2 = min(m2, (uint32_t)__shfl_xor((int)m2, o, 64));
    nkey += __shfl_xor(nkey, o, 64);
  }
  __syncthreads();
  if (valid) {
    bits[row * 64 + lane] = rowb[wid][lane];
    if (lane == 0) {
      const int h = (int)(row / (size_t)CQ), u = (int)(row % (size_t)CQ);
      const int* qo = q_offsets + (size_t)h * (CQ + 1);
      const int a = min(max(qo[u], 0), N), b = min(max(qo[u + 1], a), N);
      fam[row] = u;
      // the plan's sort-key parts: the two MinHash values, the key tiles of
      // the block's own selection, whether the block has rows
      rkey[row] = make_uint4(m1, m2, (uint32_t)((nkey + 31) >> 5), b > a ? 1u : 0u);
    }
  }
}

// k_attn_family: workgroup = a pair of 64-block tiles (tu, tv <= tu) of a
// head; thread (r, kk) holds row u = 64 tu + r in registers and compares it
// with rows v = 64 tv + kk + 4 j < u (LDS); the smallest qualifying v goes to
// fam[u] by atomicMin (order-independent).
__global__ __launch_bounds__(256) void k_attn_family(const int* __restrict__ kv_count,
                                                     const uint32_t* __restrict__ bits, int CQ,
                                                     int CK, int* __restrict__ fam) {
  __shared__ uint4 vb[64][17];  // 64 bit rows of the v tile (+1 chunk: conflict-free)
  __shared__ int vcnt[64];
  const int h = blockIdx.y, p = (int)blockIdx.x, tid = threadIdx.x;
  int tu = (int)((sqrtf(8.0f * (float)p + 1.0f) - 1.0f) * 0.5f);
  while ((tu + 1) * (tu + 2) / 2 <= p) ++tu;
  while (tu * (tu + 1) / 2 > p) --tu;
  const int tv = p - tu * (tu + 1) / 2;
  const int W4 = ((CK + 31) / 32 + 3) / 4;  // 16-byte chunks holding the selection bits
  const uint4* bh = (const uint4*)(bits + (size_t)h * CQ * 64);
  for (int e = tid; e < 64 * 16; e += 256) {
    const int k = e >> 4, c = e & 15, v = tv * 64 + k;
    vb[k][c] = v < CQ ? bh[(size_t)v * 16 + c] : make_uint4(0u, 0u, 0u, 0u);
  }
  if (tid < 64) {
    const int v = tv * 64 + tid;
    vcnt[tid] = v < CQ ? min(max(kv_count[(size_t)h * CQ + v], 0), CK) : 0;
  }
  const int r = tid & 63, kk = tid >> 6, u = tu * 64 + r;
  uint4 ur[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) ur[c] = u < CQ ? bh[(size_t)u * 16 + c] : make_uint4(0u, 0u, 0u, 0u);
  const int cu = u < CQ ? min(max(kv_count[(size_t)h * CQ + u], 0), CK) : 0;
  __syncthreads();
  if (u >= CQ || cu == 0) return;  // no barrier follows
  int cand = 0x7fffffff;
  for (int j = 0; j < 16; ++j) {
    const int k = kk + 4 * j, v = tv * 64 + k;
    if (v >= u) break;
    int inter = 0;
#pragma unroll
    for (int c = 0; c < 16; ++c)
      if (c < W4) {
        const uint4 y = vb[k][c];
        inter += __popc(ur[c].x & y.x) + __popc(ur[c].y & y.y) + __popc(ur[c].z & y.z) +
                 __popc(ur[c].w & y.w);
      }
    if (3 * inter > cu + vcnt[k]) {
      cand = v;
      break;
    }
  }
  if (cand != 0x7fffffff) atomicMin(&fam[(size_t)h * CQ + u], cand);
}

// Group plan of one head (1024 threads, CQ <= 2048):
//   order[h][i]  query block at sorted position i (-1 past the blocks with rows)
//   spre[h][i]   rows of the sorted blocks before position i (i <= CQ)
//   grp[h][g]    {first row, end row, first position, end position}: rows in
//                the coordinates of the sorted concatenation; {0,0,0,0} when
//                g is past the last group.
__global__ __launch_bounds__(1024) void k_attn_gplan(const int* __restrict__ q_offsets,
                                                     const uint4* __restrict__ rkey,
                                                     const int* __restrict__ fam, int N,
                                                     int CQ, int CK, int GPH,
                                                     int* __restrict__ order,
                                                     int* __restrict__ spre,
                                                     int4* __restrict__ grp) {
  __shared__ unsigned long long key[2048];
  __shared__ int pre[2049];
  __shared__ int tiles[2048];  // key tiles of each query block's own selection (by block id)
  __shared__ int tpos[2048];   // the same by sorted position
  __shared__ uint32_t gwk[2048];                        // window and part of each group
  __shared__ uint32_t bcost[2048 / ATTN_BUN + 1];       // key tiles of each bundle of groups
  __shared__ int wsum[16];
  const int h = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int* qo = q_offsets + (size_t)h * (CQ + 1);
  int SZ = 2;
  while (SZ < CQ) SZ <<= 1;
  // sort keys (selection family, top bits of the first MinHash, top bits of
  // the second, block id); blocks without rows sort last with the key ~0.
  // One thread per block.
  for (int u = tid; u < SZ; u += 1024) {
    unsigned long long kk = ~0ull;
    if (u < CQ) {
      // MinHash values and key tiles of the selection (k_attn_selbits)
      const uint4 rk = rkey[(size_t)h * CQ + u];
      tiles[u] = (int)rk.z;
      if (rk.w) {
        // family label: the partner of u's smallest partner (one pointer jump)
        const int* fh = fam + (size_t)h * CQ;
        int f = fh[u];
        f = (unsigned)f < (unsigned)CQ ? fh[f] : u;
        f = (unsigned)f < (unsigned)CQ ? f : u;
        kk = ((unsigned long long)f << 52) | ((unsigned long long)(rk.x >> 12) << 32) |
             (rk.y & 0xfffff800u) | (uint32_t)u;
      }
    }
    key[u] = kk;
  }
  __syncthreads();
  for (int len = 2; len <= SZ; len <<= 1)
    for (int j = len >> 1; j > 0; j >>= 1) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int i = tid + 1024 * k, ixj = i ^ j;
        if (i < SZ && ixj > i) {
          const unsigned long long x = key[i], y = key[ixj];
          const bool up = (i & len) == 0;
          if ((x > y) == up) {
            key[i] = y;
            key[ixj] = x;
          }
        }
      }
      __syncthreads();
    }
  // rows of the sorted blocks and their exclusive prefix
  int x[2], uu[2];
  int s = 0;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int pos = 2 * tid + k;
    uu[k] = -1;
    x[k] = 0;
    if (pos < CQ && key[pos] != ~0ull) {
      const int u = (int)(key[pos] & 0x7ffu);
      const int a = min(max(qo[u], 0), N), b = min(max(qo[u + 1], a), N);
      uu[k] = u;
      x[k] = b - a;
    }
    s += x[k];
  }
  int inc = s;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(inc, o, 64);
    if (lane >= o) inc += y;
  }
  if (lane == 63) wsum[wid] = inc;
  __syncthreads();
  int run = inc - s, total = 0;
  for (int i = 0; i < 16; ++i) {
    run += i < wid ? wsum[i] : 0;
    total += wsum[i];
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int pos = 2 * tid + k;
    if (pos < CQ) {
      pre[pos] = run;
      tpos[pos] = uu[k] >= 0 ? tiles[uu[k]] : 0;
      order[(size_t)h * CQ + pos] = uu[k];
      spre[(size_t)h * (CQ + 1) + pos] = run;
    }
    run += x[k];
  }
  if (tid == 0) {
    pre[CQ] = total;
    spre[(size_t)h * (CQ + 1) + CQ] = total;
  }
  __syncthreads();
  // windows of ATTN_R rows; a window with more than ATTN_LB blocks is split
  // into runs of ATTN_LB blocks.  With at most 2048 groups they are ordered by
  // bundles of ATTN_BUN neighbours, longest bundle first (summed key tiles of
  // their query blocks), so that the longest ones start first, and the groups
  // of a bundle go to one XCD (workgroup i runs on XCD i % 8): neighbours are
  // of one family and stream nearly the same keys and values at the same time,
  // which that XCD's L2 then fetches once.
  int4* gh = grp + (size_t)h * GPH;
  const int W = (total + ATTN_R - 1) / ATTN_R;
  const bool lpt = GPH <= 2048 && W < (1 << 23);
  // blocks of window wdw: sorted positions [i0, i1)
  auto window = [&](int wdw, int& i0, int& i1) {
    const int ra = wdw * ATTN_R, rb = min(ra + ATTN_R, total);
    int lo = 0, hi = CQ;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (pre[mid + 1] > ra) hi = mid;
      else lo = mid + 1;
    }
    i0 = lo;
    hi = CQ;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (pre[mid] >= rb) hi = mid;
      else lo = mid + 1;
    }
    i1 = lo;
  };
  for (int g = tid; g < 2048 / ATTN_BUN + 1; g += 1024) bcost[g] = 0u;
  __syncthreads();
  auto desc = [&](int wdw, int k, int i0, int i1) {
    const int ra = wdw * ATTN_R, rb = min(ra + ATTN_R, total);
    const int ib = i0 + k * ATTN_LB, ie = min(ib + ATTN_LB, i1);
    return make_int4(max(ra, pre[ib]), min(rb, pre[ie]), ib, ie);
  };
  int gbase = 0;
  for (int w0 = 0; w0 < W; w0 += 1024) {
    const int wdw = w0 + tid;
    int i0 = 0, i1 = 0, nsub = 0;
    if (wdw < W) {
      window(wdw, i0, i1);
      nsub = (i1 - i0 + ATTN_LB - 1) / ATTN_LB;
    }
    int sinc = nsub;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(sinc, o, 64);
      if (lane >= o) sinc += y;
    }
    __syncthreads();
    if (lane == 63) wsum[wid] = sinc;
    __syncthreads();
    int g = gbase + sinc - nsub, ctot = 0;
    for (int i = 0; i < 16; ++i) {
      g += i < wid ? wsum[i] : 0;
      ctot += wsum[i];
    }
    for (int k = 0; k < nsub; ++k, ++g) {
      if (g >= GPH) continue;
      const int4 gd = desc(wdw, k, i0, i1);
      if (lpt) {
        uint32_t c = 0;
        for (int i = gd.z; i < gd.w; ++i) c += (uint32_t)tpos[i];
        gwk[g] = ((uint32_t)wdw << 8) | (uint32_t)k;
        atomicAdd(&bcost[g / ATTN_BUN], c);
      } else {
        gh[g] = gd;
      }
    }
    gbase += ctot;
  }
  if (lpt) {
    const int G = min(gbase, GPH);
    int SG = 2;
    while (SG < G) SG <<= 1;
    __syncthreads();
    // (a last bundle of fewer groups stays last: the others keep their alignment)
    for (int g = tid; g < SG; g += 1024) {
      const bool whole = g / ATTN_BUN * ATTN_BUN + ATTN_BUN <= G;
      key[g] = g >= G ? ~0ull
                      : ((unsigned long long)(0xfffffffeu - (whole ? bcost[g / ATTN_BUN] : 0u)) << 32) |
                            (uint32_t)g;
    }
    __syncthreads();
    for (int len = 2; len <= SG; len <<= 1)
      for (int j = len >> 1; j > 0; j >>= 1) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int i = tid + 1024 * k, ixj = i ^ j;
          if (i < SG && ixj > i) {
            const unsigned long long x = key[i], y = key[ixj];
            const bool up = (i & len) == 0;
            if ((x > y) == up) {
              key[i] = y;
              key[ixj] = x;
            }
          }
        }
        __syncthreads();
      }
    for (int g = tid; g < G; g += 1024) {
      const uint32_t lo = gwk[(uint32_t)key[g]];
      const int wdw = (int)(lo >> 8), k = (int)(lo & 255u);
      int i0, i1;
      window(wdw, i0, i1);
      // eight bundles side by side: member j of bundle x at 8 j + x (x in
      // alternating direction, so that no XCD gets all the longer ones)
      constexpr int SB = 8 * ATTN_BUN;
      const int sb = g / SB * SB, r = g - sb, x = r / ATTN_BUN;
      const int at = sb + SB <= G ? sb + 8 * (r % ATTN_BUN) + ((g / SB) & 1 ? 7 - x : x) : g;
      gh[at] = desc(wdw, k, i0, i1);
    }
  }
  for (int g = gbase + tid; g < GPH; g += 1024) gh[g] = make_int4(0, 0, 0, 0);
}

template <int D, int KT, int NW>
struct GrpTile {
  static constexpr int CPR = D / 8;           // 16-byte chunks per row
  static constexpr int RPI = 64 / CPR;        // rows one wave-wide DMA fills
  // DMAs per wavefront, tensor and tile, and the wavefronts that issue them
  static constexpr int NI = KT / (NW * RPI) >= 1 ? KT / (NW * RPI) : 1;
  static constexpr int DW = KT / (NI * RPI);
  static constexpr int ELEMS = KT * D;  // bf16 elements of one K or V tile
  static_assert(DW >= 1 && DW <= NW && NI * DW * RPI == KT, "tile shape");
};

// V swizzle of the 32x32 transpose reads: the 4 rows x 64 bytes that one
// half-wavefront reads cover the 64 banks once
template <int D>
__device__ __forceinline__ int swz_v32(int r) { return D == 128 ? 4 * (r & 3) : 4 * ((r >> 1) & 1); }

template <typename OT, int D>
__global__ __launch_bounds__(2 * ATTN_R, D == 128 ? 2 : 3) void k_attn_grp(
    const bf16_t* __restrict__ Qp, const bf16_t* __restrict__ Kp, const bf16_t* __restrict__ Vp,
    const int* __restrict__ q_offsets, const int* __restrict__ k_offsets,
    const uint32_t* __restrict__ bits, const int* __restrict__ q_perm,
    const int* __restrict__ order, const int* __restrict__ spre, const int4* __restrict__ grp,
    int H, int N, int CQ, int CK, int GPH, float scale_log2, OT* __restrict__ O,
    float* __restrict__ lse) {
  constexpr int KT = 32, NW = ATTN_R / 32, NT = 64 * NW;
  constexpr int NSK = ATTN_KSLOTS, NSV = ATTN_KSLOTS + 1;  // K and V ring slots
  using TS = GrpTile<D, KT, NW>;
  constexpr int KS = D / 16;         // k-steps of S^T
  constexpr int DB = D / 32;         // 32-dimension blocks of O^T
  constexpr int EPT = AT_MAXC / NT;  // key blocks per thread in the union scan
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  bf16_t* Ks = (bf16_t*)smem;                        // [NSK][KT][D], swizzled chunks
  bf16_t* Vs = Ks + NSK * TS::ELEMS;                 // [NSV][KT][D], swizzled chunks
  bf16_t* bias = Vs + NSV * TS::ELEMS;               // [NSK][KT][ATTN_LB]: 0 or -3.39e38
  int2* ut = (int2*)(bias + NSK * KT * ATTN_LB);     // [ATTN_UCAP + 1]
  uint16_t* selw = (uint16_t*)(ut + ATTN_UCAP + 1);  // [ATTN_UCAP]
  int* srow = (int*)(selw + ATTN_UCAP);              // [2 * ATTN_SEG] rows of Kp
  uint16_t* sbit = (uint16_t*)(srow + 2 * ATTN_SEG); // [2 * ATTN_SEG] their selection bits
  __shared__ int sg_row[ATTN_LB], sg_lr[ATTN_LB], sg_u[ATTN_LB];
  __shared__ int tmp[2][NW];
  static_assert(ATTN_LB <= 16, "selection words are 16 bits");

  const int nitems = H * GPH;
  // head-major over the whole chip: consecutive workgroups (dealt to the 8
  // XCDs in turn) take the groups of one head, so only a head or two are in
  // flight at a time and their keys and values stay in the Infinity Cache
  const int item = (int)blockIdx.x;
  if (item >= nitems) return;
  const int h = item / GPH;
  const int4 gd = grp[item];
  const int ib = gd.z, ie = gd.w;
  if (gd.y <= gd.x || ib < 0 || ie <= ib || ie - ib > ATTN_LB || ie > CQ || gd.y - gd.x > ATTN_R)
    return;
  const int nb = ie - ib, tid = threadIdx.x;
  const int* qo = q_offsets + (size_t)h * (CQ + 1);
  const int* koff = k_offsets + (size_t)h * (CK + 1);
  if (tid < ATTN_LB) {
    int lr = 0x7fffffff;
    if (tid < nb) {
      const int i = ib + tid;
      const int u = min(max(order[(size_t)h * CQ + i], 0), CQ - 1);
      const int s0 = spre[(size_t)h * (CQ + 1) + i];
      const int a = max(gd.x, s0);
      sg_u[tid] = u;
      sg_row[tid] = min(max(qo[u], 0), N) + (a - s0);
      lr = a - gd.x;
    }
    sg_lr[tid] = lr;
  }
  __syncthreads();
  const bf16_t* Qh = Qp + (size_t)h * N * D;
  const bf16_t* Kh = Kp + (size_t)h * N * D;
  const bf16_t* Vh = Vp + (size_t)h * N * D;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l = tid & 63, hf = l >> 5, c32 = l & 31;

  // this lane's query row: group row 32 w + c32, query block bq of the group
  const int gr = 32 * w + c32;
  int bq = 0;
#pragma unroll
  for (int b = 1; b < ATTN_LB; ++b) bq += sg_lr[b] <= gr;  // (ascending; INT_MAX past the blocks)
  const int qr0 = sg_row[bq] + (gr - sg_lr[bq]);
  const bool qvalid = gr < gd.y - gd.x && (unsigned)qr0 < (unsigned)N;
  const int qr = qvalid ? qr0 : 0;
  bf16x8_t qf[KS];
#pragma unroll
  for (int s2 = 0; s2 < KS; ++s2) {
    uint4 raw = make_uint4(0u, 0u, 0u, 0u);
    if (qvalid) raw = *(const uint4*)(Qh + (size_t)qr * D + 16 * s2 + 8 * hf);
    qf[s2] = __builtin_bit_cast(bf16x8_t, raw);
  }
  const int dst = qvalid ? q_perm[(size_t)h * N + qr] : -1;
  // one-hot of the query block (the B operand of the bias product), the one
  // being 2^127, so that the product with a bias of -3.39e38 overflows to -inf
  // (and with 0 is 0): lanes of half hf hold blocks 8 hf .. 8 hf + 7
  const int oe = (qvalid ? bq : 0) - 8 * hf;
  uint32_t ow[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) ow[k] = (oe >> 1) == k ? 0x7f00u << (16 * (oe & 1)) : 0u;
  const bf16x8_t hot = __builtin_bit_cast(bf16x8_t, make_uint4(ow[0], ow[1], ow[2], ow[3]));

  // LDS read offsets (bytes, relative to a slot).  The swizzle only flips
  // chunk bits, so the other k-steps and dimension blocks are XORs of one
  // offset with a constant (slots are aligned to a row).
  // K (A operand of S^T): key row c32, chunk 2 s + hf at kofs ^ 32 s
  const uint32_t kofs = c32 * (2 * D) + 16 * (hf ^ swz_k<D>(c32));
  // V^T (A operand of O^T) by transpose reads: in 16-lane group G, lane j
  // gives row 4 hf + j/4 (+ 16 kappa, + 8 for the second read) and dims
  // 32 db + 16 (G % 2) + 4 (j % 4); it receives dim 32 db + 16 (G % 2) + j;
  // block db at vofs ^ 64 db
  const int G = l >> 4, jg = l & 15;
  const int vr0 = 4 * hf + (jg >> 2);
  const int vcol = 16 * (G & 1) + 4 * (jg & 3);
  const uint32_t vofs = vr0 * (2 * D) + 16 * ((vcol >> 3) ^ swz_v32<D>(vr0)) + 2 * (vcol & 7);

  // reference maximum: no finite score is below the start, and a key the row's
  // block did not select has score -inf, so its probability is 0 at any (finite)
  // reference, also before the first selected key
  constexpr float NOKEY = -3.4028235e38f;  // -FLT_MAX
  float m = NOKEY, lpart = 0.0f, tmax = NOKEY;
  f32x16_t acc[DB];
#pragma unroll
  for (int b = 0; b < DB; ++b)
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[b][q] = 0.0f;

  // DMA lanes: tile row rr[i], chunk position pch
  const int pch = l % TS::CPR;
  const bool dma_w = w < TS::DW;
  int rr[TS::NI];
#pragma unroll
  for (int i = 0; i < TS::NI; ++i) rr[i] = (w * TS::NI + i) * TS::RPI + l / TS::CPR;

  // the union (U key blocks) is streamed in chunks of at most ATTN_UCAP key
  // blocks; the online softmax state carries over from one chunk to the next
  const int lane = tid & 63, wv = tid >> 6;
  int U = ATTN_UCAP;
  for (int ch = 0; ch * ATTN_UCAP < U; ++ch) {
    // stream table of this chunk: ut[j] = {stream position, first row of Kp}
    // of its j-th key block, ut[Uc] = {end position, -1}; selw[j] its bits
    {
      // f[k], bit b: query block b of the group selected key block tid EPT + k
      // (from the bit rows of the plan: one word per block and thread)
      static_assert(32 % EPT == 0, "a thread's key blocks lie in one word of a bit row");
      int2 kb2[EPT];  // block boundaries (clamped ids)
#pragma unroll
      for (int k = 0; k < EPT; ++k) kb2[k] = *(const int2*)(koff + min(tid * EPT + k, CK - 1));
      uint32_t f[EPT] = {};
      for (int b0 = 0; b0 < nb; b0 += 4) {
        uint32_t y[4];
#pragma unroll
        for (int b = 0; b < 4; ++b)
          y[b] = bits[((size_t)h * CQ + sg_u[min(b0 + b, nb - 1)]) * 64 + tid * EPT / 32];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          y[b] = b0 + b < nb ? y[b] >> (tid * EPT % 32) : 0u;
#pragma unroll
          for (int k = 0; k < EPT; ++k) f[k] |= ((y[b] >> k) & 1u) << (b0 + b);
        }
      }
      int x[EPT], kst[EPT], c = 0, s = 0;
#pragma unroll
      for (int k = 0; k < EPT; ++k) {
        const int v = tid * EPT + k;
        if (v >= CK) f[k] = 0u;
        x[k] = 0;
        kst[k] = -1;
        if (f[k]) {
          kst[k] = kb2[k].x;
          x[k] = max(0, kb2[k].y - kst[k]);
          ++c;
        }
        s += x[k];
      }
      int ic = c, is = s;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int yc = __shfl_up(ic, o, 64), ys = __shfl_up(is, o, 64);
        if (lane >= o) {
          ic += yc;
          is += ys;
        }
      }
      if (lane == 63) {
        tmp[0][wv] = ic;
        tmp[1][wv] = is;
      }
      __syncthreads();
      int jc = ic - c, js = is - s;
      U = 0;
      for (int w2 = 0; w2 < NW; ++w2) {
        jc += w2 < wv ? tmp[0][w2] : 0;
        js += w2 < wv ? tmp[1][w2] : 0;
        U += tmp[0][w2];
      }
      const int jlo = ch * ATTN_UCAP, jhi = min(jlo + ATTN_UCAP, U);
#pragma unroll
      for (int k = 0; k < EPT; ++k)
        if (f[k]) {
          if (jc >= jlo && jc < jhi) {
            ut[jc - jlo] = make_int2(js, kst[k]);
            selw[jc - jlo] = (uint16_t)f[k];
            if (jc == jhi - 1) ut[jc - jlo + 1] = make_int2(js + x[k], -1);
          }
          ++jc;
          js += x[k];
        }
      __syncthreads();
    }
    if (U == 0) break;
    const int Uc = min(ATTN_UCAP, U - ch * ATTN_UCAP);
    const int base = ut[0].x, nk = ut[Uc].x - base;
    // stream positions [ATTN_SEG sg, ATTN_SEG (sg + 1)) of this chunk as rows of
    // Kp and selection bits (positions past the end: row 0, no bit), in the
    // half of the table that segment sg - 2 held
    auto expand = [&](int sg) {
#pragma unroll 1
      for (int k = 0; k < ATTN_SEG / NT; ++k) {
        const int q = sg * ATTN_SEG + k * NT + tid, pos = base + q;
        int lo = 0, hi = Uc - 1;
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (ut[mid].x <= pos) lo = mid;
          else hi = mid - 1;
        }
        const int2 e = ut[lo];
        const int r = e.y + (pos - e.x);
        const bool ok = q < nk && (unsigned)r < (unsigned)N;
        srow[q & (2 * ATTN_SEG - 1)] = ok ? r : 0;
        sbit[q & (2 * ATTN_SEG - 1)] = ok ? selw[lo] : (uint16_t)0;
      }
    };
    // tile T: K into slot T % NSK with the score bias of every (tile row, query
    // block), V into slot T % NSV (one step later: srcv are the rows of the
    // tile whose keys went out in the step before)
    int src[TS::NI], srcv[TS::NI];
    uint32_t kb;  // selection bits of the tile row whose bias this thread writes
    constexpr int BT = KT * ATTN_LB / 2 / NT;  // 32-bit words of the bias tile per thread
    const int brow = tid * BT / 8, bword = tid * BT % 8;
    auto rows_of = [&](int T) {
#pragma unroll
      for (int i = 0; i < TS::NI; ++i) {
        srcv[i] = src[i];
        src[i] = srow[((T * KT) & (2 * ATTN_SEG - 1)) + rr[i]];
      }
      kb = sbit[((T * KT) & (2 * ATTN_SEG - 1)) + brow];
    };
    auto issue_k = [&](int T) {
      const int sk = T % NSK;
      uint32_t* bs = (uint32_t*)(bias + sk * KT * ATTN_LB) + tid * BT;
#pragma unroll
      for (int k = 0; k < BT; ++k) {
        const uint32_t y = kb >> (2 * (bword + k));
        bs[k] = (y & 1u ? 0u : 0xff7fu) | (y & 2u ? 0u : 0xff7f0000u);
      }
      if (!dma_w) return;
      const uint32_t ks = lds_addr(Ks) + sk * (2 * TS::ELEMS) + w * TS::NI * 1024;
#pragma unroll
      for (int i = 0; i < TS::NI; ++i)  // 1 KB per wave-wide DMA
        lds_dma16(Kh, (uint32_t)src[i] * (2 * D) + 16 * (pch ^ swz_k<D>(rr[i])), ks + 1024 * i);
    };
    auto issue_v = [&](int T) {
      if (!dma_w) return;
      const uint32_t vs = lds_addr(Vs) + (T % NSV) * (2 * TS::ELEMS) + w * TS::NI * 1024;
#pragma unroll
      for (int i = 0; i < TS::NI; ++i)
        lds_dma16(Vh, (uint32_t)srcv[i] * (2 * D) + 16 * (pch ^ swz_v32<D>(rr[i])), vs + 1024 * i);
    };
    // operands of tile T's scores: the K fragments, and the bias rows (key c32,
    // blocks 8 hf ..): bias x one-hot starts a score from 0 or -inf
    bf16x8_t kf[KS], bf;
    auto load_k = [&](int T) {
      const int sk = T % NSK;
      const uint32_t ko = lds_addr(Ks) + sk * (2 * TS::ELEMS) + kofs;
      bf = *(lds_bf16x8_t*)(lds_addr(bias) + sk * (2 * KT * ATTN_LB) + 32 * c32 + 16 * hf);
#pragma unroll
      for (int s2 = 0; s2 < KS; ++s2) kf[s2] = *(lds_bf16x8_t*)(ko ^ (32 * s2));
    };
    auto bias_scores = [&]() {
      const f32x16_t zero = {};
      return __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf, hot, zero, 0, 0, 0);
    };
    auto row_max = [&](const f32x16_t& st) {
      float x = fmaxf(st[0], st[1]);
#pragma unroll
      for (int q = 2; q < 16; ++q) x = fmaxf(x, st[q]);
      tmax = max_xor32(x);
    };
    const int ntiles = (nk + KT - 1) / KT;
    // One step of the pipeline.  At the top: sc holds the scores of tile t and
    // tmax their row maxima, kf and bf the operands of tile t + 1's, tiles up
    // to K(t+3), V(t+2) are in flight.  Every LDS read is issued half a step
    // before its first use, and the vector work sits between the MFMAs:
    //   first half   S(t+1) = K Q^T        beside the probabilities of tile t
    //   second half  O += V(t)^T P(t)^T    beside the row maxima of tile t + 1
    // (scores past the last tile come from a stale slot and are never used)
    auto step = [&](int t, const f32x16_t& sc, f32x16_t& sn) {
      // K(t+2) and everything issued before it (V(t)) has landed; V(t+1),
      // K(t+3) and V(t+2) may stay in flight
      if (t + NSK < ntiles) wait_vmcnt<3 * TS::NI>();
      else wait_vmcnt<0>();
      __syncthreads();  // K(t+2), V(t) visible; K(t+1) and V(t-1) are read
      // every ATTN_SEG / KT tiles, the rows of the next segment (the prefetch
      // has left the segment before this one)
      if ((t & (ATTN_SEG / KT - 1)) == 0 && t * KT + ATTN_SEG < nk)
        expand(t / (ATTN_SEG / KT) + 1);
      // the reference maximum moves only when a row maximum exceeds it by more
      // than 2^8 in probability (softmax is invariant to the shift; p <= 2^8)
      if (__any((tmax - m) * scale_log2 > 8.0f)) {
        const float mnew = fmaxf(m, tmax);
        const float alpha = __builtin_amdgcn_exp2f((m - mnew) * scale_log2);
        lpart *= alpha;
#pragma unroll
        for (int b = 0; b < DB; ++b) acc[b] *= alpha;
        m = mnew;
      }
      bf16x8_t vf[2][DB];
      const uint32_t vo = lds_addr(Vs) + (t % NSV) * (2 * TS::ELEMS) + vofs;
#pragma unroll
      for (int kp = 0; kp < 2; ++kp)
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          const uint32_t v1 = (vo ^ (64 * db)) + 32 * kp * D;
          const i16x4_t t1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t*)v1);
          const i16x4_t t2 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t*)(v1 + 16 * D));
          vf[kp][db] = __builtin_bit_cast(
              bf16x8_t, (short __attribute__((ext_vector_type(8)))){t1[0], t1[1], t1[2], t1[3],
                                                                    t2[0], t2[1], t2[2], t2[3]});
        }
      // probabilities: step kp of the product takes scores 8 kp .. 8 kp + 7
      // (keys 16 kp + 4 hf + r and 16 kp + 8 + 4 hf + r)
      constexpr int EP = 16 / KS;  // scores per MFMA of the first half
      const float nms = -m * scale_log2;
      bf16x8_t pb[2];
      float ls[2] = {0.0f, 0.0f};
      sn = bias_scores();
#pragma unroll
      for (int s2 = 0; s2 < KS; ++s2) {
        sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s2], qf[s2], sn, 0, 0, 0);
#pragma unroll
        for (int e = EP * s2; e < EP * (s2 + 1); e += 2) {
          const float p0 = __builtin_amdgcn_exp2f(fmaf(sc[e], scale_log2, nms));
          const float p1 = __builtin_amdgcn_exp2f(fmaf(sc[e + 1], scale_log2, nms));
          ls[0] += p0;
          ls[1] += p1;
          const bf16x2_t two = __builtin_convertvector(f32x2_t{p0, p1}, bf16x2_t);
          pb[e / 8][e % 8] = two[0];
          pb[e / 8][e % 8 + 1] = two[1];
        }
        // (the sums are taken here, so that the probabilities need not be kept)
        asm volatile("" : "+v"(ls[0]), "+v"(ls[1]));
      }
      lpart += ls[0] + ls[1];
      load_k(t + 2);
      rows_of(t + NSK + 1);  // (past the end: row 0, or a stale row; not issued)
#pragma unroll
      for (int kp = 0; kp < 2; ++kp)
#pragma unroll
        for (int db = 0; db < DB; ++db)
          acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[kp][db], pb[kp], acc[db], 0, 0, 0);
      row_max(sn);
      if (t + NSK + 1 < ntiles) issue_k(t + NSK + 1);
      if (t + NSK < ntiles) issue_v(t + NSK);
    };
    expand(0);
    __syncthreads();
    static_assert(NSK == 3 && NSV == 4, "the pipeline's look-ahead");
    // fill: K(0), K(1) V(0), K(2) V(1); S(0), the operands of S(1); K(3) V(2)
    f32x16_t s0, s1;
    if (ntiles > 0) {
      // (Q has arrived: from here on the counted waits see only the DMAs)
#pragma unroll
      for (int s2 = 0; s2 < KS; ++s2) asm volatile("" ::"v"(qf[s2]));
      asm volatile("" ::"v"(dst));
#pragma unroll
      for (int p = 0; p < NSK; ++p) {
        rows_of(p);  // (past the end: row 0, no bit)
        issue_k(p);
        if (p > 0) issue_v(p - 1);
      }
      wait_vmcnt<3 * TS::NI>();  // K(0), K(1)
      __syncthreads();
      load_k(0);
      s0 = bias_scores();
#pragma unroll
      for (int s2 = 0; s2 < KS; ++s2)
        s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s2], qf[s2], s0, 0, 0, 0);
      load_k(1);
      row_max(s0);
      __syncthreads();  // K(0) is read
      rows_of(NSK);
      if (NSK < ntiles) issue_k(NSK);
      if (NSK - 1 < ntiles) issue_v(NSK - 1);
    }
    for (int t = 0; t < ntiles; t += 2) {
      step(t, s0, s1);
      if (t + 1 < ntiles) step(t + 1, s1, s0);
    }
    __syncthreads();  // every wavefront is done with this chunk's tables and ring
  }
  const float lsum = lpart + __shfl_xor(lpart, 32, 64);
  if ((unsigned)dst >= (unsigned)N) return;
  const float inv = lsum > 0.0f ? 1.0f / lsum : 0.0f;
  // natural-log normaliser: the probabilities are exp2((s - m) scale_log2) of
  // raw scores s, so sum_j exp(s_j / sqrt(d)) = exp(m / sqrt(d)) lsum
  if (lse && hf == 0)
    lse[(size_t)h * N + dst] =
        lsum > 0.0f ? m * (scale_log2 * 0.69314718055994531f) + logf(lsum) : -INFINITY;
  OT* o = O + ((size_t)h * N + dst) * D + 4 * hf;
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int b4 = 0; b4 < 4; ++b4)
      store_out4<OT>(o + 32 * db + 8 * b4, acc[db][4 * b4 + 0] * inv, acc[db][4 * b4 + 1] * inv,
                     acc[db][4 * b4 + 2] * inv, acc[db][4 * b4 + 3] * inv);
}

template <typename OT>
static park_status attn_f32_d(const void* Qp, const void* Kp, const void* Vp, const int* qo,
                              const int* ko, const int* kc, const int* ki, const int* qp, int H,
                              int N, int D, int CQ, int CK, void* O, float* lse, hipStream_t st) {
  // 32-row workgroups for query blocks up to twice the mean size (larger ones
  // take several rounds; the block sizes are known on the device only)
  const unsigned nz = (unsigned)std::min((size_t)65535, 2 * (((size_t)N + 32u * CQ - 1) / (32u * (size_t)CQ)));
  const dim3 g(CQ, H, nz);
  const float sc = (float)(1.0 / sqrt((double)D)), sl2 = (float)(1.4426950408889634 / sqrt((double)D));
  if (D == 128)
    PARK_LAUNCH("attn_f32", (k_attn_f32<OT, 128>), g, dim3(512), 0, st, (const float*)Qp,
                (const float*)Kp, (const float*)Vp, qo, ko, kc, ki, qp, N, CQ, CK, sc, sl2, (OT*)O,
                lse);
  else
    PARK_LAUNCH("attn_f32", (k_attn_f32<OT, 64>), g, dim3(512), 0, st, (const float*)Qp,
                (const float*)Kp, (const float*)Vp, qo, ko, kc, ki, qp, N, CQ, CK, sc, sl2, (OT*)O,
                lse);
  return PARK_OK;
}

size_t attn_grp_offset(int H, int CQ);
// the families [H][CQ], padded to 16 bytes (the bit rows follow)
static size_t attn_fam_bytes(int H, int CQ) { return ((size_t)H * CQ * sizeof(int) + 15) & ~(size_t)15; }

template <typename OT, int D>
static park_status attn_grp_launch(const void* Qp, const void* Kp, const void* Vp, const int* qo,
                                   const int* ko, const int* kc, const int* ki, const int* qp,
                                   int H, int N, int CQ, int CK, void* plan, float sl2, void* O,
                                   float* lse, hipStream_t st) {
  const int GPH = attn_groups_per_head(N, CQ);
  int* order = (int*)plan;
  int* spre = order + (size_t)H * CQ;
  int4* grp = (int4*)((char*)plan + attn_grp_offset(H, CQ));
  int* fam = (int*)(grp + (size_t)H * GPH);
  uint32_t* bits = (uint32_t*)((char*)fam + attn_fam_bytes(H, CQ));
  uint4* rkey = (uint4*)(bits + (size_t)H * CQ * 64);
  const unsigned nrow = (unsigned)H * (unsigned)CQ, ntile = (unsigned)(CQ + 63) / 64;
  PARK_LAUNCH("attn_selbits", k_attn_selbits, dim3((nrow + 3) / 4), dim3(256), 0, st, kc, ki, qo,
              ko, H, N, CQ, CK, bits, fam, rkey);
  PARK_LAUNCH("attn_family", k_attn_family, dim3(ntile * (ntile + 1) / 2, H), dim3(256), 0, st,
              kc, bits, CQ, CK, fam);
  PARK_LAUNCH("attn_plan", k_attn_gplan, dim3(H), dim3(1024), 0, st, qo, (const uint4*)rkey,
              (const int*)fam, N, CQ, CK, GPH, order, spre, grp);
  // K ring, V ring, score biases, stream table, selection words, stream rows
  constexpr size_t lds = (size_t)(2 * ATTN_KSLOTS + 1) * 32 * D * sizeof(bf16_t) +
                         (size_t)ATTN_KSLOTS * ATTN_LB * 32 * 2 +
                         (size_t)(ATTN_UCAP + 1) * sizeof(int2) + (size_t)ATTN_UCAP * 2 +
                         (size_t)2 * ATTN_SEG * 6;
  static std::atomic<uint64_t> done{0};
  PARK_TRY(reserve_lds((const void*)k_attn_grp<OT, D>, lds, done, "attention"));
  // one workgroup per item, rounded up to whole turns over the 8 XCDs
  const unsigned nwg = 8u * (((unsigned)H * (unsigned)GPH + 7u) / 8u);
  PARK_LAUNCH("attn_mfma", (k_attn_grp<OT, D>), dim3(nwg), dim3(2 * ATTN_R), lds, st,
              (const bf16_t*)Qp, (const bf16_t*)Kp, (const bf16_t*)Vp, qo, ko, bits, qp, order, spre,
              grp, H, N, CQ, CK, GPH, sl2, (OT*)O, lse);
  return PARK_OK;
}

template <typename OT>
static park_status attn_mfma_d(const void* Qp, const void* Kp, const void* Vp, const int* qo,
                               const int* ko, const int* kc, const int* ki, const int* qp, int H,
                               int N, int D, int CQ, int CK, void* plan, void* O, float* lse,
                               hipStream_t st) {
  const float sl2 = (float)(1.4426950408889634 / sqrt((double)D));
  if (D == 128)
    return attn_grp_launch<OT, 128>(Qp, Kp, Vp, qo, ko, kc, ki, qp, H, N, CQ, CK,
                                                  plan, sl2, O, lse, st);
  return attn_grp_launch<OT, 64>(Qp, Kp, Vp, qo, ko, kc, ki, qp, H, N, CQ, CK, plan,
                                              sl2, O, lse, st);
}

// order [H][CQ], spre [H][CQ + 1], then the groups [H][GPH] at 16-byte
// alignment, the selection families [H][CQ] (padded to 16 bytes), the
// selection bit rows [H][CQ][64] and the sort-key parts [H][CQ] (uint4)
size_t attn_grp_offset(int H, int CQ) {
  return (((size_t)H * CQ + (size_t)H * (CQ + 1)) * sizeof(int) + 15) & ~(size_t)15;
}

size_t attn_plan_bytes(int H, int N, int CQ) {
  return attn_grp_offset(H, CQ) + (size_t)H * attn_groups_per_head(N, CQ) * sizeof(int4) +
         attn_fam_bytes(H, CQ) + (size_t)H * CQ * 64 * sizeof(uint32_t) +
         (size_t)H * CQ * sizeof(uint4);
}

park_status launch_attention(const void* Qp, const void* Kp, const void* Vp, const int* q_offsets,
                             const int* k_offsets, const int* kv_count, const int* kv_index,
                             const int* q_perm, int H, int N, int D, int dtype, int CQ, int CK,
                             void* O, int out_dtype, float* lse, void* plan,
                             hipStream_t st) {
  if (dtype == PARK_BF16) {
    if (out_dtype == PARK_BF16)
      return attn_mfma_d<bf16_t>(Qp, Kp, Vp, q_offsets, k_offsets, kv_count, kv_index, q_perm, H,
                                 N, D, CQ, CK, plan, O, lse, st);
    return attn_mfma_d<float>(Qp, Kp, Vp, q_offsets, k_offsets, kv_count, kv_index, q_perm, H, N,
                              D, CQ, CK, plan, O, lse, st);
  }
  if (out_dtype == PARK_BF16)
    return attn_f32_d<bf16_t>(Qp, Kp, Vp, q_offsets, k_offsets, kv_count, kv_index, q_perm, H, N,
                              D, CQ, CK, O, lse, st);
  return attn_f32_d<float>(Qp, Kp, Vp, q_offsets, k_offsets, kv_count, kv_index, q_perm, H, N, D,
                           CQ, CK, O, lse, st);
}

}  // namespace park
