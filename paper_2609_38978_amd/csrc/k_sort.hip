// Stable counting sort of cluster labels (pi = argsort(z), Alg. 3) and the
// row gathers X' = X[pi].  Two passes: per-tile histograms, then a stable
// scatter in which each tile's workgroup first derives its own bases from the
// histogram table (cluster totals scanned over clusters, plus the counts of
// the earlier tiles) and then ranks its tokens, every wavefront its own run of
// consecutive ones.  All integer work; the result is unique, so it is
// bit-exact and deterministic.
#include "common.h"
#include "kernels.h"

namespace park {

constexpr int SORT_MAXC = 2048;

// Tokens per sort tile.  Every wavefront of a scatter workgroup ranks at least
// four steps of 64: a head of up to 4096 tokens is one tile (no histogram pass) of
// eight or sixteen wavefronts, up to 8192 tokens four wavefronts take 1024 and
// beyond that eight take 2048, doubled until a head has at most 32 tiles, so that a
// scatter workgroup reads its column of the histogram table in one or two round
// trips of loads; at most 32768, since the counts inside a tile are 16 bits wide.
// Sixteen wavefronts on 4096 tokens, eight on 2048 and four on 1024 (us a call of
// 10 rounds, d = 64): 1 x 2000 259, 255, 274; 24 x 2100 303, 333, 325; 1 x 4157
// 337, 313, 309 (one wavefront on tiles of 256: 346); 24 x 4157 416, 391, 387
// (387); 24 x 6500 514, 496, 490 (517); 1 x 17019 446, 432, 443; 24 x 12000 707,
// 691, 693; 5 x 64000 1057, 1046, 1085.
int sort_tile(int H, int N, int C) {
  (void)H;
  (void)C;
  if (N > 2048 && N <= 4096) return 4096;
  int t = N > 4096 && N <= 8192 ? 1024 : 2048;
  while ((N + t - 1) / t > 32 && t < 32768) t *= 2;
  return t;
}

int sort_tiles(int H, int N, int C) {
  const int t = sort_tile(H, N, C);
  return (N + t - 1) / t;
}

// thist[h][tile][v] = #{ i in tile : z_i = v }
template <int NT>
__global__ __launch_bounds__(NT) void k_sort_hist(const int* __restrict__ labels, int N, int C,
                                                       int tile_sz, int* __restrict__ thist) {
  extern __shared__ int hist[];
  const int h = blockIdx.y, tile = blockIdx.x, nt = gridDim.x;
  for (int v = threadIdx.x; v < C; v += NT) hist[v] = 0;
  __syncthreads();
  const int i0 = tile * tile_sz, i1 = min(N, i0 + tile_sz);
  const int* z = labels + (size_t)h * N;
  // four loads in flight per thread
  for (int c0 = i0; c0 < i1; c0 += 4 * NT) {
    int v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = c0 + NT * k + threadIdx.x;
      v[k] = i < i1 ? z[i] : -1;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if ((unsigned)v[k] < (unsigned)C) atomicAdd(&hist[v[k]], 1);
  }
  __syncthreads();
  int* out = thist + ((size_t)h * nt + tile) * C;
  for (int v = threadIdx.x; v < C; v += NT) out[v] = hist[v];
}

// Stable scatter of one tile (grid: tiles x heads; thist may be null when a
// head is one tile).
//  1. Thread v sums cluster v's counts over the tiles before this one and over
//     all tiles (16 table rows in flight); the totals are scanned over the
//     clusters: base_v = start_v + earlier counts.  Tile 0 also writes the
//     cluster offsets (o[C] = N).
//  2. Every wavefront counts the clusters of its own tokens (LDS, 16-bit
//     halves), and the counts become, per cluster, the tokens of the
//     wavefronts before it.
//  3. Every wavefront walks its tokens in order, 64 at a time; equal labels
//     inside a step are matched with one ballot per label bit.
// What bounds it: a chain of round trips, not the bytes.  One wavefront per
// tile walking 64 steps alone, after 40 dependent batches of table loads per
// thread, took 66 us at 3 x 119056 tokens, C = 1861 (14 us at 12 x 17019,
// C = 266; 14.5 us at 1 x 4096; 51 us at 40 x 75600, C = 1182) as one launch on
// an otherwise idle chip; sixteen wavefronts with four steps each and 30-row
// tables take 14.6 us (6.5 at 1 x 4096), eight take 7.2 at 12 x 17019 and 26 at
// 40 x 75600 (see launch_count_sort).
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_sort_scatter(const int* __restrict__ labels, int N, int C,
                                                          int nbits, int tile_sz,
                                                          const int* __restrict__ thist,
                                                          int* __restrict__ perm,
                                                          int* __restrict__ offsets) {
  constexpr int NT = 64 * NW;
  extern __shared__ uint32_t sort_lds[];
  const int C2 = (C + 1) / 2;       // 32-bit words of one wavefront's counts
  uint32_t* cnt = sort_lds;         // [NW][C2]: two clusters per word
  int* base = (int*)(cnt + NW * C2);  // [C]
  __shared__ int wsum[NW];
  const int h = blockIdx.y, tile = blockIdx.x, nt = gridDim.x, tid = threadIdx.x;
  const int lane = tid & 63, wid = tid >> 6;
  const int* z = labels + (size_t)h * N;
  const int i0 = tile * tile_sz, i1 = min(N, i0 + tile_sz);
  const int share = tile_sz / NW;  // tokens of a wavefront (a multiple of 256)
  const int j0 = i0 + wid * share, j1 = min(i1, j0 + share);
  for (int e = tid; e < NW * C2; e += NT) cnt[e] = 0u;
  __syncthreads();
  uint32_t* cw = cnt + wid * C2;
  for (int c0 = j0; c0 < j1; c0 += 256) {
    int v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = c0 + 64 * k + lane;
      v[k] = i < j1 ? z[i] : -1;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if ((unsigned)v[k] < (unsigned)C) atomicAdd(&cw[v[k] >> 1], 1u << (16 * (v[k] & 1)));
  }
  // thread tid owns clusters tid and tid + NT in the table, and the
  // consecutive ones tid * per + k in the scan
  int before[SORT_MAXC / NT], all[SORT_MAXC / NT];
#pragma unroll
  for (int q = 0; q < SORT_MAXC / NT; ++q) {
    const int v = tid + q * NT;
    before[q] = all[q] = 0;
    if (v < C && thist) {
      const int* b = thist + (size_t)h * nt * C + v;
      for (int t0 = 0; t0 < nt; t0 += 16) {
        int c[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) c[k] = b[(size_t)min(t0 + k, nt - 1) * C];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          all[q] += t0 + k < nt ? c[k] : 0;
          before[q] += t0 + k < tile ? c[k] : 0;
        }
      }
    }
  }
  __syncthreads();
  // counts -> tokens of earlier wavefronts (two 16-bit clusters per word: a
  // tile's 32768 tokens never carry from one into the other)
  for (int e = tid; e < C2; e += NT) {
    uint32_t run = 0u;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const uint32_t x = cnt[w * C2 + e];
      cnt[w * C2 + e] = run;
      run += x;
    }
    if (!thist) {  // one tile: these are the cluster totals
      base[2 * e] = (int)(run & 0xffffu);
      if (2 * e + 1 < C) base[2 * e + 1] = (int)(run >> 16);
    }
  }
  if (thist)
#pragma unroll
    for (int q = 0; q < SORT_MAXC / NT; ++q)
      if (tid + q * NT < C) base[tid + q * NT] = all[q];
  __syncthreads();
  const int per = (C + NT - 1) / NT;
  int s = 0, tv[SORT_MAXC / NT];
#pragma unroll
  for (int k = 0; k < SORT_MAXC / NT; ++k) {
    const int v = tid * per + k;
    tv[k] = k < per && v < C ? base[v] : 0;
    s += tv[k];
  }
  int inc = s;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(inc, o, 64);
    if (lane >= o) inc += y;
  }
  if (lane == 63) wsum[wid] = inc;
  __syncthreads();
  int pre = inc - s;
#pragma unroll
  for (int q = 0; q < NW; ++q) pre += q < wid ? wsum[q] : 0;
  int* off = offsets + (size_t)h * (C + 1);
#pragma unroll
  for (int k = 0; k < SORT_MAXC / NT; ++k) {
    const int v = tid * per + k;
    if (k < per && v < C) {
      base[v] = pre;
      if (tile == 0) off[v] = pre;
      pre += tv[k];
    }
  }
  if (tile == 0 && tid == 0) off[C] = N;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < SORT_MAXC / NT; ++q)
    if (tid + q * NT < C) base[tid + q * NT] += before[q];
  __syncthreads();
  int* p = perm + (size_t)h * N;
  uint16_t* cw16 = (uint16_t*)cw;
  const uint64_t lt = (1ull << lane) - 1ull;
  const uint64_t gt = ~((2ull << lane) - 1ull);
  for (int c0 = j0; c0 < j1; c0 += 256) {
    int vv[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = c0 + 64 * k + lane;
      vv[k] = i < j1 ? z[i] : -1;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = c0 + 64 * k + lane;
      const int v = vv[k];
      const bool ok = (unsigned)v < (unsigned)C;
      uint64_t m = __ballot(ok);
      if (m == 0ull) break;
      for (int bit = 0; bit < nbits; ++bit) {
        const bool set = (v >> bit) & 1;
        const uint64_t B = __ballot(ok && set);
        m &= set ? B : ~B;
      }
      const int rank = __popcll(m & lt);
      const int own = ok ? (int)cw16[v] : 0;
      if (ok) p[base[v] + own + rank] = i;
      // the wavefront's own counts, whose LDS accesses complete in order; the
      // fences keep the compiler from moving reads and updates across each other
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (ok && (m & gt) == 0) cw16[v] = (uint16_t)(own + rank + 1);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
  }
}

template <int NW>
static park_status count_sort(const int* labels, int H, int N, int C, int* thist, int* perm,
                              int* offsets, hipStream_t st) {
  constexpr int NT = 64 * NW;
  const int tsz = sort_tile(H, N, C);
  const int nt = (N + tsz - 1) / tsz;
  int nbits = 1;
  while ((1 << nbits) < C) ++nbits;
  // one tile per head: the scatter counts for itself
  if (nt > 1)
    PARK_LAUNCH("sort_hist", k_sort_hist<NT>, dim3(nt, H), dim3(NT), (size_t)C * sizeof(int), st,
                labels, N, C, tsz, thist);
  const size_t lds = (size_t)NW * ((C + 1) / 2) * 4 + (size_t)C * 4;
  static std::atomic<uint64_t> done{0};
  PARK_TRY(reserve_lds((const void*)k_sort_scatter<NW>, NW * SORT_MAXC / 2 * 4 + SORT_MAXC * 4, done,
                       "sort"));
  PARK_LAUNCH("sort_scatter", k_sort_scatter<NW>, dim3(nt, H), dim3(NT), lds, st, labels, N, C, nbits,
              tsz, (const int*)(nt > 1 ? thist : nullptr), perm, offsets);
  return PARK_OK;
}

// Four and eight wavefronts for the tiles of 1024 and 2048.  Of larger ones, sixteen
// finish a tile soonest; with more workgroups than CUs eight serve better: twice
// as many fit beside each other and beside what the other stream runs, where a
// 1024-thread workgroup waits for a CU to clear (launch times, scatter +
// histogram, eight : sixteen; both sides of a layer in flight: 24 x 119056 75 + 18 :
// 117 + 34 us, 40 x 75600 95 + 13 : 109 + 48, the layers themselves equal within
// noise; 40 x 75600 queries alone 26 + 5 : 35 + 6; below the line, 3 x 119056
// 16.7 : 14.7).
park_status launch_count_sort(const int* labels, int H, int N, int C, int* thist, int* perm,
                              int* offsets, hipStream_t st) {
  const int t = sort_tile(H, N, C);
  if (t == 1024) return count_sort<4>(labels, H, N, C, thist, perm, offsets, st);
  if (t == 2048 || (long)H * sort_tiles(H, N, C) > 256)
    return count_sort<8>(labels, H, N, C, thist, perm, offsets, st);
  return count_sort<16>(labels, H, N, C, thist, perm, offsets, st);
}

// Xp[h][i] = X[h][perm[h][i]], 16-byte vectors.
__global__ __launch_bounds__(256) void k_gather(const uint4* __restrict__ X, const int* __restrict__ perm,
                                                int N, int vpr, uint4* __restrict__ Xp) {
  const int h = blockIdx.y;
  const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t total = (size_t)N * vpr;
  if (t >= total) return;
  const int i = (int)(t / vpr), c = (int)(t % vpr);
  const int src = perm[(size_t)h * N + i];
  uint4 val = make_uint4(0u, 0u, 0u, 0u);
  if ((unsigned)src < (unsigned)N) val = X[((size_t)h * N + src) * vpr + c];
  Xp[((size_t)h * N + i) * vpr + c] = val;
}

park_status launch_gather(const void* X, const int* perm, int H, int N, int D, int dtype, void* Xp,
                          hipStream_t st) {
  const int vpr = (int)(D * elem_size(dtype) / 16);
  const size_t total = (size_t)N * vpr;
  dim3 g((unsigned)((total + 255) / 256), H);
  PARK_LAUNCH("gather_rows", k_gather, g, dim3(256), 0, st, (const uint4*)X, perm, N, vpr,
              (uint4*)Xp);
  return PARK_OK;
}

// Fixed-tile blocks of the cluster-ordered tokens: offsets[h][v] =
// min(v b, N) for v = 0..C, b = ceil(N / C).
__global__ __launch_bounds__(256) void k_fixed_offsets(int N, int C, int b,
                                                       int* __restrict__ offsets) {
  const int h = blockIdx.y;
  const int v = blockIdx.x * 256 + threadIdx.x;
  if (v > C) return;
  const long o = (long)v * b;
  offsets[(size_t)h * (C + 1) + v] = o < (long)N ? (int)o : N;
}

park_status launch_fixed_offsets(int H, int N, int C, int* offsets, hipStream_t st) {
  const int b = (N + C - 1) / C;
  PARK_LAUNCH("fixed_offsets", k_fixed_offsets, dim3((C + 1 + 255) / 256, H), dim3(256), 0, st,
              N, C, b, offsets);
  return PARK_OK;
}

// Rows of the nonempty blocks packed in block order: row u of x (sizes[u] >
// 0) moves to row r_u = #{w < u : sizes[w] > 0} of out, and the unit
// offsets uoff[h][u] = r_u (uoff[h][C] = the count) give each nonempty block
// exactly that one row.  One workgroup per (block, head).
__global__ __launch_bounds__(256) void k_compact_rows(const float* __restrict__ x,
                                                      const int* __restrict__ sizes, int C, int D,
                                                      float* __restrict__ out,
                                                      int* __restrict__ uoff) {
  __shared__ int red[4];
  const int h = blockIdx.y, u = blockIdx.x, tid = threadIdx.x;
  const int* sz = sizes + (size_t)h * C;
  int cnt = 0;
  for (int w = tid; w < u; w += 256) cnt += sz[w] > 0 ? 1 : 0;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o);
  if ((tid & 63) == 0) red[tid >> 6] = cnt;
  __syncthreads();
  const int r = red[0] + red[1] + red[2] + red[3];
  const bool keep = sz[u] > 0;
  if (tid == 0) {
    uoff[(size_t)h * (C + 1) + u] = r;
    if (u == C - 1) uoff[(size_t)h * (C + 1) + C] = r + (keep ? 1 : 0);
  }
  if (keep)
    for (int a = tid; a < D; a += 256)
      out[((size_t)h * C + r) * D + a] = x[((size_t)h * C + u) * D + a];
}

park_status launch_compact_rows(const float* x, const int* sizes, int H, int C, int D, float* out,
                                int* uoff, hipStream_t st) {
  PARK_LAUNCH("compact_rows", k_compact_rows, dim3(C, H), dim3(256), 0, st, x, sizes, C, D, out,
              uoff);
  return PARK_OK;
}

}  // namespace park
