// Graph diffusion (Sec. 3.3, Eq. 8): g_{t+1} = A (g_t / ||g_t||_2), each
// channel normalised by its own norm.  Since the normalisation is a
// per-channel scale, step t computes y = s_t * (A g_t) with
// s_t = 1 / ||g_t|| (0 for a zero channel) and, in the same pass, the squared
// norms of y for step t+1.  CSR SpMM in three forms: spmm_rows_kernel for up to 4
// channels (a row per lane, edges staged in LDS), spmm_wide_kernel for 8, 16, 32
// and 64 (a few lanes per row, each with a piece of it), spmm_kernel for the rest
// (a group of C lanes per row, lane c on channels c, c + C, ...).
#include <algorithm>

#include "lv_internal.h"

namespace lv {

namespace {

constexpr int kNormSlots = 64;

template <lv_dtype DT>
__device__ __forceinline__ float ld(const void* p, int64_t i) {
  if constexpr (DT == LV_F32) return static_cast<const float*>(p)[i];
  else return __uint_as_float((uint32_t) static_cast<const uint16_t*>(p)[i] << 16);
}

template <lv_dtype DT>
__device__ __forceinline__ void st(void* p, int64_t i, float x) {
  if constexpr (DT == LV_F32) {
    static_cast<float*>(p)[i] = x;
  } else {
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    static_cast<uint16_t*>(p)[i] = (uint16_t)(u >> 16);
  }
}

// Squared norms are accumulated in `slots` copies of a [D] row, block b adding
// to copy b mod slots, and a step sums the copies of the norms it divides by.
// Atomics on one address complete one after the other, about 15 ns each, so
// the thousands of blocks of a step that add to the same words are held up by
// them: on a million rows of 13.6 edges a D = 64 BF16 step took 248 us with
// one copy and 202 with 64, the column norms of a D = 1 signal 59 us and 16.
// Wide rows spread over addresses by themselves; their copies are cut so that
// a block's sum of them stays at 16 KB of reads.
inline int norm_slots(int D) {
  int s = kNormSlots;
  while (s > 1 && (int64_t)s * D > 4096) s >>= 1;
  return s;
}

// The norms of the last steps: step t divides by row t mod kNormRows and adds to
// the next one; half of the rows are cleared at a time, before the first of them
// is added to again, while the row that is read lies in the other half.
constexpr int kNormRows = 64;

// Sum over the slots of channel ch, the same in every block (a fixed order);
// threads t, t + C, ... of the block's 256 hold the same channel, C a power of
// two up to 64.  A thread loads T of its 64 C / 256 slots at a time: one after
// the other they were most of a small step (500 rows, D = 64 in FP32: 10.4 us,
// 7.4 with all 16 together).  red: 4 C floats of LDS.
template <int C, int T>
__device__ __forceinline__ float slot_sum(const float* __restrict__ nrm, int slots, int D, int ch,
                                          float* red) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  float v = 0.0f;
  for (int k0 = t / C; k0 < slots; k0 += T * (256 / C)) {
    float x[T];
#pragma unroll
    for (int u = 0; u < T; u++) {
      const int k = k0 + u * (256 / C);
      x[u] = ch < D && k < slots ? nrm[(int64_t)k * D + ch] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < T; u++) v += x[u];
  }
#pragma unroll
  for (int off = C; off < 64; off <<= 1) v += __shfl_xor(v, off, 64);
  if (lane < C) red[w * C + lane] = v;
  __syncthreads();
  const int c = t & (C - 1);
  const float r = (red[c] + red[C + c]) + (red[2 * C + c] + red[3 * C + c]);
  __syncthreads();
  return r;
}

// Squared column norms of g [n][D], D <= 64, into the slots of nrm
// (pre-zeroed): 256 / D rows at a time per block, consecutive threads on
// consecutive elements.
template <lv_dtype DT>
__global__ __launch_bounds__(256) void colnorm_flat_kernel(const void* __restrict__ g, int64_t n, int D,
                                                           int slots, float* __restrict__ nrm) {
  __shared__ float part[256];
  const int t = threadIdx.x, rows = 256 / D;
  const int64_t step = (int64_t)gridDim.x * rows;
  float s = 0.0f;
  if (t < rows * D) {
    const int c = t % D;
#pragma unroll 4
    for (int64_t r = (int64_t)blockIdx.x * rows + t / D; r < n; r += step) {
      const float x = ld<DT>(g, r * D + c);
      s = __builtin_fmaf(x, x, s);
    }
  }
  part[t] = s;
  __syncthreads();
  if (t < D) {
    float a = 0.0f;
    for (int q = t; q < rows * D; q += D) a += part[q];
    if (a != 0.0f) atomicAdd(&nrm[(int64_t)(blockIdx.x % (unsigned)slots) * D + t], a);
  }
}

// The same for any D, 64 channels per grid row.
template <lv_dtype DT>
__global__ __launch_bounds__(256) void colnorm_kernel(const void* __restrict__ g, int64_t n, int D,
                                                      int rows_per_block, int slots,
                                                      float* __restrict__ nrm) {
  __shared__ float part[4][64];
  int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int c = blockIdx.y * 64 + lane;
  int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
  int64_t r1 = r0 + rows_per_block < n ? r0 + rows_per_block : n;
  float s = 0.0f;
  if (c < D)
    for (int64_t r = r0 + w; r < r1; r += 4) {
      float x = ld<DT>(g, r * D + c);
      s = __builtin_fmaf(x, x, s);
    }
  part[w][lane] = s;
  __syncthreads();
  if (w == 0 && c < D)
    atomicAdd(&nrm[(int64_t)(blockIdx.x % (unsigned)slots) * D + c], (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]));
}

// One group of C lanes per row (R = 64 / C rows per wave, 4 waves per
// block); blocks stride over the row tiles, so each block issues one atomic
// per channel for the norms of the next step instead of one per tile.  The
// row's edges are fetched C at a time, one per lane (column index and weight
// in registers), then broadcast with shuffles, so the gathers of g do not
// wait on the index loads and several are in flight at once.
template <int C, lv_dtype GT, lv_dtype VT>
__global__ __launch_bounds__(256) void spmm_kernel(const int32_t* __restrict__ row_ptr,
                                                   const int32_t* __restrict__ col,
                                                   const void* __restrict__ val, int64_t n, int D,
                                                   const void* __restrict__ g,
                                                   const float* __restrict__ nrm_in, int slots,
                                                   void* __restrict__ y, float* __restrict__ nrm_out) {
  constexpr int R = 64 / C;                 // rows per wave
  constexpr int U = C < 8 ? C : 8;          // gathers in flight per lane
  __shared__ float sq[256];
  const int t = threadIdx.x, lane = t & 63;
  const int sub = lane / C, c = lane % C, gbase = sub * C;
  const int64_t tiles = (n + 4 * R - 1) / (4 * R);
  const int cpl = (D + C - 1) / C;          // channels per lane
  nrm_out += (int64_t)(blockIdx.x % (unsigned)slots) * D;
  for (int k = 0; k < cpl; k += 1) {
    const int ch = c + k * C;
    const int64_t chc = ch < D ? ch : 0;
    const float n2 = slot_sum<C, (C < 16 ? 2 : 4)>(nrm_in, slots, D, ch, sq);
    const float scl = n2 > 0.0f ? 1.0f / sqrtf(n2) : 0.0f;
    float ss = 0.0f;  // this lane's sum of squares of channel ch
    // Workgroups go to the 8 XCDs round-robin: XCD x (= blockIdx mod 8)
    // takes the x-th eighth of the rows, so that with rows in a locality
    // order the gathered neighbours stay in that XCD's L2.
    const int64_t xcd = blockIdx.x & 7, nloc = gridDim.x >> 3;
    const int64_t t0 = tiles * xcd / 8, t1 = tiles * (xcd + 1) / 8;
    for (int64_t tile = t0 + (blockIdx.x >> 3); tile < t1; tile += nloc) {
      const int64_t row = (tile * 4 + (t >> 6)) * R + sub;
      const bool valid = row < n;
      const bool live = valid && ch < D;
      // edges in 32 unsigned bits: a step past the last of 2^31 - 1 does not wrap
      const uint32_t a = valid ? row_ptr[row] : 0, b = valid ? row_ptr[row + 1] : 0;
      float acc = 0.0f;
      for (uint32_t e0 = a; e0 < b; e0 += C) {
        const uint32_t my = e0 + c;
        const int32_t cv = my < b ? col[my] : 0;
        const float wv = my < b ? ld<VT>(val, my) : 0.0f;
        const int cnt = b - e0 < C ? (int)(b - e0) : C;
        for (int j = 0; j < cnt; j += U) {
          // U gathers in flight; slots past the row's end read column 0 of a
          // valid row with weight 0 (lanes past the end hold col 0, w 0)
          float x[U], w[U];
#pragma unroll
          for (int u = 0; u < U; u++) {
            const int src = gbase + ((j + u) < C ? (j + u) : 0);
            const int32_t cj = __shfl(cv, src, 64);
            const float wj = __shfl(wv, src, 64);
            w[u] = (j + u) < cnt ? wj : 0.0f;
            x[u] = ld<GT>(g, (int64_t)cj * D + chc);
          }
#pragma unroll
          for (int u = 0; u < U; u++) acc = __builtin_fmaf(w[u], x[u], acc);
        }
      }
      if (live) {
        float out = scl * acc;
        st<GT>(y, row * D + ch, out);
        if constexpr (GT == LV_BF16) out = ld<GT>(y, row * D + ch);  // norm of what is stored
        ss = __builtin_fmaf(out, out, ss);
      }
    }
    // per-channel sum over the block: threads t, t + C, ... hold the same
    // channel (64 is a multiple of C)
    sq[t] = ss;
    __syncthreads();
    if (t < C) {
      float acc2 = 0.0f;
      for (int q = t; q < 256; q += C) acc2 += sq[q];
      const int chn = t + k * C;
      if (chn < D && acc2 != 0.0f) atomicAdd(&nrm_out[chn], acc2);
    }
    __syncthreads();
  }
}

// The value a signal element holds once stored (BF16 storage rounds).
template <lv_dtype DT>
__device__ __forceinline__ float stored(float x) {
  if constexpr (DT == LV_F32) {
    return x;
  } else {
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return __uint_as_float(u & 0xFFFF0000u);
  }
}

// Few channels (D = ND, at most 4): one row per lane, RW consecutive rows per
// wave, whose edges are one contiguous range.  The wave takes that range 64 U
// edges at a time, one edge per lane and load: columns and weights are read
// coalesced, U gathers are in flight per lane, and the weights and gathered
// values go to LDS, where each lane then sums its own row's part in edge order
// with the same fused multiply-adds as spmm_kernel.  With each lane walking its
// row in global memory instead (8 edges at a time) every load touched one line
// per lane.  A D = 1 FP32 step on a million rows: 50 -> 27 us with 13.6 edges a
// row (121 MB: the rate of a large copy, 4.5 TB/s), 132 -> 41 us with 22.6.
// RW = 64 (a round of edges per 28 rows of 18) where there are rows enough; a
// small graph's step lasts as long as one wave's chain of rounds, and 16 rows
// are one round (see spmm_rows_launch).
template <int ND, int RW, lv_dtype GT, lv_dtype VT>
__global__ __launch_bounds__(256) void spmm_rows_kernel(const int32_t* __restrict__ row_ptr,
                                                        const int32_t* __restrict__ col,
                                                        const void* __restrict__ val, int64_t n,
                                                        const void* __restrict__ g,
                                                        const float* __restrict__ nrm_in, int slots,
                                                        void* __restrict__ y, float* __restrict__ nrm_out) {
  constexpr int U = 8, E = 64 * U;  // edges per round of a wave
  __shared__ float stage[4][ND + 1][E];
  __shared__ float sq[4 * 4];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  float scl[ND], ss[ND];
#pragma unroll
  for (int k = 0; k < ND; k++) {
    const float n2 = slot_sum<1, 1>(nrm_in, slots, ND, k, sq);
    scl[k] = n2 > 0.0f ? 1.0f / sqrtf(n2) : 0.0f;
    ss[k] = 0.0f;
  }
  float(*st_)[E] = stage[wv];
  // XCD x (= blockIdx mod 8) takes the x-th eighth of the rows (locality order)
  const int64_t tiles = (n + 4 * RW - 1) / (4 * RW);
  const int64_t xcd = blockIdx.x & 7, nloc = gridDim.x >> 3;
  const int64_t t0 = tiles * xcd / 8, t1 = tiles * (xcd + 1) / 8;
  for (int64_t tile = t0 + (blockIdx.x >> 3); tile < t1; tile += nloc) {
    const int64_t row0 = (tile * 4 + wv) * RW, row = row0 + (lane < RW ? lane : RW);
    if (row0 >= n) continue;  // wave-uniform
    // edges in 32 unsigned bits: a round past the last of 2^31 - 1 does not wrap;
    // lanes past the wave's rows have none
    const uint32_t a = row_ptr[row < n ? row : n], b = row_ptr[row < n ? (lane < RW ? row + 1 : row) : n];
    const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)a, 0);
    const uint32_t last = (uint32_t)__builtin_amdgcn_readlane((int)b, RW - 1);
    float acc[ND] = {};
    for (uint32_t base = first; base < last; base += E) {
      int32_t cj[U];
      float w[U], x[U][ND];
#pragma unroll
      for (int u = 0; u < U; u++) {
        const uint32_t e = base + 64 * u + lane;
        const bool ok = e < last;
        cj[u] = ok ? col[e] : 0;
        w[u] = ok ? ld<VT>(val, e) : 0.0f;
      }
#pragma unroll
      for (int u = 0; u < U; u++)
#pragma unroll
        for (int k = 0; k < ND; k++) x[u][k] = ld<GT>(g, (int64_t)cj[u] * ND + k);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the last round's sums have read the stage
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int u = 0; u < U; u++) {
        st_[ND][64 * u + lane] = w[u];
#pragma unroll
        for (int k = 0; k < ND; k++) st_[k][64 * u + lane] = x[u][k];
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const int e0 = (int)((a > base ? a : base) - base);
      const int e1 = (int)(b < base + E ? b - base : E);  // negative where the row ends before the round
      for (int e = e0; e < e1; e++) {
        const float we = st_[ND][e];
#pragma unroll
        for (int k = 0; k < ND; k++) acc[k] = __builtin_fmaf(we, st_[k][e], acc[k]);
      }
    }
    if (lane < RW && row < n) {
#pragma unroll
      for (int k = 0; k < ND; k++) {
        const float o = stored<GT>(scl[k] * acc[k]);  // the norm of what is stored
        st<GT>(y, row * ND + k, o);
        ss[k] = __builtin_fmaf(o, o, ss[k]);
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < ND; k++) {
    for (int off = 32; off > 0; off >>= 1) ss[k] += __shfl_xor(ss[k], off, 64);
    if (lane == 0) sq[k * 4 + wv] = ss[k];
  }
  __syncthreads();
  if (t < ND) {
    const float v = (sq[4 * t] + sq[4 * t + 1]) + (sq[4 * t + 2] + sq[4 * t + 3]);
    if (v != 0.0f) atomicAdd(&nrm_out[(int64_t)(blockIdx.x % (unsigned)slots) * ND + t], v);
  }
}

// Edges that a wave of spmm_wide_kernel stages in a round.
template <int D, int C>
constexpr int spmm_wide_edges() {
  return 64 * C / D > 32 ? 16 * (64 * C / D) : 512;
}

// D = 8, 16, 32 or 64 channels in rows of pieces of C channels, one load each (4
// channels in FP32, 8 in BF16: 16 bytes; 4 in small graphs), one piece per lane,
// L = D / C lanes per row, R = 64 / L consecutive rows per wave, whose edges are
// one contiguous range.  The wave takes that range E edges at a time: columns and
// weights are read coalesced and left in LDS as (row offset, weight); each row's
// lanes then walk the row's part, U gathers in flight, and sum in edge order with
// the same fused multiply-adds as spmm_kernel.
// What bounds a step is instructions and latency before bandwidth: with four
// channels per lane, edges broadcast by shuffles and a block per 16 rows, each
// gather cost a BF16 lane 13 instructions for 4 channels (now about 18 for 8), and
// every block began with the norms, the row pointers and the edges one after the
// other.  The blocks now stay (spmm_wide_blocks), and a tile's edges and the next
// one's row pointers are loaded while the tile before is summed.  U = 4: of 4, 6,
// 8 and 12 gathers in flight 4 is the fastest or level everywhere (D = 64 in
// FP32, 1M rows: 252, 269, 272, 303 us a step).  Steps, 16 edges a row, before and
// now: 1M rows, D = 64, BF16 207 -> 144 us (338 MB: 2.3 TB/s), FP32 260 -> 252;
// 300k rows, D = 32, BF16 50 -> 29, D = 16 30 -> 21, D = 8 28 -> 17.  In a graph
// so small that no block takes a second tile (see spmm_wide_launch) a step lasts
// as long as one wave's chain: there U = 8, and four channels per lane also in
// BF16, twice as many waves.
// kBig: offsets of g do not fit 32 bits (else they are formed when staged, and a
// gather is one addition and one load).
template <int D, int C, int U, lv_dtype GT, lv_dtype VT, bool kBig>
__global__ __launch_bounds__(256) void spmm_wide_kernel(const int32_t* __restrict__ row_ptr,
                                                        const int32_t* __restrict__ col,
                                                        const void* __restrict__ val, int64_t n,
                                                        const void* __restrict__ g,
                                                        const float* __restrict__ nrm_in, int slots,
                                                        void* __restrict__ y, float* __restrict__ nrm_out) {
  constexpr int L = D / C, R = 64 / L;
  constexpr int kPiece = C * (GT == LV_F32 ? 4 : 2), kWords = kPiece / 4;  // bytes and words of a lane's piece of a row
  typedef uint32_t piece_t __attribute__((ext_vector_type(kWords)));
  constexpr int E = spmm_wide_edges<D, C>(), P = R < 32 ? 4 : 8;  // edges per round, per lane and load
  constexpr uint32_t kRowBytes = D * (GT == LV_F32 ? 4 : 2);
  __shared__ union {
    uint2 edge[4][E];
    float sq[256 * C];
  } sh;
  __shared__ float scales[D];
  const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int sub = lane / L, cl = lane % L;
  uint2* const edge = sh.edge[wv];
  const char* const gb = static_cast<const char*>(g);
  // a gathered row's piece of this lane
  const auto gather = [&](uint32_t off) {
    if constexpr (kBig)
      return *reinterpret_cast<const piece_t*>(gb + (uint64_t)off * kRowBytes + kPiece * cl);
    else
      return *reinterpret_cast<const piece_t*>(gb + (off + (uint32_t)(kPiece * cl)));
  };
  const auto add = [&](float (&acc)[C], float w, const piece_t& r) {
#pragma unroll
    for (int k = 0; k < kWords; k++) {
      if constexpr (GT == LV_F32) {
        acc[k] = __builtin_fmaf(w, __uint_as_float(r[k]), acc[k]);
      } else {
        acc[2 * k] = __builtin_fmaf(w, __uint_as_float(r[k] << 16), acc[2 * k]);
        acc[2 * k + 1] = __builtin_fmaf(w, __uint_as_float(r[k] & 0xFFFF0000u), acc[2 * k + 1]);
      }
    }
  };
  // XCD x (= blockIdx mod 8) takes the x-th eighth of the rows (locality order)
  const int64_t tiles = (n + 4 * R - 1) / (4 * R);
  const int64_t xcd = blockIdx.x & 7, nloc = gridDim.x >> 3;
  const int64_t t0 = tiles * xcd / 8, t1 = tiles * (xcd + 1) / 8;
  // this lane's row of a tile (its edges [a, b)), and 64 P edges of a wave
  const auto load_rows = [&](int64_t tile, int32_t& a, int32_t& b) {
    const int64_t row = (tile * 4 + wv) * R + sub;
    a = row_ptr[tile < t1 && row < n ? row : n];
    b = row_ptr[tile < t1 && row < n ? row + 1 : n];
  };
  uint32_t cj[P];
  float w[P];
  const auto load_edges = [&](int32_t e0, int32_t m) {  // m > 0 edges from e0; past them the last again
#pragma unroll
    for (int u = 0; u < P; u++) {
      const int32_t q = 64 * u + lane;
      const int32_t e = e0 + (q < m ? q : m - 1);
      cj[u] = (uint32_t)col[e];
      w[u] = ld<VT>(val, e);
    }
  };
  int64_t tile = t0 + (blockIdx.x >> 3);
  int32_t a, b, an, bn;  // this tile's row and the next's
  load_rows(tile, a, b);
  load_rows(tile + nloc, an, bn);
  int32_t first = __builtin_amdgcn_readlane(a, 0), last = __builtin_amdgcn_readlane(b, 63);
  if (first < last) load_edges(first, last - first);
  {
    const float n2 = slot_sum<D, D / 4>(nrm_in, slots, D, t & (D - 1), sh.sq);
    if (t < D) scales[t] = n2 > 0.0f ? 1.0f / sqrtf(n2) : 0.0f;
    __syncthreads();
  }
  float ss[C] = {};
  for (; tile < t1; tile += nloc) {
    const int64_t row = (tile * 4 + wv) * R + sub;
    float acc[C] = {};
    int32_t base = first;
    do {
      const int32_t m = last - base < E ? last - base : E;  // edges of this round
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the last round's are read
      __builtin_amdgcn_wave_barrier();
      for (int32_t q0 = 0; q0 < m; q0 += 64 * P) {
        if (base + q0 > first) load_edges(base + q0, m - q0);
#pragma unroll
        for (int u = 0; u < P; u++)
          edge[q0 + 64 * u + lane] = make_uint2(kBig ? cj[u] : cj[u] * kRowBytes, __float_as_uint(w[u]));
      }
      if (base + m == last) {  // the next tile's first edges
        const int32_t e0 = __builtin_amdgcn_readlane(an, 0), e1 = __builtin_amdgcn_readlane(bn, 63);
        if (e0 < e1) load_edges(e0, e1 - e0);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      int32_t j = a > base ? a - base : 0;
      const int32_t j1 = b - base < m ? b - base : m;
      for (; j + U <= j1; j += U) {
        uint2 ed[U];
        piece_t x[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
          ed[u] = edge[j + u];
          x[u] = gather(ed[u].x);
        }
#pragma unroll
        for (int u = 0; u < U; u++) add(acc, __uint_as_float(ed[u].y), x[u]);
      }
      if (j < j1) {  // fewer than U left: the last edge's row again, taken as zeros
        uint2 ed[U];
        piece_t x[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
          ed[u] = edge[j + u < j1 ? j + u : j1 - 1];
          x[u] = gather(ed[u].x);
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
          const bool ok = j + u < j1;
          piece_t z;
#pragma unroll
          for (int k = 0; k < kWords; k++) z[k] = ok ? x[u][k] : 0u;
          add(acc, ok ? __uint_as_float(ed[u].y) : 0.0f, z);
        }
      }
      base += m;
    } while (base < last);
    a = an;
    b = bn;
    first = __builtin_amdgcn_readlane(a, 0);
    last = __builtin_amdgcn_readlane(b, 63);
    load_rows(tile + 2 * nloc, an, bn);
    if (row < n) {
      float o[C];
#pragma unroll
      for (int k = 0; k < C; k++) {
        o[k] = stored<GT>(scales[C * cl + k] * acc[k]);  // the norm of what is stored
        ss[k] = __builtin_fmaf(o[k], o[k], ss[k]);
      }
      piece_t q;
#pragma unroll
      for (int k = 0; k < kWords; k++) {
        if constexpr (GT == LV_F32)
          q[k] = __float_as_uint(o[k]);
        else
          q[k] = (__float_as_uint(o[2 * k]) >> 16) | __float_as_uint(o[2 * k + 1]);
      }
      *reinterpret_cast<piece_t*>(static_cast<char*>(y) + row * (int64_t)kRowBytes + kPiece * cl) = q;
    }
  }
  // per-channel sums over the block: threads t = cl (mod L) hold channels C cl ..
  // C cl + C - 1.  Where many threads share a channel (L <= 4) the lanes of a wave
  // are summed by shuffles first: 128 LDS reads in a row by few threads took 3 us
  // of a 13 us step on 5,000 rows (D = 16).
  constexpr bool kShfl = L <= 4;
  if constexpr (kShfl) {
#pragma unroll
    for (int k = 0; k < C; k++)
#pragma unroll
      for (int off = L; off < 64; off <<= 1) ss[k] += __shfl_xor(ss[k], off, 64);
  }
  __syncthreads();  // the edges are read
#pragma unroll
  for (int k = 0; k < C; k++) sh.sq[k * 256 + t] = ss[k];
  __syncthreads();
  if (t < D) {
    const int k = t % C, cc = t / C;
    float s2 = 0.0f;
    for (int q = cc; q < 256; q += kShfl ? 64 : L) s2 += sh.sq[k * 256 + q];
    if (s2 != 0.0f) atomicAdd(&nrm_out[(int64_t)(blockIdx.x % (unsigned)slots) * D + t], s2);
  }
}

template <lv_dtype GT>
__global__ void copy_kernel(const void* __restrict__ src, void* __restrict__ dst, int64_t total) {
  int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < total) st<GT>(dst, e, ld<GT>(src, e));
}

template <int C, lv_dtype GT, lv_dtype VT>
hipError_t spmm_launch(const int32_t* rp, const int32_t* col, const void* val, int64_t n, int D,
                       const void* g, const float* nin, int slots, void* y, float* nout, hipStream_t s) {
  constexpr int R = 64 / C;
  const int64_t rows_per_tile = 4 * R;
  const int64_t tiles = (n + rows_per_tile - 1) / rows_per_tile;
  // enough blocks to fill the chip several times over (a multiple of 8, one
  // share per XCD); each strides over the tiles of its XCD's share
  const int64_t want = (tiles + 7) / 8 * 8;
  const unsigned blocks = (unsigned)(want < 8192 ? want : 8192);
  hipLaunchKernelGGL((spmm_kernel<C, GT, VT>), dim3(blocks), dim3(256), 0, s, rp, col, val, n, D, g,
                     nin, slots, y, nout);
  return hipGetLastError();
}

// Five blocks per CU, all resident, sweep the rows in order: 1024, 1280, 1536 and
// 2048 blocks take 162, 144, 138 and 172 us a step (1M rows, D = 64, 16 edges a
// row, BF16) and 262, 252, 260 and 293 in FP32.  Where the staged edges leave room
// for four (D = 8 in BF16), four: 1M rows 50.2 us, 61.0 with a fifth in a round of
// its own.
template <int D, int C>
constexpr int64_t spmm_wide_blocks() {
  constexpr int lds = std::max(4 * 8 * spmm_wide_edges<D, C>(), 4 * 256 * C) + 4 * D;
  return 256 * std::min(5, 160 * 1024 / lds);
}

// Up to this many tiles the small form of spmm_wide_kernel runs (C = 4, U = 8).
// Steps of 18 edges a row, small / large form: D = 64, 5,000 rows (313 tiles) FP32
// 7.2 / 7.6 us, BF16 7.2 / 8.8; 15,000 rows (938) 9.3 / 9.0 and 9.1 / 9.5; 50,000
// rows (3125) 17.4 / 16.9 and 17.2 / 14.0; D = 8, 50,000 rows (391) 9.2 / 9.3 and
// 9.2 / 10.3; 300,000 rows (2344) 28.8 / 26.0 and 26.0 / 25.3.
constexpr int64_t kFewTiles = 1024;

template <int D, lv_dtype GT, lv_dtype VT>
hipError_t spmm_wide_launch(const int32_t* rp, const int32_t* col, const void* val, int64_t n,
                            const void* g, const float* nin, int slots, void* y, float* nout,
                            hipStream_t s) {
  constexpr int C = GT == LV_F32 ? 4 : 8;  // channels of a 16-byte piece
  const bool few = n * D <= kFewTiles * 1024;
  const int rows = 256 * (few ? 4 : C) / D;  // per tile
  const int64_t tiles = (n + rows - 1) / rows;
  const int64_t want = (tiles + 7) / 8 * 8;
  const unsigned blocks = (unsigned)std::min(want, spmm_wide_blocks<D, C>());
  const bool big = n * D * (GT == LV_F32 ? 4 : 2) > (int64_t)1 << 32;
  hipLaunchKernelGGL((few   ? spmm_wide_kernel<D, 4, 8, GT, VT, false>
                      : big ? spmm_wide_kernel<D, C, 4, GT, VT, true>
                            : spmm_wide_kernel<D, C, 4, GT, VT, false>),
                     dim3(blocks), dim3(256), 0, s, rp, col, val, n, g, nin, slots, y, nout);
  return hipGetLastError();
}

// The fewest rows per wave, 16, 32 or 64, that need at most 2048 waves (two per
// SIMD), else 64.  D = 1 in FP32, 18 edges a row, a step of 16 / 32 / 64 rows per
// wave: 5,000 rows 6.9 / 8.7 / 10.9 us, 15,000 7.6 / 8.7 / 11.0, 50,000 11.1 / 10.3
// / 11.3, 120,000 18.4 / 13.9 / 13.1; D = 4, 15,000 8.7 / 11.2 / 13.7, 50,000 15.6 /
// 12.0 / 13.7, 120,000 23.2 / 21.2 / 15.5.
template <int ND, lv_dtype GT, lv_dtype VT>
hipError_t spmm_rows_launch(const int32_t* rp, const int32_t* col, const void* val, int64_t n,
                            const void* g, const float* nin, int slots, void* y, float* nout,
                            hipStream_t s) {
  const int rows = n <= 16 * 2048 ? 16 : n <= 32 * 2048 ? 32 : 64;
  const int64_t tiles = (n + 4 * rows - 1) / (4 * rows);
  const int64_t want = (tiles + 7) / 8 * 8;
  const unsigned blocks = (unsigned)(want < 8192 ? want : 8192);
  hipLaunchKernelGGL((rows == 16   ? spmm_rows_kernel<ND, 16, GT, VT>
                      : rows == 32 ? spmm_rows_kernel<ND, 32, GT, VT>
                                   : spmm_rows_kernel<ND, 64, GT, VT>),
                     dim3(blocks), dim3(256), 0, s, rp, col, val, n, g, nin, slots, y, nout);
  return hipGetLastError();
}

template <lv_dtype GT, lv_dtype VT>
hipError_t spmm_dispatch(const int32_t* rp, const int32_t* col, const void* val, int64_t n, int D,
                         const void* g, const float* nin, int slots, void* y, float* nout,
                         hipStream_t s) {
  if (D == 1) return spmm_rows_launch<1, GT, VT>(rp, col, val, n, g, nin, slots, y, nout, s);
  if (D == 2) return spmm_rows_launch<2, GT, VT>(rp, col, val, n, g, nin, slots, y, nout, s);
  if (D == 3) return spmm_rows_launch<3, GT, VT>(rp, col, val, n, g, nin, slots, y, nout, s);
  if (D == 4) return spmm_rows_launch<4, GT, VT>(rp, col, val, n, g, nin, slots, y, nout, s);
  // 16-byte pieces of rows where the arrays are aligned to them
  if (((uintptr_t)g % 16 == 0) && ((uintptr_t)y % 16 == 0)) {
    if (D == 64) return spmm_wide_launch<64, GT, VT>(rp, col, val, n, g, nin, slots, y, nout, s);
    if (D == 32) return spmm_wide_launch<32, GT, VT>(rp, col, val, n, g, nin, slots, y, nout, s);
    if (D == 16) return spmm_wide_launch<16, GT, VT>(rp, col, val, n, g, nin, slots, y, nout, s);
    if (D == 8) return spmm_wide_launch<8, GT, VT>(rp, col, val, n, g, nin, slots, y, nout, s);
  }
  if (D >= 64) return spmm_launch<64, GT, VT>(rp, col, val, n, D, g, nin, slots, y, nout, s);
  if (D > 16) return spmm_launch<32, GT, VT>(rp, col, val, n, D, g, nin, slots, y, nout, s);
  return spmm_launch<8, GT, VT>(rp, col, val, n, D, g, nin, slots, y, nout, s);
}

template <lv_dtype GT>
hipError_t diffuse_t(const int32_t* rp, const int32_t* col, const void* val, lv_dtype vt, int64_t n,
                     const void* g0, int D, int steps, void* out, void* b0, void* b1, float* norms,
                     hipStream_t s) {
  int64_t total = n * (int64_t)D;
  if (steps == 0) {
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(copy_kernel<GT>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, g0,
                       out, total);
    return hipGetLastError();
  }
  const int slots = norm_slots(D);
  const size_t row = (size_t)D * slots;  // the norms of one step
  hipError_t e = hipMemsetAsync(norms, 0, sizeof(float) * diffuse_norm_floats(D, steps), s);
  if (e != hipSuccess) return e;
  if (total == 0) return hipSuccess;
  if (D <= 64) {
    const int64_t want = (n + 256 / D - 1) / (256 / D);
    hipLaunchKernelGGL(colnorm_flat_kernel<GT>, dim3((unsigned)(want < 1024 ? want : 1024)), dim3(256), 0,
                       s, g0, n, D, slots, norms);
  } else {
    const int rows = 256;
    hipLaunchKernelGGL(colnorm_kernel<GT>, dim3((unsigned)((n + rows - 1) / rows), (D + 63) / 64),
                       dim3(256), 0, s, g0, n, D, rows, slots, norms);
  }
  const void* cur = g0;
  for (int t = 0; t < steps; t++) {
    void* dst = (t == steps - 1) ? out : ((t & 1) ? b1 : b0);
    const float* const nin = norms + t % kNormRows * row;
    float* const nout = norms + (t + 1) % kNormRows * row;
    if (t + 1 >= kNormRows && (t + 1) % (kNormRows / 2) == 0) {
      e = hipMemsetAsync(nout, 0, sizeof(float) * row * (kNormRows / 2), s);
      if (e != hipSuccess) return e;
    }
    e = vt == LV_F32 ? spmm_dispatch<GT, LV_F32>(rp, col, val, n, D, cur, nin, slots, dst, nout, s)
                     : spmm_dispatch<GT, LV_BF16>(rp, col, val, n, D, cur, nin, slots, dst, nout, s);
    if (e != hipSuccess) return e;
    cur = dst;
  }
  return hipSuccess;
}

// ------------------------------------------------------- locality order
// Rows of A are renumbered along a Morton (Z-order) curve of the Gaussian
// centres, so that the neighbours of a row sit close in memory and the
// gathers of g hit the caches.  The renumbering is a similarity transform
// P A P^T: Eq. 8 commutes with it, and the per-channel norms are invariant.

// Order-preserving map of a float to uint32 (for atomic min / max).
__device__ __forceinline__ uint32_t ordered(float x) {
  const uint32_t u = __float_as_uint(x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float unordered(uint32_t u) {
  return __uint_as_float((u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u);
}

__global__ void box_init_kernel(uint32_t* box) {
  if (threadIdx.x < 3) box[threadIdx.x] = 0xFFFFFFFFu;
  else if (threadIdx.x < 6) box[threadIdx.x] = 0u;
}

__global__ __launch_bounds__(256) void box_kernel(const float4* __restrict__ p0, int64_t n,
                                                  uint32_t* __restrict__ box) {
  uint32_t lo[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, hi[3] = {0u, 0u, 0u};
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float4 a = p0[i];
    const float v[3] = {a.x, a.y, a.z};
#pragma unroll
    for (int k = 0; k < 3; k++) {
      const uint32_t o = ordered(v[k]);
      lo[k] = o < lo[k] ? o : lo[k];
      hi[k] = o > hi[k] ? o : hi[k];
    }
  }
#pragma unroll
  for (int k = 0; k < 3; k++) {
    for (int off = 32; off > 0; off >>= 1) {
      const uint32_t l = __shfl_xor(lo[k], off, 64), h = __shfl_xor(hi[k], off, 64);
      lo[k] = l < lo[k] ? l : lo[k];
      hi[k] = h > hi[k] ? h : hi[k];
    }
  }
  // the block's four waves through LDS, then one atomic per bound and block
  // (few blocks: the six words would serialise thousands of wave atomics)
  __shared__ uint32_t wb[4][6];
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int k = 0; k < 3; k++) {
      wb[w][k] = lo[k];
      wb[w][3 + k] = hi[k];
    }
  }
  __syncthreads();
  if (threadIdx.x < 6) {
    const int k = threadIdx.x;
    uint32_t r = wb[0][k];
    for (int q = 1; q < (int)(blockDim.x >> 6); q++) r = k < 3 ? (wb[q][k] < r ? wb[q][k] : r) : (wb[q][k] > r ? wb[q][k] : r);
    if (k < 3) atomicMin(&box[k], r);
    else atomicMax(&box[k], r);
  }
}

__device__ __forceinline__ uint32_t spread10(uint32_t x) {  // bit i -> bit 3i
  x &= 0x3FFu;
  x = (x | (x << 16)) & 0x030000FFu;
  x = (x | (x << 8)) & 0x0300F00Fu;
  x = (x | (x << 4)) & 0x030C30C3u;
  x = (x | (x << 2)) & 0x09249249u;
  return x;
}

__global__ void morton_kernel(const float4* __restrict__ p0, int64_t n,
                              const uint32_t* __restrict__ box, uint32_t* __restrict__ key,
                              uint32_t* __restrict__ val, uint32_t* __restrict__ deg,
                              const int32_t* __restrict__ row_ptr) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float4 a = p0[i];
  const float v[3] = {a.x, a.y, a.z};
  uint32_t code = 0;
#pragma unroll
  for (int k = 0; k < 3; k++) {
    const float lo = unordered(box[k]), hi = unordered(box[3 + k]);
    const float ext = hi - lo;
    float q = ext > 0.0f ? (v[k] - lo) / ext * 1024.0f : 0.0f;
    q = fminf(fmaxf(q, 0.0f), 1023.0f);
    code |= spread10((uint32_t)q) << k;
  }
  key[i] = code;
  val[i] = (uint32_t)i;
  if (row_ptr) deg[i] = (uint32_t)(row_ptr[i + 1] - row_ptr[i]);
}

// One sort segment covering all n items.
__global__ void seg_init_kernel(uint32_t* seg, int64_t n) {
  if (threadIdx.x == 0) {
    seg[0] = 0u;
    seg[1] = (uint32_t)n;
  }
}

// perm[r] = old index of new row r; inv[perm[r]] = r.
__global__ void invert_kernel(const uint32_t* __restrict__ perm, int64_t n, uint32_t* __restrict__ inv) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r < n) inv[perm[r]] = (uint32_t)r;
}

// New row r = old row perm[r], its columns renumbered; off[r] = new row start.
// 16 lanes per row (one lane per row, its accesses a row apart from the next
// lane's, took 1200 us for 1M rows of 23 edges, 16 lanes 161); a launch takes the
// rows from `first` on, as many as its grid has (fewer than 2^32 threads).
template <typename VT>
__global__ __launch_bounds__(256) void permute_csr_kernel(
    const int32_t* __restrict__ rp, const int32_t* __restrict__ col, const VT* __restrict__ val,
    const uint32_t* __restrict__ perm, const uint32_t* __restrict__ inv, const uint32_t* __restrict__ off,
    int64_t first, int64_t n, int64_t nnz, int32_t* __restrict__ rp2, int32_t* __restrict__ col2,
    VT* __restrict__ val2) {
  const int64_t r = first + (((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 4);
  const int sub = threadIdx.x & 15;
  if (r > n) return;
  if (r == n) {
    if (sub == 0) rp2[n] = (int32_t)nnz;
    return;
  }
  const int64_t o = perm[r];
  const uint32_t a = rp[o], b = rp[o + 1];  // unsigned: a step past 2^31 - 1 does not wrap
  const int64_t d = off[r];
  if (sub == 0) rp2[r] = (int32_t)d;
  for (uint32_t e = a + sub; e < b; e += 16) {
    col2[d + (e - a)] = (int32_t)inv[col[e]];
    val2[d + (e - a)] = val[e];
  }
}

// Row gather / scatter of an [n][D] signal of `esize`-byte elements:
// dst[r] = src[perm[r]] (gather) or dst[perm[r]] = src[r] (scatter).
template <typename T>
__global__ void permute_rows_kernel(const T* __restrict__ src, T* __restrict__ dst,
                                    const uint32_t* __restrict__ perm, int64_t n, int D,
                                    bool scatter) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * (int64_t)D) return;
  const int64_t r = e / D, c = e - r * D;
  const int64_t o = perm[r];
  if (scatter) dst[o * D + c] = src[e];
  else dst[e] = src[o * D + c];
}

}  // namespace

size_t diffuse_norm_floats(int D, int steps) {
  return (size_t)D * norm_slots(D) * (size_t)(steps < kNormRows ? steps + 1 : kNormRows);
}

hipError_t launch_diffuse(const int32_t* row_ptr, const int32_t* col, const void* val,
                          lv_dtype val_dtype, int64_t n, const void* g0, lv_dtype dtype, int D,
                          int steps, void* out, float* buf0, float* buf1, float* norms,
                          hipStream_t s) {
  if (dtype == LV_F32)
    return diffuse_t<LV_F32>(row_ptr, col, val, val_dtype, n, g0, D, steps, out, buf0, buf1, norms, s);
  return diffuse_t<LV_BF16>(row_ptr, col, val, val_dtype, n, g0, D, steps, out, buf0, buf1, norms, s);
}

}  // namespace lv

namespace lv {

size_t reorder_scratch_words(int64_t n) {
  // keys/vals x2, degrees, offsets, box, seg start/len, totals, sort histogram, scan tmp
  return (size_t)n * 6 + 16 + sort_hist_size(1, n) + scan_tmp_size(n);
}

hipError_t launch_scene_box(const float4* p0, int64_t n, uint32_t* box, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const unsigned nb = (unsigned)((n + 255) / 256);
  hipLaunchKernelGGL(box_init_kernel, dim3(1), dim3(64), 0, s, box);
  hipLaunchKernelGGL(box_kernel, dim3(nb < 256 ? nb : 256), dim3(256), 0, s, p0, n, box);
  return hipGetLastError();
}

hipError_t launch_morton_order(const float4* p0, int64_t n, uint32_t* scratch, uint32_t* perm,
                               uint32_t* inv, hipStream_t s) {
  if (n == 0) return hipSuccess;
  uint32_t* k0 = scratch;
  uint32_t* v0 = k0 + n;
  uint32_t* k1 = v0 + n;
  uint32_t* v1 = k1 + n;
  uint32_t* box = v1 + n;  // within reorder_scratch_words(n)
  uint32_t* seg = box + 6;
  uint32_t* hist = box + 16;
  const unsigned nb = (unsigned)((n + 255) / 256);
  hipLaunchKernelGGL(box_init_kernel, dim3(1), dim3(64), 0, s, box);
  hipLaunchKernelGGL(box_kernel, dim3(nb < 256 ? nb : 256), dim3(256), 0, s, p0, n, box);
  hipLaunchKernelGGL(morton_kernel, dim3(nb), dim3(256), 0, s, p0, n, box, k0, v0, nullptr, nullptr);
  hipLaunchKernelGGL(seg_init_kernel, dim3(1), dim3(64), 0, s, seg, n);
  bool second = false;
  hipError_t e = radix_sort(k0, v0, k1, v1, seg, seg + 1, 1, n, 30, hist, false, &second, s);
  if (e != hipSuccess) return e;
  const uint32_t* sorted = second ? v1 : v0;
  hipLaunchKernelGGL(invert_kernel, dim3(nb), dim3(256), 0, s, sorted, n, inv);
  return hipMemcpyAsync(perm, sorted, 4 * (size_t)n, hipMemcpyDeviceToDevice, s);
}

hipError_t launch_graph_reorder(const float4* p0, int64_t n, const int32_t* rp, const int32_t* col,
                                const void* val, lv_dtype vt, int64_t nnz, uint32_t* scratch,
                                uint32_t* perm, uint32_t* inv, int32_t* rp2, int32_t* col2,
                                void* val2, hipStream_t s) {
  if (n == 0) return hipSuccess;
  uint32_t* k0 = scratch;
  uint32_t* v0 = k0 + n;
  uint32_t* k1 = v0 + n;
  uint32_t* v1 = k1 + n;
  uint32_t* deg = v1 + n;
  uint32_t* off = deg + n;
  uint32_t* box = off + n;          // 6 words
  uint32_t* seg = box + 6;          // start, len
  unsigned long long* totals = reinterpret_cast<unsigned long long*>(box + 8);  // 2 x u64, 8-aligned
  uint32_t* hist = box + 16;
  uint32_t* tmp = hist + sort_hist_size(1, n);
  const unsigned nb = (unsigned)((n + 255) / 256);
  hipLaunchKernelGGL(box_init_kernel, dim3(1), dim3(64), 0, s, box);
  hipLaunchKernelGGL(box_kernel, dim3(nb < 256 ? nb : 256), dim3(256), 0, s, p0, n, box);
  hipLaunchKernelGGL(morton_kernel, dim3(nb), dim3(256), 0, s, p0, n, box, k0, v0, deg, rp);
  hipLaunchKernelGGL(seg_init_kernel, dim3(1), dim3(64), 0, s, seg, n);
  bool second = false;
  hipError_t e = radix_sort(k0, v0, k1, v1, seg, seg + 1, 1, n, 30, hist, false, &second, s);
  if (e != hipSuccess) return e;
  const uint32_t* sorted = second ? v1 : v0;
  hipLaunchKernelGGL(invert_kernel, dim3(nb), dim3(256), 0, s, sorted, n, inv);
  e = hipMemcpyAsync(perm, sorted, 4 * (size_t)n, hipMemcpyDeviceToDevice, s);
  if (e != hipSuccess) return e;
  // new row starts: exclusive scan of the degrees in the new order
  uint32_t* dummy = k0;  // seg_start / seg_len outputs of the scan (one view)
  e = scan_counts(deg, perm, n, 1, off, dummy, dummy + 1, totals, tmp, s);
  if (e != hipSuccess) return e;
  const int64_t slice = (int64_t)1 << 27;  // rows of a launch
  for (int64_t first = 0; first <= n; first += slice) {
    const unsigned nr = (unsigned)((std::min(slice, n + 1 - first) + 15) / 16);  // 16 rows per block
    if (vt == LV_F32)
      hipLaunchKernelGGL(permute_csr_kernel<float>, dim3(nr), dim3(256), 0, s, rp, col,
                         static_cast<const float*>(val), perm, inv, off, first, n, nnz, rp2, col2,
                         static_cast<float*>(val2));
    else
      hipLaunchKernelGGL(permute_csr_kernel<uint16_t>, dim3(nr), dim3(256), 0, s, rp, col,
                         static_cast<const uint16_t*>(val), perm, inv, off, first, n, nnz, rp2, col2,
                         static_cast<uint16_t*>(val2));
  }
  return hipGetLastError();
}

hipError_t launch_permute_rows(const void* src, void* dst, const uint32_t* perm, int64_t n, int D,
                               lv_dtype dt, bool scatter, hipStream_t s) {
  const int64_t total = n * (int64_t)D;
  if (total == 0) return hipSuccess;
  const unsigned nb = (unsigned)((total + 255) / 256);
  if (dt == LV_F32)
    hipLaunchKernelGGL(permute_rows_kernel<uint32_t>, dim3(nb), dim3(256), 0, s,
                       static_cast<const uint32_t*>(src), static_cast<uint32_t*>(dst), perm, n, D,
                       scatter);
  else
    hipLaunchKernelGGL(permute_rows_kernel<uint16_t>, dim3(nb), dim3(256), 0, s,
                       static_cast<const uint16_t*>(src), static_cast<uint16_t*>(dst), perm, n, D,
                       scatter);
  return hipGetLastError();
}

}  // namespace lv
