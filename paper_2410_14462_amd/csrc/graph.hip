// The diffusion graph over the Gaussian centres, built on the device
// (Sec. 3.3: diffusion runs on a weighted graph joining each Gaussian to its
// spatial neighbours; the relation is symmetrised by the union of the
// directed kNN pairs).  Weight of a pair: exp(-|x_i - x_j|^2 / sigma^2) *
// max(0, cos(f_i, f_j)), sigma the median directed kNN distance, the larger
// directed weight where both exist; rows normalised to sum 1, a row whose
// weights are all 0 gets a self-loop of weight 1.
//
// Reproducible structure: squared distances in FP64 as ((dx dx + dy dy) +
// dz dz) of the FP32 centres, neighbours ordered by (squared distance,
// index); the union pairs with a positive FP64 weight are stored, columns
// ascending; a self-loop is the only entry of its row.
//
// The paper's own weights (Eq. 7 with the feature kernel of Eq. 9, the
// appendix on diffusion for segmentation) are the other kind: A_ij =
// exp(-|g_i - g_j|^2 / (b s_f^2)) (sqrt(P_i) sqrt(P_j)) with g the
// l2-normalised features, s_f the median feature distance over the directed
// kNN pairs, b a bandwidth and P a caller-given unary term (1 if absent); no
// row normalisation, no self-loops; optionally binarised (1 where the weight
// exceeds a threshold).
//
// Steps: bounding box; uniform grid, centres sorted by cell; exact kNN by
// shells of cells around each centre until the k-th distance is below the
// distance to the next shell; sigma from the two middle order statistics of
// the n k squared distances (radix select on their bits); per-node feature
// norms and per-edge weights (a few lanes per edge); union rows (own k entries
// plus the reversed edges that are not mutual, sorted by column in each row),
// row sums in column order, normalisation into the CSR.  Nodes are worked on
// at their position in cell order, where a node's neighbours are near in
// memory and in time; columns and the CSR's rows are the caller's indices.
#include "lv_internal.h"

namespace lv {

namespace {

// Centres per grid cell: 1M uniform centres, k = 16, the build and ten steps of
// diffusion take 4.22, 4.13, 4.19 ms with 1, 2 and 3.
constexpr int kCellCentres = 2;

// ---------------------------------------------------------------- grid
__global__ void bbox_partial_kernel(const float4* __restrict__ c, int64_t n, float* __restrict__ part) {
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float4 p = c[i];
    lo[0] = fminf(lo[0], p.x); hi[0] = fmaxf(hi[0], p.x);
    lo[1] = fminf(lo[1], p.y); hi[1] = fmaxf(hi[1], p.y);
    lo[2] = fminf(lo[2], p.z); hi[2] = fmaxf(hi[2], p.z);
  }
  __shared__ float red[6][256];
#pragma unroll
  for (int a = 0; a < 3; a++) {
    red[a][threadIdx.x] = lo[a];
    red[3 + a][threadIdx.x] = hi[a];
  }
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o)
#pragma unroll
      for (int a = 0; a < 3; a++) {
        red[a][threadIdx.x] = fminf(red[a][threadIdx.x], red[a][threadIdx.x + o]);
        red[3 + a][threadIdx.x] = fmaxf(red[3 + a][threadIdx.x], red[3 + a][threadIdx.x + o]);
      }
    __syncthreads();
  }
  if (threadIdx.x < 6) part[6 * blockIdx.x + threadIdx.x] = red[threadIdx.x][0];
}

// grid parameters: gp[0..2] = box minimum, gp[3..5] = cells per unit length
// (0 for a flat axis), gp[6..8] = cell edge lengths
__global__ void grid_params_kernel(const float* __restrict__ part, int nparts, int G, float* __restrict__ gp) {
  // one wave: lanes stride over the partials, then a wave reduction
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int b = threadIdx.x; b < nparts; b += 64)
    for (int a = 0; a < 3; a++) {
      lo[a] = fminf(lo[a], part[6 * b + a]);
      hi[a] = fmaxf(hi[a], part[6 * b + 3 + a]);
    }
  for (int a = 0; a < 3; a++)
    for (int o = 32; o > 0; o >>= 1) {
      lo[a] = fminf(lo[a], __shfl_xor(lo[a], o, 64));
      hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], o, 64));
    }
  if (threadIdx.x != 0) return;
  for (int a = 0; a < 3; a++) {
    const float ext = hi[a] - lo[a];
    gp[a] = lo[a];
    gp[3 + a] = ext > 0.0f ? (float)G / ext : 0.0f;
    gp[6 + a] = ext > 0.0f ? ext / (float)G : 0.0f;
  }
}

__device__ __forceinline__ int cell_coord(float x, float lo, float inv, int G) {
  const int c = (int)floorf((x - lo) * inv);
  return c < 0 ? 0 : (c >= G ? G - 1 : c);
}

__global__ void cell_keys_kernel(const float4* __restrict__ c, int64_t n, const float* __restrict__ gp,
                                 int G, uint32_t* __restrict__ key, uint32_t* __restrict__ id) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float4 p = c[i];
  const int cx = cell_coord(p.x, gp[0], gp[3], G), cy = cell_coord(p.y, gp[1], gp[4], G),
            cz = cell_coord(p.z, gp[2], gp[5], G);
  key[i] = ((uint32_t)cz * (uint32_t)G + (uint32_t)cy) * (uint32_t)G + (uint32_t)cx;
  id[i] = (uint32_t)i;
}

// start[c] = the first sorted position whose cell is c or later, for cells
// 0 .. cells (so that [start[a], start[b + 1]) holds cells a .. b)
__global__ void cell_starts_kernel(const uint32_t* __restrict__ key, int64_t n, int64_t cells,
                                   uint32_t* __restrict__ start) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c > cells) return;
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int64_t)key[mid] < c) lo = mid + 1;
    else hi = mid;
  }
  start[c] = (uint32_t)lo;
}

// centres in cell order, the index in w
__global__ void sort_centres_kernel(const float4* __restrict__ c, const uint32_t* __restrict__ sid, int64_t n,
                                    float4* __restrict__ sc) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  const uint32_t i = sid[p];
  const float4 a = c[i];
  sc[p] = make_float4(a.x, a.y, a.z, __uint_as_float(i));
}

// (d, j) < (bd, bj) in the (squared distance, index) order
__device__ __forceinline__ bool closer(double d, uint32_t j, double bd, uint32_t bj) {
  return d < bd || (d == bd && j < bj);
}

// Exact kNN of the centre at sorted position p: the 27 cells around it, then
// shells of cells at Chebyshev distance r = 2, 3, ...; after shell r every
// centre not yet seen is at least (r - 0.001) min(cell edge) away (0.001 of a
// cell covers the rounding of the cell assignment), so the search stops once K
// candidates are held and the k-th is strictly closer than that.  Cells of one
// row along x are one range of sorted positions; a row or cell of a shell that
// is further away than the K-th candidate is passed over.  Output: sorted
// positions.
//
// What bounds it is vector issue, most of it the K-step insertions in FP64: a
// wave runs one whenever any of its lanes accepts a candidate, which some lane
// nearly always does.  So a lane first collects kKnnBuf accepted candidates
// in LDS (against the K-th of the last insertion, which only accepts more) and
// the lanes insert theirs together, and centres are read from a copy in cell
// order, where a row of cells is one run.  1M uniform centres, k = 16: 3.0 ms
// inserting every candidate at once and reading centres by index, 1.3 now.
constexpr int kKnnBuf = 4;  // 4, 8 and 12: equal to within 2 %

// K <= 16: three waves per SIMD (168 registers; two waves 1.7 ms, four, with
// spills, 1.9).
template <int K>
__global__ __launch_bounds__(256, K <= 16 ? 3 : 1) void knn_kernel(const float4* __restrict__ sc, int64_t n,
                                                  const uint32_t* __restrict__ cstart,
                                                  const float* __restrict__ gp, int G, int k,
                                                  int32_t* __restrict__ out_pos,
                                                  double* __restrict__ out_d2) {
  __shared__ double buf_d[kKnnBuf][256];
  __shared__ uint2 buf_j[kKnnBuf][256];  // index, sorted position
  const int tid = threadIdx.x;
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + tid;
  if (p >= n) return;
  const float4 pi = sc[p];
  const double xi = pi.x, yi = pi.y, zi = pi.z;
  const int cx = cell_coord(pi.x, gp[0], gp[3], G), cy = cell_coord(pi.y, gp[1], gp[4], G),
            cz = cell_coord(pi.z, gp[2], gp[5], G);
  float hmin = INFINITY;
  for (int a = 0; a < 3; a++)
    if (gp[6 + a] > 0.0f) hmin = fminf(hmin, gp[6 + a]);
  if (!(hmin < INFINITY)) hmin = 0.0f;  // all centres equal: every shell is empty but the first
  double bd[K];
  uint32_t bj[K], bq[K];  // index (the order of ties) and sorted position
#pragma unroll
  for (int t = 0; t < K; t++) {
    bd[t] = INFINITY;
    bj[t] = 0xFFFFFFFFu;
    bq[t] = 0u;
  }
  // squared distance from x to cell c of an axis, a little less than it is
  // (0 for a flat axis)
  auto gap2 = [&](double x, int c, int own, int a) {
    const double h = gp[6 + a], lo = gp[a];
    const double g = c > own ? lo + c * h - x : c < own ? x - (lo + (c + 1) * h) : 0.0;
    const double m = g - 0.001 * h - 1e-6 * (fabs(x) + fabs(lo));
    return m > 0.0 ? m * m : 0.0;
  };
  int held = 0;  // candidates in the buffer
  for (int r = 1; r <= G; r++) {
    // the shell's cell rows along x, each of up to two ranges of cells: a row
    // on a face of the shell (or of the first box) whole, one inside dx = -r
    // and dx = +r; the last turn only empties the buffer
    const int side = 2 * r + 1, turns = 2 * side * side;
    for (int it = 0; it <= turns; it++) {
      uint32_t q = 0u, q1 = 0u;
      if (it < turns) {
        const int rw = it >> 1, dz = rw / side - r, dy = rw % side - r;
        const int y = cy + dy, z = cz + dz;
        const bool face = r == 1 || dz == -r || dz == r || dy == -r || dy == r;
        if (y >= 0 && y < G && z >= 0 && z < G && !(face && (it & 1))) {
          const double g2 = r > 1 ? gap2(yi, y, cy, 1) + gap2(zi, z, cz, 2) : 0.0;
          const int lone = (it & 1) ? cx + r : cx - r;
          const int x0 = face ? max(cx - r, 0) : lone, x1 = face ? min(cx + r, G - 1) : lone;
          const bool on = face || (lone >= 0 && lone < G);
          if (on && !(g2 + (face ? 0.0 : gap2(xi, lone, cx, 0)) > bd[K - 1])) {
            const uint32_t row = ((uint32_t)z * (uint32_t)G + (uint32_t)y) * (uint32_t)G;
            q = cstart[row + x0];
            q1 = cstart[row + x1 + 1];
          }
        }
      }
      for (;;) {
        const bool more = q < q1;
        if (more) {
          const float4 pj = sc[q];
          const double ex = xi - (double)pj.x, ey = yi - (double)pj.y, ez = zi - (double)pj.z;
          const double d = (ex * ex + ey * ey) + ez * ez;
          if (d <= bd[K - 1] && q != (uint32_t)p) {
            buf_d[held][tid] = d;
            buf_j[held][tid] = make_uint2(__float_as_uint(pj.w), q);
            held++;
          }
          q++;
        }
        // the active lanes insert together
        if (__ballot(held == kKnnBuf || (it == turns && held > 0))) {
          for (int e = 0; e < held; e++) {
            double d = buf_d[e][tid];
            uint2 j = buf_j[e][tid];
            if (closer(d, j.x, bd[K - 1], bj[K - 1])) {
#pragma unroll
              for (int t = 0; t < K; t++) {  // keeping the list sorted
                const bool in = closer(d, j.x, bd[t], bj[t]);
                const double td = bd[t];
                const uint32_t tj = bj[t], tq = bq[t];
                bd[t] = in ? d : td;
                bj[t] = in ? j.x : tj;
                bq[t] = in ? j.y : tq;
                d = in ? td : d;
                j.x = in ? tj : j.x;
                j.y = in ? tq : j.y;
              }
            }
          }
          held = 0;
        }
        if (!more) break;
      }
    }
    double kth = INFINITY;
#pragma unroll
    for (int t = 0; t < K; t++)
      if (t == k - 1) kth = bd[t];
    const double gap = (double)(r - 0.001) * (double)hmin;
    if (kth < INFINITY && kth < gap * gap) break;
  }
#pragma unroll
  for (int t = 0; t < K; t++)
    if (t < k) {
      out_pos[p * k + t] = (int32_t)bq[t];
      out_d2[p * k + t] = bd[t];
    }
}

// ---------------------------------------------------- median (radix select)
// Two order statistics (ranks rk[0], rk[1]) of N non-negative doubles, by
// their bits, 11 bits per round from the top.  st: prefix[2], rank[2]
// (uint64), advanced by the pick kernel after each round.
constexpr int kSelBins = 2048;

__global__ void select_hist_kernel(const double* __restrict__ v, int64_t N, int shift, int width,
                                   const unsigned long long* __restrict__ st,
                                   unsigned int* __restrict__ hist) {
  __shared__ unsigned int h[2][kSelBins];
  for (int e = threadIdx.x; e < 2 * kSelBins; e += blockDim.x) (&h[0][0])[e] = 0u;
  __syncthreads();
  const int top = shift + width;
  const unsigned long long p0 = top >= 64 ? 0ull : st[0] >> top, p1 = top >= 64 ? 0ull : st[1] >> top;
  const unsigned long long mask = (1ull << width) - 1ull;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < N; e += (int64_t)gridDim.x * blockDim.x) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v[e]);
    const unsigned long long hb = top >= 64 ? 0ull : b >> top;
    const unsigned int d = (unsigned int)((b >> shift) & mask);
    if (hb == p0) atomicAdd(&h[0][d], 1u);
    if (hb == p1) atomicAdd(&h[1][d], 1u);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 2 * kSelBins; e += blockDim.x) {
    const unsigned int x = (&h[0][0])[e];
    if (x) atomicAdd(&hist[e], x);
  }
}

// one block of 1024 threads: for each target, the digit whose cumulative
// count passes the residual rank; the histogram is cleared for the next round
__global__ __launch_bounds__(1024) void select_pick_kernel(unsigned int* __restrict__ hist, int shift,
                                                           unsigned long long* __restrict__ st) {
  // thread t owns bins 2t, 2t + 1 of each target; block-wide exclusive scan
  __shared__ unsigned long long wsum[2][16];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  unsigned long long rank[2], part[2], c0[2], c1[2];
#pragma unroll
  for (int g = 0; g < 2; g++) {
    rank[g] = st[2 + g];
    c0[g] = hist[g * kSelBins + 2 * t];
    c1[g] = hist[g * kSelBins + 2 * t + 1];
    unsigned long long incl = c0[g] + c1[g];
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned long long y = __shfl_up(incl, o, 64);
      if (lane >= o) incl += y;
    }
    part[g] = incl - (c0[g] + c1[g]);  // exclusive within the wave
    if (lane == 63) wsum[g][w] = incl;
  }
  __syncthreads();
#pragma unroll
  for (int g = 0; g < 2; g++) {
    unsigned long long base = part[g];
    for (int q = 0; q < w; q++) base += wsum[g][q];
    // the bin whose [cum, cum + count) holds the rank (exactly one thread)
    if (rank[g] >= base && rank[g] < base + c0[g]) {
      st[g] |= (unsigned long long)(2 * t) << shift;
      st[2 + g] = rank[g] - base;
    } else if (rank[g] >= base + c0[g] && rank[g] < base + c0[g] + c1[g]) {
      st[g] |= (unsigned long long)(2 * t + 1) << shift;
      st[2 + g] = rank[g] - base - c0[g];
    }
  }
  __syncthreads();
  for (int e = t; e < 2 * kSelBins; e += blockDim.x) hist[e] = 0u;
}

__global__ void select_init_kernel(unsigned long long* st, unsigned long long r0, unsigned long long r1,
                                   unsigned int* hist) {
  if (threadIdx.x == 0) {
    st[0] = 0ull;
    st[1] = 0ull;
    st[2] = r0;
    st[3] = r1;
  }
  for (int e = threadIdx.x; e < 2 * kSelBins; e += blockDim.x) hist[e] = 0u;
}

// sig2 = (median of the roots)^2, from the two middle squared values (their
// roots averaged)
__global__ void sigma_kernel(const unsigned long long* st, double* sig2) {
  if (threadIdx.x != 0) return;
  const double a = __longlong_as_double((long long)st[0]), b = __longlong_as_double((long long)st[1]);
  const double s = (sqrt(a) + sqrt(b)) / 2.0;
  sig2[0] = s * s;
}

// ------------------------------------------------------------ edge weights
__device__ __forceinline__ double wave_sum_f64(double x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// Dot product in FP64 of the FP32 rows a and b over the channels of lane `sub`
// of L (4 consecutive channels at a time where vec, else every L-th).
template <int L>
__device__ __forceinline__ double part_dot(const float* __restrict__ a, const float* __restrict__ b, int D,
                                           int sub, bool vec) {
  double s = 0.0;
  if (vec) {
#pragma unroll 4
    for (int ch = 4 * sub; ch < D; ch += 4 * L) {
      const float4 x = *reinterpret_cast<const float4*>(a + ch), y = *reinterpret_cast<const float4*>(b + ch);
      s += (double)x.x * (double)y.x;
      s += (double)x.y * (double)y.y;
      s += (double)x.z * (double)y.z;
      s += (double)x.w * (double)y.w;
    }
  } else {
#pragma unroll 4
    for (int ch = sub; ch < D; ch += L) s += (double)a[ch] * (double)b[ch];
  }
  return s;
}

template <int L>
__device__ __forceinline__ double lane_sum(double x) {  // over L consecutive lanes
#pragma unroll
  for (int o = 1; o < L; o <<= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// Block b of a grid in which XCD x (workgroups go round-robin) takes the x-th
// eighth of the blocks: neighbours in the order of work share an L2.
__device__ __forceinline__ int64_t xcd_block() {
  const int64_t nb = gridDim.x, per = nb / 8;
  return (int64_t)blockIdx.x < 8 * per ? (int64_t)(blockIdx.x & 7) * per + (blockIdx.x >> 3) : blockIdx.x;
}

// norms of the feature rows, L lanes per row
template <int L>
__global__ __launch_bounds__(256) void norms_kernel(const float* __restrict__ f, int64_t n, int D, bool vec,
                                                    double* __restrict__ nrm) {
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / L;
  const int sub = threadIdx.x % L;
  if (i >= n) return;
  const float* const a = f + i * D;
  const double s = lane_sum<L>(part_dot<L>(a, a, D, sub, vec));
  if (sub == 0) nrm[i] = sqrt(s);
}

// Weights of the directed edges, L lanes per edge, edges in cell order: a
// neighbour's row is then read again by its other neighbours while it is in
// the caches, and 64 / L edges share one pass of the sum, the exponential and
// the division.  1M nodes, k = 16, D = 64: 4.1 ms with a wave per node, nodes
// in the caller's order; 0.59 now (the 4.1 GB of gathered rows at 7 TB/s).  A
// launch takes the edges [first, end): a grid holds fewer than 2^32 threads.
template <int L>
__global__ __launch_bounds__(256) void edge_weights_kernel(const float* __restrict__ f, int64_t first, int64_t end,
                                                           int D, int k, bool vec, const uint32_t* __restrict__ sid,
                                                           const int32_t* __restrict__ pos,
                                                           const double* __restrict__ d2,
                                                           const double* __restrict__ nrm,
                                                           const double* __restrict__ sig2,
                                                           double* __restrict__ w) {
  const int64_t e = first + (xcd_block() * blockDim.x + threadIdx.x) / L;
  const int sub = threadIdx.x % L;
  if (e >= end) return;
  const int64_t i = sid[e / k], j = sid[pos[e]];
  const double dot = lane_sum<L>(part_dot<L>(f + i * D, f + j * D, D, sub, vec));
  if (sub == 0) {
    const double den = nrm[i] * nrm[j];
    const double cs = den > 0.0 ? dot / den : 0.0;
    w[e] = exp(-d2[e] / sig2[0]) * (cs > 0.0 ? cs : 0.0);
  }
}

// squared distances of the l2-normalised features of each directed pair
// (a zero feature stays zero), one wave per node
__global__ __launch_bounds__(256) void feature_d2_kernel(const float* __restrict__ f, int64_t n, int D,
                                                         int k, const uint32_t* __restrict__ sid,
                                                         const int32_t* __restrict__ pos,
                                                         const double* __restrict__ nrm,
                                                         double* __restrict__ fd2) {
  const int64_t p = (xcd_block() * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (p >= n) return;
  const int64_t i = sid[p];
  const double ni = nrm[i];
  for (int t = 0; t < k; t++) {
    const int64_t j = sid[pos[p * k + t]];
    const double nj = nrm[j];
    double acc = 0.0;
    for (int ch = lane; ch < D; ch += 64) {
      const double a = ni > 0.0 ? (double)f[i * D + ch] / ni : 0.0;
      const double b = nj > 0.0 ? (double)f[j * D + ch] / nj : 0.0;
      acc += (a - b) * (a - b);
    }
    acc = wave_sum_f64(acc);
    if (lane == 0) fd2[p * k + t] = acc;
  }
}

// Eq. 7 / Eq. 9 weight of each directed pair
__global__ void rbf_weights_kernel(int64_t nk, int k, const uint32_t* __restrict__ sid,
                                   const int32_t* __restrict__ pos,
                                   const double* __restrict__ fd2, const double* __restrict__ s2,
                                   double bandwidth, const float* __restrict__ unary,
                                   double* __restrict__ w) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nk) return;
  const int64_t i = sid[e / k], j = sid[pos[e]];
  const double pp = unary ? sqrt((double)unary[i]) * sqrt((double)unary[j]) : 1.0;
  w[e] = exp(-fd2[e] / (bandwidth * s2[0])) * pp;
}

// ------------------------------------------------------------ union rows
// A directed edge (p, q) also belongs to row q.  Where it is mutual (p among
// q's own k, with the same weight) that row has it already; the others take
// the next free place of row q, counted here: about 0.4 of the edges of a
// uniform scene, and the only atomics of the union.
__global__ __launch_bounds__(256) void reverse_slots_kernel(const int32_t* __restrict__ pos, int64_t nk, int k,
                                                            uint32_t* __restrict__ extra,
                                                            uint32_t* __restrict__ slot) {
  const int64_t e = xcd_block() * blockDim.x + threadIdx.x;
  if (e >= nk) return;
  const int32_t p = (int32_t)(e / k), q = pos[e];
  const int32_t* const list = pos + (int64_t)q * k;
  bool mutual = false;
  for (int t = 0; t < k; t++) mutual = mutual || list[t] == p;
  slot[e] = mutual ? ~0u : atomicAdd(&extra[q], 1u);
}

__global__ void row_cap_kernel(const uint32_t* __restrict__ extra, int64_t n, int k,
                               uint32_t* __restrict__ cap) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) cap[i] = (uint32_t)k + extra[i] + 1u;  // own, reversed, a possible self-loop
}

// row p: its own k entries first, then the reversed edges of the nodes that
// chose p (in arrival order; sorted afterwards); columns are caller indices
__global__ __launch_bounds__(256) void fill_rows_kernel(const int32_t* __restrict__ pos,
                                                        const double* __restrict__ w,
                                                        const uint32_t* __restrict__ slot,
                                                        const uint32_t* __restrict__ sid, int64_t nk, int k,
                                                        const uint32_t* __restrict__ start,
                                                        int32_t* __restrict__ ucol, double* __restrict__ uw) {
  const int64_t e = xcd_block() * blockDim.x + threadIdx.x;
  if (e >= nk) return;
  const int64_t p = e / k;
  const int t = (int)(e - p * k);
  const int32_t q = pos[e];
  const double x = w[e];
  const uint32_t o = start[p] + (uint32_t)t, sl = slot[e];
  ucol[o] = (int32_t)sid[q];
  uw[o] = x;
  if (sl != ~0u) {
    const uint32_t r = start[q] + (uint32_t)k + sl;
    ucol[r] = (int32_t)sid[p];
    uw[r] = x;
  }
}

// Row p sorted by column in place, entries that do not pass dropped, the sum in
// column order; a row left empty gets the self-loop (weight 1).  len, rsum at
// the caller's index.  Columns are distinct, so an entry's place is the number
// of kept columns below its own: W lanes per row (32, or 64 for rows of 33 to
// 64 entries), the row's columns in LDS, four compared per read.  (A bitonic
// sort of a wave per row took 813 us for 1M rows of 23 entries, this 290.)
template <int W>
__device__ __forceinline__ void sort_row(int64_t p, bool on, int m, int sub, const uint32_t* start,
                                         const uint32_t* sid, int32_t* ucol, double* uw, uint32_t* len,
                                         double* rsum, double thresh, bool binarize, bool self_loops,
                                         int32_t* lc, double* lx) {
  int32_t* const cl = ucol + (on ? start[p] : 0u);
  double* const wv = uw + (on ? start[p] : 0u);
  const bool have = on && sub < m;
  const double x = have ? wv[sub] : 0.0;
  const bool keep = have && x > thresh;
  const int32_t c = keep ? cl[sub] : 0x7FFFFFFF;
  lc[sub] = c;
  lx[sub] = 0.0;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  uint32_t rank = 0u;
#pragma unroll
  for (int t = 0; t < W; t += 4) {
    const int4 o = *reinterpret_cast<const int4*>(lc + t);
    rank += (o.x < c ? 1u : 0u) + (o.y < c ? 1u : 0u) + (o.z < c ? 1u : 0u) + (o.w < c ? 1u : 0u);
  }
  const double v = binarize ? 1.0 : x;
  if (keep) {
    cl[rank] = c;
    wv[rank] = v;
    lx[rank] = v;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  double sum = lx[sub];
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  uint32_t u = keep ? 1u : 0u;
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) u += (uint32_t)__shfl_xor((int)u, o, 64);
  if (on && sub == 0) {
    const uint32_t i = sid[p];
    if (u == 0 && self_loops) {  // self-loop
      cl[0] = (int32_t)i;
      wv[0] = 1.0;
      u = 1;
      sum = 1.0;
    }
    len[i] = u;
    rsum[i] = sum;
  }
}

__global__ __launch_bounds__(256) void sort_rows_kernel(int64_t n, int k, const uint32_t* __restrict__ start,
                                                        const uint32_t* __restrict__ extra,
                                                        const uint32_t* __restrict__ sid,
                                                        int32_t* __restrict__ ucol, double* __restrict__ uw,
                                                        uint32_t* __restrict__ len, double* __restrict__ rsum,
                                                        double thresh, bool binarize, bool self_loops) {
  __shared__ __align__(16) int32_t lc[256];
  __shared__ double lx[256];
  const int64_t p = (xcd_block() * 256 + threadIdx.x) >> 5;
  const int sub = threadIdx.x & 31, g = threadIdx.x & ~31;
  const int m = p < n ? k + (int)extra[p] : 0;
  sort_row<32>(p, p < n && m <= 32, m, sub, start, sid, ucol, uw, len, rsum, thresh, binarize, self_loops, lc + g,
               lx + g);
}

// Rows of more than 32 entries (few): each wave looks for them among 64 rows
// and takes them one by one; beyond 64 entries one lane sorts the row.
__global__ __launch_bounds__(64) void sort_long_rows_kernel(int64_t n, int k, const uint32_t* __restrict__ start,
                                                            const uint32_t* __restrict__ extra,
                                                            const uint32_t* __restrict__ sid,
                                                            int32_t* __restrict__ ucol, double* __restrict__ uw,
                                                            uint32_t* __restrict__ len,
                                                            double* __restrict__ rsum, double thresh,
                                                            bool binarize, bool self_loops) {
  __shared__ __align__(16) int32_t lc[64];
  __shared__ double lx[64];
  const int lane = threadIdx.x;
  const int64_t p0 = (int64_t)blockIdx.x * 64, mine = p0 + lane;
  const int m = mine < n ? k + (int)extra[mine] : 0;
  for (uint64_t b = __ballot(m > 32 && m <= 64); b; b &= b - 1) {
    const int r = (int)__builtin_ctzll(b);
    sort_row<64>(p0 + r, true, __shfl(m, r, 64), lane, start, sid, ucol, uw, len, rsum, thresh, binarize,
                 self_loops, lc, lx);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  if (m <= 64) return;
  int32_t* cl = ucol + start[mine];
  double* wv = uw + start[mine];
  int u = 0;
  double s = 0.0;
  for (int a = 0; a < m; a++) {  // insertion sort of the entries that pass
    const int32_t c = cl[a];
    const double x = wv[a];
    if (!(x > thresh)) continue;
    int b = u - 1;
    while (b >= 0 && cl[b] > c) {
      cl[b + 1] = cl[b];
      wv[b + 1] = wv[b];
      b--;
    }
    cl[b + 1] = c;
    wv[b + 1] = binarize ? 1.0 : x;
    u++;
  }
  for (int a = 0; a < u; a++) s += wv[a];
  const uint32_t i = sid[mine];
  if (u == 0 && self_loops) {  // self-loop
    cl[0] = (int32_t)i;
    wv[0] = 1.0;
    u = 1;
    s = 1.0;
  }
  len[i] = (uint32_t)u;
  rsum[i] = s;
}

// 16 lanes per row (one lane per row took 992 us for 1M rows of 23 entries,
// these 181)
__global__ __launch_bounds__(256) void csr_out_kernel(int64_t n, const uint32_t* __restrict__ start,
                                                      const uint32_t* __restrict__ sid,
                                                      const uint32_t* __restrict__ len,
                                                      const uint32_t* __restrict__ rp,
                                                      const int32_t* __restrict__ ucol,
                                                      const double* __restrict__ uw,
                                                      const double* __restrict__ rsum, int32_t* __restrict__ col,
                                                      float* __restrict__ val, int32_t* __restrict__ row_ptr,
                                                      uint64_t nnz, bool normalise) {
  const int64_t p = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 4;
  const uint32_t sub = threadIdx.x & 15;
  if (p >= n) return;
  const uint32_t i = sid[p], a = start[p], o = rp[i], m = len[i];
  const double s = rsum[i];
  for (uint32_t q = sub; q < m; q += 16) {
    col[o + q] = ucol[a + q];
    val[o + q] = normalise ? (float)(uw[a + q] / s) : (float)uw[a + q];
  }
  if (sub == 0) {
    row_ptr[i] = (int32_t)o;
    if (i == (uint32_t)(n - 1)) row_ptr[n] = (int32_t)nnz;
  }
}

__global__ void one_segment_kernel(uint32_t* seg, int64_t n) {
  if (threadIdx.x == 0) {
    seg[0] = 0u;
    seg[1] = (uint32_t)n;
  }
}

unsigned grid1(int64_t items) { return (unsigned)((items + 255) / 256); }

// lanes per feature row or edge: rows of a few channels one lane, wide rows 16
int lanes_for(int D) { return D <= 8 ? 1 : D <= 128 ? 4 : 16; }

}  // namespace

hipError_t build_knn_graph(const float4* centres, int64_t n, const float* feats, int D, int k,
                           const GraphWeights& gw, hipStream_t s, const GraphAlloc& alloc, int32_t** row_ptr,
                           int32_t** col, float** val, int64_t* nnz_out) {
  const bool rbf = gw.kind == LV_GRAPH_FEATURE_RBF;
  *row_ptr = nullptr;
  *col = nullptr;
  *val = nullptr;
  *nnz_out = 0;
  const int64_t nk = n * (int64_t)k;
  const int64_t ucap = n * (int64_t)(2 * k + 1);  // union entries before merging
  // grid: about kCellCentres centres per cell
  int G = 1;
  while ((int64_t)(G + 1) * (G + 1) * (G + 1) * kCellCentres <= n && G < 1024) G++;
  const int64_t cells = (int64_t)G * G * G;
  int cell_bits = 0;
  while (((int64_t)1 << cell_bits) < cells) cell_bits++;
  const bool vec = D % 4 == 0 && (uintptr_t)feats % 16 == 0;
  const int lanes = lanes_for(D);
  const int nparts = (int)std::min<int64_t>(1024, (n + 255) / 256);

  // scratch layout (bytes)
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t o = off; off += (bytes + 255) & ~(size_t)255; return o; };
  const size_t o_part = take(4 * 6 * (size_t)nparts), o_gp = take(4 * 9);
  const size_t o_k0 = take(4 * (size_t)n), o_v0 = take(4 * (size_t)n), o_k1 = take(4 * (size_t)n),
               o_v1 = take(4 * (size_t)n), o_seg = take(8), o_hist = take(4 * sort_hist_size(1, n));
  const size_t o_cs = take(4 * (size_t)(cells + 1)), o_sc = take(sizeof(float4) * (size_t)n);
  const size_t o_idx = take(4 * (size_t)nk), o_d2 = take(8 * (size_t)nk), o_w = take(8 * (size_t)nk);
  const size_t o_st = take(8 * 4), o_shist = take(4 * 2 * kSelBins), o_sig = take(8),
               o_nrm = take(8 * (size_t)n);
  const size_t o_slot = take(4 * (size_t)nk);
  const size_t o_extra = take(4 * (size_t)n), o_cap = take(4 * (size_t)n), o_start = take(4 * (size_t)n),
               o_len = take(4 * (size_t)n), o_rp = take(4 * (size_t)n),
               o_rsum = take(8 * (size_t)n);
  const size_t o_ucol = take(4 * (size_t)ucap), o_uw = take(8 * (size_t)ucap);
  const size_t o_sseg = take(8), o_tot = take(16), o_stmp = take(4 * scan_tmp_size(n));
  char* base = nullptr;
  hipError_t e = alloc.scratch((void**)&base, off);
  if (e != hipSuccess) return e;
  auto at = [&](size_t o) { return base + o; };
  float* part = (float*)at(o_part);
  float* gp = (float*)at(o_gp);
  uint32_t *k0 = (uint32_t*)at(o_k0), *v0 = (uint32_t*)at(o_v0), *k1 = (uint32_t*)at(o_k1),
           *v1 = (uint32_t*)at(o_v1), *seg = (uint32_t*)at(o_seg), *hist = (uint32_t*)at(o_hist);
  uint32_t* cs = (uint32_t*)at(o_cs);
  float4* sc = (float4*)at(o_sc);
  int32_t* pos = (int32_t*)at(o_idx);  // [n][k] neighbours, all in sorted positions
  double *d2 = (double*)at(o_d2), *w = (double*)at(o_w);
  unsigned long long* st = (unsigned long long*)at(o_st);
  unsigned int* shist = (unsigned int*)at(o_shist);
  double *sig2 = (double*)at(o_sig), *nrm = (double*)at(o_nrm);
  uint32_t *slot = (uint32_t*)at(o_slot), *extra = (uint32_t*)at(o_extra), *cap = (uint32_t*)at(o_cap),
           *start = (uint32_t*)at(o_start), *len = (uint32_t*)at(o_len), *rp = (uint32_t*)at(o_rp);
  double* rsum = (double*)at(o_rsum);
  int32_t* ucol = (int32_t*)at(o_ucol);
  double* uw = (double*)at(o_uw);
  uint32_t* sseg = (uint32_t*)at(o_sseg);
  unsigned long long* tot = (unsigned long long*)at(o_tot);
  uint32_t* stmp = (uint32_t*)at(o_stmp);
  uint64_t nnz = 0;

  do {
    // grid and centres sorted by cell
    hipLaunchKernelGGL(bbox_partial_kernel, dim3(nparts), dim3(256), 0, s, centres, n, part);
    hipLaunchKernelGGL(grid_params_kernel, dim3(1), dim3(64), 0, s, part, nparts, G, gp);
    hipLaunchKernelGGL(cell_keys_kernel, dim3(grid1(n)), dim3(256), 0, s, centres, n, gp, G, k0, v0);
    hipLaunchKernelGGL(one_segment_kernel, dim3(1), dim3(64), 0, s, seg, n);
    bool second = false;
    if ((e = radix_sort(k0, v0, k1, v1, seg, seg + 1, 1, n, cell_bits, hist, true, &second, s)) != hipSuccess) break;
    const uint32_t* skey = second ? k1 : k0;
    const uint32_t* sid = second ? v1 : v0;
    hipLaunchKernelGGL(cell_starts_kernel, dim3(grid1(cells + 1)), dim3(256), 0, s, skey, n, cells, cs);
    hipLaunchKernelGGL(sort_centres_kernel, dim3(grid1(n)), dim3(256), 0, s, centres, sid, n, sc);
    // exact kNN
    if (k <= 8)
      hipLaunchKernelGGL(knn_kernel<8>, dim3(grid1(n)), dim3(256), 0, s, sc, n, cs, gp, G, k, pos, d2);
    else if (k <= 16)
      hipLaunchKernelGGL(knn_kernel<16>, dim3(grid1(n)), dim3(256), 0, s, sc, n, cs, gp, G, k, pos, d2);
    else
      hipLaunchKernelGGL(knn_kernel<32>, dim3(grid1(n)), dim3(256), 0, s, sc, n, cs, gp, G, k, pos, d2);
    // sigma: ranks (N - 1) / 2 and N / 2 of the squared distances
    const unsigned long long N = (unsigned long long)nk;
    hipLaunchKernelGGL(select_init_kernel, dim3(1), dim3(256), 0, s, st, (N - 1) / 2, N / 2, shist);
    const unsigned sblocks = (unsigned)std::min<int64_t>(1024, (nk + 255) / 256);
    for (int shift = 53, width = 11; ; ) {
      hipLaunchKernelGGL(select_hist_kernel, dim3(sblocks), dim3(256), 0, s, d2, nk, shift, width, st, shist);
      hipLaunchKernelGGL(select_pick_kernel, dim3(1), dim3(1024), 0, s, shist, shift, st);
      if (shift == 0) break;
      width = shift >= 11 ? 11 : shift;
      shift -= width;
    }
    hipLaunchKernelGGL(sigma_kernel, dim3(1), dim3(64), 0, s, st, sig2);
    // weights
    const auto norms = lanes == 1 ? norms_kernel<1> : lanes == 4 ? norms_kernel<4> : norms_kernel<16>;
    hipLaunchKernelGGL(norms, dim3(grid1(n * lanes)), dim3(256), 0, s, feats, n, D, vec, nrm);
    if (!rbf) {
      const auto weights = lanes == 1   ? edge_weights_kernel<1>
                           : lanes == 4 ? edge_weights_kernel<4>
                                        : edge_weights_kernel<16>;
      const int64_t slice = ((int64_t)1 << 31) / lanes;  // edges of a launch
      for (int64_t first = 0; first < nk; first += slice) {
        const int64_t end = std::min(nk, first + slice);
        hipLaunchKernelGGL(weights, dim3(grid1((end - first) * lanes)), dim3(256), 0, s, feats, first, end, D, k, vec,
                           sid, pos, d2, nrm, sig2, w);
      }
    } else {
      // s_f: median feature distance over the directed pairs (d2 is reused
      // for the feature distances; sigma above is not needed)
      hipLaunchKernelGGL(feature_d2_kernel, dim3((unsigned)((n * 64 + 255) / 256)), dim3(256), 0, s, feats, n,
                         D, k, sid, pos, nrm, w);
      hipLaunchKernelGGL(select_init_kernel, dim3(1), dim3(256), 0, s, st, (N - 1) / 2, N / 2, shist);
      for (int shift = 53, width = 11; ; ) {
        hipLaunchKernelGGL(select_hist_kernel, dim3(sblocks), dim3(256), 0, s, w, nk, shift, width, st, shist);
        hipLaunchKernelGGL(select_pick_kernel, dim3(1), dim3(1024), 0, s, shist, shift, st);
        if (shift == 0) break;
        width = shift >= 11 ? 11 : shift;
        shift -= width;
      }
      hipLaunchKernelGGL(sigma_kernel, dim3(1), dim3(64), 0, s, st, sig2);
      hipLaunchKernelGGL(rbf_weights_kernel, dim3(grid1(nk)), dim3(256), 0, s, nk, k, sid, pos, w,
                         sig2, (double)gw.bandwidth, gw.unary, d2);
      double* t = w;  // the weights are in d2's buffer
      w = d2;
      d2 = t;
    }
    // union rows
    if ((e = hipMemsetAsync(extra, 0, 4 * (size_t)n, s)) != hipSuccess) break;
    hipLaunchKernelGGL(reverse_slots_kernel, dim3(grid1(nk)), dim3(256), 0, s, pos, nk, k, extra, slot);
    hipLaunchKernelGGL(row_cap_kernel, dim3(grid1(n)), dim3(256), 0, s, extra, n, k, cap);
    if ((e = scan_counts(cap, nullptr, n, 1, start, sseg, sseg + 1, tot, stmp, s)) != hipSuccess) break;
    hipLaunchKernelGGL(fill_rows_kernel, dim3(grid1(nk)), dim3(256), 0, s, pos, w, slot, sid, nk, k, start, ucol,
                       uw);
    const bool bin = rbf && gw.binarize > 0.0f;
    const double thresh = bin ? (double)gw.binarize : 0.0;
    hipLaunchKernelGGL(sort_rows_kernel, dim3(grid1(n * 32)), dim3(256), 0, s, n, k, start, extra, sid, ucol, uw,
                       len, rsum, thresh, bin, !rbf);
    hipLaunchKernelGGL(sort_long_rows_kernel, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, s, n, k, start, extra,
                       sid, ucol, uw, len, rsum, thresh, bin, !rbf);
    if ((e = scan_counts(len, nullptr, n, 1, rp, sseg, sseg + 1, tot, stmp, s)) != hipSuccess) break;
    unsigned long long th[2] = {0, 0};
    if ((e = hipMemcpyAsync(th, tot, 16, hipMemcpyDeviceToHost, s)) != hipSuccess) break;
    if ((e = hipStreamSynchronize(s)) != hipSuccess) break;
    nnz = th[0];
    if ((e = alloc.csr((int64_t)nnz, row_ptr, col, val)) != hipSuccess) break;
    hipLaunchKernelGGL(csr_out_kernel, dim3(grid1(n * 16)), dim3(256), 0, s, n, start, sid, len, rp, ucol, uw, rsum,
                       *col, *val, *row_ptr, (uint64_t)nnz, !rbf);
    e = hipGetLastError();
  } while (false);
  if (e == hipSuccess) e = hipGetLastError();
  if (e != hipSuccess) {
    (void)hipStreamSynchronize(s);
    return e;
  }
  *nnz_out = (int64_t)nnz;
  return hipSuccess;
}

}  // namespace lv
