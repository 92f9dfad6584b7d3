// Blend-and-accumulate (Sec. 3.2, Eq. 3 / Eq. 5): for every tile of every
// view, walk the tile's depth-ordered Gaussians front to back, form the
// alpha-blending weight w_i(p) = alpha_i(p) T_i(p) of each Gaussian at each
// pixel (Eq. 1), and add w_i(p) F(p) and w_i(p) into the per-Gaussian
// accumulators U_i and beta_i.  W is never materialised.
//
// One workgroup = one 8x8 quadrant of a 16x16 tile (one pixel per lane) for one
// group of up to 64 channels, as one wave64 that walks and flushes in turn or
// two that share the work; with several groups, one wave per 16x8 half tile for
// all of them (blend_pair_kernel, two pixels per lane).  Workgroups never wait
// for each other.  Per step of 64 Gaussians of the tile's list:
//   0. lane j loads Gaussian j's record (vector loads, all in flight
//      together), leaves it in LDS and tests whether its alpha >= 1/255
//      region can touch the quadrant (exact minimum of the conic over the
//      quadrant, conservative slack); a ballot gives the step's hit mask;
//   A. walk: a scalar loop over the hit Gaussians in order; each lane
//      evaluates the Gaussian at its pixel (the record read from LDS at one
//      address, a broadcast), every decision in the S32 sequence;
//   B. the Gaussian takes the next of 32 LDS rows (its weights at the 64
//      pixels; in the pair and render kernels only if some w > 0).  A full set
//      of rows (and the last, partial one) is flushed: U_rows += W_rows F on the matrix cores, one global atomic per
//      (Gaussian, channel); beta (the rows' sums, in exact fixed point, once
//      for all feature sets that take the same views) and the tail channels
//      (the rows' dot products with up to 4 further channels) by one lane
//      pair per row.
#include <algorithm>

#include "lv_internal.h"

namespace lv {

namespace {


template <lv_dtype DT>
__device__ __forceinline__ float load_feature(const void* map, int64_t idx, float scale) {
  if constexpr (DT == LV_F32) {
    return gptr(static_cast<const float*>(map))[idx];
  } else if constexpr (DT == LV_BF16) {
    uint32_t b = gptr(static_cast<const uint16_t*>(map))[idx];
    return __uint_as_float(b << 16);
  } else {
    // without branches: a subnormal (e = 0) is built as 2^-6 (1 + m/8) and
    // 2^-6 taken off again, which is exact; the sign bit goes on last
    const uint32_t b = gptr(static_cast<const uint8_t*>(map))[idx];
    const uint32_t e = (b >> 3) & 0xFu, mt = b & 7u, sub = e == 0u;
    const float mag = __uint_as_float(((e + 120u + sub) << 23) | (mt << 20)) - __uint_as_float(sub * 0x3C800000u);
    return __uint_as_float(__float_as_uint(mag) | ((b & 0x80u) << 24)) * scale;
  }
}

// Map of set sd for view v (NULL: the set does not take the view).
__device__ __forceinline__ const void* map_of(const SetDesc& sd, int v) { return gptr(sd.maps)[v]; }

// Can -power(d) <= tau hold for some d in the rectangle [X0,X1] x [Y0,Y1]
// (offsets from the Gaussian's centre)?  -power = (L11 dx + L12 dy)^2 +
// (L22 dy)^2 is convex with its minimum at 0, so outside the rectangle its
// minimum over the rectangle lies on an edge; along each edge it is a 1D
// quadratic with a clamped vertex.  Evaluated in the factored form, which
// stays accurate for thin Gaussians.
__device__ __forceinline__ float neg_power(float L11, float L12, float L22, float dx, float dy) {
  const float u = __builtin_fmaf(L12, dy, L11 * dx), w = L22 * dy;
  return __builtin_fmaf(u, u, w * w);
}

__device__ __forceinline__ bool region_hits(float4 r0, float4 r1, float X0, float X1, float Y0,
                                            float Y1) {
  const float tau = r1.z;
  if (!(tau >= 0.0f)) return false;
  if (X0 <= 0.0f && X1 >= 0.0f && Y0 <= 0.0f && Y1 >= 0.0f) return true;
  const float L11 = r0.z, L12 = r0.w, L22 = r1.x;
  const float ky = -(L11 * L12) / __builtin_fmaf(L12, L12, L22 * L22);  // edge dx = X: dy* = ky X
  const float kx = -L12 / L11;                                          // edge dy = Y: dx* = kx Y
  const float dy0 = fminf(fmaxf(ky * X0, Y0), Y1);
  const float dy1 = fminf(fmaxf(ky * X1, Y0), Y1);
  const float dx0 = fminf(fmaxf(kx * Y0, X0), X1);
  const float dx1 = fminf(fmaxf(kx * Y1, X0), X1);
  const float m0 = fminf(neg_power(L11, L12, L22, X0, dy0), neg_power(L11, L12, L22, X1, dy1));
  const float m1 = fminf(neg_power(L11, L12, L22, dx0, Y0), neg_power(L11, L12, L22, dx1, Y1));
  return fminf(m0, m1) <= tau;
}

// A wave's statistics into its copy of the set's words (copy blockIdx mod
// kStatSlots; lv_accum_stats sums the copies): one atomic instruction of
// three lanes.  With one copy the thousands of waves' adds to the same words,
// about 15 ns each, were most of a counted launch (50k Gaussians, 9 views of
// 333x251, D = 37: blend 572 us with one copy, 446 with 256).
__device__ __forceinline__ void add_stats(const SetDesc& sd, int lane, uint32_t covered, uint32_t contrib,
                                          uint32_t rows) {
  if (!sd.stats || lane >= 3) return;
  const uint32_t v = lane == 0 ? covered : lane == 1 ? contrib : rows;
  gatomic_add(sd.stats + kStatWords * (blockIdx.x % (unsigned)kStatSlots) + lane, (unsigned long long)v);
}

// The quadrant a workgroup handles.  Workgroups go to the 8 XCDs
// round-robin, so the four quadrant waves of a tile get ids that are equal
// mod 8 and consecutive within the XCD: they share that XCD's L2 for the
// tile's records.
struct Quad {
  int v, tile, cg, qx, qy;
  uint2 rg;
  ViewGeom g;
};

// empty_ok: a tile without Gaussians is kept (the render writes its zeros).
__device__ __forceinline__ bool decode_quad(const uint2* __restrict__ ranges,
                                            const ViewGeom* __restrict__ geom, int tiles_stride,
                                            int nviews, int ngroups, Quad& q,
                                            bool empty_ok = false) {
  const uint32_t L = blockIdx.x;
  const uint32_t kx = L >> 3;
  const uint32_t work = ((kx >> 2) << 3) | (L & 7u);
  if (work >= (uint32_t)tiles_stride * (uint32_t)nviews * (uint32_t)ngroups) return false;
  const int quad = (int)(kx & 3u);
  q.tile = (int)(work % (uint32_t)tiles_stride);
  q.v = (int)((work / (uint32_t)tiles_stride) % (uint32_t)nviews);
  q.cg = (int)(work / ((uint32_t)tiles_stride * (uint32_t)nviews));
  q.g = geom[q.v];
  if (q.tile >= q.g.TX * q.g.TY) return false;
  q.rg = ranges[(int64_t)q.v * tiles_stride + q.tile];
  if (q.rg.y <= q.rg.x && !empty_ok) return false;
  const int tx = q.tile % q.g.TX, ty = q.tile / q.g.TX;
  q.qx = tx * kTile + (quad & 1) * 8;
  q.qy = ty * kTile + (quad >> 1) * 8;
  return q.qx < q.g.W && q.qy < q.g.H;  // else the quadrant lies outside the image
}

// Per-lane walk state.
// Coordinates are relative to the tile: pixel offsets px - ox in [0, 16) and
// centres as (ux - (ox + 0.5)) + ux_lo (see Rec).
struct Walk {
  float pxo, pyo;  // this lane's pixel, relative to the tile
  float ocx, ocy;  // first pixel centre of the tile, ox + 0.5, oy + 0.5
  float qx0, qy0;  // the quadrant's first pixel, relative to the tile
  float T;         // transmittance; 0 once the pixel is done, or outside the image
};

__device__ __forceinline__ void walk_init(const Quad& q, int lane, Walk& s) {
  const int px = q.qx + (lane & 7), py = q.qy + (lane >> 3);
  const int ox = q.qx & ~(kTile - 1), oy = q.qy & ~(kTile - 1);
  s.pxo = (float)(px - ox);
  s.pyo = (float)(py - oy);
  s.ocx = (float)ox + 0.5f;
  s.ocy = (float)oy + 0.5f;
  s.qx0 = (float)(q.qx - ox);
  s.qy0 = (float)(q.qy - oy);
  s.T = px < q.g.W && py < q.g.H ? 1.0f : 0.0f;
}

// The records of a tile's list, one step of 64 entries after the other.
// kAhead, for a wave that issues no atomics of its own: a step's ids are loaded
// two steps ahead and its records one step ahead (past the list's end: its last
// entry again, never used).  A wave that does issue atomics gains nothing from
// it: the vector memory counter is in order, so the loads' data would be waited
// for together with the atomics.
template <bool kAhead>
struct Steps {
  const Rec* vrec;
  const uint32_t* ids;
  const uint32_t* perm;  // nullable: storage -> caller order, for the ids handed out
  uint32_t end;          // the list's end
  uint32_t id1, id2;     // this lane's entries of the next step and the one after
  uint32_t out1;         // the next step's id as handed out
  float4 n0, n1;         // the next step's record
  __device__ __forceinline__ uint32_t id_at(uint32_t e) const { return ids[e < end ? e : end - 1]; }
  __device__ __forceinline__ void load(uint32_t id) {
    out1 = perm ? perm[id] : id;
    n0 = vrec[id].r0;
    n1 = vrec[id].r1;
  }
  __device__ __forceinline__ void start(const Rec* r, const uint32_t* i, uint2 rg, int lane,
                                        const uint32_t* p = nullptr) {
    vrec = r;
    ids = i;
    perm = p;
    end = rg.y;
    if constexpr (kAhead) {
      id1 = id_at(rg.x + lane);
      id2 = id_at(rg.x + kChunk + lane);
      load(id1);
    }
  }
  // the step from entry `base`: this lane's id and record
  __device__ __forceinline__ void next(uint32_t base, int lane, uint32_t& id, float4& q0, float4& q1) {
    if constexpr (!kAhead) load(id_at(base + lane));
    id = out1;
    q0 = n0;
    q1 = n1;
    if constexpr (kAhead) {
      id1 = id2;
      id2 = id_at(base + 2 * kChunk + lane);
      load(id1);
    }
  }
};

// The step from entry `base`: this lane's record, its centre made tile-relative,
// left in rs[lane] = {(cx, cy, L11, L12), (L22, opacity, tau, -)} for the walk;
// the hit mask (the alpha >= 1/255 region can touch the quadrant).
template <bool kAhead>
__device__ __forceinline__ uint64_t step_records(Steps<kAhead>& st, uint32_t base, int lane, const Walk& s,
                                                 uint32_t& my_id, float4 (*rs)[2]) {
  float4 q0, q1;
  st.next(base, lane, my_id, q0, q1);
  const uint32_t lo = __float_as_uint(q1.w);  // centre relative to the tile (see Rec)
  q0.x = (q0.x - s.ocx) + __uint_as_float(lo << 16);
  q0.y = (q0.y - s.ocy) + __uint_as_float(lo & 0xFFFF0000u);
  rs[lane][0] = q0;
  rs[lane][1] = q1;
  const float X0 = s.qx0 - q0.x, Y0 = s.qy0 - q0.y;
  const bool hit = base + lane < st.end && region_hits(q0, q1, X0, X0 + 7.0f, Y0, Y0 + 7.0f);
  return __ballot(hit);
}

// Barrier of a workgroup's waves that orders their LDS accesses only: loads and
// atomics stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Up to this many quadrants, a quadrant gets two waves, one that walks and one
// that flushes, rather than one that does both in turn: four quadrants per SIMD
// leave room for the second wave, and the launch lasts as long as its longest
// quadrant.  Past it the chip is full either way and the second wave and queue
// only take the first ones' room.  Launch of 512x384 views (3072 quadrants
// each), one wave / two: 1 mask channel, 200k Gaussians, 1 view 113 / 86 us, 2
// views 115 / 121, 8 views 260 / 343; render, D = 16, 50k Gaussians, 1 view 67 /
// 60, 2 views 81 / 90.
constexpr int64_t kFewQuadrants = 4096;

// Mean length of the tiles' lists from which a group of more than 32 channels gets
// two waves also where the launch fills the chip: with short lists the second wave
// takes room and its start is most of what it does.  Call with 20 views of 800x600,
// D = 64, one wave / two: lists of 6 in FP32 454 / 618 us, in BF16 414 / 642; of 23
// 598 / 735 and 563 / 770; of 87 1382 / 1398 and 1361 / 1388; of 289 2874 / 2868 and
// 2881 / 2863; of 1154 (10 views) 2199 / 2191 and 2207 / 2154.
constexpr int64_t kLongLists = 128;

// Orders one wave's LDS accesses.
__device__ __forceinline__ void lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// One step of the walk: the weight w = alpha T of the Gaussian of record
// (a, b) = ((cx, cy, L11, L12), (L22, opacity, -, -)) at the pixel (pxo, pyo),
// 0 where it takes no part.  A pixel that is done (the Gaussian that would take
// its transmittance below 1e-4, which is not counted, has been met) or outside
// the image has T = 0; otherwise T >= 1e-4, so a counted weight is at least
// 1e-4 / 255 and w != 0 says that the Gaussian is counted.  No masks besides T:
// a wave's hits are a serial chain, and a wave issues an instruction every four
// cycles at most, so the chain costs what its instructions do: with the state in
// lane masks, a branch around the row and its id stored by the lane that holds
// it, an uplift of 10k Gaussians into 4 views of 128x128, D = 8, took 165 us for
// the launch instead of 133, and one of a mask (200k Gaussians, 50 views of
// 512x384) 1.84 ms instead of 1.45.
__device__ __forceinline__ float blend_step(const float4& a, const float2& b, float pxo, float pyo, float& T) {
  const float dx = pxo - a.x, dy = pyo - a.y;
  const float u = __builtin_fmaf(a.w, dy, a.z * dx), w = b.x * dy;
  const float al = fminf(kAlphaMax, b.y * exp_neg(-__builtin_fmaf(u, u, w * w)));
  const float ac = al >= kAlphaMin ? al : 0.0f;
  const float Tn = T * (1.0f - ac);  // T where the Gaussian is skipped
  const bool on = Tn >= kTEps;
  const float wj = on ? ac * T : 0.0f;
  T = on ? Tn : 0.0f;
  return wj;
}

// Lanes with x != 0.
__device__ __forceinline__ uint64_t nonzero(float x) { return __builtin_amdgcn_ballot_w64(x != 0.0f); }

// ---------------------------------------------------------------- wide kernel
// Any number of feature sets; the workgroup's channel group has up to 64
// channels made of segments of the sets plus up to 4 tail channels (summed
// per LDS row at each flush).
//
// Accumulation on the matrix cores.  The weights of 32 queued Gaussians at
// the quadrant's 64 pixels form W_s (32 x 64), and their contribution to the
// group's channels is the dense product U_s = W_s F (F: 64 pixels x 64
// channels).  It runs as 32x32x16 BF16 MFMAs
// with FP32 accumulation on split operands: x = hi + lo, hi = bf16(x) and
// lo = bf16(x - hi) (both round-to-nearest-even), so |x - hi - lo| <=
// 2^-18 |x|; U_s = W_hi F_hi + W_lo F_hi + W_hi F_lo (the dropped W_lo F_lo
// and residuals are below 2^-16 |W| |F|;
// BF16 maps are exact, F_lo = 0).  A K-step of 16 pixels is two pixel rows of
// the quadrant: steps whose rows hold no contribution are skipped.  Operand
// layouts (32x32x16): lane l holds A[l % 32][8 (l / 32) + i] and
// B[8 (l / 32) + i][l % 32], i = 0..7, and D[8 (r / 4) + 4 (l / 32) + r % 4]
// [l % 32] in accumulator r.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kWtPitch = 68;  // LDS row pitch (floats) of the transposed weights

// x = hi + lo + O(2^-18 |x|), conversions round to nearest even
__device__ __forceinline__ void split8(const float (&x)[8], bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int i = 0; i < 8; i++) {
    hi[i] = (__bf16)x[i];
    lo[i] = (__bf16)(x[i] - (float)hi[i]);
  }
}

// A operand of one K-step: this lane's 8 weights (two float4 from LDS), split
__device__ __forceinline__ void load_split_w(const float* w, bf16x8& hi, bf16x8& lo) {
  const float4 wa = *reinterpret_cast<const float4*>(w);
  const float4 wb = *reinterpret_cast<const float4*>(w + 4);
  const float w8[8] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
  split8(w8, hi, lo);
}

// The same chunk after split_w_in_place: BF16 hi in its first 16 bytes, lo
// in the next 16.
__device__ __forceinline__ void load_w(const float* w, bf16x8& hi, bf16x8& lo) {
  hi = *reinterpret_cast<const bf16x8*>(w);
  lo = *reinterpret_cast<const bf16x8*>(w + 4);
}

__device__ __forceinline__ void split_w_in_place(float* w) {
  bf16x8 hi, lo;
  load_split_w(w, hi, lo);
  *reinterpret_cast<bf16x8*>(w) = hi;
  *reinterpret_cast<bf16x8*>(w + 4) = lo;
}

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Rows (8 pixels each) of a 64-pixel mask that hold a set bit.
__device__ __forceinline__ uint32_t row_bits(uint64_t m) {
  uint32_t r = 0;
#pragma unroll
  for (int k = 0; k < 8; k++) r |= (((m >> (8 * k)) & 0xFFull) != 0ull ? 1u : 0u) << k;
  return r;
}

// This lane's channel in each 32-channel block of a group (n = l % 32):
// where its features come from and where its sums go.
struct GroupLanes {
  float* outp[2];
  int outD[2];
  const void* src[2];  // a readable map even where the lane owns no channel
  bool own[2];         // the lane owns a channel of block b
  int64_t srcc[2];
  int srcld[2];
  float srcsc[2];
};

// Fills L for group grp and view q.v; false if no segment of the group takes
// the view (wave-uniform).
template <lv_dtype DT>
__device__ __forceinline__ bool group_lanes(const ChanGroup& grp, const SetDesc* __restrict__ sets,
                                            const Quad& q, int lane, GroupLanes& L) {
  bool active = false;
#pragma unroll
  for (int b = 0; b < 2; b++) {
    L.outp[b] = nullptr;
    L.outD[b] = 0;
    L.src[b] = nullptr;
    L.own[b] = false;
    L.srcc[b] = 0;
    L.srcld[b] = 0;
    L.srcsc[b] = 1.0f;
  }
  for (int k = 0; k < grp.nseg; k++) {
    const SetDesc& sd = sets[grp.set[k]];
    const void* map = map_of(sd, q.v);
    if (!map) continue;  // this set does not take the view
    active = true;
    const int vc0 = grp.vc0[k], cnt = grp.cnt[k];
#pragma unroll
    for (int b = 0; b < 2; b++) {
      const int ch = b * 32 + (lane & 31);
      if (!L.src[b]) L.src[b] = map;  // readable, for lanes without a channel
      if (ch >= vc0 && ch < vc0 + cnt) {
        const int c = grp.c0[k] + (ch - vc0);
        L.outp[b] = u_elem(sd.U, c, sd.fixed != 0);
        L.outD[b] = sd.D;
        L.src[b] = map;
        L.own[b] = true;
        L.srcc[b] = c;
        L.srcld[b] = sd.stride;
        if constexpr (DT == LV_FP8_E4M3) L.srcsc[b] = gptr(sd.scales)[(int64_t)(sd.view_base + q.v) * sd.D + c];
      }
    }
  }
  return active;
}

// Element (y, x, channel c) of a map with pixel stride ld: HWC at
// (y W + x) ld + c; pixel-block layout (PX8) at ((y W8 + x / 8) ld + c) 8 +
// x % 8 with W8 = ceil(W / 8) (pixels past W are zeros).
template <bool PX>
__device__ __forceinline__ int64_t map_index(int y, int x, int W, int ld, int64_t c) {
  if constexpr (PX)
    return (((int64_t)y * ((W + 7) >> 3) + (x >> 3)) * ld + c) * 8 + (x & 7);
  else
    return ((int64_t)y * W + x) * ld + c;
}

// Four OCP E4M3FN codes (the bytes of w) -> their values as BF16 bits, two
// per word: the hardware FP8 -> FP32 conversion (two codes per
// instruction), then FP32 -> BF16 (exact: 3 mantissa bits).
__device__ __forceinline__ void e4m3x4_bf16(uint32_t w, uint32_t& h01, uint32_t& h23) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const f32x2 a = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, false);
  const f32x2 b = __builtin_amdgcn_cvt_pk_f32_fp8((int)w, true);
  h01 = __builtin_bit_cast(uint32_t, (bf16x2{(__bf16)a.x, (__bf16)a.y}));
  h23 = __builtin_bit_cast(uint32_t, (bf16x2{(__bf16)b.x, (__bf16)b.y}));
}

__device__ __forceinline__ bf16x8 bf16x8_of(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3) {
  return __builtin_bit_cast(bf16x8, (u32x4{w0, w1, w2, w3}));
}

// The B operand of one K-step for block b: this lane's channel at the 8
// pixels (gx0 .. gx0 + 7, gx0 a multiple of 8) of pixel row gy, as BF16
// (hi; lo = the FP32 remainder, FP32 maps only).  BF16 maps are exact in hi;
// FP8 codes too (their per-channel scale multiplies the products, see
// batch_scatter).  Every lane loads, from a safe index (block or pixel 0 of
// the map) where it has nothing to load.  Pixel blocks: the data is used as
// loaded -- a lane without a channel feeds only its own output column, which
// is never scattered, and a pixel outside the image has weight 0 in every
// queued row.  (A select of zeros there becomes a zero fill of the
// destination registers plus a masked load, and the fill waits for every
// memory operation in flight: a group's K-steps would load one round trip at
// a time.)  HWC: eight gathers per row, selected (zeros outside the image
// and for lanes without a channel), which keeps them from all being in
// flight at once.
template <lv_dtype DT, bool PX>
__device__ __forceinline__ void load_row8(const GroupLanes& L, int b, int gy, int gx0,
                                          const ViewGeom& g, bf16x8& fh, bf16x8& fl) {
  const bool okr = L.own[b] && gy < g.H;
  if constexpr (PX) {
    // one block of 8 pixels of one channel: 32, 16 or 8 contiguous bytes
    const int64_t blk = okr ? ((int64_t)gy * ((g.W + 7) >> 3) + (gx0 >> 3)) * L.srcld[b] + L.srcc[b] : 0;
    if constexpr (DT == LV_BF16) {
      const u32x4 q = gptr(static_cast<const u32x4*>(L.src[b]))[blk];
      fh = bf16x8_of(q.x, q.y, q.z, q.w);
    } else if constexpr (DT == LV_FP8_E4M3) {
      const u32x2 q = gptr(static_cast<const u32x2*>(L.src[b]))[blk];
      uint32_t h[4];
      e4m3x4_bf16(q.x, h[0], h[1]);
      e4m3x4_bf16(q.y, h[2], h[3]);
      fh = bf16x8_of(h[0], h[1], h[2], h[3]);
    } else {
      const f32x4 qa = gptr(static_cast<const f32x4*>(L.src[b]))[2 * blk];
      const f32x4 qb = gptr(static_cast<const f32x4*>(L.src[b]))[2 * blk + 1];
      const float v[8] = {qa.x, qa.y, qa.z, qa.w, qb.x, qb.y, qb.z, qb.w};
      split8(v, fh, fl);
    }
  } else {
    if constexpr (DT == LV_F32) {
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; i++) {
        const bool ok = okr && gx0 + i < g.W;
        const int64_t idx = ok ? ((int64_t)gy * g.W + gx0 + i) * L.srcld[b] + L.srcc[b] : 0;
        const float x = gptr(static_cast<const float*>(L.src[b]))[idx];
        v[i] = ok ? x : 0.0f;
      }
      split8(v, fh, fl);
    } else {
      uint32_t h[8];
#pragma unroll
      for (int i = 0; i < 8; i++) {
        const bool ok = okr && gx0 + i < g.W;
        const int64_t idx = ok ? ((int64_t)gy * g.W + gx0 + i) * L.srcld[b] + L.srcc[b] : 0;
        uint32_t x;
        if constexpr (DT == LV_BF16)
          x = gptr(static_cast<const uint16_t*>(L.src[b]))[idx];
        else
          x = gptr(static_cast<const uint8_t*>(L.src[b]))[idx];
        h[i] = ok ? x : 0u;
      }
      if constexpr (DT == LV_BF16) {
        fh = bf16x8_of(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
      } else {
        uint32_t o[4];
        e4m3x4_bf16(h[0] | (h[1] << 8) | (h[2] << 16) | (h[3] << 24), o[0], o[1]);
        e4m3x4_bf16(h[4] | (h[5] << 8) | (h[6] << 16) | (h[7] << 24), o[2], o[3]);
        fh = bf16x8_of(o[0], o[1], o[2], o[3]);
      }
    }
  }
}

// U_b = W_b F for a batch of queued rows, one or two blocks of 32 channels.
// No branch separates dependent MFMAs (the widths run in separate loops).
template <bool kSplitF>
__device__ __forceinline__ void batch_mfma(bool two, uint32_t rows, const float* wrow,
                                           const bf16x8 (&fh)[2][4], const bf16x8 (&fl)[2][4],
                                           f32x16& acc0, f32x16& acc1) {
  if (two) {
#pragma unroll
    for (int t = 0; t < 4; t++) {
      if ((rows >> (2 * t)) & 3u) {
        bf16x8 ah, al;
        load_split_w(wrow + 16 * t, ah, al);
        acc0 = mfma(ah, fh[0][t], acc0);
        acc1 = mfma(ah, fh[1][t], acc1);
        acc0 = mfma(al, fh[0][t], acc0);
        acc1 = mfma(al, fh[1][t], acc1);
        if constexpr (kSplitF) {
          acc0 = mfma(ah, fl[0][t], acc0);
          acc1 = mfma(ah, fl[1][t], acc1);
        }
      }
    }
  } else {
#pragma unroll
    for (int t = 0; t < 4; t++) {
      if ((rows >> (2 * t)) & 3u) {
        bf16x8 ah, al;
        load_split_w(wrow + 16 * t, ah, al);
        acc0 = mfma(ah, fh[0][t], acc0);
        acc0 = mfma(al, fh[0][t], acc0);
        if constexpr (kSplitF) acc0 = mfma(ah, fl[0][t], acc0);
      }
    }
  }
}

// One atomic per (queued Gaussian, channel): D row m of the batch is ring
// row m, whose Gaussian id lane m holds.  rows: how many rows are added, or
// (kMask) which.  FP8 maps: the products were formed on the codes, the
// channel's scale multiplies them here.
template <lv_dtype DT, bool FIX, bool kMask>
__device__ __forceinline__ void batch_scatter_t(const GroupLanes& L, bool two, uint32_t rows,
                                                uint32_t ring_gid, int lane, f32x16 acc0,
                                                f32x16 acc1) {
  if constexpr (DT == LV_FP8_E4M3) {
    acc0 *= L.srcsc[0];
    acc1 *= L.srcsc[1];
  }
  const bool upper = lane >= 32;
  const int count = (int)rows;
  const uint32_t mine = upper ? rows >> 4 : rows;
#pragma unroll
  for (int r = 0; r < 16; r++) {
    const int m0 = 8 * (r >> 2) + (r & 3), m1 = m0 + 4;
    if (kMask ? ((rows >> m0) & 0x11u) != 0u : m0 < count) {  // wave-uniform
      const uint32_t g0 = (uint32_t)__builtin_amdgcn_readlane((int)ring_gid, m0);
      const uint32_t g1 = (uint32_t)__builtin_amdgcn_readlane((int)ring_gid, m1);
      const int64_t gid = (int64_t)(upper ? g1 : g0);
      if (kMask ? ((mine >> m0) & 1u) != 0u : (upper ? m1 : m0) < count) {
        if (L.outp[0] && acc0[r] != 0.0f) u_atomic_add(L.outp[0], gid * L.outD[0], acc0[r], FIX);
        if (two && L.outp[1] && acc1[r] != 0.0f) u_atomic_add(L.outp[1], gid * L.outD[1], acc1[r], FIX);
      }
    }
  }
}

// fixed (a deterministic accumulator) is wave-uniform: one branch per
// flush, each side a straight run of atomics
template <lv_dtype DT, bool kMask = false>
__device__ __forceinline__ void batch_scatter(const GroupLanes& L, bool two, uint32_t rows,
                                              uint32_t ring_gid, int lane, f32x16 acc0,
                                              f32x16 acc1, bool fixed) {
  if (fixed)
    batch_scatter_t<DT, true, kMask>(L, two, rows, ring_gid, lane, acc0, acc1);
  else
    batch_scatter_t<DT, false, kMask>(L, two, rows, ring_gid, lane, acc0, acc1);
}

// One channel group (at most 64 + 4 channels), one workgroup per (view,
// quadrant); the group's F fragments are staged once in registers.  Several
// groups run on blend_pair_kernel below.  The walk is a serial chain of
// instructions, the flush waits for the atomics' queue.  kTwo: the first wave
// walks and fills two queues of 32 rows in turn, the second flushes the one just
// filled, and they meet at one barrier per queue, which neither loads nor atomics
// in flight hold up; else one wave does both with one queue.  Two waves where
// the launch has few quadrants (kFewQuadrants), or where the group has more than
// 32 channels, whose flush is long, and the lists are long (kLongLists).  Launch,
// the walk before blend_step / one wave / two: 200k Gaussians, 50 views of
// 512x384, D = 64 in BF16 3.57 / 3.52 / 3.42 ms (the atomics' rate bounds it),
// D = 1 1.84 / 1.45 / 1.94; 20 views, D = 32 in FP32 1.04 / 0.98 / 0.96, in BF16
// 1.05 / 1.02 / 0.92; 20k Gaussians, 20 views of 800x600, D = 32 in FP32 0.99 /
// 0.88 / 1.08, D = 16 0.95 / 0.83 / 1.03; 10k Gaussians, 4 views of 128x128, D = 8
// 165 / 133 / 82 us; 50k Gaussians, nine launches of a 333x251 view, D = 37 455 /
// 445 / 390 us.
// kBlocks: blocks of 32 channels that the registers hold, 1 where the group has
// no more.  Occupancy: waves per SIMD the register allocation must allow.  BF16
// maps need no low operand halves, so they fit four, except that one wave with
// two blocks from HWC maps spills then (20 views of 800x600, 2000 Gaussians,
// D = 64: 527 us with four, 414 with three).
template <lv_dtype DT, bool PX, bool kTwo, int kBlocks>
constexpr int wide_waves() {
  return DT == LV_BF16 && (PX || kTwo || kBlocks == 1) ? 4 : 3;
}

template <lv_dtype DT, bool PX, bool kTwo, int kBlocks>
__global__ __launch_bounds__(kTwo ? 128 : 64, (wide_waves<DT, PX, kTwo, kBlocks>())) void blend_wide_kernel(
    const Rec* __restrict__ rec, const uint32_t* __restrict__ ids, const uint2* __restrict__ ranges,
    const ViewGeom* __restrict__ geom, int64_t n, int tiles_stride, int nviews,
    const SetDesc* __restrict__ sets, const ChanGroup* __restrict__ groups, int ngroups) {
  constexpr bool kSplitF = DT == LV_F32;  // BF16 maps and FP8 codes are exact in one BF16 operand
  constexpr int kQueues = kTwo ? 2 : 1;
  __shared__ __align__(16) float Wts[kQueues][32 * kWtPitch];  // queued Gaussians: [row][pixel]
  __shared__ uint64_t Pix[kQueues];                            // pixels used by the rows
  __shared__ int Count[kQueues];                               // rows, + 64 with the last ones
  // ids of the hits in order, hit k at k mod kIds: a queue's rows are
  // consecutive hits, and a step's ids are written all at once, at most 64 past
  // the queues
  constexpr int kIds = kTwo ? 256 : 128;
  __shared__ uint32_t Ids[kIds];
  __shared__ float4 Rs[kChunk][2];                   // the step's records
  // tail channels: their features per pixel, summed against the queued rows at
  // each flush
  __shared__ __align__(16) float Ft[kMaxTail * 64];
  Quad q;
  if (!decode_quad(ranges, geom, tiles_stride, nviews, ngroups, q)) return;
  const int lane = threadIdx.x & 63;
  // two waves: the first walks, the second flushes
  const bool flushes = !kTwo || __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) != 0;
  const bool fixedU = sets[0].fixed != 0;  // one accumulation mode per launch (wave-uniform)
  const int px = q.qx + (lane & 7), py = q.qy + (lane >> 3);
  const bool inside = px < q.g.W && py < q.g.H;

  // whether the group takes the view, sets whose beta (and counts) are added
  // here; its tail channels
  bool has_main = false;
  int bsets = 0, ssets = 0;
  {
    const ChanGroup& grp = groups[q.cg];
    for (int b = grp.beta_sets; b; b &= b - 1)
      if (map_of(sets[__builtin_ctz(b)], q.v)) bsets |= b & -b;
    for (int b = grp.stats_sets; b; b &= b - 1)
      if (map_of(sets[__builtin_ctz(b)], q.v)) ssets |= b & -b;
    for (int k = 0; k < grp.nseg; k++) has_main = has_main || map_of(sets[grp.set[k]], q.v) != nullptr;
  }
  const ChanGroup& last = groups[q.cg];
  const int ntail = last.ntail;
  bool any_tail = false;
  for (int t = 0; t < ntail; t++) any_tail = any_tail || map_of(sets[last.tset[t]], q.v) != nullptr;
  if (!has_main && !any_tail && !bsets && !ssets) return;  // wave-uniform: nothing here takes the view

  float* tout[kMaxTail];
  int tD[kMaxTail];
  GroupLanes L1;
  bf16x8 fh[2][4], fl[2][4];
  bool two1 = false;
  if (flushes) {
#pragma unroll
    for (int t = 0; t < kMaxTail; t++) {
      float ft = 0.0f;
      tout[t] = nullptr;
      tD[t] = 0;
      if (t < ntail && map_of(sets[last.tset[t]], q.v)) {
        const SetDesc& sd = sets[last.tset[t]];
        const int c = last.tc[t];
        float sc = 1.0f;
        if constexpr (DT == LV_FP8_E4M3) sc = gptr(sd.scales)[(int64_t)(sd.view_base + q.v) * sd.D + c];
        const int64_t idx = inside ? map_index<PX>(py, px, q.g.W, sd.stride, c) : 0;
        const float x = load_feature<DT>(map_of(sd, q.v), idx, sc);  // no branch around the load
        ft = inside ? x : 0.0f;
        tout[t] = u_elem(sd.U, c, fixedU);
        tD[t] = sd.D;
      }
      Ft[t * 64 + lane] = ft;
    }
    lds_order();  // Ft is written and read by this wave only

    // the group's lanes and fragments once, in registers
    {
      const ChanGroup& grp = groups[q.cg];
      const bool takes = group_lanes<DT>(grp, sets, q, lane, L1);
      two1 = kBlocks == 2 && grp.width > 32;
      if (takes) {
#pragma unroll
        for (int b = 0; b < kBlocks; b++)
#pragma unroll
          for (int t = 0; t < 4; t++)
            load_row8<DT, PX>(L1, b, q.qy + 2 * t + (lane >> 5), q.qx, q.g, fh[b][t], fl[b][t]);
      }
      has_main = has_main && takes && __ballot(L1.outp[0] != nullptr || L1.outp[1] != nullptr) != 0ull;
    }
  }
  // contributing pixels per row, where a set counts them
  bool counting = ssets != 0;
  for (int t = bsets; t; t &= t - 1) counting = counting || sets[__builtin_ctz(t)].counts != nullptr;
  uint32_t ncontrib = 0u, nrows = 0u;  // this lane's rows (statistics)

  // the rows of a queue, its first hit hit0, into the accumulators
  auto flush = [&](const float* Wt, int count, uint64_t pix, uint32_t hit0) {
    const uint32_t ring_gid = Ids[(hit0 + (uint32_t)(lane & 31)) % kIds];
    // the rows' sums.  lane l: row l % 32, pixels [32 (l / 32), 32 (l / 32) + 32)
    const float* rp = Wt + (lane & 31) * kWtPitch + 32 * (lane >> 5);
    const float* fp = Ft + 32 * (lane >> 5);
    float bs = 0.0f, ts[kMaxTail] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < 8; k++) {
      const float4 a = *reinterpret_cast<const float4*>(rp + 4 * k);
      bs += a.x;
      bs += a.y;
      bs += a.z;
      bs += a.w;
#pragma unroll
      for (int t = 0; t < kMaxTail; t++) {
        if (t < ntail) {  // wave-uniform
          const float4 f = *reinterpret_cast<const float4*>(fp + t * 64 + 4 * k);
          ts[t] = __builtin_fmaf(a.x, f.x, ts[t]);
          ts[t] = __builtin_fmaf(a.y, f.y, ts[t]);
          ts[t] = __builtin_fmaf(a.z, f.z, ts[t]);
          ts[t] = __builtin_fmaf(a.w, f.w, ts[t]);
        }
      }
    }
    bs += __shfl_xor(bs, 32, 64);
#pragma unroll
    for (int t = 0; t < kMaxTail; t++) ts[t] += __shfl_xor(ts[t], 32, 64);
    uint32_t ring_cnt = 0u;
    if (counting) {
#pragma unroll
      for (int k = 0; k < 8; k++) {
        const float4 a = *reinterpret_cast<const float4*>(rp + 4 * k);
        ring_cnt += (a.x != 0.0f ? 1u : 0u) + (a.y != 0.0f ? 1u : 0u) + (a.z != 0.0f ? 1u : 0u) +
                    (a.w != 0.0f ? 1u : 0u);
      }
      ring_cnt += (uint32_t)__shfl_xor((int)ring_cnt, 32, 64);
      if (lane < count) {
        ncontrib += ring_cnt;
        nrows += ring_cnt ? 1u : 0u;
      }
    }
    if (lane < count && bs != 0.0f) {  // lane r < 32: row r, whose id and count it holds
      for (int b = bsets; b; b &= b - 1) {
        const SetDesc& sd = sets[__builtin_ctz(b)];
        beta_atomic_add(sd.beta + ring_gid, bs);
        if (sd.counts) gatomic_add(sd.counts + ring_gid, ring_cnt);
      }
#pragma unroll
      for (int t = 0; t < kMaxTail; t++)
        if (tout[t] && ts[t] != 0.0f) u_atomic_add(tout[t], (int64_t)ring_gid * tD[t], ts[t], fixedU);
    }
    // Rows with a contribution (a weight is at least 1e-4 / 255, so their sum is
    // not 0).  The others are zeros and are not added: their products are zero
    // only where the features are finite, and a Gaussian that no pixel counts
    // takes nothing from the view, whatever the map holds there.
    const uint32_t live = (uint32_t)__ballot(bs != 0.0f && lane < count);
    if (has_main) {
      const uint32_t rows = row_bits(pix);
      const float* wrow = Wt + (lane & 31) * kWtPitch + 8 * (lane >> 5);
      f32x16 acc0 = {}, acc1 = {};
      batch_mfma<kSplitF>(two1, rows, wrow, fh, fl, acc0, acc1);
      batch_scatter<DT, true>(L1, two1, live, ring_gid, lane, acc0, acc1, fixedU);
    }
  };
  // statistics go to every set whose statistics this work item takes
  auto write_stats = [&](uint32_t covered) {
    for (int o = 32; o > 0; o >>= 1) {
      ncontrib += (uint32_t)__shfl_xor((int)ncontrib, o, 64);
      nrows += (uint32_t)__shfl_xor((int)nrows, o, 64);
    }
    for (int t = ssets; t; t &= t - 1) add_stats(sets[__builtin_ctz(t)], lane, covered, ncontrib, nrows);
  };

  if (kTwo && flushes) {
    uint32_t hit0 = 0u;  // the queue's first hit
    for (int b = 0;; b ^= 1) {
      lds_barrier();
      const int handed = __builtin_amdgcn_readfirstlane(Count[b]), count = handed & 63;
      if (count > 0) flush(Wts[b], count, Pix[b], hit0);
      hit0 += 32u;
      if (handed & 64) break;
    }
    write_stats(0u);
    return;
  }

  Walk s;
  walk_init(q, lane, s);
  uint64_t covered = 0ull;  // pixels with a contribution (statistics)
  Steps<kTwo> st;
  st.start(rec + (int64_t)q.v * n, ids, q.rg, lane);
  int b = 0, queued = 0;    // rows [0, queued) of queue b hold hits
  uint32_t hits_done = 0u;  // hits before the step
  uint32_t hit0 = 0u;       // the queue's first hit
  float used = 0.0f;        // not 0 where the pixel has a weight in the queue
  float* wrow = Wts[0] + lane;
  // a full or last queue: flushed, or handed to the other wave, which has
  // emptied the other queue when it arrives
  auto hand_over = [&](int count) {
    const uint64_t pix = nonzero(used);
    covered |= pix;
    if constexpr (kTwo) {
      if (lane == 0) {
        Pix[b] = pix;
        Count[b] = count;
      }
      lds_barrier();
      b ^= 1;
    } else {
      lds_order();
      if (count & 63) flush(Wts[0], count & 63, pix, hit0);
      lds_order();
      hit0 += 32u;
    }
    queued = 0;
    used = 0.0f;
    wrow = Wts[b] + lane;
  };
  for (uint32_t base = q.rg.x; base < q.rg.y; base += kChunk) {
    if (nonzero(s.T) == 0ull) break;
    uint32_t my_id;
    uint64_t h = step_records(st, base, lane, s, my_id, Rs);
    if (!h) continue;
    if ((h >> lane) & 1ull)
      Ids[(hits_done + (uint32_t)__popcll(h & ((1ull << lane) - 1ull))) % kIds] = my_id;
    hits_done += (uint32_t)__popcll(h);
    lds_order();  // records in LDS
    // the hit Gaussians in order (a scalar loop over the set bits; each
    // record read from LDS, a broadcast, one hit ahead): each takes the next
    // row, also where it has no contribution (its row is then zeros and is left
    // out at the flush: nearly every hit has one, and a test would cost each hit
    // more than the few rows); a full queue is handed over
    int j = (int)__builtin_ctzll(h);
    float4 ra = Rs[j][0];
    float2 rb = *reinterpret_cast<const float2*>(&Rs[j][1]);
    do {
      h &= ~(1ull << j);
      j = (int)__builtin_ctzll(h | (1ull << 63));  // 63 after the last: a readable record
      const float4 ca = ra;
      const float2 cb = rb;
      ra = Rs[j][0];
      rb = *reinterpret_cast<const float2*>(&Rs[j][1]);
      const float wj = blend_step(ca, cb, s.pxo, s.pyo, s.T);
      *wrow = wj;
      wrow += kWtPitch;
      used = fmaxf(used, wj);
      if (++queued == 32) hand_over(32);
    } while (h);
    lds_order();  // the records are read before the next step's
  }
  hand_over(queued + 64);
  write_stats((uint32_t)__popcll(covered));
}

// ------------------------------------------------------------- pair kernel
// Several channel groups (wide D): one wave per (view, tile, half tile), the
// two 8x8 quadrants of a 16x8 half tile, two pixels per lane (lane l covers
// pixel (l % 8, l / 8) of each quadrant).  A Gaussian that reaches both
// quadrants queues one row of 128 weights instead of two rows of 64, so a
// (Gaussian, view) adds about 0.7 times as many partial sums to U as with one
// wave per quadrant -- each partial sum is D atomic adds, the binding cost at
// large D.  The walk evaluates a Gaussian only at the quadrants its
// alpha >= 1/255 region reaches.  Pixel p of a queued row: quadrant p / 64,
// pixel p % 64 of it (row-major 8x8); K-step t of the products (16 pixels)
// is pixel rows 2 (t % 4), 2 (t % 4) + 1 of quadrant t / 4.
constexpr int kPairPitch = 132;  // LDS row pitch (floats) of the 128 queued weights

struct Pair {
  int v, tile, qx, qy;  // qx, qy: the half tile's first pixel
  uint2 rg;
  ViewGeom g;
};

// The two halves of a tile get consecutive ids on the same XCD (ids equal
// mod 8), so they share that XCD's L2 for the tile's records.
__device__ __forceinline__ bool decode_pair(const uint2* __restrict__ ranges,
                                            const ViewGeom* __restrict__ geom, int tiles_stride,
                                            int nviews, Pair& q) {
  const uint32_t L = blockIdx.x;
  const uint32_t kx = L >> 3;
  const uint32_t work = ((kx >> 1) << 3) | (L & 7u);
  if (work >= (uint32_t)tiles_stride * (uint32_t)nviews) return false;
  const int half = (int)(kx & 1u);
  q.tile = (int)(work % (uint32_t)tiles_stride);
  q.v = (int)(work / (uint32_t)tiles_stride);
  q.g = geom[q.v];
  if (q.tile >= q.g.TX * q.g.TY) return false;
  q.rg = ranges[(int64_t)q.v * tiles_stride + q.tile];
  if (q.rg.y <= q.rg.x) return false;
  const int tx = q.tile % q.g.TX, ty = q.tile / q.g.TX;
  q.qx = tx * kTile;
  q.qy = ty * kTile + half * 8;
  return q.qx < q.g.W && q.qy < q.g.H;
}

// group_lanes for a half tile (only the view matters)
template <lv_dtype DT>
__device__ __forceinline__ bool group_lanes_pair(const ChanGroup& grp, const SetDesc* __restrict__ sets,
                                                 const Pair& p, int lane, GroupLanes& L) {
  Quad q;
  q.v = p.v;
  return group_lanes<DT>(grp, sets, q, lane, L);
}

template <lv_dtype DT, bool PX>
__global__ __launch_bounds__(64, 2) void blend_pair_kernel(
    const Rec* __restrict__ rec, const uint32_t* __restrict__ ids, const uint2* __restrict__ ranges,
    const ViewGeom* __restrict__ geom, int64_t n, int tiles_stride, int nviews,
    const SetDesc* __restrict__ sets, const ChanGroup* __restrict__ groups, int ngroups) {
  constexpr int G = kChunk;
  constexpr bool kSplitF = DT == LV_F32;
  __shared__ __align__(16) float Wt[32 * kPairPitch];  // queued Gaussians: [row][128 pixels]
  __shared__ float4 Rs[kChunk][2];                     // the step's records
  // tail channels per pixel [kMaxTail][128]: dynamic, allocated only when the
  // last group has a tail (without it the workgroup's 19.2 KB of LDS lets 8
  // workgroups share a CU instead of 7)
  extern __shared__ __align__(16) float Ft[];
  __shared__ uint32_t Rg[32], Rc[32];
  Pair q;
  if (!decode_pair(ranges, geom, tiles_stride, nviews, q)) return;
  const int lane = threadIdx.x;
  const bool fixedU = sets[0].fixed != 0;  // one accumulation mode per launch (wave-uniform)
  const int ox = q.qx, oy = q.qy & ~(kTile - 1);
  const float ocx = (float)ox + 0.5f, ocy = (float)oy + 0.5f;
  const float pyo = (float)(q.qy - oy + (lane >> 3));
  const float pxo0 = (float)(lane & 7), pxo1 = pxo0 + 8.0f;
  const float qy0 = (float)(q.qy - oy);
  const int py = q.qy + (lane >> 3);
  const bool in0 = q.qx + (lane & 7) < q.g.W && py < q.g.H;
  const bool in1 = q.qx + 8 + (lane & 7) < q.g.W && py < q.g.H;

  bool has_main = false;
  int bsets = 0, ssets = 0;
  uint32_t gmask = 0u;
  for (int cg = 0; cg < ngroups; cg++) {
    const ChanGroup& grp = groups[cg];
    for (int b = grp.beta_sets; b; b &= b - 1)
      if (map_of(sets[__builtin_ctz(b)], q.v)) bsets |= b & -b;
    for (int b = grp.stats_sets; b; b &= b - 1)
      if (map_of(sets[__builtin_ctz(b)], q.v)) ssets |= b & -b;
    bool any = false;
    for (int k = 0; k < grp.nseg; k++) any = any || map_of(sets[grp.set[k]], q.v) != nullptr;
    if (any) {
      gmask |= 1u << cg;
      has_main = true;
    }
  }
  const ChanGroup& last = groups[ngroups - 1];
  const int ntail = last.ntail;
  float* tout[kMaxTail];
  int tD[kMaxTail];
  bool any_tail = false;
#pragma unroll
  for (int t = 0; t < kMaxTail; t++) {
    float ft0 = 0.0f, ft1 = 0.0f;
    tout[t] = nullptr;
    tD[t] = 0;
    if (t < ntail && map_of(sets[last.tset[t]], q.v)) {
      const SetDesc& sd = sets[last.tset[t]];
      const int c = last.tc[t];
      float sc = 1.0f;
      if constexpr (DT == LV_FP8_E4M3) sc = gptr(sd.scales)[(int64_t)(sd.view_base + q.v) * sd.D + c];
      const int64_t i0 = in0 ? map_index<PX>(py, q.qx + (lane & 7), q.g.W, sd.stride, c) : 0;
      const int64_t i1 = in1 ? map_index<PX>(py, q.qx + 8 + (lane & 7), q.g.W, sd.stride, c) : 0;
      const float x0 = load_feature<DT>(map_of(sd, q.v), i0, sc);  // no branch around the loads
      const float x1 = load_feature<DT>(map_of(sd, q.v), i1, sc);
      ft0 = in0 ? x0 : 0.0f;
      ft1 = in1 ? x1 : 0.0f;
      tout[t] = u_elem(sd.U, c, fixedU);
      tD[t] = sd.D;
      any_tail = true;
    }
    if (t < ntail) {  // wave-uniform
      Ft[t * 128 + lane] = ft0;
      Ft[t * 128 + 64 + lane] = ft1;
    }
  }
  if (!has_main && !any_tail && !bsets && !ssets) return;  // wave-uniform

  float T0 = in0 ? 1.0f : 0.0f, T1 = in1 ? 1.0f : 0.0f;  // see Walk
  uint64_t cov0 = 0ull, cov1 = 0ull;
  uint32_t ncontrib = 0u, nrows = 0u;
  int queued = 0;
  uint64_t pix0 = 0ull, pix1 = 0ull;  // pixels of each quadrant used by the queued rows
  auto flush = [&](int count) {
    __syncthreads();  // queued rows written (one wave per workgroup: orders LDS)
    const uint32_t ring_gid = Rg[lane & 31], ring_cnt = Rc[lane & 31];
    cov0 |= pix0;
    cov1 |= pix1;
    nrows += (uint32_t)count;
    // bit r: pixel row r % 8 of quadrant r / 8; K-step t covers bits 2t, 2t + 1
    const uint32_t rows = row_bits(pix0) | (row_bits(pix1) << 8);
    const float* wrow = Wt + (lane & 31) * kPairPitch + 8 * (lane >> 5);
    if (bsets || any_tail) {
      // lane l: row l % 32, the pixels of quadrant l / 32
      const float* rp = Wt + (lane & 31) * kPairPitch + 64 * (lane >> 5);
      const float* fp = Ft + 64 * (lane >> 5);
      float bs = 0.0f, ts[kMaxTail] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int k = 0; k < 16; k++) {
        const float4 a = *reinterpret_cast<const float4*>(rp + 4 * k);
        bs += a.x;
        bs += a.y;
        bs += a.z;
        bs += a.w;
#pragma unroll
        for (int t = 0; t < kMaxTail; t++) {
          if (t < ntail) {  // wave-uniform
            const float4 f = *reinterpret_cast<const float4*>(fp + t * 128 + 4 * k);
            ts[t] = __builtin_fmaf(a.x, f.x, ts[t]);
            ts[t] = __builtin_fmaf(a.y, f.y, ts[t]);
            ts[t] = __builtin_fmaf(a.z, f.z, ts[t]);
            ts[t] = __builtin_fmaf(a.w, f.w, ts[t]);
          }
        }
      }
      bs += __shfl_xor(bs, 32, 64);
#pragma unroll
      for (int t = 0; t < kMaxTail; t++) ts[t] += __shfl_xor(ts[t], 32, 64);
      if (lane < count) {
        for (int b = bsets; b; b &= b - 1) {
          const SetDesc& sd = sets[__builtin_ctz(b)];
          beta_atomic_add(sd.beta + ring_gid, bs);
          if (sd.counts) gatomic_add(sd.counts + ring_gid, ring_cnt);
        }
#pragma unroll
        for (int t = 0; t < kMaxTail; t++)
          if (tout[t] && ts[t] != 0.0f) u_atomic_add(tout[t], (int64_t)ring_gid * tD[t], ts[t], fixedU);
      }
      __syncthreads();  // the FP32 weights read before they are split
    }
    // the weights of this lane's operand chunks (row l % 32, pixels
    // 16 t + 8 (l / 32) + [0, 8)) split once into BF16 hi and lo in place,
    // for all groups; each lane splits exactly the chunks it reads (the FP32
    // weights' other reader, the beta and tail sums above, is done)
#pragma unroll
    for (int t = 0; t < 8; t++)
      if ((rows >> (2 * t)) & 3u) split_w_in_place(Wt + (lane & 31) * kPairPitch + 8 * (lane >> 5) + 16 * t);
    if constexpr (!kSplitF && PX) {
      // BF16 / FP8 pixel-block maps: one operand load per K-step and block
      // (the HWC layout's eight loads per operand leave no registers for
      // this).  A group's products go out (one atomic per channel) only
      // after the next group's operand loads have been issued: the vector
      // memory counter completes in order, so waiting for those loads does
      // not wait for the atomics.
      GroupLanes Lp;  // the group whose products are pending
      bool pend = false, twop = false;
      f32x16 acc0 = {}, acc1 = {};
      for (int cg = 0; cg < ngroups; cg++) {
        GroupLanes L;
        const bool ok = ((gmask >> cg) & 1u) && group_lanes_pair<DT>(groups[cg], sets, q, lane, L);
        const bool two = groups[cg].width > 32;
        bf16x8 F[2][8];
        if (ok) {
#pragma unroll
          for (int t = 0; t < 8; t++) {
            if ((rows >> (2 * t)) & 3u) {
              bf16x8 lo;
              const int gy = q.qy + 2 * (t & 3) + (lane >> 5), gx0 = q.qx + 8 * (t >> 2);
              load_row8<DT, PX>(L, 0, gy, gx0, q.g, F[0][t], lo);
              if (two) load_row8<DT, PX>(L, 1, gy, gx0, q.g, F[1][t], lo);
            }
          }
        }
        if (pend) batch_scatter<DT>(Lp, twop, count, ring_gid, lane, acc0, acc1, fixedU);
        pend = false;
        if (!ok) continue;
        acc0 = f32x16{};
        acc1 = f32x16{};
        if (two) {
#pragma unroll
          for (int t = 0; t < 8; t++) {
            if ((rows >> (2 * t)) & 3u) {
              bf16x8 ah, al;
              load_w(wrow + 16 * t, ah, al);
              acc0 = mfma(ah, F[0][t], acc0);
              acc1 = mfma(ah, F[1][t], acc1);
              acc0 = mfma(al, F[0][t], acc0);
              acc1 = mfma(al, F[1][t], acc1);
            }
          }
        } else {
#pragma unroll
          for (int t = 0; t < 8; t++) {
            if ((rows >> (2 * t)) & 3u) {
              bf16x8 ah, al;
              load_w(wrow + 16 * t, ah, al);
              acc0 = mfma(ah, F[0][t], acc0);
              acc0 = mfma(al, F[0][t], acc0);
            }
          }
        }
        Lp = L;
        twop = two;
        pend = true;
      }
      if (pend) batch_scatter<DT>(Lp, twop, count, ring_gid, lane, acc0, acc1, fixedU);
    } else {
      for (int cg = 0; cg < ngroups; cg++) {
        if (!((gmask >> cg) & 1u)) continue;
        const ChanGroup& grp = groups[cg];
        GroupLanes L;
        if (!group_lanes_pair<DT>(grp, sets, q, lane, L)) continue;
        const bool two = grp.width > 32;
        f32x16 acc0 = {}, acc1 = {};
        if (two) {
  #pragma unroll
          for (int t = 0; t < 8; t++) {
            if ((rows >> (2 * t)) & 3u) {
              bf16x8 h0, l0, h1, l1, ah, al;
              const int gy = q.qy + 2 * (t & 3) + (lane >> 5), gx0 = q.qx + 8 * (t >> 2);
              load_row8<DT, PX>(L, 0, gy, gx0, q.g, h0, l0);
              load_row8<DT, PX>(L, 1, gy, gx0, q.g, h1, l1);
              load_w(wrow + 16 * t, ah, al);
              acc0 = mfma(ah, h0, acc0);
              acc1 = mfma(ah, h1, acc1);
              acc0 = mfma(al, h0, acc0);
              acc1 = mfma(al, h1, acc1);
              if constexpr (kSplitF) {
                acc0 = mfma(ah, l0, acc0);
                acc1 = mfma(ah, l1, acc1);
              }
            }
          }
        } else {
  #pragma unroll
          for (int t = 0; t < 8; t++) {
            if ((rows >> (2 * t)) & 3u) {
              bf16x8 h0, l0, ah, al;
              load_row8<DT, PX>(L, 0, q.qy + 2 * (t & 3) + (lane >> 5), q.qx + 8 * (t >> 2), q.g, h0, l0);
              load_w(wrow + 16 * t, ah, al);
              acc0 = mfma(ah, h0, acc0);
              acc0 = mfma(al, h0, acc0);
              if constexpr (kSplitF) acc0 = mfma(ah, l0, acc0);
            }
          }
        }
        batch_scatter<DT>(L, two, count, ring_gid, lane, acc0, acc1, fixedU);
      }
    }
    __syncthreads();  // rows read before they are written again
  };

  const Rec* vrec = rec + (int64_t)q.v * n;
  for (uint32_t base = q.rg.x; base < q.rg.y; base += G) {
    if ((nonzero(T0) | nonzero(T1)) == 0ull) break;
    const int cnt = (int)(q.rg.y - base < (uint32_t)G ? q.rg.y - base : (uint32_t)G);
    // lane j: record j, centre made tile-relative, left in LDS; hit masks of
    // the two quadrants
    float4 r0 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    float4 r1 = make_float4(0.0f, 0.0f, -1.0f, 0.0f);
    uint32_t my_id = 0;
    if (lane < cnt) {
      my_id = ids[base + lane];
      r0 = vrec[my_id].r0;
      r1 = vrec[my_id].r1;
      const uint32_t lo = __float_as_uint(r1.w);
      r0.x = (r0.x - ocx) + __uint_as_float(lo << 16);
      r0.y = (r0.y - ocy) + __uint_as_float(lo & 0xFFFF0000u);
    }
    Rs[lane][0] = r0;
    Rs[lane][1] = r1;
    const float X0 = -r0.x, Y0 = qy0 - r0.y;
    const bool h0 = lane < cnt && region_hits(r0, r1, X0, X0 + 7.0f, Y0, Y0 + 7.0f);
    const bool h1 = lane < cnt && region_hits(r0, r1, X0 + 8.0f, X0 + 15.0f, Y0, Y0 + 7.0f);
    const uint64_t hits0 = __ballot(h0), hits1 = __ballot(h1);
    uint64_t h = hits0 | hits1;
    if (!h) continue;
    __syncthreads();  // records in LDS
    while (h) {
      const int j = (int)__builtin_ctzll(h);
      h &= h - 1;
      const float4 a = Rs[j][0];
      const float2 b = *reinterpret_cast<const float2*>(&Rs[j][1]);
      float w0 = 0.0f, w1 = 0.0f;
      if ((hits0 >> j) & 1ull) w0 = blend_step(a, b, pxo0, pyo, T0);
      if ((hits1 >> j) & 1ull) w1 = blend_step(a, b, pxo1, pyo, T1);
      const uint64_t m0 = nonzero(w0), m1 = nonzero(w1);
      const uint32_t c = (uint32_t)(__popcll(m0) + __popcll(m1));
      Wt[queued * kPairPitch + lane] = w0;
      Wt[queued * kPairPitch + 64 + lane] = w1;
      Rg[queued] = (uint32_t)__builtin_amdgcn_readlane((int)my_id, j);  // every lane the same
      Rc[queued] = c;
      ncontrib += c;
      pix0 |= m0;
      pix1 |= m1;
      queued += (m0 | m1) != 0ull ? 1 : 0;
      if (queued == 32) {
        flush(32);
        queued = 0;
        pix0 = pix1 = 0ull;
      }
    }
  }
  if (queued > 0) flush(queued);
  for (int b = ssets; b; b &= b - 1) {
    add_stats(sets[__builtin_ctz(b)], lane, (uint32_t)(__popcll(cov0) + __popcll(cov1)), ncontrib, nrows);
  }
}

template <lv_dtype DT, bool PX>
hipError_t launch_blend_t(const BlendArgs& a, int m, hipStream_t s) {
  // one group: one workgroup per (view, quadrant); several: one wave per
  // (view, half tile) for all groups, sharing the walk
  const bool multi = a.ngroups > 1;
  int64_t work = (int64_t)a.tiles_stride * m;
  int64_t blocks = (work + 7) / 8 * 32;
  const bool two = 4 * work <= kFewQuadrants || (a.max_width > 32 && a.pairs >= kLongLists * work);
  if (multi) {
    // one wave per half tile: two per tile, whole rounds of 8 XCDs
    const int64_t pblocks = ((int64_t)a.tiles_stride * m + 7) / 8 * 16;
    const size_t tail_lds = a.has_tail ? sizeof(float) * kMaxTail * 128 : 0;
    hipLaunchKernelGGL((blend_pair_kernel<DT, PX>), dim3((unsigned)pblocks), dim3(64), tail_lds, s, a.rec,
                       a.ids, a.ranges, a.geom, a.n, a.tiles_stride, m, a.sets, a.groups,
                       a.ngroups);
  } else
    hipLaunchKernelGGL((two                ? blend_wide_kernel<DT, PX, true, 2>
                        : a.max_width > 32 ? blend_wide_kernel<DT, PX, false, 2>
                                           : blend_wide_kernel<DT, PX, false, 1>),
                       dim3((unsigned)blocks), dim3(two ? 128 : 64), 0, s, a.rec, a.ids, a.ranges, a.geom, a.n,
                       a.tiles_stride, m, a.sets, a.groups, a.ngroups);
  return hipGetLastError();
}

// ------------------------------------------------------------ forward render
// Eq. (4): F^(p) = sum_i w_i(p) g_i, the adjoint of the uplift.  One workgroup
// per (view, quadrant) and one or three groups of 32 NB channels walks the
// tile's list as the uplift does and, for each queue of up to 32 LDS rows, adds
// out (64 pixels x 32 NB channels) += W^T (64 x 32 rows) G (32 rows x 32 NB
// channels) on the matrix cores, split BF16 operands as in the uplift, the
// 2 x NB 32x32 output blocks held in registers until the walk ends; each (pixel,
// channel) is then written once.  The opacity sum_i w_i(p) goes to alpha[v]
// (group 0).  NB = 1 for D <= 32, 2 for D <= 64, else 4 (128 registers of output
// blocks, two waves per SIMD).
// The walk is a serial chain, the products wait for rows of g.  kSplit: the
// first wave walks and fills two queues in turn, each other wave takes a group
// of channels and the queue just filled; else one wave does both for its group.
// Split where the launch has few quadrants (half of kFewQuadrants at NB = 4,
// whose registers leave room for two waves a SIMD: D = 128, 1536 quadrants, 91
// us as one wave / 79 split; 3072: 75 / 88) and where the groups are a multiple
// of three, which share one walk: 6 views of 1008x756, 1M Gaussians, D = 384,
// 3.64 ms as three workgroups / 3.46 sharing; 8 views of 512x384, D = 257, 1.59
// / 1.39, D = 384 1.28 / 1.31.  Two groups sharing a walk lose (D = 256: 0.88 /
// 1.14 ms), and so does a last workgroup with idle waves (D = 385: 2.16 / 2.79).
// Before the walk of blend_step, one wave per group: D = 384 as above 3.99 ms, 4
// views of 512x384 with D = 3 155 us, now 136.
// kVec: D is a multiple of NB and g and the outputs are aligned to NB floats;
// a lane's channels are then consecutive (channel NB (l % 32) + b in block b),
// and each row of g and each output pixel is one load or store of NB floats
// instead of NB (4.89 -> 3.99 ms on the first job above).  Else block b's
// channels are 32 b + l % 32.
constexpr int kRenderWaves = 3;  // channel groups that share a walk

template <int NB, bool kVec, bool kSplit>
__global__ __launch_bounds__(kSplit ? 64 * (1 + (NB == 4 ? kRenderWaves : 1)) : 64,
                             (NB == 1 ? 4 : NB == 2 ? 3 : 2)) void render_kernel(
    const Rec* __restrict__ rec, const uint32_t* __restrict__ ids, const uint2* __restrict__ ranges,
    const ViewGeom* __restrict__ geom, int64_t n, int tiles_stride, int nviews, int nwork,
    const float* __restrict__ g, int D, float* const* __restrict__ outs,
    float* const* __restrict__ alphas, const uint32_t* __restrict__ perm) {
  constexpr int kQueues = kSplit ? 2 : 1;
  __shared__ __align__(16) float Wts[kQueues][32 * kWtPitch];  // queued Gaussians: [row][pixel]
  __shared__ float4 Rs[kChunk][2];                             // the step's records
  __shared__ int Count[kQueues];                               // rows, + 64 with the last ones
  constexpr int kIds = kSplit ? 256 : 128;
  __shared__ uint32_t Ids[kIds];  // the rows' Gaussians in order, row k at k mod kIds
  Quad q;
  // every in-image (pixel, channel) of every view is written, zeros where no
  // Gaussian reaches (a tile without Gaussians walks nothing)
  if (!decode_quad(ranges, geom, tiles_stride, nviews, nwork, q, true)) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int px = q.qx + (lane & 7), py = q.qy + (lane >> 3);

  const int c0 = (kSplit ? q.cg * ((int)(blockDim.x >> 6) - 1) + wave - 1 : q.cg) * 32 * NB;
  // this lane's channel in each 32-channel block (a readable one where it has none)
  int ch[NB];
  bool own[NB];
#pragma unroll
  for (int b = 0; b < NB; b++) {
    ch[b] = kVec ? c0 + NB * (lane & 31) + b : c0 + 32 * b + (lane & 31);
    own[b] = ch[b] < D;
    if (!own[b]) ch[b] = kVec ? b : 0;
  }
  typedef float fvec __attribute__((ext_vector_type(NB)));
  f32x16 acc[2][NB];  // [pixel block][channel block]
#pragma unroll
  for (int b = 0; b < NB; b++) acc[0][b] = acc[1][b] = f32x16{};

  auto flush = [&](const float* Wt, int count, uint32_t row0) {
    // K-step t: queue rows 16 t + 8 (l / 32) + i, i < 8.  Rows past count
    // have weight 0 and read the features of row 0 (in this queue), and a lane
    // without a channel feeds only its own output column, never written: the
    // loaded features are used as loaded (no select, so no zero fill that would
    // wait for every load in flight).
    for (int t = 0; t < 2 && 16 * t < count && c0 < D; t++) {
      float w0[8], w1[8];
      int64_t gid[8];
#pragma unroll
      for (int i = 0; i < 8; i++) {
        const int row = 16 * t + 8 * (lane >> 5) + i;
        const bool ok = row < count;
        gid[i] = (int64_t)Ids[(row0 + (uint32_t)(ok ? row : 0)) % kIds];
        w0[i] = ok ? Wt[row * kWtPitch + (lane & 31)] : 0.0f;
        w1[i] = ok ? Wt[row * kWtPitch + 32 + (lane & 31)] : 0.0f;
      }
      float gb[NB][8];
      if constexpr (kVec && NB > 1) {
        fvec r[8];
#pragma unroll
        for (int i = 0; i < 8; i++) r[i] = *reinterpret_cast<const fvec*>(g + gid[i] * D + ch[0]);
#pragma unroll
        for (int i = 0; i < 8; i++)
#pragma unroll
          for (int c = 0; c < NB; c++) gb[c][i] = r[i][c];
      } else {
#pragma unroll
        for (int c = 0; c < NB; c++)
#pragma unroll
          for (int i = 0; i < 8; i++) gb[c][i] = g[gid[i] * D + ch[c]];
      }
      bf16x8 a0h, a0l, a1h, a1l;
      split8(w0, a0h, a0l);
      split8(w1, a1h, a1l);
#pragma unroll
      for (int c = 0; c < NB; c++) {
        bf16x8 bh, bl;
        split8(gb[c], bh, bl);
        acc[0][c] = mfma(a0h, bh, acc[0][c]);
        acc[1][c] = mfma(a1h, bh, acc[1][c]);
        acc[0][c] = mfma(a0l, bh, acc[0][c]);
        acc[1][c] = mfma(a1l, bh, acc[1][c]);
        acc[0][c] = mfma(a0h, bl, acc[0][c]);
        acc[1][c] = mfma(a1h, bl, acc[1][c]);
      }
    }
  };

  if (wave == 0) {
    Walk s;
    walk_init(q, lane, s);
    Steps<kSplit> st;
    if (q.rg.y > q.rg.x) st.start(rec + (int64_t)q.v * n, ids, q.rg, lane, perm);
    int b = 0, queued = 0;   // rows [0, queued) of queue b hold Gaussians
    uint32_t rows_done = 0u; // rows whose ids are in Ids
    uint64_t kept = 0ull;    // hits of the step that took a row since
    uint32_t my_id = 0u;
    float asum = 0.0f;
    uint32_t row0 = 0u;      // the queue's first row
    float* wrow = Wts[0] + lane;
    auto write_ids = [&]() {
      if ((kept >> lane) & 1ull)
        Ids[(rows_done + (uint32_t)__popcll(kept & ((1ull << lane) - 1ull))) % kIds] = my_id;
      rows_done += (uint32_t)__popcll(kept);
      kept = 0ull;
    };
    auto hand_over = [&](int count) {
      write_ids();
      if constexpr (kSplit) {
        if (lane == 0) Count[b] = count;
        lds_barrier();
        b ^= 1;
      } else {
        lds_order();
        flush(Wts[0], count & 63, row0);
        lds_order();
        row0 += 32u;
      }
      queued = 0;
      wrow = Wts[b] + lane;
    };
    for (uint32_t base = q.rg.x; base < q.rg.y; base += kChunk) {
      if (nonzero(s.T) == 0ull) break;
      uint64_t h = step_records(st, base, lane, s, my_id, Rs);
      if (!h) continue;
      lds_order();  // records in LDS
      int j = (int)__builtin_ctzll(h);
      float4 ra = Rs[j][0];
      float2 rb = *reinterpret_cast<const float2*>(&Rs[j][1]);
      do {
        const uint64_t bit = 1ull << j;
        h &= ~bit;
        j = (int)__builtin_ctzll(h | (1ull << 63));  // 63 after the last: a readable record
        const float4 ca = ra;
        const float2 cb = rb;
        ra = Rs[j][0];
        rb = *reinterpret_cast<const float2*>(&Rs[j][1]);
        const float wj = blend_step(ca, cb, s.pxo, s.pyo, s.T);
        *wrow = wj;
        asum += wj;
        if (nonzero(wj)) {  // else the next hit takes the row: a row costs 32 NB channels of g
          kept |= bit;
          wrow += kWtPitch;
          if (++queued == 32) hand_over(32);
        }
      } while (h);
      write_ids();
      lds_order();  // the records are read before the next step's
    }
    hand_over(queued + 64);
    if (q.cg == 0 && alphas[q.v] && px < q.g.W && py < q.g.H)
      gptr(alphas[q.v])[(int64_t)py * q.g.W + px] = asum;
    if (kSplit) return;
  }
  if constexpr (kSplit) {
    uint32_t row0 = 0u;  // the queue's first row
    for (int b = 0;; b ^= 1) {
      lds_barrier();
      const int handed = __builtin_amdgcn_readfirstlane(Count[b]);
      flush(Wts[b], handed & 63, row0);
      row0 += 32u;
      if (handed & 64) break;
    }
  }

  // D row m of a block: pixel 32 pb + 8 (r / 4) + 4 (l / 32) + r % 4, column
  // l % 32
  float* const out = outs[q.v];
#pragma unroll
  for (int pb = 0; pb < 2; pb++) {
#pragma unroll
    for (int r = 0; r < 16; r++) {
      const int m = 32 * pb + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
      const int ox = q.qx + (m & 7), oy = q.qy + (m >> 3);
      if (ox < q.g.W && oy < q.g.H) {
        const int64_t pix = (int64_t)oy * q.g.W + ox;
        if constexpr (kVec && NB > 1) {
          fvec o;
#pragma unroll
          for (int c = 0; c < NB; c++) o[c] = acc[pb][c][r];
          if (own[0]) *gptr(reinterpret_cast<fvec*>(out + pix * D + ch[0])) = o;
        } else {
#pragma unroll
          for (int c = 0; c < NB; c++)
            if (own[c]) gptr(out)[pix * D + ch[c]] = acc[pb][c][r];
        }
      }
    }
  }
}

// D a multiple of 4, 16-byte aligned arrays: a block takes 64 Gaussians,
// each thread four channels at a time (16-byte accesses, no 64-bit division
// per element).
constexpr int kFinRows = 64;
__global__ __launch_bounds__(256) void finalize4_kernel(const float4* __restrict__ U,
                                                        const beta_t* __restrict__ beta, int64_t n,
                                                        int Q, float4* __restrict__ f,
                                                        float* __restrict__ wsum,
                                                        float4* __restrict__ usum,
                                                        const uint32_t* __restrict__ perm) {
  const int64_t r0 = (int64_t)blockIdx.x * kFinRows;
  const int rows = (int)(n - r0 < kFinRows ? n - r0 : kFinRows);
  for (int k = threadIdx.x; k < rows * Q; k += 256) {
    const int r = k / Q, q = k - r * Q;
    const int64_t i = r0 + r;
    const int64_t o = perm ? (int64_t)perm[i] : i;  // the output row
    const float bs = (float)((double)beta[i] * (1.0 / kBetaUnit));
    const float4 u = U[i * Q + q];
    const int64_t e = o * Q + q;
    if (f)
      f[e] = bs > 0.0f ? make_float4(u.x / bs, u.y / bs, u.z / bs, u.w / bs)
                       : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (usum) usum[e] = u;
    if (wsum && q == 0) wsum[o] = bs;
  }
}

__global__ void finalize_kernel(const float* __restrict__ U, const beta_t* __restrict__ beta,
                                int64_t n, int D, float* __restrict__ f, float* __restrict__ wsum,
                                float* __restrict__ usum, const uint32_t* __restrict__ perm) {
  int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * D) return;
  int64_t i = e / D;
  const int64_t c = e - i * D;
  const int64_t o = perm ? (int64_t)perm[i] : i;  // the output row
  const float bs = (float)((double)beta[i] * (1.0 / kBetaUnit));
  float u = U[e];
  if (f) f[o * D + c] = bs > 0.0f ? u / bs : 0.0f;
  if (usum) usum[o * D + c] = u;
  if (wsum && c == 0) wsum[o] = bs;
}

__global__ void finalize_fixed_kernel(const long long* __restrict__ U, const beta_t* __restrict__ beta,
                                      int64_t n, int D, float* __restrict__ f, float* __restrict__ wsum,
                                      float* __restrict__ usum, const uint32_t* __restrict__ perm) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * D) return;
  const int64_t i = e / D, c = e - i * D;
  const int64_t o = perm ? (int64_t)perm[i] : i;  // the output row
  const double b = (double)beta[i] * (1.0 / kBetaUnit);
  const double u = (double)U[e] * (1.0 / kBetaUnit);
  if (f) f[o * D + c] = b > 0.0 ? (float)(u / b) : 0.0f;
  if (usum) usum[o * D + c] = (float)u;
  if (wsum && c == 0) wsum[o] = (float)b;
}

}  // namespace

namespace {
__global__ __launch_bounds__(256) void class_add_kernel(const beta_t* __restrict__ beta,
                                                        const uint32_t* __restrict__ counts,
                                                        ClassAdd dst, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const beta_t b = beta[i];
    const uint32_t c = counts ? counts[i] : 0u;
    for (int k = 0; k < dst.nd; k++) {
      if (dst.beta[k]) dst.beta[k][i] += b;
      if (dst.counts[k]) dst.counts[k][i] += c;
    }
  }
}
}  // namespace

hipError_t launch_class_add(const beta_t* beta, const uint32_t* counts, const ClassAdd& dst,
                            int64_t n, hipStream_t s) {
  if (n == 0 || dst.nd == 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(class_add_kernel, dim3((unsigned)blocks), dim3(256), 0, s, beta, counts, dst, n);
  return hipGetLastError();
}

hipError_t launch_blend(const BlendArgs& a, lv_dtype dtype, int m, hipStream_t s) {
  if (m == 0 || a.tiles_stride == 0) return hipSuccess;
  switch (dtype) {
    case LV_F32: return launch_blend_t<LV_F32, false>(a, m, s);
    case LV_BF16: return launch_blend_t<LV_BF16, false>(a, m, s);
    case LV_FP8_E4M3: return launch_blend_t<LV_FP8_E4M3, false>(a, m, s);
    case LV_F32_PX8: return launch_blend_t<LV_F32, true>(a, m, s);
    case LV_BF16_PX8: return launch_blend_t<LV_BF16, true>(a, m, s);
    case LV_FP8_E4M3_PX8: return launch_blend_t<LV_FP8_E4M3, true>(a, m, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_render(const BlendArgs& a, int m, const float* g, int D, float* const* outs,
                         uintptr_t outs_align, float* const* alphas, const uint32_t* perm, hipStream_t s) {
  if (m == 0 || a.tiles_stride == 0) return hipSuccess;
  const int nb = D > 64 ? 4 : D > 32 ? 2 : 1;  // 32-channel blocks per wave
  const int ngroups = (D + 32 * nb - 1) / (32 * nb);
  const int waves = ngroups % kRenderWaves == 0 ? kRenderWaves : 1;  // groups per workgroup
  const int nwork = ngroups / waves;                                 // workgroups per quadrant
  const bool split = waves > 1 || (int64_t)a.tiles_stride * m * nwork * 4 <= kFewQuadrants / (nb == 4 ? 2 : 1);
  const int64_t work = (int64_t)a.tiles_stride * m * nwork;
  const int64_t blocks = (work + 7) / 8 * 32;  // 4 quadrants per tile, whole rounds of 8 XCDs
  const bool vec = D % nb == 0 && (uintptr_t)g % (4 * nb) == 0 && outs_align % (4 * nb) == 0;
  const auto kernel = nb == 1   ? (split ? render_kernel<1, false, true> : render_kernel<1, false, false>)
                      : nb == 2 ? (vec ? (split ? render_kernel<2, true, true> : render_kernel<2, true, false>)
                                       : (split ? render_kernel<2, false, true> : render_kernel<2, false, false>))
                                : (vec ? (split ? render_kernel<4, true, true> : render_kernel<4, true, false>)
                                       : (split ? render_kernel<4, false, true> : render_kernel<4, false, false>));
  hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(split ? 64 * (1 + waves) : 64), 0, s, a.rec, a.ids,
                     a.ranges, a.geom, a.n, a.tiles_stride, m, nwork, g, D, outs, alphas, perm);
  return hipGetLastError();
}

hipError_t launch_finalize_fixed(const long long* U, const beta_t* beta, int64_t n, int D, float* f,
                                 float* wsum, float* usum, const uint32_t* perm, hipStream_t s) {
  const int64_t total = n * (int64_t)D;
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(finalize_fixed_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, U, beta,
                     n, D, f, wsum, usum, perm);
  return hipGetLastError();
}

hipError_t launch_finalize(const float* U, const beta_t* beta, int64_t n, int D, float* f,
                           float* wsum, float* usum, const uint32_t* perm, hipStream_t s) {
  int64_t total = n * (int64_t)D;
  if (total == 0) return hipSuccess;
  const auto a16 = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  if (D % 4 == 0 && a16(U) && a16(f) && a16(usum)) {
    hipLaunchKernelGGL(finalize4_kernel, dim3((unsigned)((n + kFinRows - 1) / kFinRows)), dim3(256), 0, s,
                       reinterpret_cast<const float4*>(U), beta, n, D / 4, reinterpret_cast<float4*>(f),
                       wsum, reinterpret_cast<float4*>(usum), perm);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(finalize_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, U,
                     beta, n, D, f, wsum, usum, perm);
  return hipGetLastError();
}

}  // namespace lv
