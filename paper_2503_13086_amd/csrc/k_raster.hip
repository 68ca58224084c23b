// Tile rasterizer forward and backward for gfx950.
//
// Forward (Sec. III Eq. 2): one thread per pixel, each wavefront owning an 8x8 block
// of a T x T tile (T = 8, 16 or 32).  It walks the tile's depth-ordered list, one
// record per lane, keeps the records whose cutoff ellipse meets the block's pixel
// centres in its own LDS rows, and every pixel reads these by LDS broadcast.  A
// wavefront stops when all its pixels have stopped blending.  Screen centres arrive
// in FP64 and are made relative to the tile origin while staging, so per-pixel
// offsets are accurate fp32 numbers at any image size.
//
// Backward (Sec. IV-E): the same tiling and per-block candidate sets, walking each
// list back to front from the last position any pixel of the tile blended (each
// wavefront starts at the last position its own pixels blended).  Each pixel
// recovers its transmittance with one reciprocal per Gaussian and keeps the colour
// accumulated behind it.  Per Gaussian, nine sums over the block's pixels (the moments
// of dL/d(exponent) over dx, dy, dx^2, dx dy, dy^2, then opacity and colour partials)
// are formed eight Gaussians at a time from a panel in LDS (see kPanel) and added to
// the tile's totals there; the moments become centre and conic partials once per tile,
// and each workgroup issues one global atomic per (tile, Gaussian, component) instead
// of one per (pixel, Gaussian, component), consecutive lanes taking consecutive
// components so a wavefront's atomics share cache lines.
#include <type_traits>

#include "gs_internal.h"

#pragma clang fp contract(off)

namespace gsk {
namespace {

// Wave-wide mask of a per-lane predicate (the compiler keeps the predicate in a
// scalar mask instead of round-tripping it through a vector register).
__device__ inline uint64_t wave_mask(bool p) { return __builtin_amdgcn_ballot_w64(p); }


// Set bits of a wave-wide mask below this lane.
__device__ inline int mask_rank(uint64_t m) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Tile of workgroup b.  Workgroups are dealt to the chip's 8 XCDs round-robin (b
// runs on XCD b mod 8, each XCD with its own L2); XCD x takes the runs x, x + 8,
// ... of 32 consecutive tiles, so neighbouring tiles, which stage mostly the same
// records, meet in one L2, while the short runs keep the work per XCD even (1%
// faster backward than plain tile order; whole contiguous eighths were slower).
// The grid is rounded up to whole rounds of runs; workgroups past the last tile
// return at once.
constexpr int kXcdRun = 32;
__device__ inline int xcd_raster_tile(int b) {
  const int x = b % 8, q = b / 8;
  return ((q / kXcdRun) * 8 + x) * kXcdRun + q % kXcdRun;
}

// View of a (wave-uniform) tile: lane v looks at view v's first tile (at most 64
// views), so one load's latency instead of a chain of them.
__device__ inline int view_of_tile(const ViewDev* __restrict__ views, int V, int tile) {
  static_assert(GS_MAX_VIEWS <= 64, "one lane per view");
  const int v = (int)__lane_id();
  return __popcll(wave_mask(v < V && tile >= views[v < V ? v : 0].tile_off)) - 1;
}

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Negated base-2 exponent q of the 2D Gaussian at offset (dx, dy): with A = a/2,
// B = b, C = c/2 pre-scaled by log2(e), e^power = 2^-q, taken as
// dx (A dx + B dy) + C dy^2 (five operations).
__device__ inline float gauss_q(float A, float B, float C, float dx, float dy) {
  return __fmaf_rn(C * dy, dy, dx * __fmaf_rn(B, dy, A * dx));
}

// The pixel test tau <= power <= 0 as one comparison: t = -tau log2(e) >= 0 and q
// compared as unsigned integers.  A q in [0, t] orders like its bits; a negative q
// (power > 0) has the sign bit set and a NaN lies above every number, so both fail.
// (q is never -0: a difference of equal numbers and a sum of a -0 product with +0
// are +0.)  One VALU comparison costs four cycles per wavefront, a multiply or an
// add two.
__device__ inline bool passes(float q, float t) { return __float_as_uint(q) <= __float_as_uint(t); }

struct TileGeom {
  int v, tx, ty, lx, ly, px, py;
  bool inside;
  double ox, oy;
};

template <int T>
__device__ inline TileGeom tile_geom(const ViewDev* __restrict__ views, int V, int tile) {
  TileGeom t;
  t.v = view_of_tile(views, V, tile);
  const ViewDev& cv = views[t.v];
  const int lt = tile - cv.tile_off;
  t.tx = lt % cv.tiles_x;
  t.ty = lt / cv.tiles_x;
  // wavefront w covers the 8x8 block (w mod T/8, w div T/8) of the tile; lane l
  // its pixel (l & 7, l >> 3)
  constexpr int QW = T / 8;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  t.lx = ((w % QW) << 3) | (l & 7);
  t.ly = ((w / QW) << 3) | (l >> 3);
  t.px = t.tx * T + t.lx;
  t.py = t.ty * T + t.ly;
  t.inside = t.px < cv.W && t.py < cv.H;
  t.ox = (double)(t.tx * T) + 0.5;
  t.oy = (double)(t.ty * T) + 0.5;
  return t;
}

// Stage record `rid` for a tile with origin (ox, oy): centre relative to the tile,
// coefficients of q and the cutoff t in base-2 units (the comparisons are unchanged
// by the positive factor), opacity, colour, and two values for the block test below:
// the slope kC = -b / c of the line on which the exponent peaks along vertical
// lines, and a cutoff t_c = t (1 + 1e-5 kappa) slightly above the pixel test's,
// kappa = (sqrt(ac) + |b|)^2 / (ac - b^2) bounding (|A dx^2| + |B dx dy| + |C dy^2|) /
// |q|, so that fp32 rounding in either test can never make the block test drop a
// Gaussian a pixel accepts.  det = ac - b^2 is one fused multiply-add (error below
// ulp(b^2), so below 2e-4 det wherever kappa < 1e4, and every conic with det <= 0
// yields det < ulp(b^2), kappa > 1e4); kappa and kC are fp32 too (their errors only
// move the margin by as much of itself).  A conic that is not clearly positive
// definite (det <= 0 or kappa >= 1e4) gets t_c = inf, so every block lists it; a
// cutoff above 0 (opacity below 1/255) or NaN gets t_c = NaN, which no block's q is at
// or below, whatever rounding made of it: the pixel test, which only sees |tau|, never
// meets such a splat.
//   q0 = (u', w', A, B)   q1 = (C, t, t_c, kC)   q2 = (o, r, g, b)
// (the per-pixel test reads q0 and q1.xy, a blend q2).
struct RawRecord {
  double2 uw;
  float4 c, d;
};

__device__ inline RawRecord fetch(const Record* __restrict__ rec, uint32_t rid) {
  const Record* r = rec + rid;
  return RawRecord{*reinterpret_cast<const double2*>(r), reinterpret_cast<const float4*>(r)[1],
                   reinterpret_cast<const float4*>(r)[2]};
}

__device__ inline void stage(const RawRecord& r, double ox, double oy, float4& q0, float4& q1, float4& q2) {
  const float4 c = r.c, d = r.d;
  const float det = __fmaf_rn(c.x, c.z, -(c.y * c.y));
  const float t = fabsf(d.x * kLog2e);
  float tc = INFINITY, kc = 0.0f;
  if (det > 0.0f) {
    const float s = __builtin_amdgcn_sqrtf(c.x * c.z) + fabsf(c.y);
    const float kappa = (s * s) * __builtin_amdgcn_rcpf(det);
    if (kappa < 1e4f) tc = t * (1.0f + 1e-5f * kappa);
    kc = -c.y * __builtin_amdgcn_rcpf(c.z);
  }
  if (!(d.x <= 0.0f)) tc = NAN;
  q0 = make_float4((float)(r.uw.x - ox), (float)(r.uw.y - oy), (0.5f * c.x) * kLog2e, c.y * kLog2e);
  q1 = make_float4((0.5f * c.z) * kLog2e, t, tc, kc);
  q2 = make_float4(c.w, d.y, d.z, d.w);
}

// Placeholder for an entry that belongs to no Gaussian (never for a consistent
// sort): no block lists it, and no pixel would accept it.
__device__ inline void stage_empty(float4& q0, float4& q1, float4& q2) {
  q0 = make_float4(NAN, 0.f, 0.f, 0.f);
  q1 = make_float4(0.f, 0.f, NAN, 0.f);
  q2 = make_float4(0.f, 0.f, 0.f, 0.f);
}

// Does a staged record's cutoff ellipse meet this wavefront's 8x8 block of pixel
// centres [qx, qx + 7] x [qy, qy + 7] (tile-relative)?  The pixels' offsets u' - x,
// w' - y fill the box [x0, x1] x [y0, y1] (same fp32 subtractions as the pixel test),
// and the smallest q over that box lies on the edge dx = xn (the box's nearest value
// to 0), where it is least at dy = kC xn, or on the edge dy = yn, least at dx = kA yn
// (a convex quadratic's minimum over a box is at its centre, or on an edge next to
// the nearest corner); any point of the box bounds that minimum from above, so the
// rounding of those positions only costs the second-order loss already covered by
// t_c.
__device__ inline bool block_hit(const float4& a0, const float4& a1, float qx, float qy) {
  const float x0 = a0.x - (qx + 7.0f), x1 = a0.x - qx;
  const float y0 = a0.y - (qy + 7.0f), y1 = a0.y - qy;
  // (x0 <= x1 and y0 <= y1: a median of three is a clamp)
  const float xn = __builtin_amdgcn_fmed3f(0.0f, x0, x1);
  const float yn = __builtin_amdgcn_fmed3f(0.0f, y0, y1);
  const float ka = (-0.5f * a0.w) * __builtin_amdgcn_rcpf(a0.z);
  const float dy1 = __builtin_amdgcn_fmed3f(xn * a1.w, y0, y1);
  const float dx2 = __builtin_amdgcn_fmed3f(yn * ka, x0, x1);
  const float f1 = gauss_q(a0.z, a0.w, a1.x, xn, dy1);
  const float f2 = gauss_q(a0.z, a0.w, a1.x, dx2, yn);
  return fminf(f1, f2) <= a1.z;
}

// Ballots of block_hit over the staged records [0, m); bit b of mask[k] is record
// 64 k + b.
template <int NM>
__device__ inline void block_masks(const float4* s0, const float4* s1, int m, float qx, float qy,
                                      uint64_t (&mask)[NM]) {
  const int lane = (int)__lane_id();
#pragma unroll
  for (int k = 0; k < NM; ++k) {
    const int j = lane + 64 * k;
    bool hit = false;
    if (j < m) hit = block_hit(s0[j], s1[j], qx, qy);
    mask[k] = wave_mask(hit);
  }
}

// A pixel that did not blend a candidate enters every sum as alpha = 0 times finite
// numbers, which takes no select.  The numbers are finite while colours and upstream
// gradients are below kTame: their product, summed with weights of at most 1 in all and
// divided by 1 - alpha >= 0.01, stays under 1e33.  A wavefront with anything larger,
// infinite or NaN leaves out the candidates that none of its pixels blends, and in the
// backward sets the derivative of the pixels that did not blend one to zero: such a
// value then reaches no splat but those blended with it, and no block but those that
// blend it.
constexpr float kTame = 1e15f;
__device__ inline bool tame_colour(const float4& q2) { return fabsf(q2.y) + fabsf(q2.z) + fabsf(q2.w) <= kTame; }

// x << 1, with the lane's bit of a wave-wide mask shifted in (one add with carry).
__device__ inline uint32_t shift_in(uint32_t x, uint64_t m) {
  uint32_t r;
  asm("v_addc_co_u32_e64 %0, vcc, %1, %1, %2" : "=v"(r) : "v"(x), "s"(m) : "vcc");
  return r;
}

// Candidates a wavefront takes together in the forward: their tests and alphas do not
// depend on each other.  One build with 1, 2 or 4 took 692, 657 and 667 us at 1M
// Gaussians and 10 Mpix (six to eight wavefronts per SIMD hide most of it) and 74, 64 and 60 us at 10k
// Gaussians and 128x128 pixels (256 wavefronts on the whole chip).
constexpr int kFwdGroup = 4;

// One wavefront per 8x8 block of a tile, four to a workgroup and independent of each
// other (no barrier: each stops as soon as its own pixels have, and finds the
// records its neighbours staged in the same caches).  It walks the tile's list 64
// positions at a time, one record per lane with the next 64 records and the ids of
// the 64 after them in flight, and writes the records whose cutoff ellipse meets
// its block to its own LDS rows in list order; every pixel then reads them by LDS
// broadcast.  Bound by VALU issue: about 55 cycles per candidate and wavefront (a
// selection of masks held in scalar registers keeps comparisons, selects and scalar
// operands, four cycles each, to five), 85% of the issue slots taken, where one
// workgroup per tile with a barrier per batch took 81: in a training step of 1M
// Gaussians, nine views and 10 Mpix 751 -> 699 us, of 300k and 1296x864 101 -> 87, of 10k
// and 128x128 78 -> 59.
template <int T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) void k_render_fwd(
    const ViewDev* __restrict__ views, int V, int n_tiles, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ pair_rec, const Record* __restrict__ rec, uint32_t n_rec,
    float* __restrict__ color, float* __restrict__ t_final, uint32_t* __restrict__ n_contrib,
    uint32_t* __restrict__ last, float* __restrict__ asum) {
  constexpr int G = kFwdGroup, QW = T / 8, NBLK = QW * QW, ROWS = 64 + G;
  __shared__ float4 rows[4][3 * ROWS];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = (int)__lane_id();
  const int unit = 4 * xcd_raster_tile((int)blockIdx.x) + wave;
  const int tile = unit / NBLK, blk = unit % NBLK;
  if (tile >= n_tiles) return;
  const int v = view_of_tile(views, V, tile);
  const ViewDev& cv = views[v];
  const uint2 rg = ranges[tile];
  const int lt = tile - cv.tile_off;
  const int tx = lt % cv.tiles_x, ty = lt / cv.tiles_x;
  const int bx = 8 * (blk % QW), by = 8 * (blk / QW);        // block origin in the tile
  const double ox = (double)(tx * T) + 0.5, oy = (double)(ty * T) + 0.5;
  const float qx = (float)bx, qy = (float)by;
  const int px = tx * T + bx + (lane & 7), py = ty * T + by + (lane >> 3);
  const bool inside = px < cv.W && py < cv.H;
  const float fx = (float)(bx + (lane & 7)), fy = (float)(by + (lane >> 3));
  float Tr = 1.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f, A = 0.0f;
  uint32_t cnt = 0, lastp = 0;

  float4* const r0 = rows[wave];
  const auto id_at = [&](uint32_t i) {
    return i + (uint32_t)lane < rg.y ? pair_rec[i + (uint32_t)lane] : ~0u;
  };
  uint32_t rid = id_at(rg.x), rid1 = id_at(rg.x + 64u);
  RawRecord raw{}, raw1{};
  if (rid < n_rec) raw = fetch(rec, rid);
  uint64_t live = wave_mask(inside);      // the pixels that have not stopped
  for (uint32_t base = rg.x; base < rg.y && live != 0ull; base += 64u) {
    const uint32_t rid2 = id_at(base + 128u);
    if (rid1 < n_rec) raw1 = fetch(rec, rid1);
    float4 q0, q1, q2;
    stage(raw, ox, oy, q0, q1, q2);
    const bool hit = rid < n_rec && block_hit(q0, q1, qx, qy);
    const uint64_t mk = wave_mask(hit);
    const bool caps = wave_mask(hit && q2.x > kAlphaMax) != 0ull;   // some alpha may reach the cap
    const bool wild = wave_mask(hit && !tame_colour(q2)) != 0ull;
    const int n = __popcll(mk);
    __builtin_amdgcn_wave_barrier();
    if (hit) {
      const int r = mask_rank(mk);
      r0[r] = q0;
      r0[ROWS + r] = make_float4(q1.x, q1.y, __uint_as_float(base - rg.x + (uint32_t)lane + 1u), 0.0f);
      r0[2 * ROWS + r] = q2;
    }
    if (lane < G) {   // fills up the last group: no pixel accepts it
      float4 e0, e1, e2;
      stage_empty(e0, e1, e2);
      r0[n + lane] = e0;
      r0[ROWS + n + lane] = e1;
      r0[2 * ROWS + n + lane] = e2;
    }
    __builtin_amdgcn_wave_barrier();
    // Every step is straight-line over the wavefront; the masks of the pixels that
    // pass, stop or still blend live in scalar registers.  `hist` collects one bit per
    // candidate and pixel (blended or not), which gives the count and the last
    // position once per 32 candidates.
    const auto walk = [&](auto cap, auto wild_colours) {
      constexpr bool CAP = decltype(cap)::value, WILD = decltype(wild_colours)::value;
      for (int i0 = 0; i0 < n && live != 0ull; i0 += 32) {
        uint32_t hist = 0u;
        int i = i0;
        for (const int i1 = min(i0 + 32, n); i < i1 && live != 0ull; i += G) {
          float q[G], al[G];
          float4 a2[G];
          uint64_t pass[G];
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const float4 a0 = r0[i + g];
            const float2 a1 = *reinterpret_cast<const float2*>(&r0[ROWS + i + g]);
            a2[g] = r0[2 * ROWS + i + g];
            // (one 16-byte read here rather than four where its parts are used)
            asm volatile("" ::"v"(a2[g].x), "v"(a2[g].y), "v"(a2[g].z), "v"(a2[g].w));
            q[g] = gauss_q(a0.z, a0.w, a1.x, a0.x - fx, a0.y - fy);
            pass[g] = wave_mask(passes(q[g], a1.y));
            al[g] = a2[g].x * __builtin_amdgcn_exp2f(-q[g]);
            if (CAP) al[g] = fminf(kAlphaMax, al[g]);
            asm volatile("" : "+v"(al[g]));   // (formed here, not in a branch around its use)
          }
#pragma unroll
          for (int g = 0; g < G; ++g) {
            uint64_t m = pass[g] & live;
            if (WILD && m == 0ull) {   // (its colour times 0 would be NaN)
              hist = shift_in(hist, 0ull);
              continue;
            }
            float alpha = __builtin_amdgcn_inverse_ballot_w64(m) ? al[g] : 0.0f;   // 0 where it does not blend
            float Tn = Tr * (1.0f - alpha);
            const uint64_t stops = wave_mask(Tn < kTMin);
            if (stops != 0ull) {   // these blend nothing, and nothing more
              const bool stop = __builtin_amdgcn_inverse_ballot_w64(stops);
              m &= ~stops;
              live &= ~stops;
              alpha = stop ? 0.0f : alpha;
              Tn = stop ? Tr : Tn;
            }
            const float wgt = alpha * Tr;
            C0 = __fmaf_rn(a2[g].y, wgt, C0);
            C1 = __fmaf_rn(a2[g].z, wgt, C1);
            C2 = __fmaf_rn(a2[g].w, wgt, C2);
            A += alpha;
            Tr = Tn;
            hist = shift_in(hist, m);
          }
        }
        cnt += (uint32_t)__popc(hist);
        // bit b of hist is row i - 1 - b
        if (hist != 0u) lastp = __float_as_uint(r0[ROWS + i - __ffs((int)hist)].z);
      }
    };
    if (wild) walk(std::true_type{}, std::true_type{});
    else if (caps) walk(std::true_type{}, std::false_type{});
    else walk(std::false_type{}, std::false_type{});
    raw = raw1;
    rid = rid1;
    rid1 = rid2;
  }
  if (inside) {
    const size_t hw = (size_t)cv.W * cv.H;
    const size_t pix = (size_t)py * cv.W + px;
    float* img = color + 3 * (size_t)cv.pix_off;
    img[pix] = C0 + Tr * cv.bg[0];
    img[hw + pix] = C1 + Tr * cv.bg[1];
    img[2 * hw + pix] = C2 + Tr * cv.bg[2];
    const size_t gp = (size_t)cv.pix_off + pix;
    t_final[gp] = Tr;
    n_contrib[gp] = cnt;
    last[gp] = lastp;
    asum[gp] = A;
  }
}

// The forward's walk, one workgroup of T x T threads per tile (the tile's blocks meet
// at a barrier per batch of T^2 records, so that they can mark a list entry together),
// writing the number of Gaussians each pixel evaluates up to its termination (those
// that pass its cutoff test: the blended ones and, if it stopped, the one that stopped
// it) into evals, and the number of the tile's list entries that at least one of its
// pixels blends into pairs_eff[tile].  The same decisions as the forward's: the same
// staged numbers and the same arithmetic.
template <int T>
__global__ __launch_bounds__(T * T) void k_render_count(const ViewDev* __restrict__ views, int V, int n_tiles_total,
                                                      const uint2* __restrict__ ranges,
                                                      const uint32_t* __restrict__ pair_rec,
                                                      const Record* __restrict__ rec, uint32_t n_rec,
                                                      uint32_t* __restrict__ evals,
                                                      uint32_t* __restrict__ pairs_eff) {
  constexpr int NT = T * T, NM = NT / 64;
  __shared__ float4 s0[NT], s1[NT], s2[NT];
  __shared__ uint32_t s_eff[NT / 32];   // batch entries some pixel blended
  uint32_t n_eff = 0;
  const int tile = xcd_raster_tile((int)blockIdx.x);
  if (tile >= n_tiles_total) return;
  const TileGeom tg = tile_geom<T>(views, V, tile);
  const uint2 rg = ranges[tile];
  // (a pixel that has stopped moves to infinity: no test passes there)
  float fx = tg.inside ? (float)tg.lx : INFINITY;
  const float fy = (float)tg.ly;
  const float qx = (float)(tg.lx & ~7), qy = (float)(tg.ly & ~7);
  float Tr = 1.0f;
  uint32_t cnt = 0;
  for (uint32_t base = rg.x; base < rg.y; base += NT) {
    const uint32_t m = min((uint32_t)NT, rg.y - base);
    __syncthreads();
    if (threadIdx.x < NT / 32) s_eff[threadIdx.x] = 0u;
    if (threadIdx.x < m) {
      const uint32_t rid = pair_rec[base + threadIdx.x];
      if (rid < n_rec) {
        stage(fetch(rec, rid), tg.ox, tg.oy, s0[threadIdx.x], s1[threadIdx.x], s2[threadIdx.x]);
      } else {
        stage_empty(s0[threadIdx.x], s1[threadIdx.x], s2[threadIdx.x]);
      }
    }
    __syncthreads();
    if (wave_mask(fx < INFINITY) != 0ull) {   // (a block whose pixels have all stopped only keeps the barriers)
      uint64_t mask[NM];
      block_masks<NM>(s0, s1, (int)m, qx, qy, mask);
      for (int k = 0; k < NM; ++k) {
        uint64_t eff = 0ull;   // this wave's blended entries of the 64, marked together
        uint64_t mk = wave_mask(fx < INFINITY) != 0ull ? mask[k] : 0ull;
        while (mk != 0ull) {
          const uint32_t j = 64u * k + (uint32_t)__builtin_ctzll(mk);
          const uint64_t bit = mk & (0ull - mk);
          mk ^= bit;
          const float4 a0 = s0[j];
          const float4 a1 = s1[j];
          const float opacity = s2[j].x;
          const float q = gauss_q(a0.z, a0.w, a1.x, a0.x - fx, a0.y - fy);
          const bool pass = passes(q, a1.y);
          if (wave_mask(pass) == 0ull) continue;
          const float alpha = fminf(kAlphaMax, opacity * __builtin_amdgcn_exp2f(-q));
          const float Tn = Tr * (1.0f - alpha);
          const bool stop = pass & (Tn < kTMin), blend = pass & !stop;
          cnt += pass ? 1u : 0u;
          Tr = blend ? Tn : Tr;
          eff |= wave_mask(blend) != 0ull ? bit : 0ull;
          fx = stop ? INFINITY : fx;
          mk = wave_mask(fx < INFINITY) == 0ull ? 0ull : mk;
        }
        if (__lane_id() == 0u) {
          if ((uint32_t)eff) atomicOr(&s_eff[2 * k], (uint32_t)eff);
          if ((uint32_t)(eff >> 32)) atomicOr(&s_eff[2 * k + 1], (uint32_t)(eff >> 32));
        }
      }
    }
    __syncthreads();
    if (threadIdx.x == 0)
      for (int w = 0; w < NT / 32; ++w) n_eff += (uint32_t)__popc(s_eff[w]);
    if (__syncthreads_and(!(fx < INFINITY))) break;
  }
  if (tg.inside) {
    const ViewDev& cv = views[tg.v];
    evals[(size_t)cv.pix_off + (size_t)tg.py * cv.W + tg.px] = cnt;
  }
  if (threadIdx.x == 0) pairs_eff[tile] = n_eff;
}

// Lane l receives v from the lane the DPP control names (row_half_mirror = 0x141:
// lane 7 - l of its half-row; quad_perm [2,3,0,1] = 0x4E and [1,0,3,2] = 0xB1: lanes
// l ^ 2 and l ^ 1).
template <int CTRL>
__device__ inline float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

// a + b across the partner lanes of a DPP permutation that pairs each lane with
// one whose selector bit `hi` differs: lanes with hi clear keep the sum of a over
// the pair, lanes with hi set the sum of b.
template <int CTRL>
__device__ inline float fold_dpp(float a, float b, bool hi) {
  const float own = hi ? b : a, give = hi ? a : b;
  return own + dpp<CTRL>(give);
}

// The same across half-row mirrors, selected by lane bit 2 (DPP banks 1 and 3),
// without the two selects: every lane forms a plus its partner's a, then the lanes
// of the selected banks overwrite that with b plus the partner's b (a DPP add that
// writes those banks only).  A DPP read of a VGPR that the VALU wrote in the last two
// cycles needs two wait states, and the compiler does not see inside the asm: the
// nops before and after cover the asm's own read and any DPP read of its result.
__device__ inline float fold_mirror_bit2(float a, float b) {
  float t = a + dpp<0x141>(a);
  asm("s_nop 1\n\tv_add_f32_dpp %0, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xa bound_ctrl:1\n\ts_nop 1" : "+v"(t) : "v"(b));
  return t;
}

// The backward's sums over pixels.  Each wavefront walks its candidates pixel by
// lane and writes, per (candidate, pixel), the two numbers every partial is made of,
// dL/d(exponent) and the blend weight, into its own LDS panel of kPanel candidates x
// 64 pixels.  When the panel is full the wavefront turns round: lane l takes
// candidate l / 8 and row l mod 8 of the 8x8 block, and forms the row's nine sums from
// eight pixels read back with four 16-byte loads, with no cross-lane step; three DPP
// levels over the candidate's eight lanes finish them, each lane ending with one of
// the eight first totals.  Per candidate this is about 27 VALU cycles, against
// about 118 for summing every candidate's nine values across 64 lanes (permlane
// swaps take 8 cycles, DPP and selects 4, a multiply or an add 2).
// LDS float adds cost three cycles a lane on this chip (193 for a full wavefront);
// double adds cost 8 for the wavefront, so the tile's totals are doubles.
constexpr int kPanel = 8;
// Candidates whose tests and alphas a wavefront takes together (each wavefront's
// chain per candidate is long, and four wavefronts per SIMD hide it only in part):
// one build with 1, 2 or 4 at a time took 1.48, 1.33 and 1.26 ms at 1M Gaussians and 10
// Mpix, and 117, 86 and 76 us at 10k Gaussians and 128x128 pixels.  In a training step
// the kernel takes 1.30 ms and 75 us there, and 146 us at 300k and 1296x864, where the
// sums across 64 lanes took 1.69 ms, 112 and 209 us.
constexpr int kGroup = 4;
typedef __attribute__((address_space(3))) double LdsDouble;

// Panel position of pixel pair (row, u): pixels 2 u and 2 u + 1 of a row form a
// 16-byte unit, and the units of a row are permuted by xor with unit_turn.  The 16
// lanes (two slots, eight rows) that one LDS cycle serves then read 16 different
// units of the 256-byte bank row, unit u of every row in the same load.
__device__ inline int unit_turn(int slot, int row) { return (row >> 2) + 2 * (slot & 1); }

// ORDERED: instead of adding each (tile, Gaussian) partial sum into grad2d with a
// global atomic, write it to out[pair position * kGrad2D + component] (every
// position of the tile's list, zeros included), each wave keeping its totals in its
// own LDS rows and the waves' rows summed in wave order, so that every partial is the
// same bits on every run; the per-Gaussian sums are then taken in tile order by
// launch_ordered_sum.
template <int T, bool ORDERED = false>
__global__ __launch_bounds__(T * T) __attribute__((amdgpu_waves_per_eu(4))) void k_render_bwd(const ViewDev* __restrict__ views, int V, int n_tiles_total,
                                                    const uint2* __restrict__ ranges,
                                                    const uint32_t* __restrict__ pair_rec,
                                                    const Record* __restrict__ rec, uint32_t n_rec,
                                                    const float* __restrict__ t_final,
                                                    const uint32_t* __restrict__ last,
                                                    const float* __restrict__ dL_dcolor,
                                                    const float* __restrict__ dL_dG, float* __restrict__ grad2d) {
  // records are staged NB at a time; row NB is a record no pixel accepts, which fills
  // up a wavefront's last group
  constexpr int NT = T * T, NB = ORDERED || NT < 128 ? 64 : 128, NM = (NB + 63) / 64, NW = NT / 64;
  constexpr int NACC = ORDERED ? NW : 1;
  constexpr int G = kGroup;
  using Acc = typename std::conditional<ORDERED, float, double>::type;
  __shared__ float4 s0[NB + 1], s1[NB + 1], s2[NB + 1];
  __shared__ uint32_t srid[NB];
  __shared__ Acc acc[NACC][NB][kGrad2D];
  __shared__ __align__(16) float2 panel[NW][kPanel][64];
  __shared__ __align__(16) uint32_t list[NW][NB + kPanel];   // byte offsets of the wave's candidates in s0
  __shared__ uint32_t smax[NW];
  const int tile = xcd_raster_tile((int)blockIdx.x);
  if (tile >= n_tiles_total) return;
  const TileGeom tg = tile_geom<T>(views, V, tile);
  const ViewDev& cv = views[tg.v];
  const uint2 rg = ranges[tile];
  const float fx = (float)tg.lx, fy = (float)tg.ly;
  const float qx = (float)(tg.lx & ~7), qy = (float)(tg.ly & ~7);
  const int wave = threadIdx.x >> 6, lane = (int)__lane_id();

  // Sg = sum over channels of dL/dcolour times the colour accumulated behind the
  // current Gaussian (background included): the only form in which that colour
  // enters dL/dalpha.
  float Tr = 0.0f, Sg = 0.0f, g0 = 0.0f, g1 = 0.0f, g2 = 0.0f, gG = 0.0f;
  uint32_t lp = 0;
  if (tg.inside) {
    const size_t hw = (size_t)cv.W * cv.H;
    const size_t pix = (size_t)tg.py * cv.W + tg.px;
    const size_t gp = (size_t)cv.pix_off + pix;
    Tr = t_final[gp];
    lp = last[gp];
    const float* gimg = dL_dcolor + 3 * (size_t)cv.pix_off;
    g0 = gimg[pix];
    g1 = gimg[hw + pix];
    g2 = gimg[2 * hw + pix];
    if (dL_dG) gG = dL_dG[gp];
    Sg = Tr * __fmaf_rn(g2, cv.bg[2], __fmaf_rn(g1, cv.bg[1], g0 * cv.bg[0]));
  }
  uint32_t mx = lp;
  for (int off = 32; off > 0; off >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, off));
  const int wave_last = (int)mx;           // this wave never needs list positions >= wave_last
  if (lane == 0) smax[wave] = mx;
  for (int i = threadIdx.x; i < NACC * NB * kGrad2D; i += NT) (&acc[0][0][0])[i] = (Acc)0;
  if (threadIdx.x == 0) stage_empty(s0[NB], s1[NB], s2[NB]);

  // this lane's part in the panel's sums: slot ps, row pr, the row's upstream
  // gradients (through the panel's own memory), the total it ends with (pc), and the
  // selectors of the last two levels; pan[s & 1] + 64 s is where it writes as a pixel
  const int ps = lane >> 3, pr = lane & 7;
  const int pc = ((lane & 1) << 2) | (lane & 2) | ((lane >> 2) & 1);
  const bool bit1 = (lane & 2) != 0, bit0 = (lane & 1) != 0;
  float2* const pan[2] = {&panel[wave][0][lane ^ (2 * unit_turn(0, lane >> 3))],
                          &panel[wave][0][lane ^ (2 * unit_turn(1, lane >> 3))]};
  const float4* const prow = reinterpret_cast<const float4*>(&panel[wave][ps][8 * pr]);
  const int turn = unit_turn(ps, pr);
  float pg[3][8];
  {
    float* pf = reinterpret_cast<float*>(&panel[wave][0][0]);
    pf[lane] = g0;
    pf[64 + lane] = g1;
    pf[128 + lane] = g2;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int ch = 0; ch < 3; ++ch)
#pragma unroll
      for (int x = 0; x < 8; ++x) pg[ch][x] = pf[64 * ch + 8 * pr + x];
    __builtin_amdgcn_wave_barrier();
  }
  const float pgy = qy + (float)pr;
  __syncthreads();
  int jmax = 0;
  for (int w = 0; w < NW; ++w) jmax = max(jmax, (int)smax[w]);

  // the records of a batch are fetched while the one before it is walked (at four
  // waves per SIMD nothing else covers two dependent loads per batch)
  uint32_t rid = ~0u;
  RawRecord raw{};
  const auto fetch_batch = [&](int end) {
    const int beg = end > NB ? end - NB : 0;
    rid = (int)threadIdx.x < end - beg ? pair_rec[rg.x + beg + threadIdx.x] : ~0u;
    if (rid < n_rec) raw = fetch(rec, rid);
  };
  fetch_batch(jmax);
  const bool wild_pixel = wave_mask(!(fabsf(g0) + fabsf(g1) + fabsf(g2) + fabsf(gG) <= kTame &&
                                      fabsf(Sg) <= kTame * kTame)) != 0ull;
  for (int end = jmax; end > 0; end -= NB) {
    const int beg = end > NB ? end - NB : 0;
    const int m = end - beg;
    __syncthreads();
    if ((int)threadIdx.x < m) {
      srid[threadIdx.x] = rid;
      if (rid < n_rec) {
        stage(raw, tg.ox, tg.oy, s0[threadIdx.x], s1[threadIdx.x], s2[threadIdx.x]);
      } else {
        stage_empty(s0[threadIdx.x], s1[threadIdx.x], s2[threadIdx.x]);
      }
    }
    __syncthreads();
    if (beg > 0) fetch_batch(beg);
    // records this wavefront may need: positions below its own last blended one
    // whose cutoff ellipse meets its block, walked back to front
    uint64_t mask[NM];
    block_masks<NM>(s0, s1, min(m, wave_last - beg), qx, qy, mask);
    // batch positions this pixel blended (at most all NB: they are compared as byte offsets)
    const uint32_t lrel = lp > (uint32_t)beg ? min(lp - (uint32_t)beg, (uint32_t)NB) : 0u;
    int cnt = 0;
    bool opaque = false, wild_colour = false;
#pragma unroll
    for (int k = NM - 1; k >= 0; --k) {
      const uint64_t mk = mask[k];
      const int hits = __popcll(mk);
      if ((mk >> lane) & 1ull) {
        // its rank from the back
        list[wave][cnt + hits - 1 - mask_rank(mk)] = 16u * (uint32_t)(64 * k + lane);
        const float4 a2 = s2[64 * k + lane];
        opaque |= a2.x > kAlphaMax;
        wild_colour |= !tame_colour(a2);
      }
      cnt += hits;
    }
    const bool wild = wild_pixel || wave_mask(wild_colour) != 0ull;
    const bool caps = wave_mask(opaque) != 0ull || wild;   // some candidate's alpha may reach the cap
    const uint32_t lrel16 = 16u * lrel;
    if (wild) {
      // candidates that no pixel of the block blends leave the list (see kTame)
      __builtin_amdgcn_wave_barrier();
      int kept = 0;
      for (int c = 0; c < cnt; ++c) {
        const uint32_t off = list[wave][c];
        const float4 a0 = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(s0) + off);
        const float2 a1 = *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(s1) + off);
        const float q = gauss_q(a0.z, a0.w, a1.x, a0.x - fx, a0.y - fy);
        if (wave_mask((off < lrel16) & passes(q, a1.y)) != 0ull) list[wave][kept++] = off;
      }
      cnt = kept;
    }
    if (lane < kPanel) list[wave][cnt + lane] = 16u * NB;
    __builtin_amdgcn_wave_barrier();
    // candidates base + h .. base + h + G - 1: their tests and alphas do not depend on
    // each other, so G of them hide each other's latency where few waves are resident
    const auto group = [&](auto cap, int first, int h) {
      constexpr bool CAP = decltype(cap)::value;
        float alpha[G], ri[G], cg[G];
        bool none[G];   // no derivative: a capped alpha, or a pixel that did not blend (see kTame)
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const uint32_t off = list[wave][first + g];
          const float4 a0 = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(s0) + off);
          const float2 a1 = *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(s1) + off);
          const float4 a2 = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(s2) + off);
          const float q = gauss_q(a0.z, a0.w, a1.x, a0.x - fx, a0.y - fy);
          const bool on = (off < lrel16) & passes(q, a1.y);
          const float og = a2.x * __builtin_amdgcn_exp2f(-q);
          // alpha of this pixel, 0 where it did not blend: then 1 / (1 - alpha) = 1
          // exactly, transmittance and weight need no select and every sum gets zeros
          alpha[g] = on ? og : 0.0f;
          if (CAP) {
            none[g] = alpha[g] > kAlphaMax;
            alpha[g] = none[g] ? kAlphaMax : alpha[g];
            none[g] |= !on;
          }
          ri[g] = __builtin_amdgcn_rcpf(1.0f - alpha[g]);
          cg[g] = __fmaf_rn(g2, a2.w, __fmaf_rn(g1, a2.z, g0 * a2.y));
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
          Tr = Tr * ri[g];                       // transmittance in front of this Gaussian
          const float wgt = alpha[g] * Tr;
          // dL/dalpha = T (g . colour) - Sg / (1 - alpha) + gG, gG being the
          // load-balancing gradient of the pixel's soft count (each blended alpha enters
          // it with weight 1); dL/d(exponent) = alpha dL/dalpha, zero for a capped alpha
          const float dLda = __fmaf_rn(Tr, cg[g], __fmaf_rn(-Sg, ri[g], gG));
          Sg = __fmaf_rn(cg[g], wgt, Sg);
          float dpow = dLda * alpha[g];
          if (CAP) dpow = none[g] ? 0.0f : dpow;
          pan[(h + g) & 1][64 * (h + g)] = make_float2(dpow, wgt);
        }
    };
    for (int base = 0; base < cnt; base += kPanel) {
      // fill the panel, G candidates at a time
#pragma unroll
      for (int h = 0; h < kPanel; h += G) {
        if (base + h >= cnt) break;
        if (caps) group(std::true_type{}, base + h, h);
        else group(std::false_type{}, base + h, h);
      }
      __builtin_amdgcn_wave_barrier();
      // nine sums of this lane's row: the moments of dL/d(exponent) over (dx, dy,
      // dx^2, dx dy, dy^2) and itself, and the colour partials.  (The offsets are rounded
      // twice, from the splat to the block and on to the pixel; against 64 bits the 2D
      // gradients are as far off as with one rounding, 5.1e-7 to 1.2e-6 of their norm at
      // 37k Gaussians, and eight column numbers would not fit in the registers.)
      const uint32_t off = list[wave][base + ps];
      const float2 uw = *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(s0) + off);
      const float ux = uw.x - qx;
      float m0 = 0.0f, m1 = 0.0f, m2 = 0.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float4 v = prow[i ^ turn];
        const float dxa = ux - (float)(2 * i), dxb = ux - (float)(2 * i + 1);
        const float ta = v.x * dxa, tb = v.z * dxb;
        m0 += v.x;
        m1 += ta;
        m2 = __fmaf_rn(ta, dxa, m2);
        c0 = __fmaf_rn(pg[0][2 * i], v.y, c0);
        c1 = __fmaf_rn(pg[1][2 * i], v.y, c1);
        c2 = __fmaf_rn(pg[2][2 * i], v.y, c2);
        m0 += v.z;
        m1 += tb;
        m2 = __fmaf_rn(tb, dxb, m2);
        c0 = __fmaf_rn(pg[0][2 * i + 1], v.w, c0);
        c1 = __fmaf_rn(pg[1][2 * i + 1], v.w, c1);
        c2 = __fmaf_rn(pg[2][2 * i + 1], v.w, c2);
      }
      __builtin_amdgcn_wave_barrier();   // the panel may be written again
      const float dy = uw.y - pgy;
      const float n0 = dy * m0, n1 = dy * m1, n2 = dy * n0;
      // over the candidate's eight lanes: lane bits 2, 1, 0 select among the first
      // eight values; the ninth is summed in every lane
      const float e0 = fold_mirror_bit2(m1, n0), e1 = fold_mirror_bit2(m2, n1);
      const float e2 = fold_mirror_bit2(n2, m0), e3 = fold_mirror_bit2(c0, c1);
      const float f0 = fold_dpp<0x4E>(e0, e1, bit1), f1 = fold_dpp<0x4E>(e2, e3, bit1);
      const float tot = fold_dpp<0xB1>(f0, f1, bit0);
      c2 += dpp<0x141>(c2);
      c2 += dpp<0x4E>(c2);
      c2 += dpp<0xB1>(c2);
      if (base + ps < cnt) {
        const uint32_t j = off >> 4;
        if (ORDERED) {
          acc[wave][j][pc] = (Acc)tot;
          if (pr == 0) acc[wave][j][8] = (Acc)c2;
        } else {
          __hip_atomic_fetch_add((LdsDouble*)&acc[0][j][pc], (double)tot, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
          if (pr == 0)
            __hip_atomic_fetch_add((LdsDouble*)&acc[0][j][8], (double)c2, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      }
    }
    __syncthreads();
    if ((int)threadIdx.x < m) {
      Acc* ar = acc[0][threadIdx.x];
      float a[kGrad2D];
      for (int c = 0; c < kGrad2D; ++c) a[c] = (float)ar[c];
      // (two waves' rows in flight at T = 32: with all sixteen, 71 registers went to scratch memory)
      constexpr int kRowsAhead = NACC > 4 ? 2 : 4;
#pragma unroll kRowsAhead
      for (int w = 1; w < NACC; ++w)
        for (int c = 0; c < kGrad2D; ++c) a[c] += (float)acc[w][threadIdx.x][c];
      // moments -> partials: with exponent p = -(a dx^2 + 2 b dx dy + c dy^2)/2 and the
      // staged coefficients A, B, C = (a/2, b, c/2) log2(e):
      // dp/du = -ln2 (2A dx + B dy), dp/dw = -ln2 (B dx + 2C dy),
      // dp/da = -dx^2/2, dp/db = -dx dy, dp/dc = -dy^2/2
      const float A = s0[threadIdx.x].z, B = s0[threadIdx.x].w, C = s1[threadIdx.x].x;
      ar[0] = (Acc)(-kLn2 * (2.0f * A * a[0] + B * a[1]));
      ar[1] = (Acc)(-kLn2 * (B * a[0] + 2.0f * C * a[1]));
      ar[2] = (Acc)(-0.5f * a[2]);
      ar[3] = (Acc)(-a[3]);
      ar[4] = (Acc)(-0.5f * a[4]);
      // dL/dopacity: the exponent derivative summed over the tile's pixels is
      // sum dL/dalpha o G, so dividing by o gives sum dL/dalpha G
      const float o = s2[threadIdx.x].x;
      ar[5] = (Acc)(o > 0.0f ? a[5] / o : 0.0f);
      for (int c = 6; c < kGrad2D; ++c) ar[c] = (Acc)a[c];
    }
    __syncthreads();
    // one global atomic per (tile, Gaussian, component); consecutive lanes take
    // consecutive components, so a wavefront's atomics fall on a few cache lines
    // (element offsets in 64 bits: n_rec * 9 may pass 2^32 bytes)
    Acc* af = &acc[0][0][0];
    if (ORDERED) {
      float* po = grad2d + ((size_t)rg.x + (size_t)beg) * kGrad2D;
      for (int i = threadIdx.x; i < m * kGrad2D; i += NT) po[i] = srid[i / kGrad2D] < n_rec ? (float)af[i] : 0.0f;
      __syncthreads();
      for (int i = threadIdx.x; i < NACC * NB * kGrad2D; i += NT) af[i] = (Acc)0;
    } else {
      for (int i = threadIdx.x; i < m * kGrad2D; i += NT) {
        const int j = i / kGrad2D;
        const uint32_t r = srid[j];
        const float x = (float)af[i];
        if (x != 0.0f && r < n_rec)
          unsafeAtomicAdd(grad2d + ((size_t)r * kGrad2D + (size_t)(i - kGrad2D * j)), x);
        af[i] = (Acc)0;
      }
    }
  }
  if (ORDERED) {
    // list positions no pixel of the tile reached: zero partials
    const size_t len = rg.y > rg.x ? (size_t)(rg.y - rg.x) : 0;
    float* po = grad2d + (size_t)rg.x * kGrad2D;
    for (size_t i = (size_t)jmax * kGrad2D + threadIdx.x; i < len * kGrad2D; i += NT) po[i] = 0.0f;
  }
}

}  // namespace

hipError_t launch_render_fwd(const ViewDev* views, int V, int n_tiles, const uint2* ranges, const uint32_t* pair_rec,
                             const Record* rec, uint32_t n_rec, float* color, float* t_final, uint32_t* n_contrib,
                             uint32_t* last, float* asum, int tile, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  // four 8x8 blocks to a workgroup
  const int64_t groups = ((int64_t)n_tiles * (tile / 8) * (tile / 8) + 3) / 4, round = 8 * kXcdRun;
  const dim3 grid((unsigned)((groups + round - 1) / round * round));
#define GS_FWD(TT)                                                                                                  \
  hipLaunchKernelGGL(k_render_fwd<TT>, grid, dim3(256), 0, s, views, V, n_tiles, ranges, pair_rec, rec, n_rec, color, \
                     t_final, n_contrib, last, asum)
  switch (tile) {
    case 8: GS_FWD(8); break;
    case 16: GS_FWD(16); break;
    case 32: GS_FWD(32); break;
    default: return hipErrorInvalidValue;
  }
#undef GS_FWD
  return hipGetLastError();
}

hipError_t launch_render_count(const ViewDev* views, int V, int n_tiles, const uint2* ranges, const uint32_t* pair_rec,
                               const Record* rec, uint32_t n_rec, uint32_t* evals, uint32_t* pairs_eff, int tile,
                               hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  const dim3 grid((unsigned)((n_tiles + 8 * kXcdRun - 1) / (8 * kXcdRun) * (8 * kXcdRun)));
#define GS_COUNT(TT)                                                                                                  \
  hipLaunchKernelGGL(k_render_count<TT>, grid, dim3(TT * TT), 0, s, views, V, n_tiles, ranges, pair_rec, rec, n_rec, \
                     evals, pairs_eff)
  switch (tile) {
    case 8: GS_COUNT(8); break;
    case 16: GS_COUNT(16); break;
    case 32: GS_COUNT(32); break;
    default: return hipErrorInvalidValue;
  }
#undef GS_COUNT
  return hipGetLastError();
}

hipError_t launch_render_bwd(const ViewDev* views, int V, int n_tiles, const uint2* ranges, const uint32_t* pair_rec,
                             const Record* rec, uint32_t n_rec, const float* t_final, const uint32_t* last,
                             const float* dL_dcolor, const float* dL_dG, float* grad2d, int tile, int ordered,
                             hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  const dim3 grid((unsigned)((n_tiles + 8 * kXcdRun - 1) / (8 * kXcdRun) * (8 * kXcdRun)));
#define GS_BWD(TT, OO)                                                                                            \
  hipLaunchKernelGGL((k_render_bwd<TT, OO>), grid, dim3(TT * TT), 0, s, views, V, n_tiles, ranges, pair_rec, rec, \
                     n_rec, t_final, last, dL_dcolor, dL_dG, grad2d)
  switch (tile) {
    case 8: if (ordered) GS_BWD(8, true); else GS_BWD(8, false); break;
    case 16: if (ordered) GS_BWD(16, true); else GS_BWD(16, false); break;
    case 32: if (ordered) GS_BWD(32, true); else GS_BWD(32, false); break;
    default: return hipErrorInvalidValue;
  }
#undef GS_BWD
  return hipGetLastError();
}

}  // namespace gsk
