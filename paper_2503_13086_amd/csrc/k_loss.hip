// Image loss terms of Eq. 10 and dL/dimage for gfx950.
//
// Per view: w_l1 * mean|x - y| + w_dssim * (1 - mean SSIM(x, y)), SSIM per channel
// from windowed means under a normalised 11x11 Gaussian window (sigma 1.5, zero
// padding), C1 = 0.01^2, C2 = 0.03^2.  All views share one launch.  E[x^2] and E[y^2]
// enter SSIM only through their sum (in D2), so four maps are filtered: x, y,
// x^2 + y^2 and xy.
//
// Backward: with N1 = 2 mx my + C1, N2 = 2 sxy + C2, D1 = mx^2 + my^2 + C1,
// D2 = sxx + syy + C2 and S = N1 N2 / (D1 D2), the per-pixel partials of S with
// respect to the windowed statistics (mx, E[x^2], E[xy]) are
//   A = 2 my (N2 - N1) / (D1 D2) + 2 mx S (1/D2 - 1/D1),  B = -S / D2,
//   Cc = 2 N1 / (D1 D2),
// and dS_mean/dx = (window * A + 2 x (window * B) + y (window * Cc)) / N (the window
// is symmetric), with 1/D1 and 1/D2 taken once per pixel from the hardware reciprocal.
// k_ssim forms all of it in one pass over the images.
// Loss sums are taken in FP64, over blocks of a view that its own size decides and then
// over the view's blocks in order: a view's loss is the same bits in any batch.
//
// The load-balancing term of Eq. 9 (kernels at the end) works on the soft
// per-pixel Gaussian count the forward writes.
#include "gs_internal.h"

namespace gsk {
namespace {

constexpr int LT = 32;              // k_l1's tile edge
constexpr int R = 5;                // window radius
constexpr int TAPS = 2 * R + 1;
constexpr int kSsimOccupancy = 3;   // k_ssim's wavefronts per SIMD (156 registers; at four they spill)
constexpr int SW = 64 - 4 * R;      // k_ssim: output columns of a wavefront (two windows less than its lanes)
constexpr int kMaxRows = 12;        // k_ssim's strips: at most so many TAPS rows
constexpr float kC1 = 0.01f * 0.01f;
constexpr float kC2 = 0.03f * 0.03f;

struct Win {
  float w[TAPS];
};


__device__ inline double block_sum_d(double x, double* sh) {
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
  if (__lane_id() == 0) sh[threadIdx.x / 64] = x;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < (int)(blockDim.x / 64); ++w) t += sh[w];
  __syncthreads();
  return t;
}

struct TileLoc {
  int v, x0, y0;
};

// Workgroups are dealt to the chip's 8 XCDs round-robin (workgroup b runs on XCD
// b mod 8), each XCD with its own L2.  Workgroup b takes tile (b mod 8) * chunk +
// b / 8, so every XCD walks a contiguous range of tiles and the halo rows that
// neighbouring tiles share are fetched into one L2.  Tiles past the end (at most
// 7 workgroups) return at once.
constexpr int kXcds = 8;

__host__ __device__ inline int xcd_tile_chunk(int n_tiles) { return (n_tiles + kXcds - 1) / kXcds; }

__device__ inline int xcd_tile(int b, int n_tiles) { return (b % kXcds) * xcd_tile_chunk(n_tiles) + b / kXcds; }

__device__ inline int loss_view(const LossOffsets& lt, int V, int tile) {
  int v = 0;
  while (v + 1 < V && tile >= lt.off[v + 1]) ++v;
  return v;
}

__device__ inline TileLoc loss_tile(const ViewDev* __restrict__ views, const LossOffsets& lt, int V, int tile) {
  const int v = loss_view(lt, V, tile);
  const int nx = (views[v].W + LT - 1) / LT;
  const int local = tile - lt.off[v];
  return TileLoc{v, (local % nx) * LT, (local / nx) * LT};
}

__global__ __launch_bounds__(256) void k_l1(const ViewDev* __restrict__ views, int V, LossOffsets lt,
                                             const float* __restrict__ x, const float* __restrict__ y, float w_l1,
                                             float* __restrict__ grad, double2* __restrict__ partials) {
  __shared__ double sh[4];
  const int tile = xcd_tile(blockIdx.x, lt.off[V]);
  if (tile >= lt.off[V]) return;
  const TileLoc t = loss_tile(views, lt, V, tile);
  const ViewDev& cv = views[t.v];
  const size_t hw = (size_t)cv.W * cv.H;
  const size_t base = 3 * (size_t)cv.pix_off;
  const float inv = w_l1 / (float)(3 * hw);
  double s = 0.0;
  for (int i = threadIdx.x; i < LT * LT; i += blockDim.x) {
    const int px = t.x0 + i % LT, py = t.y0 + i / LT;
    if (px >= cv.W || py >= cv.H) continue;
    const size_t p = base + (size_t)py * cv.W + px;
    for (int c = 0; c < 3; ++c) {
      const float d = x[p + c * hw] - y[p + c * hw];
      s += fabs((double)d);
      grad[p + c * hw] = inv * (float)((d > 0.0f) - (d < 0.0f));
    }
  }
  const double tot = block_sum_d(s, sh);
  if (threadIdx.x == 0) partials[tile] = make_double2(tot, 0.0);
}

// Q vertical windows: acc[q][s] sums output row s mod TAPS, which the TAPS input rows
// from it on reach.  Takes input row u mod TAPS (u a constant, so that the sums rotate
// through the registers without moves) and returns the row that is then complete.
template <int Q>
__device__ inline void window_rows(int u, const float (&w)[R + 1], const float (&v)[Q], float (&acc)[Q][TAPS],
                                   float (&fin)[Q]) {
#pragma unroll
  for (int k = 0; k < TAPS; ++k) {
    const int s = (u - k + TAPS) % TAPS;
#pragma unroll
    for (int q = 0; q < Q; ++q)
      acc[q][s] = k == 0 ? w[0] * v[q] : __fmaf_rn(w[k < R ? k : TAPS - 1 - k], v[q], acc[q][s]);
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) fin[q] = acc[q][(u + 1) % TAPS];
}

// Orders a wavefront's LDS accesses (which execute in order) for the compiler: lanes
// read what other lanes wrote.
__device__ inline void lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The horizontal window: lane l's sums over lanes l .. l + TAPS - 1 of Q values, through
// one 16-byte LDS word per lane (the last TAPS - 1 lanes read past the 64 values that
// are there and have no result).  In two parts, for other work while the words travel.
template <int Q>
struct Neighbours {
  float v[TAPS][Q];
};
template <int Q>
__device__ inline void window_cols_load(float4* buf, const float (&v)[Q], Neighbours<Q>& nb) {
  static_assert(Q == 3 || Q == 4, "one 16-byte word");
  const int lane = __lane_id();
  lds_order();   // the reads of the row before
  buf[lane] = make_float4(v[0], v[1], v[2], Q > 3 ? v[Q - 1] : 0.0f);
  lds_order();
#pragma unroll
  for (int q = 0; q < Q; ++q) nb.v[0][q] = v[q];
#pragma unroll
  for (int k = 1; k < TAPS; ++k) {
    const float4 n = buf[lane + k];
    const float nv[4] = {n.x, n.y, n.z, n.w};
#pragma unroll
    for (int q = 0; q < Q; ++q) nb.v[k][q] = nv[q];
  }
}
template <int Q>
__device__ inline void window_cols_sum(const float (&w)[R + 1], const Neighbours<Q>& nb, float (&out)[Q]) {
#pragma unroll
  for (int k = 0; k < TAPS; ++k)
#pragma unroll
    for (int q = 0; q < Q; ++q)
      out[q] = k == 0 ? w[0] * nb.v[k][q] : __fmaf_rn(w[k < R ? k : TAPS - 1 - k], nb.v[k][q], out[q]);
  // the sums are formed here: left alone, the compiler moves them to where the vertical
  // windows are used and keeps every word live until then
#pragma unroll
  for (int q = 0; q < Q; ++q) asm volatile("" : "+v"(out[q]));
}

// Sums over the wavefront, a's in the lower 32 lanes and b's in the upper: half_sums pairs
// the lanes, whole_sums finishes.  By lane swaps and DPP (shuffles through LDS would hold
// a register for every lane distance).
struct Words {
  uint32_t lo, hi;
};
__device__ inline Words words(double x) {
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  return Words{(uint32_t)u, (uint32_t)(u >> 32)};
}
__device__ inline double from_words(uint32_t lo, uint32_t hi) {
  return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}
template <int CTRL>
__device__ inline double dpp_add(double x) {
  const Words w = words(x);
  return x + from_words((uint32_t)__builtin_amdgcn_update_dpp(0, (int)w.lo, CTRL, 0xf, 0xf, true),
                        (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w.hi, CTRL, 0xf, 0xf, true));
}
__device__ inline double half_sums(double a, double b) {
  const Words wa = words(a), wb = words(b);
  const auto l32 = __builtin_amdgcn_permlane32_swap(wa.lo, wb.lo, false, false);
  const auto h32 = __builtin_amdgcn_permlane32_swap(wa.hi, wb.hi, false, false);
  return from_words(l32[0], h32[0]) + from_words(l32[1], h32[1]);
}
__device__ inline double whole_sums(double x) {
  const Words w = words(x);
  const auto l16 = __builtin_amdgcn_permlane16_swap(w.lo, w.lo, false, false);
  const auto h16 = __builtin_amdgcn_permlane16_swap(w.hi, w.hi, false, false);
  x = from_words(l16[0], h16[0]) + from_words(l16[1], h16[1]);
  x = dpp_add<0x128>(x);    // lane l ^ 8
  x = dpp_add<0x141>(x);    // lane 7 - l of its eight
  x = dpp_add<0x4E>(x);     // lane l ^ 2
  return dpp_add<0xB1>(x);  // lane l ^ 1
}

// The SSIM term and both terms' gradient.  A wavefront takes one channel of SW columns
// by some rows (a strip) and walks down them, a lane per column: each row's four maps go
// through LDS into the horizontal windows and from there into the vertical ones; the row
// these finish gives S and A, B, Cc, which go through the second horizontal and vertical
// windows, and the row those finish is a row of the gradient.  So each image is read once
// (and a fifth around it), nothing else but the gradient touches HBM and no barrier is
// met.  What it does again: a strip passes over its rows + 4R rows and 64 columns for its
// SW.
// The sums of each block of a strip (some TAPS rows, see ssim_block) are kept by
// themselves, so that they do not depend on how many blocks a strip has: in LDS, folded
// over the lanes at the end (in the loop that takes 10 registers, and 10 % more time for
// the spills).
// Bound by instruction issue (about 185 vector instructions a row, of which 154 the
// windows' multiply-adds) and the 22 16-byte LDS accesses a row beside it.  It replaced
// two kernels over 32x32 tiles with the statistics in HBM between them (36 bytes a pixel
// written and read) and, for gs_loss_noalloc, one over 52x52 patches: 10.1 Mpix in 9
// views 426 -> 282 us (both terms and the final sums), 1600x1067 87 -> 74, 1296x864
// 63 -> 54, three views of 0.2 Mpix in all 38 -> 23.
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kSsimOccupancy))) void k_ssim(
    const ViewDev* __restrict__ views, int V, LossPlan plan, const float* __restrict__ x,
    const float* __restrict__ y, Win win, float w_l1, float w_dssim, float* __restrict__ grad,
    double* __restrict__ partials) {
  __shared__ float4 buf[2][64 + TAPS - 1];
  __shared__ double lane_sums[kMaxRows][64];
  const int wave = xcd_tile(blockIdx.x, 3 * plan.tiles.off[V]), tile = wave / 3, ch = wave % 3;
  if (tile >= plan.tiles.off[V]) return;
  const int v = loss_view(plan.tiles, V, tile);
  const ViewDev& cv = views[v];
  const int W = cv.W, H = cv.H, lane = __lane_id();
  const int cols = (W + SW - 1) / SW, local = tile - plan.tiles.off[v], block = plan.block[v];
  const int rows = TAPS * block * plan.blocks[v], nb = (H + TAPS * block - 1) / (TAPS * block);
  const TileLoc t{v, (local % cols) * SW, (local / cols) * rows};
  // the strip's sums: its blocks' pairs, after those of the channels and strips before it
  double* sums = partials + 2 * ((size_t)plan.sums.off[v] + (size_t)((ch * cols + local % cols) * nb) +
                                 (size_t)((local / cols) * plan.blocks[v]));
  const size_t hw = (size_t)W * H;
  const size_t plane = 3 * (size_t)cv.pix_off + ch * hw;
  const float invN = 1.0f / (float)(3 * hw);
  float w[R + 1];   // (in vector registers: a scalar operand halves the rate of an FMA)
#pragma unroll
  for (int k = 0; k <= R; ++k) {
    w[k] = win.w[k];
    asm volatile("" : "+v"(w[k]));
  }
  // Lane l reads column x0 - 2R + l, has the statistics of column x0 - R + l (l < 54) and
  // the gradient of column x0 + l (l < SW).
  const int cin = t.x0 - 2 * R + lane, cst = cin + R, cout = t.x0 + lane;
  const bool st_ok = cst >= 0 && cst < W, out_ok = lane < SW && cout < W;
  const bool st_own = st_ok && lane >= R && lane < SW + R;   // counted here
  const int y_end = min(t.y0 + rows, H);                     // rows of this strip: [y0, y_end)
  // The images go through buffer descriptors that begin at the first row read (or the
  // tile's own first row) and end with the image: what lies outside reads as zero, the
  // padding, and is not written, with no branch around a load or a store (at which all
  // loads in flight would be waited for).  Columns outside get an offset that no row
  // brings back in range.
  const uint32_t pitch = 4u * (uint32_t)W, off_image = 0x80000000u;
  const int r_in = max(t.y0 - 2 * R, 0);
  const auto rows_of = [&](const float* im, int r) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(im) + plane + (size_t)r * W, 0,
                                             (int)(pitch * (uint32_t)min(H - r, rows + 4 * R)), 0x00020000);
  };
  const __amdgpu_buffer_rsrc_t xi = rows_of(x, r_in), yi = rows_of(y, r_in), xo = rows_of(x, t.y0),
                               yo = rows_of(y, t.y0), go = rows_of(grad, t.y0);
  const auto at = [](__amdgpu_buffer_rsrc_t im, uint32_t off) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(im, off, 0, 0));
  };
  // offsets of the next row to load, of the next row whose values are loaded for the
  // gradient, and of the next gradient row to store (the last two begin above the tile)
  uint32_t off_in = (cin >= 0 && cin < W ? 4u * (uint32_t)cin : off_image) +
                    pitch * (uint32_t)(t.y0 - 2 * R - r_in);
  uint32_t off_out = (out_ok ? 4u * (uint32_t)cout : off_image) - pitch * (uint32_t)(2 * R + 1);
  float acc1[4][TAPS], acc2[3][TAPS];
#pragma unroll
  for (int j = 0; j < TAPS; ++j) {
#pragma unroll
    for (int q = 0; q < 4; ++q) acc1[q][j] = 0.0f;
#pragma unroll
    for (int q = 0; q < 3; ++q) acc2[q][j] = 0.0f;
  }
  double sl1 = 0.0, sss = 0.0, sss_block = 0.0;
  bool ends = false;   // this block's last rows are on their way
  // image values of the next AHEAD rows
  constexpr int AHEAD = 2;
  float nx[AHEAD], ny[AHEAD];
#pragma unroll
  for (int k = 0; k < AHEAD; ++k) {
    nx[k] = at(xi, off_in);
    ny[k] = at(yi, off_in);
    off_in += pitch;
  }
  // the maps of the next row of the images, through the first horizontal windows' exchange
  const auto take = [&](Neighbours<4>& nb) {
    const float xv = nx[0], yv = ny[0];
#pragma unroll
    for (int k = 0; k + 1 < AHEAD; ++k) {
      nx[k] = nx[k + 1];
      ny[k] = ny[k + 1];
    }
    nx[AHEAD - 1] = at(xi, off_in);
    ny[AHEAD - 1] = at(yi, off_in);
    off_in += pitch;
    const float maps[4] = {xv, yv, __fmaf_rn(xv, xv, yv * yv), xv * yv};
    window_cols_load<4>(buf[0], maps, nb);
  };
  // the gradient row whose sums g are (from the row above the tile's first 2R + 1 on, of
  // which nothing is stored)
  float xc = 0.0f, yc = 0.0f;
  const auto give = [&](const float (&g)[3]) {
    const float d = xc - yc;
    sl1 += fabs((double)d);   // (zero where there is no pixel)
    const float l1 = w_l1 * invN * (float)((d > 0.0f) - (d < 0.0f));
    __builtin_amdgcn_raw_buffer_store_b32(
        __float_as_uint(l1 - w_dssim * invN * (g[0] + 2.0f * xc * g[1] + yc * g[2])), go, off_out, 0, 0);
    off_out += pitch;
    xc = at(xo, off_out);
    yc = at(yo, off_out);
  };
  // Each of a row's two exchanges overlaps arithmetic of the row before or after: the
  // images are taken a row ahead, and the second vertical windows lag by a row.
  float m[4], h1[4], h2[3] = {0.0f, 0.0f, 0.0f}, g[3];
  const auto row = [&](int u, int i) {   // u = i mod TAPS
    Neighbours<4> nb1;
    take(nb1);
    window_rows<3>((u + TAPS - 1) % TAPS, w, h2, acc2, g);
    give(g);
    const int rst = t.y0 - 3 * R + i;                        // the statistics' row
    const float mx = m[0], my = m[1];
    // (fused operations written out: the statistics cancel, so their roundings show)
    const float sxy = __fmaf_rn(-mx, my, m[3]);
    const float N1 = __fmaf_rn(2.0f * mx, my, kC1), N2 = __fmaf_rn(2.0f, sxy, kC2);
    const float M2 = __fmaf_rn(mx, mx, my * my);
    const float D1 = M2 + kC1, D2 = (m[2] - M2) + kC2;
    // hardware reciprocals (1 ulp): D1, D2 >= C1 > 0
    const float r1 = __builtin_amdgcn_rcpf(D1), r2 = __builtin_amdgcn_rcpf(D2);
    const float rden = r1 * r2;
    const float S = (N1 * N2) * rden;
    const bool ok = st_ok && rst >= 0 && rst < H, own = st_own && rst >= t.y0 && rst < y_end;
    const float abc[3] = {ok ? __fmaf_rn(2.0f * my * (N2 - N1), rden, 2.0f * mx * S * (r2 - r1)) : 0.0f,
                          ok ? -S * r2 : 0.0f, ok ? 2.0f * N1 * rden : 0.0f};
    // (at u = 3R mod TAPS the statistics enter the next TAPS rows)
    if (u == 3 * R % TAPS) {
      sss_block = sss;
      sss = ends ? 0.0 : sss;
    }
    sss += own ? (double)S : 0.0;
    window_cols_sum<4>(w, nb1, h1);
    Neighbours<3> nb2;
    window_cols_load<3>(buf[1], abc, nb2);
    window_rows<4>((u + 1) % TAPS, w, h1, acc1, m);
    __builtin_amdgcn_sched_barrier(0);   // (the words' sums stay after the rows': 7 % at any size)
    window_cols_sum<3>(w, nb2, h2);
  };
#pragma unroll
  for (int u = 0; u <= 2 * R; ++u) {
    Neighbours<4> nb1;
    take(nb1);
    window_cols_sum<4>(w, nb1, h1);
    window_rows<4>(u, w, h1, acc1, m);
  }
  // After k rounds of TAPS rows the gradient has its first TAPS (k - 1) rows and the
  // statistics are R + 1 rows ahead.
  const int rounds = (y_end - t.y0 + TAPS - 1) / TAPS;
  int left = block + 1, done = 0;
  for (int k = 0; k <= rounds; ++k) {   // (rows past y_end, at the bottom of a view, are all outside)
    ends = --left == 0 || k == rounds;
#pragma unroll
    for (int u = 0; u < TAPS; ++u) row((2 * R + u) % TAPS, 2 * R + TAPS * k + u);
    lane_sums[done][lane] = half_sums(sl1, sss_block);   // (whole after the block's last round)
    sl1 = ends ? 0.0 : sl1;
    done += ends ? 1 : 0;
    left = ends ? block : left;
  }
  for (int b = 0; b < done; ++b) {
    const double sum = whole_sums(lane_sums[b][lane]);
    if ((lane & 31) == 0) sums[2 * b + (lane >> 5)] = sum;
  }
}

// One workgroup per view: the view's partial sums added up in FP64, kFinalBatch loads of a
// thread in flight (7110 sums of 1296x864 are two round trips to memory).
constexpr int kFinalBatch = 16;
__global__ __launch_bounds__(256) void k_loss_final(const ViewDev* __restrict__ views, LossOffsets lt,
                                                     const double2* __restrict__ partials, float w_l1,
                                                     float w_dssim, int ssim, double* __restrict__ out) {
  __shared__ double sh[4];
  const int v = blockIdx.x;
  const ViewDev& cv = views[v];
  const int end = lt.off[v + 1];
  double a = 0.0, b = 0.0;
  for (int t = lt.off[v] + threadIdx.x; t < end; t += 256 * kFinalBatch) {
    double2 pt[kFinalBatch];
#pragma unroll
    for (int k = 0; k < kFinalBatch; ++k) pt[k] = t + 256 * k < end ? partials[t + 256 * k] : make_double2(0.0, 0.0);
#pragma unroll
    for (int k = 0; k < kFinalBatch; ++k) {
      a += pt[k].x;
      b += pt[k].y;
    }
  }
  a = block_sum_d(a, sh);
  b = block_sum_d(b, sh);
  if (threadIdx.x == 0) {
    const double N = 3.0 * (double)cv.W * (double)cv.H;
    double l = (double)w_l1 * a / N;
    if (ssim) l += (double)w_dssim * (1.0 - b / N);
    out[v] = l;
  }
}

// ---- Eq. 9 load-balancing term on the soft per-pixel count G_p (sum of the
// alphas a pixel blended, written by the forward): per view, L = w std_p(G_p)
// (population std) and dL/dG_p = w (G_p - mean) / (P std) (0 when std = 0).
// Sums of G and G^2 are taken in FP64 per 2048-pixel chunk, then per view.
constexpr int kLoadChunk = 2048;

__global__ __launch_bounds__(256) void k_load_partial(const ViewDev* __restrict__ views,
                                                      const float* __restrict__ asum, int chunks,
                                                      double2* __restrict__ part) {
  __shared__ double sh[4];
  const ViewDev& cv = views[blockIdx.y];
  const int64_t P = (int64_t)cv.W * cv.H;
  const int64_t base = (int64_t)blockIdx.x * kLoadChunk;
  double a = 0.0, b = 0.0;
  for (int k = 0; k < kLoadChunk / 256; ++k) {
    const int64_t i = base + k * 256 + threadIdx.x;
    if (i < P) {
      const double g = (double)asum[cv.pix_off + i];
      a += g;
      b += g * g;
    }
  }
  a = block_sum_d(a, sh);
  b = block_sum_d(b, sh);
  if (threadIdx.x == 0) part[(size_t)blockIdx.y * chunks + blockIdx.x] = make_double2(a, b);
}

__global__ __launch_bounds__(256) void k_load_final(const ViewDev* __restrict__ views, int chunks,
                                                    const double2* __restrict__ part, float w,
                                                    double2* __restrict__ stats, double* __restrict__ loss_out) {
  __shared__ double sh[4];
  const int v = blockIdx.x;
  const ViewDev& cv = views[v];
  const int64_t P = (int64_t)cv.W * cv.H;
  const int nc = (int)((P + kLoadChunk - 1) / kLoadChunk);
  double a = 0.0, b = 0.0;
  for (int t = threadIdx.x; t < nc; t += blockDim.x) {
    a += part[(size_t)v * chunks + t].x;
    b += part[(size_t)v * chunks + t].y;
  }
  a = block_sum_d(a, sh);
  b = block_sum_d(b, sh);
  if (threadIdx.x == 0) {
    const double m = a / (double)P;
    const double var = fmax(b / (double)P - m * m, 0.0);
    const double sd = sqrt(var);
    stats[v] = make_double2(m, sd > 0.0 ? (double)w / ((double)P * sd) : 0.0);
    if (loss_out) loss_out[v] = (double)w * sd;
  }
}

__global__ __launch_bounds__(256) void k_load_grad(const ViewDev* __restrict__ views,
                                                   const double2* __restrict__ stats,
                                                   const float* __restrict__ asum, float* __restrict__ dG) {
  const ViewDev& cv = views[blockIdx.y];
  const int64_t P = (int64_t)cv.W * cv.H;
  const double2 st = stats[blockIdx.y];
  const int64_t base = (int64_t)blockIdx.x * kLoadChunk;
  for (int k = 0; k < kLoadChunk / 256; ++k) {
    const int64_t i = base + k * 256 + threadIdx.x;
    if (i < P) dG[cv.pix_off + i] = (float)(((double)asum[cv.pix_off + i] - st.x) * st.y);
  }
}

}  // namespace

int load_chunks(const ViewDev* hviews, int V) {
  int64_t mx = 1;
  for (int v = 0; v < V; ++v) {
    const int64_t c = ((int64_t)hviews[v].W * hviews[v].H + kLoadChunk - 1) / kLoadChunk;
    mx = c > mx ? c : mx;
  }
  return (int)mx;
}

hipError_t launch_load_balance(const ViewDev* dviews, const ViewDev* hviews, int V, const float* asum, float w,
                               double* partials, double* stats, double* loss_out, float* dG, hipStream_t s) {
  const int chunks = load_chunks(hviews, V);
  double2* part = reinterpret_cast<double2*>(partials);
  double2* st = reinterpret_cast<double2*>(stats);
  hipLaunchKernelGGL(k_load_partial, dim3(chunks, V), dim3(256), 0, s, dviews, asum, chunks, part);
  hipLaunchKernelGGL(k_load_final, dim3(V), dim3(256), 0, s, dviews, chunks, part, w, st, loss_out);
  hipLaunchKernelGGL(k_load_grad, dim3(chunks, V), dim3(256), 0, s, dviews, st, asum, dG);
  return hipGetLastError();
}

int loss_tiles(const ViewDev* hviews, int V) {
  int t = 0;
  for (int v = 0; v < V; ++v) t += ((hviews[v].W + LT - 1) / LT) * ((hviews[v].H + LT - 1) / LT);
  return t;
}

namespace {
constexpr int kSsimWaves = 1024 * kSsimOccupancy;   // wavefronts the chip holds at once

int ceil_div(int a, int b) { return (a + b - 1) / b; }

// A strip of r rows passes over r + 4R, so taller is less work, but all its rows one after
// the other: what a launch takes goes with the rounds of as many wavefronts as fit on the
// chip times the rows of a round.  In a training step (the target out of the caches)
// 1296x864 takes 62 us with strips of 22 rows (3600 wavefronts), 58 with 33 (2430), 63 with
// 44; 1600x1067 81 with 33 (3663), 72 with 44 (2775), 78 with 55; 2048x2048 148 with 77
// (3807), 126 with 99 (2961), 142 with 110; two views of 1296x864 94 with 44 (3600), 83
// with 55 (2880), 90 with 66; ten megapixels in nine views 290 with 132 (5922), 296 with 88.
int64_t ssim_cost(int64_t tiles, int rows) {
  return (3 * tiles + kSsimWaves - 1) / kSsimWaves * (rows + 4 * R);
}

// Rows of a view's blocks, in TAPS, by the view alone (its sums have to be its own): a part
// of the strip that is best for it alone, so that this is made of them, and small, so that
// the strips of a batch can be; but no more blocks than k_loss_final adds up at no cost.
int ssim_block(const ViewDev& v) {
  const int64_t cols = ceil_div(v.W, SW);
  int best = 1;
  for (int r = 2; r <= kMaxRows; ++r)
    if (ssim_cost(cols * ceil_div(v.H, TAPS * r), TAPS * r) < ssim_cost(cols * ceil_div(v.H, TAPS * best), TAPS * best))
      best = r;
  int b = 1;
  while (b < best && (best % b != 0 || 3 * cols * ceil_div(v.H, TAPS * b) > 8192)) ++b;
  return b;
}
static_assert(SW >= LT && 3 * TAPS >= LT && kLossSums >= (size_t)9 * kLossTiles,
              "at most three blocks, of three channels, to a 32x32 tile");
}  // namespace

LossPlan loss_plan(const ViewDev* hviews, int V, bool ssim) {
  LossPlan p{};
  if (!ssim) {
    for (int v = 0; v < V; ++v)
      p.tiles.off[v + 1] = p.tiles.off[v] + ceil_div(hviews[v].W, LT) * ceil_div(hviews[v].H, LT);
    p.sums = p.tiles;
    return p;
  }
  for (int v = 0; v < V; ++v) {
    const int b = ssim_block(hviews[v]);
    p.block[v] = (uint8_t)b;
    p.sums.off[v + 1] = p.sums.off[v] + 3 * ceil_div(hviews[v].W, SW) * ceil_div(hviews[v].H, TAPS * b);
  }
  // blocks of a strip: as many as fit the height that is best for the batch
  int64_t best_cost = 0;
  for (int r = 1; r <= kMaxRows; ++r) {
    int64_t tiles = 0;
    int rows = 0;
    for (int v = 0; v < V; ++v) {
      const int h = TAPS * p.block[v] * (r > p.block[v] ? r / p.block[v] : 1);
      tiles += (int64_t)ceil_div(hviews[v].W, SW) * ceil_div(hviews[v].H, h);
      rows = h > rows ? h : rows;
    }
    const int64_t cost = ssim_cost(tiles, rows);
    if (r > 1 && cost >= best_cost) continue;
    best_cost = cost;
    for (int v = 0; v < V; ++v) p.blocks[v] = (uint8_t)(r > p.block[v] ? r / p.block[v] : 1);
  }
  for (int v = 0; v < V; ++v)
    p.tiles.off[v + 1] = p.tiles.off[v] + ceil_div(hviews[v].W, SW) *
                                              ceil_div(hviews[v].H, TAPS * p.block[v] * p.blocks[v]);
  return p;
}

hipError_t launch_loss_dev(const ViewDev* dviews, int V, const LossPlan& plan, const float* color,
                           const float* target, float w_l1, float w_dssim, double* partials, double* loss_out,
                           float* dL_dcolor, hipStream_t s) {
  Win win;
  double g[TAPS], tot = 0.0;
  for (int k = 0; k < TAPS; ++k) {
    const double d = (double)(k - R);
    g[k] = exp(-(d * d) / (2.0 * 1.5 * 1.5));
    tot += g[k];
  }
  for (int k = 0; k < TAPS; ++k) win.w[k] = (float)(g[k] / tot);
  const bool ssim = w_dssim != 0.0f;
  double2* part = reinterpret_cast<double2*>(partials);
  // at least as many workgroups as tiles, see xcd_tile
  const dim3 grid(kXcds * xcd_tile_chunk((ssim ? 3 : 1) * plan.tiles.off[V]));
  if (!ssim)
    hipLaunchKernelGGL(k_l1, grid, dim3(256), 0, s, dviews, V, plan.tiles, color, target, w_l1, dL_dcolor, part);
  else
    hipLaunchKernelGGL(k_ssim, grid, dim3(64), 0, s, dviews, V, plan, color, target, win, w_l1, w_dssim, dL_dcolor,
                       partials);
  if (loss_out)
    hipLaunchKernelGGL(k_loss_final, dim3(V), dim3(256), 0, s, dviews, plan.sums, part, w_l1, w_dssim, ssim ? 1 : 0,
                       loss_out);
  return hipGetLastError();
}

}  // namespace gsk
