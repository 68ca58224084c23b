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
// Loss sums are reduced per workgroup in FP64.
//
// The load-balancing term of Eq. 9 (kernels at the end) works on the soft
// per-pixel Gaussian count the forward writes.
#include "gs_internal.h"

namespace gsk {
namespace {

constexpr int LT = 32;              // k_l1's tile edge
constexpr int R = 5;                // window radius
constexpr int TAPS = 2 * R + 1;
constexpr int kSsimOccupancy = 3;   // k_ssim's wavefronts per SIMD (147 registers; at four they spill)
constexpr int SW = 64 - 4 * R;      // k_ssim: output columns of a wavefront (two windows less than its lanes)
constexpr float kC1 = 0.01f * 0.01f;
constexpr float kC2 = 0.03f * 0.03f;

struct Win {
  float w[TAPS];
};

// global offset of each view's tiles (n_views + 1 entries): 32x32 pixels (k_l1) or SW
// columns by a number of rows (k_ssim)
struct LossTiles {
  int32_t off[GS_MAX_VIEWS + 1];
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

__device__ inline TileLoc loss_tile(const ViewDev* __restrict__ views, const LossTiles& lt, int V, int tile, int tw,
                                    int th) {
  int v = 0;
  while (v + 1 < V && tile >= lt.off[v + 1]) ++v;
  const int nx = (views[v].W + tw - 1) / tw;
  const int local = tile - lt.off[v];
  return TileLoc{v, (local % nx) * tw, (local / nx) * th};
}

__global__ __launch_bounds__(256) void k_l1(const ViewDev* __restrict__ views, int V, LossTiles lt,
                                             const float* __restrict__ x, const float* __restrict__ y, float w_l1,
                                             float* __restrict__ grad, double2* __restrict__ partials) {
  __shared__ double sh[4];
  const int tile = xcd_tile(blockIdx.x, lt.off[V]);
  if (tile >= lt.off[V]) return;
  const TileLoc t = loss_tile(views, lt, V, tile, LT, LT);
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

// The SSIM term and both terms' gradient.  A wavefront takes one channel of SW columns
// by `rows` rows and walks down them, a lane per column: each row's four maps go through
// LDS into the horizontal windows and from there into the vertical ones; the row these
// finish gives S and A, B, Cc, which go through the second horizontal and vertical
// windows, and the row those finish is a row of the gradient.  So each image is read once (and a fifth around it), nothing else but
// the gradient touches HBM and no barrier is met.  What it does again: a tile passes
// over rows + 4R rows and 64 columns for its SW.
// Bound by instruction issue (about 185 vector instructions a row, of which 154 the
// windows' multiply-adds) and the 22 16-byte LDS accesses a row beside it.  It replaced
// two kernels over 32x32 tiles with the statistics in HBM between them (36 bytes a pixel
// written and read) and, for gs_loss_noalloc, one over 52x52 patches: 10.1 Mpix in 9
// views 431 -> 290 us (both terms and the final sums), 1600x1067 91 -> 76, 1296x864
// 71 -> 56, three views of 0.2 Mpix in all 45 -> 27.
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(kSsimOccupancy))) void k_ssim(
    const ViewDev* __restrict__ views, int V, LossTiles lt, int rows, const float* __restrict__ x,
    const float* __restrict__ y, Win win, float w_l1, float w_dssim, float* __restrict__ grad,
    double2* __restrict__ partials) {
  static_assert(WAVES == 1 || WAVES == 3, "a channel or all three");
  __shared__ float4 bufs[WAVES][2][64 + TAPS - 1];
  __shared__ double2 sums[3];
  const int part = xcd_tile(blockIdx.x, WAVES == 1 ? 3 * lt.off[V] : lt.off[V]);
  const int tile = WAVES == 1 ? part / 3 : part;
  if (tile >= lt.off[V]) return;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64), ch = WAVES == 1 ? part % 3 : wave;
  float4 (*buf)[64 + TAPS - 1] = bufs[wave];
  const TileLoc t = loss_tile(views, lt, V, tile, SW, rows);
  const ViewDev& cv = views[t.v];
  const int W = cv.W, H = cv.H, lane = __lane_id();
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
  const int y_end = min(t.y0 + rows, H);                     // rows of this tile: [y0, y_end)
  const int n_in = y_end - t.y0 + 4 * R;                     // input rows y0 - 2R ..
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
  double sl1 = 0.0, sss = 0.0;
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
  for (int i = 2 * R; i < n_in; i += TAPS)   // (rows past n_in, in the last tile of a column, are all outside)
#pragma unroll
    for (int u = 0; u < TAPS; ++u) row((2 * R + u) % TAPS, i + u);
  window_rows<3>((2 * R + TAPS - 1) % TAPS, w, h2, acc2, g);
  give(g);
  for (int o = 32; o > 0; o >>= 1) {
    sl1 += __shfl_xor(sl1, o);
    sss += __shfl_xor(sss, o);
  }
  if (WAVES == 1) {
    if (lane == 0) partials[part] = make_double2(sl1, sss);
    return;
  }
  if (lane == 0) sums[ch] = make_double2(sl1, sss);
  __syncthreads();
  if (threadIdx.x == 0)
    partials[tile] = make_double2(sums[0].x + sums[1].x + sums[2].x, sums[0].y + sums[1].y + sums[2].y);
}

// One workgroup per view: the view's tile partials summed in FP64.
__global__ __launch_bounds__(256) void k_loss_final(const ViewDev* __restrict__ views, LossTiles lt,
                                                     const double2* __restrict__ partials, int per_tile,
                                                     float w_l1, float w_dssim, int ssim,
                                                     double* __restrict__ out) {
  __shared__ double sh[4];
  const int v = blockIdx.x;
  const ViewDev& cv = views[v];
  double a = 0.0, b = 0.0;
  for (int t = per_tile * lt.off[v] + threadIdx.x; t < per_tile * lt.off[v + 1]; t += blockDim.x) {
    const double2 pt = partials[t];
    a += pt.x;
    b += pt.y;
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
constexpr int kSsimParts = 65536;   // partial sums that always fit (gs_loss_noalloc's array)
constexpr int kSsimWaves = 1024 * kSsimOccupancy;   // wavefronts the chip holds at once

int64_t ssim_tiles(const ViewDev* hviews, int V, int rows) {
  int64_t t = 0;
  for (int v = 0; v < V; ++v)
    t += (int64_t)((hviews[v].W + SW - 1) / SW) * ((hviews[v].H + rows - 1) / rows);
  return t;
}

// Shape of k_ssim's launch: rows of a tile, tiles, and whether a wavefront (one channel)
// is a workgroup.  A tile of r rows passes over r + 4R, so taller is less work, but all
// its rows one after the other: the shape is the one whose rounds of as many wavefronts
// as fit on the chip, times the rows of a round, are fewest.  1296x864 takes 57 us with
// 34 rows (one round), 64 with 45, 67 with 23; 10.1 Mpix 285 with 89, 331 with 34 or
// 122; 0.2 Mpix 28 with 12, 33 with 23.  Three wavefronts (the channels) share a
// workgroup and one sum only where single sums might not fit.
struct SsimShape {
  int rows, tiles, parts;
  bool waves;
};
SsimShape ssim_shape(const ViewDev* hviews, int V) {
  SsimShape best{};
  double best_cost = 0.0;
  for (int rows = 12; rows <= 133; rows += TAPS) {   // with 2R more, whole runs of TAPS rows
    const int64_t t = ssim_tiles(hviews, V, rows);
    const bool fits = 3 * t <= kSsimParts;
    if (!fits && rows < LT) continue;   // (from LT rows on there are no more tiles than loss_tiles() counts)
    const double rounds = (double)((3 * t + kSsimWaves - 1) / kSsimWaves), cost = (rows + 4 * R) * rounds;
    if (best_cost == 0.0 || cost < best_cost) {
      best = SsimShape{rows, (int)t, (int)(fits ? 3 * t : t), fits};
      best_cost = cost;
    }
  }
  return best;
}
}  // namespace

int loss_partials(const ViewDev* hviews, int V) {
  const int t = loss_tiles(hviews, V), p = ssim_shape(hviews, V).parts;
  return t > p ? t : p;
}

hipError_t launch_loss_dev(const ViewDev* dviews, const ViewDev* hviews, int V, const float* color,
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
  const SsimShape sh = ssim ? ssim_shape(hviews, V) : SsimShape{};
  const int rows = ssim ? sh.rows : LT, cols = ssim ? SW : LT;
  LossTiles lt{};
  int t = 0;
  for (int v = 0; v < V; ++v) {
    lt.off[v] = t;
    t += ((hviews[v].W + cols - 1) / cols) * ((hviews[v].H + rows - 1) / rows);
  }
  lt.off[V] = t;
  double2* part = reinterpret_cast<double2*>(partials);
  const dim3 grid(kXcds * xcd_tile_chunk(ssim ? sh.parts : t));   // at least as many workgroups, see xcd_tile
  if (!ssim)
    hipLaunchKernelGGL(k_l1, grid, dim3(256), 0, s, dviews, V, lt, color, target, w_l1, dL_dcolor, part);
  else if (sh.waves)
    hipLaunchKernelGGL(k_ssim<1>, grid, dim3(64), 0, s, dviews, V, lt, rows, color, target, win, w_l1, w_dssim,
                       dL_dcolor, part);
  else
    hipLaunchKernelGGL(k_ssim<3>, grid, dim3(192), 0, s, dviews, V, lt, rows, color, target, win, w_l1, w_dssim,
                       dL_dcolor, part);
  if (loss_out)
    hipLaunchKernelGGL(k_loss_final, dim3(V), dim3(256), 0, s, dviews, lt, part, ssim && sh.waves ? 3 : 1, w_l1,
                       w_dssim, ssim ? 1 : 0, loss_out);
  return hipGetLastError();
}

}  // namespace gsk
