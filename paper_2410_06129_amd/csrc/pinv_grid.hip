// Adjoint b = E^H d of encodings without an off-resonance map by gridding, in FP64:
// a type-1 non-uniform FFT (spreading with the exponential-of-semicircle kernel of
// Barnett, Magland and af Klinteberg, SIAM J. Sci. Comput. 41, 2019) whose transforms
// are matrix products.
//
// Without the map every factor of E is separable, and per frame, coil and species
//   b(iy, ix) = conj(coil) sum_i d_i conj(ref_i) exp(i 2 pi (kappa_i m_x + eta_i m_y))
// with m = index - n / 2 (integer), kappa, eta the turns from one voxel to the next and
// ref the element's phase at m = 0.  With psi the kernel, 16 cells wide on a grid of
// G = 2 n cells, and t = kappa G,
//   exp(i 2 pi kappa m) = (1 / psihat(m / G)) sum_j psi(j - t) exp(i 2 pi j m / G):
//   spread:    g[jy][jx] = sum_i psi_y psi_x d_i conj(ref_i)
//   x, y DFT:  with 1 / psihat in the matrices
//   combine:   sum over coils of conj(coil) times the transform
// A sample meets 16 x 16 cells (23 x 23 as computed, in 8 x 8 tiles) with real weights
// instead of nx ny voxels with complex ones.  E^H d of 1000 frames of 64 x 64, 8 coils,
// K = 4096: 15.0 ms by the direct sum, 4.3 by gridding; 500 of 96 x 96, 16 coils,
// K = 8192: 67 and 12; 500 of 128 x 128, one coil, K = 32768: 30 and 2.5.  Error against 80-bit sums at 64 x 64,
// K = 4096: 5e-15 of the result's norm, the direct FP64 sum's 2e-15 (rounding in both).
#include <type_traits>

#include "pinv_internal.h"

namespace pinv {

constexpr int kTaps = 16;              // cells a sample spreads over, per axis
constexpr int kGridTile = 8;           // cells per side of a spread tile
constexpr int kSpreadK = 16, kSpreadLd = 68;   // samples per chunk of a spread; LDS row stride
constexpr double kGridBeta = 2.30 * kTaps;
constexpr int kGridMin = 16;           // smallest nx, ny: two windows fit the grid
constexpr size_t kGridBytes = (size_t)512 << 20;   // grids of a pass over frames

struct GridPlan {
  int gx, gy, tx, ty;      // grid cells and tiles
  int64_t entries;         // bound on the tile lists' length
  int seg, extra;          // samples per segment of a list; bound on the segments past the first
  int frames;              // frames per pass
  size_t cell, w, ref, head, segs, idx, tw, dx, dy, tables;   // offsets into the tables; their bytes
  // of a pass: grids, then half-transformed grids, whose place the partial tiles take
  // before them
  size_t grid, work;
};

static GridPlan grid_plan(const EncDev<double>& e, int F, size_t room) {
  GridPlan g{};
  g.gx = 2 * e.nx;
  g.gy = 2 * e.ny;
  g.tx = cdiv(g.gx, kGridTile);
  g.ty = cdiv(g.gy, kGridTile);
  // 16 cells meet 3 tiles of 8 at most, 4 where the last tile is cut
  const int64_t hx = g.gx % kGridTile ? 4 : 3, hy = g.gy % kGridTile ? 4 : 3;
  g.entries = std::min<int64_t>(hx * hy, (int64_t)g.tx * g.ty) * e.K;
  // no more extra segments than tiles
  g.seg = (int)std::max<int64_t>(256, cdiv(cdiv(g.entries, (int64_t)g.tx * g.ty), kSpreadK) * kSpreadK);
  g.extra = (int)(g.entries / g.seg);
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o += (bytes + 255) & ~size_t(255);
    return at;
  };
  g.cell = take(8 * (size_t)e.K);
  g.w = take(16 * kTaps * (size_t)e.K);
  g.ref = take(16 * (size_t)e.K * e.S);
  g.head = take(8 * (size_t)g.tx * g.ty + 8);
  g.segs = take(16 * ((size_t)g.tx * g.ty + g.extra));
  g.idx = take(4 * (size_t)g.entries);
  g.tw = take(16 * kGridTile * (size_t)g.entries);
  g.dx = take(16 * (size_t)g.gx * e.nx);
  g.dy = take(16 * (size_t)g.gy * e.ny);
  g.tables = o;
  const size_t half = 16 * std::max<size_t>((size_t)g.gy * e.nx, kGridTile * kGridTile * (size_t)g.extra);
  const size_t row = 16 * (size_t)g.gy * g.gx + half, rows = (size_t)e.C * e.S;
  int q = 64;   // whole 64-row tiles per pass
  while (q > 1 && (rows * (q / 2)) % 64 == 0) q /= 2;
  // as many frames as a pass may take; none where the scratch left holds neither all of
  // them nor a quarter of a pass (many short passes take longer than the direct sum)
  const size_t left = room > g.tables + 512 ? room - g.tables - 512 : 0, fit = std::min(kGridBytes, left);
  int f = (int)std::min<size_t>((size_t)F, fit / (row * rows));
  if (f < F && fit < kGridBytes / 4) f = 0;
  if (f == 0) return g;
  if (f < F) {
    if (f >= q) f = f / q * q;
    const int passes = cdiv(F, f);
    f = std::min(f, cdiv(cdiv(F, passes), q) * q);
  }
  g.frames = f;
  g.grid = 16 * (size_t)g.gy * g.gx * rows * f;
  g.work = row * rows * f;
  return g;
}

// Turns from one voxel to the next along an axis of n voxels, from the axis's phase
// factors p[0 .. n) = exp(-i 2 pi kappa (index - n / 2)): the neighbours' ratio, made
// sharp by the ends' (n - 1 steps apart, known up to whole turns).
__device__ __forceinline__ double grid_kappa(const cx<double>* p, int n) {
  auto turns = [](const cx<double>& a, const cx<double>& b) {   // -arg(a conj(b)) / 2 pi
    return -atan2(a.im * b.re - a.re * b.im, a.re * b.re + a.im * b.im) * 0.15915494309189535;
  };
  const double coarse = turns(p[1], p[0]), fine = turns(p[n - 1], p[0]);
  return (rint(coarse * (n - 1) - fine) + fine) / (n - 1);
}

// First cells and weights of every sample's windows and its conj(ref) per species, and
// an empty list counter.  Non-finite positions get cell 0 and NaN weights.
__global__ __launch_bounds__(256) void k_grid_prep(EncDev<double> e, int gx, int gy, int2* __restrict__ cell,
                                                   double* __restrict__ w, cx<double>* __restrict__ ref,
                                                   int* __restrict__ total, int4* __restrict__ segs,
                                                   int extra) {
  const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (u < 2) total[u] = 0;
  if (u < extra) segs[u] = int4{0, 0, 0, -2};   // not in use
  const int i = (int)(u / 32), a = (int)(u % 32) % kTaps;
  const bool y = u % 32 >= kTaps;
  if (i >= e.K) return;
  const cx<double>* px = reinterpret_cast<const cx<double>*>(e.px) + (size_t)i * e.nx;
  const cx<double>* py = reinterpret_cast<const cx<double>*>(e.py) + (size_t)i * e.ny;
  const int n = y ? e.ny : e.nx, G = y ? gy : gx;
  double t = grid_kappa(y ? py : px, n) * G;
  t -= G * floor(t / G);
  const double c = ceil(t - kTaps / 2), z = (c + a - t) / (kTaps / 2);
  const bool fin = t >= 0.0 && t <= G;   // false for NaN
  w[(size_t)i * 32 + u % 32] = fin ? exp(kGridBeta * (sqrt(fmax(0.0, 1.0 - z * z)) - 1.0)) : __builtin_nan("");
  if (a == 0) {
    int ci = fin ? (int)c : 0;
    if (ci < 0) ci += G;
    (y ? cell[i].y : cell[i].x) = ci;
  }
  for (int s = (int)(u % 32); s < e.S; s += 32) {
    cx<double> r = cmul(px[e.nx / 2], py[e.ny / 2]);
    if (e.q) r = cmul(r, reinterpret_cast<const cx<double>*>(e.q)[(size_t)i * e.S + s]);
    ref[(size_t)i * e.S + s] = cx<double>{r.re, -r.im};
  }
}

// The transforms' matrices: Dx[jx][ix] and Dy[iy][jy] = exp(i 2 pi j m / G) / psihat(m / G).
// psihat by the trapezoid rule over u = 8 sin(theta), 64 intervals of [0, pi / 2]: the
// integrand falls to exp(-37) at the end, so the rule converges to rounding.
__global__ __launch_bounds__(64) void k_grid_dft(int nx, int ny, int gx, int gy, cx<double>* __restrict__ Dx,
                                                 cx<double>* __restrict__ Dy) {
  const bool y = (int)blockIdx.x >= nx;
  const int n = y ? ny : nx, G = y ? gy : gx, i = (int)blockIdx.x - (y ? nx : 0), m = i - n / 2;
  const int lane = threadIdx.x;
  double sn, cs;
  sincospi(lane / 128.0, &sn, &cs);
  double v = exp(kGridBeta * (cs - 1.0)) * cs * cospi(kTaps * (double)m / G * sn);
  if (lane == 0) v *= 0.5;
  for (int o = 32; o; o >>= 1) v += __shfl_xor(v, o);
  const double scale = 1.0 / (kTaps * (3.14159265358979323846 / 128.0) * v);
  for (int j = lane; j < G; j += 64) {
    int jm = (int)((int64_t)j * m % G);
    sincospi(2.0 * jm / G, &sn, &cs);
    (y ? Dy[(size_t)i * G + j] : Dx[(size_t)j * n + i]) = cx<double>{cs * scale, sn * scale};
  }
}

// One tile's samples in ascending order, one workgroup per tile: idx the samples, tw
// the weights of the tile's 8 rows and 8 columns (zero outside the window).  A list is
// worked on in segments of `seg` samples, segs[] = (tile, first entry, entries, slot of
// the partial tile): the tile's own at segs[extra + tile] (slot -1), further ones from
// segs[head[tile].x] on, head[tile].y of them.  Where entries and segments lie depends on
// the order in which workgroups ask for room, what they hold does not.  Each wave
// takes a share of the samples and counts them first.
constexpr int kListWaves = 16;
__global__ __launch_bounds__(64 * kListWaves) void k_grid_lists(
    int K, int gx, int gy, int tx, int seg, int extra, const int2* __restrict__ cell,
    const double* __restrict__ w, int* __restrict__ total, int2* __restrict__ head,
    int4* __restrict__ segs, int* __restrict__ idx, double* __restrict__ tw) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int x0 = (int)(blockIdx.x % tx) * kGridTile, y0 = (int)(blockIdx.x / tx) * kGridTile;
  __shared__ int cnt[kListWaves], base;
  // distance of a tile's start past a window's, modulo the grid
  auto past = [](int t0, int c, int G) { const int d = t0 - c; return d < 0 ? d + G : d; };
  auto meets = [](int d, int G, int t0) { return d < kTaps || G - d < min(kGridTile, G - t0); };
  auto hit = [&](int i) {
    if (i >= K) return false;
    const int2 c = cell[i];
    return meets(past(x0, c.x, gx), gx, x0) && meets(past(y0, c.y, gy), gy, y0);
  };
  const int per = (K + kListWaves - 1) / kListWaves, i0 = wv * per, i1 = min(K, i0 + per);
  int n = 0;
#pragma unroll 4
  for (int i = i0; i < i1; i += 64) n += __popcll(__ballot(i + lane < i1 && hit(i + lane)));
  if (lane == 0) cnt[wv] = n;
  __syncthreads();
  int all = 0, at = 0;
  for (int v = 0; v < kListWaves; ++v) {
    if (v == wv) at = all;
    all += cnt[v];
  }
  if (threadIdx.x == 0) {
    base = atomicAdd(total, all);
    const int more = all > 0 ? (all - 1) / seg : 0, slot = more ? atomicAdd(total + 1, more) : 0;
    head[blockIdx.x] = int2{slot, more};
    segs[extra + blockIdx.x] = int4{(int)blockIdx.x, base, min(all, seg), -1};
    for (int q = 0; q < more; ++q)
      segs[slot + q] = int4{(int)blockIdx.x, base + (q + 1) * seg, min(seg, all - (q + 1) * seg), slot + q};
  }
  __syncthreads();
  at += base;
#pragma unroll 4
  for (int i = i0; i < i1; i += 64) {
    const bool h = i + lane < i1 && hit(i + lane);
    const uint64_t m = __ballot(h);
    if (h) idx[at + __popcll(m & ((1ull << lane) - 1))] = i + lane;
    at += __popcll(m);
  }
  __syncthreads();   // idx is visible to the workgroup
  const int first = base;
  for (int u = threadIdx.x; u < all * 16; u += 64 * kListWaves) {
    const int en = first + u / 16, a = u % kGridTile, i = idx[en];
    const bool x = u % 16 >= kGridTile;
    const int G = x ? gx : gy, t0 = x ? x0 : y0;
    const int2 c = cell[i];
    int d = past(t0, x ? c.x : c.y, G) + a;
    if (d >= G) d -= G;
    tw[(size_t)en * 16 + u % 16] = d < kTaps && t0 + a < G ? w[(size_t)i * 32 + (x ? 0 : kTaps) + d] : 0.0;
  }
}

// The spread as a matrix product per tile: rows (frame, coil, species), a contraction
// over the tile's samples, 64 cells as columns; the weight of (sample, cell) is real
// and formed on the way to LDS, the data are read in place and multiplied by
// conj(ref).  Bound by the FP64 matrix cores: 2 x 529 multiply-adds per row and sample.
// Segments past a list's first (where samples are dense) come first and go to partial
// tiles, added by k_grid_join: with whole lists the launch waited for the few
// tiles around k = 0 (a variable-density spiral of 128 x 128, K = 32768: 1303 us for
// 128 rows, 311 in segments; 64 x 64, K = 4096, 640 rows: 299 and 167, the matrix cores
// half busy).
template <bool SPECIES>
__global__ __launch_bounds__(256) void k_grid_spread(const float* __restrict__ D, int K, int S, int rows,
                                                     int gx, int gy, int tx, int nseg,
                                                     const cx<double>* __restrict__ ref,
                                                     const int4* __restrict__ segs,
                                                     const int* __restrict__ idx,
                                                     const double* __restrict__ tw,
                                                     cx<double>* __restrict__ g,
                                                     cx<double>* __restrict__ part) {
  __shared__ double sm[2][3][kSpreadK * kSpreadLd];
  const int t = xcd_contiguous(blockIdx.x, gridDim.x);
  const int r0 = t / nseg * 64;
  const int4 sg = segs[t % nseg];
  if (sg.w == -2) return;
  const int2 hd{sg.y, sg.z};
  const int cx0 = sg.x % tx, cy0 = sg.x / tx;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lk = lane >> 4, wr = wv / 2, wc = wv % 2;
  const cx<float>* Dc = reinterpret_cast<const cx<float>*>(D);
  // of a chunk this thread stages sample ks for P rows, and cell `lane` for P samples
  constexpr int P = kSpreadK / 4, RP = 256 / kSpreadK;
  const int ks = tid % kSpreadK;
  cx<float> d[P];
  cx<double> rf[P];
  double wy[P], wx[P];
  bool in;
  auto fetch = [&](int k0, int i) {
    in = k0 + ks < hd.y;
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const int row = min(r0 + tid / kSpreadK + RP * j, rows - 1);
      const int fc = SPECIES ? row / S : row;
      d[j] = Dc[(size_t)fc * K + i];
      if (SPECIES || j == 0) rf[j] = ref[SPECIES ? (size_t)i * S + (row - fc * S) : (size_t)i];
      const int en = hd.x + min(k0 + wv + 4 * j, hd.y - 1);
      wy[j] = tw[(size_t)en * 16 + lane / kGridTile];
      wx[j] = tw[(size_t)en * 16 + kGridTile + lane % kGridTile];
    }
  };
  auto store = [&](int k0, double (&s)[3][kSpreadK * kSpreadLd]) {
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const cx<double> z = cmul(cx<double>{d[j].re, d[j].im}, rf[SPECIES ? j : 0]);
      const int o = ks * kSpreadLd + tid / kSpreadK + RP * j;
      s[0][o] = in ? z.re : 0.0;
      s[1][o] = in ? z.im : 0.0;
      s[2][(wv + 4 * j) * kSpreadLd + lane] = k0 + wv + 4 * j < hd.y ? wy[j] * wx[j] : 0.0;
    }
  };
  auto sample = [&](int k0) { return idx[hd.x + min(k0 + ks, hd.y - 1)]; };
  f64x4 re[2][2], im[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) re[a][b] = im[a][b] = f64x4{0, 0, 0, 0};
  if (hd.y > 0) {
    fetch(0, sample(0));
    int next = sample(kSpreadK);
    store(0, sm[0]);
    __syncthreads();
    for (int k0 = 0, c = 0; k0 < hd.y; k0 += kSpreadK, c ^= 1) {
      const bool more = k0 + kSpreadK < hd.y;
      if (more) {
        fetch(k0 + kSpreadK, next);
        next = sample(k0 + 2 * kSpreadK);
      }
      const auto& s = sm[c];
#pragma unroll
      for (int kk = 0; kk < kSpreadK / 4; ++kk) {
        double ar[2], ai[2], b[2];
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          const int o = (kk * 4 + lk) * kSpreadLd + a * 16 + lr;
          ar[a] = s[0][o + wr * 32];
          ai[a] = s[1][o + wr * 32];
          b[a] = s[2][o + wc * 32];
        }
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            re[a][q] = mfma4(ar[a], b[q], re[a][q]);
            im[a][q] = mfma4(ai[a], b[q], im[a][q]);
          }
      }
      if (more) store(k0 + kSpreadK, sm[c ^ 1]);
      __syncthreads();
    }
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = r0 + wr * 32 + a * 16 + lk + 4 * r, o = wc * 32 + q * 16 + lr;
        const int y = cy0 * kGridTile + o / kGridTile, x = cx0 * kGridTile + o % kGridTile;
        const cx<double> z{re[a][q][r], im[a][q][r]};
        if (row >= rows) continue;
        if (sg.w >= 0) part[((size_t)sg.w * rows + row) * 64 + o] = z;
        else if (y < gy && x < gx) g[((size_t)row * gy + y) * gx + x] = z;
      }
}

// The partial tiles of a tile's further segments added to the grid, in order.  One
// workgroup per tile and kJoinRows rows.
constexpr int kJoinRows = 8;
__global__ __launch_bounds__(256) void k_grid_join(int rows, int gx, int gy, int tx,
                                                   const int2* __restrict__ head,
                                                   const cx<double>* __restrict__ part,
                                                   cx<double>* __restrict__ g) {
  const int2 h = head[blockIdx.x];
  if (h.y == 0) return;
  const int o = threadIdx.x % 64;
  const int x = (int)(blockIdx.x % tx) * kGridTile + o % kGridTile;
  const int y = (int)(blockIdx.x / tx) * kGridTile + o / kGridTile;
  if (x >= gx || y >= gy) return;
  const int r1 = min(rows, (int)(blockIdx.y + 1) * kJoinRows);
  for (int row = (int)blockIdx.y * kJoinRows + (int)(threadIdx.x / 64); row < r1; row += 4) {
    cx<double>* p = g + ((size_t)row * gy + y) * gx + x;
    cx<double> z = *p;
#pragma unroll 8
    for (int q = 0; q < h.y; ++q) {
      const cx<double> v = part[((size_t)(h.x + q) * rows + row) * 64 + o];
      z.re += v.re;
      z.im += v.im;
    }
    *p = z;
  }
}

// C[m][n] = sum_k A[m][k] B[k][n], one product per blockIdx.y (B and C advance by sb, sc).
template <class Cfg>
__global__ __launch_bounds__(256, MinBlocks<Cfg>::value) void k_grid_product(
    const cx<double>* __restrict__ A, const cx<double>* __restrict__ B, cx<double>* __restrict__ C, int m,
    int n, int k, size_t sb, size_t sc) {
  const int nbj = (n + Cfg::BN - 1) / Cfg::BN;
  const int bi = blockIdx.x / nbj, bj = blockIdx.x % nbj;
  LoadDenseKC<Cfg, Cfg::BM, Cfg::LDA, double, false> la;
  la.p = A;
  la.ld = k;
  la.o0 = bi * Cfg::BM;
  la.oend = m;
  LoadDenseOC<Cfg, Cfg::BN, Cfg::LDB, double, false> lb;
  lb.p = B + blockIdx.y * sb;
  lb.ld = n;
  lb.o0 = bj * Cfg::BN;
  lb.oend = n;
  AccTile<Cfg> acc;
  acc.zero();
  mainloop<Cfg>(la, lb, 0, k, acc, smem_base<Cfg>());
  cx<double>* O = C + blockIdx.y * sc;
  acc_foreach<Cfg>(acc, [&](int r, int c, double re, double im) {
    const int row = bi * Cfg::BM + r, col = bj * Cfg::BN + c;
    if (row < m && col < n) O[(size_t)row * n + col] = cx<double>{re, im};
  });
}

// b[f][s V + v] = sum_c conj(coil[c][v]) T[(f C + c) S + s][voxel v].
__global__ __launch_bounds__(256) void k_grid_combine(EncDev<double> e, const cx<double>* __restrict__ T,
                                                      int F, cx<double>* __restrict__ b) {
  const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= (int64_t)F * e.N) return;
  const int f = (int)(u / e.N), n = (int)(u - (int64_t)f * e.N), s = n / e.V, v = n - s * e.V;
  int ix, iy;
  voxel_xy(e, v, &ix, &iy);
  const cx<double>* coil = reinterpret_cast<const cx<double>*>(e.coil);
  const size_t img = (size_t)e.nx * e.ny;
  cx<double> z{0.0, 0.0};
  for (int c = 0; c < e.C; ++c) {
    const cx<double> t = T[(((size_t)f * e.C + c) * e.S + s) * img + (size_t)iy * e.nx + ix];
    if (coil) {
      const cx<double> a = coil[(size_t)c * e.V + v];
      z.re += t.re * a.re + t.im * a.im;
      z.im += t.im * a.re - t.re * a.im;
    } else {
      z = t;
    }
  }
  b[u] = z;
}

// Gridding does fewer multiply-adds than a sum over all voxels, but its contractions
// run at half the matrix cores' rate where a product with a stored F^H reaches 0.73.
// A refinement step by the direct sum, stored F^H and gridding (ratio of multiply-adds):
// 24 x 24, 8 coils, 200 frames 905, 546, 588 us (1.46); 28 x 28 1001, 737, 708 (1.87);
// 48 x 48, 4 coils, 100 frames 2018, 1543, 1249 (4.4); 64 x 64, 8 coils, 1 frame 4354,
// 2590, 1928 (7.5); level at one frame of 32 x 32, one coil (6e6 multiply-adds).
bool grid_adjoint(const EncDev<double>& e, int F) {
  if (e.b0 || e.nx < kGridMin || e.ny < kGridMin || F <= 0) return false;
  const double rows = (double)F * e.C * e.S, img = (double)e.nx * e.ny;
  // tables and a pass over a frame's grids at least fit 256 MB, what a call that fits the
  // fixed region of applies without allocation leaves (and a frame's rows a launch's y
  // dimension)
  const GridPlan one = grid_plan(e, 1, SIZE_MAX);
  if (one.frames == 0 || one.tables > kGridBytes / 4 - 1024 || one.work > kGridBytes / 4) return false;
  const double direct = 3.0 * rows * e.K * e.V;
  const double grid = rows * (2.0 * 529.0 * e.K + 3.0 * img * (4.0 * e.nx + 2.0 * e.ny));
  return direct >= 1.75 * grid && direct >= 1e7;
}

hipError_t launch_grid_adjoint(const EncDev<double>& e, const float* D, int F, double* b, Scratch& sc,
                               hipStream_t s) {
  const GridPlan g = grid_plan(e, F, sc.room());
  if (g.frames == 0) return hipErrorOutOfMemory;
  void *tab = nullptr, *work = nullptr;
  hipError_t err = sc.get(&tab, g.tables, s);
  if (err != hipSuccess) return err;
  if ((err = sc.get(&work, g.work, s)) != hipSuccess) {
    (void)sc.put(tab, s);
    return err;
  }
  char* T = (char*)tab;
  int2* cell = (int2*)(T + g.cell);
  double *w = (double*)(T + g.w), *tw = (double*)(T + g.tw);
  cx<double>*ref = (cx<double>*)(T + g.ref), *Dx = (cx<double>*)(T + g.dx), *Dy = (cx<double>*)(T + g.dy);
  int* total = (int*)(T + g.head);   // entries and further segments handed out
  int2* head = (int2*)(T + g.head) + 1;
  int4* segs = (int4*)(T + g.segs);
  int* idx = (int*)(T + g.idx);
  cx<double>*grid = (cx<double>*)work, *half = (cx<double>*)((char*)work + g.grid);
  const int tiles = g.tx * g.ty, nseg = tiles + g.extra;
  const int64_t prep = std::max<int64_t>((int64_t)e.K * 32, g.extra);
  hipLaunchKernelGGL(k_grid_prep, dim3((unsigned)((prep + 255) / 256)), dim3(256), 0, s, e, g.gx, g.gy, cell,
                     w, ref, total, segs, g.extra);
  hipLaunchKernelGGL(k_grid_dft, dim3(e.nx + e.ny), dim3(64), 0, s, e.nx, e.ny, g.gx, g.gy, Dx, Dy);
  hipLaunchKernelGGL(k_grid_lists, dim3(tiles), dim3(64 * kListWaves), 0, s, e.K, g.gx, g.gy, g.tx, g.seg,
                     g.extra, (const int2*)cell, (const double*)w, total, head, segs, idx, tw);
  typedef F64Cfg3 Cfg;
  const size_t img = (size_t)e.nx * e.ny;
  for (int f0 = 0; f0 < F; f0 += g.frames) {
    const int f = std::min(g.frames, F - f0), rows = f * e.C * e.S;
    const float* d = D + 2 * (size_t)f0 * e.M;
    auto spread = [&](auto kern) {
      hipLaunchKernelGGL(kern, dim3((unsigned)(cdiv(rows, 64) * nseg)), dim3(256), 0, s, d, e.K, e.S, rows,
                         g.gx, g.gy, g.tx, nseg, (const cx<double>*)ref, (const int4*)segs, (const int*)idx,
                         (const double*)tw, grid, half);
    };
    e.S > 1 ? spread(k_grid_spread<true>) : spread(k_grid_spread<false>);
    hipLaunchKernelGGL(k_grid_join, dim3(tiles, cdiv(rows, kJoinRows)), dim3(256), 0, s, rows, g.gx, g.gy, g.tx,
                       (const int2*)head, (const cx<double>*)half, grid);
    hipLaunchKernelGGL(k_grid_product<Cfg>, dim3((unsigned)(cdiv((int64_t)rows * g.gy, 64) * cdiv(e.nx, 64))),
                       dim3(256), smem_bytes<Cfg>(), s, (const cx<double>*)grid, (const cx<double>*)Dx, half,
                       rows * g.gy, e.nx, g.gx, (size_t)0, (size_t)0);
    // the images in the grids' place
    hipLaunchKernelGGL(k_grid_product<Cfg>, dim3((unsigned)(cdiv(e.ny, 64) * cdiv(e.nx, 64)), (unsigned)rows),
                       dim3(256), smem_bytes<Cfg>(), s, (const cx<double>*)Dy, (const cx<double>*)half, grid,
                       e.ny, e.nx, g.gy, (size_t)g.gy * e.nx, img);
    hipLaunchKernelGGL(k_grid_combine, dim3((unsigned)(((int64_t)f * e.N + 255) / 256)), dim3(256), 0, s, e,
                       (const cx<double>*)grid, f, (cx<double>*)b + (size_t)f0 * e.N);
    if ((err = hipGetLastError()) != hipSuccess) break;
  }
  const hipError_t e1 = sc.put(work, s), e2 = sc.put(tab, s);
  return err != hipSuccess ? err : e1 != hipSuccess ? e1 : e2;
}

}  // namespace pinv
