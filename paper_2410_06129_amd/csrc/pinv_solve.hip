// Forward model D = E X (Eq. 1), adjoint Z = E^H D, the normal-equation
// residual through the Gram (Eq. 6), triangular products on frame blocks
// (refinement correction and factor-only solves) and precision conversions.
#include <type_traits>

#include "pinv_internal.h"

namespace pinv {

// ---------------------------------------------------------------------------
// Forward model D[f][m] = sum_n X[f][n] E[m][n]  (S = storage type of X).
// With `sub` set the result is Dout = Din - E x (refinement residual).
// ---------------------------------------------------------------------------
template <class Cfg, int FEAT, typename SX, typename SD, bool AL>
__global__ __launch_bounds__(256, 2) void k_forward(EncDev<typename Cfg::T> e, const SX* __restrict__ X,
                                                 int F, const SD* __restrict__ Din,
                                                 typename Cfg::T* __restrict__ Dout) {
  typedef typename Cfg::T T;
  const int N = e.N, M = e.M;
  const int nbj = (M + Cfg::BN - 1) / Cfg::BN;
  const int t = blockIdx.x;
  const int bi = t / nbj, bj = t % nbj;
  LoadDenseKC<Cfg, Cfg::BM, Cfg::LDA, SX, false> la;
  la.p = reinterpret_cast<const cx<SX>*>(X);
  la.ld = N;
  la.o0 = bi * Cfg::BM;
  la.oend = F;
  LoadGenRow<Cfg, Cfg::BN, Cfg::LDB, false, FEAT, AL> lb;
  lb.init(e, bj * Cfg::BN);
  AccTile<Cfg> acc;
  acc.zero();
  mainloop<Cfg>(la, lb, 0, N, acc, smem_base<Cfg>());
  cx<T>* O = reinterpret_cast<cx<T>*>(Dout);
  const cx<SD>* Di = reinterpret_cast<const cx<SD>*>(Din);
  const int r0 = bi * Cfg::BM, c0 = bj * Cfg::BN;
  acc_foreach<Cfg>(acc, [&](int r, int c, T re, T im) {
    const int row = r0 + r, col = c0 + c;
    if (row < F && col < M) {
      const size_t o = (size_t)row * M + col;
      if (Di) {
        cx<SD> d = Di[o];
        O[o] = cx<T>{T(d.re) - re, T(d.im) - im};
      } else {
        O[o] = cx<T>{re, im};
      }
    }
  });
}

// Adjoint Z[f][n] = sum_m D[f][m] conj(E[m][n]);  with X given, Z -= lam * X.
// The result is written with storage type SO.
// With a split of the contraction (ksplit > 1, `work` non-null) workgroup
// blockIdx = split * tiles + tile sums rows m in [split*kchunk, +kchunk) and
// stores its raw partial tile to work[split]; k_split_reduce then adds the
// partials in split order (deterministic) and applies the -lam x term.
template <class Cfg, int FEAT, typename SD, typename SX, typename SO, bool AL>
__global__ __launch_bounds__(256, (MinBlocks<Cfg, FEAT>::value)) void k_adjoint(EncDev<typename Cfg::T> e, const SD* __restrict__ D,
                                                 int F, const SX* __restrict__ X, double lam,
                                                 SO* __restrict__ Z, int tiles, int kchunk,
                                                 typename Cfg::T* __restrict__ work) {
  typedef typename Cfg::T T;
  const int N = e.N, M = e.M;
  const int nbj = (N + Cfg::BN - 1) / Cfg::BN;
  const int split = blockIdx.x / tiles;
  const int t = blockIdx.x - split * tiles;
  const int bi = t / nbj, bj = t % nbj;
  const int k0 = split * kchunk, k1 = min(M, k0 + kchunk);
  LoadDenseKC<Cfg, Cfg::BM, Cfg::LDA, SD, false> la;
  la.p = reinterpret_cast<const cx<SD>*>(D);
  la.ld = M;
  la.o0 = bi * Cfg::BM;
  la.oend = F;
  LoadGenCol<Cfg, Cfg::BN, Cfg::LDB, true, FEAT, AL> lb;
  lb.init(e, bj * Cfg::BN);
  AccTile<Cfg> acc;
  acc.zero();
  mainloop<Cfg>(la, lb, k0, k1, acc, smem_base<Cfg>());
  const int r0 = bi * Cfg::BM, c0 = bj * Cfg::BN;
  if (work) {
    cx<T>* W = reinterpret_cast<cx<T>*>(work) + (size_t)split * F * N;
    acc_foreach<Cfg>(acc, [&](int r, int c, T re, T im) {
      const int row = r0 + r, col = c0 + c;
      if (row < F && col < N) W[(size_t)row * N + col] = cx<T>{re, im};
    });
    return;
  }
  cx<SO>* O = reinterpret_cast<cx<SO>*>(Z);
  const cx<SX>* Xc = reinterpret_cast<const cx<SX>*>(X);
  acc_foreach<Cfg>(acc, [&](int r, int c, T re, T im) {
    const int row = r0 + r, col = c0 + c;
    if (row < F && col < N) {
      const size_t o = (size_t)row * N + col;
      T zr = re, zi = im;
      if (Xc) {
        cx<SX> x = Xc[o];
        zr -= T(lam) * T(x.re);
        zi -= T(lam) * T(x.im);
      }
      O[o] = cx<SO>{SO(zr), SO(zi)};
    }
  });
}

// Apply for a few frames: X[f][n] = sum_m D[f][m] R[n][m], each wavefront

// Triangular products on frame blocks (refinement correction, factor-only solves):
//   mode 0: Y[f][i] = sum_{n <= i} Xin[f][n] Li[i][n]          (L^-1 x, per frame)
//   mode 1: X[f][i] += sum_{n >= i} Yin[f][n] conj(Li[n][i])   (L^-H y, accumulated)
//   mode 2: X[f][i] = sum_{n >= i} Yin[f][n] conj(Li[n][i])    (L^-H y)
// (S = storage type of L^-1 and of the frames.)
// With `work`, workgroup split * tiles + tile takes one of `splits` equal parts of its
// tile's contraction and stores the raw sum to work[split] (k_parts_sum adds them).
template <class Cfg, int MODE, typename SO, typename S>
__global__ __launch_bounds__(256) void k_tri_frames(const S* __restrict__ Li, const S* __restrict__ In, int F,
                                                    int N, SO* __restrict__ Out, int splits,
                                                    typename Cfg::T* __restrict__ work) {
  typedef typename Cfg::T T;
  const int nbj = (N + Cfg::BN - 1) / Cfg::BN;
  const int nbi = (F + Cfg::BM - 1) / Cfg::BM;
  // A tile's contraction length grows with its distance from the triangle's
  // short end.  Rank r = 0 is the longest tile; the grid's first half takes
  // ranks in descending length and its second half in ascending length, so
  // workgroups t and t + half, which the dispatcher tends to place on one CU,
  // carry one long and one short tile.
  const int total = nbi * nbj, half = (total + 1) / 2;
  const int split = (int)blockIdx.x / total, t = (int)blockIdx.x - split * total;
  const int r = t < half ? t : total - 1 + half - t;
  const int jr = r / nbi;                       // 0 = longest block column
  const int bi = r - jr * nbi;
  const int bj = MODE == 0 ? nbj - 1 - jr : jr;
  LoadDenseKC<Cfg, Cfg::BM, Cfg::LDA, S, false> la;
  la.p = reinterpret_cast<const cx<S>*>(In);
  la.ld = N;
  la.o0 = bi * Cfg::BM;
  la.oend = F;
  AccTile<Cfg> acc;
  acc.zero();
  int k0 = MODE == 0 ? 0 : bj * Cfg::BN, k1 = MODE == 0 ? min(N, (bj + 1) * Cfg::BN) : N;
  const int part = ((k1 - k0 + Cfg::BK - 1) / Cfg::BK + splits - 1) / splits * Cfg::BK;
  k0 = min(k1, k0 + split * part);
  k1 = min(k1, k0 + part);
  if (MODE == 0) {
    LoadDenseKC<Cfg, Cfg::BN, Cfg::LDB, S, false> lb;   // (o=i, k=n) at Li[i*N+n]
    lb.p = reinterpret_cast<const cx<S>*>(Li);
    lb.ld = N;
    lb.o0 = bj * Cfg::BN;
    lb.oend = N;
    mainloop<Cfg>(la, lb, k0, k1, acc, smem_base<Cfg>());
  } else {
    LoadDenseOC<Cfg, Cfg::BN, Cfg::LDB, S, true> lb;    // (o=i, k=n) at conj Li[n*N+i]
    lb.p = reinterpret_cast<const cx<S>*>(Li);
    lb.ld = N;
    lb.o0 = bj * Cfg::BN;
    lb.oend = N;
    mainloop<Cfg>(la, lb, k0, k1, acc, smem_base<Cfg>());
  }
  cx<SO>* O = reinterpret_cast<cx<SO>*>(Out);
  const int r0 = bi * Cfg::BM, c0 = bj * Cfg::BN;
  if (work) {
    cx<T>* W = reinterpret_cast<cx<T>*>(work) + (size_t)split * F * N;
    acc_foreach<Cfg>(acc, [&](int r, int c, T re, T im) {
      if (r0 + r < F && c0 + c < N) W[(size_t)(r0 + r) * N + c0 + c] = cx<T>{re, im};
    });
    return;
  }
  acc_foreach<Cfg>(acc, [&](int r, int c, T re, T im) {
    const int row = r0 + r, col = c0 + c;
    if (row < F && col < N) {
      const size_t o = (size_t)row * N + col;
      if (MODE != 1) {
        O[o] = cx<SO>{SO(re), SO(im)};
      } else {
        cx<SO> x = O[o];
        O[o] = cx<SO>{SO(x.re + re), SO(x.im + im)};
      }
    }
  });
}

// Normal-equation residual through the Gram (Eq. 6):
//   Out[f][a] = b[f][a] - sum_n G[a][n] X[f][n] - lam X[f][a]
// with G the full Hermitian FP64 Gram [N][N] and b = E^H d in FP64.  With `work` the
// contraction is in `splits` parts, as in k_tri_frames.
template <class Cfg, typename SX, typename SO>
__global__ __launch_bounds__(256, MinBlocks<Cfg>::value) void k_resid(const double* __restrict__ G,
                                               const double* __restrict__ b,
                                               const SX* __restrict__ X, int F, int N, double lam,
                                               SO* __restrict__ Out, int splits,
                                               double* __restrict__ work) {
  typedef typename Cfg::T T;
  const int nbj = (N + Cfg::BN - 1) / Cfg::BN;
  const int tiles = (F + Cfg::BM - 1) / Cfg::BM * nbj;
  const int split = blockIdx.x / tiles, t = blockIdx.x - split * tiles;
  const int part = ((N + Cfg::BK - 1) / Cfg::BK + splits - 1) / splits * Cfg::BK;
  const int k0 = min(N, split * part), k1 = min(N, k0 + part);
  const int bi = t / nbj, bj = t % nbj;
  LoadDenseKC<Cfg, Cfg::BM, Cfg::LDA, SX, false> la;     // X[f][n]
  la.p = reinterpret_cast<const cx<SX>*>(X);
  la.ld = N;
  la.o0 = bi * Cfg::BM;
  la.oend = F;
  LoadDenseKC<Cfg, Cfg::BN, Cfg::LDB, double, false> lb;  // (o=a, k=n) at G[a][n]
  lb.p = reinterpret_cast<const cx<double>*>(G);
  lb.ld = N;
  lb.o0 = bj * Cfg::BN;
  lb.oend = N;
  AccTile<Cfg> acc;
  acc.zero();
  mainloop<Cfg>(la, lb, k0, k1, acc, smem_base<Cfg>());
  if (work) {
    cx<double>* W = reinterpret_cast<cx<double>*>(work) + (size_t)split * F * N;
    const int r0 = bi * Cfg::BM, c0 = bj * Cfg::BN;
    acc_foreach<Cfg>(acc, [&](int r, int c, T re, T im) {
      if (r0 + r < F && c0 + c < N) W[(size_t)(r0 + r) * N + c0 + c] = cx<double>{re, im};
    });
    return;
  }
  cx<SO>* O = reinterpret_cast<cx<SO>*>(Out);
  const cx<double>* bc = reinterpret_cast<const cx<double>*>(b);
  const cx<SX>* Xc = reinterpret_cast<const cx<SX>*>(X);
  const int r0 = bi * Cfg::BM, c0 = bj * Cfg::BN;
  acc_foreach<Cfg>(acc, [&](int r, int c, T re, T im) {
    const int row = r0 + r, col = c0 + c;
    if (row < F && col < N) {
      const size_t o = (size_t)row * N + col;
      const cx<double> bb = bc[o];
      const cx<SX> x = Xc[o];
      O[o] = cx<SO>{SO(bb.re - (double)re - lam * (double)x.re),
                    SO(bb.im - (double)im - lam * (double)x.im)};
    }
  });
}


// A split contraction's parts summed in order, n values each: mode 0 or 2 Out = sum,
// mode 1 Out += sum, mode 3 Out = b - sum - lam X.
template <int MODE, typename SX, typename SO>
__global__ __launch_bounds__(256) void k_parts_sum(const double* __restrict__ work, int splits, int64_t n,
                                                   const double* __restrict__ b, const SX* __restrict__ X,
                                                   double lam, SO* __restrict__ Out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const cx<double>* W = reinterpret_cast<const cx<double>*>(work);
  cx<SO>* O = reinterpret_cast<cx<SO>*>(Out);
  cx<double> z = W[i];
  for (int q = 1; q < splits; ++q) {
    z.re += W[q * n + i].re;
    z.im += W[q * n + i].im;
  }
  if (MODE == 1) {
    const cx<SO> x = O[i];
    O[i] = cx<SO>{SO(x.re + z.re), SO(x.im + z.im)};
  } else if (MODE == 3) {
    const cx<double> bb = reinterpret_cast<const cx<double>*>(b)[i];
    const cx<SX> x = reinterpret_cast<const cx<SX>*>(X)[i];
    O[i] = cx<SO>{SO(bb.re - z.re - lam * (double)x.re), SO(bb.im - z.im - lam * (double)x.im)};
  } else {
    O[i] = cx<SO>{SO(z.re), SO(z.im)};
  }
}

// Parts of a contraction of `chunks` chunks over `tiles` workgroups: enough to put one
// workgroup on each of 512 places, of at least 8 chunks.  A refinement's residual and
// triangular products at few frames were three chains of N / 8 chunks on a few CUs, whole
// against in parts: N = 1024, 64 frames 455 / 89 us; 2304, 1 frame 991 / 162; 4096, 1 frame
// 1748 / 420, 250 frames (2 parts) 1797 / 1624; 16384, 1 frame 7.0 / 6.2 ms.
static int few_splits(long tiles, int chunks) {
  return (int)std::max<long>(1, std::min<long>(512 / std::max<long>(tiles, 1), chunks / 8));
}

// Elementwise FP64 -> FP32 complex copy (n complex values).
__global__ void k_to_f32(const double* __restrict__ in, float* __restrict__ out, size_t n2) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n2;
       i += (size_t)gridDim.x * blockDim.x)
    out[i] = (float)in[i];
}

// Elementwise FP32 -> FP64 complex copy (n complex values).
__global__ void k_to_f64(const float* __restrict__ in, double* __restrict__ out, size_t n2) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n2;
       i += (size_t)gridDim.x * blockDim.x)
    out[i] = (double)in[i];
}


// host launchers
template <typename T, typename SX, typename SD>
hipError_t launch_forward(const EncDev<T>& e, const SX* X, int F, const SD* Din, T* Dout,
                          hipStream_t s) {
  typedef typename PickCfg<T>::type Cfg;
  const int tiles = cdiv(F, Cfg::BM) * cdiv(e.M, Cfg::BN);
  if (tiles == 0) return hipSuccess;
  return with_feat_al(enc_features(e), row_aligned(e, Cfg::BK), [&](auto fc, auto al) {
    hipLaunchKernelGGL((k_forward<Cfg, decltype(fc)::value, SX, SD, decltype(al)::value>),
                       dim3(tiles), dim3(256), smem_bytes<Cfg>(), s, e, X, F, Din, Dout);
    return hipGetLastError();
  });
}

// The adjoint's tile kernel for this encoding and its contraction split:
// f(kernel, tiles, splits, kchunk) with the split chosen to fill the last
// round of the tile grid (pick_split).
template <typename T, typename SD, typename SX, typename SO, class Fn>
static hipError_t adjoint_plan(const EncDev<T>& e, int F, Fn&& f) {
  typedef typename std::conditional<std::is_same<T, double>::value, F64Cfg3, F32Cfg>::type Cfg;
  const int tiles = cdiv(F, Cfg::BM) * cdiv(e.N, Cfg::BN);
  return with_feat_al(enc_features(e), e.K % Cfg::BK == 0, [&](auto fc, auto al) {
    auto kern = k_adjoint<Cfg, decltype(fc)::value, SD, SX, SO, decltype(al)::value>;
    const int nchunks = cdiv(e.M, Cfg::BK);
    const int splits =
        tiles ? pick_split(tiles, resident_blocks(kern, 256, smem_bytes<Cfg>()), nchunks) : 1;
    return f(kern, Cfg{}, tiles, splits, cdiv(nchunks, splits) * Cfg::BK);
  });
}

template <typename T, typename SD, typename SX, typename SO>
size_t adjoint_scratch_bytes(const EncDev<T>& e, int F) {
  size_t bytes = 0;
  (void)adjoint_plan<T, SD, SX, SO>(e, F, [&](auto, auto, int tiles, int splits, int) {
    if (tiles > 0 && splits > 1) bytes = (size_t)splits * F * e.N * 2 * sizeof(T);
    return hipSuccess;
  });
  return bytes;
}

template <typename T, typename SD, typename SX, typename SO>
hipError_t launch_adjoint(const EncDev<T>& e, const SD* D, int F, const SX* X, double lam, SO* Z,
                          Scratch& sc, hipStream_t s) {
  return adjoint_plan<T, SD, SX, SO>(e, F, [&](auto kern, auto cfg, int tiles, int splits,
                                               int kchunk) {
    typedef decltype(cfg) Cfg;
    if (tiles == 0) return hipSuccess;
    // split the M contraction when one pass of the tile grid would leave the
    // GPU partly idle (the grid's last round is what the split fills)
    if (splits == 1) {
      hipLaunchKernelGGL(kern, dim3(tiles), dim3(256), smem_bytes<Cfg>(), s, e, D, F, X, lam, Z,
                         tiles, kchunk, (T*)nullptr);
      return hipGetLastError();
    }
    const int64_t n = (int64_t)F * e.N;
    void* work = nullptr;
    hipError_t err = sc.get(&work, (size_t)splits * n * 2 * sizeof(T), s);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kern, dim3(tiles * splits), dim3(256), smem_bytes<Cfg>(), s, e, D, F, X, lam,
                       Z, tiles, kchunk, (T*)work);
    err = hipGetLastError();
    if (err == hipSuccess) {
      const int blocks = (int)std::min<int64_t>((n + 255) / 256, 1 << 16);
      hipLaunchKernelGGL((k_split_reduce<T, SX, SO>), dim3(blocks), dim3(256), 0, s,
                         (const T*)work, splits, n, X, lam, Z);
      err = hipGetLastError();
    }
    const hipError_t ferr = sc.put(work, s);
    return err != hipSuccess ? err : ferr;
  });
}

// ---------------------------------------------------------------------------
// Adjoint through a stored F^H, the encoding of one coil, in FP64: T = D F^* for every
// (frame, coil) as a row, then b[f][n] = sum_c conj(coil[c][n]) T[(f, c)][n].  F^H is
// formed once per call, in slabs of columns n; the direct sum forms its elements, each
// with a sine and cosine under an off-resonance map, once per coil and 64 frames.
// ---------------------------------------------------------------------------
template <class Cfg>
__global__ __launch_bounds__(256, MinBlocks<Cfg>::value) void k_adjoint_rows(
    const float* __restrict__ D, const double* __restrict__ Fh, double* __restrict__ T, int rows, int n, int K,
    int tiles, int kchunk) {
  const int nbj = (n + Cfg::BN - 1) / Cfg::BN;
  const int split = blockIdx.x / tiles, t = blockIdx.x - split * tiles;
  const int bi = t / nbj, bj = t % nbj;
  const int k0 = split * kchunk, k1 = min(K, k0 + kchunk);
  LoadDenseKC<Cfg, Cfg::BM, Cfg::LDA, float, false> la;
  LoadDenseKC<Cfg, Cfg::BN, Cfg::LDB, double, false> lb;
  la.p = reinterpret_cast<const cx<float>*>(D);
  lb.p = reinterpret_cast<const cx<double>*>(Fh);
  la.ld = lb.ld = K;
  la.o0 = bi * Cfg::BM;
  la.oend = rows;
  lb.o0 = bj * Cfg::BN;
  lb.oend = n;
  AccTile<Cfg> acc;
  acc.zero();
  mainloop<Cfg>(la, lb, k0, k1, acc, smem_base<Cfg>());
  cx<double>* O = reinterpret_cast<cx<double>*>(T) + (size_t)split * rows * n;
  const int r0 = bi * Cfg::BM, c0 = bj * Cfg::BN;
  acc_foreach<Cfg>(acc, [&](int r, int c, double re, double im) {
    if (r0 + r < rows && c0 + c < n) O[(size_t)(r0 + r) * n + c0 + c] = cx<double>{re, im};
  });
}

// b[f][n0 + j] = sum_c conj(coil[c][(n0 + j) % V]) sum_split T[split][(f, c)][j].
__global__ __launch_bounds__(256) void k_adjoint_coils(EncDev<double> e, const double* __restrict__ T, int splits,
                                                       int F, int n0, int n, double* __restrict__ b) {
  const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= (int64_t)F * n) return;
  const int f = (int)(u / n), j = (int)(u - (int64_t)f * n);
  const cx<double>* t = reinterpret_cast<const cx<double>*>(T);
  const cx<double>* coil = reinterpret_cast<const cx<double>*>(e.coil);
  const size_t part = (size_t)F * e.C * n;
  cx<double> z{0.0, 0.0};
  for (int c = 0; c < e.C; ++c) {
    cx<double> v{0.0, 0.0};
    for (int q = 0; q < splits; ++q) {
      const cx<double> p = t[q * part + ((size_t)f * e.C + c) * n + j];
      v.re += p.re;
      v.im += p.im;
    }
    const cx<double> a = coil ? coil[(size_t)c * e.V + (n0 + j) % e.V] : cx<double>{1.0, 0.0};
    z.re += v.re * a.re + v.im * a.im;
    z.im += v.im * a.re - v.re * a.im;
  }
  reinterpret_cast<cx<double>*>(b)[(size_t)f * e.N + n0 + j] = z;
}

constexpr size_t kStoredBytes = (size_t)512 << 20;   // F^H and T of a slab

struct StoredPlan {
  int splits, kchunk, n;   // contraction split, columns per slab (0: a slab does not fit)
  size_t bytes;
};
static StoredPlan stored_plan(const EncDev<double>& e, int F, size_t room) {
  typedef F64Cfg3 Cfg;
  const int64_t rows = (int64_t)F * e.C;
  StoredPlan p{};
  const int nchunks = cdiv(e.K, Cfg::BK);
  auto columns = [&](int splits, size_t bytes) {
    const int64_t n = (int64_t)(bytes / (16 * ((size_t)e.K + splits * rows)));
    return (int)std::min<int64_t>(e.N, n >= e.N ? n : n / Cfg::BN * Cfg::BN);
  };
  // (the split, which the sums' order follows from, does not depend on the room)
  const int n1 = columns(1, kStoredBytes);
  if (n1 <= 0) return p;
  p.splits = pick_split((long)cdiv(rows, Cfg::BM) * cdiv(n1, Cfg::BN),
                        resident_blocks(k_adjoint_rows<Cfg>, 256, smem_bytes<Cfg>()), nchunks);
  if (columns(p.splits, kStoredBytes / 4) <= 0) p.splits = 1;
  p.kchunk = cdiv(nchunks, p.splits) * Cfg::BK;
  p.n = columns(p.splits, std::min(kStoredBytes, room));
  p.bytes = 16 * (size_t)p.n * ((size_t)e.K + p.splits * rows);
  return p;
}

// F^H's elements are formed once instead of once per coil and 64 frames.  A refinement
// step, direct sum against stored F^H: five species of 32 x 32 with a map, 8 coils, 200
// frames 13.2 / 8.6 ms; one, 20 frames 1316 / 569 us, 200 frames of one coil 641 / 611;
// 16 x 16 without a map, 8 coils, 500 frames 785 / 425, 8 x 8, 4 coils, 5 frames 83 / 83.
// With one coil, at most 64 frames and no map nothing is formed twice (212 / 217).
bool stored_adjoint(const EncDev<double>& e, int F) {
  return F > 0 && (e.C > 1 || e.b0 || F > F64Cfg3::BM) && stored_plan(e, F, kStoredBytes / 4).n > 0;
}

hipError_t launch_stored_adjoint(const EncDev<double>& e, const float* D, int F, double* b, Scratch& sc,
                                 hipStream_t s) {
  typedef F64Cfg3 Cfg;
  const StoredPlan p = stored_plan(e, F, sc.room());
  if (p.n == 0) return hipErrorOutOfMemory;
  void* work = nullptr;
  hipError_t err = sc.get(&work, p.bytes, s);
  if (err != hipSuccess) return err;
  double* Fh = (double*)work;
  double* T = Fh + 2 * (size_t)p.n * e.K;
  const int rows = F * e.C;
  EncDev<double> f = e;   // one coil's rows
  f.coil = nullptr;
  f.C = 1;
  f.M = e.K;
  for (int n0 = 0; n0 < e.N; n0 += p.n) {
    const int n = std::min(p.n, e.N - n0), tiles = cdiv(rows, Cfg::BM) * cdiv(n, Cfg::BN);
    if ((err = launch_gen_eh(f, Fh, s, n0, n)) != hipSuccess) break;
    hipLaunchKernelGGL(k_adjoint_rows<Cfg>, dim3(tiles * p.splits), dim3(256), smem_bytes<Cfg>(), s, D,
                       (const double*)Fh, T, rows, n, e.K, tiles, p.kchunk);
    hipLaunchKernelGGL(k_adjoint_coils, dim3((unsigned)(((int64_t)F * n + 255) / 256)), dim3(256), 0, s, e,
                       (const double*)T, p.splits, F, n0, n, b);
    if ((err = hipGetLastError()) != hipSuccess) break;
  }
  const hipError_t ferr = sc.put(work, s);
  return err != hipSuccess ? err : ferr;
}

static int resid_splits(int F, int N) {
  typedef F64Cfg3 Cfg;
  return few_splits((long)cdiv(F, Cfg::BM) * cdiv(N, Cfg::BN), cdiv(N, Cfg::BK));
}
// Triangular products in parts are summed in FP64, also from an FP32 factor: in FP32 the
// parts' rounding adds to the refined images' error (one coil of 64 x 64, 50 frames, one
// step: 4.0e-8 in one FP32 sum, 4.4e-8 in FP32 parts, 2.6e-8 like this).
static int tri_splits(int F, int N) {   // (a tile's mean contraction: N / 2)
  typedef F64Cfg3 Cfg;
  return few_splits((long)cdiv(F, Cfg::BM) * cdiv(N, Cfg::BN), cdiv(N, 2 * Cfg::BK));
}

// Scratch for a split's parts; without it the contraction runs whole (*splits = 1).
static hipError_t parts_get(void** work, int* splits, int F, int N, Scratch& sc, hipStream_t s) {
  *work = nullptr;
  if (*splits <= 1) return hipSuccess;
  hipError_t err = sc.get(work, (size_t)*splits * F * N * 16, s);
  if (err == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    *work = nullptr;
    *splits = 1;
    err = hipSuccess;
  }
  return err;
}

template <typename SX, typename SO>
hipError_t launch_resid(const double* G, const double* b, const SX* X, int F, int N, double lam,
                        SO* Out, Scratch& sc, hipStream_t s) {
  typedef F64Cfg3 Cfg;
  const int tiles = cdiv(F, Cfg::BM) * cdiv(N, Cfg::BN);
  if (tiles == 0) return hipSuccess;
  int splits = resid_splits(F, N);
  void* work = nullptr;
  hipError_t err = parts_get(&work, &splits, F, N, sc, s);
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL((k_resid<Cfg, SX, SO>), dim3(tiles * splits), dim3(256), smem_bytes<Cfg>(), s, G, b, X,
                     F, N, lam, Out, splits, (double*)work);
  if (!work) return hipGetLastError();
  const int64_t n = (int64_t)F * N;
  hipLaunchKernelGGL((k_parts_sum<3, SX, SO>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                     (const double*)work, splits, n, b, X, lam, Out);
  err = hipGetLastError();
  const hipError_t ferr = sc.put(work, s);
  return err != hipSuccess ? err : ferr;
}

template <typename T, int MODE, typename SO>
hipError_t launch_tri_frames(const T* Li, const T* In, int F, int N, SO* Out, Scratch& sc, hipStream_t s) {
  if (F <= 0 || N <= 0) return hipSuccess;
  int splits = tri_splits(F, N);
  void* work = nullptr;
  hipError_t err = parts_get(&work, &splits, F, N, sc, s);
  if (err != hipSuccess) return err;
  if (!work) {
    typedef typename PickCfg<T>::type Cfg;
    hipLaunchKernelGGL((k_tri_frames<Cfg, MODE, SO, T>), dim3(cdiv(F, Cfg::BM) * cdiv(N, Cfg::BN)), dim3(256),
                       smem_bytes<Cfg>(), s, Li, In, F, N, Out, 1, (T*)nullptr);
    return hipGetLastError();
  }
  typedef F64Cfg3 Cfg;
  hipLaunchKernelGGL((k_tri_frames<Cfg, MODE, SO, T>), dim3(cdiv(F, Cfg::BM) * cdiv(N, Cfg::BN) * splits),
                     dim3(256), smem_bytes<Cfg>(), s, Li, In, F, N, Out, splits, (double*)work);
  const int64_t n = (int64_t)F * N;
  hipLaunchKernelGGL((k_parts_sum<MODE, double, SO>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                     (const double*)work, splits, n, (const double*)nullptr, (const double*)nullptr, 0.0, Out);
  err = hipGetLastError();
  const hipError_t ferr = sc.put(work, s);
  return err != hipSuccess ? err : ferr;
}


hipError_t launch_to_f64(const float* in, double* out, size_t n_complex, hipStream_t s) {
  const size_t n2 = 2 * n_complex;
  int blocks = (int)std::min<size_t>(4096, (n2 + 255) / 256);
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_to_f64, dim3(blocks), dim3(256), 0, s, in, out, n2);
  return hipGetLastError();
}

hipError_t launch_to_f32(const double* in, float* out, size_t n_complex, hipStream_t s) {
  const size_t n2 = 2 * n_complex;
  int blocks = (int)std::min<size_t>(4096, (n2 + 255) / 256);
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_to_f32, dim3(blocks), dim3(256), 0, s, in, out, n2);
  return hipGetLastError();
}

// explicit instantiations
template hipError_t launch_forward<float, float, float>(const EncDev<float>&, const float*, int,
                                                        const float*, float*, hipStream_t);
template hipError_t launch_forward<double, double, double>(const EncDev<double>&, const double*, int,
                                                           const double*, double*, hipStream_t);
template hipError_t launch_forward<double, float, float>(const EncDev<double>&, const float*, int,
                                                         const float*, double*, hipStream_t);
template hipError_t launch_resid<float, float>(const double*, const double*, const float*, int, int,
                                               double, float*, Scratch&, hipStream_t);
template hipError_t launch_resid<double, double>(const double*, const double*, const double*, int,
                                                 int, double, double*, Scratch&, hipStream_t);
template hipError_t launch_resid<double, float>(const double*, const double*, const double*, int,
                                                int, double, float*, Scratch&, hipStream_t);
template hipError_t launch_tri_frames<float, 1, double>(const float*, const float*, int, int, double*,
                                                        Scratch&, hipStream_t);
template hipError_t launch_tri_frames<float, 2, double>(const float*, const float*, int, int, double*,
                                                        Scratch&, hipStream_t);
template hipError_t launch_tri_frames<float, 0, float>(const float*, const float*, int, int, float*,
                                                       Scratch&, hipStream_t);
template hipError_t launch_tri_frames<float, 1, float>(const float*, const float*, int, int, float*,
                                                       Scratch&, hipStream_t);
template hipError_t launch_tri_frames<double, 0, double>(const double*, const double*, int, int,
                                                         double*, Scratch&, hipStream_t);
template hipError_t launch_tri_frames<double, 1, double>(const double*, const double*, int, int,
                                                         double*, Scratch&, hipStream_t);
template hipError_t launch_tri_frames<double, 2, double>(const double*, const double*, int, int,
                                                         double*, Scratch&, hipStream_t);
template hipError_t launch_tri_frames<float, 2, float>(const float*, const float*, int, int, float*,
                                                       Scratch&, hipStream_t);
template hipError_t launch_adjoint<double, double, float, float>(const EncDev<double>&, const double*, int,
    const float*, double, float*, Scratch&, hipStream_t);
template size_t adjoint_scratch_bytes<double, double, float, float>(const EncDev<double>&, int);
template hipError_t launch_adjoint<double, double, double, double>(const EncDev<double>&, const double*, int,
    const double*, double, double*, Scratch&, hipStream_t);
template size_t adjoint_scratch_bytes<double, double, double, double>(const EncDev<double>&, int);
template hipError_t launch_adjoint<double, float, float, double>(const EncDev<double>&, const float*, int,
    const float*, double, double*, Scratch&, hipStream_t);
template size_t adjoint_scratch_bytes<double, float, float, double>(const EncDev<double>&, int);
template hipError_t launch_adjoint<double, float, float, float>(const EncDev<double>&, const float*, int,
    const float*, double, float*, Scratch&, hipStream_t);
template size_t adjoint_scratch_bytes<double, float, float, float>(const EncDev<double>&, int);
template hipError_t launch_adjoint<float, float, float, float>(const EncDev<float>&, const float*, int,
    const float*, double, float*, Scratch&, hipStream_t);
template size_t adjoint_scratch_bytes<float, float, float, float>(const EncDev<float>&, int);

}  // namespace pinv
