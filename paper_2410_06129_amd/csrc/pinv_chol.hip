// Blocked right-looking Cholesky of G + lam I in FP64 with L^-1 formed
// alongside (Eq. 6, Eq. 8; Sec. 2.3).
#include <type_traits>

#include "pinv_internal.h"

namespace pinv {

// ---------------------------------------------------------------------------
// Cholesky diagonal block (FP64, one workgroup): L_kk^-1 of the 64 x 64 Hermitian
// block A_kk + lam I = L_kk L_kk^H, in four steps of 16 columns.  Step s
//   factors the 16 x 16 block A_ss:  T_s = L_ss^-1        (one wave)
//   forms  L_is = A_is T_s^H (i > s)  and  Y_sj = T_s B_sj (j < s), Y_ss = T_s
//   updates A_ij -= L_is L_js^H (i >= j > s)  and  B_ij -= L_is Y_sj (j <= s < i)
// with B the right-hand side of L Y = I, whose rows become those of the inverse.
// Only lower blocks are kept, so the matrix stays exactly Hermitian; the diagonal's
// imaginary parts are dropped.  The products run on MFMA, a 16 x 16 block per wave;
// wave 0 updates A_{s+1,s+1} first and factors it while the others finish.
//
// Bound by latency: 64 dependent columns in one workgroup.  Eliminating one column
// of the whole block at a time, with a division and a masked rank-1 update in every
// one of 16 waves, took 57 us (up to 85 beside trailing tiles); this form takes 28,
// nearly all of it the columns of the 16 x 16 blocks (an LDS exchange, a
// reciprocal and a multiply-add each).
// ---------------------------------------------------------------------------
constexpr int kDiagWaves = 10;   // at most 9 block products in a step, and the factoring wave
constexpr int kSubLd = 17;       // row stride of a 16 x 16 block in LDS
constexpr int kSub = 16 * kSubLd;

// Lower block (i, j) of a 4 x 4 block matrix.
__device__ __forceinline__ int sub_index(int i, int j) { return i * (i + 1) / 2 + j; }

struct SubBlock { double re[kSub], im[kSub]; };

// acc = X op(Y): op(Y) = Y^H (HERM: rows of Y are the result's columns) or Y.
template <bool HERM>
__device__ __forceinline__ void sub_product(const SubBlock& X, const SubBlock& Y, f64x4& re, f64x4& im) {
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
  re = im = f64x4{0, 0, 0, 0};
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const int k = kk * 4 + lk;
    const double ar = X.re[lr * kSubLd + k], ai = X.im[lr * kSubLd + k];
    const int y = HERM ? lr * kSubLd + k : k * kSubLd + lr;
    const double br = Y.re[y], bi = HERM ? -Y.im[y] : Y.im[y];
    re = mfma4(ar, br, re);
    re = mfma4(-ai, bi, re);
    im = mfma4(ar, bi, im);
    im = mfma4(ai, br, im);
  }
}

// O = acc, or O -= acc.
template <bool SUB>
__device__ __forceinline__ void sub_store(SubBlock& O, const f64x4& re, const f64x4& im) {
  const int lane = threadIdx.x & 63, col = lane & 15;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int o = ((lane >> 4) + 4 * r) * kSubLd + col;
    O.re[o] = SUB ? O.re[o] - re[r] : re[r];
    O.im[o] = SUB ? O.im[o] - im[r] : im[r];
  }
}

// Orders a wave's own LDS accesses (which the hardware runs in order).
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// 1 / p: the hardware's 2^-24 start and two Newton steps (a fifth of the division's
// dependent instructions).  Equal to the division bit for bit for all of 2.6e8 random p
// over 2^-1000 .. 2^1000.
__device__ __forceinline__ double recip(double p) {
  double r = __builtin_amdgcn_rcp(p);
  r = fma(r, fma(-p, r, 1.0), r);
  return fma(r, fma(-p, r, 1.0), r);
}

// The value of x in lane `l` (uniform), the same for the whole wave.
__device__ __forceinline__ double lane_value(double x, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l),
                          __builtin_amdgcn_readlane(__double2loint(x), l));
}

// One wave: T = L^-1 of the Hermitian 16 x 16 block A = L L^H, by elimination of
// [A | I] without pivoting (A = Lt D Lt^H, L^-1 = D^-1/2 Lt^-1).  One complex value
// per row and column: column c of row i holds A_ic while c is still to be
// eliminated and (Lt^-1)_ic once it has been.  Lane l holds row l / 4, columns
// 4 (l % 4) .. + 4.  Column j and row j are published to LDS when final, and the
// pivot's reciprocal is formed from a lane read meanwhile; row j of A is read as the
// conjugate of column j.  Returns the first column whose pivot is
// not positive (NaN included), 16 if none.
__device__ __forceinline__ int sub_factor(const SubBlock& A, SubBlock& T, cx<double> (&xch)[2][32],
                                          double (&dpiv)[16]) {
  const int lane = threadIdx.x & 63, r = lane >> 2, q = lane & 3;
  cx<double> z[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int c = 4 * q + t;
    z[t] = cx<double>{A.re[r * kSubLd + c], c == r ? 0.0 : A.im[r * kSubLd + c]};
  }
  if (q == 0) xch[0][r] = z[0];
  wave_order();
  int bad = 16;
  // four columns unrolled: the code of all 16 would run from a cold instruction
  // cache every time
  for (int j0 = 0; j0 < 16; j0 += 4) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = j0 + u;
      const cx<double>* x = xch[u & 1];   // column j, then row j's columns below j
      const double piv = lane_value(z[u].re, 4 * j + j0 / 4);
      if (!(piv > 0.0) && bad == 16) bad = j;
      const double inv = recip(piv);
      if (lane == 0) dpiv[j] = piv;
      const cx<double> a = x[r];
      cx<double> w[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int c = 4 * q + t;
        w[t] = x[c < j ? 16 + c : c];
      }
      if (r > j) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int c = 4 * q + t;
          cx<double> p{w[t].re * inv, (c < j ? w[t].im : -w[t].im) * inv};
          cx<double> o = z[t];
          if (c == j) {
            p = cx<double>{inv, 0.0};
            o = cx<double>{0.0, 0.0};
          }
          o.re -= a.re * p.re - a.im * p.im;
          o.im -= a.re * p.im + a.im * p.re;
          z[t] = o;
        }
      }
      if (j < 15) {
        cx<double>* y = xch[(u + 1) & 1];
        if (q == (j + 1) / 4) y[r] = z[(u + 1) % 4];
        if (r == j + 1) {
#pragma unroll
          for (int t = 0; t < 4; ++t) y[16 + 4 * q + t] = z[t];
        }
      }
      wave_order();
    }
  }
  const double sc = 1.0 / sqrt(dpiv[r]);
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int c = 4 * q + t;
    T.re[r * kSubLd + c] = c < r ? z[t].re * sc : c == r ? sc : 0.0;
    T.im[r * kSubLd + c] = c < r ? z[t].im * sc : 0.0;
  }
  wave_order();
  return bad;
}

__global__ __launch_bounds__(64 * kDiagWaves) void k_chol_diag(double* __restrict__ A,
                                                               double* __restrict__ Li, int N, int k,
                                                               double lam, int* __restrict__ info) {
  __shared__ SubBlock a[10], y[10];
  __shared__ cx<double> xch[2][32];
  __shared__ double dpiv[16];
  __shared__ int bad;
  constexpr int NT = 64 * kDiagWaves, PASSES = (4096 + NT - 1) / NT;
  const int failed = *info;   // (tested below: the loads do not wait for it)
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int k0 = k * 64, nbk = min(64, N - k0);
  const cx<double>* Ac = reinterpret_cast<const cx<double>*>(A);
  cx<double>* Lc = reinterpret_cast<cx<double>*>(Li);
  if (tid == 0) bad = 64;
  cx<double> v[PASSES];
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {   // all loads in flight; rows past N re-read the last
    const int u = tid + p * NT, row = min(u / 64, nbk - 1), col = min(u % 64, row);
    v[p] = Ac[(size_t)(k0 + row) * N + k0 + col];
  }
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    const int u = tid + p * NT, row = u / 64, col = u % 64, i = row / 16, j = col / 16;
    if (u >= 4096 || j > i) continue;
    cx<double> x{0.0, 0.0};
    if (row < nbk && col <= row) x = v[p];
    if (row == col) x = cx<double>{row < nbk ? x.re + lam : 1.0, 0.0};   // rows past N: identity
    const int o = (row % 16) * kSubLd + col % 16;
    a[sub_index(i, j)].re[o] = x.re;
    a[sub_index(i, j)].im[o] = x.im;
    y[sub_index(i, j)].re[o] = y[sub_index(i, j)].im[o] = 0.0;
  }
  __syncthreads();
  if (failed) return;
  for (int s = 0; s < 4; ++s) {
    if (s > 0) {
      // step s - 1's updates; item 0 is A_ss, wave 0's, the other waves share the rest
      const int rem = 4 - s, nherk = rem * (rem + 1) / 2, items = nherk + rem * s;
      for (int t = w; t < items; t += w == 0 ? items : kDiagWaves - 1) {
        f64x4 re, im;
        if (t < nherk) {
          const int ti = t < 1 ? 0 : t < 3 ? 1 : 2, tj = t - ti * (ti + 1) / 2;
          const int i = s + ti, j = s + tj;
          sub_product<true>(a[sub_index(i, s - 1)], a[sub_index(j, s - 1)], re, im);
          sub_store<true>(a[sub_index(i, j)], re, im);
        } else {
          const int v = t - nherk, i = s + v / s, j = v % s;
          sub_product<false>(a[sub_index(i, s - 1)], y[sub_index(s - 1, j)], re, im);
          sub_store<true>(y[sub_index(i, j)], re, im);
        }
      }
    }
    if (w == 0) {
      wave_order();
      const int c = sub_factor(a[sub_index(s, s)], y[sub_index(s, s)], xch, dpiv);
      if (c < 16 && tid == 0) bad = 16 * s + c;
    }
    __syncthreads();
    if (bad < 64) {   // the same for every thread
      if (tid == 0) atomicCAS(info, 0, k0 + bad + 1);
      return;
    }
    // three products, in place: L_is for i > s, Y_sj for j < s
    if (w < 3) {
      const SubBlock& T = y[sub_index(s, s)];
      f64x4 re, im;
      if (w < 3 - s) {
        SubBlock& O = a[sub_index(s + 1 + w, s)];
        sub_product<true>(O, T, re, im);
        wave_order();
        sub_store<false>(O, re, im);
      } else {
        SubBlock& O = y[sub_index(s, w - (3 - s))];
        sub_product<false>(T, O, re, im);
        wave_order();
        sub_store<false>(O, re, im);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    const int u = tid + p * NT, row = u / 64, col = u % 64, i = row / 16, j = col / 16;
    if (u >= 4096 || row >= nbk || col >= nbk) continue;
    cx<double> x{0.0, 0.0};
    if (j <= i) {
      const int o = (row % 16) * kSubLd + col % 16;
      x = cx<double>{y[sub_index(i, j)].re[o], y[sub_index(i, j)].im[o]};
    }
    Lc[(size_t)(k0 + row) * N + k0 + col] = x;
  }
}

// Block (bi, bj) store helper for nb x nb FP64 blocks of an N x N matrix.
typedef TileCfg<double, 64, 64, 8> CholCfg;

// ---------------------------------------------------------------------------
// Short products: an RM x RN tile over at most a few times 64 columns
// ---------------------------------------------------------------------------
// The panel and, near the end or in a small matrix, the trailing update are a few
// tiles of 64 or 128 columns: bound by latency, not by the matrix cores.  All
// loads of a 64-column chunk are in flight at once (the next chunk's under this
// one's products), against eight chunks of eight with a barrier each in the long
// products' loop, and the tiles are smaller, so that more CUs share the work (a
// panel 14 -> 8 us, a trailing update of few tiles 27 -> 6 to 9 us).
// Wave w computes the 16 x 16 block (w / (RN / 16), w % (RN / 16)).
template <int RM, int RN> struct ShortTile {
  static constexpr int NT = RM / 16 * (RN / 16) * 64;
  static constexpr int LDA = RM + 1, LDB = RN + 1;   // odd: stores along k hit distinct banks
  static constexpr int PA = RM * 64 / NT, PB = RN * 64 / NT;
  double a[2][64 * LDA], b[2][64 * LDB];
};

// acc = sum_{l < kw} A[o][l] op(B)[l][n]: A rows o0a .. (k contiguous, zero at or
// past oenda), B rows o0b .. conjugated (k contiguous) or, with BOC, B[l][n] with
// columns n from o0b (zero at or past oendb).
template <int RM, int RN, bool BOC>
__device__ __forceinline__ void short_product(ShortTile<RM, RN>& sm, const cx<double>* __restrict__ A,
                                              int64_t lda, int o0a, int oenda,
                                              const cx<double>* __restrict__ B, int64_t ldb, int o0b,
                                              int oendb, int kw, f64x4& re, f64x4& im) {
  typedef ShortTile<RM, RN> S;
  const int tid = threadIdx.x;
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  cx<double> va[S::PA], vb[S::PB];
  // the clamped loads stay in bounds; what they stand for is zeroed in store()
  auto fetch = [&](int k0) {
#pragma unroll
    for (int i = 0; i < S::PA; ++i) {
      const int u = tid + i * S::NT, o = o0a + u / 64, l = k0 + u % 64;
      va[i] = A[(int64_t)min(o, oenda - 1) * lda + min(l, kw - 1)];
    }
#pragma unroll
    for (int i = 0; i < S::PB; ++i) {
      const int u = tid + i * S::NT;
      const int o = o0b + (BOC ? u % RN : u / 64), l = k0 + (BOC ? u / RN : u % 64);
      const int oc = min(o, oendb - 1), lc = min(l, kw - 1);
      vb[i] = B[BOC ? (int64_t)lc * ldb + oc : (int64_t)oc * ldb + lc];
    }
  };
  auto store = [&](int k0) {
#pragma unroll
    for (int i = 0; i < S::PA; ++i) {
      const int u = tid + i * S::NT, o = u / 64, l = u % 64;
      const bool ok = o0a + o < oenda && k0 + l < kw;
      sm.a[0][l * S::LDA + o] = ok ? va[i].re : 0.0;
      sm.a[1][l * S::LDA + o] = ok ? va[i].im : 0.0;
    }
#pragma unroll
    for (int i = 0; i < S::PB; ++i) {
      const int u = tid + i * S::NT, o = BOC ? u % RN : u / 64, l = BOC ? u / RN : u % 64;
      const bool ok = o0b + o < oendb && k0 + l < kw;
      sm.b[0][l * S::LDB + o] = ok ? vb[i].re : 0.0;
      sm.b[1][l * S::LDB + o] = ok ? (BOC ? vb[i].im : -vb[i].im) : 0.0;
    }
  };
  re = im = f64x4{0, 0, 0, 0};
  fetch(0);
  for (int k0 = 0; k0 < kw; k0 += 64) {
    if (k0) __syncthreads();   // the last chunk's reads are done
    store(k0);
    __syncthreads();
    if (k0 + 64 < kw) fetch(k0 + 64);
    const int oa = w / (RN / 16) * 16 + lr, ob = w % (RN / 16) * 16 + lr;
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      const int l = kk * 4 + lk;
      const double ar = sm.a[0][l * S::LDA + oa], ai = sm.a[1][l * S::LDA + oa];
      const double br = sm.b[0][l * S::LDB + ob], bi = sm.b[1][l * S::LDB + ob];
      re = mfma4(ar, br, re);
      re = mfma4(-ai, bi, re);
      im = mfma4(ar, bi, im);
      im = mfma4(ai, br, im);
    }
  }
}

// Visit this lane's four elements of its wave's block: f(q, row, col).
template <int RM, int RN, class F>
__device__ __forceinline__ void short_foreach(F&& f) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
  for (int q = 0; q < 4; ++q)
    f(q, w / (RN / 16) * 16 + (lane >> 4) + 4 * q, w % (RN / 16) * 16 + (lane & 15));
}

// Step k, after the diagonal block: panel blocks i > k become L_ik = A_ik L_kk^-H
// (in place, 32 of a block's rows per workgroup), and the inverse's blocks j < k of
// row k become Y_kj = L_kk^-1 B_kj (in place, 32 of a block's columns).
__global__ __launch_bounds__((ShortTile<32, 64>::NT)) void k_chol_panel(double* __restrict__ A,
                                                                      double* __restrict__ Li, int N,
                                                                      int k,
                                                                      const int* __restrict__ info) {
  const int failed = *info;   // (tested before the stores: the loads do not wait for it)
  __shared__ union {
    ShortTile<32, 64> p;
    ShortTile<64, 32> y;
  } sm;
  const int nblk = (N + 63) / 64;
  const int npanel = 2 * (nblk - k - 1);
  const int t = blockIdx.x, d0 = k * 64;
  const int kw = min(64, N - d0);
  const cx<double>* Lkk = reinterpret_cast<const cx<double>*>(Li) + (size_t)d0 * N + d0;
  f64x4 re, im;
  if (t < npanel) {
    const int r0 = (k + 1) * 64 + t * 32;
    if (r0 >= N) return;
    cx<double>* O = reinterpret_cast<cx<double>*>(A) + d0;
    short_product<32, 64, false>(sm.p, O, N, r0, N, Lkk, N, 0, kw, kw, re, im);
    if (failed) return;
    short_foreach<32, 64>([&](int q, int r, int c) {
      if (r0 + r < N && c < kw) O[(size_t)(r0 + r) * N + c] = cx<double>{re[q], im[q]};
    });
  } else {
    const int c0 = (t - npanel) * 32;   // c0 < 64 k
    cx<double>* O = reinterpret_cast<cx<double>*>(Li) + (size_t)d0 * N;
    short_product<64, 32, true>(sm.y, Lkk, N, 0, kw, O, N, c0, N, kw, re, im);
    if (failed) return;
    short_foreach<64, 32>([&](int q, int r, int c) {
      if (r < kw) O[(size_t)r * N + c0 + c] = cx<double>{re[q], im[q]};
    });
  }
}

// Trailing update after steps kb .. k = kb + kn - 1 (kn = 1, or 2 for the
// two-level factorisation): A_ij -= sum_{l=kb..k} L_il L_jl^H for k < j <= i
// ("herk" tiles) and B_ij -= sum_{l=kb..k} L_il Y_lj for i > k, j <= k
// (inverse tiles), one contraction over the kn 64-column panels, which lie
// side by side in A's columns and in Li's rows (Y_lj for j > l is zero: Li
// starts zeroed and only its lower blocks are written).  `part` selects the
// tiles of one launch:
//   0  all of them;
//   1  the look-ahead set: the next `ahead` block columns of A and block rows of B,
//      all that as many steps' diagonal blocks and panels read;
//   2  the rest, which can run beside those steps' kernels.
// The accumulators start from -(old tile), loaded together with the first
// operand chunk, and the tile is stored negated: no read after the products.
__host__ __device__ __forceinline__ int trailing_tiles(int k, int nblk, int part, int la) {
  const int rem = nblk - k - 1;                        // block rows below step k
  if (part == 1) {
    const int w = la < rem ? la : rem;
    return w * rem - w * (w - 1) / 2 + w * (k + 1);    // w columns of A, w rows of B
  }
  const int r = part == 2 ? rem - la : rem;
  return r <= 0 ? 0 : r * (r + 1) / 2 + r * (k + 1);
}

// Tile t of the list: the 64 x 64 tile's first row and column, of A (herk) or B.
__device__ __forceinline__ void trailing_tile(int t, int k, int nblk, int part, int la, bool* herk,
                                              int* r0, int* c0) {
  const int rem = nblk - k - 1;
  if (part == 1) {
    int j = 0;   // column k + 1 + j of A has rem - j tiles
    const int w = la < rem ? la : rem;
    while (j < w && t >= rem - j) t -= rem - j++;
    *herk = j < w;
    *r0 = (k + 1 + (*herk ? j + t : t / (k + 1))) * 64;
    *c0 = (*herk ? k + 1 + j : t % (k + 1)) * 64;
    return;
  }
  const int first = part == 2 ? k + 1 + la : k + 1;   // first trailing block row/column
  const int r = nblk - first;
  const int nherk = r * (r + 1) / 2;
  *herk = t < nherk;
  if (*herk) {
    int ti, tj;
    tri_index(t, &ti, &tj);
    *r0 = (first + ti) * 64;
    *c0 = (first + tj) * 64;
  } else {
    const int u = t - nherk;
    *r0 = (first + u / (k + 1)) * 64;
    *c0 = (u % (k + 1)) * 64;
  }
}

template <class Cfg>
__global__ __launch_bounds__(256) void k_chol_trailing(double* __restrict__ A, double* __restrict__ Li,
                                                       int N, int kb, int kn,
                                                       const int* __restrict__ info, int part, int ahead) {
  if (*info) return;
  const int nb = 64;
  const int k = kb + kn - 1;
  const int nblk = (N + nb - 1) / nb;
  const int t = blockIdx.x;
  const cx<double>* Ac = reinterpret_cast<const cx<double>*>(A);
  const cx<double>* Lc = reinterpret_cast<const cx<double>*>(Li);
  double* smem = smem_base<Cfg>();
  const int kw = min(N, (k + 1) * nb) - kb * nb;
  bool herk;
  int r0, c0;
  trailing_tile(t, k, nblk, part, ahead, &herk, &r0, &c0);
  cx<double>* O = reinterpret_cast<cx<double>*>(herk ? A : Li);
  AccTile<Cfg> acc;
  acc_foreach_mut<Cfg>(acc, [&](int r, int c, double& re, double& im) {
    const int row = r0 + r, col = c0 + c;
    cx<double> o{0.0, 0.0};
    if (row < N && col < N) o = O[(size_t)row * N + col];
    re = -o.re;
    im = -o.im;
  });
  LoadDenseKC<Cfg, 64, Cfg::LDA, double, false> la;      // L_il[m][.] at A[(i*nb+m)*N + kb*nb + .]
  la.p = Ac + kb * nb;
  la.ld = N;
  la.o0 = r0;
  la.oend = N;
  if (herk) {
    LoadDenseKC<Cfg, 64, Cfg::LDB, double, true> lb;     // conj(L_jl[n][.])
    lb.p = Ac + kb * nb;
    lb.ld = N;
    lb.o0 = c0;
    lb.oend = N;
    mainloop<Cfg, false>(la, lb, 0, kw, acc, smem);
  } else {
    LoadDenseOC<Cfg, 64, Cfg::LDB, double, false> lb;    // Y_lj[.][n] at Li[(kb*nb+.)*N + j*nb + n]
    lb.p = Lc + (size_t)(kb * nb) * N;
    lb.ld = N;
    lb.o0 = c0;
    lb.oend = min(N, c0 + nb);
    mainloop<Cfg, false>(la, lb, 0, kw, acc, smem);
  }
  acc_foreach<Cfg>(acc, [&](int r, int c, double re, double im) {
    const int row = r0 + r, col = c0 + c;
    if (row < N && col < N) O[(size_t)row * N + col] = cx<double>{-re, -im};
  });
}

// The same update by 32 x 32 tiles: tile blockIdx.x / 4 of k_chol_trailing's list,
// quarter blockIdx.x % 4.  kw columns from kb * 64.
__global__ __launch_bounds__((ShortTile<32, 32>::NT)) void k_chol_trailing_short(
    double* __restrict__ A, double* __restrict__ Li, int N, int kb, int kn,
    const int* __restrict__ info, int part, int ahead) {
  const int failed = *info;   // (tested before the stores: the loads do not wait for it)
  __shared__ ShortTile<32, 32> sm;
  const int k = kb + kn - 1, nblk = (N + 63) / 64;
  bool herk;
  int r0, c0;
  trailing_tile(blockIdx.x / 4, k, nblk, part, ahead, &herk, &r0, &c0);
  r0 += 32 * (blockIdx.x / 2 % 2);
  c0 += 32 * (blockIdx.x % 2);
  if (r0 >= N || (herk && (c0 >= N || c0 > r0 + 31))) return;   // past the matrix, above the diagonal
  const int kw = min(N, (k + 1) * 64) - kb * 64;
  const cx<double>* P = reinterpret_cast<const cx<double>*>(A) + kb * 64;
  cx<double>* O = reinterpret_cast<cx<double>*>(herk ? A : Li);
  const int cend = herk ? N : min(N, (k + 1) * 64);   // the inverse's columns end at block k
  cx<double> old[4];
  short_foreach<32, 32>([&](int q, int r, int c) {
    old[q] = O[(size_t)min(r0 + r, N - 1) * N + min(c0 + c, N - 1)];
  });
  f64x4 re, im;
  if (herk)
    short_product<32, 32, false>(sm, P, N, r0, N, P, N, c0, N, kw, re, im);
  else
    short_product<32, 32, true>(sm, P, N, r0, N,
                                reinterpret_cast<const cx<double>*>(Li) + (size_t)(kb * 64) * N, N, c0,
                                cend, kw, re, im);
  if (failed) return;
  short_foreach<32, 32>([&](int q, int r, int c) {
    if (r0 + r < N && c0 + c < cend)
      O[(size_t)(r0 + r) * N + c0 + c] = cx<double>{old[q].re - re[q], old[q].im - im[q]};
  });
}

// host launcher

// Up to this many block columns everything runs on one stream: a step's whole
// trailing update takes less than a look-ahead's events and second launch (6 us
// each).  Whole factorisation on one stream against with look-ahead: N = 400 300 /
// 325 us, 1024 743 / 762, 1296 1038 / 1027, 1521 1315 / 1190, 2025 1962 / 1703.
constexpr int kSerialBlocks = 20;

// Up to this many 64 x 64 trailing tiles (one per CU) go as four 32 x 32 tiles each;
// more fill the CUs as they are.  The factorisation with 0, 128, 256, 512: N = 400
// 378, 302, 300, 301 us; 1024 908, 751, 743, 748; 2025 2080, 1704, 1703, 1735; 4096
// 6646, 5991, 5981, 6003.
constexpr int kShortTiles = 256;

// One factorisation step's trailing launches of step range kb .. kb + kn - 1
// over tiles `part`, the look-ahead set being `la` blocks wide.
template <class Cfg>
static void trailing(double* A, double* Li, int N, int kb, int kn, int* info, int part, int la,
                     hipStream_t st) {
  const int tiles = trailing_tiles(kb + kn - 1, cdiv(N, 64), part, la);
  if (tiles <= 0) return;
  if (tiles <= kShortTiles) {
    hipLaunchKernelGGL(k_chol_trailing_short, dim3(4 * tiles), dim3(ShortTile<32, 32>::NT), 0, st, A, Li,
                       N, kb, kn, (const int*)info, part, la);
    return;
  }
  hipLaunchKernelGGL(k_chol_trailing<Cfg>, dim3(tiles), dim3(256), smem_bytes<Cfg>(), st, A, Li, N,
                     kb, kn, (const int*)info, part, la);
}

// Blocked right-looking factorisation, 64-column steps.  nb = 64: every
// step updates the whole trailing matrix (rank 64).  nb = 128 (two-level):
// the first step of each pair updates only the next block column (and block
// row of the inverse), and after the second step one rank-128 update covers
// the rest, so the trailing matrix is read and written half as often and
// each tile runs twice the matrix products per load of its old value (at
// N = 16384: 238 against 260 ms).
//
// With an auxiliary stream `aux` the factorisation looks ahead: the trailing
// tiles that the next group's steps read (part 1, as wide as a group) run on s, the
// rest (part 2) on aux beside those steps' kernels.  Events order part 2 after part 1
// (so that the next diagonal block's one workgroup is placed before part 2 fills the
// CUs: behind it, it waited for part 2 to end) and every later launch on s that
// touches its tiles after it.  Without aux everything runs on s in order.
template <class Cfg>
static hipError_t cholinv(double* A, double* Li, int N, double lam, int* info, hipStream_t s,
                          hipStream_t aux, int nb) {
  const int nblk = cdiv(N, 64);
  const int kn_max = nb / 64;
  if (nblk <= kSerialBlocks) aux = nullptr;
  hipEvent_t ev_part1 = nullptr, ev_rest = nullptr;
  if (aux) {
    hipError_t err = hipEventCreateWithFlags(&ev_part1, hipEventDisableTiming);
    if (err == hipSuccess) err = hipEventCreateWithFlags(&ev_rest, hipEventDisableTiming);
    if (err != hipSuccess) {
      if (ev_part1) (void)hipEventDestroy(ev_part1);
      return err;
    }
  }
  hipError_t err = hipSuccess;
  bool rest_pending = false;
  for (int kb = 0; kb < nblk && err == hipSuccess; kb += kn_max) {
    const int kn = std::min(kn_max, nblk - kb);
    for (int k = kb; k < kb + kn; ++k) {
      hipLaunchKernelGGL(k_chol_diag, dim3(1), dim3(64 * kDiagWaves), 0, s, A, Li, N, k, lam, info);
      if (nblk - 1 > 0)   // (nblk-k-1) panel tiles + k inverse tiles
        hipLaunchKernelGGL(k_chol_panel, dim3(2 * (nblk - 1)), dim3(ShortTile<32, 64>::NT), 0, s, A, Li,
                           N, k, (const int*)info);
      // inside a group: the next step's block column and row from this step alone
      if (k + 1 < kb + kn) trailing<Cfg>(A, Li, N, k, 1, info, 1, 1, s);
    }
    const int last = kb + kn - 1;
    if ((err = hipGetLastError()) != hipSuccess || nblk - last - 1 <= 0) break;
    if (!aux) {
      trailing<Cfg>(A, Li, N, kb, kn, info, 0, kn_max, s);
      err = hipGetLastError();
      continue;
    }
    // part 1 (s) after the previous part 2
    if (rest_pending && (err = hipStreamWaitEvent(s, ev_rest, 0)) != hipSuccess) break;
    rest_pending = false;
    trailing<Cfg>(A, Li, N, kb, kn, info, 1, kn_max, s);
    if (trailing_tiles(last, nblk, 2, kn_max) > 0) {
      if ((err = hipEventRecord(ev_part1, s)) != hipSuccess) break;
      if ((err = hipStreamWaitEvent(aux, ev_part1, 0)) != hipSuccess) break;
      trailing<Cfg>(A, Li, N, kb, kn, info, 2, kn_max, aux);
      if ((err = hipEventRecord(ev_rest, aux)) != hipSuccess) break;
      rest_pending = true;
    }
    err = hipGetLastError();
  }
  if (aux) {
    // everything after the factorisation on s sees the last part-2 updates
    if (err == hipSuccess && rest_pending) err = hipStreamWaitEvent(s, ev_rest, 0);
    (void)hipEventDestroy(ev_part1);
    (void)hipEventDestroy(ev_rest);
  }
  if (err != hipSuccess) return err;
  return hipGetLastError();
}

// The trailing tiles run four real products per complex product: three (Gauss)
// took longer at N = 16384 (321 against 260 ms at nb = 64, 277 against 238
// at nb = 128), the third LDS plane and the extra accumulators (one wavefront
// per SIMD instead of two) outweighing the fewer matrix products.
hipError_t launch_cholinv(double* A, double* Li, int N, double lam, int* info, hipStream_t s,
                          hipStream_t aux, int nb) {
  if (nb != 64 && nb != 128) return hipErrorInvalidValue;
  return cholinv<CholCfg>(A, Li, N, lam, info, s, aux, nb);
}

}  // namespace pinv
