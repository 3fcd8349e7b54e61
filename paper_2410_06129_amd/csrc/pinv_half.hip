// FP32 products on the f16 matrix pipe: W = L^-1 E^H, R = L^-H W (Eq. 8) and
// the many-frame apply image = R data (Eq. 3) of FP32 plans.
//
// v_mfma_f32_16x16x32_f16 multiplies sixteen times faster than
// v_mfma_f32_16x16x4_f32, so each FP32 operand value is written as a sum of
// f16 pieces, x = 2^-s (h + l [+ t]), each piece the rounding of what the ones
// before it leave, and a real product is the sum of the pieces' products:
//
//   two pieces by two:    h h + h l + l h                (12 MFMAs per complex product)
//   three pieces by two:  h h + h l + l h + t h          (16)
//
// accumulated in FP32.  s is a power of two per row and segment that puts the
// row's largest value in [2^13, 2^14): two pieces then hold 23 bits of every
// value within 2^-15 of the row's largest and 2^-39 of the largest below that,
// three pieces ten bits more.  One instruction sums 32 products of a pair of
// pieces before the FP32 accumulator rounds, against four on the FP32
// instruction, and the dropped l l products (2^-24 relative, of random sign)
// are smaller than what that saves.
//
// The factor takes three pieces, split straight from FP64: its rounding enters
// W and R alike, adds up coherently in R data, and with FP32 values made most
// of an FP32 plan's unrefined error.  E, W, R and the data are rounded
// independently from one value to the next and take two.
//
// Packed layout.  A matrix of `rows` rows and k columns is stored in chunks of
// 32 columns (zero past k): for each row and chunk 256 bytes, the planes re_h,
// re_l, im_h, im_l of the 32 columns, 64 bytes each; a third piece is kept
// beside it, 128 bytes per row and chunk (re_t, im_t).  A tile's chunk is
// copied to LDS by the memory pipe itself (global_load_lds, 16 bytes a lane, no
// registers and no store instructions).  The instruction writes a wave's 64
// pieces side by side, so the order within a row is chosen on the global side:
// the 16-byte piece j of tile row r comes to slot j ^ (r % 16), and the 16 rows
// that a fragment read touches at one j then lie in distinct banks.
#include <type_traits>

#include "pinv_internal.h"

namespace pinv {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void lds_void;
typedef const __attribute__((address_space(1))) void glb_void;

__device__ __forceinline__ f32x4 mfma_f16(f16x8 a, f16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// h and l pieces of x0 and x1, each pair in a 32-bit word (x0 in the low half).
__device__ __forceinline__ void split_h2(float x0, float x1, uint32_t& h, uint32_t& l) {
  const f16x2 hv{(_Float16)x0, (_Float16)x1};
  const f16x2 lv{(_Float16)(x0 - (float)hv[0]), (_Float16)(x1 - (float)hv[1])};
  h = __builtin_bit_cast(uint32_t, hv);
  l = __builtin_bit_cast(uint32_t, lv);
}

__device__ __forceinline__ void split_h2(double x0, double x1, uint32_t& h, uint32_t& l) {
  const f16x2 hv{(_Float16)(float)x0, (_Float16)(float)x1};
  const f16x2 lv{(_Float16)(float)(x0 - (double)hv[0]), (_Float16)(float)(x1 - (double)hv[1])};
  h = __builtin_bit_cast(uint32_t, hv);
  l = __builtin_bit_cast(uint32_t, lv);
}

// The power of two that brings a row whose largest |value| has the FP32 (FP64
// high word's) exponent field `e` into [2^13, 2^14).  Rows of zeros keep 1;
// rows that hold an infinity or a NaN stay non-finite at any scale.
__device__ __forceinline__ int row_shift(int e, int bias) { return e == 0 ? 0 : 13 + bias - e; }

// W^T is stored as 2^12 W: no entry of W exceeds 1 (W W^H = I - lam L^-1 L^-H).
constexpr int kWShift = 12;

// ---------------------------------------------------------------------------
// Tiles
// ---------------------------------------------------------------------------
// WGM x WGN wavefronts, each WTM x WTN of a BM x BN tile; PA pieces in operand
// A (rows), two in B (columns).  Two LDS stages: the next chunk is copied in
// while this one computes, one barrier per chunk.
template <int BM_, int BN_, int WGM_, int WGN_, int PA_> struct HalfCfg {
  static constexpr int BM = BM_, BN = BN_, WGM = WGM_, WGN = WGN_, PA = PA_;
  static constexpr int NW = WGM * WGN, NT = 64 * NW;
  static constexpr int WTM = BM / WGM, WTN = BN / WGN, MB = WTM / 16, NB = WTN / 16;
  static constexpr int A_BYTES = BM * 256, T_BYTES = PA == 3 ? BM * 128 : 0, B_BYTES = BN * 256;
  static constexpr int STAGE = A_BYTES + T_BYTES + B_BYTES;
  static_assert(A_BYTES % (1024 * NW) == 0 && T_BYTES % (1024 * NW) == 0 &&
                    B_BYTES % (1024 * NW) == 0 && (4 * NW) % 16 == 0,
                "whole wave-wide copies, their row mod 16 the same in every pass");
};

// Rows row0 .. of a packed matrix: `main` (256 bytes per row and chunk) and,
// with a third piece, `third` (128).  nc: chunks per row.  Rows past `last`
// are read as row `last` (their products are not stored).
struct HalfOperand {
  const char* main;
  const char* third;
  int nc, row0, last;
};

template <class C> struct HalfAcc { f32x4 re[C::MB][C::NB], im[C::MB][C::NB]; };

template <class C> struct HalfLoader {
  static constexpr int IA = C::A_BYTES / 1024 / C::NW, IT = C::T_BYTES / 1024 / C::NW,
                       IB = C::B_BYTES / 1024 / C::NW;
  const char *a, *t, *b;
  uint32_t oa[IA], ot[IT ? IT : 1], ob[IB];
  int w;
  __device__ __forceinline__ void init(const HalfOperand& A, const HalfOperand& B) {
    const int lane = threadIdx.x & 63;
    w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    a = A.main + (size_t)A.row0 * A.nc * 256;
    b = B.main + (size_t)B.row0 * B.nc * 256;
    t = C::PA == 3 ? A.third + (size_t)A.row0 * A.nc * 128 : nullptr;
    const int r4 = 4 * w + (lane >> 4);       // four rows of 16 pieces per copy
    const uint32_t j4 = ((lane & 15) ^ (r4 & 15)) * 16;
#pragma unroll
    for (int i = 0; i < IA; ++i)
      oa[i] = (uint32_t)min(r4 + 4 * C::NW * i, A.last - A.row0) * (uint32_t)A.nc * 256u + j4;
#pragma unroll
    for (int i = 0; i < IB; ++i)
      ob[i] = (uint32_t)min(r4 + 4 * C::NW * i, B.last - B.row0) * (uint32_t)B.nc * 256u + j4;
    if constexpr (C::PA == 3) {
      const int r8 = 8 * w + (lane >> 3);     // eight rows of 8 pieces
      const uint32_t j8 = ((lane & 7) ^ (r8 & 7)) * 16;
#pragma unroll
      for (int i = 0; i < IT; ++i)
        ot[i] = (uint32_t)min(r8 + 8 * C::NW * i, A.last - A.row0) * (uint32_t)A.nc * 128u + j8;
    }
  }
  __device__ __forceinline__ void load(char* s, int c) const {
    const char* pa = a + (size_t)c * 256;
    const char* pb = b + (size_t)c * 256;
#pragma unroll
    for (int i = 0; i < IA; ++i)
      __builtin_amdgcn_global_load_lds((glb_void*)(pa + oa[i]),
                                       (lds_void*)(s + (w + i * C::NW) * 1024), 16, 0, 0);
    if constexpr (C::PA == 3) {
      const char* pt = t + (size_t)c * 128;
#pragma unroll
      for (int i = 0; i < IT; ++i)
        __builtin_amdgcn_global_load_lds((glb_void*)(pt + ot[i]),
                                         (lds_void*)(s + C::A_BYTES + (w + i * C::NW) * 1024), 16, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < IB; ++i)
      __builtin_amdgcn_global_load_lds(
          (glb_void*)(pb + ob[i]),
          (lds_void*)(s + C::A_BYTES + C::T_BYTES + (w + i * C::NW) * 1024), 16, 0, 0);
  }
};

// One chunk from the stage `s`: lane l holds row l % 16 (of a block of A or B)
// and columns 8 (l / 16) .. + 8.
//
// The chunk's products are summed from zero and then added to the tile's
// accumulators, so the sums between FP32 roundings of the whole are 32 columns
// long.  The instruction aligns the products of a group of eight to the largest
// and cuts what falls below towards minus infinity when they meet a larger sum:
// a bias of one sign in every element, which adds up coherently over the samples of an
// apply.  So every second chunk of operand A is stored negated, and its sums are
// subtracted (SUB): the bias of one chunk cancels the next one's, at the same speed.  One
// 64 x 64 coil, M = 8192, E from FP32 tables: unrefined images 2.1e-3 off with the bias,
// 5.9e-4 without, FP32 instructions 1.75e-3; after one refinement step 1.0e-6, 3.8e-8,
// 3.8e-8.  Sums kept apart by their sign instead, ar br - ai bi, cost 12% of the
// products' time and left 7.6e-8.
template <class C, bool SUB>
__device__ __forceinline__ void half_compute(const char* s, HalfAcc<C>& acc) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const char* sa = s + (w / C::WGN) * C::WTM * 256 + lr * 256;
  const char* st = s + C::A_BYTES + (w / C::WGN) * C::WTM * 128 + lr * 128;
  const char* sb = s + C::A_BYTES + C::T_BYTES + (w % C::WGN) * C::WTN * 256 + lr * 256;
  f16x8 b[C::NB][4];
#pragma unroll
  for (int j = 0; j < C::NB; ++j)
#pragma unroll
    for (int p = 0; p < 4; ++p)
      b[j][p] = *reinterpret_cast<const f16x8*>(sb + j * 4096 + ((p * 4 + lk) ^ lr) * 16);
#pragma unroll
  for (int i = 0; i < C::MB; ++i) {
    f16x8 a[4];
#pragma unroll
    for (int p = 0; p < 4; ++p)
      a[p] = *reinterpret_cast<const f16x8*>(sa + i * 4096 + ((p * 4 + lk) ^ lr) * 16);
    const f16x8 nh = -a[2], nl = -a[3];
    f16x8 rt, it, nt;
    if constexpr (C::PA == 3) {
      rt = *reinterpret_cast<const f16x8*>(st + i * 2048 + (lk ^ (lr & 7)) * 16);
      it = *reinterpret_cast<const f16x8*>(st + i * 2048 + ((4 + lk) ^ (lr & 7)) * 16);
      nt = -it;
    }
    f32x4 re[C::NB], im[C::NB];   // this chunk's sums
#pragma unroll
    for (int j = 0; j < C::NB; ++j) {
      const f32x4 zero{0.f, 0.f, 0.f, 0.f};
      if constexpr (C::PA == 3) {
        re[j] = mfma_f16(rt, b[j][0], zero);
        im[j] = mfma_f16(rt, b[j][2], zero);
        re[j] = mfma_f16(nt, b[j][2], re[j]);
        im[j] = mfma_f16(it, b[j][0], im[j]);
        re[j] = mfma_f16(a[1], b[j][0], re[j]);
        im[j] = mfma_f16(a[1], b[j][2], im[j]);
      } else {
        re[j] = mfma_f16(a[1], b[j][0], zero);
        im[j] = mfma_f16(a[1], b[j][2], zero);
      }
    }
#pragma unroll
    for (int j = 0; j < C::NB; ++j) {
      re[j] = mfma_f16(nl, b[j][2], re[j]);
      im[j] = mfma_f16(a[3], b[j][0], im[j]);
      re[j] = mfma_f16(a[0], b[j][1], re[j]);
      im[j] = mfma_f16(a[0], b[j][3], im[j]);
      re[j] = mfma_f16(nh, b[j][3], re[j]);
      im[j] = mfma_f16(a[2], b[j][1], im[j]);
      re[j] = mfma_f16(a[0], b[j][0], re[j]);
      im[j] = mfma_f16(a[0], b[j][2], im[j]);
      re[j] = mfma_f16(nh, b[j][2], re[j]);
      im[j] = mfma_f16(a[2], b[j][0], im[j]);
    }
#pragma unroll
    for (int j = 0; j < C::NB; ++j) {
      acc.re[i][j] = SUB ? acc.re[i][j] - re[j] : acc.re[i][j] + re[j];
      acc.im[i][j] = SUB ? acc.im[i][j] - im[j] : acc.im[i][j] + im[j];
    }
  }
}

// The copies into `nxt` run under the products from `cur`.  The two are
// different stages; `__restrict__` lets the compiler order no read of one
// behind the copies into the other.
template <class C, bool SUB>
__device__ __forceinline__ void half_step(const HalfLoader<C>& ld, char* __restrict__ nxt, int c,
                                          const char* __restrict__ cur, HalfAcc<C>& acc) {
  ld.load(nxt, c);
  __builtin_amdgcn_sched_barrier(0);   // the copies first
  half_compute<C, SUB>(cur, acc);
}

// vmcnt(0): this wave's copies into LDS have landed; the barrier publishes
// them and retires every wave's reads of the stage the next copies overwrite.
__device__ __forceinline__ void half_publish() {
  __builtin_amdgcn_s_waitcnt(0x0f70);
  __syncthreads();
}

// acc = sum over chunks c0 .. c1 - 1 (at least one), from the top with DOWN; the
// second, fourth, ... chunk in that order is negated in A.
template <class C, bool DOWN>
__device__ __forceinline__ void half_mainloop(const HalfOperand& A, const HalfOperand& B, int c0,
                                              int c1, char* s0, char* s1, HalfAcc<C>& acc) {
#pragma unroll
  for (int i = 0; i < C::MB; ++i)
#pragma unroll
    for (int j = 0; j < C::NB; ++j) acc.re[i][j] = acc.im[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  HalfLoader<C> ld;
  ld.init(A, B);
  const int n = c1 - c0;
  auto at = [&](int k) { return DOWN ? c1 - 1 - min(k, n - 1) : c0 + min(k, n - 1); };
  ld.load(s0, at(0));
  half_publish();
  int k = 0;
  for (; k + 2 <= n; k += 2) {
    half_step<C, false>(ld, s1, at(k + 1), s0, acc);
    half_publish();
    half_step<C, true>(ld, s0, at(k + 2), s1, acc);   // the last pass copies a chunk it does not use
    half_publish();
  }
  if (k < n) half_compute<C, false>(s0, acc);
}

// ---------------------------------------------------------------------------
// The factor: row and column scales, and L^-1 and L^-H in three pieces
// ---------------------------------------------------------------------------
// row_e[n], col_e[n]: the largest exponent field of row and column n of the
// lower triangle (zeroed before).  One workgroup per 64 x 64 block.
__global__ __launch_bounds__(256) void k_factor_exps(const double* __restrict__ Li, int N,
                                                     int* __restrict__ row_e, int* __restrict__ col_e) {
  int bi, bj;
  tri_index(blockIdx.x, &bi, &bj);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const cx<double>* L = reinterpret_cast<const cx<double>*>(Li);
  __shared__ int cmax[4][64];
  const int col = bj * 64 + lane;
  int cm = 0;
#pragma unroll 4
  for (int q = 0; q < 16; ++q) {
    const int row = bi * 64 + w * 16 + q;
    int e = 0;
    if (row < N && col < N) {
      const cx<double> v = L[(size_t)row * N + col];
      const int hr = __double2hiint(v.re) & 0x7fffffff, hi = __double2hiint(v.im) & 0x7fffffff;
      e = max(hr, hi) >> 20;
    }
    cm = max(cm, e);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) e = max(e, __shfl_xor(e, off));
    if (lane == 0 && row < N) atomicMax(row_e + row, e);
  }
  cmax[w][lane] = cm;
  __syncthreads();
  if (w == 0 && col < N)
    atomicMax(col_e + col, max(max(cmax[0][lane], cmax[1][lane]), max(cmax[2][lane], cmax[3][lane])));
}

// Packed rows of L^-1 (TRANS false: row n, k = n' <= n) or L^-H (TRANS: row i,
// value conj(Li[k][i]), k >= i), 8 columns per thread.  Only the chunks that
// the products read are written: k up to, or from, the row's block of 128.  Odd
// chunks are negated, counted from k = 0 for L^-1 and from the end for L^-H, as
// the products visit them.
template <bool TRANS>
__global__ __launch_bounds__(256) void k_factor_pack(const double* __restrict__ Li, int N, int nc,
                                                     const int* __restrict__ e_max,
                                                     char* __restrict__ main, char* __restrict__ third) {
  const cx<double>* L = reinterpret_cast<const cx<double>*>(Li);
  const int64_t total = (int64_t)N * nc * 4;
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < total;
       u += (int64_t)gridDim.x * blockDim.x) {
    int r, g;   // row, 8-group: neighbours take one row's groups, or one group's rows
    if constexpr (TRANS) {
      g = (int)(u / N);
      r = (int)(u - (int64_t)g * N);
    } else {
      r = (int)(u / (nc * 4));
      g = (int)(u - (int64_t)r * (nc * 4));
    }
    const int blk = r / 128 * 128;
    if (TRANS ? 8 * g < blk : 8 * g >= blk + 128) continue;
    const int s = row_shift(e_max[r], 1023);
    const bool neg = ((TRANS ? nc - 1 - g / 4 : g / 4) & 1) != 0;
    f16x8 p[6];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = 8 * g + j;
      cx<double> v{0.0, 0.0};
      if (k < N) v = TRANS ? L[(size_t)k * N + r] : L[(size_t)r * N + k];
      const double x[2] = {ldexp(neg ? -v.re : v.re, s), ldexp(TRANS != neg ? -v.im : v.im, s)};
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const _Float16 h = (_Float16)x[c];
        const double r1 = x[c] - (double)h;
        const _Float16 l = (_Float16)r1;
        p[2 * c][j] = h;
        p[2 * c + 1][j] = l;
        p[4 + c][j] = (_Float16)(r1 - (double)l);
      }
    }
    char* m = main + ((size_t)r * nc + g / 4) * 256 + (g % 4) * 16;
    char* t = third + ((size_t)r * nc + g / 4) * 128 + (g % 4) * 16;
#pragma unroll
    for (int q = 0; q < 4; ++q) *reinterpret_cast<f16x8*>(m + q * 64) = p[q];
    *reinterpret_cast<f16x8*>(t) = p[4];
    *reinterpret_cast<f16x8*>(t + 64) = p[5];
  }
}

// ---------------------------------------------------------------------------
// conj(E), packed: rows m0 .. m0 + rows of samples, columns n, scaled by 2^es
// ---------------------------------------------------------------------------
// Workgroup b takes 64 rows and kGenChunksH chunks; thread t generates columns
// 8 (t % 4) .. + 8 of row t / 4 of each chunk, in FP64, so that the split is E's only
// rounding.  Four neighbouring lanes read 512 contiguous bytes of a row's table and write
// 64 of each plane: 620 us for N = 4096, M = 32768 (928 with a column group's rows side by
// side; 522 from FP32 tables, whose roundings come on top of the split's), 5.5 ms for N =
// 9216, M = 131072.
constexpr int kGenChunksH = 16;
struct GenHCfg { static constexpr int NT = 256, BK = 32; };

template <int FEAT, bool AL>
__global__ __launch_bounds__(256) void k_gen_e_h(EncDev<double> e, int m0, int rows, int nc, double scale,
                                                 char* __restrict__ Es) {
  const int nbc = (nc + kGenChunksH - 1) / kGenChunksH;
  const int r0 = (int)(blockIdx.x / nbc) * 64, cb = (int)(blockIdx.x % nbc);
  LoadGenRowSP<GenHCfg, 64, true, FEAT, AL, double, true> g;
  g.init(e, m0 + r0);
  const int o = threadIdx.x / 4, gq = (int)(threadIdx.x % 4);
  const bool live = r0 + o < rows;
  for (int c = 0; c < kGenChunksH; ++c) {
    const int ck = cb * kGenChunksH + c;
    if (ck >= nc) break;
    g.fetch(ck * 32, e.N);
    uint32_t pk[4][4];
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
      double re[2], im[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const cx<double> el = gen_product<FEAT>(g.raw[j + u]);
        re[u] = g.ok[j + u] ? el.re * scale : 0.0;
        im[u] = g.ok[j + u] ? -el.im * scale : 0.0;
      }
      split_h2(re[0], re[1], pk[0][j / 2], pk[1][j / 2]);
      split_h2(im[0], im[1], pk[2][j / 2], pk[3][j / 2]);
    }
    if (live) {
      char* d = Es + ((size_t)(r0 + o) * nc + ck) * 256 + gq * 16;
#pragma unroll
      for (int p = 0; p < 4; ++p)
        *reinterpret_cast<uint4*>(d + p * 64) = uint4{pk[p][0], pk[p][1], pk[p][2], pk[p][3]};
    }
  }
}

// ---------------------------------------------------------------------------
// W^T (packed, rows m, k = n) and R
// ---------------------------------------------------------------------------
// Bound by the f16 pipe and its power budget: at N = 16384, M = 262144 the two products
// take 880 and 876 ms, 1290 TFLOP/s of executed f16 products, with the pipe 0.67 busy at
// a shader clock of 1.84 GHz (counters; 2.2 GHz under the kernels around them) and no LDS
// bank conflicts; three real FP32 products per complex one took 2057 and 1969.  At N =
// 9216, M = 131072: 137 and 138 ms, 1310 TFLOP/s, where a plain bf16 library product of
// 16384^3 reaches 1330; 329 and 313 on FP32.  128 x 128 tiles over eight wavefronts fill
// the 160 KB of LDS with two stages of 80 KB; the LDS moves 344 KB a chunk (2700 cycles)
// against 4096 cycles of matrix products.
typedef HalfCfg<128, 128, 2, 4, 3> TrmmH;

__global__ __launch_bounds__(TrmmH::NT, 1) void k_trmm_wh(const char* __restrict__ Lm,
                                                          const char* __restrict__ Lt,
                                                          const int* __restrict__ row_e, int es,
                                                          const char* __restrict__ Es,
                                                          char* __restrict__ Wt, int N, int nc, int m0,
                                                          int rows) {
  typedef TrmmH C;
  __shared__ __attribute__((aligned(1024))) char s0[C::STAGE];
  __shared__ __attribute__((aligned(1024))) char s1[C::STAGE];
  const int nbi = (N + C::BM - 1) / C::BM, nbj = (rows + C::BN - 1) / C::BN;
  int r, bj;
  grouped_tile<8>(xcd_contiguous(blockIdx.x, nbi * nbj), nbi, nbj, &r, &bj);
  const int bi = nbi - 1 - r;   // longest ranges first
  HalfAcc<C> acc;
  half_mainloop<C, false>(HalfOperand{Lm, Lt, nc, bi * C::BM, N - 1},
                          HalfOperand{Es, nullptr, nc, bj * C::BN, rows - 1}, 0,
                          min(nc, (bi + 1) * (C::BM / 32)), s0, s1, acc);
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = w / C::WGN, wc = w % C::WGN;
#pragma unroll
  for (int i = 0; i < C::MB; ++i) {
    const int n = bi * C::BM + wr * C::WTM + i * 16 + 4 * (lane >> 4);   // four rows n .. n + 3
    if (n >= nc * 32) continue;
    int sh[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      sh[q] = n + q < N ? kWShift - es - row_shift(row_e[n + q], 1023) : 0;
#pragma unroll
    for (int j = 0; j < C::NB; ++j) {
      const int m = bj * C::BN + wc * C::WTN + j * 16 + (lane & 15);
      if (m >= rows) continue;
      float re[4], im[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {   // k past N is zero
        re[q] = n + q < N ? ldexpf(acc.re[i][j][q], sh[q]) : 0.f;
        im[q] = n + q < N ? ldexpf(acc.im[i][j][q], sh[q]) : 0.f;
      }
      uint2 o[4];
      split_h2(re[0], re[1], o[0].x, o[1].x);
      split_h2(re[2], re[3], o[0].y, o[1].y);
      split_h2(im[0], im[1], o[2].x, o[3].x);
      split_h2(im[2], im[3], o[2].y, o[3].y);
      char* d = Wt + ((size_t)(m0 + m) * nc + n / 32) * 256 + (n % 32) * 2;
#pragma unroll
      for (int p = 0; p < 4; ++p) *reinterpret_cast<uint2*>(d + p * 64) = o[p];
    }
  }
}

__global__ __launch_bounds__(TrmmH::NT, 1) void k_trmm_rh(const char* __restrict__ Hm,
                                                          const char* __restrict__ Ht,
                                                          const int* __restrict__ col_e,
                                                          const char* __restrict__ Wt,
                                                          float* __restrict__ R, int N, int M, int nc) {
  typedef TrmmH C;
  __shared__ __attribute__((aligned(1024))) char s0[C::STAGE];
  __shared__ __attribute__((aligned(1024))) char s1[C::STAGE];
  const int nbi = (N + C::BM - 1) / C::BM, nbj = (M + C::BN - 1) / C::BN;
  int bi, bj;
  grouped_tile<8>(xcd_contiguous(blockIdx.x, nbi * nbj), nbi, nbj, &bi, &bj);
  HalfAcc<C> acc;
  half_mainloop<C, true>(HalfOperand{Hm, Ht, nc, bi * C::BM, N - 1},
                         HalfOperand{Wt, nullptr, nc, bj * C::BN, M - 1}, bi * (C::BM / 32), nc, s0,
                         s1, acc);
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = w / C::WGN, wc = w % C::WGN;
  cx<float>* O = reinterpret_cast<cx<float>*>(R);
#pragma unroll
  for (int i = 0; i < C::MB; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int n = bi * C::BM + wr * C::WTM + i * 16 + 4 * (lane >> 4) + q;
      if (n >= N) continue;
      const int sh = -kWShift - row_shift(col_e[n], 1023);
#pragma unroll
      for (int j = 0; j < C::NB; ++j) {
        const int m = bj * C::BN + wc * C::WTN + j * 16 + (lane & 15);
        if (m < M)
          O[(size_t)n * M + m] = cx<float>{ldexpf(acc.re[i][j][q], sh), ldexpf(acc.im[i][j][q], sh)};
      }
    }
}

// ---------------------------------------------------------------------------
// Apply: X[f][n] = sum_m D[f][m] R[n][m] for more frames than the streamed apply
// takes
// ---------------------------------------------------------------------------
// The contraction is cut into segments of at most kHalfSegCols columns, each with
// row scales of its own, so a running FP32 sum covers one segment.  A slab of
// segments of R and of the data is packed into scratch, multiplied (one tile grid
// per segment) and its segments' partial images are added into X.  A slab is at
// most kHalfApplyBytes, which the 256 MB memory-side cache holds between the pass
// that writes it and the product that reads it.
constexpr int kHalfSegCols = 4096;
constexpr size_t kHalfApplyBytes = 256ull << 20;
constexpr int kHalfFrames = 2048;   // frames per pass over R

// Rows r of `src` (complex64, ld columns a row), columns c0 + seg_len g .. of
// segment g (zero at and past `cols`): dst[g][r][chunk], and the power of two that
// scales the row in exps[g][r].  NEG: odd chunks negated (operand A of the
// tiles).  One workgroup per row and segment, a pair of columns per thread and
// step.
template <int VEC, bool NEG>
__global__ __launch_bounds__(256) void k_pack_half(const float* __restrict__ src, int64_t ld, int rows,
                                                   int64_t c0, int64_t cols, int seg_len,
                                                   char* __restrict__ dst, int* __restrict__ exps) {
  constexpr int STEPS = kHalfSegCols / 512;
  const int r = (int)(blockIdx.x % rows), g = (int)(blockIdx.x / rows);
  const cx<float>* z = reinterpret_cast<const cx<float>*>(src) + (int64_t)r * ld + c0 + (int64_t)g * seg_len;
  const int64_t left = cols - c0 - (int64_t)g * seg_len;
  const int live = (int)(left < seg_len ? left : seg_len);
  float4 v[STEPS];
  int e = 0;
#pragma unroll
  for (int i = 0; i < STEPS; ++i) {
    const int k = 2 * (threadIdx.x + 256 * i);
    v[i] = float4{0.f, 0.f, 0.f, 0.f};
    if (VEC == 2) {   // an even number of columns, 16-byte aligned rows and segments
      if (k < live) v[i] = *reinterpret_cast<const float4*>(z + k);
    } else {
      if (k < live) v[i].x = z[k].re, v[i].y = z[k].im;
      if (k + 1 < live) v[i].z = z[k + 1].re, v[i].w = z[k + 1].im;
    }
#pragma unroll
    for (const float x : {v[i].x, v[i].y, v[i].z, v[i].w})
      e = max(e, (__float_as_int(x) & 0x7fffffff) >> 23);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) e = max(e, __shfl_xor(e, off));
  __shared__ int we[4];
  if ((threadIdx.x & 63) == 0) we[threadIdx.x >> 6] = e;
  __syncthreads();
  const int s = row_shift(max(max(we[0], we[1]), max(we[2], we[3])), 127);
  if (threadIdx.x == 0) exps[(size_t)g * rows + r] = s;
  char* d = dst + ((size_t)g * rows + r) * (seg_len / 32) * 256;
#pragma unroll
  for (int i = 0; i < STEPS; ++i) {
    const int k = 2 * (threadIdx.x + 256 * i);
    if (k >= seg_len) break;
    uint32_t o[4];
    split_h2(ldexpf(v[i].x, s), ldexpf(v[i].z, s), o[0], o[1]);
    split_h2(ldexpf(v[i].y, s), ldexpf(v[i].w, s), o[2], o[3]);
    const uint32_t sign = NEG && (k / 32 & 1) ? 0x80008000u : 0u;
#pragma unroll
    for (int p = 0; p < 4; ++p)
      *reinterpret_cast<uint32_t*>(d + (k / 32) * 256 + p * 64 + (k % 32) * 2) = o[p] ^ sign;
  }
}

// Tiles of BM frames x BN unknowns, one grid of `tiles` per segment.  With
// `work` the partial image of segment g goes to work[g][F][N]; else to X (added
// to what is there with `add`).
template <class C>
__global__ __launch_bounds__(C::NT, 1) void k_apply_half(const char* __restrict__ Dp,
                                                         const int* __restrict__ de,
                                                         const char* __restrict__ Rp,
                                                         const int* __restrict__ re, int F, int N, int nc,
                                                         int64_t cols, int tiles, float* __restrict__ X,
                                                         float* __restrict__ work, int add) {
  __shared__ __attribute__((aligned(1024))) char s0[C::STAGE];
  __shared__ __attribute__((aligned(1024))) char s1[C::STAGE];
  const int u = xcd_contiguous(blockIdx.x, gridDim.x);
  const int g = u / tiles, t = u - g * tiles;
  const int nbi = (F + C::BM - 1) / C::BM;
  const int bi = t % nbi, bj = t / nbi;
  const int64_t left = cols - (int64_t)g * nc * 32;   // the last segment may be short
  const int n = (int)min((int64_t)nc, (left + 31) / 32);
  HalfAcc<C> acc;
  half_mainloop<C, false>(HalfOperand{Dp + (size_t)g * F * nc * 256, nullptr, nc, bi * C::BM, F - 1},
                          HalfOperand{Rp + (size_t)g * N * nc * 256, nullptr, nc, bj * C::BN, N - 1}, 0, n,
                          s0, s1, acc);
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = w / C::WGN, wc = w % C::WGN;
  cx<float>* O = reinterpret_cast<cx<float>*>(work ? work + (size_t)g * F * N * 2 : X);
#pragma unroll
  for (int j = 0; j < C::NB; ++j) {
    const int col = bj * C::BN + wc * C::WTN + j * 16 + (lane & 15);
    if (col >= N) continue;
    const int sr = re[(size_t)g * N + col];
#pragma unroll
    for (int i = 0; i < C::MB; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int f = bi * C::BM + wr * C::WTM + i * 16 + 4 * (lane >> 4) + q;
        if (f >= F) continue;
        const int sh = -sr - de[(size_t)g * F + f];
        cx<float> x{ldexpf(acc.re[i][j][q], sh), ldexpf(acc.im[i][j][q], sh)};
        cx<float>* o = O + (size_t)f * N + col;
        if (add) {
          const cx<float> old = *o;
          x.re += old.re;
          x.im += old.im;
        }
        *o = x;
      }
  }
}

// X = (add ? X : 0) + sum_g work[g] in segment order, in FP64, rounded once.
__global__ __launch_bounds__(256) void k_half_reduce(const float* __restrict__ work, int segs, int64_t n,
                                                     float* __restrict__ X, int add) {
  const cx<float>* w = reinterpret_cast<const cx<float>*>(work);
  cx<float>* x = reinterpret_cast<cx<float>*>(X);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    double re = add ? x[i].re : 0.0, im = add ? x[i].im : 0.0;
    for (int g = 0; g < segs; ++g) {
      re += w[(int64_t)g * n + i].re;
      im += w[(int64_t)g * n + i].im;
    }
    x[i] = cx<float>{(float)re, (float)im};
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// Tiles of 128 frames x 128 unknowns, or of 64 x 256 where they leave less of the
// last frame tile empty or fill the CUs better.  1000 frames at N = 4096, M = 65536:
// 5.2 ms of products (410 TFLOP/s of complex products, 1240 executed; the power
// budget again) and 1.0 ms of packing, where the FP32 tiles took 15.6 (18.8 in
// segments); 300 frames 2.7 ms against 5.9 (7.1).  At 33 to 64 frames the packing
// (R read and written once) is most of the 1.5 ms, against 2.0 (2.4).
typedef HalfCfg<128, 128, 2, 4, 2> ApplyH128;
typedef HalfCfg<64, 256, 1, 8, 2> ApplyH64;

// Segments, slabs and tiles of an apply: a function of F, N and M only.
struct HalfApply {
  int frames;     // frames per pass
  bool wide;      // tiles of 128 frames (else 64)
  int seg_len, nseg, slab;   // columns per segment, segments, segments per slab
  size_t r_bytes, d_bytes, e_bytes, w_bytes;
  size_t bytes() const { return r_bytes + d_bytes + e_bytes + w_bytes; }
};

static HalfApply half_apply_plan(int F, int N, int M) {
  HalfApply best{};
  double best_cost = 1e300;
  const int64_t fr = std::min(F, kHalfFrames);
  for (int wide = 0; wide < 2; ++wide) {
    const int64_t tiles = (int64_t)cdiv(fr, wide ? 128 : 64) * cdiv(N, wide ? 128 : 256);
    for (int len = kHalfSegCols; len >= 256; len /= 2) {
      const int nseg = cdiv(M, len);
      const int sl = cdiv(cdiv(M, nseg), 32) * 32;
      const size_t per = (size_t)(N + fr) * sl * 8 + (size_t)(N + fr) * 4;
      const size_t part = (size_t)fr * N * 8;
      int64_t slab = std::min<int64_t>(nseg, (int64_t)(kHalfApplyBytes / (per + part)));
      if (slab < 1) slab = per <= kHalfApplyBytes ? 1 : 0;
      for (; slab >= 1; slab = slab > 1 ? slab / 2 : 0) {
        // rounds of the tile grid over the 256 CUs, in chunks, with a fixed part
        // for the tile's start and end; a tile of 64 frames takes 0.55 of one of 128
        const int nslab = cdiv(nseg, slab);
        const double cost = (double)nslab * (((int64_t)tiles * slab + 255) / 256) *
                            ((sl / 32) * (wide ? 1.0 : 1.1) + 6.0) + 4.0 * nslab;
        if (cost < best_cost * 0.999) {
          best_cost = cost;
          best.frames = (int)fr;
          best.wide = wide;
          best.seg_len = sl;
          best.nseg = cdiv(M, sl);
          best.slab = (int)slab;
          auto al = [](size_t n) { return (n + 255) & ~size_t(255); };
          best.r_bytes = al((size_t)N * sl * 8 * slab);
          best.d_bytes = al((size_t)fr * sl * 8 * slab);
          best.e_bytes = al((size_t)(N + fr) * 4 * slab);
          best.w_bytes = slab > 1 ? al(part * slab) : 0;
        }
      }
    }
  }
  return best;
}

hipError_t launch_apply_half(const float* R, const float* D, float* X, int N, int M, int F, Scratch& sc,
                             hipStream_t s) {
  if (F <= 0 || N <= 0) return hipSuccess;
  const HalfApply p = half_apply_plan(F, N, M);
  if (p.slab < 1) return hipErrorInvalidValue;
  void* ws = nullptr;
  hipError_t err = sc.get(&ws, p.bytes(), s);
  if (err != hipSuccess) return err;
  char* rp = (char*)ws;
  char* dp = rp + p.r_bytes;
  int* re = (int*)(dp + p.d_bytes);
  int* de = re + (size_t)N * p.slab;
  float* work = p.w_bytes ? (float*)(dp + p.d_bytes + p.e_bytes) : nullptr;
  const bool vec = M % 2 == 0 && ((uintptr_t)R % 16) == 0 && ((uintptr_t)D % 16) == 0;
  auto pack = [&](auto neg, const float* src, int rows, int64_t c0, int segs, char* dst, int* exps) {
    constexpr bool NEG = decltype(neg)::value;
    const dim3 grid((unsigned)((int64_t)rows * segs)), block(256);
    if (vec)
      hipLaunchKernelGGL((k_pack_half<2, NEG>), grid, block, 0, s, src, (int64_t)M, rows, c0, (int64_t)M,
                         p.seg_len, dst, exps);
    else
      hipLaunchKernelGGL((k_pack_half<1, NEG>), grid, block, 0, s, src, (int64_t)M, rows, c0, (int64_t)M,
                         p.seg_len, dst, exps);
    return hipGetLastError();
  };
  for (int f0 = 0; f0 < F && err == hipSuccess; f0 += p.frames) {
    const int f = std::min(p.frames, F - f0);
    const float* d = D + 2 * (size_t)f0 * M;
    float* x = X + 2 * (size_t)f0 * N;
    const int tiles = cdiv(f, p.wide ? 128 : 64) * cdiv(N, p.wide ? 128 : 256);
    for (int g0 = 0; g0 < p.nseg && err == hipSuccess; g0 += p.slab) {
      const int segs = std::min(p.slab, p.nseg - g0);
      const int64_t c0 = (int64_t)g0 * p.seg_len;
      const int add = g0 > 0;
      if ((err = pack(std::true_type{}, d, f, c0, segs, dp, de)) != hipSuccess) break;
      if ((err = pack(std::false_type{}, R, N, c0, segs, rp, re)) != hipSuccess) break;
      auto tile = [&](auto cfg) {
        typedef decltype(cfg) C;
        hipLaunchKernelGGL(k_apply_half<C>, dim3((unsigned)(tiles * segs)), dim3(C::NT), 0, s,
                           (const char*)dp, (const int*)de, (const char*)rp, (const int*)re, f, N,
                           p.seg_len / 32, (int64_t)M - c0, tiles, x, work, work ? 0 : add);
        return hipGetLastError();
      };
      err = p.wide ? tile(ApplyH128{}) : tile(ApplyH64{});
      if (err == hipSuccess && work) {
        const int64_t n = (int64_t)f * N;
        hipLaunchKernelGGL(k_half_reduce, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 8192)), dim3(256),
                           0, s, (const float*)work, segs, n, x, add);
        err = hipGetLastError();
      }
    }
  }
  const hipError_t ferr = sc.put(ws, s);
  return err != hipSuccess ? err : ferr;
}

static int grid_1d(int64_t n, int most) {
  return (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, most));
}

size_t half_factor_bytes(int64_t N) {
  return (size_t)(N * (half_cols(N) / 32) * 384 + ((2 * N * 4 + 255) & ~int64_t(255)));
}

static hipError_t pack_factor(const double* Li, int N, bool trans, const int* e, char* main,
                              char* third, hipStream_t s) {
  const int nc = (int)(half_cols(N) / 32);
  const int grid = grid_1d((int64_t)N * nc * 4, 16384);
  if (trans)
    hipLaunchKernelGGL(k_factor_pack<true>, dim3(grid), dim3(256), 0, s, Li, N, nc, e, main, third);
  else
    hipLaunchKernelGGL(k_factor_pack<false>, dim3(grid), dim3(256), 0, s, Li, N, nc, e, main, third);
  return hipGetLastError();
}

hipError_t launch_trmm_wh(const EncDev<double>& e, const double* Li, void* factor, void* Es,
                          int64_t slab_rows, int es, void* Wt, hipStream_t s) {
  const int N = e.N, M = e.M;
  if (N <= 0 || M <= 0) return hipSuccess;
  if (slab_rows <= 0) return hipErrorInvalidValue;
  const int nc = (int)(half_cols(N) / 32);
  char* main = (char*)factor;
  char* third = main + (size_t)N * nc * 256;
  int* row_e = (int*)(third + (size_t)N * nc * 128);
  hipError_t err = hipMemsetAsync(row_e, 0, 2 * (size_t)N * 4, s);
  if (err != hipSuccess) return err;
  const int nb = cdiv(N, 64);
  hipLaunchKernelGGL(k_factor_exps, dim3((unsigned)((int64_t)nb * (nb + 1) / 2)), dim3(256), 0, s, Li,
                     N, row_e, row_e + N);
  if ((err = hipGetLastError()) != hipSuccess) return err;
  if ((err = pack_factor(Li, N, false, row_e, main, third, s)) != hipSuccess) return err;
  const int nbc = cdiv(nc, kGenChunksH);
  const double scale = ldexp(1.0, es);
  for (int64_t m0 = 0; m0 < M; m0 += slab_rows) {
    const int rows = (int)std::min<int64_t>(slab_rows, M - m0);
    err = with_feat_al(enc_features(e), row_aligned(e, 32), [&](auto fc, auto al) {
      hipLaunchKernelGGL((k_gen_e_h<decltype(fc)::value, decltype(al)::value>),
                         dim3((unsigned)(cdiv(rows, 64) * nbc)), dim3(256), 0, s, e, (int)m0, rows, nc,
                         scale, (char*)Es);
      return hipGetLastError();
    });
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(k_trmm_wh, dim3((unsigned)(cdiv(N, TrmmH::BM) * cdiv(rows, TrmmH::BN))),
                       dim3(TrmmH::NT), 0, s, (const char*)main, (const char*)third,
                       (const int*)row_e, es, (const char*)Es, (char*)Wt, N, nc, (int)m0, rows);
    if ((err = hipGetLastError()) != hipSuccess) return err;
  }
  return hipSuccess;
}

hipError_t launch_trmm_rh(const double* Li, void* factor, const void* Wt, float* R, int N, int M,
                          hipStream_t s) {
  if (N <= 0 || M <= 0) return hipSuccess;
  const int nc = (int)(half_cols(N) / 32);
  char* main = (char*)factor;
  char* third = main + (size_t)N * nc * 256;
  const int* col_e = (const int*)(third + (size_t)N * nc * 128) + N;
  hipError_t err = pack_factor(Li, N, true, col_e, main, third, s);
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(k_trmm_rh, dim3((unsigned)(cdiv(N, TrmmH::BM) * cdiv(M, TrmmH::BN))),
                     dim3(TrmmH::NT), 0, s, (const char*)main, (const char*)third, col_e,
                     (const char*)Wt, R, N, M, nc);
  return hipGetLastError();
}

}  // namespace pinv
