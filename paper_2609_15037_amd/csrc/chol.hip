// Blocked Cholesky factorisation and triangular inverse of the fp64 Gram
// matrices of a refresh batch (CholeskyQR: Z = Q R with R^T R = Z^T Z, then
// Q = Z R^{-1}). 64 x 64 blocks; every launch covers all matrices of the batch:
//   block row 0:   diag      factor C_00 = R_00^T R_00 and invert R_00 (one WG per matrix)
//   block row k:   row(k)    apply R's factored rows to C, right- or left-looking (one WG per block, k >= 1);
//                            the WG of the diagonal block (k, k) then factors C_kk and inverts
//                            R_kk while the launch's other WGs still run
//                  panel(k)  R_kc = R_kk^{-T} C_kc for c > k           (one WG per block)
//   then X = R^{-1} by recursive doubling over the blocks (k_trtri).
// A pivot not above 1e-13 * max(diag C) marks a numerically dependent column (a
// rank-deficient iterate): its row of R and its row and column of X = R^{-1} are set to
// zero, which is the Cholesky factor and inverse of the independent columns alone, so
// Q = Z X has orthonormal independent columns and zero dependent ones (raising such a
// pivot to a floor instead leaves chains of 1 / sqrt(floor) factors in R^{-1} that
// overflow its fp32 copy). An all-zero Gram gives R = I.
#include <algorithm>

#include "refresh.h"

namespace {

constexpr int NB = 64;
constexpr int LDB = NB + 1;

__device__ __forceinline__ int find_pref(const uint32_t* pref, int n, uint32_t t) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (pref[mid] <= t) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__device__ __forceinline__ int nblk(int w) { return (w + NB - 1) / NB; }
__device__ __forceinline__ int bsz(int w, int b) { return min(NB, w - b * NB); }

// load a kb_r x kb_c block (zero padded to 64 x 64) of a w x w row-major matrix into LDS
__device__ __forceinline__ void load_blk(double (*dst)[LDB], const double* M, int w, int br, int bc) {
  const int r0 = br * NB, c0 = bc * NB;
  for (int e = threadIdx.x; e < NB * NB; e += 256) {
    const int i = e >> 6, j = e & 63;
    dst[i][j] = (r0 + i < w && c0 + j < w) ? M[(int64_t)(r0 + i) * w + c0 + j] : 0.0;
  }
}

// fp64 MFMA form of the 64 x 64 block products (v_mfma_f64_16x16x4: lane l supplies
// A[l%16][l/16] and B[l/16][l%16] and receives D[4r + l/16][l%16] in register r).
// Wave w accumulates rows [16w, 16w+16) of the product, all 64 columns (four 16 x 16
// tiles): acc[jt] += op(A)[rows][t] * B[t][16 jt ..], op(A) = A^T when TA.
typedef double f64x4 __attribute__((ext_vector_type(4)));
template <bool TA>
__device__ __forceinline__ void mfma_blk(const double (*A)[LDB], const double (*Bm)[LDB], f64x4 (&acc)[4]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = 16 * wave + (lane & 15);
#pragma unroll 4
  for (int ks = 0; ks < NB / 4; ++ks) {
    const int t = 4 * ks + (lane >> 4);
    const double a = TA ? A[t][i] : A[i][t];
#pragma unroll
    for (int jt = 0; jt < 4; ++jt)
      acc[jt] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Bm[t][16 * jt + (lane & 15)], acc[jt], 0, 0, 0);
  }
}
// element (row, col) of the 64 x 64 block held in acc[jt][r]
__device__ __forceinline__ int mfma_row(int r) { return 16 * (threadIdx.x >> 6) + 4 * r + ((threadIdx.x & 63) >> 4); }
__device__ __forceinline__ int mfma_col(int jt) { return 16 * jt + (threadIdx.x & 15); }

// Factorisation of one 64 x 64 diagonal block and inverse of its factor by a workgroup of
// four waves, in 16 x 16 sub-blocks. What bounds it is the chain of 64 pivots (a reciprocal
// square root, then the next pivot's update), so only the 16 x 16 diagonal sub-blocks are
// worked entry by entry, by one wave in registers (16 values per lane, pivots and rows
// broadcast by v_readlane); everything between them is 16 x 16 x 16 products on fp64 MFMA.
// Measured against the whole 64 x 64 block in one wave's registers (64 values per lane, rows
// broadcast through LDS): a launch that factors one block 28 us instead of 74 (d = 256 layer),
// the left-looking k_chol_row over a Llama-2-7B-shaped layer 90 us on average instead of 151, its refresh 311
// ms instead of 353 (four 300M-shaped layers 50.9 instead of 60.7, d = 256 10.5 instead of 13.4).
constexpr int SB = 16, LDX = SB + 1;
struct DiagLds {
  double D[NB][LDB];        // the block; then R in its upper part and, in the strictly lower
                            // sub-blocks (j, i), the sub-blocks X_ij (i < j) of X = R^{-1}
  double Xd[4][SB][LDX];    // X_kk of the diagonal sub-blocks
};

// a lane's double as a wave-uniform value (the source lane is a compile-time constant)
__device__ __forceinline__ double lane_d(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}

// An empty asm on a value keeps the compiler from deferring the updates before it to their
// last use and from carrying the 120 row broadcasts and the lane masks of one loop into the
// next: both spill.
__device__ __forceinline__ void pin(double& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// One wave: factor the 16 x 16 sub-block (k, k) in place (R_kk, zero below its diagonal) and
// write its inverse. Lane l works on column l % 16 (the four quarters of the wave alike).
//   column j: R_jj = sqrt(D_jj) (0 for a dependent column), R_jc = D_jc / R_jj (c > j),
//             D_ac -= R_ja R_jc for a > j
//   inverse from the last row up: a_ic = sum_{t > i} R_it X_tc, X_cc = 1 / R_cc,
//             X_ic = -a_ic / R_ii (i < c); a zero R_ii gives a zero row of X.
__device__ __forceinline__ void factor16(DiagLds& S, int k, double floor_piv) {
  const int lane = threadIdx.x & 63, c = lane & 15;
  double col[SB], ri[SB];
#pragma unroll
  for (int i = 0; i < SB; ++i) col[i] = S.D[SB * k + i][SB * k + c];
#pragma unroll
  for (int j = 0; j < SB; ++j) {
    const double v = lane_d(col[j], j);
    const bool dep = !(v > floor_piv);
    double root, rinv;
    sqrt_rsqrt(dep ? 1.0 : v, root, rinv);
    root = dep ? 0.0 : root;
    rinv = dep ? 0.0 : rinv;
    ri[j] = rinv;
    const int cj = fresh(c);
    const double rjc = cj == j ? root : (cj > j ? col[j] * rinv : 0.0);
    col[j] = rjc;
#pragma unroll
    for (int a = j + 1; a < SB; ++a) pin(col[a] = fma(-lane_d(rjc, a), rjc, col[a]));
  }
  double x[SB];
#pragma unroll
  for (int i = 0; i < SB; ++i) {
    pin(col[i]);
    x[i] = 0.0;
  }
#pragma unroll
  for (int t = SB - 1; t >= 0; --t) {
    const int ct = fresh(c);
    x[t] = ct >= t ? ((ct == t ? 1.0 : 0.0) - x[t]) * ri[t] : 0.0;
#pragma unroll
    for (int i = 0; i < t; ++i) pin(x[i] = fma(lane_d(col[i], t), x[t], x[i]));
  }
  if (lane < SB) {
#pragma unroll
    for (int i = 0; i < SB; ++i) {
      S.D[SB * k + i][SB * k + c] = col[i];
      S.Xd[k][i][c] = x[i];
    }
  }
}

// acc += op(A) B on 16 x 16 sub-blocks (v_mfma_f64_16x16x4): fa(i, t) = op(A)[i][t] and
// fb(ks) = this lane's B operand of rows 4 ks .. 4 ks + 3. Register r of acc holds row
// 4 r + l / 16, column l % 16, which is the B operand of ks = r: products chain through
// registers.
template <class FA, class FB>
__device__ __forceinline__ void prod16(f64x4& acc, FA fa, FB fb) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(fa(lane & 15, 4 * ks + (lane >> 4)), fb(ks), acc, 0, 0, 0);
}

// LDS accesses of one wave complete in program order: keep the compiler's order too
__device__ __forceinline__ void wave_lds_order() { asm volatile("" ::: "memory"); }

// S.D holds the updated block (identity in the padding of a ragged block; the identity as a
// whole for an all-zero Gram, which gives R_kk = X_kk = I). Called by all 256 threads after a
// barrier; writes R_kk, X_kk and the fp32 copy of X_kk.
__device__ __forceinline__ void diag_factor(DiagLds& S, int kb, double floor_piv, const RefDev& d, int r0) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lr = lane >> 4, lc = lane & 15;
  const f64x4 zero = f64x4{0.0, 0.0, 0.0, 0.0};
  if (wave == 0) factor16(S, 0, floor_piv);
#pragma unroll 1
  for (int k = 0; k < 3; ++k) {
    __syncthreads();
    if (wave < 3 - k) {   // row k of R: R_kj = X_kk^T D_kj
      const int j = k + 1 + wave;
      f64x4 acc = zero;
      prod16(acc, [&](int i, int t) { return S.Xd[k][t][i]; },
             [&](int ks) { return S.D[SB * k + 4 * ks + lr][SB * j + lc]; });
#pragma unroll
      for (int r = 0; r < 4; ++r) S.D[SB * k + 4 * r + lr][SB * j + lc] = acc[r];
    }
    __syncthreads();
    // D_ij -= R_ki^T R_kj for k < i <= j: the next diagonal sub-block by wave 0, which then
    // factors it while the other waves update the rest
    int q = 0;
    for (int i = k + 1; i < 4; ++i)
      for (int j = i; j < 4; ++j, ++q) {
        if ((q == 0 ? 0 : 1 + (q - 1) % 3) != wave) continue;
        f64x4 acc = zero;
        prod16(acc, [&](int a, int t) { return S.D[SB * k + t][SB * i + a]; },
               [&](int ks) { return S.D[SB * k + 4 * ks + lr][SB * j + lc]; });
#pragma unroll
        for (int r = 0; r < 4; ++r) S.D[SB * i + 4 * r + lr][SB * j + lc] -= acc[r];
      }
    if (wave == 0) {
      wave_lds_order();
      factor16(S, k + 1, floor_piv);
    }
  }
  __syncthreads();
  // X by doubling: X_01 = -X_00 (R_01 X_11) and X_23 likewise, then the 2 x 2 sub-blocks
  // X_ij = -sum_{u = i, 1} X_iu T_uj, T_uj = sum_{t = 2 .. j} R_ut X_tj (i < 2 <= j)
  auto X = [&](int i, int j, int a, int b) { return i == j ? S.Xd[i][a][b] : S.D[SB * j + a][SB * i + b]; };
  auto R = [&](int i, int j, int a, int b) { return S.D[SB * i + a][SB * j + b]; };
  auto put = [&](int i, int j, const f64x4& acc) {
#pragma unroll
    for (int r = 0; r < 4; ++r) S.D[SB * j + 4 * r + lr][SB * i + lc] = -acc[r];
  };
  if (wave < 2) {
    const int i = 2 * wave, j = i + 1;
    f64x4 T = zero, acc = zero;
    prod16(T, [&](int a, int t) { return R(i, j, a, t); }, [&](int ks) { return X(j, j, 4 * ks + lr, lc); });
    prod16(acc, [&](int a, int t) { return X(i, i, a, t); }, [&](int ks) { return T[ks]; });
    put(i, j, acc);
  }
  __syncthreads();
  {
    const int i = wave >> 1, j = 2 + (wave & 1);
    f64x4 acc = zero;
    for (int u = i; u < 2; ++u) {
      f64x4 T = zero;
      for (int t = 2; t <= j; ++t)
        prod16(T, [&](int a, int b) { return R(u, t, a, b); }, [&](int ks) { return X(t, j, 4 * ks + lr, lc); });
      prod16(acc, [&](int a, int b) { return X(i, u, a, b); }, [&](int ks) { return T[ks]; });
    }
    put(i, j, acc);   // sub-blocks (j, i): read by nobody before the barrier
  }
  __syncthreads();
  const int w = d.w;
  for (int e = threadIdx.x; e < NB * NB; e += 256) {
    const int i = e >> 6, j = e & 63, bi = i >> 4, bj = j >> 4;
    if (i >= kb || j >= kb) continue;
    const int64_t g = (int64_t)(r0 + i) * w + r0 + j;
    const double x = bi > bj ? 0.0 : X(bi, bj, i & 15, j & 15);
    d.C[g] = bi > bj ? 0.0 : S.D[i][j];
    d.X[g] = x;
    d.Rinv[g] = (float)x;
  }
}

// Block 0 (no update before it): one workgroup per matrix; also records the pivot floor's
// reference, the largest diagonal entry of the untouched Gram.
__global__ __launch_bounds__(256) void k_chol_diag(const RefDev* __restrict__ ds) {
  __shared__ DiagLds S;
  const RefDev& d = ds[blockIdx.x];
  const int w = d.w;
  const int tid = threadIdx.x;
  const int kb = bsz(w, 0);
  double mx = 0.0;
  for (int i = tid; i < w; i += 256) mx = fmax(mx, d.C[(int64_t)i * w + i]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
  double* red = &S.Xd[0][0][0];   // free until the factorisation
  if ((tid & 63) == 0) red[tid >> 6] = mx;
  __syncthreads();
  mx = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
  if (tid == 0) d.cmax[0] = mx;
  for (int e = tid; e < NB * NB; e += 256) {
    const int i = e >> 6, j = e & 63;
    S.D[i][j] = (mx > 0.0 && i < kb && j < kb) ? d.C[(int64_t)i * w + j] : (i == j ? 1.0 : 0.0);
  }
  __syncthreads();
  diag_factor(S, kb, mx * 1e-13, d, 0);
}

__global__ __launch_bounds__(256, 4) void k_chol_panel(const RefDev* __restrict__ ds, const uint32_t* __restrict__ pref,
                                                       int n, int k) {
  const uint32_t t = blockIdx.x;
  const int mi = find_pref(pref, n, t);
  const RefDev& d = ds[mi];
  const int w = d.w;
  const int j = k + 1 + (int)(t - pref[mi]);
  // R_kj = X_kk^T C_kj: C_kj in LDS, each wave's 16 columns of X_kk straight into its MFMA
  // operand registers (A[i][t] = X_kk[t][16 w + i])
  __shared__ double Cb[NB][LDB];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double av[NB / 4];
  {
    const int col = k * NB + 16 * wave + (lane & 15);
#pragma unroll
    for (int ks = 0; ks < NB / 4; ++ks) {
      const int row = k * NB + 4 * ks + (lane >> 4);
      av[ks] = (row < w && col < w) ? d.X[(int64_t)row * w + col] : 0.0;
    }
  }
  load_blk(Cb, d.C, w, k, j);
  __syncthreads();
  f64x4 acc[4];
#pragma unroll
  for (int jt = 0; jt < 4; ++jt) acc[jt] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int ks = 0; ks < NB / 4; ++ks) {
    const int tr = 4 * ks + (lane >> 4);
#pragma unroll
    for (int jt = 0; jt < 4; ++jt)
      acc[jt] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[ks], Cb[tr][16 * jt + (lane & 15)], acc[jt], 0, 0, 0);
  }
  const bool zero = !(d.cmax[0] > 0.0);
#pragma unroll
  for (int jt = 0; jt < 4; ++jt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = k * NB + mfma_row(r), col = j * NB + mfma_col(jt);
      if (row < w && col < w) d.C[(int64_t)row * w + col] = zero ? 0.0 : acc[jt][r];
    }
}

// Update before the factorisation of block row k (k >= 1), and factorisation of the diagonal
// block k. One workgroup per (matrix, block), in one of two forms:
//   right-looking:  C_ic -= R_{k-1,i}^T R_{k-1,c}              for k <= i <= c
//   left-looking:   C_kc -= sum_{j < k} R_jk^T R_jc, j rising  for k <= c
// Both apply the same MFMA steps to a block in the same order (the block itself is the accumulator,
// and in memory between launches a double as well), so the factor does not depend on the form.
// What bounds a factorisation of few matrices is its chain of launches, one per block row, and in it
// the diagonal block's workgroup: right-looking, that is one block product and diag_factor, and
// the trailing blocks' traffic runs beside it while most CUs are idle (35 us a launch on average
// in a Llama-2-7B-shaped layer; left-looking, up to 31 products at w = 2048, 90 us). In a batch whose
// trailing blocks keep the chip busy by themselves that traffic is what counts, and left-looking
// reads and writes every block of C once (32 such layers: 345 ms of a refresh against 201). See
// chol_left_looking. Applying two or four block rows at a time, right-looking, measured 0 and 2 %
// more at one 7B-shaped layer (refresh 255, 255, 261 ms) and 1.5 and 4 % at four 300M-shaped ones.
// R_jc through LDS, R_ji's 16 columns of each wave straight into its MFMA operand registers
// (A[a][t] = R_ji[t][16 w + a]), the next pair loaded while the current one is multiplied.
template <bool LEFT>
__global__ __launch_bounds__(256, 2) void k_chol_row(const RefDev* __restrict__ ds, const uint32_t* __restrict__ pref,
                                                     int n, int k) {
  // workgroups 0 .. n-1: the diagonal block of matrix t (updated, then factored here);
  // the rest: the other blocks (i, c) row by row (LEFT: of row k only), matrices by prefix
  const uint32_t t = blockIdx.x;
  const bool diag = t < (uint32_t)n;
  const int mi = diag ? (int)t : find_pref(pref, n, t - n);
  const RefDev& d = ds[mi];
  const int w = d.w, nb = nblk(w);
  if (diag && k >= nb) return;
  int ib = k, c = k;
  if (!diag) {
    int rem = 1 + (int)(t - n - pref[mi]);
    if (!LEFT)
      while (rem >= nb - ib) { rem -= nb - ib; ++ib; }
    c = ib + rem;
  }
  __shared__ DiagLds S;
  double (*Rb)[LDB] = S.D;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double av[NB / 4], pb[16];
  auto fetch_a = [&](int j, double (&a)[NB / 4]) {
    const int col = ib * NB + 16 * wave + (lane & 15);
#pragma unroll
    for (int ks = 0; ks < NB / 4; ++ks) {
      const int row = j * NB + 4 * ks + (lane >> 4);
      a[ks] = (row < w && col < w) ? d.C[(int64_t)row * w + col] : 0.0;
    }
  };
  auto fetch_b = [&](int j) {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int e = threadIdx.x + 256 * q, row = j * NB + (e >> 6), col = c * NB + (e & 63);
      pb[q] = (row < w && col < w) ? d.C[(int64_t)row * w + col] : 0.0;
    }
  };
  auto publish_b = [&]() {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int e = threadIdx.x + 256 * q;
      Rb[e >> 6][e & 63] = pb[q];
    }
  };
  const int j0 = LEFT ? 0 : k - 1;
  fetch_a(j0, av);
  fetch_b(j0);
  f64x4 acc[4];
#pragma unroll
  for (int jt = 0; jt < 4; ++jt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = ib * NB + mfma_row(r), col = c * NB + mfma_col(jt);
      acc[jt][r] = (row < w && col < w) ? d.C[(int64_t)row * w + col] : 0.0;
    }
  publish_b();
  const double cmax = d.cmax[0];
  __syncthreads();
  for (int j = j0; j < k; ++j) {
    double an[NB / 4];
    if (LEFT && j + 1 < k) {
      fetch_a(j + 1, an);
      fetch_b(j + 1);
    }
#pragma unroll
    for (int ks = 0; ks < NB / 4; ++ks) {
      const int tr = 4 * ks + (lane >> 4);
#pragma unroll
      for (int jt = 0; jt < 4; ++jt)
        acc[jt] = __builtin_amdgcn_mfma_f64_16x16x4f64(-av[ks], Rb[tr][16 * jt + (lane & 15)], acc[jt], 0, 0, 0);
    }
    if (LEFT && j + 1 < k) {
      __syncthreads();
      publish_b();
#pragma unroll
      for (int ks = 0; ks < NB / 4; ++ks) av[ks] = an[ks];
      __syncthreads();
    }
  }
  if (!diag) {
#pragma unroll
    for (int jt = 0; jt < 4; ++jt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = ib * NB + mfma_row(r), col = c * NB + mfma_col(jt);
        if (row < w && col < w) d.C[(int64_t)row * w + col] = acc[jt][r];
      }
    return;
  }
  // diagonal block: the updated C_kk goes to LDS and is factored while the other workgroups of
  // the launch run on
  __syncthreads();
  const int kb = bsz(w, k);
#pragma unroll
  for (int jt = 0; jt < 4; ++jt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = mfma_row(r), j = mfma_col(jt);
      Rb[i][j] = (cmax > 0.0 && i < kb && j < kb) ? acc[jt][r] : (i == j ? 1.0 : 0.0);
    }
  __syncthreads();
  diag_factor(S, kb, cmax * 1e-13, d, k * NB);
}

// Triangular inverse X = R^{-1} by recursive doubling over the 64 x 64 blocks. Level l
// (l = 1, 2, ...) pairs the already inverted halves A = blocks [p 2^l, p 2^l + 2^(l-1))
// and B = [p 2^l + 2^(l-1), min((p + 1) 2^l, nb)) of every super-block p and forms
//   X_AB = -X_AA R_AB X_BB
// in two launches: phase 0 T = R_AB X_BB, phase 1 X_AB = -X_AA T. T waits in the
// (otherwise unused) strictly lower part of X, its block (i, j) transposed at block
// (j, i), which holds exactly the rows and columns of T's block even at a partial edge block. The
// diagonal blocks X_kk come from k_chol_diag. A dependency chain is at most 2^(l-1)
// block products long, against up to nb - 1 for a column-by-column inverse. One
// workgroup per 64 x 64 output block; its K loop loads the next block pair into
// registers while the current one is multiplied from LDS.
__global__ __launch_bounds__(256, 2) void k_trtri(const RefDev* __restrict__ ds, const uint32_t* __restrict__ pref,
                                               int n, int l, int phase) {
  const uint32_t t = blockIdx.x;
  const int mi = find_pref(pref, n, t);
  const RefDev& d = ds[mi];
  const int w = d.w, nb = nblk(w);
  const int h = 1 << (l - 1);
  int rem = (int)(t - pref[mi]), A0 = 0, nB = 1;
  for (int p = 0; p * 2 * h + h < nb; ++p) {   // pairs with a non-empty B half
    const int a0 = p * 2 * h, cnt = h * (min(a0 + 2 * h, nb) - a0 - h);
    if (rem < cnt) { A0 = a0; nB = min(a0 + 2 * h, nb) - a0 - h; break; }
    rem -= cnt;
  }
  const int B0 = A0 + h;
  const int I = A0 + rem / nB, J = B0 + rem % nB;
  // phase 0: sum over tb = B0 .. J of R_{I,tb} X_{tb,J}   (R in the upper part of C)
  // phase 1: sum over tb = I .. B0-1 of X_{I,tb} T_{tb,J} (T_{tb,J}^T parked at X block (J, tb))
  const int tlo = phase == 0 ? B0 : I, thi = phase == 0 ? J : B0 - 1;
  __shared__ double Ab[NB][LDB];
  __shared__ double Bb[NB][LDB];
  f64x4 acc[4];
#pragma unroll
  for (int jt = 0; jt < 4; ++jt) acc[jt] = f64x4{0.0, 0.0, 0.0, 0.0};
  double pa[16], pb[16];
  auto fetch = [&](int tb) {
    const double* Am = phase == 0 ? d.C : d.X;
    const int ar = I, ac = tb;                       // A block (I, tb)
    const int br = phase == 0 ? tb : J, bc = phase == 0 ? J : tb;   // B block (phase 1: transposed)
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int e = threadIdx.x + 256 * q, i = e >> 6, j = e & 63;
      const int ra = ar * NB + i, ca = ac * NB + j, rb = br * NB + i, cb = bc * NB + j;
      pa[q] = (ra < w && ca < w) ? Am[(int64_t)ra * w + ca] : 0.0;
      pb[q] = (rb < w && cb < w) ? d.X[(int64_t)rb * w + cb] : 0.0;
    }
  };
  auto publish = [&]() {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int e = threadIdx.x + 256 * q, i = e >> 6, j = e & 63;
      Ab[i][j] = pa[q];
      if (phase == 0) Bb[i][j] = pb[q];
      else Bb[j][i] = pb[q];   // X block (J, tb) holds T_{tb,J}^T
    }
  };
  fetch(tlo);
  publish();
  __syncthreads();
  for (int tb = tlo; tb <= thi; ++tb) {
    if (tb < thi) fetch(tb + 1);
    mfma_blk<false>(Ab, Bb, acc);
    __syncthreads();
    if (tb < thi) {
      publish();
      __syncthreads();
    }
  }
  if (phase == 0) {   // park T_{I,J}^T at block (J, I), transposed through LDS
#pragma unroll
    for (int jt = 0; jt < 4; ++jt)
#pragma unroll
      for (int r = 0; r < 4; ++r) Ab[mfma_col(jt)][mfma_row(r)] = acc[jt][r];
    __syncthreads();
    for (int e = threadIdx.x; e < NB * NB; e += 256) {
      const int i = e >> 6, j = e & 63, row = J * NB + i, col = I * NB + j;
      if (row < w && col < w) d.X[(int64_t)row * w + col] = Ab[i][j];
    }
  } else {
#pragma unroll
    for (int jt = 0; jt < 4; ++jt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = I * NB + mfma_row(r), col = J * NB + mfma_col(jt);
        if (row < w && col < w) {
          const int64_t g = (int64_t)row * w + col;
          d.X[g] = -acc[jt][r];
          d.Rinv[g] = (float)(-acc[jt][r]);
        }
      }
  }
}

}  // namespace

int chol_blocks(int32_t w) { return (w + NB - 1) / NB; }
uint32_t chol_row_tiles(int nb, int k, bool left) {
  if (k < 1 || k >= nb) return 0;
  return left ? (uint32_t)(nb - k - 1) : (uint32_t)((nb - k) * (nb - k + 1) / 2 - 1);
}
// What the right-looking form adds is traffic, all trailing blocks once per block row (sum over the
// matrices of nb^3 / 3 block updates); what the left-looking one adds is a chain of nbmax^2 / 2
// block products before the diagonal blocks. Refresh, right against left (ms): a d = 256 layer 7.1 and
// 7.2; 24 layers of 300M shapes (ratio 675) 135.7 and 137.0; 1, 4, 8, 16, 32 layers of Llama-2-7B
// shapes (ratio 112 each) 228 and 266, 626 and 655, 1131 and 1143, 2160 and 2151, 4234 and 4181.
bool chol_left_looking(int64_t sum_nb3, int nbmax) { return sum_nb3 > 1300 * (int64_t)nbmax * nbmax; }

hipError_t launch_chol_diag(const RefDev* d, int n, hipStream_t st) {
  if (!n) return hipSuccess;
  hipLaunchKernelGGL(k_chol_diag, dim3(n), dim3(256), 0, st, d);
  return hipGetLastError();
}
hipError_t launch_chol_panel(const RefDev* d, const uint32_t* pref, int n, uint32_t total, int k, hipStream_t st) {
  if (!total) return hipSuccess;
  hipLaunchKernelGGL(k_chol_panel, dim3(total), dim3(256), 0, st, d, pref, n, k);
  return hipGetLastError();
}
hipError_t launch_chol_row(const RefDev* d, const uint32_t* pref, int n, uint32_t total, int k, bool left,
                           hipStream_t st) {
  if (!n || k < 1 || total < (uint32_t)n) return hipSuccess;
  if (left) hipLaunchKernelGGL(k_chol_row<true>, dim3(total), dim3(256), 0, st, d, pref, n, k);
  else hipLaunchKernelGGL(k_chol_row<false>, dim3(total), dim3(256), 0, st, d, pref, n, k);
  return hipGetLastError();
}
int trtri_levels(int32_t nbmax) { int l = 0; while ((1 << l) < nbmax) ++l; return l; }
uint32_t trtri_tiles(int32_t w, int l) {
  const int nb = (w + NB - 1) / NB, h = 1 << (l - 1);
  uint32_t c = 0;
  for (int a0 = 0; a0 + h < nb; a0 += 2 * h) c += (uint32_t)(h * (std::min(a0 + 2 * h, nb) - a0 - h));
  return c;
}
hipError_t launch_trtri(const RefDev* d, const uint32_t* pref, int n, uint32_t total, int l, int phase, hipStream_t st) {
  if (!total) return hipSuccess;
  hipLaunchKernelGGL(k_trtri, dim3(total), dim3(256), 0, st, d, pref, n, l, phase);
  return hipGetLastError();
}
