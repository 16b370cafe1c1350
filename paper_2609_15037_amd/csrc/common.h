// Shared device-side definitions of the MoARa HIP library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

enum { SIDE_LEFT = 1, SIDE_RIGHT = 2 };

// ---------------------------------------------------------------- descriptors
// One projected matrix as seen by the step kernels. Rebuilt on the host for
// every call (pointers to W and G change between calls) and uploaded as one
// array; per-kernel tile prefixes let one launch cover every matrix.
struct MatDev {
  const float* G;      // m x n fp32, row-major
  void* W;             // m x n, weight dtype
  int64_t m, n;        // rows, cols
  int32_t k;           // blocks per row = ceil(n / B)
  int32_t r;           // rank
  int32_t side;        // SIDE_LEFT (P is m x r) or SIDE_RIGHT (Q is n x r)
  int32_t L, s;        // L = uncompressed state dim, s = projected dim
  float* inv;          // m x k: 1 / (M + eps_d) (the one-pass kernel leaves block sums of squares here)
  float* dM;           // m x k: Optimizer_M output
  float* mag1;         // m x k: Optimizer_M moments
  float* mag2;
  float* exp1;         // L x r, row stride ldr: Optimizer_V moments (row l, column j)
  float* exp2;
  void* N;             // L x r: Optimizer_V output in operand dtype
  const void* Pop;     // s x r projector, operand dtype
  const void* Ptop;    // r x s projector (transposed copy), operand dtype
  float bc1, bc2;      // 1 - beta1^t, 1 - beta2^t for this step
  uint32_t tile_dec;   // first WG index of this matrix in the decompose launch
  uint32_t tile_proj;  // ... in the projection launch
  uint32_t tile_back;  // ... in the back-projection launch
  int32_t vt;          // V output layout: 0 row-major m x n, 1 transposed n x m
  bf16* Vb;            // bf16 direction tensor V written by the decomposition (nullptr: none); its
                       // padding up to whole 32-wide K panels is zero and stays so
  int32_t n_bf16;      // zero-gradient step: N is bf16 (else fp32) ...
  int32_t n_kp;        // ... in the blocked layout kp_index(l, j, L)
  int32_t mom_bf16;    // zero-gradient step: exp1 / exp2 hold bf16 values
  int32_t ldr;         // row stride of exp1 / exp2
  int32_t parts;       // transposed decomposition: column parts of a row group, one workgroup each
  int32_t pad_;
};

struct StepParams {
  int32_t B;            // block size
  int32_t nmat;
  int32_t decompose;    // 0: V = G, dM = 1
  int32_t weight_bf16;  // 1: W is bf16
  float beta1, beta2, adam_eps, decomp_eps;
  float lr, scale;
  uint32_t total_dec, total_proj, total_back;
};

// ---------------------------------------------------------------- helpers
// Blocked ("K-panel") layout of a bf16 GEMM operand with `rows` rows and reduction
// length K (rounded up to a multiple of 32, the last panel's tail zero): element (i, k) sits
// at ((k / 32) * rows + i) * 32 + k % 32.
// The 64-byte row segments of one 32-wide K step of consecutive rows are then one
// contiguous run, which the large-tile GEMM streams with whole-line DMA loads.
__host__ __device__ __forceinline__ int64_t kp_index(int64_t i, int64_t k, int64_t rows) {
  return ((k >> 5) * rows + i) * 32 + (k & 31);
}

__device__ __forceinline__ float bf2f(bf16 x) { return (float)x; }
__device__ __forceinline__ bf16 f2bf(float x) { return (bf16)x; }   // round to nearest even

// Bijective remaps of the hardware dispatch order (workgroup b runs on XCD b % 8) so that
// neighbouring logical tiles run on the same XCD and share its L2.
// xcd_remap: each XCD takes one contiguous eighth of the tiles.
__device__ __forceinline__ uint32_t xcd_remap(uint32_t bid, uint32_t nblk) {
  const uint32_t X = 8;
  const uint32_t xcd = bid % X, per = nblk / X, rem = nblk % X;
  return xcd * per + (xcd < rem ? xcd : rem) + bid / X;
}
// xcd_remap_list: with `groups` the XCDs take groups of XCD_GROUP tiles in turn (what is left past
// whole rounds in eighths), so that each gets a share of every problem in a list; the GEMM lists
// choose by gemm_xcd_groups. Groups of 32 measured the same, of 64 235 instead of 229 ms (refresh
// of a 7B-shaped layer). The one-pass projection streams the gradient and keeps the eighths (24
// layers of 300M shapes 10 us faster).
constexpr uint32_t XCD_GROUP = 16;
__device__ __forceinline__ uint32_t xcd_remap_list(uint32_t bid, uint32_t nblk, int groups) {
  const uint32_t X = 8, G = XCD_GROUP;
  const uint32_t full = groups ? nblk / (X * G) * (X * G) : 0;   // tiles in groups
  const uint32_t i = bid / X;
  const uint32_t in_groups = ((i / G) * X + bid % X) * G + i % G;
  const uint32_t in_eighths = full + xcd_remap(bid - full, nblk - full);   // full: a multiple of X
  return bid < full ? in_groups : in_eighths;
}

// Largest i with prefix(i) <= t, prefix read through a member pointer of MatDev.
template <typename F>
__device__ __forceinline__ int find_mat(const MatDev* mats, int nmat, uint32_t t, F prefix) {
  int lo = 0, hi = nmat - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (prefix(mats[mid]) <= t) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__device__ __forceinline__ float wave_sum(float v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_sum_d(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// The multiply-adds below are written out: left to the compiler, their contraction depends on the
// kernel they are inlined into, and a matrix's step must not depend (to the last bit) on which
// kernel it takes. The sum of squares keeps the order that fp32 operands have always seen: a
// refresh's first update is close to sign(R), so one element of R near zero turns an ulp of a
// block norm into 1e-2 of a weight's root mean square.
__device__ __forceinline__ float sumsq4(float4 v) {
  return fmaf(v.w, v.w, fmaf(v.z, v.z, fmaf(v.x, v.x, v.y * v.y)));
}

// Adam step of Kingma & Ba with bias correction terms passed in (no weight decay).
__device__ __forceinline__ float adam_out(float x, float& e, float& q, float b1, float b2,
                                          float eps, float bc1, float bc2) {
  e = fmaf(b1, e, (1.0f - b1) * x);
  q = fmaf((1.0f - b2) * x, x, b2 * q);
  return (e / bc1) / (sqrtf(q / bc2) + eps);
}

// The same step with the moments stored in bf16: the updated moments are rounded to bf16
// (nearest even) for storage and the output is formed from the stored values.
__device__ __forceinline__ float adam_out_bf16(float x, bf16& e, bf16& q, float b1, float b2, float eps,
                                               float bc1, float bc2) {
  const float e1 = bf2f(f2bf(fmaf(b1, bf2f(e), (1.0f - b1) * x)));
  const float q1 = bf2f(f2bf(fmaf((1.0f - b2) * x, x, b2 * bf2f(q))));
  e = f2bf(e1);
  q = f2bf(q1);
  return (e1 / bc1) / (sqrtf(q1 / bc2) + eps);
}

// ---------------------------------------------------------------- launchers
// All launchers return hipError_t from hipGetLastError after the launch.
struct GemmProb;
// pinned host memory -> device, 16-byte aligned, both blocks padded to 16 bytes
hipError_t launch_upload(void* dst, const void* host_src, size_t bytes, hipStream_t st);
// bf16 -> fp32 (exact) of up to CAST_MAX buffers of any alignment in one launch
constexpr int CAST_MAX = 64;
struct CastList {
  const void* src[CAST_MAX];
  float* dst[CAST_MAX];
  int64_t count[CAST_MAX];
  uint32_t start[CAST_MAX];   // first workgroup
  int n;
};
uint32_t cast_tiles(int64_t count);
hipError_t launch_cast(const CastList& l, uint32_t total, hipStream_t st);
// One launch covers matrices that are all plain (decompose_plain) or all not. adam_m: also run
// Optimizer_M.
bool decompose_plain(const float* G, int64_t n, int k, bool decompose, bool transposed);
hipError_t launch_decompose(const MatDev* mats_dev, const StepParams& p, int adam_m, bool plain, hipStream_t st);
// split: some matrix of the list has parts > 1
hipError_t launch_decompose_vt(const MatDev* mats_dev, const StepParams& p, int adam_m, bool plain, bool split,
                               hipStream_t st);
int decompose_tiles(int64_t m);
int decompose_vt_tiles(int64_t m);          // row groups; times MatDev::parts workgroups
int decompose_vt_max_parts(int64_t n);
// Optimizer_M and Optimizer_V of a matrix whose gradient is exactly zero (no G is read):
// magnitude moments -> dM (when p.decompose), direction moments -> N; tile_dec holds the
// matrix's first workgroup, zero_grad_tiles(...) workgroups per matrix.
uint32_t zero_grad_tiles(int64_t mk, int64_t Lr);
hipError_t launch_zero_grad(const MatDev* mats_dev, const StepParams& p, hipStream_t st);
// limits of the V-writing decomposition paths (blocks per row)
constexpr int DEC_VT_MAX_K = 160;    // transposed path: blocks held in LDS at a time (any k runs)
constexpr int DEC_ROW_MAX_K = 512;   // row-major path, 16 rows per workgroup
hipError_t launch_project(const MatDev* mats_dev, const StepParams& p, int operand_bf16, hipStream_t st);
hipError_t launch_backproject(const MatDev* mats_dev, const StepParams& p, int operand_bf16, hipStream_t st);
