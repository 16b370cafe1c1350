// Block-wise magnitude/direction decomposition (Section 3.1, Appendix B.1)
// fused with Optimizer_M (Adam on the block magnitudes, Algorithm 1).
//
// For every row i and block j (columns [jB, min(jB+B, n)) -- the zero padding of
// the last block contributes nothing to the norm):
//   M[i,j]   = ||G[i, block j]||_2
//   inv[i,j] = 1 / (M[i,j] + eps_d)        (V = G * inv is formed on the fly by the GEMMs)
//   dM[i,j]  = Adam(M[i,j])                (when p.adam_m != 0)
//
// Memory-bound: reads G once (4 B/element), writes 4 (inv, dM, two moments)
// and reads 2 fp32 values per block. A block of B <= 256 columns maps onto B/4
// consecutive lanes and is reduced with xor shuffles inside that lane group
// (fixed order, so results are bit-reproducible; the butterfly leaves the same
// sum in every lane of the group). Other block sizes take a generic per-block
// path.
//
// When the step's GEMMs take bf16 operands, the same pass also writes the
// direction tensor V = G * inv in bf16 (2 B/element), oriented so that the
// projection's reduction index runs along its rows (m x n for a RIGHT projection
// V Q, transposed n x m for a LEFT one P^T V) and stored in the blocked K-panel
// layout of the large-tile GEMM (kp_index). The transposed form comes from
// k_decompose_vt, which stages a 32-row x 256-column slab in LDS.
#include "common.h"

namespace {
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
constexpr int DEC_ROWS = 16;   // rows per workgroup (4 waves x 4 rows)

// Columns c .. c + 3 of a gradient row of n columns (zeros past its end). PLAIN: n % 4 == 0 and
// rows 16-byte aligned. Otherwise rows start at any multiple of 4 bytes, which a 16-byte global
// load takes, and a group may end inside the row. One code path with the tail test made the
// transposed decomposition 3 to 40 % slower at aligned sizes (more live masks around its 8 loads
// in flight), so the kernels are instantiated for both and each matrix goes to its own launch.
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
template <bool PLAIN>
__device__ __forceinline__ float4 load_g4(const float* row, int64_t c, int64_t n) {
  if (PLAIN) return c < n ? *reinterpret_cast<const float4*>(row + c) : make_float4(0.f, 0.f, 0.f, 0.f);
  if (c + 4 <= n) {
    const f32x4_a4 v = *reinterpret_cast<const f32x4_a4*>(row + c);
    return make_float4(v.x, v.y, v.z, v.w);
  }
  return make_float4(c < n ? row[c] : 0.f, c + 1 < n ? row[c + 1] : 0.f, c + 2 < n ? row[c + 2] : 0.f, 0.f);
}

// Sum over aligned groups of gl lanes (gl a power of two <= 64). The first four
// levels use DPP lane permutations (pairs within a quad, then the two quads of an
// 8-lane half-row, then the two halves of a 16-lane row: mirror permutations pair
// lanes whose values are already equal to their group's partial sum), the fifth a
// ds_swizzle xor 16, the sixth a cross-half shuffle. Each level adds two equal
// partial sums in either order, so every lane of a group ends with the same,
// bit-identical total.
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float group_sum(float v, int gl) {
  if (gl >= 2) v += dpp_f<0xB1>(v);    // quad_perm [1,0,3,2]
  if (gl >= 4) v += dpp_f<0x4E>(v);    // quad_perm [2,3,0,1]
  if (gl >= 8) v += dpp_f<0x141>(v);   // row_half_mirror
  if (gl >= 16) v += dpp_f<0x140>(v);  // row_mirror
  if (gl >= 32) v += __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x401F));   // lane ^ 16
  if (gl >= 64) v += __shfl_xor(v, 32, 64);
  return v;
}

__device__ __forceinline__ void block_out(const MatDev& d, const StepParams& p, int64_t row, int j,
                                          float ss, int adam_m) {
  const float M = sqrtf(ss);
  const int64_t idx = row * d.k + j;
  d.inv[idx] = 1.0f / (M + p.decomp_eps);
  if (adam_m) {
    float e = d.mag1[idx], q = d.mag2[idx];
    const float out = adam_out(M, e, q, p.beta1, p.beta2, p.adam_eps, d.bc1, d.bc2);
    d.mag1[idx] = e;
    d.mag2[idx] = q;
    d.dM[idx] = out;
  }
}

// Phase 1: the block sums of squares of the workgroup's DEC_ROWS rows go to LDS
// (each wave streams one row at a time with UNR 16-byte loads in flight).
// Phase 2: all threads run Optimizer_M over those DEC_ROWS * k blocks, which are
// contiguous in the m x k layout, so the moment/inv/dM traffic is coalesced.
constexpr int DEC_LDS = 8192;   // floats of LDS for block sums (phase 1 -> 2)

template <bool PLAIN>
__global__ __launch_bounds__(256) void k_decompose(const MatDev* __restrict__ mats, StepParams p, int adam_m) {
  __shared__ float sums[DEC_LDS];
  const uint32_t t = blockIdx.x;
  const int mi = find_mat(mats, p.nmat, t, [](const MatDev& d) { return d.tile_dec; });
  const MatDev d = mats[mi];
  const int64_t row0 = (int64_t)(t - d.tile_dec) * DEC_ROWS;
  const int rows = (int)((d.m - row0 < DEC_ROWS) ? d.m - row0 : DEC_ROWS);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // without the decomposition V = G: only V is written (any group width does)
  const bool dec = PLAIN || p.decompose != 0;
  const int B = dec ? p.B : 128;
  const int64_t n = d.n;
  const int k = d.k;
  const bool staged = !dec || (int64_t)rows * k <= DEC_LDS;
  const bool fast = staged && B >= 4 && B <= 256 && (B & (B - 1)) == 0;
  if (!staged) {
    // generic path (very many blocks per row): one block at a time, Optimizer_M inline
    for (int rr = wave; rr < rows; rr += 4) {
      const int64_t row = row0 + rr;
      const float* g = d.G + row * n;
      for (int j = 0; j < k; ++j) {
        const int64_t cs = (int64_t)j * B;
        const int64_t ce = (cs + B < n) ? cs + B : n;
        float ss = 0.f;
        for (int64_t c = cs + lane; c < ce; c += 64) { const float v = g[c]; ss += v * v; }
        ss = wave_sum(ss);
        if (lane == 0) block_out(d, p, row, j, ss, adam_m);
      }
    }
    return;
  }
  if (fast && B <= 128) {
    // Row pairs: the two half-waves take rows 2p and 2p + 1 (blocks of B <= 128 columns
    // stay inside a half-wave), so that each bf16 store of V covers both rows of a
    // 32-column block, i.e. whole 128-byte lines of the blocked layout.
    constexpr int UNR = 8;
    const int gl = B >> 2;   // lanes per block
    const int lgB = __builtin_ctz(B);
    const int hl = lane & 31;
    for (int rp = wave; 2 * rp < rows; rp += 4) {
      const int rr = 2 * rp + (lane >> 5);
      const bool rok = rr < rows;
      const int64_t row = row0 + rr;
      const float* g = d.G + row * n;
      for (int64_t c00 = 0; c00 < n; c00 += 128 * UNR) {
        float4 v[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          const int64_t c = c00 + 128 * u + 4 * hl;
          v[u] = load_g4<PLAIN>(g, rok ? c : n, n);
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          const int64_t c = c00 + 128 * u + 4 * hl;
          float ss = sumsq4(v[u]);
          ss = group_sum(ss, gl);
          if (rok && c < n) {
            if (dec && (hl & (gl - 1)) == 0) sums[rr * k + (int)(c >> lgB)] = ss;
            if (d.Vb) {
              const float inv = dec ? 1.0f / (sqrtf(ss) + p.decomp_eps) : 1.0f;
              bf16x4 o;
              o[0] = f2bf(v[u].x * inv); o[1] = f2bf(v[u].y * inv); o[2] = f2bf(v[u].z * inv); o[3] = f2bf(v[u].w * inv);
              *reinterpret_cast<bf16x4*>(d.Vb + kp_index(row, c, d.m)) = o;   // blocked, K = n
            }
          }
        }
      }
    }
  } else
  for (int rr = wave; rr < rows; rr += 4) {
    const int64_t row = row0 + rr;
    const float* g = d.G + row * n;
    if (fast) {
      constexpr int UNR = 8;
      const int gl = B >> 2;   // lanes per block
      const int lgB = __builtin_ctz(B);
      for (int64_t c00 = 0; c00 < n; c00 += 256 * UNR) {
        float4 v[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          const int64_t c = c00 + 256 * u + 4 * lane;
          v[u] = load_g4<PLAIN>(g, c, n);
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          const int64_t c = c00 + 256 * u + 4 * lane;
          float ss = sumsq4(v[u]);
          ss = group_sum(ss, gl);
          if ((lane & (gl - 1)) == 0 && c < n) sums[rr * k + (int)(c >> lgB)] = ss;
          if (d.Vb && c < n) {
            const float inv = 1.0f / (sqrtf(ss) + p.decomp_eps);
            bf16x4 o;
            o[0] = f2bf(v[u].x * inv); o[1] = f2bf(v[u].y * inv); o[2] = f2bf(v[u].z * inv); o[3] = f2bf(v[u].w * inv);
            *reinterpret_cast<bf16x4*>(d.Vb + kp_index(row, c, d.m)) = o;   // blocked, K = n
          }
        }
      }
    } else {
      for (int j = 0; j < k; ++j) {
        const int64_t cs = (int64_t)j * B;
        const int64_t ce = (cs + B < n) ? cs + B : n;
        float ss = 0.f;
        for (int64_t c = cs + lane; c < ce; c += 64) { const float v = g[c]; ss += v * v; }
        ss = wave_sum(ss);
        if (lane == 0) sums[rr * k + j] = ss;
      }
    }
  }
  if (!dec) return;
  __syncthreads();
  const int total = rows * k;
  for (int e = threadIdx.x; e < total; e += 256) {
    const int rr = e / k, j = e - (e / k) * k;
    block_out(d, p, row0 + rr, j, sums[e], adam_m);
  }
}

// Transposed-V variant (LEFT projections): one workgroup per VT_ROWS (32) rows. For each
// 256-column slab every wave loads VT_RPW of the rows (float4 per lane, all in
// flight), reduces the block sums, writes V in bf16 into an LDS slab
// T[VT_ROWS][256] (row-major, conflict-free 4-byte stores) and records the sums; the
// slab is then written out transposed, VT_ROWS / 8 lanes per output column (16 bytes
// each), i.e. 64-byte (one K panel) segments of Vt. The odd 4-byte pitch of T keeps the
// row groups read by one instruction on distinct banks. Optimizer_M then runs over the
// VT_ROWS x k sums as in k_decompose. 32-row slabs (143 VGPRs, three waves per SIMD)
// measured 1.7 % faster than 64-row ones (231 VGPRs, two). The sums of DEC_VT_MAX_K blocks per
// row fit in LDS; longer rows run in column ranges of that many blocks. SPLIT: a row group's columns
// go to MatDev::parts workgroups (short lists, whose few row groups would each walk all columns). Rows past m are zero in
// the last K panel. Preconditions (checked by the host): B a power of two in [4, 256], or no
// decomposition (V = G); PLAIN: decompose_plain.
#ifndef DEC_VT_ROWS
#define DEC_VT_ROWS 32
#endif
constexpr int VT_ROWS = DEC_VT_ROWS, VT_COLS = 256, VT_PITCH = VT_COLS + 2;   // bf16 elements
constexpr int VT_RPW = VT_ROWS / 4;    // rows per wave
constexpr int VT_GRP = VT_ROWS / 8;    // 8-row groups of a column (16-byte output runs)
static_assert(VT_ROWS % 32 == 0, "whole 32-row K panels of the blocked output");

template <bool PLAIN, bool SPLIT>
__global__ __launch_bounds__(256) void k_decompose_vt(const MatDev* __restrict__ mats, StepParams p, int adam_m) {
  __shared__ float sums[VT_ROWS * DEC_VT_MAX_K];
  __shared__ __attribute__((aligned(16))) bf16 T[VT_ROWS * VT_PITCH];
  const uint32_t t = blockIdx.x;
  const int mi = find_mat(mats, p.nmat, t, [](const MatDev& d) { return d.tile_dec; });
  const MatDev d = mats[mi];
  const uint32_t lt = t - d.tile_dec, parts = SPLIT ? (uint32_t)d.parts : 1u;
  const int64_t row0 = (int64_t)(lt / parts) * VT_ROWS;
  const int rows = (int)((d.m - row0 < VT_ROWS) ? d.m - row0 : VT_ROWS);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const bool dec = PLAIN || p.decompose != 0;
  const int B = dec ? p.B : 128, gl = B >> 2, k = d.k, lgB = __builtin_ctz(B);
  const int64_t n = d.n;
  // the slab loop is software-pipelined: the VT_RPW loads of the next slab are issued
  // before the current slab is reduced, transposed and written out
  float4 va[VT_RPW], vb[VT_RPW];
  auto load = [&](int64_t c0, float4 (&v)[VT_RPW]) {
    const int64_t c = c0 + 4 * lane;
#pragma unroll
    for (int i = 0; i < VT_RPW; ++i) {
      const int rr = wave + 4 * i;
      v[i] = load_g4<PLAIN>(d.G + (row0 + rr) * n, rr < rows ? c : n, n);
    }
  };
  int kc0 = 0, kc = 0;   // blocks of the current column range: [kc0, kc0 + kc)
  auto process = [&](int64_t c0, const float4 (&v)[VT_RPW]) {
    const int64_t c = c0 + 4 * lane;
#pragma unroll
    for (int i = 0; i < VT_RPW; ++i) {
      const int rr = wave + 4 * i;
      float ss = sumsq4(v[i]);
      ss = group_sum(ss, gl);
      if (dec && rr < rows && c < n && (lane & (gl - 1)) == 0) sums[rr * kc + (int)(c >> lgB) - kc0] = ss;
      // rows past m are K padding of V and have to stay zero, also where 1 / (0 + eps_d) is infinite
      const float scale = dec ? 1.0f / (sqrtf(ss) + p.decomp_eps) : 1.0f, inv = rr < rows ? scale : 0.0f;
      bf16x2 a, b;
      a[0] = f2bf(v[i].x * inv); a[1] = f2bf(v[i].y * inv);
      b[0] = f2bf(v[i].z * inv); b[1] = f2bf(v[i].w * inv);
      *reinterpret_cast<bf16x2*>(T + rr * VT_PITCH + 4 * lane) = a;
      *reinterpret_cast<bf16x2*>(T + rr * VT_PITCH + 4 * lane + 2) = b;
    }
    __syncthreads();
#pragma unroll 2
    for (int it = 0; it < VT_GRP; ++it) {
      const int q = it * 256 + (int)threadIdx.x;
      const int cl = q / VT_GRP, g = q % VT_GRP;
      const int64_t col = c0 + cl;
      if (col < n && 8 * g < rows) {
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = T[(8 * g + e) * VT_PITCH + cl];
        *reinterpret_cast<bf16x8*>(d.Vb + kp_index(col, row0 + 8 * g, n)) = o;   // blocked V' (n x m), K = m
      }
    }
    __syncthreads();
  };
  auto adam_m_blocks = [&]() {
    const int total = rows * kc;
    for (int e = threadIdx.x; e < total; e += 256) {
      const int rr = e / kc, j = e - (e / kc) * kc;
      block_out(d, p, row0 + rr, kc0 + j, sums[e], adam_m);
    }
  };
  // this workgroup's columns: whole slabs, parts of equal length but for the last ones
  const int64_t len = SPLIT ? ((n + VT_COLS - 1) / VT_COLS + parts - 1) / parts * VT_COLS : n;
  const int64_t cb = lt % parts * len, cend = cb + len < n ? cb + len : n;
  if (SPLIT && cb >= cend) return;
  load(cb, va);
  if (PLAIN) {
    kc0 = (int)(cb >> lgB);
    kc = (int)((cend + B - 1) >> lgB) - kc0;
    for (int64_t c0 = cb; c0 < cend; c0 += 2 * VT_COLS) {
      if (c0 + VT_COLS < cend) load(c0 + VT_COLS, vb);
      process(c0, va);
      if (c0 + VT_COLS >= cend) break;
      if (c0 + 2 * VT_COLS < cend) load(c0 + 2 * VT_COLS, va);
      process(c0 + VT_COLS, vb);
    }
    adam_m_blocks();
    return;
  }
  // column ranges of at most DEC_VT_MAX_K blocks, whole slabs (B divides VT_COLS)
  const int64_t span = dec ? (int64_t)DEC_VT_MAX_K * B / VT_COLS * VT_COLS : n;
  for (int64_t cr = cb; cr < cend; cr += span) {
    const int64_t ce = cr + span < cend ? cr + span : cend;
    kc0 = (int)(cr >> lgB);
    kc = (int)((ce + B - 1) >> lgB) - kc0;
    for (int64_t c0 = cr; c0 < ce; c0 += 2 * VT_COLS) {
      if (c0 + VT_COLS < cend) load(c0 + VT_COLS, vb);
      process(c0, va);
      if (c0 + VT_COLS >= ce) {   // odd number of slabs: the next range starts with vb's columns
#pragma unroll
        for (int i = 0; i < VT_RPW; ++i) va[i] = vb[i];
        break;
      }
      if (c0 + 2 * VT_COLS < cend) load(c0 + 2 * VT_COLS, va);
      process(c0 + VT_COLS, vb);
    }
    if (!dec) break;
    adam_m_blocks();
    __syncthreads();   // the next range's sums overwrite these
  }
}
// A zero gradient gives M = 0, V = 0 and R = P^T V = 0 (Algorithm 1 with G = 0), so the
// step reduces to decaying the moments: Optimizer_M on M = 0 and Optimizer_V on R = 0,
// through the same adam_out as the decomposition and the projection epilogue (bit for
// bit what those kernels produce from an all-zero G). Elements [0, m k) of a matrix are
// its magnitude blocks (only when the decomposition is on), the next L r its direction
// moments; ZG_PER_WG elements per workgroup, consecutive threads on consecutive elements.
constexpr int ZG_PER_WG = 2048;
__global__ __launch_bounds__(256) void k_zero_grad(const MatDev* __restrict__ mats, StepParams p) {
  const uint32_t t = blockIdx.x;
  const MatDev& d = mats[find_mat(mats, p.nmat, t, [](const MatDev& x) { return x.tile_dec; })];
  const int64_t mk = p.decompose ? d.m * d.k : 0;
  const int64_t Lr = (int64_t)d.L * d.r;
  const int64_t e0 = (int64_t)(t - d.tile_dec) * ZG_PER_WG;
  for (int64_t e = e0 + threadIdx.x; e < e0 + ZG_PER_WG && e < mk + Lr; e += 256) {
    if (e < mk) {
      float a = d.mag1[e], q = d.mag2[e];
      const float out = adam_out(0.f, a, q, p.beta1, p.beta2, p.adam_eps, d.bc1, d.bc2);
      d.mag1[e] = a;
      d.mag2[e] = q;
      d.dM[e] = out;
    } else {
      const int64_t el = e - mk, l = el / d.r, j = el - l * d.r, x = l * d.ldr + j;   // (l, j) of the moments
      float out;
      if (d.mom_bf16) {
        bf16* E1 = reinterpret_cast<bf16*>(d.exp1);
        bf16* E2 = reinterpret_cast<bf16*>(d.exp2);
        bf16 a = E1[x], q = E2[x];
        out = adam_out_bf16(0.f, a, q, p.beta1, p.beta2, p.adam_eps, d.bc1, d.bc2);
        E1[x] = a;
        E2[x] = q;
      } else {
        float a = d.exp1[x], q = d.exp2[x];
        out = adam_out(0.f, a, q, p.beta1, p.beta2, p.adam_eps, d.bc1, d.bc2);
        d.exp1[x] = a;
        d.exp2[x] = q;
      }
      if (d.n_bf16) {
        ((bf16*)d.N)[d.n_kp ? kp_index(l, j, d.L) : el] = f2bf(out);
      } else {
        ((float*)d.N)[el] = out;
      }
    }
  }
}

// Descriptors from pinned host memory, read by the kernel itself: a copy through the runtime
// leaves the stream idle for about 5 us after it (a copy and its gap 9.5 us for a small call,
// this 4). The host blocks are 16-byte aligned and padded.
__global__ __launch_bounds__(256) void k_upload(uint4* __restrict__ dst, const uint4* __restrict__ src, uint32_t n) {
  for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) dst[i] = src[i];
}

// bf16 gradients -> fp32 for the kernels that take fp32 only, all of a step's in a few launches
// (one copy per matrix took 4 us each at 0.26 to 2.9 M elements, most of it the launch's own time).
// Memory-bound, 6 bytes per element: eight elements per thread and pass.
constexpr int CAST_PER_WG = 8192;
__global__ __launch_bounds__(256) void k_cast(CastList L) {
  typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
  const uint32_t t = blockIdx.x;
  int lo = 0, hi = L.n - 1;
  while (lo < hi) { const int mid = (lo + hi + 1) >> 1; if (L.start[mid] <= t) lo = mid; else hi = mid - 1; }
  const unsigned short* src = (const unsigned short*)L.src[lo];
  float* dst = L.dst[lo];
  const int64_t e0 = (int64_t)(t - L.start[lo]) * CAST_PER_WG;
  const int64_t e1 = e0 + CAST_PER_WG < L.count[lo] ? e0 + CAST_PER_WG : L.count[lo];
  if ((((uintptr_t)src | (uintptr_t)dst) & 15) == 0) {
    for (int64_t e = e0 + 8 * threadIdx.x; e + 8 <= e1; e += 8 * 256) {
      const u16x8 v = *reinterpret_cast<const u16x8*>(src + e);
#pragma unroll
      for (int h = 0; h < 2; ++h)
        *reinterpret_cast<float4*>(dst + e + 4 * h) =
            make_float4(__uint_as_float((uint32_t)v[4 * h] << 16), __uint_as_float((uint32_t)v[4 * h + 1] << 16),
                        __uint_as_float((uint32_t)v[4 * h + 2] << 16), __uint_as_float((uint32_t)v[4 * h + 3] << 16));
    }
    const int64_t e = e1 - ((e1 - e0) & 7) + threadIdx.x;   // the last elements of the buffer
    if (e < e1) dst[e] = __uint_as_float((uint32_t)src[e] << 16);
  } else {
    for (int64_t e = e0 + threadIdx.x; e < e1; e += 256) dst[e] = __uint_as_float((uint32_t)src[e] << 16);
  }
}
}  // namespace

uint32_t cast_tiles(int64_t count) { return (uint32_t)((count + CAST_PER_WG - 1) / CAST_PER_WG); }

hipError_t launch_cast(const CastList& l, uint32_t total, hipStream_t st) {
  if (!total) return hipSuccess;
  hipLaunchKernelGGL(k_cast, dim3(total), dim3(256), 0, st, l);
  return hipGetLastError();
}

hipError_t launch_upload(void* dst, const void* host_src, size_t bytes, hipStream_t st) {
  const uint32_t n = (uint32_t)((bytes + 15) / 16);
  if (!n) return hipSuccess;
  const uint32_t g = (n + 255) / 256;
  hipLaunchKernelGGL(k_upload, dim3(g < 64 ? g : 64), dim3(256), 0, st, (uint4*)dst, (const uint4*)host_src, n);
  return hipGetLastError();
}

uint32_t zero_grad_tiles(int64_t mk, int64_t Lr) { return (uint32_t)((mk + Lr + ZG_PER_WG - 1) / ZG_PER_WG); }

hipError_t launch_zero_grad(const MatDev* mats_dev, const StepParams& p, hipStream_t st) {
  if (p.total_dec == 0) return hipSuccess;
  hipLaunchKernelGGL(k_zero_grad, dim3(p.total_dec), dim3(256), 0, st, mats_dev, p);
  return hipGetLastError();
}

int decompose_tiles(int64_t m) { return (int)((m + DEC_ROWS - 1) / DEC_ROWS); }
int decompose_vt_tiles(int64_t m) { return (int)((m + VT_ROWS - 1) / VT_ROWS); }
int decompose_vt_max_parts(int64_t n) {   // two slabs a part: the second one's loads run under the first
  const int64_t slabs = (n + VT_COLS - 1) / VT_COLS;
  return slabs < 4 ? 1 : slabs < 0x10000 ? (int)(slabs / 2) : 0x8000;
}

bool decompose_plain(const float* G, int64_t n, int k, bool decompose, bool transposed) {
  return decompose && (n & 3) == 0 && ((uintptr_t)G & 15) == 0 && (!transposed || k <= DEC_VT_MAX_K);
}

hipError_t launch_decompose_vt(const MatDev* mats_dev, const StepParams& p, int adam_m, bool plain, bool split,
                               hipStream_t st) {
  if (p.total_dec == 0) return hipSuccess;
  const dim3 g(p.total_dec), b(256);
  if (plain && !split) hipLaunchKernelGGL((k_decompose_vt<true, false>), g, b, 0, st, mats_dev, p, adam_m);
  else if (plain) hipLaunchKernelGGL((k_decompose_vt<true, true>), g, b, 0, st, mats_dev, p, adam_m);
  else if (!split) hipLaunchKernelGGL((k_decompose_vt<false, false>), g, b, 0, st, mats_dev, p, adam_m);
  else hipLaunchKernelGGL((k_decompose_vt<false, true>), g, b, 0, st, mats_dev, p, adam_m);
  return hipGetLastError();
}

hipError_t launch_decompose(const MatDev* mats_dev, const StepParams& p, int adam_m, bool plain, hipStream_t st) {
  if (p.total_dec == 0) return hipSuccess;
  if (plain) hipLaunchKernelGGL((k_decompose<true>), dim3(p.total_dec), dim3(256), 0, st, mats_dev, p, adam_m);
  else hipLaunchKernelGGL((k_decompose<false>), dim3(p.total_dec), dim3(256), 0, st, mats_dev, p, adam_m);
  return hipGetLastError();
}
