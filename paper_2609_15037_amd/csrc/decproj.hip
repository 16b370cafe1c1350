// Decomposition and projection in one pass over the gradient, for ranks up to 256:
//
//   V = G / (Rep_B(M) + eps_d)  (or V = G without the decomposition), in bf16,
//   R^(T)[l][j] = sum_k V'[l][k] P[k][j]   (V' = V for RIGHT, V^T for LEFT),
//   N = Optimizer_V(R)                      (EP_ADAM's epilogue),
//   block sums of squares of G              (Optimizer_M follows in k_opt_m).
//
// With r <= 256 one tile holds every column of R, so G needs to be read only once and V never
// leaves the CU; the two-kernel form writes V and reads it back, 4 of its 8 bytes per gradient
// element. Same V (bit for bit), same order of the products' terms.
//
// What bounds it is the gradient's stream from HBM: a tile of K = 1024 needs a quarter of its read
// time on the matrix cores. Hence two workgroups of eight waves per CU (80 KB of LDS, 128
// VGPRs): one's loads are in flight while the other converts, multiplies or runs its epilogue.
// A workgroup walks K in gradient chunks of 32 KB, four float4 per thread:
//   RIGHT: 64 rows l x 128 k;  LEFT: 128 columns l x 64 k (gradient rows).
// A half-wave reads 128 consecutive columns of one gradient row, so blocks of B <= 128 columns
// stay inside it and their sums are DPP butterflies; scaled, rounded to bf16 and stored to
// LDS as the MFMA's A operand [l][k] (LEFT: each thread holds 4 consecutive gradient rows, so the
// transposed store moves 8 bytes of consecutive k). P comes through one
// 64 KB LDS buffer (direct-to-LDS loads from the blocked layout; LEFT uses its halves in turn).
// 16-byte chunks of an A row are permuted by the row so that the fragment reads and both stores
// spread over the banks. (Eight float4 per thread, 128 rows x 128 k, spilled 50 to 150
// registers beside the 64 accumulators.)
// Measured, decomposition + projection, two kernels -> this (us, bf16 moments): 24 layers of 300M
// shapes (r = 128, 192, 256) 387 + 346 -> 514 and 27 for k_opt_m; the step 1068 -> 852. G read at
// 3.0 (r = 32) to 1.9 TB/s (r = 256) over 96 matrices of 1024 x 1024, against a copy's 4.7 (read
// and written): the latency of a chunk's phases, not HBM, is what is left.
#include <type_traits>

#include "gemm.h"

namespace {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;

constexpr int FNT = 512, FU = 4;                          // threads, float4 per thread and chunk
constexpr int R_BM = 64, R_KC = 128, L_BM = 128, L_KC = 64;   // tile rows and K chunk of either side
constexpr int A_BYTES = R_BM * R_KC * 2, B_BYTES = 256 * 128 * 2;
constexpr int SLAB_LD = 64 + 4, SLAB = 32 * SLAB_LD;      // epilogue slab of a wave (floats)
constexpr int SMEM = A_BYTES + B_BYTES > 8 * SLAB * 4 ? A_BYTES + B_BYTES : 8 * SLAB * 4;

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
// sum over aligned groups of GL = 8, 16 or 32 lanes, in the decomposition's order (every lane of
// the group gets the same value)
template <int GL>
__device__ __forceinline__ float group_sum(float v) {
  v += dpp_f<0xB1>(v);
  v += dpp_f<0x4E>(v);
  v += dpp_f<0x141>(v);
  if (GL >= 16) v += dpp_f<0x140>(v);
  if (GL >= 32) v += __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x401F));
  return v;
}

__device__ __forceinline__ uint32_t pack2(float a, float b) {   // two bf16, a in the low half
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 v;
  v[0] = f2bf(a);
  v[1] = f2bf(b);
  return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ int swz_b(int R) { return ((R >> 1) & 3) ^ ((R >> 3) & 1); }   // as the large-tile GEMM
// A rows of 256 bytes (RIGHT, 16 chunks) and of 128 bytes (LEFT, 8 chunks)
__device__ __forceinline__ int swz_r(int R) { return (R & 15) ^ ((R >> 4) & 15); }
__device__ __forceinline__ int swz_l(int R) { return ((R >> 1) ^ (R >> 4)) & 7; }

__device__ __forceinline__ void wg_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// a value the compiler cannot see to be loop-invariant: addresses derived from it are formed where
// they are used instead of being kept (and spilled) across the K loop
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// GL: lanes per block (B / 4), 0 without the decomposition. A kernel of its own for each: with the
// choice made per row inside, the branches kept the loads of a chunk from staying in registers.
// G16: the gradient is bf16 (8-byte loads, widened exactly), PLAIN only. Half the bytes are worth
// little here (24 layers of Qwen2.5-350M shapes 500 -> 460 us: a chunk's phases bound it); what
// it saves is the fp32 copy, 168 launches and 665 us there.
template <bool PLAIN, bool MOM16, int GL, bool G16>
__global__ __launch_bounds__(FNT, 4) void k_decproj(const FusedProb* __restrict__ probs, GemmUniform U) {
  constexpr bool dec = GL > 0;
  constexpr int GB = G16 ? 2 : 4;   // bytes per gradient element
  static_assert(PLAIN || !G16, "bf16 gradients: four columns at a time, 8-byte aligned");
  constexpr int gl = dec ? GL : 32, lgB = gl == 8 ? 5 : gl == 16 ? 6 : 7;
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];
  const uint32_t t = xcd_remap(blockIdx.x, gridDim.x);
  int lo = 0, hi = U.nprob - 1;
  while (lo < hi) { const int mid = (lo + hi + 1) >> 1; if (probs[mid].tile_start <= t) lo = mid; else hi = mid - 1; }
  const FusedProb& P = probs[lo];
  static_assert(SMEM <= 81920, "two workgroups per CU");
  const bool side_l = P.side == SIDE_LEFT;
  const int64_t l0 = (int64_t)(t - P.tile_start) * (side_l ? L_BM : R_BM);   // first row of R^(T)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = side_l ? wave & 3 : wave & 1, wn = side_l ? wave >> 2 : wave >> 1;   // 32-row, column groups
  const int n = (int)P.n, m = (int)P.m, r = P.r;
  const int NT = (r + 31) >> 5, per = side_l ? (NT + 1) >> 1 : (NT + 3) >> 2;       // 32-column blocks, per wave
  const int nb0 = wn * per, nbw = NT - nb0 < per ? (NT - nb0 > 0 ? NT - nb0 : 0) : per;
  const int np_all = (int)((P.s + 31) >> 5);              // K panels
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void*)P.P, (short)0, (int)P.p_bytes, 0x00020000);

  f32x16 acc[4];
#pragma unroll
  for (int nb = 0; nb < 4; ++nb)
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[nb][j] = 0.f;

  // the K loop, instantiated for either side
  auto k_loop = [&](auto side) {
  constexpr bool left = decltype(side)::value;
  constexpr int KC = left ? L_KC : R_KC;
  const int nch = (np_all + KC / 32 - 1) / (KC / 32);

  // ---- gradient chunk: thread (hw, hl) holds four columns of FU gradient rows,
  //   RIGHT: rows l0 + hw + 16 u, columns 128 c + 4 hl;  LEFT: rows 64 c + 4 hw + u, columns l0 + 4 hl
  const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc((void*)P.G, (short)0, m * n * GB, 0x00020000);
  const int row_s = left ? 1 : 16;
  auto row_of = [&](int c, int tf) { return left ? L_KC * c + 4 * (tf >> 5) : (int)l0 + (tf >> 5); };
  auto col_of = [&](int c, int tf) { return (left ? (int)l0 : R_KC * c) + 4 * (tf & 31); };
  // a chunk that lies inside the matrix (uniform)
  auto inside = [&](int c) {
    return left ? L_KC * (c + 1) <= m && (int)l0 + L_BM <= n : (int)l0 + R_BM <= m && R_KC * (c + 1) <= n;
  };
  using graw_t = std::conditional_t<G16, u32x2, u32x4>;
  graw_t graw[FU];   // the chunk in flight
  auto load_g = [&](int c) {   // always FU loads per wave: the waits count them
    const int tf = fresh(tid), row = row_of(c, tf), col = col_of(c, tf);
    const int cc = PLAIN ? col : (col < n - 4 ? col : n - 4);   // the last group's load stays inside the row
    const int off = (row * n + cc) * GB, st = row_s * n * GB;
#pragma unroll
    for (int u = 0; u < FU; ++u) {
      const int o = (row + row_s * u < m) & (col < n) ? off + u * st : 0;
      if constexpr (G16) graw[u] = __builtin_amdgcn_raw_buffer_load_b64(rg, o, 0, 0);
      else graw[u] = __builtin_amdgcn_raw_buffer_load_b128(rg, o, 0, 0);
    }
  };
  // zero what load_g read out of place (rows past m, columns past n), shift a clamped last group
  auto fix_g = [&](int c, float4 (&g)[FU]) {
    const int tf = fresh(tid), row = row_of(c, tf), col = col_of(c, tf), sh = col - (n - 4);
#pragma unroll
    for (int u = 0; u < FU; ++u) {
      if (!PLAIN) {
        const float4 v = g[u];
        if (sh == 1) g[u] = make_float4(v.y, v.z, v.w, 0.f);
        if (sh == 2) g[u] = make_float4(v.z, v.w, 0.f, 0.f);
        if (sh == 3) g[u] = make_float4(v.w, 0.f, 0.f, 0.f);
      }
      if (!(row + row_s * u < m && col < n)) g[u] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };

  // ---- P of chunk c (RIGHT four panels, LEFT two, in the buffer half c & 1): 1 KB (16 rows) per op
  char* Bl = smem + A_BYTES;
  constexpr int NPAN = KC / 32;
  auto b_buf = [&](int c) { return left ? Bl + (c & 1) * (B_BYTES / 2) : Bl; };
  auto issue_b = [&](int c) {
    const int p0 = NPAN * c, npan = np_all - p0 < NPAN ? np_all - p0 : NPAN;
    const int ops = npan * 2 * NT, lf = fresh(tid) & 63;
    char* dst = b_buf(c);
    for (int o = wave; o < ops; o += 8) {
      const int p = o / (2 * NT), q = o - p * 2 * NT;
      const int R = 16 * q + (lf >> 2);
      const int row = R < r ? R : r - 1;      // rows past r repeat the last one; never stored
      const uint32_t off = (uint32_t)(((int64_t)(p0 + p) * r + row) * 64 + (((lf & 3) ^ swz_b(R)) << 4));
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void*)(dst + o * 1024), 16, off, 0, 0, 0);
    }
  };

  auto mfma_chunk = [&](int c) {
    const int p0 = NPAN * c, npan = np_all - p0 < NPAN ? np_all - p0 : NPAN;
    // fragment addresses: A row ar, 16-byte chunk k at k ^ swz(ar), the lane's half in bit 0; B rows
    // one 32-block apart share their permutation
    const int lf = fresh(tid) & 63, ar = 32 * wm + (lf & 31), fa = (lf >> 5) ^ (left ? swz_l(ar) : swz_r(ar));
    const char* Arow = smem + ar * (2 * KC);
    const char* Brow[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
      Brow[ks] = b_buf(c) + (32 * nb0 + (lf & 31)) * 64 + (((2 * ks + (lf >> 5)) ^ swz_b(lf & 31)) << 4);
#pragma unroll 1
    for (int p = 0; p < npan; ++p) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(Arow + (((4 * p + 2 * ks) ^ fa) << 4));
        const char* bp = Brow[ks] + p * NT * 2048;
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
          if (nb < nbw) {   // uniform
            const bf16x8 b = *reinterpret_cast<const bf16x8*>(bp + nb * 2048);
            acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, acc[nb], 0, 0, 0);
          }
        }
      }
    }
  };

  issue_b(0);
  load_g(0);
  for (int c = 0; c < nch; ++c) {
    float4 g[FU];
#pragma unroll
    for (int u = 0; u < FU; ++u) {
      const graw_t x = graw[u];
      if constexpr (G16)
        g[u] = make_float4(__uint_as_float(x.x << 16), __uint_as_float(x.x & 0xFFFF0000u), __uint_as_float(x.y << 16),
                           __uint_as_float(x.y & 0xFFFF0000u));
      else
        g[u] = make_float4(__uint_as_float(x.x), __uint_as_float(x.y), __uint_as_float(x.z), __uint_as_float(x.w));
    }
    if (!inside(c)) fix_g(c, g);
    // ---- block sums, V in bf16, into LDS
    float sel = 0.f;
    const int tf = fresh(tid), hf = tf & 31, wf = tf >> 5;
    const int us = tf & (gl - 1);   // the gradient row (u) whose block sum this lane writes
    // Each lane keeps the sum of one (row, block) of its group, row us (lanes past the FU rows keep
    // zero), so the square root and the division run once per thread instead of once per row;
    // the scales come back by lane permutes.
    float inv = 1.f;
    if (dec) {
#pragma unroll
      for (int u = 0; u < FU; ++u) {
        float ss = sumsq4(g[u]);
        ss = group_sum<gl>(ss);
        sel = us == u ? ss : sel;
      }
      inv = 1.0f / (sqrtf(sel) + U.decomp_eps);
      // LEFT: gradient rows past m are K padding and have to stay zero, also where eps_d is so
      // small that 1 / (0 + eps_d) is infinite
      if (left && L_KC * (c + 1) > m && row_of(c, tf) + row_s * us >= m) inv = 0.f;
    }
    const int grp = ((tf & 63) - us) << 2;   // byte address of the group's first lane
    auto scale = [&](int u) {
      return dec ? __int_as_float(__builtin_amdgcn_ds_bpermute(grp + 4 * u, __float_as_int(inv))) : 1.f;
    };
    if (left) {
      const float i0 = scale(0), i1 = scale(1), i2 = scale(2), i3 = scale(3);
      const float* g0 = &g[0].x; const float* g1 = &g[1].x; const float* g2 = &g[2].x; const float* g3 = &g[3].x;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = 4 * hf + q;
        *reinterpret_cast<uint2*>(smem + i * 128 + (((wf >> 1) ^ swz_l(i)) << 4) + (wf & 1) * 8) =
            make_uint2(pack2(g0[q] * i0, g1[q] * i1), pack2(g2[q] * i2, g3[q] * i3));
      }
    } else {
#pragma unroll
      for (int u = 0; u < FU; ++u) {
        const float i0 = scale(u);
        const int i = wf + 16 * u;   // swz_r(i) = hw ^ u since hw < 16
        *reinterpret_cast<uint2*>(smem + i * 256 + (((hf >> 1) ^ wf ^ u) << 4) + (hf & 1) * 8) =
            make_uint2(pack2(g[u].x * i0, g[u].y * i0), pack2(g[u].z * i0, g[u].w * i0));
      }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's part of P is in LDS
    if (dec && us < FU) {
      const int col = col_of(c, tf), row = row_of(c, tf) + row_s * us;
      const int blk = col >> lgB;
      if (row < m && (blk << lgB) < n) P.ss[(int64_t)row * P.k + blk] = sel;
    }
    __syncthreads();
    // the next chunk's gradient is in flight while this one is multiplied, and P behind it: LEFT into
    // the other half of the buffer, RIGHT (which needs all of it) once every wave is done
    const bool more = c + 1 < nch;
    if (more) load_g(c + 1);
    if (left && more) issue_b(c + 1);
    mfma_chunk(c);
    wg_barrier();                       // A (and RIGHT's B) are free
    if (!left && more) issue_b(c + 1);
  }

  };
  if (side_l) k_loop(std::true_type{});
  else k_loop(std::false_type{});

  // ---- Optimizer_V, 32 rows x 64 columns of the wave at a time through its LDS slab (as the
  // large-tile GEMM's epilogue: 16 lanes x 4 columns per row, four rows per pass)
  float* slab = reinterpret_cast<float*>(smem) + wave * SLAB;
  const int cc = 4 * (lane & 15);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (2 * h >= nbw) break;
    const int col = 32 * (nb0 + 2 * h) + cc;
    const int64_t row0 = l0 + 32 * wm;
    const bool cin = col < r && (cc < 32 || 2 * h + 1 < nbw);
    // the moments of four passes (16 rows) at a time, the next four's loads behind each pass
    bf16x4 e16[4], q16[4];
    float4 e32[4], q32[4];
    auto load_m = [&](int p) {
      const int64_t row = row0 + 4 * p + (lane >> 4);
      if (row < P.L && cin) {
        const int64_t idx = row * P.ldr + col;
        if (MOM16) {
          e16[p & 3] = __builtin_bit_cast(bf16x4, __builtin_nontemporal_load(reinterpret_cast<const u32x2*>((const bf16*)P.e1 + idx)));
          q16[p & 3] = __builtin_bit_cast(bf16x4, __builtin_nontemporal_load(reinterpret_cast<const u32x2*>((const bf16*)P.e2 + idx)));
        } else {
          e32[p & 3] = *reinterpret_cast<const float4*>((const float*)P.e1 + idx);
          q32[p & 3] = *reinterpret_cast<const float4*>((const float*)P.e2 + idx);
        }
      }
    };
#pragma unroll
    for (int p = 0; p < 4; ++p) load_m(p);
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        const int c2 = 32 * b + 8 * gq + 4 * (lane >> 5);
        const f32x16& a = acc[2 * h + b];
        *reinterpret_cast<float4*>(slab + (lane & 31) * SLAB_LD + c2) = make_float4(a[4 * gq], a[4 * gq + 1], a[4 * gq + 2], a[4 * gq + 3]);
      }
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      const int rr = 4 * p + (lane >> 4);
      const int64_t row = row0 + rr;
      if (row < P.L && cin) {
        const float4 v4 = *reinterpret_cast<const float4*>(slab + rr * SLAB_LD + cc);
        const int nin = r - col;   // columns past r (r % 4 != 0): zeros, so the padding stays zero
        const float v[4] = {v4.x, nin > 1 ? v4.y : 0.f, nin > 2 ? v4.z : 0.f, nin > 3 ? v4.w : 0.f};
        const int64_t idx = row * P.ldr + col;
        bf16x4 o;
        if (MOM16) {
          bf16x4 e = e16[p & 3], w = q16[p & 3];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            bf16 ec = e[q], qc = w[q];
            o[q] = f2bf(adam_out_bf16(v[q], ec, qc, U.beta1, U.beta2, U.adam_eps, P.bc1, P.bc2));
            e[q] = ec;
            w[q] = qc;
          }
          __builtin_nontemporal_store(__builtin_bit_cast(u32x2, e), reinterpret_cast<u32x2*>((bf16*)P.e1 + idx));
          __builtin_nontemporal_store(__builtin_bit_cast(u32x2, w), reinterpret_cast<u32x2*>((bf16*)P.e2 + idx));
        } else {
          float4 e = e32[p & 3], q = q32[p & 3];
          o[0] = f2bf(adam_out(v[0], e.x, q.x, U.beta1, U.beta2, U.adam_eps, P.bc1, P.bc2));
          o[1] = f2bf(adam_out(v[1], e.y, q.y, U.beta1, U.beta2, U.adam_eps, P.bc1, P.bc2));
          o[2] = f2bf(adam_out(v[2], e.z, q.z, U.beta1, U.beta2, U.adam_eps, P.bc1, P.bc2));
          o[3] = f2bf(adam_out(v[3], e.w, q.w, U.beta1, U.beta2, U.adam_eps, P.bc1, P.bc2));
          *reinterpret_cast<float4*>((float*)P.e1 + idx) = e;
          *reinterpret_cast<float4*>((float*)P.e2 + idx) = q;
        }
        *reinterpret_cast<bf16x4*>((bf16*)P.N + kp_index(row, col, P.L)) = o;
      }
      if (p + 4 < 8) load_m(p + 4);
    }
  }
}

// Optimizer_M of the fused matrices: the block sums of squares left by k_decproj -> dM and the
// magnitude moments (the same arithmetic as the decomposition's second phase). One thread per
// block, consecutive threads on consecutive blocks: 24 bytes each, bound by HBM.
constexpr int OM_PER_WG = 1024;
__global__ __launch_bounds__(256) void k_opt_m(const FusedProb* __restrict__ probs, GemmUniform U) {
  const uint32_t t = blockIdx.x;
  int lo = 0, hi = U.nprob - 1;
  while (lo < hi) { const int mid = (lo + hi + 1) >> 1; if (probs[mid].tile_m <= t) lo = mid; else hi = mid - 1; }
  const FusedProb& P = probs[lo];
  const int64_t total = P.m * P.k, e0 = (int64_t)(t - P.tile_m) * OM_PER_WG + threadIdx.x;
#pragma unroll
  for (int u = 0; u < OM_PER_WG / 256; ++u) {
    const int64_t i = e0 + 256 * u;
    if (i < total) {
      float e = P.mag1[i], q = P.mag2[i];
      P.dM[i] = adam_out(sqrtf(P.ss[i]), e, q, U.beta1, U.beta2, U.adam_eps, P.bc1, P.bc2);
      P.mag1[i] = e;
      P.mag2[i] = q;
    }
  }
}

}  // namespace

bool decproj_fits(int64_t m, int64_t n, int64_t s, int32_t r, int B, bool decompose) {
  if (r > 256 || n < 4 || 4 * m * n > 0x7FFFFFFFLL) return false;   // four columns per load
  if (s >= 32 && (m < 32 || n < 32)) return false;   // projected onto the long side: one tile, all of K
  return !decompose || B == 32 || B == 64 || B == 128;
}
uint32_t decproj_tiles(int side, int64_t L) {
  const int bm = side == SIDE_LEFT ? L_BM : R_BM;
  return (uint32_t)((L + bm - 1) / bm);
}
uint32_t opt_m_tiles(int64_t mk) { return (uint32_t)((mk + OM_PER_WG - 1) / OM_PER_WG); }

hipError_t launch_decproj(const FusedProb* p, int n, uint32_t total, const GemmUniform& u0, bool plain, bool g16,
                          bool decompose, hipStream_t st) {
  if (!total) return hipSuccess;
  GemmUniform u = u0;
  u.nprob = n;
  const dim3 g(total), b(FNT);
  const int gl = decompose ? u.B >> 2 : 0;
#define DECPROJ(PL, MO, G, H)                                                        \
  if (plain == PL && g16 == H && (u.moment_bf16 != 0) == MO && gl == G) {            \
    hipLaunchKernelGGL((k_decproj<PL, MO, G, H>), g, b, 0, st, p, u);                \
    return hipGetLastError();                                                        \
  }
#define DECPROJ_G(PL, MO, H) DECPROJ(PL, MO, 0, H) DECPROJ(PL, MO, 8, H) DECPROJ(PL, MO, 16, H) DECPROJ(PL, MO, 32, H)
  DECPROJ_G(true, true, false)
  DECPROJ_G(true, false, false)
  DECPROJ_G(false, true, false)
  DECPROJ_G(false, false, false)
  DECPROJ_G(true, true, true)
  DECPROJ_G(true, false, true)
#undef DECPROJ_G
#undef DECPROJ
  return hipErrorInvalidValue;
}
hipError_t launch_opt_m(const FusedProb* p, int n, uint32_t total, const GemmUniform& u0, hipStream_t st) {
  if (!total) return hipSuccess;
  GemmUniform u = u0;
  u.nprob = n;
  hipLaunchKernelGGL(k_opt_m, dim3(total), dim3(256), 0, st, p, u);
  return hipGetLastError();
}
