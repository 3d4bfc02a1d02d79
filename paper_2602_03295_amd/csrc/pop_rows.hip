// Projections of 3 to 32 rows (decode steps of a batch, boundary rows of several prompts: Sec. 3.2 and 3.3) with the work
// around them done in their epilogues: weight streaming, and as few launches as possible.
//
// A work-group owns 16 or 32 weight rows (output columns) and all activation rows; its four waves split K between them and add
// their fp32 sums through LDS in wave order, so no partial product leaves the work-group and whatever follows a projection
// element by element can follow it here:
//   ROWS_ADD    h += scale * C, xn = bf16(h * gamma), and the sum of h^2 over every 16 columns: the next
//               projection's input without its row's 1 / rms, which needs the whole row and is applied by that projection to
//               its fp32 sums (bf16 rounds relative to the value: h * gamma carries the same error as h * rstd * gamma)
//   ROWS_QKV    RoPE and the append to the paged cache; a work-group's columns are rotation pairs
//   ROWS_STORE  fp32 rows
// gate|up and the LM head, whose columns are enough for 64 to 128 per work-group on every CU, have a kernel of their own below
// (rows_wide_kernel; ROWS_GLU and, for many columns, ROWS_STORE).
// Each wave stages its weights and activations (128 bytes of a row per K-step) into a ring of its own with buffer_load ... lds
// and waits for its own loads alone: no barrier before the sums are added.
#include <algorithm>
#include <type_traits>

#include "pop_device.h"
#include "pop_kernels.h"

namespace pop {

namespace rows_impl {

typedef __attribute__((address_space(3))) void* lds_ptr_t;
constexpr uint32_t kOOB = 0x80000000u;   // byte offset beyond any buffer accepted (< 2^31 bytes)

// rows_wide_kernel: blocks of 16 weight rows per work-group (one round of 256 work-groups), stages of a wave's ring.
constexpr int wide_blocks(long long w_rows) { return (int)((w_rows + 4095) / 4096); }
constexpr int wide_stages(int a8, int nb) {        // (a8 = 0: 32 KB are left for the normalised rows)
  const int st = (a8 ? 160 : 128) / (4 * (2 * nb + a8));
  return st < 4 ? st : 4;
}
constexpr int wide_ring_bytes(int a8, int nb) { return 4 * wide_stages(a8, nb) * (nb * 2048 + a8 * 1024); }
constexpr int wide_norm_lds(int M, int K) { return M * (K * 2 + 16); }

// A8: groups of 8 activation rows; NB: blocks of 16 columns; ST: stages of a wave's ring
template <int A8, int NB, int ST, int EPI>
__global__ __launch_bounds__(256) void rows_kernel(RowsArgs p) {
#if defined(__HIP_DEVICE_COMPILE__)  // the buffer-resource builtins exist in the device pass only
  constexpr int MB = (A8 + 1) / 2;                 // blocks of 16 activation rows
  constexpr int STAGE = NB * 2048 + A8 * 1024, LOADS = 2 * NB + A8;
  static_assert((ST - 1) * LOADS < 64, "vmcnt is a 6-bit counter");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];   // [4][ST][STAGE], float4 [4][MB][NB][64], rstd
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wg = blockIdx.x;
  unsigned char* const ring = smem + wave * (ST * STAGE);
  float4* const sums = reinterpret_cast<float4*>(smem + 4 * ST * STAGE);
  float* const rstd = reinterpret_cast<float*>(sums + 4 * MB * NB * 64);

  // ---- the rows' sums of squares, as the previous projection's work-groups left them: requested here, added behind the loop
  typedef __attribute__((__vector_size__(16))) unsigned int u32x4_t;
  u32x4_t ssq[2 * A8][2];
  if (p.n_sumsq > 0) {
    const __amdgpu_buffer_rsrc_t rS = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.sumsq_in), 0,
                                                                        (uint32_t)p.M * p.n_sumsq * 4, 0x00020000);
#pragma unroll
    for (int i = 0; i < 2 * A8; ++i)
#pragma unroll
      for (int u = 0; u < 2; ++u) {               // (range-checked: zeros beyond the row's sums and beyond the last row)
        const int q = u * 256 + lane * 4;
        ssq[i][u] = __builtin_amdgcn_raw_buffer_load_b128(
            rS, q < p.n_sumsq ? (uint32_t)((wave * 2 * A8 + i) * p.n_sumsq + q) * 4 : kOOB, 0, 0);
      }
  }

  // ---- columns of the work-group; ROWS_QKV: the first half are dims pair0, pair0 + 1, .. of a head, the others their partners
  constexpr int COLS = NB * 16, PAIRS = COLS / 2;
  const int half = p.hd >> 1;
  const int head = EPI == ROWS_QKV ? wg / (p.hd / COLS) : 0, pair0 = EPI == ROWS_QKV ? wg % (p.hd / COLS) * PAIRS : 0;
  auto column = [&](int r) {
    return EPI == ROWS_QKV ? head * p.hd + pair0 + r % PAIRS + r / PAIRS * half : wg * COLS + r;
  };

  const __amdgpu_buffer_rsrc_t rA = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(p.x), 0, (uint32_t)((long long)p.M * p.K * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rW = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(p.W), 0, (uint32_t)((long long)p.N * p.K * 2), 0x00020000);
  // A wave-load fills 8 rows of 128 bytes; chunk c of row r is stored at c ^ ((r >> 1) & 7) (see the tiled GEMM)
  const int lr = lane >> 3;
  uint32_t off_w[2 * NB], off_a[A8];
#pragma unroll
  for (int j = 0; j < 2 * NB; ++j)
    off_w[j] = (uint32_t)((long long)column(j * 8 + lr) * p.K * 2) + ((lane & 7) ^ (((j & 1) * 4 + (lr >> 1)) & 7)) * 16;
#pragma unroll
  for (int j = 0; j < A8; ++j) {
    const int row = j * 8 + lr;
    off_a[j] = row < p.M ? (uint32_t)((long long)row * p.K * 2) + ((lane & 7) ^ (((j & 1) * 4 + (lr >> 1)) & 7)) * 16 : kOOB;
  }
  // this wave's K-steps, started at a different place in every work-group (rows of W lie a multiple of 4 KB apart: work-groups
  // that walk K together meet on a few memory channels)
  const int nk_all = p.K >> 6, k_lo = nk_all * wave / 4, nk = nk_all * (wave + 1) / 4 - k_lo;
  const int rot = (int)((long long)wg * nk / gridDim.x);
  auto issue = [&](int i) {                        // the wave's i-th K-step (beyond the last: masked)
    int k = i + rot;
    if (k >= nk) k -= nk;
    const uint32_t mask = i < nk ? 0u : kOOB;
    const int off = (k_lo + k) * 128;
    unsigned char* s = ring + (i % ST) * STAGE;
#pragma unroll
    for (int j = 0; j < 2 * NB; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rW, (lds_ptr_t)(s + j * 1024), 16, off_w[j] | mask, off, 0, 2 /* streamed */);
#pragma unroll
    for (int j = 0; j < A8; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rA, (lds_ptr_t)(s + NB * 2048 + j * 1024), 16, off_a[j] | mask, off, 0, 0);
  };
#pragma unroll
  for (int i = 0; i < ST - 1; ++i) issue(i);

  // v_mfma_f32_16x16x32_bf16 with W first: lane l receives columns 4 (l / 16) .. + 3 of activation row l % 16
  const int r16 = lane & 15, g4 = lane >> 4;
  const int frag = r16 * 128, key = (r16 >> 1) & 7;
  // (an odd number of 8-row groups: the last block's upper rows repeat its lower ones, and are never stored)
  const int frag_last = A8 % 2 ? (r16 & 7) * 128 : frag, key_last = A8 % 2 ? ((r16 & 7) >> 1) & 7 : key;
  floatx4_t acc[MB][NB];
#pragma unroll
  for (int j = 0; j < MB; ++j)
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[j][n] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  for (int i = 0; i < nk; ++i) {
    issue(i + ST - 1);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((ST - 1) * LOADS) : "memory");
    const unsigned char* s = ring + (i % ST) * STAGE;
    bf16x8_t w[2][NB], a[2][MB];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int n = 0; n < NB; ++n)
        w[ks][n] = *reinterpret_cast<const bf16x8_t*>(s + n * 2048 + frag + ((4 * ks + g4) ^ key) * 16);
#pragma unroll
      for (int j = 0; j < MB; ++j) {
        const bool odd = A8 % 2 && j == MB - 1;
        a[ks][j] = *reinterpret_cast<const bf16x8_t*>(s + NB * 2048 + j * 2048 + (odd ? frag_last : frag) +
                                                      ((4 * ks + g4) ^ (odd ? key_last : key)) * 16);
      }
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int j = 0; j < MB; ++j)
#pragma unroll
        for (int n = 0; n < NB; ++n)
          acc[j][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][n], a[ks][j], acc[j][n], 0, 0, 0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the next iteration refills this slot's predecessor, then this slot
  }
#pragma unroll
  for (int j = 0; j < MB; ++j)
#pragma unroll
    for (int n = 0; n < NB; ++n)
      sums[((wave * MB + j) * NB + n) * 64 + lane] = make_float4(acc[j][n][0], acc[j][n][1], acc[j][n][2], acc[j][n][3]);
  if (p.n_sumsq > 0) {
#pragma unroll
    for (int i = 0; i < 2 * A8; ++i) {
      const float4 a = __builtin_bit_cast(float4, ssq[i][0]), b = __builtin_bit_cast(float4, ssq[i][1]);
      const float total = wave_sum_rows(((a.x + a.y) + (a.z + a.w)) + ((b.x + b.y) + (b.z + b.w)));
      if (lane == 0) rstd[wave * 2 * A8 + i] = rsqrtf(total / (float)p.d_norm + p.eps);
    }
  } else if (lane < 2 * A8) {
    rstd[wave * 2 * A8 + lane] = 1.f;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // masked loads still target this group's LDS
  __syncthreads();
  // ---- a wave finishes a block of 16 rows x 16 columns (ROWS_QKV: x all columns, so that a lane holds both halves of its pairs)
  constexpr int NQ = EPI == ROWS_QKV ? NB : 1;
  if (wave >= MB * NB / NQ) return;
  const int mb = wave / (NB / NQ), nb = wave % (NB / NQ);
  float c[NQ][4];
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
#pragma unroll
    for (int e = 0; e < 4; ++e) c[n][e] = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float4 v = sums[((w * MB + mb) * NB + nb + n) * 64 + lane];
      c[n][0] += v.x; c[n][1] += v.y; c[n][2] += v.z; c[n][3] += v.w;
    }
  }
  const int m = mb * 16 + r16, n0 = wg * COLS + nb * 16 + g4 * 4;
  const bool valid = m < p.M;
  const float rs = valid ? rstd[m] : 0.f;
  if constexpr (EPI == ROWS_STORE) {
    if (valid)
      *reinterpret_cast<float4*>(p.out + (size_t)m * p.ldo + n0) =
          make_float4(c[0][0] * rs, c[0][1] * rs, c[0][2] * rs, c[0][3] * rs);
  } else if constexpr (EPI == ROWS_ADD) {
    float4* o = reinterpret_cast<float4*>(p.out + (size_t)(valid ? m : 0) * p.ldo + n0);
    float4 hv = *o;
    hv.x += c[0][0] * p.scale; hv.y += c[0][1] * p.scale; hv.z += c[0][2] * p.scale; hv.w += c[0][3] * p.scale;
    if (valid) *o = hv;
    if (p.gamma) {
      const float4 g = *reinterpret_cast<const float4*>(p.gamma + n0);
      if (valid)
        *reinterpret_cast<uint2*>(p.xn + (size_t)m * p.N + n0) =
            make_uint2(pack_bf16x2(hv.x * g.x, hv.y * g.y), pack_bf16x2(hv.z * g.z, hv.w * g.w));
      float q = (hv.x * hv.x + hv.y * hv.y) + (hv.z * hv.z + hv.w * hv.w);
      q += __shfl_xor(q, 16, 64);
      q += __shfl_xor(q, 32, 64);
      if (valid && g4 == 0) p.sumsq_out[(size_t)m * (p.N / 16) + wg * NB + nb] = q;
    }
  } else {
    // lo, hi: this lane's rotation pairs; with 16 columns its own four values are one half of them, the lane 32 on has the other
    const bool rotate = head < p.n_q_heads + p.n_kv_heads;
    const int i0 = pair0 + (NB == 1 ? 4 * (g4 & 1) : 4 * g4);       // pair index of the first
    float lo[4], hi[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (NB == 1) {
        const float own = c[0][e] * rs, other = __shfl_xor(own, 32, 64);
        lo[e] = g4 < 2 ? own : other;
        hi[e] = g4 < 2 ? other : own;
      } else {
        lo[e] = c[0][e] * rs;
        hi[e] = c[NQ - 1][e] * rs;
      }
    }
    if (valid) {
      if (rotate) {
        const float4* cs = reinterpret_cast<const float4*>(p.cs + (size_t)m * half + i0);
        const float4 c01 = cs[0], c23 = cs[1];
        const float cc[4] = {c01.x, c01.z, c23.x, c23.z}, sn[4] = {c01.y, c01.w, c23.y, c23.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float a = lo[e] * cc[e] - hi[e] * sn[e], b = hi[e] * cc[e] + lo[e] * sn[e];
          lo[e] = a;
          hi[e] = b;
        }
      }
      const int hh = head < p.n_q_heads ? head : rotate ? head - p.n_q_heads : head - p.n_q_heads - p.n_kv_heads;
      const int s = p.slot[m];
      const size_t entry = (((size_t)(s / p.page_size) * p.n_kv_heads + hh) * p.page_size + (s % p.page_size)) * p.hd;
      const float inv = rotate ? p.kvq.k_inv : p.kvq.v_inv;
      bf16_t* pool = rotate ? p.k_pool : p.v_pool;
      auto store = [&](const float (&x)[4], int dim) {
        const uint2 bf = make_uint2(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]));
        if (head < p.n_q_heads)
          *reinterpret_cast<uint2*>(p.q_out + ((size_t)m * p.n_q_heads + head) * p.hd + dim) = bf;
        else if (p.kvq.fp8)
          *reinterpret_cast<uint32_t*>(reinterpret_cast<unsigned char*>(pool) + entry + dim) =
              e4m3_pack4(x[0] * inv, x[1] * inv, x[2] * inv, x[3] * inv);
        else
          *reinterpret_cast<uint2*>(pool + entry + dim) = bf;
      };
      if (NB == 2 || g4 < 2) store(lo, i0);
      if (NB == 2 || g4 >= 2) store(hi, i0 + half);
    }
  }
#endif
}

// gate|up (ROWS_GLU) and LM head (ROWS_STORE): a work-group owns NB blocks of 16 weight rows, NB chosen so that the work-groups
// are one round of at most 256.  What counts is that every CU streams weights and all of them the same amount: a CU has no
// more than the 32 KB of its L1 on the way, so that CUs without a work-group are bandwidth lost (the 64 x 128 tiles of the tiled
// GEMM leave 32 of 256 idle at 28672 columns, 64 at 24576, 124 at 16864).  The activations, which every work-group reads
// whole, are 1 : 2 NB of the weights with 8 rows.  Waves split K and add their sums in LDS as in rows_kernel.
// ROWS_GLU: a block of 16 weight rows is 8 gate and the 8 up rows of the same output columns, which makes any number of blocks a
// whole number of columns; lane l + 32 holds the up values of lane l's gate values.
// A8 = 0: one or two fp32 rows p.xf, which the work-group normalises (Sec. 2.1) into LDS with the thread layout, summation
// order and roundings of rmsnorm_kernel while its first weights travel; the ring then holds weights alone.
// Measured against the kernels it replaces, us: gate|up (28672 x 4096) of 8 rows 42.3 -> 37.9 (6.2 TB/s; loads alone take 38),
// of one row 41.1 -> 38.1, (24576 x 4096) of 32 rows 40.5 -> 35.6; LM head (16864 x 4096) of 32 rows 35.8 -> 24.7.
template <int A8, int NB, int EPI>
__global__ __launch_bounds__(256) void rows_wide_kernel(RowsArgs p) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr bool NORM = A8 == 0;
  constexpr int MB = NORM ? 1 : (A8 + 1) / 2;
  constexpr int STAGE = NB * 2048 + A8 * 1024, LOADS = 2 * NB + A8, ST = wide_stages(A8, NB);
  static_assert(ST >= 2 && (ST - 1) * LOADS < 64, "vmcnt is a 6-bit counter");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];   // [4][ST][STAGE], then float4 [4][MB][NB][64], rstd
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wg = blockIdx.x;
  unsigned char* const ring = smem + wave * (ST * STAGE);
  float4* const sums = reinterpret_cast<float4*>(smem);
  float* const rstd = reinterpret_cast<float*>(sums + 4 * MB * NB * 64);
  unsigned char* const xn_lds = smem + 4 * ST * STAGE;                      // NORM: bf16 [M][K], float [M][4]
  float4 h[2][8], gam[8];                           // NORM: this thread's share of the rows and of the norm scale
  if constexpr (NORM) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int i = (j * 256 + (int)threadIdx.x) * 4;
      gam[j] = i < p.K ? *reinterpret_cast<const float4*>(p.gamma + i) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int i = (j * 256 + (int)threadIdx.x) * 4;
        h[m][j] = m < p.M && i < p.K ? *reinterpret_cast<const float4*>(p.xf + (size_t)m * p.K + i) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
  }

  typedef __attribute__((__vector_size__(16))) unsigned int u32x4_t;
  u32x4_t ssq[NORM ? 1 : 2 * A8][2];                // the rows' sums of squares (see rows_kernel)
  if (!NORM && p.n_sumsq > 0) {
    const __amdgpu_buffer_rsrc_t rS = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.sumsq_in), 0,
                                                                        (uint32_t)p.M * p.n_sumsq * 4, 0x00020000);
#pragma unroll
    for (int i = 0; i < 2 * A8; ++i)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int q = u * 256 + lane * 4;
        ssq[i][u] = __builtin_amdgcn_raw_buffer_load_b128(
            rS, q < p.n_sumsq ? (uint32_t)((wave * 2 * A8 + i) * p.n_sumsq + q) * 4 : kOOB, 0, 0);
      }
  }

  constexpr bool GLU = EPI == ROWS_GLU;
  constexpr int COLS = GLU ? NB * 8 : NB * 16;      // output columns of the work-group
  const __amdgpu_buffer_rsrc_t rA = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(p.x), 0, (uint32_t)((long long)p.M * p.K * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rW = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(p.W), 0, (uint32_t)((long long)p.N * (GLU ? 2 : 1) * p.K * 2), 0x00020000);
  const int lr = lane >> 3;
  uint32_t off_w[2 * NB], off_a[NORM ? 1 : A8];
#pragma unroll
  for (int j = 0; j < 2 * NB; ++j) {
    const int col = wg * COLS + (GLU ? (j >> 1) * 8 + lr : j * 8 + lr);
    const int row = col + (GLU && (j & 1) ? p.N : 0);
    off_w[j] = col < p.N ? (uint32_t)((long long)row * p.K * 2) + ((lane & 7) ^ (((j & 1) * 4 + (lr >> 1)) & 7)) * 16 : kOOB;
  }
#pragma unroll
  for (int j = 0; j < A8; ++j) {
    const int row = j * 8 + lr;
    off_a[j] = row < p.M ? (uint32_t)((long long)row * p.K * 2) + ((lane & 7) ^ (((j & 1) * 4 + (lr >> 1)) & 7)) * 16 : kOOB;
  }
  const int nk_all = p.K >> 6, k_lo = nk_all * wave / 4, nk = nk_all * (wave + 1) / 4 - k_lo;
  const int rot = (int)((long long)wg * nk / gridDim.x);
  auto issue = [&](int i, int stage) {              // the wave's i-th K-step (beyond the last: masked)
    int k = i + rot;
    if (k >= nk) k -= nk;
    const uint32_t mask = i < nk ? 0u : kOOB;
    const int off = (k_lo + k) * 128;
    unsigned char* s = ring + stage * STAGE;
#pragma unroll
    for (int j = 0; j < 2 * NB; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rW, (lds_ptr_t)(s + j * 1024), 16, off_w[j] | mask, off, 0, 2 /* streamed */);
#pragma unroll
    for (int j = 0; j < A8; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rA, (lds_ptr_t)(s + NB * 2048 + j * 1024), 16, off_a[j] | mask, off, 0, 0);
  };
#pragma unroll
  for (int i = 0; i < ST - 1; ++i) issue(i, i);
  if constexpr (NORM) {
    // LDS accesses in assembly: beside loads into LDS that are under way the compiler waits for all of those before each of its own
    const uint32_t xn_addr = (uint32_t)(size_t)(lds_ptr_t)xn_lds, red = xn_addr + (uint32_t)(p.M * p.K * 2);
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      float ss = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if ((j * 256 + (int)threadIdx.x) * 4 < p.K)
          ss += h[m][j].x * h[m][j].x + h[m][j].y * h[m][j].y + h[m][j].z * h[m][j].z + h[m][j].w * h[m][j].w;
      ss = wave_sum(ss);
      if (m < p.M && lane == 0) asm volatile("ds_write_b32 %0, %1" ::"v"(red + (m * 4 + wave) * 4), "v"(ss) : "memory");
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (not __syncthreads: the weights stay in flight)
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      if (m >= p.M) break;
      floatx4_t part;
      asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(part) : "v"(red + m * 16) : "memory");
      const float total = part[0] + part[1] + part[2] + part[3];
      const float r = rsqrtf(total / (float)p.K + p.eps);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int i = (j * 256 + (int)threadIdx.x) * 4;
        if (i < p.K) {
          const float4 g = gam[j];
          const uint2 v = make_uint2(pack_bf16x2(h[m][j].x * r * g.x, h[m][j].y * r * g.y), pack_bf16x2(h[m][j].z * r * g.z, h[m][j].w * r * g.w));
          asm volatile("ds_write_b64 %0, %1" ::"v"(xn_addr + (uint32_t)(m * p.K + i) * 2), "v"(__builtin_bit_cast(unsigned long long, v)) : "memory");
        }
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
  }

  const int r16 = lane & 15, g4 = lane >> 4;
  const int frag = r16 * 128, key = (r16 >> 1) & 7;
  const int frag_last = A8 % 2 ? (r16 & 7) * 128 : frag, key_last = A8 % 2 ? ((r16 & 7) >> 1) & 7 : key;
  floatx4_t acc[MB][NB];
#pragma unroll
  for (int j = 0; j < MB; ++j)
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[j][n] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  // NORM: lanes of rows that do not exist repeat the last one (never stored)
  const unsigned char* const xn_lane = xn_lds + (size_t)min(r16, p.M - 1) * p.K * 2 + g4 * 16;
  int stage = 0;
  for (int i = 0; i < nk; ++i) {
    issue(i + ST - 1, stage == 0 ? ST - 1 : stage - 1);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((ST - 1) * LOADS) : "memory");
    const unsigned char* s = ring + stage * STAGE;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      bf16x8_t w[NB], a[MB];
#pragma unroll
      for (int n = 0; n < NB; ++n)
        w[n] = *reinterpret_cast<const bf16x8_t*>(s + n * 2048 + frag + ((4 * ks + g4) ^ key) * 16);
      if constexpr (NORM) {
        const int k = i + rot >= nk ? i + rot - nk : i + rot;
        a[0] = *reinterpret_cast<const bf16x8_t*>(xn_lane + (k_lo + k) * 128 + ks * 64);
      } else {
#pragma unroll
      for (int j = 0; j < MB; ++j) {
        const bool odd = A8 % 2 && j == MB - 1;
        a[j] = *reinterpret_cast<const bf16x8_t*>(s + NB * 2048 + j * 2048 + (odd ? frag_last : frag) +
                                                  ((4 * ks + g4) ^ (odd ? key_last : key)) * 16);
      }
      }
#pragma unroll
      for (int j = 0; j < MB; ++j)
#pragma unroll
        for (int n = 0; n < NB; ++n) acc[j][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[n], a[j], acc[j][n], 0, 0, 0);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the next iteration refills this slot's predecessor, then this slot
    stage = stage == ST - 1 ? 0 : stage + 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // masked loads still target this group's LDS
  __syncthreads();                                   // the sums take the place of the rings
#pragma unroll
  for (int j = 0; j < MB; ++j)
#pragma unroll
    for (int n = 0; n < NB; ++n)
      sums[((wave * MB + j) * NB + n) * 64 + lane] = make_float4(acc[j][n][0], acc[j][n][1], acc[j][n][2], acc[j][n][3]);
  if (!NORM && p.n_sumsq > 0) {
#pragma unroll
    for (int i = 0; i < 2 * A8; ++i) {
      const float4 a = __builtin_bit_cast(float4, ssq[i][0]), b = __builtin_bit_cast(float4, ssq[i][1]);
      const float total = wave_sum_rows(((a.x + a.y) + (a.z + a.w)) + ((b.x + b.y) + (b.z + b.w)));
      if (lane == 0) rstd[wave * 2 * A8 + i] = rsqrtf(total / (float)p.d_norm + p.eps);
    }
  } else if (lane < 2 * A8) {
    rstd[wave * 2 * A8 + lane] = 1.f;
  }
  __syncthreads();
  const float k0 = glu_k0(p.act), k1 = glu_k1(p.act);
  for (int blk = wave; blk < MB * NB; blk += 4) {    // 16 rows x 16 weight rows each
    const int mb = blk / NB, n = blk % NB, m = mb * 16 + r16;
    const bool valid = m < p.M;
    const float rs = NORM ? 1.f : valid ? rstd[m] : 0.f;
    float c[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float4 v = sums[((w * MB + mb) * NB + n) * 64 + lane];
      c[0] += v.x; c[1] += v.y; c[2] += v.z; c[3] += v.w;
    }
    if constexpr (GLU) {
      const int col = wg * COLS + n * 8 + (g4 & 1) * 4;
      float u[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float up = __shfl_xor(c[e], 32, 64);   // (lanes 0 to 31; the others compute nothing of use)
        u[e] = glu_act(c[e] * rs, k0, k1) * (up * rs);
      }
      if (valid && g4 < 2 && col < p.N)
        *reinterpret_cast<uint2*>(p.xn + (size_t)m * p.ldo + col) = make_uint2(pack_bf16x2(u[0], u[1]), pack_bf16x2(u[2], u[3]));
    } else {
      const int col = wg * COLS + n * 16 + g4 * 4;
      if (valid && col < p.N)
        *reinterpret_cast<float4*>(p.out + (size_t)m * p.ldo + col) = make_float4(c[0] * rs, c[1] * rs, c[2] * rs, c[3] * rs);
    }
  }
#endif
}

template <int A8, int NB, int EPI>
hipError_t launch_wide_cfg(const RowsArgs& a, hipStream_t st) {
  constexpr int MB = A8 ? (A8 + 1) / 2 : 1, ring = wide_ring_bytes(A8, NB), sums = 4 * MB * NB * 1024 + 8 * A8 * 4;
  static_assert(ring >= sums && ring <= 160 * 1024, "LDS budget of a gfx950 CU");
  const int smem = ring + (A8 ? 0 : wide_norm_lds(a.M, a.K));
  static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&rows_wide_kernel<A8, NB, EPI>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, A8 ? ring : 160 * 1024);
  if (attr_err != hipSuccess) return attr_err;
  constexpr int cols = EPI == ROWS_GLU ? NB * 8 : NB * 16;
  hipLaunchKernelGGL((rows_wide_kernel<A8, NB, EPI>), dim3((a.N + cols - 1) / cols), dim3(256), smem, st, a);
  return hipGetLastError();
}

template <int EPI>
hipError_t launch_wide(const RowsArgs& a, hipStream_t st) {
  auto rows = [&](auto nb_c) {
    constexpr int NB = decltype(nb_c)::value;
    if (a.xf) return launch_wide_cfg<0, NB, EPI>(a, st);
    if (a.M <= 8) return launch_wide_cfg<1, NB, EPI>(a, st);
    if (a.M <= 16) return launch_wide_cfg<2, NB, EPI>(a, st);
    if (a.M <= 24) return launch_wide_cfg<3, NB, EPI>(a, st);
    return launch_wide_cfg<4, NB, EPI>(a, st);
  };
  switch (wide_blocks(EPI == ROWS_GLU ? 2LL * a.N : a.N)) {
    case 4: return rows(std::integral_constant<int, 4>{});
    case 5: return rows(std::integral_constant<int, 5>{});
    case 6: return rows(std::integral_constant<int, 6>{});
    case 7: return rows(std::integral_constant<int, 7>{});
    default: return rows(std::integral_constant<int, 8>{});
  }
}

template <int A8, int NB, int ST, int EPI>
hipError_t launch_cfg(const RowsArgs& a, hipStream_t st) {
  constexpr int MB = (A8 + 1) / 2;
  constexpr int smem = 4 * ST * (NB * 2048 + A8 * 1024) + 4 * MB * NB * 64 * 16 + 8 * A8 * 4;
  static_assert(smem <= 160 * 1024, "LDS budget of a gfx950 CU");
  // once per instantiation; the initialisation of a function-local static is thread-safe
  static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&rows_kernel<A8, NB, ST, EPI>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  if (attr_err != hipSuccess) return attr_err;
  hipLaunchKernelGGL((rows_kernel<A8, NB, ST, EPI>), dim3(a.N / (16 * NB)), dim3(256), smem, st, a);
  return hipGetLastError();
}

template <int EPI>
hipError_t launch_epi(const RowsArgs& a, hipStream_t st) {
  // 16 columns per work-group; from 17 rows on, whose activations outweigh such a work-group's weights, 32 where there would be
  // more than 256 work-groups (QKV of 6144 columns, 32 rows: 24.5 -> 16.9 us; O of 4096: 11.0 -> 12.9).
  // Two to four stages: 32 to 48 KB are requested per CU, and its L1 has no room for more; deeper rings, as deep as LDS
  // allows, were slower (O and down of 8 rows, mean of both, by stages: 12 15.5 us, 8 15.0, 6 14.7, 5 14.4, 4 14.35, 3 14.7, 2 17.4;
  // QKV 6 12.9, 3 12.4, 2 12.1; 14 rows 9 16.4, 4 16.1, 3 15.8, 2 17.5; O of 32 rows 6 12.3, 4 12.3, 3 11.7, 2 12.2).
  const bool one = a.N / 16 <= 256;
  if (a.M <= 8) return one ? launch_cfg<1, 1, 4, EPI>(a, st) : launch_cfg<1, 1, 2, EPI>(a, st);
  if (a.M <= 16) return one ? launch_cfg<2, 1, 3, EPI>(a, st) : launch_cfg<2, 1, 2, EPI>(a, st);
  if (a.M <= 24) return one ? launch_cfg<3, 1, 3, EPI>(a, st) : launch_cfg<3, 2, 3, EPI>(a, st);
  return one ? launch_cfg<4, 1, 3, EPI>(a, st) : launch_cfg<4, 2, 3, EPI>(a, st);
}

}  // namespace rows_impl
using namespace rows_impl;

bool rows_supported(int M, int N, int K) {
  return M >= 3 && M <= 32 && N % 32 == 0 && K % 64 == 0 && K >= 256 && (long long)N * K * 2 < (1LL << 31);
}

// 64 to 128 weight rows per CU: fewer leave the ring's loads short of the memory, more are several rounds, for which the tiled
// GEMM with two work-groups per CU is the better one.
bool rows_wide_supported(int M, int N, int K, int epilogue) {
  const long long w_rows = epilogue == ROWS_GLU ? 2LL * N : N;
  return (epilogue == ROWS_GLU || epilogue == ROWS_STORE) && M >= 3 && M <= 32 && N % (epilogue == ROWS_GLU ? 8 : 4) == 0 &&
         K % 64 == 0 && K >= 256 && wide_blocks(w_rows) >= 4 && wide_blocks(w_rows) <= 8 && w_rows * K * 2 < (1LL << 31);
}

bool rows_wide_norm_supported(int M, int N, int K, int epilogue) {
  return M >= 1 && M <= 2 && K <= 8192 && rows_wide_supported(3, N, K, epilogue) &&
         wide_ring_bytes(0, wide_blocks(epilogue == ROWS_GLU ? 2LL * N : N)) + wide_norm_lds(M, K) <= 160 * 1024;
}

hipError_t launch_rows(const RowsArgs& a, hipStream_t st) {
  const bool wide = a.xf ? rows_wide_norm_supported(a.M, a.N, a.K, a.epilogue) && a.gamma && a.n_sumsq == 0
                         : rows_wide_supported(a.M, a.N, a.K, a.epilogue);
  if (a.xf && !wide) return hipErrorInvalidValue;
  if (!(wide || rows_supported(a.M, a.N, a.K)) || a.ldo % 4 || a.n_sumsq % 4 || a.n_sumsq > kRowScaledSums) return hipErrorInvalidValue;
  if (wide) return a.epilogue == ROWS_GLU ? launch_wide<ROWS_GLU>(a, st) : launch_wide<ROWS_STORE>(a, st);
  switch (a.epilogue) {
    case ROWS_ADD: return launch_epi<ROWS_ADD>(a, st);
    case ROWS_QKV:
      if (a.hd % 32 || a.N != (a.n_q_heads + 2 * a.n_kv_heads) * a.hd || a.page_size < 1) return hipErrorInvalidValue;
      return launch_epi<ROWS_QKV>(a, st);
    case ROWS_STORE: return launch_epi<ROWS_STORE>(a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace pop
