// Decode-step kernels: one row per sequence through a full layer against the paged KV cache (few-row
// projections, attention over the cache, for one or two rows with RoPE and the append of the new entry inside, greedy
// choice).
// They carry the boundary token of Sec. 3.3 ("Boundary Handling for the Last Input Token": x_N is
// the first decode step with the full model) and pop_decode_step (Sec. 3.2, decode operator).
// Every projection streams its weights once: HBM-bound (three and more rows go through the tiled GEMM, three and four of a
// K that is no multiple of 64 through the GEMV kernel here).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "pop_device.h"
#include "pop_kernels.h"

namespace pop {

namespace decode_impl {

__device__ __forceinline__ float glu_act_f(float g, int act) {
  if (act == 0) return g / (1.f + __expf(-g));
  const float u = 0.7978845608028654f * (g + 0.044715f * g * g * g);
  return 0.5f * g * (1.f + tanhf(u));
}

// acc += sum of the eight bf16 products of w and x, with v_dot2_f32_bf16 (two products and the fp32 sum per
// instruction, operands taken as packed bf16 without conversion): a quarter of the vector instructions of
// converting to fp32 and multiplying, which is what kept the forms with several batch rows below the HBM rate.
__device__ __forceinline__ void fma8(float (&acc), const uint4& w, const uint4& x) {
  typedef __bf16 bf2_t __attribute__((ext_vector_type(2)));
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf2_t, w.x), __builtin_bit_cast(bf2_t, x.x), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf2_t, w.y), __builtin_bit_cast(bf2_t, x.y), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf2_t, w.z), __builtin_bit_cast(bf2_t, x.z), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf2_t, w.w), __builtin_bit_cast(bf2_t, x.w), acc, false);
}

// Each wave owns RW weight rows (for GLU: RW gate rows and the matching RW up rows) and all M batch
// rows; lanes stride over K in 16-byte chunks; fp32 accumulation, wave reduction at the end.
// The K loop is unrolled by U with all weight loads of an unrolled step issued before the first
// multiply: with one row per step a wave has too few bytes in flight to cover HBM latency.
// NORM: the M input rows are fp32 rows xf that are RMS-normalised first (Sec. 2.1, the LN of the layer
// equations): every work-group computes the M normalised bf16 rows into LDS, with the thread layout, the
// summation order and the roundings of rmsnorm_kernel (same bits), which saves the launch of that kernel
// and the round trip of its output.
template <int M, int EPI, int RW, int U, bool NORM>
__global__ __launch_bounds__(256) void gemv_kernel(const bf16_t* __restrict__ x, const float* __restrict__ xf,
                                                   const float* __restrict__ gamma, float eps,
                                                   const bf16_t* __restrict__ W, void* __restrict__ out, int N, int K,
                                                   long long ldo, int act, float scale /* ADD: out += scale * C */,
                                                   int m_valid /* rows that exist (<= M); the others repeat the last */) {
  constexpr int NR = EPI == GEMV_GLU_BF16 ? 2 * RW : RW;  // weight rows streamed per wave
  typedef __attribute__((__vector_size__(16))) unsigned int u32x4_t;
  extern __shared__ __attribute__((aligned(16))) unsigned char gemv_smem[];   // NORM: bf16 [M][K], then float [M][4]
  const bf16_t* xs = reinterpret_cast<const bf16_t*>(gemv_smem);
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int n0 = (blockIdx.x * 4 + wave) * RW;
  const bf16_t* wr[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    int row;
    if (EPI == GEMV_GLU_BF16) row = (r < RW ? 0 : N) + min(n0 + (r % RW), N - 1);
    else row = min(n0 + r, N - 1);
    wr[r] = W + (size_t)row * K;
  }
  int k = lane * 8;
  // NORM: the weights of the first unrolled step are requested before the rows are normalised, so that
  // they travel meanwhile
  u32x4_t wl[U][NR];
  bool preloaded = NORM && k + (U - 1) * 512 < K;
  if (preloaded) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int r = 0; r < NR; ++r)
        wl[u][r] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(wr[r] + k + u * 512));
  }
  if (NORM) {
    bf16_t* xw = reinterpret_cast<bf16_t*>(gemv_smem);
    float* red = reinterpret_cast<float*>(gemv_smem + (size_t)M * K * 2);
#pragma unroll 1
    for (int m = 0; m < M; ++m) {
      const float* xr = xf + (size_t)m * K;
      float4 v[8];
      float ss = 0.f;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int i = (j * 256 + threadIdx.x) * 4;
        if (i < K) {
          v[j] = *reinterpret_cast<const float4*>(xr + i);
          ss += v[j].x * v[j].x + v[j].y * v[j].y + v[j].z * v[j].z + v[j].w * v[j].w;
        }
      }
      ss = wave_sum(ss);
      if ((threadIdx.x & 63) == 0) red[m * 4 + (threadIdx.x >> 6)] = ss;
      __syncthreads();
      const float total = red[m * 4] + red[m * 4 + 1] + red[m * 4 + 2] + red[m * 4 + 3];
      const float rstd = rsqrtf(total / (float)K + eps);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int i = (j * 256 + threadIdx.x) * 4;
        if (i < K) {
          const float4 gg = *reinterpret_cast<const float4*>(gamma + i);
          uint2 pk;
          pk.x = pack_bf16x2(v[j].x * rstd * gg.x, v[j].y * rstd * gg.y);
          pk.y = pack_bf16x2(v[j].z * rstd * gg.z, v[j].w * rstd * gg.w);
          *reinterpret_cast<uint2*>(xw + (size_t)m * K + i) = pk;
        }
      }
    }
    __syncthreads();
  }
  if (n0 >= N) return;
  auto x_chunk = [&](int m, int k) {
    return NORM ? *reinterpret_cast<const uint4*>(xs + (size_t)m * K + k)
                : *reinterpret_cast<const uint4*>(x + (size_t)min(m, m_valid - 1) * K + k);
  };
  float acc[NR][M];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int m = 0; m < M; ++m) acc[r][m] = 0.f;
  for (; k + (U - 1) * 512 < K; k += U * 512) {
    if (!preloaded) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int r = 0; r < NR; ++r)
          wl[u][r] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(wr[r] + k + u * 512));
    }
    preloaded = false;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      uint4 xv[M];
#pragma unroll
      for (int m = 0; m < M; ++m) xv[m] = x_chunk(m, k + u * 512);
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const uint4 wv = make_uint4(wl[u][r][0], wl[u][r][1], wl[u][r][2], wl[u][r][3]);
#pragma unroll
        for (int m = 0; m < M; ++m) fma8(acc[r][m], wv, xv[m]);
      }
    }
  }
  for (; k < K; k += 512) {
    uint4 xv[M];
#pragma unroll
    for (int m = 0; m < M; ++m) xv[m] = x_chunk(m, k);
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const u32x4_t wt = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(wr[r] + k));
      const uint4 wv = make_uint4(wt[0], wt[1], wt[2], wt[3]);
#pragma unroll
      for (int m = 0; m < M; ++m) fma8(acc[r][m], wv, xv[m]);
    }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int m = 0; m < M; ++m) acc[r][m] = wave_sum(acc[r][m]);
  if (lane != 0) return;
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    const int n = n0 + r;
    if (n >= N) break;
#pragma unroll
    for (int m = 0; m < M; ++m) {
      if (m >= m_valid) break;
      if (EPI == GEMV_GLU_BF16) {
        reinterpret_cast<bf16_t*>(out)[(size_t)m * ldo + n] = f32_to_bf16(glu_act_f(acc[r][m], act) * acc[r + RW][m]);
      } else {
        float* o = reinterpret_cast<float*>(out) + (size_t)m * ldo + n;
        *o = EPI == GEMV_ADD_F32 ? *o + acc[r][m] * scale : acc[r][m];
      }
    }
  }
}

// The input of a projection: bf16 rows x, or (xf != nullptr) fp32 rows to be RMS-normalised with gamma / eps.
struct GemvIn {
  const bf16_t* x;
  const float* xf;
  const float* gamma;
  float eps;
  float scale;   // GEMV_ADD_F32: out += scale * C
  int m_valid = 0;   // 0: all M rows of the instantiation exist; otherwise how many do (bf16 input only)
};

template <int M, int EPI, int RW, int U>
void launch_gemv_cfg(const GemvIn& in, const bf16_t* W, void* out, int N, int K, long long ldo, int act, hipStream_t st) {
  const int blocks = (N + 4 * RW - 1) / (4 * RW);
  if (in.xf)
    hipLaunchKernelGGL((gemv_kernel<M, EPI, RW, U, true>), dim3(blocks), dim3(256), (size_t)M * K * 2 + 16 * M, st,
                       in.x, in.xf, in.gamma, in.eps, W, out, N, K, ldo, act, in.scale, M);
  else
    hipLaunchKernelGGL((gemv_kernel<M, EPI, RW, U, false>), dim3(blocks), dim3(256), 0, st, in.x, in.xf, in.gamma,
                       in.eps, W, out, N, K, ldo, act, in.scale, in.m_valid > 0 ? in.m_valid : M);
}

// Rows per wave and unroll depth: few batch rows leave registers for deep unrolling; a small N gets
// two rows per wave so that the launch still has several waves per SIMD.
template <int M, int EPI>
void launch_gemv_me(const GemvIn& x, const bf16_t* W, void* out, int N, int K, long long ldo, int act, hipStream_t st) {
  if (EPI == GEMV_GLU_BF16) {
    if (M <= 2) launch_gemv_cfg<M, EPI, 2, 4>(x, W, out, N, K, ldo, act, st);
    else launch_gemv_cfg<M, EPI, 2, 1>(x, W, out, N, K, ldo, act, st);
  } else if (M <= 2) {
    if (N <= 8192) launch_gemv_cfg<M, EPI, 2, 4>(x, W, out, N, K, ldo, act, st);
    else launch_gemv_cfg<M, EPI, 4, 4>(x, W, out, N, K, ldo, act, st);
  } else if (M <= 4) {
    launch_gemv_cfg<M, EPI, 4, 2>(x, W, out, N, K, ldo, act, st);
  } else {
    launch_gemv_cfg<M, EPI, 4, 1>(x, W, out, N, K, ldo, act, st);
  }
}

template <int M>
void launch_gemv_m(const GemvIn& x, const bf16_t* W, void* out, int N, int K, long long ldo, int epi, int act,
                   hipStream_t st) {
  switch (epi) {
    case GEMV_STORE_F32: launch_gemv_me<M, GEMV_STORE_F32>(x, W, out, N, K, ldo, act, st); break;
    case GEMV_ADD_F32: launch_gemv_me<M, GEMV_ADD_F32>(x, W, out, N, K, ldo, act, st); break;
    default: launch_gemv_me<M, GEMV_GLU_BF16>(x, W, out, N, K, ldo, act, st);
  }
}

// rows m0 .. m0 + mm - 1 of the input
GemvIn rows_from(const GemvIn& in, int m0, int K) {
  GemvIn r = in;
  if (r.xf) r.xf += (size_t)m0 * K;
  else r.x += (size_t)m0 * K;
  return r;
}

void launch_gemv_in(const GemvIn& in, const bf16_t* W, void* out, int M, int N, int K, int64_t ldo, int epilogue,
                    int act, hipStream_t st) {
  if (M <= 0 || N <= 0) return;
  // rows are processed in groups of at most 8 (weights are re-streamed per group)
  const size_t osz = epilogue == GEMV_GLU_BF16 ? 2 : 4;
  for (int m0 = 0; m0 < M; m0 += 8) {
    const int mm = M - m0 < 8 ? M - m0 : 8;
    const GemvIn xs = rows_from(in, m0, K);
    void* os = reinterpret_cast<char*>(out) + (size_t)m0 * ldo * osz;
    if (mm == 1) launch_gemv_m<1>(xs, W, os, N, K, ldo, epilogue, act, st);
    else if (mm == 2) launch_gemv_m<2>(xs, W, os, N, K, ldo, epilogue, act, st);
    else if (mm <= 4) {
      // 3 rows: the 4-row form with the last one repeated (never stored; the weights are streamed once), or 2 + 1 where the
      // kernel normalises the rows
      if (mm == 3 && !xs.xf) {
        GemvIn x4 = xs;
        x4.m_valid = mm;
        launch_gemv_m<4>(x4, W, os, N, K, ldo, epilogue, act, st);
      } else if (mm == 3) {
        launch_gemv_m<2>(xs, W, os, N, K, ldo, epilogue, act, st);
        launch_gemv_m<1>(rows_from(xs, 2, K), W, reinterpret_cast<char*>(os) + 2 * ldo * osz, N, K, ldo, epilogue, act, st);
      } else launch_gemv_m<4>(xs, W, os, N, K, ldo, epilogue, act, st);
    } else if (mm == 8 || !xs.xf) {
      // 5..7 rows of bf16 input run the 8-row form with the missing rows repeating the last one (never stored):
      // the weights are streamed once
      GemvIn x8 = xs;
      x8.m_valid = mm;
      launch_gemv_m<8>(x8, W, os, N, K, ldo, epilogue, act, st);
    } else {  // 5..7 fp32 rows to be normalised: 4 + remainder
      launch_gemv_m<4>(xs, W, os, N, K, ldo, epilogue, act, st);
      launch_gemv_in(rows_from(xs, 4, K), W, reinterpret_cast<char*>(os) + 4 * ldo * osz, mm - 4, N, K, ldo, epilogue, act, st);
    }
  }
}

}  // namespace decode_impl
using namespace decode_impl;

void launch_gemv(const bf16_t* x, const bf16_t* W, void* out, int M, int N, int K, int64_t ldo, int epilogue,
                 int act, hipStream_t st, float scale) {
  launch_gemv_in(GemvIn{x, nullptr, nullptr, 0.f, scale, 0}, W, out, M, N, K, ldo, epilogue, act, st);
}

bool gemv_norm_supported(int M, int K) {
  return M >= 1 && M <= 4 && K % 8 == 0 && K <= 8192 && (size_t)M * K * 2 + 16 * M <= 48 * 1024;
}

void launch_gemv_norm(const float* xf, const float* gamma, float eps, const bf16_t* W, void* out, int M, int N, int K,
                      int64_t ldo, int epilogue, int act, hipStream_t st) {
  launch_gemv_in(GemvIn{nullptr, xf, gamma, eps, 1.f, 0}, W, out, M, N, K, ldo, epilogue, act, st);
}

// ------------------------------------------------------------------------------------- RoPE + append
namespace decode_impl {
__global__ __launch_bounds__(128) void rope_append_kernel(const float* __restrict__ qkv, int ld,
                                                          bf16_t* __restrict__ q_out, int n_q_heads,
                                                          int n_kv_heads, int hd, const int32_t* __restrict__ pos,
                                                          const int32_t* __restrict__ slot,
                                                          double neg2_over_hd_log2theta, bf16_t* __restrict__ k_pool,
                                                          bf16_t* __restrict__ v_pool, int P,
                                                          const float* __restrict__ q_gamma,
                                                          const float* __restrict__ k_gamma, float qk_eps,
                                                          int n_parts, size_t part_stride, KvQuant kvq) {
  __shared__ float red[2];
  const int b = blockIdx.x, head = blockIdx.y;
  const int half = hd >> 1;
  const int i = threadIdx.x;
  const float* row = qkv + (size_t)b * ld + (size_t)head * hd;
  const int s = slot[b];
  // per-head QK-norm (uniform over the block): RMS over the head's hd values, before the rotation
  const float* gamma = head < n_q_heads ? q_gamma : (head < n_q_heads + n_kv_heads ? k_gamma : nullptr);
  float x = i < half ? row[i] : 0.f, y = i < half ? row[i + half] : 0.f;
  for (int p = 1; p < n_parts; ++p)
    if (i < half) {
      x += row[p * part_stride + i];
      y += row[p * part_stride + i + half];
    }
  if (gamma) {
    const float ss = wave_sum(x * x + y * y);
    if ((i & 63) == 0) red[i >> 6] = ss;
    __syncthreads();
    const float rstd = 1.0f / sqrtf((red[0] + red[1]) / (float)hd + qk_eps);
    if (i < half) {
      x *= rstd * gamma[i];
      y *= rstd * gamma[i + half];
    }
  }
  if (i >= half) return;
  if (head < n_q_heads + n_kv_heads) {
    const double ang = (double)pos[b] * exp2((double)i * neg2_over_hd_log2theta);
    double sd, cd;
    sincos(ang, &sd, &cd);
    const float c = (float)cd, sn = (float)sd;
    const float rlo = x * c - y * sn, rhi = y * c + x * sn;
    const bf16_t lo = f32_to_bf16(rlo), hi = f32_to_bf16(rhi);
    if (head < n_q_heads) {
      bf16_t* o = q_out + ((size_t)b * n_q_heads + head) * hd;
      o[i] = lo;
      o[i + half] = hi;
    } else {
      const int hh = head - n_q_heads;
      const size_t eoff = (((size_t)(s / P) * n_kv_heads + hh) * P + (s % P)) * hd;
      if (kvq.fp8) {     // one-byte e4m3 codes
        unsigned char* o = reinterpret_cast<unsigned char*>(k_pool) + eoff;
        o[i] = (unsigned char)e4m3_encode(rlo * kvq.k_inv);
        o[i + half] = (unsigned char)e4m3_encode(rhi * kvq.k_inv);
      } else {
        bf16_t* o = k_pool + eoff;
        o[i] = lo;
        o[i + half] = hi;
      }
    }
  } else {
    const int hh = head - n_q_heads - n_kv_heads;
    const size_t eoff = (((size_t)(s / P) * n_kv_heads + hh) * P + (s % P)) * hd;
    if (kvq.fp8) {
      unsigned char* o = reinterpret_cast<unsigned char*>(v_pool) + eoff;
      o[i] = (unsigned char)e4m3_encode(x * kvq.v_inv);
      o[i + half] = (unsigned char)e4m3_encode(y * kvq.v_inv);
    } else {
      bf16_t* o = v_pool + eoff;
      o[i] = f32_to_bf16(x);
      o[i + half] = f32_to_bf16(y);
    }
  }
}
}  // namespace decode_impl
using namespace decode_impl;

void launch_rope_append(const float* qkv, int ld, bf16_t* q_out, int n_q_heads, int n_kv_heads, int hd,
                        const int32_t* pos, const int32_t* slot, double theta, bf16_t* k_pool, bf16_t* v_pool,
                        int page_size, int B, hipStream_t st, const float* q_gamma, const float* k_gamma,
                        float qk_eps, int n_parts, size_t part_stride, KvQuant kvq) {
  if (B <= 0) return;
  hipLaunchKernelGGL(rope_append_kernel, dim3(B, n_q_heads + 2 * n_kv_heads), dim3(128), 0, st, qkv, ld, q_out,
                     n_q_heads, n_kv_heads, hd, pos, slot, -2.0 / (double)hd * log2(theta), k_pool, v_pool,
                     page_size, q_gamma, k_gamma, qk_eps, n_parts, part_stride, kvq);
}

// ------------------------------------------------------------------------------------- decode attention
namespace decode_impl {

constexpr int GMAX = 8;   // query heads per KV head

// grid (n_splits, Hkv, B), 256 threads.  Split s of sequence b covers keys lo + s * split_keys .., lo = first visible
// key (window start, or the first position the layer holds an entry for); wave w of the work-group takes its key
// blocks (NB groups of 16 keys) w, w + 4, ... with a running maximum and sum of its own.
//   S = K Q^T on the MFMA (v_mfma_f32_16x16x32_bf16): lane l takes chunks of 8 dims of key l % 16, which are the operand as they
//   are (8-bit codes become bf16, exactly).  Column c of the 16 is query head c % GT: the heads stand there several times.
//   O^T += V^T P^T on the MFMA (v_mfma_f32_16x16x16_bf16) without rounding P: the 24 bits of a probability are three bf16 numbers
//   (cut off, not rounded, so that their sum is the probability), which go to three columns of the same head, c / GT = 0, 1, 2, and
//   are added at the end (eight heads: two columns each, and a second product for the third).  A lane then scales and splits
//   the four keys that S left it, and nothing crosses lanes.  V, whose rows are contiguous in the head-dim, goes through LDS
//   (a wave's own 16 rows per group) and comes back transposed, four keys of a dim per lane (ds_read_b64_tr_b16); 32-byte pieces of
//   row r lie at piece ^ (r & 7), so that the 16 rows of a read fall on different banks.
//   K goes through LDS too, as it is stored, so that every load takes whole rows (16 bytes of 16 rows per load, the operand's
//   own layout, reads slower), and the next block's K and V are requested as soon as this block's are in LDS.
// Where the time goes: with P V in fp32 on the vector ALU and K loaded in operand layout a step's attention took, per layer of 8
// sequences, 15.0 us (2048 keys) and 35.0 (8192, 8-bit); P V on the MFMA alone changed nothing (15.0, 35.6), loads of whole rows
// 14.1 and 28.8, fewer splits the rest (see choose_decode_splits).  Three work-groups per CU need the launch bound.
// GT: compile-time bound of the number of query heads per KV head (registers and loops are sized by it).
// FUSED: RoPE + append inside this kernel (a.qkv_raw given).
template <int HD, int GT, bool FUSED, bool FP8, int NB>
__global__ __launch_bounds__(256, (HD <= 128 && GT <= 4) ? 3 : 1 /* work-groups per CU */) void attn_decode_split_kernel(AttnDecodeArgs a, float scale) {
  constexpr int KS = HD / 32;                       // MFMA steps over the head dim
  constexpr int LPK = HD / 8, KPL = 64 / LPK;       // lanes per V row, V rows per load
  constexpr int VL = 16 / KPL;                      // V loads per 16 keys
  constexpr int HALF = HD / 2;
  typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
  typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
  typedef typename std::conditional<FP8, u32x2_t, u32x4_t>::type chunk_t;   // 8 elements
  typedef short s16x4_t __attribute__((ext_vector_type(4)));
  constexpr int HB = HD / 16;                       // 16-dim blocks of a head
  // K (as stored) and V (bf16) of a wave's block; after its last one V's place holds the wave's float [GT][HD]
  __shared__ __attribute__((aligned(16))) unsigned char k_lds[4][NB * 16 * LPK * sizeof(chunk_t)];
  __shared__ __attribute__((aligned(16))) unsigned char v_lds[4][NB * 16 * HD * 2];
  static_assert(GT * 4 <= NB * 32, "the wave's sums fit its share");
  auto red = [&](int w, int g, int e) -> float& { return reinterpret_cast<float*>(v_lds[w])[g * HD + e]; };
  __shared__ float stat[4][2][GT];

  const int split = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
  const int G = a.n_q_heads / a.n_kv_heads;
  const int P = a.page_size, lgP = __ffs(P) - 1;    // page sizes are powers of two
  const int qpos = a.pos[b];
  int lo = a.window > 0 ? max(0, qpos - a.window + 1) : 0;
  if (a.kv_first) lo = max(lo, min(a.kv_first[b], qpos));   // the query token's own entry always exists
  const int k_first = lo + split * a.split_keys;
  const int n_keys = min(a.split_keys, qpos + 1 - k_first);  // <= 0: this split is empty
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g4 = lane >> 4;        // key (K operand) or column (Q operand); k chunk
  const int hcol = r16 % GT, piece = r16 / GT;      // the column's query head, and which bf16 piece of its probabilities
  const int li = lane % LPK, vs = lane / LPK;       // V: head-dim chunk, row of the load
  const int32_t* bt = a.block_table + (size_t)b * a.max_pages;
  float* part = a.part + (((size_t)b * a.n_q_heads + (size_t)kvh * G) * a.n_splits + split) * (HD + 2);
  const size_t part_head_stride = (size_t)a.n_splits * (HD + 2);
  if (n_keys <= 0) {                                // the merge skips a split whose maximum is -inf
    if (tid < G) part[tid * part_head_stride + HD] = -INFINITY;
    return;
  }
  const chunk_t* k_pool = reinterpret_cast<const chunk_t*>(a.k_pool);
  const chunk_t* v_pool = reinterpret_cast<const chunk_t*>(a.v_pool);
  // row (of HD elements) of entry `key` in page `page`; chunk index of a row
  auto row_of = [&](int key, int page) { return ((uint32_t)(page * a.n_kv_heads + kvh) << lgP) + (uint32_t)(key & (P - 1)); };
  auto chunk_of = [&](uint32_t row) { return (size_t)row * LPK; };
  // Key kk of the split (kk beyond the last one repeats it, masked below).
  auto key_of = [&](int kk) { return k_first + min(kk, n_keys - 1); };
  const int n_blocks = (n_keys + NB * 16 - 1) / (NB * 16);
  // A load takes KPL whole rows, K and V alike: lane (vs, li) has chunk li of row i * KPL + vs of each group of 16 keys.
  chunk_t kw[NB][VL], vw[NB][VL];
  // Pages are looked up a block further ahead than entries are: loads return in order, so that a page looked up when its entries
  // are due arrives behind the rows on their way.
  int32_t page[NB];                                 // page of key r16 of each group of the block after
  auto load_pages = [&](int blk) {
#pragma unroll
    for (int n = 0; n < NB; ++n) page[n] = bt[key_of((blk * NB + n) * 16 + r16) >> lgP];
  };
  auto load_kv = [&](int blk) {                     // (its pages have been looked up)
    uint32_t row[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) row[n] = row_of(key_of((blk * NB + n) * 16 + r16), page[n]);
    load_pages(blk + 4);
    size_t at[NB][VL];
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int i = 0; i < VL; ++i) at[n][i] = chunk_of((uint32_t)__shfl((int)row[n], i * KPL + vs, 64)) + li;
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int i = 0; i < VL; ++i) kw[n][i] = k_pool[at[n][i]];
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int i = 0; i < VL; ++i) vw[n][i] = v_pool[at[n][i]];
  };
  // the first block's entries travel while the query rows are prepared
  load_pages(wave);
  if (wave < n_blocks) load_kv(wave);

  auto as_chunk = [](const uint4& w) {
    if constexpr (FP8) return chunk_t{w.x, w.y};
    else return __builtin_bit_cast(chunk_t, w);
  };

  // ---- query rows: lane l holds head hcol (zeros beyond G), dims 32 ks + 8 g4 .. + 7, as bf16.  The other member of
  //      a rotation pair, HALF dims on, is the same lane's chunk ks + KS / 2.
  bf16x8_t qf[KS];
  // FUSED: the query position's own entry (K row, V row), a copy per wave
  __shared__ chunk_t entry_new[FUSED ? 4 : 1][2][LPK];
  const bool has_new = FUSED && qpos - k_first < a.split_keys;     // (uniform) its key falls into this split
  if constexpr (FUSED) {
    // the 8 * KS values of this lane of the head at column `col`: optionally RMS-normalised over the head (its four
    // lanes g4 hold it all), rotated
    float cc[KS / 2][8], sn[KS / 2][8];
    const float2* csp = a.cs + (size_t)b * HALF + g4 * 8;
#pragma unroll
    for (int ks = 0; ks < KS / 2; ++ks)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float4 t = *reinterpret_cast<const float4*>(csp + ks * 32 + 2 * e);
        cc[ks][2 * e] = t.x; sn[ks][2 * e] = t.y; cc[ks][2 * e + 1] = t.z; sn[ks][2 * e + 1] = t.w;
      }
    auto head_row = [&](int col, const float* gamma, float (&x)[KS][8]) {
      const float* row = a.qkv_raw + (size_t)b * a.ld + col + g4 * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const float4 u = *reinterpret_cast<const float4*>(row + ks * 32), w = *reinterpret_cast<const float4*>(row + ks * 32 + 4);
        x[ks][0] = u.x; x[ks][1] = u.y; x[ks][2] = u.z; x[ks][3] = u.w;
        x[ks][4] = w.x; x[ks][5] = w.y; x[ks][6] = w.z; x[ks][7] = w.w;
      }
      if (gamma) {
        float s2 = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int e = 0; e < 8; ++e) s2 += x[ks][e] * x[ks][e];
        s2 += __shfl_xor(s2, 16, 64);
        s2 += __shfl_xor(s2, 32, 64);
        const float rstd = 1.0f / sqrtf(s2 / (float)HD + a.qk_eps);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int e = 0; e < 8; ++e) x[ks][e] *= rstd * gamma[ks * 32 + g4 * 8 + e];
      }
#pragma unroll
      for (int ks = 0; ks < KS / 2; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float lo8 = x[ks][e], hi8 = x[ks + KS / 2][e];
          x[ks][e] = lo8 * cc[ks][e] - hi8 * sn[ks][e];
          x[ks + KS / 2][e] = hi8 * cc[ks][e] + lo8 * sn[ks][e];
        }
    };
    auto pack8 = [&](const float* x, float inv) {   // a cache chunk: bf16 values or e4m3 codes
      if (FP8)
        return make_uint4(e4m3_pack4(x[0] * inv, x[1] * inv, x[2] * inv, x[3] * inv),
                          e4m3_pack4(x[4] * inv, x[5] * inv, x[6] * inv, x[7] * inv), 0u, 0u);
      return make_uint4(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7]));
    };
    float x[KS][8];
    head_row((kvh * G + min(hcol, G - 1)) * HD, a.q_gamma, x);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint4 w = hcol < G ? make_uint4(pack_bf16x2(x[ks][0], x[ks][1]), pack_bf16x2(x[ks][2], x[ks][3]),
                                            pack_bf16x2(x[ks][4], x[ks][5]), pack_bf16x2(x[ks][6], x[ks][7]))
                               : make_uint4(0, 0, 0, 0);
      qf[ks] = __builtin_bit_cast(bf16x8_t, w);
    }
    if (has_new) {
      head_row((a.n_q_heads + kvh) * HD, a.k_gamma, x);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        if (r16 == 0) entry_new[wave][0][ks * 4 + g4] = as_chunk(pack8(x[ks], a.kvq.k_inv));
      float v8[8];
      const float* row = a.qkv_raw + (size_t)b * a.ld + (a.n_q_heads + a.n_kv_heads + kvh) * HD + li * 8;
#pragma unroll
      for (int e = 0; e < 8; ++e) v8[e] = row[e];
      if (vs == 0) entry_new[wave][1][li] = as_chunk(pack8(v8, a.kvq.v_inv));
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the wave's own LDS writes, read by its other lanes
    }
  } else {
    const bf16_t* q = a.q + ((size_t)b * a.n_q_heads + kvh * G + min(hcol, G - 1)) * HD + g4 * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint4 w = *reinterpret_cast<const uint4*>(q + ks * 32);
      qf[ks] = __builtin_bit_cast(bf16x8_t, hcol < G ? w : make_uint4(0, 0, 0, 0));
    }
  }
  // FUSED, in the block that holds the query position's key (the split's last): the chunks loaded for it, also by
  // lanes that repeat it, are replaced by the new entry, and the lanes whose key it is store it.
  auto patch = [&](int blk) {
    const chunk_t kn = entry_new[FUSED ? wave : 0][0][li], vn = entry_new[FUSED ? wave : 0][1][li];
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int i = 0; i < VL; ++i) {
        const int kk = (blk * NB + n) * 16 + i * KPL + vs, key = key_of(kk);
        if (key != qpos) continue;
        kw[n][i] = kn;
        vw[n][i] = vn;
        if (kk == n_keys - 1) {
          const size_t at = chunk_of(row_of(key, bt[key >> lgP])) + li;
          reinterpret_cast<chunk_t*>(const_cast<bf16_t*>(a.k_pool))[at] = kn;
          reinterpret_cast<chunk_t*>(const_cast<bf16_t*>(a.v_pool))[at] = vn;
        }
      }
  };
  // a chunk of K as the MFMA operand
  auto k_operand = [&](const chunk_t& w) {
    if constexpr (FP8) return e4m3_to_bf16x8(make_uint2(w.x, w.y));
    else return __builtin_bit_cast(bf16x8_t, w);
  };
  const float s_scale = FP8 ? scale * a.kvq.k_scale : scale;
  const uint32_t is_piece[3] = {piece == 0 ? ~0u : 0u, piece == 1 ? ~0u : 0u, piece == 2 ? ~0u : 0u};
  floatx4_t o[HB], o3[GT == 8 ? HB : 1];            // o[c][v]: dim 16 c + 4 g4 + v of column r16; o3: the third pieces
#pragma unroll
  for (int c = 0; c < HB; ++c) o[c] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < (GT == 8 ? HB : 1); ++c) o3[c] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;             // of query head hcol; l_run: this lane's keys
  // V in LDS: 32-byte piece q of row r at q ^ key(r).  Written in 16-byte chunks, read back by lane i of a group of 16 as the four
  // rows 4 g4 + 0..3 of dim 16 c + i, for which lanes 4 r .. 4 r + 3 of the group point at row r
  auto swz = [](int r) { return HD == 64 ? (r >> 1) & 3 : r & 7; };
  unsigned char* const v_wave = v_lds[wave];
  const int tr_row = 4 * g4 + (r16 >> 2), tr_key = swz(tr_row);
  const unsigned char* const tr_lane = v_wave + tr_row * (HD * 2) + (r16 & 3) * 8;
  // K in LDS: chunk c of row r at c ^ key(r), so that the 16 rows of an operand read (two reads' worth of 8-byte chunks) fall on
  // different banks
  auto kswz = [](int r) { return FP8 ? (HD == 64 ? (r >> 2 & 3) << 1 : HD == 128 ? (r >> 1 & 7) << 1 : (r & 15) << 1)
                                     : HD == 64 ? r >> 1 & 7 : r & 15; };
  chunk_t* const k_wave = reinterpret_cast<chunk_t*>(k_lds[wave]);
  const chunk_t* const k_lane = k_wave + r16 * LPK;
  const int k_key = kswz(r16);

  for (int blk = wave; blk < n_blocks; blk += 4) {
    if (FUSED && has_new && blk == n_blocks - 1) patch(blk);
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int i = 0; i < VL; ++i) {
        const int r = i * KPL + vs;                 // row of the group
        k_wave[(n * 16 + r) * LPK + (li ^ kswz(r))] = kw[n][i];
        u32x4_t w;
        if constexpr (FP8) w = __builtin_bit_cast(u32x4_t, e4m3_to_bf16x8(make_uint2(vw[n][i].x, vw[n][i].y)));
        else w = vw[n][i];
        *reinterpret_cast<u32x4_t*>(v_wave + (n * 16 + r) * (HD * 2) + ((li >> 1) ^ swz(r)) * 32 + (li & 1) * 16) = w;
      }
    if (blk + 4 < n_blocks) load_kv(blk + 4);
    floatx4_t s[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      s[n] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        s[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k_operand(k_lane[n * 16 * LPK + ((ks * 4 + g4) ^ k_key)]), qf[ks], s[n], 0, 0, 0);
    }
    // s[n][v]: query head hcol, key 16 n + 4 g4 + v of the block
    float mx = -INFINITY;
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const bool in = (blk * NB + n) * 16 + 4 * g4 + v < n_keys;
        s[n][v] = in ? s[n][v] * s_scale : -INFINITY;
        mx = fmaxf(mx, s[n][v]);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(m_run, mx);           // every block has a key: finite unless the scores are not
    const float alpha = __expf(m_run - m_new);
    float sum = 0.f;
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        s[n][v] = __expf(s[n][v] - m_new);
        sum += s[n][v];
      }
    l_run = l_run * alpha + sum;
    m_run = m_new;
    if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0) {
#pragma unroll
      for (int c = 0; c < HB; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) o[c][v] *= alpha;
      if (GT == 8) {
#pragma unroll
        for (int c = 0; c < HB; ++c)
#pragma unroll
          for (int v = 0; v < 4; ++v) o3[GT == 8 ? c : 0][v] *= alpha;
      }
    }
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      uint32_t first[4], third[4];                  // this column's piece of the four probabilities (upper halves), and the third
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const uint32_t p1 = __builtin_bit_cast(uint32_t, s[n][v]);
        const float r1 = s[n][v] - __builtin_bit_cast(float, p1 & 0xffff0000u);
        const uint32_t p2 = __builtin_bit_cast(uint32_t, r1);
        third[v] = __builtin_bit_cast(uint32_t, r1 - __builtin_bit_cast(float, p2 & 0xffff0000u));
        first[v] = (p1 & is_piece[0]) | (p2 & is_piece[1]) | (third[v] & is_piece[2]);
      }
      auto operand = [](const uint32_t (&w)[4]) {
        return __builtin_bit_cast(s16x4_t, make_uint2(__builtin_amdgcn_perm(w[1], w[0], 0x07060302u),
                                                      __builtin_amdgcn_perm(w[3], w[2], 0x07060302u)));
      };
      const s16x4_t pf = operand(first), pf3 = operand(third);
#pragma unroll
      for (int c = 0; c < HB; ++c) {
#if defined(__HIP_DEVICE_COMPILE__)  // the builtins exist in the device pass only
        typedef __attribute__((address_space(3))) s16x4_t* lds_s16x4_t;
        const s16x4_t vt = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_s16x4_t)(tr_lane + n * 16 * (HD * 2) + (c ^ tr_key) * 32));
        o[c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vt, pf, o[c], 0, 0, 0);
        if (GT == 8) o3[GT == 8 ? c : 0] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vt, pf3, o3[GT == 8 ? c : 0], 0, 0, 0);
#endif
      }
    }
  }

  // ---- the wave's key slots, then the four waves, each with its own maximum
  l_run += __shfl_xor(l_run, 16, 64);
  l_run += __shfl_xor(l_run, 32, 64);
  if (g4 == 0 && r16 < G) {
    stat[wave][0][r16 % GT] = m_run;
    stat[wave][1][r16 % GT] = l_run;
  }
  asm volatile("" ::: "memory");                    // (the sums take the place of V)
  // the pieces of a head: columns c, c + GT, c + 2 GT (row_ror:n brings lane i the value of lane i - n of its 16)
#pragma unroll
  for (int c = 0; c < HB; ++c) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      float x = o[c][v] + dpp_f32<0x120 + 16 - GT>(o[c][v]);
      if constexpr (GT == 8) x += o3[GT == 8 ? c : 0][v];
      else x += dpp_f32<0x120 + 16 - 2 * (GT == 8 ? 4 : GT)>(o[c][v]);
      if (r16 < G) red(wave, r16 % GT, c * 16 + 4 * g4 + v) = x;
    }
  }
  __syncthreads();
  const float v_scale = FP8 ? a.kvq.v_scale : 1.f;
  for (int i = tid; i < G * HD; i += 256) {
    const int g = i / HD, e = i % HD;
    const float m = fmaxf(fmaxf(stat[0][0][g], stat[1][0][g]), fmaxf(stat[2][0][g], stat[3][0][g]));
    float num = 0.f, den = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float f = stat[w][0][g] == -INFINITY ? 0.f : __expf(stat[w][0][g] - m);   // (a wave without keys)
      num += f * red(w, g, e);
      den += f * stat[w][1][g];
    }
    num *= v_scale;
    if (a.n_splits == 1) {
      a.out[((size_t)b * a.n_q_heads + kvh * G + g) * HD + e] = f32_to_bf16(den > 0.f ? num / den : 0.f);
    } else {
      part[g * part_head_stride + e] = num;
      if (e == 0) {
        part[g * part_head_stride + HD] = m;
        part[g * part_head_stride + HD + 1] = den;
      }
    }
  }
}

// grid (B * Hq), 256 threads: thread (grp, i) sums head-dim element i over the splits s = grp, grp + NG, ..
// (NG = 256 / hd groups), the groups are then added in index order: a fixed summation order.
__global__ __launch_bounds__(256) void attn_decode_combine_kernel(const float* __restrict__ part,
                                                                  bf16_t* __restrict__ out, int n_splits, int hd) {
  __shared__ float red_m[4];
  __shared__ float red_num[4][256];
  __shared__ float red_den[4];
  const size_t bh = blockIdx.x;
  const int tid = threadIdx.x;
  const int stride = hd + 2;
  const float* p = part + bh * n_splits * stride;
  float mx = -INFINITY;
  for (int s = tid; s < n_splits; s += 256) mx = fmaxf(mx, p[s * stride + hd]);
  mx = wave_max(mx);
  if ((tid & 63) == 0) red_m[tid >> 6] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red_m[0], red_m[1]), fmaxf(red_m[2], red_m[3]));
  const int ng = 256 / hd, grp = tid / hd, i = tid % hd;
  float num = 0.f, den = 0.f;
#pragma unroll 4
  for (int s = grp; s < n_splits; s += ng) {
    const float m = p[s * stride + hd];
    // (an empty split holds nothing but its maximum, -inf)
    const float w = m == -INFINITY ? 0.f : __expf(m - mx);
    const float x = p[s * stride + i], y = p[s * stride + hd + 1];
    num += m == -INFINITY ? 0.f : w * x;
    den += m == -INFINITY ? 0.f : w * y;
  }
  red_num[grp][i] = num;
  if (i == 0) red_den[grp] = den;
  __syncthreads();
  if (tid < hd) {
    float n = red_num[0][tid], d = red_den[0];
    for (int g = 1; g < ng; ++g) { n += red_num[g][tid]; d += red_den[g]; }
    out[bh * hd + tid] = f32_to_bf16(d > 0.f ? n / d : 0.f);
  }
}

template <int HD, bool FUSED, bool FP8, int NB>
void launch_decode_cfg(const AttnDecodeArgs& a, hipStream_t st) {
  const float scale = 1.f / sqrtf((float)HD);
  const dim3 grid(a.n_splits, a.n_kv_heads, a.B);
  const int G = a.n_q_heads / a.n_kv_heads;
  if (G <= 1) hipLaunchKernelGGL((attn_decode_split_kernel<HD, 1, FUSED, FP8, NB>), grid, dim3(256), 0, st, a, scale);
  else if (G <= 2) hipLaunchKernelGGL((attn_decode_split_kernel<HD, 2, FUSED, FP8, NB>), grid, dim3(256), 0, st, a, scale);
  else if (G <= 4) hipLaunchKernelGGL((attn_decode_split_kernel<HD, 4, FUSED, FP8, NB>), grid, dim3(256), 0, st, a, scale);
  else hipLaunchKernelGGL((attn_decode_split_kernel<HD, GMAX, FUSED, FP8, NB>), grid, dim3(256), 0, st, a, scale);
}

template <int HD>
void launch_decode_hd(const AttnDecodeArgs& a, hipStream_t st) {
  // Two groups of 16 keys per block where a wave has several blocks of an 8-bit cache (half the cross-lane steps per key:
  // 8 sequences of 8192 tokens 604 us a step against 629); bf16 entries, twice the registers, do better with one and
  // more waves (691 against 706 us), and with three or four neither does.
  auto go = [&](auto fused_c, auto fp8_c) {
    constexpr bool F = decltype(fused_c)::value, Q = decltype(fp8_c)::value;
    if constexpr (Q && HD <= 128) {
      if (a.split_keys >= 256) { launch_decode_cfg<HD, F, Q, 2>(a, st); return; }
    }
    launch_decode_cfg<HD, F, Q, 1>(a, st);
  };
  auto go_q = [&](auto fused_c) {
    if (a.kvq.fp8) go(fused_c, std::true_type{});
    else go(fused_c, std::false_type{});
  };
  if (a.qkv_raw) go_q(std::true_type{});
  else go_q(std::false_type{});
  if (a.n_splits > 1)
    hipLaunchKernelGGL(attn_decode_combine_kernel, dim3(a.B * a.n_q_heads), dim3(256), 0, st, a.part, a.out,
                       a.n_splits, HD);
}
}  // namespace decode_impl
using namespace decode_impl;

// ------------------------------------------------------------------------------------- greedy choice
namespace decode_impl {
// tok[b] = (step > 0 and tok[b] == eos and eos >= 0) ? eos : argmax_v logits[b, v]  (lowest index on ties),
// and out[b * out_stride + step] = tok[b].  One work-group of 1024 threads per sequence.
__global__ __launch_bounds__(1024) void argmax_kernel(const float* __restrict__ logits, int vocab,
                                                      int32_t* __restrict__ tok, int32_t* __restrict__ out,
                                                      int out_stride, int step, int eos) {
  __shared__ float bv[16];
  __shared__ int bi[16];
  const int b = blockIdx.x, tid = threadIdx.x;
  const float* row = logits + (size_t)b * vocab;
  float best = -INFINITY;
  int idx = 0x7fffffff;
  // A thread sees its elements in ascending order, so the first maximum it meets is the one it keeps.  With a
  // 16-byte aligned row it takes four consecutive logits per load and has four loads in flight (one block per
  // sequence reads half a megabyte: the latency of dependent scalar loads was 39 us at a vocabulary of 128256).
  if ((vocab & 3) == 0 && (reinterpret_cast<uintptr_t>(row) & 15) == 0) {
    const float4* row4 = reinterpret_cast<const float4*>(row);
    const int n4 = vocab >> 2;
    for (int v0 = tid; v0 < n4; v0 += 4 * 1024) {
      float4 x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int v = v0 + u * 1024;
        x[u] = v < n4 ? row4[v] : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int v = (v0 + u * 1024) * 4;
        if (x[u].x > best) { best = x[u].x; idx = v; }
        if (x[u].y > best) { best = x[u].y; idx = v + 1; }
        if (x[u].z > best) { best = x[u].z; idx = v + 2; }
        if (x[u].w > best) { best = x[u].w; idx = v + 3; }
      }
    }
  } else {
    for (int v = tid; v < vocab; v += 1024) {
      const float x = row[v];
      if (x > best) { best = x; idx = v; }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(best, o, 64);
    const int oi = __shfl_xor(idx, o, 64);
    if (ov > best || (ov == best && oi < idx)) { best = ov; idx = oi; }
  }
  if ((tid & 63) == 0) { bv[tid >> 6] = best; bi[tid >> 6] = idx; }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < 16; ++w)
      if (bv[w] > best || (bv[w] == best && bi[w] < idx)) { best = bv[w]; idx = bi[w]; }
    if (idx == 0x7fffffff) idx = 0;   // a row without any finite maximum
    if (step > 0 && eos >= 0 && tok[b] == eos) idx = eos;
    tok[b] = idx;
    out[(size_t)b * out_stride + step] = idx;
  }
}
}  // namespace decode_impl

void launch_argmax(const float* logits, int vocab, int32_t* tok, int32_t* out, int out_stride, int step, int eos,
                   int B, hipStream_t st) {
  if (B <= 0) return;
  hipLaunchKernelGGL(decode_impl::argmax_kernel, dim3(B), dim3(1024), 0, st, logits, vocab, tok, out, out_stride, step,
                     eos);
}

// Splits of the key range.  A wave's block of keys takes about 1.25 us (heads of 256: 2.5) however few work-groups run, all of
// them together no less than the entries at 6.5 TB/s, each work-group on a CU about 1 us, and the merge of the splits 5 us and
// more with their number: the least sum of these over the splits that leave at least 64 keys and at most three work-groups per
// CU.  In effect one work-group per CU where the contexts are short enough, and no merge where sequences are many (four layers of
// a step, us, three work-groups per CU always -> this:
// 32 sequences of 512 keys 559 -> 530, 8-bit 534 -> 491, 20 of 700 477 -> 461, 8 of 2048 462 -> 448, 8 of 2000 with heads of 256 752
// -> 717, one of 2048 407 -> 396, one of 16000 438 -> 430, 17 of 3500 627 -> 618; 4 of 15000, 8-bit, 555 -> 558).
// More than 256 (sequence, KV head) pairs: whole rounds of work-groups, rounded down (48 sequences of 300 keys 566, one split 585).
void choose_decode_splits(AttnDecodeArgs& a, int span) {
  const long long pairs = (long long)a.B * a.n_kv_heads;
  const long long most = std::max(1LL, std::min<long long>((span + kDecodeKeysPerSplit - 1) / kDecodeKeysPerSplit, 768 / pairs));
  auto keys_of = [&](long long splits) { return (int)(((span + splits - 1) / splits + 63) / 64 * 64); };
  a.split_keys = keys_of(most);
  if (pairs <= 256) {
    const double all_us = (double)pairs * span * a.hd * 2 * (a.kvq.fp8 ? 1 : 2) / 6.5e6, block_us = a.hd <= 128 ? 1.25 : 2.5;
    double best = 1e300;
    for (long long want = 1; want <= most; ++want) {
      const int keys = keys_of(want), splits = (span + keys - 1) / keys;
      const double groups = (double)pairs * splits, rounds = std::ceil(groups / 256);
      const int block_keys = a.kvq.fp8 && a.hd <= 128 && keys >= 256 ? 128 : 64;
      const double us = std::max((keys + block_keys - 1) / block_keys * block_us, all_us * rounds * 256 / groups) + rounds +
                        (splits > 1 ? 5 + 0.05 * splits : 0);
      if (us < best) {
        best = us;
        a.split_keys = keys;
      }
    }
  }
  a.n_splits = (span + a.split_keys - 1) / a.split_keys;
}

void launch_attention_decode(const AttnDecodeArgs& args, int span, hipStream_t st) {
  AttnDecodeArgs a = args;
  if (a.B <= 0) return;
  choose_decode_splits(a, span);
  switch (a.hd) {
    case 64: launch_decode_hd<64>(a, st); break;
    case 128: launch_decode_hd<128>(a, st); break;
    case 256: launch_decode_hd<256>(a, st); break;
  }
}

}  // namespace pop
