// Decode-step kernels: one row per sequence through a full layer against the paged KV cache (few-row
// projections, attention over the cache, for one or two rows with RoPE and the append of the new entry inside, greedy
// choice).
// They carry the boundary token of Sec. 3.3 ("Boundary Handling for the Last Input Token": x_N is
// the first decode step with the full model) and pop_decode_step (Sec. 3.2, decode operator).
// Every projection streams its weights once: HBM-bound (three and more rows go through the tiled GEMM, three and four of a
// K that is no multiple of 64 through the GEMV kernel here).
#include <algorithm>
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

// Reduces values that the lanes li, li + LPK, ... of a wave hold for the same head-dim slice, by a butterfly that
// halves the number of values a lane carries at every step (a lane sends the half its partner keeps): N values cost
// N (1 - LPK / 64) exchanges.  Returns the index of this lane's v[0]; the first N * LPK / 64 entries are its results.
template <int LPK, int N>
__device__ __forceinline__ int fold_keys(float (&v)[N], int lane) {
  int first = 0;
  auto fold = [&](auto n_c, int o) {
    constexpr int H = decltype(n_c)::value / 2;
    const bool upper = (lane & o) != 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const float send = upper ? v[i] : v[i + H];
      const float keep = upper ? v[i + H] : v[i];
      v[i] = keep + __shfl_xor(send, o, 64);
    }
    if (upper) first += H;
  };
  constexpr int N2 = LPK <= 32 ? N / 2 : N, N3 = LPK <= 16 ? N2 / 2 : N2;
  static_assert(N * LPK >= 64, "a lane keeps at least one value");
  if constexpr (LPK <= 32) fold(std::integral_constant<int, N>{}, 32);
  if constexpr (LPK <= 16) fold(std::integral_constant<int, N2>{}, 16);
  if constexpr (LPK <= 8) fold(std::integral_constant<int, N3>{}, 8);
  return first;
}

// grid (n_splits, Hkv, B), 256 threads.  Split s of sequence b covers keys lo + s * split_keys .., lo = first visible
// key (window start, or the first position the layer holds an entry for); wave w of the work-group takes its key
// blocks (NB groups of 16 keys) w, w + 4, ... with a running maximum and sum of its own.
//   S = K Q^T on the MFMA (v_mfma_f32_16x16x32_bf16; the G query heads of the KV head are columns, the others zero):
//   lane l loads 16-byte chunks of key l % 16, which are the operand as they are (8-bit codes become bf16, exactly).
//   O += P V on the vector ALU in fp32 with P in fp32: V's rows are contiguous in the head-dim, so an MFMA would need
//   them transposed; LPK = HD / 8 lanes share a V row, P crosses lanes through LDS inside the wave.
//   The next block's K is requested as soon as S is formed, its V as soon as P V is: a wave has 8 to 16 KB in flight.
// A work-group per 64 keys with everything on the vector ALU spent its time there and on 130 partial values per head
// and 64 keys; at 8 sequences: 2048 keys 27 us, 8192 keys of the 8-bit cache 70 + 10 us (with the merge).
// Per 32 keys of the 8-bit cache a wave issues about 480 vector instructions (row numbers formed once per key and passed
// between lanes, codes to bf16 two per instruction), 750 before; three work-groups per CU need the launch bound (180
// registers without it: 650 us a step).  8 sequences of 8192 tokens: 623 -> 605 us a step of four layers; steps over bf16 entries
// take what they took.
// GT: compile-time bound of the number of query heads per KV head (registers and loops are sized by it).
// FUSED: RoPE + append inside this kernel (a.qkv_raw given).
template <int HD, int GT, bool FUSED, bool FP8, int NB>
__global__ __launch_bounds__(256, (HD <= 128 && GT <= 4) ? 3 : 1 /* work-groups per CU */) void attn_decode_split_kernel(AttnDecodeArgs a, float scale) {
  constexpr int KS = HD / 32;                       // MFMA steps over the head dim
  constexpr int LPK = HD / 8, KPL = 64 / LPK;       // lanes per V row, V rows per load
  constexpr int VL = 16 / KPL;                      // V loads per 16 keys
  constexpr int HALF = HD / 2;
  typedef typename std::conditional<FP8, uint2, uint4>::type chunk_t;   // 8 elements
  __shared__ float ps[4][NB * 16][GT];              // P of a wave's block, then unused
  __shared__ float al[4][GT];                       // rescaling factors of a wave
  __shared__ float red[4][GT][HD];
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
  const int r16 = lane & 15, g4 = lane >> 4;        // key (K operand) or query head (Q operand); k chunk
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
  uint32_t row_k[NB];                               // row of this lane's key (r16) in each group of the next block
  chunk_t kw[NB][KS], vw[NB][VL];
  auto load_pages = [&](int blk) {
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const int key = key_of((blk * NB + n) * 16 + r16);
      row_k[n] = row_of(key, bt[key >> lgP]);
    }
  };
  auto load_k = [&] {
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const chunk_t* p = k_pool + chunk_of(row_k[n]) + g4;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kw[n][ks] = p[ks * 4];
    }
  };
  uint32_t row_v[NB];                               // rows of the block whose V is loaded next
  auto load_v = [&] {
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int i = 0; i < VL; ++i) vw[n][i] = v_pool[chunk_of((uint32_t)__shfl((int)row_v[n], i * KPL + vs, 64)) + li];
  };
  // the first block's entries travel while the query rows are prepared
  load_pages(wave);
#pragma unroll
  for (int n = 0; n < NB; ++n) row_v[n] = row_k[n];
  if (wave < n_blocks) {
    load_k();
    load_v();
  }

  auto as_chunk = [](const uint4& w) {
    if constexpr (FP8) return make_uint2(w.x, w.y);
    else return w;
  };

  // ---- query rows: lane l holds head r16 (zeros beyond G), dims 32 ks + 8 g4 .. + 7, as bf16.  The other member of
  //      a rotation pair, HALF dims on, is the same lane's chunk ks + KS / 2.
  bf16x8_t qf[KS];
  // FUSED: the query position's own entry, in registers as loaded from the pools; with two key groups per block in LDS (K row, V
  // row), a copy per wave: in registers it made the form for three and four heads of 128 spill at three work-groups per CU
  // (four layers of a step over an 8-bit cache, us: 1 sequence of 32000 tokens 493 -> 470, of 64000 567 -> 544, with three heads
  // per KV head 482 -> 465 and 562 -> 540).  Where nothing spills the way through LDS only delays
  // the wave (bf16 entries, one sequence of 2048 tokens: 406.7 -> 408.3).
  constexpr bool NEW_IN_LDS = FUSED && NB == 2;
  __shared__ chunk_t entry_new[NEW_IN_LDS ? 4 : 1][2][LPK];
  chunk_t k_new[KS], v_new = as_chunk(make_uint4(0, 0, 0, 0));
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
    head_row((kvh * G + min(r16, G - 1)) * HD, a.q_gamma, x);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint4 w = r16 < G ? make_uint4(pack_bf16x2(x[ks][0], x[ks][1]), pack_bf16x2(x[ks][2], x[ks][3]),
                                           pack_bf16x2(x[ks][4], x[ks][5]), pack_bf16x2(x[ks][6], x[ks][7]))
                              : make_uint4(0, 0, 0, 0);
      qf[ks] = __builtin_bit_cast(bf16x8_t, w);
    }
    if (has_new) {
      head_row((a.n_q_heads + kvh) * HD, a.k_gamma, x);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        k_new[ks] = as_chunk(pack8(x[ks], a.kvq.k_inv));
        if (NEW_IN_LDS && r16 == 0) entry_new[wave][0][ks * 4 + g4] = k_new[ks];
      }
      float v8[8];
      const float* row = a.qkv_raw + (size_t)b * a.ld + (a.n_q_heads + a.n_kv_heads + kvh) * HD + li * 8;
#pragma unroll
      for (int e = 0; e < 8; ++e) v8[e] = row[e];
      v_new = as_chunk(pack8(v8, a.kvq.v_inv));
      if constexpr (NEW_IN_LDS) {
        if (vs == 0) entry_new[wave][1][li] = v_new;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the wave's own LDS writes, read by its other lanes
      }
    }
  } else {
    const bf16_t* q = a.q + ((size_t)b * a.n_q_heads + kvh * G + min(r16, G - 1)) * HD + g4 * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint4 w = *reinterpret_cast<const uint4*>(q + ks * 32);
      qf[ks] = __builtin_bit_cast(bf16x8_t, r16 < G ? w : make_uint4(0, 0, 0, 0));
    }
  }
  // FUSED, in the block that holds the query position's key (the split's last): the chunks loaded for it, also by
  // lanes that repeat it, are replaced by the new entry, and the lanes whose key it is store it.
  auto patch_k = [&](int blk) {
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const int kk = (blk * NB + n) * 16 + r16, key = key_of(kk);
      if (key != qpos) continue;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kw[n][ks] = NEW_IN_LDS ? entry_new[wave][0][ks * 4 + g4] : k_new[ks];
      if (kk == n_keys - 1) {
        chunk_t* o = reinterpret_cast<chunk_t*>(const_cast<bf16_t*>(a.k_pool)) + chunk_of(row_of(key, bt[key >> lgP])) + g4;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) o[ks * 4] = kw[n][ks];
      }
    }
  };
  auto patch_v = [&](int blk) {
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int i = 0; i < VL; ++i) {
        const int kk = (blk * NB + n) * 16 + i * KPL + vs, key = key_of(kk);
        if (key != qpos) continue;
        vw[n][i] = NEW_IN_LDS ? entry_new[wave][1][li] : v_new;
        if (kk == n_keys - 1)
          reinterpret_cast<chunk_t*>(const_cast<bf16_t*>(a.v_pool))[chunk_of(row_of(key, bt[key >> lgP])) + li] = vw[n][i];
      }
  };
  // a chunk of K as the MFMA operand
  auto k_operand = [&](const chunk_t& w) {
    if constexpr (FP8) return e4m3_to_bf16x8(w);
    else return __builtin_bit_cast(bf16x8_t, w);
  };
  const float s_scale = FP8 ? scale * a.kvq.k_scale : scale;
  float acc[GT][8];
#pragma unroll
  for (int g = 0; g < GT; ++g)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[g][e] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;             // of query head r16; l_run: this lane's keys

  for (int blk = wave; blk < n_blocks; blk += 4) {
    const bool last_block = blk == n_blocks - 1;
    if (FUSED && has_new && last_block) {
      patch_k(blk);
      patch_v(blk);
    }
    if (blk + 4 < n_blocks) load_pages(blk + 4);
    floatx4_t s[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      s[n] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        s[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k_operand(kw[n][ks]), qf[ks], s[n], 0, 0, 0);
    }
    if (blk + 4 < n_blocks) load_k();
    // s[n][v]: query head r16, key 16 n + 4 g4 + v of the block
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
    if (r16 < G) {
#pragma unroll
      for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int v = 0; v < 4; ++v) ps[wave][n * 16 + 4 * g4 + v][r16 % GT] = s[n][v];
    }
    l_run = l_run * alpha + sum;
    const bool moved = __builtin_amdgcn_ballot_w64(r16 < G && alpha != 1.f) != 0;
    if (moved && g4 == 0 && r16 < G) al[wave][r16 % GT] = alpha;
    m_run = m_new;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the wave's own LDS writes, read by its other lanes
    if (moved) {
#pragma unroll
      for (int g = 0; g < GT; ++g)
        if (g < G) {
          const float f = al[wave][g];
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[g][e] *= f;
        }
    }
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int i = 0; i < VL; ++i) {
        float vf[8];
        if constexpr (FP8) {
          e4m3_decode4_hw(vw[n][i].x, vf);
          e4m3_decode4_hw(vw[n][i].y, vf + 4);
        } else {
          const uint4 w = vw[n][i];
          vf[0] = bf16lo(w.x); vf[1] = bf16hi(w.x); vf[2] = bf16lo(w.y); vf[3] = bf16hi(w.y);
          vf[4] = bf16lo(w.z); vf[5] = bf16hi(w.z); vf[6] = bf16lo(w.w); vf[7] = bf16hi(w.w);
        }
#pragma unroll
        for (int g = 0; g < GT; ++g)
          if (GT <= 4 || g < G) {     // (three of four heads: the fourth's sums are formed and dropped)
            const float pv = ps[wave][n * 16 + i * KPL + vs][g];
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[g][e] += pv * vf[e];
          }
      }
    if (blk + 4 < n_blocks) {
#pragma unroll
      for (int n = 0; n < NB; ++n) row_v[n] = row_k[n];
      load_v();
    }
    asm volatile("" ::: "memory");                  // the next block's P is written after this block's was read
  }

  // ---- the wave's key slots, then the four waves, each with its own maximum
  l_run += __shfl_xor(l_run, 16, 64);
  l_run += __shfl_xor(l_run, 32, 64);
  if (g4 == 0 && r16 < G) {
    stat[wave][0][r16 % GT] = m_run;
    stat[wave][1][r16 % GT] = l_run;
  }
  {
    constexpr int NV = GT * 8;
    float v[NV];
#pragma unroll
    for (int g = 0; g < GT; ++g)
#pragma unroll
      for (int e = 0; e < 8; ++e) v[g * 8 + e] = acc[g][e];
    const int first = fold_keys<LPK, NV>(v, lane);
#pragma unroll
    for (int i = 0; i < NV * LPK / 64; ++i) {
      const int idx = first + i, g = idx >> 3, e = idx & 7;
      if (g < G) red[wave][g][li * 8 + e] = v[i];
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
      num += f * red[w][g][e];
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

// Splits of the key range: about three work-groups per CU (what the kernel's registers allow), but no split of fewer
// than kDecodeKeysPerSplit = 64 keys (16 per wave); equal shares, in whole rounds of the four waves.  At most three, so that no few are left
// for a second round (four layers of a decode step, us, rounded up -> down: 64 sequences of 400 / 700 keys 665 -> 653 /
// 734 -> 706, 40 of 1000 664 -> 649, 8-bit 637 -> 619, 28 of 700 592 -> 587, 10 of 4000 632 -> 626); head size 256, with
// twice the bytes per work-group, keeps the finer cut (20 sequences of 700 keys 916, rounded down 922).
void choose_decode_splits(AttnDecodeArgs& a, int span) {
  const long long pairs = (long long)a.B * a.n_kv_heads;
  const long long per_pair = a.hd <= 128 ? 768 / pairs : (768 + pairs - 1) / pairs;
  const int want = (int)std::max(1LL, std::min<long long>((span + kDecodeKeysPerSplit - 1) / kDecodeKeysPerSplit, per_pair));
  const int keys = (span + want - 1) / want;
  a.split_keys = (keys + 63) / 64 * 64;
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
