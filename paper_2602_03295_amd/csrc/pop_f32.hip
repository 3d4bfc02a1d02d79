// fp32 instantiation of the POP prefill path: every step of Sec. 2.1 / Sec. 3.3 with fp32 weights,
// activations and cache entries and fp32 accumulation.  It exists for tight numerical checks on small
// models (max relative error 1e-4 against an fp64 reference instead of the 2e-2 of the bf16 path).  Such models are
// small: a call is a chain of short launches whose latency counts, so the kernels cut every step into many waves and
// keep the chain short (the norms run inside the projections that read them).  All products on the fp32 MFMA
// (v_mfma_f32_16x16x4_f32, fp32 inputs and accumulation).
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "pop_device.h"
#include "pop_kernels.h"

namespace pop {
namespace f32 {

namespace impl {

// h[t,:] = row_src[t] < 0 ? table[tokens[t],:] : embeds[row_src[t],:]
__global__ void embed_kernel(const float* __restrict__ table, const int32_t* __restrict__ tokens,
                             const int32_t* __restrict__ row_src, const float* __restrict__ embeds,
                             float* __restrict__ h, int T, int d, RopeTables tabs) {
  const int t = blockIdx.x;
  if (t >= T) {                // the blocks after the rows: the RoPE tables
    rope_tables_block(tabs, t - T);
    return;
  }
  const int rs = row_src ? row_src[t] : -1;
  const float* src = rs < 0 ? table + (size_t)tokens[t] * d : embeds + (size_t)rs * d;
  for (int i = threadIdx.x; i < d; i += blockDim.x) h[(size_t)t * d + i] = src[i];
}

__device__ __forceinline__ float glu_act(float g, int act) {
  if (act == 0) return g / (1.f + expf(-g));
  const float u = 0.7978845608028654f * (g + 0.044715f * g * g * g);
  return 0.5f * g * (1.f + tanhf(u));
}

// C = A[M,K] W[N,K]^T.  A wave computes TM x TN blocks of 16 x 16 (GLU: of the gate and of the up columns); the
// work-group is KW waves that share a tile and split K between them (their sums meet in LDS, in wave order), or
// KW = 1 and 2 x 2 waves with a tile each.  Operands come straight from global memory: lane l of a load holds 4
// consecutive k of row l % 16, at 4 (l / 16) of a 16-wide k chunk, so one 16-byte load per operand block feeds four
// MFMAs (MFMA j contracts k = 4 g + j of the chunk, g = 0..3, the same on both sides).
// Bound by latency at the sizes this path is for, hence the split of K inside the work-group: 128 rows, N = 512,
// K = 256: 256 work-groups of 8 waves with 2 chunks each (64 x 64 tiles with one wave's worth of parallelism per SIMD
// took 47 us, this 5 us; N = 256, K = 688: 160 and 6 us).
// A wave's last chunks are loaded two at a time: with four, of which K = 256 leaves a wave two, the masked ones cost as much as the
// others (128 rows: gate|up of 2 x 688 columns 10.5 -> 7.7 us, O 4.6 -> 3.8; a call of 8 layers 271 -> 232 us).
// NORM: the rows of A are RMS-normalised on the way (the LN of Sec. 2.1): C = rstd (A * gamma) W^T, with the sum of
// squares taken from the same loads.  row_idx: row m of A is A[row_idx[m]].
// EPI: 0 store, 1 out += scale C, 2 out = act(A Wg^T) * (A Wu^T) with Wg = W rows 0..N-1, Wu = rows N..2N-1,
// EPI_QKV (KW > 1): RoPE and the append (RopeAppend).  A work-group's columns are then rotation pairs, the first half of them
// dims pair0, pair0 + 1, .. of a head and the others their partners, and the tables are read before the products.  The append
// as a kernel of its own, which formed its angles in fp64, was one launch in six: 8 layers of 128 rows 288 -> 271 us.
constexpr int EPI_QKV = 3;
struct GemmF32 {
  const float* A;
  const float* W;
  float* out;
  const int32_t* row_idx;
  const float* gamma;
  int lda, ldw, ldc, M, N, K, act;
  float eps, scale;
  RopeAppend ra;     // EPI_QKV
};

template <int TM, int TN, int KW, int EPI, bool NORM>
__global__ __launch_bounds__(KW == 1 ? 256 : 64 * KW) void gemm_kernel(GemmF32 p) {
  constexpr int NB = EPI == EPI_GLU ? 2 * TN : TN;     // W blocks of a wave
  constexpr int U = TM * NB >= 8 ? 2 : 4;              // chunks of 16 k requested together (2 where no more are left)
  __shared__ float4 red[KW > 1 ? KW : 1][KW > 1 ? TM * NB : 1][64];
  __shared__ float red_ss[KW][TM][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r16 = lane & 15, g = lane >> 4;
  const int kw = KW > 1 ? wave : 0;
  const int m0 = (KW > 1 ? blockIdx.y : blockIdx.y * 2 + (wave >> 1)) * TM * 16;
  const int n0 = (KW > 1 ? blockIdx.x : blockIdx.x * 2 + (wave & 1)) * TN * 16;
  static_assert(EPI != EPI_QKV || (KW >= TM && KW > 1 && TN <= 2), "a wave finishes all columns of 16 rows");
  // Who finishes a block of a split (EPI_QKV: 16 rows with all their columns): with more waves than blocks ES waves, each NE of
  // the four columns that a lane holds, where one wave added eight parts and evaluated four activations per lane while the
  // others idled (128 rows: gate|up of 2 x 688 columns 7.7 -> 7.4 us, QKV 4.8 -> 4.7).
  constexpr int JN = EPI == EPI_QKV ? 1 : TN, UP = EPI == EPI_GLU ? TN : EPI == EPI_QKV ? TN - 1 : 0;   // `up`: the block UP on
  constexpr int ES = KW < 2 * TM * JN ? 1 : KW < 4 * TM * JN ? 2 : 4, NE = 4 / ES;
  const int hd = EPI == EPI_QKV ? p.ra.hd : 0, half = hd >> 1;
  const int head = EPI == EPI_QKV ? n0 / hd : 0, pair0 = EPI == EPI_QKV ? n0 % hd / 2 : 0;
  // rows and columns beyond the matrix repeat its last one (never stored)
  const float* ar[TM];
  const float* wr[NB];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = min(m0 + i * 16 + r16, p.M - 1);
    ar[i] = p.A + (size_t)(p.row_idx ? p.row_idx[m] : m) * p.lda + 4 * g;
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    int n = min(n0 + (j % TN) * 16 + r16, p.N - 1);
    if (EPI == EPI_QKV) {      // (N is a multiple of the tile's columns)
      const int c = j * 16 + r16;
      n = head * hd + pair0 + c % (TN * 8) + c / (TN * 8) * half;
    }
    wr[j] = p.W + (size_t)(j < TN ? n : p.N + n) * p.ldw + 4 * g;
  }
  floatx4_t acc[TM][NB];
  float ss[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    ss[i] = 0.f;
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  }
  // EPI_QKV: (cos, sin) of the pairs that this wave will finish, NE per lane, and the rows' slots
  float2 cs[NE];
  int slot = 0;
  if (EPI == EPI_QKV) {
    const int m = min(m0 + min(wave / ES, TM - 1) * 16 + r16, p.M - 1);
    const float2* c = p.ra.cs + (size_t)(p.ra.cs_row ? p.ra.cs_row[m] : m) * half + pair0 + (TN == 1 ? 4 * (g & 1) : 4 * g) + wave % ES * NE;
#pragma unroll
    for (int e = 0; e < NE; ++e) cs[e] = c[e];
    slot = p.ra.slot[m];
  }
  const int chunks = (p.K + 15) >> 4, per = (chunks + KW - 1) / KW;
  const int c_end = min(chunks, (kw + 1) * per);
  auto step = [&](int c0, auto u_c) {
    constexpr int U = decltype(u_c)::value;
    // Loads without branches, so that all of a step are in flight together: a lane beyond K, or of a chunk beyond
    // this wave's, reads the row's start and its activations are replaced by zeros.
    float4 a[U][TM], w[U][NB], gm[U];
    bool in[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      in[u] = c0 + u < c_end && (c0 + u) * 16 + 4 * g < p.K;      // (K is a multiple of 4)
      const int k = in[u] ? (c0 + u) * 16 : -4 * g;
#pragma unroll
      for (int i = 0; i < TM; ++i) a[u][i] = *reinterpret_cast<const float4*>(ar[i] + k);
#pragma unroll
      for (int j = 0; j < NB; ++j) w[u][j] = *reinterpret_cast<const float4*>(wr[j] + k);
      if (NORM) gm[u] = *reinterpret_cast<const float4*>(p.gamma + k + 4 * g);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        float4& v = a[u][i];
        v.x = in[u] ? v.x : 0.f; v.y = in[u] ? v.y : 0.f; v.z = in[u] ? v.z : 0.f; v.w = in[u] ? v.w : 0.f;
      }
      if (NORM) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          float4& v = a[u][i];
          ss[i] += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
          v.x *= gm[u].x; v.y *= gm[u].y; v.z *= gm[u].z; v.w *= gm[u].w;
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int i = 0; i < TM; ++i)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32((&w[u][j].x)[e], (&a[u][i].x)[e], acc[i][j], 0, 0, 0);
    }
  };
  int c0 = kw * per;
  if (U > 2)
    for (; c_end - c0 > 2; c0 += U) step(c0, std::integral_constant<int, U>{});
  for (; c0 < c_end; c0 += 2) step(c0, std::integral_constant<int, 2>{});
  // acc[i][j][v]: row m0 + 16 i + lane % 16, column n0 + 16 j + 4 (lane / 16) + v
  if (NORM) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      ss[i] += __shfl_xor(ss[i], 16, 64);
      ss[i] += __shfl_xor(ss[i], 32, 64);
      if (KW > 1 && g == 0) red_ss[kw][i][r16] = ss[i];
    }
  }
  if (KW > 1) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
        red[kw][i * NB + j][lane] = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
    __syncthreads();
  }
  // wave w of a split finishes blocks w / ES, (w + KW) / ES, ...; without a split every wave its own
  for (int item = KW > 1 ? wave : 0; item < TM * JN * ES; item += KW) {
    const int blk = item / ES, e0 = item % ES * NE, i = blk / JN, j = blk % JN;
    float c[NE], up[NE];
    float sq = 0.f;
    if (KW > 1) {
      auto part = [&](int k, int b) { return reinterpret_cast<const float*>(&red[k][i * NB + b][lane]) + e0; };
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        c[e] = part(0, j)[e];
        up[e] = part(0, UP + j)[e];
      }
      if (NORM) sq = red_ss[0][i][r16];
#pragma unroll
      for (int k = 1; k < KW; ++k) {
#pragma unroll
        for (int e = 0; e < NE; ++e) {
          c[e] += part(k, j)[e];
          if (UP > 0) up[e] += part(k, UP + j)[e];
        }
        if (NORM) sq += red_ss[k][i][r16];
      }
    } else {
      // (constant indices: the loop is unrolled over the blocks)
#pragma unroll
      for (int q = 0; q < TM * TN; ++q)
        if (q == blk) {
          const floatx4_t x = acc[q / TN][q % TN], y = acc[q / TN][EPI == EPI_GLU ? TN + q % TN : q % TN];
#pragma unroll
          for (int e = 0; e < NE; ++e) {
            c[e] = x[e];
            up[e] = y[e];
          }
          sq = ss[q / TN];
        }
    }
    const float rstd = NORM ? 1.0f / sqrtf(sq / (float)p.K + p.eps) : 1.f;
    const int m = m0 + i * 16 + r16, n = n0 + j * 16 + 4 * g + e0;
    auto store_ne = [&](float* o, const float (&v)[NE]) {
      if constexpr (NE == 4) *reinterpret_cast<float4*>(o) = make_float4(v[0], v[1], v[2], v[3]);
      else if constexpr (NE == 2) *reinterpret_cast<float2*>(o) = make_float2(v[0], v[1]);
      else *o = v[0];
    };
    if constexpr (EPI == EPI_QKV) {
      // x: this lane's values (with 32 columns the low halves of its pairs), y: their partners.  16 columns: lane groups 0, 1
      // have the low halves of 8 pairs, lane groups 2, 3 the high ones
      float x[NE], y[NE];
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        x[e] = c[e] * rstd;
        y[e] = TN == 1 ? __shfl_xor(x[e], 32, 64) : up[e] * rstd;
      }
      const bool low = TN == 2 || g < 2;
      const RopeAppend& ra = p.ra;
      const bool rotate = head < ra.n_q_heads + ra.n_kv_heads;
      if (rotate) {
#pragma unroll
        for (int e = 0; e < NE; ++e) {
          const float a = low ? x[e] * cs[e].x - y[e] * cs[e].y : x[e] * cs[e].x + y[e] * cs[e].y;
          y[e] = y[e] * cs[e].x + x[e] * cs[e].y;      // (used with 32 columns)
          x[e] = a;
        }
      }
      if (m >= p.M) continue;
      auto store = [&](const float (&v)[NE], int dim) {
        if (head < ra.n_q_heads) {
          store_ne(p.out + (size_t)m * p.ldc + head * hd + dim, v);
          return;
        }
        const int hh = rotate ? head - ra.n_q_heads : head - ra.n_q_heads - ra.n_kv_heads;
        float* o = (rotate ? ra.k_pool : ra.v_pool) +
                   (((size_t)(slot / ra.page_size) * ra.n_kv_heads + hh) * ra.page_size + slot % ra.page_size) * hd + dim;
        float w[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e)   // 8-bit cache: the fp32 entry holds the value of the e4m3 code the element rounds to
          w[e] = !ra.kvq.fp8 ? v[e]
                             : e4m3_decode(e4m3_encode(v[e] * (rotate ? ra.kvq.k_inv : ra.kvq.v_inv))) *
                                   (rotate ? ra.kvq.k_scale : ra.kvq.v_scale);
        store_ne(o, w);
      };
      const int dim = pair0 + (TN == 1 ? 4 * (g & 1) : 4 * g) + e0;
      store(x, low ? dim : dim + half);
      if (TN == 2) store(y, dim + half);
      continue;
    }
    if (m >= p.M) continue;
    float* o = p.out + (size_t)m * p.ldc + n;
    if (n + NE - 1 < p.N && (p.ldc & 3) == 0) {     // all columns at once
      float old[NE], r[NE];
      if (EPI == EPI_ADD) {
#pragma unroll
        for (int e = 0; e < NE; ++e) old[e] = o[e];
      }
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const float x = c[e] * rstd;
        r[e] = EPI == EPI_ADD ? old[e] + x * p.scale : EPI == EPI_GLU ? glu_act(x, p.act) * (up[e] * rstd) : x;
      }
      store_ne(o, r);
      continue;
    }
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      if (n + e >= p.N) break;
      const float x = c[e] * rstd;
      if (EPI == EPI_STORE) o[e] = x;
      else if (EPI == EPI_ADD) o[e] += x * p.scale;
      else o[e] = glu_act(x, p.act) * (up[e] * rstd);
    }
  }
}

// RoPE (half-split pairs, angle formed in fp64) of the q and k heads of `rows` rows in place, and
// append of k, v to the paged cache at slot[row].  grid (rows, Hq + 2 Hkv), hd/2 threads rounded up to whole
// waves.  With q_gamma / k_gamma every query / key head is RMS-normalised over hd first (per-head QK-norm).
__global__ void rope_write_kernel(float* __restrict__ qkv, int ld, int q_col, int k_col, int v_col, int n_q_heads,
                                  int n_kv_heads, int hd, const int32_t* __restrict__ pos,
                                  const int32_t* __restrict__ slot, double neg2_over_hd_log2theta,
                                  float* __restrict__ k_pool, float* __restrict__ v_pool, int P,
                                  const float* __restrict__ q_gamma, const float* __restrict__ k_gamma, float qk_eps,
                                  KvQuant kvq) {
  __shared__ float red[2];
  const int r = blockIdx.x, head = blockIdx.y;
  const int half = hd >> 1;
  const int i = threadIdx.x;      // whole waves: 64 or 128 threads, the first `half` of them work
  const bool act = i < half;
  const int s = slot[r];
  float* row = qkv + (size_t)r * ld;
  if (head < n_q_heads + n_kv_heads) {
    const bool is_q = head < n_q_heads;
    if (is_q && q_col < 0) return;
    float* x = row + (is_q ? q_col + head * hd : k_col + (head - n_q_heads) * hd);
    float a = act ? x[i] : 0.f, b = act ? x[i + half] : 0.f;
    const float* gamma = is_q ? q_gamma : k_gamma;
    if (gamma) {   // per-head QK-norm before the rotation (uniform over the block)
      const float ss = wave_sum(a * a + b * b);
      if ((i & 63) == 0) red[i >> 6] = ss;
      __syncthreads();
      const float tot = blockDim.x > 64 ? red[0] + red[1] : red[0];
      const float rstd = 1.0f / sqrtf(tot / (float)hd + qk_eps);
      if (act) {
        a *= rstd * gamma[i];
        b *= rstd * gamma[i + half];
      }
    }
    if (!act) return;
    const double ang = (double)pos[r] * exp2((double)i * neg2_over_hd_log2theta);
    double sd, cd;
    sincos(ang, &sd, &cd);
    const float c = (float)cd, sn = (float)sd;
    const float lo = a * c - b * sn, hi = b * c + a * sn;
    x[i] = lo;
    x[i + half] = hi;
    if (!is_q) {
      // 8-bit cache: the fp32 entry holds the value of the e4m3 code the element rounds to
      float* o = k_pool + (((size_t)(s / P) * n_kv_heads + (head - n_q_heads)) * P + (s % P)) * hd;
      o[i] = kvq.fp8 ? e4m3_decode(e4m3_encode(lo * kvq.k_inv)) * kvq.k_scale : lo;
      o[i + half] = kvq.fp8 ? e4m3_decode(e4m3_encode(hi * kvq.k_inv)) * kvq.k_scale : hi;
    }
  } else {
    if (!act) return;
    const int hh = head - n_q_heads - n_kv_heads;
    const float* x = row + v_col + hh * hd;
    float* o = v_pool + (((size_t)(s / P) * n_kv_heads + hh) * P + (s % P)) * hd;
    o[i] = kvq.fp8 ? e4m3_decode(e4m3_encode(x[i] * kvq.v_inv)) * kvq.v_scale : x[i];
    o[i + half] = kvq.fp8 ? e4m3_decode(e4m3_encode(x[i + half] * kvq.v_inv)) * kvq.v_scale : x[i + half];
  }
}

// First key a row at position pos of sequence b sees: max(0, pos - window + 1) (window > 0) or 0, and not below the
// first position the layer holds an entry for (kv_first[b], if given; the row's own entry always exists).
__device__ __forceinline__ int first_key(int pos, int b, int window, const int32_t* kv_first) {
  const int lo = window > 0 ? max(0, pos - window + 1) : 0;
  return kv_first ? max(lo, min(kv_first[b], pos)) : lo;
}

struct AttnF32 {
  const float* q;
  int ldq, q_col;
  float* out;
  const int32_t* row_seq;
  const int32_t* row_pos;
  const float* k_pool;
  const float* v_pool;
  const int32_t* block_table;
  int max_pages, lgP, window;      // pages of 2^lgP entries
  const int32_t* kv_first;
  int rows, n_q_heads, n_kv_heads;
  float scale;
};

// Attn of Sec. 2.1 for one (row, query head) per work-group against the paged cache of the row's sequence (rows of
// different sequences: decode steps, boundary rows).  HD/4 lanes share a key, 16 bytes each; scores live in LDS.
// Every four passes wait for the block table and then for the entries, for K and again for V, hence NT = 1024 threads where
// 256 take more than four passes (heads of 64: 64 keys) and the work-groups find a CU each: one row of 4 heads over 128 keys
// 8.2 -> 6.5 us.  With fewer keys the barriers of 16 waves cost more (5 rows over 4 to 12 keys, a call 222 us, 224 with 1024).
template <int HD, int NT>
__global__ __launch_bounds__(NT) void attention_kernel(AttnF32 a) {
  constexpr int LPK = HD / 4, KPI = NT / LPK, NW = NT / 64;   // lanes per key, keys per pass of the work-group, waves
  extern __shared__ float sc[];                    // [n keys]
  __shared__ float red[NW];
  __shared__ float4 red_o[NW][LPK];
  auto over_waves = [&](auto op) {
    float v = red[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) v = op(v, red[w]);
    return v;
  };
  const int r = blockIdx.x, head = blockIdx.y, tid = threadIdx.x;
  const int b = a.row_seq[r], pos = a.row_pos[r];
  const int lo = first_key(pos, b, a.window, a.kv_first);
  const int n = pos - lo + 1;
  const int kvh = head / (a.n_q_heads / a.n_kv_heads);
  const int32_t* bt = a.block_table + (size_t)b * a.max_pages;
  const int li = tid % LPK, ks = tid / LPK;
  auto entry = [&](const float* pool, int key) {
    return *reinterpret_cast<const float4*>(
        pool + ((((size_t)bt[key >> a.lgP] * a.n_kv_heads + kvh) << a.lgP) + (key & ((1 << a.lgP) - 1))) * HD + li * 4);
  };
  const float4 qv = *reinterpret_cast<const float4*>(a.q + (size_t)r * a.ldq + a.q_col + head * HD + li * 4);
  float mx = -INFINITY;
#pragma unroll 4
  for (int j0 = 0; j0 < n; j0 += KPI) {            // (uniform over the block: the sums below cross lanes)
    const int j = j0 + ks;
    const float4 kv = entry(a.k_pool, lo + min(j, n - 1));
    float s = qv.x * kv.x + qv.y * kv.y + qv.z * kv.z + qv.w * kv.w;
    s = group_sum<16>(s);
    if (LPK > 16) s += __shfl_xor(s, 16, 64);
    if (LPK > 32) s += __shfl_xor(s, 32, 64);
    s *= a.scale;
    if (j < n) {
      if (li == 0) sc[j] = s;
      mx = fmaxf(mx, s);
    }
  }
  mx = wave_max(mx);
  if ((tid & 63) == 0) red[tid >> 6] = mx;
  __syncthreads();
  mx = over_waves([](float x, float y) { return fmaxf(x, y); });
  __syncthreads();
  float sum = 0.f;
  for (int j = tid; j < n; j += NT) {
    const float pv = expf(sc[j] - mx);
    sc[j] = pv;
    sum += pv;
  }
  sum = wave_sum(sum);
  if ((tid & 63) == 0) red[tid >> 6] = sum;
  __syncthreads();
  const float tot = over_waves([](float x, float y) { return x + y; });
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
  for (int j = ks; j < n; j += KPI) {
    const float4 v = entry(a.v_pool, lo + j);
    const float pv = sc[j];
    acc.x += pv * v.x; acc.y += pv * v.y; acc.z += pv * v.z; acc.w += pv * v.w;
  }
  // the keys of a wave, then the waves in order
#pragma unroll
  for (int w = LPK; w < 64; w *= 2) {
    acc.x += __shfl_xor(acc.x, w, 64); acc.y += __shfl_xor(acc.y, w, 64);
    acc.z += __shfl_xor(acc.z, w, 64); acc.w += __shfl_xor(acc.w, w, 64);
  }
  if ((tid & 63) < LPK) red_o[tid >> 6][li] = acc;
  __syncthreads();
  if (tid < LPK) {
    float4 o = red_o[0][tid];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      const float4 x = red_o[w][tid];
      o.x += x.x; o.y += x.y; o.z += x.z; o.w += x.w;
    }
    *reinterpret_cast<float4*>(a.out + (size_t)r * a.n_q_heads * HD + head * HD + tid * 4) =
        make_float4(o.x / tot, o.y / tot, o.z / tot, o.w / tot);
  }
}

// The same for packed prompt rows: a work-group takes 16 consecutive rows of one query head, its waves the blocks of 16
// keys in turn (four waves; eight with heads of 64 and more than 64 keys, where a second block per wave is a second chain of dependent loads: 128
// rows of 4 heads 7.0 -> 6.7 us, pages found by shifts instead of divisions included).  S^T = K Q^T and O^T += V^T P^T on the MFMA with a running maximum and sum per wave; a
// lane then holds 4 keys of one row, which are the operand of the second product as they are (MFMA j takes key
// 4 g + j from lane group g).  The waves' results meet in LDS.  Rows of different sequences in one tile are taken
// sequence by sequence.  One work-group per row and head re-read every entry 16 times as often and waited for each
// (30 us for 128 rows of 4 heads, 5 us now).
template <int HD, int NW>
__global__ __launch_bounds__(64 * NW) void attention_tile_kernel(AttnF32 a) {
  constexpr int C = HD / 16;
  extern __shared__ float smem[];                  // [NW waves][16 rows][HD + 4]
  __shared__ float red_m[NW][16], red_l[NW][16], red_f[NW][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r16 = lane & 15, g = lane >> 4;
  const int head = blockIdx.y, kvh = head / (a.n_q_heads / a.n_kv_heads);
  const int t0 = blockIdx.x * 16, tile_end = min(t0 + 16, a.rows);
  // lane i (and i + 16, ..) looks at row t0 + i; the rows of a sequence are found without further loads
  const int seq_i = a.row_seq[min(t0 + r16, a.rows - 1)], pos_i = a.row_pos[min(t0 + r16, a.rows - 1)];
  for (int r0 = t0; r0 < tile_end;) {
    const int b = __builtin_amdgcn_readlane(seq_i, r0 - t0);
    const uint32_t others = (uint32_t)__builtin_amdgcn_ballot_w64(seq_i != b) & 0xffffu & (0xffffffffu << (r0 - t0));
    const int r1 = others ? min(t0 + __ffs(others) - 1, tile_end) : tile_end;   // rows r0 .. r1-1 of sequence b
    const int row = min(r0 + r16, r1 - 1);
    const int pos = __shfl(pos_i, row - t0, 64);                                // positions ascending
    const int lo = first_key(pos, b, a.window, a.kv_first);
    const int k_lo = __builtin_amdgcn_readfirstlane(lo);                        // lane 0 has row r0
    const int k_hi = __builtin_amdgcn_readlane(pos_i, r1 - 1 - t0);
    // keys that all rows see: from the last row's first one (lane 15 has that row) to the first row's position
    const int all_lo = __builtin_amdgcn_readlane(lo, 15), all_hi = __builtin_amdgcn_readfirstlane(pos);
    const int32_t* bt = a.block_table + (size_t)b * a.max_pages;
    auto entry = [&](const float* pool, int key) {
      return pool + ((((size_t)bt[key >> a.lgP] * a.n_kv_heads + kvh) << a.lgP) + (key & ((1 << a.lgP) - 1))) * HD;
    };
    float4 qf[C];
#pragma unroll
    for (int c = 0; c < C; ++c)
      qf[c] = *reinterpret_cast<const float4*>(a.q + (size_t)row * a.ldq + a.q_col + head * HD + c * 16 + 4 * g);
    floatx4_t o[C];
#pragma unroll
    for (int c = 0; c < C; ++c) o[c] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;
    for (int k0 = k_lo + wave * 16; k0 <= k_hi; k0 += NW * 16) {
      // keys beyond the last one repeat it (masked below)
      const float* kp = entry(a.k_pool, min(k0 + r16, k_hi)) + 4 * g;
      const float* vp[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) vp[j] = entry(a.v_pool, min(k0 + 4 * g + j, k_hi)) + r16;
      float4 kf[C];
      float vf[C][4];
#pragma unroll
      for (int c = 0; c < C; ++c) kf[c] = *reinterpret_cast<const float4*>(kp + c * 16);
      if (HD <= 128) {
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int j = 0; j < 4; ++j) vf[c][j] = vp[j][c * 16];
      }
      floatx4_t s = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          s = __builtin_amdgcn_mfma_f32_16x16x4f32((&kf[c].x)[e], (&qf[c].x)[e], s, 0, 0, 0);
      // s[v]: row r16, key k0 + 4 g + v
      float mx = -INFINITY;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int key = k0 + 4 * g + v;
        s[v] = key >= lo && key <= pos ? s[v] * a.scale : -INFINITY;
        mx = fmaxf(mx, s[v]);
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float m_new = fmaxf(m_run, mx);
      const float m_use = m_new == -INFINITY ? 0.f : m_new;     // (no key of this row yet)
      const float alpha = expf(m_run - m_use);
      float p[4], sum = 0.f;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        p[v] = expf(s[v] - m_use);
        sum += p[v];
      }
      l_run = l_run * alpha + sum;       // this lane group's keys; the groups are added at the end
      m_run = m_new;
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) o[c][v] *= alpha;
      // A row must not meet a key that it does not see, not even with P = 0 if that key's V is not finite: such blocks
      // (only those that some row sees in part can hold one) are added key by key.
      bool by_key = false;
      if (k0 < all_lo || k0 + 15 > all_hi) {
        float z = 0.f;
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int j = 0; j < 4; ++j) z += 0.f * (HD <= 128 ? vf[c][j] : vp[j][c * 16]);
        by_key = __builtin_amdgcn_ballot_w64(!(z == 0.f)) != 0;
      }
      if (by_key) {
#pragma unroll 1
        for (int kg = 0; kg < 4; ++kg) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int key = k0 + 4 * kg + j;
            const float pk = __shfl(p[j], 16 * kg + r16, 64);
            const bool seen = key >= lo && key <= pos;
            const float* vk = entry(a.v_pool, min(key, k_hi)) + 4 * g;
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
              for (int v = 0; v < 4; ++v) o[c][v] += seen ? pk * vk[c * 16 + v] : 0.f;
          }
        }
      } else {
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            o[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(HD <= 128 ? vf[c][j] : vp[j][c * 16], p[j], o[c], 0, 0, 0);
      }
    }
    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);
    // o[c][v]: row r16, head-dim 16 c + 4 g + v
    if (g == 0) { red_m[wave][r16] = m_run; red_l[wave][r16] = l_run; }
#pragma unroll
    for (int c = 0; c < C; ++c)
      *reinterpret_cast<float4*>(smem + (wave * 16 + r16) * (HD + 4) + c * 16 + 4 * g) =
          make_float4(o[c][0], o[c][1], o[c][2], o[c][3]);
    __syncthreads();
    if (threadIdx.x < NW * 16) {                                 // every wave's factor, once
      const int w = threadIdx.x >> 4, r = threadIdx.x & 15;
      float m = red_m[0][r];
#pragma unroll
      for (int v = 1; v < NW; ++v) m = fmaxf(m, red_m[v][r]);
      red_f[w][r] = expf(red_m[w][r] - m);                       // (a wave without keys: exp(-inf) = 0)
    }
    __syncthreads();
    for (int it = threadIdx.x; it < (r1 - r0) * (HD / 4); it += 64 * NW) {
      const int r = it / (HD / 4), i = it % (HD / 4) * 4;
      float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
      float den = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float f = red_f[w][r];
        const float4 x = *reinterpret_cast<const float4*>(smem + (w * 16 + r) * (HD + 4) + i);
        num.x += f * x.x; num.y += f * x.y; num.z += f * x.z; num.w += f * x.w;
        den += f * red_l[w][r];
      }
      *reinterpret_cast<float4*>(a.out + (size_t)(r0 + r) * a.n_q_heads * HD + head * HD + i) =
          make_float4(num.x / den, num.y / den, num.z / den, num.w / den);
    }
    __syncthreads();                                             // before the next sequence reuses LDS
    r0 = r1;
  }
}

}  // namespace impl

void launch_embed(const float* table, const int32_t* tokens, const int32_t* row_src, const float* embeds, float* h,
                  int T, int d, hipStream_t st, const RopeTables& tabs) {
  if (T <= 0) return;
  hipLaunchKernelGGL(impl::embed_kernel, dim3(T + tabs.blocks()), dim3(256), 0, st, table, tokens, row_src, embeds, h, T, d, tabs);
}

namespace impl {
template <int EPI, bool NORM>
void launch_gemm_en(const GemmF32& p, hipStream_t st) {
  auto up = [](int x, int t) { return (x + t - 1) / t; };
  // The smallest tiles until every CU has two work-groups, then 32 x 32, from four rounds of those on 64 x 64 per
  // wave (128 x 128 per work-group; GLU half as wide), which need a quarter of the loads per product.
  if ((long long)up(p.M, 16) * up(p.N, 16) <= 512) {
    hipLaunchKernelGGL((gemm_kernel<1, 1, 8, EPI, NORM>), dim3(up(p.N, 16), up(p.M, 16)), dim3(512), 0, st, p);
  } else if ((long long)up(p.M, 32) * up(p.N, 32) <= 4096) {
    hipLaunchKernelGGL((gemm_kernel<2, 2, 4, EPI, NORM>), dim3(up(p.N, 32), up(p.M, 32)), dim3(256), 0, st, p);
  } else {
    constexpr int TN = EPI == EPI_GLU ? 2 : 4;
    hipLaunchKernelGGL((gemm_kernel<4, TN, 1, EPI, NORM>), dim3(up(p.N, 32 * TN), up(p.M, 128)), dim3(256), 0, st, p);
  }
}
// The two forms whose waves split K; more work than that (where one launch less is nothing) takes the append kernel.
bool qkv_small(int M, int N) { return (long long)((M + 15) / 16) * ((N + 15) / 16) <= 512; }
template <bool NORM>
void launch_gemm_n(const GemmF32& p, int epi, hipStream_t st) {
  if (p.M <= 0 || p.N <= 0) return;
  if (epi == EPI_STORE) launch_gemm_en<EPI_STORE, NORM>(p, st);
  else if (epi == EPI_ADD) launch_gemm_en<EPI_ADD, NORM>(p, st);
  else launch_gemm_en<EPI_GLU, NORM>(p, st);
}
}  // namespace impl

void launch_gemm(const float* A, int lda, const float* W, int ldw, float* out, int ldc, int M, int N, int K, int epi,
                 int act, hipStream_t st, float scale) {
  impl::launch_gemm_n<false>(impl::GemmF32{A, W, out, nullptr, nullptr, lda, ldw, ldc, M, N, K, act, 0.f, scale, {}}, epi, st);
}

void launch_norm_gemm(const float* x, const int32_t* row_idx, const float* gamma, float eps, const float* W, float* out,
                      int ldc, int M, int N, int K, int epi, int act, hipStream_t st) {
  impl::launch_gemm_n<true>(impl::GemmF32{x, W, out, row_idx, gamma, K, K, ldc, M, N, K, act, eps, 1.f, {}}, epi, st);
}

bool norm_qkv_supported(int M, int N, int hd) {
  return hd % 32 == 0 && N % hd == 0 && (impl::qkv_small(M, N) || (long long)((M + 31) / 32) * ((N + 31) / 32) <= 4096);
}

void launch_norm_qkv(const float* x, const int32_t* row_idx, const float* gamma, float eps, const float* W, float* out,
                     int ldc, int M, int K, const RopeAppend& ra, hipStream_t st) {
  if (M <= 0) return;
  const int N = (ra.n_q_heads + 2 * ra.n_kv_heads) * ra.hd;
  const impl::GemmF32 p{x, W, out, row_idx, gamma, K, K, ldc, M, N, K, 0, eps, 1.f, ra};
  if (impl::qkv_small(M, N))
    hipLaunchKernelGGL((impl::gemm_kernel<1, 1, 8, impl::EPI_QKV, true>), dim3(N / 16, (M + 15) / 16), dim3(512), 0, st, p);
  else
    hipLaunchKernelGGL((impl::gemm_kernel<2, 2, 4, impl::EPI_QKV, true>), dim3(N / 32, (M + 31) / 32), dim3(256), 0, st, p);
}

void launch_rope_write(float* qkv, int ld, int q_col, int k_col, int v_col, int n_q_heads, int n_kv_heads, int hd,
                       const int32_t* pos, const int32_t* slot, double theta, float* k_pool, float* v_pool, int P,
                       int rows, hipStream_t st, const float* q_gamma, const float* k_gamma, float qk_eps, KvQuant kvq) {
  if (rows <= 0) return;
  hipLaunchKernelGGL(impl::rope_write_kernel, dim3(rows, n_q_heads + 2 * n_kv_heads), dim3((hd / 2 + 63) / 64 * 64), 0, st, qkv, ld,
                     q_col, k_col, v_col, n_q_heads, n_kv_heads, hd, pos, slot, -2.0 / (double)hd * log2(theta), k_pool,
                     v_pool, P, q_gamma, k_gamma, qk_eps, kvq);
}

namespace impl {
template <int HD, int NW>
hipError_t launch_attention_tile(const AttnF32& a, hipStream_t st) {
  constexpr size_t smem = (size_t)NW * 16 * (HD + 4) * sizeof(float);
  // once per form; the initialisation of a function-local static is thread-safe
  static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&attention_tile_kernel<HD, NW>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (attr_err != hipSuccess) return attr_err;
  hipLaunchKernelGGL((attention_tile_kernel<HD, NW>), dim3((a.rows + 15) / 16, a.n_q_heads), dim3(64 * NW), smem, st, a);
  return hipGetLastError();
}
template <int HD>
hipError_t launch_attention_hd(const AttnF32& a, bool packed, int max_len, hipStream_t st) {
  if (packed) {
    if constexpr (HD == 64) {       // (wider heads spill with eight waves)
      if (max_len > 64) return launch_attention_tile<HD, 8>(a, st);
    }
    return launch_attention_tile<HD, 4>(a, st);
  } else {
    const dim3 grid(a.rows, a.n_q_heads);
    if (max_len > 64 && (long long)a.rows * a.n_q_heads <= 256) {
      static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&attention_kernel<HD, 1024>),
                                                             hipFuncAttributeMaxDynamicSharedMemorySize, kMaxContext * (int)sizeof(float));
      if (attr_err != hipSuccess) return attr_err;
      hipLaunchKernelGGL((attention_kernel<HD, 1024>), grid, dim3(1024), (size_t)max_len * sizeof(float), st, a);
    } else {
      hipLaunchKernelGGL((attention_kernel<HD, 256>), grid, dim3(256), (size_t)max_len * sizeof(float), st, a);
    }
  }
  return hipGetLastError();
}
}  // namespace impl

hipError_t launch_attention(const float* q, int ldq, int q_col, float* out, const int32_t* row_seq,
                            const int32_t* row_pos, const float* k_pool, const float* v_pool,
                            const int32_t* block_table, int max_pages, int P, int window, const int32_t* kv_first, int rows, int n_q_heads,
                            int n_kv_heads, int hd, int max_len, bool packed, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  if (max_len > kMaxContext) return hipErrorInvalidValue;
  const impl::AttnF32 a{q, ldq, q_col, out, row_seq, row_pos, k_pool, v_pool, block_table, max_pages, __builtin_ctz(P), window, kv_first,
                        rows, n_q_heads, n_kv_heads, 1.f / sqrtf((float)hd)};
  switch (hd) {
    case 64: return impl::launch_attention_hd<64>(a, packed, max_len, st);
    case 128: return impl::launch_attention_hd<128>(a, packed, max_len, st);
    case 256: return impl::launch_attention_hd<256>(a, packed, max_len, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace f32
}  // namespace pop
