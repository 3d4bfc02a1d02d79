// Causal grouped-query flash attention for the prompt body (the Attn block of Sec. 2.1 applied to
// all body rows of a kept layer at once), packed variable-length sequences, optional sliding window.
//
// A wave owns 32 query rows of one query head.  Keys/values stream through LDS in tiles of 64, staged with
// buffer_load ... lds in a ring.  What bounds it at head size 128: power.  The matrix pipe is busy 63 % of the cycles at 8192
// tokens and 70 % at 32768, at the 1.62 and 1.56 GHz that the power limit leaves; per step of 64 keys and 256 rows, 2048
// cycles of MFMAs, 2 x 790 of vector instructions, 512 of the address unit for the staged tiles.  At 2048 tokens it is busy 37 %
// at 1.84 GHz: two rounds of work-groups of unequal length, with a start and an end each (profiles/attention_prefill_hd128_*).
//
// Inside this kernel Q, K, V and P are fp16 (the RoPE/append kernel hands over fp16 copies; the cache
// itself stays bf16): with random-like V the softmax average shrinks signal and rounding noise alike, so
// the relative error of the output equals that of the individual probabilities, and bf16's 8-bit
// mantissa in q, k and P was the largest error source of a whole layer.  P <= 2^kMaxLag and
// saturating conversions keep fp16's range safe.
//
// MFMA arrangement (v_mfma_f32_32x32x16_f16, D = A * B with A rows / B columns spread over lanes):
//   S^T = K * Q^T   : A = K tile rows (keys), B = Q rows.  A lane then owns ONE query row (lane & 31)
//                     and 16 keys per 32-key block, so the softmax row reductions are in-lane plus a
//                     single exchange with lane ^ 32.
//   O^T = V^T * P^T : A = rows of the pre-transposed V (head-dim index), B = P^T.  The S^T
//                     accumulator registers 8G..8G+7 of a block are exactly the B operand of the
//                     G-th 16-key step, because the keys are fed to the first MFMA in the permuted
//                     order key(i) below; no cross-lane data movement is needed for P.
// Softmax is computed in fp32 with exp2 and running (lagging) max / sum (online softmax); P is rounded to fp16
// for the second MFMA, O accumulates in fp32.
#include <type_traits>

#include "pop_device.h"
#include "pop_kernels.h"

namespace pop {

namespace attn_impl {

typedef __attribute__((address_space(3))) void* lds_ptr_t;
constexpr int BQ = 128;   // query rows per work-group
constexpr int BKV = 64;   // keys per LDS stage
// The running maximum is raised only when a row outgrows it by this much (in powers of two): P <= 2^8 stays far inside
// fp16, whose relative rounding does not depend on the magnitude, and O is rescaled a few times per row instead of in
// every tile that moves one of a wave's 32 maxima (prompts of 6144 / 32768 tokens: 7057 -> 6969, 61739 -> 60776 us).
constexpr float kMaxLag = 8.f;

// MFMA row i (0..31) of the S^T block is fed key row key_of_row(i) of the 32-key block, chosen so
// that accumulator registers 8G..8G+7 of lane-half h hold keys 16G + 8h + (0..7).
__device__ __forceinline__ int key_of_row(int i) {
  const int a = i >> 3, hb = (i >> 2) & 1, r = i & 3;
  return 16 * (a >> 1) + 8 * hb + 4 * (a & 1) + r;
}
// LDS swizzle of the K tile.  gfx950 serves a ds_read_b128 sixteen lanes (256 B = all 64 banks) per
// cycle, and the sixteen lanes of a phase read the sixteen rows of an aligned group (key_of_row
// permutes inside such a group).  Rows of >= 256 B each fill whole bank lines, so the sixteen rows need
// sixteen different chunk positions: key = row & 15.  128-byte rows (head_dim 64) share a bank line in
// pairs: key = (row >> 1) & 7 (the row's parity already selects the half line).
template <int ROW_BYTES>
__device__ __forceinline__ int k_swz(int row) {
  return ROW_BYTES >= 256 ? (row & 15) : ((row >> 1) & 7);
}

// Head size 256, whose O and Q leave no registers for two waves per SIMD: one or two tiles of 128 query rows of one query head
// per work-group (a late tile paired with an early one, which balances the causal triangle); 4 waves x 32 rows, one per SIMD.
__global__ __launch_bounds__(256) void attn_prefill256_kernel(AttnPrefillArgs a, float scale_log2) {
#if defined(__HIP_DEVICE_COMPILE__)  // the buffer-resource builtins exist in the device pass only
  constexpr int HD = 256;
  constexpr int KS = HD / 16;            // MFMA steps over the head dim for S
  constexpr int OB = HD / 32;            // 32-row blocks of O^T
  constexpr int K_ROW_BYTES = HD * 2;
  constexpr int K_CPR = HD / 8;          // 16-byte chunks per K row
  constexpr int K_RPL = 64 / K_CPR;      // K rows per wave-load
  constexpr int K_BYTES = BKV * K_ROW_BYTES;
  constexpr int V_BYTES = HD * BKV * 2;  // V^T tile: HD rows of 64 keys (128 B)
  constexpr int STAGE = K_BYTES + V_BYTES;
  constexpr int NST = 2;                 // LDS ring: K and V^T tiles are requested NST-1 iterations ahead
  constexpr int DPF = NST - 1;
  constexpr uint32_t kOOB = 0x80000000u;   // pushes a byte offset out of range: the lane stages zeros
  constexpr int K_LOADS = K_BYTES / 1024 / 4, V_LOADS = V_BYTES / 1024 / 4;  // per wave
  constexpr int LPI = K_LOADS + V_LOADS;   // wave-loads per iteration

  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

  const AttnTile tile = a.tiles[blockIdx.x];
  const int head = blockIdx.y;
  const int kvh = head / (a.n_q_heads / a.n_kv_heads);
  const int seq0 = tile.seq0, len = tile.len;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = lane >> 5;
  // one or two query tiles per work-group (a late and an early tile of the same sequence)
  for (int part = 0; part < 2; ++part) {
  const int q0 = part == 0 ? tile.start : tile.start2;
  if (q0 < 0) break;
  if (part == 1) __builtin_amdgcn_s_barrier();  // everyone is done with the first tile's LDS stages
  const int qrow = q0 + wave * 32 + (lane & 31);  // position of this lane's query row
  const bool qvalid = qrow < len;

  // ---- key range of this query tile
  const int q_last = min(q0 + BQ, len) - 1;
  int j_begin = 0;
  if (a.window > 0) j_begin = max(0, q0 - a.window + 1) & ~(BKV - 1);
  const int j_end = q_last + 1;  // exclusive
  const int n_kv = (j_end - j_begin + BKV - 1) / BKV;

  // ---- buffer descriptors
  const __amdgpu_buffer_rsrc_t rK = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(a.qkv), 0, (uint32_t)((long long)a.T * a.ld * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rV = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(a.vT), 0, (uint32_t)((long long)a.n_kv_heads * HD * a.Tp * 2), 0x00020000);

  // staging offsets (K: rows = keys; V^T: rows = head-dim index)
  uint32_t offK[K_LOADS], offV[V_LOADS];
#pragma unroll
  for (int j = 0; j < K_LOADS; ++j) {
    const int row = (j * 4 + wave) * K_RPL + lane / K_CPR;
    const int pchunk = lane % K_CPR;
    const int c = pchunk ^ k_swz<K_ROW_BYTES>(row);
    offK[j] = (uint32_t)((((long long)seq0 + row) * a.ld + a.k_col + kvh * HD + c * 8) * 2);
  }
#pragma unroll
  for (int j = 0; j < V_LOADS; ++j) {
    const int row = (j * 4 + wave) * 8 + (lane >> 3);
    const int c = (lane & 7) ^ ((row >> 1) & 7);
    offV[j] = (uint32_t)((((long long)kvh * HD + row) * a.Tp + tile.vt_off + c * 8) * 2);
  }
  // The key offset goes into the per-lane offset (not the scalar one) so that rows beyond the end of
  // the buffer are range-checked and read as zero.
  // Key tile `it` of this query tile goes to ring slot it % NST.  Tiles beyond the key range are
  // requested with every lane out of range (zeros are staged), so that each iteration issues the same
  // number of loads and the vmcnt bookkeeping below stays uniform.
  auto issue_k1 = [&](int j, int it) {
    const int j0 = j_begin + it * BKV;
    unsigned char* sk = smem + (it % NST) * STAGE;
    const uint32_t mask = it < n_kv ? 0u : kOOB;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rK, (lds_ptr_t)(sk + (j * 4 + wave) * 1024), 16,
                                             (offK[j] + (uint32_t)(j0 * a.ld * 2)) | mask, 0, 0, 0);
  };
  auto issue_v1 = [&](int j, int it) {
    const int j0 = j_begin + it * BKV;
    unsigned char* sv = smem + (it % NST) * STAGE + K_BYTES;
    const uint32_t mask = it < n_kv ? 0u : kOOB;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rV, (lds_ptr_t)(sv + (j * 4 + wave) * 1024), 16,
                                             (offV[j] + (uint32_t)(j0 * 2)) | mask, 0, 0, 0);
  };
  auto issue_k = [&](int it) {
#pragma unroll
    for (int j = 0; j < K_LOADS; ++j) issue_k1(j, it);
  };
  auto issue_v = [&](int it) {
#pragma unroll
    for (int j = 0; j < V_LOADS; ++j) issue_v1(j, it);
  };

  // ---- Q fragments (B operand: lane = query row, 8 consecutive head-dim values per step)
  f16x8_t qf[KS];
  {
    const bf16_t* qp = a.qkv + ((long long)seq0 + (qvalid ? qrow : 0)) * a.ld + a.q_col + head * HD + h * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const f16x8_t*>(qp + ks * 16);
  }

  floatx16_t o[OB];
#pragma unroll
  for (int i = 0; i < OB; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[i][v] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;

  // LDS fragment addresses
  const int krow = key_of_row(lane & 31);
  const int k_frag = krow * K_ROW_BYTES;
  const int k_sw = k_swz<K_ROW_BYTES>(krow);  // same for krow + 32 (only bits 0..3 of the row are used)
  const int v_frag = (lane & 31) * 128;
  const int v_sw = ((lane & 31) >> 1) & 7;

  const int wave_first = q0 + wave * 32;       // first / last query position this wave owns
  const int wave_last = wave_first + 31;

  // The key loop is software pipelined so that the matrix pipe and the vector ALU work at the same
  // time inside one wave: iteration t runs the softmax of key tile t on the vector ALU and, sprinkled
  // between its instructions, the MFMAs of O^T += V^T P^T for tile t-1 and of S^T = K Q^T for tile
  // t+1.  The MFMAs of an iteration are cut into 32 slots, one per exponential.  LDS stage (t+1)&1
  // holds K of tile t+1 and V^T of tile t-1 during iteration t; K of tile t+2 and V^T of tile t are
  // requested at its start into the other stage, whose contents were consumed in iteration t-1.
  constexpr int PVN = 4 * OB;          // MFMAs of one O update, index (kb*2+g)*OB + i
  constexpr int SN = 2 * KS;           // MFMAs of one S tile, index ks*2 + kb
  constexpr int NM = PVN + SN;
  constexpr int DIST = 4;              // fragment reads run this many MFMAs ahead
  // S^T of the current and of the next tile, the packed fp16 P^T of the current and of the last one (copied at the end of an
  // iteration: there are no registers to spare for a loop unrolled by two)
  floatx16_t s_cur[2], s_next[2];
  uint32_t pw[2][2][4], pw_prev[2][2][4];
  typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
  typedef float float2_t __attribute__((ext_vector_type(2)));
  const floatx16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  // mask of a diagonal / window-edge tile: register v of block kb on lane-half h holds key
  // j0 + kb*32 + 16*(v/8) + 8*h + (v%8)
  auto mask_tile = [&](floatx16_t(&sv_)[2], int j0) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int key = j0 + kb * 32 + 16 * (v >> 3) + 8 * h + (v & 7);
        bool ok = key <= qrow;
        if (a.window > 0) ok = ok && (key > qrow - a.window);
        if (!ok) sv_[kb][v] = -INFINITY;
      }
  };
  auto tile_needs_mask = [&](int j0) {
    return (j0 + BKV - 1 > wave_first) || (a.window > 0 && j0 < wave_last - a.window + 1);
  };
  // row maximum of the tile the next iteration works on: this lane's half (mx_part) and the other
  // half of the row (mx_other, lane ^ 32, fetched through the LDS crossbar)
  float mx_part = -INFINITY, mx_other = -INFINITY;

  auto body = [&](int t, auto has_pv_c, auto has_s_c) {
    constexpr bool HAS_PV = decltype(has_pv_c)::value, HAS_S = decltype(has_s_c)::value;
    // MFMAs of this iteration in issue order: S^T of tile t+1 (slots 0..15), then the O update with
    // tile t-1 (slots 16..31).  Once S^T is complete its row maximum is formed in the later slots, so
    // the next iteration starts its exponentials at once.
    constexpr int NS = HAS_S ? SN : 0, NP = HAS_PV ? PVN : 0, CNT = NS + NP;
    // K of tile t+1 and V^T of tile t-1 were requested DPF iterations ago; the loads of the
    // iterations in between may still be in flight (loads return in order).
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((DPF - 1) * LPI) : "memory");
    __builtin_amdgcn_s_barrier();
    const unsigned char* sk = smem + ((t + 1) % NST) * STAGE;
    const unsigned char* sv = smem + ((t + NST - 1) % NST) * STAGE + K_BYTES;
    const int tk = t + 1 + DPF, tv = t - 1 + DPF;   // tiles requested during this iteration

    f16x8_t fr[SN + PVN];
    auto frag_read = [&](int n) {          // n-th MFMA of this iteration
      if (n < NS) {
        const int ks = n / 2, kb = n % 2;
        const int pc = ((2 * ks + h) ^ k_sw) * 16;
        fr[n] = *reinterpret_cast<const f16x8_t*>(sk + k_frag + kb * 32 * K_ROW_BYTES + pc);
      } else {
        const int idx = n - NS;
        const int kb = idx / (2 * OB), g = (idx / OB) % 2, i = idx % OB;
        const int pc = ((4 * kb + 2 * g + h) ^ v_sw) * 16;
        fr[n] = *reinterpret_cast<const f16x8_t*>(sv + v_frag + i * 32 * 128 + pc);
      }
    };
    auto do_mfma = [&](int n) {
      if (n < NS) {
        const int ks = n / 2, kb = n % 2;
        s_next[kb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fr[n], qf[ks], ks == 0 ? zero16 : s_next[kb], 0, 0, 0);
      } else {
        const int idx = n - NS;
        const int kb = idx / (2 * OB), g = (idx / OB) % 2, i = idx % OB;
        const uint4 w4 = make_uint4(pw_prev[kb][g][0], pw_prev[kb][g][1], pw_prev[kb][g][2], pw_prev[kb][g][3]);
        o[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fr[n], __builtin_bit_cast(f16x8_t, w4), o[i], 0, 0, 0);
      }
    };
    auto first_of = [](int slot) {   // MFMAs issued before `slot`
      const int s1 = slot < 16 ? slot : 16, s2 = slot < 16 ? 0 : slot - 16;
      return s1 * NS / 16 + s2 * NP / 16;
    };
#pragma unroll
    for (int n = 0; n < DIST && n < CNT; ++n) frag_read(n);

    const float mx = fmaxf(mx_part, mx_other) * scale_log2;
    const bool raise = mx > m_run + kMaxLag;                     // (m_run = -inf: any finite maximum)
    const float m_new = raise ? mx : m_run;
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    float psum = 0.f;
    // the exponentials are skewed over the slots (argument two slots ahead, exp one slot ahead, sum
    // and packing in the slot itself) so that consecutive vector instructions do not wait on each other
    float xa[32], ea[32];
    xa[0] = s_cur[0][0] * scale_log2 - m_use;
    xa[1] = s_cur[0][1] * scale_log2 - m_use;
    ea[0] = __builtin_amdgcn_exp2f(xa[0]);
    float mxa = -INFINITY, mxb = -INFINITY;   // two chains of the next tile's row maximum
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int slot = 0; slot < 32; ++slot) {
      const int lo = first_of(slot), hi = first_of(slot + 1);
#pragma unroll
      for (int n = lo + DIST; n < hi + DIST; ++n)
        if (n < CNT) frag_read(n);
      if (slot % (32 / LPI) == 0) {   // one global load every few slots
        const int q = slot / (32 / LPI);
        if (q < K_LOADS) issue_k1(q, tk);
        else issue_v1(q - K_LOADS, tv);
      }
      if (slot + 2 < 32) {
        xa[slot + 2] = s_cur[(slot + 2) >> 4][(slot + 2) & 15] * scale_log2 - m_use;
        asm volatile("" : "+v"(xa[slot + 2]));
      }
      if (slot + 1 < 32) {
        ea[slot + 1] = __builtin_amdgcn_exp2f(xa[slot + 1]);
        asm volatile("" : "+v"(ea[slot + 1]));
      }
      {
        const int kb = slot >> 4, v = slot & 15;
        psum += ea[slot];
        if (v & 1) {
          // 0 <= P <= 2^kMaxLag: plain round-to-nearest packing, no saturation needed
          const float2_t pp = {ea[slot - 1], ea[slot]};
          pw[kb][v >> 3][(v & 7) >> 1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pp, half2_t));
          // keep the softmax arithmetic inside its slot (otherwise it is sunk below the loop's
          // last branch, behind all MFMAs, and nothing overlaps)
          asm volatile("" : "+v"(pw[kb][v >> 3][(v & 7) >> 1]), "+v"(psum));
        } else {
          asm volatile("" : "+v"(psum));
        }
      }
      if (HAS_S) {
        if (slot == 18) {
          const int j0n = j_begin + (t + 1) * BKV;
          if (tile_needs_mask(j0n)) mask_tile(s_next, j0n);
        }
        if (slot >= 20 && slot < 28) {   // 4 values per slot, two independent chains
          const int kb = (slot - 20) >> 2, v0 = ((slot - 20) & 3) * 4;
          mxa = fmaxf(fmaxf(mxa, s_next[kb][v0]), s_next[kb][v0 + 1]);
          mxb = fmaxf(fmaxf(mxb, s_next[kb][v0 + 2]), s_next[kb][v0 + 3]);
          asm volatile("" : "+v"(mxa), "+v"(mxb));
        }
        if (slot == 28) {
          mx_part = fmaxf(mxa, mxb);
          mx_other = __shfl_xor(mx_part, 32, 64);
        }
      }
#pragma unroll
      for (int n = lo; n < hi; ++n) do_mfma(n);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (__builtin_amdgcn_ballot_w64(raise)) {  // the running max moves for some row of this wave
      const float alpha = raise ? __builtin_amdgcn_exp2f(m_run - m_use) : 1.f;   // m_run = -inf -> 0
      l_run *= alpha;
#pragma unroll
      for (int i = 0; i < OB; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[i][v] *= alpha;
    }
    l_run += psum;
    m_run = m_new;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      if (HAS_S) s_cur[kb] = s_next[kb];
#pragma unroll
      for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) pw_prev[kb][g][e] = pw[kb][g][e];
    }
  };
  using std::true_type;
  using std::false_type;

  if (n_kv > 0) {
    // prologue: request K of tiles 0..DPF and V^T of tiles 0..DPF-2, then S of tile 0
    issue_k(0);
#pragma unroll
    for (int i = 1; i <= DPF; ++i) issue_k(i);
#pragma unroll
    for (int i = 0; i <= DPF - 2; ++i) issue_v(i);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(DPF * K_LOADS + (DPF - 1) * V_LOADS) : "memory");
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int pc = ((2 * ks + h) ^ k_sw) * 16;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const f16x8_t kf = *reinterpret_cast<const f16x8_t*>(smem + k_frag + kb * 32 * K_ROW_BYTES + pc);
        s_cur[kb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf, qf[ks], ks == 0 ? zero16 : s_cur[kb], 0, 0, 0);
      }
    }
    if (tile_needs_mask(j_begin)) mask_tile(s_cur, j_begin);
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int v = 0; v < 16; ++v) mx_part = fmaxf(mx_part, s_cur[kb][v]);
    mx_other = __shfl_xor(mx_part, 32, 64);
    // O update of the last tile (all remaining loads are masked ones; drain them before the ring is reused)
    auto last_pv = [&] {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      const unsigned char* sv = smem + ((n_kv - 1) % NST) * STAGE + K_BYTES;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          const int pc = ((4 * kb + 2 * g + h) ^ v_sw) * 16;
          const uint4 w4 = make_uint4(pw_prev[kb][g][0], pw_prev[kb][g][1], pw_prev[kb][g][2], pw_prev[kb][g][3]);
#pragma unroll
          for (int i = 0; i < OB; ++i) {
            const f16x8_t vf = *reinterpret_cast<const f16x8_t*>(sv + v_frag + i * 32 * 128 + pc);
            o[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf, __builtin_bit_cast(f16x8_t, w4), o[i], 0, 0, 0);
          }
        }
    };
    if (n_kv == 1) {
      body(0, false_type{}, false_type{});
    } else {
      body(0, false_type{}, true_type{});
      for (int t = 1; t < n_kv - 1; ++t) body(t, true_type{}, true_type{});
      body(n_kv - 1, true_type{}, false_type{});
    }
    last_pv();
  }

  // ---- normalise and store: lane owns query row qrow, head-dim i*32 + (v/4)*8 + 4h + v%4
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  if (!qvalid) continue;
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  bf16_t* op = a.out + ((long long)seq0 + qrow) * ((long long)a.n_q_heads * HD) + head * HD;
#pragma unroll
  for (int i = 0; i < OB; ++i)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      uint2 pk;
      pk.x = pack_bf16x2(o[i][g * 4 + 0] * inv, o[i][g * 4 + 1] * inv);
      pk.y = pack_bf16x2(o[i][g * 4 + 2] * inv, o[i][g * 4 + 3] * inv);
      *reinterpret_cast<uint2*>(op + i * 32 + g * 8 + h * 4) = pk;
    }
  }  // part
#endif
}

// Head sizes 64 and 128, a sequence of one key tile (up to 64 tokens): K and V^T are staged once by NW waves, two of which
// have 32 query rows each.  Through the loop of the eight-wave kernel such a sequence asks for four masked loads beside every
// real one, and a masked load takes the address unit as long (31 sequences of 40 tokens and one of 300, 32 query heads of
// 128, RoPE kernel included: 77.8 -> 69.5 us).
template <int HD, int NW>
__device__ __forceinline__ void attend_one_tile(const AttnPrefillArgs& a, float scale_log2, const AttnTile& tile, int head, int kvh,
                                                unsigned char* sk, unsigned char* sv) {
#if defined(__HIP_DEVICE_COMPILE__)  // the buffer-resource builtins exist in the device pass only
  constexpr int KS = HD / 16, OB = HD / 32, ROW = HD * 2, K_CPR = HD / 8, K_RPL = 64 / K_CPR;   // (as below)
  constexpr int LOADS = BKV * ROW / 1024 / NW;
  const int seq0 = tile.seq0, len = tile.len;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = lane >> 5, qrow = wave * 32 + (lane & 31);
  const bool qvalid = qrow < len;

  f16x8_t qf[KS];
  {
    const bf16_t* qp = a.qkv + ((long long)seq0 + (qvalid ? qrow : 0)) * a.ld + a.q_col + head * HD + h * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const f16x8_t*>(qp + ks * 16);
  }
  const __amdgpu_buffer_rsrc_t rK = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(a.qkv), 0, (uint32_t)((long long)a.T * a.ld * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rV = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(a.vT), 0, (uint32_t)((long long)a.n_kv_heads * HD * a.Tp * 2), 0x00020000);
#pragma unroll
  for (int j = 0; j < LOADS; ++j) {      // (rows beyond the end of the buffer read as zero)
    const int row = (j * NW + wave) * K_RPL + lane / K_CPR, c = (lane % K_CPR) ^ k_swz<ROW>(row);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        rK, (lds_ptr_t)(sk + (j * NW + wave) * 1024), 16,
        (uint32_t)((((long long)seq0 + row) * a.ld + a.k_col + kvh * HD + c * 8) * 2), 0, 0, 0);
  }
#pragma unroll
  for (int j = 0; j < LOADS; ++j) {
    const int row = (j * NW + wave) * 8 + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        rV, (lds_ptr_t)(sv + (j * NW + wave) * 1024), 16,
        (uint32_t)((((long long)kvh * HD + row) * a.Tp + tile.vt_off + c * 8) * 2), 0, 0, 0);
  }
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS) : "memory");      // K has landed
  __builtin_amdgcn_s_barrier();
  floatx16_t s[2];
  uint32_t pw[2][2][4];
  float l_run = 0.f;
  if (wave * 32 < len) {
    typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
    typedef float float2_t __attribute__((ext_vector_type(2)));
    const int krow = key_of_row(lane & 31);        // (same swizzle for krow + 32)
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
      for (int v = 0; v < 16; ++v) s[kb][v] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const f16x8_t kf = *reinterpret_cast<const f16x8_t*>(sk + (kb * 32 + krow) * ROW + ((2 * ks + h) ^ k_swz<ROW>(krow)) * 16);
        s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf, qf[ks], s[kb], 0, 0, 0);
      }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int key = kb * 32 + 16 * (v >> 3) + 8 * h + (v & 7);
        if (key > qrow || (a.window > 0 && key <= qrow - a.window)) s[kb][v] = -INFINITY;
        mx = fmaxf(mx, s[kb][v]);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * scale_log2;
    if (mx == -INFINITY) mx = 0.f;
    float sum0 = 0.f, sum1 = 0.f;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int v = 0; v < 16; v += 2) {
        const float2_t pp = {__builtin_amdgcn_exp2f(s[kb][v] * scale_log2 - mx), __builtin_amdgcn_exp2f(s[kb][v + 1] * scale_log2 - mx)};
        sum0 += pp.x;      // (two chains, as in the loop of the eight-wave kernel: the same bits)
        sum1 += pp.y;
        pw[kb][v >> 3][(v & 7) >> 1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pp, half2_t));
      }
    l_run = sum0 + sum1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                  // V^T has
  __builtin_amdgcn_s_barrier();
  if (wave * 32 >= len) return;
  floatx16_t o[OB];
  const int v_sw = ((lane & 31) >> 1) & 7;
#pragma unroll
  for (int i = 0; i < OB; ++i) {
#pragma unroll
    for (int v = 0; v < 16; ++v) o[i][v] = 0.f;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const f16x8_t vf = *reinterpret_cast<const f16x8_t*>(sv + (i * 32 + (lane & 31)) * 128 + ((4 * kb + 2 * g + h) ^ v_sw) * 16);
        const uint4 w4 = make_uint4(pw[kb][g][0], pw[kb][g][1], pw[kb][g][2], pw[kb][g][3]);
        o[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf, __builtin_bit_cast(f16x8_t, w4), o[i], 0, 0, 0);
      }
  }
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  if (!qvalid) return;
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  bf16_t* op = a.out + ((long long)seq0 + qrow) * ((long long)a.n_q_heads * HD) + head * HD + h * 4;
#pragma unroll
  for (int i = 0; i < OB; ++i)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<uint2*>(op + i * 32 + g * 8) = make_uint2(pack_bf16x2(o[i][g * 4] * inv, o[i][g * 4 + 1] * inv),
                                                                  pack_bf16x2(o[i][g * 4 + 2] * inv, o[i][g * 4 + 3] * inv));
#endif
}

// Head sizes 64 and 128: eight waves of 32 query rows, two per SIMD.  A wave's work on a tile of 64 keys is a matrix phase
// (S^T of the next tile, then O^T += V^T P^T of the last one: 32 MFMAs at head size 128) and a vector phase (softmax of
// S^T).  Waves 4-7 meet a step's barrier half a step later than waves 0-3, so that on every SIMD one wave feeds the matrix
// pipe while the other one computes exponentials.
//   SPLIT false: a tile of 256 query rows; a step is one tile of 64 keys that all waves share.
//   SPLIT true:  a tile of 128 query rows; a step is two tiles of keys, one for waves 0-3 and one for waves 4-7 (the same
//                rows), merged through LDS at the end: half the steps, for calls whose tiles do not fill the chip.
// One wave per SIMD that interleaved both phases (128 rows, three slots), against this kernel: 300 tokens 12.7 -> 11.8 us, 1000
// 27.2 -> 22.8, 2048 55.6 -> 48.6, 6144 378 -> 315, 8192 634 -> 520, 32768 9.9 -> 7.8 ms (0.87 -> 1.1 PFLOP/s).  Two key
// tiles per step throughout (twice the bytes through the address unit) took 9.1 ms there.
template <int HD, bool SPLIT>
__global__ __launch_bounds__(512) void attn_prefill8_kernel(AttnPrefillArgs a, float scale_log2) {
#if defined(__HIP_DEVICE_COMPILE__)  // the buffer-resource builtins exist in the device pass only
  constexpr int KS = HD / 16;            // MFMA steps over the head dim for S
  constexpr int OB = HD / 32;            // 32-row blocks of O^T
  constexpr int ROW = HD * 2;            // bytes of a K row
  constexpr int K_CPR = HD / 8;          // 16-byte chunks per K row
  constexpr int K_RPL = 64 / K_CPR;      // K rows per wave-load
  constexpr int TILE = BKV * ROW;        // bytes of a K tile, and of a V^T tile (HD rows of 64 keys)
  constexpr int TPS = SPLIT ? 2 : 1;     // key tiles per step
  constexpr int NST = SPLIT ? 2 : 4;     // LDS slots, of a step's K tiles and V^T tiles
  constexpr int SLOT = 2 * TPS * TILE;
  constexpr int LOADS = TPS * TILE / 1024 / 8;   // wave-loads of K (and of V^T) per wave and step
  constexpr uint32_t kOOB = 0x80000000u;       // pushes a byte offset out of range: the lane stages zeros

  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

  // consecutive work-groups (neighbouring XCDs) take different KV heads: the query heads of one share an XCD's L2
  const int kvh = blockIdx.x % a.n_kv_heads;
  const int head = kvh * (a.n_q_heads / a.n_kv_heads) + blockIdx.x / a.n_kv_heads;
  const AttnTile tile = a.tiles[blockIdx.y];
  if (tile.len <= BKV) {     // (a short sequence among longer ones)
    attend_one_tile<HD, 8>(a, scale_log2, tile, head, kvh, smem, smem + TILE);
    return;
  }
  const int q0 = tile.start, seq0 = tile.seq0, len = tile.len;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = wave >> 2;
  const int h = lane >> 5;
  // query positions of this wave (the two waves of a SIMD, w and w + 4, take neighbouring rows: nearly the same keys)
  const int wave_first = q0 + (SPLIT ? wave & 3 : (wave & 3) * 2 + grp) * 32, wave_last = wave_first + 31;
  const int qrow = wave_first + (lane & 31);      // position of this lane's query row
  const bool qvalid = qrow < len;

  // ---- key range of this query tile
  const int q_last = min(q0 + (SPLIT ? 128 : 256), len) - 1;
  int j_begin = 0;
  if (a.window > 0) j_begin = max(0, q0 - a.window + 1) & ~(BKV - 1);
  const int n_kv = (q_last + 1 - j_begin + BKV - 1) / BKV;
  const int n_steps = (n_kv + TPS - 1) / TPS;

  const __amdgpu_buffer_rsrc_t rK = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(a.qkv), 0, (uint32_t)((long long)a.T * a.ld * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rV = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(a.vT), 0, (uint32_t)((long long)a.n_kv_heads * HD * a.Tp * 2), 0x00020000);

  // ---- Q fragments (B operand: lane = query row, 8 consecutive head-dim values per step)
  f16x8_t qf[KS];
  {
    const bf16_t* qp = a.qkv + ((long long)seq0 + (qvalid ? qrow : 0)) * a.ld + a.q_col + head * HD + h * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const f16x8_t*>(qp + ks * 16);
  }

  // staging offsets of this wave's first wave-load (K: rows = keys; V^T: rows = head-dim index); the j-th one is 8 KB further
  // on in LDS: 8 * K_RPL keys, or 64 head-dim rows and from TILE on the second tile's keys
  uint32_t offK, offV;
  {
    const int row = wave * K_RPL + lane / K_CPR;
    const int c = (lane % K_CPR) ^ k_swz<ROW>(row);
    offK = (uint32_t)((((long long)seq0 + row) * a.ld + a.k_col + kvh * HD + c * 8) * 2);
    const int vrow = wave * 8 + (lane >> 3);
    const int vc = (lane & 7) ^ ((vrow >> 1) & 7);
    offV = (uint32_t)((((long long)kvh * HD + vrow) * a.Tp + tile.vt_off + vc * 8) * 2);
  }
  // Step t reads K of its tiles and V^T of those of step t - 1 (the O update runs a step behind), from slot t % NST.  The key
  // offset goes into the per-lane offset (not the scalar one) so that rows beyond the end of the buffer are range-checked
  // and read as zero; tiles outside the range are requested with every lane out of range, which keeps the number of loads
  // per step uniform for the vmcnt bookkeeping below.
  auto issue1 = [&](int t, int j) {      // wave-load j of step t: K, then V^T
    unsigned char* base = smem + (t % NST) * SLOT + wave * 1024;
    const int jj = j % LOADS, sub = jj * TPS / LOADS;            // sub: which of the step's tiles
    if (j < LOADS)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rK, (lds_ptr_t)(base + jj * 8192), 16,
          (offK + (uint32_t)((j_begin + t * TPS * BKV + jj * 8 * K_RPL) * a.ld * 2)) | (t * TPS + sub < n_kv ? 0u : kOOB), 0, 0, 0);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rV, (lds_ptr_t)(base + TPS * TILE + jj * 8192), 16,
          (offV + (uint32_t)((j_begin + ((t - 1) * TPS + sub) * BKV + (jj % (LOADS / TPS)) * 64 * a.Tp) * 2)) |
              (t > 0 && (t - 1) * TPS + sub < n_kv ? 0u : kOOB), 0, 0, 0);
  };
  auto issue = [&](int t) {
#pragma unroll
    for (int j = 0; j < 2 * LOADS; ++j) issue1(t, j);
  };
  // Barrier t: step t's tiles have landed (loads return in order) and nobody reads those of step t - 1 any more, whose slot is
  // refilled during step t.  With four slots those of step t + 1 have landed too (only the loads of step t + 2 may still
  // be in flight), which lets a wave read its first fragments ahead of the barrier.
  constexpr bool AHEAD = NST == 4;
  auto sync = [&] {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(AHEAD ? 2 * LOADS : 0) : "memory");
    __builtin_amdgcn_s_barrier();
  };
#pragma unroll
  for (int t = 0; t < NST - 1; ++t) issue(t);

  // LDS fragment addresses: chunk c of a row is at c ^ key(row), so that steps over the head dim (K) or the keys (V^T) are an
  // exclusive or on the address
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)smem;
  const int krow = key_of_row(lane & 31);        // (same key for krow + 32)
  const uint32_t k_frag = lds0 + (SPLIT ? grp : 0) * TILE + krow * ROW + (h ^ k_swz<ROW>(krow)) * 16;
  const uint32_t v_frag = lds0 + (TPS + (SPLIT ? grp : 0)) * TILE + (lane & 31) * 128 + (h ^ (((lane & 31) >> 1) & 7)) * 16;
  typedef const __attribute__((address_space(3))) f16x8_t* lds_frag_t;

  typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
  typedef float float2_t __attribute__((ext_vector_type(2)));
  const floatx16_t zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  floatx16_t o[OB];
#pragma unroll
  for (int i = 0; i < OB; ++i) o[i] = zero16;
  float m_run = -INFINITY, m_use = 0.f, l_run = 0.f;
  floatx16_t s[2];                     // S^T of the current tile
  uint32_t pw[2][2][4];                // and its packed fp16 P^T

  // the steps t_lo .. t_hi - 1 bring this wave a tile with a key that some of its rows see
  const int j_own = j_begin + (SPLIT ? grp : 0) * BKV;   // first key of this wave's tile in step 0
  int t_lo = 0, t_hi = 0;
  if (wave_first < len) {
    t_hi = min(n_steps, (wave_last - j_own + TPS * BKV) / (TPS * BKV));
    if (a.window > 0)      // tiles whose last key is before the window of the first row
      t_lo = max(0, wave_first - a.window + 1 - j_own - BKV + TPS * BKV) / (TPS * BKV);
  }
  constexpr int PVN = 4 * OB, SN = 2 * KS, DIST = 6;   // fragment reads run DIST MFMAs ahead
  f16x8_t pre[DIST];                     // the first fragments of the next matrix phase
  auto read_k = [&](int t, int n) {      // fragment of the n-th S^T MFMA of step t
    const int ks = n / 2, kb = n % 2;
    return *(lds_frag_t)(((k_frag + (uint32_t)(t % NST) * SLOT) ^ (ks * 32)) + kb * 32 * ROW);
  };
  auto prefetch = [&](int t) {
#pragma unroll
    for (int n = 0; n < DIST; ++n) pre[n] = read_k(t, n);
  };
  // matrix phase of step t; its share of the loads of step t + NST - 1 goes between the MFMAs (in one burst behind the
  // barrier the eight waves queue at the CU's one address unit)
  auto matrix_phase = [&](int t, auto has_s_c, auto has_pv_c) {
    constexpr bool HAS_S = decltype(has_s_c)::value, HAS_PV = decltype(has_pv_c)::value;
    constexpr int NS = HAS_S ? SN : 0, CNT = NS + (HAS_PV ? PVN : 0), GAP = CNT / (2 * LOADS);
    const uint32_t sv = v_frag + (uint32_t)(t % NST) * SLOT;
    f16x8_t fr[CNT];
    auto frag_read = [&](int n) {
      if (n < NS) {
        fr[n] = read_k(t, n);
      } else {
        const int idx = n - NS, kb = idx / (2 * OB), g = (idx / OB) % 2, i = idx % OB;
        fr[n] = *(lds_frag_t)((sv ^ (kb * 64 + g * 32)) + i * 32 * 128);
      }
    };
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int n = 0; n < DIST && n < CNT; ++n) {
      if (HAS_S && AHEAD) fr[n] = pre[n];
      else frag_read(n);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int n = 0; n < CNT; ++n) {
      if (n + DIST < CNT) frag_read(n + DIST);
      if (n < NS) {
        const int ks = n / 2, kb = n % 2;
        s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fr[n], qf[ks], ks == 0 ? zero16 : s[kb], 0, 0, 0);
      } else {
        const int idx = n - NS, kb = idx / (2 * OB), g = (idx / OB) % 2, i = idx % OB;
        const uint4 w4 = make_uint4(pw[kb][g][0], pw[kb][g][1], pw[kb][g][2], pw[kb][g][3]);
        o[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fr[n], __builtin_bit_cast(f16x8_t, w4), o[i], 0, 0, 0);
      }
      if (n % GAP == 0) issue1(t + NST - 1, n / GAP);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // vector phase: softmax of S^T of tile t (register v of block kb on lane-half h: key j0 + kb*32 + 16*(v/8) + 8*h + v%8)
  auto vector_phase = [&](int t) {
    const int j0 = j_own + t * TPS * BKV;
    if (j0 + BKV - 1 > wave_first || (a.window > 0 && j0 < wave_last - a.window + 1)) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int key = j0 + kb * 32 + 16 * (v >> 3) + 8 * h + (v & 7);
          bool ok = key <= qrow;
          if (a.window > 0) ok = ok && (key > qrow - a.window);
          if (!ok) s[kb][v] = -INFINITY;
        }
    }
    float mxa = -INFINITY, mxb = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      mxa = fmaxf(fmaxf(mxa, s[0][v]), s[0][v + 1]);
      mxb = fmaxf(fmaxf(mxb, s[1][v]), s[1][v + 1]);
    }
    // a lane sees half of its row's keys; the other half (lane ^ 32) matters only where some lane outgrows the maximum
    const float mx = fmaxf(mxa, mxb);
    if (__builtin_amdgcn_ballot_w64(mx * scale_log2 > m_run + kMaxLag)) {
      const float row_max = fmaxf(mx, __shfl_xor(mx, 32, 64)) * scale_log2;
      const bool raise = row_max > m_run + kMaxLag;                // (m_run = -inf: any finite maximum)
      const float m_new = raise ? row_max : m_run;
      const float alpha = raise ? __builtin_amdgcn_exp2f(m_run - m_new) : 1.f;   // m_run = -inf -> 0
      l_run *= alpha;
#pragma unroll
      for (int i = 0; i < OB; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[i][v] *= alpha;
      m_run = m_new;
      m_use = m_new == -INFINITY ? 0.f : m_new;
    }
    float sum0 = 0.f, sum1 = 0.f;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int v = 0; v < 16; v += 2) {
        const float e0 = __builtin_amdgcn_exp2f(s[kb][v] * scale_log2 - m_use);
        const float e1 = __builtin_amdgcn_exp2f(s[kb][v + 1] * scale_log2 - m_use);
        sum0 += e0;
        sum1 += e1;
        // 0 <= P <= 2^kMaxLag: plain round-to-nearest packing, no saturation needed
        const float2_t pp = {e0, e1};
        pw[kb][v >> 3][(v & 7) >> 1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pp, half2_t));
      }
    l_run += sum0 + sum1;
    __builtin_amdgcn_sched_barrier(0);
    if (AHEAD) prefetch(t + 1);
  };
  using std::true_type;
  using std::false_type;
  // Waves 0-3 meet barrier t before their matrix phase t, waves 4-7 meet barrier t + 1 after it: the same work in the same
  // order, half a step apart.  (Loops with the test at the end: with it at the start the compiler keeps two copies of O.)
  auto before = [&](int t) { if (grp == 0 && t > 0) sync(); };
  auto after = [&](int t) { if (grp == 1 && t < n_steps) sync(); };
  auto idle = [&](int t) { before(t); issue(t + NST - 1); after(t); };
  sync();
  int t = 0;
  if (t_hi > t_lo) {
    for (; t < t_lo; ++t) idle(t);
    before(t);
    if (AHEAD) prefetch(t);
    matrix_phase(t, true_type{}, false_type{});
    after(t);
    vector_phase(t);
    ++t;
    if (t < t_hi) {
      do {
        before(t);
        matrix_phase(t, true_type{}, true_type{});
        after(t);
        vector_phase(t);
      } while (++t < t_hi);
    }
    before(t);
    matrix_phase(t, false_type{}, true_type{});
    after(t);
    ++t;
  }
  for (; t <= n_steps; ++t) idle(t);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the masked loads of the last steps still target this group's LDS

  // ---- normalise and store.  A lane holds head-dims 32 i + 8 g + 4 h + (0..3) of its row; the halves of two groups g change
  // places with lane ^ 32, so that a lane stores 16 consecutive bytes.
  bf16_t* op = a.out + ((long long)seq0 + qrow) * ((long long)a.n_q_heads * HD) + head * HD + h * 8;
  auto store_pair = [&](bf16_t* p, uint2 lo, uint2 hi) {      // groups g, g + 1
    typedef uint32_t u2_t __attribute__((ext_vector_type(2)));
    const u2_t x = __builtin_amdgcn_permlane32_swap(lo.x, hi.x, false, false);
    const u2_t y = __builtin_amdgcn_permlane32_swap(lo.y, hi.y, false, false);
    if (qvalid) *reinterpret_cast<uint4*>(p) = make_uint4(x[0], y[0], x[1], y[1]);
  };
  if constexpr (!SPLIT) {
    const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
#pragma unroll
    for (int i = 0; i < OB; ++i)
#pragma unroll
      for (int g = 0; g < 4; g += 2) {
        uint2 pk[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int v = (g + e) * 4;
          pk[e] = make_uint2(pack_bf16x2(o[i][v] * inv, o[i][v + 1] * inv), pack_bf16x2(o[i][v + 2] * inv, o[i][v + 3] * inv));
        }
        store_pair(op + i * 32 + g * 8, pk[0], pk[1]);
      }
  } else {
    // the waves w and w + 4 hold partial results of the same rows: each hands half of its O blocks over (in the ring, which is
    // free once all have arrived) and stores the other half
    __builtin_amdgcn_s_barrier();
    constexpr int HB = OB / 2;
    float4* const mo = reinterpret_cast<float4*>(smem);                       // [wave][HB * 4][64]
    float2* const ms = reinterpret_cast<float2*>(smem + 8 * HB * 4 * 1024);   // [wave][64]
#pragma unroll
    for (int i = 0; i < HB; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const floatx16_t& x = grp == 0 ? o[i + HB] : o[i];
        mo[(wave * HB * 4 + i * 4 + g) * 64 + lane] = make_float4(x[g * 4], x[g * 4 + 1], x[g * 4 + 2], x[g * 4 + 3]);
      }
    ms[wave * 64 + lane] = make_float2(m_run, l_run);
    __syncthreads();
    const float2 other = ms[(wave ^ 4) * 64 + lane];
    const float m_all = fmaxf(m_run, other.x), m_ref = m_all == -INFINITY ? 0.f : m_all;
    const float f_own = __builtin_amdgcn_exp2f(m_run - m_ref), f_other = __builtin_amdgcn_exp2f(other.x - m_ref);
    float l_tot = l_run * f_own + other.y * f_other;
    l_tot += __shfl_xor(l_tot, 32, 64);
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    const float wo = f_own * inv, wx = f_other * inv;
#pragma unroll
    for (int i = 0; i < HB; ++i)
#pragma unroll
      for (int g = 0; g < 4; g += 2) {
        uint2 pk[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const floatx16_t& x = grp == 0 ? o[i] : o[i + HB];
          const float4 y = mo[((wave ^ 4) * HB * 4 + i * 4 + g + e) * 64 + lane];
          const int v = (g + e) * 4;
          pk[e] = make_uint2(pack_bf16x2(x[v] * wo + y.x * wx, x[v + 1] * wo + y.y * wx),
                             pack_bf16x2(x[v + 2] * wo + y.z * wx, x[v + 3] * wo + y.w * wx));
        }
        store_pair(op + (grp * HB + i) * 32 + g * 8, pk[0], pk[1]);
      }
  }
#endif
}

// Sequences of one key tile by themselves.  In the kernel above six of its eight waves idle with them, and its ring leaves
// room for one work-group per CU: latency bound, four rounds for 32 sequences.  Here a CU holds five work-groups.  32 query
// heads of 128, RoPE kernel included, there -> here: 32 sequences of 16 tokens 52.4 -> 38.6 us, of 64 tokens 66.9 -> 51.7, 64
// of 40 tokens 99.9 -> 63.8 (four waves with a work-group per tile of 128 rows took 49.3, 62.9 and 89.7).
template <int HD>
__global__ __launch_bounds__(128, 2) void attn_prefill64_kernel(AttnPrefillArgs a, float scale_log2) {
  __shared__ __attribute__((aligned(1024))) unsigned char sk[BKV * HD * 2], sv[BKV * HD * 2];
  const int kvh = blockIdx.x % a.n_kv_heads;
  const int head = kvh * (a.n_q_heads / a.n_kv_heads) + blockIdx.x / a.n_kv_heads;
  attend_one_tile<HD, 2>(a, scale_log2, a.tiles[blockIdx.y], head, kvh, sk, sv);
}

template <int HD, bool SPLIT>
hipError_t launch8(const AttnPrefillArgs& a, hipStream_t st) {
  constexpr int smem = 8 * BKV * HD * 2;
  static_assert(smem >= 8 * (HD / 64) * 4 * 1024 + 8 * 64 * 8, "the merge uses the ring");
  // once per form; the initialisation of a function-local static is thread-safe
  static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_prefill8_kernel<HD, SPLIT>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  if (attr_err != hipSuccess) return attr_err;
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)HD);
  hipLaunchKernelGGL((attn_prefill8_kernel<HD, SPLIT>), dim3(a.n_q_heads, a.n_tiles), dim3(512), smem, st, a, scale_log2);
  return hipGetLastError();
}

template <int HD>
hipError_t launch64(const AttnPrefillArgs& a, hipStream_t st) {
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)HD);
  hipLaunchKernelGGL(attn_prefill64_kernel<HD>, dim3(a.n_q_heads, a.n_tiles), dim3(128), 0, st, a, scale_log2);
  return hipGetLastError();
}

hipError_t launch256(const AttnPrefillArgs& a, hipStream_t st) {
  constexpr int smem = 2 * 2 * BKV * 256 * 2;
  // once; the initialisation of a function-local static is thread-safe
  static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_prefill256_kernel),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  if (attr_err != hipSuccess) return attr_err;
  const float scale_log2 = 1.4426950408889634f / 16.f;
  hipLaunchKernelGGL(attn_prefill256_kernel, dim3(a.n_tiles, a.n_q_heads), dim3(256), smem, st, a, scale_log2);
  return hipGetLastError();
}

}  // namespace attn_impl
using namespace attn_impl;

hipError_t launch_attention_prefill(const AttnPrefillArgs& a, hipStream_t st) {
  if (a.n_tiles <= 0) return hipSuccess;
  if ((long long)a.T * a.ld * 2 >= (1LL << 31) || (long long)a.n_kv_heads * a.hd * a.Tp * 2 >= (1LL << 31))
    return hipErrorInvalidValue;
  switch (a.hd) {
    case 64: return a.tile_rows == 64 ? launch64<64>(a, st) : a.tile_rows == 128 ? launch8<64, true>(a, st) : launch8<64, false>(a, st);
    case 128: return a.tile_rows == 64 ? launch64<128>(a, st) : a.tile_rows == 128 ? launch8<128, true>(a, st) : launch8<128, false>(a, st);
    case 256: return launch256(a, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace pop
