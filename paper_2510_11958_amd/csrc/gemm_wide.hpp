// Projection GEMM for many activation rows of a bf16 model on gfx950 (prefill, whole-sequence scoring, batches whose
// steps carry more than 128 rows): y[m, n] = sum_k W[n, k] * x[m, k] with x in two bf16 planes (see gemv_mfma.hpp).
//
// With hundreds of rows the projection is a matrix-core problem, not a weight stream.  A block computes a tile of 128
// rows x 256 weight rows (SwiGLU: 128 gate and the same 128 up rows) with 8 waves of 64 x 64 (2 x 2 tiles of
// v_mfma_f32_32x32x16_bf16, the activations as the A operand, so that a lane's results are 16 rows of one output and a
// store instruction covers 32 neighbouring outputs).  K is walked in steps of 32: weights and both activation planes go
// from memory straight into LDS (global_load ... lds), 32 pieces of 1 KiB per step, each piece holding 16 rows in the
// order [16-byte chunk of k][row], which is the order the weights are stored in; a fragment read then takes 256 contiguous
// bytes per 16 lanes (no bank conflicts).  Two LDS buffers; the next step's loads fly while a step is computed.
// What bounds it: getting the pieces out of L2 in time.  A step is 8 MFMAs of 32 cycles per wave; two blocks fit a CU
// (64 KiB of LDS, 112 registers), so one block's waits are covered by the other's MFMAs.  Measured on a 2048 x 19456 x 2560
// product without epilogue (TFLOP/s counting both planes): 8 waves, 2 buffers, 2 blocks per CU 1108; 4 waves of 64 x 128 with 2
// blocks per CU 900, with 4 buffers and one block 888; 256 x 256 tiles with 3 buffers 984; fragments of the next half step read
// ahead of a step's MFMAs 954 to 1018 (the earlier wait costs more than the read-ahead gains).
// Blocks go round-robin over the 8 compute dies; a die takes a contiguous run of tiles with the row tiles fastest, so a
// weight byte enters one die's L2 only and its row tiles share it there.
// Against passes of 128 rows through gemm_mfma.hpp (4B shapes, 2048 rows, us with the finishing launch, before / now):
// gate/up 660 / 454, QKV 390 / 166, down + O 763 / 345.
#pragma once
#include "gemm_mfma.hpp"

namespace dmtd {

constexpr int GW_BM = 128, GW_BN = 256;      // activation rows, weight rows of a block's tile
constexpr int GW_WAVES = 8;
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Tile index of a block: die x = id % 8 owns tiles [x * q + min(x, rem), ...), q = total / 8.
// Tiles are numbered by groups of 8 row tiles, within a group the row tiles fastest, then the splits of K, then the weight
// tiles: what a die computes at a time is about square.
__device__ __forceinline__ void gw_tile(int id, int total, int mt, int ksplit, int& mb, int& nb, int& ks) {
  const int x = id & 7, j = id >> 3, q = total >> 3, rem = total & 7;
  const int t = x * q + (x < rem ? x : rem) + j;
  const int per_group = 8 * (total / mt), grp = t / per_group, in = t - grp * per_group, rows = min(8, mt - grp * 8);
  mb = grp * 8 + in % rows;
  const int rest = in / rows;
  ks = rest % ksplit;
  nb = rest / ksplit;
}

template <int EPI, bool NORM, bool SPLITK>
__global__ void __launch_bounds__(64 * GW_WAVES, 4) gemm_wide_mfma_kernel(const bf16_t* W_, const bf16_t* W2_, const bf16_t* xb_, const bf16_t* xb_lo_,
                                                                int M_, int N_, int K_, int ldxb_, int ksplit_, int mt_, MfmaArgs a) {
  constexpr int STAGE = 32 * 512;                    // elements of a k-step's slice: 16 weight pieces, 8 high, 8 low activation pieces
  __shared__ __attribute__((aligned(1024))) bf16_t ring[2 * STAGE];
  __shared__ float rs_s[GW_BM];
  __shared__ unsigned long long key_s[EPI == EPI_LOGITS ? GW_BM : 1];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = M_, N = N_, K = K_, KS = K >> 6;
  int mb, nb, ks;
  gw_tile(blockIdx.x, gridDim.x, mt_, SPLITK ? ksplit_ : 1, mb, nb, ks);
  // k-steps of 32 of this block
  const int s_lo = SPLITK ? 2 * (int)((long)ks * KS / ksplit_) : 0;
  const int s_hi = SPLITK ? 2 * (int)((long)(ks + 1) * KS / ksplit_) : 2 * KS;
  const int n_tiles = (N + 15) >> 4;

  // loads: wave w brings weight pieces 2w, 2w + 1 and activation pieces 2w, 2w + 1 of every step; the bases are uniform over
  // the wave, a lane adds its 16 bytes.  Weight rows beyond N repeat the last tile, activation rows beyond M the last row
  // (their results are never stored).
  const bf16_t* wsrc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int p = 2 * w + j;
    int gt = EPI == EPI_SWIGLU ? nb * 8 + (p & 7) : nb * 16 + p;
    if (gt >= n_tiles) gt = n_tiles - 1;
    wsrc[j] = ((EPI == EPI_SWIGLU && p >= 8) ? W2_ : W_) + ((size_t)gt * KS) * 1024 + (size_t)s_lo * 512;
  }
  const bf16_t* xsrc = (w >= 4 ? xb_lo_ : xb_) + (size_t)mb * GW_BM * ldxb_ + (size_t)s_lo * 32;
  int xoff[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int row = ((2 * w + j) & 7) * 16 + (lane & 15);
    xoff[j] = min(row, M - 1 - mb * GW_BM) * ldxb_ + (lane >> 4) * 8;
  }
  auto issue = [&](int buf) {
    bf16_t* dst = ring + buf * STAGE;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(wsrc[j] + lane * 8),
                                       (__attribute__((address_space(3))) void*)(dst + (2 * w + j) * 512), 16, 0, 0);
      wsrc[j] += 512;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(xsrc + xoff[j]),
                                       (__attribute__((address_space(3))) void*)(dst + (16 + 2 * w + j) * 512), 16, 0, 0);
    xsrc += 32;
  };

  const int wm = w & 1, wn = w >> 1;
  // 32-row weight tiles of this wave (SwiGLU: a gate tile and the up tile of the same outputs)
  auto wtile = [&](int j) { return EPI == EPI_SWIGLU ? 4 * j + wn : 2 * wn + j; };
  const int frag = ((lane >> 4) & 1) * 512 + (lane >> 5) * 128 + (lane & 15) * 8;   // this lane's 16 bytes of a 32-row tile, k chunk 0
  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  issue(0);
  for (int s = s_lo; s < s_hi; ++s) {
    const int buf = (s - s_lo) & 1;
    // this step's pieces have landed (nothing newer is in flight), and every wave is done with the other buffer
    __builtin_amdgcn_s_waitcnt(7 << 4);      // vmcnt(0) lgkmcnt(0), expcnt untouched
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (s + 1 < s_hi) issue(buf ^ 1);
    const bf16_t* base = ring + buf * STAGE + frag;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      bf16x8_t xh[2], xl[2], wf[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        xl[i] = __builtin_bit_cast(bf16x8_t, *(const u32x4*)(base + (24 + (2 * wm + i) * 2) * 512 + c * 256));
        xh[i] = __builtin_bit_cast(bf16x8_t, *(const u32x4*)(base + (16 + (2 * wm + i) * 2) * 512 + c * 256));
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) wf[j] = __builtin_bit_cast(bf16x8_t, *(const u32x4*)(base + wtile(j) * 1024 + c * 256));
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xl[i], wf[j], acc[i][j], 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xh[i], wf[j], acc[i][j], 0, 0, 0);
    }
  }

  // lane (column n = lane % 32 of a weight tile): element e of acc[i][j] is row 32 i + 8 (e / 4) + 4 (lane / 32) + e % 4 of the wave
  const int m_w = mb * GW_BM + wm * 64, m_l = 4 * (lane >> 5), col = lane & 31;
  if (SPLITK) {
    float* part = a.part + (size_t)ks * M * a.ldp;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int n = EPI == EPI_SWIGLU ? nb * 128 + wn * 32 + col : nb * GW_BN + wtile(j) * 32 + col;
      const int no = n + ((EPI == EPI_SWIGLU && j == 1) ? N : 0);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int m = m_w + 32 * i + 8 * (e >> 2) + m_l + (e & 3);
          if (m < M && n < N) part[(size_t)m * a.ldp + no] = acc[i][j][e];
        }
    }
    return;
  }
  if (NORM) {
    // the rows' 1/rms: four threads per row sum interleaved partial sums of squares
    const int m = mb * GW_BM + (tid >> 2);
    float ss = 0.f;
    for (int p = tid & 3; p < a.n_parts; p += 4) ss += a.ssp[(size_t)p * a.ssp_ld + min(m, M - 1)];
    ss += __shfl_xor(ss, 1, 64);
    ss += __shfl_xor(ss, 2, 64);
    if ((tid & 3) == 0) rs_s[tid >> 2] = rsqrtf(ss / (float)K + a.eps);
  }
  if (EPI == EPI_LOGITS && tid < GW_BM) key_s[tid] = 0ull;
  __syncthreads();
  const int r_w = wm * 64 + m_l;
  if (EPI == EPI_SWIGLU) {
    const int n = nb * 128 + wn * 32 + col;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int ml = 32 * i + 8 * (e >> 2) + (e & 3);
        const float rs = rs_s[r_w + ml];
        const float gt = acc[i][0][e] * rs, up = acc[i][1][e] * rs;
        bf16_t hi, lo;
        split_bf16(gt / (1.0f + __expf(-gt)) * up, hi, lo);
        // neighbouring lanes pair up: the even lane stores both high parts, the odd lane both low parts (4 bytes each)
        const uint32_t mine = (uint32_t)hi | ((uint32_t)lo << 16);
        const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)mine, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
        const uint32_t pair = (lane & 1) ? (other >> 16) | (mine & 0xFFFF0000u) : (mine & 0xFFFFu) | (other << 16);
        const int m = m_w + m_l + ml;
        if (m < M && n < N) *(uint32_t*)((lane & 1 ? a.yb_lo : a.yb) + (size_t)m * a.ldyb + (n & ~1)) = pair;
      }
    return;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int ml = 32 * i + 8 * (e >> 2) + (e & 3), m = m_w + m_l + ml;
      const float rs = NORM ? rs_s[r_w + ml] : 1.f;
      unsigned long long best = 0ull;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int n = nb * GW_BN + wtile(j) * 32 + col;
        const float v = acc[i][j][e] * rs;
        if (m < M && n < N) {
          a.y[(size_t)m * a.ldy + n] = v;
          if (EPI == EPI_LOGITS) { const unsigned long long k = argmax_key(v, n); if (k > best) best = k; }
        }
      }
      if (EPI == EPI_LOGITS && a.amax && best != 0ull) atomicMax(&key_s[r_w + ml], best);
    }
  if (EPI == EPI_LOGITS && a.amax) {
    __syncthreads();
    if (tid < GW_BM && mb * GW_BM + tid < M) atomicMax(a.amax + (size_t)(nb % AMAX_CELLS) * a.amax_ld + mb * GW_BM + tid, key_s[tid]);
  }
}

}  // namespace dmtd
