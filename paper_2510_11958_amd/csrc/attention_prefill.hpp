// Attention for passes with many rows per sequence (prefill, whole-sequence scoring) over a bf16 KV cache on gfx950.
// The rows' keys and values are in the cache already (kv_append_kernel); the output goes to the O projection as two
// bf16 planes.
//
// A block takes 128 query vectors of one KV head and sequence (128 / GQ rows x the GQ query heads that share the head), 32 per
// wave, and walks the visible keys in tiles of 64: K and V pass through LDS once per block instead of once per 16 query
// vectors.  Launches with at most a block per CU use two groups of 4 waves (KG = 2) that take the even and the odd tiles and
// meet at the end through LDS: the block with the most keys, which such a launch waits for, walks half as many tiles one
// after the other.  With more blocks two of 4 waves share a CU and need no common barrier (32 prompts of 2048: the pass
// 57.6 against 60.7 ms with KG = 2; one prompt of 1003: 2.17 against 2.13).  Per tile and wave, with v_mfma_f32_32x32x16_bf16:
//   scores   S^T[key, q] = sum_d K[key, d] Q[q, d]; K rows from LDS as the A operand, the queries (normalised, rotated, scaled
//            by log2(e) / sqrt(HD), split into bf16 high and low parts, held in registers) as the B operand.  A lane ends up
//            with 16 keys of ONE query per 32-key tile, so the softmax statistics need one exchange with lane ^ 32.
//   output   O^T[d, q] += sum_key V^T[d, key] P^T[key, q]: a lane's own probabilities are the B operand as they stand (the
//            contraction runs over the keys in the order the scores left them), V^T comes from LDS.  A probability goes in as
//            three bf16 parts that add up to all 24 bits of it, so P.V keeps fp32 probabilities at three quarters of
//            the bf16 rate per part instead of the fp32 matrix rate (1/16).
// K goes from the cache straight into LDS (global_load ... lds; rows of HD with their 16-byte chunks permuted by the key
// number), V through registers, transposed on the way (4 keys x HD/16 dims per thread, 8-byte pieces of 4 keys permuted by
// the dim): fragment reads of both spread over all banks.  Two buffers of each; the next tile's loads fly during a tile.
// What bounds it: the matrix cores (40 MFMAs of 32 cycles per 32 keys and wave at HD = 128; they work 70 % of the time behind 6k keys) at
// the clock the card's power leaves them (1.75 to 1.83 GHz there), and the softmax and three-way split, about 0.8 times as many vector cycles.
// So a tile's work is laid out by hand: a K fragment is read a step, a V fragment three products ahead of its use, the next tile's
// loads are issued one beside each step of the scores, and the exponentials and parts of a contraction step stand six vector
// instructions beside each product of the step before.  2048 rows behind 0 / 2k / 4k / 6k keys (the passes of a prompt of 8192), us per
// launch: read and waited for in place 115 / 252 / 392 / 523; in this order 108 / 245 / 378 / 510; the blocks paired long with short
// (launcher) 97 / 231 / 367 / 500; loads' addresses from two registers a tile 93 / 220 / 347 / 475.
// Wave priorities (by block, or raised around the softmax) changed nothing.
// Against the decode kernel (attention_mfma.hpp, one pass over K and V per 16 query vectors, the same products) on the same passes,
// 32/8 heads of 128, us per launch: one prompt of 1003 111 -> 49; 2048 rows against 2k to 8k keys 1044 -> 314 (the prompt of
// 8192, 2 layers: 14.5 -> 8.7 ms); 32 prompts of 2048 in passes of 64 rows 386 -> 95; one prompt of 400 33 -> 28.
// The product runs over a whole tile with probability 0 for the keys a row does not see, and 0 * inf is NaN.  So a block looks at the
// values of its own rows' positions first; if one is not finite, it and its like behind it go into LDS as 0, and the rows at or
// behind the first of them come out as NaN, which their own products would give; the rows before it are as if it were not there.
#pragma once
#include "attention_mfma.hpp"
#include "gemm_wide.hpp"

namespace dmtd {

// dynamic LDS: per group two buffers of K and V tiles
constexpr size_t attn_prefill_lds(int hd, int kg) { return (size_t)kg * 4 * 64 * hd * 2; }
constexpr int AP_QV = 128, AP_KT = 64;       // query vectors of a block, keys of a tile

template <int HD, int KG>
__global__ void __launch_bounds__(256 * KG, HD == 64 && KG == 1 ? 3 : 2) attn_prefill_mfma_kernel(
    const float* __restrict__ qkv, int ldq, const bf16_t* __restrict__ kc, const bf16_t* __restrict__ vc, int nh, int nkv, int s_max,
    int r_total, const DevState* st, int sel, int offset, const bf16_t* __restrict__ q_gain, const float2* __restrict__ rope_tab,
    float eps, bf16_t* __restrict__ out, bf16_t* __restrict__ out_lo, int ldo, int blocked, int n_down) {
  constexpr int T = HD / 16;           // MFMA steps over d for the scores
  constexpr int DT = HD / 32;          // 32-dim tiles of the output
  constexpr int DV = HD / 16;          // dims of V a thread carries
  constexpr int CH = HD / 8;           // 16-byte chunks of a K row
  constexpr int KI = AP_KT * CH / 256; // K pieces (16 bytes per lane) per wave and tile
  typedef unsigned int vraw_t __attribute__((ext_vector_type(DV / 2)));
  constexpr int TILE = AP_KT * HD;     // elements of a K or V tile
  extern __shared__ float4 attn_dyn_smem[];
  __shared__ int poison_s;             // first of the block's own positions, but its first, with a value that is not finite
  const int tid = threadIdx.x, lane = tid & 63;
  const int w8 = __builtin_amdgcn_readfirstlane(tid >> 6), w = w8 & 3, kg = KG == 2 ? w8 >> 2 : 0;      // wave of its group; group (tiles of that parity)
  bf16_t* ring = (bf16_t*)attn_dyn_smem + kg * 4 * TILE;                // the group's buffers: K, K, V^T, V^T
    // the tiles with the most keys start first; behind n_down of them the shortest first (see the launcher)
  const int g = blockIdx.x, b = blockIdx.y, z = blockIdx.z, qt = z < n_down ? (int)gridDim.z - 1 - z : z - n_down;
  const int GQ = nh / nkv, rpb = AP_QV / GQ, row0 = qt * rpb;
  const int rows = min(rpb, r_total - row0);
  const int hi = lane >> 5, qv = 32 * w + (lane & 31);
  const bool valid = qv < rows * GQ;
  const int row = row0 + (valid ? qv / GQ : 0), head = g * GQ + (valid ? qv % GQ : 0);
  const int pos0 = row_base(st, sel, offset, b) + row0;
  const int key_end = pos0 + rows, my_pos = pos0 + (row - row0);
  // a sequence's rows of one head are addressed with 32-bit element offsets (the launcher checks that they fit)
  kc += ((size_t)b * nkv + g) * s_max * HD;
  vc += ((size_t)b * nkv + g) * s_max * HD;

  // Piece i of a wave's share of a K tile holds keys (w KI + i) * 64 / CH + ln / CH, a chunk of one per lane ln, permuted by the key number.
  // The walk hands the lane number in anew for every tile: what follows from it, kept in registers through the loop, would push the kernel
  // beyond the 256 that two blocks per CU allow.
  auto load_k_piece = [&](int ln, int base, int buf, int i) {
    static_assert(64 / CH <= CH, "the permutation of a piece is that of piece 0, exclusive-or its first key");
    const int k0 = ln / CH, c0 = (ln % CH) ^ k0, ki = (w * KI + i) * (64 / CH);
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(kc + (uint32_t)(min(base + ki + k0, key_end - 1) * HD + (c0 ^ (ki & (CH - 1))) * 8)),
                                     (__attribute__((address_space(3))) void*)(ring + buf * TILE + (w * KI + i) * 512), 16, 0, 0);
  };
  auto load_k = [&](int base, int buf) {
#pragma unroll
    for (int i = 0; i < KI; ++i) load_k_piece(lane, base, buf, i);
  };
  // this thread's 4 keys of a tile, its dims, and where its pieces go in a V^T row: 16 keys' groups of 4 in the order 0, 2, 1, 3, so
  // that the two groups a lane of the PV product needs (kg, kg + 2) are one 16-byte slot; slots permuted by the dim
  const int kgp = lane & 15, dg = w * 4 + (lane >> 4), vslot = 2 * (kgp >> 2) + (kgp & 1), vhalf = ((kgp >> 1) & 1) * 4;
  vraw_t vr[4];
  auto load_v_piece = [&](int ln, int base, int m) {
    vr[m] = *(const vraw_t*)(vc + (uint32_t)(min(base + 4 * (ln & 15) + m, key_end - 1) * HD + (w * 4 + (ln >> 4)) * DV));
  };
  auto load_v = [&](int base) {
#pragma unroll
    for (int m = 0; m < 4; ++m) load_v_piece(lane, base, m);
  };
  auto drop_bad = [&](int base) {       // values from poison_s on that are not finite become 0
#pragma unroll
    for (int m = 0; m < 4; ++m)
      if (min(base + 4 * kgp + m, key_end - 1) >= poison_s) {
#pragma unroll
        for (int u = 0; u < DV / 2; ++u)
          vr[m][u] = ((vr[m][u] & 0x7F80u) == 0x7F80u ? 0u : vr[m][u] & 0xFFFFu) | ((vr[m][u] & 0x7F800000u) == 0x7F800000u ? 0u : vr[m][u] & 0xFFFF0000u);
      }
  };
  auto store_v_piece = [&](int buf, int u) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int d = dg * DV + 2 * u + h;
      const unsigned int s = h ? 0x07060302u : 0x05040100u;
      *(uint2*)(ring + (2 + buf) * TILE + d * AP_KT + ((vslot ^ ((d >> 1) & 7)) * 8 + vhalf)) =
          make_uint2(__builtin_amdgcn_perm(vr[1][u], vr[0][u], s), __builtin_amdgcn_perm(vr[3][u], vr[2][u], s));
    }
  };
  auto store_v = [&](int buf) {
#pragma unroll
    for (int u = 0; u < DV / 2; ++u) store_v_piece(buf, u);
  };
  const int n_tiles = (key_end + AP_KT - 1) / AP_KT;
  if (kg < n_tiles) { load_k(kg * AP_KT, 0); load_v(kg * AP_KT); }
  if (tid == 0) poison_s = 0x7FFFFFFF;
  // values of the keys that some row does not see, 16 bytes each: is one of them not finite?
  constexpr int NT = 256 * KG, SC = 2;
  const int n_scan = (rows - 1) * CH;
  auto scan_key = [&](int c) { return min(pos0 + 1 + c / CH, key_end - 1); };
  auto scan_load = [&](int c) { return *(const u32x4*)(vc + (uint32_t)(scan_key(c) * HD + c % CH * 8)); };
  auto scan_check = [&](const u32x4& v, int c) {
    bool bad = false;
#pragma unroll
    for (int u = 0; u < 4; ++u) bad |= (v[u] & 0x7F80u) == 0x7F80u || (v[u] & 0x7F800000u) == 0x7F800000u;
    if (bad) atomicMin(&poison_s, scan_key(c));
  };
  u32x4 sc[SC];
#pragma unroll
  for (int j = 0; j < SC; ++j) sc[j] = scan_load(tid + j * NT);

  // the lane's query vector: dims 16 t + 8 hi + 0..7; its rotary partner dims (i, i + HD/2) are the lane's own
  bf16x8_t qh[T], ql[T];
  {
    float x[T][8];
    const float* src = qkv + (size_t)(b * r_total + row) * ldq + (size_t)head * HD + 8 * hi;
    float ss = 0.f;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const f32x4 a = *(const f32x4*)(src + 16 * t), c = *(const f32x4*)(src + 16 * t + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) { x[t][e] = a[e]; x[t][4 + e] = c[e]; }
    }
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int e = 0; e < 8; ++e) ss += x[t][e] * x[t][e];
    ss = pair_sum<32>(ss);
    const float rs = rsqrtf(ss / (float)HD + eps);
    const float scale = rsqrtf((float)HD) * 1.4426950408889634f;
    const float2* rp = rope_tab + (size_t)my_pos * (HD / 2) + 8 * hi;
#pragma unroll
    for (int t = 0; t < T / 2; ++t) {
      float g0[8], g1[8];
      Elem<bf16_t>::unpack(*(const u32x4*)(q_gain + 16 * t + 8 * hi), g0);
      Elem<bf16_t>::unpack(*(const u32x4*)(q_gain + HD / 2 + 16 * t + 8 * hi), g1);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float2 cs = rp[16 * t + e];
        const float a0 = x[t][e] * (rs * g0[e]), a1 = x[t + T / 2][e] * (rs * g1[e]);
        x[t][e] = (a0 * cs.x - a1 * cs.y) * scale;
        x[t + T / 2][e] = (a1 * cs.x + a0 * cs.y) * scale;
      }
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
      uint32_t h4[4], l4[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        h4[e] = pack_bf16x2(x[t][2 * e], x[t][2 * e + 1]);
        l4[e] = pack_bf16x2(x[t][2 * e] - __uint_as_float(h4[e] << 16), x[t][2 * e + 1] - __uint_as_float(h4[e] & 0xFFFF0000u));
      }
      qh[t] = __builtin_bit_cast(bf16x8_t, u32x4{h4[0], h4[1], h4[2], h4[3]});
      ql[t] = __builtin_bit_cast(bf16x8_t, u32x4{l4[0], l4[1], l4[2], l4[3]});
    }
  }
  float m_run = -INFINITY, l_run = 0.f;
  f32x16 acc[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
  __builtin_amdgcn_s_waitcnt(0xC07F);      // lgkmcnt(0): poison_s is set before a wave adds to it; the loads stay in flight
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int j = 0; j < SC; ++j) scan_check(sc[j], tid + j * NT);
  for (int c = tid + SC * NT; c < n_scan; c += NT) scan_check(scan_load(c), c);
  if (kg < n_tiles) store_v(0);
  __builtin_amdgcn_s_waitcnt(7 << 4);      // vmcnt(0) lgkmcnt(0): this wave's share of K has landed too
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");

  // One tile's work; MORE: with the next one's loads beside it (beyond the last: its last key again, never used).  Waves whose group has one tile in
  // all do without (us per launch, with / without: 32/8 heads of 128, 40 prompts of 30 22.6 / 20.2, 48 of 50 31.4 / 30.5, 3 of 90 17.7 / 17.0; 14/2 heads
  // of 64, 48 of 50 11.2 / 10.8).
  auto tile = [&](int it, auto drop_c, auto more_c) {
    constexpr bool DROP = decltype(drop_c)::value, MORE = decltype(more_c)::value;
    const int buf = it & 1, base = (KG * it + kg) * AP_KT, ahead = base + KG * AP_KT;
    // Fragment offsets: chunk 2 t + hi of a K row and slot 2 q + hi of a V^T row, permuted, differ from chunk and slot hi by an exclusive or
    int ko = (lane & 31) * HD + ((hi ^ (lane & (CH - 1))) << 3), vo = (lane & 31) * AP_KT + ((hi ^ ((lane >> 1) & 7)) << 3);
    int ln = lane;
    asm volatile("" : "+v"(ko), "+v"(vo), "+v"(ln));
    const bf16_t* kb = ring + buf * TILE;
    const bf16_t* vb = ring + (2 + buf) * TILE;
    auto read_k = [&](int k, int t) { return __builtin_bit_cast(bf16x8_t, *(const u32x4*)(kb + (ko ^ (t << 4)) + k * 32 * HD)); };
    auto read_v = [&](int q, int t) { return __builtin_bit_cast(bf16x8_t, *(const u32x4*)(vb + (vo ^ (q << 4)) + t * 32 * AP_KT)); };
    // scores (in units of log2) of keys base + 32 k + 8 (e / 4) + 4 hi + e % 4 for the lane's query
    f32x16 s[2];
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int e = 0; e < 16; ++e) s[k][e] = 0.f;
    bf16x8_t kf[2][2];
    kf[0][0] = read_k(0, 0);
    kf[0][1] = read_k(1, 0);
    constexpr int LD = MORE ? KI + 4 : 0;          // loads of the next tile, shared out over the steps
#pragma unroll
    for (int t = 0; t < T; ++t) {
      if (t + 1 < T) {
        kf[(t + 1) & 1][0] = read_k(0, t + 1);
        kf[(t + 1) & 1][1] = read_k(1, t + 1);
      }
      s[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t & 1][0], ql[t], s[0], 0, 0, 0);
      s[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t & 1][1], ql[t], s[1], 0, 0, 0);
#pragma unroll
      for (int z = t * LD / T; z < (t + 1) * LD / T; ++z) {
        if (z < KI) load_k_piece(ln, ahead, buf ^ 1, z);
        else load_v_piece(ln, ahead, z - KI);
      }
      s[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t & 1][0], qh[t], s[0], 0, 0, 0);
      s[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t & 1][1], qh[t], s[1], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    bf16x8_t vf[2];
    vf[0] = read_v(0, 0);
    if (base + AP_KT > pos0 + 1) {      // keys beyond some row's position in this tile
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (base + 32 * k + 8 * (e >> 2) + 4 * hi + (e & 3) > my_pos) s[k][e] = -INFINITY;
    }
    float mx = s[0][0];
#pragma unroll
    for (int e = 1; e < 16; ++e) mx = fmaxf(mx, s[0][e]);
#pragma unroll
    for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[1][e]);
    mx = pair_max<32>(mx);
    // (A reference that follows only growth beyond 2^8 leaves most tiles' sums alone, 2 % of a launch, but then values beyond 2^120 overflow
    // them: a probability may be 2^8.)
    const float m_new = fmaxf(m_run, mx);       // -inf: the odd tiles so far hold no key this row sees
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    if (__any(m_new > m_run)) {
      const float f = __builtin_amdgcn_exp2f(m_run - m_use);
      l_run *= f;
#pragma unroll
      for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] *= f;
      m_run = m_new;
    }
    // The 8 probabilities of a contraction step q as three bf16 parts (truncated leading 8 bits, the next 8, the rest: exact), pair j of them
    // in three pieces of about six vector instructions
    uint32_t pp[2][3][4];
    float r0[4], r1[4];
    auto piece = [&](int q, int j, int z) {
      const int e = 8 * (q & 1) + 2 * j;
      const float a = s[q >> 1][e], d = s[q >> 1][e + 1];
      if (z == 0) {
        s[q >> 1][e] = __builtin_amdgcn_exp2f(a - m_use);
        s[q >> 1][e + 1] = __builtin_amdgcn_exp2f(d - m_use);
      } else if (z == 1) {
        l_run += a;
        l_run += d;
        pp[q & 1][0][j] = __builtin_amdgcn_perm(__float_as_uint(d), __float_as_uint(a), 0x07060302u);
        r0[j] = a - __uint_as_float(__float_as_uint(a) & 0xFFFF0000u);
        r1[j] = d - __uint_as_float(__float_as_uint(d) & 0xFFFF0000u);
      } else {
        pp[q & 1][1][j] = __builtin_amdgcn_perm(__float_as_uint(r1[j]), __float_as_uint(r0[j]), 0x07060302u);
        const float a2 = r0[j] - __uint_as_float(__float_as_uint(r0[j]) & 0xFFFF0000u), d2 = r1[j] - __uint_as_float(__float_as_uint(r1[j]) & 0xFFFF0000u);
        pp[q & 1][2][j] = __builtin_amdgcn_perm(__float_as_uint(d2), __float_as_uint(a2), 0x07060302u);
      }
    };
    constexpr int PG = 4 / DT;          // pairs of the next step beside a V fragment's three products
#pragma unroll
    for (int z = 0; z < 3; ++z)
#pragma unroll
      for (int j = 0; j < 4; ++j) piece(0, j, z);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
      for (int t = 0; t < DT; ++t) {
        const int n = q * DT + t;
        if (n + 1 < 4 * DT) vf[(n + 1) & 1] = read_v((n + 1) / DT, (n + 1) % DT);
#pragma unroll
        for (int z = 0; z < 3; ++z) {
          const uint32_t* f = pp[q & 1][2 - z];
          acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[n & 1], __builtin_bit_cast(bf16x8_t, u32x4{f[0], f[1], f[2], f[3]}), acc[t], 0, 0, 0);
          if (q < 3) {
#pragma unroll
            for (int j = 0; j < PG; ++j) piece(q + 1, t * PG + j, z);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    if (MORE) {
      if (DROP) drop_bad(ahead);
      store_v(buf ^ 1);
    }
  };
  auto walk = [&](auto drop_c) {
    for (int it = 0; KG * it < n_tiles; ++it) {
      if (KG * it + kg < n_tiles) tile(it, drop_c, std::integral_constant<bool, true>());      // uniform over the wave; every wave meets the barrier
      __builtin_amdgcn_s_waitcnt(7 << 4);
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    }
  };
  if (n_tiles <= KG && __builtin_amdgcn_readfirstlane(poison_s) == 0x7FFFFFFF) {
    if (kg < n_tiles) tile(0, std::integral_constant<bool, false>(), std::integral_constant<bool, false>());
    if (KG == 2) __syncthreads();
  } else if (__builtin_amdgcn_readfirstlane(poison_s) == 0x7FFFFFFF) {
    walk(std::integral_constant<bool, false>());
  } else {                            // seldom; the first tile's values once more
    if (kg < n_tiles) { load_v(kg * AP_KT); drop_bad(kg * AP_KT); store_v(0); }
    __builtin_amdgcn_s_waitcnt(7 << 4);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    walk(std::integral_constant<bool, true>());
  }
  l_run = pair_sum<32>(l_run);
  if constexpr (KG == 2) {
  // the odd tiles' results go through LDS (the ring is free: every wave is past the last tile's barrier) to the even tiles' waves
  float* mine = (float*)attn_dyn_smem + (size_t)w * (DT * 16 + 2) * 64 + lane;
  if (kg == 1) {
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) mine[(t * 16 + e) * 64] = acc[t][e];
    mine[DT * 16 * 64] = m_run;
    mine[(DT * 16 + 1) * 64] = l_run;
  }
  __syncthreads();
  if (kg == 1) return;
  {
    const float m1 = mine[DT * 16 * 64], mm = fmaxf(m_run, m1);      // m_run is finite: the first tile holds key 0, which every row sees
    const float f0 = __builtin_amdgcn_exp2f(m_run - mm), f1 = __builtin_amdgcn_exp2f(m1 - mm);
    l_run = l_run * f0 + mine[(DT * 16 + 1) * 64] * f1;
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[t][e] = acc[t][e] * f0 + mine[(t * 16 + e) * 64] * f1;
  }
  }
  // where the vector goes, likewise
  int ln = lane;
  asm volatile("" : "+v"(ln));
  const int qo = 32 * w + (ln & 31), ro = qo / GQ;
  if (qo >= rows * GQ) return;
  const float inv_l = my_pos >= poison_s ? __uint_as_float(0x7FC00000u) : 1.0f / l_run;
  const size_t at0 = packed_at(blocked, b * r_total + row0 + ro, (g * GQ + qo - ro * GQ) * HD + 4 * (ln >> 5), ldo);
  const int t_step = blocked ? 512 : 32, q_step = blocked ? 128 : 8;        // 32 and 8 dims further
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      bf16_t h4[4], l4[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) split_bf16(acc[t][4 * q + e] * inv_l, h4[e], l4[e]);
      const size_t at = at0 + t * t_step + q * q_step;
      *(uint2*)(out + at) = make_uint2(h4[0] | ((uint32_t)h4[1] << 16), h4[2] | ((uint32_t)h4[3] << 16));
      *(uint2*)(out_lo + at) = make_uint2(l4[0] | ((uint32_t)l4[1] << 16), l4[2] | ((uint32_t)l4[3] << 16));
    }
}

}  // namespace dmtd
