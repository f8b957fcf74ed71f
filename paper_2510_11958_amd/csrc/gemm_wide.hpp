// Projection GEMM for many activation rows of a bf16 model on gfx950 (prefill, whole-sequence scoring, batches whose
// steps carry more than 192 rows): y[m, n] = sum_k W[n, k] * x[m, k] with x in two bf16 planes (see gemv_mfma.hpp).
//
// With hundreds of rows the projection is a matrix-core problem, not a weight stream.  A block computes a tile of 256
// rows x 256 weight rows (SwiGLU: 128 gate and the same 128 up rows, 16 of each in turn) with 8 waves of 64 x 128 (2 x 4 tiles of
// v_mfma_f32_32x32x16_bf16).  Gate/up and QKV also come with 192 weight rows, where these leave fewer CUs idle
// (choose_wide).  Tiles of 320 weight rows, all that the registers (240 of 256) and LDS hold, would take gate/up of 1003 rows of 2560 in one round of whole
// tiles (us with the finishing launch 184 -> 159, 2048 rows 337 -> 308); they are not here, since they sum in one chain what 256 sum in five parts
// (below).  K is walked in steps of 32: weights and both activation planes go from memory straight into
// LDS (global_load ... lds), 48 pieces of 1 KiB per step, each piece holding 16 rows in the order [16-byte chunk of k][row],
// which is the order the weights and the blocked activations (packed_at) are stored in; a fragment read then takes 256
// contiguous bytes per 16 lanes (no bank conflicts).  A ring of three LDS buffers (144 KiB, one block per CU); a step is waited for by the
// exact count of its loads.  The block's barrier stands in the middle of a step, where the fragments of its second half are in registers
// and the next step's first ones are read beside the products (see the loop).
// What bounds it: the card's power in part.  Gate/up at 2048 rows (608 tiles, 19456 x 2560, cold weights, without the finishing launch), us, barrier in front
// of a step with all its reads and loads behind it / barrier in the middle: on zeros 263 / 233, on normally distributed data 333 / 314, where
// the clock falls to 1.9 GHz; one 2560 x 9728 launch in 240 blocks 160 / 154; tiles of 128 rows, 1003 rows of 2560 x 4096 41.3 / 40.2.  With the
// same tile loaded by every block the launch takes 302, so memory is not it.  But at that clock a loop of nothing but MFMAs on random
// operands does 1.7 PFLOP/s, and a launch 1.1 to 1.3 with its matrix cores idle for 16 % (down) or 20 % (gate/up) to 37 % (QKV) of a busy CU's time: a step's barrier and reads, a
// block's start and end, and rounds that are not full (a round of split tails behind a full one).  Of a launch's end the stores are the most: 50
// MB of QKV sums or 63 MB of raw ones take 10 to 12 us with the matrix cores idle.  Reads two at a time behind their pairs of products, without a branch each (2048 rows of 2560, us
// before / now): gate/up in tiles of 320 weight rows 301 / 294, down 158 / 154; QKV in tiles of 256 x 192 with its loop laid out likewise 121 / 116
// (without any loads 100, the same tile for every block 114, chains of both row tiles in turn 116).  Also measured at the middle barrier, no faster: other orders of
// the products (each weight tile or each row tile held over 4 of them) 312 to 316, raised wave priority 320, 4 waves of 128 x 128 (a quarter
// less LDS traffic) 5 % slower, tiles of 128 rows in 4 waves of 64 x 128 6 % slower.
// Blocks go round-robin over the 8 compute dies; a die takes a contiguous run of tiles with the row tiles fastest, so a
// weight byte enters one die's L2 only and its row tiles share it there.
// A block costs 10 to 13 us beside its steps; of the SwiGLU epilogue's 6, its divisions are 2 to 4 (tiles of 320 weight rows, us, v_rcp_f32 in their
// place / divisions: 1003 rows of 2560 149 / 152, 2048 rows 287 / 291).  Without loads, reads and barriers in the loop the products alone take 140
// of these 152, on zeros 113.
// Tiles of 128 rows (waves of 64 x 64, a ring of four buffers, 0.8 instead of 1.3 us per step) where they pad a launch's rows less.
// Against passes of 128 rows through gemm_mfma.hpp (4B shapes, 2048 rows, us with the finishing launch, before / now; the card of the 2nd figures is
// one of those that run 5 to 8 % slower than that of the others above): gate/up 660 / 337, QKV 390 / 129, down + O 763 / 283.
// Sums: a tile that takes its whole K in one block sums it in one fp32 chain, a rounding per 8 products, 4.4e-7 of the result's norm at
// K = 2560 in two planes; five parts summed apart (gemm_mfma.hpp with 128 rows) leave 2.0e-7.  In the QKV projection, whose K and V are
// then rounded to bf16, that decides roundings; there a chain has 4 k-steps (tiles of 128 rows) or one (256 rows, 128 additions beside
// 32 MFMAs), about 1.3e-7 (low and high parts alternate by half steps: 2 % more than with a step's low parts first).  Logits of a prompt of 1003, 2560 wide, against 64 bits with the cache's rounding taken
// along, 1 / 2 layers: one chain 8.5e-5 / 1.14e-4, short chains 5.1e-5 / 7.2e-5, 128-row parts 5.2e-5 / 7.5e-5.  QKV, us, one chain /
// short ones: 2048 rows of 2560 118 / 123, 1003 rows 61 / 65, 2048 rows of 1024 34.4 / 35.8 (chains of 8 steps are no nearer than parts at K = 1024).
// Chains of a step in all projections cost 9 to 10 % of a pass at 2560 wide, for no smaller an error.
#pragma once
#include "gemm_mfma.hpp"

namespace dmtd {

constexpr int GW_BN = 256;                   // weight rows of a block's tile (SwiGLU: gate and up rows together), unless the plan takes another width
constexpr int GW_WAVES = 8;
// The tile's shape by its activation rows BM and weight rows BN: waves along the rows and the weight rows, tiles of 32 rows (RT) and of 32
// weight rows (NJ) per wave, LDS buffers, 1 KiB pieces of a step (BN / 16 of weights, BM / 16 per activation plane), loads a wave issues
// per step (waves below HEAVY; the others one less).
template <int BM, int BN> struct GwTile {
  static constexpr int WM = BM == 256 || BN % 256 != 0 ? 4 : 2, WN = GW_WAVES / WM, RT = BM / 32 / WM, NJ = BN / 32 / WN, BUF = BM == 256 ? 3 : 4;
  static constexpr int WP = BN / 16, XT = BM / 16, PIECES = WP + 2 * XT, STAGE = PIECES * 512, LPS = (PIECES + GW_WAVES - 1) / GW_WAVES;
  static constexpr int HEAVY = PIECES - (LPS - 1) * GW_WAVES;
  static constexpr size_t LDS = (size_t)BUF * STAGE * 2;
  static constexpr int PART = BM * BN;       // floats of a tile's raw sums
  static_assert(WM * RT * 32 == BM && WN * NJ * 32 == BN, "a tile is whole waves");
  static_assert(LDS + 2048 <= 160 * 1024, "a CU's LDS");
};
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Which tile a block computes, and which part of K.  The launch has n_full blocks with a tile each and, behind them, ksplit blocks
// for each of the other n_tail tiles.  Either segment goes round-robin over the dies: die x = id % 8 owns the contiguous run
// [x * q + min(x, rem), ...) of it, q = size / 8.  Tiles are numbered by groups of 8 row tiles, within a group the row tiles
// fastest: what a die computes at a time is about square.
struct GwPlace { int t, mb, nb, ks; bool tail; };
__device__ __forceinline__ GwPlace gw_place(int id, int blocks, int n_full, int n_tail, int mt, int nt) {
  GwPlace p;
  p.tail = id >= n_full;
  if (p.tail) { id -= n_full; blocks -= n_full; } else blocks = n_full;
  const int x = id & 7, q = blocks >> 3, rem = blocks & 7;
  const int i = x * q + (x < rem ? x : rem) + (id >> 3);
  p.ks = p.tail ? i / n_tail : 0;
  p.t = p.tail ? n_full + i - p.ks * n_tail : i;
  const int per_group = 8 * nt, grp = p.t / per_group, in = p.t - grp * per_group, rows = min(8, mt - grp * 8);
  p.nb = in / rows;
  p.mb = grp * 8 + in - p.nb * rows;
  return p;
}

template <int EPI, bool NORM, int BM, int BN>
__global__ void __launch_bounds__(64 * GW_WAVES, 2) gemm_wide_mfma_kernel(const bf16_t* W_, const bf16_t* W2_, const bf16_t* xb_, const bf16_t* xb_lo_,
                                                                int M_, int N_, int K_, int n_full_, int n_tail_, int ksplit_, int mt_, int nt_, MfmaArgs a) {
  // which operand gives the result's rows: with the weights there a lane holds 4 consecutive outputs of one activation row (8-byte
  // pieces of the blocked layout, 512 contiguous bytes per two row groups and store), else 16 rows of one output (128 bytes of a row)
  constexpr bool WA = EPI == EPI_SWIGLU || EPI == EPI_NLL;
  typedef GwTile<BM, BN> T;
  constexpr int NJ = T::NJ, RT = T::RT;
  extern __shared__ float4 gemm_dyn_smem[];
  bf16_t* ring = (bf16_t*)gemm_dyn_smem;
  __shared__ float rs_s[BM];
  __shared__ unsigned long long key_s[EPI == EPI_LOGITS ? BM : 1];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = M_, N = N_, K = K_, KS = K >> 6;
  const GwPlace pl = gw_place(blockIdx.x, gridDim.x, n_full_, n_tail_, mt_, nt_);
  const int mb = pl.mb, nb = pl.nb;
  // k-steps of 32 of this block
  const int s_lo = pl.tail ? 2 * (int)((long)pl.ks * KS / ksplit_) : 0;
  const int s_hi = pl.tail ? 2 * (int)((long)(pl.ks + 1) * KS / ksplit_) : 2 * KS;
  const int n_tiles = (N + 15) >> 4;

  // loads: wave w brings pieces w, w + 8, ... of every step, which are the weights' (SwiGLU: 16 gate rows and the up rows of the same outputs
  // in turn), the high plane's and the low plane's; the bases are uniform over the wave, a lane adds its 16 bytes.  Weight tiles beyond
  // N and activation tiles beyond M repeat the last one, and the last activation tile's rows beyond M hold whatever the buffer
  // held: each is an output row of its own that is never stored.
  const int m_tiles = (M + 15) >> 4;
  const bf16_t* src[T::LPS];
  int slot[T::LPS];                            // the piece's place in a buffer
#pragma unroll
  for (int j = 0; j < T::LPS; ++j) {
    const int p = min(w + GW_WAVES * j, T::PIECES - 1), q = p - T::WP;
    const bool up = EPI == EPI_SWIGLU && p >= T::WP / 2;
    const int gt = min(EPI == EPI_SWIGLU ? nb * (BN / 32) + p - (up ? T::WP / 2 : 0) : nb * T::WP + p, n_tiles - 1);
    const bf16_t* base = p < T::WP ? (up ? W2_ : W_) : (q >= T::XT ? xb_lo_ : xb_);
    const int tile = p < T::WP ? gt : min(mb * T::XT + (q >= T::XT ? q - T::XT : q), m_tiles - 1);
    src[j] = base + (size_t)tile * KS * 1024 + (size_t)s_lo * 512;
    slot[j] = EPI == EPI_SWIGLU && p < T::WP ? (up ? 2 * p - T::WP + 1 : 2 * p) : w + GW_WAVES * j;
  }
  auto issue_one = [&](int buf, int j) {       // load j of a step into ring buffer buf
    if (j == T::LPS - 1 && T::HEAVY < GW_WAVES && w >= T::HEAVY) return;
    bf16_t* dst = ring + buf * T::STAGE + slot[j] * 512;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[j] + lane * 8), (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
    src[j] += 512;
  };
  auto issue = [&](int buf) {
#pragma unroll
    for (int j = 0; j < T::LPS; ++j) issue_one(buf, j);
  };
  const int wm = w % T::WM, wn = w / T::WM;
  auto wtile = [&](int j) { return NJ * wn + j; };     // 32-row weight tiles of this wave (SwiGLU: 16 gate rows, then the up rows of the same outputs)
  const int frag = ((lane >> 4) & 1) * 512 + (lane >> 5) * 128 + (lane & 15) * 8;   // this lane's 16 bytes of a 32-row tile, k chunk 0
  f32x16 acc[RT][NJ];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

#pragma unroll
  for (int s = 0; s < T::BUF - 1; ++s)
    if (s_lo + s < s_hi) issue(s);
  if (NORM && !pl.tail) {
    // the rows' 1/rms while the first steps' pieces are on their way: two or four threads per row, eight parts each at a time
    constexpr int TR = 64 * GW_WAVES / BM;
    const int m = min(mb * BM + tid / TR, M - 1);
    float ss = 0.f;
    for (int p0 = tid % TR; p0 < a.n_parts; p0 += 8 * TR) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = a.ssp[(size_t)min(p0 + TR * u, a.n_parts - 1) * a.ssp_ld + m];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (p0 + TR * u < a.n_parts) ss += v[u];
    }
    ss += lane_dpp<kDppQuad1>(ss);
    if (TR == 4) ss += lane_dpp<kDppQuad2>(ss);
    if (tid % TR == 0) rs_s[tid / TR] = rsqrtf(ss / (float)K + a.eps);
  }
  // Results that are rounded to 16 bits afterwards (QKV: the cache) are summed in short chains of their own, added to the accumulators
  // once each: 4 k-steps where the wave has registers for a second set (tiles of 128 rows), one step else
  constexpr bool SHORT_SUMS = EPI == EPI_STORE;
  auto chunk = [](const bf16_t* q) { return __builtin_bit_cast(bf16x8_t, *(const u32x4*)q); };
  auto mma = [](bf16x8_t wv, bf16x8_t xv, const f32x16& c) {
    return WA ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv, xv, c, 0, 0, 0) : __builtin_amdgcn_mfma_f32_32x32x16_bf16(xv, wv, c, 0, 0, 0);
  };
  // fragments of half a step (16 of k), in order of first use: low parts of the two row tiles, weight tiles, high parts
  constexpr int NF = 2 * RT + NJ;
  struct Frag { bf16x8_t f[NF]; };
  auto read_one = [&](Frag& f, const bf16_t* base, int c, int q) {
    const int piece = q < RT ? T::WP + T::XT + (RT * wm + q) * 2 : (q < RT + NJ ? 2 * wtile(q - RT) : T::WP + (RT * wm + q - RT - NJ) * 2);
    f.f[q] = chunk(base + piece * 512 + c * 256);
  };
  constexpr bool KEEP = SHORT_SUMS && BM == 128;      // a second set of accumulators
  f32x16 part[KEEP ? RT : 1][KEEP ? NJ : 1];
  auto clear = [&](f32x16& c) {
#pragma unroll
    for (int e = 0; e < 16; ++e) c[e] = 0.f;
  };
  if (KEEP)
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) clear(part[i][KEEP ? j : 0]);
  // the loads of a step have returned once all but those of `newer` newer steps have (they return in order); none newer for certain: all
  // vmcnt(loads) lgkmcnt(0), expcnt untouched
  auto wait_but = [&](auto newer_c) {
    constexpr int newer = decltype(newer_c)::value;
    static_assert(newer * T::LPS < 16, "the counter wait's low field");
    if (newer == 0 || T::HEAVY == GW_WAVES || w < T::HEAVY) __builtin_amdgcn_s_waitcnt(newer * T::LPS | (7 << 4));
    else __builtin_amdgcn_s_waitcnt(newer * (T::LPS - 1) | (7 << 4));
  };
  const auto wait_all = std::integral_constant<int, 0>();
  if constexpr (SHORT_SUMS && !KEEP) {
    // A step's weight tiles one after the other, its activation fragments in registers all the while.  A tile's eight products are two chains, one per
    // row tile, and a chain is added to the accumulators beside the next one's products, three products after its end.  The barrier
    // stands in front of the last tile, whose weights are in registers: behind it each fragment's last product is followed by
    // the read of the next step's, and this step's buffer is refilled.
    static_assert(RT == 2, "two row tiles");
    constexpr int NW = NJ % 2 ? 3 : 2;       // weight fragments' places: a tile's are free when the tile NW further is read
    bf16x8_t xf[2][2][2], wf[NW][2];         // [low, high part][half of the step][row tile]; [place][half]
    f32x16 sum[2];
    clear(sum[0]); clear(sum[1]);
    float total[2][NJ][16];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) total[0][j][e] = total[1][j][e] = 0.f;
    auto read_x = [&](const bf16_t* base, int p, int c, int i) { xf[p][c][i] = chunk(base + (T::WP + (1 - p) * T::XT + (2 * wm + i) * 2) * 512 + c * 256); };
    auto read_w = [&](const bf16_t* base, int j, int c) { wf[j % NW][c] = chunk(base + wtile(j) * 1024 + c * 256); };
    if (s_hi - s_lo >= T::BUF - 1) wait_but(std::integral_constant<int, T::BUF - 2>());
    else wait_but(wait_all);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");           // no LDS read of a slice moves above the barrier
#pragma unroll
    for (int u = 0; u < 8; ++u) read_x(ring + frag, (u >> 1) & 1, u & 1, u >> 2);
    read_w(ring + frag, 0, 0);
    read_w(ring + frag, 0, 1);
    if (s_hi - s_lo > T::BUF - 1) issue(T::BUF - 1);
    int buf = 0;
    for (int s = s_lo; s < s_hi; ++s) {
      const int nxt = buf + 1 == T::BUF ? 0 : buf + 1;
      const bf16_t* base = ring + buf * T::STAGE + frag;
      const bf16_t* next = ring + nxt * T::STAGE + frag;
      const bool fill = s + T::BUF < s_hi;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const bool last = j + 1 == NJ;
        if (last) {
          if (s + T::BUF - 1 < s_hi) wait_but(std::integral_constant<int, T::BUF - 2>());
          else wait_but(wait_all);
          __builtin_amdgcn_s_barrier();
          asm volatile("" ::: "memory");
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int i = u >> 2, p = (u >> 1) & 1, c = u & 1;      // low parts first
          f32x16 from = sum[i];
          if ((u & 3) == 0) clear(from);
          sum[i] = mma(wf[j % NW][c], xf[p][c][i], from);
          __builtin_amdgcn_sched_barrier(0);
          if (!last) {
            if (u < 2) read_w(base, j + 1, u);
          } else {
            read_x(next, p, c, i);           // behind the last step nobody uses what is read
            if (u >= 6) read_w(next, 0, u - 6);
            if (fill && u < T::LPS) issue_one(buf, u);
          }
          const int pi = i ^ 1, pj = i ? j : (j + NJ - 1) % NJ;      // the chain before
          if ((u & 3) > 1) {                 // (pinned: the compiler would gather the additions of a step behind a branch)
            float* t = &total[pi][pj][((u & 3) - 2) * 8];
#pragma unroll
            for (int e = 0; e < 8; ++e) t[e] += sum[pi][((u & 3) - 2) * 8 + e];
            asm volatile("" : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]), "+v"(t[4]), "+v"(t[5]), "+v"(t[6]), "+v"(t[7]));
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      buf = nxt;
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        acc[0][j][e] = total[0][j][e];
        acc[1][j][e] = total[1][j][e] + (j == NJ - 1 ? sum[1][e] : 0.f);
      }
  } else {
    // A step's two halves: while the products of one run, the fragments of the next are read.  Reads and loads stand behind a pair of products, not in
    // front: the compiler waits for all reads at a product that needs one, also for those it has just issued.  The
    // barrier stands between the halves.  Behind it the second half's fragments are in registers, so the matrix cores go on at
    // once; every wave is done reading this step's buffer, so it is refilled (a load beside every pair of products: together they would
    // hold the wave up, the memory pipe takes a load per 16 cycles of a CU); and the next step has landed for every wave.
    // BUF - 2 newer steps are on their way (at the end fewer, then all loads are waited for).
    const auto newer = std::integral_constant<int, T::BUF - 2>();
    auto half = [&](const Frag& f, auto beside) {
#pragma unroll
      for (int q = 0; q < 2 * NJ; ++q) {
        const int p = q / NJ, j = q % NJ;    // low parts first
#pragma unroll
        for (int i = 0; i < RT; ++i) {
          f32x16& c = KEEP ? part[KEEP ? i : 0][KEEP ? j : 0] : acc[i][j];
          c = mma(f.f[RT + j], f.f[p ? RT + NJ + i : i], c);
        }
        __builtin_amdgcn_sched_barrier(0);
        beside(q);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // the reads of the next fragments behind products pair q, two at a time, so that the last is back well before it is needed; the
    // loads of a step, one behind each pair
    auto reads = [&](Frag& f, const bf16_t* base, int c, int q) {
#pragma unroll
      for (int z = 2 * q; z < (q == 2 * NJ - 1 ? NF : min(2 * q + 2, NF)); ++z) read_one(f, base, c, z);
    };
    auto loads = [&](int buf, int q) {
#pragma unroll
      for (int z = q; z < (q == 2 * NJ - 1 ? T::LPS : min(q + 1, T::LPS)); ++z) issue_one(buf, z);
    };
    Frag f0, f1;
    if (s_hi - s_lo >= T::BUF - 1) wait_but(newer);
    else wait_but(wait_all);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");           // no LDS read of a slice moves above the barrier
#pragma unroll
    for (int q = 0; q < NF; ++q) read_one(f0, ring + frag, 0, q);
    if (s_hi - s_lo > T::BUF - 1) issue(T::BUF - 1);
    int buf = 0;
    for (int s = s_lo; s < s_hi; ++s) {
      const int nxt = buf + 1 == T::BUF ? 0 : buf + 1;
      const bf16_t* base = ring + buf * T::STAGE + frag;
      const bf16_t* next = ring + nxt * T::STAGE + frag;
      __builtin_amdgcn_sched_barrier(0);
      half(f0, [&](int q) { reads(f1, base, 1, q); });
      if (s + T::BUF - 1 < s_hi) wait_but(newer);
      else wait_but(wait_all);
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      const bool fill = s + T::BUF < s_hi;
      half(f1, [&](int q) {
        reads(f0, next, 0, q);               // behind the last step nobody uses what is read
        if (fill) loads(buf, q);
      });
      if (KEEP && (((s - s_lo) & 3) == 3 || s + 1 == s_hi)) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) { acc[i][j] += part[i][KEEP ? j : 0]; clear(part[i][KEEP ? j : 0]); }
      }
      buf = nxt;
    }
  }

  // lane (column n = lane % 32 of a weight tile): element e of acc[i][j] is row 32 i + 8 (e / 4) + 4 (lane / 32) + e % 4 of the wave
  const int m_w = mb * BM + wm * 32 * RT, m_l = 4 * (lane >> 5), col = lane & 31;
  if (EPI != EPI_LOGITS && EPI != EPI_NLL && BN == GW_BN && pl.tail) {
    // raw sums [BM rows][256 weight rows] of this part of K, for the finishing kernel
    float* part = a.part + ((size_t)pl.ks * n_tail_ + (pl.t - n_full_)) * T::PART + (size_t)(wm * 32 * RT) * BN;
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if (WA) {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            *(f32x4*)(part + (32 * i + col) * BN + wtile(j) * 32 + 8 * q + m_l) = f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        } else {
#pragma unroll
          for (int e = 0; e < 16; ++e) part[(32 * i + 8 * (e >> 2) + m_l + (e & 3)) * BN + wtile(j) * 32 + col] = acc[i][j][e];
        }
      }
    return;
  }
  if (EPI == EPI_LOGITS && tid < BM) key_s[tid] = 0ull;
  __syncthreads();
  const int r_w = wm * 32 * RT + m_l;
  if constexpr (EPI == EPI_NLL) {
    // What the loss and the greedy choice need of this wave's 32 NJ entries, the logits themselves go nowhere: per row the largest one and
    // the sum of exponentials against it, the target's logit if it is here, and the best entry's key.  A lane has 16 NJ entries of
    // row 32 i + lane % 32, 32 j + 8 q + 4 (lane / 32) + 0..3 from n_w on; the row's others are with lane ^ 32.
    const int n_w = nb * BN + 32 * NJ * wn;
    const int* target = (const int*)a.g_next;
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const int m = m_w + 32 * i + col, mc = min(m, M - 1);
      const bool act = m < M;
      // other blocks raise it meanwhile: with an older value the search below runs once too often
      const unsigned long long seen = __hip_atomic_load(a.amax + mc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int rel = target[mc] - n_w - m_l;
      const float rs = rs_s[wm * 32 * RT + 32 * i + col];
      float mx = -INFINITY;
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] *= rs;
      if (n_w + 32 * NJ > N) {                             // entries beyond the vocabulary
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (n_w + m_l + 32 * j + 8 * (e >> 2) + (e & 3) >= N) acc[i][j][e] = -INFINITY;
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) mx = fmaxf(mx, acc[i][j][e]);
      mx = pair_max<32>(mx);
      const float mu = mx == -INFINITY ? 0.f : mx;
      float s = 0.f;
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) s += __expf(acc[i][j][e] - mu);
      s = pair_sum<32>(s);
      if (act && lane < 32) ((float2*)a.part)[(size_t)(nb * T::WN + wn) * a.ldp + m] = make_float2(mx, s);
      const bool hit = act && rel >= 0 && rel < 32 * NJ && !(rel & 4);
      if (__any(hit)) {                                    // a target: seldom
        float z = 0.f;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) z = rel == 32 * j + 8 * (e >> 2) + (e & 3) ? acc[i][j][e] : z;
        if (hit) a.ssp_next[m] = z;
      }
      // the best entry, where the row's largest value reaches the best so far: about one wave in three with a large vocabulary (a sum
      // that is not a number hides what the maximum may have left out, and zeros of either sign are told apart by their keys only)
      const bool need = act && (!(s == s) || mx == 0.f || ordered_bits(mx) >= (uint32_t)(seen >> 32));
      if (__any(need)) {
        uint32_t bo = 0u;
        int bi = 0;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int n = n_w + m_l + 32 * j + 8 * (e >> 2) + (e & 3);
            const uint32_t o = ordered_bits(acc[i][j][e]);
            if (n < N && o > bo) { bo = o; bi = n; }       // entries in rising order: the first of equal ones stays
          }
        unsigned long long key = ((unsigned long long)bo << 32) | (uint32_t)(0x7FFFFFFF - bi);
        const LanePair<unsigned long long> p = halves<32>(key, key);
        key = p.x > p.y ? p.x : p.y;
        if (need && lane < 32) atomicMax(a.amax + m, key);
      }
    }
    return;
  }
  if (EPI == EPI_SWIGLU) {
    // activation row 32 i + lane % 32 of the wave, outputs 16 j + 8 q + 4 (lane / 32) + 0..3 of its 16 NJ; lanes 32 apart then exchange halves, so
    // that the lower one stores the 8 outputs of q = 0 and the upper one those of q = 1
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const int m = m_w + 32 * i + col;
      const float rs = rs_s[wm * 32 * RT + 32 * i + col];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int n = nb * (BN / 2) + wtile(j) * 16 + 8 * (lane >> 5);
        uint32_t hi[2][2], lo[2][2];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const float g0 = acc[i][j][4 * q + 2 * h] * rs, u0 = acc[i][j][8 + 4 * q + 2 * h] * rs;
            const float g1 = acc[i][j][4 * q + 2 * h + 1] * rs, u1 = acc[i][j][8 + 4 * q + 2 * h + 1] * rs;
            if (BM != 128) swiglu_split2(g0, u0, g1, u1, hi[q][h], lo[q][h]);
            else if (h == 0) swiglu_split2<false, true>(g0, u0, g1, u1, hi[q][h], lo[q][h]);
            else swiglu_split2<true, false>(g0, u0, g1, u1, hi[q][h], lo[q][h]);
          }
        const LanePair<uint32_t> h0 = halves<32>(hi[0][0], hi[1][0]), h1 = halves<32>(hi[0][1], hi[1][1]);
        const LanePair<uint32_t> l0 = halves<32>(lo[0][0], lo[1][0]), l1 = halves<32>(lo[0][1], lo[1][1]);
        if (m < M && n < N) {
          const size_t at = packed_at(1, m, n, a.ldyb);
          *(u32x4*)(a.yb + at) = u32x4{h0.x, h1.x, h0.y, h1.y};
          *(u32x4*)(a.yb_lo + at) = u32x4{l0.x, l1.x, l0.y, l1.y};
        }
      }
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int ml = 32 * i + 8 * (e >> 2) + (e & 3), m = m_w + m_l + ml;
      const float rs = NORM ? rs_s[r_w + ml] : 1.f;
      unsigned long long best = 0ull;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int n = nb * BN + wtile(j) * 32 + col;
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
    if (tid < BM && mb * BM + tid < M) atomicMax(a.amax + (size_t)(nb % AMAX_CELLS) * a.amax_ld + mb * BM + tid, key_s[tid]);
  }
}

// Second stage of the tiles whose K was split over blocks (and of every residual tile): epilogue(sum of the parts, in order).  A
// block takes 16 rows of a tile, a wave 16 rows x 32 outputs at a time: lane (row = lane % 16, chunk = lane / 16) has 8
// consecutive outputs, so a wave writes 1 KiB of contiguous blocked layout per plane.  (Row by row, 4 outputs per thread, the
// blocked stores are 16-byte pieces: 38 us for 2048 x 2560 from 3 parts.)  With 2048 rows memory bounds it (126 MB in 25 us); with a few
// hundred the round trips do, so every load is issued ahead of the first sum (us, one round of 4 parts of a group at a time / now: residual,
// 256 rows of 1024 10.2 / 8.6, 1003 rows of 2560 20.6 / 19.3, gate/up 2048 rows 15.8 / 12.0, QKV 13.3 / 10.1).
template <int EPI, bool NORM, int BM>
__global__ void __launch_bounds__(256) gemm_wide_finish_kernel(const float* part_, int M_, int N_, int n_full_, int n_tail_, int ksplit_, int mt_, int nt_,
                                                               MfmaArgs a) {
  __shared__ float ss_s[4][16];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int M = M_, N = N_, t = n_full_ + blockIdx.x;
  const int per_group = 8 * nt_, grp = t / per_group, in = t - grp * per_group, rows = min(8, mt_ - grp * 8);
  const int nb = in / rows, mb = grp * 8 + in - nb * rows;
  const int r = blockIdx.y * 16 + (lane & 15), m = mb * BM + r, c8 = (lane >> 4) * 8;
  constexpr int PART = GwTile<BM, GW_BN>::PART;
  if (mb * BM + (int)blockIdx.y * 16 >= M) return;
  const bool act = m < M;
  const int mc = act ? m : M - 1;
  constexpr int OUT = EPI == EPI_SWIGLU ? GW_BN / 2 : GW_BN, GROUPS = OUT / 128;      // outputs of a tile; groups of 32 of them per wave
  constexpr int PRE = EPI == EPI_RESID ? 6 : 4;          // parts of every group fetched at once
  const size_t step = (size_t)n_tail_ * PART;
  float ssv[4];                                          // the row's partial sums of squares, 16 of them up front
  if (NORM)
#pragma unroll
    for (int j = 0; j < 4; ++j) ssv[j] = a.ssp[(size_t)min((lane >> 4) + 4 * j, a.n_parts - 1) * a.ssp_ld + mc];
  float hsq = 0.f;
  // all loads of all groups first: the residual rows, the gains, and up to PRE parts (a group beyond N repeats the first)
  const int c0 = nb * OUT;
  f32x4 sum[GROUPS][2], sum2[2], res[GROUPS][2];
  u32x4 gain[GROUPS];
  const float* src[GROUPS];
#pragma unroll
  for (int gi = 0; gi < GROUPS; ++gi) {
    const int lg = (w * GROUPS + gi) * 32, lc = (c0 + lg < N ? lg : 0) + c8;
    // SwiGLU: 16 gate sums, then the up sums of the same outputs
    src[gi] = part_ + (size_t)blockIdx.x * PART + (size_t)r * GW_BN + (EPI == EPI_SWIGLU ? (lc & ~15) * 2 + (lc & 15) : lc);
    sum[gi][0] = sum[gi][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (EPI == EPI_RESID) {
      res[gi][0] = *(const f32x4*)(a.y + (size_t)mc * a.ldy + c0 + lc);
      res[gi][1] = *(const f32x4*)(a.y + (size_t)mc * a.ldy + c0 + lc + 4);
      gain[gi] = *(const u32x4*)(a.g_next + c0 + lc);
    }
  }
  sum2[0] = sum2[1] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto add_parts = [&](int k0, auto n_c) {
    constexpr int n = decltype(n_c)::value;
    f32x4 x[GROUPS][n][2], z[EPI == EPI_SWIGLU ? n : 1][2];
#pragma unroll
    for (int gi = 0; gi < GROUPS; ++gi)
#pragma unroll
      for (int k = 0; k < n; ++k) {
        const float* q = src[gi] + (size_t)(k0 + k) * step;
        x[gi][k][0] = *(const f32x4*)q; x[gi][k][1] = *(const f32x4*)(q + 4);
        if (EPI == EPI_SWIGLU) { z[k][0] = *(const f32x4*)(q + 16); z[k][1] = *(const f32x4*)(q + 20); }
      }
#pragma unroll
    for (int gi = 0; gi < GROUPS; ++gi)
#pragma unroll
      for (int k = 0; k < n; ++k) {
        sum[gi][0] += x[gi][k][0]; sum[gi][1] += x[gi][k][1];
        if (EPI == EPI_SWIGLU) { sum2[0] += z[k][0]; sum2[1] += z[k][1]; }
      }
  };
  int k0 = 0;
  for (; k0 + PRE <= ksplit_; k0 += PRE) add_parts(k0, std::integral_constant<int, PRE>());
  static_for<1, PRE>([&](auto n) {
    if (ksplit_ - k0 == decltype(n)::value) add_parts(k0, n);
  });
  float rs = 1.f;
  if (NORM) {
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) ss += (lane >> 4) + 4 * j < a.n_parts ? ssv[j] : 0.f;
    for (int p = (lane >> 4) + 16; p < a.n_parts; p += 4) ss += a.ssp[(size_t)p * a.ssp_ld + mc];
    ss = column_sum(ss);
    rs = rsqrtf(ss / (float)a.K + a.eps);
  }
#pragma unroll
  for (int gi = 0; gi < GROUPS; ++gi) {
    const int n = c0 + (w * GROUPS + gi) * 32 + c8;
    if (n - c8 >= N) continue;                                               // N is a multiple of 64 here: whole groups
    const f32x4 s0 = sum[gi][0], s1 = sum[gi][1], u0 = sum2[0], u1 = sum2[1];
    f32x4 h0 = res[gi][0], h1 = res[gi][1];
    const u32x4 graw = gain[gi];
    float v[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
    if (EPI == EPI_STORE) {
      if (act) {
        *(f32x4*)(a.y + (size_t)m * a.ldy + n) = s0 * rs;
        *(f32x4*)(a.y + (size_t)m * a.ldy + n + 4) = s1 * rs;
      }
      continue;
    }
    uint32_t hi[4], lo[4];
    if (EPI == EPI_SWIGLU) {
      const float up[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) swiglu_split2(v[2 * e] * rs, up[2 * e] * rs, v[2 * e + 1] * rs, up[2 * e + 1] * rs, hi[e], lo[e]);
    } else {
      h0 += s0; h1 += s1;
      if (act) {
        *(f32x4*)(a.y + (size_t)m * a.ldy + n) = h0;
        *(f32x4*)(a.y + (size_t)m * a.ldy + n + 4) = h1;
      }
      const float hn[8] = {h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w};
      float gn[8];
      Elem<bf16_t>::unpack(graw, gn);
#pragma unroll
      for (int e = 0; e < 8; ++e) { hsq += hn[e] * hn[e]; v[e] = hn[e] * gn[e]; }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        hi[e] = pack_bf16x2(v[2 * e], v[2 * e + 1]);
        lo[e] = pack_bf16x2(v[2 * e] - __uint_as_float(hi[e] << 16), v[2 * e + 1] - __uint_as_float(hi[e] & 0xFFFF0000u));
      }
    }
    if (act) {
      const size_t at = packed_at(1, m, n, a.ldyb);
      *(u32x4*)(a.yb + at) = u32x4{hi[0], hi[1], hi[2], hi[3]};
      *(u32x4*)(a.yb_lo + at) = u32x4{lo[0], lo[1], lo[2], lo[3]};
    }
  }
  if (EPI == EPI_RESID) {
    // one sum of squares per row and tile of 256 outputs
    hsq = column_sum(hsq);
    if (lane < 16) ss_s[w][lane] = hsq;
    __syncthreads();
    if (tid < 16 && act) a.ssp_next[(size_t)nb * a.ssp_ld + m] = ss_s[0][tid] + ss_s[1][tid] + ss_s[2][tid] + ss_s[3][tid];
  }
}

}  // namespace dmtd
