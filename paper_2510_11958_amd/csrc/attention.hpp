// GQA decode attention for gfx950, split over the KV sequence ("split-K"), with the
// QK-RMSNorm, the rotary embedding and the KV-cache append of the new rows folded in.
//
// Two launches per layer.  (1) attn_split_kernel: a block = (key range, row group, KV head,
// sequence) and the query vectors of that row group that share the KV head (rows x GQ query
// heads, at most QVT).  Its key range is fixed by the launch (range index x keys per range), so
// the K/V loads of its first iteration are issued at once, together with the load of the
// device-resident position and of the raw q/k/v rows; nothing waits on anything else.  K and V
// rows go straight from HBM into registers with 16-byte per-lane loads: HD/8 lanes cover one key,
// so a wave load instruction fetches 64/(HD/8) adjacent keys (1 KiB contiguous).  While they fly
// the block normalises and rotates its query vectors and the launch's new keys (per-head RMSNorm,
// then RoPE with half-split pairing at the row's absolute position, cos/sin from a table) into LDS; the block whose
// range holds a new position takes that key and value from LDS (rounded to the cache's type,
// exactly what later steps read back) and the last row group's block also writes them to the
// cache.  Scoring: partial dot per lane, summed inside the lane group by shuffles; running softmax
// with the maximum shared across the wave; p*V accumulated for the 8 output dims a lane owns;
// lane groups summed by shuffles, the 4 waves through LDS; the range's (max, sum, unnormalised
// output) go to a partials buffer.  (2) attn_merge_kernel: per (row, query head, sequence), merges the
// ranges in a fixed order (deterministic) and writes the normalised output; all its loads are issued
// before the first one is needed.  The kernel boundary makes the partials visible across the chip
// (fences and same-kernel grid barriers were measured to cost far more on this chip).
//
// What bounds it on a small model is the chain position -> rotary table -> queries -> scores -> totals of one block: what does not depend on
// the position is loaded ahead of it, sixteen vectors are prepared at a time, and sums across lanes are exchanges between
// registers (tiny model, 33 to 48 keys, 1 or 2 rows: 8.7 us with shuffles and a wave per vector, 6.4 now).
//
// Keys beyond the current context inside a block's range are loaded (they lie inside the cache
// allocation) and masked; ranges wholly beyond the context exit early and are skipped by the merge.
#pragma once
#include "kernels.hpp"

namespace dmtd {

constexpr int QV_MAX = 16;         // query vectors per KV head one block can carry (and query heads per KV head)
constexpr int ATT_MAX_SPLITS = 64;

// Keys a block covers per iteration: 16 lane groups x 4 keys (head_dim 128) or 32 x 4 (head_dim 64).
template <int HD> struct AttKeysPerIter { static constexpr int value = 4 * (64 / (HD / 8)) * 4; };


// Which key range and row group of a sequence a block of a decode attention launch takes.  Grid: (ranges x row groups, KV heads,
// sequences); the row groups are fastest: those of a range read the same keys at about the same time.  In a front pass over some sequences
// (fmap) most row groups behind the first may be dead (live_rows); there the ranges are fastest, and the groups
// begin at another one for every KV head and sequence.  With the row groups fastest, blocks going round-robin over the 8 dies, two
// or four row groups left the living ones to 4 or 2 dies (1536 wide, 8 sequences of 2 rows beside one of 8, us per step of 4 layers with 8k / 32k
// keys: 200 / 313, here 194 / 285; a pass of its own for the longer one 200 / 288).
// MAP, here and in the kernels: such a pass.  Told apart by the pointer, every launch's prologue took 0.2 to 0.5 us longer.
struct AttPlace { int split, rg; };
template <bool MAP> __device__ __forceinline__ AttPlace att_place(int n_splits, int n_rg) {
  const int x = blockIdx.x;
  if (MAP) return AttPlace{x % n_splits, (int)(x / n_splits + blockIdx.y + blockIdx.z) % n_rg};
  return AttPlace{x / n_rg, x % n_rg};
}

// f over the keys of a wave: a value per lane slice that holds a key (2 or 4 neighbouring lanes each), every lane gets the result
template <int HD, typename F> __device__ __forceinline__ float key_reduce(float v, F f) {
  if (HD == 64) v = f(v, lane_dpp<kDppQuad2>(v));
  v = f(v, lane_dpp<kDppHalfMirror>(v));        // quads hold one value each: lane ^ 4
  v = f(v, lane_dpp<kDppRor8>(v));
  LanePair<float> p = halves<16>(v, v);
  v = f(p.x, p.y);
  p = halves<32>(v, v);
  return f(p.x, p.y);
}

// One block iteration of the running softmax: 4 keys per lane group (kf, vf: this lane's 8 dims of
// each), scored against every query vector.  After the in-group reduction lane slice sl holds the
// score of key u = sl >> USH, whose position is my_key; keys at or beyond key_end, or beyond the
// row's own position (row i = qv / GQ sees keys <= pos0 + i), are masked.
template <int HD, int QVT>
__device__ __forceinline__ void attn_accumulate(const float (&q)[QVT][8], const float (&kf)[4][8], const float (&vf)[4][8],
                                                int my_key, int key_end, int pos0, int GQ, int QV, int lane, int sl,
                                                float (&m)[QVT], float (&l)[QVT], float (&acc)[QVT][8]) {
  constexpr int LPK = HD / 8, U = 4;
  constexpr int USH = LPK == 16 ? 2 : 1;
#pragma unroll
for (int qv = 0; qv < QVT; ++qv) {
  if (qv < QV) {
    float s4[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float d = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) d += q[qv][e] * kf[u][e];
      s4[u] = d;
    }
    // sum over the lane group; the 4 keys' sums end up in 4 different lane slices (the mirror pairs a lane with one whose lower
    // bits are flipped too: the steps behind it sum over those)
    {
      constexpr int X1 = LPK == 16 ? kDppRor8 : kDppHalfMirror, X2 = LPK == 16 ? kDppHalfMirror : kDppQuad2;
      const bool up1 = (sl & (LPK / 2)) != 0;
      const float a0 = (up1 ? s4[2] : s4[0]) + lane_dpp<X1>(up1 ? s4[0] : s4[2]);
      const float a1 = (up1 ? s4[3] : s4[1]) + lane_dpp<X1>(up1 ? s4[1] : s4[3]);
      const bool up2 = (sl & (LPK / 4)) != 0;
      float s = (up2 ? a1 : a0) + lane_dpp<X2>(up2 ? a0 : a1);
      if (LPK == 16) s += lane_dpp<kDppQuad2>(s);
      s += lane_dpp<kDppQuad1>(s);
      s4[0] = s;
    }
    // causal and range mask: row i = qv / GQ sees keys <= pos0 + i
    float s = s4[0];
    if (my_key >= key_end || my_key > pos0 + qv / GQ) s = -INFINITY;
    const float mx = key_reduce<HD>(s, [](float a, float b) { return fmaxf(a, b); });   // over keys and lane groups
    const float m_new = fmaxf(m[qv], mx);
    if (m_new != -INFINITY) {
      const float sc = __expf(m[qv] - m_new);           // exp(-inf) = 0 on the first visible key
      const float p = (s == -INFINITY) ? 0.f : __expf(s - m_new);
      l[qv] = l[qv] * sc + p;
      float pu[U];
#pragma unroll
      for (int u = 0; u < U; ++u) pu[u] = __shfl(p, (lane & ~(LPK - 1)) | (u << USH), 64);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        acc[qv][e] = acc[qv][e] * sc + ((pu[0] * vf[0][e] + pu[1] * vf[1][e]) + (pu[2] * vf[2][e] + pu[3] * vf[3][e]));
      m[qv] = m_new;
    }
  }
}
}

// End of a wave's key loop: l summed over the keys, acc over the lane groups.  The sum over the groups halves the values a lane
// holds at each step: lane (slice sl, group grp) ends up with output dims 8 sl + e .. of query qv in acc[qv][0 ..], AttOut<HD> of them from
// e = AttOut<HD>::first(lane) on.
template <int HD> struct AttOut {
  static constexpr int n = HD == 64 ? 1 : 2;
  static __device__ __forceinline__ int first(int lane) { return (lane >> 5) * 4 + ((lane >> 4) & 1) * 2 + (HD == 64 ? (lane >> 3) & 1 : 0); }
};
template <int HD, int QVT>
__device__ __forceinline__ void attn_wave_totals(float (&l)[QVT], float (&acc)[QVT][8], int QV, int lane) {
#pragma unroll
  for (int qv = 0; qv < QVT; ++qv)
    if (qv < QV) {
      l[qv] = key_reduce<HD>(l[qv], [](float a, float b) { return a + b; });
      float (&v)[8] = acc[qv];
#pragma unroll
      for (int e = 0; e < 4; ++e) { const LanePair<float> p = halves<32>(v[e], v[e + 4]); v[e] = p.x + p.y; }
#pragma unroll
      for (int e = 0; e < 2; ++e) { const LanePair<float> p = halves<16>(v[e], v[e + 2]); v[e] = p.x + p.y; }
      if (HD == 64) {
        const bool up = (lane & 8) != 0;
        const float send = up ? v[0] : v[1], keep = up ? v[1] : v[0];
        v[0] = keep + lane_dpp<kDppRor8>(send);
      }
    }
}

// Rotary table, built once: (cos, sin) of position * theta^(-2i/hd), angle and functions in double
// precision, stored rounded to float (what the attention kernel would otherwise compute per launch).
__global__ void rope_table_kernel(const double* __restrict__ inv_freq, float2* __restrict__ tab, int s_max, int half) {
  const size_t n = (size_t)s_max * half;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    double sn, cs;
    sincos((double)(i / half) * inv_freq[i % half], &sn, &cs);
    tab[i] = make_float2((float)cs, (float)sn);
  }
}

// A vector of the prologue (a query, a new key or a new value of one head) is handled by 16 neighbouring lanes; lane l holds the
// rotary pairs (HL l + e, HD/2 + HL l + e), e < HL.
template <int HD> struct AttRow {
  static constexpr int HL = HD / 32;
  typedef float vec __attribute__((ext_vector_type(HD / 32)));
  vec a, b;
  __device__ __forceinline__ void load(const float* p, int l) { a = *(const vec*)(p + HL * l); b = *(const vec*)(p + HD / 2 + HL * l); }
};
// Sum over the 16 lanes of a DPP row by rotations (every lane ends up with the total).
__device__ __forceinline__ float row16_sum(float v) {
  v += lane_dpp<0x128>(v);
  v += lane_dpp<0x124>(v);
  v += lane_dpp<0x122>(v);
  v += lane_dpp<0x121>(v);
  return v;
}

// QK-RMSNorm + RoPE + KV append as a launch of its own, for passes that carry more rows per sequence than an attention
// block keeps in LDS (prefill, the whole-sequence forward): per-head RMSNorm and rotation of the rows' keys, and their
// values, rounded to the cache's type and stored; the attention launch that follows then finds every key in the cache
// (do_append = 2).  One wave per (row, KV head).
template <typename CT, int HD>
__global__ void __launch_bounds__(64) kv_append_kernel(
    const float* __restrict__ qkv, int ldq, const void* __restrict__ k_gain, const float2* __restrict__ rope_tab,
    CT* __restrict__ kc, CT* __restrict__ vc, int nh, int nkv, int s_max, float eps, const DevState* st, int sel, int offset, int r_total) {
  constexpr int half = HD / 2;
  const int row_g = blockIdx.x, g = blockIdx.y, lane = threadIdx.x;
  const int b = row_g / r_total, i = row_g % r_total;
  const int key = row_base(st, sel, offset, b) + i;
  const float* ksrc = qkv + (size_t)row_g * ldq + (size_t)(nh + g) * HD;
  const float* vsrc = qkv + (size_t)row_g * ldq + (size_t)(nh + nkv + g) * HD;
  const bool act = lane < half;
  float x0 = act ? ksrc[lane] : 0.f, x1 = act ? ksrc[lane + half] : 0.f;
  const float rs = rsqrtf(wave_sum(x0 * x0 + x1 * x1) / (float)HD + eps);
  CT* kd = kc + (((size_t)b * nkv + g) * s_max + key) * HD;
  CT* vd = vc + (((size_t)b * nkv + g) * s_max + key) * HD;
  if (act) {
    const CT* gn = (const CT*)k_gain;
    x0 *= rs * Elem<CT>::to_f32(gn[lane]);
    x1 *= rs * Elem<CT>::to_f32(gn[lane + half]);
    const float2 cs = rope_tab[(size_t)key * half + lane];
    kd[lane] = Elem<CT>::from_f32(x0 * cs.x - x1 * cs.y);
    kd[lane + half] = Elem<CT>::from_f32(x1 * cs.x + x0 * cs.y);
  }
  for (int k = lane; k < HD; k += 64) vd[k] = Elem<CT>::from_f32(vsrc[k]);
}

template <int HD, int QVT, bool MAP>
__global__ void __launch_bounds__(256) attn_split_kernel(
    const float* __restrict__ qkv, int ldq, const void* __restrict__ q_gain, const void* __restrict__ k_gain,
    const float2* __restrict__ rope_tab /* [s_max][HD / 2] (cos, sin) of position * theta^(-2i/HD) */, float* __restrict__ kc, float* __restrict__ vc,
    float* __restrict__ part_o, float* __restrict__ part_ml, int nh, int nkv, int s_max, float eps,
    int kps /* keys per range, a multiple of the block iteration */, int n_splits, int qv_stride,
    const DevState* st, int sel, int offset, int r_total,
    int do_append /* 1: the launch appends its rows' keys and values; 0: it scores them from its inputs and leaves the cache untouched (measurement); 2: they are in the cache already */,
    const int* __restrict__ fmap /* MAP: launch sequence -> sequence slot (cache rows, positions) */,
    float* __restrict__ out, int ldo /* nullable: one range, no merge launch follows */) {
  typedef Elem<float>::Raw Raw;
  constexpr int LPK = HD / 8;          // lanes per key (16 or 8)
  constexpr int GPW = 64 / LPK;        // lane groups per wave (4 or 8)
  constexpr int NG = 4 * GPW;          // lane groups per block
  constexpr int U = 4;                 // keys per lane group per iteration
  constexpr int KPI = NG * U;          // keys per block iteration
  static_assert(KPI == AttKeysPerIter<HD>::value, "block iteration size");
  constexpr int USH = LPK == 16 ? 2 : 1;   // after the score reduction, lane slice sl holds key u = sl >> USH
  constexpr int NEW_MAX = 16;          // rows a launch can carry

  const int g = blockIdx.y, b = blockIdx.z;
  const int GQ = nh / nkv;
  const int rpb = QVT / GQ;                                    // rows per block
  const int n_rg = (r_total + rpb - 1) / rpb;
  const AttPlace pl = att_place<MAP>(n_splits, n_rg);
  const int split = pl.split, rg = pl.rg;
  // rows and partials are indexed by the launch's sequence number b, the cache and the positions by the sequence's slot:
  // the cache pointers are moved so that index b lands on the slot
  const int bs = MAP ? fmap[b] : b;
  kc += (ptrdiff_t)(bs - b) * nkv * s_max * HD;
  vc += (ptrdiff_t)(bs - b) * nkv * s_max * HD;
  if (MAP && rg > 0 && rg * rpb >= live_rows(st, bs, r_total)) return;      // no row of its own; the first group has one
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int key_begin = split * kps;
  const int sl = lane % LPK, grp = wave * GPW + lane / LPK;
  const int my_u = sl >> USH;
  // the rows this block prepares if every row is alive: its queries, then the new keys and values its queries may see
  const int QV_all = min(rpb, r_total - rg * rpb) * GQ, new_all = min(r_total, (rg + 1) * rpb);
  const int vl = tid & 15, vg = tid >> 4;              // lane of a 16-lane row; row of the block
  AttRow<HD> x0, gq, gk;
  auto vec_src = [&](int v) {                          // vector v of the prologue
    const bool is_q = v < QV_all, is_k = v < QV_all + new_all;
    const int row = is_q ? rg * rpb + v / GQ : (is_k ? v - QV_all : v - QV_all - new_all);
    return qkv + (size_t)(b * r_total + row) * ldq + (size_t)(is_q ? g * GQ + v % GQ : (is_k ? nh + g : nh + nkv + g)) * HD;
  };
  // the first vector and the gains: what does not depend on the position is on its way before that is known
  x0.load(vec_src(min(vg, QV_all + 2 * new_all - 1)), vl);
  gq.load((const float*)q_gain, vl);
  gk.load((const float*)k_gain, vl);

  __shared__ __attribute__((aligned(16))) float q_s[QVT][HD];
  __shared__ __attribute__((aligned(16))) float knew_s[NEW_MAX][HD], vnew_s[NEW_MAX][HD];
  __shared__ float wacc[4][QVT][HD];
  __shared__ float wm[4][QVT], wl[4][QVT];

  // K/V of the first iteration: addresses depend on the launch only
  const float* kbase = kc + (((size_t)b * nkv + g) * s_max) * HD + sl * 8;
  const float* vbase = vc + (((size_t)b * nkv + g) * s_max) * HD + sl * 8;
  Raw kr[U], vr[U];
  int loaded = 0;                      // the limit of the keys in kr and vr
  auto load_kv = [&](int it0, int limit) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int key = min(it0 + u * NG + grp, limit - 1);      // unconditional; a key beyond the limit becomes zero when it is used
      kr[u] = Elem<float>::load_raw(kbase + (size_t)key * HD);
      vr[u] = Elem<float>::load_raw(vbase + (size_t)key * HD);
    }
    loaded = limit;
  };
  load_kv(key_begin, min(s_max, key_begin + kps));

  const int pos_first = row_base(st, sel, offset, bs);
  const int live = MAP ? live_rows(st, bs, r_total) : r_total; // rows of this sequence; the others of its r_total are dead
  const int r = min(rpb, live - rg * rpb), QV = r * GQ;
  if (r <= 0) return;
  const int pos0 = pos_first + rg * rpb;                        // position of this block's first row
  const int ctx = pos0 + r;                                     // keys 0 .. ctx-1 are visible to its last row
  if (key_begin >= ctx) return;                                 // whole range beyond the context (block-uniform)
  const int key_end = min(ctx, key_begin + kps);
  const int n_new = rg * rpb + r;                               // new rows whose keys this block's rows can see
  const bool holds_new = do_append != 2 && key_end > pos_first; // a new position, not yet in the cache, falls into this range
  const bool writer = do_append == 1 && (rg + 1) * rpb >= live;   // the last row group's blocks append to the cache

  // Per-head RMSNorm + RoPE (cos/sin from the table) of the block's queries, scaled by 1/sqrt(HD), into q_s and, if the range holds new
  // positions, of the launch's new keys, and the new values, into knew_s / vnew_s; the writer also stores them to the cache.
  // Sixteen vectors at a time.
  {
    constexpr int HL = AttRow<HD>::HL, half = HD / 2;
    const float scale = rsqrtf((float)HD);
    const int n_vec = QV_all + (holds_new ? 2 * new_all : 0);
    for (int v = vg; v < n_vec; v += 16) {
      const bool is_q = v < QV_all, is_k = !is_q && v < QV_all + new_all;
      const int row = is_q ? rg * rpb + v / GQ : (is_k ? v - QV_all : v - QV_all - new_all);
      AttRow<HD> x = x0;
      if (v != vg) x.load(vec_src(v), vl);
      if (row >= live) continue;
      const int key = pos_first + row;
      const bool wr = !is_q && writer && key >= key_begin && key < key_end;
      const size_t at = (((size_t)b * nkv + g) * s_max + key) * HD + HL * vl;
      typename AttRow<HD>::vec ya = x.a, yb = x.b;
      if (is_q || is_k) {
        float ss = 0.f;
#pragma unroll
        for (int e = 0; e < HL; ++e) ss += x.a[e] * x.a[e] + x.b[e] * x.b[e];
        const float rs = rsqrtf(row16_sum(ss) / (float)HD + eps);
        const float2* rp = rope_tab + (size_t)key * half + HL * vl;
#pragma unroll
        for (int e = 0; e < HL; ++e) {
          const float2 cs = rp[e];
          const float a0 = x.a[e] * (rs * (is_q ? gq.a[e] : gk.a[e])), a1 = x.b[e] * (rs * (is_q ? gq.b[e] : gk.b[e]));
          ya[e] = a0 * cs.x - a1 * cs.y;
          yb[e] = a1 * cs.x + a0 * cs.y;
        }
      }
      typedef typename AttRow<HD>::vec vec;
      if (is_q) {
        *(vec*)&q_s[v][HL * vl] = ya * scale; *(vec*)&q_s[v][half + HL * vl] = yb * scale;
      } else {
        float (*dst)[HD] = is_k ? knew_s : vnew_s;
        *(vec*)&dst[row][HL * vl] = ya; *(vec*)&dst[row][half + HL * vl] = yb;
        if (wr) {
          float* c = (is_k ? kc : vc) + at;
          *(vec*)c = ya; *(vec*)(c + half) = yb;
        }
      }
    }
  }
  __syncthreads();

  float q[QVT][8];
#pragma unroll
  for (int qv = 0; qv < QVT; ++qv)
#pragma unroll
    for (int e = 0; e < 8; ++e) q[qv][e] = qv < QV ? q_s[qv][sl * 8 + e] : 0.f;
  float m[QVT], l[QVT], acc[QVT][8];
#pragma unroll
  for (int qv = 0; qv < QVT; ++qv) {
    m[qv] = -INFINITY; l[qv] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[qv][e] = 0.f;
  }

  for (int it0 = key_begin; it0 < key_end; it0 += KPI) {
    float kf[U][8], vf[U][8];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool ok = it0 + u * NG + grp < loaded;
      Elem<float>::unpack(ok ? kr[u] : Elem<float>::zero_raw(), kf[u]);
      Elem<float>::unpack(ok ? vr[u] : Elem<float>::zero_raw(), vf[u]);
    }
    if (it0 + KPI < key_end) load_kv(it0 + KPI, key_end);       // next iteration's keys fly during the scoring
    if (holds_new) {
      // new positions: key and value come from LDS, not from the cache slot (written by another block, or not yet)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = it0 + u * NG + grp - pos_first;
        if (i >= 0 && i < n_new) {
#pragma unroll
          for (int e = 0; e < 8; ++e) { kf[u][e] = knew_s[i][sl * 8 + e]; vf[u][e] = vnew_s[i][sl * 8 + e]; }
        }
      }
    }
    attn_accumulate<HD, QVT>(q, kf, vf, it0 + my_u * NG + grp, key_end, pos0, GQ, QV, lane, sl, m, l, acc);
  }

  attn_wave_totals<HD, QVT>(l, acc, QV, lane);
#pragma unroll
  for (int qv = 0; qv < QVT; ++qv)
    if (qv < QV) {
#pragma unroll
      for (int e = 0; e < AttOut<HD>::n; ++e) wacc[wave][qv][sl * 8 + AttOut<HD>::first(lane) + e] = acc[qv][e];
      if (lane == 0) { wm[wave][qv] = m[qv]; wl[wave][qv] = l[qv]; }
    }
  __syncthreads();
  // partials are indexed by the launch-wide query-vector number row * GQ + head
  const size_t slot = (((size_t)b * nkv + g) * ATT_MAX_SPLITS + split) * qv_stride + (size_t)rg * rpb * GQ;
  float* my_o = part_o + slot * HD;
  float* my_ml = part_ml + slot * 2;
  for (int e = tid; e < QV * HD; e += 256) {
    const int qv = e / HD, d = e % HD;
    const float mm = fmaxf(fmaxf(wm[0][qv], wm[1][qv]), fmaxf(wm[2][qv], wm[3][qv]));
    float o = 0.f, ll = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float f = (wm[w][qv] == -INFINITY) ? 0.f : __expf(wm[w][qv] - mm);
      o += f * wacc[w][qv][d];
      ll += f * wl[w][qv];
    }
    if (out) {       // the launch's only range: the block's result is the attention output (what the merge of one range gives)
      out[(size_t)(b * r_total + rg * rpb + qv / GQ) * ldo + (size_t)(g * GQ + qv % GQ) * HD + d] = o * (1.0f / ll);
      continue;
    }
    my_o[qv * HD + d] = o;
    if (d == 0) { my_ml[qv * 2] = mm; my_ml[qv * 2 + 1] = ll; }
  }
}

// Merge the ranges' partial results: out[row, head, :] = sum_s f_s o_s / sum_s f_s l_s with
// f_s = exp(m_s - max_s m_s).  One block (256 threads) per (row, query head, sequence): thread (group, d4) takes
// 4 consecutive d of the ranges group, group + NG, ...; every load is issued before the first one is needed; the
// maximum and the denominator are wave reductions over one lane per range; the groups' sums are added in group
// order through LDS (deterministic).
template <int HD, typename OT, bool MAP>   // OT: float, or bf16_t (the packed input of the O projection: high parts to out, low parts to out_lo)
__global__ void __launch_bounds__(256) attn_merge_kernel(
    const float* __restrict__ part_o, const float* __restrict__ part_ml, OT* __restrict__ out, OT* __restrict__ out_lo, int ldo,
    int nh, int nkv, int kps, int n_splits, int qv_stride, const DevState* st, int sel, int offset, int r_total,
    const int* __restrict__ fmap /* MAP: launch sequence -> sequence slot (positions) */, int blocked /* layout of a bf16 output (packed_at) */) {
  constexpr int T4 = HD / 4;              // threads per group: one per 4 consecutive d
  constexpr int NG = 256 / T4;            // groups (8 or 16); group sg takes ranges sg, sg + NG, ...
  constexpr int PRE = 4;                  // ranges per thread fetched before anything is waited for (4 * NG >= 32 ranges)
  static_assert(ATT_MAX_SPLITS <= 64, "one wave holds a lane per range");
  const int i = blockIdx.x, head = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x;
  const int GQ = nh / nkv, g = head / GQ, j = head % GQ;
  const int sg = tid / T4, d = (tid % T4) * 4;
  const int bs = MAP ? fmap[b] : b;
  if (MAP && i > 0 && i >= live_rows(st, bs, r_total)) return;       // a dead row; the first is alive
  __shared__ float f_s[ATT_MAX_SPLITS];
  __shared__ float inv_l_s;
  __shared__ __attribute__((aligned(16))) float red[NG][HD];
  const size_t slot0 = ((size_t)b * nkv + g) * ATT_MAX_SPLITS;
  const size_t qv = (size_t)i * GQ + j;
  float mv = -INFINITY, lv = 0.f;
  {
    const float2 ml = *(const float2*)(part_ml + ((slot0 + (tid < n_splits ? tid : 0)) * qv_stride + qv) * 2);
    if (tid < n_splits) { mv = ml.x; lv = ml.y; }
  }
  const float* po = part_o + ((slot0 + sg) * qv_stride + qv) * HD + d;
  const size_t po_step = (size_t)NG * qv_stride * HD;
  f32x4 ov[PRE];
#pragma unroll
  for (int u = 0; u < PRE; ++u) {
    // unconditional, from a clamped range index (a range beyond n_splits gets factor 0 below): a load under a
    // per-lane condition would be waited for on the spot, one memory round trip after the other
    const int uc = sg + u * NG < n_splits ? u : 0;
    ov[u] = *(const f32x4*)(po + uc * po_step);
  }
  const int pos_row = row_base(st, sel, offset, bs) + i;    // row i sees keys 0 .. pos_row
  const int n_act = min(n_splits, pos_row / kps + 1);   // ranges that hold keys visible to row i; later ones hold stale partials
  if (tid < 64) {
    // the first wave holds one range per lane: maximum and weighted sum by shuffles (a fixed tree: deterministic)
    const float m_l = tid < n_act ? mv : -INFINITY;
    const float mm = wave_max(m_l);
    const float f = (m_l != -INFINITY) ? __expf(m_l - mm) : 0.f;
    f_s[tid] = f;
    const float ll = wave_sum(f == 0.f ? 0.f : f * lv);     // a skipped range may hold anything
    if (tid == 0) inv_l_s = 1.0f / ll;
  }
  __syncthreads();
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < PRE; ++u) {
    const int s2 = sg + u * NG;
    const float f = s2 < n_act ? f_s[s2] : 0.f;
    if (f != 0.f) o += f * ov[u];
  }
  for (int s2 = sg + PRE * NG; s2 < n_act; s2 += NG) {
    const float f = f_s[s2];
    if (f != 0.f) o += f * *(const f32x4*)(po + (size_t)(s2 / NG) * po_step);
  }
  *(f32x4*)&red[sg][d] = o;
  __syncthreads();
  if (tid < T4) {
    f32x4 t = *(const f32x4*)&red[0][d];
#pragma unroll
    for (int q = 1; q < NG; ++q) t += *(const f32x4*)&red[q][d];
    const size_t at = packed_at(blocked, b * r_total + i, head * HD + d, ldo);     // 4 consecutive values stay together in both layouts
    const float inv_l = inv_l_s;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float res = t[e] * inv_l;
      const OT hi = Elem<OT>::from_f32(res);
      out[at + e] = hi;
      if (out_lo) out_lo[at + e] = Elem<OT>::from_f32(res - Elem<OT>::to_f32(hi));
    }
  }
}

}  // namespace dmtd
