// Attention over gathered cache rows with direct global -> LDS loads (BF16 compute path).
//
// Same work decomposition and arithmetic as the register-staged kernel in attention.hip:
// one workgroup of 4 wavefronts per (work item, kv head); scores computed transposed,
// S^T = K Q^T, so that every accumulator of a lane belongs to one query; online softmax in
// FP32 on raw scores with the 1/sqrt(D) scale folded into the exponent; O^T = V^T P^T.
// The difference is how key/value tiles reach LDS: with global_load_lds every lane names
// one 16-byte chunk of a cached row anywhere in HBM and the chunk lands in LDS at the
// lane's slot, so a gathered tile costs no registers and up to NS tiles are in flight per
// workgroup.  Completion is tracked with explicit vmcnt waits: every wavefront issues the
// same number of vector-memory operations per tile.
//
// What bounds it: many long units, HBM (4.4 TB/s with a BF16 cache, 1024 documents of the scale
// workload's lengths; 763 us a launch); a single unit, the chain of one tile's step (wait,
// scores, maximum, exponentials, value product).  The loop is written for that chain: the three
// cursors below step through a source with a few scalar operations (forming every tile's
// addresses from the descriptors of all three sources took half of the loop's instructions), the
// maximum crosses lanes without LDS, and no register load can make the compiler wait for the
// tiles in flight (a conditional query load did, at every tile).  One unit of 4096 keys: 189 ->
// 113 us (1.47 -> 0.88 us a tile); FP8 cache, 1024 documents: 712 -> 550 us.
//
// LDS layout of a tile part (K or V): rows in the source dtype (FP8 cache rows, BF16
// cache or own rows), chunk c of row r at slot c ^ swz(r).  The K swizzle spreads the 16
// rows read at one chunk by an S^T operand over distinct banks; the V swizzle does the
// same for the 8 rows x 2 chunks of a transposed read.  V^T operands come from
// ds_read_b64_tr_b16 (BF16 rows) or ds_read_b64_tr_b8 (FP8 rows) without a transposing
// copy; FP8 values are widened with the hardware FP8 -> BF16 conversion (exact: every E4M3
// value is a BF16 value) and their per-16-row block scales multiply scores and
// probabilities as in the register-staged kernel.
#include <algorithm>
#include <type_traits>

#include "direct_loads.h"
#include "common.h"
#include "kernels.h"

namespace kvop {

typedef short v4i16_t __attribute__((ext_vector_type(4)));
typedef int v2i32_t __attribute__((ext_vector_type(2)));

template <typename TKV, int D, int KT_, int NS_>
struct DmaCfg {
  static constexpr bool FP8 = sizeof(TKV) == 1;
  static constexpr int KT = KT_;                     // keys per cache tile
  static constexpr int NS = NS_;                     // stages (tiles resident in LDS)
  static constexpr int RBC = D * (int)sizeof(TKV);   // bytes per cached row
  static constexpr int RBO = D * 2;                  // bytes per own (BF16) row
  static constexpr int KTO = FP8 ? KT / 2 : KT;      // keys per own tile: the same bytes as a cache tile
  static constexpr int CHC = RBC / 16, CHO = RBO / 16;
  static constexpr int REGION = KT * RBC;            // bytes of the K (or V) part of a tile
  static_assert(KT * RBC == KTO * RBO, "cache and own tiles move the same bytes");
  static constexpr int NJ = 2 * REGION / 16 / 256;   // chunk loads per thread per tile
  static constexpr int NR = NJ / 2;                  // rows per thread per tile (K and V chunks share them)
  static_assert(NJ >= 2 && NJ % 2 == 0, "tile split");
  static constexpr int META = FP8 ? 3 * 64 * 4 : 0;  // ksc | vsc | unused (64 slots each)
  static constexpr int STAGE = 2 * REGION + META;
  static constexpr int LEAD = NS - 1;                // row numbers are loaded LEAD tiles before their chunks
  static constexpr int NRING = NS + LEAD;            // row-number ring: tiles ti .. ti + NS - 1 + LEAD
  static constexpr int RING = NS * STAGE;
  static constexpr int LDS = RING + NRING * 64 * 4;
  static constexpr int LDS_TOTAL = LDS;
  static constexpr int OPS = NJ + (FP8 ? 1 : 0);     // vector-memory operations of one tile (chunks, FP8 scales)
  static_assert((NS - 2) * (OPS + 1) <= 63 && NS >= 2, "vmcnt immediates");
  static_assert(kOwnRows % KTO == 0, "whole own tiles between moves of the base");
};

// log2(16 / CH): consecutive rows that share one 256-byte bank line
template <int CH> struct RowShift {
  static constexpr int v = CH >= 16 ? 0 : (CH == 8 ? 1 : (CH == 4 ? 2 : 3));
};
template <int CH> __host__ __device__ constexpr int swz_k(int r) { return (r >> RowShift<CH>::v) & (CH - 1); }
template <int CH> __host__ __device__ constexpr int swz_v(int r) { return CH >= 4 ? 2 * ((r >> RowShift<CH>::v) & (CH / 2 - 1)) : 0; }
// V swizzle of FP8 rows (read by ds_read_b64_tr_b8: rows r, r + 1, r + 2, r + 3 and the
// same + 16 at one chunk, for two lane groups): distinct (slot, bank line half) pairs
template <int CH> __device__ inline int swz_v8(int r) {
  if constexpr (CH >= 8) return ((r >> 1) & 3) | (((r >> 4) & 1) << 2);
  else return ((r >> 2) & 1) | (((r >> 4) & 1) << 1);
}

__device__ inline void ds_read_tr8_x4(const uint32_t (&ad)[4], u32x2 (&y)[4]) {
  asm volatile(
      "ds_read_b64_tr_b8 %0, %4\n\tds_read_b64_tr_b8 %1, %5\n\t"
      "ds_read_b64_tr_b8 %2, %6\n\tds_read_b64_tr_b8 %3, %7\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(y[0]), "=&v"(y[1]), "=&v"(y[2]), "=&v"(y[3])
      : "v"(ad[0]), "v"(ad[1]), "v"(ad[2]), "v"(ad[3])
      : "memory");
}

template <typename TKV, int D, int KT, int NS, int KC, bool LISTS>
__device__ void attn_dma_unit(const AttnArgs& a, int unit, uint8_t* smem) {
  using C = DmaCfg<TKV, D, KT, NS>;
  constexpr int NQ = D / 32;                 // 32-deep K steps of S^T
  constexpr int ND = D / 16;                 // 16-wide d blocks of the output
  static_assert(KT % KC == 0 && KC % 32 == 0, "compute steps of whole 32-key pairs");
  constexpr bool FP8 = C::FP8;

  const int Hkv = a.Hkv;
  const int h = unit % Hkv;
  // the work item's fields one by one: a struct that is read through selected members would live
  // in scratch memory, and a scratch load waits behind every tile load in flight
  const AttnWork* wp = a.work + unit / Hkv;
  const int64_t w_off_a = wp->off_a, w_off_b = wp->off_b, w_idx_a = wp->idx_a, w_idx_b = wp->idx_b;
  const int w_L_a = wp->L_a, w_L_b = wp->L_b, w_n_a = wp->n_a, w_n_b = wp->n_b, w_q_row0 = wp->q_row0;
  const int w_q_pos0 = wp->q_pos0, w_n_q = wp->n_q, w_own_row0 = wp->own_row0, w_n_own = wp->n_own;
  const int w_own_pos0 = wp->own_pos0, w_pad_a = wp->pad_a;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qi = lane & 15, g4 = lane >> 4;
  const int r = wave * 16 + qi;
  const int gq = r / a.Pmax, p = r % a.Pmax;
  const bool qvalid = gq < a.G && p < w_n_q;
  const bool wave_active = __any(qvalid);
  const int hq = h * a.G + (gq < a.G ? gq : 0);
  const int qpos = w_q_pos0 + p;
  const int64_t qrow = (int64_t)w_q_row0 + (qvalid ? p : 0);

  // ---- query fragments (B operand of S^T).  Joins: the fragments of the queries rotated at
  // position - L_A are loaded when the tiles of document B begin, and the plain ones again
  // after them (both sets would cost the registers of a resident workgroup).
  u32x4 qf[NQ];
  const bf16_t* q_plain = reinterpret_cast<const bf16_t*>(a.q) + qrow * a.q_stride + hq * D;
  const bf16_t* q_rot = reinterpret_cast<const bf16_t*>(a.q_alt ? a.q_alt : a.q) + qrow * a.q_stride + hq * D;
  auto load_q = [&](const bf16_t* q) {
#pragma unroll
    for (int k = 0; k < NQ; k++)
      qf[k] = qvalid ? gload(reinterpret_cast<const u32x4*>(q + 32 * k + 8 * g4)) : u32x4{0, 0, 0, 0};
  };
  load_q(q_plain);

  // ---- key sources: 0 = document A, 1 = document B, 2 = own rows.  Three cursors walk the same
  // sequence of tiles: the row numbers being fetched, the chunks being fetched, the tile being
  // computed.  Each keeps what it needs of its current source and steps through it with a few
  // scalar operations; a source's addresses are formed only when a cursor enters it.
  auto keys_of = [&](int s) { return s == 0 ? w_n_a : (s == 1 ? w_n_b : w_n_own); };
  auto iterated = [&](int s) { return s == 0 && w_n_a > 0 ? max(w_n_a, w_pad_a) : keys_of(s); };
  auto step_of = [&](int s) { return FP8 && s == 2 ? C::KTO : KT; };
  auto next_source = [&](int s) {     // the next source with keys (2 when there is none)
    do s++;
    while (s < 2 && keys_of(s) == 0);
    return s;
  };
  auto list_of = [&](int s) -> const int32_t* {
    const int64_t il = s == 0 ? w_idx_a : w_idx_b;
    return LISTS && s < 2 && il >= 0 ? a.idx + il : nullptr;
  };
  const int first = keys_of(0) > 0 ? 0 : (keys_of(1) > 0 ? 1 : 2);
  const int TA = w_n_a > 0 ? (iterated(0) + KT - 1) / KT : 0, TB = (w_n_b + KT - 1) / KT;
  const int T = TA + TB + (w_n_own + C::KTO - 1) / C::KTO;
  // a valid address for loads whose value is not used (keeps the per-tile load count fixed)
  const int32_t* dummy = reinterpret_cast<const int32_t*>(a.work + unit / Hkv);

  // Row numbers of retained lists reach LDS by direct loads too (one 4-byte load per key, lane =
  // key), LEAD tiles before the chunks that need them, into a ring of NRING slots: the loop
  // holds no register-destination memory load, so the only waits on memory are explicit.
  int* ring = reinterpret_cast<int*>(smem + C::RING);
  struct { int s, t, n, np, slot; const int32_t* idx; } rc;
  auto enter_rows = [&](int s) {
    rc.s = s;
    rc.t = 0;
    rc.n = keys_of(s);
    rc.np = iterated(s);
    rc.idx = list_of(s);
  };
  auto issue_rows = [&]() {
    if constexpr (LISTS) {
      // a padded tile (past the source's keys) loads the source's rows again from the start of
      // the list, cyclically: real rows, so the padded keys cost loads and multiplies.  Past the
      // last tile the load goes on with row numbers that nobody reads.
      const int tl = rc.t < rc.n ? rc.t : rc.t % max(rc.n, 1);
      const int32_t* g = rc.idx ? rc.idx + min(tl + lane, rc.n - 1) : dummy;
      load_to_lds<4>(g, ring + rc.slot * 64);
      rc.slot = rc.slot + 1 == C::NRING ? 0 : rc.slot + 1;
      rc.t += step_of(rc.s);
      if (rc.t >= rc.np && rc.s < 2) enter_rows(next_source(rc.s));
    }
  };

  // chunk loads of the next tile, then (FP8) one metadata load per wavefront (key = lane):
  // wave 0 the K block scales, wave 1 the V block scales, waves 2-3 none (a load of an unused
  // word keeps the count per wavefront the same)
  struct { int s, t, n, np, clampL, pitch, slot, stage; bool list; const uint8_t *k, *v; const float *ksc, *vsc; } ic;
  auto enter_tiles = [&](int s) {
    ic.s = s;
    ic.t = 0;
    ic.n = keys_of(s);
    ic.np = iterated(s);
    ic.list = list_of(s) != nullptr;
    ic.ksc = ic.vsc = nullptr;
    ic.k = ic.v = a.pool;
    if (s == 2) {
      ic.np = kOwnRows;
      ic.clampL = max(ic.n, 1);
      ic.pitch = (int)a.own_stride * 2;
      const uint8_t* ob = reinterpret_cast<const uint8_t*>(a.own) + (int64_t)w_own_row0 * a.own_stride * 2;
      ic.k = ob + (int64_t)(a.own_kcol + h * D) * 2;
      ic.v = ob + (int64_t)(a.own_vcol + h * D) * 2;
    } else if (ic.n > 0) {
      const int L = s == 0 ? w_L_a : w_L_b;
      ic.clampL = max(L, 1);
      ic.pitch = C::RBC;
      const uint8_t* base = a.pool + (s == 0 ? w_off_a : w_off_b);
      const int64_t kv_elems = (int64_t)L * D;
      const int64_t hk = (int64_t)(a.layer * Hkv + h) * 2;
      ic.k = base + hk * kv_elems * (int64_t)sizeof(TKV);
      ic.v = ic.k + kv_elems * (int64_t)sizeof(TKV);
      if constexpr (FP8) {
        const int nblk = (L + 15) >> 4;
        ic.ksc = reinterpret_cast<const float*>(base + (int64_t)2 * a.n_layers * Hkv * kv_elems) + hk * nblk;
        ic.vsc = ic.ksc + nblk;
      }
    }
  };
  auto issue_chunks = [&](auto own_c) __attribute__((always_inline)) {
    constexpr bool OWN = decltype(own_c)::value;
    constexpr int CH = OWN ? C::CHO : C::CHC;
    const int tl = ic.t < ic.n ? ic.t : ic.t % max(ic.n, 1);   // as in issue_rows
    const int* rws = ring + ic.slot * 64;
    uint8_t* sb = smem + ic.stage * C::STAGE;
    uint32_t off[C::NR];
#pragma unroll
    for (int j = 0; j < C::NR; j++) {
      const int rr = (256 * j + tid) / CH;         // key of the tile
      const int t = min(tl + rr, ic.n - 1);
      const int row = min(max(!OWN && ic.list ? rws[rr] : t, 0), ic.clampL - 1);
      off[j] = (uint32_t)row * (uint32_t)ic.pitch;
    }
#pragma unroll
    for (int v = 0; v < 2; v++)
#pragma unroll
      for (int j = 0; j < C::NR; j++) {
        const int rr = (256 * j + tid) / CH, slot = (256 * j + tid) % CH;
        const int sw = v ? (FP8 && !OWN ? swz_v8<CH>(rr) : swz_v<CH>(rr)) : swz_k<CH>(rr);
        const uint8_t* g = (v ? ic.v : ic.k) + (off[j] + (uint32_t)((slot ^ sw) * 16));
        uint8_t* l = sb + (v ? C::REGION : 0) + (256 * j + 64 * wave) * 16;
        load_to_lds<16>(g, l);
      }
    if constexpr (FP8) {
      float* meta = reinterpret_cast<float*>(sb + 2 * C::REGION);
      const void* g = dummy;
      if (!OWN && wave < 2) {
        const int row = min(max(ic.list ? rws[lane] : min(tl + lane, ic.n - 1), 0), ic.clampL - 1);
        g = (wave == 0 ? ic.ksc : ic.vsc) + (row >> 4);
      }
      load_to_lds<4>(static_cast<const uint8_t*>(g), meta + min(wave, 2) * 64);
    }
  };
  auto issue_tile = [&]() __attribute__((always_inline)) {
    if constexpr (FP8) {
      if (ic.s == 2) issue_chunks(std::true_type{});
      else issue_chunks(std::false_type{});
    } else {
      issue_chunks(std::false_type{});             // own rows have the cache's layout
    }
    ic.slot = ic.slot + 1 == C::NRING ? 0 : ic.slot + 1;
    ic.stage = ic.stage + 1 == NS ? 0 : ic.stage + 1;
    ic.t += step_of(ic.s);
    if (ic.t >= ic.np) {
      if (ic.s < 2) {
        enter_tiles(next_source(ic.s));
      } else {
        ic.t = 0;
        ic.n -= kOwnRows;
        ic.clampL = max(ic.n, 1);
        ic.k += (int64_t)kOwnRows * ic.pitch;
        ic.v += (int64_t)kOwnRows * ic.pitch;
      }
    }
  };

  // the tile being computed
  struct { int s, t, n, np, pos_add, top, slot, stage; bool list; } cc;
  auto enter_compute = [&](int s) {
    cc.s = s;
    cc.t = 0;
    cc.n = keys_of(s);
    cc.np = iterated(s);
    cc.list = list_of(s) != nullptr;
    cc.pos_add = s == 0 ? 0 : (s == 1 ? w_L_a : w_own_pos0);
    // no list row of a document lies past its length: whether a tile can hold an invisible key
    cc.top = (s == 0 ? w_L_a : w_L_b) - 1;
  };

  float m_run = -INFINITY, l_run = 0.f;
  f32x4 o[ND];
#pragma unroll
  for (int i = 0; i < ND; i++) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};

  vm_wait<0>();  // the query fragments have arrived (the loop's waits count tile loads only)
  __syncthreads();
  // Step j issues the row numbers of tile j + NS - 1 + LEAD, then the chunks of tile j + NS - 1;
  // the prologue runs steps -(NS - 1) .. -1.  The row numbers of a tile are older than the
  // chunks of the tile LEAD before it, so once tile ti has landed the row numbers that step ti
  // needs have too, while NS - 2 later tiles stay in flight.
  if (T > 0) {
    rc.slot = ic.slot = cc.slot = ic.stage = cc.stage = 0;
    enter_rows(first);
    enter_tiles(first);
    enter_compute(first);
    if constexpr (LISTS) {
#pragma unroll
      for (int q = 0; q < C::LEAD; q++) issue_rows();
      vm_wait<0>();
      __builtin_amdgcn_s_barrier();
    }
#pragma unroll
    for (int q = 0; q < NS - 1; q++) {
      issue_rows();
      if (q < T) issue_tile();
    }
  }
  constexpr int ROWS = LISTS ? NS - 2 : 0;         // row-number loads behind a tile

  // One online-softmax step over NB 16-key blocks from block kb0 of the tile at sb.
  auto compute = [&](const uint8_t* sb, auto own_c, auto nb_c, int kb0, bool need_mask) __attribute__((always_inline)) {
    constexpr bool T8 = FP8 && !decltype(own_c)::value;   // FP8 rows
    constexpr int NB = decltype(nb_c)::value;
    constexpr int RB = T8 ? C::RBC : C::RBO;
    const uint8_t* Kp = sb;
    const uint8_t* Vp = sb + C::REGION;
    const float* ksc_s = reinterpret_cast<const float*>(sb + 2 * C::REGION);
    const float* vsc_s = ksc_s + 64;
    // ---- scores S^T[key][query]: lane holds keys 16 (kb0 + b) + 4 g4 + t of query column qi
    f32x4 sc[NB];
#pragma unroll
    for (int b = 0; b < NB; b++) sc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < NB; b++) {
      const int kr = 16 * (kb0 + b) + qi;
#pragma unroll
      for (int k = 0; k < NQ; k++) {
        u32x4 kf;
        if constexpr (T8) {
          const int pc = 4 * k + g4;  // 8-byte piece of the FP8 row
          const u32x2 raw = *reinterpret_cast<const u32x2*>(Kp + kr * RB + ((pc >> 1) ^ swz_k<C::CHC>(kr)) * 16 +
                                                           (pc & 1) * 8);
          kf = fp8x8_to_bf16x8(raw[0], raw[1]);
        } else {
          kf = *reinterpret_cast<const u32x4*>(Kp + kr * RB + ((4 * k + g4) ^ swz_k<C::CHO>(kr)) * 16);
        }
        sc[b] = mfma_bf16(__builtin_bit_cast(u16x8, kf), __builtin_bit_cast(u16x8, qf[k]), sc[b]);
      }
    }
    // ---- online softmax (FP32).  Keys past the source's end and keys after the query's position
    // are masked; only tiles that can hold such keys test positions.
    if constexpr (T8) {
#pragma unroll
      for (int b = 0; b < NB; b++) sc[b] *= *reinterpret_cast<const f32x4*>(ksc_s + 16 * (kb0 + b) + 4 * g4);
    }
    if (need_mask) {
      const int n_here = cc.n - cc.t;
      const int* rows_s = ring + cc.slot * 64;
#pragma unroll
      for (int b = 0; b < NB; b++) {
        const int key = 16 * (kb0 + b) + 4 * g4;
        int kp[4] = {cc.t + key, cc.t + key + 1, cc.t + key + 2, cc.t + key + 3};
        if (LISTS && cc.list) {
          const u32x4 rw = *reinterpret_cast<const u32x4*>(rows_s + key);
#pragma unroll
          for (int t = 0; t < 4; t++) kp[t] = (int)rw[t];
        }
#pragma unroll
        for (int t = 0; t < 4; t++)
          if (!(key + t < n_here && kp[t] + cc.pos_add <= qpos)) sc[b][t] = -INFINITY;
      }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int b = 0; b < NB; b++)
#pragma unroll
      for (int t = 0; t < 4; t++) mx = fmaxf(mx, sc[b][t]);
    mx = max_over_groups(mx);
    const float c = a.scale_log2;
    const float m_new = fmaxf(m_run, mx);
    const float mc = m_new == -INFINITY ? 0.f : m_new * c;
    // rescale of the running sums: exactly 1 when the maximum did not move (the fused
    // m_run * c - mc is then the rounding error of mc, not 0), 0 when m_run = -inf.  The roundings
    // are spelled out: a tile's later steps subtract the rounded products.
    const bool moved = m_new > m_run;
    const float up = kb0 == 0 ? __builtin_fmaf(m_run, c, -mc) : scaled_minus(m_run, c, mc);
    const float alpha = moved ? __builtin_amdgcn_exp2f(up) : 1.f;
    float psum = 0.f;
#pragma unroll
    for (int b = 0; b < NB; b++)
#pragma unroll
      for (int t = 0; t < 4; t++) {
        const float pv = __builtin_amdgcn_exp2f(fmaf(sc[b][t], c, -mc));  // exp2(-inf) = 0
        sc[b][t] = pv;
        psum += pv;
      }
    l_run = l_run * alpha + psum;
    m_run = m_new;
    // (a product with exactly 1 changes nothing: skipped when no query's maximum moved, which
    // after the first tiles of a long document is the usual case)
    if (__any(moved)) {
#pragma unroll
      for (int i = 0; i < ND; i++) o[i] *= alpha;
    }

    // ---- O^T[d][query] += V^T[d][key] P^T[key][query].  K slots 0..3 of lane group g4 are
    // keys 32 b2 + 4 g4 + t, slots 4..7 keys 32 b2 + 16 + 4 g4 + t (b2: pair of the tile).
#pragma unroll
    for (int bp = 0; bp < NB / 2; bp++) {
      const int bl = 2 * bp, b2 = kb0 / 2 + bp;
      if constexpr (T8) {
        sc[bl] *= *reinterpret_cast<const f32x4*>(vsc_s + 32 * b2 + 4 * g4);
        sc[bl + 1] *= *reinterpret_cast<const f32x4*>(vsc_s + 32 * b2 + 16 + 4 * g4);
      }
      u32x4 pb;
#pragma unroll
      for (int t = 0; t < 4; t += 2) {
        pb[t / 2] = pack_bf16x2(sc[bl][t], sc[bl][t + 1]);
        pb[2 + t / 2] = pack_bf16x2(sc[bl + 1][t], sc[bl + 1][t + 1]);
      }
      if constexpr (T8) {
        // 8-bit transposed reads: within a lane group, lane qi addresses key slot qi / 2
        // (row 32 b2 + 4 g4 + (qi/2 < 4 ? qi/2 : 16 + qi/2 - 4)) at byte columns
        // 16 i + 8 (qi % 2) .. +7; lane qi receives byte column 16 i + qi of the 8 rows
        const int ks = qi >> 1;
        const int vr = 32 * b2 + 4 * g4 + (ks < 4 ? ks : 12 + ks);
        const int sv = swz_v8<C::CHC>(vr);
#pragma unroll
        for (int i0 = 0; i0 < ND; i0 += 4) {
          uint32_t ad[4];
          u32x2 y[4];
#pragma unroll
          for (int i = 0; i < 4; i++) ad[i] = lds_addr(Vp + vr * RB + (((i0 + i) ^ sv) * 16) + (qi & 1) * 8);
          ds_read_tr8_x4(ad, y);
#pragma unroll
          for (int i = 0; i < 4; i++) {
            const u32x4 va = fp8x8_to_bf16x8(y[i][0], y[i][1]);
            o[i0 + i] = mfma_bf16(__builtin_bit_cast(u16x8, va), __builtin_bit_cast(u16x8, pb), o[i0 + i]);
          }
        }
      } else {
        // 16-bit transposed reads: lane (qi, g4) addresses row 32 b2 + 4 g4 + qi / 4 and the row 16
        // after it (same swizzle), columns 16 i + 4 (qi % 4) .. +3; lane qi receives column
        // 16 i + qi of the 4 rows of its group
        const int vr = 32 * b2 + 4 * g4 + (qi >> 2);
        static_assert(swz_v<C::CHO>(16) == 0, "rows 16 apart share a swizzle");
#pragma unroll
        for (int i0 = 0; i0 < ND; i0 += 4) {
          uint32_t ad[4];
          u32x2 y[8];
#pragma unroll
          for (int i = 0; i < 4; i++) {
            const int cch = (16 * (i0 + i) + 4 * (qi & 3)) >> 3;
            ad[i] = lds_addr(Vp + vr * RB + (cch ^ swz_v<C::CHO>(vr)) * 16 + (qi & 1) * 8);
          }
          ds_read_tr16_x8<16 * RB>(ad, y);
#pragma unroll
          for (int i = 0; i < 4; i++) {
            const u32x4 va = u32x4{y[2 * i][0], y[2 * i][1], y[2 * i + 1][0], y[2 * i + 1][1]};
            o[i0 + i] = mfma_bf16(__builtin_bit_cast(u16x8, va), __builtin_bit_cast(u16x8, pb), o[i0 + i]);
          }
        }
      }
    }
  };

  for (int ti = 0; ti < T; ti++) {
    // Wait for tile ti: ROWS row-number loads and the tiles after ti (at most NS - 2) may be in
    // flight behind it.  Then a bare s_barrier makes every wavefront's loads visible and marks
    // tile ti - 1 consumed (a fence would wait for the loads still in flight).
    const int behind = T - 1 - ti;
    if (behind >= NS - 2) vm_wait<(NS - 2) * C::OPS + ROWS>();
    else vm_wait_behind<NS - 3, C::OPS, ROWS>(behind);
    __builtin_amdgcn_s_barrier();
    issue_rows();
    if (ti + NS - 1 < T) issue_tile();

    // document B is scored with the queries rotated at (position - L_A).  The wait belongs to
    // these loads alone: left to the compiler it would stand before the score products of every
    // tile, and wait there for the tiles in flight.
    if (TB > 0 && (ti == TA || ti == TA + TB)) {
      load_q(ti == TA ? q_rot : q_plain);
      vm_wait<0>();
    }
    if (wave_active) {
      const uint8_t* sb = smem + cc.stage * C::STAGE;
      const bool own = cc.s == 2;
      const int n_here = cc.n - cc.t;
      const int last = cc.list ? cc.top : min(cc.t + (own ? C::KTO : KT) - 1, own ? 0x7fffffff : cc.top);
      const bool need_mask = own || n_here < KT || last + cc.pos_add > w_q_pos0;
      if (FP8 && own) {
        constexpr int NB = C::KTO / 16 < KC / 16 ? C::KTO / 16 : KC / 16;
#pragma unroll
        for (int kb0 = 0; kb0 < C::KTO / 16; kb0 += NB)
          compute(sb, std::true_type{}, std::integral_constant<int, NB>{}, kb0, true);
      } else {
        // a tile may carry more keys than one step holds in registers
#pragma unroll 1
        for (int kb0 = 0; kb0 < KT / 16; kb0 += KC / 16)
          compute(sb, std::false_type{}, std::integral_constant<int, KC / 16>{}, kb0, need_mask);
      }
    }
    cc.slot = cc.slot + 1 == C::NRING ? 0 : cc.slot + 1;
    cc.stage = cc.stage + 1 == NS ? 0 : cc.stage + 1;
    cc.t += step_of(cc.s);
    if (cc.t >= cc.np && cc.s < 2) enter_compute(next_source(cc.s));
  }

  vm_wait<0>();  // row numbers fetched past the last tile have landed: nothing writes this LDS later

  // ---- normalise and store: lane holds O[query qi][d = 16 i + 4 g4 + t]
  float l_tot = l_run + __shfl_xor(l_run, 16, 64);
  l_tot += __shfl_xor(l_tot, 32, 64);
  __syncthreads();  // LDS reused by the workgroup's next unit
  if (!qvalid) return;
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  bf16_t* out = reinterpret_cast<bf16_t*>(a.out) + qrow * a.out_stride + hq * D;
#pragma unroll
  for (int i = 0; i < ND; i++) {
    const int d0 = 16 * i + 4 * g4;
    u32x2 pk;
    pk[0] = pack_bf16x2(o[i][0] * inv, o[i][1] * inv);
    pk[1] = pack_bf16x2(o[i][2] * inv, o[i][3] * inv);
    *reinterpret_cast<u32x2*>(out + d0) = pk;
  }
}

// One workgroup per unit.  32-key compute steps of a BF16 cache fit 128 VGPRs (four wavefronts per
// SIMD), which two stages use (34 KB of LDS: four workgroups per CU); an FP8 cache's widening
// takes 168 (three).  The register budget is capped to match.
template <typename TKV, int D, int KT, int NS, int KC, bool LISTS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(KC == 32 ? (NS == 2 ? 4 : NS == 3 ? 3 : 2) : 1)))
void attn_dma_kernel(AttnArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint8_t dma_smem[];
  attn_dma_unit<TKV, D, KT, NS, KC, LISTS>(a, blockIdx.x, dma_smem);
}

// Persistent form: a fixed grid takes units from a device counter (zeroed by the caller
// before the launch) until every unit is taken; every workgroup exits once the counter
// passes the unit count, so the grid always drains.
template <typename TKV, int D, int KT, int NS, int KC, bool LISTS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(KC == 32 ? (NS <= 3 ? 3 : 2) : 1)))
void attn_dma_persistent_kernel(AttnArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint8_t dma_smem[];
  __shared__ int next;
  const int total = a.n_work * a.Hkv;
  for (;;) {
    if (threadIdx.x == 0) next = atomicAdd(a.counter, 1);
    __syncthreads();
    const int unit = next;
    __syncthreads();
    if (unit >= total) break;
    attn_dma_unit<TKV, D, KT, NS, KC, LISTS>(a, unit, dma_smem);
  }
}

template <typename TKV, int D, int KT, int NS, int KC, bool LISTS>
static hipError_t launch_dma_t(const AttnArgs& a, hipStream_t st) {
  using C = DmaCfg<TKV, D, KT, NS>;
  const int64_t units = (int64_t)a.n_work * a.Hkv;
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)attn_dma_kernel<TKV, D, KT, NS, KC, LISTS>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_TOTAL);
    if (e == hipSuccess)
      e = hipFuncSetAttribute((const void*)attn_dma_persistent_kernel<TKV, D, KT, NS, KC, LISTS>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_TOTAL);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  if (a.counter) {
    // as many workgroups as are resident at once (registers and LDS decide: three per CU for
    // the 32-key compute steps); each takes units until the counter passes their number
    static int per_cu = 0;
    if (per_cu == 0) {
      hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &per_cu, (const void*)attn_dma_persistent_kernel<TKV, D, KT, NS, KC, LISTS>, 256, C::LDS_TOTAL);
      if (e != hipSuccess || per_cu < 1) per_cu = 2;
    }
    const int64_t wgs = (int64_t)per_cu * std::max(a.n_cu, 1);
    hipLaunchKernelGGL((attn_dma_persistent_kernel<TKV, D, KT, NS, KC, LISTS>),
                       dim3((unsigned)std::min<int64_t>(units, wgs)), dim3(256), C::LDS_TOTAL, st, a);
  } else {
    hipLaunchKernelGGL((attn_dma_kernel<TKV, D, KT, NS, KC, LISTS>), dim3((unsigned)units), dim3(256), C::LDS_TOTAL, st, a);
  }
  return hipGetLastError();
}

// prefill reads whole documents (no retained lists): its form has no row numbers to fetch
template <typename TKV, int D, int KT, int NS, int KC = KT>
static hipError_t launch_dma(const AttnArgs& a, hipStream_t st) {
  return a.idx ? launch_dma_t<TKV, D, KT, NS, KC, true>(a, st) : launch_dma_t<TKV, D, KT, NS, KC, false>(a, st);
}

// variant: 0 = KT 64 / 2 stages, 1 = KT 64 / 3 stages, 2 = 32-key compute steps over tiles of
// 16 KiB of keys and values: 32-key tiles of a BF16 cache, 64-key tiles of an FP8 cache (its
// rows are half as long, so the tile moves the same bytes), each computed in 32-key steps.
// The BF16 form runs two stages and four resident workgroups per CU (one tile in flight per
// workgroup, four per CU): a step's chain of dependent operations is then hidden by four
// wavefronts per SIMD instead of three, and HBM needs no more bytes in flight per CU than
// that; its persistent form keeps three stages (at four wavefronts per SIMD it would spill).
// The FP8 form needs more registers (three workgroups per CU whatever the stages) and keeps
// three stages.  The stage count changes no arithmetic: all forms of a variant agree bit
// for bit.  (D = 64 has no 32-key variant: its FP8 tile would be under one chunk load per
// thread.)
// Few documents of very different lengths: the launch ends with its longest unit, whose tiles are
// one chain (0.9 us each while its CU is quiet; one unit of 4096 keys 113 us), so two workgroups
// per CU with three tiles in flight serve it better than four with one.  192 documents of 16 to
// 3072 rows: 133 us against 156; 1024 of 16 to 4096 rows, bound by HBM: 772 against 765.  The line
// is where the chain takes half the time that the bytes take at 4.4 TB/s.
static bool longest_unit_bound(const AttnArgs& a, int D) {
  const double chain_us = a.longest_keys / 32.0 * 0.9;
  const double bytes_us = (double)a.total_keys * a.Hkv * D * 4.0 / 4.4e6;
  return 2.0 * chain_us > bytes_us;
}

int attention_dma_stages(int kvdt, int D, int variant, const AttnArgs& a) {
  if (variant == 0) return 2;
  if (variant == 1 || D == 64 || kvdt == DT_FP8 || a.counter) return 3;
  return longest_unit_bound(a, D) ? 4 : 2;
}

template <typename TKV, int D>
static hipError_t launch_dma_variant(int kvdt, int variant, const AttnArgs& a, hipStream_t st) {
  const int stages = attention_dma_stages(kvdt, D, variant, a);
  if (variant == 0) return launch_dma<TKV, D, 64, 2>(a, st);
  if constexpr (D == 64) return launch_dma<TKV, D, 64, 3>(a, st);
  else {
    if (variant == 1) return launch_dma<TKV, D, 64, 3>(a, st);
    if constexpr (sizeof(TKV) == 1) return launch_dma<TKV, D, 64, 3, 32>(a, st);
    else if (stages == 3) return launch_dma<TKV, D, 32, 3>(a, st);
    else if (stages == 4) return launch_dma<TKV, D, 32, 4>(a, st);
    else return launch_dma<TKV, D, 32, 2>(a, st);
  }
}

// The attention kernels' FP8 -> BF16 widening applied to a code array (n a multiple of 8),
// for an exhaustive check against the format's definition.
__global__ void fp8_widen_kernel(const uint8_t* __restrict__ codes, uint16_t* __restrict__ out, int n8) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n8) return;
  const u32x2 raw = *reinterpret_cast<const u32x2*>(codes + 8 * i);
  *reinterpret_cast<u32x4*>(out + 8 * i) = fp8x8_to_bf16x8(raw[0], raw[1]);
}

hipError_t fp8_widen(const uint8_t* codes, uint16_t* out, int n, hipStream_t st) {
  if (n <= 0 || n % 8) return hipErrorInvalidValue;
  const int n8 = n / 8;
  hipLaunchKernelGGL(fp8_widen_kernel, dim3((n8 + 255) / 256), dim3(256), 0, st, codes, out, n8);
  return hipGetLastError();
}

hipError_t attention_dma(int kvdt, int D, int variant, const AttnArgs& a, hipStream_t st) {
  if (a.n_work <= 0) return hipSuccess;
  if (a.counter && a.persistent_wgs < 1) return hipErrorInvalidValue;
  if (a.G * a.Pmax > 64 || a.G < 1 || a.Pmax < 1) return hipErrorInvalidValue;
  if (kvdt == DT_BF16) {
    if (D == 128) return launch_dma_variant<bf16_t, 128>(kvdt, variant, a, st);
    if (D == 64) return launch_dma_variant<bf16_t, 64>(kvdt, variant, a, st);
  } else if (kvdt == DT_FP8) {
    if (D == 128) return launch_dma_variant<fp8_t, 128>(kvdt, variant, a, st);
    if (D == 64) return launch_dma_variant<fp8_t, 64>(kvdt, variant, a, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace kvop
