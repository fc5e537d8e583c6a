// Attention over gathered cache rows, FP32 compute and FP32 caches.
//
// The work decomposition of the register-staged kernel in attention.hip: one workgroup of 4
// wavefronts per (work item, kv head), each wavefront 16 of its query rows; scores computed
// transposed, S^T = K Q^T, online softmax in FP32, O^T = V^T P^T, both products on
// v_mfma_f32_16x16x4f32.  Tiles of KT keys reach LDS by direct global -> LDS loads, NS - 1 of them
// in flight, as in attention_dma.hip.
//
// What bounds it: with 64 query rows the MFMAs (64 of 32 cycles per 16 keys of 128 columns and
// wavefront: 0.85 us), with one query row per head the bytes; one unit alone, its chain of steps
// (1.6 us each).  A long item is one such chain (4096 keys: 415 us; 700 with register-staged tiles
// of 32 keys and 4-byte reads of V), so where few items are long its keys go to several workgroups,
// kAttnChunkKeys to each, and a second launch puts their results together.  64 documents of 16 to
// 4096 rows, D = 128, 8 kv heads: 64 query rows 695 -> 206 us, 2 query rows 670 -> 144 us; 1024
// documents: 2800 -> 2040 and 2350 -> 1230 us.  That is for a call whose items share one suffix; mixed
// batches and a map's decoding steps bring no room for the states and run each unit whole.
//
// LDS layout of a tile part (K or V): FP32 rows, 16-byte chunk c of row r at slot c ^ swz(r), so
// that the 16 rows read at one chunk (K) lie on distinct banks.  Output column ND q + i is row q of
// the i-th product (ND = D / 16): a lane's ND values of a key are then contiguous, one or two
// 16-byte reads instead of ND 4-byte ones; at D = 128, of two, every other chunk of a row at a time,
// two to a bank (a third of the LDS cycles are conflicts, with the MFMAs 50 to 79% busy).
#include <algorithm>
#include <type_traits>

#include "direct_loads.h"
#include "common.h"
#include "kernels.h"

namespace kvop {

template <int D, int NS_>
struct F32Cfg {
  static constexpr int KT = attn_f32_tile(D);        // keys per tile
  static constexpr int NS = NS_;                     // stages (tiles resident in LDS)
  static constexpr int CH = D / 4;                   // 16-byte chunks per row
  static constexpr int RB = D * 4;                   // bytes per row
  static constexpr int REGION = KT * RB;             // bytes of the K (or V) part of a tile
  static constexpr int NR = REGION / 16 / 256;       // chunk loads per thread and part
  static_assert(NR >= 1 && REGION % 4096 == 0, "whole chunk loads per thread");
  static_assert(kOwnRows % KT == 0, "whole own tiles between moves of the base");
  static constexpr int STAGE = 2 * REGION;
  static constexpr int LEAD = NS - 1;                // row numbers are loaded LEAD tiles before their chunks
  static constexpr int NRING = NS + LEAD;
  static constexpr int RING = NS * STAGE;
  static constexpr int LDS = RING + NRING * 64 * 4;
  static constexpr int OPS = 2 * NR;                 // vector-memory operations of one tile
  static constexpr int CT = kAttnChunkKeys / KT;     // tiles per chunk
  // consecutive rows that share one 256-byte bank line differ in the low bits that are shifted out
  __device__ static constexpr int swz(int r) { return (r >> (CH >= 16 ? 0 : 1)) & (std::min(CH, 16) - 1); }
};

// The keys of an item are taken in chunks.  Each chunk has an online softmax of its own, and the
// chunks' maxima, sums and outputs are put together in order by this one step, whether one
// workgroup takes them all or one workgroup each: the split changes no bit.  (m, l, o) is the
// state so far, (mc, lc, oc) the next chunk's.  A state's probabilities are relative to its maximum's
// scaled and rounded value, so the factors are of the differences of those: taken of the exact
// products, the roundings of large maxima (half an ulp: 1e-3 at a maximum of 2^14) stayed in.
struct MergeFactors {
  float run, next;
};
__device__ inline MergeFactors merge_stats(float& m, float& l, float mc, float lc, float scale_log2) {
  const float mn = fmaxf(m, mc), mns = mn * scale_log2;
  MergeFactors f;
  f.run = m == mn ? 1.f : __builtin_amdgcn_exp2f(scaled_minus(m, scale_log2, mns));
  f.next = mc == mn ? 1.f : __builtin_amdgcn_exp2f(scaled_minus(mc, scale_log2, mns));
  l = __builtin_fmaf(lc, f.next, l * f.run);
  m = mn;
  return f;
}
__device__ inline float merge_out(float o, float oc, const MergeFactors& f) {
  return __builtin_fmaf(oc, f.next, o * f.run);
}

__device__ inline int item_tiles(const AttnWork* w, int kt) {
  return (w->n_a + kt - 1) / kt + (w->n_b + kt - 1) / kt + (w->n_own + kt - 1) / kt;
}

// One (work item, kv head) unit; SPLIT: one chunk of its keys, whose state goes to a.part unless
// the item has no other chunk.
template <int D, int NS, bool LISTS, bool SPLIT>
__device__ void attn_f32_unit(const AttnArgs& a, int unit, int chunk, uint8_t* smem) {
  using C = F32Cfg<D, NS>;
  constexpr int KT = C::KT, NB = KT / 16, NQ = D / 16, ND = D / 16, CH = C::CH;

  const int Hkv = a.Hkv;
  const int h = unit % Hkv;
  const AttnWork* wp = a.work + unit / Hkv;
  const int w_n_a = wp->n_a, w_n_b = wp->n_b, w_n_own = wp->n_own, w_n_q = wp->n_q;
  const int w_q_row0 = wp->q_row0, w_q_pos0 = wp->q_pos0, w_part0 = wp->part0;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qi = lane & 15, g4 = lane >> 4;
  const int r = wave * 16 + qi;
  const int gq = r / a.Pmax, p = r % a.Pmax;
  const bool qvalid = gq < a.G && p < w_n_q;
  const bool wave_active = __any(qvalid);
  const int hq = h * a.G + (gq < a.G ? gq : 0);
  const int qpos = w_q_pos0 + p;
  const int64_t qrow = (int64_t)w_q_row0 + (qvalid ? p : 0);

  // ---- sources (0 = document A, 1 = document B, 2 = own rows) and this workgroup's tiles
  const int TA = (w_n_a + KT - 1) / KT, TB = (w_n_b + KT - 1) / KT;
  const int T = TA + TB + (w_n_own + KT - 1) / KT;
  const int t0 = SPLIT ? chunk * C::CT : 0, t1 = SPLIT ? min(T, t0 + C::CT) : T;
  const bool whole = T <= C::CT;                     // one chunk: nothing to put together
  const int s0 = t0 < TA ? 0 : (t0 < TA + TB ? 1 : 2);
  const int k0 = (t0 - (s0 == 0 ? 0 : (s0 == 1 ? TA : TA + TB))) * KT;
  // What a source has is read from the item when a cursor enters it, into scalar registers there and
  // then: a choice between two captured locals becomes one between their addresses, a load from
  // scratch memory, and a vector load's wait would move to the value's first use in the loop and
  // stand there, at every tile, for the tiles in flight.
  auto val = [](int x) __attribute__((always_inline)) { return __builtin_amdgcn_readfirstlane(x); };
  auto val64 = [](int64_t x) __attribute__((always_inline)) {
    const int lo = __builtin_amdgcn_readfirstlane((int)x), hi = __builtin_amdgcn_readfirstlane((int)(x >> 32));
    return (int64_t)((uint64_t)(uint32_t)hi << 32 | (uint32_t)lo);
  };
  auto keys_of = [&](int s) __attribute__((always_inline)) {
    return val(s == 0 ? wp->n_a : (s == 1 ? wp->n_b : wp->n_own));
  };
  auto next_source = [&](int s) {
    do s++;
    while (s < 2 && keys_of(s) == 0);
    return s;
  };
  auto list_of = [&](int s) -> const int32_t* {
    const int64_t il = val64(s == 0 ? wp->idx_a : wp->idx_b);
    return LISTS && s < 2 && il >= 0 ? a.idx + il : nullptr;
  };
  const int32_t* dummy = reinterpret_cast<const int32_t*>(wp);   // for loads whose value is not used

  // ---- query fragments (B operand of S^T); document B's keys are scored with the queries rotated
  // at position - L_A
  u32x4 qf[NQ];
  const float* q_plain = reinterpret_cast<const float*>(a.q) + qrow * a.q_stride + hq * D;
  const float* q_rot = reinterpret_cast<const float*>(a.q_alt ? a.q_alt : a.q) + qrow * a.q_stride + hq * D;
  auto load_q = [&](const float* q) {
#pragma unroll
    for (int k = 0; k < NQ; k++)
      qf[k] = qvalid ? gload(reinterpret_cast<const u32x4*>(q + 16 * k + 4 * g4)) : u32x4{0, 0, 0, 0};
  };
  load_q(s0 == 1 ? q_rot : q_plain);

  // ---- three cursors walk the same sequence of tiles: the row numbers of retained lists being
  // fetched (LEAD tiles before the chunks that need them), the chunks being fetched, the tile
  // being computed
  int* ring = reinterpret_cast<int*>(smem + C::RING);
  struct { int s, t, n, slot; const int32_t* idx; } rc;
  auto enter_rows = [&](int s, int t) __attribute__((always_inline)) {
    rc.s = s;
    rc.t = t;
    rc.n = keys_of(s);
    rc.idx = list_of(s);
  };
  auto issue_rows = [&]() __attribute__((always_inline)) {
    if constexpr (LISTS) {
      // past the last tile the load goes on with row numbers that nobody reads
      const int32_t* g = rc.idx ? rc.idx + min(rc.t + lane, rc.n - 1) : dummy;
      load_to_lds<4>(g, ring + rc.slot * 64);
      rc.slot = rc.slot + 1 == C::NRING ? 0 : rc.slot + 1;
      rc.t += KT;
      if (rc.t >= rc.n && rc.s < 2) enter_rows(next_source(rc.s), 0);
    }
  };
  struct { int s, t, n, np, clampL, pitch, slot, stage; bool list; const uint8_t *k, *v; } ic;
  auto enter_tiles = [&](int s, int t) __attribute__((always_inline)) {
    ic.s = s;
    ic.t = t;
    ic.n = ic.np = keys_of(s);
    ic.list = list_of(s) != nullptr;
    ic.k = ic.v = a.pool;
    if (s == 2) {
      ic.t = 0;
      ic.n -= t;
      ic.np = kOwnRows;
      ic.clampL = max(ic.n, 1);
      ic.pitch = (int)a.own_stride * 4;
      const uint8_t* ob = reinterpret_cast<const uint8_t*>(a.own) + (int64_t)(val(wp->own_row0) + t) * a.own_stride * 4;
      ic.k = ob + (int64_t)(a.own_kcol + h * D) * 4;
      ic.v = ob + (int64_t)(a.own_vcol + h * D) * 4;
    } else if (ic.n > 0) {
      const int L = val(s == 0 ? wp->L_a : wp->L_b);
      ic.clampL = max(L, 1);
      ic.pitch = C::RB;
      const int64_t kv_bytes = (int64_t)L * C::RB;
      ic.k = a.pool + val64(s == 0 ? wp->off_a : wp->off_b) + (int64_t)(a.layer * Hkv + h) * 2 * kv_bytes;
      ic.v = ic.k + kv_bytes;
    }
  };
  auto issue_tile = [&]() __attribute__((always_inline)) {
    const int* rws = ring + ic.slot * 64;
    uint8_t* sb = smem + ic.stage * C::STAGE;
    uint32_t off[C::NR];
#pragma unroll
    for (int j = 0; j < C::NR; j++) {
      const int rr = (256 * j + tid) / CH, slot = (256 * j + tid) % CH;
      const int row = min(max(ic.list ? rws[rr] : min(ic.t + rr, ic.n - 1), 0), ic.clampL - 1);
      off[j] = (uint32_t)row * (uint32_t)ic.pitch + (uint32_t)((slot ^ C::swz(rr)) * 16);
    }
#pragma unroll
    for (int v = 0; v < 2; v++)
#pragma unroll
      for (int j = 0; j < C::NR; j++)
        load_to_lds<16>((v ? ic.v : ic.k) + off[j], sb + (v ? C::REGION : 0) + (256 * j + 64 * wave) * 16);
    ic.slot = ic.slot + 1 == C::NRING ? 0 : ic.slot + 1;
    ic.stage = ic.stage + 1 == NS ? 0 : ic.stage + 1;
    ic.t += KT;
    if (ic.t >= ic.np) {
      if (ic.s < 2) {
        enter_tiles(next_source(ic.s), 0);
      } else {
        ic.t = 0;
        ic.n -= kOwnRows;
        ic.clampL = max(ic.n, 1);
        ic.k += (int64_t)kOwnRows * ic.pitch;
        ic.v += (int64_t)kOwnRows * ic.pitch;
      }
    }
  };
  struct { int s, t, n, pos_add, top, slot, stage; bool list; } cc;
  auto enter_compute = [&](int s, int t) __attribute__((always_inline)) {
    cc.s = s;
    cc.t = t;
    cc.n = keys_of(s);
    cc.list = list_of(s) != nullptr;
    cc.pos_add = s == 0 ? 0 : val(s == 1 ? wp->L_a : wp->own_pos0);
    // no list row of a document lies past its length: whether a tile can hold an invisible key
    cc.top = val(s == 0 ? wp->L_a : wp->L_b) - 1;
  };

  float m_run = -INFINITY, l_run = 0.f;
  f32x4 o[ND];
#pragma unroll
  for (int i = 0; i < ND; i++) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  // state put together from the chunks before (all chunks by this workgroup)
  constexpr int NM = SPLIT ? 1 : ND;
  f32x4 om[NM];
  float m_all = -INFINITY, l_all = 0.f;
#pragma unroll
  for (int i = 0; i < NM; i++) om[i] = f32x4{0.f, 0.f, 0.f, 0.f};

  vm_wait<0>();  // the query fragments have arrived (the loop's waits count tile loads only)
  __syncthreads();
  if (t0 < t1) {
    rc.slot = ic.slot = cc.slot = ic.stage = cc.stage = 0;
    enter_rows(s0, k0);
    enter_tiles(s0, k0);
    enter_compute(s0, k0);
    if constexpr (LISTS) {
#pragma unroll
      for (int q = 0; q < C::LEAD; q++) issue_rows();
      vm_wait<0>();
      __builtin_amdgcn_s_barrier();
    }
#pragma unroll
    for (int q = 0; q < NS - 1; q++) {
      issue_rows();
      if (t0 + q < t1) issue_tile();
    }
  }
  constexpr int ROWS = LISTS ? NS - 2 : 0;         // row-number loads behind a tile

  for (int ti = t0; ti < t1; ti++) {
    // Wait for tile ti: ROWS row-number loads and the tiles after ti (at most NS - 2) may be in
    // flight behind it.  Then a bare s_barrier makes every wavefront's loads visible and marks
    // tile ti - 1 consumed (a fence would wait for the loads still in flight).
    const int behind = t1 - 1 - ti;
    if (behind >= NS - 2) vm_wait<(NS - 2) * C::OPS + ROWS>();
    else vm_wait_behind<NS - 3, C::OPS, ROWS>(behind);
    __builtin_amdgcn_s_barrier();
    issue_rows();
    if (ti + NS - 1 < t1) issue_tile();
    if (TB > 0 && ti > t0 && (ti == TA || ti == TA + TB)) {
      load_q(ti == TA ? q_rot : q_plain);
      vm_wait<0>();
    }
    if (wave_active) {
      const float* Kp = reinterpret_cast<const float*>(smem + cc.stage * C::STAGE);
      const float* Vp = Kp + KT * D;
      const int n_here = cc.n - cc.t;
      const bool own = cc.s == 2;
      const int last = cc.list ? cc.top : min(cc.t + KT - 1, own ? 0x7fffffff : cc.top);
      // ---- scores S^T[key][query]: lane holds keys 16 b + 4 g4 + t of query column qi
      f32x4 sc[NB];
#pragma unroll
      for (int b = 0; b < NB; b++) {
        sc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int kr = 16 * b + qi;
        f32x4 kf[NQ];
#pragma unroll
        for (int k = 0; k < NQ; k++)
          kf[k] = *reinterpret_cast<const f32x4*>(Kp + kr * D + ((4 * k + g4) ^ C::swz(kr)) * 4);
#pragma unroll
        for (int k = 0; k < NQ; k++)
#pragma unroll
          for (int t = 0; t < 4; t++) sc[b] = mfma_f32(kf[k][t], as_f32(qf[k][t]), sc[b]);
        // reads and products in groups (one read at a time, each with its wait, cost as much as the
        // products; more than four at once cost the registers of a resident workgroup)
        constexpr int RG = NQ < 4 ? NQ : 4;
#pragma unroll
        for (int k = 0; k < NQ / RG; k++) {
          __builtin_amdgcn_sched_group_barrier(0x100, RG, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 4 * RG, 0);
        }
      }
      // ---- online softmax on raw scores, the scale folded into the exponent.  Keys past the
      // source's end and keys after the query's position are masked; only tiles that can hold
      // such keys test positions.
      if (own || n_here < KT || last + cc.pos_add > w_q_pos0) {
        const int* rows_s = ring + cc.slot * 64;
#pragma unroll
        for (int b = 0; b < NB; b++) {
          const int key = 16 * b + 4 * g4;
#pragma unroll
          for (int t = 0; t < 4; t++) {
            const int kp = LISTS && cc.list ? rows_s[key + t] : cc.t + key + t;
            if (!(key + t < n_here && kp + cc.pos_add <= qpos)) sc[b][t] = -INFINITY;
          }
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
      // exactly 1 when the maximum did not move, 0 when m_run = -inf
      const bool moved = m_new > m_run;
      const float alpha = moved ? __builtin_amdgcn_exp2f(scaled_minus(m_run, c, mc)) : 1.f;
      float psum = 0.f;
#pragma unroll
      for (int b = 0; b < NB; b++)
#pragma unroll
        for (int t = 0; t < 4; t++) {
          const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[b][t], c, -mc));  // exp2(-inf) = 0
          sc[b][t] = pv;
          psum += pv;
        }
      l_run = __builtin_fmaf(l_run, alpha, psum);
      m_run = m_new;
      if (__any(moved)) {
#pragma unroll
        for (int i = 0; i < ND; i++) o[i] *= alpha;
      }
      // ---- O^T[d][query] += V^T[d][key] P^T[key][query]
#pragma unroll
      for (int b = 0; b < NB; b++) {
        float vb[4][ND];
#pragma unroll
        for (int t = 0; t < 4; t++) {
          const int vr = 16 * b + 4 * g4 + t;
          const float* vp = Vp + vr * D;
          float (&v)[ND] = vb[t];
          if constexpr (ND == 2) {
            const u32x2 x = *reinterpret_cast<const u32x2*>(vp + (((qi >> 1) ^ C::swz(vr)) * 4) + (qi & 1) * 2);
            v[0] = as_f32(x[0]);
            v[1] = as_f32(x[1]);
          } else {
#pragma unroll
            for (int j = 0; j < ND / 4; j++) {
              const f32x4 x = *reinterpret_cast<const f32x4*>(vp + ((ND / 4 * qi + j) ^ C::swz(vr)) * 4);
#pragma unroll
              for (int e = 0; e < 4; e++) v[4 * j + e] = x[e];
            }
          }
        }
#pragma unroll
        for (int t = 0; t < 4; t++)
#pragma unroll
          for (int i = 0; i < ND; i++) o[i] = mfma_f32(vb[t][i], sc[b][t], o[i]);
#pragma unroll
        for (int g = 0; g < (ND > 4 ? 2 : 1); g++) {
          __builtin_amdgcn_sched_group_barrier(0x100, 4, 1);
          __builtin_amdgcn_sched_group_barrier(0x008, ND > 4 ? 2 * ND : 4 * ND, 1);
        }
      }
      if constexpr (!SPLIT) {
        if (!whole && ((ti + 1) % C::CT == 0 || ti + 1 == T)) {
          float l_chunk = l_run + __shfl_xor(l_run, 16, 64);
          l_chunk += __shfl_xor(l_chunk, 32, 64);
          if (ti < C::CT) {
            m_all = m_run;
            l_all = l_chunk;
#pragma unroll
            for (int i = 0; i < ND; i++) om[i] = o[i];
          } else {
            const MergeFactors f = merge_stats(m_all, l_all, m_run, l_chunk, c);
#pragma unroll
            for (int i = 0; i < ND; i++)
#pragma unroll
              for (int t = 0; t < 4; t++) om[i][t] = merge_out(om[i][t], o[i][t], f);
          }
          m_run = -INFINITY;
          l_run = 0.f;
#pragma unroll
          for (int i = 0; i < ND; i++) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
    }
    cc.slot = cc.slot + 1 == C::NRING ? 0 : cc.slot + 1;
    cc.stage = cc.stage + 1 == NS ? 0 : cc.stage + 1;
    cc.t += KT;
    if (cc.t >= cc.n && cc.s < 2) enter_compute(next_source(cc.s), 0);
  }

  vm_wait<0>();  // row numbers fetched past the last tile have landed: nothing writes this LDS later

  // ---- store: lane holds O[query qi][d = ND (4 g4 + t) + i]
  float l_tot = l_run + __shfl_xor(l_run, 16, 64);
  l_tot += __shfl_xor(l_tot, 32, 64);
  if constexpr (!SPLIT) {
    if (!whole) {
      l_tot = l_all;
#pragma unroll
      for (int i = 0; i < ND; i++) o[i] = om[i];
    }
  }
  __syncthreads();  // LDS reused by the workgroup's next unit
  if (!qvalid) return;
  float* out = reinterpret_cast<float*>(a.out) + qrow * a.out_stride + hq * D;
  float scale = l_tot > 0.f ? 1.f / l_tot : 0.f;
  if (SPLIT && !whole) {
    const int R = a.G * a.Pmax;
    const int64_t row = ((int64_t)(w_part0 + chunk) * Hkv + h) * R + r;
    out = a.part + row * D;
    scale = 1.f;
    if (g4 == 0) {
      float* ml = a.part + (int64_t)a.n_part * Hkv * R * D + 2 * row;
      ml[0] = m_run;
      ml[1] = l_tot;
    }
  }
#pragma unroll
  for (int t = 0; t < 4; t++) {
    float* od = out + ND * (4 * g4 + t);
    if constexpr (ND == 2) {
      od[0] = o[0][t] * scale;
      od[1] = o[1][t] * scale;
    } else {
#pragma unroll
      for (int i = 0; i < ND; i += 4)
        *reinterpret_cast<f32x4*>(od + i) = f32x4{o[i][t], o[i + 1][t], o[i + 2][t], o[i + 3][t]} * scale;
    }
  }
}

// One workgroup per unit, or (SPLIT) per chunk of a unit: chunks that an item does not have end at
// once.  A chunk takes 128 VGPRs and two stages (33 KB), four workgroups per CU; a whole unit keeps
// a second set of outputs, 166 VGPRs, three workgroups per CU, and three stages.
template <int D, int NS, bool LISTS, bool SPLIT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(SPLIT ? 4 : 2))) void attn_f32_kernel(AttnArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint8_t f32_smem[];
  if constexpr (SPLIT) {
    using C = F32Cfg<D, NS>;
    const int units = a.n_work * a.Hkv;
    const int chunk = (int)(blockIdx.x / (unsigned)units), unit = (int)(blockIdx.x % (unsigned)units);
    if (chunk > 0 && chunk * C::CT >= item_tiles(a.work + unit / a.Hkv, C::KT)) return;
    attn_f32_unit<D, NS, LISTS, true>(a, unit, chunk, f32_smem);
  } else {
    attn_f32_unit<D, NS, LISTS, false>(a, blockIdx.x, 0, f32_smem);
  }
}

// Persistent form: a fixed grid takes units from a device counter (zeroed by the caller before the
// launch) until every unit is taken; every workgroup exits once the counter passes the unit
// count, so the grid always drains.
template <int D, int NS, bool LISTS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void attn_f32_persistent_kernel(AttnArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint8_t f32_smem[];
  __shared__ int next;
  const int total = a.n_work * a.Hkv;
  for (;;) {
    if (threadIdx.x == 0) next = atomicAdd(a.counter, 1);
    __syncthreads();
    const int unit = next;
    __syncthreads();
    if (unit >= total) break;
    attn_f32_unit<D, NS, LISTS, false>(a, unit, 0, f32_smem);
  }
}

// The chunks of the items that have several, put together: workgroups per unit and part of its
// rows, a thread per four columns of a row.  Four chunks are loaded at a time.
template <int D>
__global__ __launch_bounds__(256) void attn_f32_merge_kernel(AttnArgs a) {
  constexpr int KT = attn_f32_tile(D);
  const int unit = blockIdx.x, h = unit % a.Hkv;
  const AttnWork* w = a.work + unit / a.Hkv;
  const int nch = (item_tiles(w, KT) + kAttnChunkKeys / KT - 1) / (kAttnChunkKeys / KT);
  if (nch <= 1) return;
  const int R = a.G * a.Pmax;
  const int64_t step = (int64_t)a.Hkv * R, row0 = ((int64_t)w->part0 * a.Hkv + h) * R;
  const float* ml = a.part + (int64_t)a.n_part * a.Hkv * R * D;
  for (int i = blockIdx.y * 256 + threadIdx.x; i < R * (D / 4); i += gridDim.y * 256) {
    const int r = i / (D / 4), d = (i % (D / 4)) * 4;
    const int gq = r / a.Pmax, p = r % a.Pmax;
    if (p >= w->n_q) continue;
    const float* po = a.part + (row0 + r) * D + d;
    const float* pm = ml + 2 * (row0 + r);
    f32x4 o = *reinterpret_cast<const f32x4*>(po);
    float m = pm[0], l = pm[1];
    for (int c0 = 1; c0 < nch; c0 += 4) {
      f32x4 oc[4];
      float mc[4], lc[4];
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const int64_t c = min(c0 + j, nch - 1);
        oc[j] = *reinterpret_cast<const f32x4*>(po + c * step * D);
        mc[j] = pm[2 * c * step];
        lc[j] = pm[2 * c * step + 1];
      }
#pragma unroll
      for (int j = 0; j < 4; j++)
        if (c0 + j < nch) {
          const MergeFactors f = merge_stats(m, l, mc[j], lc[j], a.scale_log2);
#pragma unroll
          for (int t = 0; t < 4; t++) o[t] = merge_out(o[t], oc[j][t], f);
        }
    }
    const float inv = l > 0.f ? 1.f / l : 0.f;
    float* out = reinterpret_cast<float*>(a.out) + (int64_t)(w->q_row0 + p) * a.out_stride + (h * a.G + gq) * D + d;
    *reinterpret_cast<f32x4*>(out) = o * inv;
  }
}

// The chunks of long items go to workgroups of their own where the longest item's chain of tiles
// (1.6 us per 16 keys of 128 columns) takes longer than all keys and values at the rate that many
// units reach (3.3 TB/s with more than one block of 16 query rows, 4.9 with one).  D = 128, 8 kv
// heads, 64 query rows: 64 documents of 16 to 4096 rows 441 us whole, 206 split; 192 of 16 to 3072
// 423 and 366; 1024 of 16 to 4096, where the chunks' states only add traffic, 2040 and 2234.
bool attention_f32_splits(int D, const AttnArgs& a) {
  const double chain_us = a.longest_keys / 16.0 * 1.6 * D / 128.0;
  const double bytes_us = (double)a.total_keys * a.Hkv * D * 8.0 / (a.G * a.Pmax > 16 ? 3.3e6 : 4.9e6);
  return a.longest_keys > kAttnChunkKeys && chain_us > bytes_us;
}

template <int D, bool LISTS>
static hipError_t allow_lds() {
  hipError_t e = hipFuncSetAttribute((const void*)attn_f32_kernel<D, 3, LISTS, false>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, F32Cfg<D, 3>::LDS);
  if (e == hipSuccess)
    e = hipFuncSetAttribute((const void*)attn_f32_persistent_kernel<D, 3, LISTS>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, F32Cfg<D, 3>::LDS);
  if (e == hipSuccess)
    e = hipFuncSetAttribute((const void*)attn_f32_kernel<D, 2, LISTS, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            F32Cfg<D, 2>::LDS);
  return e;
}

template <int D, bool LISTS>
static hipError_t launch_f32(const AttnArgs& a, hipStream_t st) {
  const int64_t units = (int64_t)a.n_work * a.Hkv;
  constexpr int lds = F32Cfg<D, 3>::LDS;
  static const hipError_t attr = allow_lds<D, LISTS>();
  if (attr != hipSuccess) return attr;
  if (a.counter) {
    hipLaunchKernelGGL((attn_f32_persistent_kernel<D, 3, LISTS>),
                       dim3((unsigned)std::min<int64_t>(units, a.persistent_wgs)), dim3(256), lds, st, a);
    return hipGetLastError();
  }
  // a last, partial tile from each of the three sources
  using C = F32Cfg<D, 2>;
  const int64_t chunks = (a.longest_keys / C::KT + 3 + C::CT - 1) / C::CT;
  if (a.part && units * chunks <= INT32_MAX) {
    hipLaunchKernelGGL((attn_f32_kernel<D, 2, LISTS, true>), dim3((unsigned)(units * chunks)), dim3(256), C::LDS, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int per_unit = std::max(1, a.G * a.Pmax * (D / 4) / 512);
    hipLaunchKernelGGL((attn_f32_merge_kernel<D>), dim3((unsigned)units, per_unit), dim3(256), 0, st, a);
  } else {
    hipLaunchKernelGGL((attn_f32_kernel<D, 3, LISTS, false>), dim3((unsigned)units), dim3(256), lds, st, a);
  }
  return hipGetLastError();
}

template <int D>
static hipError_t launch_f32_d(const AttnArgs& a, hipStream_t st) {
  return a.idx ? launch_f32<D, true>(a, st) : launch_f32<D, false>(a, st);
}

hipError_t attention_f32(int D, const AttnArgs& a, hipStream_t st) {
  switch (D) {
    case 32: return launch_f32_d<32>(a, st);
    case 64: return launch_f32_d<64>(a, st);
    case 128: return launch_f32_d<128>(a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace kvop
