// Exact-token routed attention, forward (Sec. 2.1 item 3).
//
// One workgroup per (query block, kv head, slice of GW query heads). Each of
// its 2*GW waves owns 32 queries of one query head. The routed key set
// [sink | local | selected groups] is gathered 64 tokens at a time into LDS,
// double-buffered: the next tile's global loads are in flight while the
// matrix cores work on the current one. K and V stay row-major in LDS; the V
// operand of P.V is read with the LDS transpose load (fp32 inputs, which have
// no such load, stage V transposed instead).
//
// Per tile and wave, on 32x32 MFMA tiles:
//   S^T = K . Q^T      (A = K rows from LDS, B = the wave's Q held in registers)
//   online softmax     (every lane holds scores of a single query, so the
//                       running max / sum are per lane plus one cross-half swap)
//   O^T += V^T . P^T   (A = transposed V from LDS, B = P straight from the
//                       S^T accumulators, rounded to the input precision)
// Scores are kept raw; p = exp2(s*c - m*c) with c = softmax_scale*log2(e) is one
// FMA and one v_exp_f32. The running max m is raised lazily: only when a row's
// new maximum exceeds it by more than 2^8 (in exp2 units) are O and the sum
// rescaled, so p stays below 2^8 and most tiles skip the rescale entirely.
#include "route_device.h"
#include "routed_tile.h"

namespace hga {

// The attention of one workgroup: (query block wc.b, kv head wc.h, query heads
// wc.hs * GW ...), on 2 * GW waves whose thread ids are `tid` (0 .. 128 GW).
// Window tiles (sink and local, known without the routing) come first and
// their gathers go out with the query rows. The selected groups follow:
//  - LATE == false: `routed(rs)` completes rs from the routing row once the
//    window gathers are out; `sync` then makes its LDS writes visible. Two
//    register slots alternate: while tile t is computed, tile t+1 waits in
//    one and tile t+2 is in flight in the other.
//  - LATE == true: the routing is computed by other waves of the workgroup
//    while these attend the window tiles. `ready()` polls whether it has
//    landed (each wave on its own); the gathers of selected groups go out as
//    soon as a wave sees it, and a wave waits for it only when it has no
//    window tile left to compute. Two register slots (the routing waves
//    share the SIMDs' registers).
// Every slot is named statically at each gather and each use (the loop is
// unrolled over the slot rotation), so the compiler waits for exactly the
// gather a use needs and the later ones stay in flight.
// PREC (bf16 only, chosen when the caller asks for the float32 copy of O):
// P enters P.V as a bf16 hi + lo pair, so that copy is accurate to ~2^-17
// relative and the backward's row term D = rowsum(dO * O) is exact enough.
template <typename T, int D, int GW, bool PREC, bool LATE, bool CMP, typename Sync, typename Ready, typename Routed>
__device__ __forceinline__ void attend_block(const AttnArgs& a, const WgCoord wc, char* smem, const int* sel_lds,
                                             const int tid, Sync& sync, Ready&& ready, Routed&& routed) {
  using EL = Elem<T>;
  using Frag = typename EL::Frag;
  using TL = Tile<T, D>;
  // padding keys are masked to -inf below, so their rows need no zeroing
  using KV = KVRegs<T, D, 128 * GW, false>;
  constexpr int E = EL::E, KS = EL::KSTEP, EB = EL::kBytes;
  constexpr int NKS = D / KS;   // MFMAs over the head dim per S tile
  constexpr int NDT = D / 32;   // 32-wide head-dim tiles of O^T
  constexpr int VPS = 16 / E;  // P.V k-steps per 32-key half tile
  constexpr bool TR = EB == 2;  // V operand through the LDS transpose load
  constexpr int STAGE = TL::kRowBytes + (TR ? TL::kRowBytes : TL::kTBytes);

  const int lane = tid & 63, wave = tid >> 6;
  const int hh = lane >> 5, l32 = lane & 31;
  const int hq = wc.h * a.gqa + wc.hs * GW + (wave >> 1);
  const int qoff = (wave & 1) * 32 + l32;  // query offset inside the block
  const int row = wc.b * 64 + qoff;

  const char* Qb = static_cast<const char*>(a.Q);
  const char* Kb = static_cast<const char*>(a.K);
  const char* Vb = static_cast<const char*>(a.V);
  const int64_t k_head_b = (int64_t)wc.h * a.k_head * EB, v_head_b = (int64_t)wc.h * a.v_head * EB;

  // The wave's 32 query rows: bf16 goes through the wave's share of the stages
  // before the first tile does (131,072 queries: 1,612 us with direct loads,
  // 1,579 so). float32 rows would not fit, and with LATE the barrier that this
  // takes costs what it gains: there the fragments are loaded directly.
  constexpr bool QL = EB == 2 && !LATE;
  Frag qf[NKS];
  RowFrags<T, D> qrows;
  {
    const char* q0 = Qb + (((int64_t)wc.b * 64 + (wave & 1) * 32) * a.q_tok + (int64_t)hq * a.q_head) * EB;
    if constexpr (QL) {
      static_assert(2 * GW * RowFrags<T, D>::kBytes <= 2 * STAGE, "the waves' rows fit the stages");
      qrows.load(q0, a.q_tok * EB, lane);
    } else {
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) qf[ks] = EL::load_frag(q0 + l32 * a.q_tok * EB + (ks * KS + E * hh) * EB);
    }
  }
  auto take_queries = [&] {
    if constexpr (QL) qrows.fragments(smem + wave * RowFrags<T, D>::kBytes, lane, qf);
  };
  // CMP: K and V are the compact copies of hga_gather_routed, rows of this
  // (block, kv head)'s routed set in tile order, padding rows zero
  const int64_t cslot = CMP ? ((int64_t)wc.b * a.n_kv_heads + wc.h) * a.r_cap * D * EB : 0;
  const char* kb = CMP ? Kb + cslot : Kb + k_head_b;
  const char* vb = CMP ? Vb + cslot : Vb + v_head_b;
  const int64_t ktb = CMP ? D * EB : a.k_tok * EB, vtb = CMP ? D * EB : a.v_tok * EB;

  // The query fragments are waited for here, before the tile loop: a first
  // use inside the loop would leave their wait in every iteration, where it
  // also waits for every gather issued after them.
  auto settle = [](Frag (&f)[NKS]) {
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) asm volatile("" : "+v"(f[ks]));
  };
  RoutedSet rs = window_set(a, wc.b, sel_lds);
  const int nwt = rs.nw >> 6;  // window tiles (>= 1: the diagonal block)
  int ntl = nwt;               // tiles known so far
  bool have = false;           // routing known to this wave
  // gather of tile x into slot r: a window tile before the routing is
  // known, any tile after (rs.token covers both)
  auto gather_w = [&](KV& r, int x) {
    r.load_contiguous(kb, ktb, vb, vtb, CMP ? (int64_t)64 * x : rs.window_first(x), tid);
  };
  auto gather = [&](KV& r, int x) {
    if constexpr (CMP) r.load_contiguous(kb, ktb, vb, vtb, (int64_t)64 * x, tid);
    else if (64 * x < rs.nw) r.load_contiguous(kb, ktb, vb, vtb, rs.window_first(x), tid);
    else r.load_groups(kb, ktb, vb, vtb, rs, x, tid);
  };
  auto take_routing = [&] {
    routed(rs);
    have = true;
    ntl = (rs.R + 63) >> 6;
  };
  auto put = [&](const KV& r, char* dst) {
    r.store_rows(dst, false, tid);
    if constexpr (TR) r.store_rows(dst + TL::kRowBytes, true, tid);
    else r.store_transposed(dst + TL::kRowBytes, true, tid);
  };

  f32x16 oacc[NDT];
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt) oacc[dt] = f32x16{};
  float m_run = -__builtin_inff(), l_run = 0.0f;
  const float c = a.scale_log2;
  const float lazy = 8.0f / c;  // raise the max only when it grows by > 2^8 in exp2 units

  // One 64-key tile from LDS stage `st` into the running softmax and O, as
  // two 32-key halves, each an online-softmax step of its own: the second
  // half's S products and the first half's P.V products overlap the other
  // half's max and exponentials.
  auto compute = [&](int tile, const char* st) __attribute__((always_inline)) {
    // S^T = K . Q^T : two 32-key tiles, raw scores
    f32x16 sacc[2] = {f32x16{}, f32x16{}};
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        const Frag kf = EL::load_frag(st + TL::row_off(32 * t + l32, ks * KS + E * hh));
        sacc[t] = EL::mma(kf, qf[ks], sacc[t]);
      }
    }
    // the same for every lane of the wave; read as a scalar so the masked
    // path is a branch, not a select over every tile
    const bool need_mask = __builtin_amdgcn_readfirstlane((int)rs.tile_needs_mask(tile * 64, (wave & 1) * 32)) != 0;
    if (need_mask) {  // both halves under one branch: under two, the second became selects in every tile
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int p = tile * 64 + 32 * t + 8 * (v >> 2) + 4 * hh + (v & 3);
          if (rs.masked(p, qoff)) sacc[t][v] = -__builtin_inff();
        }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      float mx = -__builtin_inff();
#pragma unroll
      for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sacc[t][v]);
      mx = half_max(mx);
      const bool raise = mx > m_run + lazy;  // also true on the first half-tile (m_run = -inf)
      if (__any(raise)) {
        const float m_new = raise ? mx : m_run;
        const float corr = __builtin_amdgcn_exp2f((m_run - m_new) * c);
        m_run = m_new;
        l_run *= corr;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) oacc[dt] *= corr;
      }
      const float mc = m_run * c;
      float psum = 0.0f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float p = __builtin_amdgcn_exp2f(fmaf(sacc[t][v], c, -mc));
        sacc[t][v] = p;
        psum += p;
      }
      l_run += psum;
      // O^T += V^T . P^T over this half's keys
#pragma unroll
      for (int s2 = 0; s2 < VPS; ++s2) {
        const int s = t * VPS + s2;
        float pv[E], plo[E];
#pragma unroll
        for (int j = 0; j < E; ++j) {
          pv[j] = sacc[t][E * s2 + j];
          if constexpr (PREC) plo[j] = pv[j] - bf16_bits_to_float(float_to_bf16_bits(pv[j]));
        }
        const Frag pf = EL::frag_from(pv);
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
          Frag vf;
          if constexpr (TR) vf = tr_frag<TL>(st + TL::kRowBytes, 32 * dt, 16 * s + 4 * hh, 16 * s + 8 + 4 * hh, lane);
          else vf = EL::load_frag(st + TL::kRowBytes + TL::t_off(32 * dt + l32, KS * s + E * hh));
          oacc[dt] = EL::mma(vf, pf, oacc[dt]);
          if constexpr (PREC) oacc[dt] = EL::mma(vf, EL::frag_from(plo), oacc[dt]);
        }
      }
    }
  };

  if constexpr (!LATE) {
    // Tile x lives in kv0 for even x, kv1 for odd x; its LDS stage is x & 1.
    KV kv0, kv1;
    gather_w(kv0, 0);  // always a window tile
    if (nwt > 1) gather_w(kv1, 1);
    take_routing();
    take_queries();
    sync();  // the routing row's LDS copy is there, the waves' query rows have been read
    const int last = ntl - 1;
    if (nwt <= 1) gather(kv1, min(1, last));
    put(kv0, smem);
    gather(kv0, min(2, last));
    settle(qf);
    sync();
    // Two tiles per round, so that each slot and stage is named statically. A
    // slot chosen at run time (three of them, before) made the compiler load
    // into the free S registers, wait, and copy: every tile then waited for
    // the gather that it had just sent. Refills are unconditional, on tile
    // indices clamped to the last (loaded again and not used).
    // The loop leaves no round half done: an exit between the refills would
    // make every store wait for both slots.
    int tile = 0;
#pragma unroll 1
    for (; tile + 2 <= last; tile += 2) {
      compute(tile, smem);
      put(kv1, smem + STAGE);
      gather(kv1, min(tile + 3, last));
      sync();
      compute(tile + 1, smem + STAGE);
      put(kv0, smem);
      gather(kv0, min(tile + 4, last));
      sync();
    }
    compute(tile, smem);
    if (tile < last) {
      put(kv1, smem + STAGE);
      sync();
      compute(tile + 1, smem + STAGE);
    }
    sync();  // the last tile's stage is no longer read
  } else {
    // Slots A, B: tile x lives in kv0 for even x, kv1 for odd x. nl is the
    // next tile to gather; a selected-group tile whose routing this wave has
    // not seen yet waits in nl.
    KV kv0, kv1;
    gather_w(kv0, 0);
    int nl = 1;
    if (nwt > 1) { gather_w(kv1, 1); nl = 2; }
    // next tile x (nl == x) into slot r, if it is known or the routing has
    // landed meanwhile
    auto try_gather = [&](KV& r, int x) {
      if (nl != x) return;
      if (!have && x >= ntl && ready()) take_routing();
      if (x < ntl) { gather(r, x); ++nl; }
    };
    put(kv0, smem);
    try_gather(kv0, 2);
    settle(qf);
    sync();
    // iteration t: compute tile t; tile t+1 (slot A) to LDS; gathers of
    // t+2 (slot B, free since tile t went to LDS) and t+3 (slot A)
    auto iter = [&](int t, KV& A, KV& B) -> bool {
      compute(t, smem + (t & 1) * STAGE);
      if (t + 1 >= ntl) {
        if (have) return false;
        while (!ready()) __builtin_amdgcn_s_sleep(2);
        take_routing();
        if (t + 1 >= ntl) return false;
      }
      if (nl == t + 1) { gather(A, t + 1); ++nl; }  // a selected-group tile not gathered yet
      put(A, smem + ((t + 1) & 1) * STAGE);
      try_gather(B, t + 2);
      try_gather(A, t + 3);
      sync();
      return true;
    };
    for (int tile = 0;; tile += 2) {
      if (!iter(tile, kv1, kv0)) break;
      if (!iter(tile + 1, kv0, kv1)) break;
    }
  }

  // Epilogue: O = O^T / l, LSE = (m + log2 l) * ln 2. A lane holds half the
  // head dim of one query row, so storing from registers would scatter every
  // store instruction over 32 rows; each wave's 32 rows go through its share
  // of LDS instead (the stages are free now), as output elements, and leave
  // as 16-byte pieces with consecutive lanes on consecutive pieces of a row.
  // No barrier: a wave reads only its own rows.
  if constexpr (LATE) sync();  // the last tile's stage is no longer read
  const float l = half_sum(l_run);
  const float inv = 1.0f / l;
  if (hh == 0) a.lse[(int64_t)row * a.n_q_heads + hq] = (m_run * c + __log2f(l)) * kLn2;
  constexpr int OP = EB == 2 ? D * 2 + 16 : D * 4;  // byte pitch of a staged row
  constexpr int WB = 2 * STAGE / (2 * GW) / 16 * 16;  // a wave's share
  static_assert(32 * OP <= WB, "a wave's rows fit its share");
  char* ost = smem + wave * WB;
  const int64_t row0 = (int64_t)wc.b * 64 + (wave & 1) * 32;  // the wave's first row
  // the wave's staged rows to rows `stride` bytes apart
  auto drain = [&](char* dst, int64_t stride) __attribute__((always_inline)) {
    constexpr int CPR = (EB == 2 ? D * 2 : D * 4) / 16;
#pragma unroll
    for (int it = 0; it < 32 * CPR / 64; ++it) {
      const int cc = (lane + 64 * it) % CPR, r = (lane + 64 * it) / CPR;
      *reinterpret_cast<u32x4*>(dst + r * stride + cc * 16) = *reinterpret_cast<const u32x4*>(ost + r * OP + cc * 16);
    }
  };
  auto scaled = [&](int dt, int v4) __attribute__((always_inline)) {
    return f32x4{oacc[dt][4 * v4] * inv, oacc[dt][4 * v4 + 1] * inv, oacc[dt][4 * v4 + 2] * inv,
                 oacc[dt][4 * v4 + 3] * inv};
  };
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int v4 = 0; v4 < 4; ++v4) {
      const f32x4 x = scaled(dt, v4);
      char* dst = ost + l32 * OP + (32 * dt + 8 * v4 + 4 * hh) * EB;
      if constexpr (EB == 2)
        *reinterpret_cast<uint2*>(dst) = uint2{float_to_bf16_bits(x[0]) | (float_to_bf16_bits(x[1]) << 16),
                                               float_to_bf16_bits(x[2]) | (float_to_bf16_bits(x[3]) << 16)};
      else
        *reinterpret_cast<f32x4*>(dst) = x;
    }
  __builtin_amdgcn_wave_barrier();
  drain(static_cast<char*>(a.Out) + (row0 * a.out_tok + (int64_t)hq * a.out_head) * EB, a.out_tok * EB);
  if (a.o32) {
    char* dst = reinterpret_cast<char*>(a.o32 + (row0 * a.n_q_heads + hq) * D);
    const int64_t stride = (int64_t)a.n_q_heads * D * 4;
    if constexpr (EB == 2) {  // float32 rows are twice as long: half the head dim at a time
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int dt = 0; dt < NDT / 2; ++dt)
#pragma unroll
          for (int v4 = 0; v4 < 4; ++v4)
            *reinterpret_cast<f32x4*>(ost + l32 * OP + (32 * dt + 8 * v4 + 4 * hh) * 4) = scaled(p * (NDT / 2) + dt, v4);
        __builtin_amdgcn_wave_barrier();
        drain(dst + p * D * 2, stride);
      }
    } else {
      drain(dst, stride);
    }
  }
}

// bf16 with head dim 64, two heads: 37 KB of LDS and few enough registers for
// three workgroups per CU.
template <typename T, int D, int GW>
constexpr bool three_per_simd() { return Elem<T>::kBytes == 2 && D == 64 && GW == 2; }

// CMP: over the compact copies of hga_gather_routed (only the routing counts
// are read; the rows come in tile order).
//
// What bounds it: at d = 128 a CU holds one workgroup (two waves per SIMD), and
// a tile's LDS reads, matrix products and exponentials take about as long
// each; they overlap only as far as the two waves are apart. 131,072 queries,
// Qwen3-8B layer, 576 routed keys: 1,938 us when every tile waited for its own
// gather and the softmax maximum went through the LDS crossbar, 1,579 us (742
// TFLOP/s) now.
template <typename T, int D, int GW, bool PREC, bool CMP>
__global__ __launch_bounds__(128 * GW) __attribute__((amdgpu_waves_per_eu(three_per_simd<T, D, GW>() ? 3 : 1))) void
attend_fwd_kernel(AttnArgs a) {
  __shared__ __attribute__((aligned(16))) char smem[2 * (Tile<T, D>::kRowBytes +
                                                         (Elem<T>::kBytes == 2 ? Tile<T, D>::kRowBytes
                                                                               : Tile<T, D>::kTBytes))];
  __shared__ int s_sel[64];
  prefetch_args(a);
  WgCoord wc = decode_wg(blockIdx.x, a.n_kv_heads, a.gqa / GW);
  // last blocks first when a block's routed set grows with its position (a
  // sink window covering the context, i.e. dense causal attention): the
  // longest workgroups start first and the tail of the grid is short ones
  if (a.heavy_last) wc.b = a.n_qb - 1 - wc.b;
  const int tid = threadIdx.x;
  // the routing row is requested before anything else
  RouteRow rrow;
  if constexpr (CMP) {
    rrow.nsel = a.n_sel[(int64_t)wc.b * a.n_kv_heads + wc.h];
    rrow.sel = -1;
  } else {
    rrow = load_route_row(a, wc.b, wc.h, tid);
  }
  WgSync sync;
  attend_block<T, D, GW, PREC, false, CMP>(a, wc, smem, s_sel, tid, sync, [] { return true; }, [&](RoutedSet& rs) {
    if (tid < a.top_groups) s_sel[tid] = rrow.sel;
    set_groups(rs, rrow.nsel, s_sel);
  });
}

// Routing and forward in one launch, for calls whose (query block, kv head)
// pairs alone do not fill the chip. Each workgroup of a two-head slice has
// eight waves in two teams that run side by side, each with its own barrier:
// waves 0-3 route the block (the routing kernel's single-block path,
// route_blocks with TB = 1; the first slice also writes the routing tables)
// and leave the selection in LDS; waves 4-7 attend the block's window tiles
// meanwhile and take the selected groups as soon as the routing lands.
template <typename T, int D, bool PREC>
__global__ __launch_bounds__(512) void route_attend_kernel(RouteArgs ra, AttnArgs a) {
  __shared__ __attribute__((aligned(16))) char smem[2 * (Tile<T, D>::kRowBytes +
                                                         (Elem<T>::kBytes == 2 ? Tile<T, D>::kRowBytes
                                                                               : Tile<T, D>::kTBytes))];
  __shared__ int s_route[65];  // selected group ids, then their count
  __shared__ int s_sync[3];    // the two teams' barrier counters, the routing-done flag
  prefetch_args(ra);
  prefetch_args(a);
  const WgCoord wc = decode_wg(blockIdx.x, a.n_kv_heads, a.gqa / 2);
  if (threadIdx.x < 3) s_sync[threadIdx.x] = 0;
  __syncthreads();  // the last workgroup-wide barrier: the teams part here
  if (threadIdx.x < 256) {
    WaveGroupSync sync{&s_sync[0], 4};
    // the first summary row goes out after the query rows have landed: the
    // team's waves share the SIMDs' registers with the attention team's
    route_blocks<T, D, 1, false>(ra, wc.b * a.n_kv_heads + wc.h, wc.hs == 0, s_route, (int)threadIdx.x, sync);
    if (threadIdx.x < 64) publish_flag(&s_sync[2]);  // wave 0 wrote s_route
    return;
  }
  const int tid = (int)threadIdx.x - 256;
  WaveGroupSync sync{&s_sync[1], 4};
  attend_block<T, D, 2, PREC, true, false>(a, wc, smem, s_route, tid, sync, [&] { return flag_set(&s_sync[2]); },
                                    [&](RoutedSet& rs) { set_groups(rs, s_route[64], s_route); });
}

template <typename T, int D, bool PREC, bool CMP = false>
static hipError_t fwd_dispatch(const AttnArgs& a, hipStream_t s) {
  // four query heads per workgroup share each gathered tile; with fewer
  // (block, kv head) pairs than the chip has CUs, two heads per workgroup
  // fill it instead. bf16 with d = 64 takes two heads always: three such
  // workgroups fit a CU and hide each other's start and end, which outweighs
  // gathering each tile twice and a few spilled registers (us with two heads
  // and, before, four heads and one workgroup per CU: 10,048 queries, G = 8,
  // 320 keys 53 and 65, 1,216 keys 139 and 163, 4,352 keys 339 and 407; 40,000
  // queries 202 and 256; with o_f32 77 and 81; 2,048 queries 14 and 16, with
  // o_f32 20 and 20). At d = 128, where two fit, 131,072 queries took 1,759
  // against 1,590.
  int gw = a.gqa >= 4 ? 4 : a.gqa;
  if (gw == 4 && three_per_simd<T, D, 2>()) gw = 2;
  if (gw == 4 && (int64_t)a.n_qb * a.n_kv_heads * (a.gqa / 4) < 256) gw = 2;
  const dim3 grid(a.n_qb * a.n_kv_heads * (a.gqa / gw));
  if (gw == 4) {
    if constexpr (!three_per_simd<T, D, 2>())
      hipLaunchKernelGGL((attend_fwd_kernel<T, D, 4, PREC, CMP>), grid, dim3(512), 0, s, a);
  } else if (gw == 2)
    hipLaunchKernelGGL((attend_fwd_kernel<T, D, 2, PREC, CMP>), grid, dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((attend_fwd_kernel<T, D, 1, PREC, CMP>), grid, dim3(128), 0, s, a);
  return hipGetLastError();
}

// The forward's own choice for such calls is two heads per workgroup (see
// fwd_dispatch): G = 2, or G = 4 with fewer than 256 (block, kv head) pairs.
// The fused kernel's static LDS plus the routing's must fit a CU.
bool route_attend_fusable(const AttnArgs& a, size_t route_lds) {
  const bool two_heads = a.gqa == 2 || (a.gqa == 4 && (int64_t)a.n_qb * a.n_kv_heads < 256);
  const size_t fixed = 2 * (2 * Tile<__bf16, 128>::kRowBytes) + 2 * 64 * 4 + 24 * 1024;
  return two_heads && fixed + route_lds <= 160 * 1024;
}

hipError_t launch_route_attend(const RouteArgs& ra, const AttnArgs& a, bool bf16, int head_dim,
                               size_t route_lds, hipStream_t s) {
  const dim3 grid(a.n_qb * a.n_kv_heads * (a.gqa / 2));
#define HGA_RA(T, D, P) hipLaunchKernelGGL((route_attend_kernel<T, D, P>), grid, dim3(512), route_lds, s, ra, a)
  if (bf16) {
    if (head_dim == 64) { if (a.o32) HGA_RA(__bf16, 64, true); else HGA_RA(__bf16, 64, false); }
    else { if (a.o32) HGA_RA(__bf16, 128, true); else HGA_RA(__bf16, 128, false); }
  } else {
    HGA_RA(float, 64, false);  // float32 is built for head_dim 64 only
  }
#undef HGA_RA
  return hipGetLastError();
}

hipError_t launch_attend_fwd(const AttnArgs& a, bool bf16, int head_dim, hipStream_t s) {
  if (bf16) {
    if (a.o32) return head_dim == 64 ? fwd_dispatch<__bf16, 64, true>(a, s) : fwd_dispatch<__bf16, 128, true>(a, s);
    return head_dim == 64 ? fwd_dispatch<__bf16, 64, false>(a, s) : fwd_dispatch<__bf16, 128, false>(a, s);
  }
  return fwd_dispatch<float, 64, false>(a, s);  // float32 is built for head_dim 64 only
}

hipError_t launch_attend_gathered_fwd(const AttnArgs& a, bool bf16, int head_dim, hipStream_t s) {
  if (bf16) {
    if (a.o32)
      return head_dim == 64 ? fwd_dispatch<__bf16, 64, true, true>(a, s) : fwd_dispatch<__bf16, 128, true, true>(a, s);
    return head_dim == 64 ? fwd_dispatch<__bf16, 64, false, true>(a, s) : fwd_dispatch<__bf16, 128, false, true>(a, s);
  }
  return fwd_dispatch<float, 64, false, true>(a, s);  // float32 is built for head_dim 64 only
}

}  // namespace hga
