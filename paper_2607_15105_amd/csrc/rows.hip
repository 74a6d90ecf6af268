// Per-query routing and attention: every query row routes on its own (the
// block descriptor of Sec. 2.1 item 1 taken over a block of one query), and
// attends its own routed set. This is routing at generation time, one or a
// few queries per call (Sec. 1, last result: routed generation; Sec. 7),
// and, applied to every row of a training segment, a strictly causal
// variant of the method (Sec. 6.1: with a routing decision shared by a whole
// block, an early query's attended set depends on later queries; here it
// depends only on its own row and on keys before its block).
//
// A query keeps the windows and the candidate chunks of the 64-token block
// holding it (sink window, local window ending at the block end, chunks
// closed before the local window) and attends only tokens up to its own
// position: keys after it never enter its result.
//
// Routing: one workgroup per (four consecutive query rows, or one row when the
// call is too small to fill the chip that way, kv head), of four waves, or of
// sixteen for a row with a long candidate list. A row's descriptor is the exact
// float64 mean of its G query-head rows; chunk and group scores (one
// candidate per thread, against every row of the workgroup) are float64 FMA
// chains over the float32 summaries, selected by wave_top_k, one wave per row
// (larger score first, lower index on ties; sets returned ascending).
//
// Attention, bf16: rows of one block in groups of up to 16 (row, query head)
// pairs on the matrix cores (attend_rows_fwd_mfma_kernel below).
// Attention, float32: one workgroup of four waves per (query row, kv head),
// all G query heads together, on the vector units: lane = key for the scores
// (each lane reads its key's K and V rows), an online softmax with
// wave-uniform maxima, and lane = head-dim slice for P.V over the tile's V
// rows staged in LDS. The four waves take every fourth 64-key tile of the
// routed set and merge their partial softmax states at the end.
#include "route_device.h"

namespace hga {

// ---------------------------------------------------------------- routing

template <typename T, int D>
__device__ inline float load_elem(const char* p) {
  if constexpr (Elem<T>::kBytes == 2) return bf16_bits_to_float(*reinterpret_cast<const uint16_t*>(p));
  else return *reinterpret_cast<const float*>(p);
}

// Float64 dot product of the descriptor with summary row r of a quad-major
// table (two FMA chains over the even and odd head-dim elements).
template <int D>
__device__ inline double summary_dot(const float* table, int64_t r, int64_t cap, const double* q) {
  const f32x4* t = reinterpret_cast<const f32x4*>(table) + r;
  f32x4 v[D / 4];
#pragma unroll
  for (int k = 0; k < D / 4; ++k) v[k] = t[(int64_t)k * cap];  // every load in flight
  double a0 = 0.0, a1 = 0.0;
#pragma unroll
  for (int k = 0; k < D / 4; ++k) {
    a0 = fma((double)v[k][0], q[4 * k], a0);
    a1 = fma((double)v[k][1], q[4 * k + 1], a1);
    a0 = fma((double)v[k][2], q[4 * k + 2], a0);
    a1 = fma((double)v[k][3], q[4 * k + 3], a1);
    // keep each quad's conversions and descriptor reads with it (hoisting
    // them all ahead doubles the live registers)
    __builtin_amdgcn_sched_barrier(0);
  }
  return a0 + a1;
}

// Float64 dots of summary row r with the descriptors q[0..nv): per
// descriptor the two FMA chains of summary_dot, in the same order, with the
// row read and converted once for all of them. Sixteen elements at a time in
// two load slots, so that the kernel keeps four waves per SIMD.
template <int D, int RB>
__device__ inline void summary_dots(const float* table, int64_t r, int64_t cap, const double (*q)[D], int nv,
                                    double (&out)[RB]) {
  constexpr int U = D / 16;  // units of a row
  f32x4 va[4], vb[4];
  double a0[RB], a1[RB];
#pragma unroll
  for (int w = 0; w < RB; ++w) a0[w] = a1[w] = 0.0;
  load_unit<D, U>(va, table, r, cap, 0);
  load_unit<D, U>(vb, table, r, cap, 1);
#pragma unroll
  for (int u = 0; u < U; u += 2) {
    unit_dots<D, U, RB>(va, q, u, nv, a0, a1);
    if (u + 2 < U) load_unit<D, U>(va, table, r, cap, u + 2);
    unit_dots<D, U, RB>(vb, q, u + 1, nv, a0, a1);
    if (u + 3 < U) load_unit<D, U>(vb, table, r, cap, u + 3);
  }
#pragma unroll
  for (int w = 0; w < RB; ++w) out[w] = a0[w] + a1[w];
}

// One workgroup of four waves per (RB consecutive query rows, kv head).
// Every chunk-summary row the call scores is read once per workgroup and
// scored against the RB row descriptors (rows of one block share their
// candidate list; rows of two blocks score the longer list, each keeping its
// own prefix); wave w then selects for row w. Candidates are taken in rounds
// of RR: after each round a row's selection is the top-k_c of [its running
// selection | the round's scores]. The kept entries sit ahead of the round's
// and have lower chunk ids, so positions keep chunk order, ties still go to
// the lower chunk, and the selection is the whole list's. `stride`: doubles
// of dynamic LDS per row.
template <int RB>
struct RowsRoute {
  static constexpr int RR = RB == 1 ? kRowsRouteRound : 512;
};

// NT threads: 256, or 1,024 for one row with more than 512 candidates. There
// the sixteen waves score 1,024 candidates a pass and each selects from a
// sixteenth of the round (contiguous, so that kept positions stay in chunk
// order); wave 0 then selects from the kept entries of all. (Decode step at
// 131K, 2,027 candidates: 34 us with four waves and one selection by ranks,
// 20 us so. The scoring takes half of it: the CU's float64 conversions and the
// descriptor's LDS reads, not the summary rows; four load slots were no faster.)
// WHOLE (one row, 256 threads): a summary row's loads all in flight at once, one
// workgroup per CU. It is the shortest for a workgroup on its own, so it serves
// calls with at most one per CU (one row at 16K: 9.9 us against 12.8 with ranks);
// with more, the sixteen-element units let four share a CU (64 rows at 16K,
// 512 workgroups: 18 us whole, 10.9 in units; 15.4 with ranks).
template <typename T, int D, int RB, int NT, bool WHOLE>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WHOLE ? 1 : 4, 8))) void
route_rows_kernel(RouteArgs a, int64_t n_rows, int stride) {
  constexpr int EB = Elem<T>::kBytes;
  constexpr int RR = RowsRoute<RB>::RR;
  static_assert(RB <= 4, "one selecting wave per row");
  extern __shared__ double dyn[];  // per row: [kept | the round's scores], then its group scores
  __shared__ __attribute__((aligned(16))) double s_q[RB][D];
  __shared__ TopKScratch s_tk[RB];
  __shared__ double s_kv[RB][64];
  __shared__ int s_ki[RB][64];
  __shared__ int s_chunks[RB][64];
  constexpr int NWS = NT / 64;  // waves that share a selection (RB == 1, NT > 256)
  __shared__ double s_cv[NT > 256 ? NWS * 64 : 1];  // their kept entries, compacted
  __shared__ int s_ci[NT > 256 ? NWS * 64 : 1];
  __shared__ TopKScratch s_tkw[NT > 256 ? NWS : 1];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.x % a.n_kv_heads;
  const int64_t row0 = (int64_t)(blockIdx.x / a.n_kv_heads) * RB;
  const int nv = (int)(n_rows - row0 < RB ? n_rows - row0 : RB);  // rows of this workgroup
  const int G = a.gqa;

  // descriptors: the mean of each row's G head rows of kv head h (a sum of G
  // bf16 or float32 values and a division by a power of two: exact)
  for (int x = tid; x < RB * D; x += NT) {
    const int w = x / D, e = x % D;
    double s = 0.0;
    if (w < nv) {
      const char* qrow = static_cast<const char*>(a.Q) + ((row0 + w) * a.q_tok + (int64_t)h * G * a.q_head) * EB;
      for (int g = 0; g < G; ++g) s += (double)load_elem<T, D>(qrow + ((int64_t)g * a.q_head + e) * EB);
      s /= (double)G;
    }
    s_q[w][e] = s;
  }
  __syncthreads();

  // candidates [c_lo, c_lo + n) of row w: a prefix of the longest list
  const int c_lo = a.first_cand;
  auto n_cand_of = [&](int w) {
    return max(0, last_cand((a.q_begin + row0 + w) / 64, a.local_tokens) - c_lo);
  };
  int n_max = 0;
  for (int w = 0; w < nv; ++w) n_max = max(n_max, n_cand_of(w));
  const int my_n = wave < nv ? n_cand_of(wave) : 0;
  const float* cs = a.chunk_sum + quad_off(h, 0, 0, D, a.chunk_cap);
  const int n_rounds = max(1, (n_max + RR - 1) / RR);
  double* mine = dyn + wave * stride;  // this wave's row (wave < nv)
  int n_kept = 0;
  for (int r = 0; r < n_rounds; ++r) {
    const int nr = max(0, min(RR, n_max - r * RR));
    const int r0 = c_lo + r * RR;
    for (int i0 = 0; i0 < nr; i0 += NT) {
      const int i = i0 + tid;
      double v[RB];
      if constexpr (WHOLE) v[0] = summary_dot<D>(cs, r0 + min(i, nr - 1), a.chunk_cap, s_q[0]);
      else summary_dots<D, RB>(cs, r0 + min(i, nr - 1), a.chunk_cap, s_q, nv, v);
      if (i < nr) {
#pragma unroll
        for (int w = 0; w < RB; ++w)
          if (w < nv) dyn[w * stride + 64 + i] = no_nan(v[w]);
      }
    }
    __syncthreads();
    int nr_w = max(0, min(RR, my_n - r * RR));
    bool listed = false;
    if constexpr (NT > 256) {
      // every wave its slice; the kept entries of all replace the round's
      const int per = (nr + NWS - 1) / NWS, lo = min(wave * per, nr), cnt = min(per, nr - lo);
      const int ke = min(a.top_chunks, per);  // entries a full slice keeps
      listed = ke * NWS < nr;
      if (listed) {
        const int p = wave_top_k(dyn + 64 + lo, cnt, ke, lane, s_tkw[wave]);
        if (lane < ke) {
          s_cv[wave * ke + lane] = lane < cnt ? dyn[64 + lo + p] : -__builtin_inf();
          s_ci[wave * ke + lane] = lane < cnt ? r0 + lo + p : kNoIdx;
        }
        __syncthreads();
        nr_w = nr / per * ke + min(ke, nr % per);  // full slices, then at most one short one
        for (int i = tid; i < NWS * ke; i += NT) dyn[64 + i] = s_cv[i];
        __syncthreads();
      }
    }
    if (wave < nv && nr_w > 0) {
      double* base = mine + 64 - n_kept;
      if (lane < n_kept) base[lane] = s_kv[wave][lane];
      __builtin_amdgcn_wave_barrier();
      const int n = n_kept + nr_w;
      const int pc = wave_top_k(base, n, a.top_chunks, lane, s_tk[wave]);
      const int k_eff = min(a.top_chunks, n);
      double v = 0.0;
      int idx = -1;
      if (lane < k_eff) {  // pc is a position only on those lanes
        v = base[pc];
        idx = pc < n_kept ? s_ki[wave][pc] : NT > 256 && listed ? s_ci[pc - n_kept] : r0 + (pc - n_kept);
      }
      __builtin_amdgcn_wave_barrier();
      if (lane < k_eff) {
        s_kv[wave][lane] = v;
        s_ki[wave][lane] = idx;
      }
      n_kept = k_eff;
    }
    __syncthreads();  // the round's scores are read: the next round may overwrite them
  }
  const int kc_eff = min(a.top_chunks, my_n);  // this wave's row
  const int64_t slot = (row0 + wave) * a.n_kv_heads + h;
  if (wave < nv) {
    const int chunk = lane < kc_eff ? s_ki[wave][lane] : -1;
    if (lane < a.top_chunks) a.sel_chunks[slot * a.top_chunks + lane] = chunk;
    s_chunks[wave][lane] = lane < kc_eff ? chunk : 0;
  }
  __syncthreads();

  // group scores over every group of each row's chosen chunks (ascending
  // ids): item f of row w is group f of its list
  const int gpc_shift = 6 - a.group_shift;
  const int gmask = (1 << gpc_shift) - 1;
  const int gslot = a.top_chunks << gpc_shift;  // items per row
  if (a.top_groups > 0 && gslot > 0) {
    const float* gs = a.group_sum + quad_off(h, 0, 0, D, a.group_cap);
    for (int f0 = 0; f0 < nv * gslot; f0 += NT) {
      const int fa = f0 + tid, w = fa / gslot, f = fa - w * gslot;
      if (w < nv && f < (min(a.top_chunks, n_cand_of(w)) << gpc_shift)) {
        const int64_t j = ((int64_t)s_chunks[w][f >> gpc_shift] << gpc_shift) + (f & gmask);
        if constexpr (WHOLE) {
          dyn[w * stride + f] = no_nan(summary_dot<D>(gs, j, a.group_cap, s_q[w]));
        } else {
          double v[1];
          summary_dots<D, 1>(gs, j, a.group_cap, s_q + w, 1, v);
          dyn[w * stride + f] = no_nan(v[0]);
        }
      }
    }
  }
  __syncthreads();
  if (wave >= nv) return;
  const int n_gc = kc_eff << gpc_shift;
  if (a.top_groups > 0) {
    const int kg_eff = min(a.top_groups, n_gc);
    const int pg = wave_top_k(mine, n_gc, a.top_groups, lane, s_tk[wave]);
    const int pgs = lane < kg_eff ? pg : 0;  // pg is a position only on those lanes
    const int gid = (s_chunks[wave][pgs >> gpc_shift] << gpc_shift) + (pgs & gmask);
    if (lane < a.top_groups) a.sel_groups[slot * a.top_groups + lane] = lane < kg_eff ? gid : -1;
    if (lane == 0) a.n_sel[slot] = kg_eff;
  } else if (lane == 0) {
    a.n_sel[slot] = 0;
  }
}

// Candidates of a row from which on sixteen waves route it: four waves take
// 256 a pass, and the merging of sixteen selections costs about a pass (Qwen3-8B
// layer, one row, k_c 8: 286 to 478 candidates 12.3-13.7 us with four waves and
// 15.1-16.1 with sixteen, 542 to 766 15.4 and 15.4, 1,022 17.7 and 15.6).
constexpr int kRowsRouteWide = 512;

// Rows per routing workgroup: four when the call still fills the chip with
// (four rows, kv head) workgroups (each summary row read then serves four
// rows), else one (decode steps and short calls keep one workgroup per row).
static int route_rows_per_wg(int64_t n_rows, int n_kv_heads) {
  return (n_rows + 3) / 4 * n_kv_heads >= 256 ? 4 : 1;
}

hipError_t launch_route_rows(const RouteArgs& a, int64_t n_rows, int n_cand_max, int group_cand, bool bf16,
                             int head_dim, hipStream_t s) {
  const int rb = route_rows_per_wg(n_rows, a.n_kv_heads);
  const int rr = rb == 1 ? RowsRoute<1>::RR : RowsRoute<4>::RR;
  const int nc = 64 + (n_cand_max < rr ? n_cand_max : rr);
  const int stride = nc > group_cand ? nc : group_cand;
  const size_t lds = (size_t)rb * stride * sizeof(double);
  const dim3 grid((unsigned)((n_rows + rb - 1) / rb * a.n_kv_heads));
#define HGA_RR(T, D, RB, NT, WHOLE) \
  hipLaunchKernelGGL((route_rows_kernel<T, D, RB, NT, WHOLE>), grid, dim3(NT), lds, s, a, n_rows, stride)
#define HGA_RRT(RB, NT, WHOLE)                          \
  do {                                                  \
    if (!bf16) HGA_RR(float, 64, RB, NT, WHOLE);        \
    else if (head_dim == 64) HGA_RR(__bf16, 64, RB, NT, WHOLE); \
    else HGA_RR(__bf16, 128, RB, NT, WHOLE);            \
  } while (0)
  const bool alone = n_rows * a.n_kv_heads <= 256;  // one workgroup per CU at most
  if (rb == 4) HGA_RRT(4, 256, false);
  else if (!alone) HGA_RRT(1, 256, false);
  else if (n_cand_max > kRowsRouteWide) HGA_RRT(1, 1024, false);
  else HGA_RRT(1, 256, true);
#undef HGA_RRT
#undef HGA_RR
  return hipGetLastError();
}

// ---------------------------------------------------------------- attention

// The float32 kernels are for head dim 64, which is what float32 is built for.
__device__ inline float load_f32(const char* p) { return *reinterpret_cast<const float*>(p); }

// Wave-wide maximum and sum, the same value in every lane: DPP steps inside
// each 16-lane row (swap neighbours, swap pairs, mirror each half-row,
// mirror the row), then the four rows' values read as scalars. No step goes
// through the LDS crossbar.
template <int CTRL>
__device__ inline float dpp_src(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}
__device__ inline float row_lane(float x, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), l));
}
__device__ inline float wave_max(float v) {
  v = fmaxf(v, dpp_src<0xB1>(v));   // quad_perm [1,0,3,2]
  v = fmaxf(v, dpp_src<0x4E>(v));   // quad_perm [2,3,0,1]
  v = fmaxf(v, dpp_src<0x141>(v));  // row_half_mirror
  v = fmaxf(v, dpp_src<0x140>(v));  // row_mirror
  return fmaxf(fmaxf(row_lane(v, 0), row_lane(v, 16)), fmaxf(row_lane(v, 32), row_lane(v, 48)));
}
__device__ inline float wave_sum(float v) {
  v += dpp_src<0xB1>(v);
  v += dpp_src<0x4E>(v);
  v += dpp_src<0x141>(v);
  v += dpp_src<0x140>(v);
  return (row_lane(v, 0) + row_lane(v, 16)) + (row_lane(v, 32) + row_lane(v, 48));
}

// Token at position p of a row's routed set [sink | selected groups | local
// window up to the row].
__device__ inline int64_t row_token(int p, int n_sink, int n_grp_tok, int64_t ls, const int32_t* sel,
                                    int gshift) {
  if (p < n_sink) return p;
  if (p < n_sink + n_grp_tok) {
    const int q = p - n_sink;
    return ((int64_t)sel[q >> gshift] << gshift) + (q & ((1 << gshift) - 1));
  }
  return ls + (p - n_sink - n_grp_tok);
}

// The routed set of query row `row` for kv head h.
struct RowSet {
  int64_t pos, ls;
  int n_sink, n_grp_tok, R;
  const int32_t* sel;
};

__device__ inline RowSet row_set(const AttnArgs& a, int64_t row, int h) {
  RowSet r;
  r.pos = a.q_begin + row;
  const int64_t block_end = (r.pos / 64 + 1) * 64;
  r.ls = block_end - a.local_tokens > 0 ? block_end - a.local_tokens : 0;
  r.n_sink = (int)min((int64_t)a.sink_tokens, r.ls);
  const int64_t slot = row * a.n_kv_heads + h;
  const int n_sel = a.top_groups > 0 ? a.n_sel[slot] : 0;
  r.n_grp_tok = n_sel << a.group_shift;
  r.R = r.n_sink + r.n_grp_tok + (int)(r.pos + 1 - r.ls);
  r.sel = a.top_groups > 0 ? a.sel_groups + slot * a.top_groups : nullptr;
  return r;
}

template <int G>
__global__ __launch_bounds__(256) void attend_rows_fwd_kernel(AttnArgs a) {
  constexpr int D = 64;                 // a lane per head-dim element in P.V
  constexpr int NP = D / 4;             // 16-byte pieces of a key row
  constexpr int VP = D * 4 + 16;        // LDS pitch of a staged V row (padded against bank conflicts)
  __shared__ __attribute__((aligned(16))) float s_q[G][D];
  __shared__ float s_m[4][G], s_l[4][G];
  __shared__ float s_o[4][G][D];
  __shared__ __attribute__((aligned(16))) char s_v[4][64 * VP];  // each wave's current V tile, row = key
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.x % a.n_kv_heads;
  const int64_t row = blockIdx.x / a.n_kv_heads;
  const char* Qb = static_cast<const char*>(a.Q);
  const char* Kb = static_cast<const char*>(a.K);
  const char* Vb = static_cast<const char*>(a.V);

  for (int x = tid; x < G * D; x += 256) {
    const int g = x / D, e = x % D;
    s_q[g][e] = load_f32(Qb + (row * a.q_tok + (int64_t)(h * G + g) * a.q_head + e) * 4);
  }
  const RowSet rs = row_set(a, row, h);
  __syncthreads();

  float m[G], l[G], o[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m[g] = -__builtin_inff();
    l[g] = 0.0f;
    o[g] = 0.0f;
  }
  const int64_t k_stride = a.k_tok * 4, v_stride = a.v_tok * 4;
  const int64_t k_head = (int64_t)h * a.k_head * 4, v_head = (int64_t)h * a.v_head * 4;
  for (int tb = wave * 64; tb < rs.R; tb += 256) {
    const int p = tb + lane;
    const bool valid = p < rs.R;
    const int64_t t = row_token(min(p, rs.R - 1), rs.n_sink, rs.n_grp_tok, rs.ls, rs.sel, a.group_shift);
    // scores of this lane's key for the G query heads; its V row goes out
    // with its K row and is staged in LDS for P.V
    const char* kr = row_ptr(Kb, t, k_stride) + k_head;
    const char* vrow = row_ptr(Vb, t, v_stride) + v_head;
    u32x4 kw[NP], vw[NP];
#pragma unroll
    for (int c = 0; c < NP; ++c) kw[c] = *reinterpret_cast<const u32x4*>(kr + 16 * c);
#pragma unroll
    for (int c = 0; c < NP; ++c) vw[c] = *reinterpret_cast<const u32x4*>(vrow + 16 * c);
    float s[G];
#pragma unroll
    for (int g = 0; g < G; ++g) s[g] = 0.0f;
#pragma unroll
    for (int c = 0; c < NP; ++c) {
      const f32x4 kx = __builtin_bit_cast(f32x4, kw[c]);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const f32x4 qq = *reinterpret_cast<const f32x4*>(&s_q[g][4 * c]);
#pragma unroll
        for (int e = 0; e < 4; ++e) s[g] = fmaf(qq[e], kx[e], s[g]);
      }
      // one piece at a time: its query reads stay with it
      __builtin_amdgcn_sched_barrier(0);
    }
    // online softmax in log2 units; the maximum is uniform over the wave
    float pr[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float sg = valid ? s[g] * a.scale_log2 : -__builtin_inff();
      const float mn = fmaxf(m[g], wave_max(sg));
      const float alpha = exp2f(m[g] - mn);
      pr[g] = exp2f(sg - mn);
      l[g] = l[g] * alpha + pr[g];
      o[g] *= alpha;
      m[g] = mn;
    }
    // P.V: the tile's V rows through LDS (row = key), then lane = head-dim
    // element reads each key's (consecutive lanes, consecutive words)
    char* sv = s_v[wave];
#pragma unroll
    for (int c = 0; c < NP; ++c) *reinterpret_cast<u32x4*>(sv + lane * VP + 16 * c) = vw[c];
    __builtin_amdgcn_wave_barrier();
    const int nk = min(64, rs.R - tb);
#pragma unroll 1
    for (int j0 = 0; j0 < nk; j0 += 8) {
      float vv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) vv[u] = load_f32(sv + (j0 + u) * VP + lane * 4);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (j0 + u < nk) {
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const float pj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pr[g]), j0 + u));
            o[g] = fmaf(pj, vv[u], o[g]);
          }
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
  // merge the four waves' partial softmax states
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const float lt = wave_sum(l[g]);
    if (lane == 0) {
      s_m[wave][g] = m[g];
      s_l[wave][g] = lt;
    }
    s_o[wave][g][lane] = o[g];
  }
  __syncthreads();
  char* Ob = static_cast<char*>(a.Out);
  for (int x = tid; x < G * D; x += 256) {
    const int g = x / D, e = x % D;
    float M = -__builtin_inff();
#pragma unroll
    for (int w = 0; w < 4; ++w) M = fmaxf(M, s_m[w][g]);
    float num = 0.0f, den = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float f = s_m[w][g] == -__builtin_inff() ? 0.0f : exp2f(s_m[w][g] - M);
      num = fmaf(f, s_o[w][g][e], num);
      den = fmaf(f, s_l[w][g], den);
    }
    const float out = num / den;
    *reinterpret_cast<float*>(Ob + (row * a.out_tok + (int64_t)(h * G + g) * a.out_head + e) * 4) = out;
    if (a.o32) a.o32[(row * a.n_q_heads + h * G + g) * D + e] = out;
    if (e == 0) a.lse[row * a.n_q_heads + h * G + g] = (M + log2f(den)) * kLn2;
  }
}

// bf16: rows in groups, scores and P.V on the matrix cores.
//
// A group is RPW consecutive rows at positions RPW * i .. (RPW divides 64: one
// block, one set of windows), at most 16 (row, query head) pairs, the columns
// of the 16 x 16 x 32 products. Its key lists are walked 32 keys at a time:
// first the shared one (sink window, local window up to the group's last
// row), every row at once; then each row's private one (its selected groups),
// in the same products with the other rows' columns computed and dropped. The
// columns are 3/4 idle there, which costs little: the kernel is bound by the
// gathered bytes, and by how they are gathered.
//  - Loads: consecutive lanes take consecutive 16-byte pieces of a row (four
//    rows of 256 bytes per instruction) and the rows go through LDS. With one
//    lane per key, or with each lane its operand's piece, neighbouring lanes
//    lie in different rows: every lane is then a cache access of its own, and
//    the issue of the loads took longer than all else.
//  - S^T = K Q^T: K rows from LDS (A operand), the pairs' Q rows in registers.
//  - online softmax: lane l holds 8 scores of pair l % 16; the maximum over
//    the four lanes of a pair goes by lane swaps.
//  - O^T += V^T P^T: P^T from the registers that hold S^T, V from LDS through
//    the transpose load. P enters as a bf16 hi + lo pair. As one bf16 value the
//    lazily raised maximum would leave the heaviest key's P unrepresentable,
//    which is exactly 1 under an exact maximum: 1.6e-3 of O's norm (float32
//    copy, 320 keys) against 1.3e-3, and the backward's D carries it on to dQ.
//    The exact maximum alone gives back 1.2e-3 where several waves share a row
//    and each has its own, but not with a wave per group. The pair gives
//    3e-6, for 0 to 4% of the time (9% with 8,192 keys a row).
// One register set of K and one of V: the next step's rows go out when these
// are in LDS (one buffer per wave, K and then V).
//
// KW == 1: a wave per group, four groups per workgroup. KW > 1 (few rows):
// the KW waves of a workgroup take every KW-th step of one group's lists (of one
// row's, where RPW == 1) and merge their softmax states through LDS.
//
// Strictly causal 1,024-row segment at 16K (Qwen3-8B layer): 172 us with one
// workgroup per row and one lane per key, 46 us so; a decode step at 16K 9.6 and
// 6.8 us.
constexpr int kRowsStep = 32;  // keys of a step
// Which form a call takes. A wave per group from 1,024 (group, kv head) pairs on;
// below, rows on their own while they are few, else four waves per group. (Qwen3-8B
// layer, forward, a wave and four per group, us: 320 keys a row, 256 rows or 512
// group pairs 32 and 20, 512 rows 31 and 33, 768 43 and 47, 1,024 46 and 61. The line
// is for such lists: of 96 keys 320 rows take 12.7 and 14.9, of 1,216 keys 512 rows
// 166 and 139, 768 228 and 204, 1,024 243 and 266; at d = 64 512 rows 22 and 17,
// 1,024 28 and 30.)
constexpr int64_t kRowsWaveGroups = 1024;

// The keys of the last row's block in the windows, and those of a row's
// selected groups, at most.
static int64_t window_keys(const AttnArgs& a, int64_t n_rows) {
  const int64_t end = ((a.q_begin + n_rows - 1) / 64 + 1) * 64;
  const int64_t ls = end > a.local_tokens ? end - a.local_tokens : 0;
  return (a.sink_tokens < ls ? a.sink_tokens : ls) + end - ls;
}
static int64_t private_keys(const AttnArgs& a) { return (int64_t)a.top_groups << a.group_shift; }

// Rows on their own, or in groups of `rpw` that share the windows' keys: up to
// 256 (row, kv head) pairs, one workgroup per CU, always on their own; up to
// `most` pairs where the windows do not outweigh what the rows have for
// themselves. Two rows' workgroups share a CU then and take about 1.5 (windows +
// private) keys' time, a group windows + rpw private. (Forward, Qwen3-8B layer,
// own rows and groups, us: 512 pairs, windows 192 and private 128 keys 10.5 and
// 13.4, 192 and 1,024 25 and 53, 8,320 and 128 123 and 86; 640 pairs 13.5 and
// 13.8, 800 16.3 and 14.0. Eight heads a row, groups of two, 512 pairs: 192 and
// 128 11.2 and 10.8, 192 and 1,024 26 and 32. dQ: 512 pairs 23.2 and 24.6, 39.6
// and 60, 149 and 97; 640 pairs 30 and 26.)
static bool rows_apart(const AttnArgs& a, int64_t n_rows, int rpw, int64_t most) {
  const int64_t pairs = n_rows * a.n_kv_heads;
  return pairs <= 256 || (pairs <= most && window_keys(a, n_rows) < (2 * rpw - 3) * private_keys(a));
}

// Waves for a row on its own: four, or many (twelve, dQ eight) where it has a CU
// to itself and more than sixteen steps to walk. (One row, the same inputs again
// and again: forward, 320 keys 7.5 us with four and 8.0 with twelve, 576 9.8 and
// 10.0, 704 11.0 and 11.0, 1,216 15.9 and 13.7; dQ with the rest, 320 keys 13.8
// with four and 14.3 with eight, 576 16.1 and 15.9, 1,216 22.7 and 20.8. A decode
// step at 131K with inputs that change, 576 keys: 33.7 and 33.3.)
static bool many_waves(const AttnArgs& a, int64_t n_rows) {
  return n_rows * a.n_kv_heads <= 256 && window_keys(a, n_rows) + private_keys(a) > 16 * kRowsStep;
}

// Maximum and sum over the four lanes l % 16 + 16 i, the same in each.
__device__ inline float quad_max(float x) {
  float y = x;
  swap16(x, y);
  x = y = fmaxf(x, y);
  swap32(x, y);
  return fmaxf(x, y);
}
__device__ inline float quad_sum(float x) {
  float y = x;
  swap16(x, y);
  x = y = x + y;
  swap32(x, y);
  return x + y;
}

// A product that no sum takes up unrounded.
__device__ inline float mul_rounded(float x, float y) {
#pragma clang fp contract(off)
  return x * y;
}

// Natural logarithm of l 2^m, rounded once: log2 of l's mantissa is below 1 in
// size, and the sum is taken in float64.
__device__ inline float lse_of(float m, float l) {
  const double e = (double)m + (double)__builtin_amdgcn_frexp_expf(l);
  return (float)((e + (double)__log2f(__builtin_amdgcn_frexp_mantf(l))) * 0.69314718055994530942);
}

// A group of rows and its key lists. List 0 is shared (n_sh keys: the sink
// window, then the local window up to the last row; a row takes those up to
// its own position); list 1 + r is row r's: its selected groups.
struct RowGroup {
  int64_t pos0;   // position of the first row
  int64_t row0;   // its row in the call
  int nr;         // rows
  int64_t ls;     // local window start
  int ns;         // sink tokens
  int n_sh;       // keys of the shared list
  int gshift;
  int cnt;        // lane r: tokens of row r's selected groups
  const int* sel; // this wave's LDS [row][64]: selected group ids

  // Keys of list u (u the same in every lane), and the steps they take.
  __device__ inline int len(int u) const {
    return u == 0 ? n_sh : __builtin_amdgcn_readlane(cnt, u - 1);
  }
  __device__ inline int steps(int u) const { return (len(u) + kRowsStep - 1) / kRowsStep; }
  // Tokens of keys p, p + dp, ... of list u (clamped to the list). The list
  // is chosen once, so that the reads of the selected ids go out together.
  template <int N>
  __device__ inline void tokens(int u, int p, int dp, uint32_t (&t)[N]) const {
    if (u == 0) {
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const int q = min(p + dp * j, n_sh - 1);
        t[j] = (uint32_t)q + (q < ns ? 0u : (uint32_t)ls - (uint32_t)ns);
      }
    } else {
      const int last = __builtin_amdgcn_readlane(cnt, u - 1) - 1;
      const int* s = sel + (u - 1) * 64;
#pragma unroll
      for (int j = 0; j < N; ++j) t[j] = (uint32_t)s[min(p + dp * j, last) >> gshift];
#pragma unroll
      for (int j = 0; j < N; ++j)
        t[j] = (t[j] << gshift) + ((uint32_t)min(p + dp * j, last) & ((1u << gshift) - 1u));
    }
  }
};

// The group of `nr` rows of the call from row `row0` on (all in one block),
// without its selected groups (cnt).
__device__ inline RowGroup row_group(const AttnArgs& a, int64_t row0, int nr, const int* s_sel) {
  RowGroup g;
  g.row0 = row0;
  g.pos0 = a.q_begin + row0;
  g.nr = nr;
  const int64_t block_end = (g.pos0 / 64 + 1) * 64;
  g.ls = block_end - a.local_tokens > 0 ? block_end - a.local_tokens : 0;
  g.ns = (int)min((int64_t)a.sink_tokens, g.ls);
  g.n_sh = g.ns + (int)(g.pos0 + nr - g.ls);
  g.gshift = a.group_shift;
  g.cnt = 0;
  g.sel = s_sel;
  return g;
}

// The routing rows of a group, one entry per lane: requested at the start,
// taken (to the wave's LDS list) when the windows' loads are out.
template <int RPW>
struct RowRoutes {
  int n;
  int sel[RPW];
  __device__ inline void load(const AttnArgs& a, const RowGroup& g, int h, int lane) {
    n = 0;
    if (a.top_groups > 0) {
      // lanes and rows past the end repeat the last entry
      n = a.n_sel[(g.row0 + min(lane, g.nr - 1)) * a.n_kv_heads + h];
#pragma unroll
      for (int r = 0; r < RPW; ++r)
        sel[r] = a.sel_groups[((g.row0 + min(r, g.nr - 1)) * a.n_kv_heads + h) * a.top_groups +
                              min(lane, a.top_groups - 1)];
    }
  }
  __device__ inline void take(const AttnArgs& a, RowGroup& g, int* s_sel, int lane) const {
    g.cnt = n << a.group_shift;
    if (a.top_groups > 0) {
#pragma unroll
      for (int r = 0; r < RPW; ++r) s_sel[r * 64 + lane] = sel[r];
    }
    __builtin_amdgcn_wave_barrier();
  }
};

// A step of a walk over the lists of a group: keys [32 f, 32 f + 32) of list
// u. A wave starts at its index and advances by the number of waves.
struct RowStep {
  int u, f, n;  // n: steps of list u
  __device__ inline void settle(const RowGroup& g) {
    while (u <= g.nr) {
      n = g.steps(u);
      if (f < n) return;
      f -= n;
      ++u;
    }
  }
};

// One lane's share of a step's 32 rows of K or V: 16-byte pieces, a row's
// pieces on consecutive lanes; their tokens serve both tensors.
template <int D>
struct RowRegs {
  static constexpr int PPR = D / 8;         // pieces of a row
  static constexpr int RPI = 64 / PPR;      // rows per load instruction
  static constexpr int NJ = kRowsStep / RPI;
  u32x4 x[NJ];
  static __device__ inline void tokens(const RowGroup& g, const RowStep& st, int lane, uint32_t (&t)[NJ]) {
    g.tokens(st.u, kRowsStep * st.f + lane / PPR, RPI, t);
  }
  __device__ inline void load(const char* base, int64_t stride, const uint32_t (&t)[NJ], int lane) {
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      x[j] = *reinterpret_cast<const u32x4*>(row_ptr(base, t[j], stride) + 16 * (lane % PPR));
  }
  __device__ inline void store(char* dst, int pitch, int lane) const {
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      *reinterpret_cast<u32x4*>(dst + (RPI * j + lane / PPR) * pitch + 16 * (lane % PPR)) = x[j];
  }
};

template <int D, int G, int RPW, int KW>
__global__ __launch_bounds__(KW == 1 ? 256 : 64 * KW) __attribute__((amdgpu_waves_per_eu(2))) void
attend_rows_fwd_mfma_kernel(AttnArgs a, int64_t n_rows, int64_t n_groups) {
  constexpr int NS = D / 32;       // k steps of S
  constexpr int NT = D / 16;       // 16-row tiles of O^T
  constexpr int KP = D * 2 + 16;   // LDS pitch of a K row: an operand read's sixteen rows start 4 banks apart
  constexpr int VP = D * 2 + 32;   // and of a V row: a transpose load's eight rows start 8 banks apart
  constexpr int NW = KW == 1 ? 4 : KW;
  constexpr int NG = KW == 1 ? 4 : 1;  // groups per workgroup
  // V tiles at a time, so that a tile's two products are not one after the
  // other (d = 64: two keep it at four waves per SIMD; four took 52 us where
  // two take 44, 2,048 rows)
  constexpr int NV = D / 32;
  static_assert(RPW * G <= 16, "a group's pairs are the columns of one product");
  // each wave's K, then V rows of its current step; with KW > 1, at the end, its O
  __shared__ __attribute__((aligned(16))) char s_v[NW][kRowsStep * VP];
  __shared__ int s_sel[NW][RPW * 64];
  __shared__ float s_m[NW][16], s_l[NW][16];
  __shared__ int s_bad[NW];
  static_assert(16 * D * 4 <= kRowsStep * VP, "a wave's partial O fits its V buffer");
  typedef __attribute__((address_space(3))) s16x4* lds_s4;
  prefetch_args(a);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.x % a.n_kv_heads;
  const int64_t gi = (int64_t)(blockIdx.x / a.n_kv_heads) * NG + (KW == 1 ? wave : 0);
  if (KW == 1 && gi >= n_groups) return;  // no barrier follows with KW == 1
  // rows [r_lo, r_hi) of the call: positions RPW * i .. RPW * i + RPW - 1
  const int64_t p_lo = (a.q_begin / RPW + gi) * RPW - a.q_begin;
  const int64_t r_lo = p_lo > 0 ? p_lo : 0;
  const int64_t r_hi = min(p_lo + RPW, n_rows);
  const int pr = lane & 15, quad = lane >> 4;  // this lane's pair (column) and quarter
  const int hq = h * G + pr % G;
  const char* Kb = static_cast<const char*>(a.K) + (int64_t)h * a.k_head * 2;
  const char* Vb = static_cast<const char*>(a.V) + (int64_t)h * a.v_head * 2;
  const int64_t k_stride = a.k_tok * 2, v_stride = a.v_tok * 2;
  const float c = a.scale_log2;
  char* sv = s_v[wave];
  const char* tr = sv + (4 * quad + (pr >> 2)) * VP + 8 * (pr & 3);  // this lane's transpose-load address
  char* Ob = static_cast<char*>(a.Out);

  // The rows all at once; then, if an infinity or a NaN came out, each alone:
  // it may stem from a V row that only some of them attend and that met a
  // zero weight in the others' columns.
  int64_t row0 = r_lo;
  int nr = (int)(r_hi - r_lo);
  bool alone = nr == 1;
  for (;;) {
    RowGroup g = row_group(a, row0, nr, s_sel[wave]);
    RowRoutes<RPW> routes;
    routes.load(a, g, h, lane);
    const int ri = min(pr / G, nr - 1);  // this lane's row in the group (surplus columns repeat the last row)
    const int64_t row = row0 + ri;
    bf16x8 qf[NS];
    {
      const char* qr = static_cast<const char*>(a.Q) + (row * a.q_tok + (int64_t)hq * a.q_head) * 2;
#pragma unroll
      for (int s = 0; s < NS; ++s) qf[s] = *reinterpret_cast<const bf16x8*>(qr + 64 * s + 16 * quad);
    }
    // with few rows the routing and query rows go ahead of every wave's K and V rows
    if constexpr (KW > 1) __builtin_amdgcn_s_barrier();

    // this lane's pair: running maximum (scores in log2 units, as rounded to
    // float32: every p, correction and the LSE are relative to that), sum, O
    float m = -__builtin_inff(), l = 0.0f;
    f32x4 o[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) o[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // one step, its rows in kr and vr, which refill with the rows of step `ld`
    auto step = [&](const RowStep& st, RowRegs<D>& kr, RowRegs<D>& vr, const RowStep& ld,
                    bool more) __attribute__((always_inline)) {
      kr.store(sv, KP, lane);
      uint32_t tok[RowRegs<D>::NJ];
      if (more) {
        RowRegs<D>::tokens(g, ld, lane, tok);
        kr.load(Kb, k_stride, tok, lane);
      }
      __builtin_amdgcn_wave_barrier();
      f32x4 s[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        s[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < NS; ++k)
          s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              *reinterpret_cast<const bf16x8*>(sv + (16 * t + pr) * KP + 64 * k + 16 * quad), qf[k], s[t], 0, 0, 0);
      }
      __builtin_amdgcn_wave_barrier();
      vr.store(sv, VP, lane);
      if (more) vr.load(Vb, v_stride, tok, lane);
      // this lane's keys of the list are [0, last): in the shared list those
      // up to its row, in a row's list all or, in other rows' columns, none
      const int last = st.u == 0 ? g.n_sh - (nr - 1) + ri : ri == st.u - 1 ? g.len(st.u) : 0;
      const int end = kRowsStep * (st.f + 1);
      if (st.u > 0 || end > g.n_sh - (nr - 1)) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (end - kRowsStep + 16 * t + 4 * quad + i >= last) s[t][i] = -__builtin_inff();
      }
      float mx = -__builtin_inff();
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) mx = fmaxf(mx, s[t][i]);
      mx = mul_rounded(quad_max(mx), c);
      const bool raise = mx > m + 8.0f;  // the maximum is raised when it grows by more than 2^8
      if (__any(raise)) {
        const float f = raise ? __builtin_amdgcn_exp2f(m - mx) : 1.0f;
        if (raise) m = mx;
        l *= f;
#pragma unroll
        for (int t = 0; t < NT; ++t) o[t] *= f;
      }
      const float mc = m == -__builtin_inff() ? 0.0f : m;  // nothing attended yet: every p is 0
      bf16x8 hi, lo;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float p = __builtin_amdgcn_exp2f(fmaf(s[t][i], c, -mc));
          l += p;
          hi[4 * t + i] = (__bf16)p;
          lo[4 * t + i] = (__bf16)(p - (float)hi[4 * t + i]);
        }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int t0 = 0; t0 < NT; t0 += NV) {
        bf16x8 vt[NV];
#pragma unroll
        for (int j = 0; j < NV; ++j) {
          const int t = t0 + j;
          const s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(tr + 32 * t));
          const s16x4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(tr + 16 * VP + 32 * t));
          typedef short s16x8 __attribute__((ext_vector_type(8)));
          vt[j] = __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7));
        }
#pragma unroll
        for (int j = 0; j < NV; ++j)
          o[t0 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[j], hi, o[t0 + j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < NV; ++j)
          o[t0 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[j], lo, o[t0 + j], 0, 0, 0);
      }
      __builtin_amdgcn_wave_barrier();
    };
    // a wave that starts in the windows does not wait for the routing rows
    RowStep s0{0, KW == 1 ? 0 : wave, g.steps(0)};
    RowRegs<D> k0, v0;
    const bool early = s0.f < s0.n;
    uint32_t tok0[RowRegs<D>::NJ];
    if (early) {
      RowRegs<D>::tokens(g, s0, lane, tok0);
      k0.load(Kb, k_stride, tok0, lane);
      v0.load(Vb, v_stride, tok0, lane);
    }
    routes.take(a, g, s_sel[wave], lane);
    s0.settle(g);
    if (!early && s0.u <= nr) {
      RowRegs<D>::tokens(g, s0, lane, tok0);
      k0.load(Kb, k_stride, tok0, lane);
      v0.load(Vb, v_stride, tok0, lane);
    }
    while (s0.u <= nr) {
      RowStep nx = s0;
      nx.f += KW;
      nx.settle(g);
      // past the end a wave of many steps loads its last rows again, unused:
      // with conditional loads the compiler waits for both register sets at
      // each use; a wave of few steps does without them
      const bool more = nx.u <= nr;
      const RowStep ld = RowStep{more ? nx.u : s0.u, more ? nx.f : s0.f, more ? nx.n : s0.n};
      step(s0, k0, v0, ld, KW == 1 || more);
      s0 = nx;
    }
    l = quad_sum(l);
    bool bad = false;  // a result of the pass is not finite
    if (!alone) {
      float sum = l;
#pragma unroll
      for (int t = 0; t < NT; ++t) sum += (o[t][0] + o[t][1]) + (o[t][2] + o[t][3]);
      bad = __any(!(fabsf(sum) < __builtin_inff())) != 0;
    }
    if constexpr (KW == 1) {
      if (!bad && pr < nr * G) {
        const float inv = 1.0f / l;
        if (quad == 0) a.lse[row * a.n_q_heads + hq] = lse_of(m, l);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const int d0 = 16 * t + 4 * quad;
          const f32x4 v = o[t] * inv;
          *reinterpret_cast<uint2*>(Ob + (row * a.out_tok + (int64_t)hq * a.out_head + d0) * 2) =
              uint2{float_to_bf16_bits(v[0]) | (float_to_bf16_bits(v[1]) << 16),
                    float_to_bf16_bits(v[2]) | (float_to_bf16_bits(v[3]) << 16)};
          if (a.o32) *reinterpret_cast<f32x4*>(a.o32 + (row * a.n_q_heads + hq) * D + d0) = v;
        }
      }
    } else {
      float* so = reinterpret_cast<float*>(sv);
      if (quad == 0) {
        s_m[wave][pr] = m;
        s_l[wave][pr] = l;
      }
      if (RPW > 1 && lane == 0) s_bad[wave] = bad;
      if (pr < RPW * G) {
#pragma unroll
        for (int t = 0; t < NT; ++t) *reinterpret_cast<f32x4*>(so + pr * D + 16 * t + 4 * quad) = o[t];
      }
      __syncthreads();
      if constexpr (RPW > 1) {
        bad = false;
#pragma unroll
        for (int w = 0; w < KW; ++w) bad |= __builtin_amdgcn_readfirstlane(s_bad[w]) != 0;
      }
      for (int x = tid; !bad && x < nr * G * (D / 4); x += 64 * KW) {
        const int p = x / (D / 4), d0 = 4 * (x % (D / 4));
        float M = -__builtin_inff();
#pragma unroll
        for (int w = 0; w < KW; ++w) M = fmaxf(M, s_m[w][p]);
        f32x4 num = {0.0f, 0.0f, 0.0f, 0.0f};
        float den = 0.0f;
#pragma unroll
        for (int w = 0; w < KW; ++w) {
          const float f = s_m[w][p] == -__builtin_inff() ? 0.0f : __builtin_amdgcn_exp2f(s_m[w][p] - M);
          num += f * *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(s_v[w]) + p * D + d0);
          den = fmaf(f, s_l[w][p], den);
        }
        const f32x4 v = num * (1.0f / den);
        const int64_t r = row0 + p / G;
        const int hp = h * G + p % G;
        *reinterpret_cast<uint2*>(Ob + (r * a.out_tok + (int64_t)hp * a.out_head + d0) * 2) =
            uint2{float_to_bf16_bits(v[0]) | (float_to_bf16_bits(v[1]) << 16),
                  float_to_bf16_bits(v[2]) | (float_to_bf16_bits(v[3]) << 16)};
        if (a.o32) *reinterpret_cast<f32x4*>(a.o32 + (r * a.n_q_heads + hp) * D + d0) = v;
        if (d0 == 0) a.lse[r * a.n_q_heads + hp] = lse_of(M, den);
      }
      if constexpr (RPW > 1) __syncthreads();  // the buffers are read: a further pass may overwrite them
    }
    // the next pass: the first row alone, then the one after it, ...
    if constexpr (RPW == 1) {
      return;
    } else {
      if (alone ? row0 + 1 == r_hi || nr == (int)(r_hi - r_lo) : !bad) return;
      row0 = alone ? row0 + 1 : r_lo;
      alone = true;
      nr = 1;
    }
  }
}

// Rows per group with several rows: four, two where a row has eight heads.
template <int G>
constexpr int rows_per_group() { return G >= 8 ? 2 : 4; }

// Groups of `rpw` rows by position that hold a row of the call.
static int64_t n_row_groups(const AttnArgs& a, int64_t n_rows, int rpw) {
  return (a.q_begin + n_rows + rpw - 1) / rpw - a.q_begin / rpw;
}

template <int D, int G>
hipError_t rows_fwd_mfma(const AttnArgs& a, int64_t n_rows, hipStream_t s) {
  constexpr int R = rows_per_group<G>();
  const int64_t ng = n_row_groups(a, n_rows, R);
  if (ng * a.n_kv_heads >= kRowsWaveGroups) {
    hipLaunchKernelGGL((attend_rows_fwd_mfma_kernel<D, G, R, 1>), dim3((unsigned)((ng + 3) / 4 * a.n_kv_heads)),
                       dim3(256), 0, s, a, n_rows, ng);
  } else if (!rows_apart(a, n_rows, R, 640)) {
    hipLaunchKernelGGL((attend_rows_fwd_mfma_kernel<D, G, R, 4>), dim3((unsigned)(ng * a.n_kv_heads)), dim3(256), 0,
                       s, a, n_rows, ng);
  } else if (many_waves(a, n_rows)) {
    hipLaunchKernelGGL((attend_rows_fwd_mfma_kernel<D, G, 1, 12>), dim3((unsigned)(n_rows * a.n_kv_heads)),
                       dim3(768), 0, s, a, n_rows, n_rows);
  } else {
    hipLaunchKernelGGL((attend_rows_fwd_mfma_kernel<D, G, 1, 4>), dim3((unsigned)(n_rows * a.n_kv_heads)),
                       dim3(256), 0, s, a, n_rows, n_rows);
  }
  return hipGetLastError();
}

template <int D>
hipError_t rows_fwd_bf16(const AttnArgs& a, int64_t n_rows, hipStream_t s) {
  switch (a.gqa) {
    case 1: return rows_fwd_mfma<D, 1>(a, n_rows, s);
    case 2: return rows_fwd_mfma<D, 2>(a, n_rows, s);
    case 4: return rows_fwd_mfma<D, 4>(a, n_rows, s);
    default: return rows_fwd_mfma<D, 8>(a, n_rows, s);
  }
}

hipError_t launch_attend_rows_fwd(const AttnArgs& a, int64_t n_rows, bool bf16, int head_dim, hipStream_t s) {
  if (bf16) return head_dim == 64 ? rows_fwd_bf16<64>(a, n_rows, s) : rows_fwd_bf16<128>(a, n_rows, s);
  const dim3 grid((unsigned)(n_rows * a.n_kv_heads)), block(256);
  switch (a.gqa) {
    case 1: hipLaunchKernelGGL(attend_rows_fwd_kernel<1>, grid, block, 0, s, a); break;
    case 2: hipLaunchKernelGGL(attend_rows_fwd_kernel<2>, grid, block, 0, s, a); break;
    case 4: hipLaunchKernelGGL(attend_rows_fwd_kernel<4>, grid, block, 0, s, a); break;
    default: hipLaunchKernelGGL(attend_rows_fwd_kernel<8>, grid, block, 0, s, a); break;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------- backward
//
// The backward of hga_attend_rows_fwd with the routing held constant:
//   dQ                  query-major: the rows' routed sets in tiles, P
//                       recomputed from the LSE, dS = P (dP - D) and
//                       dQ = scale dS K. bf16: rows_dq_mfma_kernel, which also
//                       forms D = rowsum(dO * O); float32: rows_rowdot_kernel
//                       for D, then rows_dq_kernel;
//   dK, dV              key-major and deterministic: one workgroup per (16
//                       keys of a 64-token chunk of the active tokens, kv
//                       head). It lists, in row order, the rows whose routed
//                       set touches those keys (window or selected groups)
//                       with the mask of the keys each attends, then walks the
//                       list (rows_dkv_mfma_kernel for bf16, rows_dkv_kernel
//                       for float32). No atomics: results are bitwise
//                       reproducible.

__global__ __launch_bounds__(256) void rows_rowdot_kernel(AttnArgs a, int64_t n_rows) {
  constexpr int D = 64;
  const int lane = threadIdx.x & 63;
  const int64_t x = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);  // (row, query head)
  if (x >= n_rows * a.n_q_heads) return;
  const int64_t row = x / a.n_q_heads;
  const int hq = (int)(x % a.n_q_heads);
  const char* dob = static_cast<const char*>(a.dO) + (row * a.do_tok + (int64_t)hq * a.do_head) * 4;
  const float o = a.o32 ? a.o32[x * D + lane]
                        : load_f32(static_cast<const char*>(a.O) + (row * a.o_tok + (int64_t)hq * a.o_head + lane) * 4);
  const float sum = wave_sum(fmaf(load_f32(dob + lane * 4), o, 0.0f));
  if (lane == 0) a.dvec[x] = sum;
}

// float32 dQ on the vector units: the four waves stage each tile's K and V
// rows together in LDS (double-buffered); each wave takes a query head,
// forms dS (lane = key), then dQ = scale dS K (lane = head-dim slice, keys in
// tile order).
template <int G>
__global__ __launch_bounds__(256) void rows_dq_kernel(AttnArgs a) {
  constexpr int D = 64;                 // a lane per head-dim element of dQ
  constexpr int NP = D / 4;             // 16-byte pieces of a key row
  constexpr int KP = D * 4 + 16;        // LDS pitch of a staged K / V row (padded against bank conflicts)
  constexpr int HPW = (G + 3) / 4;      // query heads of a wave
  constexpr int PER = 2 * 64 * NP / 256;  // 16-byte pieces of a K/V tile per thread
  __shared__ __attribute__((aligned(16))) float s_q[G][D];
  __shared__ __attribute__((aligned(16))) float s_do[G][D];
  __shared__ float s_lse[G], s_dd[G];
  __shared__ float s_ds[G][64];
  // the K and V rows of the current 64-key tile, double-buffered
  __shared__ __attribute__((aligned(16))) char s_kv[2][2][64 * KP];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.x % a.n_kv_heads;
  const int64_t row = blockIdx.x / a.n_kv_heads;
  const char* Kb = static_cast<const char*>(a.K);
  const char* Vb = static_cast<const char*>(a.V);
  for (int x = tid; x < G * D; x += 256) {
    const int g = x / D, e = x % D;
    const int64_t hq = h * G + g;
    s_q[g][e] = load_f32(static_cast<const char*>(a.Q) + (row * a.q_tok + hq * a.q_head + e) * 4);
    s_do[g][e] = load_f32(static_cast<const char*>(a.dO) + (row * a.do_tok + hq * a.do_head + e) * 4);
  }
  if (tid < G) {
    s_lse[tid] = a.lse[row * a.n_q_heads + h * G + tid] * kLog2e;
    s_dd[tid] = a.dvec[row * a.n_q_heads + h * G + tid];
  }
  const RowSet rs = row_set(a, row, h);
  const int ntiles = (rs.R + 63) / 64;

  // a tile's K and V rows: thread items (tensor, row, piece), all loads in
  // flight together, then stored to the tile's buffer
  const int64_t k_stride = a.k_tok * 4, v_stride = a.v_tok * 4;
  const int64_t k_head = (int64_t)h * a.k_head * 4, v_head = (int64_t)h * a.v_head * 4;
  auto fetch = [&](int tile, u32x4 (&st)[PER]) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int item = tid + 256 * u;
      const int which = item / (64 * NP), rem = item % (64 * NP);
      const int r = rem / NP, c = rem % NP;
      const int p = min(tile * 64 + r, rs.R - 1);  // padding positions read the last row (their P is 0)
      const int64_t t = row_token(p, rs.n_sink, rs.n_grp_tok, rs.ls, rs.sel, a.group_shift);
      const char* src = which == 0 ? row_ptr(Kb, t, k_stride) + k_head : row_ptr(Vb, t, v_stride) + v_head;
      st[u] = *reinterpret_cast<const u32x4*>(src + 16 * c);
    }
  };
  auto stage = [&](int buf, const u32x4 (&st)[PER]) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int item = tid + 256 * u;
      const int which = item / (64 * NP), rem = item % (64 * NP);
      const int r = rem / NP, c = rem % NP;
      *reinterpret_cast<u32x4*>(s_kv[buf][which] + r * KP + 16 * c) = st[u];
    }
  };
  if (ntiles > 0) {
    u32x4 st[PER];
    fetch(0, st);
    stage(0, st);
  }
  __syncthreads();

  float dq[HPW];
#pragma unroll
  for (int i = 0; i < HPW; ++i) dq[i] = 0.0f;
  for (int tile = 0; tile < ntiles; ++tile) {
    const int buf = tile & 1;
    u32x4 nx[PER];
    if (tile + 1 < ntiles) fetch(tile + 1, nx);  // the next tile's rows are in flight during this one
    const char* sk = s_kv[buf][0];
    const char* sv = s_kv[buf][1];
    const int nk = min(64, rs.R - tile * 64);
    // S and dP: lane = key, this wave's query heads
#pragma unroll
    for (int i = 0; i < HPW; ++i) {
      const int g = wave + 4 * i;
      if (g < G) {
        float sg = 0.0f, dg = 0.0f;
#pragma unroll 4
        for (int c = 0; c < NP; ++c) {
          const f32x4 kx = *reinterpret_cast<const f32x4*>(sk + lane * KP + 16 * c);
          const f32x4 vx = *reinterpret_cast<const f32x4*>(sv + lane * KP + 16 * c);
          const f32x4 qq = *reinterpret_cast<const f32x4*>(&s_q[g][4 * c]);
          const f32x4 dd = *reinterpret_cast<const f32x4*>(&s_do[g][4 * c]);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            sg = fmaf(qq[e], kx[e], sg);
            dg = fmaf(dd[e], vx[e], dg);
          }
        }
        const float pr = lane < nk ? exp2f(sg * a.scale_log2 - s_lse[g]) : 0.0f;
        s_ds[g][lane] = pr * (dg - s_dd[g]);
      }
    }
    __builtin_amdgcn_wave_barrier();  // a wave reads only the dS rows it wrote
    // dQ += dS K: lane = head-dim element, keys of the tile in order
#pragma unroll
    for (int i = 0; i < HPW; ++i) {
      const int g = wave + 4 * i;
      if (g < G) {
#pragma unroll 8
        for (int j = 0; j < nk; ++j) dq[i] = fmaf(s_ds[g][j], load_f32(sk + j * KP + lane * 4), dq[i]);
      }
    }
    if (tile + 1 < ntiles) {
      // the other buffer held tile - 1, which every wave finished before the
      // previous barrier
      stage(buf ^ 1, nx);
      __syncthreads();
    }
  }
#pragma unroll
  for (int i = 0; i < HPW; ++i) {
    const int g = wave + 4 * i;
    if (g < G) a.dQ[(row * a.n_q_heads + h * G + g) * D + lane] = dq[i] * a.scale;
  }
}

// bf16: dQ (and D = rowsum(dO * O)) on the forward's groups of rows and key
// lists, with its loads. S^T = K Q^T and dP^T = V dO^T leave, in lane l, eight
// keys' scores and dP of pair l % 16; P comes from the LSE, dS = P (dP - D)
// enters dQ^T += K^T dS^T as a bf16 hi + lo pair (as in the block kernels: dQ
// scales dS by raw key magnitudes), with K read from LDS by rows for S and
// through the transpose load for dQ. The kernel also forms its rows' D and
// leaves it in a.dvec for the dK/dV kernel.
//
// Strictly causal 1,024-row segment at 16K (Qwen3-8B layer): 255 us (dQ, one
// workgroup per row, one lane per key) + 8.8 us (D, a kernel of its own)
// before, 53 us in all so.
template <int D, int G, int RPW, int KW>
__global__ __launch_bounds__(KW == 1 ? 256 : 64 * KW) __attribute__((amdgpu_waves_per_eu(2))) void
rows_dq_mfma_kernel(AttnArgs a, int64_t n_rows, int64_t n_groups) {
  using TL = Tile<__bf16, D>;
  constexpr int NS = D / 32;       // k steps of S and dP
  constexpr int NT = D / 16;       // 16-row tiles of dQ^T
  constexpr int TB = kRowsStep * TL::kRowPitch;  // bytes of 32 rows
  constexpr int NW = KW == 1 ? 4 : KW;
  constexpr int NG = KW == 1 ? 4 : 1;            // groups per workgroup
  static_assert(RPW * G <= 16, "a group's pairs are the columns of one product");
  // each wave's K and V rows of its current step; with KW > 1, at the end, its dQ
  __shared__ __attribute__((aligned(16))) char s_kv[NW][2 * TB];
  __shared__ int s_sel[NW][RPW * 64];
  __shared__ int s_bad[NW];
  static_assert(16 * D * 4 <= 2 * TB, "a wave's partial dQ fits its buffer");
  typedef __attribute__((address_space(3))) s16x4* lds_s4;
  prefetch_args(a);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.x % a.n_kv_heads;
  const int64_t gi = (int64_t)(blockIdx.x / a.n_kv_heads) * NG + (KW == 1 ? wave : 0);
  if (KW == 1 && gi >= n_groups) return;  // no barrier follows with KW == 1
  const int64_t p_lo = (a.q_begin / RPW + gi) * RPW - a.q_begin;
  const int64_t r_lo = p_lo > 0 ? p_lo : 0;
  const int64_t r_hi = min(p_lo + RPW, n_rows);
  const int pr = lane & 15, quad = lane >> 4;  // this lane's pair (column) and quarter
  const int hq = h * G + pr % G;
  const char* Kb = static_cast<const char*>(a.K) + (int64_t)h * a.k_head * 2;
  const char* Vb = static_cast<const char*>(a.V) + (int64_t)h * a.v_head * 2;
  const int64_t k_stride = a.k_tok * 2, v_stride = a.v_tok * 2;
  const float c = a.scale_log2;
  char* sk = s_kv[wave];
  char* sv = sk + TB;
  const int rd = TL::row_off(pr, 0) + 16 * quad;               // this lane's operand rows (tile 0)
  const int tr = TL::row_off(4 * quad + (pr >> 2), 4 * (pr & 3));  // and its transpose-load address

  // The rows all at once; then, if an infinity or a NaN came out, each alone
  // (see the forward; here K rows meet a zero dS).
  int64_t row0 = r_lo;
  int nr = (int)(r_hi - r_lo);
  bool alone = nr == 1;
  for (;;) {
    RowGroup g = row_group(a, row0, nr, s_sel[wave]);
    RowRoutes<RPW> routes;
    routes.load(a, g, h, lane);
    const int ri = min(pr / G, nr - 1);  // this lane's row in the group (surplus columns repeat the last row)
    const int64_t row = row0 + ri;
    const int64_t rh = row * a.n_q_heads + hq;
    RowStep s0{0, KW == 1 ? 0 : wave, g.steps(0)};
    RowRegs<D> kr, vr;
    uint32_t tok0[RowRegs<D>::NJ];
    const bool early = s0.f < s0.n;
    if (early) {
      RowRegs<D>::tokens(g, s0, lane, tok0);
      kr.load(Kb, k_stride, tok0, lane);
      vr.load(Vb, v_stride, tok0, lane);
    }
    bf16x8 qf[NS], df[NS];
    float dd = 0.0f;
    {
      const char* qr = static_cast<const char*>(a.Q) + (row * a.q_tok + (int64_t)hq * a.q_head) * 2;
      const char* dr = static_cast<const char*>(a.dO) + (row * a.do_tok + (int64_t)hq * a.do_head) * 2;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        qf[s] = *reinterpret_cast<const bf16x8*>(qr + 64 * s + 16 * quad);
        df[s] = *reinterpret_cast<const bf16x8*>(dr + 64 * s + 16 * quad);
      }
      if (a.o32) {
        const float* orow = a.o32 + rh * D;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const f32x4 x = *reinterpret_cast<const f32x4*>(orow + 32 * s + 8 * quad);
          const f32x4 y = *reinterpret_cast<const f32x4*>(orow + 32 * s + 8 * quad + 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) dd = fmaf((float)df[s][e], x[e], dd);
#pragma unroll
          for (int e = 0; e < 4; ++e) dd = fmaf((float)df[s][4 + e], y[e], dd);
        }
      } else {
        const char* orow = static_cast<const char*>(a.O) + (row * a.o_tok + (int64_t)hq * a.o_head) * 2;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const bf16x8 x = *reinterpret_cast<const bf16x8*>(orow + 64 * s + 16 * quad);
#pragma unroll
          for (int e = 0; e < 8; ++e) dd = fmaf((float)df[s][e], (float)x[e], dd);
        }
      }
      dd = quad_sum(dd);
    }
    const float lse2 = a.lse[rh] * kLog2e;
    if ((KW == 1 || wave == 0) && quad == 0 && pr < nr * G) a.dvec[rh] = dd;
    routes.take(a, g, s_sel[wave], lane);
    s0.settle(g);
    if (!early && s0.u <= nr) {
      RowRegs<D>::tokens(g, s0, lane, tok0);
      kr.load(Kb, k_stride, tok0, lane);
      vr.load(Vb, v_stride, tok0, lane);
    }
    f32x4 dq[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) dq[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    while (s0.u <= nr) {
      RowStep nx = s0;
      nx.f += KW;
      nx.settle(g);
      const bool more = nx.u <= nr;
      const RowStep ld = RowStep{more ? nx.u : s0.u, more ? nx.f : s0.f, more ? nx.n : s0.n};
      // the step's rows to LDS, the next step's requested (unconditionally,
      // as in the forward)
#pragma unroll
      for (int j = 0; j < RowRegs<D>::NJ; ++j) {
        const int off = TL::row_off(RowRegs<D>::RPI * j + lane / RowRegs<D>::PPR, 8 * (lane % RowRegs<D>::PPR));
        *reinterpret_cast<u32x4*>(sk + off) = kr.x[j];
        *reinterpret_cast<u32x4*>(sv + off) = vr.x[j];
      }
      uint32_t tok[RowRegs<D>::NJ];
      RowRegs<D>::tokens(g, ld, lane, tok);
      kr.load(Kb, k_stride, tok, lane);
      vr.load(Vb, v_stride, tok, lane);
      __builtin_amdgcn_wave_barrier();
      f32x4 s[2], dp[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        s[t] = dp[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < NS; ++k) {
          const int off = rd + 16 * t * TL::kRowPitch + 64 * k;
          s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8*>(sk + off), qf[k], s[t], 0, 0, 0);
          dp[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8*>(sv + off), df[k], dp[t], 0, 0, 0);
        }
      }
      // this lane's keys of the list are [0, last) (see the forward)
      const int last = s0.u == 0 ? g.n_sh - (nr - 1) + ri : ri == s0.u - 1 ? g.len(s0.u) : 0;
      const int first = kRowsStep * s0.f + 4 * quad;
      bf16x8 hi, lo;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float p = __builtin_amdgcn_exp2f(fmaf(s[t][i], c, -lse2));
          const float ds = first + 16 * t + i < last ? p * (dp[t][i] - dd) : 0.0f;
          hi[4 * t + i] = (__bf16)ds;
          lo[4 * t + i] = (__bf16)(ds - (float)hi[4 * t + i]);
        }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(sk + tr + 32 * t));
        const s16x4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(sk + tr + 16 * TL::kRowPitch + 32 * t));
        typedef short s16x8 __attribute__((ext_vector_type(8)));
        const bf16x8 kt = __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7));
        dq[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kt, hi, dq[t], 0, 0, 0);
        dq[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kt, lo, dq[t], 0, 0, 0);
      }
      __builtin_amdgcn_wave_barrier();
      s0 = nx;
    }
    bool bad = false;  // a result of the pass is not finite
    if (!alone) {
      float sum = 0.0f;
#pragma unroll
      for (int t = 0; t < NT; ++t) sum += (dq[t][0] + dq[t][1]) + (dq[t][2] + dq[t][3]);
      bad = __any(!(fabsf(sum) < __builtin_inff())) != 0;
    }
    if constexpr (KW == 1) {
      if (!bad && pr < nr * G) {
#pragma unroll
        for (int t = 0; t < NT; ++t) *reinterpret_cast<f32x4*>(a.dQ + rh * D + 16 * t + 4 * quad) = dq[t] * a.scale;
      }
    } else {
      float* so = reinterpret_cast<float*>(sk);
      if (lane == 0) s_bad[wave] = bad;
      if (pr < RPW * G) {
#pragma unroll
        for (int t = 0; t < NT; ++t) *reinterpret_cast<f32x4*>(so + pr * D + 16 * t + 4 * quad) = dq[t];
      }
      __syncthreads();
      bad = false;
#pragma unroll
      for (int w = 0; w < KW; ++w) bad |= __builtin_amdgcn_readfirstlane(s_bad[w]) != 0;
      for (int x = tid; !bad && x < nr * G * (D / 4); x += 64 * KW) {  // the waves' parts in wave order
        const int p = x / (D / 4), d0 = 4 * (x % (D / 4));
        f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int w = 0; w < KW; ++w)
          v += *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(s_kv[w]) + p * D + d0);
        *reinterpret_cast<f32x4*>(a.dQ + ((row0 + p / G) * a.n_q_heads + h * G + p % G) * D + d0) = v * a.scale;
      }
      __syncthreads();  // the buffers are read: a further pass may overwrite them
    }
    // the next pass: the first row alone, then the one after it, ...
    if (alone ? row0 + 1 == r_hi || nr == (int)(r_hi - r_lo) : !bad) return;
    row0 = alone ? row0 + 1 : r_lo;
    alone = true;
    nr = 1;
  }
}

// The rows of the call whose routed set touches keys [k0, k0 + KW) of chunk c
// (k0 = 64 c + part KW): listed in row order in s_rows, each with the mask of
// those keys it attends (window or selected groups, cut at its position) in
// s_mask; returns their number. Called by all 256 threads of a workgroup.
template <int KW>
__device__ inline int rows_attending(const AttnArgs& a, int64_t n_rows, int h, int64_t c, int part, int* s_rows,
                                     uint32_t* s_mask, int* s_cnt) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t c0 = c * 64;
  const int64_t k0 = c0 + part * KW;
  const int g_sz = 1 << a.group_shift;
  const int gpc_shift = 6 - a.group_shift;
  const uint64_t kmask = (1ull << KW) - 1;
  int base = 0;
  for (int64_t r0 = 0; r0 < n_rows; r0 += 256) {
    const int64_t r = r0 + tid;
    uint64_t m = 0;
    if (r < n_rows) {
      const int64_t pos = a.q_begin + r;
      if (pos >= k0) {
        const int64_t block_end = (pos / 64 + 1) * 64;
        const int64_t ls = block_end - a.local_tokens > 0 ? block_end - a.local_tokens : 0;
        const int64_t sink_end = min((int64_t)a.sink_tokens, ls);
        if ((c0 >= ls && c0 < block_end) || c0 < sink_end) {
          m = ~0ull;
        } else if (a.top_groups > 0) {
          const int64_t slot = r * a.n_kv_heads + h;
          const int n = a.n_sel[slot];
          const int32_t* sel = a.sel_groups + slot * a.top_groups;
          const uint64_t gm = g_sz == 64 ? ~0ull : (1ull << g_sz) - 1;
          // sixteen entries in flight (past the end the last one again), not
          // one after the other
          for (int j0 = 0; j0 < n; j0 += 16) {
            int gid[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) gid[u] = sel[min(j0 + u, n - 1)];
#pragma unroll
            for (int u = 0; u < 16; ++u)
              if ((gid[u] >> gpc_shift) == c) m |= gm << ((gid[u] & ((1 << gpc_shift) - 1)) << a.group_shift);
          }
        }
        const int64_t last = pos - c0;  // keys after the row are not attended
        if (last < 63) m &= (2ull << last) - 1;
        m = (m >> (part * KW)) & kmask;
      }
    }
    const uint64_t bal = __ballot(m != 0);
    if (lane == 0) s_cnt[wave] = __popcll(bal);
    __syncthreads();
    int off = base;
    for (int w = 0; w < wave; ++w) off += s_cnt[w];
    if (m != 0) {
      const int at = off + lanes_below(bal);
      s_rows[at] = (int)r;
      s_mask[at] = (uint32_t)m;
    }
    base += s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
    __syncthreads();
  }
  return base;
}

// float32 dK and dV on the vector units: the list is walked four rows at a
// time; the waves split the (row, query head) pairs for S and dP (lane = key
// and a quarter of the head dim, quarters added across lanes), share P and dS
// through LDS, and each thread accumulates a slice of dK and dV for one key.
template <int G>
__global__ __launch_bounds__(256) void rows_dkv_kernel(AttnArgs a, int64_t n_rows) {
  constexpr int D = 64;
  constexpr int KW = kRowsDkvKeys;     // keys of this workgroup
  constexpr int NQ = 64 / KW;          // lanes per key: head-dim parts of a dot product
  constexpr int DQ = D / NQ;           // head dims of one part
  constexpr int NPQ = DQ / 4;          // 16-byte pieces of one part of a row
  constexpr int DE = DQ / 4;           // dK / dV dims a thread accumulates
  __shared__ int s_rows[kRowsBwdMaxRows];  // the row lists live in LDS: calls of at most this many rows
  __shared__ uint32_t s_mask[kRowsBwdMaxRows];
  __shared__ int s_cnt[4];
  constexpr int RB = 4;                // listed rows per step
  __shared__ __attribute__((aligned(16))) float s_q[2][RB][G][D];
  __shared__ __attribute__((aligned(16))) float s_do[2][RB][G][D];
  __shared__ float s_lse[2][RB][G], s_dd[2][RB][G];
  __shared__ float s_p[RB][G][KW], s_ds[RB][G][KW];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.x % a.n_kv_heads;
  const int part = (blockIdx.x / a.n_kv_heads) % (64 / KW);
  const int64_t c = a.grad_begin / 64 + blockIdx.x / a.n_kv_heads / (64 / KW);  // absolute chunk
  const int64_t k0 = c * 64 + part * KW;  // this workgroup's first key
  const int64_t q_end = a.q_begin + n_rows;

  // ---- the rows that attend one of this workgroup's keys, in row order,
  // with the mask of those keys each attends
  const int L = rows_attending<KW>(a, n_rows, h, c, part, s_rows, s_mask, s_cnt);

  // ---- this lane's key and head-dim part for the dot products
  const int kk = lane % KW, qd = lane / KW;
  const int64_t tk = min(k0 + kk, q_end - 1);  // keys past the call's end are never attended
  const char* kr = row_ptr(static_cast<const char*>(a.K), tk, a.k_tok * 4) + ((int64_t)h * a.k_head + qd * DQ) * 4;
  const char* vr = row_ptr(static_cast<const char*>(a.V), tk, a.v_tok * 4) + ((int64_t)h * a.v_head + qd * DQ) * 4;
  u32x4 kw[NPQ], vw[NPQ];
#pragma unroll
  for (int p = 0; p < NPQ; ++p) kw[p] = *reinterpret_cast<const u32x4*>(kr + 16 * p);
#pragma unroll
  for (int p = 0; p < NPQ; ++p) vw[p] = *reinterpret_cast<const u32x4*>(vr + 16 * p);
  // this thread's dK / dV dims: key kk, dims [dd0, dd0 + DE)
  const int dd0 = qd * DQ + wave * DE;
  float dk[DE], dv[DE];
#pragma unroll
  for (int e = 0; e < DE; ++e) dk[e] = dv[e] = 0.0f;

  // The list is walked RB rows at a time: the query-side data of the RB
  // rows (all G heads) is staged in LDS, double-buffered, with the next
  // batch's loads in flight while this one is used.
  constexpr int NV = 2 * RB * G * D;            // staged values per batch (Q and dO rows)
  constexpr int PER = (NV + 255) / 256;         // values per thread
  auto fetch = [&](int kb, float (&st)[PER]) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int x = tid + 256 * u;
      const int which = x / (RB * G * D), rem = x % (RB * G * D);
      const int r = rem / (G * D), g = (rem / D) % G, e = rem % D;
      const int64_t rr = s_rows[min(kb + r, L - 1)];
      const int64_t hq = h * G + g;
      st[u] = 0.0f;
      if (x < NV)
        st[u] = which == 0
            ? load_f32(static_cast<const char*>(a.Q) + (rr * a.q_tok + hq * a.q_head + e) * 4)
            : load_f32(static_cast<const char*>(a.dO) + (rr * a.do_tok + hq * a.do_head + e) * 4);
    }
  };
  auto stage = [&](int kb, int buf, const float (&st)[PER]) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int x = tid + 256 * u;
      const int which = x / (RB * G * D), rem = x % (RB * G * D);
      const int r = rem / (G * D), g = (rem / D) % G, e = rem % D;
      if (x < NV) {
        if (which == 0) s_q[buf][r][g][e] = st[u];
        else s_do[buf][r][g][e] = st[u];
      }
    }
    if (tid < RB * G) {
      const int r = tid / G, g = tid % G;
      const int64_t rr = s_rows[min(kb + r, L - 1)];
      s_lse[buf][r][g] = a.lse[rr * a.n_q_heads + h * G + g] * kLog2e;
      s_dd[buf][r][g] = a.dvec[rr * a.n_q_heads + h * G + g];
    }
  };
  if (L > 0) {
    float st[PER];
    fetch(0, st);
    stage(0, 0, st);
  }
  __syncthreads();
  for (int kb = 0; kb < L; kb += RB) {
    const int buf = (kb / RB) & 1;
    const int nrb = min(RB, L - kb);
    float nx[PER];
    fetch(kb + RB, nx);  // the next batch's data is in flight during this one
    // S and dP of the batch's (row, head) pairs, split over the waves: lane =
    // (key, head-dim part); the NQ parts are added across lanes in a fixed
    // order, so every lane of a key holds the same sums
#pragma unroll 1
    for (int pi = wave; pi < RB * G; pi += 4) {
      const int r = pi / G, g = pi % G;
      if (r < nrb) {
        float s = 0.0f, dp = 0.0f;
#pragma unroll
        for (int p = 0; p < NPQ; ++p) {
          const f32x4 kx = __builtin_bit_cast(f32x4, kw[p]), vx = __builtin_bit_cast(f32x4, vw[p]);
          const f32x4 qq = *reinterpret_cast<const f32x4*>(&s_q[buf][r][g][qd * DQ + 4 * p]);
          const f32x4 dd = *reinterpret_cast<const f32x4*>(&s_do[buf][r][g][qd * DQ + 4 * p]);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            s = fmaf(qq[e], kx[e], s);
            dp = fmaf(dd[e], vx[e], dp);
          }
        }
#pragma unroll
        for (int m = KW; m < 64; m <<= 1) {
          s += __shfl_xor(s, m);
          dp += __shfl_xor(dp, m);
        }
        if (qd == 0) {
          const bool attend = (s_mask[kb + r] >> kk) & 1u;
          const float pr = attend ? exp2f(s * a.scale_log2 - s_lse[buf][r][g]) : 0.0f;
          s_p[r][g][kk] = pr;
          s_ds[r][g][kk] = pr * (dp - s_dd[buf][r][g]);
        }
      }
    }
    __syncthreads();
    // dV += P^T dO and dK += dS^T Q: key kk, dims [dd0, dd0 + DE)
#pragma unroll 1
    for (int pi = 0; pi < nrb * G; ++pi) {
      const int r = pi / G, g = pi % G;
      const float pj = s_p[r][g][kk], dj = s_ds[r][g][kk];
#pragma unroll
      for (int e4 = 0; e4 < DE / 4; ++e4) {
        const f32x4 dd = *reinterpret_cast<const f32x4*>(&s_do[buf][r][g][dd0 + 4 * e4]);
        const f32x4 qq = *reinterpret_cast<const f32x4*>(&s_q[buf][r][g][dd0 + 4 * e4]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          dv[4 * e4 + e] = fmaf(pj, dd[e], dv[4 * e4 + e]);
          dk[4 * e4 + e] = fmaf(dj, qq[e], dk[4 * e4 + e]);
        }
      }
    }
    if (kb + RB < L) stage(kb + RB, buf ^ 1, nx);
    __syncthreads();
  }
  // keys of this workgroup that exist in this call (all tokens >= grad_begin)
  const int64_t t = k0 + kk;
  if (t < q_end) {
    float* dkr = a.dK + ((t - a.grad_begin) * a.n_kv_heads + h) * D + dd0;
    float* dvr = a.dV + ((t - a.grad_begin) * a.n_kv_heads + h) * D + dd0;
#pragma unroll
    for (int e4 = 0; e4 < DE / 4; ++e4) {
      *reinterpret_cast<f32x4*>(dkr + 4 * e4) =
          f32x4{dk[4 * e4] * a.scale, dk[4 * e4 + 1] * a.scale, dk[4 * e4 + 2] * a.scale, dk[4 * e4 + 3] * a.scale};
      *reinterpret_cast<f32x4*>(dvr + 4 * e4) = f32x4{dv[4 * e4], dv[4 * e4 + 1], dv[4 * e4 + 2], dv[4 * e4 + 3]};
    }
  }
}

// bf16: dK and dV on the matrix cores. The waves take every fourth batch of
// 16 (row, query head) pairs of the list (16 / G rows each). S = Q K^T and
// dP = dO V^T are 16 x 16 x d products (v_mfma_f32_16x16x32_bf16, lane l
// holding row l % 16 of A and column l % 16 of B over eight k values):
// A = the batch's Q or dO rows, B = the workgroup's 16 K or V rows, held in
// registers for the whole walk. Their result holds, in lane l, pairs
// 4 (l / 16) .. + 3 of key l % 16, which is the A operand of the 16 x 16 x 16
// product with keys as rows: P and dS, each as a bf16 hi + lo pair (two
// products sharing the B operand, so both enter to about 2^-17), feed
// dV += P^T dO and dK += dS^T Q straight from the registers, with dO and Q
// read from LDS through the transpose load. Each wave keeps its own dK and
// dV; the four are added in wave order at the end, so results are bitwise
// reproducible. Query rows are loaded with a row's pieces on consecutive lanes
// and go through LDS also where they are operands by rows. (Strictly causal
// 1,024-row segment at 16K: 44 us with each lane loading its operand's pieces
// and the routing rows read entry by entry, 33 us so.)
template <int D, int G>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void rows_dkv_mfma_kernel(AttnArgs a,
                                                                                     int64_t n_rows) {
  constexpr int KW = kRowsDkvKeys;  // keys of this workgroup
  static_assert(KW == 16, "one 16 x 16 product per batch");
  constexpr int PR = 16 / G;        // rows of a batch
  constexpr int NS = D / 32;        // k steps of S and dP
  constexpr int NT = D / 16;        // 16-column tiles of dK and dV
  constexpr int QP = D * 2 + 16;    // LDS pitch of a staged Q / dO row (padded against bank conflicts)
  __shared__ int s_rows[kRowsBwdMaxRows];  // the row lists live in LDS: calls of at most this many rows
  __shared__ uint32_t s_mask[kRowsBwdMaxRows];
  __shared__ int s_cnt[4];
  // each wave's Q and dO rows of its current batch; at the end, its partial dV, then dK
  __shared__ __attribute__((aligned(16))) char s_st[4][2][16 * QP];
  static_assert(KW * D * 4 <= 2 * 16 * QP, "a wave's partial dK or dV fits its staging buffer");
  typedef __attribute__((address_space(3))) s16x4* lds_s4;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.x % a.n_kv_heads;
  const int part = (blockIdx.x / a.n_kv_heads) % (64 / KW);
  const int64_t c = a.grad_begin / 64 + blockIdx.x / a.n_kv_heads / (64 / KW);  // absolute chunk
  const int64_t k0 = c * 64 + part * KW;  // this workgroup's first key
  const int64_t q_end = a.q_begin + n_rows;

  const int L = rows_attending<KW>(a, n_rows, h, c, part, s_rows, s_mask, s_cnt);

  // lane l: key kk of the workgroup (B column of S and dP, pair row of their
  // A), and quad, which selects the eight-value k slices it holds
  const int kk = lane & 15, quad = lane >> 4;
  const int64_t tk = min(k0 + kk, q_end - 1);  // keys past the call's end are never attended
  const char* kr = row_ptr(static_cast<const char*>(a.K), tk, a.k_tok * 2) + (int64_t)h * a.k_head * 2;
  const char* vr = row_ptr(static_cast<const char*>(a.V), tk, a.v_tok * 2) + (int64_t)h * a.v_head * 2;
  u32x4 kb[NS], vb[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    kb[s] = *reinterpret_cast<const u32x4*>(kr + (4 * s + quad) * 16);
    vb[s] = *reinterpret_cast<const u32x4*>(vr + (4 * s + quad) * 16);
  }
  f32x4 dk[NT], dv[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) dk[t] = dv[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  // a batch's operands: this lane's share of its Q and dO rows (16-byte
  // pieces, a row's pieces on consecutive lanes) and the softmax data of its
  // four result pairs 4 quad + i; entries past the list repeat its last row
  // and attend nothing
  constexpr int PPR = D / 8, RPI = 64 / PPR;  // pieces of a row, rows per load instruction
  constexpr int NJ = 16 / RPI;
  const int lr = lane / PPR, lp = lane % PPR;
  struct Batch {
    u32x4 q[NJ], d[NJ];
    float lse[4], dd[4];
    uint32_t att;
  };
  auto fetch = [&](int kb0, Batch& b) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int p = RPI * j + lr;
      const int64_t ra = s_rows[min(kb0 + p / G, L - 1)];
      const int64_t hqa = (int64_t)h * G + p % G;
      b.q[j] = *reinterpret_cast<const u32x4*>(static_cast<const char*>(a.Q) + (ra * a.q_tok + hqa * a.q_head) * 2 + 16 * lp);
      b.d[j] = *reinterpret_cast<const u32x4*>(static_cast<const char*>(a.dO) + (ra * a.do_tok + hqa * a.do_head) * 2 + 16 * lp);
    }
    b.att = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int p = 4 * quad + i, e = kb0 + p / G, ec = min(e, L - 1);
      const int64_t x = (int64_t)s_rows[ec] * a.n_q_heads + h * G + p % G;
      b.lse[i] = a.lse[x] * kLog2e;
      b.dd[i] = a.dvec[x];
      if (e < L && ((s_mask[ec] >> kk) & 1u)) b.att |= 1u << i;
    }
  };
  char* sq = s_st[wave][0];
  char* sdo = s_st[wave][1];
  const int rd = (4 * quad + (kk >> 2)) * QP + 4 * (kk & 3) * 2;  // this lane's transpose-load address in a tile
  Batch cur;
  if (wave * PR < L) fetch(wave * PR, cur);
  for (int kb0 = wave * PR; kb0 < L; kb0 += 4 * PR) {
    Batch nxt;
    if (kb0 + 4 * PR < L) fetch(kb0 + 4 * PR, nxt);  // the next batch's loads are in flight during this one
    // the batch's Q and dO rows into this wave's staging tiles (row = pair),
    // and from there as operands
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      *reinterpret_cast<u32x4*>(sq + (RPI * j + lr) * QP + 16 * lp) = cur.q[j];
      *reinterpret_cast<u32x4*>(sdo + (RPI * j + lr) * QP + 16 * lp) = cur.d[j];
    }
    __builtin_amdgcn_wave_barrier();
    f32x4 sacc = {0.0f, 0.0f, 0.0f, 0.0f}, pacc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int off = kk * QP + (4 * s + quad) * 16;
      sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8*>(sq + off),
                                                     __builtin_bit_cast(bf16x8, kb[s]), sacc, 0, 0, 0);
      pacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8*>(sdo + off),
                                                     __builtin_bit_cast(bf16x8, vb[s]), pacc, 0, 0, 0);
    }
    // P and dS = P (dP - D) of pairs 4 quad + i against key kk
    s16x4 pa, pl, sa, sl;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float pr = (cur.att >> i) & 1u ? exp2f(sacc[i] * a.scale_log2 - cur.lse[i]) : 0.0f;
      const float ds = pr * (pacc[i] - cur.dd[i]);
      const uint32_t ph = float_to_bf16_bits(pr), dh = float_to_bf16_bits(ds);
      pa[i] = (short)ph;
      pl[i] = (short)float_to_bf16_bits(pr - bf16_bits_to_float(ph));
      sa[i] = (short)dh;
      sl[i] = (short)float_to_bf16_bits(ds - bf16_bits_to_float(dh));
    }
    // dV += P^T dO and dK += dS^T Q, sixteen columns per product
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const s16x4 bo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(sdo + rd + 32 * t));
      const s16x4 bq = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(sq + rd + 32 * t));
      dv[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pa, bo, dv[t], 0, 0, 0);
      dv[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pl, bo, dv[t], 0, 0, 0);
      dk[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(sa, bq, dk[t], 0, 0, 0);
      dk[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(sl, bq, dk[t], 0, 0, 0);
    }
    __builtin_amdgcn_wave_barrier();
    cur = nxt;
  }
  // the four waves' partial dV, then dK, added in wave order; lane l holds
  // keys 4 quad + i, column 16 t + kk
  __syncthreads();
  for (int which = 0; which < 2; ++which) {
    float* pd = reinterpret_cast<float*>(s_st[wave]);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) pd[(4 * quad + i) * D + 16 * t + kk] = which == 0 ? dv[t][i] : dk[t][i];
    __syncthreads();
    for (int x = tid; x < KW * D / 4; x += 256) {
      const int key = x / (D / 4), col = 4 * (x % (D / 4));
      f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int w = 0; w < 4; ++w) acc += *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(s_st[w]) + key * D + col);
      const int64_t t = k0 + key;
      if (t < q_end) {  // keys of this workgroup that exist in this call (all tokens >= grad_begin)
        float* dst = (which == 0 ? a.dV : a.dK) + ((t - a.grad_begin) * a.n_kv_heads + h) * D + col;
        *reinterpret_cast<f32x4*>(dst) = which == 0 ? acc : acc * a.scale;
      }
    }
    __syncthreads();
  }
}

// Workgroups of the dK/dV kernels: 16 keys of an active chunk, kv head.
static dim3 rows_dkv_grid(const AttnArgs& a, int64_t n_rows) {
  const int n_act = (int)((a.q_begin + n_rows - a.grad_begin + 63) / 64);
  return dim3((unsigned)(n_act * a.n_kv_heads * (64 / kRowsDkvKeys)));
}

template <int D, int G>
hipError_t rows_bwd_mfma(const AttnArgs& a, int64_t n_rows, hipStream_t s) {
  constexpr int R = rows_per_group<G>();
  const int64_t ng = n_row_groups(a, n_rows, R);
  const dim3 each((unsigned)(n_rows * a.n_kv_heads));
  if (ng * a.n_kv_heads >= kRowsWaveGroups)
    hipLaunchKernelGGL((rows_dq_mfma_kernel<D, G, R, 1>), dim3((unsigned)((ng + 3) / 4 * a.n_kv_heads)), dim3(256), 0,
                       s, a, n_rows, ng);
  else if (!rows_apart(a, n_rows, R, 512))
    hipLaunchKernelGGL((rows_dq_mfma_kernel<D, G, R, 4>), dim3((unsigned)(ng * a.n_kv_heads)), dim3(256), 0, s, a,
                       n_rows, ng);
  else if (many_waves(a, n_rows))
    hipLaunchKernelGGL((rows_dq_mfma_kernel<D, G, 1, 8>), each, dim3(512), 0, s, a, n_rows, n_rows);
  else
    hipLaunchKernelGGL((rows_dq_mfma_kernel<D, G, 1, 4>), each, dim3(256), 0, s, a, n_rows, n_rows);
  hipLaunchKernelGGL((rows_dkv_mfma_kernel<D, G>), rows_dkv_grid(a, n_rows), dim3(256), 0, s, a, n_rows);
  return hipGetLastError();
}

template <int D>
hipError_t rows_bwd_bf16(const AttnArgs& a, int64_t n_rows, hipStream_t s) {
  switch (a.gqa) {
    case 1: return rows_bwd_mfma<D, 1>(a, n_rows, s);
    case 2: return rows_bwd_mfma<D, 2>(a, n_rows, s);
    case 4: return rows_bwd_mfma<D, 4>(a, n_rows, s);
    default: return rows_bwd_mfma<D, 8>(a, n_rows, s);
  }
}

template <int G>
hipError_t rows_bwd_f32(const AttnArgs& a, int64_t n_rows, hipStream_t s) {
  const int64_t pairs = n_rows * a.n_q_heads;
  hipLaunchKernelGGL(rows_rowdot_kernel, dim3((unsigned)((pairs + 3) / 4)), dim3(256), 0, s, a, n_rows);
  hipLaunchKernelGGL(rows_dq_kernel<G>, dim3((unsigned)(n_rows * a.n_kv_heads)), dim3(256), 0, s, a);
  hipLaunchKernelGGL(rows_dkv_kernel<G>, rows_dkv_grid(a, n_rows), dim3(256), 0, s, a, n_rows);
  return hipGetLastError();
}

hipError_t launch_attend_rows_bwd(const AttnArgs& a, int64_t n_rows, bool bf16, int head_dim, hipStream_t s) {
  if (bf16) return head_dim == 64 ? rows_bwd_bf16<64>(a, n_rows, s) : rows_bwd_bf16<128>(a, n_rows, s);
  switch (a.gqa) {
    case 1: return rows_bwd_f32<1>(a, n_rows, s);
    case 2: return rows_bwd_f32<2>(a, n_rows, s);
    case 4: return rows_bwd_f32<4>(a, n_rows, s);
    default: return rows_bwd_f32<8>(a, n_rows, s);
  }
}

}  // namespace hga
