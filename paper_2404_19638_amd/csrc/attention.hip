// Fused masked attention forward over a localized block (an extension built
// on the paper's two kernels, not part of the paper).  For every stored entry
// p of local row i with column j:
//
//   score  e_p     = <q_i, k_j>                          (SDDMM, Eq. (1), s == 1)
//   weight alpha_p = exp(e_p - m_i) / s_i,  m_i = max of row i's scores,
//                    s_i = sum over row i of exp(e_q - m_i)
//   output out_i   = sum_p alpha_p v_j                   (SpMM, Eq. (2))
//
// in one pass over the block, so neither the scores nor the weights are
// written to memory (the SDDMM -> softmax -> SpMM fusion the paper's related
// work calls FusedMM).  Each row segment keeps a running triple (m, s, a): the
// largest score so far, the sum of exp(e - m) and the sum of exp(e - m) v.  A
// new score e costs one exponential: when e > m the sums so far are rescaled
// by exp(m - e) and e becomes the maximum, otherwise exp(e - m) is added.  Two
// partial triples of one row merge by rescaling both to the larger maximum.
// At the row's end out_i = a / s, and (m_i, s_i) are stored so that the
// backward pass can rebuild alpha from recomputed scores.
//
// Work decomposition.  Group g (LPN lanes) of a wavefront owns the contiguous
// run of S = 2^lg_s slots [b + g*S, b + (g+1)*S) of its work item (S <= 64,
// so a run lies inside one 64-bit head word), walked in steps of U slots.  The
// item's column indices are staged in LDS, so that the loop waits for gathered
// rows only (vector loads return in order: an index load that misses to HBM
// would hold back the rows issued after it); the U key and value rows of a
// step (and the query rows of the rows that start in it) are loaded as raw
// 16-byte vectors before any is used.  A step's scores come first, then each
// slot's running maximum, and then one evaluation of the exponential serves
// the step, lane u of every quad computing slot u's.  Row triples are finished
// where the next row starts; the part of a row before a run's first row start
// (kept in LDS) and the part after its last meet in a segmented suffix scan
// over the groups (shuffles, log2 G steps), and rows cut by work-item
// boundaries leave head / tail carries that k_attn_fixup merges in a fixed
// order.  All merge orders depend only on the structure, so results are
// deterministic.
//
// What bounds it: vector instructions.  At R-MAT 2^18, degree 32, bfloat16,
// K = 64 it issues 87.6 million (92 per slot of eight groups), 143 of 159 us
// at four cycles each on 1024 SIMDs and 2.4 GHz; the 790 MB read beyond L2
// take 121 us at the card's copy rate, underneath.  The count is that of the
// kernel before; what went is the waiting.  Registers decide how much overlaps:
// 92 for bfloat16 rows of 128 bytes, five wavefronts a SIMD; a second loop body
// for steps without a row start needed 118 to 156 and took 180 to 192 us.
// us before and after (MI355X, inference, bfloat16, K = 64): R-MAT 2^18,
// degree 32 218 to 159, degree 8 91 to 65; 2^16, degree 32 69 to 54; 2^14,
// degree 16 48 to 23; FP32 2^16, degree 32 93 to 73.
#include <cmath>

#include "run.h"

namespace spc3d {

template <int NCH, int VEC>
struct Tri {
  float m, s;
  float a[NCH][VEC];
};

template <int NCH, int VEC>
__device__ inline void tri_init(Tri<NCH, VEC>& t) {
  t.m = -INFINITY;
  t.s = 0.f;
  zero(t.a);
}

// x <- x (+) y: both rescaled to the larger maximum (equal maxima, including
// two empty triples, scale by exactly 1).
template <int NCH, int VEC>
__device__ inline void tri_merge(Tri<NCH, VEC>& x, const Tri<NCH, VEC>& y) {
  const float m = fmaxf(x.m, y.m);
  const float cx = (x.m == m) ? 1.f : expf(x.m - m);
  const float cy = (y.m == m) ? 1.f : expf(y.m - m);
  x.s = fmaf(x.s, cx, y.s * cy);
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
    for (int k = 0; k < VEC; ++k) x.a[ch][k] = fmaf(x.a[ch][k], cx, y.a[ch][k] * cy);
  x.m = m;
}

// Adds score e with value row v to a triple of maximum m; x = exp(-|e - m|).
template <int NCH, int VEC>
__device__ inline void tri_push(Tri<NCH, VEC>& t, float e, float m, float x,
                                const float (&v)[NCH][VEC]) {
  const bool up = e > m;
  const float c = up ? x : 1.f;
  const float p = up ? 1.f : x;
  t.s = fmaf(t.s, c, p);
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
    for (int k = 0; k < VEC; ++k) t.a[ch][k] = fmaf(t.a[ch][k], c, p * v[ch][k]);
  t.m = up ? e : m;
}

template <int NCH, int VEC>
__device__ inline void tri_shfl(const Tri<NCH, VEC>& t, Tri<NCH, VEC>& o, int from) {
  o.m = __shfl(t.m, from);
  o.s = __shfl(t.s, from);
  shfl_vec<VEC, NCH>(t.a, o.a, from);
}

// Carry record of kz + 4 floats: the kz weighted sums, then m and s.
template <int LPN, int NCH, int VEC>
__device__ inline void tri_store(float* __restrict__ rec, int kz, int nvec, int q,
                                 const Tri<NCH, VEC>& t) {
  store_vec<VEC, NCH>(rec, nvec, q, LPN, t.a);
  if (q == 0) {
    rec[kz] = t.m;
    rec[kz + 1] = t.s;
  }
}

template <int LPN, int NCH, int VEC>
__device__ inline void tri_load(const float* __restrict__ rec, int kz, int nvec, int q,
                                Tri<NCH, VEC>& t) {
  zero(t.a);
  add_vec<VEC, NCH>(rec, nvec, q, LPN, t.a);
  t.m = rec[kz];
  t.s = rec[kz + 1];
}

// out row i = a / s; stats[2i] = m, stats[2i+1] = s.
template <int LPN, int NCH, int VEC>
__device__ inline void tri_finish(float* __restrict__ out, float* __restrict__ stats, int64_t row,
                                  int kz, int nvec, int q, const Tri<NCH, VEC>& t) {
  // a / s by the reciprocal and one residual step: within an ulp of the
  // correctly rounded quotient's last bit, at half the instructions of a
  // division per element
  const float inv = 1.f / t.s;
  float o[NCH][VEC];
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
    for (int k = 0; k < VEC; ++k) {
      const float d = t.a[ch][k] * inv;
      const float e = fmaf(fmaf(-d, t.s, t.a[ch][k]), inv, d);
      o[ch][k] = fabsf(d) < INFINITY ? e : d;   // an infinite sum has no residual
    }
  store_row<VEC, NCH>(out, row, kz, nvec, q, LPN, o, 0);
  if (stats && q == 0) {
    stats[2 * row] = t.m;
    stats[2 * row + 1] = t.s;
  }
}

// Loads this lane's vectors of the row at byte offset off.
template <int LPN, int NCH, typename Off>
__device__ inline void load_raw(const char* __restrict__ base, Off off, int q, uint4 (&r)[NCH]) {
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
    r[ch] = *reinterpret_cast<const uint4*>(base + (off + (Off)((q + ch * LPN) * 16)));
}

// Byte offset of row i: 32 bits (ids of 24 and operands below 4 GiB) or 64.
__device__ inline void row_offset(int i, uint32_t ldb, uint32_t& off) {
  off = __umul24((uint32_t)i, ldb);
}
__device__ inline void row_offset(int i, uint32_t ldb, uint64_t& off) { off = (uint64_t)i * ldb; }

// Keeps the conversion of a raw row where it is used: hoisted above the row
// ends of a step, the converted rows of all its slots would be live together.
template <int NCH>
__device__ inline void pin_raw(uint4 (&r)[NCH]) {
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
    asm volatile("" : "+v"(r[ch].x), "+v"(r[ch].y), "+v"(r[ch].z), "+v"(r[ch].w));
}

// Lane u of this lane's group (groups of 4 or more lanes: lane u of the own
// quad, which holds the same slot).
__device__ inline int quad_bcast(int v, int u) {
  switch (u) {
    case 0: return __builtin_amdgcn_update_dpp(v, v, 0x00, 0xF, 0xF, true);
    case 1: return __builtin_amdgcn_update_dpp(v, v, 0x55, 0xF, 0xF, true);
    case 2: return __builtin_amdgcn_update_dpp(v, v, 0xAA, 0xF, 0xF, true);
    default: return __builtin_amdgcn_update_dpp(v, v, 0xFF, 0xF, 0xF, true);
  }
}

// The part of a row that runs into a lane's run, kept in LDS until the scan.
template <int NCH, int VEC>
constexpr int kLeadWords = NCH * VEC + 2;

template <int NCH, int VEC>
__device__ inline void lead_put(float* __restrict__ s, const Tri<NCH, VEC>& t) {
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
    for (int k = 0; k < VEC; ++k) s[(ch * VEC + k) * 64] = t.a[ch][k];
  s[NCH * VEC * 64] = t.m;
  s[(NCH * VEC + 1) * 64] = t.s;
}

template <int NCH, int VEC>
__device__ inline void lead_get(const float* __restrict__ s, Tri<NCH, VEC>& t) {
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
    for (int k = 0; k < VEC; ++k) t.a[ch][k] = s[(ch * VEC + k) * 64];
  t.m = s[NCH * VEC * 64];
  t.s = s[(NCH * VEC + 1) * 64];
}

// Lanes of a group cover the row exactly: LPN * NCH * VEC == kz.
template <typename T, int VEC, int LPN, int NCH, int U, typename Off>
__global__ __launch_bounds__(256) void k_attn_fwd(int64_t nnz, int64_t nitems, int64_t nblocks,
                                                  int lg_s, const int32_t* __restrict__ idx,
                                                  const uint64_t* __restrict__ head,
                                                  const int32_t* __restrict__ tile_row,
                                                  const char* __restrict__ Q,
                                                  const char* __restrict__ Kf,
                                                  const char* __restrict__ V, int kz,
                                                  float* __restrict__ out,
                                                  float* __restrict__ stats,
                                                  float* __restrict__ carry) {
  static_assert(LPN >= 4 && LPN <= 16 && (U == 2 || U == 4), "attention shape");
  using Tr = Tri<NCH, VEC>;
  constexpr int G = 64 / LPN;
  extern __shared__ __align__(16) char smem[];
  const int lane = threadIdx.x & 63, g = lane / LPN, q = lane % LPN;
  const int64_t item = xcd_block(nblocks) * 4 + (threadIdx.x >> 6);
  if (item >= nitems) return;   // uniform per wavefront; no barriers below
  const int S = 1 << lg_s, P = S + 4;
  const int64_t W = (int64_t)G << lg_s;
  const int64_t b = item * W;
  const int64_t e = (b + W < nnz) ? b + W : nnz;
  const int64_t gs = b + ((int64_t)g << lg_s);
  const int nrun = gs >= e ? 0 : (e - gs < S ? (int)(e - gs) : S);
  const int nvec = kz / VEC;
  const int CS = kz + 4;
  const uint32_t ldb = (uint32_t)kz * (uint32_t)sizeof(T);
  const bool ends_at_e = (e >= nnz) || is_head(head, e);
  int* s_col = reinterpret_cast<int*>(smem) + (threadIdx.x >> 6) * (G * P + 64 * kLeadWords<NCH, VEC>);
  float* s_lead = reinterpret_cast<float*>(s_col + G * P) + lane;   // this lane's, 64 apart
  for (int i = lane; i < (int)W; i += 64)
    s_col[(i >> lg_s) * P + (i & (S - 1))] = b + i < e ? ld_stream(idx + b + i) : 0;

  // head bits of the run (bit t: slot gs + t starts a row) and the row of gs
  const int64_t gw = (gs < nnz ? gs : nnz - 1) >> 6;
  const uint64_t hword = head[gw];
  const int sh = (int)(gs & 63);
  const uint64_t vmask = nrun >= 64 ? ~0ull : ((1ull << nrun) - 1ull);
  uint64_t run = (hword >> sh) & vmask;
  const bool first = run & 1ull;
  run &= ~1ull;
  int r = tile_row[gw] + __popcll(hword & lanemask_le(sh) & ~1ull);

  Tr cur;
  tri_init(cur);
  float qv[NCH][VEC];   // the current row of Q
  Off qoff;
  row_offset(r, ldb, qoff);
  {
    uint4 q0[NCH];
    load_raw<LPN, NCH>(Q, qoff, q, q0);
    unpack_raw<T, VEC, NCH>(q0, qv);
  }
  bool seen = first;
  const int steps = S / U;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  for (int m = 0; m < steps; ++m) {
    int col[U];
    read_words<U>(s_col + g * P + m * U, col);
    const unsigned hb = (unsigned)run & ((1u << U) - 1u);
    run >>= U;
    uint4 kr[U][NCH], vr[U][NCH], qr[U][NCH];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      Off off;
      row_offset(col[u], ldb, off);
      load_raw<LPN, NCH>(Kf, off, q, kr[u]);
      load_raw<LPN, NCH>(V, off, q, vr[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if ((hb >> u) & 1u) {
        qoff += ldb;
        load_raw<LPN, NCH>(Q, qoff, q, qr[u]);
      }
    }
    float sc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if ((hb >> u) & 1u) unpack_raw<T, VEC, NCH>(qr[u], qv);
      float kx[NCH][VEC];
      pin_raw<NCH>(kr[u]);
      unpack_raw<T, VEC, NCH>(kr[u], kx);
      float d = 0.f;
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
        for (int k = 0; k < VEC; ++k) d = fmaf(qv[ch][k], kx[ch][k], d);
      sc[u] = group_sum<LPN>(d);
    }
    // the row maximum before each slot, and from it the slot's exponential
    // (lane u of each quad computes slot u's)
    float before[U], x = 0.f;
    float top = cur.m;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      before[u] = ((hb >> u) & 1u) ? -INFINITY : top;
      top = sc[u] > before[u] ? sc[u] : before[u];
      const float below = (sc[u] == before[u]) ? 0.f : -fabsf(sc[u] - before[u]);
      x = (q & 3) == u ? below : x;
    }
    const int y = __float_as_int(expf(x));
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if ((hb >> u) & 1u) {   // the row before this slot is complete
        if (seen)
          tri_finish<LPN, NCH, VEC>(out, stats, r, kz, nvec, q, cur);
        else
          lead_put<NCH, VEC>(s_lead, cur);
        tri_init(cur);
        ++r;
        seen = true;
      }
      if (m * U + u < nrun) {
        float vx[NCH][VEC];
        pin_raw<NCH>(vr[u]);
        unpack_raw<T, VEC, NCH>(vr[u], vx);
        tri_push(cur, sc[u], before[u], __int_as_float(quad_bcast(y, u)), vx);
      }
    }
  }

  // (P, f): the run's lead (the whole run when no row starts in it) and
  // whether a row starts in the run.  Suffix scan over the groups:
  // Sv_g = P_g (+) Sv_{g+1} unless f_g;  F_g = f_g | F_{g+1}.
  const bool f = seen;
  Tr sv = cur;
  if (f) {
    tri_init(sv);   // a run that starts with a row has no lead
    if (!first) lead_get<NCH, VEC>(s_lead, sv);
  }
  bool F = f;
#pragma unroll
  for (int d = 1; d < G; d <<= 1) {
    const bool inr = g + d < G;
    const int src = inr ? lane + d * LPN : lane;
    Tr o;
    tri_shfl(sv, o, src);
    const bool of = __shfl((int)F, src) != 0;
    if (inr && !F) tri_merge(sv, o);
    F = F || (inr && of);
  }
  const bool has_next = g + 1 < G;
  const int nsrc = has_next ? lane + LPN : lane;
  Tr nx;
  tri_shfl(sv, nx, nsrc);
  const bool nF = (__shfl((int)F, nsrc) != 0) && has_next;
  if (f) {
    // the run's last row: its tail and the leads of the runs it continues into
    if (has_next) tri_merge(cur, nx);
    if (nF || ends_at_e)
      tri_finish<LPN, NCH, VEC>(out, stats, r, kz, nvec, q, cur);
    else
      tri_store<LPN, NCH, VEC>(carry + (item * 2 + 1) * CS, kz, nvec, q, cur);
  }
  // the item starts inside a row: its head carry for the row's owner
  if (g == 0 && nrun > 0 && !first)
    tri_store<LPN, NCH, VEC>(carry + (item * 2) * CS, kz, nvec, q, sv);
}

// Rows cut by item boundaries: item j whose last row starts inside it and
// runs past its end owns the row; it merges its tail carry with the head
// carries of the items the row runs through (blocked per group, then a
// butterfly over the groups: a fixed order).
template <int VEC, int LPN, int NCH>
__global__ __launch_bounds__(256) void k_attn_fixup(int64_t nnz, int64_t nitems, int64_t wslots,
                                                    const int32_t* __restrict__ ptr,
                                                    const uint64_t* __restrict__ head,
                                                    const int32_t* __restrict__ tile_row, int kz,
                                                    float* __restrict__ out,
                                                    float* __restrict__ stats,
                                                    const float* __restrict__ carry) {
  using Tr = Tri<NCH, VEC>;
  constexpr int G = 64 / LPN;
  constexpr int BLK = 16;
  const int lane = threadIdx.x & 63, g = lane / LPN, q = lane % LPN;
  const int64_t j = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (j >= nitems) return;
  const int64_t b = j * wslots, e = b + wslots;
  if (e >= nnz) return;
  const int nvec = kz / VEC;
  const int CS = kz + 4;
  // the common case, a row that ends in item j + 1, needs these two carries:
  // their loads overlap the look-up of the row
  Tr res, tot;
  tri_load<LPN, NCH, VEC>(carry + (j * 2 + 1) * CS, kz, nvec, q, res);
  tri_load<LPN, NCH, VEC>(carry + ((j + 1) * 2) * CS, kz, nvec, q, tot);
  if (is_head(head, e)) return;
  const int r = row_of(head, tile_row, e - 1);
  const int64_t start = ptr[r], end = ptr[r + 1];
  if (start < b) return;
  const int64_t jl = (end - 1) / wslots;
  if (jl > j + 1) {
    tri_init(tot);
    for (int64_t j0 = j + 1 + g; j0 <= jl; j0 += (int64_t)G * BLK) {
      Tr blk;
      tri_init(blk);
      for (int m = 0; m < BLK; ++m) {
        const int64_t jj = j0 + (int64_t)m * G;
        if (jj > jl) break;
        Tr c;
        tri_load<LPN, NCH, VEC>(carry + (jj * 2) * CS, kz, nvec, q, c);
        tri_merge(blk, c);
      }
      tri_merge(tot, blk);
    }
#pragma unroll
    for (int m = G / 2; m >= 1; m >>= 1) {
      Tr o;
      tri_shfl(tot, o, lane ^ (m * LPN));
      tri_merge(tot, o);
    }
  }
  if (g == 0) {
    tri_merge(res, tot);
    tri_finish<LPN, NCH, VEC>(out, stats, r, kz, nvec, q, res);
  }
}

namespace {

struct AttnShape {
  int vec, lanes, nch, lg_s;
};

// variant: -1, or lg_lanes (bits 0-3, 2..4) | lg_s << 4 (4..6).
spc3d_status attn_shape(int32_t kz, spc3d_dtype t, int variant, int64_t nnz, AttnShape* sh) {
  sh->vec = t == SPC3D_F32 ? 4 : 8;
  if (kz % sh->vec != 0)
    return fail(SPC3D_ERR_UNSUPPORTED, "fused attention needs kz %% %d == 0 (kz=%d)", sh->vec, kz);
  const int nvec = kz / sh->vec;
  if (variant < 0) {
    sh->lanes = nvec < 16 ? nvec : 16;
    // Runs of 64 slots, shorter where that leaves under 3500 wavefronts.  us for
    // runs of 16, 32, 64 (bfloat16, K = 64, eight groups): 261,000 entries 18.9,
    // 25.4, 39.6; 523,000 26.5, 29.0, 42.1; 2.09 million 73.0, 71.1, 70.2; 8.4
    // million 349, 338, 333.
    const int64_t groups = sh->lanes > 0 ? 64 / sh->lanes : 1;
    sh->lg_s = nnz >= 3500 * 64 * groups ? 6 : nnz >= 3500 * 32 * groups ? 5 : 4;
  } else {
    const int lg = variant & 15, lgs = (variant >> 4) & 15;
    if (lg < 2 || lg > 4 || lgs < 4 || lgs > 6 || (variant >> 8))
      return fail(SPC3D_ERR_INVALID_ARG, "bad attention variant %d", variant);
    sh->lanes = 1 << lg;
    sh->lg_s = lgs;
  }
  if (sh->lanes < 4 || nvec % sh->lanes != 0 || nvec / sh->lanes > 2 ||
      (sh->lanes & (sh->lanes - 1)))
    return fail(SPC3D_ERR_UNSUPPORTED, "fused attention does not cover kz=%d with %d lanes", kz,
                sh->lanes);
  sh->nch = nvec / sh->lanes;
  return SPC3D_OK;
}

int64_t attn_items(const Plan* p, const AttnShape& sh) {
  const int64_t W = (int64_t)(64 / sh.lanes) << sh.lg_s;
  return (p->nnz + W - 1) / W;
}

template <typename T, int VEC>
void launch_attn(const AttnShape& sh, hipStream_t st, const Plan* p, int64_t nitems,
                 const void* Q, const void* K, const void* V, int kz, float* out, float* stats,
                 float* carry) {
  const int64_t nblocks = (nitems + 3) / 4;
  const int64_t W = (int64_t)(64 / sh.lanes) << sh.lg_s;
  const size_t lds =
      (size_t)4 * 4 * ((64 / sh.lanes) * ((1 << sh.lg_s) + 4) + 64 * (sh.nch * VEC + 2));
  const char* q = static_cast<const char*>(Q);
  const char* k = static_cast<const char*>(K);
  const char* v = static_cast<const char*>(V);
  const int64_t most = p->R > p->C ? p->R : p->C;
  const bool small = most < (1 << 24) && most * kz * (int64_t)sizeof(T) < (int64_t(1) << 32);
#define SPC3D_ATTN_OFF(LPN, NCH, U, OFF)                                                         \
  hipLaunchKernelGGL((k_attn_fwd<T, VEC, LPN, NCH, U, OFF>), dim3((unsigned)nblocks), dim3(256), \
                     lds, st, p->nnz, nitems, nblocks, sh.lg_s, p->colidx, p->head, p->tile_row, \
                     q, k, v, kz, out, stats, carry)
#define SPC3D_ATTN(LPN, NCH, U)                                                                  \
  do {                                                                                           \
    if (small) SPC3D_ATTN_OFF(LPN, NCH, U, uint32_t);                                            \
    else SPC3D_ATTN_OFF(LPN, NCH, U, uint64_t);                                                  \
    hipLaunchKernelGGL((k_attn_fixup<VEC, LPN, NCH>), dim3((unsigned)((nitems + 3) / 4)),        \
                       dim3(256), 0, st, p->nnz, nitems, W, p->rowptr, p->head, p->tile_row, kz, \
                       out, stats, carry);                                                       \
  } while (0)
  if (sh.nch == 1) {
    if (sh.lanes == 4) SPC3D_ATTN(4, 1, 4);
    else if (sh.lanes == 8) SPC3D_ATTN(8, 1, 4);
    else SPC3D_ATTN(16, 1, 4);
  } else {
    if (sh.lanes == 4) SPC3D_ATTN(4, 2, 2);
    else if (sh.lanes == 8) SPC3D_ATTN(8, 2, 2);
    else SPC3D_ATTN(16, 2, 2);
  }
#undef SPC3D_ATTN
#undef SPC3D_ATTN_OFF
}

}  // namespace
}  // namespace spc3d

using namespace spc3d;

extern "C" {

spc3d_status spc3d_attention_fwd_buffer_size(spc3d_plan h, int32_t kz, spc3d_dtype t, int variant,
                                             size_t* bytes) {
  Plan* p;
  spc3d_status st = get_plan(h, &p);
  if (st != SPC3D_OK) return st;
  if (!bytes) return fail(SPC3D_ERR_INVALID_ARG, "bytes is NULL");
  if (t != SPC3D_F32 && t != SPC3D_BF16) return fail(SPC3D_ERR_INVALID_ARG, "bad dtype");
  if (kz < 1 || kz > kMaxKz) return fail(SPC3D_ERR_INVALID_ARG, "kz=%d outside [1,%d]", kz, kMaxKz);
  AttnShape sh;
  st = attn_shape(kz, t, variant, p->nnz, &sh);
  if (st != SPC3D_OK) return st;
  const int64_t nitems = attn_items(p, sh);
  *bytes = (size_t)(nitems > 0 ? nitems : 1) * 2 * (size_t)(kz + 4) * 4;
  return SPC3D_OK;
}

spc3d_status spc3d_attention_fwd(spc3d_plan h, const void* d_Q, const void* d_K, const void* d_V,
                                 spc3d_dtype t, int32_t kz, float* d_out, float* d_stats,
                                 int variant, void* d_buf, size_t buf_bytes, hipStream_t stream) {
  Plan* p;
  spc3d_status st = get_plan(h, &p);
  if (st != SPC3D_OK) return st;
  if (t != SPC3D_F32 && t != SPC3D_BF16) return fail(SPC3D_ERR_INVALID_ARG, "bad dtype");
  if (kz < 1 || kz > kMaxKz) return fail(SPC3D_ERR_INVALID_ARG, "kz=%d outside [1,%d]", kz, kMaxKz);
  AttnShape sh;
  st = attn_shape(kz, t, variant, p->nnz, &sh);
  if (st != SPC3D_OK) return st;
  if (p->nnz == 0) return SPC3D_OK;
  if (!d_Q || !d_K || !d_V || !d_out || !d_buf) return fail(SPC3D_ERR_INVALID_ARG, "NULL buffer");
  if (!aligned16(d_Q) || !aligned16(d_K) || !aligned16(d_V) || !aligned16(d_out))
    return fail(SPC3D_ERR_INVALID_ARG, "Q, K, V and out must be 16-byte aligned");
  if (d_stats && (reinterpret_cast<uintptr_t>(d_stats) & 7u))
    return fail(SPC3D_ERR_INVALID_ARG, "stats must be 8-byte aligned");
  if (reinterpret_cast<uintptr_t>(d_buf) & 255u)
    return fail(SPC3D_ERR_INVALID_ARG, "buffer must be 256-byte aligned");
  // shorter runs mean more carries: a buffer for fewer takes longer runs
  while (variant < 0 && sh.lg_s < 6 &&
         buf_bytes < (size_t)attn_items(p, sh) * 2 * (size_t)(kz + 4) * 4)
    ++sh.lg_s;
  const int64_t nitems = attn_items(p, sh);
  const size_t need = (size_t)nitems * 2 * (size_t)(kz + 4) * 4;
  if (buf_bytes < need)
    return fail(SPC3D_ERR_WORKSPACE, "attention buffer %zu bytes < %zu required", buf_bytes, need);
  DeviceGuard dg;
  st = dg.enter(p);
  if (st != SPC3D_OK) return st;
  SPC3D_DEBUG_CHECK(p, stream);
  float* carry = static_cast<float*>(d_buf);
  if (t == SPC3D_F32)
    launch_attn<float, 4>(sh, stream, p, nitems, d_Q, d_K, d_V, kz, d_out, d_stats, carry);
  else
    launch_attn<bf16_t, 8>(sh, stream, p, nitems, d_Q, d_K, d_V, kz, d_out, d_stats, carry);
  SPC3D_LAUNCHED("attention_fwd");
  return SPC3D_OK;
}

}  // extern "C"
