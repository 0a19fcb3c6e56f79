// SpMM and the fused SDDMM + SpMM pass, run family (k_run).
//
// Work decomposition.  A work item is W = G * S consecutive slots (G = 64 /
// LPN lane groups, S = 2^lg_s <= 64), one item per wavefront.  Group g walks
// the run of S slots [b + g*S, b + (g+1)*S) in steps of U: the U gathered rows
// (and, fused, the U rows of A) are loaded as raw 16-byte vectors before any
// is used.  The item's columns and values are staged in LDS first, so that the
// loop's only loads are the gathered rows: vector loads return in order, and
// an index load that misses to HBM would hold back every row load issued after
// it.  A row that starts and ends in a run is stored where the next one
// starts; the parts of rows that cross runs meet in a segmented suffix scan
// over the groups (shuffles, log2 G steps), and a row that crosses items
// leaves carries for k_run_fixup.  The summation order depends only on the
// structure, so results are deterministic.
//
// Rows whose width is not LPN * NCH * VEC elements (FULL = false) keep the
// 16-byte loads: the last lanes' vectors are moved back to end at the row's
// last element.  The elements such a vector shares with its neighbour are
// skipped in dots; in row sums both lanes compute and store the same value.
// Loads and stores need the element's alignment only.
//
// Columns [k0, k0 + kw) of the rows can be taken alone (a slice); blockIdx.y
// counts slices.
//
// What bounds it: the lines of gathered rows that miss L2.  Against the
// group-run family (k_spmm), which the default took before: 21.6M against 31.8M
// vector, 5.0M against 15.5M scalar and 0.9M against 2.2M LDS instructions (the
// fused pass on the share of a 2^24-vertex R-MAT graph, 4.1M entries, kz = 32), and
// in us, fused / SpMM, MI355X: the share 92.2 to 78.3 / 72.9 to 63.5; R-MAT 2^16 kz =
// 32 45.2 to 28.2 / 33.5 to 23.8, kz = 64 59.5 to 47.7 / 45.6 to 36.4; 2^18 kz = 32
// 139.9 to 95.6 / 92.1 to 79.2; kz = 30 (2^18, degree 16) 122.8 to 81.5 / 85.8 to
// 66.7.  Loading indices from global memory in the loop instead of staging them
// costs 20 to 40%: 109 us (fused, the share), 1057 against 834 us (2^20, kz = 64).
#pragma once

#include <type_traits>

#include "kernels.h"

namespace spc3d {

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_e4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4_e2 __attribute__((ext_vector_type(4), aligned(2)));

struct RunArgs {
  int64_t nnz, nitems, nblocks;
  int lg_s;
  int kz;                    // elements of a packed row: the stride of X, A and Y
  int kw;                    // elements taken of each row
  int k0;                    // first of them, for blockIdx.y = 0 (then kw more each)
  const int32_t* idx;
  const uint64_t* head;
  const int32_t* tile_row;
  const float* vals;         // nullptr: all ones
  const int32_t* vidx;       // slot of the value array, or nullptr (slot order)
  const char* X;
  const char* A;             // fused
  YOut Y;
  float* carry;
  float* out;                // fused
  int acc_out;
  float* dots;               // fused, PARTS: sums of the slices before this one
  int part_first, part_last; // fused, PARTS: this slice is the row's first, last
};

// Where a finished row goes.
enum { kPut = 0, kAddPacked = 1, kAddSlab = 2 };

// LDS words of one wavefront: an item's columns, then its values (fused: then
// its outputs), each run padded by 4 words so that the groups' 16-byte reads
// fall on different banks.
__host__ __device__ inline int run_words(int G, int S) { return 2 * G * (S + 4); }

template <int U>
__device__ inline void read_words(const int32_t* p, int32_t (&o)[U]) {
  if constexpr (U % 4 == 0) {
#pragma unroll
    for (int u = 0; u < U; u += 4) {
      const i32x4 c = *reinterpret_cast<const i32x4*>(p + u);
      o[u] = c.x; o[u + 1] = c.y; o[u + 2] = c.z; o[u + 3] = c.w;
    }
  } else if constexpr (U == 1) {
    o[0] = p[0];
  } else {
    static_assert(U == 2, "steps of 1, 2 or a multiple of 4 slots");
    const i32x2 c = *reinterpret_cast<const i32x2*>(p);
    o[0] = c.x; o[1] = c.y;
  }
}

// A lane's NCH vectors of a row: their first elements, and how many of each
// vector's elements belong to the lane before (0 when FULL).
template <int VEC, int LPN, int NCH, bool FULL>
struct LaneCols {
  uint32_t at[NCH];
  int32_t dup[NCH];
  __device__ inline LaneCols(int q, int kw) {
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      const int w = (q + ch * LPN) * VEC;
      const int m = FULL ? w : (w < kw - VEC ? w : kw - VEC);
      at[ch] = (uint32_t)m;
      dup[ch] = w - m;
    }
  }
};

template <typename T, int VEC, int LPN, int NCH, bool FULL>
__device__ inline void load_at(const char* __restrict__ base, uint32_t rowoff,
                               const LaneCols<VEC, LPN, NCH, FULL>& lc, uint4 (&r)[NCH]) {
  using V = typename std::conditional<sizeof(T) == 4, u32x4_e4, u32x4_e2>::type;
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    const V w = *reinterpret_cast<const V*>(base + (rowoff + lc.at[ch] * (uint32_t)sizeof(T)));
    r[ch] = make_uint4(w.x, w.y, w.z, w.w);
  }
}

template <int VEC, int LPN, int NCH, bool FULL, bool STREAM = FULL>
__device__ inline void put_at(float* __restrict__ row, const LaneCols<VEC, LPN, NCH, FULL>& lc,
                              const float (&acc)[NCH][VEC]) {
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
    for (int t = 0; t < VEC; t += 4) {
      const f32x4_e4 o = {acc[ch][t], acc[ch][t + 1], acc[ch][t + 2], acc[ch][t + 3]};
      f32x4_e4* y = reinterpret_cast<f32x4_e4*>(row + lc.at[ch] + t);
      if constexpr (STREAM)
        __builtin_nontemporal_store(o, y);
      else
        *y = o;   // lanes overlap: let the cache merge them
    }
}

template <int VEC, int LPN, int NCH, bool FULL>
__device__ inline void get_at(const float* __restrict__ row,
                              const LaneCols<VEC, LPN, NCH, FULL>& lc, float (&v)[NCH][VEC]) {
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
    for (int t = 0; t < VEC; t += 4) {
      const f32x4_e4 w = *reinterpret_cast<const f32x4_e4*>(row + lc.at[ch] + t);
      v[ch][t] = w.x; v[ch][t + 1] = w.y; v[ch][t + 2] = w.z; v[ch][t + 3] = w.w;
    }
}

template <int VEC, int NCH>
__device__ inline void add_to(float (&a)[NCH][VEC], const float (&b)[NCH][VEC]) {
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
    for (int t = 0; t < VEC; ++t) a[ch][t] += b[ch][t];
}

template <int VEC, int NCH>
__device__ inline void copy_to(float (&a)[NCH][VEC], const float (&b)[NCH][VEC]) {
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
    for (int t = 0; t < VEC; ++t) a[ch][t] = b[ch][t];
}

// Where vectors of neighbouring lanes overlap (FULL = false), every lane's loads
// of a row that is added to come before any lane's stores to it.  A lane's own
// vectors do not overlap, so only this keeps the compiler from storing one
// before it loads the next, which may hold elements of the neighbour's.
template <bool FULL>
__device__ inline void loads_before_stores() {
  if constexpr (!FULL) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// Puts (or adds) the finished local row r.  What a row is added to is read
// here, where the row ends.  Read with the step's gathered rows (kAhead) it holds U
// rows more in registers, which costs more wavefronts than the wait saves but on
// very short rows of cold slabs (folded pass, us, with the step / here: FP32 kz = 32, R-MAT 2^19, 13.6M entries, 251 / 197,
// 5.5M banded 169 / 128; kz = 60, R-MAT 2^17, 3.4M, 156 / 132; bfloat16 kz = 128,
// 3.4M, 288 / 184).
template <int OUTM, int VEC, int LPN, int NCH, bool FULL, bool STREAM = FULL>
__device__ inline void finish_row(const RunArgs& a, int64_t r, int k0,
                                  const LaneCols<VEC, LPN, NCH, FULL>& lc,
                                  const float (&acc)[NCH][VEC]) {
  const int64_t d = OUTM == kAddSlab ? a.Y.map[r] - a.Y.lo : r;
  float* row = a.Y.base + d * a.Y.ld + k0;
  if constexpr (OUTM == kPut) {
    put_at<VEC, LPN, NCH, FULL, STREAM>(row, lc, acc);
  } else {
    float v[NCH][VEC];
    get_at<VEC, LPN, NCH, FULL>(row, lc, v);
    loads_before_stores<FULL>();
    add_to<VEC, NCH>(v, acc);
    put_at<VEC, LPN, NCH, FULL>(row, lc, v);
  }
}

enum { kPlain = 0, kAhead = 1, kStream = 2 };

// AROW: how the fused pass gets its rows of A.
enum { kNoA = 0, kEachSlot = 1, kEachRow = 2 };

// DEST: kAhead, what the rows that end in a step are added to is read with the step's
// gathered rows, their map entries a step before that; kStream, ragged rows are stored past
// the caches (see pick_run).
//
// PARTS: a fused pass over one slice of several.  The slices' dots are summed
// in a.dots, and the last slice multiplies the sum by the entry's value: a
// product with a part of the dot could overflow, or be infinite with the other
// sign, where the product with the whole is not.
template <typename T, int VEC, int LPN, int NCH, int U, bool FULL, int AROW, int OUTM, bool PARTS,
          int DEST>
__global__ __launch_bounds__(256) void k_run(const RunArgs a) {
  constexpr bool FUSED = AROW != kNoA, AHEAD = DEST == kAhead;
  constexpr int G = 64 / LPN;
  static_assert(U <= LPN, "one lane per slot of a step");
  using LC = LaneCols<VEC, LPN, NCH, FULL>;
  extern __shared__ __align__(16) char smem[];
  const int lane = threadIdx.x & 63, g = lane / LPN, q = lane % LPN;
  const int64_t item = xcd_block(a.nblocks) * 4 + (threadIdx.x >> 6);
  if (item >= a.nitems) return;   // uniform per wavefront; no barriers below
  const int S = 1 << a.lg_s, W = G << a.lg_s, P = S + 4;
  const int kz = a.kz;
  const int k0 = a.k0 + (int)blockIdx.y * a.kw;
  const uint32_t ldb = (uint32_t)kz * (uint32_t)sizeof(T);
  const char* X = a.X + (size_t)k0 * sizeof(T);
  const char* A = FUSED ? a.A + (size_t)k0 * sizeof(T) : nullptr;
  float* carry = a.carry + item * 2 * kz + k0;
  int32_t* s_col = reinterpret_cast<int32_t*>(smem) + (threadIdx.x >> 6) * 2 * G * P;
  int32_t* s_val = s_col + G * P;
  const LC lc(q, a.kw);

  const int64_t b = item * W;
  const int64_t e = (b + W < a.nnz) ? b + W : a.nnz;
  for (int i = lane; i < W; i += 64) {
    const bool ok = b + i < e;
    const int at = (i >> a.lg_s) * P + (i & (S - 1));
    s_col[at] = ok ? ld_stream(a.idx + b + i) : 0;
    float v = 1.f;
    if (a.vals)
      v = ok ? (a.vidx ? a.vals[a.vidx[b + i]] : ld_stream(a.vals + b + i)) : 0.f;
    s_val[at] = __float_as_int(v);
  }
  const int64_t gs = b + ((int64_t)g << a.lg_s);
  const int nrun = gs >= e ? 0 : (e - gs < S ? (int)(e - gs) : S);
  const bool ends_at_e = (e >= a.nnz) || is_head(a.head, e);
  const int64_t gw = (gs < a.nnz ? gs : a.nnz - 1) >> 6;
  const uint64_t hword = a.head[gw];
  const int sh = (int)(gs & 63);
  const uint64_t vmask = nrun >= 64 ? ~0ull : ((1ull << nrun) - 1ull);
  uint64_t run = (hword >> sh) & vmask;   // bit t: a row starts at slot gs + t
  const int rbase = a.tile_row[gw] + __popcll(hword & lanemask_le(sh) & ~1ull);
  const bool first = run & 1ull;
  run &= ~1ull;
  bool seen = first;   // a row starts in the part of the run walked so far
  int r = rbase;
  uint32_t aoff = FUSED ? (uint32_t)rbase * ldb : 0u;

  float acc[NCH][VEC], lead[NCH][VEC];
  zero(acc);
  zero(lead);
  auto end_row = [&]() {
    finish_row<OUTM, VEC, LPN, NCH, FULL, FULL || DEST == kStream>(a, r, k0, lc, acc);
  };
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();

  auto walk = [&](auto ragged) {
    constexpr bool TAIL = decltype(ragged)::value;   // the block's last item
    const int steps = S / U;
    uint4 acur[AROW == kEachRow ? NCH : 1];   // the current row of A
    if constexpr (AROW == kEachRow) load_at<T, VEC, LPN, NCH, FULL>(A, aoff, lc, acur);
    int64_t place[AHEAD ? U : 1];
    auto look_up = [&](uint32_t ends, int rr) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if ((ends >> u) & 1u) place[u] = a.Y.map[rr++];   // used a step later
    };
    if constexpr (AHEAD) look_up((uint32_t)run & ((1u << U) - 1u), r);
    for (int m = 0; m < steps; ++m) {
      int32_t col[U], vb[U];
      read_words<U>(s_col + g * P + m * U, col);
      read_words<U>(s_val + g * P + m * U, vb);
      const uint32_t hb = (uint32_t)run & ((1u << U) - 1u);
      run >>= U;
      uint4 x[U][NCH], ar[FUSED ? U : 1][NCH];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        load_at<T, VEC, LPN, NCH, FULL>(X, __umul24((uint32_t)col[u], ldb), lc, x[u]);
        if constexpr (AROW == kEachSlot) {
          aoff += __umul24((hb >> u) & 1u, ldb);
          load_at<T, VEC, LPN, NCH, FULL>(A, aoff, lc, ar[u]);
        }
      }
      if constexpr (AROW == kEachRow) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if ((hb >> u) & 1u) {
            aoff += ldb;
            load_at<T, VEC, LPN, NCH, FULL>(A, aoff, lc, ar[u]);
          }
        }
      }
      float held[AHEAD ? U : 1][NCH][VEC];
      float* dst[AHEAD ? U : 1];
      if constexpr (AHEAD) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if ((hb >> u) & 1u) {
            dst[u] = a.Y.base + (place[u] - a.Y.lo) * a.Y.ld + k0;
            get_at<VEC, LPN, NCH, FULL>(dst[u], lc, held[u]);
          }
        }
        if (m + 1 < steps) look_up((uint32_t)run & ((1u << U) - 1u), r + __popc(hb));
      }
      float res = 0.f;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float v = __int_as_float(vb[u]);
        float xv[NCH][VEC];
        unpack_raw<T, VEC, NCH>(x[u], xv);
        if ((hb >> u) & 1u) {   // the row before this slot is complete
          if (!seen) {
            copy_to<VEC, NCH>(lead, acc);
          } else if constexpr (AHEAD) {
            loads_before_stores<FULL>();
            add_to<VEC, NCH>(acc, held[u]);
            put_at<VEC, LPN, NCH, FULL>(dst[u], lc, acc);
          } else {
            end_row();
          }
          zero(acc);
          if constexpr (AROW == kEachRow) {
#pragma unroll
            for (int ch = 0; ch < NCH; ++ch) acur[ch] = ar[u][ch];
          }
          ++r;
          seen = true;
        }
        if constexpr (FUSED) {
          float av[NCH][VEC];
          if constexpr (AROW == kEachRow)
            unpack_raw<T, VEC, NCH>(acur, av);
          else
            unpack_raw<T, VEC, NCH>(ar[u], av);
          float d = 0.f;
#pragma unroll
          for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
            for (int t = 0; t < VEC; ++t) {
              const float f = fmaf(av[ch][t], xv[ch][t], d);
              d = (FULL || t >= lc.dup[ch]) ? f : d;
            }
          d = group_sum<LPN>(d);
          if constexpr (!PARTS) d = v * d;
          res = (q == u) ? d : res;
        }
        if (!TAIL || m * U + u < nrun) {
#pragma unroll
          for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
            for (int t = 0; t < VEC; ++t) acc[ch][t] = fmaf(v, xv[ch][t], acc[ch][t]);
        }
      }
      if constexpr (FUSED) {
        if (q < U) s_val[g * P + m * U + q] = __float_as_int(res);
      }
    }
  };
  if (b + W <= a.nnz)
    walk(std::false_type{});
  else
    walk(std::true_type{});

  if constexpr (FUSED) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int i = lane; i < (int)(e - b); i += 64) {
      float o = __int_as_float(s_val[(i >> a.lg_s) * P + (i & (S - 1))]);
      if constexpr (PARTS) {
        if (!a.part_first) o = ld_stream(a.dots + b + i) + o;
        if (!a.part_last) {
          st_stream(a.dots + b + i, o);
          continue;
        }
        if (a.vals) o = ld_stream(a.vals + b + i) * o;
      }
      st_stream(a.out + b + i, a.acc_out ? ld_stream(a.out + b + i) + o : o);
    }
  }
  // Segmented suffix scan: sv of group g is the part of the row that runs
  // into g, through the groups up to the first one in which a row starts.
  float sv[NCH][VEC];
  copy_to<VEC, NCH>(sv, acc);
  if (seen) copy_to<VEC, NCH>(sv, lead);
  bool F = seen;   // a row starts in group g or a later one scanned
#pragma unroll
  for (int d = 1; d < G; d <<= 1) {
    const bool inr = g + d < G;
    const int src = inr ? lane + d * LPN : lane;
    float o[NCH][VEC];
    shfl_vec<VEC, NCH>(sv, o, src);
    const bool of = __shfl((int)F, src) != 0;
    if (inr && !F) add_to<VEC, NCH>(sv, o);
    F = F || (inr && of);
  }
  const bool has_next = g + 1 < G;
  const int nsrc = has_next ? lane + LPN : lane;
  float nx[NCH][VEC];
  shfl_vec<VEC, NCH>(sv, nx, nsrc);
  const bool nF = (__shfl((int)F, nsrc) != 0) && has_next;
  if (seen) {
    // the run's last row, with the runs it continues into
    if (has_next) add_to<VEC, NCH>(acc, nx);
    if (nF || ends_at_e)
      end_row();
    else
      put_at<VEC, LPN, NCH, FULL>(carry + kz, lc, acc);
  }
  // the item starts inside a row: its part of that row
  if (g == 0 && !first) put_at<VEC, LPN, NCH, FULL>(carry, lc, sv);
}

// Rows cut by item boundaries: the item j in which such a row starts adds its
// tail carry and the head carries of the items the row runs through, in item
// order (blocked per group, then a butterfly over the groups).
template <int VEC, int LPN, int NCH, bool FULL, int OUTM>
__global__ __launch_bounds__(256) void k_run_fixup(const RunArgs a, const int32_t* __restrict__ ptr) {
  constexpr int G = 64 / LPN;
  constexpr int BLK = 16;
  using LC = LaneCols<VEC, LPN, NCH, FULL>;
  const int lane = threadIdx.x & 63, g = lane / LPN, q = lane % LPN;
  const int64_t j = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (j >= a.nitems) return;   // uniform per wavefront, as are the returns below
  const int64_t I = G << a.lg_s;
  const int64_t b = j * I, e = b + I;
  if (e >= a.nnz) return;      // the last item ends with the block
  const int kz = a.kz;
  const int k0 = a.k0 + (int)blockIdx.y * a.kw;
  const float* carry = a.carry + k0;
  const LC lc(q, a.kw);
  // the common case, a row that ends in item j + 1, needs these two carries:
  // their loads overlap the look-up of the row
  float tail[NCH][VEC], tot[NCH][VEC];
  get_at<VEC, LPN, NCH, FULL>(carry + (j * 2 + 1) * kz, lc, tail);
  get_at<VEC, LPN, NCH, FULL>(carry + (j + 1) * 2 * kz, lc, tot);
  if (is_head(a.head, e)) return;
  const int r = row_of(a.head, a.tile_row, e - 1);
  const int64_t start = ptr[r], end = ptr[r + 1];
  if (start < b) return;       // an earlier item owns the row
  const int64_t jl = (end - 1) / I;
  if (jl > j + 1) {
    zero(tot);
    for (int64_t j0 = j + 1 + g; j0 <= jl; j0 += (int64_t)G * BLK) {
      float blk[NCH][VEC];
      zero(blk);
      for (int m = 0; m < BLK; ++m) {
        const int64_t jj = j0 + (int64_t)m * G;
        if (jj > jl) break;
        float c[NCH][VEC];
        get_at<VEC, LPN, NCH, FULL>(carry + jj * 2 * kz, lc, c);
        add_to<VEC, NCH>(blk, c);
      }
      add_to<VEC, NCH>(tot, blk);
    }
#pragma unroll
    for (int m = G / 2; m >= 1; m >>= 1) {
      float o[NCH][VEC];
      shfl_vec<VEC, NCH>(tot, o, lane ^ (m * LPN));
      add_to<VEC, NCH>(tot, o);
    }
  }
  if (g == 0) {
    add_to<VEC, NCH>(tail, tot);
    finish_row<OUTM, VEC, LPN, NCH, FULL>(a, r, k0, lc, tail);
  }
}

// ------------------------------------------------------------------ launch

struct RunShape {
  int vec, lanes, nch;
  int lg_s;          // log2 of the run length
  int kw, slices;    // elements per slice, slices of a row
  bool full;         // lanes cover a slice exactly
  bool each_row;     // fused: a row of A is loaded where it starts, not for every slot
  bool ahead;        // adding: destinations are read with a step's gathered rows
  bool step4;        // putting: steps of 4 slots with two vectors a lane
  bool stream;       // putting: ragged rows are stored past the caches
  int64_t item() const { return (64 / lanes) << lg_s; }
};

// Launches the pass and its fix-up over slices [s0, s0 + ns) of the rows.
template <typename T, int VEC, bool FUSED>
void launch_run(const RunShape& sh, RunArgs a, int outm, const int32_t* ptr, int s0, int ns,
                hipStream_t st) {
  a.lg_s = sh.lg_s;
  a.kw = sh.kw;
  a.k0 = s0 * sh.kw;
  a.nitems = (a.nnz + sh.item() - 1) / sh.item();
  a.nblocks = (a.nitems + 3) / 4;
  const dim3 grid((unsigned)a.nblocks, (unsigned)ns);
  const size_t lds = (size_t)4 * 4 * run_words(64 / sh.lanes, 1 << sh.lg_s);
#define SPC3D_RUN_GO(L, N, U, F, M, O, P, H)                                                    \
  do {                                                                                          \
    hipLaunchKernelGGL((k_run<T, VEC, L, N, U, F, M, O, P, H>), grid, dim3(256), lds, st, a);    \
    hipLaunchKernelGGL((k_run_fixup<VEC, L, N, F, O>), grid, dim3(256), 0, st, a, ptr);          \
  } while (0)
#define SPC3D_RUN_H(L, N, U, F, M, O, P)                                       \
  do {                                                                         \
    if constexpr (O == kAddSlab && !P && N * VEC <= 8 && (F || VEC == 4)) {    \
      if (sh.ahead) SPC3D_RUN_GO(L, N, 4, F, M, O, P, kAhead);                 \
      else SPC3D_RUN_GO(L, N, U, F, M, O, P, kPlain);                          \
    } else if constexpr (O == kPut && !F && !P) {                              \
      if (sh.stream) SPC3D_RUN_GO(L, N, U, F, M, O, P, kStream);               \
      else SPC3D_RUN_GO(L, N, U, F, M, O, P, kPlain);                          \
    } else {                                                                   \
      SPC3D_RUN_GO(L, N, U, F, M, O, P, kPlain);                               \
    }                                                                          \
  } while (0)
#define SPC3D_RUN_A(L, N, U, F, O, P)                                          \
  do {                                                                         \
    if constexpr (!FUSED) SPC3D_RUN_H(L, N, U, F, kNoA, O, false);             \
    else if constexpr (N > 1) SPC3D_RUN_H(L, N, U, F, kEachRow, O, P);         \
    else if (sh.each_row) SPC3D_RUN_H(L, N, U, F, kEachRow, O, P);             \
    else SPC3D_RUN_H(L, N, U, F, kEachSlot, O, P);                             \
  } while (0)
// slices of a fused pass are 8 or 16 vectors, which 8 lanes cover
#define SPC3D_RUN_OUT(L, N, U, F, O)                                           \
  do {                                                                         \
    if constexpr (FUSED && L == 8 && N <= 2 &&                                 \
                  (F || (VEC == 8 && N == 2 && O != kPut))) {                  \
      if (sh.slices > 1) SPC3D_RUN_A(L, N, U, F, O, true);                     \
      else SPC3D_RUN_A(L, N, U, F, O, false);                                  \
    } else {                                                                   \
      SPC3D_RUN_A(L, N, U, F, O, false);                                       \
    }                                                                          \
  } while (0)
#define SPC3D_RUN_FULL(L, N, U, F)                                      \
  do {                                                                  \
    if (outm == kPut) SPC3D_RUN_OUT(L, N, U, F, kPut);                  \
    else if (outm == kAddPacked) SPC3D_RUN_OUT(L, N, U, F, kAddPacked); \
    else if constexpr (FUSED) SPC3D_RUN_OUT(L, N, U, F, kAddSlab);      \
  } while (0)
// Steps of 2 slots with two vectors a lane and of 1 with four: with steps twice
// as long two wavefronts a SIMD fewer fit (us, steps of 4 / 2, R-MAT 2^17, 3.4M
// entries: bfloat16 kz = 128 fused 107 / 104, folded 184 / 157; FP32 kz = 40
// folded 123 / 115; of 2 / 1, FP32 kz = 128 folded 231 / 178).  But steps of 4 with
// two vectors where rows are put and RunShape::step4 says so.  Adding, two
// bfloat16 vectors a lane take the general form, which fits 128 registers where
// the full one takes 129 (folded 156 / 130).
#define SPC3D_RUN_SHAPE(L, N, U)                                                    \
  if (sh.lanes == L && sh.nch == N) {                                               \
    if (sh.full && !(VEC == 8 && N == 2 && outm != kPut)) SPC3D_RUN_FULL(L, N, U, true); \
    else SPC3D_RUN_FULL(L, N, U, false);                                            \
  }
  SPC3D_RUN_SHAPE(4, 1, 4)
  SPC3D_RUN_SHAPE(8, 1, 4)
  if (outm == kPut && sh.step4 && sh.lanes == 8 && sh.nch == 2 &&
      (!FUSED || sh.slices == 1)) {
    if (sh.full) SPC3D_RUN_A(8, 2, 4, true, kPut, false);
    else SPC3D_RUN_A(8, 2, 4, false, kPut, false);
    return;
  }
  SPC3D_RUN_SHAPE(8, 2, 2)
  SPC3D_RUN_SHAPE(8, 4, 1)
#undef SPC3D_RUN_SHAPE
#undef SPC3D_RUN_FULL
#undef SPC3D_RUN_OUT
#undef SPC3D_RUN_A
#undef SPC3D_RUN_H
#undef SPC3D_RUN_GO
}

#define SPC3D_RUN_LAUNCH_ARGS const RunShape&, RunArgs, int, const int32_t*, int, int, hipStream_t

}  // namespace spc3d
