// PreComm / PostComm, local side: SpC-BB packing and unpacking of data units
// (paper: Section "Sparse communication model", Method 1 — copy each global
// id's data unit into a buffer; at the receiver, put each one back at the
// location of its global id).  Here a data unit is the K-slice [k0, k0+kz) of
// one dense row, the packed buffer holds the units of the block's non-empty
// rows (or columns) in local-id order, and unpacking reduces (+=) into the
// owner's rows as the SpMM PostComm does ("Building SpMM with SpComm3D").
//
// Both kernels move a row in chunks of 16 bytes of packed data (4 FP32 or 8
// bfloat16 values; 32 bytes of an FP32 source converted to bfloat16).  A
// wavefront takes `rpw` consecutive rows: it loads their global ids in one
// access, then walks the rows' chunks as one sequence (chunk j of the group is
// chunk j % c of row j / c), all lanes busy whatever the width, kBatch chunks
// a lane loaded before the first is stored.  The last chunk of a row whose
// width is not a multiple of a chunk is moved back to end with the row; a
// gather then writes the shared elements twice with the same value, a scatter
// leaves them to the chunk before.  Rows and buffers need the element's
// alignment only.
#include <type_traits>

#include "internal.h"
#include "vec.h"

namespace spc3d {

constexpr int kBatch = 2;

// What bounds both: the slab rows, which come from HBM through an Infinity
// Cache (256 MB) full of the step's other data.  Nontemporal accesses keep what
// is not read again from evicting the rest; where a step's data fits, they only
// lose what the cache would have kept.  So each hint has its own line.  us for a
// whole step (both gathers, the pass, the scatter-reduce; inputs that change
// between steps), MI355X:
//
// kStreamSource, nontemporal loads of a gather, by the bytes of the source rows
// (cached / nontemporal): R-MAT 2^17, 10 MB 55.3 / 55.9, 18 MB 99.7 / 97.2, 36 MB
// 151 / 149; R-MAT share, 55 MB 180 / 171, 110 MB 326 / 305; uniform, 28 MB 134 /
// 131.5.  A conversion to bfloat16 reads 32 bytes a lane in two loads, the second
// from a line that a nontemporal first one need not leave behind: 5 MB 61.5 / 63.4,
// 19 MB 73.6 / 76.7, 38 MB 120 / 116.
//
// kStreamPacked, nontemporal stores of packed rows, which the pass reads next
// (cached / nontemporal): 229 MB uniform share 418 / 409, 55 MB R-MAT share 167 /
// 169, banded kz = 16 of two entries a row, 134 MB 418 / 389, uniform kz = 16, 114
// MB 363 / 368 (and 357 / 368 from cold caches).  Rows that are not whole 64-byte granules gain earlier
// (kStreamPackedRagged): R-MAT share kz = 40, 69 MB 270 / 282, banded, 11 a row, 80 MB
// 292 / 305, 3 a row, kz = 20, 84 MB 295 / 286, bfloat16 kz = 40, 84 MB 450 / 431,
// kz = 30, 126 MB 454 / 421; share kz = 60 (103 MB) 430 / 400.
//
// kStreamSlab, nontemporal loads of the slab rows a scatter adds to, and
// kStreamSlabStored, of the stores as well (cached / loads / both): R-MAT share, 55 MB
// 179 / 171 / 172, 220 MB 586 / 585 / 596; banded, 179 MB 395 / 395 / 386, 268 MB
// 583 / 585 / 573, 537 MB 828 / 831 / 792; 18 MB 172 / 175 / 174.  What is stored
// cached the next scatter into the same slab may find there: 55 MB 31.8 us against
// 36.4, 220 MB 113 against 126; but what is left there is written back during the
// step's other kernels, which costs more where the slab rows near the cache's size, and
// from 128 MB on (kStreamSlabSpread) where whole 128-byte lines of a slab row are
// taken and all of those rows are larger than it (a step that adds to one slab again
// and again, cached / past the caches: uniform, 229 of 916 MB 463 / 455, banded, 268 MB
// of 1 GB 496 / 484; whole rows, banded, 5 a row, bfloat16 kz = 128, 256 MB 469 / 431,
// R-MAT share kz = 128, 220 MB 575 / 590; half lines, kz = 16, uniform, 114 of 916 MB
// 366 / 369, banded, 134 MB of 1 GB 389 / 396).  Slab rows that are not whole 64-byte granules
// (kz, k0 or ld no multiple of 16, or an address) stay cached: a granule that
// two rows share is then read or written twice (kz = 24, 41 MB 219 / 223 / 226; kz =
// 60, 103 MB 387 / 400 / 417; banded, 168 MB 510 / 533 / 536).
constexpr int64_t kStreamSource = 12 << 20;
constexpr int64_t kStreamSourceConverted = 32 << 20;
constexpr int64_t kStreamPacked = 120 << 20;
constexpr int64_t kStreamPackedRagged = 78 << 20;
constexpr int64_t kStreamSlab = 32 << 20;
constexpr int64_t kStreamSlabStored = 220 << 20;
constexpr int64_t kStreamSlabSpread = 128 << 20;

typedef uint32_t vec4u_e4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t vec4u_e2 __attribute__((ext_vector_type(4), aligned(2)));
typedef float vec4f_e4 __attribute__((ext_vector_type(4), aligned(4)));

// The rows a wavefront moves.
struct RowGroup {
  int64_t r0;      // first local row
  int64_t off;     // of row r0 + lane: first element in the slab
  int total;       // chunks
  __device__ inline RowGroup(int64_t n, int rpw, int c, const int64_t* __restrict__ gmap,
                             int64_t lo, int64_t ld, int k0) {
    const int lane = threadIdx.x & 63;
    r0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * rpw;
    const int rows = n - r0 < rpw ? (n > r0 ? (int)(n - r0) : 0) : rpw;
    off = lane < rows ? (gmap[r0 + lane] - lo) * ld + k0 : 0;
    total = rows * c;
  }
};

// Row and first element of chunk j.  magic = ceil(2^32 / c): exact for the
// j < 64 * 256 of a group.
struct ChunkAt {
  int l, e;
  __device__ inline ChunkAt(int j, int c, uint32_t magic, int vo, int kz) {
    l = c == 1 ? j : (int)__umulhi((uint32_t)j, magic);
    const int w = (j - l * c) * vo;
    e = w < kz - vo ? w : kz - vo;
  }
};

// packed[l*kz + k] = conv(src[(gmap[l]-lo)*ld + k0 + k]).
template <typename Tin, typename Tout, bool NTLD, bool NTST>
__global__ __launch_bounds__(256) void k_gather(int64_t n, int rpw, int c, uint32_t magic,
                                                const int64_t* __restrict__ gmap, int64_t lo,
                                                const Tin* __restrict__ src, int64_t ld, int k0,
                                                int kz, Tout* __restrict__ dst) {
  constexpr int VO = 16 / sizeof(Tout);
  constexpr int NL = VO * sizeof(Tin) / 16;   // 16-byte loads of a chunk
  using VI = typename std::conditional<sizeof(Tin) == 4, vec4u_e4, vec4u_e2>::type;
  using VOUT = typename std::conditional<sizeof(Tout) == 4, vec4u_e4, vec4u_e2>::type;
  const RowGroup rg(n, rpw, c, gmap, lo, ld, k0);
  const int lane = threadIdx.x & 63;
  Tout* out = dst + rg.r0 * kz;
  for (int base = 0; base < rg.total; base += 64 * kBatch) {
    VI v[kBatch][NL];
    int at[kBatch];
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int j0 = base + i * 64 + lane;
      const int j = j0 < rg.total ? j0 : rg.total - 1;   // spare lanes repeat the last chunk
      const ChunkAt ch(j, c, magic, VO, kz);
      const VI* s = reinterpret_cast<const VI*>(src + __shfl(rg.off, ch.l) + ch.e);
#pragma unroll
      for (int h = 0; h < NL; ++h) v[i][h] = NTLD ? __builtin_nontemporal_load(s + h) : s[h];
      at[i] = ch.l * kz + ch.e;
    }
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      VOUT o;
      if constexpr (sizeof(Tin) == sizeof(Tout)) {
        o = v[i][0];
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const VI w = v[i][t >> 1];
          o[t] = (uint32_t)f32_to_bf16(__uint_as_float(w[(t & 1) * 2])) |
                 ((uint32_t)f32_to_bf16(__uint_as_float(w[(t & 1) * 2 + 1])) << 16);
        }
      }
      VOUT* d = reinterpret_cast<VOUT*>(out + at[i]);
      if constexpr (NTST)
        __builtin_nontemporal_store(o, d);
      else
        *d = o;
    }
  }
}

// dst[(gmap[l]-lo)*ld + k0 + k] += packed[l*kz + k].
template <bool NTLD, bool NTST>
__global__ __launch_bounds__(256) void k_scatter_add(int64_t n, int rpw, int c, uint32_t magic,
                                                     const int64_t* __restrict__ gmap, int64_t lo,
                                                     const float* __restrict__ packed, int kz,
                                                     float* __restrict__ dst, int64_t ld, int k0) {
  const RowGroup rg(n, rpw, c, gmap, lo, ld, k0);
  const int lane = threadIdx.x & 63;
  const float* in = packed + rg.r0 * kz;
  for (int base = 0; base < rg.total; base += 64 * kBatch) {
    vec4f_e4 v[kBatch], w[kBatch];
    float* at[kBatch];
    int skip[kBatch];   // leading elements that are another lane's
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int j0 = base + i * 64 + lane;
      const int j = j0 < rg.total ? j0 : rg.total - 1;
      const ChunkAt ch(j, c, magic, 4, kz);
      skip[i] = j0 < rg.total ? (j - ch.l * c) * 4 - ch.e : 4;
      at[i] = dst + __shfl(rg.off, ch.l) + ch.e;
      const vec4f_e4* p = reinterpret_cast<const vec4f_e4*>(in + ch.l * kz + ch.e);
      const vec4f_e4* d = reinterpret_cast<const vec4f_e4*>(at[i]);
      v[i] = __builtin_nontemporal_load(p);   // read for the last time
      w[i] = NTLD ? __builtin_nontemporal_load(d) : *d;
    }
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const vec4f_e4 s = w[i] + v[i];
      vec4f_e4* d = reinterpret_cast<vec4f_e4*>(at[i]);
      if (skip[i] == 0) {
        if constexpr (NTST)
          __builtin_nontemporal_store(s, d);
        else
          *d = s;
      } else {
#pragma unroll
        for (int t = 1; t < 4; ++t)
          if (t >= skip[i]) at[i][t] = s[t];
      }
    }
  }
}

// Rows narrower than a chunk: one element a thread.
template <typename Tin, typename Tout>
__global__ __launch_bounds__(256) void k_gather_narrow(int64_t n, const int64_t* __restrict__ gmap,
                                                       int64_t lo, const Tin* __restrict__ src,
                                                       int64_t ld, int k0, int kz,
                                                       Tout* __restrict__ dst) {
  const int64_t total = n * kz;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t l = i / kz;
    const Tin v = src[(gmap[l] - lo) * ld + k0 + (i - l * kz)];
    if constexpr (sizeof(Tin) == sizeof(Tout))
      dst[i] = v;
    else
      dst[i] = f32_to_bf16(v);
  }
}

__global__ __launch_bounds__(256) void k_scatter_add_narrow(int64_t n,
                                                            const int64_t* __restrict__ gmap,
                                                            int64_t lo,
                                                            const float* __restrict__ packed,
                                                            int kz, float* __restrict__ dst,
                                                            int64_t ld, int k0) {
  const int64_t total = n * kz;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t l = i / kz;
    dst[(gmap[l] - lo) * ld + k0 + (i - l * kz)] += packed[i];
  }
}

namespace {

unsigned blocks_narrow(int64_t total) {
  const int64_t b = (total + 255) / 256;
  return (unsigned)(b < 1 ? 1 : b > (1 << 20) ? 1 << 20 : b);
}

// Rows per wavefront: as many as fill its kBatch chunks a lane.  More rows a
// wavefront were slower (banded block, 2.1M rows of 64 bfloat16 values, whole
// step: 811 us with 32 rows of 16 chunks each against 781).
struct RowSplit {
  int rpw, c;
  uint32_t magic;
  dim3 grid;
  RowSplit(int64_t n, int kz, int vo) {
    c = (kz + vo - 1) / vo;
    magic = c == 1 ? 0u : (uint32_t)(((1ull << 32) + c - 1) / c);
    rpw = 64 * kBatch / c;
    rpw = rpw < 1 ? 1 : rpw > 64 ? 64 : rpw;
    grid = dim3((unsigned)(((n + rpw - 1) / rpw + 3) / 4));
  }
};

template <typename Tin, typename Tout>
void launch_gather(int64_t n, const int64_t* gmap, int64_t lo, const void* src, int64_t ld, int k0,
                   int kz, void* dst, hipStream_t stream) {
  constexpr int VO = 16 / sizeof(Tout);
  const Tin* s = static_cast<const Tin*>(src);
  Tout* d = static_cast<Tout*>(dst);
  if (kz < VO) {
    hipLaunchKernelGGL((k_gather_narrow<Tin, Tout>), dim3(blocks_narrow(n * kz)), dim3(256), 0,
                       stream, n, gmap, lo, s, ld, k0, kz, d);
    return;
  }
  const RowSplit sp(n, kz, VO);
  const int64_t from = n * kz * (int64_t)sizeof(Tin), to = n * kz * (int64_t)sizeof(Tout);
  const bool ntld = from > (sizeof(Tin) == sizeof(Tout) ? kStreamSource : kStreamSourceConverted);
  const bool ntst = to > (kz * sizeof(Tout) % 64 ? kStreamPackedRagged : kStreamPacked);
#define SPC3D_GATHER(LD, ST)                                                                      \
  hipLaunchKernelGGL((k_gather<Tin, Tout, LD, ST>), sp.grid, dim3(256), 0, stream, n, sp.rpw,     \
                     sp.c, sp.magic, gmap, lo, s, ld, k0, kz, d)
  if (ntld && ntst) SPC3D_GATHER(true, true);   // rows to store this way are many enough to load so
  else if (ntld) SPC3D_GATHER(true, false);
  else SPC3D_GATHER(false, false);
#undef SPC3D_GATHER
}

}  // namespace
}  // namespace spc3d

using namespace spc3d;

extern "C" {

spc3d_status spc3d_gather(spc3d_plan h, spc3d_axis axis, const void* d_src, spc3d_dtype src_t,
                          int64_t ld_src, int32_t k0, int32_t kz, void* d_packed,
                          spc3d_dtype packed_t, hipStream_t stream) {
  Plan* p;
  spc3d_status st = get_plan(h, &p);
  if (st != SPC3D_OK) return st;
  if (axis != SPC3D_ROWS && axis != SPC3D_COLS) return fail(SPC3D_ERR_INVALID_ARG, "bad axis");
  if (src_t != SPC3D_F32 && src_t != SPC3D_BF16) return fail(SPC3D_ERR_INVALID_ARG, "bad src_t");
  if (packed_t != SPC3D_F32 && packed_t != SPC3D_BF16)
    return fail(SPC3D_ERR_INVALID_ARG, "bad packed_t");
  if (src_t == SPC3D_BF16 && packed_t == SPC3D_F32)
    return fail(SPC3D_ERR_UNSUPPORTED, "bfloat16 source to FP32 packing");
  if (kz < 1 || kz > kMaxKz) return fail(SPC3D_ERR_INVALID_ARG, "kz=%d outside [1,%d]", kz, kMaxKz);
  if (k0 < 0 || ld_src < (int64_t)k0 + kz)
    return fail(SPC3D_ERR_INVALID_ARG, "k0=%d kz=%d do not fit ld_src=%lld", k0, kz,
                (long long)ld_src);
  const int64_t n = axis == SPC3D_ROWS ? p->R : p->C;
  if (n == 0) return SPC3D_OK;
  if (!d_src || !d_packed) return fail(SPC3D_ERR_INVALID_ARG, "NULL buffer");
  DeviceGuard dg;
  st = dg.enter(p);
  if (st != SPC3D_OK) return st;
  SPC3D_DEBUG_CHECK(p, stream);
  const int64_t* gmap = axis == SPC3D_ROWS ? p->gmap_r : p->gmap_c;
  const int64_t lo = axis == SPC3D_ROWS ? p->row_lo : p->col_lo;
  if (src_t == SPC3D_BF16)
    launch_gather<bf16_t, bf16_t>(n, gmap, lo, d_src, ld_src, k0, kz, d_packed, stream);
  else if (packed_t == SPC3D_BF16)
    launch_gather<float, bf16_t>(n, gmap, lo, d_src, ld_src, k0, kz, d_packed, stream);
  else
    launch_gather<float, float>(n, gmap, lo, d_src, ld_src, k0, kz, d_packed, stream);
  SPC3D_LAUNCHED("gather");
  return SPC3D_OK;
}

spc3d_status spc3d_scatter_reduce(spc3d_plan h, spc3d_axis axis, const float* d_packed,
                                  int32_t kz, float* d_dst, int64_t ld_dst, int32_t k0,
                                  hipStream_t stream) {
  Plan* p;
  spc3d_status st = get_plan(h, &p);
  if (st != SPC3D_OK) return st;
  if (axis != SPC3D_ROWS && axis != SPC3D_COLS) return fail(SPC3D_ERR_INVALID_ARG, "bad axis");
  if (kz < 1 || kz > kMaxKz) return fail(SPC3D_ERR_INVALID_ARG, "kz=%d outside [1,%d]", kz, kMaxKz);
  if (k0 < 0 || ld_dst < (int64_t)k0 + kz)
    return fail(SPC3D_ERR_INVALID_ARG, "k0=%d kz=%d do not fit ld_dst=%lld", k0, kz,
                (long long)ld_dst);
  const int64_t n = axis == SPC3D_ROWS ? p->R : p->C;
  if (n == 0) return SPC3D_OK;
  if (!d_packed || !d_dst) return fail(SPC3D_ERR_INVALID_ARG, "NULL buffer");
  DeviceGuard dg;
  st = dg.enter(p);
  if (st != SPC3D_OK) return st;
  SPC3D_DEBUG_CHECK(p, stream);
  const int64_t* gmap = axis == SPC3D_ROWS ? p->gmap_r : p->gmap_c;
  const int64_t lo = axis == SPC3D_ROWS ? p->row_lo : p->col_lo;
  if (kz < 4) {
    hipLaunchKernelGGL(k_scatter_add_narrow, dim3(blocks_narrow(n * kz)), dim3(256), 0, stream, n,
                       gmap, lo, d_packed, kz, d_dst, ld_dst, k0);
  } else {
    const RowSplit sp(n, kz, 4);
    const bool granules = ((kz | k0 | ld_dst) & 15) == 0 &&
                          (reinterpret_cast<uintptr_t>(d_dst) & 63u) == 0;
    const int64_t bytes = granules ? n * kz * 4 : 0;
    const bool spread = kz % 32 == 0 && n * ld_dst * 4 > kStreamSlabStored;
    if (bytes > (spread ? kStreamSlabSpread : kStreamSlabStored))
      hipLaunchKernelGGL((k_scatter_add<true, true>), sp.grid, dim3(256), 0, stream, n, sp.rpw,
                         sp.c, sp.magic, gmap, lo, d_packed, kz, d_dst, ld_dst, k0);
    else if (bytes > kStreamSlab)
      hipLaunchKernelGGL((k_scatter_add<true, false>), sp.grid, dim3(256), 0, stream, n, sp.rpw, sp.c,
                         sp.magic, gmap, lo, d_packed, kz, d_dst, ld_dst, k0);
    else
      hipLaunchKernelGGL((k_scatter_add<false, false>), sp.grid, dim3(256), 0, stream, n, sp.rpw, sp.c,
                         sp.magic, gmap, lo, d_packed, kz, d_dst, ld_dst, k0);
  }
  SPC3D_LAUNCHED("scatter_reduce");
  return SPC3D_OK;
}

}  // extern "C"
