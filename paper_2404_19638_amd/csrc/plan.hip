// Setup phase: localization of a sparse block (globalMap / localMap, empty
// rows and columns removed) and construction of its row-major and optional
// column-major slot structure.  Paper: Section "Data distribution" (localized
// blocks and the two maps) and Section "General structure" (a setup phase run
// once per sparsity pattern, after which iterations only move data).
//
// Device pipeline, both axes in each of the first five launches:
//   mark ids      one byte flag per id of the range (range violations raise a
//                 flag of their own)
//   rank words    64 flags to a bitmap word with the number of ids before it
//   compact       lmap[g - lo] = rank or -1; gmap[rank] = g
//   key/value     key = lr << bits(C) | lc (ranks from the words, which fit L2
//                 where localMap would not), value = caller index
//   radix sort    LSD, 8-bit digits, stable (so equal keys keep caller order)
//   build slots   colidx, perm, rowptr, per-64-slot head bitmaps and tile rows
// For the column-major view the slots are sorted again by column alone: the
// sort is stable and the slots ascend by row.
// What bounds setup: the sort's passes, and 2 random accesses an entry in each
// of marking and key construction (a 128-byte line each, from L2).  An R-MAT
// share of 4.1M entries (ranges of 2^21) took 677 us before and takes 464 after the
// byte flags, rank words and sort described below, with the value permutation
// (59 us); a CSR graph of 1.8M entries with both views 526 and 323.
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <unordered_set>

#include "internal.h"

namespace spc3d {

// ------------------------------------------------------------- errors

static thread_local std::string g_last_error;

spc3d_status fail(spc3d_status s, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return s;
}

spc3d_status hip_fail(hipError_t e, const char* what) {
  return fail(SPC3D_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

static std::mutex g_plans_mu;
static std::unordered_set<const void*> g_plans;

spc3d_status get_plan(spc3d_plan h, Plan** out) {
  std::lock_guard<std::mutex> lk(g_plans_mu);
  if (!h || !g_plans.count(static_cast<const void*>(h)))
    return fail(SPC3D_ERR_BAD_HANDLE, "not a live plan");
  Plan* p = reinterpret_cast<Plan*>(h);
  if (p->magic != kPlanMagic) return fail(SPC3D_ERR_BAD_HANDLE, "corrupt plan");
  *out = p;
  return SPC3D_OK;
}

spc3d_status DeviceGuard::enter(const Plan* p) {
  int cur = -1;
  SPC3D_HIP(hipGetDevice(&cur));
  if (cur != p->device) {
    SPC3D_HIP(hipSetDevice(p->device));
    prev_ = cur;
  }
  return SPC3D_OK;
}

// ------------------------------------------------------------- kernels

__device__ inline int wave_inclusive_sum(int v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    int t = __shfl_up(v, d, 64);
    if (lane >= d) v += t;
  }
  return v;
}

// Exclusive prefix of v over the block (NT threads); *total gets the sum.
template <int NT>
__device__ inline int block_exclusive_sum(int v, int* total) {
  __shared__ int wsum[NT / 64];
  const int inc = wave_inclusive_sum(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  int off = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) {
    int s = wsum[i];
    off += (i < w) ? s : 0;
    tot += s;
  }
  __syncthreads();
  *total = tot;
  return off + inc - v;
}

__global__ void k_fill_i32(int32_t* p, int64_t n, int32_t v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// One axis of a block during localization.
struct Axis {
  const int64_t* gid;    // nullptr: flags were set from a CSR row pointer
  int64_t lo, range;
  uint8_t* flag;         // one byte per id, in the localMap's memory
  struct RankWord* word;
  int32_t* partial;      // ids of each tile of kWordTile ids
  int32_t* lmap;
  int64_t* gmap;
  int64_t cap;           // ids gmap has room for, min(nnz, range)
  int32_t* count;        // ids in use
};

// 64 ids: which are in use, and how many in use come before them.
struct alignas(16) RankWord {
  uint64_t bits;
  int32_t before;
  int32_t pad;
};

constexpr int kWordTile = 256 * 64;   // ids per block of k_rank_words

__device__ inline int rank_of(const RankWord* __restrict__ word, int64_t id) {
  const RankWord w = word[id >> 6];
  return w.before + __popcll(w.bits & ((1ull << (id & 63)) - 1ull));
}

__global__ __launch_bounds__(256) void k_clear_flags(Axis r, Axis c) {
  const Axis& ax = blockIdx.y ? c : r;
  uint4* p = reinterpret_cast<uint4*>(ax.flag);
  const int64_t n = (ax.range + 15) / 16;   // the memory holds 4 bytes per id
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = make_uint4(0, 0, 0, 0);
}

// Flags every id.  Reading a flag first to store only where it is clear was
// slower (89 against 58 us for 2 x 4.1M ids in ranges of 2^21): a random read
// moves a 128-byte line into L1, a store one byte.
__global__ __launch_bounds__(256) void k_mark(int64_t nnz, Axis r, Axis c,
                                              int32_t* __restrict__ err) {
  const Axis& ax = blockIdx.y ? c : r;
  if (!ax.gid) return;
  constexpr int U = 4;
  const int64_t p0 = blockIdx.x * (int64_t)(256 * U) + threadIdx.x;
  int64_t g[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t p = p0 + u * 256;
    g[u] = p < nnz ? __builtin_nontemporal_load(ax.gid + p) - ax.lo : -1;
    if (p < nnz && (g[u] < 0 || g[u] >= ax.range)) {
      err[0] = 1;
      g[u] = -1;
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (g[u] >= 0) ax.flag[g[u]] = 1;
}

// Bitmap word and ids before it inside the tile; the tile's total to partial.
__global__ __launch_bounds__(256) void k_rank_words(Axis r, Axis c) {
  const Axis& ax = blockIdx.y ? c : r;
  const int64_t w = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (blockIdx.x * (int64_t)kWordTile >= ax.range) return;   // uniform per block
  uint64_t bits = 0;
  if (w * 64 < ax.range) {
    const uint4* p = reinterpret_cast<const uint4*>(ax.flag + w * 64);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (w * 64 + i * 16 >= ax.range) break;   // past the cleared flags
      const uint4 v = p[i];
      const uint64_t a = v.x | ((uint64_t)v.y << 32), b = v.z | ((uint64_t)v.w << 32);
      // eight 0/1 bytes to eight bits
      const uint64_t m = ((a * 0x0102040810204080ull) >> 56) |
                         (((b * 0x0102040810204080ull) >> 56) << 8);
      bits |= m << (i * 16);
    }
  }
  int total;
  const int before = block_exclusive_sum<256>(__popcll(bits), &total);
  if (w * 64 < ax.range) {
    RankWord o;
    o.bits = bits;
    o.before = before;
    o.pad = 0;
    ax.word[w] = o;
  }
  if (threadIdx.x == 0) ax.partial[blockIdx.x] = total;
}

// Exclusive scan of each axis' partials in place; the totals are the counts.
__global__ __launch_bounds__(1024) void k_scan_partials(Axis r, Axis c) {
  const Axis& ax = blockIdx.x ? c : r;
  const int64_t m = (ax.range + kWordTile - 1) / kWordTile;
  int carry = 0;
  for (int64_t base = 0; base < m; base += 1024) {
    const int64_t j = base + threadIdx.x;
    const int v = (j < m) ? ax.partial[j] : 0;
    int tot;
    const int ex = block_exclusive_sum<1024>(v, &tot);
    if (j < m) ax.partial[j] = carry + ex;
    carry += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) *ax.count = carry;
}

// Words -> localMap (rank or -1) and globalMap (rank -> global id); the words'
// counts become global.  A wavefront takes kCompactWords words, lane i id i of
// each.  Only a bad row pointer, which the host refuses after this kernel, flags
// more ids than gmap has room for (a row counts as used where the pointer
// increases, whether or not it ends at nnz): those are not stored.
constexpr int kCompactWords = 16;
__global__ __launch_bounds__(256) void k_compact(Axis r, Axis c) {
  const Axis& ax = blockIdx.y ? c : r;
  const int lane = threadIdx.x & 63;
  const int64_t nw = (ax.range + 63) / 64;
  const int64_t w0 = (blockIdx.x * (int64_t)4 + (threadIdx.x >> 6)) * kCompactWords;
  if (w0 >= nw) return;
  const int nwd = nw - w0 < kCompactWords ? (int)(nw - w0) : kCompactWords;
  RankWord mine;
  mine.bits = 0;
  mine.before = 0;
  mine.pad = 0;
  if (lane < nwd) {
    mine = ax.word[w0 + lane];
    mine.before += ax.partial[(w0 + lane) / 256];
    ax.word[w0 + lane] = mine;
  }
#pragma unroll
  for (int i = 0; i < kCompactWords; ++i) {   // words past the range hold no ids
    const uint64_t bits = __shfl(mine.bits, i);
    const int rank = __shfl(mine.before, i) + __popcll(bits & ((1ull << lane) - 1ull));
    const int64_t id = (w0 + i) * 64 + lane;
    const bool on = (bits >> lane) & 1ull;
    if (id < ax.range) ax.lmap[id] = on ? rank : -1;
    if (on && rank < ax.cap) ax.gmap[rank] = ax.lo + id;
  }
}

// ---------------------------------------------------------- radix sort
//
// One pass: a histogram per tile (counts[tile][digit]), a scan of each digit's
// counts with the digit's total, and a stable scatter.  Consecutive tiles run
// on one XCD, where the ends of their neighbouring runs meet in one L2 line.
// Per pass, us before and after (block barriers in each of the eight ranking
// rounds, counts[digit][tile] written and scanned by three kernels): 4.1M
// entries scatter 40 to 23, histogram 11 to 8, scans 16 to 6; 31.4M entries
// scatter 278 to 180 (tiles of 2048 there: 202), histogram 84 to 51.  What bounds a pass is
// the scatter's traffic (24 bytes an entry) and, below some millions of
// entries, how few tiles there are; tiles of 2048 entries serve smaller inputs
// and tiles of 4096, whose digits' runs are 16 entries (128 bytes of keys) on
// average, larger ones.

constexpr int kSortThreads = 256;
constexpr int64_t kSortLarge = int64_t(6) << 20;   // entries from which tiles are large

inline int64_t sort_tiles(int64_t n) {
  const int64_t tile = n < kSortLarge ? 2048 : 4096;
  return (n + tile - 1) / tile;
}

// Adds this thread's digits to a tile's histogram (one copy per wavefront).
struct TileHist {
  int h[kSortThreads / 64][256];
};

__device__ inline void hist_clear(TileHist& th) {
#pragma unroll
  for (int w = 0; w < kSortThreads / 64; ++w) th.h[w][threadIdx.x] = 0;
  __syncthreads();
}

__device__ inline void hist_write(TileHist& th, int64_t tile, int32_t* __restrict__ counts) {
  __syncthreads();
  int s = 0;
#pragma unroll
  for (int w = 0; w < kSortThreads / 64; ++w) s += th.h[w][threadIdx.x];
  counts[tile * 256 + threadIdx.x] = s;
}

template <int ITEMS>
__global__ __launch_bounds__(kSortThreads) void k_radix_hist(const uint64_t* __restrict__ key,
                                                             int64_t n, int shift,
                                                             int32_t* __restrict__ counts) {
  __shared__ TileHist th;
  const int64_t tile = xcd_block(gridDim.x);
  const int64_t base = tile * (kSortThreads * ITEMS) + threadIdx.x;
  uint64_t k[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int64_t j = base + r * kSortThreads;
    k[r] = j < n ? key[j] : 0;
  }
  hist_clear(th);
#pragma unroll
  for (int r = 0; r < ITEMS; ++r)
    if (base + r * kSortThreads < n)
      atomicAdd(&th.h[threadIdx.x >> 6][(int)(k[r] >> shift) & 255], 1);
  hist_write(th, tile, counts);
}

// Keys and the first pass' histogram.  A local id comes from the rank words,
// or from localMap where the axis was regrouped.
template <int ITEMS>
__global__ __launch_bounds__(kSortThreads) void k_make_keys(
    int64_t nnz, const int64_t* __restrict__ rgid, const int64_t* __restrict__ cgid, int64_t rlo,
    int64_t clo, const RankWord* __restrict__ word_r, const RankWord* __restrict__ word_c,
    const int32_t* __restrict__ lmap_r, const int32_t* __restrict__ lmap_c, int bits_c,
    uint64_t* __restrict__ key, int32_t* __restrict__ val, int32_t* __restrict__ counts) {
  __shared__ TileHist th;
  constexpr int U = 4;   // entries of a thread in flight
  const int64_t tile = xcd_block(gridDim.x);
  const int64_t base = tile * (kSortThreads * ITEMS) + threadIdx.x;
  hist_clear(th);
#pragma unroll 1
  for (int r0 = 0; r0 < ITEMS; r0 += U) {
    int64_t gr[U], gc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t p = base + (r0 + u) * kSortThreads;
      gr[u] = p < nnz ? __builtin_nontemporal_load(rgid + p) - rlo : 0;
      gc[u] = p < nnz ? __builtin_nontemporal_load(cgid + p) - clo : 0;
    }
    uint32_t lr[U], lc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      lr[u] = (uint32_t)(lmap_r ? lmap_r[gr[u]] : rank_of(word_r, gr[u]));
      lc[u] = (uint32_t)(lmap_c ? lmap_c[gc[u]] : rank_of(word_c, gc[u]));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t p = base + (r0 + u) * kSortThreads;
      if (p < nnz) {
        const uint64_t k = ((uint64_t)lr[u] << bits_c) | lc[u];
        key[p] = k;
        val[p] = (int32_t)p;
        atomicAdd(&th.h[threadIdx.x >> 6][(int)k & 255], 1);
      }
    }
  }
  hist_write(th, tile, counts);
}

// Keys of the column-major view from the row-major slots, (lc << bits_r) | lr,
// value = row-major slot, and the histogram of the column's lowest digit.
template <int ITEMS>
__global__ __launch_bounds__(kSortThreads) void k_make_keys_t(
    int64_t nnz, const uint64_t* __restrict__ skey, int bits_c, int bits_r,
    uint64_t* __restrict__ key, int32_t* __restrict__ val, int32_t* __restrict__ counts) {
  __shared__ TileHist th;
  const uint64_t cmask = bits_c ? ((1ull << bits_c) - 1ull) : 0ull;
  const int64_t tile = xcd_block(gridDim.x);
  const int64_t base = tile * (kSortThreads * ITEMS) + threadIdx.x;
  uint64_t k[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int64_t j = base + r * kSortThreads;
    k[r] = j < nnz ? skey[j] : 0;
  }
  hist_clear(th);
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int64_t j = base + r * kSortThreads;
    if (j < nnz) {
      key[j] = ((k[r] & cmask) << bits_r) | (k[r] >> bits_c);
      val[j] = (int32_t)j;
      atomicAdd(&th.h[threadIdx.x >> 6][(int)(k[r] & cmask) & 255], 1);
    }
  }
  hist_write(th, tile, counts);
}

// Exclusive scan of four digits' counts over the tiles, in place, and their
// totals.  Thread t takes digit t % 4 of kScanRows consecutive tiles, so a
// block covers 2048 tiles per round and reads 16 bytes of each.
constexpr int kScanRows = 8;
__global__ __launch_bounds__(1024) void k_scan_digits(int32_t* __restrict__ counts, int64_t nblk,
                                                      int32_t* __restrict__ total) {
  __shared__ int wsum[16][4];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, j = t & 3;
  const int d = blockIdx.x * 4 + j;
  int carry = 0;
  for (int64_t base = 0; base < nblk; base += 256 * kScanRows) {
    const int64_t row = base + (int64_t)(t >> 2) * kScanRows;
    int v[kScanRows], sum = 0;
#pragma unroll
    for (int i = 0; i < kScanRows; ++i) {
      v[i] = row + i < nblk ? counts[(row + i) * 256 + d] : 0;
      sum += v[i];
    }
    int inc = sum;   // over the lanes of this digit
#pragma unroll
    for (int s = 4; s < 64; s <<= 1) {
      const int o = __shfl_up(inc, s, 64);
      if (lane >= s) inc += o;
    }
    if (lane >= 60) wsum[w][j] = inc;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int x = wsum[i][j];
      before += i < w ? x : 0;
      all += x;
    }
    __syncthreads();
    int ex = carry + before + inc - sum;
#pragma unroll
    for (int i = 0; i < kScanRows; ++i) {
      if (row + i < nblk) counts[(row + i) * 256 + d] = ex;
      ex += v[i];
    }
    carry += all;
  }
  if (t < 4) total[d] = carry;
}

// Stable scatter of one tile.  A wavefront owns ITEMS * 64 consecutive
// entries and ranks them in rounds of 64 against its own digit counters
// (ballots give a lane's rank among the round's equal digits), so only the
// merge of the wavefronts' counters needs the block's barriers.  The tile is
// then put in digit order in LDS and written out in that order: consecutive
// threads store consecutive entries of one digit's run.
template <int ITEMS>
__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(
    const uint64_t* __restrict__ kin, const int32_t* __restrict__ vin, int64_t n, int shift,
    const int32_t* __restrict__ offsets, const int32_t* __restrict__ total,
    uint64_t* __restrict__ kout, int32_t* __restrict__ vout) {
  constexpr int TILE = kSortThreads * ITEMS;
  constexpr int NW = kSortThreads / 64;
  __shared__ uint64_t s_key[TILE];
  __shared__ int32_t s_val[TILE];
  __shared__ int cnt[NW][256];     // per wavefront: count, then first position
  __shared__ int64_t dest[256];    // global position of a digit's run minus its tile position
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t tile = xcd_block(gridDim.x);
  const int64_t mine = tile * TILE + w * (ITEMS * 64) + lane;
  uint64_t k[ITEMS];
  int32_t v[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int64_t j = mine + r * 64;
    k[r] = j < n ? kin[j] : 0;
    v[r] = j < n ? vin[j] : 0;
  }
#pragma unroll
  for (int i = 0; i < NW; ++i) cnt[i][t] = 0;
  const int64_t off = offsets[tile * 256 + t];
  int tot;
  const int64_t first = block_exclusive_sum<kSortThreads>(total[t], &tot);   // has barriers
  int rank[ITEMS];
  volatile int* my = cnt[w];   // touched by this wavefront alone until the barrier
  const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const bool valid = mine + r * 64 < n;
    const int d = (int)(k[r] >> shift) & 255;
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const uint64_t bb = __ballot((d >> bit) & 1);
      peers &= ((d >> bit) & 1) ? bb : ~bb;
    }
    const int below = __popcll(peers & lt);
    const int seen = my[d];
    rank[r] = seen + below;
    __builtin_amdgcn_wave_barrier();
    if (valid && below == 0) my[d] = seen + __popcll(peers);
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  int sum = 0, part[NW];
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    part[i] = sum;
    sum += cnt[i][t];
  }
  int items;
  const int start = block_exclusive_sum<kSortThreads>(sum, &items);
#pragma unroll
  for (int i = 0; i < NW; ++i) cnt[i][t] = start + part[i];
  dest[t] = first + off - start;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    if (mine + r * 64 < n) {
      const int pos = cnt[w][(int)(k[r] >> shift) & 255] + rank[r];
      s_key[pos] = k[r];
      s_val[pos] = v[r];
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int i = r * kSortThreads + t;
    if (i < items) {
      const uint64_t key = s_key[i];
      const int64_t g = dest[(int)(key >> shift) & 255] + i;
      kout[g] = key;
      vout[g] = s_val[i];
    }
  }
}

// Sorted keys -> slot arrays.  One thread per slot; lanes of a wavefront hold
// 64 consecutive slots, so the head bitmap word is one ballot.
__global__ __launch_bounds__(256) void k_build_slots(int64_t nnz, int64_t nrows,
                                                     const uint64_t* __restrict__ key,
                                                     const int32_t* __restrict__ val, int bits_minor,
                                                     int32_t* __restrict__ minor_out,
                                                     int32_t* __restrict__ val_out,
                                                     int32_t* __restrict__ ptr,
                                                     uint64_t* __restrict__ head,
                                                     int32_t* __restrict__ tile_row) {
  const int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const uint64_t mmask = bits_minor ? ((1ull << bits_minor) - 1ull) : 0ull;
  const bool valid = s < nnz;
  bool is_head = false;
  int32_t major = 0;
  if (valid) {
    const uint64_t k = key[s];
    major = (int32_t)(k >> bits_minor);
    minor_out[s] = (int32_t)(k & mmask);
    val_out[s] = val[s];
    is_head = (s == 0) || ((int32_t)(key[s - 1] >> bits_minor) != major);
    if (is_head) ptr[major] = (int32_t)s;
    if (s == nnz - 1) ptr[nrows] = (int32_t)nnz;
  }
  const uint64_t hb = __ballot(is_head);
  if ((threadIdx.x & 63) == 0 && valid) {
    head[s >> 6] = hb;
    tile_row[s >> 6] = major;
  }
}

// ------------------------------------------------------- CSR input

constexpr int kCsrChunk = 512;   // entries of a wavefront of k_csr_rows

// Checks the row pointer, flags the rows with entries and notes the row of
// every kCsrChunk-th entry: rows over more than kCsrMany chunks one after
// another by the whole wavefront.  (One thread a row, one row of 30M entries took
// 3233 us for the whole setup, 1786 so; the same entries searched one by one
// 2698.)
constexpr int kCsrMany = 8;
__global__ void k_csr_flags(int64_t n, const int64_t* __restrict__ rowptr, int64_t nnz,
                            uint8_t* __restrict__ flag, int32_t* __restrict__ chunk_row,
                            int32_t* __restrict__ err) {
  const int lane = threadIdx.x & 63;
  for (int64_t i0 = blockIdx.x * (int64_t)blockDim.x + (threadIdx.x & ~63); i0 <= n;
       i0 += (int64_t)gridDim.x * blockDim.x) {   // uniform per wavefront
    const int64_t i = i0 + lane;
    int64_t c = 0, ce = 0;   // the chunks whose first entry is row i's
    if (i <= n) {
      const int64_t v = rowptr[i];
      const int64_t next = i < n ? rowptr[i + 1] : v;
      const bool bad = (i == 0 && v != 0) || (i == n && v != nnz) || next < v || v < 0 || v > nnz;
      if (bad) err[0] = 1;
      if (i < n) {
        flag[i] = next > v;
        if (!bad && next <= nnz) {
          c = (v + kCsrChunk - 1) / kCsrChunk;
          ce = (next + kCsrChunk - 1) / kCsrChunk;
        }
      }
    }
    const bool many = ce - c > kCsrMany;
    if (!many)
      for (; c < ce; ++c) chunk_row[c] = (int32_t)i;
    for (uint64_t left = __ballot(many); left; left &= left - 1) {
      const int l = __ffsll((unsigned long long)left) - 1;
      const int64_t to = __shfl(ce, l);
      for (int64_t k = __shfl(c, l) + lane; k < to; k += 64) chunk_row[k] = (int32_t)(i0 + l);
    }
  }
}

// rows[p] = lo + i for the entries p in [rowptr[i], rowptr[i+1]): each entry's
// row is searched between the rows of its chunk's ends, all of a lane's
// entries in step.  (With a bad row pointer, which is reported, chunk_row may
// hold anything: the rows found still lie in the range.)
__global__ __launch_bounds__(256) void k_csr_rows(int64_t n, const int64_t* __restrict__ rowptr,
                                                  int64_t nnz, int64_t lo,
                                                  const int32_t* __restrict__ chunk_row,
                                                  int64_t* __restrict__ rows) {
  constexpr int U = kCsrChunk / 64;
  const int lane = threadIdx.x & 63;
  const int64_t w = blockIdx.x * (int64_t)4 + (threadIdx.x >> 6);
  const int64_t p0 = w * kCsrChunk;
  if (p0 >= nnz) return;
  int64_t a = chunk_row[w], b = p0 + kCsrChunk < nnz ? chunk_row[w + 1] : n - 1;
  a = a < 0 ? 0 : a >= n ? n - 1 : a;
  b = b < a ? a : b >= n ? n - 1 : b;
  int64_t x[U], y[U];   // the row lies in [x, y)
#pragma unroll
  for (int u = 0; u < U; ++u) {
    x[u] = a;
    y[u] = b + 1;
  }
  for (int64_t span = b + 1 - a; span > 1; span = (span + 1) >> 1) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t m = (x[u] + y[u]) >> 1;   // x itself once y == x + 1
      if (rowptr[m] <= p0 + u * 64 + lane) x[u] = m; else y[u] = m;
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t p = p0 + u * 64 + lane;
    if (p < nnz) rows[p] = lo + x[u];
  }
}

// ------------------------------------------- owner-grouped local order
//
// Method 2 of the paper's sparse communication model (SpC-SB / SpC-RB) stores
// local data as the concatenation of the data units exchanged with each peer,
// so that a message is sent or received in place.  With a group key per
// global id (for example 0 for the rows a processor owns and 1 + peer rank
// for the others), local ids are re-assigned in order of (key, global id):
// one stable radix pass over the used ids keyed by the group, whose values
// are the ids' offsets in the range, then the maps are rewritten.

// keys[l] = group of the l-th used id (in ascending id order), vals[l] = its
// offset in the range; a key outside [0, ngroups) raises *err.
__global__ void k_group_keys(int64_t n, const int64_t* __restrict__ gmap, int64_t lo,
                             const int32_t* __restrict__ group, int32_t ngroups,
                             uint64_t* __restrict__ keys, int32_t* __restrict__ vals,
                             int32_t* __restrict__ err) {
  for (int64_t l = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; l < n;
       l += (int64_t)gridDim.x * blockDim.x) {
    const int64_t off = gmap[l] - lo;
    const int32_t k = group[off];
    const bool ok = k >= 0 && k < ngroups;
    if (!ok) err[0] = 1;
    keys[l] = ok ? (uint64_t)k : 0ull;
    vals[l] = (int32_t)off;
  }
}

// New local id j for the id at range offset sv[j].
__global__ void k_apply_order(int64_t n, const int32_t* __restrict__ sv, int64_t lo,
                              int64_t* __restrict__ gmap, int32_t* __restrict__ lmap) {
  for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < n;
       j += (int64_t)gridDim.x * blockDim.x) {
    const int32_t off = sv[j];
    gmap[j] = lo + off;
    lmap[off] = (int32_t)j;
  }
}

// goff[q] = number of used ids with key < q, for q = 0..ngroups (sorted keys).
__global__ void k_group_offsets(int32_t ngroups, int64_t n, const uint64_t* __restrict__ sk,
                                int32_t* __restrict__ goff) {
  for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q <= ngroups;
       q += (int64_t)gridDim.x * blockDim.x) {
    int64_t a = 0, b = n;
    while (a < b) {
      const int64_t m = (a + b) >> 1;
      if (sk[m] < (uint64_t)q) a = m + 1; else b = m;
    }
    goff[q] = (int32_t)a;
  }
}

// gather (out[p] = in[perm[p]]) or scatter (out[perm[p]] = in[p]) of one
// value per entry; perm is the plan's slot -> caller map, or its column-major
// slot -> row-major slot map.
__global__ void k_permute(int64_t nnz, const int32_t* __restrict__ perm, int gather,
                          const float* __restrict__ in, float* __restrict__ out) {
  for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < nnz;
       p += (int64_t)gridDim.x * blockDim.x) {
    if (gather)
      out[p] = in[perm[p]];
    else
      out[perm[p]] = in[p];
  }
}

// --------------------------------------------------------------- host side

namespace {

inline unsigned grid_for(int64_t n, int threads, int64_t cap = 1 << 20) {
  int64_t b = (n + threads - 1) / threads;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (unsigned)b;
}

struct Bump {
  size_t off = 0;
  size_t take(size_t bytes) {
    size_t o = off;
    off += (bytes + 255) & ~size_t(255);
    return o;
  }
};

struct Layout {
  size_t gmap_r, gmap_c, lmap_r, lmap_c, rowptr, colidx, perm, head, tile_row;
  size_t colptr, rowidx_t, slot_t, head_t, tile_col, small, goff_r, goff_c;
  size_t keys0, keys1, vals0, vals1, counts, digits, word_r, word_c, partial_r, partial_c;
  size_t total;
};

Layout make_layout(int64_t nnz, int64_t rr, int64_t cr, uint32_t flags) {
  Layout L{};
  Bump b;
  const int64_t cap_r = nnz < rr ? nnz : rr;
  const int64_t cap_c = nnz < cr ? nnz : cr;
  const int64_t ntiles = (nnz + 63) / 64;
  const bool csc = flags & SPC3D_BUILD_CSC;
  L.gmap_r = b.take(8 * (size_t)cap_r);
  L.gmap_c = b.take(8 * (size_t)cap_c);
  L.lmap_r = b.take(4 * (size_t)rr);
  L.lmap_c = b.take(4 * (size_t)cr);
  L.rowptr = b.take(4 * (size_t)(cap_r + 1));
  // colidx and perm are one region: before the slots are built it holds the
  // int64 row ids expanded from a CSR input (plan_create_csr)
  L.colidx = b.take(8 * (size_t)nnz);
  L.perm = L.colidx + 4 * (size_t)nnz;
  L.head = b.take(8 * (size_t)ntiles);
  L.tile_row = b.take(4 * (size_t)ntiles);
  L.colptr = csc ? b.take(4 * (size_t)(cap_c + 1)) : 0;
  L.rowidx_t = csc ? b.take(4 * (size_t)nnz) : 0;
  L.slot_t = csc ? b.take(4 * (size_t)nnz) : 0;
  L.head_t = csc ? b.take(8 * (size_t)ntiles) : 0;
  L.tile_col = csc ? b.take(4 * (size_t)ntiles) : 0;
  L.small = b.take(256);
  L.goff_r = b.take(4 * (size_t)(kMaxGroups + 1));
  L.goff_c = b.take(4 * (size_t)(kMaxGroups + 1));
  // temporaries (dead after plan creation)
  L.keys0 = b.take(8 * (size_t)nnz);
  L.keys1 = b.take(8 * (size_t)nnz);
  L.vals0 = b.take(4 * (size_t)nnz);
  L.vals1 = b.take(4 * (size_t)nnz);
  L.counts = b.take(4 * (size_t)(256 * ((nnz + 2047) / 2048)));   // tiles of either size
  L.digits = b.take(4 * 256);
  L.word_r = b.take(sizeof(RankWord) * (size_t)((rr + 63) / 64));
  L.word_c = b.take(sizeof(RankWord) * (size_t)((cr + 63) / 64));
  L.partial_r = b.take(4 * (size_t)((rr + kWordTile - 1) / kWordTile));
  L.partial_c = b.take(4 * (size_t)((cr + kWordTile - 1) / kWordTile));
  L.total = b.off;
  return L;
}

// Localize both axes: flags -> words -> localMap, globalMap and the counts.
// rowptr: the block is in CSR (the row axis has no ids to mark).
spc3d_status localize(int64_t nnz, const Axis& r, const Axis& c, const int64_t* rowptr,
                      int32_t* chunk_row, int32_t* d_err, int32_t* d_csr_err, hipStream_t s) {
  const int64_t most = r.range > c.range ? r.range : c.range;
  hipLaunchKernelGGL(k_clear_flags, dim3(grid_for((most + 15) / 16, 256, 4096), 2), dim3(256), 0, s,
                     r, c);
  if (rowptr)
    hipLaunchKernelGGL(k_csr_flags, dim3(grid_for(r.range + 1, 256)), dim3(256), 0, s, r.range,
                       rowptr, nnz, r.flag, chunk_row, d_csr_err);
  if (nnz > 0)
    hipLaunchKernelGGL(k_mark, dim3(grid_for(nnz, 1024, INT32_MAX), 2), dim3(256), 0, s, nnz, r, c,
                       d_err);
  hipLaunchKernelGGL(k_rank_words, dim3(grid_for(most, kWordTile, INT32_MAX), 2), dim3(256), 0, s,
                     r, c);
  hipLaunchKernelGGL(k_scan_partials, dim3(2), dim3(1024), 0, s, r, c);
  hipLaunchKernelGGL(k_compact, dim3(grid_for((most + 63) / 64, 4 * kCompactWords, INT32_MAX), 2),
                     dim3(256), 0, s, r, c);
  SPC3D_LAUNCHED("localize");
  return SPC3D_OK;
}

// The sort's scratch.
struct SortTemp {
  uint64_t *k0, *k1;
  int32_t *v0, *v1, *counts, *digits;
};

// Stable LSD sort of (t.k0, t.v0) over bits [from, to).  counted: the first
// digit's histogram is in t.counts already.  *out_k / *out_v point at the
// result, the other pair is free.
spc3d_status radix_sort(const SortTemp& t, int64_t n, int from, int to, bool counted,
                        hipStream_t s, uint64_t** out_k, int32_t** out_v) {
  uint64_t *ks = t.k0, *kd = t.k1;
  int32_t *vs = t.v0, *vd = t.v1;
  const int64_t nblk = sort_tiles(n);
  const dim3 grid((unsigned)nblk), block(kSortThreads);
  const bool small = n < kSortLarge;
  for (int shift = from; shift < to; shift += 8) {
    if (!(counted && shift == from)) {
      if (small)
        hipLaunchKernelGGL(k_radix_hist<8>, grid, block, 0, s, ks, n, shift, t.counts);
      else
        hipLaunchKernelGGL(k_radix_hist<16>, grid, block, 0, s, ks, n, shift, t.counts);
    }
    hipLaunchKernelGGL(k_scan_digits, dim3(64), dim3(1024), 0, s, t.counts, nblk, t.digits);
    if (small)
      hipLaunchKernelGGL(k_radix_scatter<8>, grid, block, 0, s, ks, vs, n, shift, t.counts,
                         t.digits, kd, vd);
    else
      hipLaunchKernelGGL(k_radix_scatter<16>, grid, block, 0, s, ks, vs, n, shift, t.counts,
                         t.digits, kd, vd);
    SPC3D_LAUNCHED("radix pass");
    uint64_t* tk = ks; ks = kd; kd = tk;
    int32_t* tv = vs; vs = vd; vd = tv;
  }
  *out_k = ks;
  *out_v = vs;
  return SPC3D_OK;
}

// Re-assigns the local ids of one axis in (group, id) order (see above).
spc3d_status group_axis(int64_t n, int64_t lo, int64_t* gmap, int32_t* lmap,
                        const int32_t* group, int32_t ngroups, int32_t* goff, const SortTemp& t,
                        int32_t* d_err, hipStream_t s) {
  if (n > 0) {
    hipLaunchKernelGGL(k_group_keys, dim3(grid_for(n, 256)), dim3(256), 0, s, n, gmap, lo, group,
                       ngroups, t.k0, t.v0, d_err);
    SPC3D_LAUNCHED("group keys");
    uint64_t* sk;
    int32_t* sv;
    spc3d_status st = radix_sort(t, n, 0, ceil_log2(ngroups), false, s, &sk, &sv);
    if (st != SPC3D_OK) return st;
    hipLaunchKernelGGL(k_apply_order, dim3(grid_for(n, 256)), dim3(256), 0, s, n, sv, lo, gmap,
                       lmap);
    hipLaunchKernelGGL(k_group_offsets, dim3(grid_for(ngroups + 1, 256)), dim3(256), 0, s,
                       ngroups, n, sk, goff);
  } else {
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(ngroups + 1, 256)), dim3(256), 0, s, goff,
                       (int64_t)ngroups + 1, 0);
  }
  SPC3D_LAUNCHED("group order");
  return SPC3D_OK;
}

spc3d_status validate_ranges(int64_t nnz, int64_t row_lo, int64_t row_hi, int64_t col_lo,
                             int64_t col_hi) {
  if (nnz < 0 || nnz > INT32_MAX - 64)
    return fail(SPC3D_ERR_INVALID_ARG, "nnz=%lld outside [0, 2^31-65]", (long long)nnz);
  // hi > lo first, so the unsigned difference is the exact width of the range
  if (row_hi <= row_lo || (uint64_t)row_hi - (uint64_t)row_lo > (uint64_t)INT32_MAX - 1 ||
      col_hi <= col_lo || (uint64_t)col_hi - (uint64_t)col_lo > (uint64_t)INT32_MAX - 1)
    return fail(SPC3D_ERR_INVALID_ARG, "id ranges must hold 1..2^31-2 ids");
  return SPC3D_OK;
}

}  // namespace
}  // namespace spc3d

using namespace spc3d;

extern "C" {

spc3d_status spc3d_plan_workspace_size(int64_t nnz, int64_t row_lo, int64_t row_hi,
                                       int64_t col_lo, int64_t col_hi, uint32_t flags,
                                       size_t* bytes) {
  if (!bytes) return fail(SPC3D_ERR_INVALID_ARG, "bytes is NULL");
  spc3d_status st = validate_ranges(nnz, row_lo, row_hi, col_lo, col_hi);
  if (st != SPC3D_OK) return st;
  if (flags & ~uint32_t(SPC3D_BUILD_CSC)) return fail(SPC3D_ERR_INVALID_ARG, "unknown flags");
  *bytes = make_layout(nnz, row_hi - row_lo, col_hi - col_lo, flags).total;
  return SPC3D_OK;
}

}  // extern "C"

namespace {

spc3d_status create_plan(spc3d_plan* out, int64_t nnz, const int64_t* d_row_gid,
                         const int64_t* d_rowptr, const int64_t* d_col_gid, int64_t row_lo,
                         int64_t row_hi,
                         int64_t col_lo, int64_t col_hi, const int32_t* d_group_r,
                         int32_t ngroups_r, const int32_t* d_group_c, int32_t ngroups_c,
                         uint32_t flags, void* d_ws, size_t ws_bytes, hipStream_t stream) {
  if (!out) return fail(SPC3D_ERR_INVALID_ARG, "out is NULL");
  *out = nullptr;
  spc3d_status st = validate_ranges(nnz, row_lo, row_hi, col_lo, col_hi);
  if (st != SPC3D_OK) return st;
  if (flags & ~uint32_t(SPC3D_BUILD_CSC)) return fail(SPC3D_ERR_INVALID_ARG, "unknown flags");
  if (nnz > 0 && ((!d_row_gid && !d_rowptr) || !d_col_gid))
    return fail(SPC3D_ERR_INVALID_ARG, "id arrays are NULL");
  if (!d_ws) return fail(SPC3D_ERR_INVALID_ARG, "workspace is NULL");
  if (reinterpret_cast<uintptr_t>(d_ws) & 255u)
    return fail(SPC3D_ERR_INVALID_ARG, "workspace must be 256-byte aligned");
  const int64_t rr = row_hi - row_lo, cr = col_hi - col_lo;
  const Layout L = make_layout(nnz, rr, cr, flags);
  if (ws_bytes < L.total)
    return fail(SPC3D_ERR_WORKSPACE, "workspace %zu bytes < %zu required", ws_bytes, L.total);

  int device = 0;
  SPC3D_HIP(hipGetDevice(&device));
  char* w = static_cast<char*>(d_ws);
  Plan* p = new Plan();
  p->magic = kPlanMagic;
  p->device = device;
  p->flags = flags;
  p->nnz = nnz;
  p->row_lo = row_lo; p->row_hi = row_hi; p->col_lo = col_lo; p->col_hi = col_hi;
  p->ntiles = (nnz + 63) / 64;
  p->gmap_r = reinterpret_cast<int64_t*>(w + L.gmap_r);
  p->gmap_c = reinterpret_cast<int64_t*>(w + L.gmap_c);
  p->lmap_r = reinterpret_cast<int32_t*>(w + L.lmap_r);
  p->lmap_c = reinterpret_cast<int32_t*>(w + L.lmap_c);
  p->rowptr = reinterpret_cast<int32_t*>(w + L.rowptr);
  p->colidx = reinterpret_cast<int32_t*>(w + L.colidx);
  p->perm = reinterpret_cast<int32_t*>(w + L.perm);
  p->head = reinterpret_cast<uint64_t*>(w + L.head);
  p->tile_row = reinterpret_cast<int32_t*>(w + L.tile_row);
  if (flags & SPC3D_BUILD_CSC) {
    p->colptr = reinterpret_cast<int32_t*>(w + L.colptr);
    p->rowidx_t = reinterpret_cast<int32_t*>(w + L.rowidx_t);
    p->slot_t = reinterpret_cast<int32_t*>(w + L.slot_t);
    p->head_t = reinterpret_cast<uint64_t*>(w + L.head_t);
    p->tile_col = reinterpret_cast<int32_t*>(w + L.tile_col);
  }
  int32_t* small = reinterpret_cast<int32_t*>(w + L.small);
  const SortTemp tmp{reinterpret_cast<uint64_t*>(w + L.keys0),
                     reinterpret_cast<uint64_t*>(w + L.keys1),
                     reinterpret_cast<int32_t*>(w + L.vals0),
                     reinterpret_cast<int32_t*>(w + L.vals1),
                     reinterpret_cast<int32_t*>(w + L.counts),
                     reinterpret_cast<int32_t*>(w + L.digits)};
  if (d_group_r) {
    p->ngroups_r = ngroups_r;
    p->goff_r = reinterpret_cast<int32_t*>(w + L.goff_r);
  }
  if (d_group_c) {
    p->ngroups_c = ngroups_c;
    p->goff_c = reinterpret_cast<int32_t*>(w + L.goff_c);
  }

  auto bail = [&](spc3d_status s) {
    delete p;
    return s;
  };
  hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, stream, small, (int64_t)64, 0);
  const Axis ax_r{d_rowptr ? nullptr : d_row_gid, row_lo, rr,
                  reinterpret_cast<uint8_t*>(p->lmap_r),
                  reinterpret_cast<RankWord*>(w + L.word_r),
                  reinterpret_cast<int32_t*>(w + L.partial_r), p->lmap_r, p->gmap_r,
                  nnz < rr ? nnz : rr, small + 0};
  const Axis ax_c{d_col_gid, col_lo, cr, reinterpret_cast<uint8_t*>(p->lmap_c),
                  reinterpret_cast<RankWord*>(w + L.word_c),
                  reinterpret_cast<int32_t*>(w + L.partial_c), p->lmap_c, p->gmap_c,
                  nnz < cr ? nnz : cr, small + 1};
  int32_t* chunk_row = tmp.counts;   // free until the sort
  st = localize(nnz, ax_r, ax_c, d_rowptr, chunk_row, small + 2, small + 4, stream);
  if (st != SPC3D_OK) return bail(st);
  if (d_rowptr && nnz > 0) {
    // CSR input: expand the row pointer to one row id per entry in the colidx
    // / perm region (free until the slots are built)
    int64_t* rows_tmp = reinterpret_cast<int64_t*>(w + L.colidx);
    hipLaunchKernelGGL(k_csr_rows, dim3(grid_for(nnz, 4 * kCsrChunk, INT32_MAX)), dim3(256), 0, stream, rr,
                       d_rowptr, nnz, row_lo, chunk_row, rows_tmp);
    SPC3D_LAUNCHED("csr rows");
    d_row_gid = rows_tmp;
  }
  int32_t host_small[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  hipError_t e = hipMemcpyAsync(host_small, small, sizeof host_small, hipMemcpyDeviceToHost,
                                stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return bail(hip_fail(e, "plan_create sync"));
  if (host_small[4])
    return bail(fail(SPC3D_ERR_INVALID_ARG,
                     "rowptr must start at 0, not decrease, and end at nnz"));
  if (host_small[2])
    return bail(fail(SPC3D_ERR_OUT_OF_RANGE, "a global id lies outside its [lo, hi) range"));
  p->R = host_small[0];
  p->C = host_small[1];
  if (d_group_r || d_group_c) {
    if (d_group_r) {
      st = group_axis(p->R, row_lo, p->gmap_r, p->lmap_r, d_group_r, ngroups_r, p->goff_r, tmp,
                      small + 3, stream);
      if (st != SPC3D_OK) return bail(st);
    }
    if (d_group_c) {
      st = group_axis(p->C, col_lo, p->gmap_c, p->lmap_c, d_group_c, ngroups_c, p->goff_c, tmp,
                      small + 3, stream);
      if (st != SPC3D_OK) return bail(st);
    }
    int32_t host_err = 0;
    e = hipMemcpyAsync(&host_err, small + 3, sizeof host_err, hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return bail(hip_fail(e, "plan_create group sync"));
    if (host_err) return bail(fail(SPC3D_ERR_INVALID_ARG, "a group key lies outside [0, ngroups)"));
  }

  const int bits_r = ceil_log2(p->R), bits_c = ceil_log2(p->C);
  if (nnz > 0) {
    const int64_t nblk = sort_tiles(nnz);
    const dim3 tiles((unsigned)nblk), threads(kSortThreads);
    const bool small_sort = nnz < kSortLarge;
    const int32_t* map_r = d_group_r ? p->lmap_r : nullptr;
    const int32_t* map_c = d_group_c ? p->lmap_c : nullptr;
    if (small_sort)
      hipLaunchKernelGGL(k_make_keys<8>, tiles, threads, 0, stream, nnz, d_row_gid, d_col_gid,
                         row_lo, col_lo, ax_r.word, ax_c.word, map_r, map_c, bits_c, tmp.k0, tmp.v0,
                         tmp.counts);
    else
      hipLaunchKernelGGL(k_make_keys<16>, tiles, threads, 0, stream, nnz, d_row_gid, d_col_gid,
                         row_lo, col_lo, ax_r.word, ax_c.word, map_r, map_c, bits_c, tmp.k0, tmp.v0,
                         tmp.counts);
    SPC3D_LAUNCHED("make_keys");
    uint64_t* sk;
    int32_t* sv;
    st = radix_sort(tmp, nnz, 0, bits_r + bits_c, true, stream, &sk, &sv);
    if (st != SPC3D_OK) return bail(st);
    hipLaunchKernelGGL(k_build_slots, dim3(grid_for(nnz, 256, INT32_MAX)), dim3(256), 0, stream,
                       nnz, p->R, sk, sv, bits_c, p->colidx, p->perm, p->rowptr, p->head,
                       p->tile_row);
    SPC3D_LAUNCHED("build_slots");
    if (flags & SPC3D_BUILD_CSC) {
      SortTemp t = tmp;   // the sorted keys are read, the other pair written
      if (sk == tmp.k0) {
        t.k0 = tmp.k1;
        t.k1 = tmp.k0;
        t.v0 = tmp.v1;
        t.v1 = tmp.v0;
      }
      if (small_sort)
        hipLaunchKernelGGL(k_make_keys_t<8>, tiles, threads, 0, stream, nnz, sk, bits_c, bits_r,
                           t.k0, t.v0, t.counts);
      else
        hipLaunchKernelGGL(k_make_keys_t<16>, tiles, threads, 0, stream, nnz, sk, bits_c, bits_r,
                           t.k0, t.v0, t.counts);
      SPC3D_LAUNCHED("make_keys_t");
      uint64_t* sk2;
      int32_t* sv2;
      st = radix_sort(t, nnz, bits_r, bits_r + bits_c, true, stream, &sk2, &sv2);
      if (st != SPC3D_OK) return bail(st);
      hipLaunchKernelGGL(k_build_slots, dim3(grid_for(nnz, 256, INT32_MAX)), dim3(256), 0,
                         stream, nnz, p->C, sk2, sv2, bits_r, p->rowidx_t, p->slot_t, p->colptr,
                         p->head_t, p->tile_col);
      SPC3D_LAUNCHED("build_slots_t");
    }
  } else {
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, stream, p->rowptr, (int64_t)1, 0);
    if (flags & SPC3D_BUILD_CSC)
      hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, stream, p->colptr, (int64_t)1, 0);
    SPC3D_LAUNCHED("empty plan");
  }
  e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return bail(hip_fail(e, "plan_create final sync"));
  {
    std::lock_guard<std::mutex> lk(g_plans_mu);
    g_plans.insert(static_cast<const void*>(p));
  }
  *out = reinterpret_cast<spc3d_plan>(p);
  return SPC3D_OK;
}

}  // namespace

extern "C" {

spc3d_status spc3d_plan_create_coo(spc3d_plan* out, int64_t nnz, const int64_t* d_row_gid,
                                   const int64_t* d_col_gid, int64_t row_lo, int64_t row_hi,
                                   int64_t col_lo, int64_t col_hi, uint32_t flags, void* d_ws,
                                   size_t ws_bytes, hipStream_t stream) {
  return create_plan(out, nnz, d_row_gid, nullptr, d_col_gid, row_lo, row_hi, col_lo, col_hi,
                     nullptr, 0, nullptr, 0, flags, d_ws, ws_bytes, stream);
}

spc3d_status spc3d_plan_create_csr(spc3d_plan* out, int64_t nnz, const int64_t* d_rowptr,
                                   const int64_t* d_col_gid, int64_t row_lo, int64_t row_hi,
                                   int64_t col_lo, int64_t col_hi, uint32_t flags, void* d_ws,
                                   size_t ws_bytes, hipStream_t stream) {
  if (out) *out = nullptr;
  if (!d_rowptr) return fail(SPC3D_ERR_INVALID_ARG, "rowptr is NULL");
  return create_plan(out, nnz, nullptr, d_rowptr, d_col_gid, row_lo, row_hi, col_lo, col_hi,
                     nullptr, 0, nullptr, 0, flags, d_ws, ws_bytes, stream);
}

spc3d_status spc3d_plan_create_coo_grouped(spc3d_plan* out, int64_t nnz,
                                           const int64_t* d_row_gid, const int64_t* d_col_gid,
                                           int64_t row_lo, int64_t row_hi, int64_t col_lo,
                                           int64_t col_hi, const int32_t* d_group_r,
                                           int32_t ngroups_r, const int32_t* d_group_c,
                                           int32_t ngroups_c, uint32_t flags, void* d_ws,
                                           size_t ws_bytes, hipStream_t stream) {
  if (out) *out = nullptr;
  if ((d_group_r && (ngroups_r < 1 || ngroups_r > kMaxGroups)) ||
      (d_group_c && (ngroups_c < 1 || ngroups_c > kMaxGroups)))
    return fail(SPC3D_ERR_INVALID_ARG, "ngroups must lie in [1, %d]", kMaxGroups);
  return create_plan(out, nnz, d_row_gid, nullptr, d_col_gid, row_lo, row_hi, col_lo, col_hi,
                     d_group_r, ngroups_r, d_group_c, ngroups_c, flags, d_ws, ws_bytes, stream);
}

spc3d_status spc3d_plan_group_offsets(spc3d_plan h, spc3d_axis axis, const int32_t** d_offsets,
                                      int32_t* ngroups) {
  Plan* p;
  spc3d_status st = get_plan(h, &p);
  if (st != SPC3D_OK) return st;
  if (axis != SPC3D_ROWS && axis != SPC3D_COLS) return fail(SPC3D_ERR_INVALID_ARG, "bad axis");
  const int32_t* g = axis == SPC3D_ROWS ? p->goff_r : p->goff_c;
  if (!g) return fail(SPC3D_ERR_INVALID_ARG, "the plan was built without groups on this axis");
  if (d_offsets) *d_offsets = g;
  if (ngroups) *ngroups = axis == SPC3D_ROWS ? p->ngroups_r : p->ngroups_c;
  return SPC3D_OK;
}

spc3d_status spc3d_plan_query(spc3d_plan h, int64_t* R, int64_t* C, int64_t* nnz) {
  Plan* p;
  spc3d_status st = get_plan(h, &p);
  if (st != SPC3D_OK) return st;
  if (R) *R = p->R;
  if (C) *C = p->C;
  if (nnz) *nnz = p->nnz;
  return SPC3D_OK;
}

spc3d_status spc3d_plan_maps(spc3d_plan h, spc3d_maps* m) {
  Plan* p;
  spc3d_status st = get_plan(h, &p);
  if (st != SPC3D_OK) return st;
  if (!m) return fail(SPC3D_ERR_INVALID_ARG, "maps is NULL");
  m->gmap_r = p->gmap_r; m->gmap_c = p->gmap_c;
  m->lmap_r = p->lmap_r; m->lmap_c = p->lmap_c;
  m->rowptr = p->rowptr; m->colidx = p->colidx; m->perm = p->perm;
  m->colptr = p->colptr; m->rowidx_t = p->rowidx_t; m->slot_t = p->slot_t;
  return SPC3D_OK;
}

spc3d_status spc3d_plan_destroy(spc3d_plan h) {
  std::lock_guard<std::mutex> lk(g_plans_mu);
  if (!h || !g_plans.erase(static_cast<const void*>(h)))
    return fail(SPC3D_ERR_BAD_HANDLE, "not a live plan");
  Plan* p = reinterpret_cast<Plan*>(h);
  p->magic = 0;
  delete p;
  return SPC3D_OK;
}

spc3d_status spc3d_permute_values(spc3d_plan h, int direction, const float* d_in, float* d_out,
                                  hipStream_t stream) {
  Plan* p;
  spc3d_status st = get_plan(h, &p);
  if (st != SPC3D_OK) return st;
  if (direction < SPC3D_CALLER_TO_SLOT || direction > SPC3D_COLUMN_TO_SLOT)
    return fail(SPC3D_ERR_INVALID_ARG, "bad direction %d", direction);
  const bool csc = direction == SPC3D_SLOT_TO_COLUMN || direction == SPC3D_COLUMN_TO_SLOT;
  if (csc && !(p->flags & SPC3D_BUILD_CSC))
    return fail(SPC3D_ERR_INVALID_ARG, "column-major order needs a plan built with BUILD_CSC");
  if (p->nnz == 0) return SPC3D_OK;
  if (!d_in || !d_out) return fail(SPC3D_ERR_INVALID_ARG, "NULL array");
  if (d_in == d_out) return fail(SPC3D_ERR_INVALID_ARG, "in and out alias");
  DeviceGuard dg;
  st = dg.enter(p);
  if (st != SPC3D_OK) return st;
  SPC3D_DEBUG_CHECK(p, stream);
  const int gather = direction == SPC3D_CALLER_TO_SLOT || direction == SPC3D_SLOT_TO_COLUMN;
  hipLaunchKernelGGL(k_permute, dim3(grid_for(p->nnz, 256)), dim3(256), 0, stream, p->nnz,
                     csc ? p->slot_t : p->perm, gather, d_in, d_out);
  SPC3D_LAUNCHED("permute_values");
  return SPC3D_OK;
}

const char* spc3d_status_string(spc3d_status s) {
  switch (s) {
    case SPC3D_OK: return "ok";
    case SPC3D_ERR_INVALID_ARG: return "invalid argument";
    case SPC3D_ERR_OUT_OF_RANGE: return "global id out of range";
    case SPC3D_ERR_WORKSPACE: return "workspace or buffer too small";
    case SPC3D_ERR_UNSUPPORTED: return "unsupported";
    case SPC3D_ERR_HIP: return "HIP runtime error";
    case SPC3D_ERR_BAD_HANDLE: return "bad plan handle";
  }
  return "unknown status";
}

const char* spc3d_last_error(void) { return g_last_error.c_str(); }

int spc3d_version(void) { return 100; }

}  // extern "C"
