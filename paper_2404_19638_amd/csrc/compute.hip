// SDDMM / SpMM entry points: argument checks, variant choice and launch.
// The kernels and their design notes are in kernels.h; their instantiations
// are spread over inst_*.hip so they compile in parallel.
#include <cmath>
#include <mutex>

#include "run.h"

namespace spc3d {

#define SPC3D_EXTERN_LAUNCHERS(T, V)                                                          \
  extern template void launch_sddmm<T, V>(SPC3D_SDDMM_LAUNCH_ARGS);                            \
  extern template void launch_spmm<T, V, false>(SPC3D_SPMM_LAUNCH_ARGS);                      \
  extern template void launch_spmm<T, V, true>(SPC3D_SPMM_LAUNCH_ARGS);
SPC3D_EXTERN_LAUNCHERS(float, 4)
SPC3D_EXTERN_LAUNCHERS(float, 1)
SPC3D_EXTERN_LAUNCHERS(bf16_t, 8)
SPC3D_EXTERN_LAUNCHERS(bf16_t, 1)
#undef SPC3D_EXTERN_LAUNCHERS
extern template void launch_sddmm_ragged<bf16_t, 8>(SPC3D_SDDMM_LAUNCH_ARGS);
extern template void launch_run<float, 4, true>(SPC3D_RUN_LAUNCH_ARGS);
extern template void launch_run<float, 4, false>(SPC3D_RUN_LAUNCH_ARGS);
extern template void launch_run<bf16_t, 8, true>(SPC3D_RUN_LAUNCH_ARGS);
extern template void launch_run<bf16_t, 8, false>(SPC3D_RUN_LAUNCH_ARGS);

namespace {

// The entries use fewer rows of the gathered table than entries at uniform
// positions would (0.8 of the expected number).
bool skewed(const Plan* p, int transpose) {
  const int64_t rows = transpose ? p->R : p->C;
  const double ids = transpose ? (double)(p->row_hi - p->row_lo) : (double)(p->col_hi - p->col_lo);
  return rows < 0.8 * ids * -expm1(-(double)p->nnz / ids);
}

// Slices of a packed row that a pass takes one after another (1: the whole
// row).  A pass over a large table is bound by the row lines that miss L2 (they
// arrive at 6.5 to 7.5 TB/s from the Infinity Cache and HBM alike).  Where
// columns are skewed, each XCD's 4 MB L2 holds the hot rows; of rows cut to a
// 128- or 256-byte slice it holds two to four times as many, at the price of
// reading the indices once per slice.  FP32 SpMM, R-MAT graphs of degree 32
// (us, whole row / 256-byte / 128-byte slices): 2^20 vertices kz = 64 (157 MB
// of rows) 775 / - / 643, kz = 128 1781 / 1473 / 1290; 2^19 kz = 128 743 / 631 /
// 569; 2^18 kz = 128 (85 MB) 340 / 277 / 278, kz = 64 (42 MB) 141 / - / 145;
// 2^17 kz = 128 (44 MB) 147 / 126 / 140, kz = 64 72 / - / 76.  Uniform
// columns do not gain: 2^20 columns, 32 entries each, kz = 64 1248 / - / 1344.
// So only skewed blocks are sliced.  The fused pass reads A and adds to
// the dots once more per slice, so it slices only rows of 512 bytes or more of
// tables beyond 128 MB: R-MAT 2^20 kz = 128 1867 / 1662 / 1712, 2^19 833 /
// 767 / 874, 2^18 372 / 368 / 451, kz = 64 2^20 820 / - / 829; at kz = 96, three
// slices of 128 bytes, 2^20 vertices of degree 8 took 449 against 401.
int slice_count(const Plan* p, int transpose, bool fused, int64_t row_bytes) {
  const int64_t rows = transpose ? p->R : p->C;   // of the gathered table
  if (row_bytes % 128 || !skewed(p, transpose)) return 1;
  const int64_t lines = row_bytes / 128, table = rows * row_bytes;
  constexpr int64_t MB = 1 << 20;
  if (lines < (fused ? 4 : 2)) return 1;
  if (table <= (fused ? 128 : lines == 2 ? 64 : 40) * MB) return 1;
  if (lines % 2 == 0 && lines >= 4 && (fused || table / (lines / 2) <= 64 * MB))
    return (int)(lines / 2);
  return (int)lines;
}

// The run family's shape for a default-variant call, if it takes the call:
// rows of 3 to 32 vectors (a lane of 8 then holds at most 4), byte offsets
// into the packed operands of 32 bits and ids of 24 (one multiply-add per
// gathered row).  Wider, narrower and larger operands keep the shapes of
// pick_shape.
//
// Run length.  Longer runs mean fewer carries and scans, shorter ones more
// wavefronts and less imbalance.  64 slots pay on rows of 16 entries and more
// (fused pass, us at 32 / 64: R-MAT 2^18 kz = 64 171 / 166, 2^20 kz = 64 844 /
// 815; at 9.5 entries a row kz = 32 80 / 86, at 3 (banded) kz = 128 357 / 381);
// the SpMM alone, whose wavefronts are lighter, already gains at 8 (66.1 /
// 63.8 at 9.5 entries, kz = 32), except at 4 vectors a lane (banded, 12
// entries, kz = 128 524 / 574).  Below about 7000 wavefronts (7 per SIMD) the
// shorter run is faster: R-MAT 2^16, kz = 32 at 16 / 32 / 64 slots 34.6 / 28.2 /
// 33.6, 2^15 20.8 / 21.9 / 24.8.  Small blocks take runs of 8 and 4 slots: with
// runs of 16 there were too few wavefronts, and each walks its run from one
// memory round trip to the next (SpMM, us, the shapes before the run family /
// runs of 16 / 8 / 4: FP32 kz = 16 40,000 entries 6.6 / 7.9 / 6.7 / 6.2, 148,000
// 7.5 / 9.3 / 7.8 / 7.4, 298,670 9.8 / 10.8 / 8.8 / 9.0, 704,939 15.6 / 14.1 / 12.9
// / 16.1, 1.6M 31.2 / 20.7 / 22.9; kz = 32 40,000 6.9 / 7.5 / 6.5 / 6.4, 298,670
// 12.4 / 10.1 / 9.9, 401,951 12.9 / 11.1 / 11.4; kz = 128 106,242 19.3 / 15.3 /
// 15.0 / 17.9, 235,037 16.4 / 15.0 / 16.1).  Groups of 4 lanes, whose items are
// twice as long, change at more wavefronts, and stop at 32: with 64 an item's
// indices take 35 KB of LDS, four blocks a CU (kz = 16, 13.6M entries, runs of 32
// / 64 125 / 154).
//
// With two or more vectors a lane the SpMM takes 64 from 4000 wavefronts on
// (R-MAT 2^18, degree 12, kz = 96 101 / 98; uniform, 3M entries, kz = 128 218 /
// 214) and 32 from 6000 (uniform, 1.6M, kz = 96 84.0 at 16 / 81.6), and the fused
// pass 64 from 4000 at four vectors (uniform, 3M, kz = 128 232 / 225).
//
// Left to the shapes of pick_shape from 2^17 entries on, where those read whole
// vectors (vec_ok: the operands' alignment; us there / here):
// - four vectors a lane on short rows, whose row ends cost more than the steps
//   between them: SpMM below 10 entries a row (banded, 7, kz = 96 32.6 / 33.8,
//   uniform, 4, 62.8 / 64.6), fused below 20 (uniform, 4, kz = 96 75.6 / 82.1,
//   banded, 12, 40,000 rows, kz = 128 28.2 / 30.7);
// - four bfloat16 vectors a lane, which take 185 registers: the fused pass (kz =
//   256, uniform, 401,951 entries, 0.83 times as fast, R-MAT 2^16, 1.6M, 0.85,
//   folded 0.91 and 0.86), and SpMM but on skewed columns (uniform 0.88, R-MAT
//   1.07);
// - two bfloat16 vectors a lane: fused below 5 entries a row (uniform, 4, 67.3 /
//   71.6), SpMM from 2^21 entries on, where pick_shape's items of 512 slots begin
//   (R-MAT 2^18, degree 12, 76.0 / 79.7; 2^17, degree 24, 66.2 / 70.8; banded kz =
//   96 197 / 230, though 2^18, degree 32, 165 / 157), and between 2^19 and 2^20, but
//   on skewed columns (kz = 96, uniform 632,099 23.4 / 25.0, banded 704,939 26.5 /
//   28.2; R-MAT 999,239 39.0 / 34.5).
//
// Slices of the fused pass.  Each ends every row again, so rows below a number of
// entries are taken whole (us, the plain and the folded pass, whole / sliced).
// Rows of 512 bytes, 36 entries: FP32, R-MAT 2^19 at 25 entries a row 391 / 409
// and 445 / 518, 33 529 / 531 and 578 / 635, 42 718 / 696 and 766 / 799; 2^20 at
// 39 1366 / 1305 and 1427 / 1426, 49 1860 / 1664 and 1914 / 1787; bfloat16, which
// goes to pick_shape below, 2^19 at 25 550 / 488 and 602 / 674, 2^20 at 39 1672 /
// 1433 and 1785 / 1793; the share at 9.3, FP32, 318 / 340.  Wider ones, 28, left to
// pick_shape below: kz = 192, 2^20 at 24 1187 / 1107 and 1258 / 1316, 29 1536 / 1399
// and 1616 / 1583.
//
// Destinations ahead.  Adding to a slab whose rows come from HBM, on rows so short
// that nearly every step ends some, a destination read where its row ends is waited
// for each time; read with the step's gathered rows it costs registers (folded, us,
// where the row ends / with the step, two vectors a lane in steps of 4: uniform, 4.0M
// entries, 2.2 a row, FP32 kz = 16 216 / 195, 32 263 / 252, 64 514 / 489, bfloat16 kz =
// 64 370 / 362; banded, 2 a row, 4.2M 213 / 198, 259 / 250, 490 / 461, 367 / 364; 3 a
// row, 3.1M 116 / 114, 162 / 162, 301 / 277, 235 / 224.  Uniform, 3.9 a row, 8M 332 /
// 319, 363 / 372, 730 / 712, 499 / 516; 4.1 a row, slab rows of 25 MB, kz = 16 63 / 64,
// of 50, kz = 32 72 / 77; banded, 11 a row, 95 / 103, 119 / 141).  FP32 rows on 4 lanes,
// 16 groups a wavefront that each wait, take it below 10 entries a row at any size
// (kz = 16: the share at 9.3, a whole step 135 / 123; uniform, 8.7 59 / 58; banded,
// 226,000 entries, 2 a row, 14.9 / 13.5; uniform, 16 a row, 47.6 / 55.8).  On 8 lanes
// FP32 rows take it where there are no more than 4 wavefronts a SIMD, with two
// vectors a lane 2, for which the registers suffice, and below 20 entries a row
// (whole steps: kz = 32 R-MAT 2^16, 494,000, 15 a row, 33.7 / 30.8, kz = 20 32.9 / 30.1,
// 575,000, 26 a row, 31.6 / 32.6, uniform, 600,000 34.0 / 38.8, 284,000, 28 a row, 17.7 /
// 20.6; kz = 64 banded, 239,000, 5 a row, 38.8 / 34.6, kz = 40 37.2 / 32.6, R-MAT 2^15,
// 244,000 35.4 / 31.1, 2^16 41.3 / 43.5, uniform, 284,000 24.9 / 25.9; bfloat16 kz = 64
// 239,000 28.7 / 32.4).  Read where the row
// starts instead: kz = 16 208, 213 and 115, 32 251, 258 and 157, 64 478, 473 and 272.
//
// Steps of 4 with two vectors a lane, which hold two wavefronts a SIMD fewer but
// twice the rows in flight, pay where rows are put and a row end costs little: in
// SpMM (us, steps of 2 / 4: FP32 kz = 64 banded, 11 a row, 134 / 120, 5 a row 85.4 /
// 80.5, uniform, 16 a row, 98.4 / 96.3, R-MAT 2^17, 23 a row, 44.1 / 43.2; kz = 60
// banded, 11 a row, 157 / 144, 2 a row 416 / 382) but for ragged FP32 rows of 12
// entries and more on skewed columns (R-MAT 2^17 kz = 48 39.0 / 40.9, 60 51.7 / 54.1;
// 2^19, 16 a row, 123 / 126; 2^20, 10 a row, 131.5 / 131.0), and in the fused pass
// below 4 entries a row (uniform, 2.2, kz = 64 350 / 345, 60 494 / 485, bfloat16 kz =
// 100 563 / 544, 3.9 kz = 64 511 / 505; 8.7 a row 100.5 / 103.1; banded, 11 a row,
// 156 / 160, 5 a row, bfloat16 kz = 100 148 / 157).
//
// Ragged rows past the caches.  They are merged there unless Y is too large (us,
// cached / past the caches: banded, 5.5M entries, Y of 120 MB, kz = 60, SpMM 172 /
// 152, fused 212 / 214, bfloat16 110 / 102 and 178 / 152; uniform, Y of 188 MB,
// bfloat16 kz = 120 SpMM 141 / 130; uniform, Y of 94 MB, kz = 60 80 / 83).
//
// Rows of A.  With one vector a lane, loading the slot's row of A for every
// slot (from L1 mostly) costs less than loading it under a mask where a row
// starts, unless rows are long: 79.6 against 84.2 us on the 2^24-vertex share
// (9.5 entries a row), 100.7 against 95.6 on R-MAT 2^18 (44), kz = 32.  With
// more vectors a lane the L1 traffic decides: banded, 12 entries, kz = 128 892
// against 682 us.
bool pick_run(const Plan* p, int transpose, bool fused, int kz, spc3d_dtype t, bool vec_ok,
              RunShape* sh) {
  const int esz = t == SPC3D_F32 ? 4 : 2;
  sh->vec = 16 / esz;
  const int64_t most = p->R > p->C ? p->R : p->C;
  if (kz < sh->vec || most >= (1 << 24) || most * kz * esz >= (int64_t(1) << 32)) return false;
  const int64_t rows = transpose ? p->C : p->R;
  // a slice of a fused pass ends every row again, and reads its row of A
  const int64_t entries = kz * esz > 512 ? 28 : 36;
  sh->slices =
      fused && p->nnz < entries * rows ? 1 : slice_count(p, transpose, fused, (int64_t)kz * esz);
  sh->kw = kz / sh->slices;
  const int nvec = (sh->kw + sh->vec - 1) / sh->vec;
  if (nvec < 3 || nvec > 32) return false;
  sh->lanes = nvec <= 4 ? 4 : 8;
  sh->nch = nvec <= 8 ? 1 : nvec <= 16 ? 2 : 4;
  sh->full = sh->kw == sh->lanes * sh->nch * sh->vec;
  const bool len16 = p->nnz >= 16 * rows;
  if (vec_ok && kz % sh->vec == 0 && p->nnz >= (int64_t(1) << 17)) {
    const int64_t halves = p->nnz >> 19;   // of 2^20 entries
    if (sh->nch == 4 && p->nnz < (fused ? 20 : 10) * rows) return false;
    if (t == SPC3D_BF16 && sh->nch == 4 && (fused || !skewed(p, transpose))) return false;
    if (t == SPC3D_BF16 && sh->nch == 2) {
      if (fused && p->nnz < 5 * rows) return false;
      if (!fused && sh->slices == 1 &&
          (halves >= 4 || (halves == 1 && !skewed(p, transpose)))) return false;
    }
  }
  sh->each_row = len16;
  sh->step4 = fused ? p->nnz < 4 * rows
                    : sh->full || t == SPC3D_BF16 || p->nnz < 12 * rows || !skewed(p, transpose);
  sh->stream = rows * kz * 4 > (int64_t(100) << 20);
  const int64_t G = 64 / sh->lanes;
  const bool long_runs = len16 || (!fused && sh->nch < 4 && p->nnz >= 8 * rows);
  const int64_t from64 = (fused ? sh->nch == 4 : sh->nch >= 2) ? 4000 : 7000;
  const int64_t from32 = !fused && sh->nch >= 2 ? 6000 : 7000;
  const int64_t from16 = sh->lanes == 4 ? 4000 : sh->nch >= 2 ? 1800 : 2500;
  const int64_t from8 = sh->lanes == 4 ? 1500 : 1000;
  sh->lg_s = long_runs && sh->lanes == 8 && p->nnz >= from64 * 64 * G ? 6
             : p->nnz >= from32 * 32 * G                            ? 5
             : p->nnz >= from16 * 16 * G                            ? 4
             : p->nnz >= from8 * 8 * G                              ? 3
                                                                    : 2;
  const int64_t waves = p->nnz / (G << sh->lg_s);
  sh->ahead = (sh->full && p->nnz < 3 * rows && rows * kz * 4 >= (int64_t(48) << 20)) ||
              (t == SPC3D_F32 &&
               (sh->lanes == 4 ? p->nnz < 10 * rows
                               : p->nnz < 20 * rows && waves < (sh->nch == 1 ? 4096 : 2048)));
  return true;
}

int64_t carry_bytes(int64_t nnz, int64_t item, int kz) {
  const int64_t n = (nnz + item - 1) / item;
  return (n > 0 ? n : 1) * 2 * kz * 4;
}

inline int row_bytes(int kz, spc3d_dtype t) { return kz * (t == SPC3D_F32 ? 4 : 2); }
constexpr int kWholeRow = 512;   // bytes of the widest row that is taken whole

// Scratch of a call through the run family: the carries, and the sums of the
// dots of a sliced fused pass that adds to out (see run_family).
int64_t run_bytes(const Plan* p, const RunShape& sh, bool fused, int kz, spc3d_dtype t,
                  bool acc_out) {
  const bool sums = fused && acc_out && sh.slices > 1 && row_bytes(kz, t) != kWholeRow;
  return carry_bytes(p->nnz, sh.item(), kz) + (sums ? 4 * p->nnz : 0);
}

// Runs the pass through the run family.
void run_family(const Plan* p, RunShape sh, int transpose, const float* d_vals,
                const void* d_X, spc3d_dtype t, int kz, const YOut& Y, int acc, float* carry,
                hipStream_t stream, const void* d_A, float* d_out) {
  Orient o = transpose ? p->csc() : p->csr();
  RunArgs a{};
  a.nnz = p->nnz;
  a.kz = kz;
  a.idx = o.idx;
  a.head = o.head;
  a.tile_row = o.tile_row;
  a.vals = d_vals;
  a.vidx = transpose == 2 ? nullptr : o.vidx;
  a.X = static_cast<const char*>(d_X);
  a.A = static_cast<const char*>(d_A);
  a.Y = Y;
  a.carry = carry;
  a.out = d_out;
  a.acc_out = (acc & kAccOut) != 0;
  const int outm = Y.map ? kAddSlab : (acc & kAccY) ? kAddPacked : kPut;
  if (!d_A) {
    if (t == SPC3D_F32)
      launch_run<float, 4, false>(sh, a, outm, o.ptr, 0, sh.slices, stream);
    else
      launch_run<bf16_t, 8, false>(sh, a, outm, o.ptr, 0, sh.slices, stream);
    return;
  }
  a.dots = d_out;
  if (sh.slices > 1 && a.acc_out) {
    // out holds what is added to: rows of 512 bytes are taken whole, with the
    // runs and so the row sums of the slices; the dots of wider ones are summed
    // behind the carries
    if (row_bytes(kz, t) == kWholeRow) {
      sh.slices = 1;
      sh.kw = kz;
      sh.nch = kWholeRow / 16 / sh.lanes;
    } else {
      a.dots = carry + carry_bytes(p->nnz, sh.item(), kz) / 4;
    }
  }
  for (int s = 0; s < sh.slices; ++s) {
    a.part_first = s == 0;
    a.part_last = s == sh.slices - 1;
    if (t == SPC3D_F32)
      launch_run<float, 4, true>(sh, a, outm, o.ptr, s, 1, stream);
    else
      launch_run<bf16_t, 8, true>(sh, a, outm, o.ptr, s, 1, stream);
  }
}

// Shared body of spc3d_spmm, spc3d_sddmm_spmm, spc3d_sddmm_spmm_static and
// spc3d_sddmm_spmm_scatter.  Y: where finished rows go; acc: kAccY / kAccOut
// bits; static_buf: d_buf is the library's own scratch array.
spc3d_status run_spmm(Plan* p, int transpose, const float* d_vals, const void* d_X,
                      spc3d_dtype x_t, int32_t kz, const YOut& Y, int acc, int variant,
                      void* d_buf, size_t buf_bytes, hipStream_t stream, const void* d_A,
                      float* d_out, bool static_buf = false) {
  const bool fused = d_A != nullptr;
  // The shape, and with it the order of every sum, follows from the operands:
  // the same rows put in Y or added to a slab of any ld and k0 have the same
  // bits.  The destination's alignment decides only what is refused (rows wider
  // than the scalar shapes take).
  const bool al_in = aligned16(d_X) && (!fused || aligned16(d_A));
  const bool al_out = aligned16(Y.base) && Y.ld % 4 == 0;
  const auto lds_of = [&](const Shape& s) {
    return s.window ? size_t(0) : 4 * spmm_wave_lds(s.items, s.lanes, s.nch, s.vec, fused);
  };
  Shape sh;
  spc3d_status st = pick_shape(kz, x_t, al_in && al_out, variant, fused ? 2 : 1, p->nnz, &sh);
  if (st != SPC3D_OK) return st;
  if (al_in && !al_out) {
    Shape vec;
    if (pick_shape(kz, x_t, true, variant, fused ? 2 : 1, p->nnz, &vec) == SPC3D_OK &&
        lds_of(vec) <= 65536)
      sh = vec;
  }
  RunShape rs;
  const bool run = variant < 0 && pick_run(p, transpose, fused, kz, x_t, al_in, &rs) &&
                   buf_bytes >= (size_t)run_bytes(p, rs, fused, kz, x_t, (acc & kAccOut) != 0);
  const int64_t nitems = (p->nnz + sh.items - 1) / sh.items;
  const size_t need = (size_t)nitems * 2 * (size_t)kz * 4;
  if (!run && buf_bytes < need) {
    if (static_buf)
      return fail(SPC3D_ERR_WORKSPACE,
                  "this call needs %zu bytes of scratch; the library's static scratch holds %zu "
                  "(use spc3d_sddmm_spmm with a caller buffer)", need, buf_bytes);
    return fail(SPC3D_ERR_WORKSPACE, "SpMM buffer %zu bytes < %zu required", buf_bytes, need);
  }
  const size_t lds = lds_of(sh);
  if (lds > 65536) return fail(SPC3D_ERR_UNSUPPORTED, "variant needs %zu bytes of LDS", lds);
  DeviceGuard dg;
  st = dg.enter(p);
  if (st != SPC3D_OK) return st;
  SPC3D_DEBUG_CHECK(p, stream);
  if (run) {
    run_family(p, rs, transpose, d_vals, d_X, x_t, kz, Y, acc, static_cast<float*>(d_buf), stream,
               d_A, d_out);
    SPC3D_LAUNCHED(fused ? "sddmm_spmm" : "spmm");
    return SPC3D_OK;
  }
  const int64_t nblocks = (nitems + 3) / 4;
  Orient o = transpose ? p->csc() : p->csr();
  if (transpose == 2) o.vidx = nullptr;   // values already in column-major slot order
  float* carry = static_cast<float*>(d_buf);
#define SPC3D_RUN(T, V)                                                                        \
  do {                                                                                         \
    if (fused)                                                                                 \
      launch_spmm<T, V, true>(sh, stream, p->nnz, nitems, nblocks, o, d_vals, d_X, kz, Y, acc, \
                              carry, lds, d_A, d_out);                                         \
    else                                                                                       \
      launch_spmm<T, V, false>(sh, stream, p->nnz, nitems, nblocks, o, d_vals, d_X, kz, Y, acc,\
                               carry, lds, nullptr, nullptr);                                  \
  } while (0)
  if (x_t == SPC3D_F32) {
    if (sh.vec == 4) SPC3D_RUN(float, 4);
    else SPC3D_RUN(float, 1);
  } else {
    if (sh.vec == 8) SPC3D_RUN(bf16_t, 8);
    else SPC3D_RUN(bf16_t, 1);
  }
#undef SPC3D_RUN
  SPC3D_LAUNCHED(fused ? "sddmm_spmm" : "spmm");
  return SPC3D_OK;
}

// The kernels' accumulate bits for an output mode that applies to both outputs.
int acc_bits(int mode) { return mode == SPC3D_ACCUMULATE ? (kAccY | kAccOut) : 0; }

// Arguments common to the fused entry points.
spc3d_status check_fused_args(spc3d_plan h, Plan** p, spc3d_dtype ab_t, int32_t kz, int mode) {
  spc3d_status st = get_plan(h, p);
  if (st != SPC3D_OK) return st;
  if (ab_t != SPC3D_F32 && ab_t != SPC3D_BF16) return fail(SPC3D_ERR_INVALID_ARG, "bad ab_t");
  if (mode != SPC3D_OVERWRITE && mode != SPC3D_ACCUMULATE)
    return fail(SPC3D_ERR_INVALID_ARG, "bad mode");
  if (kz < 1 || kz > kMaxKz) return fail(SPC3D_ERR_INVALID_ARG, "kz=%d outside [1,%d]", kz, kMaxKz);
  return SPC3D_OK;
}

// The scratch of spc3d_sddmm_spmm_static: the SpMM carries of one call, in a
// device array the library owns.  Each GPU the library runs on holds its own
// copy (kept until the process ends); host code reaches it only through the
// device address hipGetSymbolAddress gives with that GPU current.
static __device__ __align__(256) char scratch[SPC3D_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_addr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up once per device).
spc3d_status static_scratch(void** out) {
  int dev = -1;
  SPC3D_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices)
    return fail(SPC3D_ERR_UNSUPPORTED, "device %d beyond the %d the static scratch serves", dev,
                kMaxDevices);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_addr[dev]) {
    void* addr = nullptr;
    SPC3D_HIP(hipGetSymbolAddress(&addr, HIP_SYMBOL(scratch)));
    if (!addr) return fail(SPC3D_ERR_HIP, "hipGetSymbolAddress gave no address for the scratch");
    g_scratch_addr[dev] = addr;
  }
  *out = g_scratch_addr[dev];
  return SPC3D_OK;
}

}  // namespace
}  // namespace spc3d

using namespace spc3d;

extern "C" {

spc3d_status spc3d_sddmm(spc3d_plan h, const float* d_vals, const void* d_A, const void* d_B,
                         spc3d_dtype ab_t, int32_t kz, float* d_out, int mode, int variant,
                         hipStream_t stream) {
  Plan* p;
  spc3d_status st = get_plan(h, &p);
  if (st != SPC3D_OK) return st;
  if (ab_t != SPC3D_F32 && ab_t != SPC3D_BF16) return fail(SPC3D_ERR_INVALID_ARG, "bad ab_t");
  if (mode != SPC3D_OVERWRITE && mode != SPC3D_ACCUMULATE)
    return fail(SPC3D_ERR_INVALID_ARG, "bad mode");
  if (kz < 1 || kz > kMaxKz) return fail(SPC3D_ERR_INVALID_ARG, "kz=%d outside [1,%d]", kz, kMaxKz);
  if (p->nnz == 0) return SPC3D_OK;
  if (!d_A || !d_B || !d_out) return fail(SPC3D_ERR_INVALID_ARG, "NULL buffer");
  Shape sh;
  st = pick_shape(kz, ab_t, aligned16(d_A) && aligned16(d_B), variant, 0, p->nnz, &sh);
  if (st != SPC3D_OK) return st;
  DeviceGuard dg;
  st = dg.enter(p);
  if (st != SPC3D_OK) return st;
  SPC3D_DEBUG_CHECK(p, stream);
  const int64_t nitems = (p->nnz + sh.items - 1) / sh.items;
  const int64_t nblocks = (nitems + 3) / 4;
  const Orient o = p->csr();
  const int acc = mode == SPC3D_ACCUMULATE;
  if (variant < 0 && pick_ragged(kz, ab_t, d_A, d_B, &sh)) {
    launch_sddmm_ragged<bf16_t, 8>(sh, stream, p->nnz, nitems, nblocks, o, d_vals, d_A, d_B, kz,
                                   d_out, acc);
  } else if (ab_t == SPC3D_F32) {
    if (sh.vec == 4)
      launch_sddmm<float, 4>(sh, stream, p->nnz, nitems, nblocks, o, d_vals, d_A, d_B, kz, d_out,
                             acc);
    else
      launch_sddmm<float, 1>(sh, stream, p->nnz, nitems, nblocks, o, d_vals, d_A, d_B, kz, d_out,
                             acc);
  } else {
    if (sh.vec == 8)
      launch_sddmm<bf16_t, 8>(sh, stream, p->nnz, nitems, nblocks, o, d_vals, d_A, d_B, kz,
                              d_out, acc);
    else
      launch_sddmm<bf16_t, 1>(sh, stream, p->nnz, nitems, nblocks, o, d_vals, d_A, d_B, kz,
                              d_out, acc);
  }
  SPC3D_LAUNCHED("sddmm");
  return SPC3D_OK;
}

spc3d_status spc3d_spmm_buffer_size(spc3d_plan h, int transpose, int32_t kz, int variant,
                                    size_t* bytes) {
  Plan* p;
  spc3d_status st = get_plan(h, &p);
  if (st != SPC3D_OK) return st;
  if (!bytes) return fail(SPC3D_ERR_INVALID_ARG, "bytes is NULL");
  if (kz < 1 || kz > kMaxKz) return fail(SPC3D_ERR_INVALID_ARG, "kz=%d outside [1,%d]", kz, kMaxKz);
  // The work-item size, and so the number of carries, depends on the shape a
  // call takes: the operand type, whether the operands are 16-byte aligned
  // and whether the pass is fused.  The size covers every shape that can run.
  int64_t items = 0;
  bool any = false;
  spc3d_status first = SPC3D_OK;
  for (int op = 1; op <= 2; ++op)
    for (int t = 0; t < 2; ++t)
      for (int al = 1; al >= 0; --al) {
        Shape sh;
        st = pick_shape(kz, t ? SPC3D_BF16 : SPC3D_F32, al != 0, variant, op, p->nnz, &sh);
        if (st == SPC3D_OK) {
          any = true;
          const int64_t n = (p->nnz + sh.items - 1) / sh.items;
          items = n > items ? n : items;
        } else if (first == SPC3D_OK) {
          first = st;
        }
      }
  if (!any) return first;
  *bytes = (size_t)(items > 0 ? items : 1) * 2 * (size_t)kz * 4;
  if (variant < 0)
    for (int f = 0; f < 2; ++f)
      for (int t = 0; t < 2; ++t) {
        RunShape rs;
        if (!pick_run(p, transpose, f != 0, kz, t ? SPC3D_BF16 : SPC3D_F32, false, &rs)) continue;
        const size_t n = (size_t)run_bytes(p, rs, f != 0, kz, t ? SPC3D_BF16 : SPC3D_F32, true);
        if (n > *bytes) *bytes = n;
      }
  return SPC3D_OK;
}

spc3d_status spc3d_spmm(spc3d_plan h, int transpose, const float* d_vals, const void* d_X,
                        spc3d_dtype x_t, int32_t kz, float* d_Y, int mode, int variant,
                        void* d_buf, size_t buf_bytes, hipStream_t stream) {
  Plan* p;
  spc3d_status st = get_plan(h, &p);
  if (st != SPC3D_OK) return st;
  if (transpose < 0 || transpose > 2) return fail(SPC3D_ERR_INVALID_ARG, "bad transpose");
  if (transpose && !(p->flags & SPC3D_BUILD_CSC))
    return fail(SPC3D_ERR_INVALID_ARG, "transposed SpMM needs a plan built with BUILD_CSC");
  if (x_t != SPC3D_F32 && x_t != SPC3D_BF16) return fail(SPC3D_ERR_INVALID_ARG, "bad x_t");
  if (mode != SPC3D_OVERWRITE && mode != SPC3D_ACCUMULATE)
    return fail(SPC3D_ERR_INVALID_ARG, "bad mode");
  if (kz < 1 || kz > kMaxKz) return fail(SPC3D_ERR_INVALID_ARG, "kz=%d outside [1,%d]", kz, kMaxKz);
  if (p->nnz == 0) return SPC3D_OK;
  if (!d_X || !d_Y || !d_buf) return fail(SPC3D_ERR_INVALID_ARG, "NULL buffer");
  if (reinterpret_cast<uintptr_t>(d_buf) & 255u)
    return fail(SPC3D_ERR_INVALID_ARG, "buffer must be 256-byte aligned");
  const YOut Y{d_Y, nullptr, 0, kz, 0};
  return run_spmm(p, transpose, d_vals, d_X, x_t, kz, Y, acc_bits(mode), variant, d_buf,
                  buf_bytes, stream, nullptr, nullptr);
}

spc3d_status spc3d_sddmm_spmm(spc3d_plan h, const float* d_vals, const void* d_A, const void* d_B,
                              spc3d_dtype ab_t, int32_t kz, float* d_out, float* d_Y, int mode,
                              int variant, void* d_buf, size_t buf_bytes, hipStream_t stream) {
  Plan* p;
  spc3d_status st = check_fused_args(h, &p, ab_t, kz, mode);
  if (st != SPC3D_OK) return st;
  if (p->nnz == 0) return SPC3D_OK;
  if (!d_A || !d_B || !d_out || !d_Y || !d_buf) return fail(SPC3D_ERR_INVALID_ARG, "NULL buffer");
  if (reinterpret_cast<uintptr_t>(d_buf) & 255u)
    return fail(SPC3D_ERR_INVALID_ARG, "buffer must be 256-byte aligned");
  const YOut Y{d_Y, nullptr, 0, kz, 0};
  return run_spmm(p, 0, d_vals, d_B, ab_t, kz, Y, acc_bits(mode), variant, d_buf, buf_bytes,
                  stream, d_A, d_out);
}

spc3d_status spc3d_sddmm_spmm_static(spc3d_plan h, const float* d_vals, const void* d_A,
                                     const void* d_B, spc3d_dtype ab_t, int32_t kz, float* d_out,
                                     float* d_Y, int mode, int variant, hipStream_t stream) {
  Plan* p;
  spc3d_status st = check_fused_args(h, &p, ab_t, kz, mode);
  if (st != SPC3D_OK) return st;
  if (p->nnz == 0) return SPC3D_OK;
  if (!d_A || !d_B || !d_out || !d_Y) return fail(SPC3D_ERR_INVALID_ARG, "NULL buffer");
  DeviceGuard dg;
  st = dg.enter(p);
  if (st != SPC3D_OK) return st;
  void* buf = nullptr;
  st = static_scratch(&buf);
  if (st != SPC3D_OK) return st;
  const YOut Y{d_Y, nullptr, 0, kz, 0};
  return run_spmm(p, 0, d_vals, d_B, ab_t, kz, Y, acc_bits(mode), variant, buf,
                  SPC3D_STATIC_SCRATCH_BYTES, stream, d_A, d_out, true);
}

spc3d_status spc3d_sddmm_spmm_scatter(spc3d_plan h, const float* d_vals, const void* d_A,
                                      const void* d_B, spc3d_dtype ab_t, int32_t kz, float* d_out,
                                      int out_mode, float* d_dst, int64_t ld_dst, int32_t k0,
                                      int variant, void* d_buf, size_t buf_bytes,
                                      hipStream_t stream) {
  Plan* p;
  spc3d_status st = check_fused_args(h, &p, ab_t, kz, out_mode);
  if (st != SPC3D_OK) return st;
  if (k0 < 0 || ld_dst < (int64_t)k0 + kz)
    return fail(SPC3D_ERR_INVALID_ARG, "k0=%d kz=%d do not fit ld_dst=%lld", k0, kz,
                (long long)ld_dst);
  if (p->nnz == 0) return SPC3D_OK;
  if (!d_A || !d_B || !d_out || !d_dst || !d_buf) return fail(SPC3D_ERR_INVALID_ARG, "NULL buffer");
  if (reinterpret_cast<uintptr_t>(d_buf) & 255u)
    return fail(SPC3D_ERR_INVALID_ARG, "buffer must be 256-byte aligned");
  const YOut Y{d_dst + k0, p->gmap_r, p->row_lo, ld_dst, p->R};
  const int acc = kAccY | (out_mode == SPC3D_ACCUMULATE ? kAccOut : 0);
  return run_spmm(p, 0, d_vals, d_B, ab_t, kz, Y, acc, variant, d_buf, buf_bytes, stream, d_A,
                  d_out);
}

spc3d_status spc3d_variant_check(int op, int32_t kz, spc3d_dtype ab_t, int variant) {
  if (op < SPC3D_OP_SDDMM || op > SPC3D_OP_SDDMM_SPMM) return fail(SPC3D_ERR_INVALID_ARG, "bad op %d", op);
  if (ab_t != SPC3D_F32 && ab_t != SPC3D_BF16) return fail(SPC3D_ERR_INVALID_ARG, "bad ab_t");
  if (kz < 1 || kz > kMaxKz) return fail(SPC3D_ERR_INVALID_ARG, "kz=%d outside [1,%d]", kz, kMaxKz);
  Shape sh;
  return pick_shape(kz, ab_t, true, variant, op, 0, &sh);
}

}  // extern "C"
