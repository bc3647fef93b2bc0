// The stage-launch policy of the C ABI: which stage kernel runs (the
// automatic choice), the alternating work-item order, and the stage
// parameters of a context.

#include <algorithm>

#include "api_internal.h"

namespace wadg {
namespace host {

// LSRK(5,4) 2N-storage coefficients (Carpenter & Kennedy 1994), the
// integrator of the paper's experiments (Section 5.2).
const double kRkA[5] = {0.0,
                        -567301805773.0 / 1357537059087.0,
                        -2404267990393.0 / 2016746695238.0,
                        -3550918686646.0 / 2091501179385.0,
                        -1275806237668.0 / 842570457699.0};
const double kRkB[5] = {1432997174477.0 / 9575080441755.0,
                        5161836677717.0 / 13612068292357.0,
                        1720146321549.0 / 2090206949498.0,
                        3134564353537.0 / 4481467310338.0,
                        2277821191437.0 / 14882151754819.0};

// The base variant of a launch: the selectable kernel that its context,
// precision and mode lead to without regard to its size (but S = 1).  An
// explicit choice launches it; the automatic one starts from it
// (launch_kernel).  From measurement on MI355X (64x64 and 128x128 elements, N
// = 3, FP64 and FP32): LSRK stages of two or more slices take the pipelined
// kernel where its LDS plan fits, else the split-work kernel; right-hand
// sides the resident-geometry kernel where the geometry fits in LDS, else
// the split-work kernel; the adjoint's apply-A launches the split-work
// kernel (the resident kernel has no apply-A mode, so an explicit RESIDENT
// or STREAMED choice runs them streamed).
int kernel_path(wadg_ctx c, bool fp32, int mode, int32_t S) {
  if (mode == wadg::kStage && (c->kernel == WADG_KERNEL_PIPE || c->kernel == WADG_KERNEL_AUTO) &&
      S >= kPipeMinSlices && wadg::pipe_supported(c->N, c->nq1, fp32))
    return WADG_KERNEL_PIPE;
  if (c->kernel == WADG_KERNEL_PIPE) return WADG_KERNEL_SPLIT;  // its other launches
  const bool fits = wadg::resident_supported(c->N, c->nq1, fp32);
  if (mode == wadg::kApplyAMass) return WADG_KERNEL_SPLIT;   // split kernel only
  if (mode == wadg::kApplyA)   // no resident apply-A mode
    return c->kernel == WADG_KERNEL_AUTO || c->kernel == WADG_KERNEL_SPLIT ? WADG_KERNEL_SPLIT
                                                                           : WADG_KERNEL_STREAMED;
  if (c->kernel == WADG_KERNEL_RESIDENT && fits) return WADG_KERNEL_RESIDENT;
  if (c->kernel != WADG_KERNEL_AUTO) return c->kernel == WADG_KERNEL_RESIDENT
                                                ? WADG_KERNEL_STREAMED : c->kernel;
  if (mode == wadg::kRhs && fits) return WADG_KERNEL_RESIDENT;
  return WADG_KERNEL_SPLIT;
}

namespace {

int64_t sets_of(wadg_ctx c, int32_t S) { return (int64_t)((c->K + 15) / 16) * S; }

// Whether an automatic launch over `sets` sets of 16 elements, S slices, takes
// the quarter kernel: up to about as many sets as fill the CUs once.  Its
// launch takes the time of one short item, but each workgroup reads its own
// copy of the geometry and exchanges every intermediate through LDS, so it
// loses where several sets queue on a CU.  Measured on MI355X (256 CUs), one
// launch against the kernel that otherwise runs, us:
//   FP64 stages and the adjoint's launches, N = 3, nq1 = 5: 8.3 -> 5.8 at 64
// sets, 9.4 -> 6.9 at 256, 9.6 -> 8.6 at 384, 11.7 -> 12.1 at 1024; N = 4,
// nq1 = 6: 12.7 -> 9.0 at 64, 15.8 -> 13.9 at 384, 14.8 -> 16.0 at 576.
// Stages stop at 256 sets at nq1 <= 3, whose items are short (N = 2, nq1 = 3:
// 5.8 -> 6.0 at 384), and at N = 3, nq1 = 6, whose instance spills (12.0 ->
// 12.7 at 324, 12.2 -> 13.1 at 381; right-hand sides 9 % faster there).
//   FP32 of one slice, against the split kernel: N = 3: 6.7 -> 4.8 at 64 sets,
// 9.3 -> 8.5 at 1024; N = 2: 5.4 -> 4.9 at 484, 6.33 -> 6.39 at 1024.
//   FP32 of more slices, against the pipelined kernel, which holds two
// workgroups per CU: N = 3, nq1 = 5: 10 % faster at 512 sets, 1 % at 576, 7.9
// -> 8.5 at 800, 8.2 -> 9.5 at 1024; N = 4, nq1 = 5: 9.3 -> 9.6 at 628, 10.2
// -> 12.4 at 1024; nq1 = 7: 13.0 -> 15.4 at 785; N = 1, 2: nq1 <= 3 even at 256
// to 384, 3.8 -> 4.05 at 512; nq1 = 4, 5: 4 % faster at 512.
bool takes_quarter(wadg_ctx c, int mode, bool fp32, int32_t S, int64_t sets) {
  if (c->kernel != WADG_KERNEL_AUTO) return false;
  const int64_t cus = c->cus;
  const bool shortest = c->nq1 <= 3;
  if (!fp32)
    return sets <= (mode == wadg::kStage && (shortest || (c->N == 3 && c->nq1 == 6))
                        ? cus : cus * 3 / 2);
  if (S == 1) return sets <= (c->N >= 3 ? cus * 4 : cus * 2);
  return sets <= (c->N >= 3 ? cus * 9 / 4 : shortest ? cus : cus * 2);
}

// Whether an automatic FP64 stage or right-hand side whose geometry does not
// fit on chip (N = 4; N = 3 with nq1 = 6) takes the pipelined kernel's form
// that streams it, rather than the split kernel.  Each workgroup a CU runs
// walks ceil(S / chunks) slices and takes one step more to drain the
// pipeline, and a CU runs the split kernel's items two at a time; a step
// takes about two thirds of such a round's time, so the shorter sum decides
// (a run of one slice per workgroup stays split).  Measured on MI355X (256
// CUs), stage and right-hand side, us, split -> pipelined: N = 4, nq1 = 6:
// 50x50 elements and 32 slices (5 rounds, 7 steps) 72.5 -> 66.4, 64.9 -> 52.8;
// 128x128 and 64 slices (64, 65) 875 -> 659, 752 -> 514; 50x50 and 12 (2, 3)
// 30.2 -> 28.1; but 96x96 and 16 (9, 17) 126 -> 142; 50x50 and 6 (1, 2) 16.4
// -> 17.9; nq1 = 5, 50x50 and 32: 59 -> 46.8, 50 -> 37.8; nq1 = 7: 94 -> 77, 82
// -> 64; N = 3, nq1 = 6, 64x64 and 64: 164 -> 112, 135 -> 86; 24x24 and 30
// (2, 3) 24.3 -> 18.5; 200x200 and 3 (8, 3 x 4) 84 -> 76.
bool takes_streamed_pipe(wadg_ctx c, int32_t S) {
  const int64_t nEG = c->groups(), chunks = wadg::pipe_chunks((int)nEG, S, c->cus);
  // (workgroups one after another on a CU)
  const int64_t runs = (nEG * chunks + c->cus - 1) / c->cus;
  const int64_t steps = runs * ((S + chunks - 1) / chunks + 1);
  const int64_t rounds = (nEG * S + c->cus - 1) / c->cus;
  return 3 * rounds >= 2 * steps;
}

}  // namespace

// The kernel of a launch of S slices: the base variant, or in an automatic
// choice the quarter kernel (few elements) or the pipelined kernel (right-hand
// sides, and FP64 launches whose geometry it streams).
//
// An automatic right-hand side whose geometry fits on chip runs on the
// pipelined kernel, which holds it there too and overlaps one slice's loads
// and face terms with another's mass inverse.  Measured on MI355X against
// the resident kernel, bitwise the same: 128x128 elements, N = 3, nq1 = 5,
// 256 slices 1,178 -> 909 us, 2 slices 20.4 -> 16.6, 1 slice 18.5 -> 11.1;
// 81x81, N = 2, 24 slices 39.9 -> 30.7; 64x64, N = 1, 64 slices 28.4 ->
// 19.3 (never slower at any size measured).
int launch_kernel(wadg_ctx c, int mode, bool fp32, int32_t S) {
  const int base = kernel_path(c, fp32, mode, S);
  if (c->kernel != WADG_KERNEL_AUTO) return base;
  if (takes_quarter(c, mode, fp32, S, sets_of(c, S))) return WADG_KERNEL_QUARTER;
  if (!fp32 && wadg::pipe_supported(c->N, c->nq1, false))
    return mode == wadg::kRhs ? WADG_KERNEL_PIPE : base;
  if (!fp32 && (mode == wadg::kStage || mode == wadg::kRhs) && takes_streamed_pipe(c, S))
    return WADG_KERNEL_PIPE;
  return base;
}

int launch_stage(wadg_ctx c, int mode, bool fp32, const wadg::StageParams& p0, void* stream) {
  const int kernel = launch_kernel(c, mode, fp32, p0.S);
  if (kernel == WADG_KERNEL_PIPE)
    return fp32 ? wadg::launch_stage_pipe_fp32(c->N, c->nq1, p0, c->cus, stream)
                : wadg::launch_stage_pipe(c->N, c->nq1, mode, p0, c->cus, stream);
  // alternate the item order from one launch to the next (item_of)
  wadg::StageParams p = p0;
  c->order_flip ^= 1;
  p.reverse = (int32_t)c->order_flip;
  if (kernel == WADG_KERNEL_QUARTER)
    return fp32 ? wadg::launch_stage_quarter_fp32(c->N, c->nq1, p, stream)
                : wadg::launch_stage_quarter(c->N, c->nq1, mode, p, stream);
  if (kernel == WADG_KERNEL_SPLIT)
    return fp32 ? wadg::launch_stage_split_fp32(c->N, c->nq1, p, stream)
                : wadg::launch_stage_split(c->N, c->nq1, mode, p, stream);
  if (kernel == WADG_KERNEL_RESIDENT) {
    const int ranges = wadg::resident_ranges(p.nEG, p.S, c->cus);
    return fp32 ? wadg::launch_stage_resident_fp32(c->N, c->nq1, p, ranges, stream)
                : wadg::launch_stage_resident(c->N, c->nq1, mode, p, ranges, stream);
  }
  return fp32 ? wadg::launch_stage_streamed_fp32(c->N, c->nq1, p, stream)
              : wadg::launch_stage_streamed(c->N, c->nq1, mode, p, stream);
}

int launch_stage_pair(wadg_ctx c, int mode_a, const wadg::StageParams& a0,
                      const wadg::StageParams& b0, void* stream) {
  wadg::StageParams a = a0, b = b0;
  c->order_flip ^= 1;
  a.reverse = b.reverse = (int32_t)c->order_flip;
  if (takes_quarter(c, mode_a, false, a0.S, sets_of(c, a0.S) + sets_of(c, b0.S)))
    return wadg::launch_stage_quarter_pair(c->N, c->nq1, mode_a, a, b, stream);
  return wadg::launch_stage_pair(c->N, c->nq1, mode_a, a, b, stream);
}

// One launch for the whole sweep where a slice's mesh fits in one workgroup
// (quarter_sweep_kernel), by its sets of 16 elements:
//   one or two: always;
//   three, N >= 3: always, but for N = 3, nq1 = 5 with more than 8 slices per
// CU whose stages find their three arrays in the 256 MB memory-side cache;
//   three, N <= 2: up to 4 slices per CU; four: up to 2.  Beyond, many slices
// fill the chip better from the stage kernels;
//   FP64 workgroups of 15 or 16 waves at N >= 3, nq1 >= 5 (three sets at nq1 =
// 7, else four), which are held to 128 registers per lane and spill: only
// where there are too many slices for the quarter kernel's stages, and few
// enough to run at once.
// Measured per stage on MI355X (256 CUs), us, the stage launches against this
// one: N = 3, nq1 = 5, FP64: 16 elements, 1 slice 7.9 -> 2.6, 4096 slices 61.6
// -> 19.0; 25 elements, 4096 slices 64 -> 49; 36 elements, 2048 slices 34.4 ->
// 33.1, 3072 47.1 -> 49.0, 16384 294 -> 261; 64 elements, 1 slice 6.0 -> 7.6 (one step; 5.4 ->
// 5.7 of eight), 128 slices 1.41x, 512 1.18x, 2048 36.7 -> 53.8.  FP32: 36
// elements, 2048 slices 21.3 -> 19.7, 4096 34.0 -> 38.5, 6144 49.4 -> 57.6,
// 12288 1.25x; nq1 = 4 and 6 there 1.17x, 1.06x.  nq1 = 6, FP64: 64 elements, 1
// slice 8.4 -> 10.3, 256 slices 1.48x, 512 19.5 -> 22.7.  N = 4: 36 elements,
// FP64, nq1 = 5, 6: 1.13x to 2.5x at any number; nq1 = 7: 1 slice 8.8 ->
// 14.4, 256 1.31x, 1024 54 -> 61, 16384 739 -> 967 (25 elements: 1.28x to 3.0x); FP32
// 1.2x to 2.7x.  N = 1, nq1 = 3, 36 elements: 1024 slices 1.22x, 4096 19.9 ->
// 27.4; N = 2, nq1 = 5: 1.24x, 46.5 -> 53.2.
bool one_launch_sweep(wadg_ctx c, bool fp32, int32_t S) {
  if (c->kernel != WADG_KERNEL_AUTO ||
      c->K > wadg::quarter_sweep_elements(c->N, c->nq1, fp32))
    return false;
  const int sets = (c->K + 15) / 16;
  const int64_t cus = c->cus;
  if (sets <= 2) return true;
  if (!fp32 && c->N >= 3 && c->nq1 >= 5 && sets == (c->nq1 == 7 ? 3 : 4))
    return S <= (c->nq1 == 5 ? 2 * cus : cus) &&
           !takes_quarter(c, wadg::kStage, fp32, S, sets_of(c, S));
  if (sets == 4) return S <= 2 * cus;
  if (c->N < 3) return S <= 4 * cus;
  const int64_t arrays = 3 * (int64_t)c->state_doubles(S) * (fp32 ? 4 : 8);
  return !(c->N == 3 && c->nq1 == 5 && S > 8 * cus && arrays <= (int64_t)256 << 20);
}

// A launch of quarter_sweep_kernel holds its CUs until its last step, so a
// sweep of many steps is cut: at most 512 steps of as many slices as there
// are CUs, or fewer steps of more slices.  Such a launch takes 7 ms (16
// elements, N = 3; 31 ms at the slowest kernel measured, 12 us per stage),
// its start 10 us: below 0.2 %.  A step starts from A = 0 and nothing but the
// state is carried over (in FP32 exactly, through FP64), so the cut changes
// no bit.
int launch_sweep(wadg_ctx c, const double* Qin, double* Qout, const wadg::StageParams& p,
                 int32_t nsteps, bool fp32, void* stream) {
  wadg::SweepCoefs rk;
  for (int i = 0; i < 5; ++i) {
    rk.A[i] = kRkA[i];
    rk.B[i] = kRkB[i];
  }
  const int32_t rounds = (p.S - 1) / c->cus + 1;
  const int32_t most = std::max(1, 512 / rounds);
  for (int32_t done = 0; done < nsteps; done += std::min(most, nsteps - done)) {
    int e = wadg::launch_sweep_quarter(c->N, c->nq1, done ? Qout : Qin, Qout, p, rk,
                                       std::min(most, nsteps - done), fp32, stream);
    if (e) return e;
  }
  return 0;
}

wadg::StageParams base_params(wadg_ctx c, int32_t S) {
  wadg::StageParams p{};
  p.vol = c->d_vol;
  p.face = c->d_face;
  p.nbr = c->d_nbr;
  p.K = c->K;
  p.S = S;
  p.nEG = (c->K + wadg::kWave - 1) / wadg::kWave;
  p.tile_groups = c->tile_groups < p.nEG ? c->tile_groups : p.nEG;
  // (a scattered mesh: an eighth of the slices per tile, so that each XCD
  // walks slices of its own, as in the pipelined kernel; split kernel, N = 4,
  // nq1 = 6, 64x64 elements at random x 8 slices 40.3 -> 38.1 us per stage)
  const int ts = c->tile_slices >= 0 ? c->tile_slices : c->scattered ? (S + 7) / 8 : 0;
  p.tile_slices = (ts == 0 || ts > S) ? S : ts;
  p.scattered = c->scattered;
  p.tau_p = c->tau_p;
  p.tau_u = c->tau_u;
  p.c2_scale = c->c2_scale;
  p.res_out = nullptr;
  p.res_dead = 0;
  return p;
}

}  // namespace host
}  // namespace wadg
