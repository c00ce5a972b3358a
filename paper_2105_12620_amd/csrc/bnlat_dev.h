// Internal interface between the C-ABI host code and the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lattice_lines.h"

namespace bnlat {

// Philox stream tags (fourth counter word).
constexpr uint32_t S_INIT = 0xA;
constexpr uint32_t S_INTEG = 0xB;
constexpr uint32_t S_PROP = 0xC;

// Integrand rows are padded to a multiple of this many entries; padded rows
// have normal (0, 0) and threshold 0, so their hit count is always 0 and they
// contribute nothing to energies.
constexpr uint32_t T_ALIGN = 128;
constexpr uint32_t MAX_RADIUS = 8;
constexpr uint32_t MAX_N = 4096;
// Size of the per-GPU scratch array of the allocation-free entry point.
constexpr size_t NOALLOC_SCRATCH_BYTES = (size_t)32 << 20;

// MODE_SWEEP: proposals of every pixel of a sweep, rows grouped by colour
// class ([class][class pixel]); the kernel argument kappa is then the sweep
// look-ahead added to the device sweep counter.
enum CountMode : int { MODE_ALL = 0, MODE_CLASS = 1, MODE_LIST = 2, MODE_SWEEP = 3 };

// Operands of the colour phases: uint16 counts, or int8 deviations (phase_gram.h).
enum FieldForm : int { FIELD_WIDE = 0, FIELD_NARROW = 1, FIELD_SPLIT = 2 };

// Everything a kernel needs to know about one problem, passed by value.
struct DevView {
  uint32_t n, log2n, w, h, t, tp, k, cw, ch, pc;
  uint32_t problem, seed_lo, seed_hi;
  int32_t objective;
  uint32_t radius, ncls;
  const uint32_t* lat;       // [n] lattice points, x | y << 16, index order i
  const int2* ihp;           // [tp] (nx | ny << 16, D' = n . (C - 2^15))
  uint32_t lines;            // lattice lines of the line counter (a template size; 0: sample counter)
  uint32_t gx, gy;           // lattice generator
  const uint32_t* lrow;      // [n][line_row_words(lines)] lattice lines of each shift class
  const LineRec* lrec;       // [tp]
  const float* area;         // [tp] FP32 exact integrals (0 for padding)
  const int32_t* dcls;       // [2 radius^2 + 1] class of a squared distance
  const double* wd;          // [ncls] class weights exp(-d / sigma^2)
  uint32_t* U;               // [P] offsets, x | y << 16
  uint32_t* seen;            // [P] offsets whose counts d8 holds, where the caller owns offsets and counts,
                             // else null
  uint16_t* cnt;             // [tp/8][P][8] hit counts (16-byte integrand tiles)
  float* err;                // [P][tp] error vectors
  uint32_t* u_new;           // [M] proposals of the current phase / list
  uint16_t* c_new;           // [tp/8][M][8] recounted hits of the proposals
  uint32_t form;             // FieldForm of the colour phases
  int8_t* d8;                // narrow forms: [tp/16][P][16] counts less their integrand's base, else null
  int8_t* n8;                // narrow forms: [tp/16][M][16] the same of the proposals (c_new is null)
  const uint32_t* bias8;     // [tp/2] 0x00800080 - (base of 2 i | base of 2 i + 1 << 16)
  // sweeps on narrow forms (moves_wait): the accepted moves of the classes
  // before this one are still proposals, committed together after the last class
  uint32_t decided;          // classes whose moves wait (0 otherwise)
  uint8_t* accepts;          // [K^2][pc] the sweep's decisions, else null
  const int8_t* n8_sweep;    // n8 of class 0
  double* delta;             // [M] energy change
  uint8_t* accept;           // [M] decision
  const uint32_t* pix_list;  // [M] pixels (list mode)
  unsigned long long* ctr;   // [0] sweep index, [1] accepted total, [2] BF16 vetoes,
                             // [3] the overlapped schedule's recount index
  uint32_t span;             // words of 8 counts whose class sums fit int32 (wide form)
  uint32_t slices;           // integrand slices of a colour phase (phase_slices)
  long long* xsum;           // [slices][pc][ncls + 1] their class sums and self terms (null: one slice)
  long long* xpart;          // [ncls][pc] integer class sums of the BF16 pass (kept zero between phases), else null
  uint32_t* unsure;          // [pc] matrix-core results not certified exact (kept zero between phases)
  uint32_t mfma;             // colour phases' evaluation: 0 FP32 form (exact integer stencil), 1 BF16 matrix
                             // cores on exact counts (N <= 256, Heaviside rows only), 2 BF16 matrix cores on
                             // rounded error vectors with exact re-evaluation of accepted moves
  uint32_t tb;               // rows of the BF16 field: tp + tgp
  uint16_t* bf;              // [tb/8][P][8] BF16 field (mode 1: counts; mode 2: errors), else null
  double* delta_bf;          // [M] energy change the BF16 pass computed (before re-evaluation), else null
  double xscale;             // energy change = xscale * sum_d w_d X_d of the class sums X_d
  uint32_t tch;              // integrands per wave in the counting kernels (launch shape)
  uint32_t slice_target;     // workgroups the BF16 pass aims for
  uint32_t count_cap;        // workgroup cap of the sweep-wide recount launch (0: none)
  // Gaussian integrands (tgp = 0 when there are none)
  uint32_t tg, tgp;          // count, padded to 64
  const double* gcoef;       // [tgp][4] exponent coefficients a, bx, by, c (base 2; 0 for padding)
  uint32_t glines, gwords;   // Gaussian line form: lines (0: sample by sample), doubles per table
  const uint32_t* grow;      // [n][1 + glines] lattice lines of each shift class (lattice_lines.h)
  const int* gspans;         // [glines][4] steps, full_lo, full_hi, steps of b1 from O + b2 to the next origin
  const double* gtab;        // [tg / 4 rounded up][gwords][4] tables (lattice_lines.h)
  const double* gint;        // [tgp] exact integrals
  float* gest;               // [P][tgp] estimates
  float* gerr;               // [P][tgp] errors g - I (refreshed on demand)
  float* g_new;              // [M][tgp] estimates of the proposals
  double* gdelta;            // [M] Gaussian part of the energy change
  // line form in sweeps: moves decided again from estimates sample by sample
  double* gmargin;           // [M] how far gdelta can be from theirs, else null
  uint32_t* gunsure;         // count, then the moves within it ([1 + M]; 0 between phases)
  double* hpart;             // [M] their Heaviside part
  double* gpart;             // [M][tgp/16] their Gaussian parts by 16
};

hipError_t launch_init_offsets(const DevView& v, hipStream_t s);
hipError_t launch_count(const DevView& v, int mode, uint32_t kappa, uint32_t m, hipStream_t s);
hipError_t launch_delta(const DevView& v, int mode, uint32_t kappa, uint32_t m, hipStream_t s);
// a colour phase of the FP32 form with a phase kernel (K = 1, 2, 4)
bool staged_phases(const DevView& v);
hipError_t launch_phase(const DevView& v, uint32_t kappa, hipStream_t s);
// advance: also the sweep counter
hipError_t launch_commit(const DevView& v, uint32_t kappa, hipStream_t s, bool advance = false);
uint32_t commit_blocks(const DevView& v);
bool moves_wait(const DevView& v);
// d8 of the pixels whose offset the caller has replaced, from their counts
hipError_t launch_follow(const DevView& v, hipStream_t s);
hipError_t launch_follow_batch(const DevView* views, const uint32_t* pre, uint32_t nmem, uint32_t blocks, hipStream_t s);
// the waiting moves of all classes (v: a sweep's view) in one launch
hipError_t launch_commit_sweep(const DevView& v, hipStream_t s, bool advance);
uint32_t commit_sweep_blocks(const DevView& v);
hipError_t launch_commit_sweep_batch(const DevView* views, const uint32_t* pre, uint32_t nmem, uint32_t blocks,
                                     hipStream_t s);
hipError_t launch_errors(const DevView& v, hipStream_t s);
hipError_t launch_pack_errors(const DevView& v, uint32_t first, uint32_t n, float* out, hipStream_t s);
hipError_t launch_advance(const DevView& v, hipStream_t s);
hipError_t launch_recount_index(const DevView& v, hipStream_t s);
hipError_t launch_recount_advance_pair(const DevView& v, hipStream_t s);
hipError_t launch_points(const DevView& v, uint32_t pixel, uint32_t* out, hipStream_t s);
constexpr uint32_t ENERGY_ROWS = 64;   // rows of class sums that k_energy spreads its atomics over
hipError_t launch_energy(const DevView& v, unsigned long long* y, hipStream_t s);
// Taps of a blur on the device: BLUR_BLOCK - 1 readable floats past the last,
// runs of consecutive distances (first, count).
constexpr uint32_t BLUR_BLOCK = 16;
struct BlurTaps {
  const float* taps;
  const int2* runs;
  uint32_t nruns;
};
hipError_t launch_blur(const DevView& v, const float* field, uint32_t pitch, uint32_t valid, const BlurTaps& x,
                       const BlurTaps& y, float* tmp, double* partial, uint32_t* npartial, hipStream_t s);
uint32_t blur_partials(const DevView& v, uint32_t pitch);
bool gauss_lines_pay(const DevView& v, uint32_t m);
hipError_t launch_gauss_again(const DevView& v, uint32_t kappa, hipStream_t s);
hipError_t launch_gauss_lines(const DevView& v, bool all, uint32_t m, hipStream_t s);
hipError_t launch_gauss_est(const DevView& v, int mode, uint32_t m, hipStream_t s);
hipError_t launch_gauss_delta(const DevView& v, int mode, uint32_t kappa, uint32_t m, hipStream_t s);
hipError_t launch_gauss_commit(const DevView& v, uint32_t kappa, hipStream_t s);
hipError_t launch_gauss_errors(const DevView& v, hipStream_t s);
hipError_t launch_gauss_energy(const DevView& v, double* gsum, hipStream_t s);

// energy change and decision of a colour phase, one source per form
hipError_t launch_phase_wide(const DevView& v, uint32_t kappa, hipStream_t s);
hipError_t launch_phase_batch_wide(uint32_t radius, uint32_t k, bool sliced, const DevView* views, const uint32_t* pre,
                               uint32_t nmem, uint32_t blocks, uint32_t kappa, hipStream_t s);
uint32_t phase_blocks_wide(const DevView& v);
hipError_t launch_phase_narrow(const DevView& v, uint32_t kappa, hipStream_t s);
hipError_t launch_phase_batch_narrow(uint32_t radius, uint32_t k, bool sliced, const DevView* views, const uint32_t* pre,
                               uint32_t nmem, uint32_t blocks, uint32_t kappa, hipStream_t s);
uint32_t phase_blocks_narrow(const DevView& v);
hipError_t launch_phase_split(const DevView& v, uint32_t kappa, hipStream_t s);
hipError_t launch_phase_batch_split(uint32_t radius, uint32_t k, bool sliced, const DevView* views, const uint32_t* pre,
                               uint32_t nmem, uint32_t blocks, uint32_t kappa, hipStream_t s);
uint32_t phase_blocks_split(const DevView& v);
// workgroups of a phase launch: those of its class pixels, for each slice
uint32_t phase_blocks(const DevView& v);
// the integrand slices of v's phases where `blocks` workgroups have one slice
uint32_t phase_slices(const DevView& v, uint32_t blocks);
// decisions from the slices' class sums
hipError_t launch_phase_decide(const DevView& v, uint32_t kappa, hipStream_t s);
uint32_t decide_blocks(const DevView& v);
hipError_t launch_phase_decide_batch(uint32_t radius, const DevView* views, const uint32_t* pre, uint32_t nmem,
                                     uint32_t blocks, uint32_t kappa, hipStream_t s);
// words of 8 counts whose class sums fit int32 (wide form)
uint32_t phase_span_wide(uint32_t n);

// batched launches: member i of a group owns blocks pre[i] .. pre[i+1]-1
int count_kind(const DevView& v);
uint32_t count_blocks(const DevView& v);
hipError_t launch_count_batch(int kind, const DevView* views, const uint32_t* pre, uint32_t nmem,
                              uint32_t blocks, uint32_t kappa, hipStream_t s);
// sliced: a member has several integrand slices
hipError_t launch_phase_batch(uint32_t form, uint32_t radius, uint32_t k, bool sliced, const DevView* views, const uint32_t* pre,
                              uint32_t nmem, uint32_t blocks, uint32_t kappa, hipStream_t s);
hipError_t launch_commit_batch(const DevView* views, const uint32_t* pre, uint32_t nmem, uint32_t blocks,
                               uint32_t kappa, hipStream_t s);
hipError_t launch_advance_batch(const DevView* views, uint32_t nmem, hipStream_t s);

// BF16 precision form (mfma.hip): the field from counts / estimates, the
// colour phase's evaluation (Gram pass + decision + exact re-evaluation), the
// field's energy
bool bf16_supported_k(uint32_t k);
hipError_t launch_bf_field(const DevView& v, hipStream_t s);
// raises the LDS launch limit of the BF16 kernels of this radius and K (once per process)
hipError_t prepare_bf_kernels(uint32_t radius, uint32_t k);
hipError_t launch_delta_bf16(const DevView& v, uint32_t kappa, hipStream_t s);
hipError_t launch_energy_bf16(const DevView& v, double* ysum, hipStream_t s);
// decision from the summed class sums of a colour phase (clears them)
hipError_t launch_finish(const DevView& v, hipStream_t s);
// Gaussian rows' part of the energy change into gdelta, whatever the form
hipError_t launch_gauss_delta_exact(const DevView& v, uint32_t kappa, hipStream_t s);

// error spectrum (spectrum.hip): DFT of SPEC_CHUNK integrand rows along x
// into rows [H][W][chunk] (complex), then along y with |.|^2 summed over the
// chunk into power [H][W] (added to)
uint32_t spectrum_chunk();
// chunks of `rows` integrand rows that one launch takes
uint32_t spectrum_chunks(const DevView& v, uint32_t rows);
// entries of the scratch buffers of such a launch
struct SpectrumScratch {
  size_t rows, power;
};
SpectrumScratch spectrum_scratch(const DevView& v, uint32_t chunks);
// the twiddles along a side of n: the n values, or their matrix
bool spectrum_matrix(const DevView& v, uint32_t n, uint32_t rows);
size_t spectrum_matrix_size(uint32_t n);
hipError_t launch_twiddles(const float2* tw, uint32_t n, float2* mat, hipStream_t s);
struct SpectrumTwiddles {
  const float2* tw;
  bool matrix;
};
// integrands t0 ..; first: of a spectrum (sum starts with theirs)
hipError_t launch_spectrum_chunks(const DevView& v, const float* field, uint32_t pitch, uint32_t valid, uint32_t t0,
                                  uint32_t chunks, bool first, const SpectrumTwiddles& x, const SpectrumTwiddles& y,
                                  float2* rows, double* power, double* sum, hipStream_t s);

// device peak loops: kind 0 copy (buf -> buf2, size bytes), 1 dot2 chains,
// 2 BF16 MFMA accumulations (iters iterations each); blocks workgroups of 256
hipError_t peak_launch(int kind, void* buf, void* buf2, uint64_t size, uint32_t iters, uint32_t blocks,
                       hipStream_t s);

// allocation-free entry point: device address of the scratch array on
// `device` (located once per device), and tiled counts -> host row layout
hipError_t noalloc_scratch(int device, void** ptr);
hipError_t launch_untile_counts(const uint16_t* tiled, uint32_t rows, uint32_t first, uint32_t n, uint32_t t,
                                uint16_t* out, hipStream_t s);
hipError_t launch_untile_narrow(const int8_t* tiled, const uint32_t* bias8, uint32_t rows, uint32_t first, uint32_t n,
                                uint32_t t, uint16_t* out, hipStream_t s);

}  // namespace bnlat
