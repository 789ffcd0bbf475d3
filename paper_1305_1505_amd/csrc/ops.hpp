// Host-side table of the kernel launchers for one (precision, N).  Each supported pair is
// instantiated in its own translation unit (inst.hip compiled with PIN_INST_N / PIN_INST_FP64).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "host_math.hpp"

namespace pin {

struct LaunchShape {
  int grid;
  int block;
};

// One batch of the collapse z pass.
struct CollapseStep {
  const void* in;     // 3 packed slots per radius
  const void* gin;    // 2 packed gradient slots per radius, or null (no v_max)
  const void* tw;
  void* F;
  uint8_t* ridx;
  void* vmax;
  void* part;         // groups > 1: groups * N^3 reals and as many bytes of scratch
  int r0, nb;         // first radius index, radii
  int groups;         // workgroups along the radii (1 with v_max)
  bool whole;         // part of a call over all radii, taken from the last to the first
  bool fresh;         // no state before this batch
  double sphere_gain, vscale;
};

// Growing-mode tables of the collapse redshift (host_math.hpp: GrowthTable).
struct GrowthArgs {
  const double* d;
  const double* dd;
  int m;
  double y0, h, a_per_D, lambda_over_m;
  const int32_t* guide;   // last node with d <= 2^(l0 + b / inv), per bucket b < k
  int k;
  float l0, inv;
  int f_base, f_count, e_base, e_count;
  double f_inf, f_none;
};
// All of it on the device: a call recorded in a graph reads the tables and the numbers that belong to
// them as pin_plan_set_growth last left them.
struct GrowthTables {
  GrowthArgs args;
  double poly[kMaxBuckets * kBucketStride];   // kBucketStride values per bucket: f_count of F, then e_count of e
  double d[kGrowthNodes], dd[kGrowthNodes];
  int32_t guide[kGrowthGuide];
};

struct SizeOps {
  int n;
  bool fp64;
  // radius-independent Hessian input g0 = M dk scale / f^2 into one aligned slot
  void (*prep)(const void* dk, void* g0, double scale, hipStream_t s);
  // x pass.  mode 0: Hessian from g0 (3 outputs per radius, nb radii with consecutive window rows
  // from wtab); mode 1: gradient from the user half spectrum (2 outputs).  out = first workspace
  // slot of the outputs.
  void (*xpass)(int mode, const void* dk, void* out, const void* wtab, const void* tw, double scale, int nb,
                hipStream_t s);
  // fused forward-x / inverse-x of a second-order source: one input slot -> two output slots
  // (gradient, 2LPT) or three (hess: the Hessian x-pass outputs)
  void (*xpass_fwdinv)(bool hess, const void* in, void* out, const void* tw, double scale, hipStream_t s);
  // fused forward-x / inverse-x of the third-order displacement: four source slots -> three
  void (*xpass_lpt3)(const void* in, void* out, const void* tw, double scale, hipStream_t s);
  // y pass: recipe 0 Hessian (3 half slots -> 3 packed slots), 1 gradient (2 half -> 2 packed),
  // 2 forward (1 half -> 1 half, nb = 1), 4 three finished components (3 half -> 2 packed); nb radii,
  // the slots of one behind the other's
  void (*ypass)(int recipe, const void* in, void* out, const void* tw, int nb, hipStream_t s);
  // Hessian y pass that also writes the v_max gradient (2 packed slots per radius) to gout
  void (*ypass_hess_grad)(const void* in, void* out, void* gout, const void* tw, int nb, hipStream_t s);
  // z pass (packed slots in) with the collapse epilogue over a batch of radii, and v_max if gin is
  // not null; with several groups, `part` takes each group's result and a second launch merges them
  void (*zcollapse)(const CollapseStep& c, hipStream_t s);
  // waves of one group of that pass; most radii one launch of the collapse passes takes, without
  // and with v_max
  int zwaves, batch, batch_v;
  // z pass storing nc = 6 (Hessian) or 3 (gradient) real components to out[nc][N^3]
  void (*zpass_store)(int nc, const void* in, const void* tw, void* out, hipStream_t s);
  // z pass computing the 2LPT source and its forward transform along z into one slot; the six
  // tensor components are also stored to t6[6][N^3] when t6 is not null
  void (*zpass_mu2)(const void* in, const void* tw, void* out_slot, void* t6, hipStream_t s);
  // z pass of the second-order tensor with the third-order source epilogue: reads T1 [6][N^3],
  // writes the z-forward transforms of (sl, cx, cy, cz) to four half slots
  void (*zpass_lpt3)(const void* in, const void* t1, const void* tw, void* out_slots, hipStream_t s);
  // the field of `seed`, mode amplitudes from the plan's table (mode_amplitudes)
  void (*grf)(void* dk, uint64_t seed, const double* amp, hipStream_t s);
  void (*reset)(void* F, uint8_t* ridx, hipStream_t s);
  // collapse redshift of count F values (*t on the device, see k_redshift)
  void (*redshift)(const void* F, size_t count, const GrowthTables* t, void* z, hipStream_t s);
  // count reals of the plan's precision set to zero
  void (*zero)(void* p, size_t count, hipStream_t s);
  // per-point collapse model on [6][count] tensors
  void (*collapse_points)(const void* t6, size_t count, void* F, double sphere_gain, hipStream_t s);
  // launch shapes, for reports
  LaunchShape shape_x, shape_y, shape_z;
};

const SizeOps* find_ops(int n, bool fp64);

}  // namespace pin
