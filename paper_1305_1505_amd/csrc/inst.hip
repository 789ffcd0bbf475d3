// Instantiation of the kernels and their launchers for one grid size and precision.
// Compiled once per supported (N, precision) with -DPIN_INST_N=<N> -DPIN_INST_FP64=<0|1>.
#include "grf.hpp"
#include "kernels.hpp"
#include "launch.hpp"
#include "ops.hpp"

#ifndef PIN_INST_N
#error "PIN_INST_N must be defined"
#endif
#ifndef PIN_INST_FP64
#error "PIN_INST_FP64 must be defined"
#endif

namespace pin {
namespace {

constexpr int NN = PIN_INST_N;
using RR = std::conditional_t<PIN_INST_FP64 != 0, double, float>;
using VV = Cplx<RR>::type;
static_assert(size_ok(NN) && NN % 2 == 0, "grid size");

void prep(const void* dk, void* g0, double scale, hipStream_t s) {
  const size_t total = (size_t)NN * NN * (NN / 2);
  const int block = 256;
  const int grid = (int)((total + block - 1) / block);
  launch(k_prep<RR, NN>, dim3(grid), dim3(block), s, static_cast<const VV*>(dk),
         static_cast<VV*>(g0), (RR)scale);
}

void xpass(int mode, const void* dk, void* out, const void* wtab, const void* tw, double scale, int nb,
           hipStream_t s) {
  using S = Strided<RR, NN, +1>;
  if (mode == 0) {
    launch(k_xpass<RR, NN, 0>, dim3(S::GRID, nb, S::SPLIT ? 3 : 1), dim3(S::T), s, static_cast<const VV*>(dk),
           static_cast<VV*>(out), static_cast<const RR*>(wtab), static_cast<const VV*>(tw), (RR)scale);
  } else {
    launch(k_xpass<RR, NN, 1>, dim3(S::GRID, 1, S::SPLIT ? 2 : 1), dim3(S::T), s, static_cast<const VV*>(dk),
           static_cast<VV*>(out), static_cast<const RR*>(nullptr), static_cast<const VV*>(tw), (RR)scale);
  }
}

void xpass_fwdinv(bool hess, const void* in, void* out, const void* tw, double scale, hipStream_t s) {
  using S = Strided<RR, NN, +1>;
  if (hess) {
    launch(k_xpass_fwdinv<RR, NN, true>, dim3(S::GRID), dim3(S::T), s, static_cast<const VV*>(in),
           static_cast<VV*>(out), static_cast<const VV*>(tw), (RR)scale);
  } else {
    launch(k_xpass_fwdinv<RR, NN, false>, dim3(S::GRID), dim3(S::T), s, static_cast<const VV*>(in),
           static_cast<VV*>(out), static_cast<const VV*>(tw), (RR)scale);
  }
}

void xpass_lpt3(const void* in, void* out, const void* tw, double scale, hipStream_t s) {
  using S = Strided<RR, NN, +1>;
  launch(k_xpass_lpt3<RR, NN>, dim3(S::GRID), dim3(S::T), s, static_cast<const VV*>(in),
         static_cast<VV*>(out), static_cast<const VV*>(tw), (RR)scale);
}

template <int RECIPE> void ypass_packed(const void* in, void* out, void* out2, const void* tw, int nb, hipStream_t s) {
  using S = Strided<RR, NN, +1>;
  launch(k_ypass_packed<RR, NN, RECIPE>, dim3(S::GRID, nb, S::SPLIT ? YRecipe<RECIPE>::Q : 1), dim3(S::T), s,
         static_cast<const VV*>(in), static_cast<VV*>(out), static_cast<const VV*>(tw), static_cast<VV*>(out2));
}

void ypass(int recipe, const void* in, void* out, const void* tw, int nb, hipStream_t s) {
  if (recipe == 0) {
    ypass_packed<0>(in, out, nullptr, tw, nb, s);
  } else if (recipe == 1) {
    ypass_packed<1>(in, out, nullptr, tw, nb, s);
  } else if (recipe == 4) {
    ypass_packed<4>(in, out, nullptr, tw, nb, s);
  } else {
    using S = Strided<RR, NN, -1>;
    launch(k_ypass_fwd<RR, NN>, dim3(S::GRID), dim3(S::T), s, static_cast<const VV*>(in), static_cast<VV*>(out),
           static_cast<const VV*>(tw));
  }
}

// Hessian (3 packed slots to out) and v_max gradient (2 packed slots to gout) in one y pass.
void ypass_hess_grad(const void* in, void* out, void* gout, const void* tw, int nb, hipStream_t s) {
  ypass_packed<5>(in, out, gout, tw, nb, s);
}

template <bool VEL, bool WHOLE> void zcollapse_launch(const CollapseStep& c, const ZCollapseArgs& a, hipStream_t s) {
  using Z = ZCollapse<RR, NN, VEL, WHOLE>;
  if constexpr (BatchRule<RR, NN>::MANY) {
    if (c.nb > 1) {
      launch(k_zcollapse<RR, NN, VEL, WHOLE, true>, dim3(Z::GRID, c.groups), dim3(Z::T), s,
             static_cast<const VV*>(c.in), static_cast<const VV*>(c.tw), a);
      return;
    }
  }
  launch(k_zcollapse<RR, NN, VEL, WHOLE, false>, dim3(Z::GRID), dim3(Z::T), s,
         static_cast<const VV*>(c.in), static_cast<const VV*>(c.tw), a);
}

void zcollapse(const CollapseStep& c, hipStream_t s) {
  constexpr size_t vol = (size_t)NN * NN * NN;
  RR* Fg = static_cast<RR*>(c.groups > 1 ? c.part : c.F);
  uint8_t* rg = c.groups > 1 ? reinterpret_cast<uint8_t*>(Fg + (size_t)c.groups * vol) : c.ridx;
  ZCollapseArgs a{c.F, Fg, rg, c.r0, c.nb, c.fresh, CollapseConst{c.sphere_gain}, c.gin, c.vmax, c.vscale};
  if (c.gin != nullptr)
    c.whole ? zcollapse_launch<true, true>(c, a, s) : zcollapse_launch<true, false>(c, a, s);
  else
    c.whole ? zcollapse_launch<false, true>(c, a, s) : zcollapse_launch<false, false>(c, a, s);
  if (c.groups > 1) {
    const int block = 256;
    launch(k_merge<RR>, dim3((unsigned)((vol + block - 1) / block)), dim3(block), s, Fg, rg, c.groups,
           vol, static_cast<RR*>(c.F), c.ridx, c.whole, c.fresh);
  }
}

void zpass_store(int nc, const void* in, const void* tw, void* out, hipStream_t s) {
  ZArgs a{};
  a.out = out;
  a.nc = nc;
  if (nc == 6) {
    using Z = ZPass<RR, NN, 3, EPI_STORE>;
    launch(k_zpass<RR, NN, 3, EPI_STORE>, dim3(Z::GRID), dim3(Z::T), s,
           static_cast<const VV*>(in), static_cast<const VV*>(tw), a);
  } else {
    using Z = ZPass<RR, NN, 2, EPI_STORE>;
    launch(k_zpass<RR, NN, 2, EPI_STORE>, dim3(Z::GRID), dim3(Z::T), s,
           static_cast<const VV*>(in), static_cast<const VV*>(tw), a);
  }
}

void zpass_mu2(const void* in, const void* tw, void* out_slot, void* t6, hipStream_t s) {
  using Z = ZPass<RR, NN, 3, EPI_MU2>;
  ZArgs a{};
  a.out = out_slot;
  a.t6 = t6;
  launch(k_zpass<RR, NN, 3, EPI_MU2>, dim3(Z::GRID), dim3(Z::T), s,
         static_cast<const VV*>(in), static_cast<const VV*>(tw), a);
}

void zpass_lpt3(const void* in, const void* t1, const void* tw, void* out_slots, hipStream_t s) {
  using Z = ZPass<RR, NN, 3, EPI_LPT3>;
  ZArgs a{};
  a.out = out_slots;
  a.t6 = const_cast<void*>(t1);
  launch(k_zpass<RR, NN, 3, EPI_LPT3>, dim3(Z::GRID), dim3(Z::T), s,
         static_cast<const VV*>(in), static_cast<const VV*>(tw), a);
}

void grf(void* dk, uint64_t seed, const double* amp, hipStream_t s) {
  GrfArgs g{seed, amp};
  const size_t total = (size_t)NN * NN * (NN / 2 + 1);
  const int block = 256;
  const int grid = (int)((total + block - 1) / block);
  launch(k_grf<RR>, dim3(grid), dim3(block), s, static_cast<VV*>(dk), NN, g);
}

void reset(void* F, uint8_t* ridx, hipStream_t s) {
  const size_t total = (size_t)NN * NN * NN;
  const int block = 256;
  const int grid = (int)((total + block - 1) / block);
  launch(k_reset<RR>, dim3(grid), dim3(block), s, static_cast<RR*>(F), ridx, total);
}

void redshift(const void* F, size_t count, const GrowthTables* t, void* z, hipStream_t s) {
  if (count == 0) return;
  if (count <= kRedshiftFew) {
    launch(k_redshift_few<RR>, dim3((unsigned)((count + 255) / 256)), dim3(256), s, static_cast<const RR*>(F), count, t,
           static_cast<RR*>(z));
    return;
  }
  constexpr size_t span = (size_t)kRedshiftThreads * kRedshiftValues;
  const size_t need = (count + span - 1) / span, most = 512;   // two workgroups on each of 256 CUs
  launch(k_redshift<RR>, dim3((unsigned)(need < most ? need : most)), dim3(kRedshiftThreads), s,
         static_cast<const RR*>(F), count, t, static_cast<RR*>(z));
}

void zero(void* p, size_t count, hipStream_t s) {
  if (count == 0) return;
  const int block = 256;
  const int grid = (int)((count + block - 1) / block);
  launch(k_zero<RR>, dim3(grid), dim3(block), s, static_cast<RR*>(p), count);
}

void collapse_points(const void* t6, size_t count, void* F, double sphere_gain, hipStream_t s) {
  if (count == 0) return;
  CollapseConst cc{sphere_gain};
  const int block = 256;
  const int grid = (int)((count + block - 1) / block);
  launch(k_collapse_points<RR>, dim3(grid), dim3(block), s, static_cast<const RR*>(t6), count,
         static_cast<RR*>(F), cc);
}

}  // namespace

#define PIN_CAT2(a, b, c) a##b##_##c
#define PIN_CAT(a, b, c) PIN_CAT2(a, b, c)

const SizeOps* PIN_CAT(ops_, PIN_INST_FP64, PIN_INST_N)() {
  static const SizeOps ops = {
      NN, PIN_INST_FP64 != 0, prep, xpass, xpass_fwdinv, xpass_lpt3, ypass, ypass_hess_grad, zcollapse,
      ZCollapse<RR, NN, false, true>::GRID * ZCollapse<RR, NN, false, true>::WAVES, BatchRule<RR, NN>::RADII,
      BatchRule<RR, NN>::RADII_V, zpass_store, zpass_mu2, zpass_lpt3, grf, reset, redshift, zero, collapse_points,
      LaunchShape{Strided<RR, NN, +1>::GRID, Strided<RR, NN, +1>::T},
      LaunchShape{Strided<RR, NN, +1>::GRID, Strided<RR, NN, +1>::T},
      LaunchShape{ZCollapse<RR, NN, false, true>::GRID, ZCollapse<RR, NN, false, true>::T}};
  return &ops;
}

}  // namespace pin
