// Instantiates the row kernels for one grid, selected at compile time by
// -DGL1=<log2 n1> -DGL2=<log2 n2>.
#include "row_kernels.hpp"
#include "grids.hpp"

#include <type_traits>

#ifndef GL1
#error "GL1 / GL2 must be defined"
#endif

namespace tmk {

#define TM_CAT2(a, b, c) a##_##b##_##c
#define TM_CAT(a, b, c) TM_CAT2(a, b, c)

// FP64 residual: 8 values per thread (at 128 x 64: 1024 threads, 128 VGPRs, four
// waves per SIMD; 16 values per thread took 248 VGPRs and two waves)
using PLd = Plan<GL1, GL2, (GL1 + GL2 >= 3) ? 3 : GL1 + GL2>;

// Configurations 0 and 1: the mixed-axis plan where it is compiled (32 x 32 to
// 128 x 64; it has no digit order), else one axis per pass in either digit
// order. At 2286 x 8192 it runs the Lanczos step in 287 us against 384, the
// cyclic sweep in 251 against 372 and the gradient in 250 against 379; at
// 1500 x 4096 85 against 103, 73 against 99 and 78 against 105; at 512 x 1024
// 23 against 27, 22 against 27 and 25 against 27. With few rows it is the faster
// one as well or level (64 x 8192: cyclic sweep 36 us against 40, Lanczos step
// 40 and 40; 100 x 1024: 21 against 27, 22 against 27), so no row count decides.
constexpr bool kWide = wide_compiled(GL1, GL2);
template <int VAR>
using Default = std::conditional_t<kWide, WidePlan<kWide ? GL1 : 6, kWide ? GL2 : 6>, Plan<GL1, GL2, -1, VAR>>;

// Up to eight waves per CU (two per SIMD, 2048 on 256 CUs) the mixed-axis kernels need no
// more than two waves' registers, and take the form that loads a mask ahead. Lanczos step /
// gradient / training backward step, 4 masks, us: 128 x 64, 64 rows 38.9 / 37.9 / 30.5 -> 35.7
// / 34.6 / 25.7; 64 x 64, 400 rows 35.3 / 33.7 / 74.0 -> 32.1 / 32.3 / 46.1; 64 x 32, 900 rows
// 34.6 / 33.7 / 54.3 -> 31.8 / 31.7 / 46.5; 32 x 32, 512 rows 23.2 / 23.6 / 36.4 -> 22.0 / 22.3
// / 30.3. Adjoint, 6 masks: 32 x 32, 64 rows 21.1 -> 16.9, 64 x 32, 900 rows 31.6 -> 30.1; with
// larger workgroups only to half as many waves (64 x 64, 256 rows 27.0 -> 25.9, 500 rows 33.6
// -> 34.2). The L-BFGS line sums of 900 rows of 64 x 32, whose prologue has twice the loads in
// flight, 64 -> 55. Error reduction gains nothing steady (averaged, 64 x 32, 900 rows: 33.9 ->
// 35.7; cyclic level) and keeps the one form.
static int64_t few_waves(const RowArgs& a) { return 8 * (int64_t)a.cus; }

template <class PLg, typename IT>
static bool launch_few(int mode, const RowArgs& a, dim3 grid, dim3 block, hipStream_t s) {
  switch (mode) {
    case M_GRAD:
      if (a.sums || a.fout) row_kernel_few<PLg, M_GRAD, IT, true><<<grid, block, 0, s>>>(a);
      else row_kernel_few<PLg, M_GRAD, IT, false><<<grid, block, 0, s>>>(a);
      return true;
    case M_AGRAD:
      if (a.sums || a.fout) row_kernel_few<PLg, M_AGRAD, IT, true><<<grid, block, 0, s>>>(a);
      else row_kernel_few<PLg, M_AGRAD, IT, false><<<grid, block, 0, s>>>(a);
      return true;
    case M_ADJ:
      if (Launch<PLg>::WG > 128 && (int64_t)grid.x * (Launch<PLg>::WG / 64) > few_waves(a) / 2) return false;
      row_kernel_few<PLg, M_ADJ, IT><<<grid, block, 0, s>>>(a);
      return true;
    case M_LS: row_kernel_few<PLg, M_LS, IT><<<grid, block, 0, s>>>(a); return true;
    case M_ALS: row_kernel_few<PLg, M_ALS, IT><<<grid, block, 0, s>>>(a); return true;
    case M_FILT: row_kernel_few<PLg, M_FILT, IT><<<grid, block, 0, s>>>(a); return true;
    case M_SPEC: row_kernel_few<PLg, M_SPEC, IT><<<grid, block, 0, s>>>(a); return true;
    case M_LANCZOS: row_kernel_few<PLg, M_LANCZOS, IT><<<grid, block, 0, s>>>(a); return true;
    case M_LANCZOS_T: row_kernel_few<PLg, M_LANCZOS_T, IT><<<grid, block, 0, s>>>(a); return true;
    case M_WAPPLY: row_kernel_few<PLg, M_WAPPLY, IT><<<grid, block, 0, s>>>(a); return true;
    case M_WBACK: row_kernel_few<PLg, M_WBACK, IT><<<grid, block, 0, s>>>(a); return true;
    default: return false;
  }
}

// One-axis plan of 8192 points (64 x 128) with at most one row per CU: the second workgroup
// per CU, for which the kernels with one LDS copy save registers, does not come. Two copies
// (no barrier between the adjoint's masks) and all registers (the cyclic sweep's loads
// together) take, few / many rows' kernel: 256 rows, 6 masks, adjoint 45 / 48.6 us, ten sweeps
// 663 / 683; from the next row on the many rows' kernel wins (1000 rows, 4 masks: 134 / 99,
// 1725 / 1291).
template <class PLg, typename IT>
static bool launch_two(int mode, const RowArgs& a, dim3 grid, dim3 block, hipStream_t s) {
  switch (mode) {
    case M_ADJ: row_kernel_few<PLg, M_ADJ, IT><<<grid, block, 0, s>>>(a); return true;
    case M_ERC:
      if (a.sums) row_kernel_few<PLg, M_ERC, IT, true><<<grid, block, 0, s>>>(a);
      else row_kernel_few<PLg, M_ERC, IT, false><<<grid, block, 0, s>>>(a);
      return true;
    default: return false;
  }
}

template <class PLg, typename IT>
static int launch_t(int mode, const RowArgs& a, hipStream_t s) {
  using LC = Launch<PLg>;
  if (a.P <= 0) return 0;
  if (split_mode(mode) && (a.split < 1 || a.split > a.K)) return (int)hipErrorInvalidValue;
  dim3 grid((a.P + LC::RPW - 1) / LC::RPW * (split_mode(mode) ? a.split : 1)), block(LC::WG);
  if constexpr (PLg::WIDE) {
    if ((int64_t)grid.x * (LC::WG / 64) <= few_waves(a) && launch_few<PLg, IT>(mode, a, grid, block, s))
      return (int)hipGetLastError();
  } else if constexpr (PLg::T == 512) {
    if ((int)grid.x <= a.cus && launch_two<PLg, IT>(mode, a, grid, block, s)) return (int)hipGetLastError();
  }
  switch (mode) {
    case M_FWD_FIELD: row_kernel<PLg, M_FWD_FIELD, IT><<<grid, block, 0, s>>>(a); break;
    case M_FWD_INT: row_kernel<PLg, M_FWD_INT, IT><<<grid, block, 0, s>>>(a); break;
    case M_ADJ: row_kernel<PLg, M_ADJ, IT><<<grid, block, 0, s>>>(a); break;
    case M_ER:
      if (a.sums) row_kernel<PLg, M_ER, IT, true><<<grid, block, 0, s>>>(a);
      else row_kernel<PLg, M_ER, IT, false><<<grid, block, 0, s>>>(a);
      break;
    case M_ERC:
      if (a.sums) row_kernel<PLg, M_ERC, IT, true><<<grid, block, 0, s>>>(a);
      else row_kernel<PLg, M_ERC, IT, false><<<grid, block, 0, s>>>(a);
      break;
    case M_GRAD:
      if (a.sums || a.fout) row_kernel<PLg, M_GRAD, IT, true><<<grid, block, 0, s>>>(a);
      else row_kernel<PLg, M_GRAD, IT, false><<<grid, block, 0, s>>>(a);
      break;
    case M_SPEC: row_kernel<PLg, M_SPEC, IT><<<grid, block, 0, s>>>(a); break;
    case M_LANCZOS: row_kernel<PLg, M_LANCZOS, IT><<<grid, block, 0, s>>>(a); break;
    case M_LANCZOS_T: row_kernel<PLg, M_LANCZOS_T, IT><<<grid, block, 0, s>>>(a); break;
    case M_WAPPLY: row_kernel<PLg, M_WAPPLY, IT><<<grid, block, 0, s>>>(a); break;
    case M_WBACK: row_kernel<PLg, M_WBACK, IT><<<grid, block, 0, s>>>(a); break;
    case M_LS: row_kernel<PLg, M_LS, IT><<<grid, block, 0, s>>>(a); break;
    case M_AGRAD:
      if (a.sums || a.fout) row_kernel<PLg, M_AGRAD, IT, true><<<grid, block, 0, s>>>(a);
      else row_kernel<PLg, M_AGRAD, IT, false><<<grid, block, 0, s>>>(a);
      break;
    case M_ALS: row_kernel<PLg, M_ALS, IT><<<grid, block, 0, s>>>(a); break;
    case M_FILT: row_kernel<PLg, M_FILT, IT><<<grid, block, 0, s>>>(a); break;
    case M_BACKPROP: row_kernel<PLg, M_BACKPROP, IT><<<grid, block, 0, s>>>(a); break;
    case M_RES64: {
      using LD = Launch<PLd>;
      size_t lds = (size_t)LD::RPW * PLd::LDS_ROW * sizeof(cx<double>) + (LD::WG / 64 + 1) * sizeof(double);
      auto fn = res64_kernel<PLd, IT>;
      hipError_t e = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return (int)e;
      fn<<<dim3((a.P + LD::RPW - 1) / LD::RPW), dim3(LD::WG), lds, s>>>(a);
      break;
    }
    default: return (int)hipErrorInvalidValue;
  }
  return (int)hipGetLastError();
}

// Digit-order variant 1 differs from variant 0 only when an axis splits
// into digits of unequal size.
constexpr bool uneven(int b) { return ndigits(b) >= 2 && b % ndigits(b) != 0; }
constexpr bool kHasVar = uneven(GL1) || uneven(GL2);

int TM_CAT(row_launch, GL1, GL2)(int mode, int ibf16, const RowArgs& a, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  using P0 = Default<0>;
  return ibf16 ? launch_t<P0, uint16_t>(mode, a, s) : launch_t<P0, float>(mode, a, s);
}

int TM_CAT(row_launchv, GL1, GL2)(int mode, int ibf16, const RowArgs& a, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  if constexpr (kHasVar && !kWide) {
    using P1 = Plan<GL1, GL2, -1, 1>;
    return ibf16 ? launch_t<P1, uint16_t>(mode, a, s) : launch_t<P1, float>(mode, a, s);
  } else {
    return TM_CAT(row_launch, GL1, GL2)(mode, ibf16, a, stream);
  }
}

// Wider configurations for the autotuner, cfg bits: 1 the digit order
// (variant 1), 2 eight values per thread instead of sixteen, 4 twice the rows
// per workgroup. They apply to the iteration and start kernels the batch also
// runs (error reduction, averaged and cyclic; heavy-ball spectral and Lanczos
// steps) and to the L-BFGS solvers' gradient kernels and the amplitude cost's
// line search (the intensity cost's line search, which holds both transforms
// of a mask at once, spills at eight values per thread and keeps the default
// plan); every other mode runs the default plan of the same digit order.
// Compiled for the grids of the benchmark workloads.
constexpr bool kExt = (GL1 == 5 && GL2 == 5) || (GL1 == 6 && GL2 == 5) || (GL1 == 6 && GL2 == 6) ||
                      (GL1 == 7 && GL2 == 6);

template <int CFG>
struct XCfg {
  static constexpr int LE = (CFG & 2) ? 3 : -1;
  using PX = Plan<GL1, GL2, LE, (CFG & 1) && kHasVar ? 1 : 0>;
  static constexpr int WG0 = Launch<PX>::WG;
  static constexpr int WG = (CFG & 4) ? 2 * WG0 : WG0;
  // twice the rows only up to 512 threads (two waves per SIMD keep a 256-register budget)
  static constexpr bool ok = kExt && (CFG & 6) != 0 && (GL1 + GL2 >= 3) && ((CFG & 4) ? WG <= 512 : WG <= 1024);
};

template <class PX, int WG, typename IT>
static int launch_x(int mode, const RowArgs& a, hipStream_t s) {
  constexpr int RPW = WG / PX::T;
  static_assert(RPW >= 1 && RPW * PX::T == WG, "whole rows per workgroup");
  if (a.P <= 0) return 0;
  dim3 grid((a.P + RPW - 1) / RPW), block(WG);
  switch (mode) {
    case M_LANCZOS: row_kernel_w<PX, M_LANCZOS, IT, true, WG><<<grid, block, 0, s>>>(a); break;
    case M_LANCZOS_T: row_kernel_w<PX, M_LANCZOS_T, IT, true, WG><<<grid, block, 0, s>>>(a); break;
    case M_SPEC: row_kernel_w<PX, M_SPEC, IT, true, WG><<<grid, block, 0, s>>>(a); break;
    case M_ER:
      if (a.sums) row_kernel_w<PX, M_ER, IT, true, WG><<<grid, block, 0, s>>>(a);
      else row_kernel_w<PX, M_ER, IT, false, WG><<<grid, block, 0, s>>>(a);
      break;
    case M_ERC:
      if (a.sums) row_kernel_w<PX, M_ERC, IT, true, WG><<<grid, block, 0, s>>>(a);
      else row_kernel_w<PX, M_ERC, IT, false, WG><<<grid, block, 0, s>>>(a);
      break;
    case M_GRAD:
      if (a.sums || a.fout) row_kernel_w<PX, M_GRAD, IT, true, WG><<<grid, block, 0, s>>>(a);
      else row_kernel_w<PX, M_GRAD, IT, false, WG><<<grid, block, 0, s>>>(a);
      break;
    case M_AGRAD:
      if (a.sums || a.fout) row_kernel_w<PX, M_AGRAD, IT, true, WG><<<grid, block, 0, s>>>(a);
      else row_kernel_w<PX, M_AGRAD, IT, false, WG><<<grid, block, 0, s>>>(a);
      break;
    case M_ALS: row_kernel_w<PX, M_ALS, IT, true, WG><<<grid, block, 0, s>>>(a); break;
    default: return (int)hipErrorInvalidValue;
  }
  return (int)hipGetLastError();
}

template <int CFG>
static int launch_cfg(int mode, int ibf16, const RowArgs& a, void* stream) {
  using X = XCfg<CFG>;
  if constexpr (!X::ok) {
    return (int)hipErrorInvalidValue;
  } else {
    hipStream_t s = (hipStream_t)stream;
    if (mode == M_LANCZOS || mode == M_ERC || mode == M_ER || mode == M_SPEC || mode == M_GRAD || mode == M_AGRAD ||
        mode == M_ALS)
      return ibf16 ? launch_x<typename X::PX, X::WG, uint16_t>(mode, a, s)
                   : launch_x<typename X::PX, X::WG, float>(mode, a, s);
    if (mode == M_LANCZOS_T && !ibf16) return launch_x<typename X::PX, X::WG, float>(mode, a, s);
    return (CFG & 1) ? TM_CAT(row_launchv, GL1, GL2)(mode, ibf16, a, stream)
                     : TM_CAT(row_launch, GL1, GL2)(mode, ibf16, a, stream);
  }
}

#define TM_CFG_FN(k)                                                                      \
  int TM_CAT(row_launchc##k, GL1, GL2)(int mode, int ibf16, const RowArgs& a, void* s) { \
    return launch_cfg<k>(mode, ibf16, a, s);                                             \
  }
TM_CFG_FN(2)
TM_CFG_FN(3)
TM_CFG_FN(4)
TM_CFG_FN(5)
TM_CFG_FN(6)
TM_CFG_FN(7)

// bit k set: configuration k is compiled for this grid
int TM_CAT(row_cfgmask, GL1, GL2)() {
  return 3 | (XCfg<2>::ok << 2) | (XCfg<3>::ok << 3) | (XCfg<4>::ok << 4) | (XCfg<5>::ok << 5) |
         (XCfg<6>::ok << 6) | (XCfg<7>::ok << 7);
}

// threads per workgroup, rows per workgroup, values per thread of configuration cfg
void TM_CAT(row_cfgshape, GL1, GL2)(int cfg, int* wg, int* rpw, int* ept) {
  *wg = *rpw = *ept = 0;
  auto put = [&](int w, int t, int e) { *wg = w; *rpw = w / t; *ept = e; };
  switch (cfg) {
    case 0: case 1: put(Launch<Plan<GL1, GL2>>::WG, Plan<GL1, GL2>::T, Plan<GL1, GL2>::E); break;
    case 2: if (XCfg<2>::ok) put(XCfg<2>::WG, XCfg<2>::PX::T, XCfg<2>::PX::E); break;
    case 3: if (XCfg<3>::ok) put(XCfg<3>::WG, XCfg<3>::PX::T, XCfg<3>::PX::E); break;
    case 4: if (XCfg<4>::ok) put(XCfg<4>::WG, XCfg<4>::PX::T, XCfg<4>::PX::E); break;
    case 5: if (XCfg<5>::ok) put(XCfg<5>::WG, XCfg<5>::PX::T, XCfg<5>::PX::E); break;
    case 6: if (XCfg<6>::ok) put(XCfg<6>::WG, XCfg<6>::PX::T, XCfg<6>::PX::E); break;
    case 7: if (XCfg<7>::ok) put(XCfg<7>::WG, XCfg<7>::PX::T, XCfg<7>::PX::E); break;
    default: break;
  }
}

// The lowest configuration whose kernels cfg runs (-1: not compiled), and their shape.
int TM_CAT(row_cfgkernel, GL1, GL2)(int cfg, int* wg, int* rpw, int* ept) {
  TM_CAT(row_cfgshape, GL1, GL2)(cfg, wg, rpw, ept);
  if (*wg == 0) return -1;
  if (cfg < 2) {
    *wg = Launch<Default<0>>::WG;  // the same in both digit orders
    *rpw = Launch<Default<0>>::RPW;
    *ept = Default<0>::E;
  }
  return (cfg & 1) && (!kHasVar || (cfg < 2 && kWide)) ? cfg - 1 : cfg;
}

void TM_CAT(row_shape, GL1, GL2)(int* wg, int* rpw) {
  *wg = Launch<Default<0>>::WG;
  *rpw = Launch<Default<0>>::RPW;
}

}  // namespace tmk
