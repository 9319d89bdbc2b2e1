// Ensemble stage kernels: many meshes of different size and order in one
// launch per stage (or one per order); the stage itself is in dgsw_stage.hpp.
#include "dgsw_stage.hpp"
#include "dgsw_stage_m4.hpp"

namespace dgsw {

// ------------------------------------------------------------------ ensemble
// What a line stage takes in the kernel over all orders (kFused), the persistent
// kernel of one order and the flat one (kFlat; kFlatLarge: of an ensemble whose
// states, read and written, exceed the Infinity Cache).  An item is short and comes
// with loads of its own, so strips and freely moved table loads pay less often than
// in a mesh, strips at r = 2 and 5 only where memory is the limit.  Microseconds a
// stage of 32 members 33x17 .. 180x90 and one of 360x180, FP32:
//   strips / rows           r = 1        2            4            5            6
//     flat              14.2 / 14.6  25.8 / 24.7  62.7 / 72.0  95.1 / 93.9  138.8 / 147.1
//     persistent        14.3 / 14.3  28.9 / 27.3  84.1 / 82.4   122 / 113    164 / 154
//   (8 members, r = 4 persistent with two wavefronts 20.0 / 19.8, r = 1 6.2 / 5.8)
//   flat, members 90x45 .. 360x180, by the packed state: r = 2 82 MB 68.0 / 65.2,
//     109 MB 90.4 / 96.7, 164 MB 139 / 157; r = 5 52 MB 57.0 / 55.7, 105 MB 105.5 /
//     106.7, 210 MB 221 / 226, 630 MB 580 / 611
//   tables moved freely / in order: r = 5 rows 93.9 / 92.4, r = 7 flat 187 / 179,
//     persistent 186 / 193
// In the fused kernel both cost a wavefront per SIMD and a hundred spilled scalars
// (64 members 1.75 -> 2.4 ms a step).
enum { kFused, kPersistent, kFlat, kFlatLarge };
template <typename T, int NP, int FORM>
constexpr bool ens_strips = sizeof(T) == 4 && ((NP == 5 && FORM != kFused) || ((NP == 2 || NP == 7) && FORM >= kFlat) ||
                                               ((NP == 3 || NP == 6) && FORM == kFlatLarge));
template <typename T, int NP, int FORM>
constexpr bool ens_moved = sizeof(T) == 4 && FORM != kFused && (NP != 6 || FORM == kFlatLarge) && !(NP == 8 && FORM == kFlat);
// the orders whose flat kernel has the two forms
template <typename T, int NP, int LAY>
constexpr bool ens_two_flat = LAY == 0 && ens_strips<T, NP, kFlat> != ens_strips<T, NP, kFlatLarge>;
// Wavefronts a SIMD: r = 6 FP32 in strips needs a few registers more than three
// allow (148.4 -> 138.8 us; the persistent kernel would spill, 164 -> 221; with four
// wavefronts a workgroup the LDS allows two).  The
// matrix-core items hold 113 .. 122 registers and 22 accumulation registers, so
// three; held to four, flat items take 54.7 us for 55.2 and persistent ones spill
// (81 for 73).
template <typename T, int NP, int LAY, int WPB>
constexpr int ens_flat_waves = sizeof(T) == 4 && NP == 7 && LAY == 0 && WPB < 4 ? 3 : 1;
// LDS of one wavefront for any order up to NPMAX (the fused kernel)
template <typename T, int NPMAX>
struct LdsMax {
  using S_ = Shape<T, NPMAX>;
  static constexpr int tab = S_::cmax(S_::TB, LdsMax<T, NPMAX - 1>::tab);
  // (a wavefront's slice on 16 bytes: wide accesses at other addresses made this
  // kernel 5 .. 12 % slower with several wavefronts a workgroup)
  static constexpr int sh = S_::cmax((S_::wave(false) + 3) / 4 * 4, LdsMax<T, NPMAX - 1>::sh);
};
template <typename T>
struct LdsMax<T, 0> {
  static constexpr int tab = 0, sh = 0;
};

template <typename T, int NP, int CM, int FORM>
__device__ __forceinline__ void ens_case(const EnsItem &m, const unsigned char *__restrict__ tabs, const T *q,
                                         const T *q0, T *out, int combine, T c0, T ce, int lane, T *tab, T *sh) {
  StageArgs<T, NP> A;
  A.q = q + m.off;
  A.q0 = q0 ? q0 + m.off : nullptr;
  A.out = out + m.off;
  A.forcing = nullptr;
  A.qa = A.qb = nullptr;
  A.ca = A.cb = T(0);
  A.gt = reinterpret_cast<const GlobTab<T, NP> *>(tabs + m.glob);
  A.rows = reinterpret_cast<const RowTab<T, NP> *>(tabs + m.rows);
  A.n_lon = m.n_lon;
  A.n_lat = m.n_lat;
  A.alpha_global = m.alpha_global;
  A.periodic_y = 0;
  A.combine = combine;
  A.c0 = c0;
  A.c1 = T(0);
  A.ce = ce;
  A.dt = T(m.dt);
  stage_wave<T, NP, CM, ens_strips<T, NP, FORM>, ens_moved<T, NP, FORM>>(A, m.j, m.seg, lane, tab, sh);
}

// One launch per Runge-Kutta stage for a whole ensemble of meshes of different
// size and order, packed back to back in q / q0 / out.  Work unit: one
// wavefront of one member (items[k] = {member, wave index}).  Workgroup b
// (renumbered so each XCD gets a contiguous range) works through the
// contiguous item range [bounds[b], bounds[b+1]), balanced by cost on the host;
// its WPB wavefronts take every WPB-th item.  The order of each member is a
// wave-uniform switch.
template <typename T, int NPMAX, int WPB, int CM>
__global__ __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 && NPMAX <= 5 && WPB == 4 ? 3 : 1)))   // one register over otherwise
__launch_bounds__(64 * WPB) void k_ens_stage(const T *__restrict__ q, const T *q0, T *out,
                                                        const unsigned char *__restrict__ tabs,
                                                        const EnsItem *__restrict__ items,
                                                        const int *__restrict__ bounds, int combine,
                                                        T c0, T ce) {
  __shared__ T tab_all[WPB][LdsMax<T, NPMAX>::tab];
  __shared__ __attribute__((aligned(16))) T sh_all[WPB][LdsMax<T, NPMAX>::sh];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  T *tab = tab_all[wv], *sh = sh_all[wv];
  const int part = xcd_block(blockIdx.x, gridDim.x);
  const int end = bounds[part + 1];
  for (int it = bounds[part] + wv; it < end; it += WPB) {
    const EnsItem m = items[it];
    switch (m.np) {
      case 1: ens_case<T, 1, CM, kFused>(m, tabs, q, q0, out, combine, c0, ce, lane, tab, sh); break;
      case 2: ens_case<T, 2, CM, kFused>(m, tabs, q, q0, out, combine, c0, ce, lane, tab, sh); break;
      case 3: ens_case<T, 3, CM, kFused>(m, tabs, q, q0, out, combine, c0, ce, lane, tab, sh); break;
      case 4: ens_case<T, 4, CM, kFused>(m, tabs, q, q0, out, combine, c0, ce, lane, tab, sh); break;
      case 5: ens_case<T, 5, CM, kFused>(m, tabs, q, q0, out, combine, c0, ce, lane, tab, sh); break;
      default:
        if constexpr (NPMAX > 5) {
          switch (m.np) {
            case 6: ens_case<T, (NPMAX > 5 ? 6 : 1), CM, kFused>(m, tabs, q, q0, out, combine, c0, ce, lane, tab, sh); break;
            case 7: ens_case<T, (NPMAX > 6 ? 7 : 1), CM, kFused>(m, tabs, q, q0, out, combine, c0, ce, lane, tab, sh); break;
            case 8: ens_case<T, (NPMAX > 7 ? 8 : 1), CM, kFused>(m, tabs, q, q0, out, combine, c0, ce, lane, tab, sh); break;
            default: break;
          }
        }
        break;
    }
  }
}

// The same for the half layout (2 NP lanes per element); items give their
// element range.
template <typename T, int NP>
__device__ __forceinline__ StageArgs<T, NP> ens_args(const EnsItem &m, const unsigned char *__restrict__ tabs,
                                                     const T *q, const T *q0, T *out, int combine, T c0, T ce) {
  StageArgs<T, NP> A;
  A.q = q + m.off;
  A.q0 = q0 ? q0 + m.off : nullptr;
  A.out = out + m.off;
  A.forcing = nullptr;
  A.qa = A.qb = nullptr;
  A.ca = A.cb = T(0);
  A.gt = reinterpret_cast<const GlobTab<T, NP> *>(tabs + m.glob);
  A.rows = reinterpret_cast<const RowTab<T, NP> *>(tabs + m.rows);
  A.n_lon = m.n_lon;
  A.n_lat = m.n_lat;
  A.alpha_global = m.alpha_global;
  A.periodic_y = 0;
  A.combine = combine;
  A.c0 = c0;
  A.c1 = T(0);
  A.ce = ce;
  A.dt = T(m.dt);
  A.levels = 1;
  A.lstride = 0;
  return A;
}

// LDS of one wavefront per layout: the line and half variants, on 16 bytes
template <typename T, int NP, int LAY, int FORM>
struct EnsLds {
  static constexpr bool G4 = M4<T, NP> && LAY == 1;
  static constexpr int TB = G4 ? 2 : (LAY == 0 ? Shape<T, NP>::TB : ShapeH2<T, NP>::TB);
  static constexpr int USED = G4 ? kM4Lds
                                 : (LAY == 0 ? Shape<T, NP>::wave(ens_strips<T, NP, FORM>)
                                             : ShapeH2<T, NP>::SLOTS * ShapeH2<T, NP>::SH);
  static constexpr int SH = (USED + 3) / 4 * 4;
};

template <typename T, int NP, int LAY, int CM, int FORM>
__device__ __forceinline__ void ens_item(const EnsItem &m, const unsigned char *__restrict__ tabs, const T *q,
                                         const T *q0, T *out, int combine, T c0, T ce, int lane, T *tab, T *sh) {
  if constexpr (LAY == 0) {
    ens_case<T, NP, CM, FORM>(m, tabs, q, q0, out, combine, c0, ce, lane, tab, sh);
  } else if constexpr (M4<T, NP>) {
    const StageArgs<T, NP> A = ens_args<T, NP>(m, tabs, q, q0, out, combine, c0, ce);
    m4_run<CM, false>(
        A, (m.e_end - m.seg + kM4Elems - 1) / kM4Elems,
        [&](int k) {
          const int e0 = m.seg + kM4Elems * k;
          return M4Group{e0, m.e_end, k == 0 ? m.j : (int)((unsigned)e0 / (unsigned)m.n_lon), 0};
        },
        lane, (lds_double *)sh);
    m4_have_read();   // before the wavefront's next item arrives
  } else {
    stage_wave_h2<T, NP, CM, true>(ens_args<T, NP>(m, tabs, q, q0, out, combine, c0, ce), m.j, m.seg, m.e_end, lane,
                                   tab, sh);
  }
}

// Ensemble stage restricted to the members of one order and layout (the work
// list is sorted by both; bounds cover this group's items): the kernel is
// compiled for that order and layout alone, so it keeps their register
// budget and occupancy.
template <typename T, int NP, int LAY, int WPB, int CM>
__global__ __launch_bounds__(64 * WPB) void k_ens_stage_np(const T *__restrict__ q, const T *q0, T *out,
                                                           const unsigned char *__restrict__ tabs,
                                                           const EnsItem *__restrict__ items,
                                                           const int *__restrict__ bounds, int combine,
                                                           T c0, T ce) {
  __shared__ T tab_all[WPB][EnsLds<T, NP, LAY, kPersistent>::TB];
  __shared__ __attribute__((aligned(16))) T sh_all[WPB][EnsLds<T, NP, LAY, kPersistent>::SH];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int part = xcd_block(blockIdx.x, gridDim.x);
  const int end = bounds[part + 1];
  for (int it = bounds[part] + wv; it < end; it += WPB) {
    const EnsItem m = items[it];
    ens_item<T, NP, LAY, CM, kPersistent>(m, tabs, q, q0, out, combine, c0, ce, lane, tab_all[wv], sh_all[wv]);
  }
}

// Flat form: workgroup b takes items begin + b*WPB + wv, one item per
// wavefront, so the hardware schedules the ensemble like an ordinary grid
// (no loop: same register budget as the single-mesh kernel).
template <typename T, int NP, int LAY, int WPB, int CM, int FORM>
__global__ __attribute__((amdgpu_waves_per_eu(ens_flat_waves<T, NP, LAY, WPB>)))
__launch_bounds__(64 * WPB) void k_ens_stage_flat(const T *__restrict__ q, const T *q0, T *out,
                                                             const unsigned char *__restrict__ tabs,
                                                             const EnsItem *__restrict__ items,
                                                             int begin, int end, int combine, T c0, T ce) {
  __shared__ T tab_all[WPB][EnsLds<T, NP, LAY, FORM>::TB];
  __shared__ __attribute__((aligned(16))) T sh_all[WPB][EnsLds<T, NP, LAY, FORM>::SH];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int it = begin + xcd_block(blockIdx.x, gridDim.x) * WPB + wv;
  if (it >= end) return;
  const EnsItem m = items[it];
  ens_item<T, NP, LAY, CM, FORM>(m, tabs, q, q0, out, combine, c0, ce, lane, tab_all[wv], sh_all[wv]);
}

// the combination mode is a template parameter of the ensemble kernels too:
// 0 (right-hand side) or 1 (Shu-Osher stage)
template <typename T, int NP, int LAY, int WPB, int FORM>
static hipError_t launch_ens_flat_f(const EnsLaunch &a, hipStream_t s) {
  const int n = a.end - a.begin;
  const dim3 grid((n + WPB - 1) / WPB), block(64 * WPB);
  if (a.combine)
    hipLaunchKernelGGL((k_ens_stage_flat<T, NP, LAY, WPB, 1, FORM>), grid, block, 0, s, static_cast<const T *>(a.q),
                       static_cast<const T *>(a.q0), static_cast<T *>(a.out),
                       static_cast<const unsigned char *>(a.tabs), a.items, a.begin, a.end, 1, T(a.c0),
                       T(a.c0 + a.c1 - 1.0));
  else
    hipLaunchKernelGGL((k_ens_stage_flat<T, NP, LAY, WPB, 0, FORM>), grid, block, 0, s, static_cast<const T *>(a.q),
                       static_cast<const T *>(a.q0), static_cast<T *>(a.out),
                       static_cast<const unsigned char *>(a.tabs), a.items, a.begin, a.end, 0, T(a.c0),
                       T(a.c0 + a.c1 - 1.0));
  return hipGetLastError();
}

template <typename T, int NP, int LAY, int WPB>
static hipError_t launch_ens_flat_t(const EnsLaunch &a, hipStream_t s) {
  if constexpr (ens_two_flat<T, NP, LAY>)
    if (a.large) return launch_ens_flat_f<T, NP, LAY, WPB, kFlatLarge>(a, s);
  return launch_ens_flat_f<T, NP, LAY, WPB, kFlat>(a, s);
}

template <typename T, int NP, int LAY, int WPB>
static hipError_t launch_ens_np_t(const EnsLaunch &a, hipStream_t s) {
  if (a.combine)
    hipLaunchKernelGGL((k_ens_stage_np<T, NP, LAY, WPB, 1>), dim3(a.parts), dim3(64 * WPB), 0, s,
                       static_cast<const T *>(a.q), static_cast<const T *>(a.q0), static_cast<T *>(a.out),
                       static_cast<const unsigned char *>(a.tabs), a.items,
                       a.bounds, 1, T(a.c0), T(a.c0 + a.c1 - 1.0));
  else
    hipLaunchKernelGGL((k_ens_stage_np<T, NP, LAY, WPB, 0>), dim3(a.parts), dim3(64 * WPB), 0, s,
                       static_cast<const T *>(a.q), static_cast<const T *>(a.q0), static_cast<T *>(a.out),
                       static_cast<const unsigned char *>(a.tabs), a.items,
                       a.bounds, 0, T(a.c0), T(a.c0 + a.c1 - 1.0));
  return hipGetLastError();
}

template <typename T, int NP, int LAY>
static hipError_t launch_ens_np_l(int wpb, const EnsLaunch &a, hipStream_t s) {
  if (a.flat) {
    switch (wpb) {
      case 1: return launch_ens_flat_t<T, NP, LAY, 1>(a, s);
      case 2: return launch_ens_flat_t<T, NP, LAY, 2>(a, s);
      case 4: return launch_ens_flat_t<T, NP, LAY, 4>(a, s);
      default: return hipErrorInvalidValue;
    }
  }
  switch (wpb) {
    case 1: return launch_ens_np_t<T, NP, LAY, 1>(a, s);
    case 2: return launch_ens_np_t<T, NP, LAY, 2>(a, s);
    case 4: return launch_ens_np_t<T, NP, LAY, 4>(a, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename T, int NP>
static hipError_t launch_ens_np_w(int layout, int wpb, const EnsLaunch &a, hipStream_t s) {
  switch (layout) {
    case 0: return launch_ens_np_l<T, NP, 0>(wpb, a, s);
    case 1: return launch_ens_np_l<T, NP, 1>(wpb, a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_ens_stage_np(int dtype, int np, int layout, int wpb, const EnsLaunch &a, hipStream_t s) {
  DGSW_DISPATCH(dtype, np, launch_ens_np_w, layout, wpb, a, s)
  return hipErrorInvalidValue;
}

template <typename T, int NPMAX, int WPB>
static hipError_t launch_ens_t(const EnsLaunch &a, hipStream_t s) {
  if (a.combine)
    hipLaunchKernelGGL((k_ens_stage<T, NPMAX, WPB, 1>), dim3(a.parts), dim3(64 * WPB), 0, s,
                       static_cast<const T *>(a.q), static_cast<const T *>(a.q0), static_cast<T *>(a.out),
                       static_cast<const unsigned char *>(a.tabs), a.items,
                       a.bounds, 1, T(a.c0), T(a.c0 + a.c1 - 1.0));
  else
    hipLaunchKernelGGL((k_ens_stage<T, NPMAX, WPB, 0>), dim3(a.parts), dim3(64 * WPB), 0, s,
                       static_cast<const T *>(a.q), static_cast<const T *>(a.q0), static_cast<T *>(a.out),
                       static_cast<const unsigned char *>(a.tabs), a.items,
                       a.bounds, 0, T(a.c0), T(a.c0 + a.c1 - 1.0));
  return hipGetLastError();
}

hipError_t launch_ens_stage(int dtype, int npmax, int wpb, const EnsLaunch &a, hipStream_t s) {
#define DGSW_ENS(NPM, W)                                                                  \
  if (npmax <= NPM && wpb == W)                                                           \
    return dtype == 0 ? launch_ens_t<double, NPM, W>(a, s) : launch_ens_t<float, NPM, W>(a, s);
  DGSW_ENS(5, 1) DGSW_ENS(5, 2) DGSW_ENS(5, 4) DGSW_ENS(8, 1) DGSW_ENS(8, 2) DGSW_ENS(8, 4)
#undef DGSW_ENS
  return hipErrorInvalidValue;
}

}  // namespace dgsw
