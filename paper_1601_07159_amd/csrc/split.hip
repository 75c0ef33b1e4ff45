// Launches of the slab and plane passes on split lines (split_passes.h) and of
// the orbital transposition they take their inputs from.
#include "split_passes.h"

namespace ace {
namespace {

// Waves per SIMD that the registers are budgeted for (the most that needs no
// spills; four lanes per line leave 60 to 126 registers to a lane).
template <int N, typename R>
constexpr int kSplitWaves = sizeof(R) == 4 ? 4 : N >= 64 ? 2 : 3;

// Pairs per workgroup: up to `most`, fewer while the launch has less than
// eight workgroups for every CU.
int run_length(int n, int np, int most) {
  const long r = (long)n * np / (256 * 8);
  return (int)(r < 1 ? 1 : r > most ? most : r);
}

template <int N, typename R>
ace_status slab_n(ace_ctx c, const cx<R>* phi, const cx<R>* psi, cx<R>* buf, int mode, int i0,
                  int A, int j0, long p0, int np) {
  const int run = run_length(N, np, kSlabRun);
  const long runs = (np + run - 1) / run;
  return launch(c, "pair_fwd_slab", k_slab_split<N, R, kSplitWaves<N, R>>,
                dim3(xcd_pad(N * runs)), dim3(kSplitThreads<N>), 0, phi, psi, buf, mode, i0, A,
                j0, p0, np, run);
}

template <int N, typename R>
ace_status plane_n(ace_ctx c, cx<R>* buf, const ace_kspec& ks, int np) {
  const int run = run_length(N, np, kPlaneRun);
  const long runs = (np + run - 1) / run;
  return launch(c, "plane_kernel", k_plane_split<N, R, kSplitWaves<N, R>>,
                dim3(xcd_pad(N * runs)), dim3(kSplitThreads<N>), 0, buf, ks, np, run);
}

}  // namespace

template <typename R>
ace_status split_slab(ace_ctx c, int n, const cx<R>* phi, const cx<R>* psi, cx<R>* buf, int mode,
                      int i0, int A, int j0, long p0, int np) {
  switch (n) {
#define ACE_CASE(NV) \
  case NV:           \
    if constexpr (NV >= kSplitSlabN<R>) return slab_n<NV, R>(c, phi, psi, buf, mode, i0, A, j0, p0, np); \
    break;
    ACE_FOR_EACH_N(ACE_CASE)
#undef ACE_CASE
  }
  return fail(c, ACE_E_UNSUPPORTED, "grid size not compiled into the library");
}

template <typename R>
ace_status split_plane(ace_ctx c, int n, cx<R>* buf, const ace_kspec& ks, int np) {
  switch (n) {
#define ACE_CASE(NV) \
  case NV:           \
    if constexpr (NV >= kSplitPlaneN<R>) return plane_n<NV, R>(c, buf, ks, np); \
    break;
    ACE_FOR_EACH_N(ACE_CASE)
#undef ACE_CASE
  }
  return fail(c, ACE_E_UNSUPPORTED, "grid size not compiled into the library");
}

template <typename V>
ace_status orbital_transpose(ace_ctx c, int n, const V* x, long ldx, int count, V* y) {
  switch (n) {
#define ACE_CASE(NV)                                                                        \
  case NV:                                                                                  \
    if constexpr (NV >= 40)                                                                 \
      return launch(c, "orbital_transpose", k_orbital_transpose<NV, V>,                     \
                    dim3((unsigned)count * NV), dim3(256), 0, x, ldx, y);                   \
    break;
    ACE_FOR_EACH_N(ACE_CASE)
#undef ACE_CASE
  }
  return fail(c, ACE_E_UNSUPPORTED, "grid size not compiled into the library");
}

template ace_status split_slab<float>(ace_ctx, int, const cx<float>*, const cx<float>*, cx<float>*,
                                      int, int, int, int, long, int);
template ace_status split_slab<double>(ace_ctx, int, const cx<double>*, const cx<double>*,
                                       cx<double>*, int, int, int, int, long, int);
template ace_status split_plane<float>(ace_ctx, int, cx<float>*, const ace_kspec&, int);
template ace_status split_plane<double>(ace_ctx, int, cx<double>*, const ace_kspec&, int);
template ace_status orbital_transpose<cx<float>>(ace_ctx, int, const cx<float>*, long, int,
                                                 cx<float>*);
template ace_status orbital_transpose<cx<double>>(ace_ctx, int, const cx<double>*, long, int,
                                                  cx<double>*);

}  // namespace ace
