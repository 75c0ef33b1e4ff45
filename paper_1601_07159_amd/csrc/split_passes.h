// Slab and plane passes on split lines (fft_split, fft_core.h).
//
// Every pass transforms two axes of a plane: the first straight from global
// memory (lanes on consecutive lines), then, through LDS, the second, whose
// lines are the rows of the first.  The slab pass takes the orbitals with axes
// 1 and 2 exchanged, f'[x0][x2][x1] (k_orbital_transpose, once per build): its
// lanes then end on consecutive k2, so that one trip through LDS leaves the
// spectrum in its natural order, stored as contiguous runs.  The plane pass
// ends with its lanes on x0 and takes a second trip to store rows of x2.
//   slab   f'[x0][x2][x1] of phi and psi -> buf[x0][k1][k2]
//   plane  buf[x0][k1][k2] -> (in place, every k1) buf[x0][k1][x2]
// The arithmetic of every line and the order of the axes are those of the quad
// forms (fft_quad_*), bit for bit in FP32.
#pragma once

#include "pass_bodies.h"

namespace ace {
namespace {

// One N x N plane per workgroup, four lanes per line; LDS rows an odd number of
// elements apart (rows at one offset fall into different banks).
template <int N>
constexpr int kSplitThreads = (N * 4 + 63) / 64 * 64;
template <int N>
constexpr int kSplitLd = N + 1 - (N & 1);

// Line l and part h of a thread.  Threads past the last line repeat it and
// store nothing (live).
template <int N>
struct SplitLane {
  int l, h;
  bool live;
  __device__ __forceinline__ explicit SplitLane(int t) {
    constexpr int LPW = 16;  // lines per wave
    const int line = (t >> 6) * LPW + (t & (LPW - 1));
    h = (t & 63) / LPW;
    live = N % LPW == 0 || line < N;
    l = live ? line : N - 1;
  }
};

// A block of complex values addressed by a wave-uniform base and a 32-bit lane
// offset: with the constant part of every access on the base (scalar
// arithmetic) the strided accesses of a line share one address register.
template <typename R>
struct LaneBlock {
  const char* base;
  __device__ __forceinline__ explicit LaneBlock(const cx<R>* p) : base((const char*)p) {}
  // element lane + fixed
  __device__ __forceinline__ cx<R> load(int lane, int fixed) const {
    const char* row = base + (size_t)fixed * sizeof(cx<R>);
    return *(const cx<R>*)(row + (size_t)(unsigned)(lane * (int)sizeof(cx<R>)));
  }
  template <bool STREAM>
  __device__ __forceinline__ void store(int lane, int fixed, cx<R> v) const {
    char* row = const_cast<char*>(base) + (size_t)fixed * sizeof(cx<R>);
    cx<R>* q = (cx<R>*)(row + (size_t)(unsigned)(lane * (int)sizeof(cx<R>)));
    if constexpr (STREAM)
      store_nt(q, v);
    else
      *q = v;
  }
};

// Position of register r of part h = fixed part of r + lane part of h (the
// registers past the last whole group have a lane part of their own).
template <int N>
struct SplitLanePos {
  int grouped, rest;
  __device__ __forceinline__ SplitLanePos(int h, int stride, int base)
      : grouped(base + h * stride),
        rest(base + N / 4 * ((h >> 1) | ((h & 1) << 1)) * stride) {}
  __device__ __forceinline__ int lane(int r) const {
    return r < Split<N>::kGrouped ? grouped : rest;
  }
  __device__ static constexpr int fixed(int r) {
    return r >= Split<N>::kGrouped ? r : r - r % 4 + N / 4 * (r % 4);
  }
};

// y[b][x0][x2][x1] = x[b][x0][x1][x2]: one x0 plane per workgroup through LDS.
template <int N, typename V>
__global__ __launch_bounds__(256) void k_orbital_transpose(const V* __restrict__ x, long ldx,
                                                           V* __restrict__ y) {
  constexpr int NN = N * N, LD = kSplitLd<N>;
  __shared__ V s[N * LD];
  const int b = blockIdx.x / N, x0 = blockIdx.x - b * N;
  const V* src = x + (size_t)b * ldx + (size_t)x0 * NN;
  V* dst = y + ((size_t)b * N + x0) * NN;
#pragma unroll
  for (int e = threadIdx.x; e < NN; e += 256) s[e / N * LD + e % N] = src[e];
  __syncthreads();
#pragma unroll
  for (int e = threadIdx.x; e < NN; e += 256) dst[e] = s[e % N * LD + e / N];
}

// The twiddle tables (both signs) into LDS, visible after the workgroup's next
// barrier.
template <int N, typename R>
__device__ __forceinline__ void split_tw_stage(cx<R>* s) {
  for (int e = threadIdx.x; e < 2 * N; e += blockDim.x) s[e] = kSplitRoots<N, R>.w[0][e];
}

// Pairs of one slab that a workgroup takes in a row: the twiddles, and the
// psi slab for as long as the band stays the same, are loaded once for all of
// them.  The quad form was bound by its vector memory instructions (16 clocks
// each in the CU's address unit, whatever their width) and by accesses of 32
// contiguous bytes; here 16 lanes cover a run of 128 (FP32), the stores of a
// spectrum need no second trip through LDS, and two loads in three remain.
// 72^3 FP32, 1,146 pairs: 1.85 -> 1.18 ms (2.9 TB/s of spectra); 40^3 FP64,
// 1,353 pairs: one thread per line 0.47 -> 0.34 ms (4.1 TB/s).
constexpr int kSlabRun = 8;  // at most (`run`)

template <int N, typename R, int WPE>
__global__ __launch_bounds__(kSplitThreads<N>) __attribute__((amdgpu_waves_per_eu(WPE))) void
k_slab_split(const cx<R>* __restrict__ phi, const cx<R>* __restrict__ psi, cx<R>* __restrict__ buf,
             int mode, int i0, int A, int j0, long p0, int npairs, int run) {
  constexpr int NN = N * N, LD = kSplitLd<N>, M = N / 4;
  __shared__ cx<R> s[N * LD];
  __shared__ cx<R> s_tw[2 * N];
  const int nruns = (npairs + run - 1) / run;
  const long lid = xcd_logical(blockIdx.x, gridDim.x);
  if (lid >= (long)N * nruns) return;
  const SplitLane<N> ln((int)threadIdx.x);
  const int l = ln.l, h = ln.h;
  const int x0 = (int)(lid / nruns);
  int p = (int)(lid - (long)x0 * nruns) * run;
  const int pend = p + run < npairs ? p + run : npairs;
  int i, j;
  pair_of(mode, i0, A, j0, p0, p, &i, &j);
  const int ibeg = mode == 3 ? 0 : i0;
  split_tw_stage<N, R>(s_tw);
  const SplitTw<N, R> tw(h, s_tw);
  const SplitLanePos<N> row(h, LD, l), col(h, N, l);
  cx<R> va[M], vb[M];
  auto load = [&](cx<R> (&x)[M], const cx<R>* f, int orb) {
    const LaneBlock<R> b(f + ((size_t)orb * N + x0) * NN);
#pragma unroll
    for (int m = 0; m < M; ++m) x[m] = b.load(h * N + l, 4 * m * N);
  };
  load(vb, psi, j);
  __syncthreads();
  for (bool first = true;; first = false) {
    cx<R> v[M];
    load(va, phi, i);
#pragma unroll
    for (int m = 0; m < M; ++m) v[m] = cmulc_fma(va[m], vb[m]);
    const LaneBlock<R> out(buf + ((size_t)p * N + x0) * NN);
    // the next pair: along the row of band j, then the next band
    const bool more = ++p < pend;
    if (more) {
      const int last = mode == 0 ? ibeg + A - 1 : mode == 1 ? j : j < A ? j : A - 1;
      if (i == last) {
        i = ibeg;
        ++j;
        load(vb, psi, j);
      } else {
        ++i;
      }
        }
    fft_split<N, -1, TwRound::kIm>(v, h, tw);  // axis 2 of column l = x1
    if (!first) __syncthreads();       // the rows of the pair before are read
#pragma unroll
    for (int r = 0; r < M; ++r) s[row.lane(r) + LD * row.fixed(r)] = v[r];
    __syncthreads();
#pragma unroll
    for (int m = 0; m < M; ++m) v[m] = s[l * LD + h + 4 * m];
    fft_split<N, -1, TwRound::kImSums>(v, h, tw);  // axis 1 of row l = k2
    if (ln.live) {
#pragma unroll
      for (int r = 0; r < M; ++r)
        out.template store<(N * sizeof(cx<R>)) % 128 == 0>(col.lane(r), N * col.fixed(r), v[r]);
    }
    if (!more) break;  // uniform
  }
}

// A workgroup takes kPlaneRun pairs at one k1: K' (the same for all of them)
// and the twiddles are formed once.  Runs of pairs first, then k1: the
// workgroups of a run work on neighbouring rows of the same pairs.  Bound by
// the strided rows of a plane (each read and written once): 72^3 FP32, 1,146
// pairs: quads 2.39 -> 1.79 ms (3.8 TB/s both ways); 40^3 FP64, 1,353 pairs:
// 0.80 -> 0.55 ms (5.1 TB/s).  Loading the next pair's plane ahead costs the
// registers of a resident workgroup (72^3 1.64 -> 1.95 ms in an earlier form),
// forming K' again for every pair as much.
constexpr int kPlaneRun = 4;  // at most (`run`)
// Whether the last transform of the plane pass runs from decimated to split
// positions (as the staged quad form, N <= 64) or the other way round.
template <int N, typename R>
constexpr bool kPlaneDif = N <= 64;

template <int N, typename R, int WPE>
__global__ __launch_bounds__(kSplitThreads<N>) __attribute__((amdgpu_waves_per_eu(WPE))) void
k_plane_split(cx<R>* __restrict__ buf, ace_kspec ks, int npairs, int run) {
  constexpr int NN = N * N, LD = kSplitLd<N>, M = N / 4;
  __shared__ cx<R> s[N * LD];
  __shared__ cx<R> s_tw[2 * N];
  const int nruns = (npairs + run - 1) / run;
  const long lid = xcd_logical(blockIdx.x, gridDim.x);
  if (lid >= (long)N * nruns) return;
  const SplitLane<N> ln((int)threadIdx.x);
  const int l = ln.l, h = ln.h;
  int p = (int)(lid / N) * run;
  const int k1 = (int)(lid % N);
  const int pend = p + run < npairs ? p + run : npairs;
  split_tw_stage<N, R>(s_tw);
  const SplitTw<N, R> tw(h, s_tw);
  const SplitLanePos<N> row(h, 1, l * LD);
  R kk[M];
  {
    const KEval<R> ke(ks);
    const R s12 = ke.part12(k1, l);
#pragma unroll
    for (int r = 0; r < M; ++r) kk[r] = ke.at(split_pos<N>(r, h), s12);
  }
  __syncthreads();
  for (bool first = true;; first = false) {
    const LaneBlock<R> plane(buf + (size_t)p * N * NN + (size_t)k1 * N);
    cx<R> v[M];
#pragma unroll
    for (int m = 0; m < M; ++m) v[m] = plane.load(h * NN + l, 4 * m * NN);
    const bool more = ++p < pend;
    fft_split<N, -1, TwRound::kIm>(v, h, tw);  // axis 0 of column l = k2
#pragma unroll
    for (int r = 0; r < M; ++r) {
      v[r].x *= kk[r];
      v[r].y *= kk[r];
      keep_rounded(v[r]);
    }
    fft_unsplit<N, +1, TwRound::kIm>(v, h, tw);
    if (!first) __syncthreads();  // the planes of the pair before are stored
#pragma unroll
    for (int m = 0; m < M; ++m) s[(h + 4 * m) * LD + l] = v[m];
    __syncthreads();
    // axis 2 of row l = x0, read and rewritten by its own lanes only
    if constexpr (kPlaneDif<N, R>) {
#pragma unroll
      for (int m = 0; m < M; ++m) v[m] = s[l * LD + h + 4 * m];
      fft_split<N, +1, TwRound::kImSums>(v, h, tw);
      if (ln.live) {
#pragma unroll
        for (int r = 0; r < M; ++r) s[row.lane(r) + row.fixed(r)] = v[r];
      }
    } else {
#pragma unroll
      for (int r = 0; r < M; ++r) v[r] = s[row.lane(r) + row.fixed(r)];
      fft_unsplit<N, +1, TwRound::kRe>(v, h, tw);
      if (ln.live) {
#pragma unroll
        for (int m = 0; m < M; ++m) s[l * LD + h + 4 * m] = v[m];
      }
    }
    __syncthreads();
    if (ln.live) {
#pragma unroll
      for (int m = 0; m < M; ++m)
        plane.template store<false>(h * NN + l, 4 * m * NN, s[(h + 4 * m) * LD + l]);
    }
    if (!more) break;  // uniform
  }
}

}  // namespace
}  // namespace ace
