// Building blocks of the linear eigensolver inside the self-consistent loops
// of Section 2 (Alg. 1: the exchange operator applied as V_X[phi] by pair
// Poisson solves) and Section 3 (Alg. 2: the same loop with V_ACE), for a
// Hamiltonian H = -1/2 Laplacian + V_loc + V_ex of the form of Eq. HFlineig
// with a fixed local potential:
//   ace_apply_h        Y = H X, the exchange part V_ACE (from xi), V_X[phi]
//                      (pair solves) or absent;
//   ace_combine        D = a A + b B + c C on orbital blocks (the three-term
//                      recurrences of polynomial filters);
//   ace_rayleigh_ritz  S = dV X^H (HX), S = Q diag(e) Q^H by a parallel
//                      cyclic Jacobi method, X Q and (HX) Q.
// The kinetic term runs on the pair FFT passes: one "orbital" of ones and the
// kernel |G|^2 / 2 make them compute ifftn(|G|^2/2 fftn(x)) for every x.
#include <cmath>
#include <cstdio>

#include "ace_internal.h"

#define ACE_EXPORT extern "C" __attribute__((visibility("default")))

namespace ace {
namespace {

template <typename T>
__global__ __launch_bounds__(256) void k_fill_ones(cx<T>* __restrict__ x, long ng) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i < ng) x[i] = cx<T>{T(1), T(0)};
}

// Y_b[r] += V(r) X_b[r] for b < n (V real, one value per grid point).
template <typename T>
__global__ __launch_bounds__(256) void k_add_local(const cx<T>* __restrict__ X, long ldx,
                                                   const T* __restrict__ V, cx<T>* __restrict__ Y,
                                                   long ldy, long ng, int n) {
  const long total = ng * n;
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < total; e += (long)gridDim.x * 256) {
    const long b = e / ng, r = e - b * ng;
    const cx<T> x = X[b * ldx + r];
    const T v = V[r];
    cx<T> y = Y[b * ldy + r];
    y.x += v * x.x;
    y.y += v * x.y;
    Y[b * ldy + r] = y;
  }
}

// D_b[r] = a A_b[r] + b B_b[r] + c C_b[r]  (B, C nullable: their term absent).
template <typename T>
__global__ __launch_bounds__(256) void k_combine(double a, const cx<T>* __restrict__ A, long lda,
                                                 double b, const cx<T>* __restrict__ B, long ldb,
                                                 double c, const cx<T>* __restrict__ C, long ldc,
                                                 cx<T>* __restrict__ D, long ldd, long ng, int n) {
  const long total = ng * n;
  const T ta = (T)a, tb = (T)b, tc = (T)c;
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < total; e += (long)gridDim.x * 256) {
    const long k = e / ng, r = e - k * ng;
    const cx<T> x = A[k * lda + r];
    cx<T> y = {ta * x.x, ta * x.y};
    if (B) {
      const cx<T> u = B[k * ldb + r];
      y.x += tb * u.x;
      y.y += tb * u.y;
    }
    if (C) {
      const cx<T> u = C[k * ldc + r];
      y.x += tc * u.x;
      y.y += tc * u.y;
    }
    D[k * ldd + r] = y;
  }
}

inline unsigned stream_blocks(long total) {
  const long b = (total + 255) / 256;
  return (unsigned)(b < 8192 ? b : 8192);
}

// ---------------------------------------------------------------------------
// Hermitian eigensolver for n <= kJacobiMax: the parallel cyclic Jacobi method
// (Brent-Luk order) in two kernels.  A sweep visits every pair (p, q) once in
// n - 1 steps (n even; a zero row and column pad odd n) of n/2 disjoint pairs,
// scheduled by the circle method (index m = n - 1 fixed, the others rotating).
// For the pair (p, q) with a = A_pp, b = A_qq, A_pq = |c| e^{i phi}: the phase
// D = diag(1, e^{-i phi}) makes the pair block real, then the real rotation
// [[cs, sn], [-sn, cs]] with t = tan(theta) the smaller root of
// t^2 + 2 tau t - 1 = 0, tau = (b - a) / (2 |c|), annihilates it:
//   rows:    p <- cs p - sn e^{i phi} q,   q <- sn p + cs e^{i phi} q
//   columns: p <- cs p - sn e^{-i phi} q,  q <- sn p + cs e^{-i phi} q.
// Sweeps stop when the off-diagonal Frobenius norm falls below tol times the
// whole norm (or after max_sweeps).  The eigenvalues (real parts of the final
// diagonal) are sorted ascending, ties by index, and the columns of V follow.
//
// k_jacobi_sweeps (one workgroup) rotates A alone and records the rotations;
// k_jacobi_vectors forms V from them.  The sweeps are a serial chain of
// (n - 1) x sweeps steps of two barriers, so what a step does decides the
// time: a thread takes whole 2 x 2 blocks (pair k's rows x pair l's columns)
// and applies both sides to them in registers, rows first (one pass over A in
// LDS and one barrier where rows and columns in turn take two of each), and V,
// whose rows never mix, leaves the workgroup: one wave per row of V replays
// the recorded rotations, all rows in parallel.  Measured, against one kernel
// with separate row and column passes and V in global memory: n = 88 (A in
// LDS) 5.98 -> 1.75 + 0.11 ms, the whole Rayleigh-Ritz step at n = 128 (A in
// global memory) 29.2 -> 6.5 ms, at n = 256 303 -> 137 ms.
// A is kept in LDS up to kJacobiLds rows, in global scratch beyond.
constexpr int kJacobiMax = 512;
constexpr int kJacobiLds = 88;  // 88^2 complex128 = 121 KiB of LDS
constexpr int kJacobiSmall = 32;  // up to here the vectors turn along with A
constexpr int kJacobiSweeps = 30;

struct alignas(16) JacobiRot {
  double cs, sn, er, ei;  // cosine, sine, e^{i phi}; sn = 0: not rotated
};

// Pair k of step st: (st, m) for k = 0, else (st + k, st - k) mod m; p < q.
__device__ __forceinline__ void jacobi_pair(int st, int k, int m, int* p, int* q) {
  int x = st, y = m;
  if (k != 0) {
    x = st + k;
    x = x >= m ? x - m : x;
    y = st - k;
    y = y < 0 ? y + m : y;
  }
  *p = x < y ? x : y;
  *q = x < y ? y : x;
}

// The rotation of pair (p, q) from its block's entries a = A_pp, b = A_qq, c = A_pq.
// (Here and in jacobi_rows / jacobi_cols the fused multiply-adds are explicit:
// the vector a rotation ends on depends on the rounding of nearly converged
// entries, so every form must round alike.)
__device__ __forceinline__ JacobiRot jacobi_rotation(double a, double b, cx<double> c) {
  JacobiRot r{1.0, 0.0, 1.0, 0.0};
  const double ac = sqrt(fma(c.x, c.x, c.y * c.y));
  if (ac > 1e-300 && ac > 1e-18 * sqrt(fabs(a * b))) {
    const double tau = (b - a) / (2.0 * ac);
    const double tt = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(fma(tau, tau, 1.0)));
    r.cs = 1.0 / sqrt(fma(tt, tt, 1.0));
    r.sn = tt * r.cs;
    r.er = c.x / ac;
    r.ei = c.y / ac;
  }
  return r;
}

// Rows p, q of one column: p <- cs p - sn e^{i phi} q, q <- sn p + cs e^{i phi} q.
__device__ __forceinline__ void jacobi_rows(cx<double>& p, cx<double>& q, const JacobiRot& r) {
  const cx<double> ap = p;
  const double ex = fma(r.er, q.x, -(r.ei * q.y)), ey = fma(r.ei, q.x, r.er * q.y);
  p = {fma(r.cs, ap.x, -(r.sn * ex)), fma(r.cs, ap.y, -(r.sn * ey))};
  q = {fma(r.sn, ap.x, r.cs * ex), fma(r.sn, ap.y, r.cs * ey)};
}
// Columns p, q of one row: p <- cs p - sn e^{-i phi} q, q <- sn p + cs e^{-i phi} q.
__device__ __forceinline__ void jacobi_cols(cx<double>& p, cx<double>& q, const JacobiRot& r) {
  const cx<double> ap = p;
  const double ex = fma(r.er, q.x, r.ei * q.y), ey = fma(r.er, q.y, -(r.ei * q.x));
  p = {fma(r.cs, ap.x, -(r.sn * ex)), fma(r.cs, ap.y, -(r.sn * ey))};
  q = {fma(r.sn, ap.x, r.cs * ex), fma(r.sn, ap.y, r.cs * ey)};
}

// Both sides of the rotations on one block: rows of pair k, then columns of
// pair l.
__device__ __forceinline__ void jacobi_block(cx<double> (&b)[2][2], const JacobiRot& rk,
                                             const JacobiRot& rl) {
  if (rk.sn != 0.0) {
    jacobi_rows(b[0][0], b[1][0], rk);
    jacobi_rows(b[0][1], b[1][1], rk);
  }
  if (rl.sn != 0.0) {
    jacobi_cols(b[0][0], b[0][1], rl);
    jacobi_cols(b[1][0], b[1][1], rl);
  }
}

// A = (S + S^H)/2 (ne x ne, the padding of odd n zero).
template <int NT>
__device__ __forceinline__ void jacobi_load(const cx<double>* __restrict__ S, int lds_, int n,
                                            int ne, cx<double>* A, int lda) {
  for (int e = threadIdx.x; e < ne * ne; e += NT) {
    const int i = e % ne, j = e / ne;
    cx<double> v = {0.0, 0.0};
    if (i < n && j < n) {
      const cx<double> u = S[i + (size_t)j * lds_], w = S[j + (size_t)i * lds_];
      v = {0.5 * (u.x + w.x), 0.5 * (u.y - w.y)};
    }
    A[i + j * lda] = v;
  }
  __syncthreads();
}

// Whether the off-diagonal Frobenius norm of A is at most tol times the whole
// one (the same answer in every thread).
template <int NT>
__device__ __forceinline__ bool jacobi_converged(const cx<double>* A, int lda, int n, double tol) {
  __shared__ double red[2][NT];
  const int t = threadIdx.x;
  double off = 0.0, all = 0.0;
  for (int e = t; e < n * n; e += NT) {
    const int i = e % n, j = e / n;
    const cx<double> u = A[i + j * lda];
    const double v = fma(u.x, u.x, u.y * u.y);
    all += v;
    if (i != j) off += v;
  }
  red[0][t] = off;
  red[1][t] = all;
  __syncthreads();
  for (int w = NT / 2; w > 0; w >>= 1) {
    if (t < w) {
      red[0][t] += red[0][t + w];
      red[1][t] += red[1][t + w];
    }
    __syncthreads();
  }
  const bool done = !(red[0][0] > tol * tol * red[1][0]);
  __syncthreads();
  return done;
}

// ctl[0] = the number of sweeps; the eigenvalues in ascending order (ties by
// index) and the rank of diagonal entry i in ctl[1 + i].
template <int NT>
__device__ __forceinline__ void jacobi_finish(const cx<double>* A, int lda, int n, int sweeps,
                                              int* __restrict__ ctl, double* __restrict__ evals) {
  if (threadIdx.x == 0) ctl[0] = sweeps;
  for (int i = threadIdx.x; i < n; i += NT) {
    const double ei = A[i + i * lda].x;
    int rank = 0;
    for (int j = 0; j < n; ++j) {
      const double ej = A[j + j * lda].x;
      rank += (ej < ei || (ej == ei && j < i)) ? 1 : 0;
    }
    evals[rank] = ei;
    ctl[1 + i] = rank;
  }
}

// Sweeps for n <= kJacobiLds, A in LDS.  Rotations of all steps, in order:
// rots[(sweep m + st) np + k].  A thread owns the blocks (k, l) and
// (k, l + dl) of every step.  The last wave forms the step's rotations (a
// serial chain of square roots and divisions) while every wave reads its
// blocks; after a barrier they are rotated and written back.  At n = 88 a step
// takes 2.0 us on the one CU: the rotations 0.55, then LDS traffic (busy 56% of
// the cycles) and the FP64 products (35% VALU issue) in turn.  The indices of a
// pair are kept as byte offsets into A that advance by one index per step (and
// are back at the first step's after m of them): no multiply or remainder in
// the loop.
struct JacobiPos {  // the two indices of a pair, as offsets of one stride
  int x, y, dy, end, step;
  __device__ __forceinline__ JacobiPos(int k, int m, int stride)
      : x(k * stride), y((k ? m - k : m) * stride), dy(k ? stride : 0),
        end(m * stride), step(stride) {}
  __device__ __forceinline__ int p() const { return x < y ? x : y; }
  __device__ __forceinline__ int q() const { return x < y ? y : x; }
  __device__ __forceinline__ void advance() {
    x += step;
    x = x == end ? 0 : x;
    y += dy;
    y = y == end && dy ? 0 : y;  // pair 0 keeps the fixed index m
  }
};

//
// VEC (n <= kJacobiSmall): threads without blocks turn the vectors V along, each
// one pair of columns of one row, instead of a second launch that replays the
// rotations: the Rayleigh-Ritz step on 16 vectors at 16^3 181 -> 158 us, on 8
// 95 -> 82 us, with 256 threads up to n = 16 (170 and 86 us with 1,024).
template <int LD, bool VEC, int NT>
__global__ __launch_bounds__(NT) void k_jacobi_sweeps_lds(const cx<double>* __restrict__ S,
                                                            int lds_, int n,
                                                            JacobiRot* __restrict__ rots,
                                                            int* __restrict__ ctl,
                                                            double* __restrict__ evals,
                                                            int max_sweeps, double tol,
                                                            cx<double>* __restrict__ Vout) {
  constexpr int RB = (int)sizeof(cx<double>), CB = LD * RB;  // row and column strides in bytes
  typedef double v2d __attribute__((ext_vector_type(2)));
  __shared__ alignas(16) cx<double> A[LD * LD];
  __shared__ v2d rot[2][LD / 2];  // (cs, sn) and (er, ei): 16-byte strides, no bank conflicts
  constexpr int LV = LD + 1;
  __shared__ cx<double> V[VEC ? LD * LV : 1];
  constexpr int kFirstV = (LD / 2) * ((LD / 2 + 1) / 2);  // threads before have blocks
  static_assert(!VEC || kFirstV + LD * (LD / 2) <= NT - 64, "a thread per row and pair of V");
  static_assert((LD / 2) * ((LD / 2 + 1) / 2) <= NT && LD / 2 <= 64, "two blocks per thread");
  const int t = threadIdx.x;
  const int ne = n + (n & 1), m = ne - 1, np = ne / 2, dl = (np + 1) / 2;
  jacobi_load<NT>(S, lds_, n, ne, A, LD);
  const int k = t % np;
  const bool has0 = t / np < dl, has1 = has0 && t / np + dl < np;
  const int l0 = has0 ? t / np : 0, l1 = has1 ? l0 + dl : 0;
  const int kr = t - (NT - 64);  // pair whose rotation this thread forms (last wave)
  const bool rotator = kr >= 0 && kr < np;
  const int kc = rotator ? kr : 0;
  JacobiPos rk(k, m, RB), c0(l0, m, CB), c1(l1, m, CB), rr(kc, m, RB), rc(kc, m, CB);
  const int tv = t - kFirstV;
  const bool turner = VEC && tv >= 0 && tv < n * np;
  const int rowv = turner ? tv / np : 0, kv = turner ? tv - rowv * np : 0;
  JacobiPos pv(kv, m, 1);
  if constexpr (VEC)
    for (int e = t; e < LD * LV; e += NT) V[e] = {e / LV == e % LV ? 1.0 : 0.0, 0.0};
  auto at = [&](int off) {
    const v2d v = *reinterpret_cast<const v2d*>(reinterpret_cast<const char*>(A) + off);
    return cx<double>{v.x, v.y};
  };
  auto rotation = [&](int i) {
    const v2d u = rot[0][i], w = rot[1][i];
    return JacobiRot{u.x, u.y, w.x, w.y};
  };
  auto put = [&](int off, cx<double> v) {
    *reinterpret_cast<v2d*>(reinterpret_cast<char*>(A) + off) = v2d{v.x, v.y};
  };
  int sweep = 0;
  for (; sweep < max_sweeps; ++sweep) {
    if (jacobi_converged<NT>(A, LD, n, tol)) break;
    JacobiRot* out = rots + (size_t)sweep * m * np + kc;
    for (int st = 0; st < m; ++st, out += np) {
      if (rotator) {
        JacobiRot r{1.0, 0.0, 1.0, 0.0};
        const int p = rr.p(), q = rr.q(), pc = rc.p(), qc = rc.q();
        if (q < n * RB) r = jacobi_rotation(at(p + pc).x, at(q + qc).x, at(p + qc));
        rot[0][kr] = v2d{r.cs, r.sn};
        rot[1][kr] = v2d{r.er, r.ei};
        if constexpr (!VEC) *out = r;
      }
      rr.advance();
      rc.advance();
      cx<double> b0[2][2], b1[2][2];
      const int pk = rk.p(), qk = rk.q();
      const int p0 = c0.p(), q0 = c0.q(), p1 = c1.p(), q1 = c1.q();
      rk.advance();
      c0.advance();
      c1.advance();
      b0[0][0] = at(pk + p0);
      b0[1][0] = at(qk + p0);
      b0[0][1] = at(pk + q0);
      b0[1][1] = at(qk + q0);
      b1[0][0] = at(pk + p1);
      b1[1][0] = at(qk + p1);
      b1[0][1] = at(pk + q1);
      b1[1][1] = at(qk + q1);
      __syncthreads();
      const JacobiRot r = rotation(k);
      if (has0) {
        jacobi_block(b0, r, rotation(l0));
        put(pk + p0, b0[0][0]);
        put(qk + p0, b0[1][0]);
        put(pk + q0, b0[0][1]);
        put(qk + q0, b0[1][1]);
      }
      if (has1) {
        jacobi_block(b1, r, rotation(l1));
        put(pk + p1, b1[0][0]);
        put(qk + p1, b1[1][0]);
        put(pk + q1, b1[0][1]);
        put(qk + q1, b1[1][1]);
      }
      if constexpr (VEC) {
        const int p = pv.p(), q = pv.q();
        pv.advance();
        if (turner) {
          const JacobiRot x = rotation(kv);
          if (x.sn != 0.0) {
            cx<double> vp = V[rowv * LV + p], vq = V[rowv * LV + q];
            jacobi_cols(vp, vq, x);
            V[rowv * LV + p] = vp;
            V[rowv * LV + q] = vq;
          }
        }
      }
      __syncthreads();
    }
  }
  jacobi_finish<NT>(A, LD, n, sweep, ctl, evals);
  if constexpr (VEC) {
    __syncthreads();
    for (int e = t; e < n * n; e += NT) {
      const int row = e % n, c = e / n;
      Vout[row + (size_t)ctl[1 + c] * n] = V[row * LV + c];
    }
  }
}

// Sweeps for larger n: A (ne x ne) in global memory (L2), block by block.
__global__ __launch_bounds__(1024) void k_jacobi_sweeps(const cx<double>* __restrict__ S, int lds_,
                                                        int n, cx<double>* __restrict__ A,
                                                        JacobiRot* __restrict__ rots,
                                                        int* __restrict__ ctl,
                                                        double* __restrict__ evals,
                                                        int max_sweeps, double tol) {
  __shared__ JacobiRot rot[kJacobiMax / 2];
  const int t = threadIdx.x;
  const int ne = n + (n & 1), m = ne - 1, np = ne / 2;
  jacobi_load<1024>(S, lds_, n, ne, A, ne);
  // the thread's first block (k, l) and the step to its next one
  const int k0 = t % np, l0 = t / np, dk = 1024 % np, dl = 1024 / np;
  int sweep = 0;
  for (; sweep < max_sweeps; ++sweep) {
    if (jacobi_converged<1024>(A, ne, n, tol)) break;
    JacobiRot* out = rots + (size_t)sweep * m * np;
    for (int st = 0; st < m; ++st, out += np) {
      for (int k = t; k < np; k += 1024) {
        int p, q;
        jacobi_pair(st, k, m, &p, &q);
        JacobiRot r{1.0, 0.0, 1.0, 0.0};
        if (q < n) r = jacobi_rotation(A[p + p * ne].x, A[q + q * ne].x, A[p + q * ne]);
        rot[k] = r;
        out[k] = r;
      }
      __syncthreads();
      int k = k0, l = l0;
      while (l < np) {
        int pk, qk, pl, ql;
        jacobi_pair(st, k, m, &pk, &qk);
        jacobi_pair(st, l, m, &pl, &ql);
        cx<double> b[2][2] = {{A[pk + pl * ne], A[pk + ql * ne]},
                              {A[qk + pl * ne], A[qk + ql * ne]}};
        jacobi_block(b, rot[k], rot[l]);
        A[pk + pl * ne] = b[0][0];
        A[pk + ql * ne] = b[0][1];
        A[qk + pl * ne] = b[1][0];
        A[qk + ql * ne] = b[1][1];
        k += dk;
        l += dl;
        if (k >= np) {
          k -= np;
          ++l;
        }
      }
      __syncthreads();
    }
  }
  jacobi_finish<1024>(A, ne, n, sweep, ctl, evals);
}

// V = the product of the recorded rotations, columns in the order of the
// ranks: one wave per row of V (the row in LDS; its DS operations stay in
// order, so steps need no barrier).  The rotations of kJacobiAhead steps are
// loaded while the previous ones are applied.
constexpr int kJacobiAhead = 4;
template <int PPL>  // pairs per lane: n <= 128 PPL
__global__ __launch_bounds__(64) void k_jacobi_vectors(const JacobiRot* __restrict__ rots,
                                                       const int* __restrict__ ctl, int n,
                                                       cx<double>* __restrict__ Vout, int ldv) {
  __shared__ cx<double> v[kJacobiMax];
  const int row = blockIdx.x, lane = threadIdx.x;
  const int ne = n + (n & 1), m = ne - 1, np = ne / 2;
  for (int c = lane; c < ne; c += 64) v[c] = {c == row ? 1.0 : 0.0, 0.0};
  const int steps = ctl[0] * m;
  constexpr int D = kJacobiAhead;
  JacobiRot r[D][PPL];
  auto load = [&](JacobiRot (&x)[PPL], int s) {
    const int sc = s < steps ? s : steps - 1;
#pragma unroll
    for (int u = 0; u < PPL; ++u) {
      const int k = lane + 64 * u;
      x[u] = rots[(size_t)sc * np + (k < np ? k : np - 1)];
    }
  };
  int st = 0;
  if (steps > 0)
#pragma unroll
    for (int d = 0; d < D; ++d) load(r[d], d);
  for (int s0 = 0; s0 < steps; s0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (s0 + d < steps) {  // uniform
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < PPL; ++u) {
          const int k = lane + 64 * u;
          const JacobiRot x = r[d][u];
          if (k < np && x.sn != 0.0) {
            int p, q;
            jacobi_pair(st, k, m, &p, &q);
            cx<double> vp = v[p], vq = v[q];
            jacobi_cols(vp, vq, x);
            v[p] = vp;
            v[q] = vq;
          }
        }
        st = st + 1 == m ? 0 : st + 1;
      }
      load(r[d], s0 + d + D);
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  for (int c = lane; c < n; c += 64) Vout[row + (size_t)ctl[1 + c] * ldv] = v[c];
}

}  // namespace

// Y = H X with H = -1/2 Laplacian + V_loc + V_ex (see ace_apply_h).
template <typename T>
ace_status hamiltonian_t(ace_ctx c, const GridInfo& g, const T* vloc, const cx<T>* xi, int nxi,
                         long ldxi, const cx<T>* phi, int nphi, long ldphi, double scale_x,
                         const cx<T>* X, int nx, long ldx, cx<T>* Y, long ldy) {
  ace_status st = ACE_OK;
  bool have = false;  // Y holds a term already
  if (xi) {
    // V_ACE X = -xi (dV xi^H X)
    const size_t mat = align_up((size_t)nxi * nx * sizeof(cx<double>), 256);
    ACE_TRY(ws_begin(c, mat + gemm_cn_partial_bytes(nxi, nx, g.ng, sizeof(cx<T>), kFp32Chunks, false)));
    cx<double>* C = (cx<double>*)ws_take(c, mat, &st);
    if (!C) return st;
    ACE_TRY(gemm_cn<T>(c, xi, ldxi, nxi, X, ldx, nx, g.ng, -g.dV, C, nxi, kFp32Chunks));
    ACE_TRY(gemm_nn<T>(c, xi, ldxi, nxi, C, nxi, nx, Y, ldy, g.ng, false));
    have = true;
  } else if (phi) {
    // scale_x V_X[phi] X by pair Poisson solves
    ACE_TRY(build_W_impl<T>(c, g, phi, nphi, ldphi, X, nx, ldx, Y, ldy, scale_x));
    have = true;
  }
  // kinetic term through the pair passes: one orbital of ones, kernel |G|^2/2;
  // the ones sit in a workspace prefix that the build's own pieces skip
  GridInfo gk = g;
  gk.kind = kKindKinetic;
  const size_t ones_bytes = align_up((size_t)g.ng * sizeof(cx<T>), 256);
  const BuildPlan pl = plan_build(c, gk, sizeof(cx<T>), 1, nx, false);
  ACE_TRY(ws_begin(c, ones_bytes + pl.bytes));
  cx<T>* ones = (cx<T>*)ws_take(c, (size_t)g.ng * sizeof(cx<T>), &st);
  if (!ones) return st;
  ACE_TRY(launch(c, "fill_ones", k_fill_ones<T>, dim3((unsigned)((g.ng + 255) / 256)), dim3(256),
                 0, ones, g.ng));
  c->ws_prefix = ones_bytes;
  st = build_W_impl<T>(c, gk, ones, 1, g.ng, X, nx, ldx, Y, ldy, -1.0, nullptr, have);
  c->ws_prefix = 0;
  if (st != ACE_OK) return st;
  if (vloc)
    ACE_TRY(launch(c, "add_local", k_add_local<T>, dim3(stream_blocks((long)g.ng * nx)), dim3(256),
                   0, X, ldx, vloc, Y, ldy, g.ng, nx));
  return ACE_OK;
}

size_t hamiltonian_ws_bytes(ace_ctx c, const GridInfo& g, size_t eb, int nx, int nxi, int nphi,
                            bool copies) {
  GridInfo gk = g;
  gk.kind = kKindKinetic;
  size_t need = align_up((size_t)g.ng * eb, 256) + plan_build(c, gk, eb, 1, nx, false).bytes;
  if (nxi > 0)
    need = std::max(need, align_up((size_t)nxi * nx * sizeof(cx<double>), 256) +
                              gemm_cn_partial_bytes(nxi, nx, g.ng, eb, kFp32Chunks, false));
  if (nphi > 0) need = std::max(need, plan_build(c, g, eb, nphi, nx, false).size(copies));
  return need;
}

// Rotations of up to kJacobiSweeps sweeps (at least one element for n = 1).
static size_t jacobi_rot_bytes(int n) {
  const size_t ne = n + (n & 1);
  return kJacobiSweeps * (ne - 1) * (ne / 2) * sizeof(JacobiRot);
}

size_t ritz_ws_bytes(int n, long ng) {
  const size_t mat = align_up((size_t)n * n * sizeof(cx<double>), 256);
  const size_t ne = n + (n & 1);
  return 2 * mat + align_up(ne * ne * sizeof(cx<double>), 256) +
         align_up((1 + (size_t)n) * sizeof(int), 256) +
         std::max(gemm_cn_scratch_bytes(n, n, ng), align_up(jacobi_rot_bytes(n), 256));
}

namespace {

template <typename T>
ace_status rayleigh_ritz_t(ace_ctx c, const GridInfo& g, const cx<T>* X, long ldx,
                           const cx<T>* HX, long ldhx, int n, cx<T>* Xout, cx<T>* HXout,
                           long ldo, double* evals) {
  const size_t mat = align_up((size_t)n * n * sizeof(cx<double>), 256);
  const size_t ne = n + (n & 1);
  ACE_TRY(ws_begin(c, ritz_ws_bytes(n, g.ng)));
  ace_status st = ACE_OK;
  cx<double>* S = (cx<double>*)ws_take(c, mat, &st);
  cx<double>* Q = (cx<double>*)ws_take(c, mat, &st);
  cx<double>* A = (cx<double>*)ws_take(c, ne * ne * sizeof(cx<double>), &st);
  int* ctl = (int*)ws_take(c, (1 + (size_t)n) * sizeof(int), &st);
  if (!S || !A || !ctl || !Q) return st;
  const size_t used = c->ws_used;
  // S = dV X^H (H X), Hermitian for Hermitian H: upper tiles, lower mirrored.
  // By tiles, in one order of summation: the sweeps end at a threshold, and
  // rounding differences of S turn the vectors of close eigenvalues (by 1e-4,
  // 96 vectors at 48^3; 0.05 ms of 2.2).
  ACE_TRY(gemm_cn<T>(c, X, ldx, n, HX, ldhx, n, g.ng, g.dV, S, n, kFp64Tiles, false, true));
  // the rotations take the place of the reduction's partial sums, which the
  // stream has consumed by then
  c->ws_used = used;
  JacobiRot* rots = (JacobiRot*)ws_take(c, jacobi_rot_bytes(n), &st);
  if (!rots) return st;
  if (n <= 16)
    ACE_TRY(launch(c, "jacobi_sweeps", k_jacobi_sweeps_lds<17, true, 256>, dim3(1), dim3(256), 0,
                   (const cx<double>*)S, n, n, rots, ctl, evals, kJacobiSweeps, 1e-15, Q));
  else if (n <= kJacobiSmall)
    ACE_TRY(launch(c, "jacobi_sweeps", k_jacobi_sweeps_lds<kJacobiSmall + 1, true, 1024>, dim3(1),
                   dim3(1024), 0, (const cx<double>*)S, n, n, rots, ctl, evals, kJacobiSweeps,
                   1e-15, Q));
  else if (n <= kJacobiLds)
    ACE_TRY(launch(c, "jacobi_sweeps", k_jacobi_sweeps_lds<kJacobiLds, false, 1024>, dim3(1),
                   dim3(1024), 0, (const cx<double>*)S, n, n, rots, ctl, evals, kJacobiSweeps,
                   1e-15, Q));
  else
    ACE_TRY(launch(c, "jacobi_sweeps", k_jacobi_sweeps, dim3(1), dim3(1024), 0,
                   (const cx<double>*)S, n, n, A, rots, ctl, evals, kJacobiSweeps, 1e-15));
  const auto vectors = n <= 128   ? k_jacobi_vectors<1>
                       : n <= 256 ? k_jacobi_vectors<2>
                                  : k_jacobi_vectors<4>;
  if (n > kJacobiSmall)
    ACE_TRY(launch(c, "jacobi_vectors", vectors, dim3(n), dim3(64), 0, (const JacobiRot*)rots,
                   (const int*)ctl, n, Q, n));
  ACE_TRY(gemm_nn<T>(c, X, ldx, n, Q, n, n, Xout, ldo, g.ng, true));
  if (HXout) ACE_TRY(gemm_nn<T>(c, HX, ldhx, n, Q, n, n, HXout, ldo, g.ng, true));
  return ACE_OK;
}

}  // namespace
}  // namespace ace

using namespace ace;

ACE_EXPORT ace_status ace_apply_h(ace_ctx c, const ace_grid* grid, ace_prec prec, const void* vloc,
                                  const void* xi, int n_xi, long ld_xi, const void* phi,
                                  int n_phi, long ld_phi, double scale_x, const void* X, int n_x,
                                  long ld_x, void* Y, long ld_y) {
  if (!c) return ACE_E_ARG;
  GridInfo g;
  ACE_TRY(check_grid(c, grid, prec, &g));
  if (prec == ACE_REAL32 || prec == ACE_REAL64)
    return fail(c, ACE_E_UNSUPPORTED, "ace_apply_h takes complex orbitals");
  if (xi && phi) return fail(c, ACE_E_ARG, "give xi (V_ACE) or phi (V_X), not both");
  ACE_TRY(check_block(c, X, n_x, ld_x, g, "X"));
  ACE_TRY(check_block(c, Y, n_x, ld_y, g, "Y"));
  if (xi) ACE_TRY(check_block(c, xi, n_xi, ld_xi, g, "xi"));
  if (phi) ACE_TRY(check_block(c, phi, n_phi, ld_phi, g, "phi"));
  if (!std::isfinite(scale_x)) return fail(c, ACE_E_ARG, "scale_x must be finite");
  const size_t eb = elem_bytes(prec);
  const Span sy = span_of(Y, n_x, ld_y, g.ng, eb);
  if (overlap(sy, span_of(X, n_x, ld_x, g.ng, eb)) ||
      (xi && overlap(sy, span_of(xi, n_xi, ld_xi, g.ng, eb))) ||
      (phi && overlap(sy, span_of(phi, n_phi, ld_phi, g.ng, eb))))
    return fail(c, ACE_E_ARG, "Y overlaps an input");
  if (prec == ACE_FP64)
    return hamiltonian_t<double>(c, g, (const double*)vloc, (const cx<double>*)xi, n_xi, ld_xi,
                                 (const cx<double>*)phi, n_phi, ld_phi, scale_x,
                                 (const cx<double>*)X, n_x, ld_x, (cx<double>*)Y, ld_y);
  return hamiltonian_t<float>(c, g, (const float*)vloc, (const cx<float>*)xi, n_xi, ld_xi,
                              (const cx<float>*)phi, n_phi, ld_phi, scale_x, (const cx<float>*)X,
                              n_x, ld_x, (cx<float>*)Y, ld_y);
}

ACE_EXPORT ace_status ace_combine(ace_ctx c, const ace_grid* grid, ace_prec prec, int n, double a,
                                  const void* A, long lda, double b, const void* B, long ldb,
                                  double cc, const void* C, long ldc, void* D, long ldd) {
  if (!c) return ACE_E_ARG;
  GridInfo g;
  ACE_TRY(check_grid(c, grid, prec, &g));
  if (prec == ACE_REAL32 || prec == ACE_REAL64)
    return fail(c, ACE_E_UNSUPPORTED, "ace_combine takes complex orbitals");
  if (!std::isfinite(a) || !std::isfinite(b) || !std::isfinite(cc))
    return fail(c, ACE_E_ARG, "coefficients must be finite");
  ACE_TRY(check_block(c, A, n, lda, g, "A"));
  ACE_TRY(check_block(c, D, n, ldd, g, "D"));
  if (B) ACE_TRY(check_block(c, B, n, ldb, g, "B"));
  if (C) ACE_TRY(check_block(c, C, n, ldc, g, "C"));
  const dim3 grd(stream_blocks((long)g.ng * n));
  if (prec == ACE_FP64)
    return launch(c, "combine", k_combine<double>, grd, dim3(256), 0, a, (const cx<double>*)A, lda,
                  b, (const cx<double>*)B, ldb, cc, (const cx<double>*)C, ldc, (cx<double>*)D, ldd,
                  g.ng, n);
  return launch(c, "combine", k_combine<float>, grd, dim3(256), 0, a, (const cx<float>*)A, lda, b,
                (const cx<float>*)B, ldb, cc, (const cx<float>*)C, ldc, (cx<float>*)D, ldd, g.ng,
                n);
}

ACE_EXPORT ace_status ace_rayleigh_ritz(ace_ctx c, const ace_grid* grid, ace_prec prec,
                                        const void* X, long ld_x, const void* HX, long ld_hx,
                                        int n, void* Xout, void* HXout, long ld_out,
                                        double* evals_dev) {
  if (!c) return ACE_E_ARG;
  GridInfo g;
  ACE_TRY(check_grid(c, grid, prec, &g));
  if (prec == ACE_REAL32 || prec == ACE_REAL64)
    return fail(c, ACE_E_UNSUPPORTED, "ace_rayleigh_ritz takes complex orbitals");
  if (n < 1 || n > kJacobiMax) return fail(c, ACE_E_UNSUPPORTED, "n must be 1..512");
  if (!evals_dev) return fail(c, ACE_E_ARG, "evals_dev is NULL");
  ACE_TRY(check_block(c, X, n, ld_x, g, "X"));
  ACE_TRY(check_block(c, HX, n, ld_hx, g, "HX"));
  ACE_TRY(check_block(c, Xout, n, ld_out, g, "Xout"));
  if (HXout) ACE_TRY(check_block(c, HXout, n, ld_out, g, "HXout"));
  const size_t eb = elem_bytes(prec);
  const Span ins[2] = {span_of(X, n, ld_x, g.ng, eb), span_of(HX, n, ld_hx, g.ng, eb)};
  const Span so = span_of(Xout, n, ld_out, g.ng, eb);
  if (overlap(so, ins[0]) || overlap(so, ins[1]) ||
      (HXout && (overlap(span_of(HXout, n, ld_out, g.ng, eb), ins[0]) ||
                 overlap(span_of(HXout, n, ld_out, g.ng, eb), ins[1]) ||
                 overlap(span_of(HXout, n, ld_out, g.ng, eb), so))))
    return fail(c, ACE_E_ARG, "outputs overlap inputs or each other");
  if (prec == ACE_FP64)
    return rayleigh_ritz_t<double>(c, g, (const cx<double>*)X, ld_x, (const cx<double>*)HX, ld_hx,
                                   n, (cx<double>*)Xout, (cx<double>*)HXout, ld_out, evals_dev);
  return rayleigh_ritz_t<float>(c, g, (const cx<float>*)X, ld_x, (const cx<float>*)HX, ld_hx, n,
                                (cx<float>*)Xout, (cx<float>*)HXout, ld_out, evals_dev);
}
