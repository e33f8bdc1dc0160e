// Jacobi-CG of one system run entirely by one workgroup of BLOCK threads
// (paper Sec. 6 recurrences, the K1..K3 path's order of tests and
// statuses), shared by the single-system small solve (cg.hip) and the
// persistent batched solve (batched.hip).  The SpMV is the in-order stream
// walk over tiles of ROWS <= BLOCK rows, its products staged in `prod`
// (LDS, at least as many doubles as the largest tile has entries); the dots
// are workgroup sums.  No kernel is launched per iteration and no other
// workgroup is waited for.  cg_solve_regs does the same, bit for bit, with
// the rows' entries and vectors in registers, for systems that fit them.
#pragma once

#include <cmath>

#include "common.hpp"
#include "device.hpp"
#include "spmv_core.hpp"

namespace spx {
namespace one {

// Workgroup sum returned to every thread (every thread adds the per-wave
// sums in the same order).  lds: BLOCK / 64 doubles.
template <int BLOCK>
__device__ __forceinline__ double allsum(double v, double* lds) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) lds[w] = v;
  __syncthreads();
  double r = 0.0;
#pragma unroll
  for (int i = 0; i < BLOCK / 64; ++i) r += lds[i];
  __syncthreads();
  return r;
}

// Solves A x = b from the guess in x with D^-1 in dinv; r, p, q are n-entry
// work vectors.  status0 / maxit: the solve's entry status (a nonzero one,
// e.g. a zero diagonal, stops it before any iteration) and iteration limit.
// Thread 0 stores the outcome in *st (done = 1).
// EAGER: the products' loads issued together (stream_rows): faster with
// many workgroups solving at once (the persistent batch), not for one
// system alone.  Members per thread and chunk: 8, or 6 in the eager form
// (2048 small systems: CG 12.4 ms at 6, 12.5 at 8, 13.1 at 4).
template <bool EAGER>
constexpr int kOneDepth = EAGER ? 6 : 8;
template <int BLOCK, int ROWS, bool EAGER = false>
__device__ __forceinline__ void cg_solve(int64_t n, const int32_t* __restrict__ rowptr,
                                         const int32_t* __restrict__ col,
                                         const double* __restrict__ val,
                                         const double* __restrict__ b, double* __restrict__ x,
                                         double* __restrict__ r, double* __restrict__ p,
                                         double* __restrict__ q, const double* __restrict__ dinv,
                                         int32_t status0, int32_t maxit, double rtol,
                                         CgScalars* st, double* prod, double* lds) {
  static_assert(ROWS <= BLOCK, "one thread per row of a tile");
  const int tid = threadIdx.x;
  // r = b - A x; p = D^-1 r
  double rz = 0.0, rr = 0.0, bb = 0.0;
  for (int64_t r0 = 0; r0 < n; r0 += ROWS) {
    const int64_t r1 = r0 + ROWS < n ? r0 + ROWS : n;
    const double ax = stream_rows<BLOCK, kOneDepth<EAGER>, double, double, double, false, EAGER>(
        rowptr, col, val, x, r0, r1, prod);
    if (tid < r1 - r0) {
      const int64_t row = r0 + tid;
      const double bi = b[row];
      const double ri = bi - ax;
      const double zi = dinv[row] * ri;
      r[row] = ri;
      p[row] = zi;
      rz += ri * zi;
      rr += ri * ri;
      bb += bi * bi;
    }
  }
  rz = allsum<BLOCK>(rz, lds);
  rr = allsum<BLOCK>(rr, lds);
  bb = allsum<BLOCK>(bb, lds);
  const double bnorm = sqrt(bb);
  const double thresh = rtol * bnorm;
  int32_t status = status0, iters = 0;
  double rho = rz, pq = 0.0;
  bool done = true;
  if (status != SPX_OK) {
  } else if (sqrt(rr) <= thresh) {
  } else if (maxit <= 0) {
    status = SPX_NOT_CONVERGED;
  } else {
    done = false;
  }
  for (int32_t k = 1; !done; ++k) {
    // q = A p; p.q
    double pqs = 0.0;
    for (int64_t r0 = 0; r0 < n; r0 += ROWS) {
      const int64_t r1 = r0 + ROWS < n ? r0 + ROWS : n;
      const double s = stream_rows<BLOCK, kOneDepth<EAGER>, double, double, double, false, EAGER>(
          rowptr, col, val, p, r0, r1, prod);
      if (tid < r1 - r0) {
        q[r0 + tid] = s;
        pqs += p[r0 + tid] * s;
      }
    }
    pq = allsum<BLOCK>(pqs, lds);
    if (!(pq > 0.0) || !isfinite(pq)) {
      status = SPX_BREAKDOWN;
      iters = k - 1;
      break;
    }
    const double alpha = rho / pq;
    double rzs = 0.0, rrs = 0.0;
    for (int64_t i = tid; i < n; i += BLOCK) {
      const double xi = x[i] + alpha * p[i];
      const double ri = r[i] - alpha * q[i];
      const double zi = dinv[i] * ri;
      x[i] = xi;
      r[i] = ri;
      rzs += ri * zi;
      rrs += ri * ri;
    }
    rz = allsum<BLOCK>(rzs, lds);
    rr = allsum<BLOCK>(rrs, lds);
    iters = k;
    if (sqrt(rr) <= thresh) {
      status = SPX_OK;
      break;
    }
    if (k >= maxit) {
      status = SPX_NOT_CONVERGED;
      break;
    }
    const double beta = rz / rho;
    rho = rz;
    for (int64_t i = tid; i < n; i += BLOCK) p[i] = dinv[i] * r[i] + beta * p[i];
    __syncthreads();  // p is gathered by every thread in the next product
  }
  if (tid == 0) {
    st->rho[0] = rho;
    st->pq = pq;
    st->rr = rr;
    st->bb = bb;
    st->bnorm = bnorm;
    st->thresh = thresh;
    st->iters = iters;
    st->status = status;
    st->done = 1;
  }
}

// N sums over H * BLOCK values of as many threads of a larger workgroup,
// H of which each thread here stands for (v[k][h] is the value of thread
// tid + h BLOCK), formed as allsum<H * BLOCK> forms them (N x H x BLOCK / 64
// doubles of lds).  The caller alternates between two such areas, so no
// barrier is needed after the reads.
template <int BLOCK, int H, int N>
__device__ __forceinline__ void allsum_n(double (&v)[N][H], double* lds) {
  constexpr int W = BLOCK / 64;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int k = 0; k < N; ++k) {
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const double t = wave_sum(v[k][h]);
      if (lane == 0) lds[(k * H + h) * W + w] = t;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N; ++k) {
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < W * H; ++i) t += lds[k * W * H + i];
    v[k][0] = t;
  }
}

// cg_solve for systems of at most BLOCK * RPT rows of at most K entries
// (BLOCK * RPT <= 8192), with every vector and the matrix in the compute
// unit: thread t holds rows t, t + BLOCK, ... with their values and 16-bit
// columns, r, A p, and (unless LDSV) x and D^-1 in registers; p, which the
// product reads at any row, is in LDS, with LDSV x and D^-1 too.  The walk
// over a matrix and vectors in L2 is a chain of round trips per tile (25 us
// an iteration on a 4,096-row 5-point system alone on its compute unit);
// here an iteration is K LDS reads per row and three barriers.  Each row's
// products are rounded and added in entry order (a row's unused entries are
// 0 times its own p and change nothing) and each dot takes the rows of
// cg_solve<H * BLOCK, H * BLOCK> in the same order, so every bit is
// cg_solve's (the multiply-adds are written out: the compiler would fuse a
// thread's first two squares the other way round).  vec: BLOCK * RPT doubles (3 times that with LDSV); lds: 6 x H
// x BLOCK / 64.
template <int BLOCK, int H, int RPT, int K, bool LDSV>
__device__ __forceinline__ void cg_solve_regs(int32_t n, const int32_t* __restrict__ rowptr,
                                              const int32_t* __restrict__ col,
                                              const double* __restrict__ val,
                                              const int32_t* __restrict__ dpos,
                                              const double* __restrict__ b,
                                              double* __restrict__ xg, int32_t maxit, double rtol,
                                              CgScalars* st, double* vec, double* lds) {
  static_assert(BLOCK * RPT <= 8192, "byte offsets in 16 bits");
  static_assert(RPT % H == 0, "as many rows for every thread stood for");
  constexpr int W = H * BLOCK / 64, R = LDSV ? 1 : RPT;
  const int tid = threadIdx.x;
  double* pv = vec;
  double* xv = vec + BLOCK * RPT;
  double* dv = vec + 2 * BLOCK * RPT;
  double a[RPT][K], r[RPT], q[RPT], xr[R], dr[R];
  uint32_t c[RPT][(K + 1) / 2];
  double bad[1][H] = {};
  // Rows past n are empty rows with x = r = p = D^-1 = 0: they add +0.0 to
  // every sum, and nothing below branches on them.  All loads are
  // unconditional (an entry past its row loads the row's first; the tail
  // padding keeps an empty last row's inside the arrays): branches here made
  // the compiler keep the matrix in memory.
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int32_t row = tid + k * BLOCK;
    const bool own = row < n;
    const int32_t rc = own ? row : 0;
    const int32_t t0 = rowptr[rc], t1 = rowptr[rc + 1], dp = dpos[rc];
    const int32_t len = own ? t1 - t0 : 0;
    const double xg0 = xg[rc], d0 = val[dp >= 0 ? dp : 0];
    const double d = dp >= 0 ? d0 : 0.0;
    bad[0][0] = own && d == 0.0 ? 1.0 : bad[0][0];
    const double inv = own && d != 0.0 ? 1.0 / d : 0.0, x0 = own ? xg0 : 0.0;
#pragma unroll
    for (int j = 0; j < (K + 1) / 2; ++j) c[k][j] = 0;
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const bool in = j < len;
      const int32_t t = in ? t0 + j : t0;
      const double v = val[t];
      const int32_t cj = col[t];
      a[k][j] = in ? v : 0.0;
      c[k][j / 2] |= (uint32_t)((in ? cj : row) * 8) << (16 * (j & 1));
    }
    pv[row] = x0;
    if constexpr (LDSV) {
      xv[row] = x0;
      dv[row] = inv;
    } else {
      xr[k] = x0;
      dr[k] = inv;
    }
    __builtin_amdgcn_sched_barrier(0);  // one row's loads at a time: registers
  }
  // A v for this thread's row k, v in pv.  The columns (byte offsets, two to
  // a register) are unpacked here each time: kept unpacked they would not fit.
  auto product = [&](int k) {
#pragma clang fp contract(off)
    double t = 0.0;
#pragma unroll
    for (int j = 0; j < (K + 1) / 2; ++j) asm volatile("" : "+v"(c[k][j]));
#pragma unroll
    for (int j = 0; j < K; ++j)
      t += a[k][j] * *reinterpret_cast<const double*>(
                         reinterpret_cast<const char*>(pv) +
                         ((c[k][j / 2] >> (16 * (j & 1))) & 0xffffu));
    return t;
  };
  allsum_n<BLOCK, H, 1>(bad, lds);  // and pv is complete
  int32_t status = bad[0][0] != 0.0 ? SPX_ZERO_DIAGONAL : SPX_OK, iters = 0;
  double s3[3][H] = {};  // r.z, r.r, b.b
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int32_t row = tid + k * BLOCK;
    const double bg = b[row < n ? row : 0], bi = row < n ? bg : 0.0;
    const double ri = bi - product(k);
    const double zi = (LDSV ? dv[row] : dr[LDSV ? 0 : k]) * ri;
    r[k] = ri;
    q[k] = zi;  // p below
    s3[0][k % H] = fma(ri, zi, s3[0][k % H]);
    s3[1][k % H] = fma(ri, ri, s3[1][k % H]);
    s3[2][k % H] = fma(bi, bi, s3[2][k % H]);
    __builtin_amdgcn_sched_barrier(0);
  }
  allsum_n<BLOCK, H, 3>(s3, lds + 3 * W);
#pragma unroll
  for (int k = 0; k < RPT; ++k) pv[tid + k * BLOCK] = q[k];
  __syncthreads();
  double rho = s3[0][0], rr = s3[1][0], pq = 0.0;
  const double bb = s3[2][0], bnorm = sqrt(bb), thresh = rtol * bnorm;
  bool done = true;
  if (status != SPX_OK) {
  } else if (sqrt(rr) <= thresh) {
  } else if (maxit <= 0) {
    status = SPX_NOT_CONVERGED;
  } else {
    done = false;
  }
  for (int32_t it = 1; !done; ++it) {
    double s1[1][H] = {};
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      q[k] = product(k);
      s1[0][k % H] = fma(pv[tid + k * BLOCK], q[k], s1[0][k % H]);
      if (k % 2) __builtin_amdgcn_sched_barrier(0);  // two rows' reads in flight: registers
    }
    allsum_n<BLOCK, H, 1>(s1, lds);
    pq = s1[0][0];
    if (!(pq > 0.0) || !isfinite(pq)) {
      status = SPX_BREAKDOWN;
      iters = it - 1;
      break;
    }
    const double alpha = rho / pq;
    double s2[2][H] = {};
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int32_t row = tid + k * BLOCK;
      double& x = LDSV ? xv[row] : xr[LDSV ? 0 : k];
      const double dinv = LDSV ? dv[row] : dr[LDSV ? 0 : k];
      x = fma(alpha, pv[row], x);
      r[k] = fma(-alpha, q[k], r[k]);
      const double zi = dinv * r[k];
      s2[0][k % H] = fma(r[k], zi, s2[0][k % H]);
      s2[1][k % H] = fma(r[k], r[k], s2[1][k % H]);
      if (k % 2) __builtin_amdgcn_sched_barrier(0);
    }
    allsum_n<BLOCK, H, 2>(s2, lds + 3 * W);
    rr = s2[1][0];
    iters = it;
    if (sqrt(rr) <= thresh) {
      status = SPX_OK;
      break;
    }
    if (it >= maxit) {
      status = SPX_NOT_CONVERGED;
      break;
    }
    const double beta = s2[0][0] / rho;
    rho = s2[0][0];
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int32_t row = tid + k * BLOCK;
      const double dinv = LDSV ? dv[row] : dr[LDSV ? 0 : k];
      pv[row] = fma(dinv, r[k], beta * pv[row]);
    }
    __syncthreads();  // p is read by every thread in the next product
  }
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int32_t row = tid + k * BLOCK;
    if (row < n) xg[row] = LDSV ? xv[row] : xr[LDSV ? 0 : k];
  }
  if (tid == 0) {
    st->rho[0] = rho;
    st->pq = pq;
    st->rr = rr;
    st->bb = bb;
    st->bnorm = bnorm;
    st->thresh = thresh;
    st->iters = iters;
    st->status = status;
    st->done = 1;
  }
}

}  // namespace one
}  // namespace spx
