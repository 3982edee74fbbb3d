// Diffusion closing stage: the collided flux of step 2 of Sec. 2.2 from a
// cell-centred finite-volume diffusion equation (the cheap deterministic
// solver the paper suggests in place of S_N),
//   sigma_r phi - div(D grad phi) = sigma_s phi_post,
//   sigma_r = sigma_a + tau/(c dt),  D = 1/(3 (sigma_t + tau/(c dt)))
// (no tau/(c dt) in steady state), harmonic-mean face coefficients, Marshak
// vacuum sides and zero-current reflective sides.  The symmetric positive
// definite system is solved by Jacobi-preconditioned conjugate gradients
// from phi = 0, each iteration two kernels:
//   k_cg_spmv:     p_k = z + beta p_{k-1} (every cell also forms its four
//                  neighbours' p_k, so the update needs no separate pass),
//                  q = A p_k, block partials of p_k . q;
//   k_cg_update:   alpha = rz / (p_k . q) (each block sums the partials in
//                  the same fixed order), x += alpha p_k, r -= alpha q,
//                  z = r / diag, block partials of r . z and r . r; the last
//                  block to leave its partials: beta, the stopping test ||r||
//                  <= tol ||b||, the iteration count, in the source-iteration
//                  state, so the graph batching of the S_N path applies (a
//                  launch of its own took 3-4 us of every iteration).
// Reductions use fixed association orders: results do not depend on
// scheduling.  The two p buffers alternate by iteration parity.  Meshes of
// up to 4096 cells run the whole solve in one workgroup instead
// (k_cg_solve_one_block), with barriers in place of launches: there the
// launches cost more than the work (a 1500-cell solve of 279 iterations
// 2.4 ms against 4.4 ms), while on larger meshes one compute unit's share of
// the bandwidth is the limit (19600 cells: 1.8 against 1.1 ms per step).
#include "slh_common.hpp"

namespace slh {

constexpr int kCgBlock = 256;

int cg_partials(long long n) {
  long long b = (n + kCgBlock - 1) / kCgBlock;
  return (int)(b < 1024 ? (b < 1 ? 1 : b) : 1024);
}

// Per-cell coefficients: diagonal, coupling to the x+1 neighbour (cE) and to
// the y+1 neighbour (cN), zero across the domain boundary.
__global__ void k_diff_coef(int nx, int ny, const double2* __restrict__ mat, double tt,
                            double hx, double hy, int bc, double* __restrict__ diag,
                            double* __restrict__ cE, double* __restrict__ cN) {
  const long long n = (long long)nx * ny;
  for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < n;
       k += (long long)gridDim.x * blockDim.x) {
    const int i = (int)(k % nx), j = (int)(k / nx);
    const double2 m = mat[k];  // (sigma_s, sigma_a)
    const double D = 1.0 / (3.0 * (m.y + m.x + tt));
    double d = m.y + tt;
    double e = 0.0, no = 0.0;
    // x faces
    if (i + 1 < nx) {
      const double2 mn = mat[k + 1];
      const double Dn = 1.0 / (3.0 * (mn.y + mn.x + tt));
      e = 2.0 * D * Dn / (D + Dn) / (hx * hx);
      d += e;
    } else if (!(bc & 2)) {
      d += 2.0 * D / (hx * (hx + 4.0 * D));
    }
    if (i > 0) {
      const double2 mw = mat[k - 1];
      const double Dw = 1.0 / (3.0 * (mw.y + mw.x + tt));
      d += 2.0 * Dw * D / (Dw + D) / (hx * hx);
    } else if (!(bc & 1)) {
      d += 2.0 * D / (hx * (hx + 4.0 * D));
    }
    // y faces
    if (j + 1 < ny) {
      const double2 mn = mat[k + nx];
      const double Dn = 1.0 / (3.0 * (mn.y + mn.x + tt));
      no = 2.0 * D * Dn / (D + Dn) / (hy * hy);
      d += no;
    } else if (!(bc & 8)) {
      d += 2.0 * D / (hy * (hy + 4.0 * D));
    }
    if (j > 0) {
      const double2 ms = mat[k - nx];
      const double Ds = 1.0 / (3.0 * (ms.y + ms.x + tt));
      d += 2.0 * Ds * D / (Ds + D) / (hy * hy);
    } else if (!(bc & 4)) {
      d += 2.0 * D / (hy * (hy + 4.0 * D));
    }
    diag[k] = d;
    cE[k] = e;
    cN[k] = no;
  }
}

hipError_t launch_diff_coef(int nx, int ny, const double2* mat, double tt, double hx, double hy,
                            int bc, double* diag, double* cE, double* cN, hipStream_t s) {
  const long long n = (long long)nx * ny;
  hipLaunchKernelGGL(k_diff_coef, dim3(cg_partials(n)), dim3(kCgBlock), 0, s, nx, ny, mat, tt,
                     hx, hy, bc, diag, cE, cN);
  return hipGetLastError();
}

// Sum of a block's values in the association order of a tree that halves the
// block from 128 threads to 1; in thread 0.  The two widest levels read LDS
// behind one barrier, the others stay in the first wave (a barrier per level
// cost 1-2 us of every launch).
__device__ __forceinline__ double block_tree(double v, double* s) {
  const int t = threadIdx.x;
  s[t] = v;
  __syncthreads();
  if (t < 64) {
    v = (s[t] + s[t + 128]) + (s[t + 64] + s[t + 192]);
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
  }
  return v;
}

// Leaves the block's sums of two values per thread in part[2 block + {0, 1}]
// and says whether the block is the grid's last to do so.  The partials cross
// the XCDs as agent-scope stores and loads; the stores have reached memory
// when the block counts itself.
__device__ __forceinline__ bool leave_partials(double a, double b, double* part, int block,
                                               RedCounter* red) {
  __shared__ double s_a[kCgBlock], s_b[kCgBlock];
  __shared__ int s_last;
  a = block_tree(a, s_a);
  b = block_tree(b, s_b);
  if (threadIdx.x == 0) {
    __hip_atomic_store(&part[2 * block], a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&part[2 * block + 1], b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    s_last = count_block(red);
  }
  __syncthreads();
  return s_last != 0;
}

// Fixed-order sum of the first (w = 0) or second (w = 1) value of n_part
// block partials of an earlier kernel; every thread of the block gets it.
__device__ __forceinline__ double sum_partials(const double* part, int n_part, int w) {
  __shared__ double s[kCgBlock];
  __shared__ double s_sum;
  double v = 0.0;
  for (int b = threadIdx.x; b < n_part; b += kCgBlock) v += part[2 * b + w];
  v = block_tree(v, s);
  if (threadIdx.x == 0) s_sum = v;
  __syncthreads();
  return s_sum;
}

// The same sums of both values of this kernel's partials, in thread 0.
__device__ __forceinline__ void sum_left(const double* part, int n_part, double& a, double& b) {
  __shared__ double s_a[kCgBlock], s_b[kCgBlock];
  a = b = 0.0;
  for (int k = threadIdx.x; k < n_part; k += kCgBlock) {
    a += __hip_atomic_load(&part[2 * k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    b += __hip_atomic_load(&part[2 * k + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  a = block_tree(a, s_a);
  b = block_tree(b, s_b);
}

// Both kernels of an iteration are bound by memory on large meshes (1024^2: 56
// and 64 MB in 12 and 17 us, 17 and 20 us before) and by launch and reduction
// latency on small ones (140^2: 4.6 and 6.0 us; with the decision of 3.7 us as
// a launch of its own and a barrier per level 17 us an iteration, now 10.6).
// Blocks take runs of the mesh XCD by XCD, so that a row's neighbours are read
// by the same L2; partials are indexed by the run, which keeps the order of the
// sums.  The update loads kCgAhead cells (all of a thread's on 1024^2) before it
// waits for the first.
constexpr int kCgAhead = 4;
__device__ __forceinline__ int cg_block() {
  return gridDim.x % 8u ? (int)blockIdx.x
                        : (int)((blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3));
}

// State of a new solve from the partials of r . z and b . b (one block).
__device__ __forceinline__ void start_state(const double* part, int n_part, IterState* cs,
                                            int max_iter) {
  double rz, bb;
  sum_left(part, n_part, rz, bb);
  if (threadIdx.x == 0) {
    cs->iter = 0;
    cs->bad = 0;
    cs->rz = rz;
    cs->beta = 0.0;
    cs->bb = bb;
    cs->dn2 = bb;
    cs->dn2_prev = 0.0;
    cs->nrm2 = bb;
    // a zero source has the exact solution 0
    const int conv = max_iter == 0 || bb == 0.0;
    cs->conv = conv;
    cs->done = conv;
    if (bb == 0.0) cs->dn2 = 0.0;
  }
}

// Start: b = sigma_s phi_post, x = 0, r = b, z = r / diag, p_{-1} = 0
// (buffer 1), r . z and b . b, and the state of the solve.
__global__ __launch_bounds__(kCgBlock) void k_cg_start(
    long long n, const double* __restrict__ sig_s, const double* __restrict__ phi_post,
    const double* __restrict__ diag, double* __restrict__ x, double* __restrict__ r,
    double* __restrict__ z, double* __restrict__ p1, double* part, RedCounter* red,
    IterState* cs, int max_iter, const int* halt) {
  if (*halt) return;
  double rz = 0.0, bb = 0.0;
  for (long long k = (long long)blockIdx.x * kCgBlock + threadIdx.x; k < n;
       k += (long long)gridDim.x * kCgBlock) {
    const double b = sig_s[k] * phi_post[k];
    const double zk = b / diag[k];
    x[k] = 0.0;
    r[k] = b;
    z[k] = zk;
    p1[k] = 0.0;
    rz += b * zk;
    bb += b * b;
  }
  if (leave_partials(rz, bb, part, blockIdx.x, red))
    start_state(part, gridDim.x, cs, max_iter);
}

// Start of the diffusion correction of a source iteration: b = sigma_s times
// the cell average of phi^{k+1/2} - phi^k (dnode, four nodes per cell), x = 0,
// r = b, z = r / diag, p_{-1} = 0, r . z and b . b, and the state of the solve.
__global__ __launch_bounds__(kCgBlock) void k_dsa_start(
    long long n, const double* __restrict__ sig_s, const double* __restrict__ dnode,
    const double* __restrict__ diag, double* __restrict__ x, double* __restrict__ r,
    double* __restrict__ z, double* __restrict__ p1, double* part, RedCounter* red,
    IterState* cs, int max_iter, const int* gate) {
  if (*gate) return;
  double rz = 0.0, bb = 0.0;
  for (long long k = (long long)blockIdx.x * kCgBlock + threadIdx.x; k < n;
       k += (long long)gridDim.x * kCgBlock) {
    const double4 d = reinterpret_cast<const double4*>(dnode)[k];
    const double b = sig_s[k] * (0.25 * ((d.x + d.y) + (d.z + d.w)));
    const double zk = b / diag[k];
    x[k] = 0.0;
    r[k] = b;
    z[k] = zk;
    p1[k] = 0.0;
    rz += b * zk;
    bb += b * b;
  }
  if (leave_partials(rz, bb, part, blockIdx.x, red))
    start_state(part, gridDim.x, cs, max_iter);
}

__global__ __launch_bounds__(kCgBlock) void k_cg_spmv(
    int nx, int ny, const double* __restrict__ diag, const double* __restrict__ cE,
    const double* __restrict__ cN, const double* __restrict__ z, double* __restrict__ P,
    double* __restrict__ q, double* __restrict__ part, const IterState* cs, const int* gate) {
  if ((gate && *gate) || cs->done) return;
  const long long n = (long long)nx * ny;
  const int it = cs->iter;
  const double beta = cs->beta;
  double* __restrict__ pk = P + (long long)(it & 1) * n;
  const double* __restrict__ pm = P + (long long)((it + 1) & 1) * n;
  double pq = 0.0;
  // at most 1024 blocks (cg_partials): the stride and the first cells are 32-bit
  const int block = cg_block();
  const unsigned stride = gridDim.x * kCgBlock, first = block * kCgBlock + threadIdx.x;
  int i = (int)(first % (unsigned)nx), j = (int)(first / (unsigned)nx);
  const int di = (int)(stride % (unsigned)nx), dj = (int)(stride / (unsigned)nx);
  for (long long k = first; k < n; k += stride) {
    // a side without a neighbour reads the cell itself and counts zero, so that
    // the loads need no branches between them
    const bool hE = i + 1 < nx, hW = i > 0, hN = j + 1 < ny, hS = j > 0;
    const long long kE = hE ? k + 1 : k, kW = hW ? k - 1 : k;
    const long long kN = hN ? k + nx : k, kS = hS ? k - nx : k;
    const double c0 = cE[k], c1 = cE[kW], c2 = cN[k], c3 = cN[kS];
    const double pc = z[k] + beta * pm[k];
    const double pE = z[kE] + beta * pm[kE], pW = z[kW] + beta * pm[kW];
    const double pN = z[kN] + beta * pm[kN], pS = z[kS] + beta * pm[kS];
    double a = 0.0;
    a += (hE ? c0 : 0.0) * (hE ? pE : 0.0);
    a += (hW ? c1 : 0.0) * (hW ? pW : 0.0);
    a += (hN ? c2 : 0.0) * (hN ? pN : 0.0);
    a += (hS ? c3 : 0.0) * (hS ? pS : 0.0);
    const double qk = diag[k] * pc - a;
    pk[k] = pc;
    q[k] = qk;
    pq += pc * qk;
    i += di;
    j += dj;
    if (i >= nx) {
      i -= nx;
      ++j;
    }
  }
  __shared__ double s_pq[kCgBlock];
  pq = block_tree(pq, s_pq);
  if (threadIdx.x == 0) part[2 * block] = pq;
}

__global__ __launch_bounds__(kCgBlock) void k_cg_update(
    long long n, const double* __restrict__ diag, const double* __restrict__ P,
    const double* __restrict__ q, double* __restrict__ x, double* __restrict__ r,
    double* __restrict__ z, const double* __restrict__ part_pq, int n_part, double* part,
    RedCounter* red, IterState* cs, const int* gate, double tol, int max_iter) {
  if ((gate && *gate) || cs->done) return;
  const double pq = sum_partials(part_pq, n_part, 0);
  const double alpha = cs->rz / pq;
  const double* __restrict__ pk = P + (long long)(cs->iter & 1) * n;
  double rz = 0.0, rr = 0.0;
  const int block = cg_block();
  const long long stride = (long long)gridDim.x * kCgBlock;
  for (long long k0 = (long long)block * kCgBlock + threadIdx.x; k0 < n; k0 += kCgAhead * stride) {
    double xk[kCgAhead], rk[kCgAhead], p[kCgAhead], qk[kCgAhead], d[kCgAhead];
#pragma unroll
    for (int m = 0; m < kCgAhead; ++m) {
      const long long k = k0 + m * stride < n ? k0 + m * stride : k0;
      xk[m] = x[k];
      rk[m] = r[k];
      p[m] = pk[k];
      qk[m] = q[k];
      d[m] = diag[k];
    }
#pragma unroll
    for (int m = 0; m < kCgAhead; ++m) {
      const long long k = k0 + m * stride;
      if (k >= n) break;
      x[k] = xk[m] + alpha * p[m];
      const double rm = rk[m] - alpha * qk[m];
      const double zm = rm / d[m];
      r[k] = rm;
      z[k] = zm;
      rz += rm * zm;
      rr += rm * rm;
    }
  }
  if (!leave_partials(rz, rr, part, block, red)) return;
  sum_left(part, n_part, rz, rr);
  if (threadIdx.x == 0) {
    const double bb = cs->bb;
    cs->iter += 1;
    cs->dn2_prev = cs->dn2;
    cs->dn2 = rr;
    cs->nrm2 = bb;
    const int bad = !isfinite(rr) || !isfinite(rz);
    const int conv = !bad && rr <= tol * tol * bb;
    cs->bad = bad;
    cs->conv = conv;
    cs->done = bad || conv || cs->iter >= max_iter;
    cs->beta = cs->rz != 0.0 ? rz / cs->rz : 0.0;
    cs->rz = rz;
  }
}

// Small meshes (n <= kCgOneBlockMax): the whole solve in one workgroup of
// 1024 threads, the iterations separated by barriers instead of launches.
// Same iteration as above; a thread keeps its (at most four) cells' vectors and
// coefficients in registers, and only the direction p, which the neighbours
// read, goes through LDS.  The sums are formed per wave (shuffles in a fixed
// pattern) and then over the 16 wave sums in index order, by every thread,
// so every thread holds the same alpha, beta and decision.  What is left are
// the latencies of three barriers and two wave sums: 64^2 6.6 us an iteration (16
// with the vectors in global memory, a step of 39 iterations 0.77 -> 0.41 ms),
// 30 x 50 5 us (7.5).
constexpr int kCgOneBlock = 1024;
constexpr int kCgPer = 4;
constexpr long long kCgOneBlockMax = kCgPer * kCgOneBlock;

__device__ __forceinline__ double wave_sum(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

__global__ __launch_bounds__(kCgOneBlock) void k_cg_solve_one_block(
    int nx, int ny, const double* __restrict__ diag, const double* __restrict__ cE,
    const double* __restrict__ cN, double* __restrict__ x, const double* __restrict__ r,
    const double* __restrict__ z, const double* __restrict__ P, IterState* cs, const int* gate,
    double tol, int max_iter) {
  if ((gate && *gate) || cs->done) return;
  constexpr int nw = kCgOneBlock / 64;
  __shared__ double s_p[kCgOneBlockMax];
  __shared__ double s_pq[nw], s_rz[nw], s_rr[nw];
  if (threadIdx.x < nw)  // waves that the launch leaves out count nothing
    s_pq[threadIdx.x] = s_rz[threadIdx.x] = s_rr[threadIdx.x] = 0.0;
  const int n = nx * ny;
  const int t = threadIdx.x, wv = t >> 6, lane = t & 63;
  int it = cs->iter;
  double beta = cs->beta, rz = cs->rz;
  const double bb = cs->bb;
  double xk[kCgPer], rk[kCgPer], zk[kCgPer], pk[kCgPer], dk[kCgPer];
  double c0[kCgPer], c1[kCgPer], c2[kCgPer], c3[kCgPer];  // E, W, N, S; 0 without a neighbour
#pragma unroll
  for (int m = 0; m < kCgPer; ++m) {
    const int k = t + m * kCgOneBlock;
    const bool ok = k < n;
    const int i = k % nx, j = k / nx;
    xk[m] = ok ? x[k] : 0.0;
    rk[m] = ok ? r[k] : 0.0;
    zk[m] = ok ? z[k] : 0.0;
    pk[m] = ok ? P[(long long)((it + 1) & 1) * n + k] : 0.0;
    dk[m] = ok ? diag[k] : 1.0;
    c0[m] = ok && i + 1 < nx ? cE[k] : 0.0;
    c1[m] = ok && i > 0 ? cE[k - 1] : 0.0;
    c2[m] = ok && j + 1 < ny ? cN[k] : 0.0;
    c3[m] = ok && j > 0 ? cN[k - nx] : 0.0;
  }
  double rr = 0.0;
  int done = 0, conv = 0, bad = 0;
  while (!done) {
#pragma unroll
    for (int m = 0; m < kCgPer; ++m) {
      const int k = t + m * kCgOneBlock;
      pk[m] = zk[m] + beta * pk[m];
      if (k < n) s_p[k] = pk[m];
    }
    __syncthreads();
    double pq = 0.0, qk[kCgPer];
#pragma unroll
    for (int m = 0; m < kCgPer; ++m) {
      const int k = t + m * kCgOneBlock;
      if (k < n) {
        double a = 0.0;
        a += c0[m] * s_p[k + 1 < n ? k + 1 : k];
        a += c1[m] * s_p[k > 0 ? k - 1 : k];
        a += c2[m] * s_p[k + nx < n ? k + nx : k];
        a += c3[m] * s_p[k >= nx ? k - nx : k];
        qk[m] = dk[m] * pk[m] - a;
        pq += pk[m] * qk[m];
      }
    }
    pq = wave_sum(pq);
    if (lane == 0) s_pq[wv] = pq;
    __syncthreads();
    pq = 0.0;
    for (int w = 0; w < nw; ++w) pq += s_pq[w];
    const double alpha = rz / pq;
    double rzn = 0.0, rrn = 0.0;
#pragma unroll
    for (int m = 0; m < kCgPer; ++m) {
      if (t + m * kCgOneBlock < n) {
        xk[m] += alpha * pk[m];
        rk[m] = rk[m] - alpha * qk[m];
        zk[m] = rk[m] / dk[m];
        rzn += rk[m] * zk[m];
        rrn += rk[m] * rk[m];
      }
    }
    rzn = wave_sum(rzn);
    rrn = wave_sum(rrn);
    if (lane == 0) {
      s_rz[wv] = rzn;
      s_rr[wv] = rrn;
    }
    __syncthreads();
    rzn = 0.0;
    rrn = 0.0;
    for (int w = 0; w < nw; ++w) {
      rzn += s_rz[w];
      rrn += s_rr[w];
    }
    it += 1;
    rr = rrn;
    bad = !isfinite(rrn) || !isfinite(rzn);
    conv = !bad && rrn <= tol * tol * bb;
    done = bad || conv || it >= max_iter;
    beta = rz != 0.0 ? rzn / rz : 0.0;
    rz = rzn;
  }
#pragma unroll
  for (int m = 0; m < kCgPer; ++m)
    if (t + m * kCgOneBlock < n) x[t + m * kCgOneBlock] = xk[m];
  if (t == 0) {
    cs->iter = it;
    cs->dn2_prev = 0.0;
    cs->dn2 = rr;
    cs->nrm2 = bb;
    cs->bad = bad;
    cs->conv = conv;
    cs->done = 1;
    cs->beta = beta;
    cs->rz = rz;
  }
}

// phi_c nodal = the cell value at all four nodes.
__global__ void k_cg_to_nodal(long long n, const double* __restrict__ x,
                              double* __restrict__ phi_c, const int* halt) {
  if (*halt) return;
  for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < n;
       k += (long long)gridDim.x * blockDim.x) {
    const double v = x[k];
    reinterpret_cast<double4*>(phi_c)[k] = make_double4(v, v, v, v);
  }
}

hipError_t launch_cg_start(const CgArgs& a, const double* sig_s, const double* phi_post,
                           int max_iter, const int* halt, hipStream_t s) {
  const long long n = (long long)a.nx * a.ny;
  hipLaunchKernelGGL(k_cg_start, dim3(a.n_part), dim3(kCgBlock), 0, s, n, sig_s, phi_post,
                     (const double*)a.diag, a.x, a.r, a.z, a.P + n, a.part_a, a.red, a.cs,
                     max_iter, halt);
  return hipGetLastError();
}

hipError_t launch_dsa_start(const CgArgs& a, const double* sig_s, const double* dnode,
                            int max_iter, hipStream_t s) {
  const long long n = (long long)a.nx * a.ny;
  hipLaunchKernelGGL(k_dsa_start, dim3(a.n_part), dim3(kCgBlock), 0, s, n, sig_s, dnode,
                     (const double*)a.diag, a.x, a.r, a.z, a.P + n, a.part_a, a.red, a.cs,
                     max_iter, a.gate);
  return hipGetLastError();
}

bool cg_one_block(long long n) { return n <= kCgOneBlockMax; }

hipError_t launch_cg_solve_one_block(const CgArgs& a, double tol, int max_iter, hipStream_t s) {
  const long long n = (long long)a.nx * a.ny;
  if (n < 1 || !cg_one_block(n)) return hipErrorInvalidValue;  // more than registers and LDS hold
  const int cells = (int)n;  // below kCgOneBlock: the waves that have cells
  const int threads = cells < kCgOneBlock ? (cells + 63) & ~63 : kCgOneBlock;
  hipLaunchKernelGGL(k_cg_solve_one_block, dim3(1), dim3(threads), 0, s, a.nx, a.ny,
                     (const double*)a.diag, (const double*)a.cE, (const double*)a.cN, a.x,
                     (const double*)a.r, (const double*)a.z, (const double*)a.P, a.cs, a.gate,
                     tol, max_iter);
  return hipGetLastError();
}

hipError_t launch_cg_iteration(const CgArgs& a, double tol, int max_iter, hipStream_t s) {
  const long long n = (long long)a.nx * a.ny;
  if (cg_one_block(n)) return launch_cg_solve_one_block(a, tol, max_iter, s);  // the whole rest
  hipLaunchKernelGGL(k_cg_spmv, dim3(a.n_part), dim3(kCgBlock), 0, s, a.nx, a.ny,
                     (const double*)a.diag, (const double*)a.cE, (const double*)a.cN,
                     (const double*)a.z, a.P, a.q, a.part_a, (const IterState*)a.cs, a.gate);
  hipLaunchKernelGGL(k_cg_update, dim3(a.n_part), dim3(kCgBlock), 0, s, n,
                     (const double*)a.diag, (const double*)a.P, (const double*)a.q, a.x, a.r,
                     a.z, (const double*)a.part_a, a.n_part, a.part_b, a.red, a.cs,
                     a.gate, tol, max_iter);
  return hipGetLastError();
}

hipError_t launch_cg_to_nodal(const CgArgs& a, double* phi_c, const int* halt, hipStream_t s) {
  const long long n = (long long)a.nx * a.ny;
  hipLaunchKernelGGL(k_cg_to_nodal, dim3(a.n_part), dim3(kCgBlock), 0, s, n,
                     (const double*)a.x, phi_c, halt);
  return hipGetLastError();
}

}  // namespace slh
