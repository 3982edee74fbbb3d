// Collided solve of the hybrid step (step 2 of Sec. 2.2): discrete ordinates
// with bilinear discontinuous Galerkin in space, upwind faces, vacuum inflow,
// and a step-averaged time closure sigma_e = sigma_t + tau/(c dt).  One
// transport sweep per direction and source-iteration sweep.
//
// The element equation.  On a cell of size hx x hy with nodal values
// X[kx][ky], in coordinates mirrored so that both direction components are
// positive (a = |Omega_x| / hx, b = |Omega_y| / hy), the element matrix divided
// by the mass matrix is a sum of one-dimensional operators:
//   a T X + b X T^t + sig_e X = S + a nu ux^t + b uy nu^t,
//   T = [[3, 1], [-3, 1]],  nu = (4, -2),
// ux[ky], uy[kx] the upwind traces on the x and y inflow faces (zero on a
// vacuum side).  T has the eigenvalues lambda = 2 +- i sqrt 2 whatever the
// direction, so its left eigenvector l (scaled to l.nu = 1) and right
// eigenvector v (l.v = 1) turn the element's 4x4 system into two complex
// scalar equations.  With the coefficients X1 = l_kx l_ky X (mode lambda,
// lambda), X2 = l_kx conj(l_ky) X (mode lambda, conj lambda), S1 and S2 of the
// source, and l.ux, l.uy of the traces:
//   X1 = c1 (S1 + a ux + b uy),        c1 = 1 / ((a + b) lambda + sig_e),
//   X2 = c2 (S2 + a conj(ux) + b uy),  c2 = 1 / (a lambda + b conj(lambda) + sig_e),
// and the coefficients of the outflow traces, which the next cells take, are
//   ux' = v1 X1 + conj(v1 X2),  uy' = v1 X1 + conj(v1) X2.
// Sources and angular fluxes are kept as these coefficients in each quadrant
// of directions; the reduction returns to nodal values.  A cell and direction
// then takes about 30 FP64 operations and two complex numbers c1, c2 that
// depend on the material alone, where the 4x4 block factorisation took about
// 150 and a table of its inverses 32 numbers per material.
//
// The sweep.  A wave owns a strip of 64 rows along one axis of the mesh (the
// v axis) and walks it along the other (the u axis), lane l one column behind
// lane l - 1: at step t lane l holds cell (u = t - l, v = 64 strip + l).  The
// trace across a u face stays in the lane's registers, the trace across a v
// face moves to the next lane by a lane shift, so a step needs no barrier and
// no LDS exchange.  The strips of a direction are the waves of one workgroup
// (a wave takes several when there are more than 16): the last lane of a strip
// leaves its trace of every column in an LDS row, from which the first lane of
// the next strip takes it, a few columns at a time, once the strip's progress
// word says that they are there.  What bounds the sweep is the chain of nu +
// nv dependent steps on small meshes (0.16 us each, the issue of a step's
// instructions, where a workgroup barrier per diagonal took 0.45 us; 256^2,
// S_8: 264 -> 91 us a sweep, 140^2, S_12: 130 -> 52) and the traffic of the planes
// on large ones; there each wave sweeps four directions, which share the
// sources and leave one plane: the sum of w_m psi_m over them.
//
// Every quadrant has its own copy of the source (and of the material ids) in
// its own order of visits (dg_slot): the cells that a wave holds at one step
// are neighbours in memory; so are they in sigma_e, which is kept by diagonals
// (dg_diag) where there is no table of materials.  Cells outside the mesh take no
// storage: the columns of a strip wrap around (slot row (u + l) mod nu).
#include <algorithm>

#include "slh_common.hpp"

namespace slh {

// 1/a from the hardware reciprocal estimate refined by two Newton steps
// (quadratic convergence from ~2^-26 to full FP64 precision).
__device__ __forceinline__ double recip(double a) {
  double r = __builtin_amdgcn_rcp(a);
  r = fma(fma(-a, r, 1.0), r, r);
  r = fma(fma(-a, r, 1.0), r, r);
  return r;
}

// lambda = 2 + i sqrt 2; l = (l0, l1), v = (v0, v1) as above.  A cell without
// sources and absorption passes a constant trace on times 2 Re(v1 / lambda) = 1.
// In doubles that is 1 + 1.3e-16 with the nearest ones to sqrt 2 and 2.5 sqrt 2, in
// every cell alike, and a path of hundreds of cells adds it up; with the double
// below sqrt 2 it is 1 - 2.7e-17, the least of any neighbours.  (Relative L2 error
// of a sweep against 80-bit arithmetic: 512^2 S_16 of 0.1 per unit length 1.8e-14
// -> 2.4e-15, 300^2 S_4 of 0.01 1.8e-14 -> 5.4e-15.)
constexpr double kSqrt2 = 1.414213562373095;
constexpr double kL0r = 5.0 / 18.0, kL0i = -kSqrt2 / 18.0;
constexpr double kL1r = 1.0 / 18.0, kL1i = -2.0 * kSqrt2 / 18.0;
constexpr double kV0r = 2.0, kV0i = -0.5 * kSqrt2;
constexpr double kV1r = -1.0, kV1i = 3.5355339059327378;

// Coefficients of the mirrored nodal values s<ku><kv> of a cell.
__device__ __forceinline__ void to_modes(double s00, double s01, double s10, double s11,
                                         double2& m1, double2& m2) {
  // the v transform at ku = 0, 1, then the u transform
  const double q0r = kL0r * s00 + kL1r * s01, q0i = kL0i * s00 + kL1i * s01;
  const double q1r = kL0r * s10 + kL1r * s11, q1i = kL0i * s10 + kL1i * s11;
  const double rr = kL0r * q0r + kL1r * q1r, ii = kL0i * q0i + kL1i * q1i;
  const double ri = kL0r * q0i + kL1r * q1i, ir = kL0i * q0r + kL1i * q1r;
  m1 = make_double2(rr - ii, ir + ri);
  m2 = make_double2(rr + ii, ir - ri);
}

// Mirrored nodal values s[2 ku + kv] of coefficients.
__device__ __forceinline__ void from_modes(double2 m1, double2 m2, double s[4]) {
  constexpr double vr[2] = {kV0r, kV1r}, vi[2] = {kV0i, kV1i};
#pragma unroll
  for (int kv = 0; kv < 2; ++kv) {
    // v_kv m1 + conj(v_kv) m2
    const double pr = vr[kv] * (m1.x + m2.x) - vi[kv] * (m1.y - m2.y);
    const double pi = vr[kv] * (m1.y + m2.y) + vi[kv] * (m1.x - m2.x);
#pragma unroll
    for (int ku = 0; ku < 2; ++ku) s[2 * ku + kv] = 2.0 * (vr[ku] * pr - vi[ku] * pi);
  }
}

// Index (node kx + 2 ky) of the mirrored node (ku, kv) of quadrant q (bit 0:
// Omega_x < 0, bit 1: Omega_y < 0).
__device__ __forceinline__ int quad_node(int q, int swap, int ku, int kv) {
  return ((swap ? kv : ku) ^ (q & 1)) + 2 * ((swap ? ku : kv) ^ (q >> 1));
}

// Start of a step's source iteration: phi_c = 0, the iteration state reset
// (block 0), the source of the first iterate S = sigma_s/(4 pi) (phi_c +
// phi_post) with phi_c = 0, one value at the four nodes of a cell, in every
// quadrant (later iterates get theirs from the flux reduction), and with
// reflective sides the buffer of reflected traces that the first sweep reads
// set to zero.
__global__ void k_si_start(DgArgs g, double* __restrict__ bnd0, long long n_bnd, int si_max) {
  DevState* st = g.st;
  if (st->halt) return;
  const int n = g.nx * g.ny;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->si.iter = 0;
    st->si.conv = si_max == 0 ? 1 : 0;
    st->si.done = si_max == 0 ? 1 : 0;
    st->si.bad = 0;
    st->si.dn2 = 0.0;
    st->si.dn2_prev = 0.0;
    st->si.nrm2 = 0.0;
    st->dsa_unconv = 0;
    st->dsa_corrections = 0;
    st->dsa_iter_total = 0;
    st->dsa_iter_max = 0;
  }
  const double inv4pi = 0.25 / M_PI;
  const long long i0 = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long str = (long long)gridDim.x * blockDim.x;
  for (long long i = i0; i < n; i += str) {
    const double ssc = g.sig_s[i] * inv4pi;
    const double v = ssc * (0.0 + g.phi_post[i]);
    const int ci = (int)i % g.nx, cj = (int)i / g.nx;
    reinterpret_cast<double4*>(g.phi_c)[i] = make_double4(0.0, 0.0, 0.0, 0.0);
    if (!g.src) continue;  // no sweep in this solver
    double2 m1, m2;
    to_modes(v, v, v, v, m1, m2);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      double2* S = reinterpret_cast<double2*>(g.src) + (long long)q * 2 * n;
      const int pos = dg_slot(g, q, ci, cj);
      S[2 * pos] = m1;
      S[2 * pos + 1] = m2;
    }
  }
  for (long long k = i0; k < n_bnd; k += str) bnd0[k] = 0.0;
}

// The LDS row of traces has room for the columns that a strip's first and
// last lanes touch before and after the mesh.
constexpr int kDgAhead = 8;  // the most columns a strip takes at a time
constexpr int kDgSplit = 4;  // directions per wave on large meshes
constexpr int kDgFront = 63, kDgPad = kDgFront + kDgAhead;

// The value of the lane below, `first` in lane 0.
__device__ __forceinline__ double lane_shift(double first, double v) {
  const long long o = __double_as_longlong(first), s = __double_as_longlong(v);
  constexpr int kWaveShr1 = 0x138;
  const int lo = __builtin_amdgcn_update_dpp((int)o, (int)s, kWaveShr1, 0xf, 0xf, false);
  const int hi =
      __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(s >> 32), kWaveShr1, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Buffer loads and stores of the sweep: a lane's constant byte offset plus the
// step's (uniform) one, so that an access takes no address arithmetic; an
// access past the buffer's length reads zero or is dropped, so that lanes
// without a cell store without a branch (a conditional store would make the
// compiler's wait for a load drain the younger loads).
using u32x4 = unsigned int __attribute__((ext_vector_type(4)));
constexpr int kBufferFlags = 0x00020000;  // raw 32-bit data, no swizzle
constexpr int kNoCell = 0x40000000;       // beyond any buffer of the sweep

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, kBufferFlags);
}
__device__ __forceinline__ double2 buffer_load2(__amdgpu_buffer_rsrc_t r, int lane_off, int off) {
  return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, off, 0));
}
// NT: non-temporal (planes that do not fit the caches, read once)
template <bool NT>
__device__ __forceinline__ void buffer_store2(__amdgpu_buffer_rsrc_t r, int lane_off, int off,
                                              double x, double y) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, make_double2(x, y)), r,
                                         lane_off, off, NT ? 2 : 0);
}

// c1 and c2 of a material: 1/z by Smith's division (the real part, at least
// 2 (a + b), is never below the imaginary part in size, so nothing
// overflows that the element matrix itself would not).
__device__ __forceinline__ void mode_inverse(double a, double b, double se, double2& c1,
                                             double2& c2) {
  const double dr = 2.0 * (a + b) + se;
  const double ir = recip(dr);
  const double d1 = kSqrt2 * (a + b), d2 = kSqrt2 * (a - b);
  const double r1 = d1 * ir, r2 = d2 * ir;
  const double e1 = recip(fma(d1, r1, dr)), e2 = recip(fma(d2, r2, dr));
  c1 = make_double2(e1, -r1 * e1);
  c2 = make_double2(e2, -r2 * e2);
}

// One workgroup sweeps the PER directions of one group of a quadrant, one
// wave per strip (see the head of this file).  TABLE: c1, c2 of every material
// in LDS (n_mat + 1 rows per direction, the last one zero, for lanes that have
// not reached their first column); else they are computed per cell.  AHEAD:
// columns whose sources are in flight; a strip takes at most eight at a time
// from the one before.
//
// A step of a wave issues about 50 instructions (28 FP64 per direction); one
// wave per SIMD issues one every four cycles or so, so on small meshes the
// instruction count of a step is its time, and everything that can be is kept
// out of it: addresses are uniform offsets, the lanes without a cell neither
// branch nor store, the traces carry no factor, and with one direction per
// wave the reduction applies the weight.
//
// With four directions per wave (large meshes, where the planes' traffic
// counts: a plane then holds the sum of four directions) the strips of a group
// are spread over several workgroups of four strips, one wave per SIMD.  The
// trace rows between workgroups go through global memory in tagged words: each
// 8-byte word holds half a double and the sweep's tag, so that a word that
// carries the tag is there, whatever the order in which words arrive.  A
// workgroup takes its task by a ticket of its class (the blocks that share an
// XCD), first strips first: it waits only for tasks of smaller tickets, which
// running workgroups hold, so every wait ends however the blocks are
// dispatched.
template <int PER, bool TABLE, bool REFL, int AHEAD, int THREADS>
__global__ __launch_bounds__(THREADS) void k_dg_sweep(DgArgs g) {
  if (g.st->si.done) return;  // the whole workgroup: no barrier is left pending
  constexpr bool SPLIT = PER == kDgSplit;
  static_assert(!SPLIT || 2 * PER * AHEAD == 64, "a lane per double of a block of columns");
  extern __shared__ double smem[];
  const int nu = g.nu, nv = g.nv, n = g.nx * g.ny;
  // the workgroups of a quadrant on two XCDs, so that they share its sources
  // in the L2 (1024^2, S_16: all four quadrants' sources through every L2
  // otherwise)
  const bool pairs = (g.n_grp & 1) == 0;
  const int n_all = 4 * g.n_grp;
  int task = (int)blockIdx.x, blk = 0;
  if (SPLIT) {
    int* const s_ticket = reinterpret_cast<int*>(smem);
    const int cls = (int)blockIdx.x & 7;
    if (threadIdx.x == 0)
      *s_ticket = (int)__hip_atomic_fetch_add(&g.st->ticket[cls], 1u, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int ticket = __builtin_amdgcn_readfirstlane(*s_ticket);
    __syncthreads();  // the word belongs to the trace row
    const int n_cls = (n_all - cls + 7) / 8;  // the class's groups: cls, cls + 8, ...
    blk = n_cls > 0 ? ticket / n_cls : g.n_blk;
    if (blk >= g.n_blk) return;
    task = cls + 8 * (ticket - blk * n_cls);
  }
  const int q = pairs ? (task & 7) >> 1 : task / g.n_grp;
  const int grp = pairs ? (task >> 3) * 2 + (task & 1) : task - q * g.n_grp;
  const int m0 = q * g.n_quad + grp * PER;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const int n_waves = blockDim.x >> 6;
  // LDS: row of v-face traces [nu + kDgPad][PER] and room for idle lanes' traces |
  // reflective sides: traces of the u side [PER][rows] | table [n_mat + 1][PER] of
  // c1, c2 (SPLIT: 1/|z1|^2, 1/|z2|^2 for c = conj(z)/|z|^2, half the space, and
  // [n_mat + 1] sigma_e) | progress word of each strip
  const int n_row = TABLE ? g.n_mat + 1 : 0;
  const int n_col = nu + kDgPad;
  const int n_xf = SPLIT ? 64 * n_waves : nv;  // rows of the workgroup
  double2* const yf = reinterpret_cast<double2*>(smem);
  double2* const idle = yf + PER * n_col;
  double2* const xf = idle + PER * 64;
  double2* const tab = xf + (REFL ? PER * n_xf : 0);
  double* const tab_se = reinterpret_cast<double*>(tab + (SPLIT ? PER : 2 * PER) * n_row);
  int* const prog = reinterpret_cast<int*>(tab_se + (SPLIT ? n_row : 0));

  double a[PER], b[PER], w[PER];
  int md[PER];
#pragma unroll
  for (int d = 0; d < PER; ++d) {
    // a group past the end of its quadrant repeats the last direction with weight 0
    const int m = m0 + d < (q + 1) * g.n_quad ? m0 + d : (q + 1) * g.n_quad - 1;
    md[d] = m;
    const double x = fabs(g.dir[3 * m]) / g.hx, y = fabs(g.dir[3 * m + 1]) / g.hy;
    a[d] = g.swap ? y : x;
    b[d] = g.swap ? x : y;
    w[d] = m == m0 + d ? g.dir[3 * m + 2] : 0.0;
  }
  double dr0[PER], d1[PER], d2[PER];  // z1 = dr0 + sig_e + i d1, z2 = dr0 + sig_e + i d2
#pragma unroll
  for (int d = 0; d < PER; ++d) {
    dr0[d] = 2.0 * (a[d] + b[d]);
    d1[d] = kSqrt2 * (a[d] + b[d]);
    d2[d] = kSqrt2 * (a[d] - b[d]);
  }
  if (TABLE) {
    for (int k = threadIdx.x; k < n_row; k += blockDim.x) {
      const double se = k < g.n_mat ? g.sig_e_mat[k] : 0.0;
      if (SPLIT) tab_se[k] = se;
#pragma unroll
      for (int d = 0; d < PER; ++d) {
        double2 c1 = make_double2(0.0, 0.0), c2 = c1;
        if (SPLIT) {
          const double dr = dr0[d] + se;
          if (k < g.n_mat)
            c1 = make_double2(recip(fma(dr, dr, d1[d] * d1[d])), recip(fma(dr, dr, d2[d] * d2[d])));
          tab[PER * k + d] = c1;
        } else {
          if (k < g.n_mat) mode_inverse(a[d], b[d], se, c1, c2);
          tab[2 * k] = c1;
          tab[2 * k + 1] = c2;
        }
      }
    }
  }
  // reflective sides: the inflow is the outflow of the mirrored direction in
  // the previous iteration, at the same place along the side
  const int it = REFL ? g.st->si.iter : 0;
  const bool unegative = (q & (g.swap ? 2 : 1)) != 0, vnegative = (q & (g.swap ? 1 : 2)) != 0;
  const int ubc = g.swap ? g.bc >> 2 : g.bc, vbc = g.swap ? g.bc : g.bc >> 2;
  const bool u_in = REFL && (ubc & (unegative ? 2 : 1));
  const bool u_out = REFL && (ubc & (unegative ? 1 : 2));
  const bool v_in = REFL && (vbc & (vnegative ? 2 : 1));
  const bool v_out = REFL && (vbc & (vnegative ? 1 : 2));
  const int* const ru = g.swap ? g.refl_y : g.refl_x;
  const int* const rv = g.swap ? g.refl_x : g.refl_y;
  const double2* const b_in =
      REFL ? reinterpret_cast<const double2*>(g.bnd) + (size_t)((it + 1) & 1) * g.n_dir * (nu + nv)
           : nullptr;
  double2* const b_out =
      REFL ? reinterpret_cast<double2*>(g.bnd) + (size_t)(it & 1) * g.n_dir * (nu + nv) : nullptr;
#pragma unroll
  for (int d = 0; d < PER; ++d)
    for (int k = threadIdx.x; k < n_col; k += blockDim.x) {
      const int u = k - kDgFront;
      yf[k * PER + d] = REFL && v_in && u >= 0 && u < nu
                              ? b_in[(size_t)rv[md[d]] * (nu + nv) + nv + u]
                              : make_double2(0.0, 0.0);
    }
  for (int k = threadIdx.x; k < (SPLIT ? n_waves : g.n_strips); k += blockDim.x) prog[k] = 0;
  __syncthreads();

  const unsigned bytes = 32u * (unsigned)n;  // of a source or plane (n < 2^23)
  const __amdgpu_buffer_rsrc_t src =
      buffer_of(reinterpret_cast<const double2*>(g.src) + (size_t)q * 2 * n, bytes);
  const __amdgpu_buffer_rsrc_t out = buffer_of(
      reinterpret_cast<double2*>(g.psi) + (size_t)(q * g.n_grp + grp) * 2 * n, bytes);
  const __amdgpu_buffer_rsrc_t ids =
      TABLE ? buffer_of(g.mat_off + (size_t)q * n, 4u * n)
            : buffer_of(g.sig_e + (unegative != vnegative ? (size_t)n : 0), 8u * n);
  constexpr double kap = kV1i;  // v1 = -1 + i kap

  // SPLIT: this lane's double of a block of columns, two tagged words
  unsigned long long *take = nullptr, *give = nullptr;  // at column 0
  const unsigned long long tag = SPLIT ? (unsigned long long)g.st->sweep_tag << 32 : 0ull;
  const int h_d = lane / (2 * AHEAD), h_k = lane / 2 % AHEAD;  // direction, column in the block
  double* const h_row = reinterpret_cast<double*>(yf) + 2 * (kDgFront * PER + h_d) + (lane & 1);
  if (SPLIT) {
    // [group][boundary][column][direction][part][word]
    const size_t row = (size_t)nu * (4 * PER);
    unsigned long long* const h =
        g.hand + (size_t)(q * g.n_grp + grp) * (g.n_blk - 1) * row + 4 * h_d + 2 * (lane & 1);
    if (wave == 0 && blk > 0) take = h + (blk - 1) * row;
    if (wave == n_waves - 1 && blk < g.n_blk - 1) give = h + blk * row;
  }

  const int s0 = SPLIT ? blk * n_waves : 0;  // the workgroup's first strip
  const int s_end = SPLIT && s0 + n_waves < g.n_strips ? s0 + n_waves : g.n_strips;
  for (int s = s0 + wave; s < s_end; s += n_waves) {
    const int rows = nv - 64 * s < 64 ? nv - 64 * s : 64;
    const int lr = lane < rows ? lane : rows - 1;  // a real row for every lane's loads
    const int first = lane < rows ? lane : 1 << 30;  // the step of the lane's first column
    const int steps = nu + rows - 1;
    const bool last = s + 1 == g.n_strips;
    // The lane whose v traces go to the LDS row, for the next strip or for a
    // reflective side; the others write to a word of their own (masking them
    // off would split the step's schedule).
    const bool leaves = last ? (v_out && lane == rows - 1) : lane == 63;
    double2* leave_at = leaves ? yf + PER * (kDgFront - lane) : idle + PER * lane;
    const int leave_by = leaves ? PER : 0;
    // without a table, sigma_e by diagonals (dg_diag): a step's cells lie on one,
    // the next step's on the next (negative u: on the one before)
    int e_lane = 0, e_off = 0, e_step = 0;
    if (!TABLE) {
      const int v = 64 * s + lr;
      e_lane = 8 * (vnegative ? nv - 1 - v : v);
      e_step = unegative ? -8 * nv : 8 * nv;
      const int u0 = unegative ? nu - 1 : 0, v0 = vnegative ? nv - 1 - 64 * s : 64 * s;
      e_off = 8 * nv * dg_diag_row(nu, unegative != vnegative, u0, v0);
    }
    double2 r1[AHEAD], r2[AHEAD];  // sources in flight
    int rk[AHEAD];                 // byte offsets of the materials' table rows
    double re[AHEAD];              // sigma_e
    int ro[AHEAD];                 // byte offset of the step's slot row
    const int row_bytes = 32 * rows, o_begin = 32 * 64 * s * nu, o_end = o_begin + nu * row_bytes;
    int f_off = o_begin;  // the next step's to fetch
    auto fetch = [&](int k) __attribute__((always_inline)) {
      r1[k] = buffer_load2(src, 32 * lr, f_off);
      r2[k] = buffer_load2(src, 32 * lr + 16, f_off);
      if (TABLE) {
        rk[k] = (int)__builtin_amdgcn_raw_buffer_load_b32(ids, 4 * lr, f_off >> 3, 0);
      } else {
        re[k] = __builtin_bit_cast(double,
                                   __builtin_amdgcn_raw_buffer_load_b64(ids, e_lane, e_off, 0));
        e_off += e_step;
        e_off += e_off < 0 ? 8 * n : 0;
        e_off -= e_off >= 8 * n ? 8 * n : 0;
      }
      ro[k] = f_off;
      f_off += row_bytes;
      if (f_off == o_end) f_off = o_begin;
    };
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) fetch(k);
    // traces of the lane's cell: u face of its previous column, v face
    double uxr[PER], uxi[PER], uyr[PER], uyi[PER];
    double2 ui[PER];  // reflected inflow on the u side
#pragma unroll
    for (int d = 0; d < PER; ++d) {
      uxr[d] = uxi[d] = uyr[d] = uyi[d] = 0.0;
      if (REFL)
        ui[d] = u_in ? b_in[(size_t)ru[md[d]] * (nu + nv) + 64 * s + lr] : make_double2(0.0, 0.0);
    }
    // the next step: whether the lane has a cell, and with a table its c1 and
    // c2, read a step early
    bool next_act = false;
    double2 n1[PER], n2[PER];
    double n_se = 0.0;
    auto look_up = [&](int t, int k) __attribute__((always_inline)) {
      next_act = (unsigned)(t - first) < (unsigned)nu;
      if (!TABLE) return;
      const int off = next_act ? rk[k] : 32 * g.n_mat;
      const double2* const row = reinterpret_cast<const double2*>(
          reinterpret_cast<const char*>(tab) + (SPLIT ? PER / 2 : 1) * off);
      if (SPLIT) {
        n_se = *reinterpret_cast<const double*>(reinterpret_cast<const char*>(tab_se) + (off >> 2));
#pragma unroll
        for (int d = 0; d < PER; ++d) n1[d] = row[d];
      } else {
        n1[0] = row[0];
        n2[0] = row[1];
      }
    };
    // every source has arrived: the loop's waits then count its own accesses
    // only, and leave the younger ones in flight (vmcnt 0)
    __builtin_amdgcn_s_waitcnt(0x0f70);
    look_up(0, 0);
    // the words of the block of columns at t0 (a column past the mesh: the last)
    unsigned long long in0 = 0ull, in1 = 0ull;
    auto peek = [&](int t0) __attribute__((always_inline)) {
      const int u = t0 + h_k < nu ? t0 + h_k : nu - 1;
      in0 = __hip_atomic_load(take + (size_t)u * (4 * PER), __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_AGENT);
      in1 = __hip_atomic_load(take + (size_t)u * (4 * PER) + 1, __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_AGENT);
    };
    if (SPLIT && take) peek(0);
    // After the traces of all steps before t have been left (columns before
    // t - 63): for the next workgroup, its last eight columns; for the next
    // strip, how many there are.
    auto publish = [&](int t) __attribute__((always_inline)) {
      if (SPLIT && give) {
        const int u = t - 63 - AHEAD + h_k;
        if (u >= 0 && u < nu) {
          const unsigned long long v = (unsigned long long)__double_as_longlong(h_row[2 * PER * u]);
          __hip_atomic_store(give + (size_t)u * (4 * PER), tag | v >> 32, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(give + (size_t)u * (4 * PER) + 1, tag | (v & 0xffffffffull),
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      } else if (!last) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        if (lane == 0)
          __hip_atomic_store(&prog[s - s0], t - 63, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    };
    for (int t0 = 0; t0 < steps; t0 += AHEAD) {
      if (SPLIT && take) {
        if (t0 < nu) {
          // the workgroup before has left the traces of these columns; those of
          // the next block are looked at a block early
          while (!__all((in0 >> 32 << 32) == tag && (in1 >> 32 << 32) == tag)) {
            __builtin_amdgcn_s_sleep(1);
            peek(t0);
          }
          if (t0 + h_k < nu)
            h_row[2 * PER * (t0 + h_k)] = __longlong_as_double((long long)(in0 << 32 |
                                                                      (in1 & 0xffffffffull)));
          peek(t0 + AHEAD < nu ? t0 + AHEAD : t0);
        }
      } else if (s > s0 && t0 < nu) {
        // the strip before has left the traces of these columns
        const int need = t0 + AHEAD < nu ? t0 + AHEAD : nu;
        while (__hip_atomic_load(&prog[s - s0 - 1], __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP) < need)
          __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
      }
      // the first lane's v trace of the next step, read a step early too
      const double2* const yin = yf + PER * (kDgFront + (t0 < nu ? t0 : nu));
      double2 y0[PER], y1[PER];
#pragma unroll
      for (int d = 0; d < PER; ++d) y1[d] = yin[d];
#pragma unroll
      for (int k = 0; k < AHEAD; ++k) {
        const bool act = next_act;
        double2 c1[PER], c2[PER];
#pragma unroll
        for (int d = 0; d < PER; ++d) {
          if (TABLE && SPLIT) {
            const double dr = dr0[d] + n_se;
            c1[d] = make_double2(dr * n1[d].x, -d1[d] * n1[d].x);
            c2[d] = make_double2(dr * n1[d].y, -d2[d] * n1[d].y);
          } else if (TABLE) {
            c1[d] = n1[d];
            c2[d] = n2[d];
          } else {
            mode_inverse(a[d], b[d], re[k], c1[d], c2[d]);
            // no flux before the lane's first column
            c1[d] = make_double2(act ? c1[d].x : 0.0, act ? c1[d].y : 0.0);
            c2[d] = make_double2(act ? c2[d].x : 0.0, act ? c2[d].y : 0.0);
          }
        }
        look_up(t0 + k + 1, (k + 1) % AHEAD);
#pragma unroll
        for (int d = 0; d < PER; ++d) {
          y0[d] = y1[d];
          if (k + 1 < AHEAD) y1[d] = yin[PER * (k + 1) + d];
        }
        // the reads for the next step stay ahead of this step's arithmetic
        __builtin_amdgcn_sched_barrier(0);
        const double2 S1 = r1[k], S2 = r2[k];
        double2 acc1, acc2;
#pragma unroll
        for (int d = 0; d < PER; ++d) {
          const double yr = lane_shift(y0[d].x, uyr[d]);
          const double yi = lane_shift(y0[d].y, uyi[d]);
          if (REFL && u_in && t0 + k < rows) {  // uniform: some lane's first column
            const bool now = t0 + k == lane;
            uxr[d] = now ? ui[d].x : uxr[d];
            uxi[d] = now ? ui[d].y : uxi[d];
          }
          const double sr = fma(a[d], uxr[d], b[d] * yr);
          const double t1r = S1.x + sr, t1i = fma(a[d], uxi[d], fma(b[d], yi, S1.y));
          const double t2r = S2.x + sr, t2i = fma(-a[d], uxi[d], fma(b[d], yi, S2.y));
          const double X1r = c1[d].x * t1r - c1[d].y * t1i, X1i = c1[d].x * t1i + c1[d].y * t1r;
          const double X2r = c2[d].x * t2r - c2[d].y * t2i, X2i = c2[d].x * t2i + c2[d].y * t2r;
          const double Pr = X1r + X2r, Pi = X1i + X2i, Qr = X1r - X2r, Qi = X1i - X2i;
          uxr[d] = fma(-kap, Pi, -Pr);
          uxi[d] = fma(kap, Qr, -Qi);
          uyr[d] = fma(-kap, Qi, -Pr);
          uyi[d] = fma(kap, Qr, -Pi);
          if (PER == 1) {  // the reduction applies the weight
            acc1 = make_double2(X1r, X1i);
            acc2 = make_double2(X2r, X2i);
          } else if (d == 0) {
            acc1 = make_double2(w[d] * X1r, w[d] * X1i);
            acc2 = make_double2(w[d] * X2r, w[d] * X2i);
          } else {
            acc1.x += w[d] * X1r;
            acc1.y += w[d] * X1i;
            acc2.x += w[d] * X2r;
            acc2.y += w[d] * X2i;
          }
        }
        const int lane_off = act ? 32 * lane : kNoCell;
        buffer_store2<SPLIT>(out, lane_off, ro[k], acc1.x, acc1.y);
        buffer_store2<SPLIT>(out, lane_off + 16, ro[k], acc2.x, acc2.y);
#pragma unroll
        for (int d = 0; d < PER; ++d) leave_at[d] = make_double2(uyr[d], uyi[d]);
        leave_at += leave_by;
        if (REFL && u_out && t0 + k >= nu - 1) {  // uniform: some lane's last column
          if (t0 + k - first == nu - 1) {
#pragma unroll
            for (int d = 0; d < PER; ++d)
              xf[d * n_xf + 64 * (s - s0) + lane] = make_double2(uxr[d], uxi[d]);
          }
        }
        fetch(k);  // after the last use of the stage's registers
      }
      publish(t0 + AHEAD);
    }
  }
  if (REFL) {  // the outflow traces on reflective sides, for the mirrored directions
    __syncthreads();
#pragma unroll
    for (int d = 0; d < PER; ++d) {
      double2* const o = b_out + (size_t)md[d] * (nu + nv);
      if (u_out)
        for (int k = threadIdx.x; k < n_xf && 64 * s0 + k < nv; k += blockDim.x)
          o[64 * s0 + k] = xf[d * n_xf + k];
      if (v_out && s_end == g.n_strips)
        for (int k = threadIdx.x; k < nu; k += blockDim.x)
          o[nv + k] = yf[PER * (kDgFront + k) + d];
    }
  }
}

// A mesh of one row (nv = 1): its cells form a chain only through the u traces,
// and a cell maps its inflow trace to its outflow trace by ux' = A ux + B with
//   A = a (v1 c1 + conj(v1 c2)),
//   B = v1 c1 (S1 + b uy) + conj(v1 c2 (S2 + b uy)),
// since conj(X2) is linear in ux.  Such maps compose associatively, so a
// workgroup per direction finds the inflow traces of all cells by a prefix scan
// of the maps, a thread taking `per` successive cells (one up to 1024), where
// the strips' walk takes a step per cell (S_4 with reflective sides: 5.4 us a sweep
// of 400 cells, 7.4 of 1000, launch and memory latency for the most part; the walk
// took 19 us for 80).
constexpr int kRowWaves = 16;

struct TraceMap {
  double ar, ai, br, bi;
};
// the map `second` after the map `first`
__device__ __forceinline__ TraceMap after(const TraceMap& first, const TraceMap& second) {
  TraceMap t;
  t.ar = second.ar * first.ar - second.ai * first.ai;
  t.ai = second.ar * first.ai + second.ai * first.ar;
  t.br = fma(second.ar, first.br, fma(-second.ai, first.bi, second.br));
  t.bi = fma(second.ar, first.bi, fma(second.ai, first.br, second.bi));
  return t;
}
__device__ __forceinline__ TraceMap shuffle_up(const TraceMap& m, int off) {
  return {__shfl_up(m.ar, off), __shfl_up(m.ai, off), __shfl_up(m.br, off),
          __shfl_up(m.bi, off)};
}
__device__ __forceinline__ double2 apply(const TraceMap& m, double2 x) {
  return make_double2(fma(m.ar, x.x, fma(-m.ai, x.y, m.br)), fma(m.ar, x.y, fma(m.ai, x.x, m.bi)));
}

__device__ __forceinline__ double2 times(double2 p, double2 r) {
  return make_double2(p.x * r.x - p.y * r.y, p.x * r.y + p.y * r.x);
}
// v1 X1 + conj(v1 X2)
__device__ __forceinline__ double2 trace_of(double2 X1, double2 X2) {
  return make_double2(fma(-kV1i, X1.y + X2.y, -(X1.x + X2.x)),
                      fma(kV1i, X1.x - X2.x, -(X1.y - X2.y)));
}

template <bool REFL>
__global__ __launch_bounds__(64 * kRowWaves) void k_dg_sweep_row(DgArgs g) {
  if (g.st->si.done) return;
  __shared__ TraceMap s_map[kRowWaves];  // of each wave's cells
  constexpr double kap = kV1i;           // v1 = -1 + i kap
  const int nu = g.nu, q = (int)blockIdx.x / g.n_grp;
  const int m = q * g.n_quad + ((int)blockIdx.x - q * g.n_grp);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double x = fabs(g.dir[3 * m]) / g.hx, y = fabs(g.dir[3 * m + 1]) / g.hy;
  const double a = g.swap ? y : x, b = g.swap ? x : y;
  // reflective sides as in k_dg_sweep
  const bool back = (q & (g.swap ? 2 : 1)) != 0, vnegative = (q & (g.swap ? 1 : 2)) != 0;
  const int ubc = g.swap ? g.bc >> 2 : g.bc, vbc = g.swap ? g.bc : g.bc >> 2;
  const bool u_in = REFL && (ubc & (back ? 2 : 1)), u_out = REFL && (ubc & (back ? 1 : 2));
  const bool v_in = REFL && (vbc & (vnegative ? 2 : 1));
  const bool v_out = REFL && (vbc & (vnegative ? 1 : 2));
  const int it = REFL ? g.st->si.iter : 0;
  const size_t n_tr = (size_t)nu + 1;  // traces of a direction: the u face's, then the v faces'
  const double2* b_u = nullptr;
  const double2* b_v = nullptr;
  double2* b_out = nullptr;
  if (REFL) {
    const double2* const b_in =
        reinterpret_cast<const double2*>(g.bnd) + (size_t)((it + 1) & 1) * g.n_dir * n_tr;
    b_u = b_in + (g.swap ? g.refl_y : g.refl_x)[m] * n_tr;
    b_v = b_in + (g.swap ? g.refl_x : g.refl_y)[m] * n_tr + 1;
    b_out = reinterpret_cast<double2*>(g.bnd) + ((size_t)(it & 1) * g.n_dir + m) * n_tr;
  }
  const double2* const src = reinterpret_cast<const double2*>(g.src) + (size_t)q * 2 * nu;
  double2* const out =
      reinterpret_cast<double2*>(g.psi) + (size_t)blockIdx.x * 2 * nu;

  struct Cell {
    double2 c1, c2, t1, t2;  // t = S + b uy
  };
  auto load = [&](int u) {
    double se;
    if (g.mat_off)
      se = g.sig_e_mat[g.mat_off[(size_t)q * nu + u] >> 5];
    else
      se = g.sig_e[back ? nu - 1 - u : u];
    Cell c;
    c.t1 = src[2 * u];
    c.t2 = src[2 * u + 1];
    if (v_in) {
      const double2 uy = b_v[u];
      c.t1.x = fma(b, uy.x, c.t1.x);
      c.t1.y = fma(b, uy.y, c.t1.y);
      c.t2.x = fma(b, uy.x, c.t2.x);
      c.t2.y = fma(b, uy.y, c.t2.y);
    }
    mode_inverse(a, b, se, c.c1, c.c2);
    return c;
  };

  const int per = (nu + (int)blockDim.x - 1) / (int)blockDim.x;
  const int u0 = (int)threadIdx.x * per, u1 = u0 + per < nu ? u0 + per : nu;
  const double2 ux0 = u_in ? b_u[0] : make_double2(0.0, 0.0);
  TraceMap map = {1.0, 0.0, 0.0, 0.0};  // of the thread's cells
  Cell mine;                            // its first cell
  for (int u = u0; u < u1; ++u) {
    const Cell c = load(u);
    if (u == u0) mine = c;
    const double2 A = trace_of(c.c1, c.c2), B = trace_of(times(c.c1, c.t1), times(c.c2, c.t2));
    map = after(map, {a * A.x, a * A.y, B.x, B.y});
  }
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const TraceMap before = shuffle_up(map, off), both = after(before, map);
    if (lane >= off) map = both;
  }
  if (lane == 63) s_map[wave] = map;
  __syncthreads();
  double2 ux = ux0;  // into the wave's first cell, then into the thread's
  for (int k = 0; k < wave; ++k) ux = apply(s_map[k], ux);
  const TraceMap before = shuffle_up(map, 1);
  if (lane > 0) ux = apply(before, ux);
  for (int u = u0; u < u1; ++u) {
    const Cell c = u == u0 ? mine : load(u);
    const double2 X1 = times(c.c1, make_double2(fma(a, ux.x, c.t1.x), fma(a, ux.y, c.t1.y)));
    const double2 X2 = times(c.c2, make_double2(fma(a, ux.x, c.t2.x), fma(-a, ux.y, c.t2.y)));
    ux = trace_of(X1, X2);
    out[2 * u] = X1;  // the reduction applies the weight
    out[2 * u + 1] = X2;
    if (v_out)
      b_out[1 + u] = make_double2(fma(-kap, X1.y - X2.y, -(X1.x + X2.x)),
                                  fma(kap, X1.x - X2.x, -(X1.y + X2.y)));
    if (u_out && u == nu - 1) b_out[0] = ux;
  }
}

// ---------------------------------------------------------------------------
// Plan of the sweep
// ---------------------------------------------------------------------------
constexpr int kDgMaxWaves = 16;
constexpr int kDgSplitWaves = 4;  // strips of a workgroup with four directions per wave

size_t dg_sweep_lds_bytes(const DgPlan& p, int n_mat, bool refl) {
  const size_t rows = n_mat > 0 ? (size_t)n_mat + 1 : 0;
  const bool split = p.per == kDgSplit;
  return sizeof(double2) * (size_t)p.per *
             (p.nu + kDgPad + 64 + (refl ? (split ? 64 * p.n_waves : p.nv) : 0) +
              (split ? 1 : 2) * rows) +
         sizeof(double) * (split ? rows : 0) +
         sizeof(int) * (size_t)(split ? p.n_waves : p.n_strips);
}

size_t dg_hand_words(const DgPlan& p) {
  return (size_t)4 * p.n_grp * (p.n_blk - 1) * p.nu * 4 * p.per;
}

size_t dg_plane_bytes(const DgPlan& p, long long cells) {
  return (size_t)4 * p.n_grp * cells * 32 + dg_hand_words(p) * 8;
}

DgPlan dg_plan(int nx, int ny, int n_dir, long long n_mat, bool squares, bool refl, size_t lds) {
  DgPlan p;
  // wave-steps of a direction with the lanes along y or along x
  auto cost = [](int nu, int nv) {
    return (long long)((nv + 63) / 64) * (nu + (nv < 64 ? nv : 64) - 1);
  };
  auto axis = [&](int swap) {
    p.swap = swap;
    p.nu = swap ? ny : nx;
    p.nv = swap ? nx : ny;
    p.n_strips = (p.nv + 63) / 64;
  };
  const int cheap = cost(ny, nx) < cost(nx, ny) || nx == 1 ? 1 : 0;  // one column: as one row
  const long long nc = (long long)nx * ny;
  auto fill = [&](int per) {
    p.per = per;
    const int most = per == kDgSplit ? kDgSplitWaves : kDgMaxWaves;
    p.n_waves = p.n_strips < most ? p.n_strips : most;
    p.n_blk = per == kDgSplit ? (p.n_strips + most - 1) / most : 1;
    p.n_grp = (n_dir / 4 + per - 1) / per;
    // A table entry costs about 60 operations per material and direction in
    // each sweep's workgroup, a step about 50 per wave and the inverses per cell 25
    // more: the table where it is the cheaper of the two and fits (and, with
    // 1/|z|^2 in it, where that is a normal number).  A large table also keeps
    // other workgroups off the compute unit, and many directions take turns (50^2,
    // 2500 materials, S_32: 0.16 ms an iteration with the table, 83 KB for a
    // workgroup of one wave, in four turns; 0.09 without).
    const int rows = (int)std::min<long long>(n_mat, 1 << 20);
    auto turns = [&](int n) {
      const long long here = lds / dg_sweep_lds_bytes(p, n, refl);
      // (waves of four directions fill their SIMDs, of one need company)
      const long long waves = (per == 1 ? 16 : 4) / p.n_waves;
      const long long at_once = 256 * std::max(1ll, std::min(here, waves));
      return (4 * p.n_grp * p.n_blk + at_once - 1) / at_once;
    };
    const long long walk = 64ll * p.n_waves * (p.nu + p.nv);
    p.table = n_mat > 0 && (per == 1 || squares) &&
              dg_sweep_lds_bytes(p, rows, refl) <= lds &&
              turns(rows) * (60 * n_mat + 50 * walk) <= turns(0) * 75 * walk;
    return dg_sweep_lds_bytes(p, p.table ? (int)n_mat : 0, refl) <= lds;
  };
  DgPlan cand[4];
  int n_cand = 0;
  auto add = [&](int swap, int per) {
    axis(swap);
    if (fill(per)) cand[n_cand++] = p;
    return n_cand > 0;
  };
  if (!add(cheap, 1) || p.nv == 1) return p;  // (a row: the scan of its cells)
  add(1 - cheap, 1);
  if (n_dir >= 4 * kDgSplit) {
    add(cheap, kDgSplit);
    add(1 - cheap, kDgSplit);
  }
  // Microseconds of a sweep and its reduction.  The chain of steps: a strip starts
  // 72 steps after the one before, so that at most (nu + 63) / 72 + 1 work at a time.
  // With four directions per wave a step takes 0.5 us, 0.65 with the inverses per
  // cell; with one 0.23, or 0.033 (0.038) times the strips at work, which share a
  // compute unit, and up to 2.1 times that where rows of more than 600 columns
  // leave the caches.  The planes: what stays in the 256 MB last-level cache costs
  // 0.2 us a MB, what does not 0.3 more, which four directions per wave quarter;
  // one direction per wave, with four times their memory, has to gain 5%.
  // Fitted to 300 measured pairs of mesh and order (40^2 to 2048^2, 3500 x 30 to
  // 3800 x 250, S_2 to S_16, table and cells; other sizes are extrapolated): the
  // choice is at most 10% slower than the best of the four, 0.2% on average.
  // Milliseconds with one along either axis, four along either: 2300 x 65 S_4 0.50,
  // 0.42, 1.18, 1.06; 3000 x 1000 S_16 13.8, -, -, 5.2 (four's traces do not fit the
  // LDS above some 2400 columns); 1024^2 S_16 5.1, -, 1.83, 1.88; 256^2 S_8 0.13, -,
  // 0.27, 0.27; 512^2 S_8 0.59, -, 0.59, 0.58.
  auto us = [&](const DgPlan& c, bool table) {
    const bool four = c.per == kDgSplit;
    const double strips = c.n_strips - 1, steps = c.nu + 72.0 * strips + c.nv - 64.0 * strips;
    const double work = std::min(c.n_waves, (c.nu + 63) / 72 + 1);
    const double far = std::max(0, c.nu - 600) * 1e-3 * std::min(1.0, nc / 0.9e6);
    const double busy = (0.033 * (1.0 + std::min(1.1, far)) + (table ? 0.0 : 0.005)) * work;
    const double step = four ? (table ? 0.5 : 0.65) : std::max(0.23, busy);
    const double mb = 128e-6 * c.n_grp * (double)nc, past = std::max(0.0, mb - 200.0);
    const double t = steps * step + (four ? 0.24 : 0.2) * mb + (four ? 0.12 : 0.32) * past;
    return four ? t : 1.05 * t;
  };
  int best = 0;
  if (n_mat >= 0) {
    for (int k = 1; k < n_cand; ++k)
      if (us(cand[k], cand[k].table) < us(cand[best], cand[best].table)) best = k;
    return cand[best];
  }
  // not known: of those that some materials would choose, the largest
  double most = us(cand[0], false);
  for (int k = 1; k < n_cand; ++k) most = std::min(most, us(cand[k], false));
  size_t bytes = 0;
  for (int k = 0; k < n_cand; ++k)
    if (us(cand[k], true) <= most && dg_plane_bytes(cand[k], nc) > bytes) {
      bytes = dg_plane_bytes(cand[k], nc);
      best = k;
    }
  return cand[best];
}

hipError_t launch_si_start(const DgArgs& a, int si_max, hipStream_t s) {
  const long long nc = (long long)a.nx * a.ny;
  long long b = (nc + 255) / 256;
  const int grid = (int)(b < 2048 ? (b < 1 ? 1 : b) : 2048);
  const long long nb = a.bnd ? (long long)a.n_dir * 2 * (a.nx + a.ny) : 0;
  hipLaunchKernelGGL(k_si_start, dim3(grid), dim3(256), 0, s, a, a.bnd ? a.bnd + nb : nullptr, nb,
                     si_max);
  return hipGetLastError();
}

__global__ void k_si_check(DevState* st) {
  if (threadIdx.x == 0 && !st->halt && !st->si.done) {
    st->halt = 1;
    st->si.done = 1;
  }
}

__global__ void k_dsa_check(DevState* st) {
  if (threadIdx.x == 0 && !st->halt && !st->si.done && !st->dsa.done) {
    st->halt = 1;
    st->si.done = 1;
  }
}

hipError_t launch_dsa_check(DevState* st, hipStream_t s) {
  hipLaunchKernelGGL(k_dsa_check, dim3(1), dim3(64), 0, s, st);
  return hipGetLastError();
}

hipError_t launch_si_check(DevState* st, hipStream_t s) {
  hipLaunchKernelGGL(k_si_check, dim3(1), dim3(64), 0, s, st);
  return hipGetLastError();
}

// Sixteen waves leave 128 vector registers to each, eight 256: sources of
// four or of eight columns in flight.
template <bool TABLE, bool REFL>
static void sweep_launch(const DgArgs& a, size_t lds, hipStream_t s) {
  const dim3 block(64 * a.n_waves);
  const int n_all = 4 * a.n_grp;
  if (a.per == kDgSplit)  // a grid that gives every class its tasks
    hipLaunchKernelGGL((k_dg_sweep<kDgSplit, TABLE, REFL, 8, 64 * kDgSplitWaves>),
                       dim3((n_all + 7) / 8 * 8 * a.n_blk), block, lds, s, a);
  else if (a.n_waves <= 8)
    hipLaunchKernelGGL((k_dg_sweep<1, TABLE, REFL, 8, 512>), dim3(n_all), block, lds, s, a);
  else
    hipLaunchKernelGGL((k_dg_sweep<1, TABLE, REFL, 4, 1024>), dim3(n_all), block, lds, s, a);
}

hipError_t launch_dg_sweep(const DgArgs& a, hipStream_t s) {
  const bool table = a.mat_off != nullptr;
  const bool refl = a.bc != 0 && a.bnd != nullptr, split = a.per == kDgSplit;
  const size_t lds = dg_sweep_lds_bytes(a, table ? a.n_mat : 0, refl);
  if ((a.per != 1 && !split) || a.n_waves < 1 || a.n_strips != (a.nv + 63) / 64 ||
      a.n_waves > (split ? kDgSplitWaves : kDgMaxWaves) || a.n_grp * a.per < a.n_quad ||
      a.n_blk * a.n_waves < (split ? a.n_strips : 1) || (split && a.n_blk > 1 && !a.hand) ||
      (!split && a.n_blk != 1) || a.nx * a.ny >= 1 << 23)
    return hipErrorInvalidValue;
  if (a.nv == 1 && a.per == 1) {
    const int waves = std::min(kRowWaves, (a.nu + 63) / 64);
    if (refl)
      hipLaunchKernelGGL((k_dg_sweep_row<true>), dim3(4 * a.n_grp), dim3(64 * waves), 0, s, a);
    else
      hipLaunchKernelGGL((k_dg_sweep_row<false>), dim3(4 * a.n_grp), dim3(64 * waves), 0, s, a);
  } else if (table) {
    if (refl) sweep_launch<true, true>(a, lds, s);
    else sweep_launch<true, false>(a, lds, s);
  } else {
    if (refl) sweep_launch<false, true>(a, lds, s);
    else sweep_launch<false, false>(a, lds, s);
  }
  return hipGetLastError();
}

// The reduction of a source iteration (k_dg_combine): phi_new = the nodal
// values of the four quadrants' sums over their planes, in place (the sweep
// read only the sources); the next iterate's source S = sigma_s/(4 pi)
// (phi_new + phi_post) in every quadrant's coefficients (unused when the
// iteration stops here); block partials of |phi_new - phi_old|^2 and
// |phi_new|^2, or |phi_new + phi_pre + phi_post|^2 when phi_pre is given (the
// step's whole flux as the reference of the stopping test).  With the
// diffusion correction the combine keeps phi_new - phi_old in dnode instead
// and leaves the source and the residual to k_dsa_apply.  The last block of a
// grid to leave its partials takes the iteration's decision.
constexpr int kTile = 8;                  // cells of a tile's side
constexpr int kRedCells = kTile * kTile;  // one wave per quadrant
constexpr int kRedWaves = 4;
constexpr int kRedBlock = 64 * kRedWaves;

int dg_reduce_partials(int nx, int ny) {
  const long long tiles = (long long)((nx + kTile - 1) / kTile) * ((ny + kTile - 1) / kTile);
  return (int)(tiles < 1024 ? tiles : 1024);
}

__device__ __forceinline__ double wave_sum(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// Leaves the block's partials (the first wave's sums, in a fixed order) and,
// in the last block of the grid to do so, sums all of them in a fixed order
// (strided per-thread sums, wave sums, the waves in order) and takes the
// iteration's decision: done when |phi_new - phi_old| <= tol |phi_new|
// (converged), when the iteration limit is reached, or when the residual is
// not finite.  After a diffusion correction (dsa) it also books that
// correction's conjugate-gradient iterations and whether they reached their
// tolerance.  The partials cross the XCDs as agent-scope stores and loads;
// the stores have reached memory when the block counts itself.  (As a launch
// of its own the decision took 3-4 us of every iteration.)
__device__ __forceinline__ void residual(double dsum, double nsum, double* partials, DevState* st,
                                         double si_tol, int si_max, int dsa) {
  __shared__ double s_d[kRedWaves], s_n[kRedWaves];
  __shared__ int s_last;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (wave == 0) {
    dsum = wave_sum(dsum);
    nsum = wave_sum(nsum);
    if (lane == 0) {
      __hip_atomic_store(&partials[2 * blockIdx.x], dsum, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&partials[2 * blockIdx.x + 1], nsum, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      if (lane == 0) s_last = count_block(st->red);
    }
  }
  __syncthreads();
  if (!s_last) return;
  double d = 0.0, n = 0.0;
  for (int b = threadIdx.x; b < (int)gridDim.x; b += kRedBlock) {
    d += __hip_atomic_load(&partials[2 * b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    n += __hip_atomic_load(&partials[2 * b + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  d = wave_sum(d);
  n = wave_sum(n);
  if (lane == 0) {
    s_d[wave] = d;
    s_n[wave] = n;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double dn2 = s_d[0], nrm2 = s_n[0];
    for (int k = 1; k < kRedWaves; ++k) {
      dn2 += s_d[k];
      nrm2 += s_n[k];
    }
    const double dn = sqrt(dn2), nrm = sqrt(nrm2);
    st->si.dn2_prev = st->si.iter > 0 ? st->si.dn2 : 0.0;
    st->si.dn2 = dn2;
    st->si.nrm2 = nrm2;
    st->si.iter += 1;
    const int bad = !isfinite(dn) || !isfinite(nrm);
    const int conv = !bad && dn <= si_tol * nrm;
    st->si.bad = bad;
    st->si.conv = conv;
    st->si.done = bad || conv || st->si.iter >= si_max;
    if (dsa) {
      st->dsa_corrections += 1;
      st->dsa_iter_total += st->dsa.iter;
      if (st->dsa.iter > st->dsa_iter_max) st->dsa_iter_max = st->dsa.iter;
      if (!st->dsa.conv) st->dsa_unconv += 1;
    }
  }
}

// A cell's contribution to the stopping test.
__device__ __forceinline__ void add_norms(double4 v, double4 d, double r, double& dsum,
                                          double& nsum) {
  dsum += d.x * d.x + d.y * d.y + d.z * d.z + d.w * d.w;
  nsum += (v.x + r) * (v.x + r) + (v.y + r) * (v.y + r) + (v.z + r) * (v.z + r) +
          (v.w + r) * (v.w + r);
}

// A block takes tiles of 8 x 8 cells; wave q works in quadrant q: it sums the
// quadrant's planes at the lane's cell, the four nodal sums meet in LDS, and
// after the cells' update (wave 0) it forms the quadrant's next source.  The
// cells of a slot row lie on a diagonal of the mesh, so a wave takes its tile
// along the diagonals of its quadrant: eight lanes then read, and write, two
// whole cache lines.  Bound by the planes' traffic and, with few tiles, by the
// latency of the planes' batches; 26 us a reduction at 140x140, S_12 (the choices,
// when they were made, in means over launches of which a quarter return at once:
// 29 us; cells in row-major order, a line for every lane, 75; the two modes in
// arrays of their own, one line for eight lanes, 40; tiles of 16 x 16, 33).
constexpr int kNodeRow = kRedCells + 1;  // LDS stride of a node: [node][cell]

// Tile cell of lane l in quadrant q: column (d - e) mod 8 of the u axis and row e
// of the v axis, d and e the lane's octal digits, u and v mirrored as the quadrant
// is.
struct TileCell {
  int cell, slot, at;  // the cell, its slot, its place in the tile (row-major)
  bool ok;
};
__device__ __forceinline__ TileCell tile_cell(const DgArgs& g, int2 tile, int q, int lane) {
  const int e = lane % kTile, d = lane / kTile, f = (d - e) & (kTile - 1);
  const int x = g.swap ? e : f, y = g.swap ? f : e;
  const int i = (q & 1) ? kTile - 1 - x : x, j = (q & 2) ? kTile - 1 - y : y;
  const int ci = tile.x * kTile + i, cj = tile.y * kTile + j;
  TileCell t;
  t.ok = ci < g.nx && cj < g.ny;
  // a real cell for every lane's loads
  const int ri = ci < g.nx ? ci : g.nx - 1, rj = cj < g.ny ? cj : g.ny - 1;
  t.cell = rj * g.nx + ri;
  t.slot = dg_slot(g, q, ri, rj);
  t.at = j * kTile + i;
  return t;
}

__device__ __forceinline__ int dg_tiles(const DgArgs& g) {
  return ((g.nx + kTile - 1) / kTile) * ((g.ny + kTile - 1) / kTile);
}

// The k-th tile.  A slot row's run of eight cells belongs to two tiles that are
// neighbours along u, and its cache lines to neighbours along v: where every
// tile has its block, the blocks of an XCD (k mod 8) take a run of tiles in the
// order of v, then u (333 x 187, S_8: 38 -> 31 us a reduction, 128^2, S_16: 31 ->
// 28, 140^2, S_12: 27 -> 26).  On larger meshes the rows' order is the better
// one: the runs' starts, an eighth of a power of two apart, meet in the same
// memory channels (1024^2: 0.46 against 0.51 ms; patches of 8 x 8 tiles 0.47).
__device__ __forceinline__ int2 dg_tile(const DgArgs& g, int k) {
  const int tx = (g.nx + kTile - 1) / kTile, ty = (g.ny + kTile - 1) / kTile;
  if (tx * ty > (int)gridDim.x) return make_int2(k % tx, k / tx);
  const int xcd = k & 7, base = tx * ty >> 3, more = tx * ty & 7;
  const int p = xcd * base + (xcd < more ? xcd : more) + (k >> 3);
  const int along = g.swap ? tx : ty, tu = p / along, tv = p - tu * along;
  return g.swap ? make_int2(tv, tu) : make_int2(tu, tv);
}

// The quadrant's next source at the lane's cell from the nodal one in LDS.
__device__ __forceinline__ void put_source(const DgArgs& g, int q, const TileCell& t,
                                           const double* s_src) {
  const int n = g.nx * g.ny;
  double2 m1, m2;
  to_modes(s_src[quad_node(q, g.swap, 0, 0) * kNodeRow + t.at],
           s_src[quad_node(q, g.swap, 0, 1) * kNodeRow + t.at],
           s_src[quad_node(q, g.swap, 1, 0) * kNodeRow + t.at],
           s_src[quad_node(q, g.swap, 1, 1) * kNodeRow + t.at], m1, m2);
  double2* const S = reinterpret_cast<double2*>(g.src) + (size_t)q * 2 * n;
  S[2 * t.slot] = m1;
  S[2 * t.slot + 1] = m2;
}

// Nodal source of a cell into LDS (wave 0).
__device__ __forceinline__ void nodal_source(double* s_src, int at, double ssc, double4 v,
                                             double pp) {
  s_src[0 * kNodeRow + at] = ssc * (v.x + pp);
  s_src[1 * kNodeRow + at] = ssc * (v.y + pp);
  s_src[2 * kNodeRow + at] = ssc * (v.z + pp);
  s_src[3 * kNodeRow + at] = ssc * (v.w + pp);
}

__global__ __launch_bounds__(kRedBlock) void k_dg_combine(DgArgs g, double* partials,
                                                          double si_tol, int si_max) {
  DevState* const st = g.st;
  if (st->si.done) return;
  if (blockIdx.x == 0 && threadIdx.x < 8) {  // ready for the next sweep
    st->ticket[threadIdx.x] = 0u;
    if (threadIdx.x == 0) st->sweep_tag += 1u;
  }
  __shared__ double s_phi[4][4 * kNodeRow];  // nodal sums of each quadrant
  __shared__ double s_src[4 * kNodeRow];     // nodal source
  const double inv4pi = 0.25 / M_PI;
  const int n = g.nx * g.ny;
  const int lane = threadIdx.x & 63;
  const int q = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const double2* const plane =
      reinterpret_cast<const double2*>(g.psi) + (size_t)q * g.n_grp * 2 * n;
  const double* const dir = g.dir + 3 * (size_t)q * g.n_quad;
  const int n_tiles = dg_tiles(g);
  double dsum = 0.0, nsum = 0.0;
  for (int k = blockIdx.x; k < n_tiles; k += gridDim.x) {
    const TileCell t = tile_cell(g, dg_tile(g, k), q, lane);
    // wave 0: the cell's data for the update, in flight with the planes
    double4 o = make_double4(0.0, 0.0, 0.0, 0.0);
    double ssc = 0.0, pp = 0.0, pre = 0.0;
    if (q == 0) {
      o = reinterpret_cast<const double4*>(g.phi_c)[t.cell];
      if (!g.dnode) {
        ssc = g.sig_s[t.cell];
        pp = g.phi_post[t.cell];
        if (g.phi_pre) pre = g.phi_pre[t.cell];
      }
    }
    double2 m1 = make_double2(0.0, 0.0), m2 = m1;
    auto add = [&](int u, double2 t1, double2 t2) __attribute__((always_inline)) {
      const double w = g.per == 1 ? dir[3 * u + 2] : 1.0;
      m1.x += w * t1.x;
      m1.y += w * t1.y;
      m2.x += w * t2.x;
      m2.y += w * t2.y;
    };
    int u = 0;
    for (; u + 8 <= g.n_grp; u += 8) {  // eight planes' loads in flight
      double2 t1[8], t2[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        t1[e] = plane[((size_t)(u + e) * n + t.slot) * 2];
        t2[e] = plane[((size_t)(u + e) * n + t.slot) * 2 + 1];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) add(u + e, t1[e], t2[e]);
    }
    if (u < g.n_grp) {  // the rest as one batch too (past the end, loads of the last one)
      double2 t1[7], t2[7];
#pragma unroll
      for (int e = 0; e < 7; ++e) {
        const int v = u + e < g.n_grp ? u + e : g.n_grp - 1;
        t1[e] = plane[((size_t)v * n + t.slot) * 2];
        t2[e] = plane[((size_t)v * n + t.slot) * 2 + 1];
      }
#pragma unroll
      for (int e = 0; e < 7; ++e)
        if (u + e < g.n_grp) add(u + e, t1[e], t2[e]);
    }
    double x[4];
    from_modes(m1, m2, x);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      s_phi[q][quad_node(q, g.swap, k >> 1, k & 1) * kNodeRow + t.at] = x[k];
    __syncthreads();
    if (q == 0 && t.ok) {
      double f[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int at = k * kNodeRow + t.at;
        f[k] = (s_phi[0][at] + s_phi[3][at]) + (s_phi[1][at] + s_phi[2][at]);
      }
      const double4 v = make_double4(f[0], f[1], f[2], f[3]);
      const double4 d = make_double4(v.x - o.x, v.y - o.y, v.z - o.z, v.w - o.w);
      reinterpret_cast<double4*>(g.phi_c)[t.cell] = v;
      if (g.dnode) {  // the correction, the source and the residual come later
        reinterpret_cast<double4*>(g.dnode)[t.cell] = d;
      } else {
        nodal_source(s_src, t.at, ssc * inv4pi, v, pp);
        add_norms(v, d, g.phi_pre ? pre + pp : 0.0, dsum, nsum);
      }
    }
    __syncthreads();
    if (!g.dnode && t.ok) put_source(g, q, t, s_src);
  }
  if (g.dnode) return;  // the same for the whole grid
  residual(dsum, nsum, partials, st, si_tol, si_max, 0);
}

// phi += delta (per cell) at every node, the next source, and the residual of
// |dnode + delta|^2 and |phi|^2 (or of the whole-flux norm).
__global__ __launch_bounds__(kRedBlock) void k_dsa_apply(DgArgs g,
                                                         const double* __restrict__ delta,
                                                         double* partials, double si_tol,
                                                         int si_max) {
  DevState* const st = g.st;
  if (st->si.done) return;
  __shared__ double s_src[4 * kNodeRow];
  const double inv4pi = 0.25 / M_PI;
  const int lane = threadIdx.x & 63;
  const int q = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int n_tiles = dg_tiles(g);
  double dsum = 0.0, nsum = 0.0;
  for (int k = blockIdx.x; k < n_tiles; k += gridDim.x) {
    const TileCell t = tile_cell(g, dg_tile(g, k), q, lane);
    if (q == 0 && t.ok) {
      const double dl = delta[t.cell];
      const double4 o = reinterpret_cast<const double4*>(g.phi_c)[t.cell];
      const double4 dn = reinterpret_cast<const double4*>(g.dnode)[t.cell];
      const double4 v = make_double4(o.x + dl, o.y + dl, o.z + dl, o.w + dl);
      const double4 d = make_double4(dn.x + dl, dn.y + dl, dn.z + dl, dn.w + dl);
      reinterpret_cast<double4*>(g.phi_c)[t.cell] = v;
      const double pp = g.phi_post[t.cell];
      nodal_source(s_src, t.at, g.sig_s[t.cell] * inv4pi, v, pp);
      add_norms(v, d, g.phi_pre ? g.phi_pre[t.cell] + pp : 0.0, dsum, nsum);
    }
    __syncthreads();
    if (t.ok) put_source(g, q, t, s_src);
    __syncthreads();
  }
  residual(dsum, nsum, partials, st, si_tol, si_max, 1);
}

hipError_t launch_dg_reduce(const DgArgs& a, double* partials, int n_part, double si_tol,
                            int si_max, hipStream_t s) {
  hipLaunchKernelGGL(k_dg_combine, dim3(n_part), dim3(kRedBlock), 0, s, a, partials, si_tol,
                     si_max);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Source iterations of a short row in one workgroup
// ---------------------------------------------------------------------------
// Meshes of one row and up to 128 cells: the whole batch of source iterations
// in one workgroup, the iterations separated by barriers instead of launches
// (k_dg_sweep_row and k_dg_combine take 11 us an iteration, nearly all of it
// launches and memory latency).  Sixteen lanes sweep a direction, K cells each,
// by a scan of the cells' trace maps along the direction's travel; the four
// rows of a wave are the four quadrants, wave w takes their direction w (so at
// most eight per quadrant).  The fluxes meet in LDS, where a thread per node
// sums them to the next iterate and its source; then every thread takes the
// same decision from the waves' partial norms.  What bounds an iteration is the
// issue of the busiest SIMD's two waves: S_4 with reflective sides takes 2.5 us on
// 16 cells, 6 us on 80 and 10 us on 128 (one launch each for sweep and reduction:
// 10, 11 and 11.5 us).  More cells or directions keep the separate kernels; c1
// and c2 would then leave the registers, which cost twice the time.
constexpr int kRowSolveWaves = 8;
constexpr int kRowSolveBlock = 64 * kRowSolveWaves;
constexpr int kRowSolveCells = 128;  // a thread per node

template <int CTRL>
__device__ __forceinline__ double dpp_or(double otherwise, double v) {
  const long long o = __double_as_longlong(otherwise), s = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp((int)o, (int)s, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(s >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// The map of the lane `OFF` before in the row of sixteen, else the identity.
template <int OFF>
__device__ __forceinline__ TraceMap row_before(const TraceMap& m) {
  constexpr int kRowShr = 0x110 + OFF;
  return {dpp_or<kRowShr>(1.0, m.ar), dpp_or<kRowShr>(0.0, m.ai), dpp_or<kRowShr>(0.0, m.br),
          dpp_or<kRowShr>(0.0, m.bi)};
}

template <int K>
__global__ __launch_bounds__(kRowSolveBlock) void k_dg_row_solve(DgArgs g, int n_it, double si_tol,
                                                                 int si_max) {
  DevState* const st = g.st;
  if (st->si.done) return;
  constexpr int row = 16 * K;  // places of a node's row: cell p at (p % K) * 16 + p / K
  constexpr double kap = kV1i;
  extern __shared__ double smem[];
  double* const s_src = smem;            // nodal source [node][place]
  double* const s_norm = smem + 4 * row; // partial norms [2][wave]
  double* const s_phi = s_norm + 2 * kRowSolveWaves;  // sums [wave][quadrant][node][place]
  const int nu = g.nu, t = threadIdx.x, wave = t >> 6, q = (t >> 4) & 3;
  const bool back = (q & (g.swap ? 2 : 1)) != 0, vnegative = (q & (g.swap ? 1 : 2)) != 0;
  const int ubc = g.swap ? g.bc >> 2 : g.bc, vbc = g.swap ? g.bc : g.bc >> 2;
  const bool refl = g.bc != 0 && g.bnd != nullptr;
  const bool u_in = refl && (ubc & (back ? 2 : 1)), u_out = refl && (ubc & (back ? 1 : 2));
  const bool v_in = refl && (vbc & (vnegative ? 2 : 1));
  const bool v_out = refl && (vbc & (vnegative ? 1 : 2));
  const size_t n_tr = (size_t)nu + 1;
  double2* const bnd = reinterpret_cast<double2*>(g.bnd);
  // the lane's chunk of K cells; lanes and cells in order of travel
  const int c = back ? 15 - (t & 15) : t & 15;
  auto cell_of = [&](int k) { return c * K + (back ? K - 1 - k : k); };
  auto place_of = [&](int k) { return (back ? K - 1 - k : k) * 16 + c; };

  // the sixteen lanes' direction
  const bool sweeps = wave < g.n_quad;
  const int m = q * g.n_quad + (sweeps ? wave : 0);
  const double ox = fabs(g.dir[3 * m]) / g.hx, oy = fabs(g.dir[3 * m + 1]) / g.hy;
  const double a = g.swap ? oy : ox, b = g.swap ? ox : oy, weight = g.dir[3 * m + 2];
  const double2* u_from = nullptr;  // its inflow traces in the first buffer
  const double2* v_from = nullptr;
  if (refl) {
    u_from = bnd + (g.swap ? g.refl_y : g.refl_x)[m] * n_tr;
    v_from = bnd + (g.swap ? g.refl_x : g.refl_y)[m] * n_tr + 1;
  }
  const size_t n_bnd = (size_t)g.n_dir * n_tr;  // of a buffer
  double2 c1[K], c2[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int p = cell_of(k), pc = p < nu ? p : nu - 1;
    double se;
    if (g.mat_off)
      se = g.sig_e_mat[g.mat_off[(size_t)q * nu + (back ? nu - 1 - pc : pc)] >> 5];
    else
      se = g.sig_e[pc];
    mode_inverse(a, b, se, c1[k], c2[k]);
  }

  // the thread's node
  const bool node_ok = t < 4 * nu;
  const int node = t & 3, at = node * row + (t >> 2) % K * 16 + (t >> 2) / K;
  double phi = 0.0, ssc = 0.0, pp = 0.0, ref = 0.0;
  if (node_ok) {
    phi = g.phi_c[t];
    ssc = g.sig_s[t >> 2] * (0.25 / M_PI);
    pp = g.phi_post[t >> 2];
    if (g.phi_pre) ref = g.phi_pre[t >> 2] + pp;
  }
  for (int k = t; k < 4 * row; k += kRowSolveBlock) s_src[k] = 0.0;
  __syncthreads();
  if (node_ok) s_src[at] = ssc * (phi + pp);
  __syncthreads();

  const int it0 = st->si.iter;
  int it = it0, bad = 0, conv = 0, done = 0;
  double dn2 = st->si.dn2, dn2_prev = 0.0, nrm2 = 0.0;
  while (it < it0 + n_it && !done) {
    if (sweeps) {
      const size_t in = (it + 1) & 1 ? n_bnd : 0;
      double2* const b_out = bnd + (it & 1 ? n_bnd : 0) + m * n_tr;
      double2 ux = make_double2(0.0, 0.0);
      if (u_in) ux = u_from[in];
      double2 X1[K], X2[K];  // S + b uy, then the cells' modes
#pragma unroll
      for (int k = 0; k < K; ++k) {
        double s[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
          s[j] = s_src[quad_node(q, g.swap, j >> 1, j & 1) * row + place_of(k)];
        to_modes(s[0], s[1], s[2], s[3], X1[k], X2[k]);
        if (v_in) {
          const int p = cell_of(k), pc = p < nu ? p : nu - 1;
          const double2 uy = v_from[in + (back ? nu - 1 - pc : pc)];
          X1[k] = make_double2(fma(b, uy.x, X1[k].x), fma(b, uy.y, X1[k].y));
          X2[k] = make_double2(fma(b, uy.x, X2[k].x), fma(b, uy.y, X2[k].y));
        }
      }
      TraceMap map = {1.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const double2 A = trace_of(c1[k], c2[k]);
        const double2 B = trace_of(times(c1[k], X1[k]), times(c2[k], X2[k]));
        const bool ok = cell_of(k) < nu;  // else the identity
        map = after(map, {ok ? a * A.x : 1.0, ok ? a * A.y : 0.0, ok ? B.x : 0.0,
                          ok ? B.y : 0.0});
      }
      map = after(row_before<1>(map), map);
      map = after(row_before<2>(map), map);
      map = after(row_before<4>(map), map);
      map = after(row_before<8>(map), map);
      ux = apply(row_before<1>(map), ux);
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const int p = cell_of(k), u = back ? nu - 1 - p : p;
        X1[k] = times(c1[k], make_double2(fma(a, ux.x, X1[k].x), fma(a, ux.y, X1[k].y)));
        X2[k] = times(c2[k], make_double2(fma(a, ux.x, X2[k].x), fma(-a, ux.y, X2[k].y)));
        const bool ok = p < nu;
        const double2 next = trace_of(X1[k], X2[k]);
        ux = make_double2(ok ? next.x : ux.x, ok ? next.y : ux.y);
        if (v_out && ok)
          b_out[1 + u] = make_double2(fma(-kap, X1[k].y - X2[k].y, -(X1[k].x + X2[k].x)),
                                      fma(kap, X1[k].x - X2[k].x, -(X1[k].y + X2[k].y)));
        if (u_out && u == nu - 1) b_out[0] = ux;
        double f[4];
        from_modes(X1[k], X2[k], f);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          s_phi[((wave * 4 + q) * 4 + quad_node(q, g.swap, j >> 1, j & 1)) * row + place_of(k)] =
              weight * f[j];
      }
    }
    __syncthreads();
    double d2 = 0.0, v2 = 0.0;
    if (node_ok) {
      double f[4] = {0.0, 0.0, 0.0, 0.0};
      for (int w = 0; w < g.n_quad; ++w)
#pragma unroll
        for (int k = 0; k < 4; ++k) f[k] += s_phi[(w * 4 + k) * 4 * row + at];
      const double v = (f[0] + f[3]) + (f[1] + f[2]), d = v - phi;
      phi = v;
      s_src[at] = ssc * (v + pp);
      d2 = d * d;
      v2 = (v + ref) * (v + ref);
    }
    d2 = wave_sum(d2);
    v2 = wave_sum(v2);
    if ((t & 63) == 0) {
      s_norm[wave] = d2;
      s_norm[kRowSolveWaves + wave] = v2;
    }
    __syncthreads();
    dn2_prev = it > 0 ? dn2 : 0.0;
    dn2 = nrm2 = 0.0;
    for (int w = 0; w < kRowSolveWaves; ++w) {
      dn2 += s_norm[w];
      nrm2 += s_norm[kRowSolveWaves + w];
    }
    it += 1;
    const double dn = sqrt(dn2), nrm = sqrt(nrm2);
    bad = !isfinite(dn) || !isfinite(nrm);
    conv = !bad && dn <= si_tol * nrm;
    done = bad || conv || it >= si_max;
  }
  if (node_ok) g.phi_c[t] = phi;
  if (t == 0) {
    st->si.dn2_prev = dn2_prev;
    st->si.dn2 = dn2;
    st->si.nrm2 = nrm2;
    st->si.iter = it;
    st->si.bad = bad;
    st->si.conv = conv;
    st->si.done = done;
  }
}

static size_t row_solve_lds(const DgArgs& a, int K) {
  return sizeof(double) * (size_t)(16 * K * 4 * (1 + 4 * a.n_quad) + 2 * kRowSolveWaves);
}

// Cells per lane of the one-workgroup iteration, 0 where it does not apply.
static int row_solve_cells(const DgArgs& a) {
  if (a.nv != 1 || a.per != 1 || a.dnode || a.nu > kRowSolveCells || a.n_quad > kRowSolveWaves)
    return 0;
  return (a.nu + 15) / 16;
}

bool dg_row_solve(const DgArgs& a, size_t lds) {
  const int K = row_solve_cells(a);
  return K && row_solve_lds(a, K) <= lds;
}

template <int K>
static void row_solve_launch(const DgArgs& a, int n_it, double si_tol, int si_max, hipStream_t s) {
  hipLaunchKernelGGL((k_dg_row_solve<K>), dim3(1), dim3(kRowSolveBlock), row_solve_lds(a, K), s, a,
                     n_it, si_tol, si_max);
}

hipError_t launch_dg_row_solve(const DgArgs& a, int n_it, double si_tol, int si_max,
                               hipStream_t s) {
  switch (row_solve_cells(a)) {
    case 1: row_solve_launch<1>(a, n_it, si_tol, si_max, s); break;
    case 2: row_solve_launch<2>(a, n_it, si_tol, si_max, s); break;
    case 3: row_solve_launch<3>(a, n_it, si_tol, si_max, s); break;
    case 4: row_solve_launch<4>(a, n_it, si_tol, si_max, s); break;
    case 5: row_solve_launch<5>(a, n_it, si_tol, si_max, s); break;
    case 6: row_solve_launch<6>(a, n_it, si_tol, si_max, s); break;
    case 7: row_solve_launch<7>(a, n_it, si_tol, si_max, s); break;
    case 8: row_solve_launch<8>(a, n_it, si_tol, si_max, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_dsa_apply(const DgArgs& a, const double* delta, double* partials, int n_part,
                            double si_tol, int si_max, hipStream_t s) {
  hipLaunchKernelGGL(k_dsa_apply, dim3(n_part), dim3(kRedBlock), 0, s, a, delta, partials, si_tol,
                     si_max);
  return hipGetLastError();
}

}  // namespace slh
