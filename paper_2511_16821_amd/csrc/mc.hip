// (Q)MC pass of the scatter-limited hybrid method (Sec. 2.3 of the paper):
// emission stratified by cell, tracking with at most n_lim scatters per
// history, or per-cell limits N_s(x) (implicit capture with sigma_a before
// the limit, attenuation with sigma_t after it), exact track-length tallies
// w (1 - e^{-sigma l}) / sigma per segment, and the census write of the remap
// pass.
//
// Execution model: a persistent grid sized to the device's occupancy.  Every
// lane owns one history at a time and, when it ends, takes the next work
// index of its wave's chunk of consecutive indices.  A wave whose chunk is
// used up takes the next one: on large passes (four or more chunks of
// kWorkChunk per wave) from the pass's counter, which balances the load; on
// smaller ones, where a shared counter would be contended, chunk w + k W of
// W waves, sized to about eight per wave.  (140^2 checkerboard, 2e6 items:
// passes 0.16 / 0.14 ms against 0.24 / 0.20 from the counter; 256^2 thick
// medium, 2e7 items: 1.27 ms from the counter against 1.41 cyclic.)  Lanes refill without waiting for
// the slowest history of their wave, and the histories of a wave start close
// together (the work index follows the cell order of the banks), so their
// material reads and tally adds meet in the caches.  The work index g maps to
// census particle g (g < n_in) or source particle g - n_in; every random
// number of a history is a pure function of its (stream, dimension, point
// index), so results do not depend on which lane or wave ran it.  Tallies and balance sums are fixed point with integer atomics
// and are therefore independent of the schedule.  Each wave adds into one of
// several private copies of the tally (summed afterwards), through a small
// cache of tally words in LDS, so that simultaneous updates of a busy cell do
// not queue on one cache line.
#include <atomic>
#include "slh_common.hpp"
#include "sobol_dirs.inc"

namespace slh {

const uint32_t* sobol_table_host() {
  struct Table {
    alignas(16) uint32_t w[kSobolNibbleWords];
    Table() {
      for (int e = 0; e < kSobolNibbleWords; ++e) {
        const int d = e >> 7, pos = (e >> 4) & 7;
        w[e] = 0u;
        for (int k = 0; k < 4; ++k)
          if (e >> k & 1) w[e] ^= slh_sobol_v[d * 32 + 4 * pos + k];
      }
    }
  };
  static const Table t;  // initialised once, whichever thread comes first
  return t.w;
}

template <typename R> struct Real;
template <> struct Real<double> {
  using V2 = double2;
  static __device__ __forceinline__ void scpi(double x, double* s, double* c) {
    sincospi(x, s, c);
  }
  static __device__ __forceinline__ SrcRec<double>* src(const PassArgs& a) { return a.src64; }
  // w e^{-z} = w + w (e^{-z} - 1): the weight minus what the segment removed
  static __device__ __forceinline__ double attenuate(double w, double, double em) {
    return fma(w, em, w);
  }
  static __device__ __forceinline__ double2 mat(const PassArgs& a, int c) {
    return a.mat_id16 ? a.mtab64[a.mat_id16[c]] : a.mat64[c];
  }
  static __device__ __forceinline__ double inf() { return __builtin_huge_val(); }
  static __device__ __forceinline__ const StageRec<double>* in(const PassArgs& a) {
    return a.in64;
  }
  static __device__ __forceinline__ StageRec<double>* out(const PassArgs& a) { return a.out64; }
  static __device__ __forceinline__ void stage(StageRec<double>* p, double px, double py,
                                               double ox, double oy, double w, uint64_t hid,
                                               int cell) {
    double2* o = reinterpret_cast<double2*>(p);
    o[0] = make_double2(px, py);
    o[1] = make_double2(ox, oy);
    o[2] = make_double2(w, __longlong_as_double((long long)hid));
    o[3] = make_double2(__longlong_as_double((long long)(unsigned)cell), 0.0);
  }
  static __device__ __forceinline__ void put_src(SrcRec<double>* p, double px, double py,
                                                 double ox, double oy, double w, double trel,
                                                 double tau, int cell, uint32_t lidx) {
    double2* o = reinterpret_cast<double2*>(p);
    o[0] = make_double2(px, py);
    o[1] = make_double2(ox, oy);
    o[2] = make_double2(w, trel);
    o[3] = make_double2(tau, __longlong_as_double((long long)(((uint64_t)lidx << 32) |
                                                              (uint32_t)cell)));
  }
};
template <> struct Real<float> {
  using V2 = float2;
  static __device__ __forceinline__ void scpi(float x, float* s, float* c) {
    sincospif(x, s, c);
  }
  static __device__ __forceinline__ SrcRec<float>* src(const PassArgs& a) { return a.src32; }
  static __device__ __forceinline__ float attenuate(float w, float z, float) {
    return w * expf(-z);
  }
  static __device__ __forceinline__ float2 mat(const PassArgs& a, int c) {
    return a.mat_id16 ? a.mtab32[a.mat_id16[c]] : a.mat32[c];
  }
  static __device__ __forceinline__ float inf() { return __builtin_huge_valf(); }
  static __device__ __forceinline__ const StageRec<float>* in(const PassArgs& a) {
    return a.in32;
  }
  static __device__ __forceinline__ StageRec<float>* out(const PassArgs& a) { return a.out32; }
  static __device__ __forceinline__ void stage(StageRec<float>* p, float px, float py, float ox,
                                               float oy, float w, uint64_t hid, int cell) {
    float4* o = reinterpret_cast<float4*>(p);
    o[0] = make_float4(px, py, ox, oy);
    o[1] = make_float4(w, __int_as_float(cell), __uint_as_float((unsigned)hid),
                       __uint_as_float((unsigned)(hid >> 32)));
  }
  static __device__ __forceinline__ void put_src(SrcRec<float>* p, float px, float py, float ox,
                                                 float oy, float w, float trel, float tau,
                                                 int cell, uint32_t lidx) {
    float4* o = reinterpret_cast<float4*>(p);
    o[0] = make_float4(px, py, ox, oy);
    o[1] = make_float4(w, trel, tau, __int_as_float(cell));
    o[2] = make_float4(__uint_as_float(lidx), 0.f, 0.f, 0.f);
    o[3] = make_float4(0.f, 0.f, 0.f, 0.f);  // the padding too: whole sectors
  }
};

enum { END_NONE = 0, END_CENSUS, END_LEAK, END_CUTOFF };

// States of a lane: without a history, tracking one, its history at a
// collision, its history at its end.  A segment is cheap and every iteration
// has one for each running lane; a collision (three points, a sine and cosine,
// a logarithm) and the change from a finished history to the next (balance,
// census record, bank record, first optical depth) cost as much as several
// segments, and in any one iteration only a few lanes are there.  So lanes
// wait until a quarter of the wave's live lanes have a collision, or kRefillAt
// lanes are free, or none runs.  (The order of a wave's work does not show in
// the results.)  1024^2, N_s = 3, 2e8 histories: passes of 27.1 and 21.4 ms
// served at once, 21.9 / 19.9 with 12 free and 8 colliding lanes, 20.5 / 18.6
// as here, 22.3 / 18.7 with 32 and 24 (all before the segment's branches went;
// since then 17.4 / 15.4, 17.9 / 15.9 with 18 free, and a third colliding the
// same; all in a run's third step: in the mean of 50 the passes take 18.5 and
// 15.7); 30x50 steady, where a wave has 16 histories: 0.38 ms at once, 0.43
// with twelve colliding lanes, 0.34 with a quarter of the live ones.
enum { LN_IDLE = 0, LN_RUN, LN_COL, LN_END };
constexpr int kRefillAt = 24;
constexpr int kCollideShare = 4;

__device__ __forceinline__ double maxabs4(const double* q) {
  return fmax(fmax(fabs(q[0]), fabs(q[1])), fmax(fabs(q[2]), fabs(q[3])));
}

// Bilinear interpolation of nodal values (nodes (0,0),(1,0),(0,1),(1,1)) at
// local coordinates (a, b); equal corners give exactly q[0].
__device__ __forceinline__ double bilinear(const double* q, double a, double b) {
  return q[0] + a * (q[1] - q[0]) + b * (q[2] - q[0]) + a * b * (q[0] - q[1] - q[2] + q[3]);
}

// Cell of source particle s: descend the count tree (leaf i = n_i, exact
// integers) with target s + 1/2, going left while the target is below the
// left count, else subtracting it and going right.  Particles are numbered
// in cell order, so this finds the cell j with P_j <= s < P_j + n_j
// (P_j = counts of the cells before j), and l = s - P_j.  A thread descends
// NP particles' paths together, one level at a time, so that their loads of
// the lower levels (from global memory) are in flight at once.
constexpr int kTreeTop = 1024;  // nodes [0, kTreeTop) of the tree are staged in LDS

struct CellPick {
  long long cell;
  uint32_t l;
};

template <int NP>
__device__ __forceinline__ void count_pick_n(const double* __restrict__ t,
                                             const double* __restrict__ top, long long L,
                                             const long long* s, CellPick* out) {
  double target[NP];
  long long k[NP];
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    target[j] = (double)s[j] + 0.5;
    k[j] = 1;
  }
  // at the level of nodes [lev, 2 lev) the children [2 lev, 4 lev) are all
  // in LDS or all in global memory
  for (long long lev = 1; lev < L; lev <<= 1) {
    const bool in_lds = 4 * lev <= kTreeTop;
    double2 lr[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j)
      lr[j] = in_lds ? make_double2(top[2 * k[j]], top[2 * k[j] + 1])
                     : reinterpret_cast<const double2*>(t)[k[j]];
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      if (target[j] < lr[j].x || lr[j].y == 0.0) {  // (an empty right subtree is never reached)
        k[j] = 2 * k[j];
      } else {
        target[j] -= lr[j].x;
        k[j] = 2 * k[j] + 1;
      }
    }
  }
#pragma unroll
  for (int j = 0; j < NP; ++j)
    out[j] = CellPick{k[j] - L, (uint32_t)target[j]};  // target = s - P_j + 1/2
}

// One fixed-point tally add.  A copy is only ever added to by workgroups of one
// XCD, so a workgroup-scope atomic, resolved in that XCD's L2, is exact;
// kernel boundaries write the L2 back before the copies are summed.
__device__ __forceinline__ void tally_add(unsigned long long* p, unsigned long long v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Work indices a wave takes from the pass's counter at a time (on the
// 1024x1024 solve 1024 gave the shortest passes: 64 queue on the counter,
// 16384 balance worse).
constexpr long long kWorkChunk = 1024;

// Tally-word cache of a wave in LDS: kTcSlots slots of (word, pending sum).  A
// lane's add goes to the slot its word hashes to: into the slot's sum when
// the slot holds that word or is free (claimed with a compare and swap), else
// straight to the tally.  Every kTcFlush loop iterations, and at the end, the
// wave adds each held sum to its word and frees the slots.  The histories of
// a wave start on neighbouring work items (cell order) and stay near each
// other, so many adds of a busy region meet in the cache instead of queueing
// at the same L2 lines; integer sums make the result the same as with one
// atomic per add.  FP64: 512 slots per wave (24 KB per block),
// three blocks per compute unit, which the registers allow; FP32: 256, four
// blocks (256^2, 2e7 histories: passes of 0.87 and 0.65 ms against 0.97 and
// 0.68 with three).
//
// The hash is multiplicative and the copy is the wave's: the cells that a wave
// visits are a disc of the mesh, whose rows fell on the same slots by the low
// bits of their words where the mesh has 2^k columns, and whose words were as
// many as copies where each lane had its own (1024^2, 1e8 particles, 1e9 adds
// a pass: six in ten went past the cache; the passes take 30.2 and 21.1 ms
// against 33.6 and 29.9, and 28.7 and 20.3 without any tally).  Flushing every
// 16, 32, 64, 128 iterations: 30.5, 30.2, 30.2, 30.4 ms.
template <typename R> constexpr int kTcBits = sizeof(R) == 4 ? 8 : 9;
template <typename R> constexpr int kPassWaves = sizeof(R) == 4 ? 4 : 3;  // per SIMD
constexpr int kTcFlush = 32;

// Copies of a tracking block's balance in LDS (odd stride: the copies start
// in different banks).
constexpr int kBalCopies = 8;
constexpr int kBalStride = 2 * B_NFIELDS + 1;

// Adds v, in fixed point (hi, lo) of unit 1/inv_W, to balance field f.
__device__ __forceinline__ void bal_add(unsigned long long* bal, int f, double v, double inv_W) {
  long long hi, lo;
  fix_split(v, inv_W, hi, lo);
  atomicAdd(&bal[2 * f], (unsigned long long)hi);
  atomicAdd(&bal[2 * f + 1], (unsigned long long)lo);
}

// A value every lane of the wave holds alike (read from the solver state,
// which the compiler cannot take as uniform), moved to scalar registers so
// that it takes no vector register in the tracking loop.
__device__ __forceinline__ long long wave_uniform(long long v) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v);
  const unsigned hi =
      (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)((unsigned long long)v >> 32));
  return (long long)(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double wave_uniform(double v) {
  return __longlong_as_double(wave_uniform((long long)__double_as_longlong(v)));
}
__device__ __forceinline__ float wave_uniform(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// Emission of the pass's source particles (Sec. 2.3: birth proportional to
// q, isotropic direction, weights that integrate q in expectation),
// stratified by cell: cell j emits the n_j particles of the emission plan
// (floor(r_j) or floor(r_j) + 1, E[n_j] = r_j = M_j / w_q), numbered in cell
// order.  Particle l of cell j takes its points from the cell's stream at
// index l: position (dims 0-1), birth time (dim 2), direction (dims 3-4,
// sincospi), the first optical depth (dim 5) when the pass allows scatters,
// and weight w_q q(x,y) / qbar_j, qbar_j the cell's power-of-two majorant of
// |q| (so |w| <= w_q; the expected weight of the cell is r_j w_q mean(q) /
// qbar_j = A dt mean(q), or A mean(q) per unit time in steady state, where
// every particle starts at time 0).
//
// A thread emits runs of consecutive particles, up to kEmitRun of them when
// the plan has that many per thread of the grid (one otherwise, so that a
// small plan still spreads over the whole grid).  With tens of particles per
// cell a run nearly always lies in one emitter: the descents of its first
// and last particles then show it, and the emitter's stream and
// per-dimension scramble seeds are computed once for the run.  A run that
// spans emitters descends the tree for each of its inner particles.
//
// The records of a wave's particles leave through LDS: a lane's record is four
// 16-byte words, and lanes of a run apart would write one word to each of 64
// sectors in every store; transposed, four neighbouring lanes write one whole
// 64-byte record (1e7 particles on 256^2: FP64 0.32 -> 0.26 ms, FP32 0.33 ->
// 0.24, with the six dimensions' tables loaded instead of built).
constexpr long long kEmitRun = 8;
constexpr int kEmitDims = 6;   // dimensions that a source particle's emission draws
constexpr int kEmitWaves = 4;  // waves per block
constexpr int kEmitRow = 5;    // LDS words of 16 bytes per record (padded against conflicts)

template <typename R, int KIND>
__global__ __launch_bounds__(256) void k_emit(PassArgs a) {
  if (a.st->halt) return;
  __shared__ __align__(16) uint32_t s_sobol[kEmitDims * 128];
  __shared__ double s_top[kTreeTop];
  __shared__ uint4 s_rec[kEmitWaves][64 * kEmitRow];
  sobol_nibbles_load(a.sobol, s_sobol, kEmitDims, threadIdx.x, blockDim.x);
  {
    const long long ntop = 2 * a.tree_L < kTreeTop ? 2 * a.tree_L : kTreeTop;
    for (int k = threadIdx.x; k < kTreeTop; k += blockDim.x)
      s_top[k] = (k >= 1 && k < ntop) ? a.ctree[k] : 0.0;
  }
  __syncthreads();
  const long long n_emit = a.st->n_emit;  // the plan's count, clamped to the bank
  const uint64_t step = a.st->step;
  const double wq = a.st->wq[KIND - 1];
  const R hx = (R)a.hx, hy = (R)a.hy, dt_birth = (R)a.dt_birth;
  SrcRec<R>* const b = Real<R>::src(a);
  const long long T = (long long)gridDim.x * blockDim.x;
  const long long run = n_emit / T < 1 ? 1 : (n_emit / T > kEmitRun ? kEmitRun : n_emit / T);
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  SrcRec<R>* const row = reinterpret_cast<SrcRec<R>*>(s_rec[wv] + lane * kEmitRow);
  uint4* const out = reinterpret_cast<uint4*>(b);
  static_assert(sizeof(SrcRec<R>) == 4 * sizeof(uint4), "a record is four words");
  // the wave's particles [w0, w0 + 64 run), the lane's run from r0
  for (long long w0 = ((long long)blockIdx.x * kEmitWaves + wv) * 64 * run; w0 < n_emit;
       w0 += run * T) {
    const long long r0 = w0 + lane * run;
    const long long r1 = (r0 + run < n_emit ? r0 + run : n_emit) - 1;
    // (a lane past the last particle looks up the last one)
    long long sj[2] = {r0 < n_emit ? r0 : n_emit - 1, r1};
    CellPick pk[2];
    count_pick_n<2>(a.ctree, s_top, a.tree_L, sj, pk);
    const bool one = pk[0].cell == pk[1].cell;
    long long cur = -1;  // the emitter whose stream and seeds are held
    uint64_t stream = 0;
    uint32_t sd[6];
#pragma unroll 1
    for (int k = 0; k < (int)run; ++k) {
      const long long s = r0 + k;
      if (s <= r1) {
        CellPick pc;
        if (one) pc = CellPick{pk[0].cell, pk[0].l + (uint32_t)(s - r0)};
        else if (s == r0) pc = pk[0];
        else if (s == r1) pc = pk[1];
        else count_pick_n<1>(a.ctree, s_top, a.tree_L, &s, &pc);
        const long long ci = pc.cell;  // the emitter: a cell, or a boundary face after them
        const uint32_t l = pc.l;
        if (ci != cur) {
          cur = ci;
          stream = stream_seed(a.seed, step, (uint32_t)KIND, 0u, (uint64_t)ci);
#pragma unroll
          for (int d = 0; d < 6; ++d) sd[d] = point_seed(stream, (uint32_t)d);
        }
        const R u1 = PointU<R>::u(point_u32s(s_sobol, a.points, stream, sd[0], 0u, l));
        const R u2 = PointU<R>::u(point_u32s(s_sobol, a.points, stream, sd[1], 1u, l));
        const R u3 = PointU<R>::u(point_u32s(s_sobol, a.points, stream, sd[2], 2u, l));
        const R u4 = PointU<R>::u(point_u32s(s_sobol, a.points, stream, sd[3], 3u, l));
        const R tau = a.n_lim > 0
                          ? -log(PointU<R>::u(point_u32s(s_sobol, a.points, stream, sd[5], 5u, l)))
                          : (R)0;
        if (ci < a.n_cells) {
          const R u5 = PointU<R>::u(point_u32s(s_sobol, a.points, stream, sd[4], 4u, l));
          const R sn = (R)2 * sqrt(u4 * ((R)1 - u4));
          R sp, cp;
          Real<R>::scpi((R)2 * u5, &sp, &cp);
          const double* q = a.qn + 4 * ci;
          const double wscale = wq / pow2_ceil(maxabs4(q));  // exact: a power-of-two ratio
          const R w = (R)(bilinear(q, (double)u1, (double)u2) * wscale);
          Real<R>::put_src(row, hx * u1, hy * u2, sn * cp, sn * sp, w, u3 * dt_birth, tau,
                           (int)ci, l);
        } else {
          // entering through boundary face f (the inflow G): uniform along the
          // face (dim 0) and in time (dim 1), the cosine law about the inward
          // normal, mu = sqrt(u) (dim 2), the in-plane tangential component
          // sqrt(1 - mu^2) cos(2 pi u) (dim 3); weight w_q G_f / pow2_ceil(|G_f|)
          int along;
          const int f = (int)(ci - a.n_cells);
          const int side = face_side(f, a.nx, a.ny, &along);
          const R mu = sqrt(u3);
          R sp, cp;
          Real<R>::scpi((R)2 * u4, &sp, &cp);
          const R tg = sqrt((R)1 - u3) * cp;
          const double G = a.em.inflow[f];
          const R w = (R)(G * (wq / pow2_ceil(fabs(G))));
          R px, py, ox, oy;
          if (side < 2) {
            px = side == 0 ? (R)0 : hx;
            py = hy * u1;
            ox = side == 0 ? mu : -mu;
            oy = tg;
          } else {
            px = hx * u1;
            py = side == 2 ? (R)0 : hy;
            oy = side == 2 ? mu : -mu;
            ox = tg;
          }
          Real<R>::put_src(row, px, py, ox, oy, w, u2 * dt_birth, tau, (int)ci, l);
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int of = (64 * j + lane) >> 2, part = lane & 3;  // whose record, which word
        const long long d = w0 + of * run + k;
        if (d < n_emit) out[4 * d + part] = s_rec[wv][of * kEmitRow + part];
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  }
}

template <typename R, int KIND>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kPassWaves<R>)))
void k_mc_pass(PassArgs a) {
  if (a.st->halt) return;
  constexpr int kTcSlots = 1 << kTcBits<R>;
  // Block balance in kBalCopies LDS copies picked by lane: with a per-lane
  // address the adds are plain LDS atomics, where one shared address would
  // make the compiler serialise them over the active lanes in a scalar loop.
  // The emitted weight is not added per history: it is the sum of the source
  // and census-in weights (exact in fixed point).
  __shared__ unsigned long long s_bal[kBalCopies * kBalStride];
  __shared__ unsigned long long s_cnt[4];
  __shared__ __align__(16) uint32_t s_sobol[kSobolNibbleWords];
  __shared__ unsigned s_tc_tag[4 * kTcSlots];  // four waves per block
  __shared__ unsigned long long s_tc_sum[4 * kTcSlots];
  for (int k = threadIdx.x; k < 4 * kTcSlots; k += blockDim.x) {
    s_tc_tag[k] = 0u;
    s_tc_sum[k] = 0ull;
  }
  for (int k = threadIdx.x; k < kBalCopies * kBalStride; k += blockDim.x) s_bal[k] = 0ull;
  if (threadIdx.x < 4) s_cnt[threadIdx.x] = 0ull;
  sobol_nibbles_load(a.sobol, s_sobol, kSobolDims, threadIdx.x, blockDim.x);
  __syncthreads();

  DevState* st = a.st;
  const int lane = __lane_id();
  const long long n_in = wave_uniform(st->n_in);
  const long long n_emit = wave_uniform(st->n_emit);  // the plan's count, clamped to the bank
  const unsigned long long n_tot = (unsigned long long)(n_in + n_emit);
  const double w_q = wave_uniform(st->wq[KIND - 1]);
  const R w_cut = wave_uniform((R)(a.w_cut_rel * w_q));
  const double inv_T = wave_uniform(st->inv_T);
  const double inv_W = wave_uniform(st->inv_W);
  const uint64_t step = (uint64_t)wave_uniform((long long)st->step);
  const uint64_t thin_stream = KIND == 2 ? thin_stream_seed(a.seed, step) : 0ull;
  const R hx = (R)a.hx, hy = (R)a.hy, dt = (R)a.dt, c = (R)a.c;
  const R INF = Real<R>::inf();
  const StageRec<R>* const bin = Real<R>::in(a);
  StageRec<R>* const bout = Real<R>::out(a);
  const int n_lim = a.n_lim;

  int ls = LN_IDLE;     // the lane's state
  int end = END_NONE;   // how its history ended (LN_END)
  long long q_next = 0, q_end = 0;  // the wave's current chunk of work indices (uniform)
  bool q_done = false;              // no chunk is left for this wave
  const long long n_wv = (long long)gridDim.x * (blockDim.x / 64);
  const long long per_wave = (long long)n_tot / n_wv;
  const bool q_dyn = per_wave >= 4 * kWorkChunk;  // chunks from the pass's counter
  const long long chunk = q_dyn ? kWorkChunk : (per_wave / 8 > 16 ? per_wave / 8 : 16);
  // (the wave's index, read as a wave-uniform value so that the chunk state
  // stays in scalar registers)
  long long q_chunk = (long long)blockIdx.x * (blockDim.x / 64) +
                      __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  // tally copy of this wave, one of its XCD's (the hardware XCC id, not the
  // dispatch order, decides which L2 resolves the adds)
  unsigned xcc = 0;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
  constexpr unsigned per = kTallyCopies / kNumXcd;
  const long long my_copy =
      (long long)(xcc % kNumXcd * per + (unsigned)q_chunk % per) * a.copy_stride;
  // A tally word is named by 1 + its cell, in the scatter-limited pass 1 + 2
  // cell + (1 after the limit); 0 names none.
  unsigned long long* const Ta = a.Ta + my_copy;
  unsigned long long* const Tb = a.Tb + my_copy;
  auto to_tally = [&](unsigned word, unsigned long long v) __attribute__((always_inline)) {
    const unsigned k = word - 1u;
    if (KIND == 2) tally_add(Tb + kTallyStride * (size_t)k, v);
    else tally_add((k & 1u ? Tb : Ta) + kTallyStride * (size_t)(k >> 1), v);
  };
  long long g = 0;
  unsigned p_word = 0u;  // the lane's pending tally word and sum
  unsigned long long p_val = 0ull;
  // material of the history's current cell, loaded when the history starts
  // and, after a face crossing, at the end of the iteration, so that the
  // gather is in flight while the loop turns around
  typename Real<R>::V2 m_cur;
  m_cur.x = (R)0;
  m_cur.y = (R)0;
  R px = 0, py = 0, ox = 0, oy = 0, w = 0, trel = 0, tau = 0;
  R iox = 0, ioy = 0;  // 1/ox, 1/oy (0 for a zero component)
  int ix = 0, iy = 0, n = 0;
  uint64_t stream = 0, hid = 0;
  uint32_t pidx = 0, dcur = 0, seg_p = 0;
  double w0 = 0.0, acc_abs = 0.0, acc_sca = 0.0;
  bool from_census = false;
  unsigned int lane_seg = 0, lane_hist = 0, lane_alive = 0, lane_killed = 0, lane_bad = 0;
  unsigned long long* my_bal = s_bal + (lane % kBalCopies) * kBalStride;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // wave in the block
  unsigned* const tc_tag = s_tc_tag + wv * kTcSlots;
  unsigned long long* const tc_sum = s_tc_sum + wv * kTcSlots;
  int tc_it = 0;
  // the wave's held sums to their words (all lanes of the wave together)
  auto tc_flush = [&]() __attribute__((always_inline)) {
    for (int k = lane; k < kTcSlots; k += 64) {
      const unsigned tg = tc_tag[k];
      if (tg) {
        to_tally(tg, tc_sum[k]);
        tc_tag[k] = 0u;
        tc_sum[k] = 0ull;
      }
    }
  };

  for (;;) {
    const unsigned long long m_run = __ballot(ls == LN_RUN);
    const bool more = !q_done || q_next < q_end;  // work is left for this wave
    const unsigned long long m_free = __ballot(ls == LN_END || (more && ls == LN_IDLE));
    bool fresh = false;
    if (m_free && (!m_run || __popcll(m_free) >= kRefillAt)) {
      if (ls == LN_END) {
        if (KIND == 2 && end == END_CENSUS && a.keep_census) {
          const long long slot = from_census ? g : a.out_src_base + (g - n_in);
          Real<R>::stage(bout + slot, px, py, ox, oy, w, hid, iy * a.nx + ix);
          a.alive[slot] =
              (uint8_t)(kAliveBit | (unsigned)(mix64(thin_stream ^ hid) >> kThinShift));
          a.cell[slot] = iy * a.nx + ix;
          lane_alive++;
        }
        // fold the history's balance into the block (fixed point, exact)
        const double wend = (double)w;
        if (!isfinite(wend) || !isfinite(acc_abs) || !isfinite(acc_sca)) lane_bad++;
        bal_add(my_bal, from_census ? B_CENSUS_IN_W : B_SOURCE_W, w0, inv_W);
        bal_add(my_bal, B_ABSORBED, acc_abs, inv_W);
        if (acc_sca != 0.0) bal_add(my_bal, B_SCATTERED, acc_sca, inv_W);
        bal_add(my_bal, end == END_CENSUS ? B_CENSUS : (end == END_LEAK ? B_LEAKED : B_CUTOFF),
                wend, inv_W);
        ls = LN_IDLE;
      }
      // idle lanes take the next indices of the wave's chunk, in lane order; a
      // used-up chunk is replaced by the wave's next one
      if (q_next >= q_end && !q_done) {
        unsigned long long base = 0ull;
        if (q_dyn) {
          if (lane == 0) base = atomicAdd(&st->work, (unsigned long long)chunk);
          base = (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)base) |
                 ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane(
                      (int)(unsigned)(base >> 32)) << 32);
        } else {
          base = (unsigned long long)(q_chunk * chunk);
          q_chunk += n_wv;
        }
        q_next = base < n_tot ? (long long)base : (long long)n_tot;
        q_end = base + chunk < n_tot ? (long long)(base + chunk) : (long long)n_tot;
        q_done = base + chunk >= n_tot;
      }
      const unsigned long long need = __ballot(ls == LN_IDLE);
      const uint32_t rank = __builtin_amdgcn_mbcnt_hi(
          (uint32_t)(need >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)need, 0u));
      const long long avail = q_end - q_next;
      if (ls == LN_IDLE && (long long)rank < avail) {
        g = q_next + rank;
        fresh = true;
      }
      q_next += (long long)__popcll(need) < avail ? (long long)__popcll(need) : avail;
    }
    if (fresh) {
      ls = LN_RUN;
      lane_hist++;
      seg_p = 0;
      acc_abs = 0.0;
      acc_sca = 0.0;
      n = 0;
      if (g < n_in) {
        // census particle at the start of the step, counter reset
        from_census = true;
        const StageRec<R> rec = bin[g];
        px = rec.px; py = rec.py; ox = rec.ox; oy = rec.oy; w = rec.w;
        const int cell = rec.cell;
        ix = cell % a.nx; iy = cell / a.nx;
        hid = rec.hid;
        trel = (R)0;
        // census_qmc: its cell's census cohort, the cell's census stream at
        // the particle's rank in the cohort (the bank is ordered by cell);
        // else its own stream, keyed by its identity, at point index 0
        if (KIND == 1 && n_lim > 0) {
          stream = stream_seed(a.seed, step, (uint32_t)KIND, 1u,
                               a.census_qmc ? (uint64_t)cell : hid);
          pidx = a.census_qmc ? a.in_rank[g] : 0u;
        } else {
          stream = 0ull;
          pidx = 0u;
        }
        dcur = 0;
      } else {
        // source particle, emitted by k_emit
        from_census = false;
        const SrcRec<R> sr = Real<R>::src(a)[g - n_in];
        px = sr.px; py = sr.py; ox = sr.ox; oy = sr.oy; w = sr.w;
        trel = sr.trel;
        tau = sr.tau;
        const int cell = sr.cell;  // the emitter: a cell, or a boundary face after them
        pidx = sr.lidx;
        if (cell < a.n_cells) {
          ix = cell % a.nx; iy = cell / a.nx;
        } else {  // the cell inside boundary face f
          int k;
          const int side = face_side(cell - (int)a.n_cells, a.nx, a.ny, &k);
          ix = side < 2 ? (side == 0 ? 0 : a.nx - 1) : k;
          iy = side < 2 ? k : (side == 2 ? 0 : a.ny - 1);
        }
        // the emitter's stream at the particle's index in it
        stream = stream_seed(a.seed, step, (uint32_t)KIND, 0u, (uint64_t)cell);
        hid = history_id(step, cell, pidx);
        dcur = 6;  // dims 0-4 emission, 5 the first optical depth
      }
      iox = ox != (R)0 ? (R)1 / ox : (R)0;
      ioy = oy != (R)0 ? (R)1 / oy : (R)0;
      w0 = (double)w;
      m_cur = Real<R>::mat(a, iy * a.nx + ix);
      if (from_census && n_lim > 0) {
        tau = -log(PointU<R>::u(point_u32n(s_sobol, a.points, stream, 0u, pidx)));
        dcur = 1;
      }
    }
    const unsigned long long m_col = __ballot(ls == LN_COL);
    if (m_col && (!m_run || kCollideShare * __popcll(m_col) >= __popcll(m_col | m_run))) {
      if (ls == LN_COL) {
        // isotropic re-emission, scatter counter n <- n + 1
        const R ua = PointU<R>::u(point_u32n(s_sobol, a.points, stream, dcur, pidx));
        const R ub = PointU<R>::u(point_u32n(s_sobol, a.points, stream, dcur + 1u, pidx));
        dcur += 2;
        const R sn = (R)2 * sqrt(ua * ((R)1 - ua));
        R sp, cp;
        Real<R>::scpi((R)2 * ub, &sp, &cp);
        ox = sn * cp;
        oy = sn * sp;
        iox = ox != (R)0 ? (R)1 / ox : (R)0;
        ioy = oy != (R)0 ? (R)1 / oy : (R)0;
        n++;
        if (n < n_lim) {
          tau = -log(PointU<R>::u(point_u32n(s_sobol, a.points, stream, dcur, pidx)));
          dcur++;
        }
        ls = LN_RUN;
      }
    }
    if (!__any(ls == LN_RUN)) break;  // no lane runs, collides or ends, and no work is left
    // One segment of each running lane.  The passes are bound by the issue of
    // vector instructions, and a branch here would be taken by some lane of the
    // wave and, where its sides leave different values, cost a register copy per
    // value: the event is a set of lane masks, and the new state is selected by
    // them (290 -> 190 vector instructions a segment; 1024^2, 1e8 particles,
    // N_s = 3, third step of a run: passes of 20.1 and 18.1 -> 17.4 and 15.4 ms; 256^2
    // FP32, 1e7: 0.86 and 0.67 -> 0.76 and 0.56).
    if (ls == LN_RUN) {
      const int cell = iy * a.nx + ix;
      const R ss = m_cur.x, sa = m_cur.y, stt = sa + ss;
      const bool pre = n < (a.ns_cell ? a.ns_cell[cell] : n_lim);
      R d_cen = c * (dt - trel);
      if (d_cen < (R)0) d_cen = (R)0;
      R d_col = INF;
      if (pre && ss > (R)0) { d_col = tau / ss; if (d_col < (R)0) d_col = (R)0; }
      const bool right = ox > (R)0, up = oy > (R)0;
      R d_x = ((right ? hx : (R)0) - px) * iox, d_y = ((up ? hy : (R)0) - py) * ioy;
      if (d_x < (R)0) d_x = (R)0;
      if (d_y < (R)0) d_y = (R)0;
      if (ox == (R)0) d_x = INF;
      if (oy == (R)0) d_y = INF;
      R l = d_cen;
      const bool by_col = d_col < l;
      if (by_col) l = d_col;
      const bool by_x = d_x < l;
      if (by_x) l = d_x;
      const bool cross_y = d_y < l;
      if (cross_y) l = d_y;
      const bool cross_x = by_x && !cross_y;
      const bool collide = by_col && !by_x && !cross_y;
      const bool census = !by_col && !by_x && !cross_y;

      const R sig = pre ? sa : stt;
      const R z = sig * l;
      const R em = expm1(-z);  // e^{-z} - 1
      const R contrib = (sig > (R)0) ? w * (-em) / sig : w * l;
      const unsigned t_word =
          1u + (KIND == 2 ? (unsigned)cell : 2u * (unsigned)cell + (pre ? 0u : 1u));
      const double cd = (double)contrib;
      const unsigned long long t_val = (unsigned long long)fix_round(cd, inv_T);
      acc_abs += (double)sa * cd;
      if (!pre) acc_sca += (double)ss * cd;
      w = Real<R>::attenuate(w, z, em);
      if (pre && ss > (R)0) tau -= ss * l;
      trel += l / c;
      seg_p++;
      lane_seg++;

      const R nx_p = px + ox * l, ny_p = py + oy * l;
      // a reflective side mirrors the direction; the history stays in its cell
      bool mir_x = false, mir_y = false;
      if (a.bc) {
        mir_x = cross_x && ix == (right ? a.nx - 1 : 0) && (a.bc & (right ? 2 : 1));
        mir_y = cross_y && iy == (up ? a.ny - 1 : 0) && (a.bc & (up ? 8 : 4));
        ox = mir_x ? -ox : ox;
        iox = mir_x ? -iox : iox;
        oy = mir_y ? -oy : oy;
        ioy = mir_y ? -ioy : ioy;
      }
      px = cross_x ? (right != mir_x ? (R)0 : hx) : nx_p;
      py = cross_y ? (up != mir_y ? (R)0 : hy) : ny_p;
      ix += cross_x && !mir_x ? (right ? 1 : -1) : 0;
      iy += cross_y && !mir_y ? (up ? 1 : -1) : 0;
      const bool leak = (unsigned)ix >= (unsigned)a.nx || (unsigned)iy >= (unsigned)a.ny;
      const bool killed = seg_p >= a.max_segments;
      const bool over = census || leak, cut = fabs(w) < w_cut;
      lane_killed += killed && !over && !cut ? 1u : 0u;
      end = census ? END_CENSUS : (leak ? END_LEAK : END_CUTOFF);
      ls = over || cut || killed ? LN_END : (collide ? LN_COL : LN_RUN);
      // the next cell's material before the tally atomic: memory operations
      // complete in issue order, so the wait for the material at the next
      // segment does not include the atomic's round trip
      if (ls == LN_RUN) m_cur = Real<R>::mat(a, iy * a.nx + ix);

      // A lane's consecutive adds to one word (segments that end in a
      // collision or at the census stay in their cell) are summed in registers;
      // the pending sum goes to the wave's cache when the lane moves to another
      // word.
      const bool same = t_word == p_word;
      const unsigned f_word = same ? 0u : p_word;
      const unsigned long long f_val = p_val;
      p_val = (same ? p_val : 0ull) + t_val;
      p_word = t_word;
      if (f_word) {
        const int slot = (int)((f_word * 0x9E3779B1u) >> (32 - kTcBits<R>));
        unsigned tg = tc_tag[slot];
        if (tg == 0u) {
          const unsigned old = atomicCAS(&tc_tag[slot], 0u, f_word);
          tg = old == 0u ? f_word : old;
        }
        if (tg == f_word) atomicAdd(&tc_sum[slot], f_val);
        else to_tally(f_word, f_val);
      }
    }
    if (++tc_it == kTcFlush) {
      tc_it = 0;
      tc_flush();
    }
  }

  if (p_word) to_tally(p_word, p_val);  // the last pending add
  tc_flush();

  // wave totals of the integer counters, one atomic per wave
  unsigned long long v0 = lane_seg, v1 = lane_hist, v2 = lane_alive, v3 = lane_killed;
  for (int off = 32; off > 0; off >>= 1) {
    v0 += __shfl_xor(v0, off);
    v1 += __shfl_xor(v1, off);
    v2 += __shfl_xor(v2, off);
    v3 += __shfl_xor(v3, off);
  }
  if (lane_bad) atomicOr(&st->numeric, 2);
  if (lane == 0) {
    atomicAdd(&s_cnt[0], v0);
    atomicAdd(&s_cnt[1], v1);
    atomicAdd(&s_cnt[2], v2);
    atomicAdd(&s_cnt[3], v3);
  }
  __syncthreads();
  if (threadIdx.x < 2 * B_NFIELDS) {
    const int f = threadIdx.x >> 1, wd = threadIdx.x & 1;
    unsigned long long v = 0ull;
    for (int k = 0; k < kBalCopies; ++k) {
      const unsigned long long* b = s_bal + k * kBalStride;
      v += f == B_EMITTED ? b[2 * B_SOURCE_W + wd] + b[2 * B_CENSUS_IN_W + wd] : b[threadIdx.x];
    }
    if (v) atomicAdd(&st->bal[threadIdx.x], v);
  } else if (threadIdx.x >= 64 && threadIdx.x < 68) {
    const int k = threadIdx.x - 64;
    unsigned long long* dst = k == 0 ? &st->segments
                              : k == 1 ? &st->particles
                              : k == 2 ? &st->alive : &st->killed;
    if (s_cnt[k]) atomicAdd(dst, s_cnt[k]);
  }
}

// Blocks of the persistent tracking grid: as many as can be resident at once
// (occupancy x compute units), never more than the work needs.
int mc_pass_grid(bool fp32, int kind, long long max_work) {
  // solvers and servers are created from several threads: every thread that
  // finds the entry empty computes the same value and stores it atomically
  static std::atomic<int> cached[2][2];
  std::atomic<int>& slot = cached[fp32 ? 1 : 0][kind == 1 ? 0 : 1];
  int nb = slot.load(std::memory_order_relaxed);
  if (nb == 0) {
    int dev = 0, cus = 0, per = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    hipError_t e;
    if (kind == 1)
      e = fp32 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_mc_pass<float, 1>, 256, 0)
               : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_mc_pass<double, 1>, 256, 0);
    else
      e = fp32 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_mc_pass<float, 2>, 256, 0)
               : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_mc_pass<double, 2>, 256, 0);
    if (e != hipSuccess || per < 1) per = 2;
    if (cus < 1) cus = 256;
    nb = cus * per;
    slot.store(nb, std::memory_order_relaxed);
  }
  long long want = (max_work + 255) / 256;
  if (want > nb) want = nb;
  return (int)(want < 1 ? 1 : want);
}

hipError_t launch_emit(const PassArgs& a, bool fp32, hipStream_t s) {
  if (a.n_src <= 0) return hipSuccess;
  // Runs of eight on at most 2048 blocks; fewer particles first give up the
  // blocks above 1024 and then the length of their runs (1e6 particles: 38 us
  // on 1024 blocks in runs of four, 51 on 2048 in runs of one or two, 58 on
  // 512 in runs of eight; 1e7: 0.26 ms on 2048, 0.29 on 1280)
  const long long b = (a.n_src + 255) / 256;
  const long long few = b < 1024 ? b : 1024, runs = b / kEmitRun;
  const int grid = (int)(runs < few ? few : (runs < 2048 ? runs : 2048));
  if (a.kind == 1) {
    if (fp32) hipLaunchKernelGGL((k_emit<float, 1>), dim3(grid), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_emit<double, 1>), dim3(grid), dim3(256), 0, s, a);
  } else {
    if (fp32) hipLaunchKernelGGL((k_emit<float, 2>), dim3(grid), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_emit<double, 2>), dim3(grid), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_mc_pass(const PassArgs& a, bool fp32, int grid, hipStream_t s) {
  if (a.kind == 1) {
    if (fp32) hipLaunchKernelGGL((k_mc_pass<float, 1>), dim3(grid), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_mc_pass<double, 1>), dim3(grid), dim3(256), 0, s, a);
  } else {
    if (fp32) hipLaunchKernelGGL((k_mc_pass<float, 2>), dim3(grid), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_mc_pass<double, 2>), dim3(grid), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

// The tracking kernels' point function (nibble tables), one word per thread.
__global__ __launch_bounds__(256) void k_qmc_points(uint64_t stream, uint32_t dim0,
                                                    uint32_t nd, uint32_t idx0, uint32_t n,
                                                    int mode, const uint32_t* sobol,
                                                    uint32_t* out) {
  __shared__ __align__(16) uint32_t s_nib[kSobolNibbleWords];
  sobol_nibbles_load(sobol, s_nib, kSobolDims, threadIdx.x, blockDim.x);
  __syncthreads();
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long long)n * nd) return;
  const uint32_t k = (uint32_t)(t / nd), d = (uint32_t)(t % nd);
  out[t] = point_u32n(s_nib, mode, stream, dim0 + d, idx0 + k);
}

hipError_t launch_qmc_points(uint64_t stream, uint32_t dim0, uint32_t nd, uint32_t idx0,
                             uint32_t n, int mode, const uint32_t* sobol, uint32_t* out,
                             hipStream_t s) {
  const long long tot = (long long)n * nd;
  if (tot == 0) return hipSuccess;
  const int grid = (int)((tot + 255) / 256);
  hipLaunchKernelGGL(k_qmc_points, dim3(grid), dim3(256), 0, s, stream, dim0, nd, idx0, n,
                     mode, sobol, out);
  return hipGetLastError();
}

}  // namespace slh
