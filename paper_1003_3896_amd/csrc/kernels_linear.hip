// O(N) kernels of libnbody for gfx950: fused kick + drift + centre-of-mass partials, and the
// energy / momentum diagnostics.  All are HBM-bound; one block of kBlock threads
// handles one chunk of kChunk particles of one cluster, so per-cluster reductions never mix
// clusters.  Every reduction runs in a fixed order (bitwise reproducible).  The update's chunk
// partials are combined by a second kernel; the energy pass, which runs rarely, lets the last
// block of a cluster to finish (device-scope atomic counter) combine them and reset the counter.
#include "nb_device.h"

namespace nb {

enum { NB_FP32 = 0, NB_FP32C = 1, NB_FP32DS = 2, NB_FP64 = 3 };

// Returns true in every thread of the block that finished cluster `cl` last (after its partial
// was published by thread 0).
__device__ __forceinline__ bool last_block_of_cluster(int* counter, int nchunks) {
  __shared__ int s_last;
  __threadfence();
  if (threadIdx.x == 0) s_last = (atomicAdd(counter, 1) == nchunks - 1);
  __syncthreads();
  const bool last = s_last;
  if (last) __threadfence();
  return last;
}

// Sum of the j-ranges of a split (or deferred) one-sided cluster for its particle at (sorted) position
// li, in range order; pure-FP32 mode adds the ranges in FP32.
__device__ __forceinline__ void sum_ranges(const Args& a, const DevCluster& c, int li, bool r32, double& ax,
                                           double& ay, double& az, double& pt) {
  ax = ay = az = pt = 0.0;
  float fx = 0.0f, fy = 0.0f, fz = 0.0f, fp = 0.0f;
  constexpr int kBatch = 8;  // ranges in flight
  for (int s = 0; s < c.split; s += kBatch) {
    double4 p[kBatch];
#pragma unroll
    for (int b = 0; b < kBatch; ++b)
      p[b] = s + b < c.split ? a.part[c.part_off + (long long)(s + b) * c.n + li] : make_double4(0.0, 0.0, 0.0, 0.0);
#pragma unroll
    for (int b = 0; b < kBatch; ++b) {
      if (s + b >= c.split) break;
      if (r32) {
        fx += (float)p[b].x;
        fy += (float)p[b].y;
        fz += (float)p[b].z;
        fp += (float)p[b].w;
      } else {
        ax += p[b].x;
        ay += p[b].y;
        az += p[b].z;
        pt += p[b].w;
      }
    }
  }
  if (r32) {
    ax = fx;
    ay = fy;
    az = fz;
    pt = fp;
  }
}

// x + c y as the mode stores it.
__device__ __forceinline__ double axpy(bool r32, double c, double y, double x) {
  return r32 ? (double)fmaf((float)c, (float)y, (float)x) : fma(c, y, x);
}

// Rows of one band of the symmetric path (SymRows in nb_internal.h) for one particle, and the running sums
// of the bands before, in row order: thread q of Q (4 for clusters too small to fill the chip with one
// thread per particle, else 1) takes rows q, q + Q, ....  Returns true after the cluster's last band, with
// the particle's sums in the threads with q == 0 (all threads of the block must call it); else stores
// the running sums.  HBM-bound (24 bytes per particle and row).
template <int NC>
__device__ __forceinline__ bool sum_rows(const Args& a, const DevCluster& c, int li, bool valid, int q, int Q, int band,
                                         double (&sum)[NC], double (*sh)[4][64]) {
  const SymRows rows = sym_rows(c.n, c.nseg, NC == 4, c.sym_doubles);
  if (band < 0) band = rows.nbands - 1;
  const int n = c.n, r0 = rows.row0(band), r1 = rows.row1(band);
  double* const base = a.sym + c.part_off;
  double* const run = base + ((size_t)rows.cap + q) * NC * n + li;  // running sums (more than one band)
#pragma unroll
  for (int d = 0; d < NC; ++d) sum[d] = band ? run[(size_t)d * n] : 0.0;
  constexpr int kBatch = 8;  // rows in flight per thread
  const int first = r0 + ((q - r0) & (Q - 1));
  for (int r = first; r < r1; r += kBatch * Q) {
    double v[kBatch][NC];
#pragma unroll
    for (int b = 0; b < kBatch; ++b)
#pragma unroll
      for (int d = 0; d < NC; ++d)
        v[b][d] = r + b * Q < r1 ? base[((size_t)(r + b * Q - r0) * NC + d) * n + li] : 0.0;
#pragma unroll
    for (int b = 0; b < kBatch; ++b)
      if (r + b * Q < r1)
#pragma unroll
        for (int d = 0; d < NC; ++d) sum[d] += v[b][d];
  }
  if (band < rows.nbands - 1) {
    if (valid)
#pragma unroll
      for (int d = 0; d < NC; ++d) run[(size_t)d * n] = sum[d];
    return false;
  }
  if (Q > 1) {
    const int e = threadIdx.x & 63;
#pragma unroll
    for (int d = 0; d < NC; ++d) sh[d][q][e] = sum[d];
    __syncthreads();
    if (q == 0)
#pragma unroll
      for (int d = 0; d < NC; ++d)
        for (int s = 1; s < Q; ++s) sum[d] += sh[d][s][e];
  }
  return true;
}

// Kick (v += kick_pre a) and drift (x += drift v) of one chunk (when `update`), and the chunk's
// partial sums for its cluster's reference point ref = sum m x / sum m of the (new) positions,
// mass-uniformity flag and bounding box (combined by k_reduce or chunk_frame: a kernel boundary rather
// than a device-scope fence orders the two, a fence would write back the XCD's L2 in every block).
// FINISH: a stage of an integrator step ends and the next begins; the pass first adds the pair sums of the
// clusters that were not finished before it (symmetric: the last band's rows; small one-sided clusters:
// their j-ranges), stores the acceleration and ends the stage with its kick, then starts the next
// stage.  One kernel and one trip over the state in place of two (N = 1024, FP64: 8.2 us of combine and
// update in 4.6; N = 7680: 10.0 in 6.3).  Block (x, y) takes chunk x, y = 0; with four threads per
// particle (sum_rows), 64 of its particles.  Launch-latency bound at the sizes where it matters.
// Always launched before the pair kernels, whose work counters it clears.
// SYM: there may be symmetric clusters (without them N = 1024 takes 0.4 us less per step).
template <bool FINISH, bool SYM>
__global__ __launch_bounds__(kBlock) void k_update(Args a, int update) {
  __shared__ double sh[FINISH && SYM ? 3 : 1][4][64];
  __shared__ double red[6][kBlock / 64];
  if (blockIdx.x == 0 && blockIdx.y == 0)  // the pair kernels that follow start at item 0
    for (int q = threadIdx.x; q < a.ncounters; q += kBlock) a.item_counter[q] = 0;
  const Chunk ch = load_chunk(a);
  const DevCluster c = load_cluster(a, ch.cluster);
  const int t = threadIdx.x;
  const bool sym = FINISH && SYM && c.seg;
  const int nrec = SYM ? chunk_records(c.n, c.seg) : 1, Q = sym ? sym_sums(c.n) : 1;
  if (Q == 1 && blockIdx.y) return;
  const int q = Q == 1 ? 0 : t >> 6, sub = Q == 1 ? t >> 6 : blockIdx.y;
  const int e = 64 * sub + (t & 63);
  const bool valid = e < ch.count, r32 = a.prec == NB_FP32;
  const int li = ch.start + (valid ? e : 0);
  long long i = c.off + li;
  double g[3];
  if (sym) {
    sum_rows<3>(a, c, li, valid, q, Q, -1, g, sh);
    if (q) return;
    i = particle_index(a, c, li);
    const double mc = a.mconst[ch.cluster];  // equal masses: the sums leave the mass out
    if (mc != 0.0)
#pragma unroll
      for (int d = 0; d < 3; ++d) g[d] *= mc;
  }
  double x[3] = {0.0, 0.0, 0.0}, m = 0.0, odd = 0.0;
  if (valid) {
    m = a.mass[i];
    odd = m != a.mass[c.off] ? 1.0 : 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) x[d] = a.pos[3 * i + d];
    if (update) {
      const double* const cf = FINISH ? a.coef_next : a.coef;
      const double kc = cf ? cf[3 * ch.cluster] : FINISH ? a.pre_next : a.kick_pre;
      const double dc = cf ? cf[3 * ch.cluster + 1] : FINISH ? a.drift_next : a.drift;
      double v[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) v[d] = a.vel[3 * i + d];
      bool ends = sym;  // this pass ends the cluster's stage
      if (FINISH && small_cluster(c) && (c.split > 1 || (c.flags & kFlagDefer))) {
        double pt;
        sum_ranges(a, c, li, r32, g[0], g[1], g[2], pt);
        ends = true;
      }
      if (ends) {
        finish_accel<true>(a, c, i, g[0], g[1], g[2], r32);
        const double kp = a.coef ? a.coef[3 * ch.cluster + 2] : a.kick_post;
        const bool kick = a.coef || kp != 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          a.acc[3 * i + d] = g[d];
          if (kick) v[d] = axpy(r32, kp, g[d], v[d]);
        }
      } else {
#pragma unroll
        for (int d = 0; d < 3; ++d) g[d] = a.acc[3 * i + d];
      }
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        v[d] = axpy(r32, kc, g[d], v[d]);
        x[d] = axpy(r32, dc, v[d], x[d]);
        a.vel[3 * i + d] = v[d];
        a.pos[3 * i + d] = x[d];
      }
    }
  }
  // FP64 and pure FP32 take absolute coordinates: of the partial sums they use the mass flag alone, which
  // the first stage of the call has left (the masses stay the same).  N = 1024, FP64: 5.4 us -> 4.2
  if (FINISH && (a.prec == NB_FP64 || a.prec == NB_FP32)) return;
  double val[5] = {m * x[0], m * x[1], m * x[2], m, odd};
  double mn[3], mx[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    mn[d] = valid ? x[d] : INFINITY;
    mx[d] = valid ? x[d] : -INFINITY;
  }
  if (nrec > 1) {  // a record for each wave
    wave_sum<5>(val);
    if (c.nstiles) wave_minmax<3>(mn, mx);
  } else {
    block_reduce<5>(val, red);
    if (c.nstiles) block_minmax<3>(mn, mx, red);  // only the sort wants the box
  }
  if ((nrec > 1 ? t & 63 : t) == 0) {
    double* p = const_cast<double*>(partial_record(a, c, blockIdx.x - c.chunk0, nrec > 1 ? sub : 0));
    for (int d = 0; d < 5; ++d) p[d] = val[d];
    for (int d = 0; d < 3; ++d) {
      p[5 + d] = mn[d];
      p[8 + d] = mx[d];
    }
  }
}

// One block per cluster: combines the chunk partials in a fixed order into the reference point,
// the common mass (mconst = the mass when all are equal, else 0) and the bounding box.
__global__ __launch_bounds__(kBlock) void k_reduce(Args a) {
  __shared__ double sh[6][kBlock / 64];
  const DevCluster c = a.cl[blockIdx.x];
  const int t = threadIdx.x;
  double tot[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int q = t; q < chunks_of(c); q += kBlock) {
    for (int r = 0; r < 5; ++r) tot[r] += chunk_sum(a, c, q, r);
    const double* p = partial_record(a, c, q, 0);
    if (c.nstiles)
      for (int w = 0; w < chunk_records(c.n, c.seg); ++w, p += kPartials)
        for (int d = 0; d < 3; ++d) {
          lo[d] = fmin(lo[d], p[5 + d]);
          hi[d] = fmax(hi[d], p[8 + d]);
        }
  }
  block_reduce<5>(tot, sh);
  if (c.nstiles) block_minmax<3>(lo, hi, sh);
  if (t == 0) {
    const double M = tot[3];
    a.ref[blockIdx.x] = M > 0.0 ? make_double4(tot[0] / M, tot[1] / M, tot[2] / M, M)
                                : make_double4(0.0, 0.0, 0.0, 0.0);
    a.mconst[blockIdx.x] = tot[4] == 0.0 ? a.mass[c.off] : 0.0;
    double* b = a.box + 6 * (size_t)blockIdx.x;
    for (int d = 0; d < 3; ++d) {
      b[d] = lo[d];
      b[3 + d] = hi[d];
    }
  }
}

// Diagnostics of one chunk, then per cluster in the last block.  Sums (kEnergySums):
//   0 K  1 W  2 Uext  3-5 P  6-8 L  9-11 torque  12 M  13-15 F = sum m a_int  16 sum m |a_int|
// where a_int is the internal acceleration and pot_ws the pair potential of the pass before.
// Output per cluster (kEnergyOut): K, W, Uext, E, P, L, torque, M, F, |F|, sum m |a_int|, and a
// non-finite flag.
__global__ __launch_bounds__(kBlock) void k_energy(Args a) {
  constexpr int NS = kEnergySums;
  __shared__ double sh[NS][kBlock / 64];
  const Chunk ch = load_chunk(a);
  const DevCluster c = load_cluster(a, ch.cluster);
  const int t = threadIdx.x;
  double q[NS];
#pragma unroll
  for (int k = 0; k < NS; ++k) q[k] = 0.0;
  if (t < ch.count) {
    const long long i = c.off + ch.start + t;
    const double m = a.mass[i];
    const double x = a.pos[3 * i], y = a.pos[3 * i + 1], z = a.pos[3 * i + 2];
    const double vx = a.vel[3 * i], vy = a.vel[3 * i + 1], vz = a.vel[3 * i + 2];
    const double ax = a.eacc_ws[3 * i], ay = a.eacc_ws[3 * i + 1], az = a.eacc_ws[3 * i + 2];
    q[0] = 0.5 * m * (vx * vx + vy * vy + vz * vz);
    q[1] = 0.5 * m * a.pot_ws[i];
    q[3] = m * vx;
    q[4] = m * vy;
    q[5] = m * vz;
    q[6] = m * (y * vz - z * vy);
    q[7] = m * (z * vx - x * vz);
    q[8] = m * (x * vy - y * vx);
    q[12] = m;
    q[13] = m * ax;
    q[14] = m * ay;
    q[15] = m * az;
    q[16] = m * sqrt(ax * ax + ay * ay + az * az);
    if (c.flags & kFlagField) {
      double ex, ey, ez;
      galaxy_accel<true>(a.gal, a.G, x, y, z, ex, ey, ez);
      q[2] = m * galaxy_potential(a.gal, a.G, x, y, z);
      q[9] = m * (y * ez - z * ey);
      q[10] = m * (z * ex - x * ez);
      q[11] = m * (x * ey - y * ex);
    }
  }
  block_reduce<NS>(q, sh);
  if (t == 0) {
#pragma unroll
    for (int k = 0; k < NS; ++k) a.epart[(size_t)blockIdx.x * NS + k] = q[k];
  }
  if (!last_block_of_cluster(&a.chunk_counter[ch.cluster], chunks_of(c))) return;
  double tot[NS];
#pragma unroll
  for (int k = 0; k < NS; ++k) tot[k] = 0.0;
  for (int p = t; p < chunks_of(c); p += kBlock) {
    const double* e = a.epart + (size_t)(c.chunk0 + p) * NS;
#pragma unroll
    for (int k = 0; k < NS; ++k) tot[k] += e[k];
  }
  __syncthreads();
  block_reduce<NS>(tot, sh);
  if (t == 0) {
    double* o = a.eout + (size_t)ch.cluster * kEnergyOut;
    const double K = tot[0], W = tot[1], U = tot[2];
    o[0] = K;
    o[1] = W;
    o[2] = U;
    o[3] = K + W + U;
    for (int k = 3; k < 16; ++k) o[k + 1] = tot[k];  // P, L, torque, M, F
    o[17] = sqrt(tot[13] * tot[13] + tot[14] * tot[14] + tot[15] * tot[15]);
    o[18] = tot[16];
    bool finite = true;
    for (int k = 0; k < 19; ++k) finite = finite && isfinite(o[k]);
    o[19] = finite ? 0.0 : 1.0;
    a.chunk_counter[ch.cluster] = 0;
  }
}

// Finish a particle of a split (or deferred) one-sided cluster: sum its ranges, then scale by G, galaxy
// field, store, optional kick, optional potential, as the pair kernel does for clusters that are not
// split.  Block (x, 0) takes chunk x.
__device__ __forceinline__ void combine_split(const Args& a, const Chunk& ch, const DevCluster& c, int potmode,
                                              int kick) {
  const int t = threadIdx.x;
  if ((c.split <= 1 && !(c.flags & kFlagDefer)) || t >= ch.count) return;
  const int li = ch.start + t;  // position in the cluster's (sorted) order
  const long long gi = particle_index(a, c, li);
  const bool r32 = a.prec == NB_FP32;
  double ax, ay, az, pt;
  sum_ranges(a, c, li, r32, ax, ay, az, pt);
  finish_particle<true>(a, c, ch.cluster, gi, ax, ay, az, r32, kick);
  if (potmode && a.pot) a.pot[gi] = r32 ? (double)(-(float)a.G * (float)pt) : -a.G * pt;
}

// Symmetric cluster: the rows of `band` into the running sums, which the clusters that end with that band (or
// had fewer) leave to the pass that finishes them; or, with band < 0, the cluster's own last band and the end of
// its stage.  Exactly one pass finishes a cluster: this one, or k_update between two stages.  Block (x, y)
// as in k_update.
template <int NC>
__device__ __forceinline__ void combine_sym(const Args& a, const Chunk& ch, const DevCluster& c, int band, int kick,
                                            double (*sh)[4][64]) {
  if (band >= 0 && band >= sym_rows(c.n, c.nseg, NC == 4, c.sym_doubles).nbands - 1) return;
  const int Q = sym_sums(c.n), t = threadIdx.x;
  if (Q == 1 && blockIdx.y) return;
  const int q = Q == 1 ? 0 : t >> 6, e = Q == 1 ? t : 64 * blockIdx.y + (t & 63);
  const bool valid = e < ch.count;
  const int li = ch.start + (valid ? e : 0);
  double sum[NC];
  if (!sum_rows<NC>(a, c, li, valid, q, Q, band, sum, sh) || q) return;
  if (!valid) return;
  const double mc = a.mconst[ch.cluster];
  if (mc != 0.0)
#pragma unroll
    for (int d = 0; d < NC; ++d) sum[d] *= mc;
  const long long gi = particle_index(a, c, li);
  const bool r32 = a.prec == NB_FP32;
  finish_particle<true>(a, c, ch.cluster, gi, sum[0], sum[1], sum[2], r32, kick);
  if constexpr (NC == 4) {
    if (a.pot) a.pot[gi] = r32 ? (double)(-(float)a.G * (float)sum[3]) : -a.G * sum[3];
  }
}

template <int NC>
__global__ __launch_bounds__(kBlock) void k_combine(Args a, CombineWhat what, int band, int kick) {
  __shared__ double sh[NC][4][64];
  const Chunk ch = load_chunk(a);
  const DevCluster c = load_cluster(a, ch.cluster);
  if (c.seg) {
    if (what != kCombineLarge) combine_sym<NC>(a, ch, c, what == kCombineBand ? band : -1, kick, sh);
  } else if (blockIdx.y == 0 && (what == kCombineAll || (what == kCombineLarge && !small_cluster(c)))) {
    combine_split(a, ch, c, NC == 4, kick);
  }
}

hipError_t launch_combine(const Args& a, CombineWhat what, int band, bool potmode, bool kick, hipStream_t s) {
  const dim3 grid(a.nchunks, a.sym ? 4 : 1);
  if (potmode)
    hipLaunchKernelGGL(k_combine<4>, grid, dim3(kBlock), 0, s, a, what, band, kick ? 1 : 0);
  else
    hipLaunchKernelGGL(k_combine<3>, grid, dim3(kBlock), 0, s, a, what, band, kick ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_update(const Args& a, bool update, bool finish, hipStream_t s) {
  if (!finish)
    hipLaunchKernelGGL((k_update<false, true>), dim3(a.nchunks), dim3(kBlock), 0, s, a, update ? 1 : 0);
  else if (a.sym)
    hipLaunchKernelGGL((k_update<true, true>), dim3(a.nchunks, 4), dim3(kBlock), 0, s, a, 1);
  else
    hipLaunchKernelGGL((k_update<true, false>), dim3(a.nchunks), dim3(kBlock), 0, s, a, 1);
  return hipGetLastError();
}

hipError_t launch_reduce(const Args& a, int B, hipStream_t s) {
  hipLaunchKernelGGL(k_reduce, dim3(B), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_energy(const Args& a, hipStream_t s) {
  hipLaunchKernelGGL(k_energy, dim3(a.nchunks), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

}  // namespace nb
