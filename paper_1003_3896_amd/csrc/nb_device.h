// Device helpers for the gfx950 kernels of libnbody.
#pragma once
#include "nb_internal.h"

namespace nb {

// x + (its value in the lane that the DPP control CTRL names; nothing where there is none, or in rows outside
// ROWS).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_sum(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, ROWS, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, ROWS, 0xf, true);
  return x + __hiloint2double(hi, lo);
}

// Fixed-order reductions of V doubles per thread: inside each wave, all of whose lanes call it (sums: valid in
// every lane; minima and maxima: in lane 0), then over the block the waves in order (valid in thread 0).
// sh needs [V] (minima and maxima: [2 V]).
// Sums go by DPP row shifts and row broadcasts: the kernels of small clusters are chains of latencies, and a
// shuffle through the LDS takes several times as long as the addition (N = 480, 8 steps: 134.0 -> 130.9 us).
template <int V>
__device__ __forceinline__ void wave_sum(double (&val)[V]) {
#pragma unroll
  for (int q = 0; q < V; ++q) {
    double x = val[q];
    x = dpp_sum<0x111, 0xf>(x);  // row_shr:1, 2, 4, 8: lane 15 of a row holds its sum
    x = dpp_sum<0x112, 0xf>(x);
    x = dpp_sum<0x114, 0xf>(x);
    x = dpp_sum<0x118, 0xf>(x);
    x = dpp_sum<0x142, 0xa>(x);  // row_bcast:15 into rows 1 and 3
    x = dpp_sum<0x143, 0xc>(x);  // row_bcast:31 into rows 2 and 3: lane 63 holds the wave's
    val[q] = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 63),
                              __builtin_amdgcn_readlane(__double2loint(x), 63));
  }
}
template <int V>
__device__ __forceinline__ void wave_minmax(double (&mn)[V], double (&mx)[V]) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1)
#pragma unroll
    for (int q = 0; q < V; ++q) {
      mn[q] = fmin(mn[q], __shfl_down(mn[q], m));
      mx[q] = fmax(mx[q], __shfl_down(mx[q], m));
    }
}
template <int V>
__device__ __forceinline__ void block_reduce(double (&val)[V], double (*sh)[kBlock / 64]) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  wave_sum<V>(val);
  __syncthreads();  // sh is free (a previous reduction has been read)
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < V; ++q) sh[q][wave] = val[q];
  __syncthreads();
  if (t == 0)
#pragma unroll
    for (int q = 0; q < V; ++q) {
      double s = sh[q][0];
      for (int w = 1; w < kBlock / 64; ++w) s += sh[q][w];
      val[q] = s;
    }
}
template <int V>
__device__ __forceinline__ void block_minmax(double (&mn)[V], double (&mx)[V], double (*sh)[kBlock / 64]) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  wave_minmax<V>(mn, mx);
  __syncthreads();
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < V; ++q) {
      sh[q][wave] = mn[q];
      sh[V + q][wave] = mx[q];
    }
  __syncthreads();
  if (t == 0)
#pragma unroll
    for (int q = 0; q < V; ++q)
      for (int w = 1; w < kBlock / 64; ++w) {
        mn[q] = fmin(mn[q], sh[q][w]);
        mx[q] = fmax(mx[q], sh[V + q][w]);
      }
}

// External galaxy field at (X,Y,Z) in FP64 (the F_ext term of Eq. 3), acceleration = -grad Phi:
// model 0, Hernquist bulge + Miyamoto-Nagai disk + logarithmic halo; model 1, the Allen & Santillan
// (1991) Galaxy (a spherical bulge Phi = -G Mb / sqrt(r^2 + ab^2), the same disk, and a spherical
// halo of mass M(r) = Mh (r/ah)^2.02 / (1 + (r/ah)^1.02) inside r, constant beyond rcut); both with
// an optional softened point mass at the centre (the black hole of Sect. 6.2).  ALL_MODELS = false
// compiles model 0 only: the pair kernel never finishes a particle in model 1's field (those
// clusters are finished by the combine pass), and model 1's transcendental functions would take
// registers there.

// Model 1's halo: the mass inside min(r, rcut).
__device__ __forceinline__ double as91_halo_mass(const Galaxy& g, double r) {
  const double s = fmin(r, g.rcut) / g.ah;
  const double q = pow(s, 1.02);
  return g.Mh * s * q / (1.0 + q);
}

template <bool ALL_MODELS>
__device__ __forceinline__ void galaxy_accel(const Galaxy& g, double G, double X, double Y, double Z, double& ax,
                                             double& ay, double& az) {
  const double R2 = X * X + Y * Y;
  const double r2 = R2 + Z * Z;
  const double r = sqrt(r2);
  double fb, fh;  // |grad Phi_b| / r and |grad Phi_h| / r
  if (ALL_MODELS && g.model == kGalaxyAllenSantillan) {
    const double q = r2 + g.ab * g.ab;
    fb = G * g.Mb / (q * sqrt(q));
    fh = r > 0.0 ? G * as91_halo_mass(g, r) / (r2 * r) : 0.0;  // the field of the mass inside r
  } else {
    const double rb = r + g.ab;
    fb = r > 0.0 ? G * g.Mb / (r * rb * rb) : 0.0;
    fh = g.vh * g.vh / (r2 + g.dh * g.dh);
  }
  const double zs = sqrt(Z * Z + g.bd * g.bd);
  const double as = g.ad + zs;
  const double D2 = R2 + as * as;
  const double fd = G * g.Md / (D2 * sqrt(D2));                // (1/R) dPhi_d/dR
  const double fz = fd * as / zs;                               // (1/z) dPhi_d/dz
  const double q2 = r2 + g.ebh * g.ebh;
  const double fbh = g.Mbh > 0.0 ? G * g.Mbh / (q2 * sqrt(q2)) : 0.0;  // (1/r) dPhi_bh/dr
  const double fxy = fb + fd + fh + fbh;
  ax = -fxy * X;
  ay = -fxy * Y;
  az = -(fb + fz + fh + fbh) * Z;
}

// Model 1's halo potential: -G M(r)/r minus the work against the field of the mass inside from r out
// to rcut, G Mh / (1.02 ah) [H(rcut) - H(r)] with H(s) = ln(1 + (s/ah)^1.02) - 1.02 / (1 + (s/ah)^1.02),
// the closed form of that integral; beyond rcut the point-mass potential of M(rcut).
__device__ __forceinline__ double as91_halo_potential(const Galaxy& g, double G, double r) {
  if (r >= g.rcut) return -G * as91_halo_mass(g, g.rcut) / r;
  const double qc = pow(g.rcut / g.ah, 1.02), q = pow(r / g.ah, 1.02);
  const double Hc = log(1.0 + qc) - 1.02 / (1.0 + qc), H = log(1.0 + q) - 1.02 / (1.0 + q);
  const double inner = r > 0.0 ? -G * as91_halo_mass(g, r) / r : 0.0;  // M(r) ~ r^2.02 at the centre
  return inner - G * g.Mh / (1.02 * g.ah) * (Hc - H);
}

__device__ __forceinline__ double galaxy_potential(const Galaxy& g, double G, double X, double Y, double Z) {
  const double R2 = X * X + Y * Y;
  const double r2 = R2 + Z * Z;
  const double r = sqrt(r2);
  const double zs = sqrt(Z * Z + g.bd * g.bd);
  const double as = g.ad + zs;
  const double pbh = g.Mbh > 0.0 ? -G * g.Mbh / sqrt(r2 + g.ebh * g.ebh) : 0.0;
  const double pd = -G * g.Md / sqrt(R2 + as * as);
  if (g.model == kGalaxyAllenSantillan)
    return -G * g.Mb / sqrt(r2 + g.ab * g.ab) + pd + as91_halo_potential(g, G, r) + pbh;
  return -G * g.Mb / (r + g.ab) + pd + 0.5 * g.vh * g.vh * log(r2 + g.dh * g.dh) + pbh;
}

// 1/sqrt(x) in FP64: the hardware estimate (relative error ~2^-24) refined by one
// third-order Newton step y' = y + y e (1/2 + 3/8 e), e = 1 - x y^2 (error O(e^3)).
__device__ __forceinline__ double rsqrt_f64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double h = x * y;
  const double e = fma(-h, y, 1.0);
  const double t = fma(0.375, e, 0.5);
  return fma(y * e, t, y);
}

// j-record of a particle (record64) as the pair kernels consume it:
//   NB_FP32   (x, y, z, m) rounded to FP32 (absolute coordinates)
//   NB_FP32C  (x - ref, m) rounded to FP32, ref = the cluster's FP64 centre of mass
//   NB_FP32DS hi = fl32(x - ref), lo = fl32((x - ref) - hi)   (double-single coordinates)
//   NB_FP64   (x, y, z, m) in FP64 (absolute)
__device__ __forceinline__ void record32(const Args& a, const double4& r, const double4& ref, float4& hi, float4& lo) {
  const double x = r.x, y = r.y, z = r.z;
  const float m = (float)r.w;
  if (a.prec == 0) {
    hi = make_float4((float)x, (float)y, (float)z, m);
    lo = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    return;
  }
  const double dx = x - ref.x, dy = y - ref.y, dz = z - ref.z;
  const float hx = (float)dx, hy = (float)dy, hz = (float)dz;
  hi = make_float4(hx, hy, hz, m);
  lo = make_float4((float)(dx - (double)hx), (float)(dy - (double)hy), (float)(dz - (double)hz), 0.0f);
}

__device__ __forceinline__ double4 record64(const Args& a, long long gi) {
  return make_double4(a.pos[3 * gi], a.pos[3 * gi + 1], a.pos[3 * gi + 2], a.mass[gi]);
}

// A partial record of a chunk (or of 64 particles, chunk_records): sums m x, m y, m z, m, count of masses !=
// the cluster's first; then min x, y, z and max x, y, z.
constexpr int kPartials = 11;
__device__ __forceinline__ const double* partial_record(const Args& a, const DevCluster& c, int chunk, int sub) {
  return a.partials + ((size_t)c.rec0 + (size_t)chunk * chunk_records(c.n, c.seg) + sub) * kPartials;
}
// Sum q of the cluster's chunk, its records in order.
__device__ __forceinline__ double chunk_sum(const Args& a, const DevCluster& c, int chunk, int q) {
  const double* p = partial_record(a, c, chunk, 0) + q;
  double s = p[0];
  for (int w = 1; w < chunk_records(c.n, c.seg); ++w) s += p[w * kPartials];
  return s;
}

// Reference point (centre of mass) and common mass of a small cluster, by each wave that needs them: without
// the launch of k_reduce, which cost more (3.3 us per evaluation) than the microsecond that this takes at the
// start of an item, unless the items are many (kReduceItems) or other clusters need k_reduce anyway: then the
// kernels read its results, which are the same bits.  (The symmetric kernel has more items and chunks: there it
// cost N = 15360 7 us to save 5, and the 512-cluster ensemble 5%.)  Called by whole waves.
template <bool CENTRE>
__device__ __forceinline__ double4 chunk_frame(const Args& a, const DevCluster& c, double& mc) {
  const int lane = threadIdx.x & 63;
  const bool has = lane < chunks_of(c);
  const double* p = partial_record(a, c, has ? lane : 0, 0);
  mc = __any(has && p[4] != 0.0) ? 0.0 : a.mass[c.off];
  if (!CENTRE) return make_double4(0.0, 0.0, 0.0, 0.0);
  double v[4];
#pragma unroll
  for (int d = 0; d < 4; ++d) v[d] = has ? p[d] : 0.0;
  wave_sum<4>(v);
  return v[3] > 0.0 ? make_double4(v[0] / v[3], v[1] / v[3], v[2] / v[3], v[3]) : make_double4(0.0, 0.0, 0.0, 0.0);
}

// Acceleration of one particle from its pair sum: scale by G, add the galaxy field (unless the pass wants
// the internal acceleration alone).  ALL_MODELS: as in galaxy_accel.
template <bool ALL_MODELS>
__device__ __forceinline__ void finish_accel(const Args& a, const DevCluster& c, long long gi, double& ax, double& ay,
                                             double& az, bool round32) {
  ax *= a.G;
  ay *= a.G;
  az *= a.G;
  if (round32) {
    ax = (float)ax;
    ay = (float)ay;
    az = (float)az;
  }
  if ((c.flags & kFlagField) && !a.internal_only) {
    double ex, ey, ez;
    galaxy_accel<ALL_MODELS>(a.gal, a.G, a.pos[3 * gi], a.pos[3 * gi + 1], a.pos[3 * gi + 2], ex, ey, ez);
    ax += ex;
    ay += ey;
    az += ez;
    if (round32) {
      ax = (float)ax;
      ay = (float)ay;
      az = (float)az;
    }
  }
}

// Epilogue of one particle: scale by G, add the galaxy field (unless the pass wants the internal
// acceleration alone), store, optional kick.  ALL_MODELS: as in galaxy_accel.
template <bool ALL_MODELS>
__device__ __forceinline__ void finish_particle(const Args& a, const DevCluster& c, int cluster, long long gi,
                                                double ax, double ay, double az, bool round32, int kick) {
  finish_accel<ALL_MODELS>(a, c, gi, ax, ay, az, round32);
  if (a.acc) {
    a.acc[3 * gi] = ax;
    a.acc[3 * gi + 1] = ay;
    a.acc[3 * gi + 2] = az;
  }
  if (kick) {
    const double kp = a.coef ? a.coef[3 * cluster + 2] : a.kick_post;
    double* v = a.vel + 3 * gi;
    if (round32) {
      v[0] = fmaf((float)kp, (float)ax, (float)v[0]);
      v[1] = fmaf((float)kp, (float)ay, (float)v[1]);
      v[2] = fmaf((float)kp, (float)az, (float)v[2]);
    } else {
      v[0] = fma(kp, ax, v[0]);
      v[1] = fma(kp, ay, v[1]);
      v[2] = fma(kp, az, v[2]);
    }
  }
}

}  // namespace nb
