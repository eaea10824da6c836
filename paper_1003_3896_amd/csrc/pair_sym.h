// Symmetric all-pairs gravity (Sect. 2, Eq. 5) for gfx950: every unordered pair of particles is
// evaluated once and both of its accelerations are kept (the forces of Eq. 2 are antisymmetric).
//
// A cluster is cut into segments of S particles (nb_internal.h: sym_segment).  A work item is a pair
// of segments (I, J): one block evaluates the S x S pairs between them and writes S partial sums for
// I's particles and S for J's, each into its own row of the partial-sum table, which the combine pass
// adds in row order.  No atomics on global memory: which rows an item writes and in what order they
// are added depend on the cluster's size alone, so results are bitwise reproducible.  A segment with
// itself is evaluated one-sided (all S x S ordered terms; the self term vanishes or is masked).
//
// Wave: K i-particles per lane in registers (a group of 64 K), against strips of 64 j-particles.
// Lane l of a 16-lane row meets particle (l + n) mod 16 of its row's chunk in step n = 0..15, read
// from LDS at a fixed offset from the lane's address (each chunk is stored twice in a row, so the
// wrap needs no address arithmetic); the four rows hold the strip's four chunks in turn (phases).  The
// reaction on the j-particles, summed over the lane's K terms first, returns to the j-particle's lane
// by a row rotation (DPP) and stays in a register for the 16 steps, then goes to an FP64
// accumulator in LDS.  Per pair that is 3 differences, 3 FMAs, rsq, 2 products, 2 x 3 FMAs and
// 3/4 of a rotating add (K = 4): 7.4 instructions and half a v_rsq_f32 per interaction, where the
// one-sided loop needs 11 and one.
//
// What bounds it: the VALU issue rate.  A gfx950 SIMD issues plain FP32 instructions of two waves at a
// time (2.07 SIMD cycles per wave64 instruction at 2, 4, 6 or 8 waves; 3 waves: 3.3), while
// v_rsq_f32 (8.1 cycles) and DPP instructions (4.2) issue alone, and one of these in a stream of plain
// ones drops the whole stream to about 4 cycles per instruction, unless an s_nop next to it lets the
// waves fall back into step: 11 FMAs + 1 rsq take 4.4 cycles per instruction bare and 2.8 with
// s_nop 0 on both sides; 15 FMAs + 1 DPP move 4.0 bare and 2.25 with one s_nop 0.  Hence rsq_sym and
// ror_add below, and an even number of waves per SIMD (4).  The loop by itself runs one FP32 pair in 53
// cycles at 2.27 GHz (44 by those rates), a double-single one in 68, an FP64 one in 105.
//
// Why 8 waves to an item and 2 blocks per CU: SIMDs serve their oldest waves first, so when the items
// run out every CU still holds all its blocks' items, half done on average; fewer, faster items per CU
// shorten that tail (N = 65536 in NB_FP32DL 1.22 -> 1.10 ms against 4 blocks of 4 waves, N = 15360 in
// NB_FP32DS 101 -> 88 us; with segments of 512 instead of 1024 particles at 65536, 0.97 ms).  Two blocks per CU of 4 waves (2 waves per SIMD) were 11 to 18% slower.
// Against the one-sided kernels: N = 262144 in NB_FP32DL 17.0 -> 12.8 ms, N = 65536 1.25 -> 0.95 ms,
// N = 15360 in NB_FP32DS 140 -> 88 us, N = 65536 in FP64 with the potential 3.0 -> 2.1 ms, 512 clusters
// of 256..16384 in NB_FP32DS 5.6 -> 4.2 ms.
#pragma once
#include "nb_device.h"
#include <type_traits>

namespace nb {

constexpr int kSymBlock = 512;            // threads: 8 waves
constexpr int kSymWaves = kSymBlock / 64;
// LDS accumulators of one block (groups x chunk): 1024 (half the flushes, each two barriers) against 512 made
// the N = 15360 to 262144 steps 0.5 to 1.5% faster; with the potential they would not fit beside the staged
// strips.
template <bool POT>
constexpr int kSymAcc = POT ? 512 : 1024;

// v_rsq_f32 between two s_nop (see the top of the file; the second one is also the wait state its
// consumer needs).
__device__ __forceinline__ float rsq_sym(float x) {
  float r;
  asm("s_nop 0\n\tv_rsq_f32_e32 %0, %1\n\ts_nop 0" : "=v"(r) : "v"(x));
  return r;
}
__device__ __forceinline__ double rsq_sym(double x) { return rsqrt_f64(x); }
__device__ __forceinline__ float fma_sym(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_sym(double a, double b, double c) { return fma(a, b, c); }

// acc += t of lane (l - N) mod 16 of the same 16-lane row (two wait states between the producer of t
// and the DPP read).
template <int N>
__device__ __forceinline__ void ror_add(float& acc, float t) {
  if constexpr (N == 0)
    acc += t;
  else
    asm("s_nop 1\n\tv_add_f32_dpp %0, %1, %0 row_ror:%2 row_mask:0xf bank_mask:0xf\n\ts_nop 0"
        : "+v"(acc)
        : "v"(t), "n"(N));
}
template <int N>
__device__ __forceinline__ void ror_add3(float& ax, float& ay, float& az, float tx, float ty, float tz) {
  if constexpr (N == 0) {
    ax += tx;
    ay += ty;
    az += tz;
  } else {
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %3, %0 row_ror:%6 row_mask:0xf bank_mask:0xf\n\ts_nop 0\n\t"
        "v_add_f32_dpp %1, %4, %1 row_ror:%6 row_mask:0xf bank_mask:0xf\n\ts_nop 0\n\t"
        "v_add_f32_dpp %2, %5, %2 row_ror:%6 row_mask:0xf bank_mask:0xf\n\ts_nop 0"
        : "+v"(ax), "+v"(ay), "+v"(az)
        : "v"(tx), "v"(ty), "v"(tz), "n"(N));
  }
}
template <int N>
__device__ __forceinline__ double ror(double x) {
  if constexpr (N == 0) return x;
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, 0x120 + N, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x120 + N, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <int N>
__device__ __forceinline__ void ror_add(double& acc, double t) {
  acc += ror<N>(t);
}
template <int N>
__device__ __forceinline__ void ror_add3(double& ax, double& ay, double& az, double tx, double ty, double tz) {
  ax += ror<N>(tx);
  ay += ror<N>(ty);
  az += ror<N>(tz);
}

// One wave's strip of 64 j-records in LDS, every chunk of 16 twice in a row: record e of chunk c at
// 32 c + e and 32 c + 16 + e.
template <int FAM>
struct SymStage {
  float4 hi[128];
};
template <>
struct SymStage<FAM_DS> {
  float4 hi[128], lo[128];
};
template <>
struct SymStage<FAM_DL> : SymStage<FAM_DS> {};
template <>
struct SymStage<FAM_F64> {
  double2 xy[128], zm[128];
};

// i-particles and sums of one lane.
template <class R, int K>
struct SymLane {
  R x[K], y[K], z[K], m[K];
  float lx[K], ly[K], lz[K];   // low parts (double-single families)
  R ax[K], ay[K], az[K], p[K];
};

template <class R>
struct SymRec {
  R x, y, z, m;
  float lx, ly, lz;
};

template <int FAM, bool LO, class R>
__device__ __forceinline__ SymRec<R> sym_read(const SymStage<FAM>& st, int e) {
  SymRec<R> r;
  if constexpr (FAM == FAM_F64) {
    const double2 a = st.xy[e], b = st.zm[e];
    r.x = a.x;
    r.y = a.y;
    r.z = b.x;
    r.m = b.y;
  } else {
    const float4 a = st.hi[e];
    r.x = a.x;
    r.y = a.y;
    r.z = a.z;
    r.m = a.w;
    if constexpr (LO) {
      const float4 b = st.lo[e];
      r.lx = b.x;
      r.ly = b.y;
      r.lz = b.z;
    }
  }
  return r;
}

// Steps N .. 15 of one phase: the lane's K particles against record e0 + n of the staged strip.
// bx, by, bz, bp: the reaction on the lane's own j-particle (l of its chunk).  self0 (one-sided potential, the
// j = i term is left out): i-particle k would be entry self0 + 64 k of the row's chunk.
template <int N, int FAM, bool LO, bool EQ, bool SYM, bool MASK, bool POT, class R, int K>
__device__ __forceinline__ void sym_steps(const SymStage<FAM>& st, int e0, SymLane<R, K>& v, R e2, R& bx, R& by, R& bz,
                                          R& bp, int l16, int self0) {
  if constexpr (N < 16) {
    const SymRec<R> j = sym_read<FAM, LO, R>(st, e0 + N);
    R tx = 0, ty = 0, tz = 0, tp = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      R dx = j.x - v.x[k], dy = j.y - v.y[k], dz = j.z - v.z[k];
      if constexpr (LO) {
        dx += j.lx - v.lx[k];
        dy += j.ly - v.ly[k];
        dz += j.lz - v.lz[k];
      }
      R r2 = fma_sym(dx, dx, e2);
      r2 = fma_sym(dy, dy, r2);
      r2 = fma_sym(dz, dz, r2);
      const R inv = rsq_sym(r2);
      // si, sj: r^-3 times the other particle's mass; qi, qj: r^-1 times it (potential).  Equal masses: the mass is
      // applied once, in the combine pass.  The FP32 families take the mass into the first factor: r^-3 alone
      // leaves their range for |d| outside 1e-12 .. 1e12 (one product more per pair: 65536 Salpeter stars, a
      // leapfrog step, 1.01 -> 1.05 ms in NB_FP32DL and 1.12 -> 1.16 in NB_FP32DS).
      constexpr bool RANGE = !EQ && sizeof(R) == 4;
      const R inv2 = inv * inv, s = inv * inv2;
      const R qi = EQ ? inv : j.m * inv, qj = EQ ? inv : v.m[k] * inv;
      R si = RANGE ? qi * inv2 : EQ ? s : s * j.m, sj = RANGE ? qj * inv2 : EQ ? s : s * v.m[k];
      if (MASK) {
        si = r2 > R(0) ? si : R(0);
        sj = r2 > R(0) ? sj : R(0);
      }
      v.ax[k] = fma_sym(dx, si, v.ax[k]);
      v.ay[k] = fma_sym(dy, si, v.ay[k]);
      v.az[k] = fma_sym(dz, si, v.az[k]);
      if constexpr (POT) v.p[k] += (SYM || ((l16 + N) & 15) != self0 + 64 * k) ? qi : R(0);
      if constexpr (SYM) {
        tx = k ? fma_sym(dx, sj, tx) : dx * sj;
        ty = k ? fma_sym(dy, sj, ty) : dy * sj;
        tz = k ? fma_sym(dz, sj, tz) : dz * sj;
        if constexpr (POT) tp = !k ? qj : EQ ? tp + qj : fma_sym(inv, v.m[k], tp);
      }
    }
    if constexpr (SYM) {
      ror_add3<N>(bx, by, bz, tx, ty, tz);
      if constexpr (POT) ror_add<N>(bp, tp);
    }
    sym_steps<N + 1, FAM, LO, EQ, SYM, MASK, POT, R, K>(st, e0, v, e2, bx, by, bz, bp, l16, self0);
  }
}

__device__ __forceinline__ void lds_add(double* p, double x) {
  __hip_atomic_fetch_add(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);  // ds_add_f64
}

// FP64 sums of one lane's i-particles (the FP32 sums are folded into them every 16 or 32 terms, the FP64
// family adds to them directly).
template <int K>
struct SymSums {
  double x[K], y[K], z[K], p[K];
};

template <bool POT, int K>
__device__ __forceinline__ void sym_fold(SymLane<float, K>& v, SymSums<K>& A) {
#pragma unroll
  for (int k = 0; k < K; ++k) {
    A.x[k] += (double)v.ax[k];
    A.y[k] += (double)v.ay[k];
    A.z[k] += (double)v.az[k];
    v.ax[k] = v.ay[k] = v.az[k] = 0.0f;
    if (POT) {
      A.p[k] += (double)v.p[k];
      v.p[k] = 0.0f;
    }
  }
}

// The lane's K i-particles against one staged strip.  acc: the wave group's LDS accumulators of the
// strip's 64 j-particles (only this wave adds to them now), component q at acc[q * kSymAcc].
// jmi: first j of the strip minus the lane's i-particle 0 (one-sided potential).
// last: the wave's last strip of the item.
template <int FAM, bool LO, bool EQ, bool SYM, bool MASK, bool POT, class R, int K>
__device__ __forceinline__ void sym_strip(const SymStage<FAM>& st, SymLane<R, K>& v, SymSums<K>& A, R e2, double* acc,
                                          int jmi, bool last) {
  const int lane = threadIdx.x & 63, l16 = lane & 15;
#pragma unroll 1
  for (int p = 0; p < 4; ++p) {
    if (p == 2 && last) __builtin_amdgcn_s_setprio(0);
    const int c = ((lane >> 4) + p) & 3;
    R bx = 0, by = 0, bz = 0, bp = 0;
    sym_steps<0, FAM, LO, EQ, SYM, MASK, POT, R, K>(st, 32 * c + l16, v, e2, bx, by, bz, bp, l16, -jmi - 16 * c);
    if constexpr (SYM) {
      double* a = acc + 16 * c + l16;
      lds_add(a, (double)bx);
      lds_add(a + kSymAcc<POT>, (double)by);
      lds_add(a + 2 * kSymAcc<POT>, (double)bz);
      if constexpr (POT) lds_add(a + 3 * kSymAcc<POT>, (double)bp);
    }
    // Into FP64 every 32 terms; every 16 in near strips of the local mode, whose sorted order puts a particle's
    // near neighbours one after the other: a sum then grows early and rounds all that follow at its size (the
    // one-sided kernel deals successive terms to two sums).  Mean error of FP32DL accelerations, uniform
    // sphere of 9000: 4.81e-8 with 32, 4.06e-8 with 16, one-sided kernel 4.60e-8; far strips with 16 too:
    // 4.05e-8, but N = 65536 takes 988 us for 958 (954 with 32).
    if constexpr (FAM != FAM_F64) {
      if ((FAM == FAM_DL && LO) || (p & 1)) sym_fold<POT, K>(v, A);
    }
  }
}

// Raw FP64 source, fetched one strip ahead.
struct SymRaw {
  double x, y, z, m;
};
template <bool SORTED>
__device__ __forceinline__ SymRaw sym_fetch(const Args& a, long long g, bool valid) {
  SymRaw r{0.0, 0.0, 0.0, 0.0};
  if (valid) {
    if constexpr (SORTED) {
      const double4 q = a.spos[g];
      r = SymRaw{q.x, q.y, q.z, q.w};
    } else {
      r = SymRaw{a.pos[3 * g], a.pos[3 * g + 1], a.pos[3 * g + 2], a.mass[g]};
    }
  }
  return r;
}

// Coordinates that stand for a missing particle: so far away that every term with a real one is
// exactly zero (FP32: r^2 overflows and rsq gives 0; FP64: r^-3 underflows), and never NaN.
template <class R>
__device__ __forceinline__ constexpr R sym_pad() {
  return sizeof(R) == 4 ? (R)1e30f : (R)1e150;
}

// Record of one particle as in record32: FP32 coordinates relative to ref (absolute in NB_FP32) and,
// when asked for, their low parts, or FP64.
template <int FAM, class R>
__device__ __forceinline__ SymRec<R> sym_record(const SymRaw& q, const double4& ref, bool absolute, bool valid,
                                                bool low) {
  SymRec<R> r;
  r.lx = r.ly = r.lz = 0.0f;
  if (!valid) {
    r.x = r.y = r.z = sym_pad<R>();
    r.m = 0;
    return r;
  }
  r.m = (R)q.m;
  if constexpr (FAM == FAM_F64) {
    r.x = q.x;
    r.y = q.y;
    r.z = q.z;
  } else {
    const double dx = absolute ? q.x : q.x - ref.x, dy = absolute ? q.y : q.y - ref.y, dz = absolute ? q.z : q.z - ref.z;
    r.x = (float)dx;
    r.y = (float)dy;
    r.z = (float)dz;
    if (low) {
      r.lx = (float)(dx - (double)r.x);
      r.ly = (float)(dy - (double)r.y);
      r.lz = (float)(dz - (double)r.z);
    }
  }
  return r;
}

template <int FAM, class R>
__device__ __forceinline__ void sym_stage(SymStage<FAM>& st, const SymRec<R>& r, bool low) {
  const int lane = threadIdx.x & 63, e = 32 * (lane >> 4) + (lane & 15);
  if constexpr (FAM == FAM_F64) {
    st.xy[e] = st.xy[e + 16] = make_double2(r.x, r.y);
    st.zm[e] = st.zm[e + 16] = make_double2(r.z, r.m);
  } else {
    st.hi[e] = st.hi[e + 16] = make_float4(r.x, r.y, r.z, r.m);
    if constexpr (FAM == FAM_DS || FAM == FAM_DL) {
      if (low) st.lo[e] = st.lo[e + 16] = make_float4(r.lx, r.ly, r.lz, 0.0f);
    }
  }
}

// Orders this wave's own LDS writes before its reads of other lanes' data (and the reverse).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Reads through the scalar cache what is the same for the whole wave (tables and per-cluster values
// that kernels before this one wrote).
template <class T>
using ScalarPtr = const __attribute__((address_space(4))) T*;
template <class T>
__device__ __forceinline__ ScalarPtr<T> scalar(const T* p) {
  return (ScalarPtr<T>)(unsigned long long)p;
}

// Which entry item `t` of a band belongs to: the last k with first <= t, 64 entries per look.
__device__ __forceinline__ int sym_find(const SymEntry* e, int count, int t) {
  int lo = 0, len = count;  // e[lo].first <= t; the answer is in [lo, lo + len)
  while (len > 1) {
    const int step = (len + 63) >> 6, at = lo + (threadIdx.x & 63) * step;
    const unsigned long long m = __ballot(at < lo + len && e[at].first <= t);
    const int hit = 63 - __clzll(m);  // lane 0 always hits
    lo += hit * step;
    len = min(step, count - lo);
  }
  return uniform(lo);
}

// K i-particles per lane; G = 64 K of one wave.  The block's 8 waves are GI groups of i-particles
// times GJ waves that take every GJ-th strip of the chunk: (GI, GJ) = (4, 2) for segments of 1024, else
// (2, 4).
template <int FAM, bool MASK, bool POT, int K>
__global__ __launch_bounds__(kSymBlock, 4) void k_pair_sym(Args a, SymBand band) {
  using R = typename std::conditional<FAM == FAM_F64, double, float>::type;
  constexpr bool SORTED = FAM == FAM_DL, DS = FAM == FAM_DS || FAM == FAM_DL;
  constexpr int NC = POT ? 4 : 3, G = 64 * K, ACC = kSymAcc<POT>;
  struct Work {
    SymStage<FAM> st[kSymWaves];
    double acc[NC * ACC];
  };
  constexpr size_t kReduce = sizeof(double) * NC * G * 6;  // sums of the waves with gj > 0
  __shared__ __align__(16) char lds[sizeof(Work) > kReduce ? sizeof(Work) : kReduce];
  __shared__ int s_item;
  Work& sh = *reinterpret_cast<Work*>(lds);
  const int tid = threadIdx.x, wave = uniform(tid >> 6), lane = tid & 63;
  SymStage<FAM>& st = sh.st[wave];
  for (int e = tid; e < NC * ACC; e += kSymBlock) sh.acc[e] = 0.0;
  __syncthreads();
  for (int it = blockIdx.x; it < band.nitems;) {
    // a wave that is not in the pair loops (set-up, sums, stores) goes before those that are: its
    // latencies then lie under their arithmetic
    __builtin_amdgcn_s_setprio(3);
    int next = 0;
    if (tid == 0) next = gridDim.x + atomicAdd(band.counter, 1);  // used at the end of this item
    const ScalarPtr<SymEntry> en = scalar(band.entries + sym_find(band.entries, band.ncl, it));
    const int ci = en->cluster;
    const ScalarPtr<DevCluster> c = scalar(a.cl + ci);
    const int n = c->n, S = c->seg, nseg = c->nseg;
    const long long off = c->off;
    const int u = it - en->first, du = u / nseg, delta = en->delta0 + du, A = u - du * nseg;
    const int B = A + delta >= nseg ? A + delta - nseg : A + delta;
    const bool diag = delta == 0, half = 2 * delta == nseg;
    double* const part = a.sym + c->part_off;
    double* const rowi = part + (size_t)((diag ? 0 : 2 * delta - 1) - en->row0) * NC * n;
    double* const rowj = half ? rowi : part + (size_t)(2 * delta - en->row0) * NC * n;
    const int ib = A * S, ie = min(n, ib + S), jb = B * S, je = min(n, jb + S);
    const int GI = S >= 4 * G ? 4 : 2, GJ = kSymWaves / GI;
    const int gi = wave / GJ, gj = wave - gi * GJ;
    const int CH = ACC / GI;  // j-particles between two flushes
    const bool eq = scalar(a.mconst)[ci] != 0.0;
    const R e2 = FAM == FAM_F64 ? (R)c->eps2 : (R)c->eps2f;
    const bool absolute = a.prec == 0;
    double* const acc = sh.acc + gi * CH;
    const int wb = ib + gi * G;  // this wave's group (the block's cover the segment)
    const bool active = wb < ie;
    // the frame: the cluster's centre of mass, in the local mode the box of the group's chunk
    const ScalarPtr<double> f = scalar(reinterpret_cast<const double*>(
        FAM == FAM_DL ? a.gbox + c->chunk0 + min(wb, n - 1) / kChunk : a.ref + ci));
    const double4 ref = make_double4(f[0], f[1], f[2], f[3]);
    SymRaw raw = sym_fetch<SORTED>(a, off + jb + 64 * gj + lane, jb + 64 * gj + lane < je);
    SymLane<R, K> v;
    SymSums<K> s;
#pragma unroll
    for (int q = 0; q < K; ++q) {
      const int li = wb + 64 * q + lane;
      const bool ok = li < ie;
      const SymRec<R> r = sym_record<FAM, R>(sym_fetch<SORTED>(a, off + li, ok), ref, absolute, ok, DS);
      v.x[q] = r.x;
      v.y[q] = r.y;
      v.z[q] = r.z;
      v.m[q] = r.m;
      v.lx[q] = r.lx;
      v.ly[q] = r.ly;
      v.lz[q] = r.lz;
      v.ax[q] = v.ay[q] = v.az[q] = v.p[q] = 0;
      s.x[q] = s.y[q] = s.z[q] = s.p[q] = 0.0;
    }
    for (int jc = jb; jc < je; jc += CH) {
      const int jce = min(je, jc + CH);
      for (int j0 = jc + 64 * gj; j0 < jce; j0 += 64 * GJ) {
        const bool ok = j0 + lane < je;
        const SymRaw cur = raw;
        // the next strip of this wave (strips are 64 GJ apart, also across chunks)
        const int jn = j0 + 64 * GJ + lane;
        raw = sym_fetch<SORTED>(a, off + jn, jn < je);
        if (!active) continue;
        bool lo = FAM == FAM_DS;
        if constexpr (FAM == FAM_DL) {
          // far strip: every source at least 3/4 of the group's box diagonal from its centre, so the
          // FP32 difference of the local coordinates is within 1.5 x 2^-22 of the exact one
          const double dx = cur.x - ref.x, dy = cur.y - ref.y, dz = cur.z - ref.z;
          lo = !__all(!ok || dx * dx + dy * dy + dz * dz >= ref.w);
        }
        wave_sync();
        sym_stage<FAM, R>(st, sym_record<FAM, R>(cur, ref, absolute, ok, lo), lo);
        wave_sync();
        // Waves of equal priority are served oldest first: the younger one of a SIMD's two would end late and,
        // alone there, run at a third of the rate.  With the priority going down in the second half of the
        // item and again in the last half of its last strip they end together.  FP32-DS, N = 15360: 93 us
        // -> 86; FP32 with the potential, 30011: 291 -> 266; FP32C, 12 clusters of 1024 .. 65536: 4.09 ms
        // -> 3.85; local mode, 65536: 7.58 -> 7.24, 262144: 13.52 either way.
        const bool last = j0 - jb + 64 * GJ >= S;
        if (!last && 2 * (j0 - jb) < S)
          __builtin_amdgcn_s_setprio(2);
        else
          __builtin_amdgcn_s_setprio(1);
        double* const sa = acc + (j0 - jc);
        const int jmi = j0 - (wb + lane);
#define NB_STRIP(LO, EQ, SYM) sym_strip<FAM, LO, EQ, SYM, MASK, POT, R, K>(st, v, s, e2, sa, jmi, last)
        if constexpr (DS) {
          if (lo) {
            if (diag)
              eq ? NB_STRIP(true, true, false) : NB_STRIP(true, false, false);
            else
              eq ? NB_STRIP(true, true, true) : NB_STRIP(true, false, true);
          }
        }
        if constexpr (FAM != FAM_DS) {
          if (!lo) {
            if (diag)
              eq ? NB_STRIP(false, true, false) : NB_STRIP(false, false, false);
            else
              eq ? NB_STRIP(false, true, true) : NB_STRIP(false, false, true);
          }
        }
#undef NB_STRIP
        __builtin_amdgcn_s_setprio(3);
      }
      if (!diag) {  // the chunk's reactions, groups in order, into J's row
        __syncthreads();
        if (tid < CH && jc + tid < je) {
          const int li = jc + tid;
#pragma unroll
          for (int q = 0; q < NC; ++q) {
            double t = 0.0;
            for (int g = 0; g < GI; ++g) {
              double* const e = sh.acc + q * ACC + g * CH + tid;
              t += *e;
              *e = 0.0;
            }
            if (q < 3) t = -t;
            rowj[(size_t)q * n + li] = t;
          }
        }
        __syncthreads();
      }
    }
    if constexpr (FAM == FAM_F64) {
#pragma unroll
      for (int q = 0; q < K; ++q) {
        s.x[q] = v.ax[q];
        s.y[q] = v.ay[q];
        s.z[q] = v.az[q];
        s.p[q] = v.p[q];
      }
    }
    // the waves that shared a group, in order
    double* const red = reinterpret_cast<double*>(lds) + (size_t)(gi * (GJ - 1)) * G * NC + lane;
    __syncthreads();
    if (gj > 0) {
      double* const e = red + (size_t)(gj - 1) * G * NC;
#pragma unroll
      for (int q = 0; q < K; ++q) {
        e[0 * G + 64 * q] = s.x[q];
        e[1 * G + 64 * q] = s.y[q];
        e[2 * G + 64 * q] = s.z[q];
        if (POT) e[3 * G + 64 * q] = s.p[q];
      }
    }
    __syncthreads();
    if (gj == 0 && active) {
      for (int h = 0; h < GJ - 1; ++h) {
        const double* const e = red + (size_t)h * G * NC;
#pragma unroll
        for (int q = 0; q < K; ++q) {
          s.x[q] += e[0 * G + 64 * q];
          s.y[q] += e[1 * G + 64 * q];
          s.z[q] += e[2 * G + 64 * q];
          if (POT) s.p[q] += e[3 * G + 64 * q];
        }
      }
#pragma unroll
      for (int q = 0; q < K; ++q) {
        const int li = wb + 64 * q + lane;
        if (li < ie) {
          rowi[li] = s.x[q];
          rowi[(size_t)n + li] = s.y[q];
          rowi[2 * (size_t)n + li] = s.z[q];
          if (POT) rowi[3 * (size_t)n + li] = s.p[q];
        }
      }
    }
    __syncthreads();
    for (int e = tid; e < NC * ACC; e += kSymBlock) sh.acc[e] = 0.0;  // the sums may have lain over them
    if (tid == 0) s_item = next;
    __syncthreads();
    it = uniform(s_item);
    __syncthreads();  // every wave has read s_item
  }
}

template <int FAM>
hipError_t launch_sym_family(const Args& a, const SymBand& b, int grid, bool mask, bool pot, hipStream_t s) {
  void (*fn)(Args, SymBand);
  if (b.seg == 256)
    fn = mask ? (pot ? k_pair_sym<FAM, true, true, 2> : k_pair_sym<FAM, true, false, 2>)
              : (pot ? k_pair_sym<FAM, false, true, 2> : k_pair_sym<FAM, false, false, 2>);
  else
    fn = mask ? (pot ? k_pair_sym<FAM, true, true, 4> : k_pair_sym<FAM, true, false, 4>)
              : (pot ? k_pair_sym<FAM, false, true, 4> : k_pair_sym<FAM, false, false, 4>);
  hipLaunchKernelGGL(fn, dim3(grid), dim3(kSymBlock), 0, s, a, b);
  return hipGetLastError();
}

}  // namespace nb
