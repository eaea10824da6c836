// Internal types shared by the gfx950 kernels and the host runtime of libnbody.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nb {

// Threads per block of every kernel, and particles per O(N) chunk (one per thread).
constexpr int kBlock = 256;
constexpr int kChunk = 256;

// Precision families of the pair kernel (FAM_DL: double-single near j-tiles, FP32 on coordinates
// centred on the i-tile for far ones, particles in Hilbert-curve order).
enum Family { FAM_F32 = 0, FAM_DS = 1, FAM_F64 = 2, FAM_DL = 3 };
constexpr int kFamilies = 4;
// Cluster-size classes of the launch-shape table (largest cluster < 2048, < 32768, < 131072, larger).
constexpr int kSizeClasses = 4;

// Hilbert-curve sort of the NB_FP32DL mode: particles per sort tile (one block), radix digit bits.
constexpr int kSortTile = 2048;
constexpr int kRadixBits = 10;
constexpr int kRadix = 1 << kRadixBits;

// Per-cluster descriptor in device memory (uploaded with every call).  72 bytes: the table limit of
// nbody_accel_noalloc counts them.
struct DevCluster {
  long long off;       // first particle of the cluster in the concatenated arrays
  long long part_off;  // first row of the cluster's partial sums ([split][n] rows), when split > 1
                       // or kFlagDefer; symmetric path: first double of its rows in Args::sym
  int n;               // particles
  int flags;           // kFlagField | kFlagMaskSelf | kFlagDefer
  double eps2;         // eps^2 in FP64
  float eps2f;         // eps^2 rounded to FP32
  int chunk0;          // first O(N) chunk of the cluster
  union {
    struct {           // one-sided path
      int split;       // the j-sum of every particle is split into this many ranges (1 = none)
      int jlen;        // sources per range (the last range may be shorter)
    };
    long long sym_doubles;  // symmetric path: room for its rows (doubles)
  };
  int stile0;          // first sort tile of the cluster (NB_FP32DL)
  int nstiles;         // sort tiles of the cluster
  int tbox0;           // first j-tile box of the cluster (NB_FP32DL; room for split x ceil(jlen/128))
  int seg;             // symmetric path: particles per segment (0: the cluster takes the one-sided path)
  int nseg;            // symmetric path: segments
  int rec0;            // first partial record of the cluster (chunk_records per chunk)
};
static_assert(sizeof(DevCluster) == 72, "the uploaded tables' layout");
// O(N) chunks of a cluster
__host__ __device__ inline int chunks_of(const DevCluster& c) { return (c.n + kChunk - 1) / kChunk; }
constexpr int kFlagField = 1;     // add the galaxy field
constexpr int kFlagMaskSelf = 2;  // eps == 0: the j = i term must be excluded explicitly
constexpr int kFlagDefer = 4;     // finished by the combine pass even when unsplit (its galaxy model
                                  // is one the pair kernel leaves out)

// O(N) chunk: kChunk consecutive particles of one cluster (also used for sort tiles of
// kSortTile particles).
struct Chunk {
  int cluster, start, count, pad;
};

// Diagnostics: sums reduced per cluster by the energy pass, and doubles written per cluster.
constexpr int kEnergySums = 17;
constexpr int kEnergyOut = 20;

// Pair work item: one i-tile of one cluster against one j-range (js) of it.  In the local mode
// `flag0` is the item's first word of far-tile bits (bits 2t and 2t + 1 of the item's words: its
// j-tile t is far, and far enough for the expanded form of r^2).
struct PairItem {
  int cluster, i0, js, flag0;
};

// ---- The symmetric path (pair_sym.h) ---------------------------------------------------------
// Clusters of kSymMin to kSymMax particles.  Below, one cluster alone is too few items to fill the
// chip (N = 3840 in FP64: 52 us per step one-sided).  Up to 2^20 a cluster's least room (at most 192 bytes per
// particle, 96 from 131072 on) is less than its j-ranges would take (256 to 512, 128 at 2^20), so whatever fitted
// nbody_accel_noalloc with ranges fits with rows.  Above, there are 2 ranges or 1 (64 bytes or none) and that
// no longer holds by itself: one cluster fits up to about 2 million particles (in NB_FP32DL up to its limit
// of 1.4), batches near the scratch limit do not.  The path has not been measured there.
constexpr int kSymMin = 4096, kSymMax = 1 << 20;
constexpr int kSymBlocksPerCu = 2;  // of 8 waves: 4 per SIMD, an even number (pair_sym.h)
// Particles per segment, a function of the cluster's size alone (its sums, and so its bits, depend on
// it): small enough that one cluster has a few items per CU, large enough that the rows (48 bytes
// written and read per particle and segment) stay a small part of the time (the combine pass took 8%
// of the 512-cluster ensemble's step with 256 up to 16383, 4% with 512 from 8192 on; N = 65536: 8.04 ms
// per sym6 step with 1024, 7.65 with 512).  The block's waves cover a segment with their i-groups: 2 x
// 128, 2 x 256 or 4 x 256.
__host__ __device__ inline int sym_segment(int n) { return n < 8192 ? 256 : n < 131072 ? 512 : 1024; }
// Running sums the combine pass keeps per particle between bands (also its threads per particle): four
// while there are too few particles to fill the chip with one thread each.
__host__ __device__ inline int sym_sums(int n) { return n < 131072 ? 4 : 1; }

// Partial records per chunk: the combine pass of a symmetric cluster with four threads per particle takes 64
// particles per block.
__host__ __device__ inline int chunk_records(int n, int seg) { return seg && sym_sums(n) == 4 ? 4 : 1; }

// Rows of the partial-sum table.  Segment pairs are ordered by their circular distance delta = 0 ..
// nseg / 2: the item (A, A + delta) writes row 2 delta - 1 of A's particles and row 2 delta of the
// other's (row 0 of A for delta = 0; row nseg - 1 of both for delta = nseg / 2, which has half the
// items), so every particle gets each of its nseg rows once.  When the room does not hold nseg rows,
// the distances are taken in bands, each a launch of the pair kernel and one of the combine pass,
// which adds the band's rows to the running sums; the order of the additions, and so the result, does
// not depend on the room.
struct SymRows {
  int nseg, ndelta, d_first, d_next;  // distances; distances of the first band and of the later ones
  int cap;                            // rows a band may use
  int nbands;
  __host__ __device__ int delta0(int band) const { return band ? d_first + d_next * (band - 1) : 0; }
  __host__ __device__ int delta1(int band) const {
    const int d = d_first + d_next * band;
    return d < ndelta ? d : ndelta;
  }
  __host__ __device__ int row0(int band) const { return band ? 2 * delta0(band) - 1 : 0; }
  __host__ __device__ int row1(int band) const {
    const int r = 2 * delta1(band) - 1;
    return r < nseg ? r : nseg;
  }
  __host__ __device__ int items(int band) const {
    const int d1 = delta1(band), half = nseg % 2 == 0 && d1 == ndelta;
    return (d1 - delta0(band)) * nseg - (half ? nseg / 2 : 0);
  }
};
__host__ __device__ inline SymRows sym_rows(int n, int nseg, bool pot, long long doubles) {
  SymRows r;
  const long long row = (long long)(pot ? 4 : 3) * n;
  r.nseg = nseg;
  r.ndelta = nseg / 2 + 1;
  if (row * nseg <= doubles) {
    r.cap = nseg;
    r.d_first = r.ndelta;
    r.d_next = 1;
    r.nbands = 1;
  } else {
    r.cap = (int)(doubles / row) - sym_sums(n);
    r.d_first = (r.cap + 1) / 2;
    r.d_next = r.cap / 2;
    r.nbands = 1 + (r.ndelta - r.d_first + r.d_next - 1) / r.d_next;
  }
  return r;
}

// One band of a launch: its work counter, its items, and the clusters that take part.  The first
// item of block b is item b; further ones come from the counter.
struct SymEntry {
  int first;    // the cluster's first item
  int cluster;
  int delta0;   // the band's first distance
  int row0;     // and first row, of this cluster
};
struct SymBand {
  int* counter;
  const SymEntry* entries;  // [ncl]
  int ncl, nitems, index;
  int seg;  // 256: clusters with segments of 256 (two i-particles per lane), else the others
};

// Galaxy models (the values of the C interface's NB_GALAXY_* constants).
constexpr int kGalaxyHernquistLog = 0, kGalaxyAllenSantillan = 1;
struct Galaxy {
  double Mb, ab, Md, ad, bd, vh, dh, Mbh, ebh;
  int model;  // kGalaxyHernquistLog or kGalaxyAllenSantillan
  double Mh, ah, rcut;
};

// Everything the kernels of one call need; passed by value.
struct Args {
  const DevCluster* cl;
  const Chunk* chunks;
  int nchunks;
  int B;               // clusters
  DevCluster cl0;      // the cluster when there is only one (load_cluster, load_chunk)
  const PairItem* items;
  int nitems;
  int* item_counter;   // dynamic work distribution of the persistent pair kernel
  int* chunk_counter;  // [B] chunks finished per cluster (last-block reductions)
  double* partials;    // records of kPartials doubles (nb_device.h)
  double* box;         // [B][6] bounding box of each cluster (min xyz, max xyz)
  // Hilbert-curve sort (NB_FP32DL): keys and local indices (double-buffered), per-tile digit counts and
  // offsets, and the result: perm[off + l] = local index of the particle at sorted position l
  const Chunk* stiles;
  int nstiles;
  unsigned* skey[2];
  int* sval[2];
  int* shist;          // [nstiles][kRadix] digit counts, then each tile's offsets within the digit
  int* sbase;          // [B][kRadix] first destination of each digit in its cluster
  const int* perm;     // null: particles in their own order
  double4* spos;       // [Ntot] (x, y, z, m) in sorted order (NB_FP32DL), else null
  double4* ibox;       // [items] centre of each item's i-particle box, w = (3/4 diagonal)^2 (NB_FP32DL)
  double* tbox;        // [ntboxes][6] bounding box (min xyz, max xyz) of every j-tile (NB_FP32DL)
  int ntboxes;         // box slots (NB_FP32DL)
  unsigned* farflags;  // far-tile bits of every item (NB_FP32DL; item.flag0 is its first word)
  int item_tile;       // i-particles of one work item (64 K (4/W))
  int jtile;           // j-records of one LDS tile (T)
  double* mconst;      // [B] the common mass of a cluster whose masses are all equal, else 0
  double4* ref;        // [B] reference point of each cluster (centre of mass), w = total mass
  int reduced;         // ref and mconst hold the small clusters too (else: chunk_frame)
  double4* part;       // partial sums (ax, ay, az, pot) of split clusters
  double* sym;         // partial-sum rows of the symmetric path's clusters
  double4* gbox;       // [nchunks] centre of each sorted chunk's box, w = (3/4 diagonal)^2 (NB_FP32DL)
  int ncounters;       // work counters from item_counter on
  double* epart;       // [nchunks * kEnergySums] energy partials
  double* pot_ws;      // [Ntot] pair potential scratch for the energy pass
  double* eacc_ws;     // [Ntot * 3] internal accelerations of the energy pass
  double* coef;        // [B*3] per-cluster (kick_pre, drift, kick_post), or null
  // state
  double* pos;
  double* vel;
  double* acc;
  double* pot;
  const double* mass;
  double* eout;  // [B * kEnergyOut] energy output
  int internal_only;  // 1: the pair pass stores the internal acceleration alone (no galaxy field)
  // uniform coefficients (used when coef == null)
  double kick_pre, drift, kick_post;
  const double* coef_next;  // [B*3] or null, and uniform: those of the next stage, which the fused
  double pre_next, drift_next;  // combine + update pass starts
  double G;
  Galaxy gal;
  int prec;  // NB_FP32 .. NB_FP64
};

// Pair-kernel launch shape: K i-particles per lane, W waves sharing an i-group, T j-records per
// LDS tile, bpc persistent blocks per CU.
struct TileCfg {
  int k, w, tile, bpc, phase;
};

// Launchers (kernels_*.hip).  All return hipSuccess or the launch error.
// kick + drift (when update) and chunk partials; `finish`: first the last band of the symmetric clusters'
// rows and the small clusters' ranges (small_cluster), with the kick that ends their stage, then the next
// stage's kick and drift
hipError_t launch_update(const Args& a, bool update, bool finish, hipStream_t s);
// reference point, common mass and box of every cluster from the chunk partials
hipError_t launch_reduce(const Args& a, int B, hipStream_t s);

// the one-sided pair kernel of a mode and shape (null: not compiled in)
typedef void (*PairFn)(Args, int);
PairFn pair_kernel(int prec, const TileCfg& t, bool mask, bool potmode);
hipError_t launch_pair(PairFn fn, const Args& a, int grid, bool kick, hipStream_t s);
hipError_t launch_energy(const Args& a, hipStream_t s);
// kCombineBand: the running sums of the symmetric clusters that have bands after `band`.  kCombineAll ends the
// stage of every cluster that the pair kernels have not finished (symmetric: from its own last band);
// kCombineLarge only of the one-sided ones above the symmetric path.
enum CombineWhat { kCombineBand, kCombineLarge, kCombineAll };
hipError_t launch_combine(const Args& a, CombineWhat what, int band, bool potmode, bool kick, hipStream_t s);
hipError_t launch_pair_sym(const Args& a, const SymBand& b, int grid, bool mask, bool potmode, hipStream_t s);
hipError_t launch_sym_f32(const Args& a, const SymBand& b, int grid, bool mask, bool pot, hipStream_t s);
hipError_t launch_sym_ds(const Args& a, const SymBand& b, int grid, bool mask, bool pot, hipStream_t s);
hipError_t launch_sym_dl(const Args& a, const SymBand& b, int grid, bool mask, bool pot, hipStream_t s);
hipError_t launch_sym_f64(const Args& a, const SymBand& b, int grid, bool mask, bool pot, hipStream_t s);
// Hilbert-curve sort: leaves the permutation in sval[1] and the sorted (x, y, z, m) in spos
hipError_t launch_sort(const Args& a, int B, hipStream_t s);


bool tile_supported(int family, const TileCfg& t);
// the shape's kernel with four i-particles per lane exists (the runtime's choice only)
bool wide_compiled(int family, const TileCfg& t);
// i-particles of one pair work item for a shape
inline int item_tile(const TileCfg& t) { return 64 * t.k * (4 / t.w); }

PairFn pair_kernel_f32(const TileCfg& t, bool fold, bool mask, bool pot);
PairFn pair_kernel_ds(const TileCfg& t, bool fold, bool mask, bool pot);
PairFn pair_kernel_f64(const TileCfg& t, bool fold, bool mask, bool pot);
PairFn pair_kernel_dl(const TileCfg& t, bool fold, bool mask, bool pot);

// Cluster b, and this block's O(N) chunk.  A single cluster comes with the kernel arguments: the loads
// from the tables would be one after the other, about a microsecond of every kernel of a small system.
__device__ __forceinline__ DevCluster load_cluster(const Args& a, int b) { return a.B == 1 ? a.cl0 : a.cl[b]; }
__device__ __forceinline__ Chunk load_chunk(const Args& a) {
  if (a.B != 1) return a.chunks[blockIdx.x];
  const int start = blockIdx.x * kChunk;
  return Chunk{0, start, min(kChunk, a.cl0.n - start), 0};
}

// Index in the state arrays of the particle at (sorted) local position l of cluster c.
__device__ __forceinline__ long long particle_index(const Args& a, const DevCluster& c, int l) {
  return c.off + (a.perm && c.nstiles ? a.perm[c.off + l] : l);
}

// Clusters of the one-sided path below the symmetric one: never sorted, few enough chunks for the pair
// kernel to reduce their partials by itself (chunk_frame).
static_assert(kSymMin / kChunk <= 64, "one chunk per lane");
__host__ __device__ inline bool small_cluster(const DevCluster& c) { return c.n < kSymMin; }

}  // namespace nb
