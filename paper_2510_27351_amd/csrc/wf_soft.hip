// Smooth (soft-min) variant of the wavefront recurrence on gfx950: the adjoint
// (wf_soft_backward in include/wf.h).  The forward runs in the min-plus forward's band
// pipeline (wf_fwd.hip) with the soft-min cell in place of the minimum.
//
// The minimum of the north-west, north and west neighbours is replaced by the soft minimum
// of temperature gamma,  softmin(x) = -gamma log sum_k exp(-x_k / gamma).  The adjoint of
// L = sum(gD * D) + gscore * score  is
//     A[i][j] = gD[i][j] + [last] gscore + w(i+1,j+1) A[i+1][j+1] + w(i+1,j) A[i+1][j]
//             + w(i,j+1) A[i][j+1],       w(succ) = 2^((V(succ) - D[i][j]) log2e / gamma),
// with V(succ) = D(succ) - C(succ) the successor's soft minimum, so the weight is the
// derivative of the successor's soft minimum with respect to D[i][j].  gC = A.  The
// exponent is evaluated as (D(succ) - D[i][j]) log2e/gamma - C(succ) log2e/gamma, one fused
// multiply-add after the difference of two neighbouring table values, which is exact in
// floating point, so the weight's error is that of numbers of the size of C, not of the
// table.  (Forming V first would round it at the table's magnitude, and along a path of L
// cells those roundings add up: at 16384 x 16384 in float32 that made the first cell's
// gradient 8% off.)
//
// Structure.  The weights depend on C and D alone, so only three fused multiply-adds per cell
// are serial; the three exponentials are taken by the waves that load the inputs.  Seen from
// the far corner the sweep is a forward sweep: with row i' = m-1-i and column c' = n-1-c a
// cell reads its west, north and north-west neighbours, and this is the forward's band
// pipeline (wf_fwd.hip) over 64-row bands of i', lane r owning row i' = 64b + r and handling
// column t - r at step t.  Three LDS rings hold the weights of the three neighbours (and a
// fourth gD, when given) at slot (c' + r) mod RING, so that at step t every lane touches slot
// t and four steps are one aligned 16-byte read per ring; A overwrites the west weight, from
// where it is stored as gC.  The waves:
//   wave 0        compute    per 4 steps: the vectors of every ring, 4 x (DPP shift of A from
//                            the lane above, 3 fused multiply-adds), the A vector back to LDS;
//   wave 1        publisher  the band's last row of A as epoch-tagged words for the next band;
//   wave 2        top        polls those of the band before into the top ring, 64 columns per
//                            pass;
//   NL waves      loaders    64 / NL rows each: D and C of the row and of the row below it, the
//                            weights into the rings;
//   one wave      storer     each finished sub-chunk of A back to gC;
//   one wave      gD loader  (only with gD).
// Every wait is bounded.  What bounds it: the compute wave's issue (six VALU instructions per
// step and its LDS accesses) and 63 + 16 steps of skew plus the handoff (about 1.1 us) from
// band to band; in float64 the loaders' exponentials.  With the exponentials in the compute
// wave and (A, D, C) handed on, 4096 x 4096 float32 took 1181 us and one band 64 ns per step.
#include "wf_common.h"
#include "wf_soft.h"

namespace wf {
namespace {

// Four consecutive columns of one row, as one (float) or two (double) 16-byte transfers.
template <typename T>
__device__ __forceinline__ Vec4<T> load4(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  Vec4<T> v;
  if constexpr (sizeof(T) == 4) {
    v = __builtin_bit_cast(Vec4<T>, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
  } else {
    using H = struct alignas(16) { uint32_t w[4]; };
    H lo = __builtin_bit_cast(H, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
    H hi = __builtin_bit_cast(H, __builtin_amdgcn_raw_buffer_load_b128(r, off + 16, 0, 0));
    uint32_t w[8];
    for (int q = 0; q < 4; ++q) {
      w[q] = lo.w[q];
      w[4 + q] = hi.w[q];
    }
    __builtin_memcpy(&v, w, sizeof(v));
  }
  return v;
}

template <typename T>
__device__ __forceinline__ T load1(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
  } else {
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
  }
}

template <typename T>
__device__ __forceinline__ void store1(__amdgpu_buffer_rsrc_t r, uint32_t off, T x) {
  if constexpr (sizeof(T) == 4) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), r, off, 0, 0);
  } else {
    using V2 = __attribute__((ext_vector_type(2))) uint32_t;
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(V2, x), r, off, 0, 0);
  }
}

template <typename T>
__device__ __forceinline__ void store4(__amdgpu_buffer_rsrc_t r, uint32_t off, const Vec4<T>& v) {
  typedef int v4i __attribute__((ext_vector_type(4)));
  if constexpr (sizeof(T) == 4) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, v), r, off, 0, 0);
  } else {
    struct Hf { v4i lo, hi; };
    const Hf h = __builtin_bit_cast(Hf, v);
    __builtin_amdgcn_raw_buffer_store_b128(h.lo, r, off, 0, 0);
    __builtin_amdgcn_raw_buffer_store_b128(h.hi, r, off + 16, 0, 0);
  }
}

template <typename T>
__device__ __forceinline__ Vec4<T> reversed(const Vec4<T>& v) {
  Vec4<T> o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o.v[e] = v.v[3 - e];
  return o;
}

// wave_shl:1 -- lane r receives lane r+1's value; lane 63 keeps its own.
template <typename T>
__device__ __forceinline__ T shl1(T x) {
  auto mv = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x130, 0xf, 0xf, false); };
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, mv(__builtin_bit_cast(uint32_t, x)));
  } else {
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    const uint64_t lo = mv((uint32_t)b), hi = mv((uint32_t)(b >> 32));
    return __builtin_bit_cast(T, (hi << 32) | lo);
  }
}

// Returns x unchanged, but hides its value from the optimiser at this point: each role
// launders the kernel-wide sizes it uses, or the compiler hoists every role's address
// arithmetic out of the band loop and keeps all of it live across all roles.
template <typename V>
__device__ __forceinline__ V opaque(V x) {
  asm volatile("" : "+s"(x));
  return x;
}

template <typename T>
struct SbCfg {
  static constexpr int RING = sizeof(T) == 4 ? 128 : 64;    // slots per row (about 34 KiB a ring)
  static constexpr int PITCH = RING + 16 / (int)sizeof(T);  // row pitch 16 mod 256 bytes
  static constexpr int MASK = RING - 1;
  static constexpr int SUB = RING / 4;       // slots per loader / storer sub-chunk
  static constexpr int LPR = SUB / 4;        // lanes side by side that hold a row of a sub-chunk
  static constexpr int RPV = 64 / LPR;       // rows one vector index spans across the wave
  static constexpr int G = 16;               // columns per handoff unit
  static constexpr int GPS = SUB / G;        // units per sub-chunk
  static constexpr int NG = G / 4;           // 4-step groups per unit
  static constexpr int NVS = kBand / RPV;    // the storer's (and the gD loader's)
  static_assert(GPS >= 1 && SUB % G == 0, "bad tiling");
};

// The weight loaders.  Their loads' latency bounds a band (a sub-chunk of 32 columns is read in
// 0.6 us): many loaders of few rows keep more sub-chunks in flight in the registers a wave may
// use.  float: 8 of 8 rows with 4 sub-chunks each against 4 of 16 rows with 2: one band 124 us
// against 154 per 4096 columns, 4096 x 4096 401 against 434; with gD the ninth and tenth waves'
// share of the registers makes four loaders the faster (531 against 552).
template <typename T, bool HAS_GD>
struct SbLoad {
  using K = SbCfg<T>;
  static constexpr int NL = sizeof(T) == 4 && !HAS_GD ? 8 : 4;
  static constexpr int ROWS = kBand / NL;    // rows of each
  static constexpr int NV = ROWS / K::RPV;   // vectors per lane and sub-chunk
  static constexpr int PF = sizeof(T) == 4 ? (HAS_GD ? 3 : 4) : 2;  // sub-chunks in flight
  static_assert(NV >= 1, "bad tiling");
};

template <typename T, bool HAS_GD>
constexpr int kSbThreads = 64 * (4 + SbLoad<T, HAS_GD>::NL + (HAS_GD ? 1 : 0));

struct alignas(64) SoftShared {
  // 0..7: sub-chunks of weights loaded by loader h, 8: top units loaded, 9: sub-chunks of gD
  // loaded, 10..15: always 0; 16: steps done, 17: units published, 18: sub-chunks stored
  uint32_t ctr[24];
  uint32_t item;
  uint32_t abort;
};
constexpr int kCtrTop = 8, kCtrGd = 9, kCtrSteps = 16, kCtrPub = 17, kCtrStored = 18;
constexpr uint32_t kAllReady = 0x7fffffffu;

// The matrix as a band sees it.  Band b holds rows i' = 64b .. 64b+63, i.e. matrix rows
// row_hi = m-1-64b down; rows below 0 (the last band's) do not exist.  'base' is the band's
// lowest existing matrix row.
struct BandRows {
  int64_t base;
  int hi;     // row_hi - base: the band's first row, relative to base
  int below;  // 1 if the matrix has a row row_hi + 1
};
__device__ __forceinline__ BandRows band_rows(int64_t m, int band) {
  BandRows r;
  const int64_t row_hi = m - 1 - (int64_t)band * kBand;
  r.base = row_hi >= kBand - 1 ? row_hi - (kBand - 1) : 0;
  r.hi = (int)(row_hi - r.base);
  r.below = band > 0 ? 1 : 0;
  return r;
}
// Range-checked resource over 'rows' rows from 'base' of a matrix with leading dimension ld:
// the last row ends at its n-th element.  A negative element offset wraps to a huge one, so
// rows below 0 read as zero and are not stored.
template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const void* p, int64_t base, int rows, int64_t ld, int64_t n) {
  return make_rsrc(static_cast<const T*>(p) + base * ld, (uint32_t)(((int64_t)(rows - 1) * ld + n) * (int64_t)sizeof(T)));
}

// Vector k of a lane in sub-chunk s, of the rows from r0 on: band row l, slots t .. t+3, columns
// c' = t - l .. t - l + 3, i.e. matrix columns c_lo + 3 down to c_lo.
template <typename T>
struct SbVec {
  int l, t;
  __device__ __forceinline__ SbVec(int r0, int k, int s) {
    using K = SbCfg<T>;
    const int lane = threadIdx.x & 63;
    l = r0 + K::RPV * k + lane / K::LPR;
    t = K::SUB * s + 4 * (lane & (K::LPR - 1));
  }
  __device__ __forceinline__ int c_lo(int n) const { return n - 4 - t + l; }
  __device__ __forceinline__ int lds() const { return l * SbCfg<T>::PITCH + (t & SbCfg<T>::MASK); }
};

// Four elements from element offset e of a resource.  EDGE: offsets below 0 read element 0
// instead (a vector that straddles column 0 of the lowest row would otherwise lose its valid
// elements with the others).  32-bit arithmetic: a band spans less than 2^30 bytes.
template <typename T, bool EDGE>
__device__ __forceinline__ Vec4<T> at4(__amdgpu_buffer_rsrc_t r, int e) {
  if constexpr (!EDGE) return load4<T>(r, (uint32_t)e * (uint32_t)sizeof(T));
  Vec4<T> v;
#pragma unroll
  for (int q = 0; q < 4; ++q) v.v[q] = load1<T>(r, (uint32_t)(e + q > 0 ? e + q : 0) * (uint32_t)sizeof(T));
  return v;
}
template <typename T>
__device__ __forceinline__ T at1(__amdgpu_buffer_rsrc_t r, int e) {
  return load1<T>(r, (uint32_t)(e > 0 ? e : 0) * (uint32_t)sizeof(T));
}

// Sub-chunks from here on hold columns below 0 (or element offsets below 0).
template <typename T>
__device__ __forceinline__ bool left_edge(int s, int n) {
  return SbCfg<T>::SUB * (s + 1) > n;
}

// ---------------------------------------------------------------------------------------
// The weight loaders.  A lane's vector needs D of its row at columns c_lo .. c_lo+4,
// D of the row below at the same columns, C of its row at c_lo+1 .. c_lo+4 and C of the row
// below at c_lo .. c_lo+4.
template <typename T>
struct WeightIn {
  Vec4<T> d, db, c, cb;  // c_lo .. c_lo+3 (c: c_lo+1 .. c_lo+4)
  T d4, db4, cb4;        // c_lo+4
};

template <typename T, bool EDGE, int NV>
__device__ __forceinline__ void load_weights(WeightIn<T> (&in)[NV], __amdgpu_buffer_rsrc_t rd,
                                             __amdgpu_buffer_rsrc_t rc, int ldd, int ldc, int n, int hi, int r0, int s) {
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const SbVec<T> v(r0, k, s);
    const int c = v.c_lo(n), i = hi - v.l;
    const int ed = i * ldd + c, ec = i * ldc + c;
    in[k].d = at4<T, EDGE>(rd, ed);
    in[k].d4 = at1<T>(rd, ed + 4);
    in[k].db = at4<T, EDGE>(rd, ed + ldd);
    in[k].db4 = at1<T>(rd, ed + ldd + 4);
    in[k].c = at4<T, EDGE>(rc, ec + 1);
    in[k].cb = at4<T, EDGE>(rc, ec + ldc);
    in[k].cb4 = at1<T>(rc, ec + ldc + 4);
  }
}

// The weights of the lane's cells into the rings.  A weight between cells one of which lies
// outside the matrix is 0; that of the corner's virtual north-west neighbour, which carries
// gscore, is 1.
template <typename T, int NV>
__device__ __forceinline__ void store_weights(T* Ww, T* Wn, T* Wx, const WeightIn<T> (&in)[NV], T kx, int n, int hi, int below, int r0, int s) {
  using M = SoftMath<T>;
  using K = SbCfg<T>;
  // every column c' of the sub-chunk in [1, n), every row and the row below it in the matrix
  const bool interior = K::SUB * s >= kBand && K::SUB * (s + 1) <= n && hi >= kBand - 1 && below != 0;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const SbVec<T> v(r0, k, s);
    const WeightIn<T>& x = in[k];
    const T d5[5] = {x.d.v[0], x.d.v[1], x.d.v[2], x.d.v[3], x.d4};
    const T b5[5] = {x.db.v[0], x.db.v[1], x.db.v[2], x.db.v[3], x.db4};
    T cb[5] = {x.cb.v[0], x.cb.v[1], x.cb.v[2], x.cb.v[3], x.cb4};
#pragma unroll
    for (int q = 0; q < 5; ++q) cb[q] *= kx;
    Vec4<T> w, nn, xx;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int q = 3 - e;  // matrix column c_lo + q
      w.v[e] = M::exp2_(M::fma_(d5[q + 1] - d5[q], kx, -(x.c.v[q] * kx)));
      nn.v[e] = M::exp2_(M::fma_(b5[q] - d5[q], kx, -cb[q]));
      xx.v[e] = M::exp2_(M::fma_(b5[q + 1] - d5[q], kx, -cb[q + 1]));
    }
    if (!interior) {
      const bool row = hi - v.l >= 0, rowb = row && (v.l > 0 || below != 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c1 = v.t - v.l + e;  // c'
        const bool in_w = c1 >= 1 && c1 < n, in_n = c1 >= 0 && c1 < n;
        if (!(row && in_w)) w.v[e] = T(0);
        if (!(rowb && in_n)) nn.v[e] = T(0);
        if (!(rowb && in_w)) xx.v[e] = v.l == 0 && below == 0 && c1 == 0 ? T(1) : T(0);
      }
    }
    *reinterpret_cast<Vec4<T>*>(Ww + v.lds()) = w;
    *reinterpret_cast<Vec4<T>*>(Wn + v.lds()) = nn;
    *reinterpret_cast<Vec4<T>*>(Wx + v.lds()) = xx;
  }
}

template <typename T, bool HAS_GD>
__device__ __forceinline__ bool weight_loader(T* Ww, T* Wn, T* Wx, SoftShared& sh, const SoftArgs& a, int band, int h,
                                              int Ks) {
  using K = SbCfg<T>;
  constexpr int NV = SbLoad<T, HAS_GD>::NV, PF = SbLoad<T, HAS_GD>::PF;
  const int n = (int)opaque(a.n), ldd = (int)opaque(a.ldd), ldc = (int)opaque(a.ldc);
  const BandRows br = band_rows(opaque(a.m), band);
  const __amdgpu_buffer_rsrc_t rd = rows_rsrc<T>(a.Din, br.base, br.hi + 1 + br.below, ldd, n);
  const __amdgpu_buffer_rsrc_t rc = rows_rsrc<T>(a.C, br.base, br.hi + 1 + br.below, ldc, n);
  const T kx = (T)a.kx;
  const int r0 = SbLoad<T, HAS_GD>::ROWS * h;
  uint64_t waited = 0;
  WeightIn<T> in[PF][NV];
  auto load = [&](WeightIn<T> (&x)[NV], int s) {
    __builtin_amdgcn_sched_barrier(0);
    if (left_edge<T>(s, n)) {
      load_weights<T, true, NV>(x, rd, rc, ldd, ldc, n, br.hi, r0, s);
    } else {
      load_weights<T, false, NV>(x, rd, rc, ldd, ldc, n, br.hi, r0, s);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int p = 0; p < PF; ++p) load(in[p], p);
  for (int s0 = 0; s0 < Ks; s0 += PF) {
#pragma unroll
    for (int p = 0; p < PF; ++p) {
      const int s = s0 + p;
      if (s < Ks) {
        // sub-chunk s reuses the slots of sub-chunk s - 4, which must be stored and whose last
        // row must be published
        const int older = s - K::RING / K::SUB;
        if (older >= 0 &&
            (!lds_wait_ge<false>(&sh.ctr[kCtrStored], (uint32_t)(older + 1), &sh.abort, a.ctl, waited) ||
             !lds_wait_ge<false>(&sh.ctr[kCtrPub], (uint32_t)(K::GPS * (older + 1)), &sh.abort, a.ctl, waited)))
          return false;
        store_weights<T, NV>(Ww, Wn, Wx, in[p], kx, n, br.hi, br.below, r0, s);
        lds_signal(&sh.ctr[h], s + 1 < Ks ? (uint32_t)(s + 1) : kAllReady);
        if (s + PF < Ks) load(in[p], s + PF);
      }
    }
  }
  return true;
}

// The gD loader: gD into its ring, 0 outside the matrix.
template <typename T>
__device__ __forceinline__ bool gd_loader(T* Gd, SoftShared& sh, const SoftArgs& a, int band, int Ks) {
  using K = SbCfg<T>;
  const int n = (int)opaque(a.n), ld = (int)opaque(a.ldgd);
  const BandRows br = band_rows(opaque(a.m), band);
  const __amdgpu_buffer_rsrc_t rg = rows_rsrc<T>(a.gD, br.base, br.hi + 1, ld, n);
  uint64_t waited = 0;
  Vec4<T> x[K::NVS];
  auto load = [&](int s) {
    __builtin_amdgcn_sched_barrier(0);
    const bool edge = left_edge<T>(s, n);
#pragma unroll
    for (int k = 0; k < K::NVS; ++k) {
      const SbVec<T> v(0, k, s);
      const int e = (br.hi - v.l) * ld + v.c_lo(n);
      x[k] = edge ? at4<T, true>(rg, e) : at4<T, false>(rg, e);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  load(0);
  for (int s = 0; s < Ks; ++s) {
    // its slots are read by the compute wave alone
    const int older = s - K::RING / K::SUB;
    if (older >= 0 && !lds_wait_ge<false>(&sh.ctr[kCtrSteps], (uint32_t)(K::SUB * (older + 1)), &sh.abort, a.ctl, waited))
      return false;
#pragma unroll
    for (int k = 0; k < K::NVS; ++k) {
      const SbVec<T> v(0, k, s);
      Vec4<T> g = reversed(x[k]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c1 = v.t - v.l + e;
        if (c1 < 0 || c1 >= n || v.l > br.hi) g.v[e] = T(0);
      }
      *reinterpret_cast<Vec4<T>*>(Gd + v.lds()) = g;
    }
    lds_signal(&sh.ctr[kCtrGd], s + 1 < Ks ? (uint32_t)(s + 1) : kAllReady);
    if (s + 1 < Ks) load(s + 1);
  }
  return true;
}

// The storer: gC from the west weights' ring, which the compute wave overwrote with A.
template <typename T>
__device__ __forceinline__ bool sb_store(const T* S, SoftShared& sh, const SoftArgs& a, int band, int Ks) {
  using K = SbCfg<T>;
  const int n = (int)opaque(a.n), ld = (int)opaque(a.ldgc);
  const BandRows br = band_rows(opaque(a.m), band);
  const __amdgpu_buffer_rsrc_t ro = rows_rsrc<T>(a.gC, br.base, br.hi + 1, ld, n);
  constexpr uint32_t es = sizeof(T);
  uint64_t waited = 0;
  for (int s = 0; s < Ks; ++s) {
    // after the publisher has issued the boundary words of these steps, which the next band
    // waits for
    if (!lds_wait_ge(&sh.ctr[kCtrPub], (uint32_t)(K::GPS * (s + 1)), &sh.abort, a.ctl, waited)) return false;
    Vec4<T> x[K::NVS];
#pragma unroll
    for (int k = 0; k < K::NVS; ++k) x[k] = reversed(*reinterpret_cast<const Vec4<T>*>(S + SbVec<T>(0, k, s).lds()));
    if (K::SUB * s >= kBand - 1 && K::SUB * (s + 1) <= n) {  // every column in [0, n)
#pragma unroll
      for (int k = 0; k < K::NVS; ++k) {
        const SbVec<T> v(0, k, s);
        if (v.l <= br.hi) store4<T>(ro, (uint32_t)((br.hi - v.l) * ld + v.c_lo(n)) * es, x[k]);
      }
    } else {
#pragma unroll
      for (int k = 0; k < K::NVS; ++k) {
        const SbVec<T> v(0, k, s);
        if (v.l > br.hi) continue;
        const int c = v.c_lo(n), e0 = (br.hi - v.l) * ld + c;
        if (c >= 0 && c + 4 <= n) {
          store4<T>(ro, (uint32_t)e0 * es, x[k]);
          continue;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (c + q >= 0 && c + q < n) store1<T>(ro, (uint32_t)(e0 + q) * es, x[k].v[q]);
      }
    }
    lds_publish(&sh.ctr[kCtrStored], (uint32_t)(s + 1));
  }
  return true;
}

// wave 1: the band's last row (lane 63's) for the next band.
template <typename T>
__device__ __forceinline__ bool sb_publish(const T* S, SoftShared& sh, const SoftArgs& a, int band, int Us,
                                           uint32_t epoch) {
  using K = SbCfg<T>;
  using E = Elem<T>;
  constexpr int G = K::G, W = E::W;
  const int lane = threadIdx.x & 63;
  const int64_t n = opaque(a.n);
  const bool last_band = band == a.nb - 1;
  uint64_t waited = 0;
  for (int u = 0; u < Us;) {
    uint32_t done;
    if (!lds_wait_value<true, false>(&sh.ctr[kCtrSteps], (uint32_t)(G * (u + 1)), &sh.abort, a.ctl, waited, done))
      return false;
    int k = (int)(done / G) - u;
    if (k > 64 / G) k = 64 / G;
    if (k > Us - u) k = Us - u;
    if (lane < k * G && !last_band) {
      const int64_t j = (int64_t)G * u + lane - (kBand - 1);
      if (j >= 0 && j < n) {
        const T x = S[(kBand - 1) * K::PITCH + ((G * u + lane) & K::MASK)];
#pragma unroll
        for (int q = 0; q < W; ++q) store_word(a.bnd + ((int64_t)band * n + j) * W + q, tagged(E::word(x, q), epoch));
      }
    }
    u += k;
    lds_publish(&sh.ctr[kCtrPub], (uint32_t)u);
  }
  return true;
}

// wave 2: the top row of the band, i.e. the last row of the band before it (zeros for the first
// band and past the last column), one poll of 64 columns at a time.
template <typename T>
__device__ __forceinline__ bool sb_top(T* Tr, SoftShared& sh, const SoftArgs& a, int band, uint32_t epoch) {
  using K = SbCfg<T>;
  using E = Elem<T>;
  constexpr int G = K::G, W = E::W;
  // columns one poll covers: the ring must hold them beside a unit in use
  constexpr int COLS = K::RING >= 128 ? 64 : 32;
  const int lane = threadIdx.x & 63;
  const int64_t n = opaque(a.n);
  const int Ut = (int)((n + G - 1) / G);
  uint64_t waited = 0, t0 = 0;
  uint32_t polls = 0;
  int u = 0;
  while (u < Ut) {
    const int64_t j = (int64_t)G * u + lane;
    T val = E::zero();
    int k = COLS / G;
    if (band > 0) {
      // every lane loads (a lane with no column to read loads spare words of the control block
      // and ignores them)
      const uint64_t* src = j < n ? a.bnd + ((int64_t)(band - 1) * n + j) * W : reinterpret_cast<const uint64_t*>(a.ctl) + 4;
      uint32_t x[W];
      bool ok = true;
#pragma unroll
      for (int w = 0; w < W; ++w) {
        const uint64_t word = load_word(src + w);
        ok = ok && (uint32_t)(word >> 32) == epoch;
        x[w] = (uint32_t)word;
      }
      if (j < n) val = E::from_words(x);
      const uint64_t missing = ~__ballot(ok || j >= n);
      const int run = missing == 0 ? 64 : __builtin_ctzll(missing);
      k = (run < COLS ? run : COLS) / G;
    }
    if (k > Ut - u) k = Ut - u;
    if (k == 0) {
      __builtin_amdgcn_s_sleep(1);
      if ((++polls & 63u) == 0u) {
        if (lds_load(&sh.abort) != 0u || global_aborted(a.ctl)) return false;
        const uint64_t now = __builtin_amdgcn_s_memrealtime();
        if (polls == 64u) {
          t0 = now;
        } else if (now - t0 > kSpinTicks) {
          raise_timeout(a.ctl);
          return false;
        }
      }
      continue;
    }
    polls = 0;
    // the top ring slot of column j is read before step j and reused RING steps later
    const int64_t need_steps = (int64_t)G * (u + k) - K::RING;
    if (need_steps > 0 && !lds_wait_ge(&sh.ctr[kCtrSteps], (uint32_t)need_steps, &sh.abort, a.ctl, waited)) return false;
    if (lane < k * G) Tr[(int)(j & K::MASK)] = val;
    u += k;
    lds_signal(&sh.ctr[kCtrTop], (uint32_t)u);
  }
  // units past the last real column hold no values any real cell reads
  if (lane == 0) lds_signal(&sh.ctr[kCtrTop], kAllReady);
  return true;
}

// ---------------------------------------------------------------------------------------
// wave 0: the chain.
template <typename T>
struct SbState {
  T X;    // previous A (the west neighbour)
  T NW;   // previous step's north neighbour
  T top;  // the row above the band, shifted down one lane per step: lane 0 holds its next column
};

template <typename T, bool HAS_GD>
struct SbGroup {
  Vec4<T> w, n, x;  // weights of the west, north and north-west neighbours
  Vec4<T> g[1];     // gD (read only with HAS_GD)
};

template <typename T, bool HAS_GD>
__device__ __forceinline__ void sb_load_group(const T* Ww, const T* Wn, const T* Wx, const T* Gd, int at,
                                              SbGroup<T, HAS_GD>& r) {
  r.w = *reinterpret_cast<const Vec4<T>*>(Ww + at);
  r.n = *reinterpret_cast<const Vec4<T>*>(Wn + at);
  r.x = *reinterpret_cast<const Vec4<T>*>(Wx + at);
  if constexpr (HAS_GD) r.g[0] = *reinterpret_cast<const Vec4<T>*>(Gd + at);
}

// Four steps: A = ((gD + w_nw A_nw) + w_n A_n) + w_w A_w, one fused multiply-add per term, in
// this order.
template <typename T, bool HAS_GD>
__device__ __forceinline__ void sb_cells4(SbState<T>& st, const SbGroup<T, HAS_GD>& r, Vec4<T>& d) {
  using M = SoftMath<T>;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const T N = Elem<T>::shr1(st.X, st.top);
    st.top = shl1(st.top);
    T acc = M::fma_(r.x.v[q], st.NW, HAS_GD ? r.g[0].v[q] : T(0));
    acc = M::fma_(r.n.v[q], N, acc);
    st.X = M::fma_(r.w.v[q], st.X, acc);
    st.NW = N;
    d.v[q] = st.X;
  }
}

// float: one instruction block per four steps, as the forward's cells (wf_fwd.hip): shifting
// the top row and copying it into the DPP move's "old" operand fill the two states between
// the write of A and the move that reads it; the s_nop covers a copy of A or 'top' placed
// right before the block.
#define WF_SB1(T0, NW, X, D, WX, WN, WW, GD)                              \
  "v_mov_b32 " T0 ", %[top]\n\t"                                          \
  "v_mov_b32_dpp " T0 ", " X " wave_shr:1 row_mask:0xf bank_mask:0xf\n\t" \
  "v_fma_f32 " D ", " WX ", " NW ", " GD "\n\t"                           \
  "v_fma_f32 " D ", " WN ", " T0 ", " D "\n\t"                            \
  "v_fma_f32 " D ", " WW ", " X ", " D "\n\t"                             \
  "v_mov_b32_dpp %[top], %[top] wave_shl:1 row_mask:0xf bank_mask:0xf\n\t"
#define WF_SB_REGS                                                                                                  \
  [top] "+v"(st.top), [nw] "+v"(st.NW), [t] "=&v"(t), [d0] "=&v"(d.v[0]), [d1] "=&v"(d.v[1]), [d2] "=&v"(d.v[2]), \
      [d3] "=&v"(d.v[3])
#define WF_SB_IN                                                                                                   \
  [x] "v"(st.X), [x0] "v"(r.x.v[0]), [x1] "v"(r.x.v[1]), [x2] "v"(r.x.v[2]), [x3] "v"(r.x.v[3]),                   \
      [n0] "v"(r.n.v[0]), [n1] "v"(r.n.v[1]), [n2] "v"(r.n.v[2]), [n3] "v"(r.n.v[3]), [w0] "v"(r.w.v[0]),          \
      [w1] "v"(r.w.v[1]), [w2] "v"(r.w.v[2]), [w3] "v"(r.w.v[3])
template <>
__device__ __forceinline__ void sb_cells4<float, false>(SbState<float>& st, const SbGroup<float, false>& r,
                                                        Vec4<float>& d) {
  float t;
  asm("s_nop 0\n\t" WF_SB1("%[t]", "%[nw]", "%[x]", "%[d0]", "%[x0]", "%[n0]", "%[w0]", "0")
          WF_SB1("%[nw]", "%[t]", "%[d0]", "%[d1]", "%[x1]", "%[n1]", "%[w1]", "0")
              WF_SB1("%[t]", "%[nw]", "%[d1]", "%[d2]", "%[x2]", "%[n2]", "%[w2]", "0")
                  WF_SB1("%[nw]", "%[t]", "%[d2]", "%[d3]", "%[x3]", "%[n3]", "%[w3]", "0")
      : WF_SB_REGS
      : WF_SB_IN);
  st.X = d.v[3];
}
template <>
__device__ __forceinline__ void sb_cells4<float, true>(SbState<float>& st, const SbGroup<float, true>& r,
                                                       Vec4<float>& d) {
  float t;
  asm("s_nop 0\n\t" WF_SB1("%[t]", "%[nw]", "%[x]", "%[d0]", "%[x0]", "%[n0]", "%[w0]", "%[g0]")
          WF_SB1("%[nw]", "%[t]", "%[d0]", "%[d1]", "%[x1]", "%[n1]", "%[w1]", "%[g1]")
              WF_SB1("%[t]", "%[nw]", "%[d1]", "%[d2]", "%[x2]", "%[n2]", "%[w2]", "%[g2]")
                  WF_SB1("%[nw]", "%[t]", "%[d2]", "%[d3]", "%[x3]", "%[n3]", "%[w3]", "%[g3]")
      : WF_SB_REGS
      : WF_SB_IN, [g0] "v"(r.g[0].v[0]), [g1] "v"(r.g[0].v[1]), [g2] "v"(r.g[0].v[2]), [g3] "v"(r.g[0].v[3]));
  st.X = d.v[3];
}

template <typename T, bool HAS_GD>
__device__ __forceinline__ bool sb_compute(T* __restrict__ Ww, const T* __restrict__ Wn, const T* __restrict__ Wx,
                                           const T* __restrict__ Gd, const T* __restrict__ Tr, SoftShared& sh,
                                           const SoftArgs& a, int band, int Ks) {
  using K = SbCfg<T>;
  using E = Elem<T>;
  const int lane = threadIdx.x & 63;
  SbState<T> st{E::zero(), E::zero(), E::zero()};
  // the score's upstream value enters through the corner's virtual north-west neighbour
  if (band == 0 && lane == 0 && a.gscore) st.NW = *static_cast<const T*>(a.gscore);
  uint64_t waited = 0;
  // lane l's copy of counter l % 16 against what the next unit needs of it: one LDS read and
  // one compare test all of them
  const int which = lane & 15;
  const bool is_sub = which < SbLoad<T, HAS_GD>::NL || (HAS_GD && which == kCtrGd), is_top = which == kCtrTop;
  uint32_t need = is_sub || is_top ? 1u : 0u;
  const uint32_t per_unit = is_top ? 1u : 0u, per_sub = is_sub ? 1u : 0u;
  auto load_ready = [&]() -> uint32_t {
    return __hip_atomic_load(&sh.ctr[which], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  auto wait = [&]() -> bool {
    return lds_wait_until([&] { return __ballot(load_ready() < need) == 0; }, &sh.abort, a.ctl, waited);
  };
  const int row = lane * K::PITCH;
  SbGroup<T, HAS_GD> P[2];
  T top;
  auto load_unit = [&](int slot) {
    sb_load_group<T, HAS_GD>(Ww, Wn, Wx, Gd, row + slot, P[0]);
    sb_load_group<T, HAS_GD>(Ww, Wn, Wx, Gd, row + slot + 4, P[1]);
    top = Tr[slot + (lane & (K::G - 1))];
  };
  if (!wait()) return false;
  load_unit(0);
  for (int s = 0; s < Ks; ++s) {
#pragma unroll
    for (int v = 0; v < K::GPS; ++v) {
      const int base = (K::SUB * s + K::G * v) & K::MASK, next = (K::SUB * s + K::G * (v + 1)) & K::MASK;
      need += per_unit;
      if (v + 1 == K::GPS) need += per_sub;
      // one unit, as in the forward: reads two groups ahead, the next unit's first groups read
      // early and, if its inputs were not there yet, again after this unit is signalled
      const uint32_t ready = load_ready();
      __builtin_amdgcn_sched_barrier(0);
      SbGroup<T, HAS_GD> gr[K::NG];
      gr[0] = P[0];
      gr[1] = P[1];
      st.top = top;
      bool late = false;
#pragma unroll
      for (int g = 0; g < K::NG; ++g) {
        if (g + 2 < K::NG) {
          sb_load_group<T, HAS_GD>(Ww, Wn, Wx, Gd, row + base + 4 * (g + 2), gr[g + 2]);
        } else if (g + 2 == K::NG) {
          late = __ballot(ready < need) != 0;
          __builtin_amdgcn_sched_barrier(0);
          sb_load_group<T, HAS_GD>(Ww, Wn, Wx, Gd, row + next, P[0]);
          top = Tr[next + (lane & (K::G - 1))];
        } else {
          sb_load_group<T, HAS_GD>(Ww, Wn, Wx, Gd, row + next + 4, P[1]);
        }
        __builtin_amdgcn_sched_barrier(0);
        Vec4<T> d;
        sb_cells4<T, HAS_GD>(st, gr[g], d);
        *reinterpret_cast<Vec4<T>*>(Ww + row + base + 4 * g) = d;
      }
      lds_signal(&sh.ctr[kCtrSteps], (uint32_t)(K::SUB * s + K::G * (v + 1)));
      __builtin_amdgcn_sched_barrier(0);
      if (__builtin_expect(late, 0)) {
        if (!wait()) return false;
        // hidden from the optimiser, which would take these reads for repeats of the early ones
        load_unit(opaque(next));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  return true;
}

template <typename T, bool HAS_GD>
__global__ __launch_bounds__((kSbThreads<T, HAS_GD>), 1) void soft_bwd_kernel(SoftArgs a) {
  using K = SbCfg<T>;
  constexpr int NL = SbLoad<T, HAS_GD>::NL;
  constexpr int NV4 = kBand * K::PITCH / 4;
  __shared__ Vec4<T> W4[3][NV4];
  __shared__ Vec4<T> G4[HAS_GD ? NV4 : 1];
  __shared__ Vec4<T> Tr4[K::RING / 4];
  __shared__ SoftShared sh;
  T* Ww = reinterpret_cast<T*>(W4[0]);
  T* Wn = reinterpret_cast<T*>(W4[1]);
  T* Wx = reinterpret_cast<T*>(W4[2]);
  T* Gd = reinterpret_cast<T*>(G4);
  T* Tr = reinterpret_cast<T*>(Tr4);
  Control* ctl = a.ctl;
  const uint32_t epoch = __hip_atomic_load(&ctl->epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (threadIdx.x == 0) sh.abort = 0u;
  for (;;) {
    if (threadIdx.x < 24) sh.ctr[threadIdx.x] = 0u;
    claim_next(ctl, &sh.item, &sh.abort);
    const int band = (int)sh.item;
    if (band >= a.nb || sh.abort != 0u) break;
    bool ok = true;
    const int Ks = (int)((a.n + kBand - 1 + K::SUB - 1) / K::SUB);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // uniform branches below
    if (wave == 0) {
      ok = sb_compute<T, HAS_GD>(Ww, Wn, Wx, Gd, Tr, sh, a, band, Ks);
    } else if (wave == 1) {
      ok = sb_publish<T>(Ww, sh, a, band, Ks * K::GPS, epoch);
    } else if (wave == 2) {
      ok = sb_top<T>(Tr, sh, a, band, epoch);
    } else if (wave < 3 + NL) {
      ok = weight_loader<T, HAS_GD>(Ww, Wn, Wx, sh, a, band, wave - 3, Ks);
    } else if (wave == 3 + NL) {
      ok = sb_store<T>(Ww, sh, a, band, Ks);
    } else {
      if constexpr (HAS_GD) ok = gd_loader<T>(Gd, sh, a, band, Ks);
    }
    if (!ok) sh.abort = 1u;
    __syncthreads();
  }
  finish_launch(ctl, epoch);
}

template <typename T>
void launch_t(const SoftArgs& a, int grid, hipStream_t s) {
  if (a.gD) {
    hipLaunchKernelGGL((soft_bwd_kernel<T, true>), dim3(grid), dim3(kSbThreads<T, true>), 0, s, a);
  } else {
    hipLaunchKernelGGL((soft_bwd_kernel<T, false>), dim3(grid), dim3(kSbThreads<T, false>), 0, s, a);
  }
}

}  // namespace

hipError_t launch_soft_backward(int dtype, const SoftArgs& a, int grid, hipStream_t s) {
  if (dtype == 0) {
    launch_t<float>(a, grid, s);
  } else if (dtype == 1) {
    launch_t<double>(a, grid, s);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace wf
