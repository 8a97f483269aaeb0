// Persistent band-pipelined forward sweep (gfx950).
//
// Work decomposition.  The m x n table is cut into bands of H = 64*R rows, R = 1, 2 or 4
// (forward_rows, wf_api.hip).  A persistent workgroup claims bands in increasing order from a device
// counter and sweeps each band from left to right as a skewed wavefront.  Lane r of the
// compute wave owns the R adjacent rows R*r .. R*r+R-1 of the band: at step t it produces
// column t - r of each of them, top to bottom.  The three inputs of a cell come from registers:
//   W  the lane's previous value in the same row;
//   N  the cell just produced in the row above; for the lane's first row, the previous value
//      of lane r-1's last row moved by a DPP wave_shr:1; lane 0 takes the row above the band
//      (the "top" ring in LDS, published by the band above);
//   NW the previous step's N.
// A band takes n + 63 steps and the band below trails it by 63 + G steps plus the handoff
// latency: all m+n-1 anti-diagonals in one launch, with one handoff through global memory
// per H rows.
//
// What bounds it.  A step is a serial chain in one wave (DPP move with its wait states, then a
// v_min3 and an add per row: 5, 7 and 11 instructions of 4.1 cycles for R = 1, 2, 4) plus that
// wave's own LDS instructions, which the chain waits out: on this chip a ds_write_b128 holds
// the wave for 24 cycles, a ds_read_b128 for 4, and a change from VALU to LDS for 8.  Rows
// side by side in a lane share the DPP move and halve the handoffs, so R = 2 runs 128 rows in
// 59 cycles a step where R = 1 runs 64 in 36; against rows 64 apart in a lane (two DPP moves
// and one more skew of 65 steps per band) 512 ragged instances take 673 us instead of 1000.
//
// Skewed LDS ring.  LDS row l holds band row R*(l%64) + l/64, and its column c lies at slot
// (c + l%64) mod RING: at step t every lane touches slot t of its rows, so a lane's four
// consecutive steps are one aligned 16-byte LDS access per row.  A 16-byte chunk of slots
// [4j, 4j+4) of a row holds four consecutive columns, which are also consecutive in global
// memory, so every global transfer is one (4-byte aligned) 16-byte access paired with one
// aligned 16-byte LDS access.  The row pitch is 16 mod 256 bytes, which keeps 16-byte
// accesses of different rows on distinct banks.  D overwrites C in place.
//
// 3 + 2R waves per workgroup:
//   wave 0           compute   per 4 steps and row: one 16-byte LDS read of C, 4 cells, one
//                              16-byte LDS write of D; the top row by G or by 4 steps;
//   wave 1           publisher publishes the values of the band's last row that became final
//                              since its previous pass (whole units of G steps, up to 64
//                              columns) as tagged words for the band below, and the
//                              checkpoint rows;
//   wave 2           top       polls the band above's tagged boundary words, 64 columns per
//                              pass, and fills the top ring with every complete unit of G
//                              columns;
//   waves 3 .. 2+R   loaders   64 rows each: sub-chunks of SUB slots of C, 16-byte buffer loads
//                              and 16-byte LDS writes, PF sub-chunks in flight in registers;
//   waves 3+R ..     storers   64 rows each: every finished sub-chunk's D (16-byte LDS read,
//                              16-byte global store), the checkpoint columns and the score.
// The publisher has a wave of its own so that nothing delays the handoff, which sits on
// the critical path of the whole sweep.  G (16/32/64, the "tile width") is the handoff
// granularity.
//
// The same pipeline runs the soft-min variant of the recurrence (wf_soft_forward): with the
// SOFT option the compute wave applies the soft-min cell to values in the scaled domain
// y = D log2(e) / gamma, the publisher hands the last row on in that domain, and the storer
// writes D = y gamma ln 2.
#include <type_traits>

#include "wf_common.h"
#include "wf_soft.h"

namespace wf {
namespace {

// Returns x unchanged, but hides its value from the optimiser at this point.
template <typename V>
__device__ __forceinline__ V opaque(V x) {
  asm volatile("" : "+s"(x));
  return x;
}

template <typename T, int G, int R>
struct FwdCfg {
  using E = Elem<T>;
  static constexpr int H = kBand * R;  // rows per band
  // LDS ring: H rows x RING slots, about 128 KiB.
  static constexpr int RING = (sizeof(T) == 4 ? 512 : 256) / R;
  static constexpr int PITCH = RING + 16 / (int)sizeof(T);
  static constexpr int MASK = RING - 1;
  // Slots per loader / storer sub-chunk: four sub-chunks or more in the ring.
  static constexpr int SUB = RING >= 256 ? 64 : 32;
  // A sub-chunk of 64 rows is NV 4-column vectors per lane: LPR lanes side by side hold a row.
  static constexpr int LPR = SUB / 4;
  static constexpr int NV = 64 / (64 / LPR);
  // Sub-chunks a loader keeps in flight in registers (bounded by the registers a wave may
  // use when several share a SIMD).
  static constexpr int PF = R == 4 ? 3 : SUB * sizeof(T) <= 256 ? 2 : 1;
  static constexpr int GPS = SUB / G;   // handoff units per sub-chunk
  static constexpr int NG = G / 4;      // 4-step groups per unit
  // Waves: compute, top, publisher, and a loader and a storer for every 64 rows.
  static constexpr int WAVES = 3 + 2 * R;
  static constexpr int THREADS = 64 * WAVES;
  static_assert(RING % SUB == 0 && SUB % G == 0, "bad tiling");
  static_assert(RING >= 4 * SUB, "ring too small");
};

// LDS row l of a band holds the band's row R * (l % 64) + l / 64 (lane l % 64's row l / 64),
// whose column at step t is t - l % 64.
template <int R>
__device__ __forceinline__ int band_row(int l) {
  return R * (l & 63) + (l >> 6);
}
template <int R>
__device__ __forceinline__ int lds_row(int i) {
  return (i % R) * kBand + i / R;
}
__device__ __forceinline__ int skew(int l) { return l & 63; }

struct alignas(32) Shared {
  // 0..3: C sub-chunks loaded by loader h, 4: top units loaded, 5..7: always 0; 8: steps
  // done, 9: units published, 10..13: sub-chunks stored by storer h
  uint32_t ctr[16];
  uint32_t item;
  uint32_t abort;
  uint32_t warm;  // 1 once the compute wave has run its loop once (see compute_band)
  uint32_t spare;
};
constexpr int kCtrTop = 4, kCtrSteps = 8, kCtrPub = 9;
__device__ __forceinline__ constexpr int ctr_loaded(int h) { return h; }
__device__ __forceinline__ constexpr int ctr_stored(int h) { return 10 + h; }
constexpr uint32_t kAllReady = 0x7fffffffu;

// Every role below launders the kernel-wide sizes it uses through opaque() first:
// otherwise the compiler hoists each role's per-row address arithmetic out of the band loop
// and keeps all of it live across every role, which does not fit 256 registers per wave.

// ---------------------------------------------------------------------------------------
// wave 0: the cell chains
template <typename T, int R>
struct ComputeState {
  T X[R];  // previous value of each of the lane's rows (W of the next cell)
  T NW;    // previous N of the lane's first row (NW of its next cell)
  T top;   // without kTopVec: the row above the band, shifted down one lane per step: lane 0
           // holds the value at its next column
};

// Whether the row above the band is read from LDS with every group, the four steps' values in
// every lane, or with every unit, a column per lane, and shifted down a lane per step.
template <typename T, int R>
constexpr bool kTopVec = sizeof(T) == 8 || (R == 1 && std::is_same<T, int32_t>::value);

// C of the lane's rows at four steps, and with kTopVec the row above the band there.
template <typename T, int R>
struct GroupRegs {
  Vec4<T> c[R];
  Vec4<T> t;
};
template <typename T, int G, int R>
__device__ __forceinline__ void load_group(const T* __restrict__ S, const T* __restrict__ Tr, int slot, int lane,
                                           GroupRegs<T, R>& r) {
  using C = FwdCfg<T, G, R>;
#pragma unroll
  for (int k = 0; k < R; ++k) r.c[k] = *reinterpret_cast<const Vec4<T>*>(S + (k * kBand + lane) * C::PITCH + slot);
  if constexpr (kTopVec<T, R>) r.t = *reinterpret_cast<const Vec4<T>*>(Tr + slot);
}

// Four steps, X = C + min(NW, N, W) per cell, of a lane's R adjacent rows.  N of the first
// row is lane r-1's last row's previous value, moved by a DPP wave_shr:1 whose "old" operand
// fills lane 0 with the top row's value; NW is the previous N.  The second row's N is the
// cell just computed and its NW the first row's previous one.
//
// One asm block per four steps: a DPP move may read a register two instructions after the
// VALU wrote it at the earliest, and shifting the top row and copying it into the move's
// "old" operand are exactly those two.  Left to the compiler, the minimum (which must be
// v_min3 itself: fminf on DPP-shifted operands costs a canonicalising instruction each)
// drew a further wait state per step after every asm statement.  The s_nop covers a copy of X
// or 'top' that the compiler may place right before the block.  (int32 with one row per lane
// and double go another way: see below.)
template <typename T>
struct Cell4;

#define WF_STEP1(T0, NW, X, D, C)                                         \
  "v_mov_b32 " T0 ", %[top]\n\t"                                          \
  "v_mov_b32_dpp " T0 ", " X " wave_shr:1 row_mask:0xf bank_mask:0xf\n\t" \
  "v_min3_f32 " D ", " NW ", " T0 ", " X "\n\t"                           \
  "v_add_f32 " D ", " C ", " D "\n\t"                                     \
  "v_mov_b32_dpp %[top], %[top] wave_shl:1 row_mask:0xf bank_mask:0xf\n\t"
#define WF_STEP2(MIN3, ADD, CLAMP, T0, NW, XA, XB, DA, DB, CA, CB) \
  "v_mov_b32 " T0 ", %[top]\n\t"                                   \
  "v_mov_b32_dpp " T0 ", " XB " wave_shr:1 row_mask:0xf bank_mask:0xf\n\t" \
  MIN3 " " DA ", " NW ", " T0 ", " XA "\n\t"                       \
  ADD " " DA ", " CA ", " DA CLAMP "\n\t"                          \
  MIN3 " " DB ", " XA ", " DA ", " XB "\n\t"                       \
  ADD " " DB ", " CB ", " DB CLAMP "\n\t"                          \
  "v_mov_b32_dpp %[top], %[top] wave_shl:1 row_mask:0xf bank_mask:0xf\n\t"
#define WF_STEP4(MIN3, ADD, CLAMP, T0, NW, XA, XB, XC, XD, DA, DB, DC, DD, CA, CB, CC, CD) \
  "v_mov_b32 " T0 ", %[top]\n\t"                                   \
  "v_mov_b32_dpp " T0 ", " XD " wave_shr:1 row_mask:0xf bank_mask:0xf\n\t" \
  MIN3 " " DA ", " NW ", " T0 ", " XA "\n\t"                       \
  ADD " " DA ", " CA ", " DA CLAMP "\n\t"                          \
  MIN3 " " DB ", " XA ", " DA ", " XB "\n\t"                       \
  ADD " " DB ", " CB ", " DB CLAMP "\n\t"                          \
  MIN3 " " DC ", " XB ", " DB ", " XC "\n\t"                       \
  ADD " " DC ", " CC ", " DC CLAMP "\n\t"                          \
  MIN3 " " DD ", " XC ", " DC ", " XD "\n\t"                       \
  ADD " " DD ", " CD ", " DD CLAMP "\n\t"                          \
  "v_mov_b32_dpp %[top], %[top] wave_shl:1 row_mask:0xf bank_mask:0xf\n\t"
#define WF_CELL4(T, MIN3, ADD, CLAMP)                                                                           \
  template <>                                                                                                   \
  struct Cell4<T> {                                                                                             \
    __device__ static __forceinline__ void run(ComputeState<T, 1>& st, const GroupRegs<T, 1>& r, Vec4<T> (&d)[1]); \
    __device__ static __forceinline__ void run(ComputeState<T, 2>& st, const GroupRegs<T, 2>& r, Vec4<T> (&d)[2]) { \
      const Vec4<T>(&c)[2] = r.c;                                                                               \
      T t;                                                                                                      \
      asm("s_nop 0\n\t" WF_STEP2(MIN3, ADD, CLAMP, "%[t]", "%[nw]", "%[xa]", "%[xb]", "%[a0]", "%[b0]", "%[c0]", "%[e0]") \
              WF_STEP2(MIN3, ADD, CLAMP, "%[nw]", "%[t]", "%[a0]", "%[b0]", "%[a1]", "%[b1]", "%[c1]", "%[e1]") \
                  WF_STEP2(MIN3, ADD, CLAMP, "%[t]", "%[nw]", "%[a1]", "%[b1]", "%[a2]", "%[b2]", "%[c2]", "%[e2]") \
                      WF_STEP2(MIN3, ADD, CLAMP, "%[nw]", "%[t]", "%[a2]", "%[b2]", "%[a3]", "%[b3]", "%[c3]", "%[e3]") \
          : [top] "+v"(st.top), [nw] "+v"(st.NW), [t] "=&v"(t), [a0] "=&v"(d[0].v[0]), [a1] "=&v"(d[0].v[1]),   \
            [a2] "=&v"(d[0].v[2]), [a3] "=&v"(d[0].v[3]), [b0] "=&v"(d[1].v[0]), [b1] "=&v"(d[1].v[1]),         \
            [b2] "=&v"(d[1].v[2]), [b3] "=&v"(d[1].v[3])                                                        \
          : [xa] "v"(st.X[0]), [xb] "v"(st.X[1]), [c0] "v"(c[0].v[0]), [c1] "v"(c[0].v[1]), [c2] "v"(c[0].v[2]), \
            [c3] "v"(c[0].v[3]), [e0] "v"(c[1].v[0]), [e1] "v"(c[1].v[1]), [e2] "v"(c[1].v[2]),                 \
            [e3] "v"(c[1].v[3]));                                                                               \
      st.X[0] = d[0].v[3];                                                                                      \
      st.X[1] = d[1].v[3];                                                                                      \
    }                                                                                                           \
    template <int q>                                                                                            \
    __device__ static __forceinline__ void two(ComputeState<T, 4>& st, const Vec4<T> (&c)[4], Vec4<T> (&d)[4]) { \
      T t;                                                                                                      \
      asm("s_nop 0\n\t" WF_STEP4(MIN3, ADD, CLAMP, "%[t]", "%[nw]", "%[xa]", "%[xb]", "%[xc]", "%[xd]", "%[a0]", \
                                 "%[b0]", "%[c0]", "%[d0]", "%[ia0]", "%[ib0]", "%[ic0]", "%[id0]")             \
              WF_STEP4(MIN3, ADD, CLAMP, "%[nw]", "%[t]", "%[a0]", "%[b0]", "%[c0]", "%[d0]", "%[a1]", "%[b1]",  \
                       "%[c1]", "%[d1]", "%[ia1]", "%[ib1]", "%[ic1]", "%[id1]")                                \
          : [top] "+v"(st.top), [nw] "+v"(st.NW), [t] "=&v"(t), [a0] "=&v"(d[0].v[q]), [a1] "=&v"(d[0].v[q + 1]), \
            [b0] "=&v"(d[1].v[q]), [b1] "=&v"(d[1].v[q + 1]), [c0] "=&v"(d[2].v[q]), [c1] "=&v"(d[2].v[q + 1]),  \
            [d0] "=&v"(d[3].v[q]), [d1] "=&v"(d[3].v[q + 1])                                                    \
          : [xa] "v"(st.X[0]), [xb] "v"(st.X[1]), [xc] "v"(st.X[2]), [xd] "v"(st.X[3]), [ia0] "v"(c[0].v[q]),   \
            [ia1] "v"(c[0].v[q + 1]), [ib0] "v"(c[1].v[q]), [ib1] "v"(c[1].v[q + 1]), [ic0] "v"(c[2].v[q]),     \
            [ic1] "v"(c[2].v[q + 1]), [id0] "v"(c[3].v[q]), [id1] "v"(c[3].v[q + 1]));                          \
      for (int k = 0; k < 4; ++k) st.X[k] = d[k].v[q + 1];                                                      \
    }                                                                                                           \
    __device__ static __forceinline__ void run(ComputeState<T, 4>& st, const GroupRegs<T, 4>& r, Vec4<T> (&d)[4]) { \
      two<0>(st, r.c, d);                                                                                       \
      two<2>(st, r.c, d);                                                                                         \
    }                                                                                                           \
  };
WF_CELL4(float, "v_min3_f32", "v_add_f32", "")
// saturating, so that +inf (INT32_MAX) stays +inf on the virtual border
WF_CELL4(int32_t, "v_min3_i32", "v_add_i32", " clamp")

// One row per lane.  float: the block.  int32 and double: the compiler's code, with the row
// above read from LDS once per four steps (kTopVec): it needs no wait state beyond the DPP
// move's own there and puts the LDS instructions into those, so that a step is shorter than
// with a register to copy and to shift.  64 x 16384, scores only, us: int32 239 against 244
// in the block, double 382 against 421 with a register; float 244 in the block, 248 in one
// without a register, 264 in the compiler's code.
__device__ __forceinline__ void Cell4<float>::run(ComputeState<float, 1>& st, const GroupRegs<float, 1>& r,
                                                  Vec4<float> (&d)[1]) {
  const Vec4<float>& c = r.c[0];
  float t;
  asm("s_nop 0\n\t" WF_STEP1("%[t]", "%[nw]", "%[x]", "%[d0]", "%[c0]")
          WF_STEP1("%[nw]", "%[t]", "%[d0]", "%[d1]", "%[c1]") WF_STEP1("%[t]", "%[nw]", "%[d1]", "%[d2]", "%[c2]")
              WF_STEP1("%[nw]", "%[t]", "%[d2]", "%[d3]", "%[c3]")
      : [top] "+v"(st.top), [nw] "+v"(st.NW), [t] "=&v"(t), [d0] "=&v"(d[0].v[0]), [d1] "=&v"(d[0].v[1]),
        [d2] "=&v"(d[0].v[2]), [d3] "=&v"(d[0].v[3])
      : [x] "v"(st.X[0]), [c0] "v"(c.v[0]), [c1] "v"(c.v[1]), [c2] "v"(c.v[2]), [c3] "v"(c.v[3]));
  st.X[0] = d[0].v[3];
}
__device__ __forceinline__ void Cell4<int32_t>::run(ComputeState<int32_t, 1>& st, const GroupRegs<int32_t, 1>& r,
                                                    Vec4<int32_t> (&d)[1]) {
  using E = Elem<int32_t>;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int32_t N = E::shr1(st.X[0], r.t.v[q]);
    st.X[0] = E::add(r.c[0].v[q], E::min3(st.NW, N, st.X[0]));
    st.NW = N;
    d[0].v[q] = st.X[0];
  }
}

__device__ __forceinline__ double min_raw(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
template <>
struct Cell4<double> {
  template <int R>
  __device__ static __forceinline__ void run(ComputeState<double, R>& st, const GroupRegs<double, R>& r,
                                             Vec4<double> (&d)[R]) {
    using E = Elem<double>;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      double N = E::shr1(st.X[R - 1], r.t.v[q]), NW = st.NW;
      st.NW = N;
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const double W = st.X[k];
        st.X[k] = r.c[k].v[q] + min_raw(min_raw(NW, W), N);
        NW = W;
        N = st.X[k];
        d[k].v[q] = st.X[k];
      }
    }
  }
};

// SOFT: the soft-min cell instead (one row per lane only), on values in the scaled domain
// y = D log2(e) / gamma, the loader having scaled C the same way.  float: the operations of
// soft_cell, one instruction each, as one block per four steps like the min-plus cell's.  A
// step is issue-bound (13 instructions of 4.1 cycles and 3 transcendental ones of 8.6); left
// to the compiler it took 62 ns: it canonicalised the shifted operands, tested for +inf by a
// compare and a select, and waited a state after most inline or transcendental results.  A
// transcendental result may be read two instructions later at the earliest: the second
// exponential, an add and the top row's shift stand between.  Three inputs of +inf give
// inf - inf = NaN, which the minimum with their own minimum turns into +inf; every other
// soft minimum is not above it and stays as it is.  C is added after that: a NaN there (the
// library asks for finite inputs) shows in its cell.
__device__ __forceinline__ double max_raw(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// 2^x, x <= 0: x = n + f with |f| <= 1/2 by adding and taking away 1.5 2^52, whose sum's low
// word is n; 2^f = 1 + f p(f), p the degree-10 polynomial through (2^f - 1) / f at Chebyshev
// nodes (relative error of 2^f 9e-18).  The scaling rounds a result below 2^-1022 as it has to
// and makes one below 2^-1075 zero, and so for x = -inf or NaN (inf - inf), which the clamp turns
// into -1100: a neighbour that weighs nothing adds nothing.  (log2(1 + a) is taken from a itself,
// so a floor at 2^-64 would show: equal rows of zeros came out at -1.1e-16 gamma in 1000 columns.)
__device__ __forceinline__ double soft_exp2(double x) {
  constexpr double kP[11] = {
      0x1.62e42fefa39efp-1, 0x1.ebfbdff82c598p-3, 0x1.c6b08d704a0c2p-5, 0x1.3b2ab6fba1ddap-7,
      0x1.5d87fe78a5276p-10, 0x1.430913096fd9fp-13, 0x1.ffcbfc670dcd4p-17, 0x1.62bfd47773353p-20,
      0x1.b524fae627834p-24, 0x1.e6063f7217bc6p-28, 0x1.e9d3fe3952179p-32};
  x = max_raw(x, -1100.0);
  const double t = x + 0x1.8p52;
  const double f = x - (t - 0x1.8p52);
  double p = kP[10];
#pragma unroll
  for (int k = 9; k >= 0; --k) p = __builtin_fma(p, f, kP[k]);
  p = __builtin_fma(p, f, 1.0);
  return __builtin_ldexp(p, (int)(uint32_t)__builtin_bit_cast(uint64_t, t));
}

// log2(1 + a), 0 <= a <= 2: with z = a / (a + 2) it is (2 / ln 2) atanh(z) = z (2 / ln 2 + z^2 q),
// q the degree-13 polynomial in z^2 <= 1/4 through that function at Chebyshev nodes (relative
// error 2e-18); the quotient by the reciprocal, one Newton step and one correction.
__device__ __forceinline__ double soft_log2_1p(double a) {
  constexpr double kQ[14] = {
      0x1.ec709dc3a03fdp-1, 0x1.2776c50ef9cdfp-1, 0x1.a61762a7917abp-2, 0x1.484b13e3110a2p-2,
      0x1.0c9a8241be52dp-2, 0x1.c68feaacb37cap-3, 0x1.89e7e37c4ba1ep-3, 0x1.5c3d5cb6c4b96p-3,
      0x1.30f6db6208d67p-3, 0x1.4193f51d0a96bp-3, 0x1.228edb1e6bc77p-5, 0x1.90965137a435fp-2,
      -0x1.aaf5bcd052f13p-2, 0x1.37afb55ae6feap-1};
  constexpr double kC = 0x1.71547652b82fep+1, kCLow = 0x1.777d0ffda0d24p-55;  // 2 / ln 2
  const double b = a + 2.0;
  double r = __builtin_amdgcn_rcp(b);
  r = __builtin_fma(__builtin_fma(-b, r, 1.0), r, r);
  double z = a * r;
  z = __builtin_fma(__builtin_fma(-z, a - (b - 2.0), __builtin_fma(-b, z, a)), r, z);  // with b's rounding error
  const double w = z * z;
  double q = kQ[13];
#pragma unroll
  for (int k = 12; k >= 0; --k) q = __builtin_fma(q, w, kQ[k]);
  return __builtin_fma(z, kC, z * __builtin_fma(w, q, kCLow));
}

// double: the soft minimum of the scaled neighbours is ymn - log2(sum_k 2^(ymn - y_k)) with ymn
// their minimum, whose own term is 1: two exponentials, of the median and the maximum, and the
// logarithm of 1 plus their sum.  +inf neighbours give terms that vanish; three of them (the
// padding lanes before column 0) give +inf.  A step is a serial chain of about 70 float64
// instructions of 4.9 cycles and takes 156 ns; with the general exp2 and log2 (three and one,
// about 175 instructions: subnormal, overflow and sign cases that cannot arise here) it took
// 360 ns: 500 x 700 497 us then and 234 us now.  The table's error against 80-bit arithmetic is
// the same to 5% for gamma from 0.01 to 10 and costs from 10^-9 to 10^4 gamma.
__device__ __forceinline__ void soft_cells4(ComputeState<double, 1>& st, const GroupRegs<double, 1>& r,
                                            Vec4<double> (&d)[1]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double N = Elem<double>::shr1(st.X[0], r.t.v[q]), NW = st.NW, W = st.X[0];
    const double lo = min_raw(NW, N), hi = max_raw(NW, N);
    const double mn = min_raw(lo, W), md = max_raw(lo, min_raw(hi, W)), mx = max_raw(hi, W);
    const double a = soft_exp2(mn - md) + soft_exp2(mn - mx);
    st.X[0] = r.c[0].v[q] + (mn - soft_log2_1p(a));
    st.NW = N;
    d[0].v[q] = st.X[0];
  }
}
#define WF_SOFT1(T0, NW, X, D, C)                                         \
  "v_mov_b32 " T0 ", %[top]\n\t"                                          \
  "v_mov_b32_dpp " T0 ", " X " wave_shr:1 row_mask:0xf bank_mask:0xf\n\t" \
  "v_min3_f32 %[mn], " NW ", " T0 ", " X "\n\t"                           \
  "v_med3_f32 %[md], " NW ", " T0 ", " X "\n\t"                           \
  "v_max3_f32 %[mx], " NW ", " T0 ", " X "\n\t"                           \
  "v_sub_f32 %[md], %[mn], %[md]\n\t"                                     \
  "v_sub_f32 %[mx], %[mn], %[mx]\n\t"                                     \
  "v_exp_f32 %[md], %[md]\n\t"                                            \
  "v_exp_f32 %[mx], %[mx]\n\t"                                            \
  "v_add_f32 %[md], 1.0, %[md]\n\t"                                       \
  "v_add_f32 %[md], %[md], %[mx]\n\t"                                     \
  "v_log_f32 %[md], %[md]\n\t"                                            \
  "v_mov_b32_dpp %[top], %[top] wave_shl:1 row_mask:0xf bank_mask:0xf\n\t" \
  "v_sub_f32 %[md], %[mn], %[md]\n\t"                                     \
  "v_min_f32 %[md], %[mn], %[md]\n\t"                                     \
  "v_add_f32 " D ", " C ", %[md]\n\t"
__device__ __forceinline__ void soft_cells4(ComputeState<float, 1>& st, const GroupRegs<float, 1>& r,
                                            Vec4<float> (&d)[1]) {
  const Vec4<float>& c = r.c[0];
  float t, mn, md, mx;
  asm("s_nop 0\n\t" WF_SOFT1("%[t]", "%[nw]", "%[x]", "%[d0]", "%[c0]") "s_nop 0\n\t"
          WF_SOFT1("%[nw]", "%[t]", "%[d0]", "%[d1]", "%[c1]") "s_nop 0\n\t"
              WF_SOFT1("%[t]", "%[nw]", "%[d1]", "%[d2]", "%[c2]") "s_nop 0\n\t"
                  WF_SOFT1("%[nw]", "%[t]", "%[d2]", "%[d3]", "%[c3]")
      : [top] "+v"(st.top), [nw] "+v"(st.NW), [t] "=&v"(t), [mn] "=&v"(mn), [md] "=&v"(md), [mx] "=&v"(mx),
        [d0] "=&v"(d[0].v[0]), [d1] "=&v"(d[0].v[1]), [d2] "=&v"(d[0].v[2]), [d3] "=&v"(d[0].v[3])
      : [x] "v"(st.X[0]), [c0] "v"(c.v[0]), [c1] "v"(c.v[1]), [c2] "v"(c.v[2]), [c3] "v"(c.v[3]));
  st.X[0] = d[0].v[3];
}

template <typename T, int R, bool SOFT>
__device__ __forceinline__ void cells4(ComputeState<T, R>& st, const GroupRegs<T, R>& r, Vec4<T> (&out)[R]) {
  if constexpr (SOFT) {
    static_assert(R == 1, "the soft-min sweep uses one row per lane");
    soft_cells4(st, r, out);
  } else {
    Cell4<T>::run(st, r, out);
  }
}

// What the compute wave has read ahead of the unit it works on: the unit's first two groups
// and, without kTopVec, its columns of the top row (lane l: column G u + l, l < G).
template <typename T, int G, int R>
struct UnitRegs {
  GroupRegs<T, R> g[2];
  T top;
};

template <typename T, int G, int R>
__device__ __forceinline__ void load_unit(const T* __restrict__ S, const T* __restrict__ Tr, int slot, int lane,
                                          UnitRegs<T, G, R>& r) {
#pragma unroll
  for (int p = 0; p < 2; ++p) load_group<T, G, R>(S, Tr, slot + 4 * p, lane, r.g[p]);
  if constexpr (!kTopVec<T, R>) r.top = Tr[slot + (lane & (G - 1))];
}

// The readiness of a unit's inputs: lane l's copy of counter l % 8 against what the unit
// needs of it ('need'; the loaders' sub-chunks and the top units), so that one 4-byte LDS
// read and one compare test all of them.
__device__ __forceinline__ uint32_t load_ready(const Shared& sh, int lane) {
  return __hip_atomic_load(&sh.ctr[lane & 7], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// One unit of G steps.  'P' holds the first two groups of the unit and its top row; the
// reads of each later group are issued two groups ahead, and the last two groups issue the
// reads of the next unit's first two groups and top row -- always, so that both paths below
// leave them in the same registers (conditional reads make the compiler copy every
// prefetched register at each unit boundary).  If the next unit's inputs were not yet in
// LDS two groups before the end (by the counters read at the start of the unit), the unit is
// finished and signalled first and the wave then waits for the next unit's inputs and reads
// them again.  Waiting earlier would hold back the last steps of the unit, and with them the
// band's last row, until the band above has delivered the next unit: one unit of extra lag
// per band.  After the last unit the reads wrap around the ring and are not used.  'base' is
// the unit's first slot, 'done' the number of steps finished after it.
template <typename T, int G, int R, bool SOFT>
__device__ __forceinline__ bool compute_unit(T* __restrict__ S, const T* __restrict__ Tr, Shared& sh, Control* ctl,
                                             uint32_t* steps, int base, int next_base, uint32_t done, uint32_t need,
                                             ComputeState<T, R>& st, UnitRegs<T, G, R>& P, uint32_t (&stalls)[2],
                                             uint64_t& waited, bool trace) {
  using C = FwdCfg<T, G, R>;
  constexpr int NG = C::NG;
  const int lane = threadIdx.x & 63;
  const uint32_t ready = load_ready(sh, lane);  // for the next unit, used two groups before the end
  __builtin_amdgcn_sched_barrier(0);
  GroupRegs<T, R> gr[NG];
  gr[0] = P.g[0];
  gr[1] = P.g[1];
  if constexpr (!kTopVec<T, R>) st.top = P.top;
  bool late = false;
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    if (g + 2 < NG) {
      load_group<T, G, R>(S, Tr, base + 4 * (g + 2), lane, gr[g + 2]);
    } else if (g + 2 == NG) {
      late = __ballot(ready < need) != 0;
      if (trace && late) {
        const uint64_t b = __ballot(ready < need);
        stalls[0] += (b & 0xfu) != 0;
        stalls[1] += (b & 0x10u) != 0;
      }
      __builtin_amdgcn_sched_barrier(0);
      load_group<T, G, R>(S, Tr, next_base, lane, P.g[0]);
      if constexpr (!kTopVec<T, R>) P.top = Tr[next_base + (lane & (G - 1))];
    } else {
      load_group<T, G, R>(S, Tr, next_base + 4, lane, P.g[1]);
    }
    // keeps every group's reads two groups ahead of their use (left alone, the scheduler
    // gathers the reads of several groups into one burst just before the first of them)
    __builtin_amdgcn_sched_barrier(0);
    Vec4<T> d[R];
    cells4<T, R, SOFT>(st, gr[g], d);
#pragma unroll
    for (int k = 0; k < R; ++k) *reinterpret_cast<Vec4<T>*>(S + (k * kBand + lane) * C::PITCH + base + 4 * g) = d[k];
  }
  lds_signal(steps, done);
  __builtin_amdgcn_sched_barrier(0);
  if (__builtin_expect(late, 0)) {
    if (!lds_wait_until([&] { return __ballot(load_ready(sh, lane) < need) == 0; }, &sh.abort, ctl, waited))
      return false;
    // The slot is hidden from the optimiser: through the restrict pointers it would take
    // these reads for repeats of the early ones above and drop them.
    load_unit<T, G, R>(S, Tr, opaque(next_base), lane, P);
    __builtin_amdgcn_sched_barrier(0);
  }
  return true;
}

template <typename T, int G, int R, bool SOFT>
__device__ __forceinline__ void compute_band(T* __restrict__ S, const T* __restrict__ Tr, Shared& sh, Control* ctl,
                                             int Ks, bool first_band, uint64_t* trace) {
  using E = Elem<T>;
  using C = FwdCfg<T, G, R>;
  const int lane = threadIdx.x & 63;
  const bool tr = trace != nullptr;
  // what unit 0 needs, and what each next unit and each next sub-chunk add
  const int which = lane & 7;
  const bool is_c = which < R, is_top = which == kCtrTop;
  uint32_t stalls[2] = {0, 0};
  uint64_t t_first = 0, waited = 0;
  // The workgroup's first band runs the loop once beforehand, on the ring's last sub-chunk
  // (which the loaders fill last, and wait for this) with nothing to wait for and its
  // counter stores going to a spare word: the loop's first pass on a compute unit fetches
  // its instructions from memory, about a microsecond that would otherwise be paid after
  // the inputs have arrived, by every band in turn.
  for (int pass = sh.warm != 0u; pass < 2; ++pass) {
    const bool dry = pass == 0;
    uint32_t* steps = dry ? &sh.spare : &sh.ctr[kCtrSteps];
    uint32_t need = !dry && (is_c || is_top) ? 1u : 0u;
    const uint32_t per_unit = !dry && is_top ? 1u : 0u, per_sub = !dry && is_c ? 1u : 0u;
    const int s0 = dry ? C::RING / C::SUB - 1 : 0, s1 = dry ? C::RING / C::SUB : Ks;
    ComputeState<T, R> st;
#pragma unroll
    for (int k = 0; k < R; ++k) st.X[k] = E::inf();
    // NW of the band's first cell: the virtual corner D[-1][-1] = 0 for the first band,
    // D[row0-1][-1] = +inf for the others
    st.NW = first_band && lane == 0 ? E::zero() : E::inf();
    UnitRegs<T, G, R> P;
    if (!lds_wait_until([&] { return __ballot(load_ready(sh, lane) < need) == 0; }, &sh.abort, ctl, waited)) {
      sh.abort = 1u;
      return;
    }
    if (tr) t_first = __builtin_amdgcn_s_memrealtime();
    load_unit<T, G, R>(S, Tr, (C::SUB * s0) & C::MASK, lane, P);
    // One sub-chunk per iteration, its units unrolled: one taken branch per SUB steps.  A unit
    // reads its first groups from P and leaves the next unit's there (they are dead by the
    // time those reads are issued, so both use the same registers and nothing is copied).
    // After the band's last unit there is nothing to wait for: the loaders and the poller
    // raise their counters to kAllReady when they are through.
    for (int s = s0; s < s1; ++s) {
      const int base = (C::SUB * s) & C::MASK;
      const int next = (C::SUB * (s + 1)) & C::MASK;
#pragma unroll
      for (int v = 0; v < C::GPS; ++v) {
        need += per_unit;
        if (v + 1 == C::GPS) need += per_sub;
        if (!compute_unit<T, G, R, SOFT>(S, Tr, sh, ctl, steps, base + G * v, v + 1 < C::GPS ? base + G * (v + 1) : next,
                                         (uint32_t)(C::SUB * s + G * (v + 1)), need, st, P, stalls, waited, tr)) {
          sh.abort = 1u;
          return;
        }
        if (tr && C::GPS * s + v == 62 / G + 1) trace[16] = __builtin_amdgcn_s_memrealtime();
      }
    }
    if (dry) lds_signal(&sh.warm, 1u);
  }
  if (tr && lane == 0) {
    trace[1] = t_first;
    trace[2] = __builtin_amdgcn_s_memrealtime();
    trace[4] = stalls[0];
    trace[5] = stalls[1];
    trace[8] = waited;
  }
}

// ---------------------------------------------------------------------------------------
// waves 3 .. 2+R: global -> LDS loaders.
//
// One loader per 64 LDS rows (loader h: rows 64h .. 64h+63).  Vector k of a lane covers LDS
// row l = 64h + (64/LPR) k + lane/LPR and slots [SUB s + 4j, SUB s + 4j + 4) of sub-chunk s,
// j = lane % LPR, i.e. columns c0 .. c0+3 with c0 = SUB s + 4j - skew(l).
template <typename T, int G, int R>
struct SubVec {
  using C = FwdCfg<T, G, R>;
  int l, t;  // LDS row, slot (not wrapped)
  __device__ __forceinline__ SubVec(int h, int k, int s) {
    const int lane = threadIdx.x & 63;
    l = kBand * h + (64 / C::LPR) * k + lane / C::LPR;
    t = C::SUB * s + 4 * (lane & (C::LPR - 1));
  }
  __device__ __forceinline__ int row() const { return band_row<R>(l); }
  __device__ __forceinline__ int c0() const { return t - skew(l); }
  __device__ __forceinline__ int lds() const { return l * C::PITCH + (t & C::MASK); }
};

template <typename T, int G, int R>
using SubBuf = Vec4<T>[FwdCfg<T, G, R>::NV];

template <typename T, int G, int R>
__device__ __forceinline__ void load_sub(SubBuf<T, G, R>& buf, __amdgpu_buffer_rsrc_t rsrc, int64_t ldc, int h, int s) {
  // Loads of different sub-chunks stay in issue order, so the wait before a sub-chunk's
  // LDS write leaves the later sub-chunks in flight.  Columns outside [0, n) read
  // neighbouring row data; an offset below the band's start (possible only for a single
  // column, where row*ldc + c0 can be negative) wraps to a huge unsigned value and, like
  // reads past the band's end, returns zeros from the range-checked buffer; store_sub_lds
  // masks all of them.
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < FwdCfg<T, G, R>::NV; ++k) {
    const SubVec<T, G, R> v(h, k, s);
    const uint32_t off = (uint32_t)((int64_t)v.row() * ldc + v.c0()) * (uint32_t)sizeof(T);
    if constexpr (sizeof(T) == 4) {
      buf[k] = __builtin_bit_cast(Vec4<T>, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 0, 0));
    } else {
      struct Hf { T x[2]; };
      const Hf lo = __builtin_bit_cast(Hf, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 0, 0));
      const Hf hi = __builtin_bit_cast(Hf, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(off + 16), 0, 0));
      buf[k].v[0] = lo.x[0]; buf[k].v[1] = lo.x[1]; buf[k].v[2] = hi.x[0]; buf[k].v[3] = hi.x[1];
    }
  }
  __builtin_amdgcn_sched_barrier(0);
}

// A sub-chunk with every column in [0, n) needs no masking.  (Rows below the matrix read
// zeros and their cells hold no results: no row above depends on them, and stores to them
// fall outside the range-checked buffer.)
template <typename T, int G, int R>
__device__ __forceinline__ bool interior_sub(int s, int64_t n) {
  constexpr int SUB = FwdCfg<T, G, R>::SUB;
  return SUB * s >= kBand - 1 && (int64_t)SUB * s + SUB <= n;
}

// SOFT: scaled by kx = log2(e) / gamma on the way.
template <typename T, int G, int R, bool SOFT>
__device__ __forceinline__ void store_sub_lds(T* S, const SubBuf<T, G, R>& buf, int h, int s, int64_t n, T kx) {
  using C = FwdCfg<T, G, R>;
  using E = typename C::E;
  const bool interior = interior_sub<T, G, R>(s, n);
  if constexpr (SOFT) {
    // a branch around each vector: as one around all, a float64 sweep started 4 us later
#pragma unroll
    for (int k = 0; k < C::NV; ++k) {
      const SubVec<T, G, R> q(h, k, s);
      Vec4<T> v = buf[k];
#pragma unroll
      for (int e = 0; e < 4; ++e) v.v[e] *= kx;
      if (!interior) {
        const int64_t c0 = q.c0();
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (c0 + e < 0 || c0 + e >= n) v.v[e] = E::inf();
      }
      *reinterpret_cast<Vec4<T>*>(S + q.lds()) = v;
    }
  } else if (interior) {
#pragma unroll
    for (int k = 0; k < C::NV; ++k) *reinterpret_cast<Vec4<T>*>(S + SubVec<T, G, R>(h, k, s).lds()) = buf[k];
  } else {
    // one unsigned compare per element, no branch: a band's first sub-chunk goes this way, before
    // its first step (200 x 300: 23.0 us with a branch around each vector, 22.1 so)
#pragma unroll
    for (int k = 0; k < C::NV; ++k) {
      const SubVec<T, G, R> q(h, k, s);
      const uint32_t c0 = (uint32_t)q.c0();
      Vec4<T> v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v.v[e] = c0 + (uint32_t)e < (uint32_t)n ? buf[k].v[e] : E::inf();
      *reinterpret_cast<Vec4<T>*>(S + q.lds()) = v;
    }
  }
}

template <typename T, int G, int R, bool SOFT>
__device__ __forceinline__ void loader_band(T* S, Shared& sh, const FwdArgs& a, int band, int h, int Ks, uint64_t* tr) {
  using C = FwdCfg<T, G, R>;
  const int64_t ldc = opaque(a.ldc), n = opaque(a.n);
  const T kx = SOFT ? (T)a.kx : T(1);
  const int64_t row0 = (int64_t)band * C::H;
  const int rows = (int)(a.m - row0 < C::H ? a.m - row0 : C::H);
  const __amdgpu_buffer_rsrc_t rsrc = make_rsrc(static_cast<const T*>(a.C) + row0 * ldc,
                                                (uint32_t)(((rows - 1) * ldc + n) * (int64_t)sizeof(T)));
  uint64_t waited = 0;
  SubBuf<T, G, R> buf[C::PF];
#pragma unroll
  for (int p = 0; p < C::PF; ++p) load_sub<T, G, R>(buf[p], rsrc, ldc, h, p);
  for (int s0 = 0; s0 < Ks; s0 += C::PF) {
#pragma unroll
    for (int p = 0; p < C::PF; ++p) {
      const int s = s0 + p;
      if (s < Ks) {
        // sub-chunk s reuses the slots of sub-chunk s - RING/SUB, which must be stored (by
        // the storer of these rows) and whose last rows must be read (by the publisher)
        const int older = s - C::RING / C::SUB;
        if (older == -1 && !lds_wait_ge<false>(&sh.warm, 1u, &sh.abort, a.ctl, waited)) {
          sh.abort = 1u;
          return;
        }
        if (older >= 0 &&
            (!lds_wait_ge<false>(&sh.ctr[ctr_stored(h)], (uint32_t)(older + 1), &sh.abort, a.ctl, waited) ||
             !lds_wait_ge<false>(&sh.ctr[kCtrPub], (uint32_t)(C::GPS * (older + 1)), &sh.abort, a.ctl, waited))) {
          sh.abort = 1u;
          return;
        }
        store_sub_lds<T, G, R, SOFT>(S, buf[p], h, s, n, kx);
        lds_signal(&sh.ctr[ctr_loaded(h)], s + 1 < Ks ? (uint32_t)(s + 1) : kAllReady);
        if (s + C::PF < Ks) load_sub<T, G, R>(buf[p], rsrc, ldc, h, s + C::PF);
      }
    }
  }
  if (tr && (threadIdx.x & 63) == 0) {
    tr[9] = waited;
    tr[12] = __builtin_amdgcn_s_memrealtime();
  }
}

// ---------------------------------------------------------------------------------------
// The top boundary poller.  A poll fetches the band above's boundary words for the 64 columns
// from the first one not yet handed over, and every unit of G columns it completes is handed
// over at once, so one round trip (about 0.55 us) advances it by up to 64 columns whatever G
// is.  One poll at a time: with two, four or six in flight the words were seen later, not
// sooner (0.60 us from the store to the hand-over with one, 0.95 with two; 4096 x 256: 209,
// 224, 242 and 267 us).
template <typename T, int G, int R>
__device__ __forceinline__ void top_band(T* Tr, Shared& sh, const FwdArgs& a, int band, int Ut, uint32_t epoch,
                                         uint64_t* tr) {
  using C = FwdCfg<T, G, R>;
  using E = typename C::E;
  constexpr int W = E::W;
  const int lane = threadIdx.x & 63;
  const int64_t n = opaque(a.n);
  uint64_t waited = 0, t0 = 0;
  uint32_t polls = 0;
  int u = 0;  // units handed over
  while (u < Ut) {
    const int64_t j = (int64_t)G * u + lane;
    T val = E::inf();
    int k = 64 / G;  // units to hand over
    if (band > 0) {
      // every lane loads (a lane with no column to read loads spare words of the control
      // block and ignores them)
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
      // the leading run of ready columns (columns past the matrix count as ready), in whole
      // units
      const uint64_t missing = ~__ballot(ok || j >= n);
      k = (missing == 0 ? 64 : __builtin_ctzll(missing)) / G;
    }
    // else the first band: its top row is virtual, +inf without a round trip through memory,
    // so that the band whose pace every later one follows never waits for its poller
    if (k > Ut - u) k = Ut - u;
    if (k == 0) {
      if (polls == 0 && tr) t0 = __builtin_amdgcn_s_memrealtime();
      __builtin_amdgcn_s_sleep(1);
      if ((++polls & 63u) == 0u) {
        bool give_up = lds_load(&sh.abort) != 0u || global_aborted(a.ctl);
        const uint64_t now = __builtin_amdgcn_s_memrealtime();
        if (polls == 64u) {
          if (!tr) t0 = now;
        } else if (now - t0 > kSpinTicks) {
          raise_timeout(a.ctl);
          give_up = true;
        }
        if (give_up) {
          sh.abort = 1u;
          return;
        }
      }
      continue;
    }
    if (polls != 0u) {
      if (tr) waited += __builtin_amdgcn_s_memrealtime() - t0;
      polls = 0;
    }
    // the top ring slot of column j is read before step j and reused RING steps later
    const int64_t need_steps = (int64_t)G * (u + k) - C::RING;
    if (need_steps > 0 && !lds_wait_ge(&sh.ctr[kCtrSteps], (uint32_t)need_steps, &sh.abort, a.ctl, waited)) {
      sh.abort = 1u;
      return;
    }
    if (lane < k * G) Tr[(int)(j & C::MASK)] = val;
    const bool first = u == 0;
    u += k;
    lds_signal(&sh.ctr[kCtrTop], (uint32_t)u);
    if (tr && first && lane == 0) tr[15] = __builtin_amdgcn_s_memrealtime();
  }
  if (tr && lane == 0) {
    tr[10] = waited;
    tr[13] = __builtin_amdgcn_s_memrealtime();
  }
}

// ---------------------------------------------------------------------------------------
// waves 3+R ..: storers.  SOFT: the ring holds scaled values; D = y * gl (gl = gamma ln 2).
template <typename T, int NV, bool SOFT>
__device__ __forceinline__ void unscale(Vec4<T> (&v)[NV], T gl) {
  if constexpr (SOFT) {
#pragma unroll
    for (int k = 0; k < NV; ++k)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[k].v[e] *= gl;
  }
}

// One storer per 64 LDS rows, like the loaders.
template <typename T, int G, int R, bool SOFT, bool SKIP>
__device__ __forceinline__ void store_sub(const T* S, __amdgpu_buffer_rsrc_t drs, int64_t ldd, int rows, int64_t n,
                                          int h, int s, T gl) {
  using C = FwdCfg<T, G, R>;
  typedef int v4i __attribute__((ext_vector_type(4)));
  auto put = [&](int off, const Vec4<T>& x) {
    if constexpr (sizeof(T) == 4) {
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, x), drs, off, 0, 0);
    } else {
      struct Hf { v4i lo, hi; };
      const Hf hh = __builtin_bit_cast(Hf, x);
      __builtin_amdgcn_raw_buffer_store_b128(hh.lo, drs, off, 0, 0);
      __builtin_amdgcn_raw_buffer_store_b128(hh.hi, drs, off + 16, 0, 0);
    }
  };
  // The LDS reads first.
  Vec4<T> v[C::NV];
#pragma unroll
  for (int k = 0; k < C::NV; ++k) v[k] = *reinterpret_cast<const Vec4<T>*>(S + SubVec<T, G, R>(h, k, s).lds());
  unscale<T, C::NV, SOFT>(v, gl);
  if (interior_sub<T, G, R>(s, n)) {
    // Interior sub-chunk: one 16-byte store per 16 bytes.
#pragma unroll
    for (int k = 0; k < C::NV; ++k) {
      const SubVec<T, G, R> q(h, k, s);
      put((int)(((int64_t)q.row() * ldd + q.c0()) * (int64_t)sizeof(T)), v[k]);
    }
    return;
  }
  // Edge sub-chunk (the first and the last): per vector one 16-byte store of the rows whose four
  // cells lie inside the matrix and a store per cell of the others, the lanes that have none sent
  // past the resource's end, where stores are dropped: no branch.  (With one around each store
  // 4000 instances of 64 x 64 with tables took 211 us, 199 so; 100 x 100 alone 14.9 and 12.6.)
  // SKIP: it ends after the vectors that hold the matrix's last row (1 x 64 in float64 11.3 us
  // without, 10.2 with; 65 x 400 24.6 and 23.2).  Not in the batch kernel, where that test
  // costs more than it saves: 4000 instances of 4 to 40 rows 163 us without, 209 with, for a
  // reason not found.
  constexpr uint32_t kOut = 0x80000000u;  // a band's resource is shorter
#pragma unroll
  for (int k = 0; k < C::NV; ++k) {
    if (SKIP && k % 4 == 0 && R * (64 / C::LPR) * k + h >= rows) break;
    const SubVec<T, G, R> q(h, k, s);
    const int c0 = q.c0();
    const uint32_t off = (uint32_t)((int64_t)q.row() * ldd + c0) * (uint32_t)sizeof(T);
    const bool whole = c0 >= 0 && c0 + 4 <= (int)n;
    put((int)(whole ? off : kOut), v[k]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t o = !whole && (uint32_t)(c0 + e) < (uint32_t)n ? off + e * (uint32_t)sizeof(T) : kOut;
      if constexpr (sizeof(T) == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v[k].v[e]), drs, (int)o, 0, 0);
      } else {
        typedef int v2i __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2i, v[k].v[e]), drs, (int)o, 0, 0);
      }
    }
  }
}

template <typename T, int G, int R, bool SOFT, bool SKIP>
__device__ __forceinline__ void store_band(const T* S, Shared& sh, const FwdArgs& a, int band, int h, int Ks,
                                           uint64_t* tr) {
  using C = FwdCfg<T, G, R>;
  const int lane = threadIdx.x & 63;
  const int64_t m = opaque(a.m), n = opaque(a.n), ldd = opaque(a.ldd);
  const int64_t row0 = (int64_t)band * C::H;
  const int rows = (int)(m - row0 < C::H ? m - row0 : C::H);
  T* ck_cols = a.ckpt ? static_cast<T*>(a.ckpt) + ((m + kBand - 1) / kBand - 1) * n : nullptr;
  const int K = a.ckpt_k;
  // LDS row of the score, if it is one of this storer's rows
  const int64_t sc = m - 1 - row0;
  const int sc_l = sc >= 0 && sc < C::H && lds_row<R>((int)sc) / kBand == h ? lds_row<R>((int)sc) : -1;
  const T gl = SOFT ? (T)a.gl : T(1);
  const __amdgpu_buffer_rsrc_t drs =
      make_rsrc(a.D ? static_cast<T*>(a.D) + row0 * ldd : nullptr,
                a.D ? (uint32_t)(((rows - 1) * ldd + n) * (int64_t)sizeof(T)) : 0u);
  uint64_t waited = 0;
  for (int s = 0; s < Ks; ++s) {
    // sub-chunk s (slots [SUB s, SUB (s+1)) of every row) is final after its last step; its D
    // goes out after the publisher has issued the boundary words of those steps, which
    // the band below waits for
    if (!lds_wait_ge(&sh.ctr[kCtrPub], (uint32_t)(C::GPS * (s + 1)), &sh.abort, a.ctl, waited)) {
      sh.abort = 1u;
      return;
    }
    if (a.D) store_sub<T, G, R, SOFT, SKIP>(S, drs, ldd, rows, n, h, s, gl);
    if (ck_cols) {
      const int l = kBand * h + lane, i = band_row<R>(l);
      if (i < rows) {
        // checkpoint columns D[.][Kq-1] of row i held by sub-chunk s, from the first one on: one
        // division per sub-chunk (with one per column 64 x 16384 with K = 5 took 754 us in int32)
        const int lo = C::SUB * s - skew(l), end = lo + C::SUB < (int)n ? lo + C::SUB : (int)n - 1;
        const uint32_t q = (uint32_t)((lo > 0 ? lo : 0) + K) / (uint32_t)K;
        T* out = ck_cols + (int64_t)(q - 1) * m + row0 + i;
        for (int j = (int)q * K - 1; j < end; j += K, out += m)
          *out = S[l * C::PITCH + ((j + skew(l)) & C::MASK)];
      }
    }
    if (sc_l >= 0 && lane == sc_l % kBand) {
      const int64_t slot = n - 1 + skew(sc_l);
      if (slot / C::SUB == s) {
        const T y = S[sc_l * C::PITCH + ((int)slot & C::MASK)];
        *static_cast<T*>(a.score) = SOFT ? y * gl : y;
      }
    }
    lds_publish(&sh.ctr[ctr_stored(h)], (uint32_t)(s + 1));
  }
  if (tr && lane == 0) tr[11] = waited;
}

// ---------------------------------------------------------------------------------------
// wave 1: publisher of the band's last row (and of the checkpoint rows)
template <typename T, int G, int R>
__device__ __forceinline__ void publish_band(const T* S, Shared& sh, const FwdArgs& a, int band, int Us,
                                             uint32_t epoch, uint64_t* tr) {
  using C = FwdCfg<T, G, R>;
  using E = typename C::E;
  constexpr int W = E::W;
  const int lane = threadIdx.x & 63;
  const int64_t m = opaque(a.m), n = opaque(a.n);
  const int nb64 = (int)((m + kBand - 1) / kBand);  // 64-row bands of the checkpoint grid
  const bool last_band = band == a.nb - 1;
  T* ck_rows = static_cast<T*>(a.ckpt);
  // an injected fault (tests of the failure path) makes band 0 withhold its boundary row
  const bool withhold =
      band == 0 && __hip_atomic_load(&a.ctl->fault, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == kFaultFwdWithhold;
  uint64_t waited = 0;
  for (int u = 0; u < Us;) {
    uint32_t done;
    if (!lds_wait_value<true, false>(&sh.ctr[kCtrSteps], (uint32_t)(G * (u + 1)), &sh.abort, a.ctl, waited, done)) {
      sh.abort = 1u;
      return;
    }
    // every unit finished by now goes out in this pass, up to 64 columns
    int k = (int)(done / G) - u;
    if (k > 64 / G) k = 64 / G;
    if (k > Us - u) k = Us - u;
    const int cols = k * G;
    const bool mark = tr && u <= 62 / G + 1 && 62 / G + 1 < u + k && lane == 0;
    if (mark) tr[17] = __builtin_amdgcn_s_memrealtime();
    if (lane < cols) {
      const int slot = (G * u + lane) & C::MASK;
      // the band's last row, row H-1 (the last LDS row, lane 63's), finished this column at
      // this step
      const int64_t j = (int64_t)G * u + lane - skew(C::H - 1);
      if (!last_band && !withhold && j >= 0 && j < n) {
        const T x = S[(C::H - 1) * C::PITCH + slot];
#pragma unroll
        for (int q = 0; q < W; ++q) store_word(a.bnd + ((int64_t)band * n + j) * W + q, tagged(E::word(x, q), epoch));
      }
      // checkpoint rows: rows 63, 127, ... of the matrix except its last one
      if (ck_rows) {
#pragma unroll
        for (int h = 0; h < R; ++h) {
          const int l = lds_row<R>(kBand * h + kBand - 1);
          const int b64 = band * R + h;
          const int64_t jc = (int64_t)G * u + lane - skew(l);
          if (b64 < nb64 - 1 && jc >= 0 && jc < n) ck_rows[(int64_t)b64 * n + jc] = S[l * C::PITCH + slot];
        }
      }
    }
    if (mark) tr[14] = __builtin_amdgcn_s_memrealtime();
    u += k;
    lds_publish(&sh.ctr[kCtrPub], (uint32_t)u);
  }
  if (tr && lane == 0) tr[18] = waited;
}

// ---------------------------------------------------------------------------------------
// One band of one instance, all five roles.  The LDS counters must be zero on entry.
template <typename T, int G, int R, bool SOFT, bool BATCH>
__device__ __forceinline__ void run_band(T* S, T* Tr, Shared& sh, const FwdArgs& a, int band, uint32_t epoch,
                                         uint64_t* tr) {
  using C = FwdCfg<T, G, R>;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  // steps of a band: n + 63, rounded up to whole sub-chunks
  const int Ks = (int)((a.n + kBand - 1 + C::SUB - 1) / C::SUB);  // C sub-chunks
  const int Us = Ks * C::GPS;                                  // compute / publish units
  const int Ut = (int)((a.n + G - 1) / G);                     // top units holding real columns
  if (wave == 0) {
    compute_band<T, G, R, SOFT>(S, Tr, sh, a.ctl, Ks, band == 0, tr);
  } else if (wave == 1) {
    publish_band<T, G, R>(S, sh, a, band, Us, epoch, tr);
  } else if (wave == 2) {
    top_band<T, G, R>(Tr, sh, a, band, Ut, epoch, tr);
    // Top units beyond the last real column hold no values any real cell reads; mark
    // them loaded so that the compute wave's readiness test stays one comparison.
    if ((threadIdx.x & 63) == 0 && sh.abort == 0u) lds_signal(&sh.ctr[kCtrTop], kAllReady);
  } else if (wave < 3 + R) {
    loader_band<T, G, R, SOFT>(S, sh, a, band, wave - 3, Ks, tr);
  } else {
    store_band<T, G, R, SOFT, !BATCH>(S, sh, a, band, wave - 3 - R, Ks, tr);
  }
}

// TRACE = false compiles every trace statement out (the production instance); the traced
// instance is launched only while tracing is enabled.
template <typename T, int G, int R, bool TRACE, bool SOFT = false>
__global__ __launch_bounds__((64 * (3 + 2 * R)), 1) void fwd_kernel(FwdArgs a) {
  using C = FwdCfg<T, G, R>;
  if constexpr (!TRACE) a.trace = nullptr;
  __shared__ Vec4<T> S4[C::H * C::PITCH / 4];
  __shared__ Vec4<T> Tr4[C::RING / 4];
  __shared__ Shared sh;
  T* S = reinterpret_cast<T*>(S4);
  T* Tr = reinterpret_cast<T*>(Tr4);
  Control* ctl = a.ctl;
  const uint32_t epoch = __hip_atomic_load(&ctl->epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (threadIdx.x == 0) {
    sh.abort = 0u;
    // (a pass over the double soft-min loop costs more than its fetch: 500 x 700 234 us without,
    // 243 with)
    sh.warm = SOFT && sizeof(T) == 8 ? 1u : 0u;
  }
  for (;;) {
    if (threadIdx.x < 16) sh.ctr[threadIdx.x] = 0u;
    claim_next(ctl, &sh.item, &sh.abort);
    const int band = (int)sh.item;
    if (band >= a.nb || sh.abort != 0u) break;
    uint64_t* tr = a.trace ? a.trace + (int64_t)band * kTraceWords : nullptr;
    if (tr && threadIdx.x == 0) {
      unsigned xcc;
      asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
      tr[0] = __builtin_amdgcn_s_memrealtime();
      tr[6] = xcc;
      tr[7] = blockIdx.x;
    }
    run_band<T, G, R, SOFT, false>(S, Tr, sh, a, band, epoch, tr);
    if (tr && threadIdx.x == (3 + R) * 64) tr[3] = __builtin_amdgcn_s_memrealtime();
    __syncthreads();
  }
  finish_launch(ctl, epoch);
}

// Ragged batch: work items (instance, band) are claimed in list order; the host orders the
// list so that every band comes after the band above it of the same instance (and
// instances by decreasing critical path), so a claimed band only ever waits for bands
// that were claimed before it and are running or done.
template <typename T, int G, int R>
__global__ __launch_bounds__((64 * (3 + 2 * R)), 1) void fwd_batch_kernel(BatchArgs b) {
  using C = FwdCfg<T, G, R>;
  __shared__ Vec4<T> S4[C::H * C::PITCH / 4];
  __shared__ Vec4<T> Tr4[C::RING / 4];
  __shared__ Shared sh;
  T* S = reinterpret_cast<T*>(S4);
  T* Tr = reinterpret_cast<T*>(Tr4);
  Control* ctl = b.ctl;
  const uint32_t epoch = __hip_atomic_load(&ctl->epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (threadIdx.x == 0) {
    sh.abort = 0u;
    sh.warm = 0u;
  }
  for (;;) {
    if (threadIdx.x < 16) sh.ctr[threadIdx.x] = 0u;
    claim_next(ctl, &sh.item, &sh.abort);
    const uint32_t item = sh.item;
    if (item >= (uint32_t)b.n_items || sh.abort != 0u) break;
    const BatchItem it = b.items[item];
    const BatchInst in = b.inst[it.inst];
    FwdArgs a;
    a.C = static_cast<const T*>(b.C) + in.off;
    a.D = b.D ? static_cast<T*>(b.D) + in.off : nullptr;
    a.score = static_cast<T*>(b.scores) + it.inst;
    a.ckpt = b.ckpt ? static_cast<T*>(b.ckpt) + in.ck_off : nullptr;
    a.ldc = in.n;
    a.ldd = in.n;
    a.m = in.m;
    a.n = in.n;
    a.ckpt_k = b.ckpt ? b.ckpt_k : 0;
    a.nb = in.nb;
    a.rows = R;
    a.pad = 0;
    a.ctl = ctl;
    a.bnd = b.bnd + in.bnd_off;
    a.trace = nullptr;
    a.kx = a.gl = 1.0;
    run_band<T, G, R, false, true>(S, Tr, sh, a, it.band, epoch, nullptr);
    __syncthreads();
  }
  finish_launch(ctl, epoch);
}

template <typename T, int R, bool TRACE>
hipError_t launch_tt(int tile, const FwdArgs& a, int grid, hipStream_t s) {
  switch (tile) {
    case 16: hipLaunchKernelGGL((fwd_kernel<T, 16, R, TRACE>), dim3(grid), dim3(64 * (3 + 2 * R)), 0, s, a); break;
    case 32: hipLaunchKernelGGL((fwd_kernel<T, 32, R, TRACE>), dim3(grid), dim3(64 * (3 + 2 * R)), 0, s, a); break;
    case 64:  // 32 where the ring holds sub-chunks of 32
      hipLaunchKernelGGL((fwd_kernel<T, FwdCfg<T, 16, R>::SUB, R, TRACE>), dim3(grid), dim3(64 * (3 + 2 * R)), 0, s, a);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename T, int R>
hipError_t launch_t(int tile, const FwdArgs& a, int grid, hipStream_t s) {
  return a.trace ? launch_tt<T, R, true>(tile, a, grid, s) : launch_tt<T, R, false>(tile, a, grid, s);
}

template <typename T, int R>
hipError_t launch_batch_t(int tile, const BatchArgs& b, int grid, hipStream_t s) {
  const dim3 g(grid), t(64 * (3 + 2 * R));
  switch (tile) {
    case 16: hipLaunchKernelGGL((fwd_batch_kernel<T, 16, R>), g, t, 0, s, b); break;
    case 32: hipLaunchKernelGGL((fwd_batch_kernel<T, 32, R>), g, t, 0, s, b); break;
    case 64: hipLaunchKernelGGL((fwd_batch_kernel<T, 64, R>), g, t, 0, s, b); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_forward(int dtype, int tile, const FwdArgs& a, int grid, hipStream_t s) {
  switch (dtype * 8 + a.rows) {
    case 1: return launch_t<float, 1>(tile, a, grid, s);
    case 2: return launch_t<float, 2>(tile, a, grid, s);
    case 4: return launch_t<float, 4>(tile, a, grid, s);
    case 8 + 1: return launch_t<double, 1>(tile, a, grid, s);
    case 8 + 2: return launch_t<double, 2>(tile, a, grid, s);
    case 16 + 1: return launch_t<int32_t, 1>(tile, a, grid, s);
    case 16 + 2: return launch_t<int32_t, 2>(tile, a, grid, s);
    case 16 + 4: return launch_t<int32_t, 4>(tile, a, grid, s);
    default: return hipErrorInvalidValue;
  }
}

// The soft-min sweep's steps cost several times a min-plus step (exponentials and a
// logarithm per cell), so the finest handoff unit, 16 columns, serves it best.
hipError_t launch_forward_soft(int dtype, const FwdArgs& a, int grid, hipStream_t s) {
  switch (dtype) {
    case 0: hipLaunchKernelGGL((fwd_kernel<float, 16, 1, false, true>), dim3(grid), dim3(5 * 64), 0, s, a); break;
    case 1: hipLaunchKernelGGL((fwd_kernel<double, 16, 1, false, true>), dim3(grid), dim3(5 * 64), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_forward_batch(int dtype, int tile, int rows, const BatchArgs& b, int grid, hipStream_t s) {
  if (rows == 2 && dtype != 1) {
    return dtype == 0 ? launch_batch_t<float, 2>(tile, b, grid, s) : launch_batch_t<int32_t, 2>(tile, b, grid, s);
  }
  if (rows != 1) return hipErrorInvalidValue;
  switch (dtype) {
    case 0: return launch_batch_t<float, 1>(tile, b, grid, s);
    case 1: return launch_batch_t<double, 1>(tile, b, grid, s);
    case 2: return launch_batch_t<int32_t, 1>(tile, b, grid, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace wf
