// Device code of the 1D3V PIC hot path with radiation reaction (gfx950).
//
// Kernels (one HIP launch each):
//   k_push      gather -> Boris -> RR (electrons) -> move -> integer deposit,
//               one thread per particle over cell-sorted SoA tiles; current
//               accumulated in lane-private LDS copies of a window of nodes,
//               then one global 64-bit atomic per node and work-group.
//   k_step      for small runs: the fields of a step and the push of the next
//               in one launch (its push tiles advance their own cells' fields).
//   k_field     1D Yee advance (two B half steps around the E step), laser
//               injection and absorption at the ends, Ex as the integral of
//               the charge flux; one thread per node, halo recomputed.
//   k_sort_*    counting sort of particles by cell (histogram, scan, scatter).
//   k_diag_*    FP64 energy budget and exact integer Gauss check.
//   k_init, k_spectrum: quiet start and ion energy histogram.
//
// Templated on the storage type R (float: precision form, double: plain
// form).  Everything that decides an integer (cell index, fixed-point
// current) is computed with one IEEE rounding per operation and no fused
// multiply-add, in the order fixed by the deposition contract.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <limits.h>

namespace pic {

#ifndef PIC_PUSH_PPT
#define PIC_PUSH_PPT 20
#endif
#ifndef PIC_BATCH_PPT
#define PIC_BATCH_PPT 4
#endif
#ifndef PIC_PUSH_LDS_SLOTS
#define PIC_PUSH_LDS_SLOTS 3072
#endif
#ifndef PIC_PUSH_DEPTH
#define PIC_PUSH_DEPTH 4
#endif
#ifndef PIC_RING_UNROLL
#define PIC_RING_UNROLL 2
#endif

#ifndef PIC_PUSH_MIN_WAVES
#define PIC_PUSH_MIN_WAVES 0
#endif

constexpr int kDead = INT_MIN;        // cell index of a removed particle
constexpr int kThreads = 256;         // push work-group
constexpr int kPPT = PIC_PUSH_PPT;    // particles per thread per tile (single runs)
constexpr int kTile = kThreads * kPPT;
// Batched runs are small and many: a shorter tile lowers the latency of a
// step of one run (the window set-up and flush are paid over fewer pushes).
constexpr int kBatchPPT = PIC_BATCH_PPT;
constexpr int kBatchTile = kThreads * kBatchPPT;
#ifndef PIC_BATCH_DEPTH
#define PIC_BATCH_DEPTH 2
#endif
// The batched push keeps two particles' loads in flight per thread rather
// than the whole tile's: fewer registers, six waves per SIMD instead of five.
constexpr int kBatchDepth = PIC_BATCH_DEPTH;
// Smallest tile of a run of `cap` particles per species (its per-tile arrays
// are sized for it): one particle per thread for up to 2^16, two for up to
// 2^17, else the batched push's; see small_tile().
constexpr int min_tile(long long cap) {
  return cap <= 1 << 16 ? kThreads : cap <= 1 << 17 ? 2 * kThreads : kTile < kBatchTile ? kTile : kBatchTile;
}
constexpr int kLdsSlots = PIC_PUSH_LDS_SLOTS;  // 64-bit LDS current accumulators per work-group
constexpr int kDepth = PIC_PUSH_DEPTH;        // particles per thread whose loads are in flight
constexpr int kRingUnroll = PIC_RING_UNROLL;  // ring turns per loop iteration (renames, no copies)
constexpr int kLanes = 64;            // wavefront width
#ifndef PIC_STEPS_MIN_WAVES
#define PIC_STEPS_MIN_WAVES 4  // waves per SIMD the persistent batched-step kernel is compiled for
#endif
#ifndef PIC_STEPS_BLOCKS_PER_CU
#define PIC_STEPS_BLOCKS_PER_CU 0  // work-groups per CU of the persistent launch (0: as many as fit)
#endif
#ifndef PIC_FIELD_CHUNK
#define PIC_FIELD_CHUNK 64
#endif
constexpr int kFieldChunk = PIC_FIELD_CHUNK;  // nodes per field work-group
constexpr int kTwo24 = 1 << 24;

template <typename R>
struct SpeciesDev {
  int* cell;
  R* off;
  R* ux;
  R* uy;
  R* uz;
  R* w;
  float* rx;  // compensated RR residuals (fp32 electrons), else null
  float* ry;
  float* rz;
  R* oy;      // y offsets on a 2D grid, else null
};

// Grid fields, interleaved so that one particle gathers with four loads:
//   N[i] = (E_y, E_z) at node i = 0..n,
//   H[h] = (E_x, B_y, B_z, 0) at half-node h = 0..n+1 (x = (h - 1/2) dx).
template <typename R>
struct alignas(2 * sizeof(R)) NodeF {
  R ey, ez;
};
template <typename R>
struct alignas(16) HalfF {
  R ex, by, bz, pad;
};

template <typename R>
struct FieldsDev {
  NodeF<R>* N;
  HalfF<R>* H;
};

template <typename R>
struct PushArgs {
  SpeciesDev<R> sp[2];
  const long long* count;        // [2] particles per species as of the last sort
  int tiles0;                    // work-groups of species 0
  FieldsDev<R> f;                // E^n, B^n
  unsigned long long* J;         // currents [3 buffers][Jx (half-nodes), Jy, Jz (nodes, index node+1)][jstride]
  unsigned jstride;
  int jfix;                      // the buffer of this step's current, or -1: step mod 3
  const long long* step;         // device step counter (read when jfix < 0)
  int cap;                       // entries of the particle arrays
  double* acc;                   // [tile][4] cumulative: E_rad, E_esc_e, E_esc_i, n_stiff
  int* flags;                    // [0]: non-finite seen
  int nx;
  R cfl;                         // dt / dx
  R dt;
  R eps;                         // RR strength (4 pi / 3) r_e / lambda
  R qh[2];                       // q/m dt / 2 per species
  int Z[2];                      // charge per species
  double mass[2];
  int rr0;                       // RR on species 0 (electrons)
  int comp;                      // compensated RR accumulation (fp32 only)
  R sw;                          // 256 / w_ref (charge-weight scale)
  int qw_ref[2];                 // charge weight of a particle of weight w_ref
  int ntiles;                    // tiles of both species
  int tile0;                     // first tile of this launch (a step may be split over launches)
  // Cell range of every tile after the previous push (the particles' cells
  // now, as long as no sort or state change came between): with *pred_in
  // set, a tile sizes its current window from it instead of a pass over its
  // cells.  For a push by itself only a hint: a particle outside the window
  // deposits by global atomics.  A fused step (k_step) gathers from the fields
  // staged for this range, so there every particle must lie in it: the push
  // before, of the same call and with at most a sort (which clears *pred_in)
  // in between, has written it.  The push writes the next ranges and sets
  // *pred_out.
  const int* rng_in;             // [tile][2] min, max
  int* rng_out;
  const int* pred_in;
  int* pred_out;
};

// ---------------------------------------------------------------- helpers
// A launch's arguments (or a table no kernel writes) as constant memory, read
// where they are needed.  Taken by value, the push kernels' arguments can be
// split into scalars loaded at the kernel's entry, of which there are more
// than scalar registers: 40 to 180 of them were then spilled into lanes of
// vector registers.
template <typename T>
__device__ __forceinline__ const T& constant_ref(const T* p) {
  return *(const T*)(const __attribute__((address_space(4))) T*)p;
}
template <typename T>
__device__ __forceinline__ const T& kernel_args() {
  return *(const T*)(const __attribute__((address_space(4))) T*)__builtin_amdgcn_kernarg_segment_ptr();
}

// Approximate (about 1 ulp) reciprocal, reciprocal square root and square
// root for the Boris and RR arithmetic; the contract lines use IEEE ops.
// In FP64 they are correctly rounded (rsq: the reciprocal of the root), by
// the routines below; every argument is at least 1 there too.
__device__ __forceinline__ double sqrt_rn_ge1(double x);
__device__ __forceinline__ double rcp_rn_ge1(double x);
__device__ __forceinline__ float rsq(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double rsq(double x) { return rcp_rn_ge1(sqrt_rn_ge1(x)); }
__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rcp(double x) { return rcp_rn_ge1(x); }
__device__ __forceinline__ float fsqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ double fsqrt(double x) { return sqrt_rn_ge1(x); }

// The same where a square may overflow without the particle being dropped (a
// tracked electron has the momentum its caller gave it): infinity gives 0.
__device__ __forceinline__ float rsq_any(float x) { return rsq(x); }
__device__ __forceinline__ double rsq_any(double x) { return x == INFINITY ? 0.0 : rsq(x); }
__device__ __forceinline__ float rcp_any(float x) { return rcp(x); }
__device__ __forceinline__ double rcp_any(double x) { return x == INFINITY ? 0.0 : rcp(x); }

// Element i of an array at a wave-uniform base: a 32-bit byte offset added
// to the 64-bit base lets the compiler use scalar-base addressing instead of
// per-lane 64-bit address arithmetic.  Arrays stay below 4 GiB (capacity
// limits in the host code).
template <typename T>
__device__ __forceinline__ T ld(const T* p, unsigned i) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(p) +
                                     (size_t)(i * (unsigned)sizeof(T)));
}
// The empty asm re-creates the 32-bit offset in the store's own basic block:
// instruction selection works per block and matches the scalar-base form
// only when it sees the zero extension of the offset, which after the
// push's branches it otherwise does not (a 64-bit add per store).
template <typename T>
__device__ __forceinline__ void st(T* p, unsigned i, T v) {
  unsigned o = i * (unsigned)sizeof(T);
  asm volatile("" : "+v"(o));
  *reinterpret_cast<T*>(reinterpret_cast<char*>(p) + (size_t)o) = v;
}

__device__ __forceinline__ long long wave_sum(long long v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}
__device__ __forceinline__ int wave_min(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ int wave_max(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o));
  return v;
}

// Row-local reductions with DPP lane shifts (rows of 16 lanes).  After the
// steps 1, 2, .., N/2 of an inclusive shift-and-combine scan, the last lane of
// every aligned group of N lanes holds the group's result.  All lanes of the
// wave must be active.  Lanes shifted in from outside the row read `old`.
template <int N>
__device__ __forceinline__ int row_shr(int old, int v) {
  return __builtin_amdgcn_update_dpp(old, v, 0x110 + N, 0xf, 0xf, false);
}
template <int N>
__device__ __forceinline__ unsigned long long row_shr64(unsigned long long v) {
  const unsigned lo = (unsigned)row_shr<N>(0, (int)(unsigned)v);
  const unsigned hi = (unsigned)row_shr<N>(0, (int)(unsigned)(v >> 32));
  return ((unsigned long long)hi << 32) | lo;
}
// sum over aligned groups of g lanes, g in {1, 2, 4, 8, 16} (wave-uniform)
__device__ __forceinline__ long long group_sum(long long v, int g) {
  if (g >= 2) v += (long long)row_shr64<1>((unsigned long long)v);
  if (g >= 4) v += (long long)row_shr64<2>((unsigned long long)v);
  if (g >= 8) v += (long long)row_shr64<4>((unsigned long long)v);
  if (g >= 16) v += (long long)row_shr64<8>((unsigned long long)v);
  return v;
}
// wave sum in a fixed order: rows by DPP, then the four row sums
__device__ __forceinline__ double wave_sum_dpp(double x) {
  unsigned long long b = __double_as_longlong(x);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    unsigned long long t = 0;
    switch (k) {
      case 0: t = row_shr64<1>(b); break;
      case 1: t = row_shr64<2>(b); break;
      case 2: t = row_shr64<4>(b); break;
      default: t = row_shr64<8>(b); break;
    }
    b = __double_as_longlong(__longlong_as_double(b) + __longlong_as_double(t));
  }
  const unsigned lo = (unsigned)b, hi = (unsigned)(b >> 32);
  double r[4];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    r[k] = __longlong_as_double(((long long)__builtin_amdgcn_readlane((int)hi, 16 * k + 15) << 32) |
                                (unsigned)__builtin_amdgcn_readlane((int)lo, 16 * k + 15));
  return (r[0] + r[1]) + (r[2] + r[3]);
}
// wave minimum and maximum, wave-uniform results
__device__ __forceinline__ int wave_min_dpp(int v) {
  v = min(v, row_shr<1>(v, v));
  v = min(v, row_shr<2>(v, v));
  v = min(v, row_shr<4>(v, v));
  v = min(v, row_shr<8>(v, v));
  return min(min(__builtin_amdgcn_readlane(v, 15), __builtin_amdgcn_readlane(v, 31)),
             min(__builtin_amdgcn_readlane(v, 47), __builtin_amdgcn_readlane(v, 63)));
}
__device__ __forceinline__ int wave_max_dpp(int v) {
  v = max(v, row_shr<1>(v, v));
  v = max(v, row_shr<2>(v, v));
  v = max(v, row_shr<4>(v, v));
  v = max(v, row_shr<8>(v, v));
  return max(max(__builtin_amdgcn_readlane(v, 15), __builtin_amdgcn_readlane(v, 31)),
             max(__builtin_amdgcn_readlane(v, 47), __builtin_amdgcn_readlane(v, 63)));
}

// Correctly rounded square root and reciprocal for arguments >= 1, from the
// hardware estimates (within one ulp) and exact FMA residuals: the root
// picks among s - ulp, s, s + ulp by the signs of x - s' s; the reciprocal
// takes one Newton step r + r (1 - x r).  Compared exhaustively with the
// compiler's correctly rounded sqrtf and 1.0f / x (pic_check_rounding), they
// agree on every float in [1, 2^128) and [1, 2^126) respectively; infinity
// and NaN propagate.
__device__ __forceinline__ float sqrt_rn_ge1(float x) {
  const float s = __builtin_amdgcn_sqrtf(x);
  const float sd = __int_as_float(__float_as_int(s) - 1), su = __int_as_float(__float_as_int(s) + 1);
  const float rd = fmaf(-sd, s, x), ru = fmaf(-su, s, x);
  const float r = rd <= 0.f ? sd : s;
  return ru > 0.f ? su : r;
}
__device__ __forceinline__ float rcp_rn_ge1(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return fmaf(fmaf(-x, r, 1.0f), r, r);
}
// In FP64: the coupled Newton (Goldschmidt) iteration for sqrt(x) and
// 1 / (2 sqrt(x)) from the hardware estimate, then two residual corrections;
// two Newton steps and one residual correction of the reciprocal.  The
// general sqrt and division also scale their operands for the ends of the
// exponent range and sort out special values: 7 and 4 more instructions of 17
// and 11, some 40 of the 370 an average FP64 push issues.  Finite arguments
// in [1, 2^1000] need none of it; infinities and NaN give NaN, which the
// pushes drop as they drop infinity (a momentum past 1e30); see rsq_any() for
// tracked electrons.
__device__ __forceinline__ double sqrt_rn_ge1(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double s = x * y, h = 0.5 * y;
  const double r = fma(-h, s, 0.5);
  h = fma(h, r, h);
  s = fma(s, r, s);
  s = fma(fma(-s, s, x), h, s);
  return fma(fma(-s, s, x), h, s);
}
__device__ __forceinline__ double rcp_rn_ge1(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(fma(-x, r, 1.0), r, r);
}

// Position update of the deposition contract: gamma from the stored
// momentum in the order ((1 + ux^2) + uy^2) + uz^2, correctly rounded square
// root and division, displacement vx*cfl, offset renormalised to [0, 1).
template <typename R>
__device__ __forceinline__ void contract_move(R ux, R uy, R uz, R o, R cfl, R& g,
                                              R& vy, R& vz, R& o1, R& s) {
#pragma clang fp contract(off)
  g = sqrt_rn_ge1(((R(1) + ux * ux) + uy * uy) + uz * uz);
  const R ig = rcp_rn_ge1(g);
  const R vx = ux * ig;
  vy = uy * ig;
  vz = uz * ig;
  const R d = vx * cfl;
  s = o + d;
  R fl = floor(s);
  o1 = s - fl;
  if (o1 >= R(1)) {
    o1 = R(0);
    fl += R(1);
  }
  s = fl;  // integer cell shift
}

// Knuth's TwoSum: a + b = s + e exactly.
__device__ __forceinline__ void two_sum(float a, float b, float& s, float& e) {
#pragma clang fp contract(off)
  s = a + b;
  const float bb = s - a;
  e = (a - (s - bb)) + (b - bb);
}

// Current accumulation of one push work-group: an LDS window of W storage
// indices (starting at wlo) covering every node the tile's particles can
// touch, with R = 2^k private copies per slot (lane & (R - 1) picks the
// copy), so lanes of a wave that hit the same node add to different words.
// Tiles whose window does not fit use global atomics instead.
struct DepositCtx {
  // current / qw_ref of particles with qw == qw_ref: slot (comp, cell) of
  // copy k at lds[(comp * W + cell) * P + k], P = R + 1 (R > 1) or 1; the
  // odd stride spreads one copy of neighbouring slots over distinct banks
  unsigned long long* lds;
  unsigned long long* J[3];
  int wlo;
  int W;
  int P;
  int copy;
  int qw_ref;
  bool use_lds;
};

// Integer current of one move (cell c, offset o) -> (c1, o1); see the
// deposition contract in the library header notes.
template <typename R>
__device__ __forceinline__ void deposit(DepositCtx& d, int c, R o, int c1, R o1,
                                        R vy, R vz, int qw) {
  const int q0 = (int)(o * R(kTwo24));
  const int q1 = (int)(o1 * R(kTwo24));
  const int base = min(c, c1);
  const int d0 = c - base, d1 = c1 - base;
  const int wo0 = d0 ? 0 : kTwo24 - q0;
  const int wo1 = d0 ? kTwo24 - q0 : q0;
  const int wo2 = d0 ? q0 : 0;
  const int wn0 = d1 ? 0 : kTwo24 - q1;
  const int wn1 = d1 ? kTwo24 - q1 : q1;
  const int wn2 = d1 ? q1 : 0;
  const int F0 = wo0 - wn0;
  const int F1 = F0 + wo1 - wn1;
  const int vy24 = (int)rint(vy * R(kTwo24));  // |v| < 1: |vy24| <= 2^24
  const int vz24 = (int)rint(vz * R(kTwo24));
  // unweighted Jy, Jz terms: floor(v24 (Wo + Wn) / 2^25), |term| <= 2^24
  const int ty0 = (int)(((long long)vy24 * (wo0 + wn0)) >> 25);
  const int ty1 = (int)(((long long)vy24 * (wo1 + wn1)) >> 25);
  const int ty2 = (int)(((long long)vy24 * (wo2 + wn2)) >> 25);
  const int tz0 = (int)(((long long)vz24 * (wo0 + wn0)) >> 25);
  const int tz1 = (int)(((long long)vz24 * (wo1 + wn1)) >> 25);
  const int tz2 = (int)(((long long)vz24 * (wo2 + wn2)) >> 25);
  const bool moved = (c1 != c);
  const int j0 = base + 1;  // Jx half-node base+1/2 and Jy node base share index base+1
  const int r = j0 - d.wlo;  // 0 <= r <= W - 3 when the particle's cell is in the window
  if (d.use_lds && qw == d.qw_ref && (unsigned)r <= (unsigned)(d.W - 3)) {
    // LDS holds sums of unweighted terms; the flush multiplies by qw_ref
    // slot (comp, r + k) of this lane's copy: x0 + comp * cs + k * ss
    const int ss = d.P, cs = d.W * d.P;
    unsigned long long* x0 = d.lds + d.copy + r * d.P;
    unsigned long long* y0 = x0 + cs;
    unsigned long long* z0 = y0 + cs;
    atomicAdd(x0, (unsigned long long)(long long)F0);
    atomicAdd(y0, (unsigned long long)(long long)ty0);
    atomicAdd(y0 + ss, (unsigned long long)(long long)ty1);
    atomicAdd(z0, (unsigned long long)(long long)tz0);
    atomicAdd(z0 + ss, (unsigned long long)(long long)tz1);
    if (moved) {
      atomicAdd(x0 + ss, (unsigned long long)(long long)F1);
      atomicAdd(y0 + 2 * ss, (unsigned long long)(long long)ty2);
      atomicAdd(z0 + 2 * ss, (unsigned long long)(long long)tz2);
    }
  } else {
    // keep the 64-bit products of this rare path out of the common one
    int F1m = F1, ty2m = ty2, tz2m = tz2;
    int t[5] = {F0, ty0, ty1, tz0, tz1};
    asm volatile("" : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]), "+v"(t[4]), "+v"(F1m), "+v"(ty2m),
                 "+v"(tz2m));
    const long long q = qw;
    atomicAdd(d.J[0] + j0, (unsigned long long)(q * t[0]));
    atomicAdd(d.J[1] + j0, (unsigned long long)(q * t[1]));
    atomicAdd(d.J[1] + j0 + 1, (unsigned long long)(q * t[2]));
    atomicAdd(d.J[2] + j0, (unsigned long long)(q * t[3]));
    atomicAdd(d.J[2] + j0 + 1, (unsigned long long)(q * t[4]));
    if (moved) {
      atomicAdd(d.J[0] + j0 + 1, (unsigned long long)(q * F1m));
      atomicAdd(d.J[1] + j0 + 2, (unsigned long long)(q * ty2m));
      atomicAdd(d.J[2] + j0 + 2, (unsigned long long)(q * tz2m));
    }
  }
}

// per-thread partial sums (a thread pushes the PPT particles of its tile; FP64 from the
// work-group sum on)
struct PushAcc {
  float rad, esc, stiff;
  int cmin1, cmax1;  // range of the new cells of the thread's particles
};

// Stored state of one particle (besides its cell).
template <typename R>
struct PData {
  int c;
  R o, ux, uy, uz, w;
  float rx, ry, rz;
};

// Partial derivatives of the fields at a particle, for the derivative term of
// Eq. (3dLL): d/dt and d/dx of E_x, E_y, E_z, B_y, B_z (B_x = 0 in 1D).
template <typename R>
struct FieldRates {
  R etx, ety, etz, bty, btz;  // d/dt
  R exx, exy, exz, bxy, bxz;  // d/dx
};

template <typename R>
struct MomentumOut {
  R Lx, Ly, Lz;     // u_L^{n+1/2}, after the Boris step
  R nx, ny, nz;     // u^{n+1/2} as stored
  R ddx, ddy, ddz;  // the RR increment added (with the carried residual under COMP)
  R gL;             // gamma of u_L (RR only)
};

// One momentum step of the paper's scheme (Section 3): Boris for the Lorentz
// force (Eq. (part1)), then the RR increment dt f_R of Eq. (f_r) at the
// mid-step estimate p^(n) = (u_L + u^{n-1/2}) / 2 of Eqs. (estim1) and
// (estimgamma), added as in Eq. (pertfull).  qh = q dt / (2 m), k = eps dt.
// COMP adds the increment by TwoSum and carries the FP32 rounding residual
// in (rx, ry, rz).  DERIV adds the derivative term of Eq. (3dLL) at the same
// p^(n) (the complete LL force, for tracking in given fields).  BX takes a
// non-zero B_x (multi-dimensional grids); without it B_x = 0, as in 1D, and
// none of its terms is evaluated.  ANY: momenta whose square overflows are
// stepped too, without RR (the runs drop them after the step).
template <typename R, bool RR, bool COMP, bool DERIV, bool BX = false, bool ANY = false>
__device__ __forceinline__ void momentum_step(R ux, R uy, R uz, R ex, R ey, R ez, R by, R bz, R qh,
                                              R k, const FieldRates<R>& fr, float& rx, float& ry,
                                              float& rz, float& stiff, MomentumOut<R>& o,
                                              R bx = R(0)) {
  // Boris
  const R hx = qh * ex, hy = qh * ey, hz = qh * ez;
  const R mx = ux + hx, my = uy + hy, mz = uz + hz;
  const R m2 = R(1) + mx * mx + my * my + mz * mz;
  const R igm = ANY ? rsq_any(m2) : rsq(m2);
  const R ty = qh * by * igm, tz = qh * bz * igm;
  R tx = R(0), den;
  if constexpr (BX) {
    tx = qh * bx * igm;
    den = R(1) + tx * tx + ty * ty + tz * tz;
  } else {
    den = R(1) + ty * ty + tz * tz;
  }
  const R sf = R(2) * (ANY ? rcp_any(den) : rcp(den));
  R px = mx + (my * tz - mz * ty);
  R py = my - mx * tz;
  R pz = mz + mx * ty;
  if constexpr (BX) {
    py += mz * tx;
    pz -= my * tx;
  }
  const R sy = sf * ty, sz = sf * tz;
  R Lx = mx + (py * sz - pz * sy) + hx;
  R Ly = my - px * sz + hy;
  R Lz = mz + px * sy + hz;
  if constexpr (BX) {
    const R sx = sf * tx;
    Ly += pz * sx;
    Lz -= py * sx;
  }

  R nx = Lx, ny = Ly, nz = Lz;
  R gL = R(0), ddx = R(0), ddy = R(0), ddz = R(0);
  if (RR) {
    // mid-step momentum (u_L + u^{n-1/2}) / 2 and its velocity
    const R qx = R(0.5) * (Lx + ux), qy = R(0.5) * (Ly + uy), qz = R(0.5) * (Lz + uz);
    const R g2 = R(1) + qx * qx + qy * qy + qz * qz;
    const R ig = rsq(g2);
    const R vx = qx * ig, vy = qy * ig, vz = qz * ig;
    // F = E + v x B = -f_L
    const R Fx = ex + (vy * bz - vz * by);
    R Fy = ey - vx * bz;
    R Fz = ez + vx * by;
    if constexpr (BX) {
      Fy += vz * bx;
      Fz -= vy * bx;
    }
    const R vE = vx * ex + vy * ey + vz * ez;
    R br = Fx * Fx + Fy * Fy + Fz * Fz - vE * vE;
    br = br > R(0) ? br : R(0);
    const R g2b = g2 * br;
    // dt f_R = dt eps [F x B + (v.E) E - gamma^2 (F^2 - (v.E)^2) v]
    if constexpr (BX) {
      ddx = k * ((Fy * bz - Fz * by) + vE * ex - g2b * vx);
      ddy = k * ((Fz * bx - Fx * bz) + vE * ey - g2b * vy);
      ddz = k * ((Fx * by - Fy * bx) + vE * ez - g2b * vz);
    } else {
      ddx = k * ((Fy * bz - Fz * by) + vE * ex - g2b * vx);
      ddy = k * (vE * ey - Fx * bz - g2b * vy);
      ddz = k * (Fx * by + vE * ez - g2b * vz);
    }
    if (DERIV) {
      // derivative term of Eq. (3dLL): -eps gamma [D E + v x D B], D = d/dt + v_x d/dx
      const R g = g2 * ig;
      const R DEx = fr.etx + vx * fr.exx, DEy = fr.ety + vx * fr.exy, DEz = fr.etz + vx * fr.exz;
      const R DBy = fr.bty + vx * fr.bxy, DBz = fr.btz + vx * fr.bxz;
      ddx -= k * g * (DEx + (vy * DBz - vz * DBy));
      ddy -= k * g * (DEy - vx * DBz);
      ddz -= k * g * (DEz + vx * DBy);
    }
    if (ddx * ddx + ddy * ddy + ddz * ddz > R(0.01) * (Lx * Lx + Ly * Ly + Lz * Lz)) stiff += 1.f;
    if (COMP) {
      // increment plus the residual carried from earlier steps, added by TwoSum;
      // the new rounding residual is carried to the next step
      const float dpx = (float)ddx + rx, dpy = (float)ddy + ry, dpz = (float)ddz + rz;
      float sxx, syy, szz;
      two_sum((float)Lx, dpx, sxx, rx);
      two_sum((float)Ly, dpy, syy, ry);
      two_sum((float)Lz, dpz, szz, rz);
      ddx = dpx;
      ddy = dpy;
      ddz = dpz;
      nx = sxx;
      ny = syy;
      nz = szz;
    } else {
      nx = Lx + ddx;
      ny = Ly + ddy;
      nz = Lz + ddz;
    }
    gL = fsqrt(R(1) + Lx * Lx + Ly * Ly + Lz * Lz);
  }

  o.Lx = Lx;
  o.Ly = Ly;
  o.Lz = Lz;
  o.nx = nx;
  o.ny = ny;
  o.nz = nz;
  o.ddx = ddx;
  o.ddy = ddy;
  o.ddz = ddz;
  o.gL = gL;
}

// All loads of one particle are independent of each other, so a thread keeps
// several particles' loads in flight while it computes an earlier one.
// Past the end of the species (i >= n, last tile only) the loads need no
// branch, and the particle is marked removed; the address is held to the
// arrays' capacity, not to n, so that the first loads of a work-group do not
// wait for the particle count.
template <typename R, bool COMP>
__device__ __forceinline__ PData<R> load_particle(const SpeciesDev<R>& sp, int i, int n, int cap) {
  PData<R> d;
  const unsigned ui = (unsigned)min(i, cap - 1);
  d.c = ld(sp.cell, ui);
  if (i >= n) d.c = kDead;
  d.o = ld(sp.off, ui);
  d.ux = ld(sp.ux, ui);
  d.uy = ld(sp.uy, ui);
  d.uz = ld(sp.uz, ui);
  d.w = ld(sp.w, ui);
  if (COMP) {
    d.rx = ld(sp.rx, ui);
    d.ry = ld(sp.ry, ui);
    d.rz = ld(sp.rz, ui);
  } else {
    d.rx = d.ry = d.rz = 0.f;
  }
  return d;
}

// The four field loads of one particle's gather: (E_y, E_z) at the nodes
// either side and (E_x, B_y, B_z) at the half-nodes either side.  They are
// issued from the particle's ring entry one particle ahead of its push, so
// that their latency overlaps the push of the particle before it.
template <typename R>
struct Gath {
  NodeF<R> n0, n1;
  HalfF<R> h0, h1;
};

template <typename R>
__device__ __forceinline__ Gath<R> gather_issue(const FieldsDev<R>& f, const PData<R>& pd) {
  const unsigned uc = pd.c == kDead ? 0u : (unsigned)pd.c;  // removed: any valid address
  const unsigned h = uc + (pd.o + R(0.5) >= R(1));
  Gath<R> g;
  g.n0 = ld(f.N, uc);
  g.n1 = ld(f.N, uc + 1);
  g.h0 = ld(f.H, h);
  g.h1 = ld(f.H, h + 1);
  return g;
}

// The fields of a tile's cells held in LDS: nodes and half-nodes c0 .. c0 +
// len - 1, of which cell c reads nodes c, c + 1 and half-nodes c .. c + 2.
template <typename R>
struct StageF {
  const HalfF<R>* H;
  const NodeF<R>* N;
  int c0, len;
};

template <typename R>
__device__ __forceinline__ Gath<R> gather_staged(const StageF<R>& f, const PData<R>& pd) {
  // (a removed particle, or one outside the range: any entry)
  const int e = min(max(pd.c - f.c0, 0), f.len - 3);
  const int h = e + (pd.o + R(0.5) >= R(1));
  Gath<R> g;
  g.n0 = f.N[e];
  g.n1 = f.N[e + 1];
  g.h0 = f.H[h];
  g.h1 = f.H[h + 1];
  return g;
}

// One particle: gather (from its field loads issued ahead), Boris, RR, move,
// deposit, store.
template <typename R, bool RR, bool COMP>
__device__ __forceinline__ void push_particle(const PushArgs<R>& a, const SpeciesDev<R>& sp,
                                              int s, int i, const PData<R>& pd, const Gath<R>& gf,
                                              DepositCtx& dc, PushAcc& acc) {
  const int c = pd.c;
  if (c == kDead) return;
  const unsigned ui = (unsigned)i;
  const R o = pd.o, ux = pd.ux, uy = pd.uy, uz = pd.uz, w = pd.w;
  float rx = pd.rx, ry = pd.ry, rz = pd.rz;

  // ---- gather E^n, B^n (linear weights; E_y,E_z on nodes, the rest on half-nodes).
  // The fused multiply-adds are written out: left to contraction, the two
  // unrolled ring slots were compiled with different roundings, and a
  // particle's result then depended on its slot, which the sort's order
  // within a cell leaves open.
  const R on = R(1) - o;
  const NodeF<R> n0 = gf.n0, n1 = gf.n1;
  const R ey = fma(o, n1.ey, on * n0.ey);
  const R ez = fma(o, n1.ez, on * n0.ez);
  const R sx = o + R(0.5);
  const unsigned hb = sx >= R(1);
  const R fh = hb ? sx - R(1) : sx;
  const R fn = R(1) - fh;
  const HalfF<R> h0 = gf.h0, h1 = gf.h1;
  const R ex = fma(fh, h1.ex, fn * h0.ex);
  const R by = fma(fh, h1.by, fn * h0.by);
  const R bz = fma(fh, h1.bz, fn * h0.bz);

  MomentumOut<R> mo;
  momentum_step<R, RR, COMP, false>(ux, uy, uz, ex, ey, ez, by, bz, a.qh[s], a.eps * a.dt,
                                    FieldRates<R>{}, rx, ry, rz, acc.stiff, mo);
  const R Lx = mo.Lx, Ly = mo.Ly, Lz = mo.Lz;
  const R nx = mo.nx, ny = mo.ny, nz = mo.nz;
  const R ddx = mo.ddx, ddy = mo.ddy, ddz = mo.ddz, gL = mo.gL;

  // ---- move (contract arithmetic)
  R g, vy, vz, o1, shift;
  contract_move<R>(nx, ny, nz, o, a.cfl, g, vy, vz, o1, shift);
  if (!(fabs(shift) < R(4)) || !(g < R(1e30))) {  // NaN/Inf momentum: drop it, raise the flag
    st(sp.cell, ui, kDead);
    atomicOr(a.flags, 1);
    return;
  }
  const int c1 = c + (int)shift;
  const int qw = a.Z[s] * (int)rint(w * a.sw);
  deposit<R>(dc, c, o, c1, o1, vy, vz, qw);

  if (RR) {
    // gamma_L - gamma_new = -(d . (2 u_L + d)) / (gamma_L + gamma_new)
    const R num = ddx * (R(2) * Lx + ddx) + ddy * (R(2) * Ly + ddy) + ddz * (R(2) * Lz + ddz);
    acc.rad -= (float)(w * num * rcp(gL + g));
  }
  if (c1 < 0 || c1 >= a.nx) {
    st(sp.cell, ui, kDead);
    acc.esc += (float)(w * (R)a.mass[s] * (g - R(1)));
  } else {
    st(sp.cell, ui, c1);
    st(sp.off, ui, o1);
    acc.cmin1 = min(acc.cmin1, c1);
    acc.cmax1 = max(acc.cmax1, c1);
  }
  st(sp.ux, ui, nx);
  st(sp.uy, ui, ny);
  st(sp.uz, ui, nz);
  if (COMP) {
    st(sp.rx, ui, rx);
    st(sp.ry, ui, ry);
    st(sp.rz, ui, rz);
  }
}

// ---------------------------------------------------------------- fields
template <typename R>
struct FieldArgs {
  FieldsDev<R> in, out;           // E^n, B^n -> E^{n+1}, B^{n+1}
  unsigned long long* J;          // currents, as in PushArgs
  unsigned jstride;
  int jfix;                       // buffer of this step's current, or -1: step mod 3
  const long long* Ex_in;         // integrals of the charge flux at n and n + 1
  long long* Ex_out;
  double* budget;                 // [0] E_in, [1] E_out_left, [2] E_out_right
  // incident (E_y, E_z) at t_{n+1/2}, in entry n & 1: the field pass of step
  // n - 1 (k_incident for a first step) leaves it, so that no pass waits for
  // the FP64 sines and no push tile has to hold them
  double* inc;                    // [2][2]
  const long long* step;          // device step counter
  long long* step_next;           // where work-group 0 leaves *step + 1 after the update, or null
  int nx;
  R a;                            // dt / dx
  R dt;
  double dtd;
  double sJx, sJy;                // fixed point -> current
  double sEx;                     // fixed point -> Ex
  double ay, az;                  // incident amplitude per component
  double tr, tf, tl;              // rise, flat, fall (1/omega)
};

// Current buffers around step n: `cur` holds (push) or receives the current
// of step n; `clear` is the one a field pass of step n zeroes.  With a fixed
// buffer the two in use alternate: the field pass of step n clears the next
// step's.  With three in rotation it clears the one after the next step's,
// which neither this launch nor a push running in it touches.  Before the
// push of step n its own buffer and, in rotation, the next one are zero.
__device__ __forceinline__ int j_buffer(int jfix, long long n) {
  return jfix >= 0 ? jfix : (int)((unsigned long long)n % 3ull);
}
__device__ __forceinline__ int j_clear(int jfix, int cur) {
  return jfix >= 0 ? jfix ^ 1 : (cur == 0 ? 2 : cur - 1);
}
template <typename A>
__device__ __forceinline__ unsigned long long* j_ptr(const A& p, int buf, int comp) {
  return p.J + (size_t)(3 * buf + comp) * p.jstride;
}

__device__ __forceinline__ double envelope(double t, double tr, double tf, double tl) {
  if (t <= 0.0) return 0.0;
  if (t < tr) {
    const double s = sin(0.5 * M_PI * t / tr);
    return s * s;
  }
  t -= tr;
  if (t < tf) return 1.0;
  t -= tf;
  if (t < tl) {
    const double c = cos(0.5 * M_PI * t / tl);
    return c * c;
  }
  return 0.0;
}

// Incident wave at x = 0 at t_{n+1/2} of step n, into its entry.
template <typename R>
__device__ __forceinline__ void incident(const FieldArgs<R>& p, long long n) {
  const double th = ((double)n + 0.5) * p.dtd;
  const double f = envelope(th, p.tr, p.tf, p.tl);
  p.inc[2 * (n & 1)] = p.ay * f * sin(th);
  p.inc[2 * (n & 1) + 1] = p.az * f * cos(th);
}

template <typename R>
__global__ void k_incident(FieldArgs<R> p, long long n) {
  incident<R>(p, n);
}

// The Yee update term by term, shared by the field pass and by the push
// tiles that advance their own cells: the fused multiply-adds are written
// out, so that both give the same bits.
template <typename R>
__device__ __forceinline__ R yee_bz(R bz, R ha, R ey_hi, R ey_lo) { return fma(-ha, ey_hi - ey_lo, bz); }
template <typename R>
__device__ __forceinline__ R yee_by(R by, R ha, R ez_hi, R ez_lo) { return fma(ha, ez_hi - ez_lo, by); }
template <typename R>
__device__ __forceinline__ R yee_ey(R ey, R a, R bz_hi, R bz_lo, R dt, R jy) {
  return fma(-dt, jy, fma(-a, bz_hi - bz_lo, ey));
}
template <typename R>
__device__ __forceinline__ R yee_ez(R ez, R a, R by_hi, R by_lo, R dt, R jz) {
  return fma(-dt, jz, fma(a, by_hi - by_lo, ez));
}
// boundary guards at t_{n+1/2} (first-order Silver-Mueller with injection)
template <typename R>
__device__ __forceinline__ void guard_left(R a, R dt, R ey, R ez, R bz1, R by1, R jy, R jz, double ey_in,
                                           double ez_in, R& bz, R& by) {
  const R d = R(1) + a;
  bz = (fma(dt, jy, fma(-(R(1) - a), bz1, fma(R(4), (R)ey_in, -(R(2) * ey))))) / d;
  by = (fma(R(-4), (R)ez_in, fma(-dt, jz, fma(R(2), ez, -((R(1) - a) * by1))))) / d;
}
template <typename R>
__device__ __forceinline__ void guard_right(R a, R dt, R ey, R ez, R bzn, R byn, R jy, R jz, R& bz, R& by) {
  const R d = R(1) + a;
  bz = (fma(-dt, jy, fma(R(2), ey, -((R(1) - a) * bzn)))) / d;
  by = (fma(dt, jz, fma(R(-2), ez, -((R(1) - a) * byn)))) / d;
}

// LDS elements of a field chunk of CH nodes
template <int CH>
constexpr int field_lds_elems() { return 8 * CH + 14; }

// One chunk of CH nodes (the work-group has CH threads) of step n, whose
// current is in buffer `jb`; `sm` holds field_lds_elems<CH>() elements of LDS.
template <typename R, int CH>
__device__ __forceinline__ void field_chunk(const FieldArgs<R>& p, int chunk, long long n_step, int jb, R* sm) {
  R* sEy = sm;                    // E^n, nodes i0-2 .. i0+CH
  R* sEz = sEy + (CH + 3);
  R* sBy = sEz + (CH + 3);        // B, half-nodes i0-1 .. i0+CH
  R* sBz = sBy + (CH + 2);
  R* sJy = sBz + (CH + 2);        // J, nodes i0-1 .. i0+CH-1
  R* sJz = sJy + (CH + 1);
  R* nEy = sJz + (CH + 1);        // E^{n+1}, nodes i0-1 .. i0+CH-1
  R* nEz = nEy + (CH + 1);
  const int t = threadIdx.x;
  const int i0 = chunk * CH;
  const int n = p.nx;
  const R a = p.a, ha = R(0.5) * p.a, dt = p.dt;
  const long long* J0 = (const long long*)j_ptr(p, jb, 0);
  const long long* J1 = (const long long*)j_ptr(p, jb, 1);
  const long long* J2 = (const long long*)j_ptr(p, jb, 2);

  // loads needed only at the end are issued first, so that their latency
  // overlaps the staged update below
  const int h = i0 + t;  // this thread's half-node (and node) output
  long long ex_old = 0, jx = 0;
  if (h <= n + 1) {
    ex_old = p.Ex_in[h];
    jx = J0[h];
  }
  // incident wave at t_{n+1/2} (work-group 0 only)
  double ey_in = 0.0, ez_in = 0.0;
  if (t == 0 && i0 == 0) {
    ey_in = p.inc[2 * (n_step & 1)];
    ez_in = p.inc[2 * (n_step & 1) + 1];
  }

  for (int k = t; k < CH + 3; k += CH) {
    const int i = i0 - 2 + k;
    const bool ok = i >= 0 && i <= n;
    const NodeF<R> v = ok ? p.in.N[i] : NodeF<R>{R(0), R(0)};
    sEy[k] = v.ey;
    sEz[k] = v.ez;
  }
  for (int k = t; k < CH + 2; k += CH) {
    const int h = i0 - 1 + k;
    const bool ok = h >= 0 && h <= n + 1;
    const HalfF<R> v = ok ? p.in.H[h] : HalfF<R>{R(0), R(0), R(0), R(0)};
    sBy[k] = v.by;
    sBz[k] = v.bz;
  }
  for (int k = t; k < CH + 1; k += CH) {
    const int i = i0 - 1 + k;
    const bool ok = i >= 0 && i <= n;
    sJy[k] = ok ? (R)((double)J1[i + 1] * p.sJy) : R(0);
    sJz[k] = ok ? (R)((double)J2[i + 1] * p.sJy) : R(0);
  }
  __syncthreads();

  // B^n -> B^{n+1/2} on interior half-nodes h = 1..n
  for (int k = t; k < CH + 2; k += CH) {
    const int h = i0 - 1 + k;
    if (h >= 1 && h <= n) {
      sBz[k] = yee_bz(sBz[k], ha, sEy[k + 1], sEy[k]);
      sBy[k] = yee_by(sBy[k], ha, sEz[k + 1], sEz[k]);
    }
  }
  __syncthreads();

  if (t == 0 && i0 == 0)
    // h = 0 is LDS index 1; node 0 is sEy index 2, Jy node 0 is sJy index 1
    guard_left<R>(a, dt, sEy[2], sEz[2], sBz[2], sBy[2], sJy[1], sJz[1], ey_in, ez_in, sBz[1], sBy[1]);
  if (t == 0 && n + 1 >= i0 && n + 1 <= i0 + CH) {
    const int k = n + 1 - (i0 - 1);       // LDS index of h = n+1
    const int kn = n - (i0 - 2);          // LDS index of node n in sEy
    const int kj = n - (i0 - 1);          // LDS index of node n in sJy
    guard_right<R>(a, dt, sEy[kn], sEz[kn], sBz[k - 1], sBy[k - 1], sJy[kj], sJz[kj], sBz[k], sBy[k]);
  }
  __syncthreads();

  // E^n -> E^{n+1} on nodes i0-1 .. i0+CH-1
  for (int k = t; k < CH + 1; k += CH) {
    const int i = i0 - 1 + k;
    if (i >= 0 && i <= n) {
      nEy[k] = yee_ey(sEy[k + 1], a, sBz[k + 1], sBz[k], dt, sJy[k]);
      nEz[k] = yee_ez(sEz[k + 1], a, sBy[k + 1], sBy[k], dt, sJz[k]);
    } else {
      nEy[k] = R(0);
      nEz[k] = R(0);
    }
  }
  __syncthreads();

  // boundary bookkeeping at t_{n+1/2}
  if (t == 0 && i0 == 0) {
    const double eyl = 0.5 * ((double)sEy[2] + (double)nEy[1]);
    const double ezl = 0.5 * ((double)sEz[2] + (double)nEz[1]);
    const double bzl = 0.5 * ((double)sBz[1] + (double)sBz[2]);
    const double byl = 0.5 * ((double)sBy[1] + (double)sBy[2]);
    const double L1 = eyl - bzl, L2 = ezl + byl;
    p.budget[0] += p.dtd * (ey_in * ey_in + ez_in * ez_in);
    p.budget[1] += p.dtd * 0.25 * (L1 * L1 + L2 * L2);
    if (p.step_next) *p.step_next = n_step + 1;
    incident<R>(p, n_step + 1);
  }
  if (t == 0 && i0 <= n && n < i0 + CH) {
    const int kn = n - (i0 - 2), ke = n - (i0 - 1), kb = n - (i0 - 1);
    const double eyr = 0.5 * ((double)sEy[kn] + (double)nEy[ke]);
    const double ezr = 0.5 * ((double)sEz[kn] + (double)nEz[ke]);
    const double bzr = 0.5 * ((double)sBz[kb] + (double)sBz[kb + 1]);
    const double byr = 0.5 * ((double)sBy[kb] + (double)sBy[kb + 1]);
    const double R1 = eyr + bzr, R2 = ezr - byr;
    p.budget[2] += p.dtd * 0.25 * (R1 * R1 + R2 * R2);
  }

  // own outputs: node i = i0 + t, half-node h = i0 + t
  const int jz = j_clear(p.jfix, jb);
  const int i = i0 + t;
  if (i <= n) {
    p.out.N[i] = NodeF<R>{nEy[t + 1], nEz[t + 1]};
  }
  if (h <= n + 1) {
    R bz = sBz[t + 1], byv = sBy[t + 1];
    if (h >= 1 && h <= n) {  // B^{n+1/2} -> B^{n+1} (guards keep their t_{n+1/2} value)
      bz = yee_bz(bz, ha, nEy[t + 1], nEy[t]);
      byv = yee_by(byv, ha, nEz[t + 1], nEz[t]);
    }
    const long long ex = ex_old - jx;
    p.Ex_out[h] = ex;
    p.out.H[h] = HalfF<R>{(R)((double)ex * p.sEx), byv, bz, R(0)};
    j_ptr(p, jz, 0)[h] = 0ull;
  }
  if (i0 + t <= n + 2) {
    j_ptr(p, jz, 1)[i0 + t] = 0ull;
    j_ptr(p, jz, 2)[i0 + t] = 0ull;
  }
}

template <typename R>
__global__ __launch_bounds__(kFieldChunk) void k_field(FieldArgs<R> p) {
  __shared__ R sm[field_lds_elems<kFieldChunk>()];
  const long long n = *p.step;
  field_chunk<R, kFieldChunk>(p, (int)blockIdx.x, n, j_buffer(p.jfix, n), sm);
}

// E^{n+1} at node i and (E_x, B)^{n+1} at half-node i (0 <= i <= nx + 1), by
// one thread from E^n, B^n and the current of step n: the values field_chunk
// writes, bit for bit.
template <typename R>
__device__ __forceinline__ void field_direct(const FieldArgs<R>& p, int i, long long n_step, int jb,
                                             NodeF<R>& N1, HalfF<R>& H1) {
  const int n = p.nx;
  const R a = p.a, ha = R(0.5) * p.a, dt = p.dt;
  const long long* J1 = (const long long*)j_ptr(p, jb, 1);
  const long long* J2 = (const long long*)j_ptr(p, jb, 2);
  // nodes i-2 .. i+1 and half-nodes i-1 .. i+1 (clamped: what lies outside
  // enters nothing that is used)
  NodeF<R> e[4];
  HalfF<R> b[3];
  R jy[2], jz[2];
#pragma unroll
  for (int k = 0; k < 4; ++k) e[k] = ld(p.in.N, (unsigned)min(max(i - 2 + k, 0), n));
#pragma unroll
  for (int k = 0; k < 3; ++k) b[k] = ld(p.in.H, (unsigned)min(max(i - 1 + k, 0), n + 1));
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const unsigned m = (unsigned)min(max(i - 1 + k, 0), n) + 1u;
    jy[k] = (R)((double)ld(J1, m) * p.sJy);
    jz[k] = (R)((double)ld(J2, m) * p.sJy);
  }
  const long long ex = ld(p.Ex_in, (unsigned)i) - ld((const long long*)j_ptr(p, jb, 0), (unsigned)i);
  R bz[3], by[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int h = i - 1 + k;
    bz[k] = b[k].bz;
    by[k] = b[k].by;
    if (h >= 1 && h <= n) {
      bz[k] = yee_bz(bz[k], ha, e[k + 1].ey, e[k].ey);
      by[k] = yee_by(by[k], ha, e[k + 1].ez, e[k].ez);
    }
  }
  if (i <= 1) {  // the guard h = 0: index 1 of i = 0, index 0 of i = 1
    const double ey_in = p.inc[2 * (n_step & 1)], ez_in = p.inc[2 * (n_step & 1) + 1];
    R gz, gy;
    if (i == 0) {
      guard_left<R>(a, dt, e[2].ey, e[2].ez, bz[2], by[2], jy[1], jz[1], ey_in, ez_in, gz, gy);
      bz[1] = gz;
      by[1] = gy;
    } else {
      guard_left<R>(a, dt, e[1].ey, e[1].ez, bz[1], by[1], jy[0], jz[0], ey_in, ez_in, gz, gy);
      bz[0] = gz;
      by[0] = gy;
    }
  }
  if (i >= n) {  // the guard h = n + 1: index 2 of i = n, index 1 of i = n + 1
    R gz, gy;
    if (i == n) {
      guard_right<R>(a, dt, e[2].ey, e[2].ez, bz[1], by[1], jy[1], jz[1], gz, gy);
      bz[2] = gz;
      by[2] = gy;
    } else {
      guard_right<R>(a, dt, e[1].ey, e[1].ez, bz[0], by[0], jy[0], jz[0], gz, gy);
      bz[1] = gz;
      by[1] = gy;
    }
  }
  const R ey0 = yee_ey(e[1].ey, a, bz[1], bz[0], dt, jy[0]), ez0 = yee_ez(e[1].ez, a, by[1], by[0], dt, jz[0]);
  const R ey1 = yee_ey(e[2].ey, a, bz[2], bz[1], dt, jy[1]), ez1 = yee_ez(e[2].ez, a, by[2], by[1], dt, jz[1]);
  N1 = NodeF<R>{ey1, ez1};
  R oz = bz[1], oy = by[1];
  if (i >= 1 && i <= n) {
    oz = yee_bz(oz, ha, ey1, ey0);
    oy = yee_by(oy, ha, ez1, ez0);
  }
  H1 = HalfF<R>{(R)((double)ex * p.sEx), oy, oz, R(0)};
}

// The field loads of one particle's gather when its tile's fields are not
// in LDS: computed for this particle alone.
template <typename R>
__device__ __forceinline__ Gath<R> gather_direct(const FieldArgs<R>& p, long long n_step, int jb,
                                                 const PData<R>& pd) {
  const int c = pd.c == kDead ? 0 : pd.c;
  const int hb = pd.o + R(0.5) >= R(1);
  Gath<R> g;
#pragma unroll 1
  for (int k = 0; k < 3; ++k) {
    NodeF<R> N1;
    HalfF<R> H1;
    field_direct<R>(p, c + k, n_step, jb, N1, H1);
    if (k == 0) g.n0 = N1;
    if (k == 1) g.n1 = N1;
    if (k == hb) g.h0 = H1;
    if (k == hb + 1) g.h1 = H1;
  }
  return g;
}

// ---------------------------------------------------------------- push
// PPT particles per thread, D of them with loads in flight (D = PPT: the
// whole tile is loaded up front).  FUSED: the fields at a.f are not advanced
// yet; the tile computes those of its own cells, from *fa (the field pass of
// the step before, n_step), into the front of its LDS, and gathers there.
template <typename R, bool RR, bool COMP, int PPT, int D, bool FUSED>
__device__ __forceinline__ void push_tile(const PushArgs<R>& a, int s, int tile, int base, int jw,
                                          unsigned long long* lds, const FieldArgs<R>* fa,
                                          long long n_step, int jr) {
  static_assert(PPT % D == 0, "the load ring must divide the tile");
  // the next particle's field loads are issued from its ring entry, which
  // must be a different entry from the current particle's
  static_assert(D >= 2 || PPT == 1, "a ring of one entry holds one particle per thread only");
  __shared__ int s_mn[kThreads / kLanes], s_mx[kThreads / kLanes];
  __shared__ double s_red[3][kThreads / kLanes];
  const SpeciesDev<R> sp = a.sp[s];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int n = (int)a.count[s];
  const int cap = a.cap;
  // the tile's cell range as the previous push left it, if that is known
  // (loaded beside the flag that says so)
  const int known = *a.pred_in;
  const int rlo = a.rng_in[2 * tile], rhi = a.rng_in[2 * tile + 1];

  // the first particles' loads overlap the window set-up below
  PData<R> ring[D];
#pragma unroll
  for (int k = 0; k < D; ++k) ring[k] = load_particle<R, COMP>(sp, base + k * kThreads + tid, n, cap);
  if (base >= n) return;

  // the tile's cell range: as the previous push left it, when that is
  // known, else from a pass over the cells (from the ring when it holds the
  // whole tile)
  int cmin = INT_MAX, cmax = INT_MIN;
  if (__builtin_amdgcn_readfirstlane(known)) {
    cmin = __builtin_amdgcn_readfirstlane(rlo);
    cmax = __builtin_amdgcn_readfirstlane(rhi);
  } else {
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
      int c;
      if constexpr (PPT == D) {
        c = ring[k].c;
      } else {
        const int i = base + k * kThreads + tid;
        c = i < n ? ld(sp.cell, (unsigned)i) : kDead;
      }
      if (c != kDead) {
        cmin = min(cmin, c);
        cmax = max(cmax, c);
      }
    }
    cmin = wave_min_dpp(cmin);
    cmax = wave_max_dpp(cmax);
    if (lane == 0) {
      s_mn[wid] = cmin;
      s_mx[wid] = cmax;
    }
    __syncthreads();
    cmin = min(min(s_mn[0], s_mn[1]), min(s_mn[2], s_mn[3]));
    cmax = max(max(s_mx[0], s_mx[1]), max(s_mx[2], s_mx[3]));
  }
  if (cmin > cmax) {  // every particle of the tile was removed
    if (tid == 0) {
      a.rng_out[2 * tile] = INT_MAX;
      a.rng_out[2 * tile + 1] = INT_MIN;
      *a.pred_out = 1;
    }
    return;
  }

  // FUSED: fields of nodes and half-nodes cmin .. cmax + 2 into the front of
  // the LDS, one thread per node, unless the tile is too wide to leave room
  // for its window
  int fslots = 0;
  StageF<R> stage{nullptr, nullptr, 0, 0};
  if constexpr (FUSED) {
    constexpr int kPer = (sizeof(HalfF<R>) + sizeof(NodeF<R>)) / sizeof(unsigned long long);
    const int len = cmax - cmin + 3;
    if (kPer * len + 3 * (cmax - cmin + 4) <= kLdsSlots) {
      HalfF<R>* H = reinterpret_cast<HalfF<R>*>(lds);
      NodeF<R>* N = reinterpret_cast<NodeF<R>*>(H + len);
      for (int e = tid; e < len; e += kThreads) {
        NodeF<R> N1;
        HalfF<R> H1;
        field_direct<R>(*fa, cmin + e, n_step, jr, N1, H1);
        H[e] = H1;
        N[e] = N1;
      }
      fslots = kPer * len;
      stage = StageF<R>{H, N, cmin, len};
    }
  }

  // window: storage indices cmin .. cmax + 3 (nodes cmin - 1 .. cmax + 2),
  // with as many private copies per slot (up to 64) as the LDS holds
  DepositCtx dc;
  dc.lds = lds + fslots;
#pragma unroll
  for (int k = 0; k < 3; ++k) dc.J[k] = j_ptr(a, jw, k);
  dc.wlo = cmin;
  dc.W = cmax - cmin + 4;
  dc.qw_ref = a.qw_ref[s];
  const int room = kLdsSlots - fslots;
  int sh = 6;
  while (sh > 0 && 3 * dc.W * ((1 << sh) + 1) > room) --sh;
  dc.P = sh ? (1 << sh) + 1 : 1;
  dc.copy = lane & ((1 << sh) - 1);
  const int E = 3 * dc.W * dc.P;
  dc.use_lds = E <= room;
  if (dc.use_lds)
    for (int e = tid; e < E; e += kThreads) dc.lds[e] = 0ull;
  __syncthreads();

  PushAcc acc{0.f, 0.f, 0.f, INT_MAX, INT_MIN};
  // ring slot j holds particle k0 + j; its successor D ahead is loaded
  // before particle k0 + j is computed, and the field loads of particle
  // k0 + j + 1 (whose ring entry has arrived) before those of k0 + j + D
  auto gather = [&](const PData<R>& pd) {
    if constexpr (FUSED) return gather_staged<R>(stage, pd);
    else return gather_issue<R>(a.f, pd);
  };
  if (!FUSED || fslots) {
    Gath<R> gnext = gather(ring[0]);
#pragma unroll kRingUnroll
    for (int k0 = 0; k0 < PPT; k0 += D) {
#pragma unroll
      for (int j = 0; j < D; ++j) {
        const int i = base + (k0 + j) * kThreads + tid;
        const PData<R> cur = ring[j];
        const Gath<R> gcur = gnext;
        if (k0 + j + 1 < PPT) gnext = gather(ring[(j + 1) % D]);
        if (k0 + j + D < PPT) ring[j] = load_particle<R, COMP>(sp, i + D * kThreads, n, cap);
        push_particle<R, RR, COMP>(a, sp, s, i, cur, gcur, dc, acc);
      }
    }
  } else if constexpr (FUSED) {  // a tile wider than the LDS: rare, one particle after the other
#pragma unroll 1
    for (int k = 0; k < PPT; ++k) {
      const int i = base + k * kThreads + tid;
      const PData<R> cur = load_particle<R, COMP>(sp, i, n, cap);
      push_particle<R, RR, COMP>(a, sp, s, i, cur, gather_direct<R>(*fa, n_step, jr, cur), dc, acc);
    }
  }

  const double r0 = wave_sum_dpp((double)acc.rad), r1 = wave_sum_dpp((double)acc.esc),
               r2 = wave_sum_dpp((double)acc.stiff);
  const int n0 = wave_min_dpp(acc.cmin1), n1 = wave_max_dpp(acc.cmax1);
  if (lane == 0) {
    s_red[0][wid] = r0;
    s_red[1][wid] = r1;
    s_red[2][wid] = r2;
    s_mn[wid] = n0;
    s_mx[wid] = n1;
  }
  __syncthreads();

  // flush: g lanes per slot each sum R / g copies, DPP adds the g partial
  // sums, and the group's last lane issues one global atomic
  if (dc.use_lds) {
    const int nc = 1 << sh;  // copies per slot
    const int gsh = sh < 4 ? sh : 4, g = 1 << gsh;
    const int S = 3 * dc.W, gi = tid >> gsh, t = tid & (g - 1);
    for (int s0 = 0; s0 < S; s0 += kThreads >> gsh) {
      const int sl = s0 + gi;
      long long v = 0;
      if (sl < S) {
        const unsigned long long* q = dc.lds + sl * dc.P + t;
        for (int k = 0; k < nc; k += g) v += (long long)q[k];
      }
      v = group_sum(v, g);
      if (t == g - 1 && sl < S && v != 0) {
        const int comp = sl / dc.W, j = sl - comp * dc.W;
        atomicAdd(j_ptr(a, jw, comp) + dc.wlo + j, (unsigned long long)(v * (long long)dc.qw_ref));
      }
    }
  }
  if (tid == 0) {
    double t0 = 0.0, t1 = 0.0, t2 = 0.0;
    for (int w = 0; w < kThreads / kLanes; ++w) {
      t0 += s_red[0][w];
      t1 += s_red[1][w];
      t2 += s_red[2][w];
    }
    // the tile's cells for the next push
    a.rng_out[2 * tile] = min(min(s_mn[0], s_mn[1]), min(s_mn[2], s_mn[3]));
    a.rng_out[2 * tile + 1] = max(max(s_mx[0], s_mx[1]), max(s_mx[2], s_mx[3]));
    *a.pred_out = 1;
    // one add per slot and launch, in launch order: deterministic; the
    // atomic form needs no load, so the work-group retires without waiting
    double* A = a.acc + 4 * (size_t)tile;
    unsafeAtomicAdd(A + 0, t0);
    unsafeAtomicAdd(A + 1 + s, t1);
    unsafeAtomicAdd(A + 3, t2);
  }
}

// Tile `tile` of a push whose current goes to buffer jw.  FUSED: with the
// field pass *fa of step n_step, whose current is in buffer jr, still due.
template <typename R, int PPT, int D, bool FUSED = false>
__device__ __forceinline__ void push_one_tile(const PushArgs<R>& a, int tile, int jw, unsigned long long* lds,
                                              const FieldArgs<R>* fa = nullptr, long long n_step = 0,
                                              int jr = 0) {
  const int s = tile < a.tiles0 ? 0 : 1;
  const int tl = s ? tile - a.tiles0 : tile;
  const int base = tl * (kThreads * PPT);
  if (s == 0 && a.rr0) {
    if (a.comp)
      push_tile<R, true, true, PPT, D, FUSED>(a, s, tile, base, jw, lds, fa, n_step, jr);
    else
      push_tile<R, true, false, PPT, D, FUSED>(a, s, tile, base, jw, lds, fa, n_step, jr);
  } else {
    push_tile<R, false, false, PPT, D, FUSED>(a, s, tile, base, jw, lds, fa, n_step, jr);
  }
}

#if PIC_PUSH_MIN_WAVES > 0
#define PIC_PUSH_BOUNDS __launch_bounds__(kThreads, PIC_PUSH_MIN_WAVES)
#else
#define PIC_PUSH_BOUNDS __launch_bounds__(kThreads)
#endif

// one work-group per tile
template <typename R>
__global__ PIC_PUSH_BOUNDS void k_push(PushArgs<R>) {
  const PushArgs<R>& a = kernel_args<PushArgs<R>>();
  __shared__ __align__(16) unsigned long long lds[kLdsSlots];
  const int jw = j_buffer(a.jfix, a.jfix >= 0 ? 0 : *a.step);
  push_one_tile<R, kPPT, kDepth>(a, a.tile0 + (int)blockIdx.x, jw, lds);
}

// the same push in tiles of PPT particles per thread (two particles' loads in
// flight, as in the batched push), for runs too small to fill the device with
// kTile tiles
template <typename R, int PPT>
__global__ PIC_PUSH_BOUNDS void k_push_small(PushArgs<R>) {
  const PushArgs<R>& a = kernel_args<PushArgs<R>>();
  __shared__ __align__(16) unsigned long long lds[kLdsSlots];
  const int jw = j_buffer(a.jfix, a.jfix >= 0 ? 0 : *a.step);
  push_one_tile<R, PPT, (PPT > 1 ? kBatchDepth : 1)>(a, a.tile0 + (int)blockIdx.x, jw, lds);
}

// One launch per step for small runs: the field pass of step n (f) and the
// push of step n + 1 (a) together.  Both read only E^n, B^n and the current
// of step n: every push tile advances the fields of its own cells into LDS,
// by the arithmetic of the field pass, while the work-groups after the push
// tiles advance the whole grid for the next launch and the diagnostics.  The
// push deposits into the next current buffer of three, and the field pass
// clears the third.  A step of a small run is bound by the latency of its
// launches, not by the few MB it moves: 12,800 particles in FP32 took 8.9 us
// (push) + 4.5 us (fields) and a gap per step, now 6.7 us in tiles of 256
// particles (9.3 in tiles of 1,024); 4e5 in FP64 12.7 + 4.9, now 12.2 us.
template <typename R>
struct StepArgs {
  PushArgs<R> a;
  FieldArgs<R> f;
};

template <typename R, int PPT>
__global__ PIC_PUSH_BOUNDS void k_step(StepArgs<R>) {
  const PushArgs<R>& a = kernel_args<StepArgs<R>>().a;
  const FieldArgs<R>& f = kernel_args<StepArgs<R>>().f;
  __shared__ __align__(16) unsigned long long lds[kLdsSlots];
  static_assert(field_lds_elems<kThreads>() * sizeof(R) <= sizeof(lds), "field chunk must fit the window");
  const long long n = *f.step;
  const int jr = j_buffer(-1, n), jw = jr == 2 ? 0 : jr + 1;
  const int b = (int)blockIdx.x;
  if (b < a.ntiles)
    push_one_tile<R, PPT, (PPT > 1 ? kBatchDepth : 1), true>(a, b, jw, lds, &f, n, jr);
  else
    field_chunk<R, kThreads>(f, b - a.ntiles, n, jr, reinterpret_cast<R*>(lds));
}

// ---------------------------------------------------------------- sort
template <typename R>
struct SortArgs {
  SpeciesDev<R> src[2], dst[2];
  const long long* count;  // [2] particles in the source arrays
  int* cnt[2];          // [n] per-cell counts (zero on entry to k_sort_hist)
  int* cursor[2];       // [n] scatter cursors
  int blocks0;          // blocks of species 0 in hist / scatter grids
  int blk0;             // first block of this launch (a pass may be split over launches)
  int nx;
  int comp;             // carry residuals of species 0
  int* pred;            // [2] the push's range-prediction flags, cleared: the order changes
  int ysh, bxs, bys;    // 2D grids: cell = ix << ysh | iy, sorted by blocks of 2^bxs x 2^bys cells
};

// Sort key of a 2D cell: blocks of 2^bxs x 2^bys cells column by column,
// and the cells of a block column by column, so that the particles of a
// sort tile (and of a push tile) lie in a compact patch of the grid rather
// than along one column.  A bijection of [0, roundup(nx, 2^bxs) << ysh);
// with bxs = bys = 0 the key is the cell index itself.
__device__ __forceinline__ int sort_key2(int c, int ysh, int bxs, int bys) {
  if (c == kDead) return kDead;
  const int ix = c >> ysh, iy = c & ((1 << ysh) - 1);
  return ((ix >> bxs) << (ysh + bxs)) | ((iy >> bys) << (bxs + bys)) |
         ((ix & ((1 << bxs) - 1)) << bys) | (iy & ((1 << bys) - 1));
}

constexpr int kSortThreads = 256;
constexpr int kSortPPT = 8;                        // particles per thread per sort tile
constexpr int kSortTile = kSortThreads * kSortPPT;
constexpr int kSortWin = 4096;                     // LDS cell window of a sort tile (a power of two,
                                                   // at least twice kSortTile)

// atomicAdd(ptr[key], 1) of every valid lane, returning each lane's slot
// (ptr may point to LDS or HBM).  The lanes that share the first valid lane's
// key go together, the others by themselves, in one atomic instruction: a
// wave of a dense, sorted tile has one or two keys, a wave of a heated one
// up to 64, and a round of the whole wave per distinct key then took most of
// the sort (16,384 particles in 2D: 21 us for the histogram and 29 us for the
// scatter, now 6.2 and 7.4 us).
__device__ __forceinline__ int wave_claim(int* ptr, int key, bool valid) {
  const int lane = threadIdx.x & 63;
  const unsigned long long active = __ballot(valid);
  if (!active) return 0;
  const int leader = __ffsll((long long)active) - 1;
  const bool same = valid && key == __builtin_amdgcn_readlane(key, leader);
  const unsigned long long group = __ballot(same);
  int slot = 0;
  if (lane == leader || (valid && !same)) slot = atomicAdd(ptr + key, lane == leader ? __popcll(group) : 1);
  const int base = __builtin_amdgcn_readlane(slot, leader);
  return same ? base + __popcll(group & ((1ull << lane) - 1ull)) : slot;
}

// Cell range of a sort tile (block-uniform result).
__device__ __forceinline__ void tile_range(const int* cl, int& lo, int& hi, int* sm) {
  int a = INT_MAX, b = INT_MIN;
#pragma unroll
  for (int k = 0; k < kSortPPT; ++k)
    if (cl[k] != kDead) {
      a = min(a, cl[k]);
      b = max(b, cl[k]);
    }
  a = wave_min_dpp(a);
  b = wave_max_dpp(b);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  __syncthreads();  // earlier readers of sm (previous tile) are done
  if (lane == 0) {
    sm[wid] = a;
    sm[4 + wid] = b;
  }
  __syncthreads();
  lo = min(min(sm[0], sm[1]), min(sm[2], sm[3]));
  hi = max(max(sm[4], sm[5]), max(sm[6], sm[7]));
}

// LDS table of the keys of a tile that span more than the window (fewer than
// 2^20 keys): an entry holds (key - lo) << 12 | particles, in the window's own
// memory, twice as many entries as the tile has particles.  Open addressing
// from a multiplicative hash (from the key's low bits, the runs of
// neighbouring keys made probes of hundreds of entries).  Returns the entry
// of `key` and, in *rank, how many of its particles came before.
constexpr int kTableSpan = 1 << 20;
static_assert(kSortWin == 4096 && kSortTile <= kSortWin / 2, "the table hashes to 12 bits, at most half full");
__device__ __forceinline__ int table_add(int* tab, int key, int lo, int* rank) {
  const int mine = (int)((unsigned)(key - lo) << 12);
  unsigned h = ((unsigned)(key - lo) * 0x9E3779B1u) >> 20;
  for (;;) {
    const int old = atomicCAS(tab + h, -1, mine);
    if (old == -1 || ((unsigned)old >> 12) == (unsigned)(key - lo)) break;
    h = (h + 1) & (kSortWin - 1);
  }
  *rank = atomicAdd(tab + h, 1) & 4095;
  return (int)h;
}

// Per-cell particle counts: LDS histogram over the tile's cell window, then
// one global atomic per occupied cell and tile.  Global atomics leave the
// chip's caches at some 11 per ns in all, so that one per particle bounds a
// tile of sparse, heated particles; those of 2D grids that span more
// than the window count in an LDS table of their keys instead (8.4e6 heated
// particles: histogram 235 us, now 95; scatter 577, now 318; cold ones take
// 19 and 118 us).
template <typename R, bool KEY2 = false>
__device__ __forceinline__ void sort_hist_block(const SortArgs<R>& p, int blk) {
  __shared__ int cnt[kSortWin];
  __shared__ int sm[8];
  const int s = blk < p.blocks0 ? 0 : 1;
  const int b = s ? blk - p.blocks0 : blk;
  const long long n = p.count[s];
  const long long base = (long long)b * kSortTile;
  if (base >= n) return;
  int cl[kSortPPT];
#pragma unroll
  for (int k = 0; k < kSortPPT; ++k) {
    const long long i = base + k * kSortThreads + threadIdx.x;
    cl[k] = i < n ? p.src[s].cell[i] : kDead;
    if constexpr (KEY2) cl[k] = sort_key2(cl[k], p.ysh, p.bxs, p.bys);
  }
  int lo, hi;
  tile_range(cl, lo, hi, sm);
  if (lo > hi) return;
  const int W = hi - lo + 1;
  if (W <= kSortWin) {
    for (int e = threadIdx.x; e < W; e += kSortThreads) cnt[e] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSortPPT; ++k) wave_claim(cnt, cl[k] - lo, cl[k] != kDead);
    __syncthreads();
    for (int e = threadIdx.x; e < W; e += kSortThreads)
      if (cnt[e]) atomicAdd(p.cnt[s] + lo + e, cnt[e]);
  } else if (KEY2 && W < kTableSpan) {
    for (int e = threadIdx.x; e < kSortWin; e += kSortThreads) cnt[e] = -1;
    __syncthreads();
    int rank;
#pragma unroll 1
    for (int k = 0; k < kSortPPT; ++k)
      if (cl[k] != kDead) table_add(cnt, cl[k], lo, &rank);
    __syncthreads();
    for (int e = threadIdx.x; e < kSortWin; e += kSortThreads)
      if (cnt[e] != -1) atomicAdd(p.cnt[s] + lo + ((unsigned)cnt[e] >> 12), cnt[e] & 4095);
  } else {
#pragma unroll
    for (int k = 0; k < kSortPPT; ++k) wave_claim(p.cnt[s], cl[k], cl[k] != kDead);
  }
}

template <typename R>
__global__ __launch_bounds__(kSortThreads) void k_sort_hist(SortArgs<R> p) {
  sort_hist_block<R>(p, p.blk0 + (int)blockIdx.x);
}

// inclusive prefix sum over the 64 lanes of a wave (all lanes active)
__device__ __forceinline__ int wave_incl_scan(int v) {
  v += row_shr<1>(0, v);
  v += row_shr<2>(0, v);
  v += row_shr<4>(0, v);
  v += row_shr<8>(0, v);
  const int r0 = __builtin_amdgcn_readlane(v, 15), r1 = __builtin_amdgcn_readlane(v, 31),
            r2 = __builtin_amdgcn_readlane(v, 47);
  const int row = (threadIdx.x & 63) >> 4;
  return v + (row >= 1 ? r0 : 0) + (row >= 2 ? r1 : 0) + (row >= 3 ? r2 : 0);
}

// Exclusive scan of one chunk of kScanChunk per-cell counts (one work-group
// of 1024 threads), starting from `carry`: the chunk passes through LDS so
// that every global access is coalesced; within it thread t scans cells
// 8t .. 8t + 7.  Writes the cursors, clears the counts for the next
// histogram and returns the chunk's total.
constexpr int kScanThreads = 1024, kScanPer = 8, kScanChunk = kScanThreads * kScanPer;
__device__ __forceinline__ int scan_chunk(int* cnt, int* cur, int c0, int nx, long long carry,
                                          int* stage, int* wsum) {
  const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    const int j = c0 + k * kScanThreads + t;
    stage[k * kScanThreads + t] = j < nx ? cnt[j] : 0;
  }
  __syncthreads();
  int v[kScanPer], sum = 0;
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    v[k] = stage[t * kScanPer + k];
    sum += v[k];
  }
  const int incl = wave_incl_scan(sum);
  if (lane == 63) wsum[wid] = incl;
  __syncthreads();
  int before = 0, total = 0;
  for (int w = 0; w < kScanThreads / kLanes; ++w) {
    before += w < wid ? wsum[w] : 0;
    total += wsum[w];
  }
  int run = (int)carry + before + incl - sum;
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    stage[t * kScanPer + k] = run;
    run += v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kScanPer; ++k) {
    const int j = c0 + k * kScanThreads + t;
    if (j < nx) {
      cur[j] = stage[k * kScanThreads + t];
      cnt[j] = 0;
    }
  }
  __syncthreads();  // stage and wsum are reused by the next chunk
  return total;
}

// exclusive scan of the per-cell counts of one species in one work-group,
// chunk after chunk; the alive count goes to *new_count (the count slot of
// the destination arrays)
__device__ __forceinline__ void sort_scan_species(int* cnt, int* cur, long long* new_count, int nx) {
  __shared__ int stage[kScanChunk];
  __shared__ int wsum[kScanThreads / kLanes];
  long long carry = 0;
  for (int c0 = 0; c0 < nx; c0 += kScanChunk) carry += scan_chunk(cnt, cur, c0, nx, carry, stage, wsum);
  if (threadIdx.x == 0) *new_count = carry;
}

__global__ __launch_bounds__(1024) void k_sort_scan(int* cnt0, int* cnt1, int* cur0, int* cur1,
                                                    long long* new_count, int nx) {
  if (blockIdx.x == 0)
    sort_scan_species(cnt0, cur0, new_count, nx);
  else
    sort_scan_species(cnt1, cur1, new_count + 1, nx);
}

// scatter to the destination arrays: each tile claims, per occupied cell,
// one contiguous range of the cell's bucket with a single global atomic and
// hands out positions inside it through an LDS counter (OY: particles of a
// 2D grid also carry a y offset)
template <typename R, bool OY = false>
__device__ __forceinline__ void sort_scatter_block(const SortArgs<R>& p, int blk) {
  __shared__ int cnt[kSortWin];
  __shared__ int sm[8];
  const int s = blk < p.blocks0 ? 0 : 1;
  const int b = s ? blk - p.blocks0 : blk;
  const long long n = p.count[s];
  const long long base = (long long)b * kSortTile;
  if (blk == 0 && threadIdx.x == 0) p.pred[0] = p.pred[1] = 0;
  if (base >= n) return;
  const SpeciesDev<R> src = p.src[s], dst = p.dst[s];
  const bool comp = s == 0 && p.comp;
  int cl[kSortPPT], pos[kSortPPT];
  // the particles' data is loaded with their cells, so that its latency
  // overlaps the position claims below
  R off[kSortPPT], ux[kSortPPT], uy[kSortPPT], uz[kSortPPT], w[kSortPPT], oy[kSortPPT];
  float rx[kSortPPT], ry[kSortPPT], rz[kSortPPT];
#pragma unroll
  for (int k = 0; k < kSortPPT; ++k) {
    const long long i = base + k * kSortThreads + threadIdx.x;
    cl[k] = kDead;
    if (i < n) {
      const unsigned ui = (unsigned)i;
      cl[k] = ld(src.cell, ui);
      off[k] = ld(src.off, ui);
      ux[k] = ld(src.ux, ui);
      uy[k] = ld(src.uy, ui);
      uz[k] = ld(src.uz, ui);
      w[k] = ld(src.w, ui);
      if constexpr (OY) oy[k] = ld(src.oy, ui);
      if (comp) {
        rx[k] = ld(src.rx, ui);
        ry[k] = ld(src.ry, ui);
        rz[k] = ld(src.rz, ui);
      }
    }
  }
  // bucket keys: the cell itself, or its 2D block key (OY)
  int ky[kSortPPT];
#pragma unroll
  for (int k = 0; k < kSortPPT; ++k) {
    if constexpr (OY) ky[k] = sort_key2(cl[k], p.ysh, p.bxs, p.bys);
    else ky[k] = cl[k];
  }
  int lo, hi;
  tile_range(ky, lo, hi, sm);
  if (lo > hi) return;
  const int W = hi - lo + 1;
  if (W <= kSortWin) {
    for (int e = threadIdx.x; e < W; e += kSortThreads) cnt[e] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSortPPT; ++k) pos[k] = wave_claim(cnt, ky[k] - lo, ky[k] != kDead);
    __syncthreads();
    for (int e = threadIdx.x; e < W; e += kSortThreads)
      cnt[e] = cnt[e] ? atomicAdd(p.cursor[s] + lo + e, cnt[e]) : 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSortPPT; ++k)
      if (ky[k] != kDead) pos[k] += cnt[ky[k] - lo];
  } else if (OY && W < kTableSpan) {  // (the table of the histogram)
    for (int e = threadIdx.x; e < kSortWin; e += kSortThreads) cnt[e] = -1;
    __syncthreads();
    int en[kSortPPT];
#pragma unroll
    for (int k = 0; k < kSortPPT; ++k) {
      en[k] = 0;
      pos[k] = 0;
      if (ky[k] != kDead) en[k] = table_add(cnt, ky[k], lo, &pos[k]);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kSortWin; e += kSortThreads)
      if (cnt[e] != -1) cnt[e] = atomicAdd(p.cursor[s] + lo + ((unsigned)cnt[e] >> 12), cnt[e] & 4095);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSortPPT; ++k) pos[k] += cnt[en[k]];
  } else {
#pragma unroll
    for (int k = 0; k < kSortPPT; ++k) pos[k] = wave_claim(p.cursor[s], ky[k], ky[k] != kDead);
  }
#pragma unroll
  for (int k = 0; k < kSortPPT; ++k) {
    if (cl[k] == kDead) continue;
    const unsigned j = (unsigned)pos[k];
    st(dst.cell, j, cl[k]);
    st(dst.off, j, off[k]);
    st(dst.ux, j, ux[k]);
    st(dst.uy, j, uy[k]);
    st(dst.uz, j, uz[k]);
    st(dst.w, j, w[k]);
    if constexpr (OY) st(dst.oy, j, oy[k]);
    if (comp) {
      st(dst.rx, j, rx[k]);
      st(dst.ry, j, ry[k]);
      st(dst.rz, j, rz[k]);
    }
  }
}

template <typename R>
__global__ __launch_bounds__(kSortThreads) void k_sort_scatter(SortArgs<R> p) {
  sort_scatter_block<R>(p, p.blk0 + (int)blockIdx.x);
}

// ---------------------------------------------------------------- test electrons
// Independent electrons in a given monochromatic plane wave travelling along
// +x (the single-particle tests of Section 3): A_y = a_y sin(phi + psi),
// A_z = a_z cos(phi + psi), phi = t - x, E_perp = -dA/dphi, B = (0, -E_z, E_y).
struct TrackArgs {
  double ay, az, psi;
  double dt, t0;
  double eps;
  long long steps, n;
  double* x;
  double* ux;
  double* uy;
  double* uz;
};

// sin and cos of a phase: reduction by the nearest multiple of pi / 2 in
// three parts (Cody and Waite) with fused multiply-adds, the reduced argument
// kept with its rounding error, then the Taylor series on [-pi/4, pi/4] up to
// the terms below a twentieth of an ulp (r^17 and r^16).  At most 0.8 ulp off
// for phases below 1e5 (1.5 without the kept error and the last term).  About
// 40 instructions; the library's sincos takes about 75, of the 285 of a step
// of a tracked electron whose serial chain is the launch's time.  Phases past
// 1e5, where the three parts would not suffice, and non-finite ones go to the
// library.
__device__ __forceinline__ void phase_sincos(double x, double* sn, double* cs) {
  if (!(fabs(x) < 1e5)) {
    sincos(x, sn, cs);
    return;
  }
  const double n = rint(x * 0x1.45f306dc9c883p-1);  // 2 / pi
  const double t = fma(-n, 0x1.921fb54442d18p+0, x);  // exact
  const double r = fma(-n, 0x1.1a62633145c07p-54, t);
  const double lo = fma(-n, -0x1.f1976b7ed8fbcp-110, fma(-n, 0x1.1a62633145c07p-54, t - r));
  const double z = r * r;
  double p = 1.0 / 355687428096000.0;
  p = fma(p, z, -1.0 / 1307674368000.0);
  p = fma(p, z, 1.0 / 6227020800.0);
  p = fma(p, z, -1.0 / 39916800.0);
  p = fma(p, z, 1.0 / 362880.0);
  p = fma(p, z, -1.0 / 5040.0);
  p = fma(p, z, 1.0 / 120.0);
  p = fma(p, z, -1.0 / 6.0);
  const double hz = 0.5 * z;
  const double s = r + fma(z * r, p, fma(-hz, lo, lo));  // sin r + lo cos r
  double q = 1.0 / 20922789888000.0;
  q = fma(q, z, -1.0 / 87178291200.0);
  q = fma(q, z, 1.0 / 479001600.0);
  q = fma(q, z, -1.0 / 3628800.0);
  q = fma(q, z, 1.0 / 40320.0);
  q = fma(q, z, -1.0 / 720.0);
  q = fma(q, z, 1.0 / 24.0);
  // 1 - z / 2 in two parts, so that its rounding does not enter
  const double w = 1.0 - hz;
  const double c = w + fma(z * z, q, fma(-r, lo, (1.0 - w) - hz));
  const int k = (int)n;
  const double a = k & 1 ? c : s, b = k & 1 ? s : c;
  *sn = k & 2 ? -a : a;
  *cs = (k + 1) & 2 ? -b : b;
}

// Fields (and, for the complete force, their partial derivatives) at (x, t)
template <typename R>
__device__ __forceinline__ void wave_at(const TrackArgs& a, double x, double t, R& ey, R& ez,
                                        FieldRates<R>& fr) {
  double sn, cs;
  phase_sincos(t - x + a.psi, &sn, &cs);
  ey = (R)(-a.ay * cs);
  ez = (R)(a.az * sn);
  // dE_perp/dphi = (a_y sin, a_z cos); d/dt = d/dphi, d/dx = -d/dphi
  const R dy = (R)(a.ay * sn), dz = (R)(a.az * cs);
  fr.etx = R(0);
  fr.ety = dy;
  fr.etz = dz;
  fr.bty = -dz;
  fr.btz = dy;
  fr.exx = R(0);
  fr.exy = -dy;
  fr.exz = -dz;
  fr.bxy = dz;
  fr.bxz = -dy;
}

// A tracked electron; FP32 carries the RR increment's rounding residual.
template <typename R>
struct TrackState {
  double x;
  R ux, uy, uz;
  float rx, ry, rz;
};

template <typename R>
__device__ __forceinline__ TrackState<R> track_start(const TrackArgs& a, long long i) {
  return {a.x[i], (R)a.ux[i], (R)a.uy[i], (R)a.uz[i], 0.f, 0.f, 0.f};
}

// Whether an electron was lost to a momentum whose square overflows FP64 (or
// began so): the short roots give NaN there.  It is then tracked again in the
// form that allows for it (ANY), whose selects on the chain of every step
// would take 1.16 ms to 1.29 for 10,000 electrons and 2,000 steps.
template <typename R>
__device__ __forceinline__ bool track_lost(const TrackState<R>& e) {
  return sizeof(R) == 8 && !(e.x == e.x && e.ux == e.ux && e.uy == e.uy && e.uz == e.uz);
}

// The paper's leapfrog scheme: x^n and u^{n-1/2} in, x^{n+steps} and
// u^{n+steps-1/2} out; the position advances in FP64 by dt u_x / gamma.
// MODE: 0 Lorentz only, 1 with f_R of Eq. (f_r), 2 with the complete force.
template <typename R, int MODE, bool ANY>
__device__ __forceinline__ void leapfrog(const TrackArgs& a, TrackState<R>& e) {
  constexpr bool COMP = sizeof(R) == 4 && MODE > 0;
  const R qh = (R)(-0.5 * a.dt), k = (R)(a.eps * a.dt);
  float stiff = 0.f;
  for (long long s = 0; s < a.steps; ++s) {
    R ey, ez;
    FieldRates<R> fr;
    wave_at<R>(a, e.x, a.t0 + (double)s * a.dt, ey, ez, fr);
    MomentumOut<R> o;
    momentum_step<R, (MODE > 0), COMP, (MODE == 2), false, ANY>(e.ux, e.uy, e.uz, R(0), ey, ez, -ez, ey, qh, k, fr,
                                                                e.rx, e.ry, e.rz, stiff, o);
    e.ux = o.nx;
    e.uy = o.ny;
    e.uz = o.nz;
    const double gx = (double)e.ux + e.rx, gy = (double)e.uy + e.ry, gz = (double)e.uz + e.rz;
    const double g2 = 1.0 + gx * gx + gy * gy + gz * gz;
    e.x += a.dt * gx * (ANY ? rsq_any(g2) : rsq(g2));
  }
}

template <typename R, int MODE>
__global__ void k_track_leapfrog(TrackArgs a) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  TrackState<R> e = track_start<R>(a, i);
  leapfrog<R, MODE, false>(a, e);
  if (track_lost(e)) {
    e = track_start<R>(a, i);
    leapfrog<R, MODE, true>(a, e);
  }
  a.x[i] = e.x;
  a.ux[i] = (double)e.ux + e.rx;
  a.uy[i] = (double)e.uy + e.ry;
  a.uz[i] = (double)e.uz + e.rz;
}

template <bool ANY>
__device__ __forceinline__ float inv_gamma(float g2) { return 1.0f / sqrtf(g2); }
template <bool ANY>
__device__ __forceinline__ double inv_gamma(double g2) { return ANY ? rsq_any(g2) : rsq(g2); }

// Right-hand side of Eq. (3dLL) for an electron (MODE 0: Lorentz only; 1:
// plus the non-derivative RR terms; 2: plus the derivative term).
template <typename R, int MODE, bool ANY>
__device__ __forceinline__ void ll_rhs(R ux, R uy, R uz, R ey, R ez, const FieldRates<R>& fr, R eps,
                                       R& fx, R& fy, R& fz) {
  const R by = -ez, bz = ey;
  const R g2 = R(1) + ux * ux + uy * uy + uz * uz;
  const R ig = inv_gamma<ANY>(g2);
  const R vx = ux * ig, vy = uy * ig, vz = uz * ig;
  const R Fx = vy * bz - vz * by, Fy = ey - vx * bz, Fz = ez + vx * by;  // E + v x B (E_x = 0)
  fx = -Fx;
  fy = -Fy;
  fz = -Fz;
  if (MODE > 0) {
    const R vE = vy * ey + vz * ez;
    const R br = g2 * (Fx * Fx + Fy * Fy + Fz * Fz - vE * vE);
    fx += eps * ((Fy * bz - Fz * by) - br * vx);
    fy += eps * (vE * ey - Fx * bz - br * vy);
    fz += eps * (Fx * by + vE * ez - br * vz);
  }
  if (MODE == 2) {
    const R g = g2 * ig;
    const R DEy = fr.ety + vx * fr.exy, DEz = fr.etz + vx * fr.exz;
    const R DBy = fr.bty + vx * fr.bxy, DBz = fr.btz + vx * fr.bxz;
    fx -= eps * g * (vy * DBz - vz * DBy);
    fy -= eps * g * (DEy - vx * DBz);
    fz -= eps * g * (DEz + vx * DBy);
  }
}

// Classical RK4 of (x, u) at the same time, the comparator of Section 3.
template <typename R, int MODE, bool ANY>
__device__ __forceinline__ void rk4_step(const TrackArgs& a, double t, R h, R eps, TrackState<R>& e) {
  auto stage = [&](double xs, double ts, R sx, R sy, R sz, double& dx, R& fx, R& fy, R& fz) {
    R ey, ez;
    FieldRates<R> fr;
    wave_at<R>(a, xs, ts, ey, ez, fr);
    ll_rhs<R, MODE, ANY>(sx, sy, sz, ey, ez, fr, eps, fx, fy, fz);
    dx = (double)sx * inv_gamma<ANY>(1.0 + (double)sx * sx + (double)sy * sy + (double)sz * sz);
  };
  const double x = e.x;
  const R ux = e.ux, uy = e.uy, uz = e.uz;
  double d1, d2, d3, d4;
  R a1, b1, c1, a2, b2, c2, a3, b3, c3, a4, b4, c4;
  stage(x, t, ux, uy, uz, d1, a1, b1, c1);
  stage(x + 0.5 * a.dt * d1, t + 0.5 * a.dt, ux + R(0.5) * h * a1, uy + R(0.5) * h * b1,
        uz + R(0.5) * h * c1, d2, a2, b2, c2);
  stage(x + 0.5 * a.dt * d2, t + 0.5 * a.dt, ux + R(0.5) * h * a2, uy + R(0.5) * h * b2,
        uz + R(0.5) * h * c2, d3, a3, b3, c3);
  stage(x + a.dt * d3, t + a.dt, ux + h * a3, uy + h * b3, uz + h * c3, d4, a4, b4, c4);
  e.x += a.dt / 6.0 * (d1 + 2.0 * d2 + 2.0 * d3 + d4);
  e.ux += h / R(6) * (a1 + R(2) * a2 + R(2) * a3 + a4);
  e.uy += h / R(6) * (b1 + R(2) * b2 + R(2) * b3 + b4);
  e.uz += h / R(6) * (c1 + R(2) * c2 + R(2) * c3 + c4);
}

template <typename R, int MODE>
__global__ void k_track_rk4(TrackArgs a) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  TrackState<R> e = track_start<R>(a, i);
  const R h = (R)a.dt, eps = (R)a.eps;
  for (long long s = 0; s < a.steps; ++s) rk4_step<R, MODE, false>(a, a.t0 + (double)s * a.dt, h, eps, e);
  if (MODE == 0 && track_lost(e)) {  // (with RR no form of an overflowed stage is finite)
    e = track_start<R>(a, i);
    for (long long s = 0; s < a.steps; ++s) rk4_step<R, MODE, true>(a, a.t0 + (double)s * a.dt, h, eps, e);
  }
  a.x[i] = e.x;
  a.ux[i] = e.ux;
  a.uy[i] = e.uy;
  a.uz[i] = e.uz;
}

// ---------------------------------------------------------------- self-check
__device__ __forceinline__ unsigned long long splitmix64(unsigned long long seed,
                                                         unsigned long long i) {
  unsigned long long z = seed + (i + 1ull) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Floats with bit patterns first .. first + count - 1 (those >= 1): count the
// results of sqrt_rn_ge1 and rcp_rn_ge1 (below 2^126) that differ from the
// correctly rounded sqrtf and 1.0f / x; and, for a double of the same leading
// bits with the other 29 drawn from a hash of them, of their FP64 forms that
// differ from sqrt and 1.0 / x.
__global__ void k_check_rounding(unsigned first, unsigned count, unsigned long long* bad) {
  unsigned long long mine = 0;
  const unsigned long long stride = (unsigned long long)gridDim.x * blockDim.x;
  for (unsigned long long k = blockIdx.x * (unsigned long long)blockDim.x + threadIdx.x; k < count; k += stride) {
    const float x = __uint_as_float(first + (unsigned)k);
    if (!(x >= 1.0f) || !(x <= 3.4028235e38f)) continue;
    mine += __float_as_uint(sqrt_rn_ge1(x)) != __float_as_uint(sqrtf(x));
    if (x < 0x1p126f) mine += __float_as_uint(rcp_rn_ge1(x)) != __float_as_uint(1.0f / x);
    const double d = __longlong_as_double(__double_as_longlong((double)x) |
                                          (long long)(splitmix64(0ull, first + k) >> 35));
    mine += __double_as_longlong(sqrt_rn_ge1(d)) != __double_as_longlong(sqrt(d));
    mine += __double_as_longlong(rcp_rn_ge1(d)) != __double_as_longlong(1.0 / d);
  }
  if (mine) atomicAdd(bad, mine);
}

// ---------------------------------------------------------------- batched runs
// One slot per resident run.  Everything a step needs is derived from the
// run's device step counter n: sort due iff n > 0 and n % K == 0, particle
// buffer parity (n / K) & 1 for the push (the sort at step n reads parity
// (n / K - 1) & 1), field and current parity n & 1, laser time from n.  A
// captured sequence of batched launches can therefore be replayed while
// runs join and leave: only the slot table and the work ranges change.
template <typename R>
struct SlotDev {
  PushArgs<R> push[2][2];   // [particle parity][field parity]
  FieldArgs<R> field[2];    // [field parity] (the quantum's last field pass advances the counter itself)
  SortArgs<R> sort[2];      // [source particle parity]
  int* cnt[2];
  int* cur[2];
  long long* count;         // [parity][species]
  long long* step;          // the run's device step counter
  int* done;                // field chunks of the current step finished (zero between steps)
  long long target;         // the run stops once *step reaches target
  int sort_interval;
  int nx;
};

constexpr int kMaxSlots = 1024;
// ints between two slots' done counters: one 128-byte line each, so that the
// counting atomics of different runs do not queue on one line
constexpr int kDoneStride = 32;

// A value the whole wave shares, moved to scalar registers.
__device__ __forceinline__ long long uniform(long long v) {
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)(v & 0xffffffffll));
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)((unsigned long long)v >> 32));
  return (long long)(((unsigned long long)hi << 32) | lo);
}

// Work ranges of the slots, copied to LDS once per work-group; slot(b) is
// the slot whose range [start[s], start[s + 1]) holds work item b.
struct SlotRanges {
  int* st;  // LDS, n + 1 entries
  int n;
  // b is block-uniform, so is the result: readfirstlane lets the compiler
  // keep the slot (and every argument loaded through it) in scalar registers
  __device__ __forceinline__ int slot(int b) const {
    int lo = 0, hi = n;
    while (hi - lo > 1) {
      const int m = (lo + hi) >> 1;
      if (st[m] <= b)
        lo = m;
      else
        hi = m;
    }
    return __builtin_amdgcn_readfirstlane(lo);
  }
  __device__ __forceinline__ int first(int sl) const { return __builtin_amdgcn_readfirstlane(st[sl]); }
  __device__ __forceinline__ int total() const { return __builtin_amdgcn_readfirstlane(st[n]); }
};

__device__ __forceinline__ SlotRanges load_ranges(const int* start, int n, int* lds) {
  for (int i = threadIdx.x; i <= n; i += blockDim.x) lds[i] = start[i];
  __syncthreads();
  return SlotRanges{lds, n};
}

// Batched push and field launches run one work-group per work item: the host
// sets their grids to the resident total whenever the slot table changes (a
// grid-stride loop here would keep more values live and cost occupancy).
template <typename R>
__global__ PIC_PUSH_BOUNDS void k_push_batch(const SlotDev<R>* __restrict__ slots, const int* __restrict__ start, int n) {
  __shared__ __align__(16) unsigned long long lds[kLdsSlots];
  // the slot table and the deposit window share the LDS: every wave reads
  // the table before the barrier below, the window is cleared after it
  static_assert(2 * (kMaxSlots + 1) * sizeof(int) <= sizeof(lds), "slot ranges must fit the window");
  const SlotRanges sr = load_ranges(start, n, reinterpret_cast<int*>(lds));
  const int b = (int)blockIdx.x;
  if (b >= sr.total()) return;  // block-uniform, as are the returns below
  const int sl = sr.slot(b);
  const int tile = b - sr.first(sl);
  __syncthreads();
  const SlotDev<R>& S = constant_ref(slots + sl);
  const long long st = uniform(*S.step);
  if (st >= S.target) return;
  const int pp = (int)((st / S.sort_interval) & 1), fp = (int)(st & 1);
  push_one_tile<R, kBatchPPT, kBatchDepth>(S.push[pp][fp], tile, j_buffer(-1, st), lds);
}

// k_step for every resident run: step q >= 1 of the quantum is pushed after
// step q - 1's fields (24 requests in three groups: 26 us, where the push and
// the field launch took 24.3 + 7.7 us).  The step counters stay put during the quantum (every
// launch computes its step as counter + q) and advance at its end.
template <typename R>
__global__ PIC_PUSH_BOUNDS void k_step_batch(const SlotDev<R>* __restrict__ slots,
                                             const int* __restrict__ push_start,
                                             const int* __restrict__ field_start, int n, int q) {
  __shared__ __align__(16) unsigned long long lds[kLdsSlots];
  int* rp = reinterpret_cast<int*>(lds);
  int* rf = rp + n + 1;
  for (int i = threadIdx.x; i <= n; i += kThreads) {
    rp[i] = push_start[i];
    rf[i] = field_start[i];
  }
  __syncthreads();
  const SlotRanges P{rp, n}, F{rf, n};
  int b = (int)blockIdx.x;
  const bool push = b < P.total();
  if (!push) b -= P.total();
  const SlotRanges& sr = push ? P : F;
  if (b >= sr.total()) return;
  const int sl = sr.slot(b);
  const int item = b - sr.first(sl);
  __syncthreads();  // the tables are read: the LDS is free
  const SlotDev<R>& S = constant_ref(slots + sl);
  const long long st = uniform(*S.step) + q - 1;  // the step whose fields are due
  if (st >= S.target) return;
  const int jr = j_buffer(-1, st);
  if (push) {
    if (st + 1 >= S.target) return;
    const int pp = (int)(((st + 1) / S.sort_interval) & 1), fp = (int)((st + 1) & 1);
    push_one_tile<R, kBatchPPT, kBatchDepth, true>(S.push[pp][fp], item, jr == 2 ? 0 : jr + 1, lds,
                                                   &S.field[st & 1], st, jr);
  } else {
    field_chunk<R, kThreads>(S.field[st & 1], item, st, jr, reinterpret_cast<R*>(lds));
  }
}

// The last field pass of a quantum of q steps also ends it: the last of a
// run's chunks to finish advances the run's step counter (every chunk of the
// run has read the counter before it counts itself done).
template <typename R>
__global__ __launch_bounds__(kFieldChunk) void k_field_batch(const SlotDev<R>* __restrict__ slots,
                                                            const int* __restrict__ start, int n, int q) {
  __shared__ int rng[kMaxSlots + 1];
  __shared__ R sm[field_lds_elems<kFieldChunk>()];
  const SlotRanges sr = load_ranges(start, n, rng);
  const int b = (int)blockIdx.x;
  if (b >= sr.total()) return;
  const int sl = sr.slot(b);
  const SlotDev<R>& S = constant_ref(slots + sl);
  const long long s0 = uniform(*S.step), st = s0 + q - 1;
  if (s0 >= S.target) return;
  if (st < S.target)  // (a run that ends inside the quantum had its last fields advanced before)
    field_chunk<R, kFieldChunk>(S.field[st & 1], b - sr.first(sl), st, j_buffer(-1, st), sm);
  // relaxed: a block's read of the counter has returned (its value chose the
  // buffers) before the block counts itself; acquire/release ordering here
  // would write back and invalidate the L2 once per work-group
  if (threadIdx.x == 0) {
    const int chunks = sr.first(sl + 1) - sr.first(sl);
    if (__hip_atomic_fetch_add(S.done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == chunks - 1) {
      __hip_atomic_store(S.done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      *S.step = s0 + q < S.target ? s0 + q : S.target;
    }
  }
}

template <typename R>
__device__ __forceinline__ bool sort_due(const SlotDev<R>& S, int* q) {
  const long long st = uniform(*S.step);
  if (st >= S.target || st <= 0 || st % S.sort_interval) return false;
  *q = (int)((st / S.sort_interval - 1) & 1);
  return true;
}

template <typename R>
__global__ __launch_bounds__(kSortThreads) void k_sort_hist_batch(const SlotDev<R>* __restrict__ slots,
                                                                 const int* __restrict__ start, int n) {
  __shared__ int rng[kMaxSlots + 1];
  const SlotRanges sr = load_ranges(start, n, rng);
  for (int b = (int)blockIdx.x; b < sr.total(); b += (int)gridDim.x) {
    const int sl = sr.slot(b);
    int q;
    if (!sort_due(slots[sl], &q)) continue;
    sort_hist_block<R>(slots[sl].sort[q], b - sr.first(sl));
  }
}

template <typename R>
__global__ __launch_bounds__(1024) void k_sort_scan_batch(const SlotDev<R>* slots, int n) {
  for (int w = (int)blockIdx.x; w < 2 * n; w += (int)gridDim.x) {
    const int sl = w >> 1, sp = w & 1;
    const SlotDev<R>& S = constant_ref(slots + sl);
    int q;
    if (!sort_due(S, &q)) continue;
    __syncthreads();
    sort_scan_species(S.cnt[sp], S.cur[sp], S.count + 2 * (q ^ 1) + sp, S.nx);
  }
}

template <typename R>
__global__ __launch_bounds__(kSortThreads) void k_sort_scatter_batch(const SlotDev<R>* __restrict__ slots,
                                                                    const int* __restrict__ start, int n) {
  __shared__ int rng[kMaxSlots + 1];
  const SlotRanges sr = load_ranges(start, n, rng);
  for (int b = (int)blockIdx.x; b < sr.total(); b += (int)gridDim.x) {
    const int sl = sr.slot(b);
    int q;
    if (!sort_due(slots[sl], &q)) continue;
    sort_scatter_block<R>(slots[sl].sort[q], b - sr.first(sl));
  }
}

// ---------------------------------------------------------------- persistent batched steps
// Grid-wide barrier for a launch whose work-groups are all resident at once
// (the host sizes the grid from the kernel's occupancy).  Arrivals count in
// kBarGroups group words and then in one top word, so that no word takes
// more than about G / kBarGroups same-address atomics; the last arrival
// bumps the generation word that the others poll.  A wait longer than
// `ticks` of the 100 MHz constant clock (one second in use) sets *err, and
// once *err is set every wait ends at once: a launch always finishes, and
// the host reports the error.  Words sit 128 bytes apart: [0] generation,
// [32] top, [64 + 32 g] group g.
constexpr int kBarGroups = 16;
constexpr int kBarWords = 32 * (2 + kBarGroups);
constexpr unsigned long long kBarTicks = 100000000ull;  // one second

__device__ __forceinline__ void grid_sync(unsigned* w, int* err, unsigned long long ticks) {
  // every wave's loads and stores complete, then one agent-scope release per
  // work-group (an L2 write-back), relaxed counting and polling, and one
  // acquire after the wait (polling with acquire loads would invalidate the
  // caches on every poll, under the work-groups still running)
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    const unsigned G = gridDim.x, g = blockIdx.x % kBarGroups;
    const unsigned in_g = (G - 1 - g) / kBarGroups + 1;  // blocks b < G with b % kBarGroups == g
    const unsigned groups = G < (unsigned)kBarGroups ? G : (unsigned)kBarGroups;
    unsigned* gen = w;
    const unsigned cur = __hip_atomic_load(gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bool last = false;
    unsigned* gw = w + 64 + 32 * g;
    // the last arrival of a group and the last overall pass the others'
    // releases on (acquire, then release, through a fence each)
    if (__hip_atomic_fetch_add(gw, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == in_g - 1) {
      __hip_atomic_store(gw, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
      if (__hip_atomic_fetch_add(w + 32, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == groups - 1) {
        __hip_atomic_store(w + 32, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
        __hip_atomic_fetch_add(gen, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = true;
      }
    }
    if (!last) {
      const unsigned long long t0 = wall_clock64();
      while (__hip_atomic_load(gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == cur) {
        if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
        if (wall_clock64() - t0 > ticks) {
          __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  __syncthreads();
}

// Slots a persistent launch serves (its range tables live in LDS beside the
// push window, and more of them would cost the push a work-group per CU).
constexpr int kPersistSlots = 128;

// `steps` batched steps in one launch: every work-group takes push tiles of
// all resident runs in turn, then field chunks of kThreads nodes, with a
// grid-wide barrier after each pass.  A run's step counter stays put during
// the launch (every pass computes its step as counter + k) and advances once
// at the end, by the number of steps the run had left, at most `steps`.
template <typename R>
__global__ __launch_bounds__(kThreads, PIC_STEPS_MIN_WAVES) void k_steps_batch(const SlotDev<R>* __restrict__ slots,
                                              const int* __restrict__ push_start,
                                              const int* __restrict__ field_start, int n, int steps,
                                              unsigned* bar, int* err, unsigned long long ticks) {
  __shared__ __align__(16) unsigned long long lds[kLdsSlots];
  __shared__ int rp[kPersistSlots + 1], rf[kPersistSlots + 1];
  static_assert(field_lds_elems<kThreads>() * sizeof(double) <= sizeof(lds), "field chunk must fit the window");
  for (int i = threadIdx.x; i <= n; i += blockDim.x) {
    rp[i] = push_start[i];
    rf[i] = field_start[i];
  }
  __syncthreads();
  const SlotRanges P{rp, n}, F{rf, n};
  const int G = (int)gridDim.x;
  for (int k = 0; k < steps; ++k) {
    for (int b = (int)blockIdx.x; b < P.total(); b += G) {
      const int sl = P.slot(b);
      const SlotDev<R>& S = constant_ref(slots + sl);
      const long long st = uniform(*S.step) + k;
      if (st >= S.target) continue;
      const int pp = (int)((st / S.sort_interval) & 1), fp = (int)(st & 1);
      __syncthreads();  // the block's previous tile is out of the window
      push_one_tile<R, kBatchPPT, kBatchDepth>(S.push[pp][fp], b - P.first(sl), j_buffer(-1, st), lds);
    }
    grid_sync(bar, err, ticks);
    for (int b = (int)blockIdx.x; b < F.total(); b += G) {
      const int sl = F.slot(b);
      const SlotDev<R>& S = constant_ref(slots + sl);
      const long long st = uniform(*S.step) + k;
      if (st >= S.target) continue;
      __syncthreads();
      field_chunk<R, kThreads>(S.field[st & 1], b - F.first(sl), st, j_buffer(-1, st), reinterpret_cast<R*>(lds));
    }
    grid_sync(bar, err, ticks);
  }
  // every work-group has read the counters before the last barrier
  if (blockIdx.x == 0) {
    for (int sl = threadIdx.x; sl < n; sl += blockDim.x) {
      long long* p = slots[sl].step;
      const long long v = *p, t = slots[sl].target;
      if (v < t) *p = v + steps < t ? v + steps : t;
    }
  }
}

// ---------------------------------------------------------------- init
template <typename R>
__global__ void k_init(SpeciesDev<R> e, SpeciesDev<R> ion, long long n, int c0, int ppc,
                       unsigned long long seed, double jitter, R w) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int k = (int)(i % ppc);
  const R U = (R)(splitmix64(seed, (unsigned long long)i) >> 40) * R(1.0 / 16777216.0);
  R o = ((R)k + R(0.5) + (R)jitter * (U - R(0.5))) / (R)ppc;
  if (!(o < R(1))) o = R(0);
  const int c = c0 + (int)(i / ppc);
  SpeciesDev<R> sp[2] = {e, ion};
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    sp[s].cell[i] = c;
    sp[s].off[i] = o;
    sp[s].ux[i] = R(0);
    sp[s].uy[i] = R(0);
    sp[s].uz[i] = R(0);
    sp[s].w[i] = w;
    if (sp[s].rx) {
      sp[s].rx[i] = 0.f;
      sp[s].ry[i] = 0.f;
      sp[s].rz[i] = 0.f;
    }
  }
}

// ---------------------------------------------------------------- diagnostics
constexpr int kDiagThreads = 256;
constexpr int kDiagPartBlocks = 512;   // per species, kinetic energy partials
constexpr int kDiagFieldBlocks = 256;

template <typename R>
struct DiagArgs {
  SpeciesDev<R> sp[2];
  const long long* count;
  FieldsDev<R> f;
  const long long* Ex_int;
  long long* rho;        // [n + 3] integer charge on nodes (index node + 1): zero on entry, zeroed again
  double* part;          // partials: [2][kDiagPartBlocks] kinetic, [7][kDiagFieldBlocks]: fields (3),
                         // tile accumulators (4)
  long long* ipart;      // [kDiagFieldBlocks] gauss max, [2][kDiagPartBlocks] alive counts
  const double* acc;     // [tiles][4] the push's tile accumulators
  int tiles;
  int nx;
  double mass[2];
  int Z[2];
  R sw;
  double dx;
};

__device__ __forceinline__ double block_sum(double v, double* sh) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  v = wave_sum(v);
  __syncthreads();
  if (lane == 0) sh[wid] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += sh[w];
  return t;
}

// LDS slots of the integer charge of a diagnostics tile
constexpr int kDiagSlots = kSortWin + 1;

// Sums of N doubles over the work-group, each in a fixed order; the results
// are valid on thread 0.  sh holds N * (blockDim.x / 64) doubles.
template <int N>
__device__ __forceinline__ void block_sums(double (&v)[N], double* sh) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = wave_sum(v[k]);
  __syncthreads();
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < N; ++k) sh[k * nw + wid] = v[k];
  __syncthreads();
  if (threadIdx.x == 0)
#pragma unroll
    for (int k = 0; k < N; ++k) {
      v[k] = 0.0;
      for (int w = 0; w < nw; ++w) v[k] += sh[k * nw + w];
    }
}

// Kinetic energy (FP64) and integer charge of the particles.  Each block
// walks sort-sized tiles (blocks of a species stride over its tiles in a
// fixed order); the charge of a tile is gathered in an LDS window, in up to
// 16 private copies per node at an odd stride (as the push does: a dense
// tile's lanes share a cell), and added to HBM with one atomic per node.
// A tile's values are loaded together with its cells.  Bound by the latency
// of one tile for small runs (12,800 heated particles: 8.0 us, 28 us with one
// leader round per distinct cell of a wave) and by HBM for large ones (1e8
// particles, 24 B of each: 520 us, before 725).
template <typename R>
__global__ __launch_bounds__(kDiagThreads) void k_diag_particles(DiagArgs<R> p) {
  static_assert(kDiagThreads == kSortThreads, "diag tiles reuse the sort tiling");
  __shared__ double sh[kDiagThreads / 64];
  __shared__ long long sa[kDiagThreads / 64];
  __shared__ unsigned long long rw[kDiagSlots];
  __shared__ int sm[8];
  const int s = blockIdx.x < kDiagPartBlocks ? 0 : 1;
  const int b = blockIdx.x - s * kDiagPartBlocks;
  const long long n = p.count[s];
  const SpeciesDev<R> sp = p.sp[s];
  const int lane = threadIdx.x & 63;
  double ke = 0.0;
  long long alive = 0;
  for (long long base = (long long)b * kSortTile; base < n;
       base += (long long)kDiagPartBlocks * kSortTile) {
    int cl[kSortPPT];
    R off[kSortPPT], ux[kSortPPT], uy[kSortPPT], uz[kSortPPT], w[kSortPPT];
#pragma unroll
    for (int k = 0; k < kSortPPT; ++k) {
      const long long i = base + k * kSortThreads + threadIdx.x;
      const unsigned ui = (unsigned)(i < n ? i : n - 1);
      cl[k] = ld(sp.cell, ui);
      if (i >= n) cl[k] = kDead;
      off[k] = ld(sp.off, ui);
      ux[k] = ld(sp.ux, ui);
      uy[k] = ld(sp.uy, ui);
      uz[k] = ld(sp.uz, ui);
      w[k] = ld(sp.w, ui);
    }
    int lo, hi;
    tile_range(cl, lo, hi, sm);
    if (lo > hi) continue;  // block-uniform
    const int W = hi - lo + 2;  // nodes lo .. hi + 1
    int csh = 4;
    while (csh > 0 && W * ((1 << csh) + 1) > kDiagSlots) --csh;
    const int P = csh ? (1 << csh) + 1 : 1, copy = lane & ((1 << csh) - 1);
    const bool win = W * P <= kDiagSlots;
    if (win) {
      for (int e = threadIdx.x; e < W * P; e += kSortThreads) rw[e] = 0ull;
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < kSortPPT; ++k) {
      const int c = cl[k];
      if (c == kDead) continue;
      const double vx = ux[k], vy = uy[k], vz = uz[k];
      const double g = sqrt(1.0 + vx * vx + vy * vy + vz * vz);
      ke += (double)w[k] * p.mass[s] * (g - 1.0);
      const int q = (int)(off[k] * R(kTwo24));
      const int qw = p.Z[s] * (int)rint(w[k] * p.sw);
      const long long r0 = (long long)qw * (kTwo24 - q), r1 = (long long)qw * q;
      alive += 1;
      if (win) {
        unsigned long long* x = rw + (c - lo) * P + copy;
        atomicAdd(x, (unsigned long long)r0);
        atomicAdd(x + P, (unsigned long long)r1);
      } else {
        atomicAdd((unsigned long long*)p.rho + c + 1, (unsigned long long)r0);
        atomicAdd((unsigned long long*)p.rho + c + 2, (unsigned long long)r1);
      }
    }
    if (win) {
      __syncthreads();
      for (int e = threadIdx.x; e < W; e += kSortThreads) {
        unsigned long long v = 0ull;
        for (int k = 0; k < 1 << csh; ++k) v += rw[e * P + k];
        if (v) atomicAdd((unsigned long long*)p.rho + lo + e + 1, v);
      }
      __syncthreads();
    }
  }
  const double t = block_sum(ke, sh);
  const long long na = wave_sum((long long)alive);
  if (lane == 0) sa[threadIdx.x >> 6] = na;
  __syncthreads();
  if (threadIdx.x == 0) {
    long long tot = 0;
    for (int w = 0; w < kDiagThreads / 64; ++w) tot += sa[w];
    p.part[s * kDiagPartBlocks + b] = t;
    p.ipart[kDiagFieldBlocks + s * kDiagPartBlocks + b] = tot;
  }
}

// Field energies, the Gauss residual, this block's share of the push's tile
// accumulators (a fixed set of tiles per thread), and the charge cleared for
// the next diagnostics.
template <typename R>
__global__ __launch_bounds__(kDiagThreads) void k_diag_fields(DiagArgs<R> p) {
  __shared__ double sh[7 * (kDiagThreads / 64)];
  __shared__ long long sm[kDiagThreads / 64];
  const int n = p.nx;
  double v[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};  // U_Ex, U_Et, U_B; tile accumulators
  long long gmax = 0;
  for (int i = blockIdx.x * kDiagThreads + threadIdx.x; i <= n;
       i += kDiagFieldBlocks * kDiagThreads) {
    const double wn = (i == 0 || i == n) ? 0.5 : 1.0;
    const NodeF<R> nv = p.f.N[i];
    const double ey = nv.ey, ez = nv.ez;
    v[1] += wn * (ey * ey + ez * ez);
    if (i >= 1) {  // half-node h = i covers cell i-1
      const HalfF<R> hv = p.f.H[i];
      const double ex = hv.ex, by = hv.by, bz = hv.bz;
      v[0] += ex * ex;
      v[2] += by * by + bz * bz;
    }
    if (i >= 1 && i <= n - 1) {
      long long r = p.Ex_int[i + 1] - p.Ex_int[i] - p.rho[i + 1];
      r = r < 0 ? -r : r;
      gmax = r > gmax ? r : gmax;
    }
    p.rho[i + 1] = 0;
  }
#pragma unroll 4
  for (int t = blockIdx.x * kDiagThreads + threadIdx.x; t < p.tiles;
       t += kDiagFieldBlocks * kDiagThreads) {
#pragma unroll
    for (int k = 0; k < 4; ++k) v[3 + k] += p.acc[4 * (size_t)t + k];
  }
  long long g = gmax;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const long long x = __shfl_xor(g, o);
    g = x > g ? x : g;
  }
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = g;
  block_sums<7>(v, sh);
  if (threadIdx.x == 0) {
    long long m = 0;
    for (int w = 0; w < kDiagThreads / 64; ++w) m = sm[w] > m ? sm[w] : m;
    double* part = p.part + 2 * kDiagPartBlocks + blockIdx.x;
#pragma unroll
    for (int k = 0; k < 7; ++k) part[k * kDiagFieldBlocks] = k < 3 ? 0.5 * p.dx * v[k] : v[k];
    p.ipart[blockIdx.x] = m;
  }
}

// Final reduction in fixed order into the diagnostics record, with the
// run's boundary budget, flags and step counter, so that one copy brings
// everything to the host.
struct DiagOutDev {
  double U_Ex, U_Et, U_B, K_e, K_i, E_rad, E_esc, n_stiff;
  double budget[3];  // E_in, E_out_left, E_out_right
  long long gauss_int, alive0, alive1, step;
  int nonfinite;
};

// One work-group; every partial is loaded before the first sum, so the
// launch is one memory latency and one reduction: 5.5 us (thread 0 adding
// the counts one after the other, and an LDS tree per sum: 38 us, and 358 us
// with the 98,000 tile accumulators of 1e8 particles, now summed above).
__global__ __launch_bounds__(kDiagThreads) void k_diag_final(const double* part, const long long* ipart,
                                                             const double* budget, const int* flags,
                                                             const long long* step, DiagOutDev* out) {
  static_assert(kDiagPartBlocks == 2 * kDiagThreads && kDiagFieldBlocks == kDiagThreads,
                "one or two partials per thread");
  constexpr int T = kDiagThreads, NW = T / 64;
  __shared__ double sh[9 * NW];
  __shared__ long long si[3][NW];
  const int t = threadIdx.x;
  double v[9];
  v[0] = part[t] + part[T + t];
  v[1] = part[2 * T + t] + part[3 * T + t];
#pragma unroll
  for (int k = 0; k < 7; ++k) v[2 + k] = part[(4 + k) * T + t];
  long long a0 = ipart[T + t] + ipart[2 * T + t], a1 = ipart[3 * T + t] + ipart[4 * T + t], g = ipart[t];
  a0 = wave_sum(a0);
  a1 = wave_sum(a1);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const long long x = __shfl_xor(g, o);
    g = x > g ? x : g;
  }
  if ((t & 63) == 0) {
    si[0][t >> 6] = a0;
    si[1][t >> 6] = a1;
    si[2][t >> 6] = g;
  }
  block_sums<9>(v, sh);
  if (t == 0) {
    DiagOutDev o{};
    o.K_e = v[0];
    o.K_i = v[1];
    o.U_Ex = v[2];
    o.U_Et = v[3];
    o.U_B = v[4];
    o.E_rad = v[5];
    o.E_esc = v[6] + v[7];
    o.n_stiff = v[8];
    for (int w = 0; w < NW; ++w) {
      o.alive0 += si[0][w];
      o.alive1 += si[1][w];
      o.gauss_int = si[2][w] > o.gauss_int ? si[2][w] : o.gauss_int;
    }
    for (int k = 0; k < 3; ++k) o.budget[k] = budget[k];
    o.step = *step;
    o.nonfinite = flags[0];
    *out = o;
  }
}

// ---------------------------------------------------------------- histograms
// A histogram of up to kHistBins bins is gathered in LDS, in 2^csh private
// copies per bin side by side (lane & (copies - 1) picks one), and a
// work-group adds its non-zero bins to HBM once.  Cold or bunched particles
// fall into a few bins, and one global atomic per particle then queues on a
// few addresses: 12 ns per proton (600 ms for 5e7 cold ones; in this form
// 0.17 ms, the time of streaming 20 B each).  The friction histogram of
// 1e6 electrons went from 2.60 ms to 46 us, the spectrum of 1e6 bunched
// protons from 2.05 ms to 27 us.  Histograms that do not fit keep global atomics, with one
// add for a wave whose lanes all hit the same bin.
constexpr int kHistThreads = 512;
constexpr int kHistSlots = 4096;   // 8-byte LDS slots: 32 KB, four work-groups per CU
constexpr int kHistBins = kHistSlots;
constexpr int kHistBlocks = 1024;  // four per CU; each flushes at most `bins` atomics

// log2 of the copies per bin of a histogram of `bins` bins in LDS
__host__ __device__ constexpr int hist_copies_log2(int bins) {
  int csh = 0;
  while (csh < 3 && (bins << (csh + 1)) <= kHistSlots) ++csh;
  return csh;
}

// ---------------------------------------------------------------- spectrum
template <typename R>
__global__ __launch_bounds__(kHistThreads) void k_spectrum(SpeciesDev<R> sp, const long long* count,
                                                           unsigned long long* hist, int bins,
                                                           double e_max, double mc2, R sw) {
  __shared__ unsigned long long sh[kHistSlots];
  const bool lds = bins <= kHistBins;
  const int csh = lds ? hist_copies_log2(bins) : 0, lane = threadIdx.x & 63;
  const int copy = lane & ((1 << csh) - 1);
  if (lds) {
    for (int e = threadIdx.x; e < bins << csh; e += kHistThreads) sh[e] = 0ull;
    __syncthreads();
  }
  const long long n = *count;
  for (long long i = (long long)blockIdx.x * kHistThreads + threadIdx.x; i < n;
       i += (long long)gridDim.x * kHistThreads) {
    const int c = sp.cell[i];
    const double ux = sp.ux[i], uy = sp.uy[i], uz = sp.uz[i];
    const int qw = (int)rint(sp.w[i] * sw);
    const double E = (sqrt(1.0 + ux * ux + uy * uy + uz * uz) - 1.0) * mc2;
    const long long b = (long long)floor(E / e_max * bins);
    const bool in = c != kDead && b >= 0 && b < bins;
    if (lds) {
      if (in) atomicAdd(sh + (((int)b << csh) | copy), (unsigned long long)(long long)qw);
    } else if (in) {
      // lanes of the wave's first bin together, the others one by one
      const int b0 = __builtin_amdgcn_readfirstlane((int)b), q0 = __builtin_amdgcn_readfirstlane(qw);
      const unsigned long long same = __ballot((int)b == b0 && qw == q0);
      if (!((same >> lane) & 1ull))
        atomicAdd(hist + b, (unsigned long long)(long long)qw);
      else if (lane == __ffsll((long long)same) - 1)
        atomicAdd(hist + b, (unsigned long long)((long long)qw * __popcll(same)));
    }
  }
  if (!lds) return;
  __syncthreads();
  for (int e = threadIdx.x; e < bins; e += kHistThreads) {
    unsigned long long v = 0ull;
    for (int k = 0; k < 1 << csh; ++k) v += sh[(e << csh) | k];
    if (v) atomicAdd(hist + e, v);
  }
}

// ---------------------------------------------------------------- friction coefficient
// The friction coefficient d of Eq. (damping) of every electron at the
// current step: d = eps gamma^2 [f_L^2 - (v.f_L)^2], f_L = -(E + v x B), with
// E^n, B^n gathered at x^n by the push's linear weights and v from the stored
// momentum; FP64 throughout.  Each electron adds its weight (FP64) to bin
// floor((log10 d - lo) / (hi - lo) bins), or to the under (d <= 0 or below
// lo) or over slot; a block's maximum of d and sums of w d and w go out with
// one atomic each.  out[bins + 0]: under, [+1]: over, [+2]: max d (bits: d >= 0
// orders as an integer), [+3]: sum of w d, [+4]: sum of w.
template <typename R>
__global__ __launch_bounds__(kHistThreads) void k_friction(SpeciesDev<R> sp, FieldsDev<R> f,
                                                           const long long* count, double* out,
                                                           int bins, double lo, double hi, double eps) {
  __shared__ double sh[kHistSlots];  // bins, under and over, in copies
  __shared__ double s_red[3][kHistThreads / kLanes];
  const int slots = bins + 2;
  const bool lds = slots <= kHistBins;
  const int csh = lds ? hist_copies_log2(slots) : 0, lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int copy = lane & ((1 << csh) - 1);
  if (lds) {
    for (int e = threadIdx.x; e < slots << csh; e += kHistThreads) sh[e] = 0.0;
    __syncthreads();
  }
  const long long n = *count;
  double dmax = 0.0, wd = 0.0, ws = 0.0;
  for (long long i = (long long)blockIdx.x * kHistThreads + threadIdx.x; i < n;
       i += (long long)gridDim.x * kHistThreads) {
    const int c = sp.cell[i];
    if (c == kDead) continue;
    const double o = sp.off[i], on = 1.0 - o;
    const NodeF<R> n0 = f.N[c], n1 = f.N[c + 1];
    const double ey = on * (double)n0.ey + o * (double)n1.ey;
    const double ez = on * (double)n0.ez + o * (double)n1.ez;
    const double sx = o + 0.5;
    const int hb = sx >= 1.0;
    const double fh = hb ? sx - 1.0 : sx, fn = 1.0 - fh;
    const HalfF<R> h0 = f.H[c + hb], h1 = f.H[c + hb + 1];
    const double ex = fn * (double)h0.ex + fh * (double)h1.ex;
    const double by = fn * (double)h0.by + fh * (double)h1.by;
    const double bz = fn * (double)h0.bz + fh * (double)h1.bz;
    const double ux = sp.ux[i], uy = sp.uy[i], uz = sp.uz[i];
    const double g2 = 1.0 + ux * ux + uy * uy + uz * uz, g = sqrt(g2);
    const double vx = ux / g, vy = uy / g, vz = uz / g;
    // f_L = -(E + v x B), B = (0, by, bz)
    const double fx = -(ex + (vy * bz - vz * by));
    const double fy = -(ey - vx * bz);
    const double fz = -(ez + vx * by);
    const double vf = vx * fx + vy * fy + vz * fz;
    const double d = eps * g2 * ((fx * fx + fy * fy + fz * fz) - vf * vf);
    const double w = sp.w[i];
    const double l = d > 0.0 ? log10(d) : -INFINITY;
    long long b = l < lo ? -1 : (l >= hi ? bins : (long long)floor((l - lo) / (hi - lo) * bins));
    if (b >= bins) b = l >= hi ? bins : bins - 1;  // l just below hi
    const int slot = (int)(b < 0 ? bins : (b >= bins ? bins + 1 : b));
    if (lds)
      unsafeAtomicAdd(sh + ((slot << csh) | copy), w);
    else
      unsafeAtomicAdd(out + slot, w);
    if (d > dmax) dmax = d;
    wd += w * d;
    ws += w;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) dmax = fmax(dmax, __shfl_xor(dmax, o));
  wd = wave_sum(wd);
  ws = wave_sum(ws);
  if (lane == 0) {
    s_red[0][wid] = dmax;
    s_red[1][wid] = wd;
    s_red[2][wid] = ws;
  }
  __syncthreads();
  if (lds) {
    for (int e = threadIdx.x; e < slots; e += kHistThreads) {
      double v = 0.0;
      for (int k = 0; k < 1 << csh; ++k) v += sh[(e << csh) | k];
      if (v != 0.0) unsafeAtomicAdd(out + e, v);
    }
  }
  if (threadIdx.x == 0) {
    for (int k = 1; k < kHistThreads / kLanes; ++k) {
      dmax = fmax(dmax, s_red[0][k]);
      wd += s_red[1][k];
      ws += s_red[2][k];
    }
    atomicMax(reinterpret_cast<unsigned long long*>(out + bins + 2),
              (unsigned long long)__double_as_longlong(dmax));
    unsafeAtomicAdd(out + bins + 3, wd);
    unsafeAtomicAdd(out + bins + 4, ws);
  }
}

}  // namespace pic
