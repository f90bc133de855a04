// jdob_common.h — constants and device helpers shared by the kernels of
// libjdob.so (jdob.hip: users sharing their parameters; jdob_hetero.hip:
// heterogeneous users), and the entry of the heterogeneous path.
#ifndef JDOB_COMMON_H
#define JDOB_COMMON_H

#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include "jdob.h"

namespace jdob_dev {

constexpr int WAVE = 64;
constexpr int64_t MAX_BLOCKS_PER_LAUNCH = int64_t(1) << 24;
constexpr int LDS_LIMIT = 64 * 1024;
constexpr int LDS_PER_CU = 160 * 1024;  // gfx950

__host__ __device__ inline int align8(int x) { return (x + 7) & ~7; }

template <typename T> __device__ inline T inf_of() { return T(INFINITY); }

// Four consecutive row entries, read by one LDS instruction (all lanes read
// the same address: a broadcast).
template <typename T> struct alignas(4 * sizeof(T)) Quad { T v[4]; };

// Local latency and energy of one CPU level (Eqs. (1), (2)), read together.
template <typename T> struct alignas(2 * sizeof(T)) Level { T t, e; };

// What a candidate of batch size b needs from row s, read together: the
// batch deadline lo[b] (Eq. (10)), the largest upload latency of the batch
// up[b-1] (Eq. (3)), EU[b] + SL[b] (upload energy of the batch, Eq. (4), plus
// local energy of the others) and A[s] + B[s]*b (batch latency at the top
// GPU level, Eq. (5)).
template <typename T> struct alignas(4 * sizeof(T)) Batch { T lo, upl, esl, ab; };

// A barrier for LDS that one wave shares among its lanes.  WS: the
// workgroup holds other waves, each with LDS of its own, which need not wait
// (LDS instructions of a wave take effect in program order, so ordering the
// compiler's code is enough); otherwise the workgroup's barrier.
template <bool WS> __device__ inline void lds_sync() {
  if constexpr (WS) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// The sums of a layer chain in the sequential order of the ABI contract:
// C[0] = 0, C[q+1] = C[q] + cyc[q] (q = 0..L-1) and, when A is given,
// A[L] = 0, A[q] = A[q+1] + alpha[q] and B likewise (q = L-1..0).  The alpha
// and beta rows arrive reversed (ra[i] = alpha[L-1-i], rb[i] = beta[L-1-i]),
// so that lane 0 (cycles), lane 1 (alpha) and lane 2 (beta) all run their
// chains forward, four terms per trip at immediate offsets; lanes 1 and 2
// keep their running sums in place (ra[i] = A[L-1-i]), which are then
// copied out in layer order.  Every lane returns after a barrier.
template <typename T, bool WS = false>
__device__ inline void chain_sums(const T *cyc, T *ra, T *rb, T *C, T *A, T *B, int L,
                                  int lane) {
  if (lane < (A ? 3 : 1)) {
    const T *src = lane == 0 ? cyc : (lane == 1 ? ra : rb);
    T *dst = lane == 0 ? C + 1 : (lane == 1 ? ra : rb);
    T run = T(0);
    int q = 0;
    for (; q + 4 <= L; q += 4) {
      const T x0 = src[q], x1 = src[q + 1], x2 = src[q + 2], x3 = src[q + 3];
      run = run + x0;
      dst[q] = run;
      run = run + x1;
      dst[q + 1] = run;
      run = run + x2;
      dst[q + 2] = run;
      run = run + x3;
      dst[q + 3] = run;
    }
    for (; q < L; ++q) {
      run = run + src[q];
      dst[q] = run;
    }
    if (lane == 0) C[0] = T(0);
  }
  lds_sync<WS>();
  if (A) {
    for (int q = lane; q <= L; q += WAVE) {
      A[q] = q < L ? ra[L - 1 - q] : T(0);
      B[q] = q < L ? rb[L - 1 - q] : T(0);
    }
    lds_sync<WS>();
  }
}

// Lexicographic (energy, flat index) order: the lower energy wins, equal
// energies go to the lower index.
template <typename T>
__device__ inline bool better(T e1, int i1, T e2, int i2) {
  return (e1 < e2) || (e1 == e2 && i1 < i2);
}

// Lane moves by DPP (data-parallel primitives of the VALU, no LDS round
// trip): row_shr:n inside each row of 16 lanes, row_bcast:15 and
// row_bcast:31 across rows.  Lanes without a source, and rows outside
// RMASK, receive `id`.
template <int CTRL, int RMASK> __device__ inline int dpp_mov(int id, int v) {
  return __builtin_amdgcn_update_dpp(id, v, CTRL, RMASK, 0xf, false);
}
template <int CTRL, int RMASK> __device__ inline float dpp_mov(float id, float v) {
  return __int_as_float(dpp_mov<CTRL, RMASK>(__float_as_int(id), __float_as_int(v)));
}
template <int CTRL, int RMASK> __device__ inline double dpp_mov(double id, double v) {
  const long long qi = __double_as_longlong(id), qv = __double_as_longlong(v);
  const int lo = dpp_mov<CTRL, RMASK>((int)(qi & 0xffffffff), (int)(qv & 0xffffffff));
  const int hi = dpp_mov<CTRL, RMASK>((int)(qi >> 32), (int)(qv >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Inclusive scan over the 64 lanes with an associative, commutative op
// (identity id): Hillis-Steele inside each row of 16, then the row totals.
template <typename V, typename OP> __device__ inline V wave_iscan(V v, V id, OP op) {
  v = op(v, dpp_mov<0x111, 0xf>(id, v));  // row_shr:1
  v = op(v, dpp_mov<0x112, 0xf>(id, v));  // row_shr:2
  v = op(v, dpp_mov<0x114, 0xf>(id, v));  // row_shr:4
  v = op(v, dpp_mov<0x118, 0xf>(id, v));  // row_shr:8
  v = op(v, dpp_mov<0x142, 0xa>(id, v));  // row_bcast:15 into rows 1, 3
  v = op(v, dpp_mov<0x143, 0xc>(id, v));  // row_bcast:31 into rows 2, 3
  return v;
}

__device__ inline int lane_read(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ inline float lane_read(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ inline double lane_read(double v, int l) {
  const long long q = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(q & 0xffffffff), l);
  const int hi = __builtin_amdgcn_readlane((int)(q >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// An associative, commutative op over each aligned run of 2^lg lanes; every
// lane of the run gets the result (lg is wave-uniform).  Inside a row of 16
// by DPP: quad permutes, then mirrors of the half row and the row (all lanes
// of a half already agree).
template <typename V, typename OP> __device__ inline V run_reduce(V v, int lg, OP op) {
  if (lg >= 1) v = op(v, dpp_mov<0xB1, 0xf>(v, v));   // quad_perm [1,0,3,2]
  if (lg >= 2) v = op(v, dpp_mov<0x4E, 0xf>(v, v));   // quad_perm [2,3,0,1]
  if (lg >= 3) v = op(v, dpp_mov<0x141, 0xf>(v, v));  // row_half_mirror
  if (lg >= 4) v = op(v, dpp_mov<0x140, 0xf>(v, v));  // row_mirror
  if (lg >= 5) v = op(v, __shfl_xor(v, 16, WAVE));
  if (lg >= 6) v = op(v, __shfl_xor(v, 32, WAVE));
  return v;
}

// The lane before's value, zero in lane 0 (DPP wave_shr:1).
__device__ inline float lane_before(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ inline double lane_before(double v) {
  const long long q = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(q & 0xffffffff), 0x138, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(q >> 32), 0x138, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Three chains of L <= 64 terms, one term per lane (zero past the last), as
// running sums in lane order: run[l] = run[l-1] + x[l], the additions of a
// sequential sum.  Lane l is final after l steps and stays so.  One addition
// per step and chain, no LDS (the LDS form, chain_sums, takes 1,500 cycles at
// L = 16, this one 500).
template <typename T> __device__ inline void lane_chains(T &a, T &b, T &c, int L) {
  const T x = a, y = b, z = c;
  for (int l = 1; l < L; ++l) {
    a = lane_before(a) + x;
    b = lane_before(b) + y;
    c = lane_before(c) + z;
  }
}

// Lowest (energy, index) of the wave, lexicographically; every lane gets it.
template <typename T>
__device__ inline void wave_argmin(T &e, int &idx) {
#define JDOB_ARGMIN_STEP(CTRL, RMASK)                                  \
  {                                                                   \
    const T oe = dpp_mov<CTRL, RMASK>(inf_of<T>(), e);                \
    const int oi = dpp_mov<CTRL, RMASK>(0x7fffffff, idx);             \
    const bool tk = better(oe, oi, e, idx);                           \
    e = tk ? oe : e;                                                  \
    idx = tk ? oi : idx;                                              \
  }
  JDOB_ARGMIN_STEP(0x111, 0xf);
  JDOB_ARGMIN_STEP(0x112, 0xf);
  JDOB_ARGMIN_STEP(0x114, 0xf);
  JDOB_ARGMIN_STEP(0x118, 0xf);
  JDOB_ARGMIN_STEP(0x142, 0xa);
  JDOB_ARGMIN_STEP(0x143, 0xc);
#undef JDOB_ARGMIN_STEP
  e = lane_read(e, WAVE - 1);
  idx = lane_read(idx, WAVE - 1);
}

__device__ inline int wave_max_int(int v) {
  v = wave_iscan(v, (int)0x80000000, [](int a, int b) { return a > b ? a : b; });
  return lane_read(v, WAVE - 1);
}

// Sum over the wave of non-negative values below 2^31.
__device__ inline int64_t wave_sum_i64(int v) {
  auto add = [](int a, int b) { return a + b; };
  const int lo = lane_read(wave_iscan(v & 0xffff, 0, add), WAVE - 1);
  const int hi = lane_read(wave_iscan(v >> 16, 0, add), WAVE - 1);
  return ((int64_t)hi << 16) + lo;
}

// Wave-wide minimum and maximum (every lane gets the value).
template <typename T> __device__ inline T wave_min(T v) {
  v = wave_iscan(v, inf_of<T>(), [](T a, T b) { return b < a ? b : a; });
  return lane_read(v, WAVE - 1);
}
template <typename T>
__device__ inline T wave_max(T v) {
  v = wave_iscan(v, -inf_of<T>(), [](T a, T b) { return b > a ? b : a; });
  return lane_read(v, WAVE - 1);
}

// Inclusive scan over the wave; OP is min (exact in any order) or add (used
// for energies that only rank candidates).
template <typename T, bool IS_MIN>
__device__ inline T wave_scan(T v, int) {
  if (IS_MIN) return wave_iscan(v, inf_of<T>(), [](T a, T b) { return b < a ? b : a; });
  return wave_iscan(v, T(0), [](T a, T b) { return a + b; });
}

// Wave-uniform copies of values the compiler cannot prove uniform.
__device__ inline int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline float uni(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ inline double uni(double v) {
  const long long q = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readfirstlane((int)(q & 0xffffffff));
  const int hi = __builtin_amdgcn_readfirstlane((int)(q >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Fused multiply-add for energies that only rank candidates (every decision
// uses separately rounded operations).
__device__ inline float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Energy bounds.  A candidate's ranking energy is a sum of non-negative terms,
// so a sum with every term replaced by a lower bound of it cannot exceed it by
// more than rounding: at most about 2 N roundings of 2^-24 (binary32, N <=
// 1024: 1.2e-4, and the hardware reciprocals' ulps).  A bound that exceeds the
// energy of some candidate (inc) by 2^-12 of itself therefore belongs to
// candidates that neither win nor tie: they need not be evaluated.
template <typename T> __device__ inline bool beaten(T lb, T inc) {
  return lb * T(1.0 - 0x1p-12) > inc;
}

// A bound that overflows still belongs to a feasible candidate, whose energy
// may be infinite: it stays below the +inf of those that are not.
__device__ inline float finite_bound(float lb, float part = 1) {
  return lb < 0x1.fffffep127f * part ? lb : 0x1.fffffep127f * part;
}
__device__ inline double finite_bound(double lb, double part = 1) {
  return lb < 0x1.fffffffffffffp1023 * part ? lb : 0x1.fffffffffffffp1023 * part;
}

// Hardware reciprocal, for bounds.
__device__ inline float rough_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline double rough_rcp(double x) { return __builtin_amdgcn_rcp(x); }

// A little less than 1 / x (x > 0; the hardware's reciprocal of a denormal is
// infinite), small enough for the sum over JDOB_MAX_USERS users.
__device__ inline float rcp_below(float x) {
  const float q = rough_rcp(x) * (1.0f - 0x1p-20f);
  return q < 0x1p116f ? q : 0x1p116f;
}
__device__ inline double rcp_below(double x) {
  const double q = rough_rcp(x) * (1.0 - 0x1p-20);
  return q < 0x1p1012 ? q : 0x1p1012;
}

// CPU energy kC * f^2 (kC = kappa * C[s]) of a user with budget x or less, from
// below: the lowest frequency finishing Cs cycles by then, at least f0 (also
// where x <= 0 or Cs = 0 makes the quotient negative or NaN).
template <typename T> __device__ inline T least_cpu(T Cs, T kC, T x, T f0) {
  const T q = Cs * rough_rcp(x);
  const T f = q > f0 ? q : f0;
  return kC * (f * f);
}

// Lowest GPU energy per second of batch latency at the top level, over the
// GPU levels searched: P_j * Phi_j >= rho * (A[s] + B[s]*b).
template <typename T>
__device__ inline T gpu_energy_rate(const T *sr, const T *sP, int j_low, int J, int lane) {
  T v = inf_of<T>();
  for (int j = j_low + lane; j < J; j += WAVE) {
    const T e = sP[j] * sr[j];
    v = e < v ? e : v;
  }
  return wave_min(v);
}

// The GPU energy of a batch from below.  With ab its latency at the top level
// and r = gtop / g the stretch it is ab * (c3 / r^2 + p0 * r), c3 = gc * gtop^3
// (Eq. (5)): falling in r up to the stretch of g_opt = cbrt(p0 / (2 gc)),
// rising from there.  A batch that must be done in `room` needs r <= room / ab,
// where the second term is p0 * room.  So the least is there, or at g_opt (not
// below the lowest level searched) if that is faster.  room is a difference of
// times up to lo: a little is added for its rounding.  Up to four levels, which
// may lie far apart, are tried one by one instead (two levels a factor of ten
// apart, 347 instances of 7 users, 50 layers: 199 us without, 76 us).
template <typename T> struct GpuCost {
  T c3, p0, qmin, cost;  // qmin: 1 / stretch of g_opt; cost: energy per second of ab there
  const T *r, *P;        // stretch and power of the levels searched
  int n;                 // their number
  __device__ inline GpuCost(const T *gf, const T *sr, const T *sP, int j_low, int J, T gopt, T gc,
                            T s) {
    const T gtop = gf[J - 1], lo = gf[j_low], m = gopt > lo ? gopt : lo;
    const T g = m < gtop ? m : gtop;
    c3 = uni(gc * gtop * gtop * gtop);
    p0 = s;
    qmin = uni(g * rough_rcp(gtop));
    cost = uni(fma_(c3 * qmin, qmin, p0 * rough_rcp(qmin)));
    r = sr + j_low;
    P = sP + j_low;
    n = J - j_low;
  }
  __device__ inline T least(T ab, T room, T lo) const {
    const T some = fma_(lo, T(0x1p-20), room);
    if (n <= 4) {
      T v = inf_of<T>();
      for (int j = 0; j < n; ++j) {
        const T e = P[j] * r[j];
        v = ((ab * r[j] <= some) & (e < v)) ? e : v;
      }
      return v < inf_of<T>() ? ab * v : T(0);  // (no level: infeasible)
    }
    // (where room <= 0 makes q negative or NaN, nothing is feasible)
    const T q = ab * rough_rcp(some);
    return q > qmin ? fma_(c3 * ab, q * q, p0 * room) : ab * cost;
  }
};

// The frequency at which a second of top-level batch latency costs least.
inline double best_gpu_freq(double gc, double p0) {
  return gc > 0 ? cbrt(p0 / (2.0 * gc)) : INFINITY;
}

// A copy of a uniform value in scalar registers of its own.  Kernel arguments
// arrive in wide loads (eight or sixteen registers at a time); without the
// copy, a spill under register pressure saves and restores the whole group.
template <typename X> __device__ inline X own(X v) {
  asm volatile("" : "+s"(v));
  return v;
}

// Lanes 0..31 receive the value of lane l + 32 (one v_permlane32_swap);
// lanes 32..63 keep their own.
__device__ inline int from_upper_half(int v) {
  return (int)__builtin_amdgcn_permlane32_swap(v, v, false, false)[1];
}
__device__ inline float from_upper_half(float v) {
  return __int_as_float(from_upper_half(__float_as_int(v)));
}
__device__ inline double from_upper_half(double v) {
  const long long q = __double_as_longlong(v);
  const int lo = from_upper_half((int)(q & 0xffffffff)), hi = from_upper_half((int)(q >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Inclusive wavefront prefix sum with DPP row shifts and row broadcasts (the
// summation order differs from a sequential sum: used for energies that only
// rank candidates).
__device__ inline float scan_add(float v) {
#define JDOB_DPP_ADD(CTRL, RMASK) \
  v = v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, RMASK, 0xf, false))
  JDOB_DPP_ADD(0x111, 0xf);  // row_shr:1
  JDOB_DPP_ADD(0x112, 0xf);  // row_shr:2
  JDOB_DPP_ADD(0x114, 0xf);  // row_shr:4
  JDOB_DPP_ADD(0x118, 0xf);  // row_shr:8
  JDOB_DPP_ADD(0x142, 0xa);  // row_bcast:15
  JDOB_DPP_ADD(0x143, 0xc);  // row_bcast:31
#undef JDOB_DPP_ADD
  return v;
}
__device__ inline double scan_add(double v) {
#define JDOB_DPP_ADD(CTRL, RMASK)                                                         \
  {                                                                                       \
    const long long q = __double_as_longlong(v);                                          \
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(q & 0xffffffff), CTRL, RMASK, 0xf, false); \
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(q >> 32), CTRL, RMASK, 0xf, false);        \
    v = v + __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);               \
  }
  JDOB_DPP_ADD(0x111, 0xf);
  JDOB_DPP_ADD(0x112, 0xf);
  JDOB_DPP_ADD(0x114, 0xf);
  JDOB_DPP_ADD(0x118, 0xf);
  JDOB_DPP_ADD(0x142, 0xa);
  JDOB_DPP_ADD(0x143, 0xc);
#undef JDOB_DPP_ADD
  return v;
}


__device__ inline int64_t instance_of_block(int64_t first) {
  // Consecutive workgroups are dealt round-robin to the 8 XCDs; give each XCD
  // a contiguous range of instances so that neighbouring rows and output
  // words are touched through one L2.
  const int64_t nb = gridDim.x, b = blockIdx.x;
  const int64_t xcd = b % 8, pos = b / 8;
  const int64_t q = nb / 8, r = nb % 8;
  const int64_t start = xcd * q + (xcd < r ? xcd : r);
  return first + start + pos;
}

// Eq. (20) with a continuous CPU frequency: the slowest frequency finishing
// cycles Cs within the budget, clamped to [fmin, fmax]; fmin without local
// layers.  Used only where the top frequency fits the budget.
template <typename T> __device__ inline T cont_freq(T Cs, T budget, T fmin, T fmax) {
  if (Cs == T(0)) return fmin;
  const T g = Cs / budget;
  return g < fmin ? fmin : (g > fmax ? fmax : g);
}

__device__ inline float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline double fast_rcp(double x) { return 1.0 / x; }

__device__ inline float clamp_(float v, float lo, float hi) {
  return __builtin_amdgcn_fmed3f(v, lo, hi);  // lo <= hi
}
__device__ inline double clamp_(double v, double lo, double hi) {
  return v < lo ? lo : (v > hi ? hi : v);
}

// The outer grouping keeps, per prefix of the deadline order, a front of
// states (total energy, GPU release time) that no other state dominates (no
// higher energy and no later release), sorted by energy, at most
// GROUP_FRONT of them.
constexpr int GROUP_FRONT = 16;

// Adds the state (E, Tr, src) to the front fE/fT/from[0..n) of one prefix
// and returns the new size: nothing changes if a state of the front has no
// higher energy and no later release (it came first); otherwise the states
// the new one dominates leave, it enters at its energy's place, and a front
// longer than GROUP_FRONT loses its highest energy.  Lane q holds slot q;
// E, Tr, src and n are wave-uniform; the whole wave calls it.
template <typename T>
__device__ inline int front_add(T *fE, T *fT, int16_t *from, int n, T E, T Tr, int src, int lane) {
  const bool in = lane < n;
  const T e = in ? fE[lane] : T(0), t = in ? fT[lane] : T(0);
  const int fr = in ? from[lane] : 0;
  if (__builtin_amdgcn_ballot_w64(in && e <= E && t <= Tr)) return n;
  const bool keep = in && !(E <= e && Tr <= t);
  const uint64_t km = __builtin_amdgcn_ballot_w64(keep);
  const int m = __popcll(km);
  // kept states stay in energy order; those below E come first
  const int below = __popcll(__builtin_amdgcn_ballot_w64(keep && e < E));
  const int rk = __builtin_amdgcn_mbcnt_hi((unsigned)(km >> 32),
                                           __builtin_amdgcn_mbcnt_lo((unsigned)km, 0u));
  const int pos = rk < below ? rk : rk + 1;
  __syncthreads();  // every slot read before any is written
  if (keep && pos < GROUP_FRONT) {
    fE[pos] = e;
    fT[pos] = t;
    from[pos] = (int16_t)fr;
  }
  if (lane == 0 && below < GROUP_FRONT) {
    fE[below] = E;
    fT[below] = Tr;
    from[below] = (int16_t)src;
  }
  __syncthreads();
  return m + 1 < GROUP_FRONT ? m + 1 : GROUP_FRONT;
}

// Heterogeneous users (per-user zeta, kappa, transmit power and CPU levels),
// in jdob_hetero.hip.
bool has_user_params(const jdob_problem *p);
int validate_hetero(const jdob_problem *p, bool grouped);
int launch_hetero(const jdob_problem *p, const jdob_policy *o, hipStream_t stream);
int launch_hetero_grouped(const jdob_problem *p, const jdob_grouped_policy *o, hipStream_t stream);

}  // namespace jdob_dev

#endif  // JDOB_COMMON_H
