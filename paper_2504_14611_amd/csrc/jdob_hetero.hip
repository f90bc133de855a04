// jdob_hetero.hip — batched J-DOB for heterogeneous users on MI355X (gfx950).
//
// Sec. II gives each device m its own cycles-per-work ratio zeta_m (Eq. (1)),
// switched capacitance kappa_m (Eq. (2)), transmit power p_m (Eq. (4)) and
// CPU frequency range.  Alg. 1 then sorts the users by gamma (Eq. (17)) at
// every partition point, so the order pi_s, the batch deadlines lo[b]
// (Eq. (10)), bmin and the suffix sums all depend on s, and each offloader
// has its own level table.  One wave64 evaluates one instance (N <= 64, one
// lane per user wherever per-user work is done):
//   1. coalesced loads; the sums C, A, B in the pinned order; each user's
//      local-only level and energy (constraint (8), Eq. (20));
//   2. several partition points at a time: each user's gamma, its rank by
//      comparison counting (ties: lower index) and the smallest slack at which
//      it meets (7) at its top frequency; min-, max- and sum-scans along pi_s
//      give a lower bound of the partition point's energy.  The partition
//      points are searched best bound first, until the bound exceeds the best
//      energy found (hbounds); in those, the same scans give the batch records
//      and the batches worth a pass, and the level rows are built;
//   3. passes over (GPU level j x batch b) or, in the greedy mode, one batch
//      per level found by binary search; each lane walks its offloaders:
//      the level is the number of the user's levels too slow for the budget
//      (its latencies fall with the level), counted with broadcast reads, or
//      the continuous frequency clamped to the user's range;
//   4. the argmin (lowest flat index among equal energies, local computing
//      last), the winner's levels from exact comparisons, the energy summed
//      in user index order and the release time (Eq. (22)).
// Constraint (7) for every offloader of batch b is one comparison: user i
// meets it at its top frequency exactly when the slack H = lo[b] - Phi is
// at least need_i, the smallest binary value with t_i <= H - up_i (the
// rounded difference grows with H), so the batch needs H >= max_{i<b} need_i.
// The search takes any subset of the instance's users (a bit mask): all of
// them for one solve, a group of consecutive users in deadline order for
// the outer grouping (jdob_hetero_grouped_kernel), which solves every group
// of the dynamic program as an instance of its own.

#include "jdob_common.h"

#include <type_traits>

namespace jdob_dev {
namespace {

template <typename T> struct HProblem {
  const T *cyc, *bits, *alpha, *beta, *rate, *deadline, *tfree, *lf, *gf;
  const T *uzeta, *ukappa, *uptx, *ulf;  // per user, or nullptr: the shared value
  T kappa, ptx, gc, p0;
  T gopt;  // best_gpu_freq
  int N, L, K, J;
  int s_end, j_low;
};

template <typename T> struct HPolicy {
  int32_t *status, *cut, *gpu_level, *batch;
  T *energy, *tfree_out;
  int8_t *ulevel, *uoffload;
  int32_t *nfeas;
  int64_t *nevals;
  T *ufreq;
};

template <typename T> struct HArgs {
  HProblem<T> p;
  HPolicy<T> out;
  int64_t first;
};

template <typename T> struct HGrouped {
  int32_t *status, *num_groups;
  T *energy, *tfree_out;
  int16_t *order, *group_end;
  int32_t *group_cut, *group_gpu_level, *group_batch;
  T *group_energy, *group_tfree;
  int8_t *ulevel, *uoffload, *ugroup;
  int64_t *ninner, *nfeas, *nevals;
  T *ufreq;
};

template <typename T> struct HGArgs {
  HProblem<T> p;
  HGrouped<T> out;
  int64_t first;
};

// Per-user outputs of a winner (rows of one instance; nullptr: not written).
template <typename T> struct UserOut {
  int8_t *level, *offload, *group;
  T *freq;
  int gno;
};

// Per offloader at the current partition point, read together: its upload
// latency, its work zeta*C[s], its frequency range (continuous mode).
template <typename T> struct alignas(4 * sizeof(T)) HUser { T up, z, fmin, fmax; };

// A user in the gamma order of a partition point: its upload latency, need
// (slack_needed), work zeta*C[s], and its index m.
template <typename T> struct alignas(4 * sizeof(T)) HPos { T up, need, z, m; };

// Byte offsets of the per-instance LDS arrays.
struct HLayout {
  int cyc, al, be, bits, C, A, B, r, P;           // layers and GPU levels
  int rate, dl, zet, kap, ptx, lf, kL, eL, fL;    // per user (index m)
  int gam, need, pi, usr, kc, lv, bt, term;       // per position in pi_s
  int drank, dord, fE, fT, from, fn, ends, eks;  // the grouping program
  int tab;                                        // the grouping's orders, -1: none
  int K4, total;
  int limit;  // bytes that the limit of one instance's rows counts
};

__host__ __device__ inline HLayout make_hlayout(int N, int L, int K, int J, int szT,
                                               bool grouped) {
  HLayout y;
  int o = 0, lim = 0;  // (the limit also counts a row of rank keys)
  auto take = [&](int bytes) {
    int r = o;
    o = align8(o + bytes);
    lim = align8(lim + bytes);
    return r;
  };
  auto take32 = [&](int bytes) {
    o = (o + 31) & ~31;
    lim = (lim + 31) & ~31;
    return take(bytes);
  };
  y.K4 = 4;
  while (y.K4 < K) y.K4 <<= 1;  // level row stride: a power of two, pads never too slow
  y.cyc = take(L * szT);
  y.al = take(L * szT);
  y.be = take(L * szT);
  y.bits = take((L + 1) * szT);
  y.C = take((L + 1) * szT);
  y.A = take((L + 1) * szT);
  y.B = take((L + 1) * szT);
  y.r = take(J * szT);
  y.P = take(J * szT);
  y.rate = take(N * szT);
  y.dl = take(N * szT);
  y.zet = take(N * szT);
  y.kap = take(N * szT);
  y.ptx = take(N * szT);
  y.lf = take(N * K * szT);                    // user m's levels, ascending
  y.kL = take(N * 4);
  y.eL = take(N * szT);
  y.fL = take(N * szT);
  y.gam = take(N * szT);                       // bound of the first b users' CPU energy
  lim = align8(((lim + 31) & ~31) + ((N + 1) & ~1) * 8);
  y.need = take(N * szT);
  y.pi = take(N * 4);
  y.usr = take32((N + 1) * 4 * szT);           // HUser by position (+1: read-ahead)
  y.kc = take(N * szT);                        // kappa * C[s] by position
  y.lv = take32(N * y.K4 * 2 * szT);           // Level rows by position, K4 apart
  // Batch records, b = 1..N (+ sentinels); before they are stored, the keys of
  // a gamma order and then its records (64 of each)
  y.bt = take32((N + 2 + WAVE) * 4 * szT);
  y.term = take(N * szT);
  y.drank = y.dord = y.fE = y.fT = y.from = y.fn = y.ends = y.eks = 0;
  if (grouped) {
    y.drank = take(N * 4);        // position of user m in the deadline order
    y.dord = take(N * 4);         // users by deadline ascending
    const int F = GROUP_FRONT;    // front of prefix i: slots i*F .. i*F + F-1
    y.fE = take((N + 1) * F * szT);  // total energy of the first i users
    y.fT = take((N + 1) * F * szT);  // GPU release time after them
    y.from = take((N + 1) * F * 2);  // the state it extends (prefix * F + slot)
    y.fn = take((N + 1) * 4);        // states in the front of prefix i
    y.ends = take((N + 1) * 4);      // ends of the chosen groups, in order
    y.eks = take((N + 1) * 4);       // the chosen state at each end
  }
  // The grouping meets every partition point once per group: the gamma order
  // of all users, which holds every group's, with each one's HPos record, is
  // kept per partition point where the table costs no occupancy (the
  // workgroups that fit a CU's LDS, at most 24 of one wave each) and stays
  // within the limit of one workgroup.
  y.limit = lim;
  y.tab = -1;
  const int base = (o + 31) & ~31, tab_bytes = L * N * 4 * szT;
  auto per_cu = [](int bytes) {
    const int w = LDS_PER_CU / (bytes > 0 ? bytes : 1);
    return w < 24 ? w : 24;
  };
  if (grouped && base + tab_bytes <= LDS_LIMIT && per_cu(base + tab_bytes) == per_cu(o))
    y.tab = take32(tab_bytes);
  y.total = o;
  return y;
}

template <typename T> __device__ inline const __attribute__((address_space(4))) HArgs<T> *hargs() {
  return (const __attribute__((address_space(4))) HArgs<T> *)__builtin_amdgcn_kernarg_segment_ptr();
}
template <typename T>
__device__ inline const __attribute__((address_space(4))) HGArgs<T> *hgargs() {
  return (const __attribute__((address_space(4))) HGArgs<T> *)__builtin_amdgcn_kernarg_segment_ptr();
}

// The neighbouring binary values of a finite x (IEEE values of one sign are
// ordered like their bit patterns).
__device__ inline float next_down(float x) {
  if (x == 0.0f) return -__int_as_float(1);
  const int b = __float_as_int(x);
  return __int_as_float(x > 0.0f ? b - 1 : b + 1);
}
__device__ inline float next_up(float x) {
  if (x == 0.0f) return __int_as_float(1);
  const int b = __float_as_int(x);
  return __int_as_float(x > 0.0f ? b + 1 : b - 1);
}
__device__ inline double next_down(double x) {
  if (x == 0.0) return -__longlong_as_double(1);
  const long long b = __double_as_longlong(x);
  return __longlong_as_double(x > 0.0 ? b - 1 : b + 1);
}
__device__ inline double next_up(double x) {
  if (x == 0.0) return __longlong_as_double(1);
  const long long b = __double_as_longlong(x);
  return __longlong_as_double(x > 0.0 ? b + 1 : b - 1);
}

// The smallest binary value H with t <= H - u (rounded subtraction).  The
// predicate only turns true as H grows, and it does so within an ulp or two
// of t + u; the walk is capped so that it always ends.
template <typename T> __device__ inline T slack_needed(T t, T u) {
  T h = t + u;
  if (t <= h - u) {
    for (int it = 0; it < 64; ++it) {
      const T d = next_down(h);
      if (!(t <= d - u)) break;
      h = d;
    }
  } else {
    for (int it = 0; it < 64; ++it) {
      h = next_up(h);
      if (t <= h - u) break;
    }
  }
  return h;
}

// Instance rows, the pinned sums, per-user parameters and levels, and each
// user's local-only choice.
template <typename T, bool CONT>
__device__ void hprepare(const HProblem<T> &p, int64_t inst, unsigned char *smem, const HLayout &y,
                         int lane) {
  const int N = p.N, L = p.L, K = p.K, J = p.J;
  T *scyc = (T *)(smem + y.cyc), *sal = (T *)(smem + y.al), *sbe = (T *)(smem + y.be);
  T *sbits = (T *)(smem + y.bits);
  T *sC = (T *)(smem + y.C), *sA = (T *)(smem + y.A), *sB = (T *)(smem + y.B);
  T *sr = (T *)(smem + y.r), *sP = (T *)(smem + y.P);
  T *srate = (T *)(smem + y.rate), *sdl = (T *)(smem + y.dl), *szet = (T *)(smem + y.zet);
  T *skap = (T *)(smem + y.kap), *sptx = (T *)(smem + y.ptx), *slf = (T *)(smem + y.lf);
  int *skL = (int *)(smem + y.kL);
  T *seL = (T *)(smem + y.eL), *sfL = (T *)(smem + y.fL);

  for (int l = lane; l < L; l += WAVE) {
    scyc[l] = p.cyc[inst * L + l];
    sal[L - 1 - l] = p.alpha[inst * L + l];  // reversed: see chain_sums
    sbe[L - 1 - l] = p.beta[inst * L + l];
  }
  for (int l = lane; l <= L; l += WAVE) sbits[l] = p.bits[inst * (L + 1) + l];
  for (int j = lane; j < J; j += WAVE) {  // Eq. (5): stretch and power of level j
    const T g = p.gf[j], gtop = p.gf[J - 1];
    sr[j] = gtop / g;
    sP[j] = p.gc * ((g * g) * g) + p.p0;
  }
  if (lane < N) {
    const int64_t o = inst * N + lane;
    srate[lane] = p.rate[o];
    sdl[lane] = p.deadline[o];
    szet[lane] = p.uzeta ? p.uzeta[o] : T(1);
    skap[lane] = p.ukappa ? p.ukappa[o] : p.kappa;
    sptx[lane] = p.uptx ? p.uptx[o] : p.ptx;
  }
  for (int q = lane; q < N * K; q += WAVE)
    slf[q] = p.ulf ? p.ulf[inst * N * K + q] : p.lf[q % K];
  __syncthreads();
  // the sums C, A, B in the pinned order
  chain_sums(scyc, sal, sbe, sC, sA, sB, L, lane);
  // (8) with Eq. (20): the lowest level finishing every layer by the deadline
  if (lane < N) {
    const T W = szet[lane] * sC[L];
    const T *f = slf + lane * K;
    int kL = -1;
    for (int k = K - 1; k >= 0; --k)
      if (W / f[k] <= sdl[lane]) kL = k;
    T fL = T(0), eL = inf_of<T>();
    if (kL >= 0) {
      fL = CONT ? cont_freq(W, sdl[lane], f[0], f[K - 1]) : f[kL];
      eL = (skap[lane] * (fL * fL)) * sC[L];
    }
    skL[lane] = kL;
    seL[lane] = eL;
    sfL[lane] = fL;
  }
  __syncthreads();
}

// Rank of the lane's user in the gamma order of its partition point: users
// with a lower gamma come first, ties by lower index.  An aligned run of 2^lg
// lanes holds one partition point's users (lane m of the run user m, N of
// them); `mem` marks those ranked among each other.  In binary32 the 64-bit
// key (gamma bits, index) orders them the same way (gamma >= +0: a sum of a
// non-negative quotient and +0 or more, and non-negative IEEE values order
// like their bit patterns); the others, and the pad to an even count, get the
// largest key.  Two keys per read, one compare each.
__device__ inline int gamma_rank(float g, bool mem, int N, int lg, uint64_t *skey, int lane) {
  const int m = lane & ((1 << lg) - 1);
  const uint64_t me = mem ? ((uint64_t)__float_as_uint(g) << 32) | (uint32_t)m : ~(uint64_t)0;
  skey[lane] = me;
  __syncthreads();
  const uint64_t *k = skey + (lane - m);
  int pos = 0;
  for (int q = 0; q < N; q += 2) {  // (the run holds N + 1 lanes or N is even)
    const ulonglong2 kk = *(const ulonglong2 *)(k + q);
    pos += (kk.x < me ? 1 : 0) + (kk.y < me ? 1 : 0);
  }
  return pos;
}
__device__ inline int gamma_rank(double g, bool mem, int N, int lg, uint64_t *skey, int lane) {
  const int m = lane & ((1 << lg) - 1);
  double *sg = (double *)skey;
  sg[lane] = mem ? g : inf_of<double>();
  __syncthreads();
  const double *k = sg + (lane - m);
  int pos = 0;
  for (int q = 0; q < N; ++q) pos += (k[q] < g || (k[q] == g && q < m)) ? 1 : 0;
  return pos;
}

// The record and gamma (Eq. (17)) of user m at partition point s.
template <typename T>
__device__ inline HPos<T> user_at(const unsigned char *smem, const HLayout &y, int K, int s, int m,
                                  T *gamma) {
  HPos<T> u;
  u.z = ((const T *)(smem + y.zet))[m] * ((const T *)(smem + y.C))[s];      // cycles of layers 1..s
  const T tK1 = u.z / ((const T *)(smem + y.lf))[m * K + K - 1];            // Eq. (1), top level
  u.up = ((const T *)(smem + y.bits))[s] / ((const T *)(smem + y.rate))[m];  // Eq. (3)
  u.need = slack_needed(tK1, u.up);
  u.m = T(m);
  *gamma = u.up + tK1;
  return u;
}

// The gamma order pi_s of the users in mask, position by position: index,
// record, kappa * C[s] and need.
template <typename T>
__device__ inline void horder(const HProblem<T> &p, unsigned char *smem, const HLayout &y, int lane,
                              int s, uint64_t mask) {
  const int N = p.N, K = p.K;
  const T *slf = (const T *)(smem + y.lf);
  HPos<T> u;
  bool mem;
  int pos, m;
  if (y.tab >= 0) {  // the members of the full order, in that order
    u = ((const HPos<T> *)(smem + y.tab))[s * N + (lane < N ? lane : 0)];
    m = (int)u.m;
    mem = lane < N && ((mask >> m) & 1);
    const uint64_t mm = __builtin_amdgcn_ballot_w64(mem);
    pos = __builtin_amdgcn_mbcnt_hi((unsigned)(mm >> 32),
                                    __builtin_amdgcn_mbcnt_lo((unsigned)mm, 0u));
  } else {
    m = lane;
    mem = (mask >> lane) & 1;
    T g;
    u = user_at(smem, y, K, s, lane < N ? lane : 0, &g);
    pos = gamma_rank(g, mem, N, 6, (uint64_t *)(smem + y.bt), lane);
  }
  if (mem) {
    ((int *)(smem + y.pi))[pos] = m;
    HUser<T> v;
    v.up = u.up;
    v.z = u.z;
    v.fmin = slf[m * K];
    v.fmax = slf[m * K + K - 1];
    ((HUser<T> *)(smem + y.usr))[pos] = v;
    ((T *)(smem + y.kc))[pos] = ((const T *)(smem + y.kap))[m] * ((const T *)(smem + y.C))[s];
    ((T *)(smem + y.need))[pos] = u.need;
  }
  __syncthreads();
}

// Inclusive scan over each aligned run of 2^lg >= 16 lanes (the steps of
// wave_iscan that stay inside it).
template <typename V, typename OP> __device__ inline V run_iscan(V v, V id, int lg, OP op) {
  v = op(v, dpp_mov<0x111, 0xf>(id, v));  // row_shr:1
  v = op(v, dpp_mov<0x112, 0xf>(id, v));  // row_shr:2
  v = op(v, dpp_mov<0x114, 0xf>(id, v));  // row_shr:4
  v = op(v, dpp_mov<0x118, 0xf>(id, v));  // row_shr:8
  if (lg >= 5) v = op(v, dpp_mov<0x142, 0xa>(id, v));  // row_bcast:15 into rows 1, 3
  if (lg >= 6) v = op(v, dpp_mov<0x143, 0xc>(id, v));  // row_bcast:31 into rows 2, 3
  return v;
}

// Suffix sums over lanes 0..n-1 (v is zero past n): steps of 1, 2, 4, ...
// lanes, by DPP inside a row of 16.
template <typename T> __device__ inline T suffix_sum(T v, int n, int lane) {
  if (n <= 16) {
    v = v + dpp_mov<0x101, 0xf>(T(0), v);  // row_shl:1
    if (n > 2) v = v + dpp_mov<0x102, 0xf>(T(0), v);
    if (n > 4) v = v + dpp_mov<0x104, 0xf>(T(0), v);
    if (n > 8) v = v + dpp_mov<0x108, 0xf>(T(0), v);
    return v;
  }
  for (int d = 1; d < n; d <<= 1) {
    const T o = __shfl_down(v, d, WAVE);
    v = v + ((lane + d < n) ? o : T(0));
  }
  return v;
}

// The number of GPU levels at which a batch with deadline lo, need nd and
// batch latency ab at the top level is feasible: the highest ones, down to one
// found by binary search.
template <typename T>
__device__ inline int feasible_levels(const HProblem<T> &p, const T *sr, T lo, T nd, T ab,
                                      T tfree) {
  const int Jn = p.J - p.j_low;
  int low = 0;  // levels that miss a deadline
  for (int step = 1 << (31 - __clz(Jn)); step > 0; step >>= 1) {
    const int c = low + step;
    const T H = lo - ab * sr[c <= Jn ? p.j_low + c - 1 : p.J - 1];
    low = (c <= Jn && !(H >= tfree && H >= nd)) ? c : low;
  }
  return Jn - low;
}

// Lower bounds of the partition points' energies for the users in mask, with
// the GPU free at tfree, into slb[s] (+inf: no feasible candidate).  Lanes
// take (partition point, position in its gamma order), 64, 32 or 16 lanes a
// point.  A batch size b is bounded by the least GPU energy, the upload
// energy of the first b users, the local energy of the others, and the CPU
// energy of each offloader at the lowest frequency at which it could close a
// batch of its own, which no larger batch lets it go below; feasibility
// falls with b and rises with j, so the test is that of the top GPU level.
// (16 users, 22 layers: 5.5 of 21.5 partition points with feasible candidates
// are then searched, best bound first, in 7.7 passes of 72.)
// Counts the feasible candidates into nfeas, nevals when COUNT.  (Inlined: as
// a function it kept its arguments in 1 KB of scratch a lane; grouping of 531 x
// 21 users, binary64: 47 ms, 62 as a function.)
template <typename T, bool COUNT>
__device__ __forceinline__ void hbounds(const HProblem<T> &p, unsigned char *smem,
                                        const HLayout &y, int lane, uint64_t mask, T tfree,
                                        const GpuCost<T> &gpu, T *slb, int &nfeas, int &nevals) {
  const int N = p.N, K = p.K, J = p.J;
  const T *sC = (const T *)(smem + y.C), *sA = (const T *)(smem + y.A);
  const T *sB = (const T *)(smem + y.B), *sr = (const T *)(smem + y.r);
  const int lg = N <= 16 ? 4 : (N <= 32 ? 5 : 6), W = 1 << lg;
  const int r = lane >> lg, q = lane & (W - 1);
  const T rtop = sr[J - 1];
  for (int s0 = 0; s0 < p.s_end; s0 += WAVE >> lg) {
    const bool in = q < N && s0 + r < p.s_end;
    const int s = in ? s0 + r : 0;
    HPos<T> u;
    if (y.tab >= 0) {
      u = ((const HPos<T> *)(smem + y.tab))[s * N + (in ? q : 0)];
    } else {  // this run's orders, in the room of the batch records
      HPos<T> *scratch = (HPos<T> *)(smem + y.bt);
      T g;
      const HPos<T> v = user_at(smem, y, K, s, in ? q : 0, &g);
      const int pos = gamma_rank(g, in, N, lg, (uint64_t *)(smem + y.bt), lane);
      __syncthreads();  // every lane has read the keys before a record takes their room
      if (in) scratch[(lane - q) + pos] = v;
      __syncthreads();
      u = scratch[in ? lane : 0];
    }
    const int m = in ? (int)u.m : 0;
    const bool mem = in && ((mask >> m) & 1);
    const uint64_t mm = __builtin_amdgcn_ballot_w64(mem) >> (lane - q);
    const int b = __popcll(mm & ((uint64_t(2) << q) - 1));  // batch closed by this user
    const T lo = run_iscan(mem ? ((const T *)(smem + y.dl))[m] : inf_of<T>(), inf_of<T>(), lg,
                           [](T a, T b) { return b < a ? b : a; });
    const T nd = run_iscan(mem ? u.need : -inf_of<T>(), -inf_of<T>(), lg,
                           [](T a, T b) { return b > a ? b : a; });
    const T ab = sA[s] + sB[s] * T(b), H = lo - ab * rtop;
    const T cpu = least_cpu(u.z, ((const T *)(smem + y.kap))[m] * sC[s], H - u.up,
                            ((const T *)(smem + y.lf))[m * K]);
    const T off = run_iscan(mem ? fma_(((const T *)(smem + y.ptx))[m], u.up, cpu) : T(0), T(0), lg,
                            [](T a, T b) { return a + b; });
    // the others' local energy: suffix sums less the user's own
    // (infinite only for a user that misses its deadline: one whose energy
    // overflows takes a value that 64 of cannot)
    T sl = mem ? ((const T *)(smem + y.eL))[m] : T(0);
    if (((const int *)(smem + y.kL))[m] >= 0) sl = finite_bound(sl, T(1) / WAVE);
    if (lg == 4) {
      sl = sl + dpp_mov<0x101, 0xf>(T(0), sl);  // row_shl:1
      sl = sl + dpp_mov<0x102, 0xf>(T(0), sl);
      sl = sl + dpp_mov<0x104, 0xf>(T(0), sl);
      sl = sl + dpp_mov<0x108, 0xf>(T(0), sl);
      sl = dpp_mov<0x101, 0xf>(T(0), sl);
    } else {
      for (int d = 1; d < W; d <<= 1) {
        const T o = __shfl_down(sl, d, W);
        sl = sl + (q + d < W ? o : T(0));
      }
      const T o = __shfl_down(sl, 1, W);
      sl = q + 1 < W ? o : T(0);
    }
    // (sl is infinite where a user left local misses its deadline, (8))
    const bool ok = mem & (H >= tfree) & (H >= nd) & (sl < inf_of<T>());
    if constexpr (COUNT) {
      const int c = feasible_levels(p, sr, lo, nd, ab, tfree);
      nfeas += ok ? c : 0;
      nevals += ok ? c * b : 0;
    }
    const T room = lo - (nd > tfree ? nd : tfree);
    const T lb = run_reduce(ok ? finite_bound(gpu.least(ab, room, lo) + (off + sl)) : inf_of<T>(),
                            lg, [](T a, T b) { return b < a ? b : a; });
    if (q == 0 && s0 + r < p.s_end) slb[s0 + r] = lb;
    __syncthreads();
  }
}

// Partition point s for the users in mask (n of them): the gamma order
// pi_s of those users and each one's record; then, if a batch is worth a
// pass, the batch records b = 1..n and the level rows.  A batch is worth a
// pass if it is feasible at the top GPU level and its bound (see hbounds) is
// not beaten by inc.  The tests use the scans, before anything is stored.
// Returns bmin and sets *todo, bit b - 1 for batch size b (both
// wave-uniform); counts the feasible candidates as hbounds does when COUNT.
template <typename T, bool CONT, bool COUNT>
__device__ int hrow(const HProblem<T> &p, int64_t inst, unsigned char *smem, const HLayout &y,
                    int lane, int s, T tfree, uint64_t mask, int n, T inc,
                    const GpuCost<T> &gpu, T *rb, uint64_t *todo, int &nfeas, int &nevals) {
  const int K = p.K, K4 = y.K4;
  const T *sC = (const T *)(smem + y.C), *sA = (const T *)(smem + y.A);
  const T *sB = (const T *)(smem + y.B), *sdl = (const T *)(smem + y.dl);
  const T *skap = (const T *)(smem + y.kap), *sptx = (const T *)(smem + y.ptx);
  const T *slf = (const T *)(smem + y.lf), *seL = (const T *)(smem + y.eL);
  const int *skL = (const int *)(smem + y.kL), *spi = (const int *)(smem + y.pi);
  T *scl = (T *)(smem + y.gam);
  const HUser<T> *susr = (const HUser<T> *)(smem + y.usr);
  const T *skc = (const T *)(smem + y.kc), *sneed = (const T *)(smem + y.need);
  Level<T> *slv = (Level<T> *)(smem + y.lv);
  Batch<T> *sbt = (Batch<T> *)(smem + y.bt);
  const T Cs = sC[s];
  horder<T>(p, smem, y, lane, s, mask);
  // along pi_s (lane = position): lo = prefix min of deadlines (Eq. (10)),
  // the prefix max of need, bmin, the upload energy EU and the local
  // energies SL of the others (ranking only); scans over n positions
  const bool in = lane < n;
  const int m = in ? spi[lane] : 0;
  T lo = in ? sdl[m] : inf_of<T>(), nd = in ? sneed[lane] : -inf_of<T>();
  T sl = in ? seL[m] : T(0);
  // (up to 16 users, one row of lanes holds them all)
  const int lg = n <= 16 ? 4 : 6;
  lo = run_iscan(lo, inf_of<T>(), lg, [](T a, T b) { return b < a ? b : a; });
  nd = run_iscan(nd, -inf_of<T>(), lg, [](T a, T b) { return b > a ? b : a; });
  const uint64_t nolocal = __builtin_amdgcn_ballot_w64(in && skL[m] < 0);
  const int bmin = nolocal ? 64 - __clzll((long long)nolocal) : 0;
  const int blo = bmin > 1 ? bmin : 1;
  const T *sr = (const T *)(smem + y.r);
  const T ab = sA[s] + sB[s] * T(lane + 1);  // batch size lane + 1
  const T Htop = lo - ab * sr[p.J - 1];
  // the tests, with the operations of the passes
  uint64_t ok = __builtin_amdgcn_ballot_w64(in && lane + 1 >= blo && Htop >= tfree && Htop >= nd);
  *todo = 0;
  if (!ok) return bmin;
  if constexpr (COUNT) {
    const int c = feasible_levels(p, sr, lo, nd, ab, tfree);
    if ((ok >> lane) & 1) {
      nfeas += c;
      nevals += c * (lane + 1);
    }
  }
  const HUser<T> us = susr[in ? lane : 0];
  sl = suffix_sum(sl, n, lane);
  auto add = [](T a, T b) { return a + b; };
  const T eu = run_iscan(in ? sptx[m] * us.up : T(0), T(0), lg, add);
  T slnext;  // over positions > lane
  if (n <= 16) {
    slnext = dpp_mov<0x101, 0xf>(T(0), sl);
  } else {
    slnext = __shfl_down(sl, 1, WAVE);
    slnext = lane + 1 < n ? slnext : T(0);
  }
  const T esl = eu + slnext;
  const T cl =
      run_iscan(in ? least_cpu(us.z, skc[lane], Htop - us.up, us.fmin) : T(0), T(0), lg, add);
  const T lb = gpu.least(ab, lo - (nd > tfree ? nd : tfree), lo) + (esl + cl);
  *rb = (ok >> lane) & 1 ? finite_bound(lb) : inf_of<T>();
  *todo = ok & ~__builtin_amdgcn_ballot_w64(beaten(lb, inc));
  if (!*todo) return bmin;
  if (in) {
    Batch<T> r;
    r.lo = lo;
    r.upl = nd;
    r.esl = esl;
    r.ab = ab;
    sbt[lane + 1] = r;
    scl[lane] = cl;
  }
  for (int q = lane; q < WAVE + 1; q += WAVE) {  // past n: infeasible sentinels
    Batch<T> z;
    z.lo = -inf_of<T>();
    z.upl = T(0);
    z.esl = T(0);
    z.ab = T(0);
    sbt[n + 1 + q] = z;
  }
  __syncthreads();
  if (!CONT) {
    // Eqs. (1), (2) per (position, level): K4 lanes per user, padding never
    // too slow
    const int upw = WAVE / K4, pk = lane / K4, kk = lane - pk * K4;
    for (int p0 = 0; p0 < n; p0 += upw) {
      const int q = p0 + pk;
      if (pk < upw && q < n) {
        const int mq = spi[q];
        const T f = slf[mq * K + (kk < K ? kk : 0)];
        const T Wq = susr[q].z;
        Level<T> v;
        v.t = kk < K ? Wq / f : -inf_of<T>();
        v.e = kk < K ? (skap[mq] * (f * f)) * Cs : T(0);
        slv[q * K4 + kk] = v;
      }
    }
    __syncthreads();
  }
  return bmin;
}

// The CPU energy of a lane's offloaders 0..b-1 for ranking, given its slack
// Hu (+inf on infeasible lanes, whose sum is dropped): the wave walks users
// 0..bw-1; users 0..ball-1 belong to every feasible lane's batch (no test),
// later ones past the lane's batch add nothing.  The sum runs in user order,
// over several users per trip, whose level searches are independent.  LG > 0: the
// level rows hold 2^LG entries (the halving steps unrolled, each probe an
// LDS read at an immediate offset); LG = 0: their size is read from the
// layout.
template <typename T, bool CONT, int LG = 0>
__device__ inline T offload_cpu_energy(const unsigned char *smem, const HLayout &y, int K, T Hu,
                                       int b, int ball, int bw) {
  const HUser<T> *susr = (const HUser<T> *)(smem + y.usr);
  const T *skc = (const T *)(smem + y.kc);
  const Level<T> *slv = (const Level<T> *)(smem + y.lv);
  const int K4 = y.K4;
  auto user_e = [&](int g) -> T {
    const HUser<T> u = susr[g];
    const T x = Hu - u.up;
    if (CONT) {  // Eq. (20) with its clamp, in the user's own range
      const T f = clamp_(u.z * fast_rcp(x), u.fmin, u.fmax);
      return (skc[g] * f) * f;
    }
    // Eq. (20): the levels too slow for the budget are a prefix of the row
    // (latencies fall with the level), found by binary search over the row
    // padded to a power of two with never-too-slow entries; its reads depend
    // on each other, which eight waves per SIMD hide (counting every level
    // from broadcast reads was 12 % slower on h1 there, and faster at six
    // waves)
    if constexpr (LG > 0) {
      // The search ends at the level itself: an offloader of a feasible
      // lane fits its top level (the batch's slack covers its need), so
      // fewer than K levels are too slow; elsewhere the level read (at
      // most one entry past the row, inside the block's LDS) is dropped.
      constexpr unsigned S = sizeof(Level<T>);
      unsigned a = (unsigned)y.lv + (unsigned)(g << LG) * S;
#pragma unroll
      for (int h = (1 << LG) >> 1; h > 0; h >>= 1)
        a = (*(const T *)(smem + a + (h - 1) * S) > x) ? a + h * S : a;
      return *(const T *)(smem + a + sizeof(T));
    } else {
      const Level<T> *row = slv + g * K4;
      int k = 0;
      for (int step = K4 >> 1; step > 0; step >>= 1)
        k = (row[k + step - 1].t > x) ? k + step : k;
      k = k < K ? k : K - 1;
      return row[k].e;
    }
  };
  T acc = T(0);
  int g = 0;
  if constexpr (!CONT && LG > 0) {
    // the searches of four (then two) users step together: each probe of
    // one user beside the same probe of the others
    constexpr unsigned S = sizeof(Level<T>), R = (1u << LG) * S;
    for (; g + 3 < ball; g += 4) {
      T x[4];
      unsigned a[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        x[q] = Hu - susr[g + q].up;
        a[q] = (unsigned)y.lv + (unsigned)(g + q) * R;
      }
#pragma unroll
      for (int h = (1 << LG) >> 1; h > 0; h >>= 1) {
        T t[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) t[q] = *(const T *)(smem + a[q] + (h - 1) * S);
#pragma unroll
        for (int q = 0; q < 4; ++q) a[q] = (t[q] > x[q]) ? a[q] + h * S : a[q];
      }
      T e[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) e[q] = *(const T *)(smem + a[q] + sizeof(T));
#pragma unroll
      for (int q = 0; q < 4; ++q) acc = acc + e[q];
    }
    for (; g + 1 < ball; g += 2) {
      const T x0 = Hu - susr[g].up, x1 = Hu - susr[g + 1].up;
      unsigned a0 = (unsigned)y.lv + (unsigned)g * R, a1 = a0 + R;
#pragma unroll
      for (int h = (1 << LG) >> 1; h > 0; h >>= 1) {
        const T t0 = *(const T *)(smem + a0 + (h - 1) * S);
        const T t1 = *(const T *)(smem + a1 + (h - 1) * S);
        a0 = (t0 > x0) ? a0 + h * S : a0;
        a1 = (t1 > x1) ? a1 + h * S : a1;
      }
      const T e0 = *(const T *)(smem + a0 + sizeof(T)), e1 = *(const T *)(smem + a1 + sizeof(T));
      acc = acc + e0;
      acc = acc + e1;
    }
  } else if constexpr (CONT) {
    for (; g + 1 < ball; g += 2) {
      const T e0 = user_e(g), e1 = user_e(g + 1);
      acc = acc + e0;
      acc = acc + e1;
    }
  }
  for (; g < ball; ++g) acc = acc + user_e(g);
  for (; g < bw; ++g) {
    const T e = user_e(g);
    acc = (g < b) ? acc + e : acc;
  }
  return acc;
}

// Every candidate (s, j, b) of the mode's family for the users in mask (n of
// them) with the GPU free at tfree that is not beaten by inc, the energy of
// local computing or +inf, or by a candidate found before: each lane's best
// (energy, flat index over the n users' family, lowest index among equal
// energies) in bestE, bestI, and the work of the whole family in nfeas,
// nevals when COUNT.
template <typename T, bool COUNT, bool GREEDY, bool CONT, int LG = 0>
__device__ void hsearch(const HProblem<T> &p, int64_t inst, unsigned char *smem, const HLayout &y,
                        int lane, uint64_t mask, int n, T tfree, T inc,
                        const GpuCost<T> &gpu, T &bestE, int &bestI, int &nfeas, int &nevals) {
  const int N = p.N, K = p.K, J = p.J, s_end = p.s_end, j_low = p.j_low;
  const T *sr = (const T *)(smem + y.r), *sP = (const T *)(smem + y.P);
  const Batch<T> *sbt = (const Batch<T> *)(smem + y.bt);
  const T *scl = (const T *)(smem + y.gam);
  const int Jn = J - j_low;
  const int Jw = Jn < WAVE ? Jn : WAVE;
  const int nb = WAVE / Jw;
  const int jl = lane % Jw, bo = lane / Jw;
  const bool idle = bo >= nb;  // past the pass's (j, b) pairs: never feasible
  if (GREEDY && COUNT) inc = inf_of<T>();  // its counters come from the search itself

  // inc after lanes with `take` found E
  auto lower_inc = [&](bool take, T E) {
    if (GREEDY && COUNT) return;
    if (__builtin_amdgcn_ballot_w64(take & (E < inc))) {
      const T m = wave_min(take ? E : inf_of<T>());
      inc = m < inc ? m : inc;
    }
  };

  auto search_point = [&](auto by_bounds, int s) {
    constexpr bool bounds = decltype(by_bounds)::value;
    uint64_t todo;
    T rb;  // the bound of batch size lane + 1
    const int bmin = hrow<T, CONT, COUNT && !GREEDY && !bounds>(
        p, inst, smem, y, lane, s, tfree, mask, n, inc, gpu, &rb, &todo, nfeas, nevals);
    const int blo = bmin > 1 ? bmin : 1;
    if (!todo) return;
    const int sJN = s * J * n;
    if (GREEDY) {
      // Alg. 2 at each GPU level (lane = j): the largest set whose users all
      // meet (7) at their top frequency; the test fails more as b grows
      const int top = 1 << (31 - __clz(n));
      for (int jc = j_low; jc < J; jc += WAVE) {
        const int j = jc + lane;
        const bool jok = j < J;
        const T rj = sr[jok ? j : J - 1];
        int bg = 0;
        for (int step = top; step > 0; step >>= 1) {
          const int c = bg + step;
          const Batch<T> rc = sbt[c <= n ? c : n + 1];
          const T Hc = rc.lo - rc.ab * rj;
          bg = (Hc >= rc.upl) ? c : bg;
        }
        const Batch<T> r = sbt[bg > 0 ? bg : n + 1];
        const T Phi = r.ab * rj;
        const T H = r.lo - Phi;
        const bool feas = jok & (bg >= blo) & (H >= tfree);
        const T pj = sP[jok ? j : J - 1];
        const T lb = fma_(pj, Phi, r.esl + scl[bg > 0 ? bg - 1 : 0]);
        const bool need = feas & !beaten(lb, inc);
        const uint64_t fm = __builtin_amdgcn_ballot_w64(need);
        if (COUNT) {
          nfeas += feas ? 1 : 0;
          nevals += feas ? bg : 0;
        }
        if (fm == 0) continue;
        const int bw = __builtin_amdgcn_readlane(bg, 63 - __clzll((long long)fm));
        const T cpu =
            offload_cpu_energy<T, CONT, LG>(smem, y, K, need ? H : inf_of<T>(), bg, 0, bw);
        const T E = fma_(pj, Phi, cpu + r.esl);
        const int idx = sJN + (J - 1 - j) * n + (n - bg);
        const bool take = need & better(E, idx, bestE, bestI);
        bestE = take ? E : bestE;
        bestI = take ? idx : bestI;
        lower_inc(take, E);
      }
    } else {
      // one batch size a pass: best bound first; several: in order
      while (todo) {
        int q = __builtin_ctzll(todo);
        if (nb == 1) {
          const T least = wave_min(rb);
          if (!(least < inf_of<T>()) || beaten(least, inc)) break;
          q = __builtin_ctzll(__builtin_amdgcn_ballot_w64(rb == least));
          rb = lane == q ? inf_of<T>() : rb;
        } else {
          todo = q + nb < WAVE ? todo & (~uint64_t(0) << (q + nb)) : 0;
        }
        const int b0 = q + 1;
        for (int jc = 0; jc < Jn; jc += WAVE) {
          const int j = j_low + jc + jl;
          const bool jok = !idle && j < J;
          const int b = b0 + bo;
          const Batch<T> r = sbt[b];
          const T Phi = r.ab * sr[jok ? j : J - 1];            // Eq. (5), layers s+1..L
          const T H = r.lo - Phi;                               // slack to the batch deadline
          const bool feas = jok & (H >= tfree) & (H >= r.upl);  // (6), (7); (8): b >= bmin
          const T pj = sP[jok ? j : J - 1];
          const T lb = fma_(pj, Phi, r.esl + scl[b <= n ? b - 1 : 0]);
          const bool need = feas & !beaten(lb, inc < bestE ? inc : bestE);
          const uint64_t fm = __builtin_amdgcn_ballot_w64(need);
          if (fm == 0) continue;
          const int bw = b0 + __builtin_amdgcn_readlane(bo, 63 - __clzll((long long)fm));
          // every lane of the pass has a batch of at least b0
          const T cpu =
              offload_cpu_energy<T, CONT, LG>(smem, y, K, need ? H : inf_of<T>(), b, b0, bw);
          const T E = fma_(pj, Phi, cpu + r.esl);
          const int idx = sJN + (J - 1 - j) * n + (n - b);
          const bool take = need & better(E, idx, bestE, bestI);
          bestE = take ? E : bestE;
          bestI = take ? idx : bestI;
          lower_inc(take, E);
        }
      }
    }
  };

  // By their bounds, the lowest first, until it is beaten; as they come where
  // the bounds do not pay: with one or two partition points, and with more
  // users than let the bounds take several at once (in the greedy search,
  // whose rows cost less, than four) unless the orders are at hand.  Measured
  // with CPU levels, 16,384 instances, 22 layers, 8 GPU levels: 33 users 375 us
  // as they come, 490 by bounds, 64 users 633 and 832, 32 users 325 and 309; on
  // the continuous frequency: 25,078 x 17 users 183 us as they come,
  // 130 by bounds; 16,384 x 17 users, 22 layers 232 and 251; 6,453 x 47 users,
  // greedy, 208 and 273; 1,769 x 18, greedy, 70 and 85.  Nor where the greedy search counts, for which every partition point is
  // searched: grouping of 600 x 11 users 5.23 ms by bounds, 4.37 as they come.
  if ((GREEDY && COUNT) || s_end <= 2 || !(N <= 16 || (!GREEDY && N <= 32) || y.tab >= 0)) {
    for (int s = 0; s < s_end; ++s) search_point(std::false_type{}, s);
    return;
  }
  T *slb = (T *)(smem + y.cyc);  // (the layers' cycles have been summed)
  hbounds<T, COUNT && !GREEDY>(p, smem, y, lane, mask, tfree, gpu, slb, nfeas, nevals);
  for (int s0 = 0; s0 < s_end; s0 += WAVE) {
    T lb = s0 + lane < s_end ? slb[s0 + lane] : inf_of<T>();
    while (true) {
      const T m = wave_min(lb);
      if (!(m < inf_of<T>()) || beaten(m, inc)) break;
      const int q = __builtin_ctzll(__builtin_amdgcn_ballot_w64(lb == m));
      lb = lane == q ? inf_of<T>() : lb;
      search_point(std::true_type{}, s0 + q);
    }
  }
}

// Local computing of the users in mask: whether every one of them meets
// its deadline locally (8), and their local energies summed for ranking
// (any order).  Both wave-uniform.
template <typename T>
__device__ inline bool hlocal(const unsigned char *smem, const HLayout &y, int lane, uint64_t mask,
                              int n_max, T *e) {
  const int *skL = (const int *)(smem + y.kL);
  const T *seL = (const T *)(smem + y.eL);
  const bool mem = (mask >> lane) & 1;
  const bool ok = __builtin_amdgcn_ballot_w64(mem && skL[lane] < 0) == 0;
  T v = mem ? seL[lane] : T(0);
  v = run_reduce(v, n_max <= 16 ? 4 : 6, [](T a, T b) { return a + b; });
  *e = uni(v);
  return ok;
}

// The winner idx of the users in mask (n of them; idx = L*J*n is local
// computing) with the GPU free at tfree: each member's choice from
// correctly rounded operations in the oracle's order, the energy summed
// over the members in user index order (Eq. (21)), the release time (Eq.
// (22)); each member's level, offload flag, group and frequency are stored
// through uo where its pointers are set.
template <typename T, bool CONT>
__device__ void hwinner(const HProblem<T> &p, int64_t inst, unsigned char *smem, const HLayout &y,
                        int lane, uint64_t mask, int n, int idx, T tfree, T &E, T &tf,
                        const UserOut<T> &uo, T *slack = nullptr, T *rdy = nullptr,
                        T *phi = nullptr) {
  const int L = p.L, K = p.K, J = p.J;
  const int *skL = (const int *)(smem + y.kL);
  const T *seL = (const T *)(smem + y.eL), *sfL = (const T *)(smem + y.fL);
  T *sterm = (T *)(smem + y.term);
  const bool mem = (mask >> lane) & 1;
  if (idx == L * J * n) {  // local computing
    if (mem) {
      sterm[lane] = seL[lane];
      if (uo.level) {
        uo.level[lane] = (int8_t)(CONT ? -1 : skL[lane]);
        uo.offload[lane] = 0;
        if (uo.group) uo.group[lane] = (int8_t)uo.gno;
        if (uo.freq) uo.freq[lane] = sfL[lane];
      }
    }
    __syncthreads();
    T acc = T(0);
    for (uint64_t mm = mask; mm; mm &= mm - 1) acc = acc + sterm[__builtin_ctzll(mm)];
    E = acc;
    tf = tfree;
    if (slack) *slack = inf_of<T>();
    if (rdy) *rdy = -inf_of<T>();
    if (phi) *phi = T(0);
    __syncthreads();
    return;
  }
  const int s = idx / (J * n);
  const int rem = idx - s * (J * n);
  const int j = J - 1 - rem / n;
  const int b = n - (rem - (rem / n) * n);
  horder<T>(p, smem, y, lane, s, mask);
  const T *sC = (const T *)(smem + y.C), *sA = (const T *)(smem + y.A);
  const T *sB = (const T *)(smem + y.B), *slf = (const T *)(smem + y.lf);
  const T *skap = (const T *)(smem + y.kap), *sptx = (const T *)(smem + y.ptx);
  const T *sr = (const T *)(smem + y.r), *sP = (const T *)(smem + y.P);
  const T *sdl = (const T *)(smem + y.dl);
  const bool in = lane < n;  // lane = position in pi_s
  const int m = in ? ((const int *)(smem + y.pi))[lane] : 0;
  const HUser<T> us = ((const HUser<T> *)(smem + y.usr))[in ? lane : 0];
  const T Cs = sC[s];
  const T Phi = (sA[s] + sB[s] * T(b)) * sr[j];
  const T H = wave_min(lane < b ? sdl[m] : inf_of<T>()) - Phi;  // lo[b] of Eq. (10)
  T ready = -inf_of<T>();  // the latest offloader, the GPU free time joins below
  if (in) {
    int lv;
    int8_t off;
    T fq;
    if (lane < b) {
      const T x = H - us.up;
      const T *f = slf + m * K;
      int k = K - 1;
      for (int q = K - 1; q >= 0; --q)
        if (us.z / f[q] <= x) k = q;
      fq = CONT ? cont_freq(us.z, x, f[0], f[K - 1]) : f[k];
      const T e = (skap[m] * (fq * fq)) * Cs;
      sterm[m] = e + sptx[m] * us.up;
      const T done = us.z / fq + us.up;
      ready = (done > ready) ? done : ready;
      lv = CONT ? -1 : k;
      off = 1;
    } else {
      sterm[m] = seL[m];
      lv = CONT ? -1 : skL[m];
      fq = sfL[m];
      off = 0;
    }
    if (uo.level) {
      uo.level[m] = (int8_t)lv;
      uo.offload[m] = off;
      if (uo.group) uo.group[m] = (int8_t)uo.gno;
      if (uo.freq) uo.freq[m] = fq;
    }
  }
  ready = wave_max(ready);
  __syncthreads();
  T acc = T(0);
  for (uint64_t mm = mask; mm; mm &= mm - 1) acc = acc + sterm[__builtin_ctzll(mm)];
  E = acc + sP[j] * Phi;
  tf = ((tfree > ready) ? tfree : ready) + Phi;
  if (slack) *slack = H;
  if (rdy) *rdy = ready;
  if (phi) *phi = Phi;
  __syncthreads();
}

// Eight waves per SIMD: the rows and the bounds wait on LDS (262,144 x 16
// users, 22 layers: 1.83 ms at eight waves, 1.85 at seven, 1.96 at six; 5.34
// before the bounds).  LG > 0: level rows of 2^LG
// entries (launches without the work counters).
template <typename T, bool COUNT, bool GREEDY, bool CONT, int LG = 0>
__global__ __launch_bounds__(WAVE, 8) void jdob_hetero_kernel(HArgs<T> args) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x;
  const HProblem<T> &p = args.p;
  const int64_t inst = instance_of_block(args.first);
  const int N = p.N, L = p.L, J = p.J;
  const HLayout y = make_hlayout(N, L, p.K, J, (int)sizeof(T), false);
  const T tfree = p.tfree ? p.tfree[inst] : T(0);
  const uint64_t all = (N == WAVE) ? ~uint64_t(0) : ((uint64_t(1) << N) - 1);

  hprepare<T, CONT>(p, inst, smem, y, lane);
  T bestE = inf_of<T>();
  int bestI = 0x7fffffff, nfeas = 0;
  int nevals = 0;
  const GpuCost<T> gpu(p.gf, (const T *)(smem + y.r), (const T *)(smem + y.P), p.j_low, J, p.gopt,
                       p.gc, p.p0);
  T eLC;
  const bool local = hlocal<T>(smem, y, lane, all, N, &eLC);
  hsearch<T, COUNT, GREEDY, CONT, LG>(
      p, inst, smem, y, lane, all, N, tfree, local ? eLC : inf_of<T>(), gpu, bestE, bestI, nfeas,
      nevals);
  // local computing competes last
  const int idxLC = L * J * N;
  wave_argmin(bestE, bestI);
  if (local) {
    nfeas += (lane == 0) ? 1 : 0;
    if (better(eLC, idxLC, bestE, bestI)) { bestE = eLC; bestI = idxLC; }
  }
  const auto *a = hargs<T>();
  if constexpr (COUNT) {
    const int64_t totfeas = wave_sum_i64(nfeas), totev = wave_sum_i64(nevals);
    if (lane == 0) {
      if (a->out.nfeas) a->out.nfeas[inst] = (int32_t)totfeas;
      if (a->out.nevals) a->out.nevals[inst] = totev;
    }
  }
  UserOut<T> uo;
  uo.level = a->out.ulevel + inst * N;
  uo.offload = a->out.uoffload + inst * N;
  uo.group = nullptr;
  uo.freq = a->out.ufreq ? a->out.ufreq + inst * N : nullptr;
  uo.gno = 0;
  if (bestI == 0x7fffffff) {  // nothing feasible
    if (lane == 0) {
      a->out.status[inst] = 1;
      a->out.cut[inst] = -1;
      a->out.gpu_level[inst] = -1;
      a->out.batch[inst] = 0;
      a->out.energy[inst] = inf_of<T>();
      a->out.tfree_out[inst] = inf_of<T>();
    }
    if (lane < N) {
      uo.level[lane] = -1;
      uo.offload[lane] = 0;
      if (uo.freq) uo.freq[lane] = T(0);
    }
    return;
  }
  T E, tf;
  hwinner<T, CONT>(p, inst, smem, y, lane, all, N, bestI, tfree, E, tf, uo);
  if (lane == 0) {
    int s = L, j = -1, b = 0;
    if (bestI != idxLC) {
      s = bestI / (J * N);
      const int rem = bestI - s * (J * N);
      j = J - 1 - rem / N;
      b = N - (rem - (rem / N) * N);
    }
    a->out.status[inst] = 0;
    a->out.cut[inst] = s;
    a->out.gpu_level[inst] = j;
    a->out.batch[inst] = b;
    a->out.energy[inst] = E;
    a->out.tfree_out[inst] = tf;
  }
}

// Outer grouping with heterogeneous users: users by deadline (ties: lower
// index), consecutive groups served in order, each group one search over
// its members with the GPU free at the previous group's release time.  The
// dynamic program keeps, per prefix of the deadline order, the front of
// non-dominated (total energy, GPU release time) states, as the other
// grouping kernel does.  Six waves per SIMD: at more, values spill
// to scratch (16,384 x 10 users, continuous: 3.25 ms at six waves, 3.32 at
// seven, 3.59 at eight, 3.44 at five; 9.4 before the bounds).
template <typename T, bool COUNT, bool GREEDY, bool CONT>
__global__ __launch_bounds__(WAVE, 6) void jdob_hetero_grouped_kernel(HGArgs<T> args) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x;
  const HProblem<T> &p = args.p;
  const int64_t inst = instance_of_block(args.first);
  const int N = p.N, L = p.L, J = p.J;
  const HLayout y = make_hlayout(N, L, p.K, J, (int)sizeof(T), true);
  const T *sdl = (const T *)(smem + y.dl);
  int *dr = (int *)(smem + y.drank), *dord = (int *)(smem + y.dord);
  int *fn = (int *)(smem + y.fn), *ends = (int *)(smem + y.ends), *eks = (int *)(smem + y.eks);
  T *fE = (T *)(smem + y.fE), *fT = (T *)(smem + y.fT);
  int16_t *from = (int16_t *)(smem + y.from);
  constexpr int F = GROUP_FRONT;

  hprepare<T, CONT>(p, inst, smem, y, lane);
  if (y.tab >= 0) {
    HPos<T> *tab = (HPos<T> *)(smem + y.tab);
    for (int s = 0; s < p.s_end; ++s) {
      T g;
      const HPos<T> u = user_at(smem, y, p.K, s, lane < N ? lane : 0, &g);
      const int pos = gamma_rank(g, lane < N, N, 6, (uint64_t *)(smem + y.bt), lane);
      if (lane < N) tab[s * N + pos] = u;
      __syncthreads();
    }
  }
  if (lane < N) {  // the deadline order
    const T Tm = sdl[lane];
    int r = 0;
    for (int q = 0; q < N; ++q) r += (sdl[q] < Tm || (sdl[q] == Tm && q < lane)) ? 1 : 0;
    dr[lane] = r;
    dord[r] = lane;
  }
  for (int i = lane; i <= N; i += WAVE) fn[i] = i == 0 ? 1 : 0;
  if (lane == 0) {  // the empty prefix: no energy, the GPU free at t_free
    fE[0] = T(0);
    fT[0] = p.tfree ? p.tfree[inst] : T(0);
    from[0] = -1;
  }
  __syncthreads();

  // users at deadline ranks [lo, hi) as a lane mask
  auto members = [&](int lo, int hi) -> uint64_t {
    const int r = dr[lane < N ? lane : 0];
    return __builtin_amdgcn_ballot_w64(lane < N && r >= lo && r < hi);
  };
  const GpuCost<T> gpu(p.gf, (const T *)(smem + y.r), (const T *)(smem + y.P), p.j_low, J, p.gopt,
                       p.gc, p.p0);
  // the group's winner among its candidates and local computing, with the
  // GPU free at tf0 (0x7fffffff if none is feasible); counts into nf, ne
  auto group_search = [&](uint64_t mask, int n, T tf0, int &nf, int &ne) -> int {
    T bestE = inf_of<T>();
    int bestI = 0x7fffffff;
    T eLC;
    const bool local = hlocal<T>(smem, y, lane, mask, N, &eLC);
    hsearch<T, COUNT, GREEDY, CONT>(p, inst, smem, y, lane, mask, n, tf0,
                                    local ? eLC : inf_of<T>(), gpu, bestE, bestI, nf, ne);
    wave_argmin(bestE, bestI);
    if (local) {
      if (COUNT) nf += (lane == 0) ? 1 : 0;
      if (better(eLC, L * J * n, bestE, bestI)) { bestE = eLC; bestI = L * J * n; }
    }
    return uni(bestI);
  };

  int nfeas = 0;
  int nevals = 0;
  int64_t ninner = 0, nfeas_all = 0, nevals_all = 0;
  const UserOut<T> none{nullptr, nullptr, nullptr, nullptr, 0};
  for (int i = 1; i <= N; ++i) {
    int ni = 0;  // states in the front of prefix i
    for (int j = 0; j < i; ++j) {  // last group: users at deadline ranks j..i-1
      const int nj = uni(fn[j]);
      if (nj == 0) continue;
      const int n = i - j;
      const uint64_t mask = members(j, i);
      // the states of prefix j from the earliest release on; a winner whose
      // slack meets a later state's free time is that state's winner too
      // (constraint (6) is its only test that depends on the free time)
      int k = nj - 1;
      while (k >= 0) {
        const T tf0 = uni(fT[j * F + k]);
        const int idx = group_search(mask, n, tf0, nfeas, nevals);
        ++ninner;
        if (idx == 0x7fffffff) break;  // the states left free the GPU later still
        T Eg, Tg, H, rd, Ph;
        hwinner<T, CONT>(p, inst, smem, y, lane, mask, n, idx, tf0, Eg, Tg, none, &H, &rd, &Ph);
        Eg = uni(Eg);
        H = uni(H);
        rd = uni(rd);
        Ph = uni(Ph);
        T tk = tf0;
        do {
          const T Tk = ((tk > rd) ? tk : rd) + Ph;  // Eq. (22) after free time tk
          ni = front_add(fE + i * F, fT + i * F, from + i * F, ni, uni(fE[j * F + k]) + Eg, Tk,
                         j * F + k, lane);
          --k;
          tk = k >= 0 ? uni(fT[j * F + k]) : tk;
        } while (k >= 0 && H >= tk);
      }
      if constexpr (COUNT) {  // (a lane's sums over one group stay below 2^31)
        nfeas_all += wave_sum_i64(nfeas);
        nevals_all += wave_sum_i64(nevals);
        nfeas = nevals = 0;
      }
    }
    if (lane == 0) fn[i] = ni;
    __syncthreads();
  }

  const auto *a = hgargs<T>();
  const int64_t o = inst * N;
  for (int q = lane; q < N; q += WAVE) {
    a->out.order[o + q] = (int16_t)dord[q];
    a->out.group_end[o + q] = 0;
    a->out.group_cut[o + q] = -1;
    a->out.group_gpu_level[o + q] = -1;
    a->out.group_batch[o + q] = 0;
    a->out.group_energy[o + q] = inf_of<T>();
    a->out.group_tfree[o + q] = inf_of<T>();
    a->out.ulevel[o + q] = -1;
    a->out.uoffload[o + q] = 0;
    a->out.ugroup[o + q] = -1;
    if (a->out.ufreq) a->out.ufreq[o + q] = T(0);
  }
  if constexpr (COUNT) {
    if (lane == 0) {
      if (a->out.ninner) a->out.ninner[inst] = ninner;
      if (a->out.nfeas) a->out.nfeas[inst] = nfeas_all;
      if (a->out.nevals) a->out.nevals[inst] = nevals_all;
    }
  }
  if (uni(fn[N]) == 0) {
    if (lane == 0) {
      a->out.status[inst] = 1;
      a->out.num_groups[inst] = 0;
      a->out.energy[inst] = inf_of<T>();
      a->out.tfree_out[inst] = inf_of<T>();
    }
    return;
  }
  // the lowest-energy state of the full order, back to the empty prefix;
  // its groups are then solved again in order to write the policy
  int G = 0;
  for (int st = N * F; st > 0; st = uni((int)from[st])) ++G;
  if (lane == 0) {
    int c = G;
    for (int st = N * F; st > 0; st = from[st]) {
      --c;
      ends[c] = st / F;
      eks[c] = st;
    }
  }
  __syncthreads();
  UserOut<T> uo;
  uo.level = a->out.ulevel + o;
  uo.offload = a->out.uoffload + o;
  uo.group = a->out.ugroup + o;
  uo.freq = a->out.ufreq ? a->out.ufreq + o : nullptr;
  int start = 0;
  for (int gno = 0; gno < G; ++gno) {
    const int b = uni(ends[gno]), n = b - start;
    const uint64_t mask = members(start, b);
    const T tf0 = uni(fT[from[uni(eks[gno])]]);
    int nf = 0;
    int ne = 0;
    const int idx = group_search(mask, n, tf0, nf, ne);
    uo.gno = gno;
    T Eg, Tg;
    hwinner<T, CONT>(p, inst, smem, y, lane, mask, n, idx, tf0, Eg, Tg, uo);
    if (lane == 0) {
      int s = L, jg = -1, bb = 0;
      if (idx != L * J * n) {
        s = idx / (J * n);
        const int rem = idx - s * (J * n);
        jg = J - 1 - rem / n;
        bb = n - (rem - (rem / n) * n);
      }
      a->out.group_end[o + gno] = (int16_t)b;
      a->out.group_cut[o + gno] = s;
      a->out.group_gpu_level[o + gno] = jg;
      a->out.group_batch[o + gno] = bb;
      a->out.group_energy[o + gno] = Eg;
      a->out.group_tfree[o + gno] = Tg;
    }
    start = b;
  }
  if (lane == 0) {
    a->out.status[inst] = 0;
    a->out.num_groups[inst] = G;
    a->out.energy[inst] = fE[N * F];
    a->out.tfree_out[inst] = fT[N * F];
  }
}

template <typename T> HProblem<T> to_hproblem(const jdob_problem *q) {
  HProblem<T> p;
  p.cyc = (const T *)q->layer_cycles;
  p.bits = (const T *)q->out_bits;
  p.alpha = (const T *)q->gpu_alpha;
  p.beta = (const T *)q->gpu_beta;
  p.rate = (const T *)q->uplink_rate;
  p.deadline = (const T *)q->deadline;
  p.tfree = (const T *)q->t_free;
  p.lf = (const T *)q->local_freq;
  p.gf = (const T *)q->gpu_freq;
  p.uzeta = (const T *)q->user_zeta;
  p.ukappa = (const T *)q->user_kappa;
  p.uptx = (const T *)q->user_p_tx;
  p.ulf = (const T *)q->user_local_freq;
  p.kappa = (T)q->kappa;
  p.ptx = (T)q->p_tx;
  p.gc = (T)q->gpu_c;
  p.p0 = (T)q->gpu_p_static;
  p.gopt = (T)best_gpu_freq(q->gpu_c, q->gpu_p_static);
  p.N = q->num_users;
  p.L = q->num_layers;
  p.K = q->num_local_levels;
  p.J = q->num_gpu_levels;
  p.s_end = (q->mode & JDOB_MODE_BINARY) ? 1 : p.L;
  p.j_low = (q->mode & JDOB_MODE_FIXED_EDGE_FREQ) ? p.J - 1 : 0;
  return p;
}

template <typename T> int launch_typed(const jdob_problem *q, const jdob_policy *o, hipStream_t stream) {
  HArgs<T> a;
  a.p = to_hproblem<T>(q);
  HPolicy<T> &r = a.out;
  r.status = o->status;
  r.cut = o->cut;
  r.gpu_level = o->gpu_level;
  r.batch = o->batch;
  r.energy = (T *)o->energy;
  r.tfree_out = (T *)o->t_free_out;
  r.ulevel = o->user_level;
  r.uoffload = o->user_offload;
  r.nfeas = o->num_feasible;
  r.nevals = o->num_user_evals;
  r.ufreq = (T *)o->user_freq;
  const bool greedy = (q->mode & JDOB_MODE_GREEDY) != 0;
  const bool cont = (q->mode & JDOB_MODE_CONTINUOUS_CPU) != 0;
  const bool count = r.nfeas != nullptr || r.nevals != nullptr;
  const size_t lds = (size_t)make_hlayout(a.p.N, a.p.L, a.p.K, a.p.J, (int)sizeof(T), false).total;
  const int64_t I = q->num_instances;
  const dim3 block(WAVE);
  for (int64_t first = 0; first < I; first += MAX_BLOCKS_PER_LAUNCH) {
    const int64_t n = (I - first < MAX_BLOCKS_PER_LAUNCH) ? I - first : MAX_BLOCKS_PER_LAUNCH;
    const dim3 grid((unsigned)n);
    a.first = first;
#define JDOB_HLAUNCH(CN, GR, CT) \
  hipLaunchKernelGGL((jdob_hetero_kernel<T, CN, GR, CT>), grid, block, lds, stream, a)
    if (count) {
      if (greedy) { if (cont) JDOB_HLAUNCH(true, true, true); else JDOB_HLAUNCH(true, true, false); }
      else { if (cont) JDOB_HLAUNCH(true, false, true); else JDOB_HLAUNCH(true, false, false); }
    } else if (cont) {
      if (greedy) JDOB_HLAUNCH(false, true, true);
      else JDOB_HLAUNCH(false, false, true);
    } else {
      // level rows of K4 = 2^lg entries, 4 <= K4 <= 64 (K <= JDOB_MAX_LOCAL_LEVELS)
      static_assert(JDOB_MAX_LOCAL_LEVELS <= 64, "hetero level rows of at most 2^6 entries");
#define JDOB_HLG(G)                                                                         \
  case G:                                                                                   \
    if (greedy)                                                                             \
      hipLaunchKernelGGL((jdob_hetero_kernel<T, false, true, false, G>), grid, block, lds,  \
                         stream, a);                                                        \
    else                                                                                    \
      hipLaunchKernelGGL((jdob_hetero_kernel<T, false, false, false, G>), grid, block, lds, \
                         stream, a);                                                        \
    break;
      switch (__builtin_ctz((unsigned)make_hlayout(a.p.N, a.p.L, a.p.K, a.p.J, (int)sizeof(T),
                                                   false).K4)) {
        JDOB_HLG(2) JDOB_HLG(3) JDOB_HLG(4) JDOB_HLG(5) JDOB_HLG(6)
        default: return JDOB_ERR_UNSUPPORTED;
      }
#undef JDOB_HLG
    }
#undef JDOB_HLAUNCH
    if (hipGetLastError() != hipSuccess) return JDOB_ERR_HIP;
  }
  return JDOB_OK;
}

template <typename T>
int launch_grouped_typed(const jdob_problem *q, const jdob_grouped_policy *o, hipStream_t stream) {
  HGArgs<T> a;
  a.p = to_hproblem<T>(q);
  HGrouped<T> &g = a.out;
  g.status = o->status;
  g.num_groups = o->num_groups;
  g.energy = (T *)o->energy;
  g.tfree_out = (T *)o->t_free_out;
  g.order = o->order;
  g.group_end = o->group_end;
  g.group_cut = o->group_cut;
  g.group_gpu_level = o->group_gpu_level;
  g.group_batch = o->group_batch;
  g.group_energy = (T *)o->group_energy;
  g.group_tfree = (T *)o->group_t_free;
  g.ulevel = o->user_level;
  g.uoffload = o->user_offload;
  g.ugroup = o->user_group;
  g.ninner = o->num_inner;
  g.nfeas = o->num_feasible;
  g.nevals = o->num_user_evals;
  g.ufreq = (T *)o->user_freq;
  const bool greedy = (q->mode & JDOB_MODE_GREEDY) != 0;
  const bool cont = (q->mode & JDOB_MODE_CONTINUOUS_CPU) != 0;
  const bool count = g.ninner != nullptr || g.nfeas != nullptr || g.nevals != nullptr;
  const size_t lds = (size_t)make_hlayout(a.p.N, a.p.L, a.p.K, a.p.J, (int)sizeof(T), true).total;
  const int64_t I = q->num_instances;
  const dim3 block(WAVE);
  for (int64_t first = 0; first < I; first += MAX_BLOCKS_PER_LAUNCH) {
    const int64_t n = (I - first < MAX_BLOCKS_PER_LAUNCH) ? I - first : MAX_BLOCKS_PER_LAUNCH;
    const dim3 grid((unsigned)n);
    a.first = first;
#define JDOB_HLAUNCH(CN, GR, CT) \
  hipLaunchKernelGGL((jdob_hetero_grouped_kernel<T, CN, GR, CT>), grid, block, lds, stream, a)
    if (count) {
      if (greedy) { if (cont) JDOB_HLAUNCH(true, true, true); else JDOB_HLAUNCH(true, true, false); }
      else { if (cont) JDOB_HLAUNCH(true, false, true); else JDOB_HLAUNCH(true, false, false); }
    } else {
      if (greedy) { if (cont) JDOB_HLAUNCH(false, true, true); else JDOB_HLAUNCH(false, true, false); }
      else { if (cont) JDOB_HLAUNCH(false, false, true); else JDOB_HLAUNCH(false, false, false); }
    }
#undef JDOB_HLAUNCH
    if (hipGetLastError() != hipSuccess) return JDOB_ERR_HIP;
  }
  return JDOB_OK;
}

}  // namespace

bool has_user_params(const jdob_problem *p) {
  return p->user_zeta || p->user_kappa || p->user_p_tx || p->user_local_freq;
}

// Checks beyond the shared ones (done before): the user count and the LDS
// the instance needs.
int validate_hetero(const jdob_problem *p, bool grouped) {
  if (p->num_users > JDOB_MAX_HETERO_USERS) return JDOB_ERR_UNSUPPORTED;
  const int sz = p->dtype == JDOB_F64 ? 8 : 4;
  if (make_hlayout(p->num_users, p->num_layers, p->num_local_levels, p->num_gpu_levels, sz,
                   grouped)
          .limit > LDS_LIMIT)
    return JDOB_ERR_UNSUPPORTED;
  return JDOB_OK;
}

int launch_hetero(const jdob_problem *p, const jdob_policy *o, hipStream_t stream) {
  return p->dtype == JDOB_F64 ? launch_typed<double>(p, o, stream) : launch_typed<float>(p, o, stream);
}

int launch_hetero_grouped(const jdob_problem *p, const jdob_grouped_policy *o, hipStream_t stream) {
  return p->dtype == JDOB_F64 ? launch_grouped_typed<double>(p, o, stream)
                              : launch_grouped_typed<float>(p, o, stream);
}

}  // namespace jdob_dev
