// A 64-lane wave on the CPU: what the kernels' sources use of the HIP runtime
// and of the gfx950 builtins, so that they compile as C++ and run one
// workgroup of one wave at a time, for tests that check where a kernel reads
// and writes without a GPU.
//
// The lanes are coroutines.  Each runs until it meets an operation that
// involves the others (a barrier, a ballot, a lane move); when all lanes still
// running have arrived there, each goes on with its result.  Lanes that meet
// different operations there end the run with a message.  The LDS block
// is exactly as long as the launch asks for (to its 32-byte alignment): a page
// that may not be touched follows, the bytes between are checked, and a fresh
// block is filled with NaN patterns.  Pages that may not be touched surround
// nothing else: global arrays are the caller's.
#ifndef WAVE_CPU_H
#define WAVE_CPU_H

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <math.h>
#include <stdint.h>
#include <sys/mman.h>
#include <type_traits>
#include <utility>

namespace wave_cpu {

constexpr int LANES = 64;
constexpr size_t STACK = 256 * 1024;
constexpr size_t LDS_PAGES = 160 * 1024;

struct Wave {
  void *sp[LANES];        // suspended lanes' stack pointers
  void *main_sp;
  char *stack[LANES];
  int next[LANES];        // ring of the lanes still running
  int prev[LANES];
  int lane = 0, live = 0;
  unsigned seq[LANES];    // operations met by each lane
  struct Slot { unsigned seq; const char *kind; uint64_t v; } slot[2][LANES];
  unsigned char *pages = nullptr, *lds = nullptr;
  size_t lds_bytes = 0;
  const void *kernarg = nullptr;
  unsigned block = 0, grid = 0;
  bool descending = false;  // the order in which lanes run between two operations
  void (*body)(void *) = nullptr;
  void *body_arg = nullptr;
};

inline Wave &w() {
  static Wave x;
  return x;
}

// Saves the callee-saved registers and the stack pointer at *from, and goes on
// at `to`.
extern "C" void wave_cpu_switch(void **from, void *to);
asm(".text\n.weak wave_cpu_switch\n.type wave_cpu_switch,@function\nwave_cpu_switch:\n"
    "  push %rbp\n  push %rbx\n  push %r12\n  push %r13\n  push %r14\n  push %r15\n"
    "  mov %rsp, (%rdi)\n  mov %rsi, %rsp\n"
    "  pop %r15\n  pop %r14\n  pop %r13\n  pop %r12\n  pop %rbx\n  pop %rbp\n  ret\n"
    ".size wave_cpu_switch, .-wave_cpu_switch\n");

[[noreturn]] inline void die(const char *what) {
  fprintf(stderr, "wave_cpu: %s (block %u, lane %d)\n", what, w().block, w().lane);
  fflush(stderr);
  abort();
}

inline void lane_main() {
  Wave &x = w();
  x.body(x.body_arg);
  const int me = x.lane, to = x.next[me];
  x.next[x.prev[me]] = to;
  x.prev[to] = x.prev[me];
  void *dead;
  if (--x.live == 0) wave_cpu_switch(&dead, x.main_sp);
  x.lane = to;
  wave_cpu_switch(&dead, x.sp[to]);
  abort();
}

// Every running lane's v at this operation; returns the slots.
inline const Wave::Slot *meet(const char *kind, uint64_t v, uint64_t *present) {
  Wave &x = w();
  const int me = x.lane;
  const unsigned n = ++x.seq[me];
  Wave::Slot *s = x.slot[n & 1];
  s[me] = {n, kind, v};
  const int to = x.next[me];
  if (to != me) {
    x.lane = to;
    wave_cpu_switch(&x.sp[me], x.sp[to]);
    x.lane = me;
  }
  uint64_t m = 0;
  for (int l = 0; l < LANES; ++l)
    if (s[l].seq == n) {
      if (s[l].kind != kind && strcmp(s[l].kind, kind) != 0) {
        fprintf(stderr, "wave_cpu: lane %d at %s, lane %d at %s\n", l, s[l].kind, me, kind);
        die("lanes meet different operations");
      }
      m |= uint64_t(1) << l;
    }
  *present = m;
  return s;
}

template <typename V> inline uint64_t bits(V v) {
  uint64_t u = 0;
  memcpy(&u, &v, sizeof v);
  return u;
}
template <typename V> inline V value(uint64_t u) {
  V v;
  memcpy(&v, &u, sizeof v);
  return v;
}

inline void barrier() {
  uint64_t p;
  meet("barrier", 0, &p);
}
inline uint64_t ballot(bool b) {
  uint64_t p, r = 0;
  const Wave::Slot *s = meet("ballot", b, &p);
  for (int l = 0; l < LANES; ++l)
    if ((p >> l) & 1) r |= s[l].v << l;
  return r;
}
template <typename V> inline V lane_value(const char *kind, V v, int from) {
  uint64_t p;
  const Wave::Slot *s = meet(kind, bits(v), &p);
  if (from < 0 || from >= LANES || !((p >> from) & 1)) die("a value of a lane that is not there");
  return value<V>(s[from].v);
}

inline unsigned char *lds() { return w().lds; }

template <typename F> void run_block(F &&f, unsigned block, unsigned grid, size_t lds_bytes,
                                     const void *kernarg) {
  Wave &x = w();
  if (!x.pages) {
    x.pages = (unsigned char *)mmap(nullptr, LDS_PAGES + 4096, PROT_READ | PROT_WRITE,
                                    MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (x.pages == MAP_FAILED || mprotect(x.pages + LDS_PAGES, 4096, PROT_NONE)) die("mmap");
    for (int l = 0; l < LANES; ++l) x.stack[l] = (char *)malloc(STACK);
  }
  if (lds_bytes > LDS_PAGES) die("launch asks for more LDS than there is");
  const size_t room = (lds_bytes + 31) & ~size_t(31);
  x.lds = x.pages + LDS_PAGES - room;
  x.lds_bytes = lds_bytes;
  memset(x.lds, 0xff, room);
  x.block = block;
  x.grid = grid;
  x.kernarg = kernarg;
  x.live = LANES;
  using G = typename std::remove_reference<F>::type;
  x.body = [](void *g) { (*(G *)g)(); };
  x.body_arg = &f;
  for (int l = 0; l < LANES; ++l) {
    const int up = (l + 1) % LANES, down = (l + LANES - 1) % LANES;
    x.next[l] = x.descending ? down : up;
    x.prev[l] = x.descending ? up : down;
    x.seq[l] = 0;
    x.slot[0][l].seq = x.slot[1][l].seq = 0;
    uintptr_t top = ((uintptr_t)x.stack[l] + STACK) & ~uintptr_t(63);
    void **sp = (void **)top;
    *--sp = nullptr;                 // (alignment at entry: a call pushes 8 bytes)
    *--sp = (void *)&lane_main;      // returned to by the switch
    for (int r = 0; r < 6; ++r) *--sp = nullptr;
    x.sp[l] = sp;
  }
  x.lane = x.descending ? LANES - 1 : 0;
  wave_cpu_switch(&x.main_sp, x.sp[x.lane]);
  for (size_t i = lds_bytes; i < room; ++i)
    if (x.lds[i] != 0xff) {
      fprintf(stderr, "wave_cpu: LDS byte %zu written, the launch has %zu\n", i, lds_bytes);
      die("LDS written past the launch's block");
    }
}

extern "C" inline void __attribute__((used)) wave_cpu_descending(int on) { w().descending = on != 0; }

struct Dim { unsigned x; };
template <typename V> struct Pair {
  V v[2];
  V operator[](int i) const { return v[i]; }
};

}  // namespace wave_cpu

// ---- the runtime
struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
typedef struct ihipStream_t *hipStream_t;
enum hipError_t { hipSuccess = 0 };
inline hipError_t hipGetLastError() { return hipSuccess; }

template <typename A, typename... Rest> inline const void *first_arg(const A &a, const Rest &...) {
  return &a;
}
#define hipLaunchKernelGGL(KERNEL, GRID, BLOCK, LDS, STREAM, ...)                                 \
  do {                                                                                            \
    (void)(STREAM);                                                                               \
    if ((BLOCK).x != wave_cpu::LANES) wave_cpu::die("only workgroups of one wave");               \
    for (unsigned b_ = 0; b_ < (GRID).x; ++b_)                                                    \
      wave_cpu::run_block([&] { KERNEL(__VA_ARGS__); }, b_, (GRID).x, LDS, first_arg(__VA_ARGS__)); \
  } while (0)

#define __global__
#define __device__
#define __host__
#define __align__(n) alignas(n)
#define __launch_bounds__(...)
#define __forceinline__ inline
#define threadIdx (wave_cpu::Dim{(unsigned)wave_cpu::w().lane})
#define blockIdx (wave_cpu::Dim{wave_cpu::w().block})
#define gridDim (wave_cpu::Dim{wave_cpu::w().grid})
#define __syncthreads() wave_cpu::barrier()

struct alignas(16) ulonglong2 { unsigned long long x, y; };

inline int __float_as_int(float v) { return wave_cpu::value<int>(wave_cpu::bits(v)); }
inline unsigned __float_as_uint(float v) { return (unsigned)__float_as_int(v); }
inline float __uint_as_float(unsigned v) { return wave_cpu::value<float>(wave_cpu::bits(v)); }
inline float __int_as_float(int v) { return wave_cpu::value<float>(wave_cpu::bits(v)); }
inline long long __double_as_longlong(double v) { return wave_cpu::value<long long>(wave_cpu::bits(v)); }
inline double __longlong_as_double(long long v) { return wave_cpu::value<double>(wave_cpu::bits(v)); }
inline int min(int a, int b) { return a < b ? a : b; }
inline int __clz(int v) { return v ? __builtin_clz((unsigned)v) : 32; }
inline int __clzll(long long v) { return v ? __builtin_clzll((unsigned long long)v) : 64; }
inline int __popcll(unsigned long long v) { return __builtin_popcountll(v); }

inline unsigned long long __ballot(bool b) { return wave_cpu::ballot(b); }
template <typename V> inline V __shfl_xor(V v, int m, int = 64) {
  return wave_cpu::lane_value("shfl_xor", v, wave_cpu::w().lane ^ m);
}
template <typename V> inline V __shfl_down(V v, int d, int width = 64) {
  const int l = wave_cpu::w().lane, to = (l & (width - 1)) + d;
  return wave_cpu::lane_value("shfl_down", v, to < width ? l + d : l);
}

// ---- the builtins
#define __builtin_amdgcn_ballot_w64(b) wave_cpu::ballot(b)
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_wave_barrier() wave_cpu::barrier()
#define __builtin_amdgcn_kernarg_segment_ptr() wave_cpu::w().kernarg
#define __builtin_amdgcn_readlane(v, l) wave_cpu::lane_value<int>("readlane", (v), (l))
#define __builtin_amdgcn_readfirstlane(v) wave_cpu_first(v)
#define __builtin_amdgcn_mbcnt_lo(m, b) \
  (unsigned)((b) + __builtin_popcount((unsigned)(m) & (unsigned)wave_cpu_below()))
#define __builtin_amdgcn_mbcnt_hi(m, b) \
  (unsigned)((b) + __builtin_popcount((unsigned)(m) & (unsigned)(wave_cpu_below() >> 32)))
#define __builtin_amdgcn_permlane32_swap(a, b, fi, bc) wave_cpu_swap32(a, b)
#define __builtin_amdgcn_update_dpp wave_cpu_dpp

inline uint64_t wave_cpu_below() { return (uint64_t(1) << wave_cpu::w().lane) - 1; }
inline int wave_cpu_first(int v) {
  uint64_t p;
  const wave_cpu::Wave::Slot *s = wave_cpu::meet("readfirstlane", wave_cpu::bits(v), &p);
  return wave_cpu::value<int>(s[__builtin_ctzll(p)].v);
}
inline wave_cpu::Pair<int> wave_cpu_swap32(int a, int b) {
  const int l = wave_cpu::w().lane;
  const int lo = wave_cpu::lane_value("permlane32", b, l & 31);
  const int hi = wave_cpu::lane_value("permlane32", a, l | 32);
  return {{l < 32 ? a : lo, l < 32 ? hi : b}};
}
inline int wave_cpu_dpp(int old, int v, int ctrl, int row_mask, int bank_mask, bool bound) {
  using namespace wave_cpu;
  const int l = w().lane, row = l >> 4, q = l & 15;
  uint64_t p;
  const Wave::Slot *s = meet("dpp", bits(v), &p);
  int from = -1;
  if (ctrl <= 0xff) from = (l & ~3) + ((ctrl >> (2 * (l & 3))) & 3);
  else if (ctrl > 0x100 && ctrl < 0x110) from = q + (ctrl & 15) < 16 ? l + (ctrl & 15) : -1;
  else if (ctrl > 0x110 && ctrl < 0x120) from = q - (ctrl & 15) >= 0 ? l - (ctrl & 15) : -1;
  else if (ctrl == 0x138) from = l - 1;
  else if (ctrl == 0x140) from = (l & ~15) + 15 - q;
  else if (ctrl == 0x141) from = (l & ~7) + 7 - (l & 7);
  else if (ctrl == 0x142) from = row ? (row << 4) - 1 : -1;
  else if (ctrl == 0x143) from = row > 1 ? 31 : -1;
  else die("unknown lane move");
  if (!((row_mask >> row) & 1) || !((bank_mask >> ((l >> 2) & 3)) & 1)) return old;
  if (from < 0 || !((p >> from) & 1)) return bound ? 0 : old;
  return value<int>(s[from].v);
}

// (one ulp of the hardware's reciprocals is not modelled; its flush of binary32
// denormals is)
inline float __builtin_amdgcn_rcpf(float x) {
  const float tiny = std::numeric_limits<float>::min();
  if (std::fabs(x) < tiny) return std::copysign(INFINITY, x);
  const float q = 1.0f / x;
  return std::fabs(q) < tiny ? std::copysign(0.0f, q) : q;
}
inline double __builtin_amdgcn_rcp(double x) { return 1.0 / x; }
inline float __builtin_amdgcn_fmed3f(float a, float b, float c) {
  return std::fmax(std::fmin(a, b), std::fmin(std::fmax(a, b), c));
}

#endif  // WAVE_CPU_H
