// Test infrastructure: a workgroup of 256 lanes on the CPU.  Every lane is a fiber; an operation
// across the lanes of a wave (or a barrier) is a rendezvous of its 64 (256) fibers, and a lane that
// arrives with another operation than its wave, or never, ends the program.  Lanes run one at a
// time, so data races are not shown; wrong addresses are (the buffers are built with
// AddressSanitizer around them).
#pragma once
#include <functional>

#include <stdio.h>
#include <stdlib.h>

namespace host_wave {

constexpr int kLanes = 256, kStack = 1 << 17;

extern "C" void host_wave_switch(void** save, void* load);
asm(R"(
.text
.globl host_wave_switch
host_wave_switch:
  pushq %rbp
  pushq %rbx
  pushq %r12
  pushq %r13
  pushq %r14
  pushq %r15
  movq %rsp, (%rdi)
  movq %rsi, %rsp
  popq %r15
  popq %r14
  popq %r13
  popq %r12
  popq %rbx
  popq %rbp
  ret
)");

struct Meeting {                          // of the 64 lanes of a wave or the 256 of the workgroup
  int arrived = 0, op = 0;
  unsigned turn = 0;
  uint64_t in[kLanes], out[2][kLanes];    // a lane is at most one turn ahead of the slowest
};

inline Meeting waves[4], group;
inline void* sp[kLanes];
inline void* main_sp;
inline char* stacks;
inline bool done[kLanes];
inline int current, left;
inline long idle;                         // switches since the last completed meeting
inline std::function<void()> body;

[[noreturn]] inline void die(const char* what) {
  fprintf(stderr, "host_wave: lane %d: %s\n", current, what);
  fflush(stderr);
  abort();
}

inline void leave() {                     // to the next live lane, or back to run()
  const int from = current;
  if (++idle > 8 * kLanes) die("some lanes wait for an operation that the others never reach");
  int to = from;
  do to = (to + 1) % kLanes; while (done[to] && to != from);
  if (to == from && done[to]) { host_wave_switch(&sp[from], main_sp); return; }
  current = to;
  if (to != from) host_wave_switch(&sp[from], sp[to]);
}

// All lanes of the meeting hand in a value and get everybody's.
inline const uint64_t* meet(Meeting& m, int size, int op, uint64_t v) {
  if (m.arrived == 0) m.op = op;
  if (m.op != op) die("diverged from its wave at a cross-lane operation");
  const int me = current % size;
  m.in[me] = v;
  const unsigned turn = m.turn;
  if (++m.arrived == size) {
    memcpy(m.out[turn & 1], m.in, sizeof(m.in));
    m.arrived = 0;
    ++m.turn;
    idle = 0;
  } else {
    while (m.turn == turn) leave();
  }
  return m.out[turn & 1];
}
inline const uint64_t* in_wave(int op, uint64_t v) { return meet(waves[current >> 6], 64, op, v); }

inline void entry() {
  body();
  done[current] = true;
  --left;
  idle = 0;
  leave();
  die("woken after its end");
}

// Runs f by every lane of one workgroup.
inline void run(std::function<void()> f) {
  if (!stacks) stacks = (char*)malloc((size_t)kLanes * kStack);
  body = std::move(f);
  for (Meeting& m : waves) m.arrived = 0;
  group.arrived = 0;
  left = kLanes;
  idle = 0;
  for (int i = 0; i < kLanes; ++i) {
    done[i] = false;
    void** top = (void**)(stacks + (size_t)(i + 1) * kStack - 64);
    *--top = nullptr;                     // alignment of the entry's frame
    *--top = (void*)entry;
    for (int r = 0; r < 6; ++r) *--top = nullptr;
    sp[i] = top;
  }
  current = 0;
  host_wave_switch(&main_sp, sp[0]);
  if (left != 0) die("the workgroup ended without all of its lanes");
}

struct LaneIndex {
  operator int() const { return current; }
  int operator>>(int n) const { return current >> n; }
  int operator&(int n) const { return current & n; }
};
struct Index { LaneIndex x; };

}  // namespace host_wave

static const host_wave::Index threadIdx;

enum { kOpBallot = 1, kOpReadlane, kOpFirst, kOpPermute, kOpBarrier, kOpSync, kOpDpp, kOpShuffle };

inline unsigned long long __builtin_amdgcn_ballot_w64(bool p) {
  const uint64_t* v = host_wave::in_wave(kOpBallot, p);
  unsigned long long b = 0;
  for (int i = 0; i < 64; ++i) b |= (v[i] & 1ull) << i;
  return b;
}
inline int __builtin_amdgcn_readlane(int x, int lane) {
  const uint64_t* v = host_wave::in_wave(kOpReadlane, (uint32_t)x);
  if (lane < 0 || lane > 63) host_wave::die("readlane of a lane outside the wave");
  return (int)(uint32_t)v[lane];
}
inline int __builtin_amdgcn_readfirstlane(int x) { return (int)(uint32_t)host_wave::in_wave(kOpFirst, (uint32_t)x)[0]; }
inline int __builtin_amdgcn_ds_bpermute(int at, int x) {
  return (int)(uint32_t)host_wave::in_wave(kOpPermute, (uint32_t)x)[(at >> 2) & 63];
}
inline void __builtin_amdgcn_wave_barrier() { host_wave::in_wave(kOpBarrier, 0); }
inline void __builtin_amdgcn_fence(int, const char*) {}
inline void __builtin_amdgcn_sched_barrier(int) {}
inline void __syncthreads() { host_wave::meet(host_wave::group, host_wave::kLanes, kOpSync, 0); }

// The data-parallel shifts in use: row_shr:n (0x110 + n), wave_shr:1 (0x138), row_bcast:15 (0x142) and
// row_bcast:31 (0x143).  A lane without a source, or in a row that the mask leaves out, keeps `old`.
inline int __builtin_amdgcn_update_dpp(int old, int x, int ctrl, int rows, int banks, bool) {
  const uint64_t* v = host_wave::in_wave(kOpDpp, (uint32_t)x);
  const int lane = host_wave::current & 63, row = lane >> 4;
  int from = -1;
  if (ctrl > 0x110 && ctrl <= 0x11f) from = (lane & 15) >= (ctrl & 15) ? lane - (ctrl & 15) : -1;
  else if (ctrl == 0x138) from = lane - 1;
  else if (ctrl == 0x142) from = row > 0 ? row * 16 - 1 : -1;
  else if (ctrl == 0x143) from = row > 1 ? 31 : -1;
  else host_wave::die("unknown data-parallel shift");
  if (banks != 0xf) host_wave::die("bank masks are not modelled");
  return from >= 0 && ((rows >> row) & 1) ? (int)(uint32_t)v[from] : old;
}

inline float __shfl_xor(float x, int d, int) {
  return __int_as_float((int)(uint32_t)host_wave::in_wave(kOpShuffle, (uint32_t)__float_as_int(x))[(host_wave::current & 63) ^ d]);
}
inline int __shfl_xor(int x, int d, int) {
  return (int)(uint32_t)host_wave::in_wave(kOpShuffle, (uint32_t)x)[(host_wave::current & 63) ^ d];
}

template <typename T>
inline T atomicAdd(T* p, T v) { const T old = *p; *p = old + v; return old; }
