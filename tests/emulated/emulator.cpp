// The fibers and the schedule of the CPU stand-in (hip/hip_runtime.h), and stand-ins for the launchers of the
// sources that are not compiled for the CPU. Test infrastructure, not part of libsts.so.
#include <link.h>
#include <sched.h>
#include <stdio.h>
#include <stdlib.h>
#include <sys/mman.h>

#include <string>
#include <thread>
#include <vector>

#include "common.h"

namespace emu {

thread_local Lane *lane = nullptr;
thread_local uint64_t loaded = 0;
thread_local const void *recent[128];

namespace {
constexpr size_t STACK = 64 * 1024;
int g_slow_wave = -1, g_slow_part = -1, g_cus = 256;
unsigned g_seed = 1;
uint64_t g_loaded = 0, g_barriers = 0;
uint32_t g_lds = 0;
bool g_only_names = false;
std::string g_names;

enum State { READY, IN_WAVE_OP, AT_BARRIER, SLEEPING, ENDED };
struct Fiber : Lane {
  void *sp;
  State state;
};
struct Wave {
  uint32_t in[2][64];
  uint64_t live;
  int arrived, gen, sleeps;
};
struct Group {
  std::vector<Fiber> fibers;
  std::vector<Wave> waves;
  char *stacks;
  void *sched_sp;
  void (*body)(void *);
  void *arg;
  int live, at_barrier;
  Fiber *cur;
};
thread_local Group *g_group = nullptr;

// saves the callee-saved registers on the stack, stores the stack pointer to *from and goes on at `to`
extern "C" void emu_switch(void **from, void *to);
asm(R"(
.text
.globl emu_switch
emu_switch:
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

void leave(State s) {
  Group *g = g_group;
  Fiber *f = g->cur;
  f->state = s;
  emu_switch(&f->sp, g->sched_sp);
}

Wave &wave_of(Group *g) { return g->waves[g->cur->thread.x >> 6]; }

void release_wave(Group *g, int w) {
  Wave &wv = g->waves[w];
  if (wv.arrived == 0 || wv.arrived < __builtin_popcountll(wv.live)) return;
  wv.arrived = 0;
  ++wv.gen;
  for (int l = 0; l < 64; ++l)
    if (g->fibers[64 * w + l].state == IN_WAVE_OP) g->fibers[64 * w + l].state = READY;
}
void release_barrier(Group *g) {
  if (g->at_barrier == 0 || g->at_barrier < g->live) return;
  g->at_barrier = 0;
  for (Fiber &f : g->fibers)
    if (f.state == AT_BARRIER) f.state = READY;
}

void fiber_main() {
  Group *g = g_group;
  g->body(g->arg);
  Wave &wv = wave_of(g);
  const int w = (int)(g->cur->thread.x >> 6), l = (int)(g->cur->thread.x & 63u);
  wv.live &= ~(1ull << l);
  wv.in[0][l] = wv.in[1][l] = 0;
  --g->live;
  release_wave(g, w);
  release_barrier(g);
  leave(ENDED);
  abort();
}

// LDS holds anything when a workgroup begins: every thread-local word of this library gets the value that was asked for
int fill_lds(struct dl_phdr_info *info, size_t, void *) {
  const ElfW(Addr) here = reinterpret_cast<ElfW(Addr)>(&g_lds) - info->dlpi_addr;
  bool mine = false;
  for (int i = 0; i < info->dlpi_phnum; ++i) {
    const ElfW(Phdr) &h = info->dlpi_phdr[i];
    mine |= h.p_type == PT_LOAD && here >= h.p_vaddr && here < h.p_vaddr + h.p_memsz;
  }
  for (int i = 0; mine && i < info->dlpi_phnum; ++i)
    if (info->dlpi_phdr[i].p_type == PT_TLS)
      for (size_t w = 0; w < info->dlpi_phdr[i].p_memsz / 4; ++w) static_cast<uint32_t *>(info->dlpi_tls_data)[w] = g_lds;
  return mine;
}

void run_group(Group *g, dim3 block, dim3 where) {
  loaded = 0;                                          // (this module's thread-local memory exists from here on)
  if (g_lds) dl_iterate_phdr(fill_lds, nullptr);
  loaded = 0;
  g_group = g;
  const int n = (int)block.x, nw = n / 64;
  g->fibers.assign(n, Fiber());
  g->waves.assign(nw, Wave());
  g->live = n;
  g->at_barrier = 0;
  for (Wave &w : g->waves) w.live = ~0ull;
  for (int i = 0; i < n; ++i) {
    Fiber &f = g->fibers[i];
    f.thread = dim3((unsigned)i, 0, 0);
    f.block = where;
    f.state = READY;
    void **top = reinterpret_cast<void **>(g->stacks + (size_t)(i + 1) * STACK) - 2;
    *top = reinterpret_cast<void *>(fiber_main);       // popped by ret; six registers below it
    f.sp = top - 6;
  }
  const int slow = (int)where.x == g_slow_part ? g_slow_wave : -1;
  unsigned rng = g_seed * 2654435761u + where.x * 40503u + where.y * 977u + 12345u;
  std::vector<int> can;
  while (g->live > 0) {
    // waves with a work-item that can run; one that only sleeps wakes when it is chosen
    can.clear();
    bool slow_can = false, all_patient = true;
    for (int w = 0; w < nw; ++w) {
      bool ready = false, asleep = false;
      for (int l = 0; l < 64; ++l) {
        const State s = g->fibers[64 * w + l].state;
        ready |= s == READY;
        asleep |= s == SLEEPING;
      }
      if (!ready && !asleep) continue;
      if (w == slow) {
        slow_can = true;
        continue;
      }
      if (ready || g->waves[w].sleeps < 3000) all_patient = false;
      can.push_back(w);
    }
    int w;
    if (slow_can && all_patient) w = slow;             // nobody else can go on, or they have waited long
    else if (!can.empty()) w = can[(rng = rng * 1664525u + 1013904223u) / 65536u % can.size()];
    else {
      fprintf(stderr, "emulated workgroup %u,%u: its work-items wait for each other at different places\n", where.x, where.y);
      exit(4);
    }
    for (int l = 0; l < 64; ++l)
      if (g->fibers[64 * w + l].state == SLEEPING) {
        g->fibers[64 * w + l].state = READY;
        if (l == __builtin_ctzll(g->waves[w].live)) {
          ++g->waves[w].sleeps;
          sched_yield();
        }
      }
    for (int l = 0; l < 64; ++l) {
      Fiber &f = g->fibers[64 * w + l];
      if (f.state != READY) continue;
      g->cur = &f;
      lane = &f;
      emu_switch(&g->sched_sp, f.sp);
    }
  }
}
}  // namespace

const uint32_t *exchange(uint32_t v) {
  Group *g = g_group;
  Wave &wv = wave_of(g);
  const int at = wv.gen & 1;
  wv.in[at][g->cur->thread.x & 63u] = v;
  ++wv.arrived;
  const int w = (int)(g->cur->thread.x >> 6);
  if (wv.arrived == __builtin_popcountll(wv.live)) release_wave(g, w);
  else leave(IN_WAVE_OP);
  return wv.in[at];
}
uint64_t live() { return wave_of(g_group).live; }
void barrier() {
  Group *g = g_group;
  if (g->cur->thread.x == 0) __atomic_fetch_add(&g_barriers, 1, __ATOMIC_SEQ_CST);
  wave_of(g).sleeps = 0;
  ++g->at_barrier;
  g->cur->state = AT_BARRIER;
  release_barrier(g);
  if (g->cur->state == AT_BARRIER) leave(AT_BARRIER);
}
void sleep() { leave(SLEEPING); }

bool noted(const char *kernel) {
  std::string name = kernel;
  if (name[0] == '(') name = name.substr(1, name.size() - 2);
  if (g_only_names) g_names += (g_names.empty() ? "" : " ") + name;
  return g_only_names;
}

// Workgroups start in the order of their ids, a few at a time, each on a thread of its own: the parts of a row
// run side by side, and every workgroup's LDS (thread-local statics) is its own.
void launch(void (*body)(void *), void *arg, dim3 grid, dim3 block) {
  const unsigned total = grid.x * grid.y * grid.z, at_once = grid.x > 8 ? grid.x : 8 / grid.x * grid.x;
  for (unsigned first = 0; first < total; first += at_once) {
    std::vector<std::thread> threads;
    for (unsigned b = first; b < total && b < first + at_once; ++b)
      threads.emplace_back([=] {
        Group g;
        g.body = body;
        g.arg = arg;
        const size_t bytes = block.x * STACK;
        g.stacks = static_cast<char *>(mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0));
        run_group(&g, block, dim3(b % grid.x, b / grid.x % grid.y, b / grid.x / grid.y));
        munmap(g.stacks, bytes);
        __atomic_fetch_add(&g_loaded, loaded, __ATOMIC_SEQ_CST);
      });
    for (std::thread &t : threads) t.join();
  }
}
}  // namespace emu

hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = emu::g_cus; return hipSuccess; }

// slow_wave of the workgroups with blockIdx.x == slow_part is held back (-1: none); the seed orders the others
extern "C" void emu_schedule(int seed, int slow_part, int slow_wave) {
  emu::g_seed = (unsigned)seed;
  emu::g_slow_part = slow_part;
  emu::g_slow_wave = slow_wave;
}

// what every word of a workgroup's LDS holds when it begins
extern "C" void emu_lds(uint32_t word) { emu::g_lds = word; }

// launches are noted down by name from here on (1), or run (0)
extern "C" void emu_only_names(int on) {
  emu::g_only_names = on != 0;
  emu::g_names.clear();
}
extern "C" const char *emu_names() { return emu::g_names.c_str(); }

// bytes of scores loaded since the last call
extern "C" uint64_t emu_loaded() { return __atomic_exchange_n(&emu::g_loaded, 0, __ATOMIC_SEQ_CST); }

// barriers that workgroups have passed since the last call
extern "C" uint64_t emu_barriers() { return __atomic_exchange_n(&emu::g_barriers, 0, __ATOMIC_SEQ_CST); }

sts_status sts_static_scratch(void **) { return STS_EUNSUPPORTED; }
hipError_t launch_attn_split(const AttnArgs &a, int d, int nq, bool sparse, hipStream_t) {
  const bool shared = sparse && attn_shares_cache(a, d, d == 128 && nq == 2);
  return emu::noted(shared ? "attn_split shared" : "attn_split") ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_attn_combine(const AttnArgs &, int, int, hipStream_t) {
  return emu::noted("attn_combine") ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_attn_probsum(const AttnArgs &, int, int, hipStream_t) { return hipErrorInvalidValue; }
int attn_probsum_wgs_per_cu(int, int) { return 1; }
