// The scheduler of hip/hip_runtime.h.
#include <hip/hip_runtime.h>

#include <numeric>
#include <random>

#include "common.hpp"

namespace hull {
// dynamic LDS by the names the kernels give it
__align__(16) unsigned char dyn_lds[163840];
__align__(16) int range_lds[163840 / 4];
__align__(16) unsigned long long best[163840 / 8];
}  // namespace hull

namespace emu {
State g;

asm(R"(
.text
.globl emu_switch
.type emu_switch, @function
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
.size emu_switch, .-emu_switch
)");

// A fiber runs thread after thread; one that waits keeps its fiber.
static void run_threads() {
  for (;;) {
    Fiber* f = g.cur;
    while (g.next < g.threads) {
      f->thread = g.thread_of(g.next++);
      g.of[f->thread] = f;
      g.body();
      g.of[f->thread] = nullptr;
      f->thread = -1;
    }
    emu_switch(&f->sp, g.main_sp);
  }
}

static Fiber* idle_fiber() {
  for (auto& f : g.pool)
    if (f->thread < 0) return f.get();
  constexpr size_t kStack = 256 << 10;
  auto f = std::make_unique<Fiber>();
  f->stack.reset(new char[kStack]);
  void** sp = (void**)(((uintptr_t)f->stack.get() + kStack) & ~(uintptr_t)15);
  *--sp = nullptr;  // (alignment on entry)
  *--sp = (void*)run_threads;
  for (int k = 0; k < 6; ++k) *--sp = nullptr;
  f->sp = sp;
  g.pool.push_back(std::move(f));
  return g.pool.back().get();
}

static void resume(Fiber* f) {
  f->wait = kNone;
  g.cur = f;
  emu_switch(&g.main_sp, f->sp);
}

void wait_block() {
  Fiber* f = g.cur;
  f->wait = kBlock;
  emu_switch(&f->sp, g.main_sp);
}

Fiber* wait_wave(const void* site, unsigned long long x, int group) {
  Fiber* f = g.cur;
  f->wait = kWave;
  f->site = site;
  f->group = group;
  f->in = x;
  emu_switch(&f->sp, g.main_sp);
  return f;
}

// Every live lane of the wave waits: the lanes at one place go on together.
static bool settle_wave(int w0, std::vector<Fiber*>& ready) {
  Fiber* first = nullptr;
  for (int l = 0; l < 64 && w0 + l < g.threads; ++l) {
    Fiber* f = g.of[w0 + l];
    if (f && f->wait == kNone) return false;
    if (f && f->wait == kWave && !first) first = f;
  }
  if (!first) return false;
  const void* site = first->site;
  unsigned long long peers = 0, in[64] = {};
  for (int l = 0; l < 64 && w0 + l < g.threads; ++l) {
    Fiber* f = g.of[w0 + l];
    if (f && f->wait == kWave && f->site == site) {
      peers |= 1ull << l;
      in[l] = f->in;
    }
  }
  for (int k = 0; k < 64; ++k) {
    const int l = g.order ? 63 - k : k;
    if (!((peers >> l) & 1)) continue;
    Fiber* f = g.of[w0 + l];
    f->peers = peers;
    memcpy(f->out, in, sizeof in);
    ready.push_back(f);
  }
  return true;
}

static std::mt19937 rng;  // (the same orders in every run)

static void run_block(const char* name) {
  g.next = 0;
  if (g.order == 2) std::shuffle(g.shuffle.begin(), g.shuffle.end(), rng);
  std::vector<Fiber*> ready;
  for (;;) {
    while (g.next < g.threads) resume(idle_fiber());
    bool live = false;
    ready.clear();
    for (int w0 = 0; w0 < g.threads; w0 += 64) settle_wave(w0, ready);
    if (ready.empty()) {
      bool all = true;
      for (int k = 0; k < g.threads; ++k) {
        Fiber* f = g.of[g.thread_of(k)];
        if (!f) continue;
        live = true;
        all = all && f->wait == kBlock;
        ready.push_back(f);
      }
      if (!live) return;
      if (!all) {
        fprintf(stderr, "emu: %s does not come together\n", name);
        abort();
      }
    }
    if (g.order == 2) std::shuffle(ready.begin(), ready.end(), rng);
    for (Fiber* f : ready) resume(f);
  }
}

void launch(dim3 grid, dim3 block, size_t lds, std::function<void()> body, const char* name) {
  if (lds > sizeof hull::dyn_lds || block.x > 1024 || grid.x == 0 || grid.y == 0) {
    fprintf(stderr, "emu: %s cannot be launched\n", name);
    abort();
  }
  // (no kernel uses more dynamic LDS than it was launched with)
  unsigned char* dyn[] = {hull::dyn_lds, (unsigned char*)hull::range_lds, (unsigned char*)hull::best};
  const size_t guard = std::min<size_t>(sizeof hull::dyn_lds - lds, 8192);
  for (auto d : dyn) memset(d + lds, 0x6b, guard);
  g.body = std::move(body);
  g.grid = grid;
  g.block = block;
  g.threads = (int)block.x;
  g.of.assign(block.x, nullptr);
  g.shuffle.resize(block.x);
  std::iota(g.shuffle.begin(), g.shuffle.end(), 0);
  std::vector<unsigned> blocks(grid.x);
  std::iota(blocks.begin(), blocks.end(), 0u);
  if (!strstr(name, "scan")) {  // (a chained scan waits for the blocks before its own)
    if (g.order == 1) std::reverse(blocks.begin(), blocks.end());
    if (g.order == 2) std::shuffle(blocks.begin(), blocks.end(), rng);
  }
  for (unsigned y = 0; y < grid.y; ++y)
    for (unsigned x : blocks) {
      g.block_idx = dim3(x, y);
      run_block(name);
    }
  for (auto d : dyn)
    for (size_t q = 0; q < guard; ++q)
      if (d[lds + q] != 0x6b) {
        fprintf(stderr, "emu: %s writes past its dynamic LDS\n", name);
        abort();
      }
}
}  // namespace emu

// Threads and workgroups in ascending (0), descending (1) or shuffled (2) order.
extern "C" void emu_order(int order) { emu::g.order = order; }
// Extent and filter, whatever the number of points.
extern "C" int emu_filter(const int32_t* xyz, int64_t n, char* ws, size_t bytes) {
  const hull::Plan pl = hull::make_plan(n, 1);
  if (bytes < pl.total) return HULL_EWORKSPACE;
  hull::init_call((hull::Header*)(ws + pl.header), (int64_t*)(ws + pl.off1), n, ws, pl, nullptr);
  return hull::extent_and_filter<int32_t>(xyz, n, true, ws, pl, nullptr);
}
