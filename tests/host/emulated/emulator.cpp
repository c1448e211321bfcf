// Runs the workgroups of a launch one after the other, each thread as a fibre.  x86-64.
#include <hip/hip_runtime.h>
#include <sys/mman.h>

dim3 blockIdx, gridDim;

extern "C" void emu_switch(void** from, void* to);
asm(R"(
.globl emu_switch
emu_switch:
  pushq %rbp; pushq %rbx; pushq %r12; pushq %r13; pushq %r14; pushq %r15
  movq %rsp, (%rdi)
  movq %rsi, %rsp
  popq %r15; popq %r14; popq %r13; popq %r12; popq %rbx; popq %rbp
  ret
)");

namespace emu {
alignas(16) unsigned dynamic_lds[160 * 1024 / 4];

namespace {
constexpr int MOST = 1024;
constexpr size_t STACK = size_t(64) << 10;
char* stacks;
void *fibre[MOST], *scheduler;
bool ended[MOST];
int now, live, at_barrier, live_in[MOST / 64];
uint64_t barriers, events;
struct Wave {
  uint64_t brought[64], seen[64], round;
  int arrived;
} waves[MOST / 64];
const std::function<void()>* body;

void wait() {
  const int me = now;
  emu_switch(&fibre[me], scheduler);
  now = me;
}
void pass_barrier() {
  if (live > 0 && at_barrier == live) at_barrier = 0, ++barriers;
}
void pass_wave(int w) {
  Wave& x = waves[w];
  if (live_in[w] == 0 || x.arrived != live_in[w]) return;
  memcpy(x.seen, x.brought, sizeof x.seen);
  memset(x.brought, 0, sizeof x.brought);
  x.arrived = 0;
  ++x.round;
}
void run() {
  const int me = now;
  (*body)();
  ended[me] = true;
  ++events;
  --live, --live_in[me / 64];
  pass_barrier();
  pass_wave(me / 64);
  for (;;) emu_switch(&fibre[me], scheduler);
}
}  // namespace

int thread() { return now; }

uint64_t* exchange(uint64_t mine) {
  Wave& x = waves[now / 64];
  const uint64_t round = x.round;
  x.brought[now % 64] = mine;
  ++x.arrived, ++events;
  pass_wave(now / 64);
  while (x.round == round) wait();
  return x.seen;
}

void launch(const char* kernel, dim3 grid, dim3 block, std::function<void()> f) {
  before_launch(kernel);
  if (!stacks) stacks = static_cast<char*>(mmap(nullptr, STACK * MOST, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0));
  gridDim = grid;
  body = &f;
  const int n = static_cast<int>(block.x);
  for (unsigned y = 0; y < grid.y; ++y)
    for (unsigned x = 0; x < grid.x; ++x) {
      blockIdx = dim3(x, y);
      memset(dynamic_lds, 0xcd, sizeof dynamic_lds);
      live = n, at_barrier = 0;
      for (int w = 0; w < MOST / 64; ++w) {
        live_in[w] = std::clamp(n - 64 * w, 0, 64);
        waves[w].arrived = 0;
        memset(waves[w].brought, 0, sizeof waves[w].brought);
      }
      for (int t = 0; t < n; ++t) {
        ended[t] = false;
        void** top = reinterpret_cast<void**>(stacks + STACK * (t + 1));
        *--top = nullptr;  // (run does not return)
        *--top = reinterpret_cast<void*>(&run);
        for (int r = 0; r < 6; ++r) *--top = nullptr;
        fibre[t] = top;
      }
      uint64_t before = ~uint64_t(0);
      while (live > 0) {
        if (events == before) {
          fprintf(stderr, "%s: workgroup %u, %u waits for itself\n", kernel, x, y);
          abort();
        }
        before = events;
        for (int t = 0; t < n; ++t)
          if (!ended[t]) {
            now = t;
            emu_switch(&scheduler, fibre[t]);
          }
      }
    }
}
}  // namespace emu

void __syncthreads() {
  const uint64_t round = emu::barriers;
  ++emu::at_barrier, ++emu::events;
  emu::pass_barrier();
  while (emu::barriers == round) emu::wait();
}
