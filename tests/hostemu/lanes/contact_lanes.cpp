// Test-only: csrc/contact.hip on the CPU, and the fibers behind
// hip/hip_runtime.h (x86-64).
#include <hip/hip_runtime.h>
#include <sys/mman.h>

#include "../../../paper_2109_07719_amd/csrc/contact.hip"

namespace aba {
static std::string error;
void clear_error() { error.clear(); }
int report_error(int code, const std::string& what) { return error = what, code; }
}  // namespace aba

namespace {
__shared__ __align__(16) double contact_lds[lanes::kLds / sizeof(double)];
}

namespace lanes {

Index thread, block, block_size;
int compute_units = 256;

namespace {

constexpr int kMaxThreads = 1024, kWave = 64;
constexpr size_t kStack = 1 << 18;
struct Fiber { void* sp; bool done; };
struct Wave { int live, arrived; unsigned turn; unsigned char slot[2][16 * kWave]; };
Fiber fibers[kMaxThreads];
Wave waves[kMaxThreads / kWave];
int current, live, arrived;
unsigned turn;
void* scheduler;
const std::function<void()>* kernel;
long overruns = 0;
std::string log;

extern "C" void lanes_switch(void** save, void* to);
asm(R"(.text
.globl lanes_switch
lanes_switch:
  push %rbp
  push %rbx
  push %r12
  push %r13
  push %r14
  push %r15
  mov %rsp, (%rdi)
  mov %rsi, %rsp
  pop %r15
  pop %r14
  pop %r13
  pop %r12
  pop %rbx
  pop %rbp
  ret
)");

void hand_over() { lanes_switch(&fibers[current].sp, scheduler); }
Wave& wave() { return waves[current / kWave]; }
void entry() {
  (*kernel)();
  fibers[current].done = true;
  Wave& w = wave();
  if (--w.live && w.arrived == w.live) { w.arrived = 0; ++w.turn; }
  if (--live && arrived == live) { arrived = 0; ++turn; }
  hand_over();
  std::abort();
}

}  // namespace

int lane() { return current % kWave; }
void wave_barrier() {
  Wave& w = wave();
  const unsigned t = w.turn;
  if (++w.arrived == w.live) { w.arrived = 0; ++w.turn; }
  else while (w.turn == t) hand_over();
}
void block_barrier() {
  const unsigned t = turn;
  if (++arrived == live) { arrived = 0; ++turn; }
  else while (turn == t) hand_over();
}
const unsigned char* post(const void* p, size_t n) {
  Wave& w = wave();
  unsigned char* const s = w.slot[w.turn & 1];
  std::memcpy(s + 16 * lane(), p, n);
  wave_barrier();
  return s;
}
void run(const char* name, const std::function<void()>& body, dim3 grid, dim3 threads, size_t lds) {
  static unsigned char* const stacks = (unsigned char*)mmap(nullptr, kStack * kMaxThreads, PROT_READ | PROT_WRITE,
                                                            MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  log += std::string(name) + "\n";
  if (lds > kLds) { ++overruns; return; }
  kernel = &body;
  block_size = {threads.x};
  const int n = threads.x;
  for (unsigned b = 0; b < grid.x; ++b) {
    block = {b};
    std::memset(contact_lds, 0xff, kLds);
    live = n;
    arrived = 0;
    for (int i = 0; i < n; i += kWave) waves[i / kWave].live = std::min(kWave, n - i), waves[i / kWave].arrived = 0;
    for (int i = 0; i < n; ++i) {
      void** s = (void**)(stacks + kStack * (i + 1) - 56);
      *--s = (void*)entry;
      for (int k = 0; k < 6; ++k) *--s = nullptr;
      fibers[i] = {s, false};
    }
    for (bool left = true; left;) {
      left = false;
      for (int i = 0; i < n; ++i) {
        if (fibers[i].done) continue;
        current = i;
        thread = {(unsigned)i};
        lanes_switch(&scheduler, fibers[i].sp);
        left = left || !fibers[i].done;
      }
    }
    for (size_t k = lds; k < kLds; ++k) overruns += ((const unsigned char*)contact_lds)[k] != 0xff;
  }
}

}  // namespace lanes

extern "C" {
// compute units that launches see; LDS overruns since the last call; the
// kernels launched since the last call, a line each
void lanes_set_compute_units(int n) { lanes::compute_units = n; }
long lanes_overruns() {
  const long n = lanes::overruns;
  lanes::overruns = 0;
  return n;
}
const char* lanes_log() {
  static std::string out;
  out.swap(lanes::log);
  lanes::log.clear();
  return out.c_str();
}
}
