// Host-thread executor behind tests/cpu_emul/hip/hip_runtime.h (test infrastructure only).
#include <hip/hip_runtime.h>
#include <string>

namespace hip_emul {
thread_local dim3 t_threadIdx, t_blockIdx;
dim3 g_blockDim, g_gridDim;
thread_local Wave* t_wave = nullptr;
pthread_barrier_t g_block_bar;
alignas(16) float g_dynamic_lds[40960];  // 160 KB, the LDS of one CU
Pinned g_pinned;
int g_memsets = 0;
bool g_recording = false;
bool g_off_null = false;
std::vector<std::function<void()>> g_recorded;
thread_local hipStreamCaptureMode t_capture_mode = hipStreamCaptureModeGlobal;

static std::vector<std::pair<std::string, dim3>> g_launches;
void note_launch(const char* kernel, dim3 grid) { g_launches.emplace_back(kernel, grid); }

void launch(dim3 grid, dim3 block, void (*body)(void*), void* closure) {
  const unsigned nthreads = block.x * block.y * block.z;
  const unsigned nwaves = (nthreads + 63) / 64;
  if (nthreads % 64 != 0) {
    fprintf(stderr, "hip_emul: block size %u is not a multiple of the wavefront size\n", nthreads);
    abort();
  }
  g_blockDim = block;
  g_gridDim = grid;
  std::vector<Wave> waves(nwaves);
  for (auto& w : waves) pthread_barrier_init(&w.bar, nullptr, 64);
  pthread_barrier_init(&g_block_bar, nullptr, nthreads);
  pthread_barrier_t between;
  pthread_barrier_init(&between, nullptr, nthreads);
  std::vector<std::thread> pool;
  pool.reserve(nthreads);
  for (unsigned tid = 0; tid < nthreads; ++tid) {
    pool.emplace_back([&, tid] {
      t_threadIdx = dim3(tid % block.x, (tid / block.x) % block.y, tid / (block.x * block.y));
      t_wave = &waves[tid / 64];
      for (unsigned bz = 0; bz < grid.z; ++bz)
        for (unsigned by = 0; by < grid.y; ++by)
          for (unsigned bx = 0; bx < grid.x; ++bx) {
            t_blockIdx = dim3(bx, by, bz);
            body(closure);
            pthread_barrier_wait(&between);  // workgroups run one after the other
          }
    });
  }
  for (auto& th : pool) th.join();
  for (auto& w : waves) pthread_barrier_destroy(&w.bar);
  pthread_barrier_destroy(&g_block_bar);
  pthread_barrier_destroy(&between);
}
}  // namespace hip_emul

extern "C" void hip_emul_pinned(int out[3]) {
  out[0] = hip_emul::g_pinned.allocated;
  out[1] = hip_emul::g_pinned.freed;
  out[2] = hip_emul::g_pinned.unguarded;
}

// Grid of the last launch, since the last call with NULL, whose kernel's name as written at the launch contains `kernel`;
// false if there was none.
extern "C" int hip_emul_last_grid(const char* kernel, unsigned grid[3]) {
  if (!kernel) {
    hip_emul::g_launches.clear();
    return 0;
  }
  for (auto it = hip_emul::g_launches.rbegin(); it != hip_emul::g_launches.rend(); ++it)
    if (it->first.find(kernel) != std::string::npos) {
      grid[0] = it->second.x; grid[1] = it->second.y; grid[2] = it->second.z;
      return 1;
    }
  return 0;
}

// 1: keeps the launches that follow instead of carrying them out; 0: carries launches out again.
extern "C" void hip_emul_record(int on) {
  if (on) hip_emul::g_recorded.clear();
  hip_emul::g_recording = on != 0;
}
extern "C" int hip_emul_replay() {
  for (auto& run : hip_emul::g_recorded) run();
  return (int)hip_emul::g_recorded.size();
}

extern "C" int hip_emul_memsets() { return hip_emul::g_memsets; }  // hipMemsetAsync calls so far
extern "C" int hip_emul_off_null() { return hip_emul::g_off_null; }      // a window of memory has begun at NULL plus an offset
