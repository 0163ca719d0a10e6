// The HIP calls of the library's host code without a device: memory is the
// host's, kernel launches are written down instead of run, and a stream can be
// held so that its synchronisation waits.  Loaded before the library, so that
// its calls come here.
#include <dlfcn.h>

#include <chrono>
#include <condition_variable>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>

struct Dim3 {
  uint32_t x, y, z;
};

namespace {
std::mutex mu;
std::condition_variable cv;
std::string text;
std::map<const void *, int> resident;  // workgroups of a kernel per compute unit: its own number
void *held = nullptr;
bool waiting = false;
int device = 0;
thread_local struct {
  Dim3 grid, block;
  size_t lds;
  void *stream;
} config;

void put(const std::string &line) {
  std::lock_guard<std::mutex> g(mu);
  text += line + "\n";
}

std::string name_of(const void *kernel) {
  Dl_info info{};
  return dladdr(kernel, &info) && info.dli_sname ? info.dli_sname : "?";
}
}  // namespace

extern "C" {
const char *fake_text() { return text.c_str(); }
void fake_clear() { text.clear(); }
void fake_device(int d) { device = d; }
void fake_hold(void *stream) { held = stream; }
int fake_wait_until_held() {  // until a thread waits on the held stream
  std::unique_lock<std::mutex> g(mu);
  return cv.wait_for(g, std::chrono::seconds(20), [] { return waiting; });
}
void fake_release() {
  std::lock_guard<std::mutex> g(mu);
  held = nullptr;
  cv.notify_all();
}

int hipGetDevice(int *d) { return *d = device, 0; }
int hipSetDevice(int) { return 0; }
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return "fake"; }
int hipDeviceGetAttribute(int *v, int, int d) { return *v = 16 + 8 * d, 0; }
int hipGetSymbolAddress(void **p, const void *) {
  static char scratch[64];
  return *p = scratch, 0;
}
int hipMalloc(void **p, size_t n) { return *p = calloc(1, n), 0; }
int hipFree(void *p) { return free(p), 0; }
int hipHostMalloc(void **p, size_t n, unsigned) { return *p = calloc(1, n), 0; }
int hipHostFree(void *p) { return free(p), 0; }
int hipMemcpy(void *d, const void *s, size_t n, int) {
  put("copy on the null stream");
  return memcpy(d, s, n), 0;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *stream) {
  put("copy on stream " + std::to_string((uintptr_t)stream));
  return memcpy(d, s, n), 0;
}
int hipStreamSynchronize(void *stream) {
  std::unique_lock<std::mutex> g(mu);
  if (stream && stream == held) {
    waiting = true;
    cv.notify_all();
    cv.wait_for(g, std::chrono::seconds(20), [stream] { return held != stream; });
  }
  return 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *kernel, int, size_t) {
  std::lock_guard<std::mutex> g(mu);
  *n = resident.emplace(kernel, (int)resident.size() + 1).first->second;
  return 0;
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void *stream) {
  config = {grid, block, lds, stream};
  return 0;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *lds, void **stream) {
  *grid = config.grid;
  *block = config.block;
  *lds = config.lds;
  *stream = config.stream;
  return 0;
}
int hipLaunchKernel(const void *kernel, Dim3 grid, Dim3 block, void **, size_t, void *) {
  int r = 0;
  {
    std::lock_guard<std::mutex> g(mu);
    const auto it = resident.find(kernel);
    if (it != resident.end()) r = it->second;
  }
  put("launch " + name_of(kernel) + " " + std::to_string(grid.x) + " " + std::to_string(block.x) + " " + std::to_string(r));
  return 0;
}
}
