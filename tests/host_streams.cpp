// Host-side driver of the C ABI with the HIP runtime's calls replaced by the functions
// below (the executable's definitions come before the runtime's): device memory is a
// count of bytes, kernels do nothing, and a call can be made to fail or to wait.  It
// shows what the library's calls allocate and which of them wait for each other, without
// a GPU.
#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>
#include <unistd.h>

#include <atomic>
#include <chrono>
#include <condition_variable>
#include <future>
#include <map>
#include <mutex>
#include <thread>
#include <vector>

#include "psflib.h"

namespace {

std::mutex mu;
std::condition_variable cv;
thread_local hipError_t last_error = hipSuccess;
size_t next_address = (size_t)1 << 40;
std::map<void*, size_t> live;        // pool allocations
size_t most_bytes = ~(size_t)0;      // a larger allocation runs out of memory
size_t largest_refused = 0, last_granted = 0;
hipStream_t wait_copy = nullptr, wait_launch = nullptr;  // streams whose copies or launches wait
std::atomic<int> waiting{0};

hipError_t fails(hipError_t e) { return last_error = e; }

// wait until the gate is opened (set to no stream)
void gate(hipStream_t& closed, hipStream_t s) {
  std::unique_lock<std::mutex> lock(mu);
  if (s == nullptr || closed != s) return;
  ++waiting;
  cv.notify_all();
  cv.wait(lock, [&] { return closed != s; });
  --waiting;
}

}  // namespace

extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError(void) { const hipError_t e = last_error; last_error = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipMemPoolCreate(hipMemPool_t* p, const hipMemPoolProps*) { *p = (hipMemPool_t)1; return hipSuccess; }
hipError_t hipMemPoolDestroy(hipMemPool_t) { return hipSuccess; }
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void*) { return hipSuccess; }
hipError_t hipMallocFromPoolAsync(void** p, size_t bytes, hipMemPool_t, hipStream_t) {
  std::lock_guard<std::mutex> lock(mu);
  if (bytes > most_bytes) {
    if (bytes > largest_refused) largest_refused = bytes;
    return fails(hipErrorOutOfMemory);
  }
  *p = (void*)next_address;
  next_address += (bytes + 4095) & ~(size_t)4095;
  live[*p] = last_granted = bytes;
  return hipSuccess;
}
hipError_t hipFreeAsync(void* p, hipStream_t) {
  std::lock_guard<std::mutex> lock(mu);
  return live.erase(p) ? hipSuccess : fails(hipErrorInvalidValue);
}
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t s) { gate(wait_copy, s); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) { *c = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)0x9000; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
struct Config { dim3 grid, block; size_t lds; hipStream_t s; };
static thread_local Config config;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) { config = {g, b, lds, s}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = config.grid; *b = config.block; *lds = config.lds; *s = config.s;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t s) { gate(wait_launch, s); return hipSuccess; }
}

namespace {

#define EXPECT(cond)                                                        \
  do {                                                                      \
    if (!(cond)) {                                                          \
      fprintf(stderr, "%s:%d: expected %s\n", __FILE__, __LINE__, #cond);   \
      fflush(stderr);                                                       \
      _exit(1);                                                             \
    }                                                                       \
  } while (0)

void* const kLib = (void*)((size_t)1 << 30);  // never read
float* const kCube = (float*)((size_t)1 << 28);
float* const kScene = (float*)((size_t)1 << 29);
const hipStream_t A = (hipStream_t)0x1000, B = (hipStream_t)0x2000;

psflib_status build(int n, int K, int N, int rotate, hipStream_t s, psflib_handle** h) {
  psflib_desc d;
  memset(&d, 0, sizeof(d));
  d.n = n; d.n_psf = K; d.N = N;
  d.scene_pixscale = 1.0;
  d.rotate = rotate;
  std::vector<double> radii(K);
  for (int k = 0; k < K; ++k) radii[k] = k;
  return psflib_build(&d, kCube, radii.data(), kLib, (size_t)1 << 60, s, h);
}

// f on a thread of its own: whether it ends within five seconds
template <typename F>
bool ends(F f) {
  auto task = std::make_shared<std::packaged_task<void()>>(f);
  auto done = task->get_future();
  std::thread([task] { (*task)(); }).detach();
  return done.wait_for(std::chrono::seconds(5)) == std::future_status::ready;
}

bool someone_waits() {
  std::unique_lock<std::mutex> lock(mu);
  return cv.wait_for(lock, std::chrono::seconds(5), [] { return waiting > 0; });
}

void open_gates() {
  std::lock_guard<std::mutex> lock(mu);
  wait_copy = wait_launch = nullptr;
  cv.notify_all();
}

// Scratch of 37 MB where 48 MiB are left: the rounded size of a stream's buffer, 64
// MiB, is refused, the build takes what it needs and gives it back.
void out_of_memory() {
  psflib_handle* h = nullptr;
  most_bytes = (size_t)48 << 20;
  for (int turn = 0; turn < 2; ++turn) {
    EXPECT(build(128, 100, 8, PSFLIB_ROTATE_CUBIC, A, &h) == PSFLIB_OK);
    EXPECT(largest_refused == (size_t)64 << 20);
    EXPECT(last_granted > (size_t)32 << 20 && last_granted < (size_t)40 << 20);
    size_t held = 0;
    for (auto& b : live) held += b.second;
    EXPECT(held < (size_t)1 << 20);  // the handle's workspace
    psflib_destroy(h);
  }
  most_bytes = (size_t)16 << 20;  // nor is there memory for the exact size
  EXPECT(build(128, 100, 8, PSFLIB_ROTATE_CUBIC, A, &h) == PSFLIB_ERR_DEVICE);
  EXPECT(strstr(psflib_last_error(), "out of memory") != nullptr);
  hipGetLastError();
  most_bytes = ~(size_t)0;
  EXPECT(build(128, 100, 8, PSFLIB_ROTATE_CUBIC, A, &h) == PSFLIB_OK);
  EXPECT(last_granted == (size_t)64 << 20);  // kept with the stream
  psflib_destroy(h);
}

// A build that waits on the host -- for the copy of its radii, for a launch -- does not
// keep calls on other streams waiting.
void streams() {
  psflib_handle *h = nullptr, *h2 = nullptr;
  EXPECT(build(64, 4, 64, PSFLIB_ROTATE_BILINEAR, B, &h) == PSFLIB_OK);
  auto apply = [&](hipStream_t s) { EXPECT(psflib_apply(h, kScene, kScene, s) == PSFLIB_OK); };
  for (hipStream_t* closed : {&wait_copy, &wait_launch}) {
    {
      std::lock_guard<std::mutex> lock(mu);
      *closed = A;
    }
    std::thread t([&] { EXPECT(build(64, 200, 64, PSFLIB_ROTATE_BILINEAR, A, &h2) == PSFLIB_OK); });
    EXPECT(someone_waits());
    EXPECT(ends([&] { apply(B); }));
    if (closed == &wait_copy) EXPECT(ends([&] { apply(A); }));  // nothing of the stream's is in use yet
    open_gates();
    t.join();
    psflib_destroy(h2);
  }
  // two threads on one stream: one after the other, both through
  std::vector<std::thread> ts;
  for (int i = 0; i < 8; ++i)
    ts.emplace_back([&, i] {
      for (int k = 0; k < 200; ++k) apply(i % 2 ? A : B);
    });
  for (auto& t : ts) t.join();
  psflib_destroy(h);
}

}  // namespace

int main(int argc, char** argv) {
  if (argc > 1 && !strcmp(argv[1], "memory")) out_of_memory();
  if (argc > 1 && !strcmp(argv[1], "streams")) streams();
  printf("host_streams ok\n");
  fflush(stdout);
  _exit(0);  // without the real runtime's exit handlers
}
