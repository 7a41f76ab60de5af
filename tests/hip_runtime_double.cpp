// A stand-in for the few HIP runtime calls that the library's host code makes, over host memory: it counts and checks what
// is allocated and freed, on which device, and which kernels are launched with which arguments, and runs none of them.
// Loaded with RTLD_GLOBAL before the library, whose calls then come here; for the tests of its host code without a GPU.
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace {
struct Block { size_t bytes; int device; };
std::mutex mu;
std::map<uintptr_t, Block> live;
std::vector<uintptr_t> freed;
std::map<const void*, std::string> kernels;
struct Launch { std::string name; uintptr_t stream; std::vector<uint64_t> words; };
std::vector<Launch> launches;
int device = 0, n_devices = 2, waited[8] = {};
size_t in_use = 0, capacity = SIZE_MAX;
char* packed = nullptr;                    // where the next block lies, right behind the last one; blocks of then are never used again
int host_blocks = 0;
long unsafe_calls = 0;                     // allocations, frees and waits that would break a capture
bool set_device_fails = false, get_device_fails = false, wait_fails = false;
std::vector<uintptr_t> capturing;          // streams, in the global mode
thread_local hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
struct Config { dim3 grid, block; size_t shmem; hipStream_t stream; };
thread_local std::vector<Config> configs;

void touches() { if (!capturing.empty() && mode != hipStreamCaptureModeRelaxed) ++unsafe_calls; }
}  // namespace

extern "C" {
// ---- for the test
void double_packed() { packed = static_cast<char*>(aligned_alloc(4096, 64u << 20)); }
void double_capacity(uint64_t bytes) { capacity = bytes; }
uint64_t double_in_use() { return in_use; }
uint64_t double_blocks() { return live.size(); }
int double_host_blocks() { return host_blocks; }
uint64_t double_freed() { return freed.size(); }
void double_forget() { freed.clear(); launches.clear(); unsafe_calls = 0; memset(waited, 0, sizeof(waited)); }
int double_is_live(uint64_t ptr) {
  auto it = live.upper_bound(ptr);
  if (it == live.begin()) return 0;
  --it;
  return ptr < it->first + it->second.bytes;
}
uint64_t double_launches() { return launches.size(); }
const char* double_launch_name(uint64_t i) { return launches[i].name.c_str(); }
uint64_t double_launch_word(uint64_t i, uint64_t w) { return w < launches[i].words.size() ? launches[i].words[w] : 0; }
void double_capture(uint64_t stream, int on) { capturing.clear(); if (on) capturing.push_back(stream); }
int64_t double_unsafe_calls() { return unsafe_calls; }
void double_failures(int set_device, int get_device, int wait) { set_device_fails = set_device; get_device_fails = get_device; wait_fails = wait; }
int double_waited(int d) { return waited[d]; }

// ---- the runtime
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { kernels[host] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t s) { configs.push_back({grid, block, shmem, s}); return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, hipStream_t* s) {
  const Config c = configs.back();
  configs.pop_back();
  *grid = c.grid; *block = c.block; *shmem = c.shmem; *s = c.stream;
  return hipSuccess;
}
// What the tests look at among the arguments of a launch is kept, kernel by kernel.
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t s) {
  std::lock_guard<std::mutex> lock(mu);
  Launch l{kernels[f], reinterpret_cast<uintptr_t>(s), {}};
  if (l.name.find("partition_trials") != std::string::npos)   // its scratch: counts, descriptors, work counters
    for (int a : {14, 15, 16}) {
      uint64_t w;
      memcpy(&w, args[a], 8);
      l.words.push_back(w);
    }
  if (l.name.find("affected_element") != std::string::npos) {   // its slots per row or column of tiles
    int slots;
    memcpy(&slots, args[2], 4);
    l.words.push_back((uint64_t)slots);
  }
  launches.push_back(l);
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
  std::lock_guard<std::mutex> lock(mu);
  touches();
  if (in_use + n > capacity) return hipErrorOutOfMemory;
  if (packed) {
    *p = packed;
    packed += (n + 255) / 256 * 256;
  } else {
    *p = aligned_alloc(4096, (n + 4095) / 4096 * 4096);
  }
  memset(*p, 0, n);
  live[reinterpret_cast<uintptr_t>(*p)] = {n, device};
  in_use += n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  std::lock_guard<std::mutex> lock(mu);
  touches();
  auto it = live.find(reinterpret_cast<uintptr_t>(p));
  if (it == live.end()) return hipErrorInvalidValue;
  in_use -= it->second.bytes;
  live.erase(it);
  freed.push_back(reinterpret_cast<uintptr_t>(p));
  if (!packed) free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { touches(); *p = calloc(1, n); ++host_blocks; return hipSuccess; }
hipError_t hipHostFree(void* p) { touches(); free(p); --host_blocks; return hipSuccess; }
hipError_t hipMemcpyAsync(void* to, const void* from, size_t n, hipMemcpyKind, hipStream_t) { memcpy(to, from, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { touches(); return hipSuccess; }
hipError_t hipDeviceSynchronize() { touches(); if (wait_fails) return hipErrorUnknown; ++waited[device]; return hipSuccess; }
hipError_t hipGetDevice(int* d) { if (get_device_fails) return hipErrorUnknown; *d = device; return hipSuccess; }
hipError_t hipSetDevice(int d) { if (set_device_fails || d >= n_devices) return hipErrorInvalidDevice; device = d; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) { memset(p, 0, sizeof(*p)); strcpy(p->gcnArchName, "gfx950"); return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "the runtime's error"; }
hipError_t hipGetSymbolAddress(void** p, const void*) { static char words[1 << 20]; *p = words; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* status) {
  *status = hipStreamCaptureStatusNone;
  for (uintptr_t c : capturing)
    if (c == reinterpret_cast<uintptr_t>(s)) *status = hipStreamCaptureStatusActive;
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) { std::swap(*m, mode); return hipSuccess; }
}
