// The host side of the mask builds (radial_mask.hip) on a runtime that is written here: it hands out host memory, notes launches, copies and
// waits and refuses the launch it is told to.  Of the kernels it runs nothing but the total of mask_lists_kernel, for which it puts the number of tokens.
//   refuse : for each way to build a mask and each of its launches, that launch is refused; one line
//     "way launch kernel status launches-after allocations-left"
//   unmapped : no host memory can be mapped; per way "way status copies total-is-right"
//   together : 40 threads build at a time, each its own size, and wait for each other before any reads what came back; one line
//     "threads copies wrong" and one of a build after them
//   unwaited : the stream of three builds cannot be waited for; one line "wrong slots", those of later builds that were these three's
//   ended : after 40 builds with each launch refused, one line "way copies" with the copies to the host of a build that succeeds
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <atomic>
#include <condition_variable>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "radial_mask.hip"

namespace {

std::map<const void*, std::string> kernel_names;
std::atomic<int> launches{0}, refused{-1}, allocations{0}, copies_back{0};
std::atomic<const void*> refused_kernel{nullptr};
std::atomic<bool> can_map{true}, can_wait{true};
std::atomic<void*> last_slot{nullptr};
std::mutex gate_mutex;
std::condition_variable gate;
int expected = 0, arrived = 0;  // threads that wait for each other in hipStreamSynchronize
thread_local hipError_t last_error = hipSuccess;

hipError_t noted(hipError_t e) {
  if (e != hipSuccess) last_error = e;
  return e;
}

}  // namespace

extern "C" {
// what the compiler calls around a kernel and its launch
char __hip_fatbin[64];
void** __hipRegisterFatBinary(const void*) {
  static void* handle = nullptr;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { kernel_names[host] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
static thread_local struct { dim3 grid, block; size_t lds; hipStream_t stream; } call;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  call = {grid, block, lds, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
  *grid = call.grid;
  *block = call.block;
  *lds = call.lds;
  *stream = call.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* kernel, dim3, dim3, void** args, size_t, hipStream_t) {
  if (launches++ != refused) {
    if (kernel_names.at(kernel).find("mask_lists_kernel") != std::string::npos) {
      const radial::MaskGeom& g = *(const radial::MaskGeom*)args[0];
      const radial::Meta& meta = *(const radial::Meta*)args[5];
      meta.device[radial::kTotal] = g.n;
      if (meta.host) meta.host[radial::kTotal] = g.n;
    }
    return hipSuccess;
  }
  refused_kernel = kernel;
  return noted(hipErrorLaunchFailure);
}

hipError_t hipGetLastError() {
  const hipError_t e = last_error;
  last_error = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "refused"; }
hipError_t hipGetDevice(int* device) {
  *device = 0;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t bytes) {
  ++allocations;
  *p = calloc(1, bytes);
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  allocations -= p != nullptr;
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) {
  if (!can_map) return noted(hipErrorOutOfMemory);
  *p = calloc(1, bytes);
  return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** device, void* host, unsigned) {
  *device = host;
  last_slot = host;
  return hipSuccess;
}
hipError_t hipMemcpy(void* to, const void* from, size_t bytes, hipMemcpyKind) {
  memcpy(to, from, bytes);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* to, const void* from, size_t bytes, hipMemcpyKind kind, hipStream_t) {
  copies_back += kind == hipMemcpyDeviceToHost;
  memcpy(to, from, bytes);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  if (!can_wait) return noted(hipErrorUnknown);
  std::unique_lock<std::mutex> lock(gate_mutex);
  if (arrived < expected && ++arrived == expected) gate.notify_all();
  gate.wait(lock, [] { return arrived >= expected; });
  return hipSuccess;
}
}

namespace {

constexpr uint32_t kBoth = RADIAL_MASK_TRANSPOSE;
struct Way {
  const char* name;
  int frames, tokens;  // of a radial or banded mask; tokens alone of the others
  uint32_t flags;
};
// by the size of the lists: room for every pair, counted on the host, and too many blocks for an order
const Way kWays[] = {{"radial", 4, 500, 0},       {"radial", 4, 500, kBoth},       {"radial", 4, 15000, 0},          {"radial", 4, 15000, kBoth},
                     {"radial", 1100, 1000, 0},   {"radial", 1100, 1000, kBoth},   {"banded", 4, 500, kBoth},        {"banded", 1100, 1000, kBoth},
                     {"dense", 0, 2000, 0},       {"dense", 0, 2000, kBoth},       {"dense", 0, 1100000, kBoth},     {"lists", 0, 2000, 0},
                     {"lists", 0, 2000, kBoth},   {"lists", 0, 1100000, kBoth}};

int build(const Way& way, radial_mask** m) {
  static int32_t nothing[1 << 15];
  switch (way.name[0]) {
    case 'r': {
      const radial_mask_params p = {way.frames, way.tokens, 64, 1, way.flags, 1, 1, 0};
      return radial_mask_build(&p, nullptr, m);
    }
    case 'b': return radial_mask_build_banded(way.frames, way.tokens, 64, 1, nothing, way.flags, nullptr, m);
    case 'd': return radial_mask_build_dense(way.tokens, 64, way.flags, nullptr, m);
    default: return radial_mask_from_csr(way.tokens, 64, way.flags, nothing, nothing, nullptr, m);
  }
}

int refuse() {
  for (const Way& way : kWays) {
    radial_mask* m = nullptr;
    launches = 0;
    if (build(way, &m) != RADIAL_OK) return 1;
    radial_mask_free(m);
    const int n = launches;
    for (int k = 0; k < n; ++k) {
      launches = 0;
      refused = k;
      const int rc = build(way, &m);
      refused = -1;
      printf("%s-%d-%d-%u %d %s %d %d %d\n", way.name, way.frames, way.tokens, way.flags, k, kernel_names[refused_kernel].c_str(), rc, launches - k - 1, (int)allocations);
      if ((rc == RADIAL_OK) != (m != nullptr)) return 1;
      radial_mask_free(m);
    }
  }
  return 0;
}

int unmapped() {
  can_map = false;
  for (const Way& way : kWays) {
    radial_mask* m = nullptr;
    copies_back = 0;
    const int rc = build(way, &m);
    const bool placed = (way.name[0] == 'r' || way.name[0] == 'b') && way.frames * way.tokens <= 64 * radial::kMaxOrdered;
    printf("%s-%d-%d-%u %d %d %d\n", way.name, way.frames, way.tokens, way.flags, rc, (int)copies_back, m && (!placed || m->nnz == way.frames * way.tokens));
    radial_mask_free(m);
  }
  return 0;
}

int together() {
  std::atomic<int> wrong{0};
  const auto one = [&](int size) {
    radial_mask* m = nullptr;
    const Way way = {"radial", 3, size, 0};
    wrong += build(way, &m) != RADIAL_OK || m->nnz != 3 * size;
    radial_mask_free(m);
  };
  for (int round = 0; round < 20; ++round) {
    copies_back = 0;
    expected = 40;
    arrived = 0;
    std::vector<std::thread> threads;
    for (int i = 0; i < 40; ++i) threads.emplace_back(one, 100 + i);
    for (std::thread& t : threads) t.join();
    printf("40 %d %d\n", (int)copies_back, (int)wrong);
    expected = 0;
    copies_back = 0;
    one(99);
    printf("1 %d %d\n", (int)copies_back, (int)wrong);
  }
  return 0;
}

int unwaited() {
  const Way way = {"radial", 3, 100, 0};
  radial_mask* m = nullptr;
  std::set<void*> lost;
  can_wait = false;
  for (int i = 0; i < 3; ++i) {
    if (build(way, &m) != RADIAL_EHIP) return 1;
    lost.insert(last_slot);
    (void)hipGetLastError();
  }
  can_wait = true;
  int again = 0;
  for (int i = 0; i < 5; ++i) {
    if (build(way, &m) != RADIAL_OK) return 1;
    radial_mask_free(m);
    again += (int)lost.count(last_slot);
  }
  printf("%d %d\n", again, (int)lost.size());
  return 0;
}

int ended() {
  for (const Way& way : kWays) {
    radial_mask* m = nullptr;
    for (int k = 0, n = 1; k < n; ++k)
      for (int i = 0; i < 40; ++i) {
        launches = 0;
        refused = i < 39 ? k : -1;
        const int rc = build(way, &m);
        if ((rc == RADIAL_OK) != (i == 39)) return 1;
        if (!rc) n = launches;
        radial_mask_free(m);
      }
    copies_back = 0;
    if (build(way, &m) != RADIAL_OK) return 1;
    radial_mask_free(m);
    printf("%s-%d-%d-%u %d\n", way.name, way.frames, way.tokens, way.flags, (int)copies_back);
  }
  return 0;
}

}  // namespace

int main(int argc, char** argv) {
  const std::string mode = argc > 1 ? argv[1] : "";
  if (mode == "refuse") return refuse();
  if (mode == "ended") return ended();
  if (mode == "unmapped") return unmapped();
  if (mode == "together") return together();
  if (mode == "unwaited") return unwaited();
  return 1;
}
