// The HIP runtime calls of libcausal's host code, without a GPU: launches are recorded (kernel
// name, grid, block) and refused like the runtime refuses them, copies move nothing but
// what a test has queued, everything else succeeds.  Linked with the library's objects by
// tests/test_launch_shapes.py.
#include <cstdint>
#include <cstring>
#include <map>
#include <string>
#include <vector>

struct Dim3 {
  uint32_t x, y, z;
};
struct Launch {
  std::string kernel;
  Dim3 grid, block;
};

static std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
static std::vector<Launch> launches;
static std::vector<std::vector<char>> replies;  // device-to-host copies, first one next
static Dim3 next_grid, next_block;
static size_t next_lds;
static void* next_stream;
static int last_error = 0;

extern "C" {

int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
  next_grid = grid;
  next_block = block;
  next_lds = lds;
  next_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
  *grid = next_grid;
  *block = next_block;
  *lds = next_lds;
  *stream = next_stream;
  return 0;
}
void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) {
  names()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

// Work-items along an axis fit 32 bits, workgroups along y and z 16 bits.
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void**, size_t, void*) {
  launches.push_back({names()[f], grid, block});
  const bool fits = (uint64_t)grid.x * block.x < (1ull << 32) && grid.y <= 65535 && grid.z <= 65535 &&
                    grid.x > 0 && grid.y > 0 && grid.z > 0;
  if (!fits) last_error = 9;  // hipErrorInvalidConfiguration
  return last_error;
}
int hipGetLastError() {
  const int e = last_error;
  last_error = 0;
  return e;
}
int hipMemcpyAsync(void* dst, const void*, size_t bytes, int kind, void*) {
  if (kind != 2) return 0;
  if (replies.empty() || replies.front().size() != bytes) return 1;
  memcpy(dst, replies.front().data(), bytes);
  replies.erase(replies.begin());
  return 0;
}
int hipMemcpy(void*, const void*, size_t, int) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipGetDevice(int* dev) { return *dev = 0; }
int hipGetDevicePropertiesR0600(void*, int) { return 1; }  // the library then assumes 256 CUs
int hipMalloc(void** p, size_t) {
  *p = (void*)256;
  return 0;
}
int hipFree(void*) { return 0; }
int hipEventCreate(void** e) {
  *e = nullptr;
  return 0;
}
int hipEventDestroy(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) {
  *ms = 1.0f;
  return 0;
}
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipGetSymbolAddress(void** p, const void*) {
  *p = (void*)256;
  return 0;
}
int hipGraphDestroy(void*) { return 0; }
int hipGraphExecDestroy(void*) { return 0; }
int hipGraphInstantiate(void**, void*, void*, char*, size_t) { return 1; }
int hipGraphLaunch(void*, void*) { return 1; }
int hipStreamBeginCapture(void*, int) { return 1; }
int hipStreamCreateWithFlags(void** s, unsigned) {
  *s = nullptr;
  return 0;
}
int hipStreamDestroy(void*) { return 0; }
int hipStreamEndCapture(void*, void** g) {
  *g = nullptr;
  return 1;
}

// What the tests use.
void rec_reset() {
  launches.clear();
  replies.clear();
  last_error = 0;
}
void rec_reply(const void* data, size_t bytes) {
  replies.emplace_back((const char*)data, (const char*)data + bytes);
}
int rec_count() { return (int)launches.size(); }
const char* rec_kernel(int i) { return launches[i].kernel.c_str(); }
void rec_dims(int i, uint32_t* six) {
  memcpy(six, &launches[i].grid, 12);
  memcpy(six + 3, &launches[i].block, 12);
}
}
