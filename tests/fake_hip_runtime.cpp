// The part of the HIP runtime that the library calls, without a GPU: prints the kernels the host code
// launches and the sizes of their grids.  FAKE_HIP_FAIL: launches of kernels whose name contains it fail.
#include <cxxabi.h>

#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>

namespace {
struct Dim {
  unsigned x, y, z;
};
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> n;
  return n;
}
thread_local Dim grid, block;
thread_local size_t shared;
thread_local void* stream;
thread_local int last;                     // the error since it was last asked for
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* module;
  return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*,
                           void*, int*) {
  int status = 0;
  char* plain = abi::__cxa_demangle(name, nullptr, nullptr, &status);
  names()[host] = status == 0 ? plain : name;
  std::free(plain);
}
int __hipPushCallConfiguration(Dim g, Dim b, size_t sh, void* s) {
  grid = g;
  block = b;
  shared = sh;
  stream = s;
  return 0;
}
int __hipPopCallConfiguration(Dim* g, Dim* b, size_t* sh, void** s) {
  *g = grid;
  *b = block;
  *sh = shared;
  *s = stream;
  return 0;
}
int hipLaunchKernel(const void* f, Dim g, Dim, void**, size_t, void*) {
  const std::string& name = names()[f];
  const char* fail = std::getenv("FAKE_HIP_FAIL");
  const bool fails = fail && name.find(fail) != std::string::npos;
  std::printf("%s %u %s\n", fails ? "failed" : "launched", g.x * g.y * g.z, name.c_str());
  std::fflush(stdout);                     // (whole lines: the caller prints too)
  return fails ? last = 1 : 0;
}
int hipGetLastError() {
  const int e = last;
  last = 0;
  return e;
}
int hipGetDevice(int* d) {
  *d = 0;
  return 0;
}
int hipDeviceGetAttribute(int* v, int, int) {
  *v = 256;                                // compute units
  return 0;
}
int hipGetSymbolAddress(void** p, const void*) {
  *p = (void*)0x40000000;
  return 0;
}
int hipEventCreate(void** e) {
  *e = nullptr;
  return 0;
}
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) {
  *ms = 0.f;
  return 0;
}
}
