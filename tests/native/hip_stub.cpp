// A HIP runtime without a device, for tests of the library's host code on a machine that has none: memory
// is host memory, a kernel launch is written down and otherwise does nothing, and a chosen launch fails.
// Built as libamdhip64.so.7 and loaded before the library, which then binds to it instead of the real one.
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> n;
  return n;
}
std::string launched, fail_name;
int last_error = 0;
int give(void** p, size_t bytes) {
  *p = std::calloc(bytes ? bytes : 1, 1);
  return *p ? 0 : 2;
}
}  // namespace

extern "C" {
// what the tests call: the launches since the last call of stub_launches, one name per line; the next launch
// of a kernel whose name contains `name` fails
const char* stub_launches() {
  static std::string out;
  out.swap(launched);
  launched.clear();
  return out.c_str();
}
void stub_fail_next(const char* name) { fail_name = name; }

void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device_name, unsigned, void*, void*, void*, void*, int*) {
  names()[host] = device_name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
struct Dim3 { unsigned x, y, z; };
int __hipPushCallConfiguration(Dim3, Dim3, size_t, void*) { return 0; }
int __hipPopCallConfiguration(Dim3*, Dim3*, size_t*, void**) { return 0; }
int hipLaunchKernel(const void* host, Dim3, Dim3, void**, size_t, void*) {
  const std::string& name = names()[host];
  if (!fail_name.empty() && name.find(fail_name) != std::string::npos) {
    fail_name.clear();
    return last_error = 719;
  }
  launched += name + "\n";
  return 0;
}
int hipGetLastError() {
  const int e = last_error;
  last_error = 0;
  return e;
}
const char* hipGetErrorString(int) { return "stub"; }
int hipMalloc(void** p, size_t bytes) { return give(p, bytes); }
int hipFree(void* p) { std::free(p); return 0; }
int hipHostMalloc(void** p, size_t bytes, unsigned) { return give(p, bytes); }
int hipHostFree(void* p) { std::free(p); return 0; }
int hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return 0; }
int hipGetSymbolAddress(void** p, const void*) {
  static char word[64];
  *p = word;
  return 0;
}
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { return 0; }
int hipMemsetAsync(void*, int, size_t, void*) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipSetDevice(int) { return 0; }
int hipGetDevicePropertiesR0600(void*, int) { return 100; }
int hipGetStreamDeviceId(void*) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { return give(s, 1); }
int hipStreamDestroy(void* s) { std::free(s); return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipEventCreate(void** e) { return give(e, 1); }
int hipEventCreateWithFlags(void** e, unsigned) { return give(e, 1); }
int hipEventDestroy(void* e) { std::free(e); return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 0; return 0; }
}
