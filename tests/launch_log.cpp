// The HIP runtime as libvq.so sees it on a machine without a GPU: every kernel launch is noted down -- name, grid, workgroup, LDS, the first
// words of its arguments -- and nothing runs.  Loaded in front of the library (launches.py), so that its calls end up here.
#include <cxxabi.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
struct Dim { uint32_t x, y, z; };
struct Config { Dim grid, block; size_t lds; void *stream; } g_config;
std::map<const void *, std::string> &names() {
  static std::map<const void *, std::string> all;
  return all;
}
std::string g_log;
alignas(256) unsigned char g_symbol[256];
}  // namespace

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *, void *, void *, void *, int *) {
  int status = 0;
  char *text = abi::__cxa_demangle(device, nullptr, nullptr, &status);
  std::string name = status == 0 && text ? text : device;
  free(text);
  const size_t from = name.find("(anonymous namespace)::");
  if (from != std::string::npos) name = name.substr(from + strlen("(anonymous namespace)::"));
  const size_t arguments = name.find('(');
  names()[host] = arguments == std::string::npos ? name : name.substr(0, arguments);
}
int __hipPushCallConfiguration(Dim grid, Dim block, size_t lds, void *stream) { g_config = {grid, block, lds, stream}; return 0; }
int __hipPopCallConfiguration(Dim *grid, Dim *block, size_t *lds, void **stream) {
  *grid = g_config.grid; *block = g_config.block; *lds = g_config.lds; *stream = g_config.stream;
  return 0;
}
int hipLaunchKernel(const void *kernel, Dim grid, Dim block, void **args, size_t lds, void *) {
  const std::string &name = names()[kernel];
  char line[256];
  snprintf(line, sizeof line, "|%u %u %u|%u|%zu|", grid.x, grid.y, grid.z, block.x * block.y * block.z, lds);
  g_log += name + line;
  // (of these two kinds of kernels, whose arguments are seven and more pointers and numbers)
  if (name.find("groups_finish") != std::string::npos || name.find("products_finish") != std::string::npos || name.find("gather_cols") != std::string::npos)
    for (int i = 0; i < 6; ++i) {
      uint64_t word = 0;
      memcpy(&word, args[i], name.find("finish") != std::string::npos && i >= 2 && i < 5 ? 4 : 8);
      snprintf(line, sizeof line, "%s%llu", i ? " " : "", (unsigned long long)word);
      g_log += line;
    }
  g_log += "\n";
  return 0;
}
int hipGetLastError(void) { return 0; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipGetDevice(int *device) { *device = 0; return 0; }
int hipDeviceGetAttribute(int *value, int, int) { *value = 256; return 0; }       // (the library asks for the compute units)
int hipGetSymbolAddress(void **address, const void *) { *address = g_symbol; return 0; }

const char *launch_log(void) { return g_log.c_str(); }
void launch_log_clear(void) { g_log.clear(); }
}
