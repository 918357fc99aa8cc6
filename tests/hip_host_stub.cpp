// The HIP runtime calls that liblif.so makes, without a device: nothing is run, every launch and every attribute that is set
// is written down.  Loaded (RTLD_GLOBAL) ahead of liblif.so by tests/test_launches.py, so that the host code of the library
// - argument checks, launch geometry, LDS sizes - can be looked at on a machine without a GPU.
#include <cstddef>
#include <cstdint>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Dim3 { uint32_t x, y, z; };
struct Launch { const void* kernel; Dim3 grid, block; size_t lds; };
// (never destroyed: the fat binary is unregistered behind the static destructors)
std::map<const void*, std::string>& names() { static auto* m = new std::map<const void*, std::string>; return *m; }
std::map<const void*, int>& allowed() { static auto* m = new std::map<const void*, int>; return *m; }
std::vector<Launch>& launches() { static auto* v = new std::vector<Launch>; return *v; }
Launch pushed;
void* stream_pushed;
alignas(256) unsigned char device_symbol[256];
const char kNoKernel[] = "";
}  // namespace

extern "C" {

void** __hipRegisterFatBinary(const void*) { static void* module; return &module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names()[host] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
    pushed = Launch{nullptr, grid, block, lds};
    stream_pushed = stream;
    return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
    *grid = pushed.grid;
    *block = pushed.block;
    *lds = pushed.lds;
    *stream = stream_pushed;
    return 0;
}
int hipLaunchKernel(const void* kernel, Dim3 grid, Dim3 block, void**, size_t lds, void*) {
    launches().push_back(Launch{kernel, grid, block, lds});
    return 0;
}
int hipFuncSetAttribute(const void* kernel, int attribute, int value) {
    if (attribute == 8) allowed()[kernel] = value;            // hipFuncAttributeMaxDynamicSharedMemorySize
    return 0;
}
int hipFuncGetAttributes(void* attributes, const void*) {     // (all sizes 0: no static LDS)
    memset(attributes, 0, 56);
    return 0;
}
int hipGetDevice(int* device) { *device = 0; return 0; }
int hipDeviceGetAttribute(int* value, int, int) { *value = 64 * 1024; return 0; }
int hipGetSymbolAddress(void** address, const void*) { *address = device_symbol; return 0; }
int hipHostGetDevicePointer(void** device, void* host, unsigned) { *device = host; return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "none"; }

// what was seen
void stub_clear() { launches().clear(); }
int stub_launches() { return (int)launches().size(); }
const char* stub_kernel(int i) { auto it = names().find(launches()[i].kernel); return it == names().end() ? kNoKernel : it->second.c_str(); }
void stub_geometry(int i, uint32_t* grid, uint32_t* block, size_t* lds, int* lds_allowed) {
    const Launch& l = launches()[i];
    *grid = l.grid.x * l.grid.y * l.grid.z;
    *block = l.block.x * l.block.y * l.block.z;
    *lds = l.lds;
    auto it = allowed().find(l.kernel);
    *lds_allowed = it == allowed().end() ? 0 : it->second;
}

}  // extern "C"
