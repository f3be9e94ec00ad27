// A stand-in for the HIP runtime that runs nothing and writes down what it is asked for, one line per
// call: what the library launches, copies, records and waits for, and where, can then be checked without
// a GPU.  Loaded with RTLD_GLOBAL before the library, its functions are found before the runtime's own.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>

namespace {
std::map<const void*, std::string> kernels;
std::string text;
hipMemoryType host_type = hipMemoryTypeHost;
uint64_t* word = nullptr;         // what the work that the next synchronisation waits for has written
uint64_t word_value = 0;
uintptr_t last_event = 0;

template <typename... T>
void say(const char* format, T... values) {
    char line[512];
    std::snprintf(line, sizeof line, format, values...);
    text += line;
    text += '\n';
}
// The last argument of the kernels that end with a choice made on the host.
int choice(const std::string& name, void** args) {
    const int at = name.find("window_decode_kernel") != std::string::npos ? 9
                 : name.find("17decompress_kernel") != std::string::npos ? 10 : -1;
    return at < 0 ? -1 : *static_cast<const unsigned char*>(args[at]);
}
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* stub, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    kernels[stub] = name;
}
hipError_t hipLaunchKernel(const void* stub, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t stream) {
    const std::string& name = kernels[stub];
    say("launch stream=%zu grid=%u block=%u lds=%zu choice=%d %s", reinterpret_cast<size_t>(stream), grid.x, block.x, lds,
        choice(name, args), name.c_str());
    return hipSuccess;
}
hipError_t hipGetDevice(int* device) { *device = 0; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** address, const void*) {
    *address = reinterpret_cast<void*>(uintptr_t{1} << 40);
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
    std::memset(a, 0, sizeof *a);
    a->type = host_type;
    a->devicePointer = host_type == hipMemoryTypeHost ? const_cast<void*>(p) : nullptr;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* event, unsigned flags) {
    *event = reinterpret_cast<hipEvent_t>(++last_event);
    say("create event=%zu flags=%u", last_event, flags);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t event, hipStream_t stream) {
    say("record event=%zu stream=%zu", reinterpret_cast<size_t>(event), reinterpret_cast<size_t>(stream));
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t event) {
    say("synchronize event=%zu", reinterpret_cast<size_t>(event));
    if (word != nullptr) *word = word_value;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t stream, hipEvent_t event, unsigned) {
    say("wait event=%zu stream=%zu", reinterpret_cast<size_t>(event), reinterpret_cast<size_t>(stream));
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* to, const void* from, size_t bytes, hipMemcpyKind, hipStream_t stream) {
    say("copy stream=%zu to=%zu from=%zu bytes=%zu", reinterpret_cast<size_t>(stream), reinterpret_cast<size_t>(to),
        reinterpret_cast<size_t>(from), bytes);
    return hipSuccess;
}
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }

// For the test.
const char* fake_log() { return text.c_str(); }
void fake_clear() { text.clear(); }
void fake_host_memory(int pinned) { host_type = pinned ? hipMemoryTypeHost : hipMemoryTypeUnregistered; }
void fake_written(uint64_t* at, uint64_t value) { word = at; word_value = value; }
}
