// A stand-in for the HIP runtime on a machine without a GPU: it launches nothing and writes down, in order, which kernels
// the library launches (grid, block, dynamic LDS) and which function attributes it sets.  Loaded with global symbols
// before the library, so that the library's references bind to it.
#include <cxxabi.h>

#include <cstddef>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>

namespace {
struct Dim3 {
    unsigned x, y, z;
};
struct Config {
    Dim3 grid, block;
    std::size_t shared;
    void* stream;
};
std::map<const void*, std::string>& names() {
    static std::map<const void*, std::string> m;
    return m;
}
std::string& text() {
    static std::string s;
    return s;
}
thread_local Config pushed;
thread_local int last_error = 0;
constexpr int kInvalidConfiguration = 9;
void* module = nullptr;
alignas(256) char symbol[256];
void line(const char* kind, const void* f, const Dim3& g, const Dim3& b, std::size_t bytes) {
    char q[160];
    std::snprintf(q, sizeof q, "%s\t%u\t%u\t%u\t%zu\t", kind, g.x, g.y, b.x, bytes);
    text() += q + names()[f] + "\n";
}
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { return &module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, std::size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*, int*) {
    int status = 0;
    char* plain = abi::__cxa_demangle(device, nullptr, nullptr, &status);
    names()[host] = plain ? plain : device;
    std::free(plain);
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, std::size_t shared, void* stream) {
    pushed = Config{grid, block, shared, stream};
    return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, std::size_t* shared, void** stream) {
    *grid = pushed.grid;
    *block = pushed.block;
    *shared = pushed.shared;
    *stream = pushed.stream;
    return 0;
}
// the runtime takes fewer than 2^32 work items in a dimension
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void**, std::size_t shared, void*) {
    if (1ull * grid.x * block.x >> 32 || 1ull * grid.y * block.y >> 32) return last_error = kInvalidConfiguration;
    line("launch", f, grid, block, shared);
    return 0;
}
int hipFuncSetAttribute(const void* f, int, int value) {
    line("attribute", f, Dim3{0, 0, 0}, Dim3{0, 0, 0}, static_cast<std::size_t>(value));
    return 0;
}
int hipGetDevice(int* device) {
    *device = 0;
    return 0;
}
int hipGetDeviceCount(int* count) {
    *count = 1;
    return 0;
}
int hipDeviceGetAttribute(int* value, int, int) {      // the library asks for the number of compute units only
    const char* units = std::getenv("FAKE_HIP_COMPUTE_UNITS");
    *value = units ? std::atoi(units) : 256;
    return 0;
}
int hipGetSymbolAddress(void** address, const void*) {
    *address = symbol;
    return 0;
}
int hipGetLastError() {
    const int error = last_error;
    last_error = 0;
    return error;
}

const char* launch_log() { return text().c_str(); }
void launch_log_clear() { text().clear(); }
}
