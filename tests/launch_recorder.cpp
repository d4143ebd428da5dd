// Stands in for the HIP runtime in a process without a GPU: notes every launch the library asks for, and runs nothing.
#include <cstdlib>
#include <cxxabi.h>
#include <map>
#include <string>
#include <vector>

namespace {
struct Dim {
    unsigned x, y, z;
};
struct Launch {
    std::string name;
    unsigned grid, entries, block, lds, enabled; // enabled: dynamic LDS that the kernel had been allowed at the launch
};
std::map<const void *, std::string> &names()
{
    static std::map<const void *, std::string> m;
    return m;
}
std::map<const void *, unsigned> enabled;
std::vector<Launch> launches;
Dim pushed_grid, pushed_block;
size_t pushed_lds;
void *pushed_stream;
} // namespace

extern "C" {
void **__hipRegisterFatBinary(const void *) { return nullptr; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *, void *, void *, void *, int *)
{
    names()[host] = device;
}
int __hipPushCallConfiguration(Dim grid, Dim block, size_t lds, void *stream)
{
    pushed_grid = grid, pushed_block = block, pushed_lds = lds, pushed_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(Dim *grid, Dim *block, size_t *lds, void **stream)
{
    *grid = pushed_grid, *block = pushed_block, *lds = pushed_lds, *stream = pushed_stream;
    return 0;
}
int hipLaunchKernel(const void *f, Dim grid, Dim block, void **, size_t lds, void *)
{
    char *plain = abi::__cxa_demangle(names()[f].c_str(), nullptr, nullptr, nullptr);
    std::string name = plain ? plain : names()[f];
    free(plain);
    if (name.rfind("void ", 0) == 0) name.erase(0, 5);
    name.erase(std::min(name.size(), name.rfind('('))); // its parameters
    launches.push_back({name, grid.x, grid.y, block.x, (unsigned)lds, enabled[f]});
    return 0;
}
int hipFuncSetAttribute(const void *f, int, int value)
{
    enabled[f] = (unsigned)value;
    return 0;
}
int hipGetLastError() { return 0; }
int hipGetDevice(int *device) { return *device = 0; }
int hipDeviceGetAttribute(int *value, int, int)
{
    *value = 256; // compute units
    return 0;
}

int recorded() { return (int)launches.size(); }
const char *recorded_name(int i) { return launches[i].name.c_str(); }
void recorded_shape(int i, unsigned *out)
{
    const Launch &l = launches[i];
    out[0] = l.grid, out[1] = l.entries, out[2] = l.block, out[3] = l.lds, out[4] = l.enabled;
}
void forget() { launches.clear(); }
}
