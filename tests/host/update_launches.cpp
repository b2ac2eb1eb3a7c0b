// update_launches.cpp -- the update's host side (som_update.hip compiled for the host alone)
// against a stand-in for the HIP runtime, which keeps each kernel's dynamic LDS limit and the
// launches it is asked for.
//
// The limit belongs to the process. An update must not lower it, or another thread that has
// set it and is about to launch the same kernel on a larger lattice is refused; and a runtime
// that refuses the limit must be heard before anything is enqueued.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <vector>

#include "../../paper_2608_24067_amd/csrc/som_internal.h"

namespace {

std::map<const void *, int> limit;  // dynamic LDS bytes each kernel may take
std::map<const void *, int> most;   // the largest each has been given
int launches, lowered, refused;
hipError_t set_error = hipSuccess;
dim3 g_grid, g_block;
size_t g_lds;
hipStream_t g_stream;

void check(bool ok, const char *what)
{
    if (ok) return;
    std::fprintf(stderr, "FAILED: %s\n", what);
    std::exit(1);
}

hipError_t update(int64_t E, int64_t radius, bool f16)
{
    const int64_t V = 40, N = 5000, M = E * E;
    const som::UpdateLayout L = som::update_layout(M, N, V);
    char *w = reinterpret_cast<char *>(0x100000);  // never read: no kernel runs
    som::UpdateBuffers ub = {};
    ub.flags = reinterpret_cast<uint32_t *>(w + L.flags);
    ub.cnt = reinterpret_cast<int32_t *>(w + L.cnt);
    return som::launch_update(f16, w, V, E, nullptr, nullptr, N, 9 * N, nullptr, radius, V, ub, nullptr);
}

}  // namespace

namespace som {
hipError_t launch_check_rows(const int32_t *, int64_t, int64_t, uint32_t *, hipStream_t)
{
    ++launches;
    return hipSuccess;
}
}  // namespace som

extern "C" {
extern const char __hip_fatbin[8];
const char __hip_fatbin[8] = {};
void **__hipRegisterFatBinary(const void *) { return nullptr; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *)
{
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s)
{
    g_grid = g, g_block = b, g_lds = lds, g_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s)
{
    *g = g_grid, *b = g_block, *lds = g_lds, *s = g_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **, size_t lds, hipStream_t)
{
    ++launches;
    if (lds > 0 && (!limit.count(f) || (size_t)limit[f] < lds)) ++refused;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute a, int value)
{
    check(a == hipFuncAttributeMaxDynamicSharedMemorySize, "only the LDS limit is set");
    if (set_error != hipSuccess) return set_error;
    if (most.count(f) && value < most[f]) ++lowered;
    most[f] = most.count(f) && most[f] > value ? most[f] : value;
    limit[f] = value;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
}

int main()
{
    // whole lattices and lines, windows in registers and in LDS, large ones before small ones
    const int64_t cases[][2] = {{128, 64}, {100, 12}, {64, 31}, {9, 4},    // one kernel, falling sizes
                                {128, 3},  {100, 3},  {90, 3},             // windows in registers
                                {320, 40}, {256, 12}, {200, 12},           // lines
                                {512, 3},  {256, 3},  {190, 3}};
    for (bool f16 : {false, true})
        for (auto &c : cases) check(update(c[0], c[1], f16) == hipSuccess, "an update is launched");
    check(launches > 0, "kernels are launched");
    check(refused == 0, "every launch is within the limit set for its kernel");
    check(lowered == 0, "no kernel's limit is lowered by a later update");

    launches = 0;
    set_error = hipErrorInvalidValue;
    for (auto &c : cases) check(update(c[0], c[1], true) == hipErrorInvalidValue, "a refused limit is reported");
    check(launches == 0, "nothing is enqueued once the limit is refused");
    std::printf("update launches: passed\n");
    return 0;
}
