"""The occupancy of persistent kernels, asked for once per thread, device and
kernel: kept without allocating (an exception must not cross the C interface),
right for more kernels than are kept, and a grid of a workgroup per compute unit
where the occupancy is unknown.  Runs the built library's own lookup on the CPU,
the HIP queries replaced."""
import subprocess


from paper_2312_06538_amd import crsh as X

SRC = r"""
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <dlfcn.h>
#include <new>
static bool g_full = false;             // memory has run out
static int g_asked = 0, g_dev = 0, g_per_cu = 2;
void *operator new(size_t n)
{
    if (g_full) throw std::bad_alloc();
    return malloc(n ? n : 1);
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }
extern "C" {
int hipGetDevice(int *d) { *d = g_dev; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int threads, size_t)
{
    ++g_asked;
    if (g_per_cu < 0) return 1;
    *n = g_per_cu + (int)((uintptr_t)f % 3) + threads / 256;
    return 0;
}
}
int main(int, char **argv)
{
    void *h = dlopen(argv[1], RTLD_NOW);
    if (!h) { puts(dlerror()); return 2; }
    auto blocks = (uint32_t(*)(const void *, int))dlsym(h, "_ZN4crsh15resident_blocksEPKvi");
    auto grid = (uint32_t(*)(const void *, int, uint64_t))dlsym(h, "_ZN4crsh13resident_gridEPKvim");
    if (!blocks || !grid) { puts("no lookup"); return 2; }
    g_full = true;
    try {
        for (int round = 0; round < 3; ++round)
            for (g_dev = 0; g_dev < 3; ++g_dev)
                for (uintptr_t f = 1; f <= 300; ++f)
                    for (int t = 256; t <= 512; t += 256)
                        if (blocks((const void *)f, t) != 256u * (2 + f % 3 + t / 256)) { puts("wrong"); return 3; }
        g_dev = 0;
        const int before = g_asked;
        for (int k = 0; k < 100; ++k) blocks((const void *)777, 256);
        if (g_asked - before > 1) { printf("asked %d times\n", g_asked - before); return 4; }
        g_per_cu = -1;
        if (grid((const void *)888, 256, 100000) != 256u || grid((const void *)888, 256, 7) != 7u) {
            printf("unknown: %u\n", grid((const void *)888, 256, 100000));
            return 5;
        }
    } catch (const std::bad_alloc &) {
        puts("an exception left the lookup");
        return 1;
    }
    puts("ok");
    return 0;
}
"""


def test_occupancy_lookup(tmp_path):
    src, exe = tmp_path / "occ.cpp", tmp_path / "occ"
    src.write_text(SRC)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-rdynamic", str(src), "-o", str(exe), "-ldl"])
    r = subprocess.run([str(exe), X.LIB_PATH], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), (r.returncode, r.stdout, r.stderr)
