// Host-only driver for the launch geometry of the subspace refresh: the runtime's function that a launch hands its geometry to
// is defined here (the program's symbols come before the runtime's) and tells the caller to launch nothing, so the library's
// calls run through on the host and every grid is only looked at.  No GPU is needed or used, and no pointer is dereferenced.
// Arguments: count m n r.  Prints the number of launches; exits 1 if one exceeds what the runtime accepts: fewer than 2^32
// threads in x, 65535 workgroups in y and in z, none of them zero.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "qgalore.h"

static long launches = 0, refused = 0;

struct Extent {   // the runtime's dim3
    uint32_t x, y, z;
};

extern "C" unsigned __hipPushCallConfiguration(Extent grid, Extent block, size_t, void*) {
    ++launches;
    const uint64_t x = (uint64_t)grid.x * block.x;
    if (x == 0 || x >> 32 != 0 || grid.y == 0 || grid.y > 65535 || grid.z == 0 || grid.z > 65535) {
        if (refused++ == 0) std::printf("grid %u x %u x %u of %u threads\n", grid.x, grid.y, grid.z, block.x);
    }
    return 1;   // (not zero: the kernel's stub is not called)
}
extern "C" int hipGetLastError() { return 0; }

int main(int argc, char** argv) {
    if (argc != 5) return 2;
    const int count = std::atoi(argv[1]);
    const int64_t m = std::atoll(argv[2]), n = std::atoll(argv[3]), r = std::atoll(argv[4]);
    const qg_refresh_desc d = {reinterpret_cast<const uint8_t*>(0x10000), reinterpret_cast<const float*>(0x20000),
                               reinterpret_cast<const uint16_t*>(0x30000), reinterpret_cast<uint8_t*>(0x40000),
                               reinterpret_cast<float*>(0x50000)};
    const std::vector<qg_refresh_desc> descs(count, d);
    float* const f = reinterpret_cast<float*>(0x60000);
    int32_t* const i = reinterpret_cast<int32_t*>(0x70000);
    const int status = qg_subspace_refresh_many(count, descs.data(), m, n, r, 256, 1, f, i, reinterpret_cast<void*>(0x100000),
                                                qg_refresh_workspace_bytes(count, m, n, r), nullptr);
    std::printf("status %d, %ld launches, %ld refused\n", status, launches, refused);
    return status != QG_OK || refused != 0 || launches == 0;
}
