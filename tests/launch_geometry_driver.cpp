// Host-only driver for the launch geometry of the library: the runtime's function that a launch hands its geometry to is
// defined here (the program's symbols come before the runtime's) and tells the caller to launch nothing, so the library's calls
// run through on the host and every grid is only looked at.  No GPU is needed or used, and no pointer is dereferenced.
//   refresh count m n r          the batched subspace refresh, with the workspace that it asks for
//   forward tokens m n ld_n ld_m (pitches; 0: dense)        backward ... both outputs        grad_input ... only dx
//   t_forward tokens m n         the same on a weight stored transposed; t_backward, t_grad_input
// Prints the number of launches, and for the linear layer each of them as "workgroups threads"; exits 1 if one exceeds what
// the runtime accepts: fewer than 2^32 threads in x, 65535 workgroups in y and in z, none of them zero.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "qgalore.h"

static long launches = 0, refused = 0;
static bool list = false;

struct Extent {   // the runtime's dim3
    uint32_t x, y, z;
};

extern "C" unsigned __hipPushCallConfiguration(Extent grid, Extent block, size_t, void*) {
    ++launches;
    const uint64_t x = (uint64_t)grid.x * block.x;
    if (x == 0 || x >> 32 != 0 || grid.y == 0 || grid.y > 65535 || grid.z == 0 || grid.z > 65535) {
        if (refused++ == 0) std::printf("refused: grid %u x %u x %u of %u threads\n", grid.x, grid.y, grid.z, block.x);
    }
    if (list) std::printf("%u %u\n", grid.x, block.x);
    return 1;   // (not zero: the kernel's stub is not called)
}
extern "C" int hipGetLastError() { return 0; }

template <typename T>
static T* at(uintptr_t address) { return reinterpret_cast<T*>(address); }   // aligned, never dereferenced

int main(int argc, char** argv) {
    if (argc < 5) return 2;
    std::string what = argv[1];
    int64_t a[5] = {};
    for (int i = 0; i < 5 && i + 2 < argc; ++i) a[i] = std::atoll(argv[i + 2]);
    int status = -1;
    if (what == "refresh") {
        const qg_refresh_desc d = {at<uint8_t>(0x10000), at<float>(0x20000), at<uint16_t>(0x30000), at<uint8_t>(0x40000), at<float>(0x50000)};
        const std::vector<qg_refresh_desc> descs(a[0], d);
        status = qg_subspace_refresh_many((int)a[0], descs.data(), a[1], a[2], a[3], 256, 1, at<float>(0x60000), at<int32_t>(0x70000),
                                          at<void>(0x100000), qg_refresh_workspace_bytes((int)a[0], a[1], a[2], a[3]), nullptr);
    } else {
        list = true;
        const bool t = what.rfind("t_", 0) == 0;
        if (t) what = what.substr(2);
        uint16_t *x = at<uint16_t>(0x10000), *dy = at<uint16_t>(0x20000), *out = at<uint16_t>(0x30000), *G = at<uint16_t>(0x40000);
        if (what != "backward") G = nullptr;
        const int8_t* W = at<int8_t>(0x50000);
        const float* s = at<float>(0x60000);
        if (what == "forward")
            status = t ? qg_int8_linear_t_forward(x, W, s, nullptr, a[0], a[1], a[2], 256, out, nullptr)
                       : qg_int8_linear_forward_ld(x, W, s, nullptr, a[0], a[1], a[2], a[3], a[4], 256, out, nullptr);
        else if (what == "backward" || what == "grad_input")
            status = t ? qg_int8_linear_t_backward(dy, x, W, s, a[0], a[1], a[2], 256, out, G, nullptr)
                       : qg_int8_linear_backward_ld(dy, x, W, s, a[0], a[1], a[2], a[3], a[4], 256, out, G, nullptr);
    }
    std::printf("status %d, %ld launches, %ld refused\n", status, launches, refused);
    return status != QG_OK || refused != 0 || launches == 0;
}
