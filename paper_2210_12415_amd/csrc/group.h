// Several independent convolutions in one launch.
//
// A layer of a small batch is 16 to 250 workgroups on 256 compute units, each a chain of first loads, a sum and stores, and launches
// on one stream follow one another: the chip waits for every layer's slowest workgroup and then for the next launch.  Here the workgroups
// of up to kGroupMax problems are one grid: a workgroup finds its problem by its number and runs the body of a tile kernel
// (dstream.h, dslab.h, dplanar.h) on that problem's parameters, so that all layers are in flight together and one's ends are covered by
// another's sums.  Five layers of a ResNet in one call (64 channels at 56 x 56 and so on), one launch each before and one for all now: a batch of 1
// 35 us and 10.8, of 16 in NCHW 71 and 48, of 5 in fp32 80 and 52.
//
// A family is a kernel that holds the bodies its problems choose from, with one number of threads.  Its registers are those of its
// largest body, its LDS that of the largest problem of the launch.
#pragma once

#include "dplanar.h"
#include "dslab.h"
#include "dstream.h"

namespace alt {

constexpr int kGroupMax = 8;              // (a launch's arguments are at most 4 KB)

struct GroupParams {
    int32_t n, pad_;
    int32_t first[kGroupMax];             // the problems' first workgroups: multiples of eight, so that a problem's tiles lie on the XCDs as alone
    int32_t body[kGroupMax];
    DconvParams p[kGroupMax];
};
static_assert(sizeof(GroupParams) <= 4096, "kernel arguments");

// A tile that a family offers: what the setup and the estimate know it by, and the body that runs a problem on it (-1: none).
struct GroupTile {
    IgemmLaunch k;
    int (*body)(const DconvParams &p);
};

struct GroupFamily {
    int code;                             // in alt_multi_plan_t
    const GroupTile *tiles;
    int ntiles, threads;
    double line;                          // together up to this part of the time that the calls take one by one, both as estimated
    hipError_t (*launch)(const GroupParams &g, unsigned workgroups, size_t lds, hipStream_t st);
};
const GroupFamily &group_f32();           // fp32, NHWC
const GroupFamily &group_slab();          // bf16, NHWC
const GroupFamily &group_planar();        // bf16, NCHW

// dconv.hip: launches the problems of *g, whose sliced ones have at most kDconvMaxTiles tiles together (hipErrorNotReady: no set of
// arrival counters is free for the stream).
hipError_t group_run(const GroupFamily &f, GroupParams *g, unsigned workgroups, size_t lds, hipStream_t st);

// (The parameters are read where the launch put them: indexed as a by-value argument, the compiler copies all of them to each lane's stack.)
template <typename F>
__global__ __launch_bounds__(F::kThreads, F::kWaves) void group_kernel(const GroupParams)
{
    typedef const __attribute__((address_space(4))) GroupParams *Args;
    const GroupParams &g = *(const GroupParams *)(Args)__builtin_amdgcn_kernarg_segment_ptr();
    const int bx = (int)blockIdx.x;
    int i = 0;
#pragma unroll
    for (int j = 1; j < kGroupMax; ++j) i += j < g.n && bx >= g.first[j] ? 1 : 0;
    const DconvParams &p = g.p[i];
    const int id = bx - g.first[i];
    if (id >= p.tiles_m * p.tiles_n * p.splitk) return;    // up to the next multiple of eight
    F::run(g.body[i], p, id);
}

template <typename F>
hipError_t group_launch(const GroupParams &g, unsigned workgroups, size_t lds, hipStream_t st)
{
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)group_kernel<F>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(group_kernel<F>, dim3(workgroups), dim3(F::kThreads), lds, st, g);
    return hipGetLastError();
}

// (the setup and the estimate tell these kernels from the register-staged ones by their launch; a group's tiles are launched together)
inline hipError_t group_only(const DconvParams &, size_t, hipStream_t) { return hipErrorInvalidValue; }

}  // namespace alt
