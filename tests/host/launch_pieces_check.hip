// De-quantise launches of very large tensors, on the CPU: the kernel launcher of the runtime is replaced
// by one that records grid and arguments, so nothing runs and no address is dereferenced.  A grid counts
// fewer than 2^32 threads; a tensor beyond that must be taken in pieces that cover it exactly.
// Build: hipcc --offload-arch=gfx950 this file + aux_kernels.hip.  Prints "launch_pieces cases=<n> bad=<m>".
#include <cstdio>
#include <vector>

#include "../../paper_2605_08565_amd/csrc/mxq_launch.hpp"

struct Launch { uint64_t threads, n, codes, scales, out; };
static std::vector<Launch> g_launches;

// a launch pushes its configuration, and the kernel's stub pops it and hands it to hipLaunchKernel
static dim3 g_grid, g_block;
extern "C" hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) { g_grid = grid; g_block = block; return hipSuccess; }
extern "C" hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream)
{
    *grid = g_grid; *block = g_block; *shared = 0; *stream = nullptr;
    return hipSuccess;
}
extern "C" hipError_t hipLaunchKernel(const void*, dim3 grid, dim3 block, void** args, size_t, hipStream_t)
{
    g_launches.push_back(Launch{(uint64_t)grid.x * block.x, *(uint64_t*)args[2], *(uint64_t*)args[0], *(uint64_t*)args[1], *(uint64_t*)args[6]});
    return hipSuccess;
}
extern "C" hipError_t hipGetLastError() { return hipSuccess; }

int main()
{
    int cases = 0, bad = 0;
    for (int dtype = 0; dtype < 2; ++dtype)
        for (int block : {2, 4, 8, 16, 32, 64, 128})
            for (int64_t base : {(int64_t)0, (int64_t)1 << 20, (int64_t)1 << 33, (int64_t)1 << 35, (int64_t)1 << 36, (int64_t)1 << 37, (int64_t)5 << 38})
                for (int64_t more : {(int64_t)block, (int64_t)(1 << 14) + block}) {
                    mxq::DequantArgs a{};
                    a.codes = (const uint8_t*)0x1000000; a.scales = (const uint8_t*)0x2000000; a.out = (void*)0x3000000;
                    a.n = base + more; a.block = block; a.scale_fmt = 1; a.dtype = dtype; a.T = 1.0f;
                    g_launches.clear();
                    const bool ok = mxq::launch_dequant(a) == hipSuccess;
                    uint64_t done = 0;
                    bool good = ok && !g_launches.empty();
                    for (const Launch& l : g_launches) {
                        good &= l.threads < ((uint64_t)1 << 32) && l.n > 0 && l.codes == 0x1000000 + done / 2 &&
                                l.scales == 0x2000000 + done / (uint64_t)block && l.out == 0x3000000 + done * (dtype == 0 ? 2 : 4);
                        done += l.n;
                    }
                    good &= done == (uint64_t)a.n;
                    ++cases;
                    if (!good && bad++ < 5)
                        std::printf("dtype %d block %d n %lld: %zu launches, %llu elements, %llu threads in the first\n", dtype, block, (long long)a.n,
                                    g_launches.size(), (unsigned long long)done, g_launches.empty() ? 0ull : (unsigned long long)g_launches[0].threads);
                }
    std::printf("launch_pieces cases=%d bad=%d\n", cases, bad);
    return bad != 0;
}
