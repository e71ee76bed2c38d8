// write_runs with places handed out in any order: the list kernels themselves only ever see their lanes served in order.
#include <hip/hip_runtime.h>

#include "ap_split.hpp"

namespace {
// ids: [n_tiles][kTile], M where a request is not listed; places: [n_tiles][kTile], those of a replica's requests a permutation of 0 ..
// count - 1.  One wavefront takes every gridDim.x-th tile, so that what a tile leaves in LDS is there when the next one begins.
__global__ __launch_bounds__(kWave) void k_write_runs(SplitParams p, const uint16_t* ids, const uint16_t* places) {
    extern __shared__ __align__(16) unsigned char lds[];
    const uint32_t lane = threadIdx.x;
    init_runs(p, lds, lane);
    __syncthreads();
    const uint32_t runs_at = lds_address(lds);
    uint32_t* run = reinterpret_cast<uint32_t*>(lds);
    for (uint32_t j = blockIdx.x; j < p.n_tiles; j += gridDim.x) {
        uint32_t at[kTileSteps], place[kTileSteps];
        for (uint32_t s = 0; s < kTileSteps; ++s) {
            const uint32_t id = ids[j * kTile + s * kWave + lane];
            const bool listed = id < p.M;
            if (listed) atomicAdd(&run[id], 1u);
            at[s] = runs_at + 4u * (listed ? id : p.M + lane);
            place[s] = listed ? places[j * kTile + s * kWave + lane] : p.tile_cap / 2u;
        }
        write_runs(p, j, lane, lds, at, place, [](uint32_t, uint32_t) {});
    }
}
}  // namespace

extern "C" uint32_t runs_tile_cap(uint32_t M) { return kTile + 7u * ((M + 7u) / 8u * 8u); }

// desc: [n_tiles][M], lists: [n_tiles][runs_tile_cap(M)]; every pointer is device memory.  0: done.
extern "C" int runs_write(const uint16_t* ids, const uint16_t* places, uint32_t M, uint32_t n_tiles, uint32_t* desc, uint16_t* lists) {
    if (M == 0u || M > AP_MAX_REPLICAS || n_tiles == 0u) return 1;
    SplitParams p{};
    p.M = M;
    p.n_tiles = n_tiles;
    p.tile_cap = runs_tile_cap(M);
    p.desc = desc;
    p.lists = lists;
    hipLaunchKernelGGL(k_write_runs, dim3((n_tiles + 1u) / 2u), dim3(kWave), runs_bytes(M, p.tile_cap), nullptr, p, ids, places);
    return hipGetLastError() == hipSuccess && hipDeviceSynchronize() == hipSuccess ? 0 : 2;
}
