// Reading ahead: workgroups that a launch has to spare pull weights of the launches behind it from HBM into the last-level cache
// (256 MB in front of HBM; what is read once stays there until newer reads replace it).  Nothing depends on them: they write
// nothing, and a launch that finds its weights in HBM is only slower.
//
// Why: with a few hundred rows a contraction is bound by how long a CU's fetches, which return in order, wait for HBM (768 rows,
// 3584 x 18944: 147 us with cold weights, 107 with cached ones; 512 rows, 4096 x 12288: 81 and 64), while the last round of tiles of the
// contraction in front of it leaves CUs without work.  It has to be other CUs that read: on the CU of a running tile a read-ahead
// holds up the fetches behind it (no gain, or a third slower).  Norms and attention of block rows, which leave CUs idle too, got slower by
// as much as the weight streams behind them gained.
#pragma once
#include "psd_internal.h"
#include "device_types.h"

// extra workgroup `wg` of w.wgs: its share of the units of 1 KB, eight of them in flight per wavefront
__device__ __forceinline__ void warm_part(const Warm &w, int wg) {
    const int waves = blockDim.x >> 6, lane = threadIdx.x & 63;
    const int first = (wg * waves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * 8, step = w.wgs * waves * 8;
#pragma unroll
    for (int i = 0; i < Warm::ITEMS; ++i) {
        const int units = w.rows[i] * w.kb[i];
        for (int u = first; u < units; u += step) {
            uint4 v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int at = min(u + e, units - 1);
                v[e] = *reinterpret_cast<const uint4 *>(w.p[i] + (at / w.kb[i]) * w.stride[i] + (at % w.kb[i]) * 1024 + lane * 16);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) asm volatile("" ::"v"(v[e].x), "v"(v[e].y), "v"(v[e].z), "v"(v[e].w));   // (the loads are not removed)
        }
    }
}
