// Launches of the top-k kernels: the choice between rows held on chip
// (topk_held.hpp) and streamed rows (topk.hpp), by shape.
#pragma once

#include "topk_held.hpp"

namespace osm {

// Launch of one variant for one element type (see TopkLaunch).
template <typename T, int VAR>
hipError_t launch_topk_t(const TopkLaunch& a) {
    dim3 block(TK_BLOCK);
    const T* x = static_cast<const T*>(a.x);
    uint64_t* pkeys = static_cast<uint64_t*>(a.part);
    MD* pmd = reinterpret_cast<MD*>(pkeys + a.N * a.S * a.K);
    if constexpr (VAR != TK_SAFE) {  // one read: rows and chunks short enough are held on chip
        hipError_t e;
        if (launch_topk_held<T, VAR>(a, pkeys, pmd, &e)) return e;
    }
    if (a.S <= 1) {
        if (a.waves_per_row == 1) {
            constexpr int RB = TK_BLOCK / 64;
            dim3 grid((unsigned)((a.N + RB - 1) / RB));
            hipLaunchKernelGGL((topk_fused<T, 1, topk_unroll<T, 1>(), VAR, false>), grid, block, 0,
                               a.st, x, a.vals, a.idx, nullptr, nullptr, a.N, a.V, a.K, a.V,
                               (int64_t)1);
        } else if (a.waves_per_row == 2) {
            if constexpr (VAR == TK_ONLINE) {  // the two-wavefront shape is built for Alg. 4 only
                constexpr int RB = TK_BLOCK / 128;
                dim3 grid((unsigned)((a.N + RB - 1) / RB));
                hipLaunchKernelGGL((topk_fused<T, 2, topk_unroll<T, 2>(), VAR, false>), grid,
                                   block, 0, a.st, x, a.vals, a.idx, nullptr, nullptr, a.N, a.V,
                                   a.K, a.V, (int64_t)1);
            } else {
                return hipErrorInvalidValue;
            }
        } else if (a.waves_per_row == 4) {
            dim3 grid((unsigned)a.N);
            hipLaunchKernelGGL((topk_fused<T, 4, topk_unroll<T, 4>(), VAR, false>), grid, block, 0,
                               a.st, x, a.vals, a.idx, nullptr, nullptr, a.N, a.V, a.K, a.V,
                               (int64_t)1);
        } else {
            return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    // split: chunks of a.chunk elements, one workgroup (four wavefronts) each
    dim3 grid((unsigned)(a.N * a.S));
    if (a.ctr) {  // merge by each row's last chunk, in the same kernel
        hipLaunchKernelGGL((topk_split1<T, topk_split_unroll(), VAR>), grid, block, 0, a.st, x,
                           a.vals, a.idx, pkeys, pmd, a.ctr, a.N, a.V, a.K, a.chunk, a.S);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((topk_fused<T, 4, topk_split_unroll(), VAR, true>), grid, block, 0, a.st,
                       x, nullptr, nullptr, pkeys, pmd, a.N, a.V, a.K, a.chunk, a.S);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    constexpr int WB = TK_BLOCK / 64;
    dim3 mgrid((unsigned)((a.N + WB - 1) / WB));
    hipLaunchKernelGGL((topk_merge<VAR>), mgrid, block, 0, a.st, pkeys, pmd, a.vals, a.idx, a.N,
                       a.S, a.K);
    return hipGetLastError();
}

}  // namespace osm
