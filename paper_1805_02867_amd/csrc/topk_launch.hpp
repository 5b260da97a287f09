// Launches of the top-k kernels: the choice between rows held on chip
// (topk_held.hpp) and streamed rows (topk.hpp), by shape.
#pragma once

#include "topk_held.hpp"

namespace osm {

// Split top-k in one kernel: chunk c of row r is workgroup r * segs + c (four
// wavefronts), which leaves its partial (K keys, pair) at the coherence
// point; the workgroup that completes a row (ctr[r] counts its chunks) merges
// the row's partials there and then, instead of a second kernel.  ctr starts
// at zero and is left at zero (the merger resets its row's count).
template <typename T, int U, int VAR>
__global__ __launch_bounds__(TK_BLOCK) void topk_split1(const T* __restrict__ x,
                                                       float* __restrict__ vals,
                                                       int32_t* __restrict__ idx,
                                                       uint64_t* __restrict__ pkeys,
                                                       MD* __restrict__ pmd, uint32_t* ctr,
                                                       int64_t N, int64_t V, int K, int64_t seg,
                                                       int64_t segs) {
    static_assert(topk_region<T, U>() >= TH_LIST, "the merge's list fits a region");
    __shared__ TopkSmem<T, U> sm;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t vr = blockIdx.x;
    if (lane < K) sm.region[wv][lane] = 0;
    if (lane == 0) sm.published[wv] = 0;
    __syncthreads();
    if (!topk_vrow<T, 4, U, VAR, true>(sm, x, nullptr, nullptr, pkeys, pmd, V, K, seg, segs,
                                             vr))
        return;
    // the partial's coherent stores have completed before the row's count moves
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const int64_t row = vr / segs;
    uint32_t done = 0;
    if (lane == 0)
        done = __hip_atomic_fetch_add(ctr + row, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    done = __builtin_amdgcn_readfirstlane(done);
    if (done != (uint32_t)segs - 1) return;
    // every chunk of the row is in: its partials are read at the coherence
    // point, after the count that says so
    struct {
        uint64_t (*list)[TH_LIST];
    } one = {reinterpret_cast<uint64_t(*)[TH_LIST]>(&sm.region[wv][0])};
    uint64_t key;
    MD md;
    held_merge<VAR, 1, TK_MERGE_B, Vec<T>::N == 8 ? 1u << 16 : 1u, true>(
        one, 0, pkeys + row * segs * K, pmd + row * segs, segs * K, segs, K, &key, &md);
    held_store<VAR>(key, md, vals, idx, row, K);
    if (lane == 0) __hip_atomic_store(ctr + row, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

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
            hipLaunchKernelGGL((topk_fused<T, 1, topk_unroll<T, 1>(), VAR>), grid, block, 0,
                               a.st, x, a.vals, a.idx, a.N, a.V, a.K);
        } else if (a.waves_per_row == 2) {
            if constexpr (VAR == TK_ONLINE) {  // the two-wavefront shape is built for Alg. 4 only
                constexpr int RB = TK_BLOCK / 128;
                dim3 grid((unsigned)((a.N + RB - 1) / RB));
                hipLaunchKernelGGL((topk_fused<T, 2, topk_unroll<T, 2>(), VAR>), grid,
                                   block, 0, a.st, x, a.vals, a.idx, a.N, a.V, a.K);
            } else {
                return hipErrorInvalidValue;
            }
        } else if (a.waves_per_row == 4) {
            dim3 grid((unsigned)a.N);
            hipLaunchKernelGGL((topk_fused<T, 4, topk_unroll<T, 4>(), VAR>), grid, block, 0,
                               a.st, x, a.vals, a.idx, a.N, a.V, a.K);
        } else {
            return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    // split: chunks of a.chunk elements, one workgroup (four wavefronts) each,
    // each row merged by its last chunk
    dim3 grid((unsigned)(a.N * a.S));
    hipLaunchKernelGGL((topk_split1<T, topk_split_unroll(), VAR>), grid, block, 0, a.st, x, a.vals,
                       a.idx, pkeys, pmd, a.ctr, a.N, a.V, a.K, a.chunk, a.S);
    return hipGetLastError();
}

}  // namespace osm
