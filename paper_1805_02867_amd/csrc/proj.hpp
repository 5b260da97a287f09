// Projection layer on the gfx950 matrix cores: P = X . Y^T for row-major
// bfloat16 X (nx x K) and Y (ny x K), binary32 accumulation.  The projection
// ahead of the softmax (Section 1) is logits = h . W^T; the Discussion's
// fusion runs the softmax (+ top-k) on the tile while it is still on chip.
//
// Tile: TX x TY of P per workgroup of WX x WY wavefronts, each a block of
// 32 x 32 v_mfma_f32_32x32x16_bf16 products.  K advances in steps of 64
// through two LDS stages.  Operands travel global -> LDS by buffer loads
// with the LDS as destination (no staging registers); the buffer descriptor
// of each operand starts at the tile's first row and ends at the matrix's
// end, so rows past the matrix, and chunks past K (given an offset beyond
// the descriptor), read as zeros without any branch on the load path.  The
// step count is rounded up to even, the extra step reading zeros, so that
// every tile starts in stage 0 and both stages have fixed roles in the code.
//
// MFMA 32x32x16 lane layout (checked on the hardware): lane l supplies
// A[m = l % 32][k = 8 (l / 32) + j] and B[k = 8 (l / 32) + j][n = l % 32] for
// j < 8, and receives C[m = 8 (r / 4) + 4 (l / 32) + r % 4][n = l % 32] in
// result register r < 16.
#pragma once

#include <type_traits>

#include "md.hpp"

namespace osm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int PJ_BK = 64;  // K per step

// Cache policy (non-temporal) of an operand that one workgroup reads once and
// that the 256 MB last-level cache cannot hold for the next call: the reads of
// 1.05 GB alone, in the order of the tiles below, take 172 us without it and
// 152 with it (6.1 and 6.9 TB/s), whatever the step's shape or depth.
constexpr int PJ_ONCE = 2;

// Workgroups are dealt to the eight XCDs in turn (workgroup b to XCD b % 8),
// each with its own L2.  Logical id of workgroup b when XCD k takes the k-th
// contiguous block of `per` logical ids, so that the workgroups sharing an
// L2 work on neighbouring tiles and share their operand tiles there.  The
// grid holds 8 * per workgroups; ids past the tile count have no work.
__device__ __forceinline__ int64_t xcd_logical(int64_t b, int64_t per) {
    return (b % 8) * per + b / 8;
}

// P row of result register `i` within a 32 x 32 block: 8 (i / 4) + 4 (l / 32) + i % 4.
__device__ __forceinline__ int row_in_32(int i, int lane) {
    return 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
}

// LDS slot of 16-byte chunk kc of a tile row (rows of 64 bfloat16, 128 B).
// The LDS serves a 16-byte-per-lane read 16 lanes at a time from 64
// four-byte banks (256 B); the 16 lanes of a fragment read hold 16
// consecutive rows and one chunk, two rows per 256 B of banks, so the slot
// is XORed with (row / 2) % 8: the 16 (row parity, slot) pairs are then all
// distinct and the read is free of bank conflicts.
__device__ __forceinline__ int pj_slot(int row, int kc) { return kc ^ ((row >> 1) & 7); }

template <int TX_, int TY_, int WX_, int WY_>
struct PjCfg {
    static constexpr int TX = TX_, TY = TY_, WX = WX_, WY = WY_;
    static constexpr int NW = WX * WY, NT = 64 * NW;            // wavefronts, threads
    static constexpr int MI = TX / 32 / WX, NI = TY / 32 / WY;  // blocks per wavefront
    static constexpr int LX = TX * 8 / NT, LY = TY * 8 / NT;    // loads per thread per stage
    static_assert(LX * NT == TX * 8 && LY * NT == TY * 8, "whole loads");
    // X and Y tiles of the two stages (each stage contiguous)
    struct Stage {
        uint16_t x[TX][PJ_BK];
        uint16_t y[TY][PJ_BK];
    };
    struct Smem {
        Stage st[2];
    };
};

// Buffer descriptor of `m` (rows x K) from row r0 on; reads at byte offsets
// at or past its size return zeros.  Valid offsets in a tile stay below
// 256 K 2 <= 2^29 (K <= 2^20), so the size saturates at 2^31 - 1 harmlessly.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t pj_rsrc(const uint16_t* m, int64_t rows,
                                                         int64_t K, int64_t r0) {
    const int64_t bytes = (rows - r0) * K * 2;
    return __builtin_amdgcn_make_buffer_rsrc((void*)(m + r0 * K), (short)0,
                                             (int)(bytes < 0x7FFFFFFF ? bytes : 0x7FFFFFFF),
                                             0x00020000);
}
constexpr uint32_t PJ_OOB = 0x80000000u;  // an offset past every descriptor

// Per-thread part of the load addressing: load j of a stage covers LDS chunk
// p = 64 (NW j + wave) + lane, i.e. row p / 8, slot p % 8, which holds the
// row's chunk kc = pj_slot(row, p % 8) (the map is an involution).  Row
// p / 8 = 8 (NW j + wave) + lane / 8, so kc does not depend on j, and the
// byte offset of load j is voff + j * jstride.
struct PjAddr {
    uint32_t voff, jstride;
    int kc;
    template <class C>
    __device__ __forceinline__ static PjAddr make(int64_t K) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        const int p = 64 * wave + lane;
        const int row = p >> 3, kc = pj_slot(row, p & 7);
        return PjAddr{(uint32_t)(row * K * 2 + kc * 16), (uint32_t)(8 * C::NW * K * 2), kc};
    }
};

// Loads of step k (elements 64 k ... of each row) of one operand tile.
// Wavefront index, known to the compiler to be uniform (scalar registers).
__device__ __forceinline__ int pj_wave() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// AUX: cache policy of the loads, 0 or PJ_ONCE.
template <class C, int ROWS, int L, int AUX>
__device__ __forceinline__ void pj_dma(uint16_t (&tile)[ROWS][PJ_BK], __amdgpu_buffer_rsrc_t rs,
                                       const PjAddr& a, int64_t K, int64_t k) {
    const int wave = pj_wave();
    const int64_t k0 = k * PJ_BK;
    // chunks at or past K (the last step of a ragged K, and padded steps) read zeros
    const bool oob = k0 + PJ_BK > K && k0 + a.kc * 8 >= K;
#pragma unroll
    for (int j = 0; j < L; ++j) {
        const int base = 64 * (C::NW * j + wave);  // first chunk of this load (wave-uniform)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rs, (__attribute__((address_space(3))) void*)(&tile[0][0] + base * 8), 16,
            oob ? PJ_OOB : a.voff + j * a.jstride, (int)(k0 * 2), 0, AUX);
    }
}

// Byte offsets, within a tile, of a lane's fragment reads for the blocks of
// a wavefront whose first row is `base` (a multiple of 32): sub-step ks of
// block m reads row base + 32 m + l % 32, chunk 2 ks + l / 32, at byte
// off[ks] + 4096 m.  The row adds a multiple of 16 to (row / 2) for every m,
// so the slot's XOR term is (l % 32) / 2 % 8 for all blocks: one offset per
// sub-step, and the block's part is an instruction offset.
template <int KS>
struct PjFragOff {
    uint32_t off[KS];
    __device__ __forceinline__ static PjFragOff make(int base) {
        const int lane = threadIdx.x & 63, lr = lane & 31, lh = lane >> 5;
        PjFragOff f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            f.off[ks] = (uint32_t)((base + lr) * PJ_BK * 2 + 16 * pj_slot(lr, 2 * ks + lh));
        return f;
    }
};

template <int ROWS>
__device__ __forceinline__ bf16x8 pj_frag(const uint16_t (&tile)[ROWS][PJ_BK], uint32_t off,
                                          int m) {
    const char* p = reinterpret_cast<const char*>(&tile[0][0]) + off + m * 32 * PJ_BK * 2;
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(p));
}

// acc[mi][ni] += the wavefront's (32 MI) x (32 NI) block of X-tile . Y-tile^T
// over one K step; the block starts at the X-tile row and Y-tile row whose
// fragment offsets are xo and yo.  The fragments of sub-step ks + 1 are read
// into the other register set before the products of sub-step ks are issued.
template <class C>
__device__ __forceinline__ void pj_mma(const uint16_t (&xt)[C::TX][PJ_BK],
                                       const uint16_t (&yt)[C::TY][PJ_BK],
                                       const PjFragOff<PJ_BK / 16>& xo,
                                       const PjFragOff<PJ_BK / 16>& yo,
                                       f32x16 (&acc)[C::MI][C::NI]) {
    constexpr int MI = C::MI, NI = C::NI, KS = PJ_BK / 16;
    bf16x8 a[2][MI], b[2][NI];  // [register set][block]
    auto read = [&](int set, int ks) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) a[set][mi] = pj_frag(xt, xo.off[ks], mi);
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) b[set][ni] = pj_frag(yt, yo.off[ks], ni);
    };
    read(0, 0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const int cur = ks & 1;
        if (ks + 1 < KS) read(cur ^ 1, ks + 1);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
                acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[cur][mi], b[cur][ni],
                                                                      acc[mi][ni], 0, 0, 0);
    }
    // Keep that order through scheduling: the first fragment reads, then per
    // sub-step the next sub-step's reads ahead of its products (mask 0x100:
    // LDS reads, 0x008: matrix instructions).
    __builtin_amdgcn_sched_group_barrier(0x100, MI + NI, 0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        if (ks + 1 < KS) __builtin_amdgcn_sched_group_barrier(0x100, MI + NI, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, MI * NI, 0);
    }
}

// Stage hand-over.  The loads of the next stage were issued one step
// earlier; each thread waits for its own, and for its own fragment reads of
// the stage about to be refilled (the compiler may leave the last of them
// in flight, their products scheduled after the barrier), then the
// workgroup barrier makes every thread's loads visible and tells that every
// wavefront has finished reading that stage.  (A plain s_barrier: the fenced
// __syncthreads would also make the compiler wait for everything else.)
__device__ __forceinline__ void pj_handover() {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Step count of a K: whole steps of 64, rounded up to even.
__device__ __forceinline__ int64_t pj_steps(int64_t K) {
    return ((K + PJ_BK - 1) / PJ_BK + 1) / 2 * 2;
}

// Issue both operands' loads of step k into stage `st`.
template <class C, int XA, int YA>
__device__ __forceinline__ void pj_issue(typename C::Smem& sm, int st, __amdgpu_buffer_rsrc_t rx,
                                         __amdgpu_buffer_rsrc_t ry, const PjAddr& a, int64_t K,
                                         int64_t k) {
    pj_dma<C, C::TX, C::LX, XA>(sm.st[st].x, rx, a, K, k);
    pj_dma<C, C::TY, C::LY, YA>(sm.st[st].y, ry, a, K, k);
}

// The workgroup's tiles t = t0, t0 + 1, ... < t1, each TX x TY of P at
// coords(t) = (x0, y0) (x0 < nx, y0 < ny), accumulated over all of K;
// epi(t, x0, y0, acc) runs after each tile with stage 1 of the LDS free for
// its own use (every wavefront is past its last read of it, and it is
// refilled only after the next tile's first hand-over).  The next tile's
// first stage is in flight while epi runs.  Every thread of the workgroup
// must call this, with t0 < t1.
// XA, YA: cache policy of the operands' loads.
template <class C, int XA, int YA, class Coords, class Epi>
__device__ __forceinline__ void pj_run(const uint16_t* __restrict__ X, int64_t nx,
                                       const uint16_t* __restrict__ Y, int64_t ny, int64_t K,
                                       int64_t t0, int64_t t1, typename C::Smem& sm,
                                       Coords&& coords, Epi&& epi) {
    const int wave = pj_wave();
    const int bx = (wave / C::WY) * 32 * C::MI, by = (wave % C::WY) * 32 * C::NI;
    const PjFragOff<PJ_BK / 16> xo = PjFragOff<PJ_BK / 16>::make(bx),
                                yo = PjFragOff<PJ_BK / 16>::make(by);
    const PjAddr a = PjAddr::make<C>(K);
    const int64_t nk = pj_steps(K);
    int64_t x0, y0;
    coords(t0, x0, y0);
    __amdgpu_buffer_rsrc_t rx = pj_rsrc(X, nx, K, x0), ry = pj_rsrc(Y, ny, K, y0);
    pj_issue<C, XA, YA>(sm, 0, rx, ry, a, K, 0);
    for (int64_t t = t0; t < t1; ++t) {
        const bool more = t + 1 < t1;
        int64_t xn = x0, yn = y0;
        if (more) coords(t + 1, xn, yn);
        const __amdgpu_buffer_rsrc_t rxn = pj_rsrc(X, nx, K, xn), ryn = pj_rsrc(Y, ny, K, yn);
        f32x16 acc[C::MI][C::NI];
#pragma unroll
        for (int mi = 0; mi < C::MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < C::NI; ++ni)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[mi][ni][i] = 0.0f;
        for (int64_t k = 0; k < nk; k += 2) {
            pj_handover();
            pj_issue<C, XA, YA>(sm, 1, rx, ry, a, K, k + 1);
            pj_mma<C>(sm.st[0].x, sm.st[0].y, xo, yo, acc);
            pj_handover();
            if (k + 2 < nk) pj_issue<C, XA, YA>(sm, 0, rx, ry, a, K, k + 2);
            else if (more) pj_issue<C, XA, YA>(sm, 0, rxn, ryn, a, K, 0);
            pj_mma<C>(sm.st[1].x, sm.st[1].y, xo, yo, acc);
        }
        // every wavefront's last read of stage 1 is done before epi may write it
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        epi(t, x0, y0, acc);
        x0 = xn;
        y0 = yn;
        rx = rxn;
        ry = ryn;
    }
}

// ------------------------------------------------- 256 x 256, two wave groups
// The 256 x 256 tile by eight wavefronts in two groups that take turns: while
// the four wavefronts of one group (one per SIMD) multiply, the other group's
// read their fragments and issue loads, so each SIMD's matrix core always has
// a wavefront on it.  In pj_run all eight read after each barrier together and
// the matrix cores wait for the first fragments.  Measured: matrix cores busy
// 77% of the cycles against 60%; logits of 4000 x 4096 x 32000 977 -> 893 us,
// 512 x 4096 x 128256 517 -> 482 (1.12 PF/s), 4000 x 4096 x 128256 3825 -> 3490
// (1.20 PF/s).  What bounds it now is power (the clock settles near 1.6 GHz)
// and the loads' way into the LDS: without the loads it runs at 1.45 PF/s,
// without any wait for them no faster than with.
//
// A K step of 64 is four phases, one per quadrant of a wavefront's block.
// Wavefront (wx, wy) multiplies, with each half h of the X tile (128 rows) and
// half g of the Y tile, the 64 rows 128 h + 64 wx + ... by the 32 columns
// 128 g + 32 wy + ..., so every wavefront reads all four half tiles, one per
// phase, and a half tile is free for its next load as soon as its phase is
// over:
//   phase 1 reads X half 0, multiplies with the Y half 0 already in registers;
//   phase 2 reads Y half 1, multiplies X half 0 with it;
//   phase 3 reads X half 1, multiplies it with Y half 1;
//   phase 4 reads the next step's Y half 0, multiplies X half 1 with Y half 0.
// A phase is a read section and a multiply section with a barrier after each;
// group 1 runs one section behind group 0 (an extra barrier at the start of a
// tile, one of group 0 at its end).  A read section ends with its reads done.
// The multiply section of a phase also issues the load, for the K step after
// next, of the half tile that the phase before read: group 1 read it two
// sections ago, or three, so a load never meets a read.  (Issued in the read
// sections, the loads cost 2-3% more.)
//
// Counting.  Every multiply section issues two loads a thread.  What section j
// loads is first read in section j + 7, by group 0 one barrier after group 1's
// read section j + 6 ends: so every read section waits until at most 10 loads
// (those of the last five multiply sections) are in flight.  Loads past the
// last step read beyond the descriptor (zeros), which keeps the counts uniform.
template <class C>
struct PpSmem {
    uint16_t x[2][C::TX][PJ_BK];  // [stage]
    uint16_t y[2][C::TY][PJ_BK];
};

// Row of the block's 32 x 32 blocks: X rows of block mi, Y columns of block ni
// (offsets within the tile, before the lane's own part).
__device__ __forceinline__ int pp_row(int wx, int mi) {
    return (mi >> 1) * 128 + wx * 64 + (mi & 1) * 32;
}
__device__ __forceinline__ int pp_col(int wy, int ni) { return ni * 128 + wy * 32; }

__device__ __forceinline__ void pp_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

// The workgroup's tiles t0 <= t < t1 as pj_run, for the 256 x 256 tile in 2 x 4
// wavefronts: epi(t, x0, y0, acc) with acc[mi][ni] the block at pp_row(wx, mi),
// pp_col(wy, ni).  The stages stay in use while epi runs, and nothing else may
// wait on vmcnt order: epi's own loads and stores only make later waits longer.
// XA: cache policy of X's loads.
template <class C, int XA, class Coords, class Epi>
__device__ __forceinline__ void pp_run(const uint16_t* __restrict__ X, int64_t nx,
                                       const uint16_t* __restrict__ Y, int64_t ny, int64_t K,
                                       int64_t t0, int64_t t1, PpSmem<C>& sm, Coords&& coords,
                                       Epi&& epi) {
    static_assert(C::TX == 256 && C::TY == 256 && C::WX == 2 && C::WY == 4, "four half tiles");
    constexpr int KS = PJ_BK / 16;
    constexpr int STAGE = 256 * PJ_BK * 2, HALF = 128 * PJ_BK * 2;  // bytes
    const int wave = pj_wave(), wx = wave >> 2, wy = wave & 3;
    const int lane = threadIdx.x & 63;
    // A fragment of sub-step ks is at off ^ 32 ks from the block's start: the
    // slot's XOR term is the lane's alone, and ks moves the slot's upper two
    // bits.  Kept as one offset per operand (PjFragOff's four would not fit
    // beside the fused kernel's lists), re-derived at each read section.
    uint32_t xoff = PjFragOff<1>::make(wx * 64).off[0], yoff = PjFragOff<1>::make(wy * 32).off[0];
    const char* const xb = reinterpret_cast<const char*>(&sm.x[0][0][0]);
    const char* const yb = reinterpret_cast<const char*>(&sm.y[0][0][0]);
    auto frag = [](const char* b, uint32_t off, int at) {
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(b + off + at));
    };
    // load j of a half tile: rows 64 j + 8 wave + lane / 8 of it
    const int lrow = 8 * wave + (lane >> 3), kc = pj_slot(lrow, lane & 7);
    uint32_t voff = (uint32_t)(lrow * K * 2 + kc * 16);
    const uint32_t vstep = (uint32_t)(64 * K * 2);
    auto load = [&](auto aux, uint16_t (&tile)[256][PJ_BK], int half, __amdgpu_buffer_rsrc_t rs,
                    int64_t k, int j) {
        constexpr int AUX = decltype(aux)::value;
        const int k0 = (int)(k * PJ_BK);
        const bool oob = k0 + kc * 8 >= (int)K;  // past the end of the rows
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rs,
            (__attribute__((address_space(3))) void*)(&tile[half * 128][0] +
                                                      64 * (8 * j + wave) * 8),
            16, oob ? PJ_OOB : voff + (2 * half + j) * vstep, k0 * 2, 0, AUX);
    };
    const std::integral_constant<int, XA> ax;
    const std::integral_constant<int, 0> ay;
    const int64_t nk = pj_steps(K);
    int64_t x0, y0;
    coords(t0, x0, y0);
    __amdgpu_buffer_rsrc_t rx = pj_rsrc(X, nx, K, x0), ry = pj_rsrc(Y, ny, K, y0);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            load(ay, sm.y[s], h, ry, s, 0);
            load(ay, sm.y[s], h, ry, s, 1);
            load(ax, sm.x[s], h, rx, s, 0);
            load(ax, sm.x[s], h, rx, s, 1);
        }
    bf16x8 a[2][KS], b[2][KS];  // X half (two blocks), Y halves
    asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
    pp_barrier();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) b[0][ks] = frag(yb, yoff ^ (32 * ks), 0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    pp_barrier();

    for (int64_t t = t0; t < t1; ++t) {
        int64_t xn = x0, yn = y0;
        const bool more = t + 1 < t1;
        if (more) coords(t + 1, xn, yn);
        // past the last tile: descriptors that hold nothing
        const __amdgpu_buffer_rsrc_t rxn = pj_rsrc(X, more ? nx : xn, K, xn),
                                     ryn = pj_rsrc(Y, more ? ny : yn, K, yn);
        f32x16 acc[C::MI][C::NI];
#pragma unroll
        for (int mi = 0; mi < C::MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < C::NI; ++ni)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[mi][ni][i] = 0.0f;
        auto read_x = [&](int stage, int h) {
            asm volatile("" : "+v"(xoff));
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int mi = 0; mi < 2; ++mi)
                    a[mi][ks] = frag(xb, xoff ^ (32 * ks),
                                     stage * STAGE + h * HALF + mi * 32 * PJ_BK * 2);
        };
        auto read_y = [&](int stage, int g, bf16x8 (&to)[KS]) {
            asm volatile("" : "+v"(yoff));
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                to[ks] = frag(yb, yoff ^ (32 * ks), stage * STAGE + g * HALF);
        };
        auto end_read = [&]() {
            asm volatile("s_waitcnt vmcnt(10) lgkmcnt(0)" ::: "memory");
            pp_barrier();
        };
        auto multiply = [&](int h, int g, const bf16x8 (&bb)[KS], auto&& issue) {
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int mi = 0; mi < 2; ++mi) {
                    acc[2 * h + mi][g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        a[mi][ks], bb[ks], acc[2 * h + mi][g], 0, 0, 0);
                    if (mi == 0 && (ks == 0 || ks == 2)) {
                        __builtin_amdgcn_sched_barrier(0);
                        issue(ks / 2);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            __builtin_amdgcn_s_setprio(0);
            pp_barrier();
        };
        // K step k in stage s, whose Y half 0 is in p; q is free.
        auto step = [&](int64_t k, auto s_, bf16x8 (&p)[KS], bf16x8 (&q)[KS]) {
            constexpr int s = decltype(s_)::value;
            const bool next = k + 2 >= nk;  // the loads belong to the next tile
            const int64_t lk = next ? k + 2 - nk : k + 2;
            const __amdgpu_buffer_rsrc_t lx = next ? rxn : rx, ly = next ? ryn : ry;
            read_x(s, 0);
            end_read();
            multiply(0, 0, p, [&](int j) { load(ay, sm.y[s], 0, ly, lk, j); });
            read_y(s, 1, q);
            end_read();
            multiply(0, 1, q, [&](int j) { load(ax, sm.x[s], 0, lx, lk, j); });
            read_x(s, 1);
            end_read();
            multiply(1, 1, q, [&](int j) { load(ay, sm.y[s], 1, ly, lk, j); });
            read_y(s ^ 1, 0, q);
            end_read();
            multiply(1, 0, p, [&](int j) { load(ax, sm.x[s], 1, lx, lk, j); });
        };
        if (wx == 1) pp_barrier();
        for (int64_t k = 0; k < nk; k += 2) {
            step(k, std::integral_constant<int, 0>{}, b[0], b[1]);
            step(k + 1, std::integral_constant<int, 1>{}, b[1], b[0]);
        }
        if (wx == 0) pp_barrier();
        epi(t, x0, y0, acc);
        x0 = xn;
        y0 = yn;
        rx = rxn;
        ry = ryn;
    }
    // the last loads (of nothing) have landed before the LDS is given back
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

}  // namespace osm
