// Projection kernels: the plain projection (logits written out), and the
// projection with the online softmax and top-k fused into its epilogue, so
// that the logits never leave the chip (the Discussion's proposal).
//
// Fused kernel.  Workgroup (c, b) computes P = W . h^T for the vocabulary
// tiles of chunk c against a strip of batch rows: with W as the MFMA's A
// operand, each lane's result registers hold, per tile, a run of vocabulary
// entries of each of its batch rows (columns of P), so a lane keeps, for each
// of those rows,
//  * the online pair (s, d) of the entries it has seen (Alg. 3's update,
//    with the reference moved only when the tile maximum passes it by more
//    than kLazy, as in the other one-pass kernels), and
//  * its own sorted list of the K largest keys it has seen (Alg. 4's buffer),
//    entered only by values at or above the list's K-th value.
// Every holder of a batch row in a workgroup (two lane halves in each
// wavefront along the vocabulary) writes its pair and list as a partial;
// a second kernel (topk_merge_held) combines a row's partials (Eq. 4 for the
// pairs, the key order for the lists).
#include "proj.hpp"
#include "topk_held.hpp"

namespace osm {

// Plain logits: 256 x 256 tiles for eight wavefronts when the tile count
// fills the chip twice over, else 128 x 128 tiles for four (two workgroups
// per CU), which keep small problems spread over more CUs.
using PjBig = PjCfg<256, 256, 2, 4>;
using PjSmall = PjCfg<128, 128, 2, 2>;
// Fused, by batch size and K (the vocabulary tile is 256 entries past 64 rows; the
// lanes' top-K lists live in registers):
//  * 256 x 256 (K <= 8, N > 128): the two-group core's 2 x 4 wavefronts, two
//    batch rows per lane; 128 result registers and 128 others per lane (the
//    lists and the row state are stored away once per tile, around the K
//    loop), so two wavefronts share each SIMD.  Projection + top-5, us, against
//    the same epilogue's forerunner on pj_run: 4000 x 4096 x 32000 950 -> 875,
//    4000 x 1024 x 32000 384 -> 307, 512 x 4096 x 128256 566 -> 494;
//    also for 8 < K <= 16 where the products outweigh the longer lists'
//    epilogue (H >= 2048, and at least two tiles a workgroup: 4000 x 4096 x
//    32000 top-16 1300 -> 1000 us, 1000 x 4096 x 32000 351 -> 297, 4000 x 2048
//    x 32000 630 -> 605; but 4000 x 1024 x 32000 365 -> 408, and in one tile a
//    workgroup 512 x 2048 x 32000 107 -> 118);
//  * 256 x 128 in 2 x 4 wavefronts (8 < K <= 16, N > 1024 otherwise): one batch
//    row per lane, also two wavefronts per SIMD;
//  * 256 x 128 in 1 x 4 wavefronts (otherwise, N > 64): one batch row per
//    lane, one wavefront per SIMD, measured faster than the 2 x 4 layout up
//    to N = 512;
//  * 64 rows of batch (N <= 64), one batch row per lane, so small batches do
//    not pay for a strip of 256: 256 x 64 in 2 x 2 wavefronts, two workgroups a
//    CU, for the largest vocabularies; 128 x 64 in 2 x 2 (K <= 8), three a CU,
//    while those take every tile at once; 64 x 64 in 1 x 2 for small ones, of
//    which the taller tiles would occupy half of the CUs or fewer.  Projection
//    + top-5 of 64 or 40 rows, us, in 256, 128 and 64 rows of vocabulary: 4096 x
//    8192 57.6 / 45.1 / 40.6, 4096 x 32000 77.3 / 66.8 / 63.9, 1024 x 32000 27.0
//    / 24.2 / 22.2, 4096 x 50257 108 / 96.5 / 106.6, 4096 x 90000 142 / 136 /
//    150, 4096 x 128256 167 / 175 / 187.  For K > 8 the merge of twice the lists
//    costs more: 64 x 64 only up to two tiles a CU, and past 16384 only where
//    the products weigh enough (top-16 of 40 rows, 256 against 64: 4096 x 20000
//    66.7 / 52.8, 256 x 8192 20.2 / 18.4; but 256 x 32000 22.8 / 24.3).
using PjFused8 = PjCfg<256, 256, 2, 4>;
using PjFused16W = PjCfg<256, 128, 2, 4>;
using PjFused16 = PjCfg<256, 128, 1, 4>;
using PjFusedN = PjCfg<256, 64, 2, 2>;
using PjFusedNM = PjCfg<128, 64, 2, 2>;
using PjFusedNS = PjCfg<64, 64, 1, 2>;
enum FusedCfg { FUSED_8, FUSED_16, FUSED_16W, FUSED_16T, FUSED_N, FUSED_NM, FUSED_NS };
static FusedCfg fused_cfg(int64_t N, int64_t H, int64_t V, int K, int cus) {
    if (N <= 64) {
        const int64_t t64 = (V + 63) / 64, t128 = (V + 127) / 128;
        if (K <= 8)
            return 2 * t64 <= 5 * (int64_t)cus    ? FUSED_NS
                   : t128 <= 3 * (int64_t)cus ? FUSED_NM
                                              : FUSED_N;
        return t64 <= 2 * (int64_t)cus && (H >= 1024 || t64 <= cus) ? FUSED_NS : FUSED_N;
    }
    if (N > 128) {
        if (K <= 8) return FUSED_8;
        const int64_t tiles = ((N + 255) / 256) * ((V + 255) / 256);
        if (H >= 2048 && tiles > cus) return FUSED_16;
    }
    return N > 1024 ? FUSED_16W : FUSED_16T;
}

// ------------------------------------------------------------ plain logits
// Tiles in grouped order: groups of up to 8 batch strips, each taken across
// all vocabulary tiles before the next group, so that a contiguous block of
// logical ids covers a compact block of tiles.
constexpr int64_t PJ_GROUP = 8;

// This workgroup's tile in that order; false if it has none.
template <class C>
__device__ __forceinline__ bool logits_tile(int64_t N, int64_t V, int64_t per, int64_t& x0,
                                            int64_t& y0) {
    const int64_t nb = (N + C::TX - 1) / C::TX, nt = (V + C::TY - 1) / C::TY;
    const int64_t lid = xcd_logical(blockIdx.x, per);
    if (lid >= nb * nt) return false;
    const int64_t in_group = PJ_GROUP * nt;
    const int64_t first = (lid / in_group) * PJ_GROUP;
    const int64_t gsize = nb - first < PJ_GROUP ? nb - first : PJ_GROUP;
    x0 = (first + (lid % in_group) % gsize) * C::TX;  // batch
    y0 = ((lid % in_group) / gsize) * C::TY;          // vocabulary
    return true;
}

// One 32 x 32 block of logits, whose first row and column are given.
// Streaming stores: the logits are not read again by this kernel (measured
// 11-12% faster at 4000 x 1024 x 32000, also for a top-k reading them next;
// neutral at H = 4096).
__device__ __forceinline__ void store_block(const f32x16& acc, float* __restrict__ out, int64_t N,
                                            int64_t V, int64_t row0, int64_t col0) {
    const int lane = threadIdx.x & 63;
    const int64_t col = col0 + (lane & 31);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int64_t row = row0 + row_in_32(i, lane);
        if (row < N && col < V) __builtin_nontemporal_store(acc[i], out + row * V + col);
    }
}

template <class C, int WA>
__global__ __launch_bounds__(C::NT) void proj_logits(const uint16_t* __restrict__ h,
                                                     const uint16_t* __restrict__ w,
                                                     float* __restrict__ out, int64_t N,
                                                     int64_t H, int64_t V, int64_t per) {
    __shared__ typename C::Smem sm;
    int64_t bx0, vy0;
    if (!logits_tile<C>(N, V, per, bx0, vy0)) return;  // the whole workgroup leaves
    const int wave = threadIdx.x >> 6, wx = wave / C::WY, wy = wave % C::WY;
    pj_run<C, 0, WA>(
        h, N, w, V, H, 0, 1, sm,
        [&](int64_t, int64_t& x0, int64_t& y0) {
            x0 = bx0;
            y0 = vy0;
        },
        [&](int64_t, int64_t x0, int64_t y0, f32x16 (&acc)[C::MI][C::NI]) {
#pragma unroll
            for (int mi = 0; mi < C::MI; ++mi)
#pragma unroll
                for (int ni = 0; ni < C::NI; ++ni)
                    store_block(acc[mi][ni], out, N, V, x0 + wx * 32 * C::MI + mi * 32,
                                y0 + wy * 32 * C::NI + ni * 32);
        });
}

template <class C>
__global__ __launch_bounds__(C::NT) void proj_logits_pp(const uint16_t* __restrict__ h,
                                                        const uint16_t* __restrict__ w,
                                                        float* __restrict__ out, int64_t N,
                                                        int64_t H, int64_t V, int64_t per) {
    __shared__ PpSmem<C> sm;
    int64_t bx0, vy0;
    if (!logits_tile<C>(N, V, per, bx0, vy0)) return;  // the whole workgroup leaves
    const int wave = pj_wave(), wx = wave / C::WY, wy = wave % C::WY;
    pp_run<C, 0>(
        h, N, w, V, H, 0, 1, sm,
        [&](int64_t, int64_t& x0, int64_t& y0) {
            x0 = bx0;
            y0 = vy0;
        },
        [&](int64_t, int64_t x0, int64_t y0, f32x16 (&acc)[C::MI][C::NI]) {
#pragma unroll
            for (int mi = 0; mi < C::MI; ++mi)
#pragma unroll
                for (int ni = 0; ni < C::NI; ++ni)
                    store_block(acc[mi][ni], out, N, V, x0 + pp_row(wx, mi), y0 + pp_col(wy, ni));
        });
}

// ------------------------------------------------------------ fused top-k
constexpr int64_t PJ_CB = 4, PJ_SB = 8;  // block of chunks x batch strips per XCD

// A copy of an accumulator register made where it is used.  Left to itself
// the compiler moves every accumulator of the tile into vector registers at
// once when the products end (they are read by vector instructions from
// then on), which overflows the register file; reading each one through
// this keeps the accumulators where the products left them.
__device__ __forceinline__ float acc_reread(float a) {
    float r;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(r) : "a"(a));
    return r;
}

// m = 2 m + (x >= t): one entry's bit of a candidate mask, by a compare and an
// add with its result as the carry (a compare on its own would give a
// wave-wide scalar mask per entry, to be moved into the lanes by two more
// instructions).  The first of 32 entries ends in the highest bit.
__device__ __forceinline__ void push_bit(uint32_t& m, float x, float t) {
    asm("v_cmp_ge_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc"
        : "+v"(m)
        : "v"(x), "v"(t)
        : "vcc");
}

// The least value above x (x finite or -infinity).
__device__ __forceinline__ float next_up(float x) {
    const uint32_t u = __float_as_uint(x);
    return __uint_as_float(x == 0.0f ? 1u : (int32_t)u >= 0 ? u + 1 : u - 1);
}

// The K largest values seen, in registers: KC descending values, of which the
// first KC - K are +infinity, so that the last one is the K-th largest
// (-infinity while there are fewer).  Inserting a value below it changes
// nothing.
template <int KC>
struct LaneVals {
    float v[KC];
    __device__ __forceinline__ void init(int K) {
#pragma unroll
        for (int i = 0; i < KC; ++i) v[i] = i < KC - K ? __builtin_inff() : -__builtin_inff();
    }
    __device__ __forceinline__ float kth() const { return v[KC - 1]; }
    __device__ __forceinline__ void insert(float x) {
#pragma unroll
        for (int i = KC - 1; i > 0; --i) v[i] = __builtin_amdgcn_fmed3f(v[i - 1], v[i], x);
        v[0] = __builtin_fmaxf(v[0], x);
    }
};

// The same with the values' indices: a lane's top-K list (Alg. 4's buffer).
// Offered in increasing index order, so an equal value goes after those there
// already.  Per place one compare, one median and two selects, where 64-bit
// keys took two wide compares and eight selects: the loop over a tile's
// candidates, most of the epilogue, went from 2.7-8.6 us a row and tile to
// 1.6-2.6 (stamps at 4000 x 1024 x 32000, K = 5), the epilogue of a tile from
// 8.5-21.7 us to 6.6-10.6.
template <int KC>
struct LaneList {
    LaneVals<KC> l;
    uint32_t ix[KC];
    __device__ __forceinline__ void init(int K) {
        l.init(K);
#pragma unroll
        for (int i = 0; i < KC; ++i) ix[i] = ~0u;
    }
    __device__ __forceinline__ void insert(float x, uint32_t id) {
#pragma unroll
        for (int i = KC - 1; i > 0; --i) {
            const uint32_t moved = x > l.v[i - 1] ? ix[i - 1] : id;
            ix[i] = x > l.v[i] ? moved : ix[i];
        }
        ix[0] = x > l.v[0] ? id : ix[0];
        l.insert(x);
    }
    // key of place i (0 = none)
    __device__ __forceinline__ uint64_t key(int i) const {
        return ix[i] == ~0u ? 0ull : make_key(l.v[i], ix[i]);
    }
};

// One chunk of vocabulary tiles [c * tiles, min((c + 1) * tiles, nt)) for one
// batch strip of TY rows.  Lane l of wavefront (wx, wy) holds, for batch rows
// 32 (NI wy + ni) + l % 32 (ni < NI) of the strip, the entries
// vbase + 32 mi + 8 (i / 4) + i % 4 (vbase = tile start + 32 MI wx + 4 (l / 32),
// mi < MI) in result register i of block (mi, ni); on the two-group core the
// blocks start at pp_row and pp_col instead.  The partial of a (row, chunk) pair
// written by this lane is p = 2 (WX c + wx) + l / 32: 2 WX S per row, each a
// pair and K keys (0 = none).
// PP: the two-group core (256 x 256), whose stages stay in use during the
// epilogue, so that the epilogue's columns get the LDS that the stages leave.
// WA: cache policy of the vocabulary's loads.
template <class C, int KC, bool PP, int WA>
__global__ __launch_bounds__(C::NT) void proj_topk_part(
    const uint16_t* __restrict__ h, const uint16_t* __restrict__ w, uint64_t* __restrict__ pkeys,
    MD* __restrict__ pmd, int64_t N, int64_t H, int64_t V, int K, int64_t S, int64_t tiles,
    int64_t per) {
    constexpr int NI = C::NI;
    constexpr int E = C::MI * 16;  // entries per row per lane and tile
    // entries per pass of the LDS column: the largest power of two that fits a stage
    constexpr int EC = PP                                                        ? 16
                       : sizeof(typename C::Stage) >= C::NT * 64 * sizeof(float) ? 64
                       : sizeof(typename C::Stage) >= C::NT * 32 * sizeof(float) ? 32
                                                                                 : 16;
    static_assert(PP || sizeof(typename C::Stage) >= C::NT * EC * sizeof(float), "scratch fits");
    struct PpAll {
        PpSmem<C> st;
        float scr[EC * C::NT];
    };
    __shared__ std::conditional_t<PP, PpAll, typename C::Smem> sm;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wx = wave / C::WY, wy = wave % C::WY;
    // Logical ids in blocks of PJ_CB chunks x up to PJ_SB batch strips, so
    // that the workgroups of an XCD (a contiguous range of ids) share few
    // operand tiles in its L2: a block of 4 x 8 reads 12 distinct tiles per
    // step where 2 chunks x 16 strips would read 18.
    const int64_t nb = (N + C::TY - 1) / C::TY, nt = (V + C::TX - 1) / C::TX;
    const int64_t sb = nb < PJ_SB ? nb : PJ_SB, nsb = (nb + sb - 1) / sb;
    const int64_t lid = xcd_logical(blockIdx.x, per);
    const int64_t blk = lid / (PJ_CB * sb), in = lid % (PJ_CB * sb);
    const int64_t c = (blk / nsb) * PJ_CB + in / sb;
    const int64_t strip = (blk % nsb) * sb + in % sb;
    if (c >= S || strip >= nb) return;  // the whole workgroup leaves
    const int64_t y0s = strip * C::TY;  // batch strip
    const int64_t t0 = c * tiles;
    const int64_t t1 = t0 + tiles < nt ? t0 + tiles : nt;

    float sr[NI], dacc[NI];
    float tval[NI];  // an entry below it cannot be among the row's K largest
    LaneList<KC> list[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
        sr[ni] = kEmptyS;
        dacc[ni] = 0.0f;
        // Lanes of rows past the batch take no candidates: their logits are all
        // zero, and so many ties cost more than a real row's candidates
        // (100 x 1024 x 32000 top-5: 55.6 us with them, 33.5 without;
        // 300 x 512 x 20000: 57.2 and 39.2).
        const int64_t row = y0s + (PP ? pp_col(wy, ni) : wy * 32 * NI + ni * 32) + (lane & 31);
        tval[ni] = row < N ? -__builtin_inff() : __builtin_inff();
        list[ni].init(K);
    }
    float* scr;  // this thread's column
    if constexpr (PP) scr = sm.scr + threadIdx.x;
    else scr = reinterpret_cast<float*>(&sm.st[1]) + threadIdx.x;

    auto coords = [&](int64_t t, int64_t& x0, int64_t& y0) {
        x0 = t * C::TX;
        y0 = y0s;
    };
    auto epi = [&](int64_t, int64_t x0, int64_t, f32x16 (&acc)[C::MI][C::NI]) {
        // groups of GS consecutive entries: 8, or fewer so that there
        // are at least KC groups (the bootstrap below needs K of them)
        constexpr int GS = E / KC < 8 ? E / KC : 8;
        constexpr int NG = E / GS;
        static_assert(GS % 2 == 0 && NG >= KC, "groups hold whole entry pairs");
        const uint32_t vbase = (uint32_t)x0 + (uint32_t)((PP ? pp_row(wx, 0) : wx * 32 * C::MI) +
                                                         4 * (lane >> 5));
        // offset from vbase of entry j (block j / 16, register j % 16)
        auto voff = [](int j) {
            return (PP ? pp_row(0, j >> 4) : (j >> 4) * 32) + 8 * ((j & 15) >> 2) + (j & 3);
        };
        // entries [q EC, q EC + EC) of row ni into this thread's LDS column
        auto stage = [&](int ni, int q) {
#pragma unroll
            for (int j = 0; j < EC; ++j)
                scr[j * C::NT] = acc_reread(acc[(q * EC + j) >> 4][ni][j & 15]);
        };
        // The vocabulary's last tile may run past V (once per chunk at
        // most): entries at offsets >= lim do not exist.
        const bool ragged = x0 + C::TX > V;
        const int lim = ragged ? (int)(V - (int64_t)vbase) : 1 << 30;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            // Alg. 3: move the reference to a maximum that passes it by more
            // than kLazy.
            auto raise = [&](float tm) {
                if (tm > sr[ni] + kLazy) {
                    dacc[ni] *= exp2_hw(sr[ni] - tm);
                    sr[ni] = tm;
                }
            };
            // 1. The chunk's first tile (and the ragged one): the maxima of
            //    groups of GS entries.  They set the reference, and a first
            //    threshold: they are entries of distinct groups, so the K-th
            //    largest of the maxima of this lane and of the other lane
            //    holding the row is a value that at least K entries reach.
            if (ragged || __builtin_amdgcn_ballot_w64(sr[ni] == kEmptyS) != 0) {
                float bm[NG];
#pragma unroll
                for (int g = 0; g < NG; ++g) bm[g] = -__builtin_inff();
#pragma unroll
                for (int j = 0; j < E; ++j) {
                    const float x = acc_reread(acc[j >> 4][ni][j & 15]);
                    bm[j / GS] =
                        __builtin_fmaxf(bm[j / GS], voff(j) < lim ? x : -__builtin_inff());
                }
                LaneVals<KC> best;
                best.init(K);
                float lm = bm[0];
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    best.insert(bm[g]);
                    best.insert(__shfl_xor(bm[g], 32));
                    lm = __builtin_fmaxf(lm, bm[g]);
                }
                raise(lm * kLog2e);
                tval[ni] = __builtin_fmaxf(tval[ni], best.kth());
            }
            // 2. One pass over the row's entries: their maximum, the terms
            //    against the reference, and the entries that reach the
            //    threshold, which only rises, so that every entry that can
            //    still enter the list is among them.
            float dsum[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            uint32_t cm[E / 32];
#pragma unroll
            for (int u = 0; u < E / 32; ++u) cm[u] = 0u;
            bool recompute = ragged;
            if (!ragged) {
                const float th = tval[ni];
                float lm = -__builtin_inff();
#pragma unroll
                for (int j = 0; j < E; j += 2) {
                    const float a0 = acc_reread(acc[j >> 4][ni][j & 15]);
                    const float a1 = acc_reread(acc[(j + 1) >> 4][ni][(j + 1) & 15]);
                    lm = max3_raw(lm, a0, a1);
                    dsum[j & 3] += exp2_hw(__builtin_fmaf(a0, kLog2e, -sr[ni]));
                    dsum[(j + 1) & 3] += exp2_hw(__builtin_fmaf(a1, kLog2e, -sr[ni]));
                    push_bit(cm[j >> 5], a0, th);
                    push_bit(cm[j >> 5], a1, th);
                }
                // a move of the reference: the terms are summed again below
                if (__builtin_amdgcn_ballot_w64(lm * kLog2e > sr[ni] + kLazy) != 0) {
                    raise(lm * kLog2e);
                    recompute = true;
                }
            }
            float ds = recompute ? 0.0f : (dsum[0] + dsum[1]) + (dsum[2] + dsum[3]);
            // 3. Per part of EC entries, when anything is left to do, the
            //    part goes to this thread's LDS column (the one copy of the
            //    part's registers in the code), and rolled loops finish the
            //    work: the terms again after a move of the reference, with
            //    the bound on the ragged tile, whose candidates are found
            //    here too, then Alg. 4's insertion of each candidate.
#pragma unroll
            for (int q = 0; q < E / EC; ++q) {
                // candidates of this part, the first in the highest bit
                uint64_t m;
                if constexpr (EC == 64)
                    m = (uint64_t)cm[2 * q] << 32 | cm[2 * q + 1];
                else if constexpr (EC == 32)
                    m = (uint64_t)cm[q] << 32;
                else
                    m = (uint64_t)(q % 2 == 0 ? cm[q / 2] >> 16 : cm[q / 2] & 0xFFFFu) << 48;
                if (!recompute && __builtin_amdgcn_ballot_w64(m != 0) == 0) continue;
                stage(ni, q);
                if (recompute) {
                    const float tv = tval[ni], s = sr[ni];
                    uint64_t nm = 0;
                    float pd = 0.0f;
#pragma unroll 4
                    for (int j = 0; j < EC; ++j) {
                        const float xv = scr[j * C::NT];
                        const bool valid = voff(q * EC + j) < lim;
                        const float e = exp2_hw(__builtin_fmaf(xv, kLog2e, -s));
                        pd += valid ? e : 0.0f;
                        nm |= (uint64_t)(valid && xv >= tv) << (63 - j);
                    }
                    ds += pd;
                    if (ragged) m = nm;
                }
                while (m != 0) {
                    const int j = __builtin_clzll(m);
                    m &= ~(0x8000000000000000ull >> j);
                    list[ni].insert(scr[j * C::NT], vbase + (uint32_t)voff(q * EC + j));
                }
            }
            dacc[ni] += ds;
            // An entry equal to this lane's K-th value comes after the list's
            // (a higher index), so only larger ones count from here on; the
            // other lane holding the row saw other entries, so its K-th value
            // only bounds the row's from below.
            const float own = list[ni].l.kth();
            tval[ni] = __builtin_fmaxf(
                tval[ni], __builtin_fmaxf(next_up(own), __shfl_xor(own, 32)));
        }
    };
    if constexpr (PP) pp_run<C, WA>(w, V, h, N, H, t0, t1, sm.st, coords, epi);
    else pj_run<C, WA, 0>(w, V, h, N, H, t0, t1, sm, coords, epi);

    constexpr int P = 2 * C::WX;  // partials per (row, chunk)
    const int64_t Sp = S * P;
    const int64_t p = c * P + wx * 2 + (lane >> 5);
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
        const int64_t row = y0s + (PP ? pp_col(wy, ni) : wy * 32 * NI + ni * 32) + (lane & 31);
        if (row < N) {
            uint64_t* dst = pkeys + (row * Sp + p) * K - (KC - K);
#pragma unroll
            for (int i = 0; i < KC; ++i)
                if (i >= KC - K) dst[i] = list[ni].key(i);
            pmd[row * Sp + p] = MD{sr[ni], dacc[ni]};
        }
    }
}

// ---------------------------------------------------------------- launchers
// Whether w is read once, by one strip of `rows` batch rows, and the last-level
// cache (256 MB) could not keep enough of it for the next call (us, PJ_ONCE
// against the default: projection + top-5 64 x 4096 x 128256 167 / 186, 100 x
// ... 213 / 229, 200 x ... 257 / 270, 64 x 4096 x 50000 109 / 116; logits 64 x
// 4096 x 128256 168 / 177; but on the same w again 64 x 2048 x 68000, 279 MB,
// 84 / 68, and with more strips, which share w in L2, 768 x 4096 x 128256 750 /
// 730).  The logits' 256 x 256 tiles gain nothing (256 x 4096 x 128256 345 / 345).
// Only where a tile row's 128 bytes of a step are a whole cache line: a line
// that two steps share would be fetched twice (64 x 4080 x 60000 logits 148 /
// 117, top-5 156 / 125).
static bool w_once(const void* w, int64_t N, int64_t H, int64_t V, int64_t rows) {
    return N <= rows && V * H * 2 >= ((int64_t)384 << 20) && H % PJ_BK == 0 &&
           reinterpret_cast<uintptr_t>(w) % (PJ_BK * 2) == 0;
}

template <class C, bool PP, int WA>
static hipError_t launch_logits_t(const void* h, const void* w, float* out, int64_t N, int64_t H,
                                  int64_t V, hipStream_t st) {
    const int64_t total = ((N + C::TX - 1) / C::TX) * ((V + C::TY - 1) / C::TY);
    const int64_t per = (total + 7) / 8;
    if constexpr (PP)
        hipLaunchKernelGGL((proj_logits_pp<C>), dim3((unsigned)(8 * per)), dim3(C::NT), 0, st,
                           (const uint16_t*)h, (const uint16_t*)w, out, N, H, V, per);
    else
        hipLaunchKernelGGL((proj_logits<C, WA>), dim3((unsigned)(8 * per)), dim3(C::NT), 0, st,
                           (const uint16_t*)h, (const uint16_t*)w, out, N, H, V, per);
    return hipGetLastError();
}

hipError_t launch_proj_logits(const void* h, const void* w, float* out, int64_t N, int64_t H,
                              int64_t V, int cus, hipStream_t st) {
    const int64_t big = ((N + PjBig::TX - 1) / PjBig::TX) * ((V + PjBig::TY - 1) / PjBig::TY);
    if (big >= 2 * (int64_t)cus) return launch_logits_t<PjBig, true, 0>(h, w, out, N, H, V, st);
    if (w_once(w, N, H, V, PjSmall::TX))
        return launch_logits_t<PjSmall, false, PJ_ONCE>(h, w, out, N, H, V, st);
    return launch_logits_t<PjSmall, false, 0>(h, w, out, N, H, V, st);
}

ProjTopkShape proj_topk_shape(int64_t N, int64_t H, int64_t V, int K, int cus) {
    const FusedCfg cfg = fused_cfg(N, H, V, K, cus);
    // vocabulary rows of a tile, batch rows of a strip, and partials per (row,
    // chunk): two for each wavefront along the vocabulary
    int64_t TX = PjFused8::TX, TY = PjFused8::TY;
    int parts = 2 * PjFused8::WX;
    auto of = [&](auto c) { TX = c.TX, TY = c.TY, parts = 2 * c.WX; };
    switch (cfg) {
        case FUSED_16W: of(PjFused16W{}); break;
        case FUSED_16T: of(PjFused16{}); break;
        case FUSED_N: of(PjFusedN{}); break;
        case FUSED_NM: of(PjFusedNM{}); break;
        case FUSED_NS: of(PjFusedNS{}); break;
        default: break;
    }
    // vocabulary chunks: about one workgroup per CU in all (each takes 80 KB
    // of LDS or more); as many as fit for the tiles of 64 batch rows at K <= 8
    // and 64 x 64 (80, 48 and 32 KB of LDS), where the call streams w and the
    // loads in flight pay for the merge of more partials (256 x 64 measured
    // 5-7% faster at K <= 8; at K = 16 the larger merge ate the gain)
    const int64_t nb = (N + TY - 1) / TY, nt = (V + TX - 1) / TX;
    const int64_t per_cu = cfg == FUSED_NS             ? 5
                           : cfg == FUSED_NM           ? 3
                           : cfg == FUSED_N && K <= 8 ? 2
                                                      : 1;
    int64_t s = ((int64_t)cus * per_cu + nb - 1) / nb;
    if (s > nt) s = nt;
    if (s < 1) s = 1;
    const int64_t t = (nt + s - 1) / s;
    return {cfg, (nt + t - 1) / t, t, parts};
}

size_t proj_topk_part_bytes(int64_t N, int64_t S, int parts, int K) {
    return (size_t)N * (size_t)(S * parts) * ((size_t)K * 8 + 8);
}

template <class C, int KC, bool PP, int WA>
static void launch_part(const void* h, const void* w, uint64_t* pkeys, MD* pmd, int64_t N,
                        int64_t H, int64_t V, int K, int64_t S, int64_t tiles, hipStream_t st) {
    const int64_t nb = (N + C::TY - 1) / C::TY;
    const int64_t sb = nb < PJ_SB ? nb : PJ_SB, nsb = (nb + sb - 1) / sb;
    const int64_t ids = (S + PJ_CB - 1) / PJ_CB * nsb * PJ_CB * sb;  // whole blocks
    const int64_t per = (ids + 7) / 8;
    hipLaunchKernelGGL((proj_topk_part<C, KC, PP, WA>), dim3((unsigned)(8 * per)), dim3(C::NT), 0,
                       st, (const uint16_t*)h, (const uint16_t*)w, pkeys, pmd, N, H, V, K, S,
                       tiles, per);
}

hipError_t launch_proj_topk(const void* h, const void* w, float* vals, int32_t* idx,
                            void* part, int64_t N, int64_t H, int64_t V, int K,
                            const ProjTopkShape& p, hipStream_t st) {
    const int64_t S = p.S, tiles = p.tiles, Sp = S * p.parts;  // partials per row
    uint64_t* pkeys = static_cast<uint64_t*>(part);
    MD* pmd = reinterpret_cast<MD*>(pkeys + N * Sp * K);
    auto part_of = [&](auto cfg, auto kc, auto pp, auto wa) {
        launch_part<decltype(cfg), decltype(kc)::value, decltype(pp)::value, decltype(wa)::value>(
            h, w, pkeys, pmd, N, H, V, K, S, tiles, st);
    };
    auto run = [&](auto cfg, auto kc, auto pp) {
        if (w_once(w, N, H, V, decltype(cfg)::TY))
            part_of(cfg, kc, pp, std::integral_constant<int, PJ_ONCE>{});
        else
            part_of(cfg, kc, pp, std::integral_constant<int, 0>{});
    };
    const std::integral_constant<int, 8> k8;
    const std::integral_constant<int, 16> k16;
    switch (p.cfg) {
        case FUSED_8: run(PjFused8{}, k8, std::true_type{}); break;
        case FUSED_16: run(PjFused8{}, k16, std::true_type{}); break;
        case FUSED_16W:  // more than one strip: N > 1024
            part_of(PjFused16W{}, k16, std::false_type{}, std::integral_constant<int, 0>{});
            break;
        case FUSED_16T: run(PjFused16{}, k16, std::false_type{}); break;
        case FUSED_NM: run(PjFusedNM{}, k8, std::false_type{}); break;
        case FUSED_NS:
            if (K <= 8) run(PjFusedNS{}, k8, std::false_type{});
            else run(PjFusedNS{}, k16, std::false_type{});
            break;
        default:
            if (K <= 8) run(PjFusedN{}, k8, std::false_type{});
            else run(PjFusedN{}, k16, std::false_type{});
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_merge_held<TK_ONLINE>(pkeys, pmd, vals, idx, N, Sp, K, st);
}

}  // namespace osm
