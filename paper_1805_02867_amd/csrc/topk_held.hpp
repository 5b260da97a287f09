// Softmax + top-k of rows (or chunks of rows) that fit in registers: every
// element is loaded once, all loads before any use, and the selection runs on
// the registers.
//
// What bounds these shapes is not bandwidth but the chain from the last load
// to the outputs, so the chain is kept short and the code small (8-25 KB a row
// kernel, 35-47 KB a split one, against 60-172 KB for the streaming kernels of
// topk.hpp, whose first pass through the code costs more than the work on a
// short row).  Measured against those kernels, warm, back to back:
//   4000 x 1000 binary32 top-5    9.9 -> 6.5 us   (16 MB; a launch is ~2.5 us)
//   4000 x 1000 binary32 top-50  13.9 -> 9.7
//   4000 x 10000 bfloat16 top-50 41.4 -> 23.7     (80 MB, 3.4 TB/s)
//   4000 x 10000 binary32 top-5  31.2 -> 28.2     (160 MB, 5.7 TB/s)
//   64 x 128256 bfloat16 top-50  24.7 -> 13.4     (16 MB, split)
//   10 x 10^6 binary32 top-5     18.8 -> 16.1     (40 MB, split)
// Phases of the 64 x 128256 top-50 call by wall-clock stamps (512 workgroups,
// medians): loads 1.6 us, maxima and exponentials 1.4, threshold 0.8,
// candidates 1.1, sort 1.5, partial stored 0.4, counted 0.5, merge of the
// row's partials 2.8.
//
//  1. Each lane's maximum (by 16-byte vector), and its online pair.
//  2. A threshold from the lanes' maxima: a binary search, over the bits of
//     the order-preserving image of the values, for a value that at least K
//     groups of elements reach (a group: a lane's elements, or half of them).
//     Each group holds an element that large, so every top-K element is at
//     least as large; and few others are: of 256 groups about 1.1 K elements
//     pass for K = 50.
//  3. The candidates at or above the threshold are appended to a small list of
//     keys in LDS, in rounds that take one vector per lane.  A list of more
//     than 128 keys (a threshold low among few groups) is thinned to the keys
//     that reach a bound of its own.  Where the search for the threshold ends
//     at a value that many groups share (rows of ties), the elements of that
//     value are taken in index order instead, as many as are needed, and only
//     larger ones are looked for.
//  4. One bitonic sort of the list (of 16 keys when no more are left) gives
//     the outputs in key order.
//
// The order of keys, the normalizer pair and the outputs are those of
// topk.hpp, so the results are the same indices, bit for bit.
#pragma once

#include "topk.hpp"

namespace osm {

constexpr int TH_LIST = 192;  // slots of a wavefront's key list: up to 128, and 64 appended
constexpr int TH_CUT = 128;   // a longer list is thinned
constexpr int TH_TIE_I = 4;   // vectors a lane that are searched for ties

// Order-preserving image of a value: a larger word means a larger value.
// -0.0 and +0.0 have the same image.
__device__ __forceinline__ uint32_t order_word(float x) { return (uint32_t)(make_key(x, 0u) >> 32); }
constexpr uint32_t kOrderNegInf = 0x007FFFFFu;  // image of -infinity

// A condition that few rows meet: its code goes behind the kernel's (a short
// row's time is mostly the first pass through the code it runs).
__device__ __forceinline__ bool rare(bool c) { return __builtin_expect(c, 0); }

struct KthBound {
    uint32_t lo;  // the bound
    // Many more words than K reach lo, for [lo, up) holds one value only, which
    // the K-th largest word has: a row of ties, as it seems.
    bool tied;
    uint32_t up;
};
constexpr int TH_TIED = 16;  // how many more, past the K + K / 4 + 1 of an ordinary bound

// A word that at least K of the wavefront's 64 * G words reach (K <= 64 G;
// kOrderNegInf if fewer than K are above it), given `hi`, the largest of them.
// The words' distance below hi is bracketed in powers of four from one binade
// (2^23) on, then halved until no more than K + K / 4 + 1 words reach the
// bound, or down to GRAN, the least distance of two values (2^16 for bfloat16
// values).  Logits lie within a binade or two of their maximum, so that takes
// four to six counts, where a search from the highest bit down takes about
// twelve.  (Every lane of the wavefront takes part; the result is the same in
// all.)
template <int G, uint32_t GRAN>
__device__ __forceinline__ KthBound kth_bound(const uint32_t (&m)[G], uint32_t hi, int K) {
    const int most = K + (K >> 2) + 1;
    auto count = [&](uint32_t c) {
        int n = 0;
#pragma unroll
        for (int g = 0; g < G; ++g) n += __builtin_popcountll(__builtin_amdgcn_ballot_w64(m[g] >= c));
        return n;
    };
    const KthBound none = {kOrderNegInf, true, kOrderNegInf + 1};
    if (hi <= kOrderNegInf) return none;
    int n = count(hi);
    if (n >= K) return {hi, n > most + TH_TIED, hi + 1};
    // n words reach lo, at least K; fewer than K reach up
    uint32_t lo, up = hi, step = 1u << 23;
#pragma unroll 1
    for (;;) {
        const bool last = step >= hi - kOrderNegInf;
        lo = last ? kOrderNegInf + 1 : hi - step;
        n = count(lo);
        if (n >= K) break;
        if (last) return none;
        up = lo;
        step = step < (1u << 30) ? step << 2 : 0xFFFFFFFFu;
    }
#pragma unroll 1
    while (n > most && up - lo > GRAN) {
        const uint32_t c = lo + ((up - lo) >> 1);
        const int k = count(c);
        if (k >= K) {
            lo = c;
            n = k;
        } else {
            up = c;
        }
    }
    return {lo, n > most + TH_TIED, up};
}

// The wavefront's largest value, as a scalar.
__device__ __forceinline__ float wave_max_f(float v) {
    return __uint_as_float(
        (uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(group_max<64>(v))));
}

// The largest of the wavefront's words, as a scalar.
template <int G>
__device__ __forceinline__ uint32_t wave_hi(const uint32_t (&m)[G]) {
    uint32_t h = m[0];
#pragma unroll
    for (int g = 1; g < G; ++g) h = m[g] > h ? m[g] : h;
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_max_u32(h));
}

// Sort of the wavefront's keys (lane 0 ends with the largest) when only the
// first n lanes hold any: six stages for n <= 8, ten for n <= 16, else 21.
__device__ __forceinline__ uint64_t sort_first(uint64_t v, int n) {
    v = bitonic_stage_run<2, 1>(v);
    v = bitonic_stage_run<4, 2>(v);
    v = bitonic_stage_run<8, 4>(v);
    if (n > 8) v = bitonic_stage_run<16, 8>(v);
    if (n > 16) {
        v = bitonic_stage_run<32, 16>(v);
        v = bitonic_stage_run<64, 32>(v);
    }
    return v;
}

// The 64 largest keys of two sorted sets (one key a lane, lane 0 the largest),
// sorted the same way.
__device__ __forceinline__ uint64_t merge_sorted(uint64_t a, uint64_t b) {
    b = reverse_lanes(b);
    return bitonic_merge_desc(a > b ? a : b);
}

// Of up to 192 keys (three a lane, 0: none), those that can be among the K
// largest, written to `out`: all keys whose value reaches a bound that at least
// K of them reach, K + K / 4 + 1 or fewer but for ties.  Returns how many; lo:
// the bound.  (A few counts, where sorting 192 keys takes three networks of 21
// dependent exchanges and three merges.  Rows whose largest elements lie side
// by side, so that a lane's group holds many, need it: logits that fall with
// the index, top-50, 4000 x 32000 binary32 108 -> 100 us, 4000 x 1000 13.1 ->
// 11.5, 2000 x 60000 bfloat16 69 -> 62; in any order 81.5, 9.0 and 47.8.)
__device__ __forceinline__ int thin_keys(const uint64_t (&k)[3], int K, uint64_t* out,
                                         uint32_t* lo) {
    uint32_t g[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) g[j] = (uint32_t)(k[j] >> 32);
    const uint32_t b = kth_bound<3, 1>(g, wave_hi(g), K).lo;
    int n = 0;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const bool p = g[j] >= b;
        const uint64_t mask = __builtin_amdgcn_ballot_w64(p);
        const uint32_t below = __builtin_amdgcn_mbcnt_hi(
            (uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
        if (p) out[n + below] = k[j];
        n += __builtin_popcountll(mask);
    }
    *lo = b;
    return n;
}

// A wavefront's list of candidate keys.
struct HeldList {
    uint64_t* keys;  // TH_LIST slots of LDS
    int K;
    int n;           // keys in the list (wave-uniform), at most TH_CUT between appends
    uint64_t tau;    // keys at or below it cannot be among the K largest

    // Append the lanes' keys where p holds.  (Every lane takes part.)
    __device__ __forceinline__ void offer(bool p, uint64_t key) {
        p = p && key > tau;
        const uint64_t mask = __builtin_amdgcn_ballot_w64(p);
        if (mask == 0) return;
        const uint32_t below = __builtin_amdgcn_mbcnt_hi(
            (uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
        if (p) keys[n + below] = key;
        n += __builtin_popcountll(mask);
    }
    // More than TH_CUT keys: those that can be among the K largest stay, or the
    // K largest themselves where ties leave more of them.  (Every lane takes part.)
    __device__ __forceinline__ void cut() {
        const int lane = __lane_id();
        uint64_t k[3];
        wave_sync();
#pragma unroll
        for (int j = 0; j < 3; ++j) k[j] = lane + 64 * j < n ? keys[lane + 64 * j] : 0ull;
        uint32_t lo;
        n = thin_keys(k, K, keys, &lo);
        const uint64_t t = ((uint64_t)lo << 32) - 1;
        tau = t > tau ? t : tau;
        if (n <= TH_CUT) return;
        uint64_t cur = 0;
        wave_sync();
#pragma unroll 1
        for (int b = 0; b < n; b += 64)
            cur = merge_sorted(cur, sort_desc(b + lane < n ? keys[b + lane] : 0ull));
        wave_sync();
        if (lane < K) keys[lane] = cur;
        n = K;
        tau = read_lane_key(cur, K - 1);
    }
};

// Final selection over the lists of W wavefronts, cnt[w] keys each: lane k of
// the calling wavefront returns the k-th largest key (0: none).  Batches of 64
// keys of the lists' concatenation; one batch when they hold no more.
template <int W>
__device__ __forceinline__ uint64_t held_finish(uint64_t (*lists)[TH_LIST], const int* cnt,
                                                int K) {
    const int lane = __lane_id();
    int total = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) total += cnt[w];
    total = __builtin_amdgcn_readfirstlane(total);
    // key i of the concatenation
    auto at = [&](int i) {
        int w = 0, j = i;
#pragma unroll
        for (int u = 0; u < W - 1; ++u) {
            const int c = cnt[u];
            const bool past = w == u && j >= c;
            j = past ? j - c : j;
            w = past ? u + 1 : w;
        }
        return i < total ? lists[w][j] : 0ull;
    };
    // thinned out ahead of the sort, where that saves one (a bound leaves up to
    // K + K / 4 + 1 keys, more than one sort's for K > 50)
    if (W > 1 && rare(total > (K <= 50 ? 64 : 128) && total <= TH_LIST)) {
        const uint64_t k[3] = {at(lane), at(lane + 64), at(lane + 128)};
        uint32_t lo;
        const int n = thin_keys(k, K, lists[0], &lo);
        wave_sync();
        uint64_t cur = sort_desc(lane < n ? lists[0][lane] : 0ull);
#pragma unroll 1
        for (int b = 64; b < n; b += 64)
            cur = merge_sorted(cur, sort_desc(b + lane < n ? lists[0][b + lane] : 0ull));
        return lane < K ? cur : 0ull;
    }
    uint64_t cur = 0;
#pragma unroll 1
    for (int b = 0; b < total; b += 64) {
        const uint64_t q = sort_first(at(b + lane), total - b);
        if (b == 0) cur = q;
        else cur = merge_sorted(cur, q);
    }
    return lane < K ? cur : 0ull;
}

// Writes one row's outputs from lane k's k-th key.
template <int VAR>
__device__ __forceinline__ void held_store(uint64_t key, MD md, float* __restrict__ vals,
                                           int32_t* __restrict__ idx, int64_t row, int K) {
    const int lane = __lane_id();
    if (lane < K) {
        if constexpr (VAR == TK_VALUES) {
            vals[row * K + lane] = key_value(key);
        } else {
            vals[row * K + lane] = out_elem(key_value(key), md.s, 1.0f / md.d);
        }
        idx[row * K + lane] = key_index(key);
    }
}

// LDS of a team of W wavefronts (W = 1: of the workgroup's four teams).
template <int W>
struct HeldSmem {
    static constexpr int NW = W == 1 ? TK_BLOCK / 64 : W;
    uint64_t list[NW][TH_LIST];
    uint32_t gmax[W == 1 ? 1 : 256];  // images of 256 groups' maxima
    MD wmd[NW];
    int cnt[NW];
    int tie[TH_TIE_I][NW];  // held_ties: ties of the wavefronts' first vectors
};

// A word that at least K of a workgroup's elements reach, from the maxima `m`
// of its lanes' elements: up to 256 groups (of one lane, or W / 4) go through
// LDS, and every wavefront runs the same search.  (One barrier.)
template <int W, uint32_t GRAN, class Smem>
__device__ __forceinline__ KthBound team_bound(Smem& sm, uint32_t m, int K) {
    constexpr int GL = W > 4 ? W / 4 : 1, G = W > 4 ? 4 : W;
    const int lane = threadIdx.x & 63;
    if constexpr (GL >= 2) {
        uint32_t x, y;
        bfly_operands<0>(m, x, y);
        m = x > y ? x : y;
    }
    if constexpr (GL >= 4) {
        uint32_t x, y;
        bfly_operands<1>(m, x, y);
        m = x > y ? x : y;
    }
    if (lane % GL == 0) sm.gmax[threadIdx.x / GL] = m;
    __syncthreads();
    uint32_t g[G];
#pragma unroll
    for (int i = 0; i < G; ++i) g[i] = sm.gmax[lane + 64 * i];
    return kth_bound<G, GRAN>(g, wave_hi(g), K);
}

constexpr int TK_MERGE_B = 8;  // keys per lane in one batch of a wavefront's merge

// Merge of a row's n partial keys and P partial pairs by a team of W
// wavefronts, R keys a lane at a time.  COH: the partials were written by other
// workgroups of the same kernel; slot: the wavefront's list.  The team's first
// wavefront returns true with lane k's k-th key; the LDS is free on entry, and with W > 1 the workgroup's
// wavefronts enter together.
template <int VAR, int W, int R, uint32_t GRAN, bool COH, class Smem>
__device__ __forceinline__ bool held_merge(Smem& sm, int slot, const uint64_t* pk, const MD* pm,
                                           int64_t n, int64_t P, int K, uint64_t* key, MD* md) {
    constexpr int TR = 64 * W;
    const int lane = threadIdx.x & 63, tr = W == 1 ? lane : (int)threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto load = [](const uint64_t* p) {
        if constexpr (COH) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else return *p;
    };
    auto load_md = [&](int64_t j) {
        return __builtin_bit_cast(MD, load(reinterpret_cast<const uint64_t*>(pm + j)));
    };
    MD a = md_empty();
    if constexpr (VAR != TK_VALUES) {  // requested ahead of the keys
        if (tr < P) a = load_md(tr);
    }
    HeldList hl{sm.list[slot], K, 0, 0ull};
    uint64_t top = 0;  // W = 1, K = 1: the largest key, without threshold or list
    uint32_t t = 0;    // a word that at least K of the first batch's keys reach
#pragma unroll 1
    for (int64_t b = 0; b < n; b += TR * R) {
        uint64_t k[R];
        const int64_t left = n - b;
#pragma unroll
        for (int i = 0; i < R; ++i) k[i] = tr + i * TR < left ? load(pk + b + tr + i * TR) : 0ull;
        if (W == 1 && K == 1) {
#pragma unroll
            for (int i = 0; i < R; ++i) top = k[i] > top ? k[i] : top;
            continue;
        }
        if (b > 0) {
            // the first batch's bound holds for the later ones
        } else if constexpr (W == 1) {
            static_assert(R % 4 == 0, "four groups a lane");
            uint32_t g[4] = {0, 0, 0, 0};
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const uint32_t h = (uint32_t)(k[i] >> 32);
                g[i % 4] = h > g[i % 4] ? h : g[i % 4];
            }
            t = kth_bound<4, GRAN>(g, wave_hi(g), K).lo;
        } else {
            uint32_t m = 0;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const uint32_t h = (uint32_t)(k[i] >> 32);
                m = h > m ? h : m;
            }
            t = team_bound<W, GRAN>(sm, m, K).lo;
        }
        uint32_t hm = 0;
#pragma unroll
        for (int i = 0; i < R; ++i)
            hm |= (uint32_t)(k[i] > hl.tau && (uint32_t)(k[i] >> 32) >= t) << i;
        while (__builtin_amdgcn_ballot_w64(hm != 0) != 0) {
            const int s = hm != 0 ? __builtin_ctz(hm) : 0;
            uint64_t q = k[0];
#pragma unroll
            for (int i = 1; i < R; ++i) q = s == i ? k[i] : q;
            hl.offer(hm != 0, q);
            if (rare(hl.n > TH_CUT)) hl.cut();
            hm &= hm - 1;
        }
    }
    if constexpr (VAR != TK_VALUES) {
        // pairs tr, tr + TR, ... in order, then the butterfly
        for (int64_t j = tr + TR; j < P; j += TR) a = md_merge(a, load_md(j));
        a = group_merge<64>(a);
    }
    if constexpr (W == 1) {
        wave_sync();
        if (K == 1) *key = wave_max_key(top);
        else *key = held_finish<1>(&sm.list[slot], &hl.n, K);
        *md = a;
        return true;
    } else {
        if (lane == 0) {
            sm.cnt[wv] = hl.n;
            sm.wmd[wv] = a;
        }
        __syncthreads();
        if (wv != 0) return false;
        a = sm.wmd[0];
#pragma unroll
        for (int w = 1; w < W; ++w) a = md_merge(a, sm.wmd[w]);
        *md = a;
        *key = held_finish<W>(sm.list, sm.cnt, K);
        return true;
    }
}

// The part of a row that a team works on: elements [0, L) from xr, as scalar
// head, 16-byte vectors and scalar tail.
template <typename T>
struct HeldSpan {
    const T* xr;
    const u32x4* vb;
    int head, nvec;
    int ne;         // head and tail elements together, fewer than 2 E
    uint32_t base;  // index of the first element within the row

    __device__ __forceinline__ HeldSpan(const T* x, int64_t row, int64_t start, int64_t V, int L)
        : xr(x + row * V + start), base((uint32_t)start) {
        constexpr int E = Vec<T>::N;
        head = (int)(((16 - (((uintptr_t)xr) & 15)) & 15) / sizeof(T));
        if (head > L) head = L;
        nvec = (L - head) / E;
        ne = L - nvec * E;
        vb = reinterpret_cast<const u32x4*>(xr + head);
    }
    // place of the tr-th head or tail element
    __device__ __forceinline__ int extra(int tr) const {
        return tr < head ? tr : nvec * Vec<T>::N + tr;
    }
    // index within the row of vector v's first element
    __device__ __forceinline__ uint32_t index(int v) const {
        return base + (uint32_t)(head + v * Vec<T>::N);
    }
};

// The largest element of a vector; -inf at least.
template <typename T, int VAR>
__device__ __forceinline__ float held_vmax(u32x4 q) {
    constexpr int E = Vec<T>::N;
    float xv[E];
    widen<T>(q, xv);
    float m = -__builtin_inff();
    if constexpr (VAR == TK_VALUES) {  // a NaN never counts
#pragma unroll
        for (int e = 0; e < E; ++e) m = __builtin_fmaxf(m, xv[e]);
        return m;
    } else {
        return vec_max_into(xv, m);
    }
}

// Offers the candidates of a block of R vectors a lane (lane's vectors v0,
// v0 + TR, ...; bit i of hm: vector i holds an element of at least `th`), and
// the lane's head or tail element (bit R).  Per round each lane takes one
// vector, then its candidates one at a time.
template <typename T, int R, int TR>
__device__ __forceinline__ void held_offer(HeldList& hl, const HeldSpan<T>& sp,
                                           const u32x4 (&buf)[R], int v0, uint32_t hm, float th,
                                           float ex) {
    constexpr int E = Vec<T>::N;
#pragma unroll 1
    while (__builtin_amdgcn_ballot_w64(hm != 0) != 0) {
        const int s = __builtin_ctz(hm | 0x80000000u);
        uint32_t q0 = buf[0].x, q1 = buf[0].y, q2 = buf[0].z, q3 = buf[0].w;
#pragma unroll
        for (int i = 1; i < R; ++i) {  // values, so that the buffer stays in registers
            const u32x4 c = buf[i];
            const uint32_t c0 = c.x, c1 = c.y, c2 = c.z, c3 = c.w;
            q0 = s == i ? c0 : q0;
            q1 = s == i ? c1 : q1;
            q2 = s == i ? c2 : q2;
            q3 = s == i ? c3 : q3;
        }
        const u32x4 q = u32x4{q0, q1, q2, q3};
        uint32_t i0 = sp.index(v0 + s * TR);
        float xv[E];
        widen<T>(q, xv);
        if (s == R) {
            xv[0] = ex;
            i0 = sp.base + (uint32_t)sp.extra(v0);
        }
        uint32_t em = 0;  // candidates among the vector's elements
#pragma unroll
        for (int e = 0; e < E; ++e) em |= (uint32_t)(xv[e] >= th) << e;
        if (s == R) em = 1u;
        if (hm == 0) em = 0;
#pragma unroll 1
        while (__builtin_amdgcn_ballot_w64(em != 0) != 0) {
            const int e = __builtin_ctz(em | 0x80000000u);
            float v = xv[0];
#pragma unroll
            for (int k = 1; k < E; ++k) v = e == k ? xv[k] : v;
            hl.offer(em != 0, make_key(v, i0 + (uint32_t)e));
            if (rare(hl.n > TH_CUT)) {
                hl.cut();
                th = __builtin_fmaxf(th, key_value(hl.tau + 1));
            }
            em &= em - 1;
        }
        hm &= hm - 1;
    }
}

// Rows of ties: the elements of one value, the only one in [lo, up), when the
// first few vectors of the team's lanes (vectors tr, tr + TR, ... of a lane) hold
// at least K of them.  Those are the K of lowest index: each wavefront appends
// its own, and the rest of the ties is never looked at.  False: they seem to hold
// fewer, and the list is as it was, empty.  (The team enters together.)
// Equal elements, 4000 x 32000 binary32 top-5: 239 us looked at one by one, with
// a selection after every 64 of them; 77 us in this way, as other rows.
template <typename T, int W, int R>
__device__ __forceinline__ bool held_ties(HeldSmem<W>& sm, HeldList& hl, const HeldSpan<T>& sp,
                                          const u32x4 (&buf)[R], int tr, float lo, float up) {
    constexpr int E = Vec<T>::N, TR = 64 * W, I = R < TH_TIE_I ? R : TH_TIE_I;
    int left = hl.K;  // ties still wanted
#pragma unroll 1
    for (int i = 0; i < I && i * TR < sp.nvec && left > 0; ++i) {
        u32x4 q = buf[0];
#pragma unroll
        for (int j = 1; j < I; ++j) {
            const u32x4 c = buf[j];
            const uint32_t c0 = c.x, c1 = c.y, c2 = c.z, c3 = c.w;
            q.x = i == j ? c0 : q.x;
            q.y = i == j ? c1 : q.y;
            q.z = i == j ? c2 : q.z;
            q.w = i == j ? c3 : q.w;
        }
        const bool in = tr + i * TR < sp.nvec;
        uint32_t tie = 0;       // bit e: element e is one
        int at = 0, total = 0;  // ties in the lanes before this one, and in all
        float xv[E];
        widen<T>(q, xv);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const bool is = in && xv[e] >= lo && !(xv[e] >= up);
            const uint64_t mask = __builtin_amdgcn_ballot_w64(is);
            tie |= (uint32_t)is << e;
            at += (int)__builtin_amdgcn_mbcnt_hi(
                (uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            total += __builtin_popcountll(mask);
        }
        int room = left, all = total;
        if constexpr (W > 1) {
            const int lane = threadIdx.x & 63;
            const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
            if (lane == 0) sm.tie[i][wv] = total;
            __syncthreads();
            const int counts = sm.tie[i][lane % W];
            all = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const int c = __builtin_amdgcn_readlane(counts, w);
                all += c;
                room -= w < wv ? c : 0;
            }
        }
        opaque(q);
        widen<T>(q, xv);
        const uint32_t idx0 = sp.index(tr + i * TR);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int is = tie >> e & 1;
            if (is && at < room) hl.keys[hl.n + at] = make_key(xv[e], idx0 + (uint32_t)e);
            at += is;
        }
        hl.n += room < 0 ? 0 : total < room ? total : room;
        left -= all;
        // the vectors left would not surely do, at this rate (4000 x 32000 bfloat16,
        // one element in 200 equal to the largest, top-50: 67 us without, 54 with)
        if (4 * left > 3 * all * (I - 1 - i)) break;
    }
    if (left <= 0) return true;
    hl.n = 0;
    return false;
}

// The end of a team's work: its lists' K largest keys and its pair, written as
// the row's outputs, or (PART) as chunk vr's partial; the chunk that completes
// a row merges it.  (W > 1: the wavefronts enter together.)
template <int W, int VAR, bool PART, uint32_t GRAN>
__device__ __forceinline__ void held_end(HeldSmem<W>& sm, HeldList& hl, MD md,
                                         float* __restrict__ vals, int32_t* __restrict__ idx,
                                         uint64_t* pkeys, MD* pmd, uint32_t* ctr, int64_t row,
                                         int64_t vr, int64_t segs, int K) {
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint64_t key;
    if constexpr (W == 1) {
        wave_sync();
        key = held_finish<1>(&sm.list[wv], &hl.n, K);
        held_store<VAR>(key, md, vals, idx, row, K);
    } else {
        if (lane == 0) {
            sm.cnt[wv] = hl.n;
            sm.wmd[wv] = md;
        }
        __syncthreads();
        // a merge of more partial keys than one wavefront holds takes them all
        // (the planned chunk counts stay below that)
        const bool wide = PART && segs * K > 64 * TK_MERGE_B;
        bool last = false;
        if (wv == 0) {
            key = held_finish<W>(sm.list, sm.cnt, K);
            if constexpr (VAR != TK_VALUES) {
                md = sm.wmd[0];
#pragma unroll
                for (int w = 1; w < W; ++w) md = md_merge(md, sm.wmd[w]);
            }
            if constexpr (!PART) {
                held_store<VAR>(key, md, vals, idx, row, K);
            } else {
                // the partial, at the device's coherence point; then the row's count
                if (lane < K)
                    __hip_atomic_store(pkeys + vr * K + lane, key, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                if (VAR != TK_VALUES && lane == 0)
                    __hip_atomic_store(reinterpret_cast<uint64_t*>(pmd + vr),
                                       __builtin_bit_cast(uint64_t, md), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                uint32_t done = 0;
                if (lane == 0)
                    done = __hip_atomic_fetch_add(ctr + row, 1u, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
                last = __builtin_amdgcn_readfirstlane(done) == (uint32_t)segs - 1;
            }
        }
        if constexpr (PART) {
            const uint64_t* pk = pkeys + row * segs * K;
            const MD* pm = pmd + row * segs;
            if (wide) {
                if (wv == 0 && lane == 0) sm.cnt[0] = last;
                __syncthreads();
                last = sm.cnt[0] != 0;
                __syncthreads();
            }
            if (!last) return;
            // every chunk of the row is in
            if (wide) {
                if (!held_merge<VAR, W, TK_MERGE_B, GRAN, true>(sm, wv, pk, pm, segs * K, segs, K,
                                                                &key, &md))
                    return;
            } else {
                held_merge<VAR, 1, TK_MERGE_B, GRAN, true>(sm, 0, pk, pm, segs * K, segs, K, &key,
                                                           &md);
            }
            held_store<VAR>(key, md, vals, idx, row, K);
            if (lane == 0)
                __hip_atomic_store(ctr + row, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// Wavefronts per SIMD asked of the compiler: as many as R vectors a lane leave
// registers for (64, 80 or 96 of them), without which it takes a few more.
// (Five, with workgroups of two a SIMD, let the next workgroup's loads start
// under the first wavefront's end of the one before: 511 x 50257 binary32 top-5,
// split, 25.5 us, against 27.6 with four.)
template <typename T, int W, int R, bool PART>
constexpr int held_waves() {
    const bool more = Vec<T>::N == 8 && (W == 8 || PART);  // bfloat16 widens to twice as many
    return R <= 6    ? (PART ? 7 : 8)
           : R <= 8  ? (more ? 6 : PART ? 7 : 8)
           : R <= 13 ? (more || PART ? 5 : 6)
                     : (more && W == 4 ? 4 : 5);
}

// Rows (PART = false: vr is a row, segs = 1) or chunks of rows (PART = true:
// chunk vr % segs of `seg` elements of row vr / segs) of at most 64 W R whole
// 16-byte vectors, W wavefronts each, held in registers.
template <typename T, int W, int R, int VAR, bool PART>
__global__ __launch_bounds__(W == 1 ? TK_BLOCK : 64 * W, (held_waves<T, W, R, PART>())) void topk_held(
    const T* __restrict__ x, float* __restrict__ vals, int32_t* __restrict__ idx, uint64_t* pkeys,
    MD* pmd, uint32_t* ctr, int64_t N, int64_t V, int K, int64_t seg, int64_t segs) {
    static_assert(!PART || W > 1, "chunks take a workgroup each");
    constexpr int E = Vec<T>::N, TR = 64 * W;
    constexpr uint32_t GRAN = E == 8 ? 1u << 16 : 1u;
    __shared__ HeldSmem<W> sm;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tr = W == 1 ? lane : tid;
    const int64_t vr = W == 1 ? (int64_t)blockIdx.x * (TK_BLOCK / 64) + wv : (int64_t)blockIdx.x;
    if (W == 1 && vr >= N) return;  // whole wavefronts; no barrier follows
    const int64_t row = PART ? vr / segs : vr;
    const int64_t start = PART ? (vr - row * segs) * seg : 0;
    const HeldSpan<T> sp(x, row, start, V, (int)(PART ? (V - start < seg ? V - start : seg) : V));
    const int nvec = sp.nvec;
    const float ninf = -__builtin_inff();

    // all loads first; lanes past the row load its last vector and mask it
    u32x4 buf[R];
    if (nvec > 0) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int v = tr + i * TR;
            buf[i] = __builtin_nontemporal_load(sp.vb + (v < nvec ? v : nvec - 1));
        }
    } else {
#pragma unroll
        for (int i = 0; i < R; ++i) buf[i] = u32x4{0, 0, 0, 0};
    }
    const float ex = tr < sp.ne ? load1(sp.xr + sp.extra(tr)) : ninf;

    // 1. maxima by vector, and the wavefront's
    float vm[R];
    float lm = __builtin_fmaxf(ex, ninf);  // a NaN element gives -inf
#pragma unroll
    for (int i = 0; i < R; ++i) {
        vm[i] = tr + i * TR < nvec ? held_vmax<T, VAR>(buf[i]) : ninf;
        lm = max3_raw(lm, vm[i], ninf);
    }
    const float wm = wave_max_f(lm);
    // the wavefront's pair, relative to its own maximum
    MD md = md_empty();
    if constexpr (VAR != TK_VALUES) {
        float s = wm * kLog2e;
        if (!(s > kEmptyS)) s = kEmptyS;  // no elements (or only -inf)
        float d = exp2_hw(__builtin_fmaf(ex, kLog2e, -s));
#pragma unroll
        for (int i = 0; i < R; ++i) {
            opaque(buf[i]);
            if (i == 0 || i * TR < nvec) {  // uniform
                float xv[E];
                widen<T>(buf[i], xv);
                const float p = sum_exp_fixed(0.0f, xv, s);
                d += tr + i * TR < nvec ? p : 0.0f;
            }
        }
        md = MD{s, group_sum<64>(d)};
    }
    // 2. the threshold: W = 1 from the maxima of up to four groups of each
    //    lane's elements (elements of one vector when it holds no more)
    KthBound b;
    if constexpr (W == 1) {
        constexpr int G = R == 1 ? 2 : R < 4 ? R : 4;
        float gm[G];
#pragma unroll
        for (int g = 0; g < G; ++g) gm[g] = g == 0 ? __builtin_fmaxf(ex, ninf) : ninf;
        if constexpr (R == 1) {
            float xv[E];
            widen<T>(buf[0], xv);
#pragma unroll
            for (int e = 0; e < E; ++e)
                gm[e % 2] = __builtin_fmaxf(gm[e % 2], tr < nvec ? xv[e] : ninf);
        } else {
#pragma unroll
            for (int i = 0; i < R; ++i) gm[i % G] = max3_raw(gm[i % G], vm[i], ninf);
        }
        uint32_t g[G];
#pragma unroll
        for (int i = 0; i < G; ++i) g[i] = order_word(gm[i]);
        b = kth_bound<G, GRAN>(g, order_word(wm), K);
    } else {
        b = team_bound<W, GRAN>(sm, order_word(lm), K);
    }
    // 3. the candidates: elements at or above the bound
    HeldList hl{sm.list[wv], K, 0, 0ull};
    float th = key_value((uint64_t)b.lo << 32);
    uint32_t hm = (uint32_t)(tr < sp.ne && ex >= th) << R;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        opaque(buf[i]);
        hm |= (uint32_t)(tr + i * TR < nvec && vm[i] >= th) << i;
    }
    if (rare(b.tied && nvec >= K)) {  // (not for want of elements)
        const float up = key_value((uint64_t)b.up << 32);
        if (held_ties<T, W, R>(sm, hl, sp, buf, tr, th, up)) {
            // the ties are settled: what is left are elements above them (the
            // maxima are found again, so that they need not be kept until here)
            th = up;
            hm &= 1u << R;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                opaque(buf[i]);
                hm |= (uint32_t)(tr + i * TR < nvec && held_vmax<T, VAR>(buf[i]) >= th) << i;
            }
        }
    }
    held_offer<T, R, TR>(hl, sp, buf, tr, hm, th, ex);
    // 4. the K largest, in order
    held_end<W, VAR, PART, GRAN>(sm, hl, md, vals, idx, pkeys, pmd, ctr, row, vr, segs, K);
}

// Second kernel of the projection with top-k: a row's n = S K partial keys and S
// pairs by W wavefronts (W = 1: four rows per workgroup), R keys a lane at a time.
template <int VAR, int W, int R>
__global__ __launch_bounds__(W == 1 ? TK_BLOCK : 64 * W) void topk_merge_held(
    const uint64_t* __restrict__ pkeys, const MD* __restrict__ pmd, float* __restrict__ vals,
    int32_t* __restrict__ idx, int64_t N, int64_t S, int K) {
    __shared__ HeldSmem<W> sm;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row = W == 1 ? (int64_t)blockIdx.x * (TK_BLOCK / 64) + wv : (int64_t)blockIdx.x;
    if (W == 1 && row >= N) return;
    uint64_t key;
    MD md;
    if (held_merge<VAR, W, R, 1, false>(sm, wv, pkeys + row * S * K, pmd + row * S, S * K,
                                     S, K, &key, &md))
        held_store<VAR>(key, md, vals, idx, row, K);
}

// ------------------------------------------------------------------ launchers
constexpr int TH_RMAX = 16;  // vectors per lane

// A wavefront per row while it holds the row's keys in one batch (512), then a
// workgroup of four or sixteen: the merge of 2004 pairs and 10020 keys for each
// of 64 rows took ~40 us with a wavefront per row, in twenty batches on a
// quarter of the CUs (the whole projection + top-5 at 64 x 4096 x 128256: 216
// -> 191 us; 37 x 512 x 50001 top-16: 77.5 -> 50.7).
template <int VAR>
hipError_t launch_merge_held(const uint64_t* pkeys, const MD* pmd, float* vals, int32_t* idx,
                             int64_t N, int64_t S, int K, hipStream_t st) {
    const int64_t n = S * K;
    const dim3 rows((unsigned)N), quads((unsigned)((N + 3) / 4));
    if (n <= 512)
        hipLaunchKernelGGL((topk_merge_held<VAR, 1, 8>), quads, dim3(256), 0, st, pkeys, pmd, vals,
                           idx, N, S, K);
    else if (n <= 2048)
        hipLaunchKernelGGL((topk_merge_held<VAR, 4, 8>), rows, dim3(256), 0, st, pkeys, pmd, vals,
                           idx, N, S, K);
    else if (n <= 4096)
        hipLaunchKernelGGL((topk_merge_held<VAR, 4, 16>), rows, dim3(256), 0, st, pkeys, pmd, vals,
                           idx, N, S, K);
    else
        hipLaunchKernelGGL((topk_merge_held<VAR, 16, 16>), rows, dim3(1024), 0, st, pkeys, pmd,
                           vals, idx, N, S, K);
    return hipGetLastError();
}

// Vectors per lane: the smallest of 1, 2, 3, 4, 6, 8, 12, 16 that holds the
// row's `nv` vectors (a lane's spare vectors cost a masked load each); for
// binary32 by eight wavefronts also 13, the most that leaves three workgroups a
// CU their registers (4000 x 25000 top-5 / top-30 / top-64 66.7 / 72.2 / 83.0 us
// with 16, 63.5 / 63.8 / 66.0 with 13; 14 in as many registers spills, 15 and 16
// are level).
template <typename T, int W, int VAR, bool PART>
hipError_t launch_held_w(const TopkLaunch& a, int64_t nv, uint64_t* pkeys, MD* pmd) {
    const int64_t r = (nv + 64 * W - 1) / (64 * W);
    const int64_t rows = W == 1 ? (a.N + TK_BLOCK / 64 - 1) / (TK_BLOCK / 64) : a.N * a.S;
    const dim3 grid((unsigned)rows), block(W == 1 ? TK_BLOCK : 64 * W);
    const T* x = static_cast<const T*>(a.x);
    const int64_t seg = PART ? a.chunk : a.V, segs = PART ? a.S : 1;
#define OSM_HELD(R_)                                                                             \
    hipLaunchKernelGGL((topk_held<T, W, R_, VAR, PART>), grid, block, 0, a.st, x, a.vals, a.idx, \
                       pkeys, pmd, a.ctr, a.N, a.V, a.K, seg, segs)
    if (r <= 1) OSM_HELD(1);
    else if (r <= 2) OSM_HELD(2);
    else if (r <= 3) OSM_HELD(3);
    else if (r <= 4) OSM_HELD(4);
    else if (r <= 6) OSM_HELD(6);
    else if (r <= 8) OSM_HELD(8);
    else if (r <= 12) OSM_HELD(12);
    else if (W == 8 && Vec<T>::N == 4 && r <= 13) OSM_HELD((W == 8 && Vec<T>::N == 4 ? 13 : 16));
    else if (r <= TH_RMAX) OSM_HELD(16);
    else return hipErrorInvalidValue;
#undef OSM_HELD
    return hipGetLastError();
}

// Launch of a row kernel (a.S <= 1) or of the one-kernel split (a.S > 1) whose
// rows or chunks the registers hold; false: they do not, nothing was launched.
template <typename T, int VAR>
bool launch_topk_held(const TopkLaunch& a, uint64_t* pkeys, MD* pmd, hipError_t* e) {
    const int64_t nv = (a.S > 1 ? a.chunk : a.V) / Vec<T>::N;  // at least the whole vectors
    if (a.S > 1) {
        // Chunks of eight wavefronts: two workgroups a CU are resident.  With
        // more of them than that, streamed chunks overlap the next one's loads
        // better than the selection costs at small K (400 x 50000 binary32 in
        // 800 chunks, top-1: 21.8 us streamed, 22.7 held; top-5 26.1 and 25.1),
        // most where the second round is short (top-5, streamed / held: 300 x
        // 50257 21.2 / 21.6, 350 x 50257 21.7 / 22.5, 300 x 60000 22.1 / 23.8;
        // but 257 x 50257 18.4 / 17.5, 300 x 40000, whose chunks leave room for
        // three workgroups, 17.6 / 14.4, and top-16 300 x 50257 23.9 / 22.7).
        const int64_t n = a.N * a.S, two = 2 * (int64_t)a.cus;
        const bool few = nv > 512 * 12 && 10 * n > 11 * two && 2 * n < 3 * two;
        const bool eight = n <= two || a.K > (few ? 8 : 4);
        if (nv <= 256 * TH_RMAX) *e = launch_held_w<T, 4, VAR, true>(a, nv, pkeys, pmd);
        else if (nv <= 512 * TH_RMAX && eight) *e = launch_held_w<T, 8, VAR, true>(a, nv, pkeys, pmd);
        else return false;
        return true;
    }
    if (a.waves_per_row == 1 && nv <= 64 * TH_RMAX)
        *e = launch_held_w<T, 1, VAR, false>(a, nv, pkeys, pmd);
    else if (a.waves_per_row == 4 && nv <= 256 * TH_RMAX)
        *e = launch_held_w<T, 4, VAR, false>(a, nv, pkeys, pmd);
    else if (a.waves_per_row == 4 && nv <= 512 * TH_RMAX)
        *e = launch_held_w<T, 8, VAR, false>(a, nv, pkeys, pmd);
    else
        return false;
    return true;
}

}  // namespace osm
