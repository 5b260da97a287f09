// C-ABI of the library: argument validation, kernel choice and launches.
// Declarations and the contract of every entry point are in osoftmax.h.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "kernels.h"
#include "osoftmax.h"

namespace {

constexpr int64_t kMaxDim = 2147483647;  // 2^31 - 1
constexpr int64_t kMaxThreads = 4294967295;  // of one launch, workgroups times their size
constexpr int kMaxDevices = 64;

size_t elem_size(int dtype) { return dtype == OSM_BF16 ? 2 : 4; }
int elems_per_vec(int dtype) { return dtype == OSM_BF16 ? 8 : 4; }

// ------------------------------------------------------------ device state
// Scratch of the split kernels, cached per stream: work on one stream runs in
// order, so successive calls on a stream share a buffer without allocating;
// distinct streams get distinct buffers.
struct ScratchSlot {
    hipStream_t stream;
    void* ptr;
    size_t bytes;
};
constexpr int kScratchSlots = 64;
constexpr size_t kScratchMin = 256 * 1024;

// Fixed scratch of softmax_topk_ex_noalloc: one copy per device, held until
// the process ends.  In host code `scratch` names a host-side stand-in, not
// device memory: its device address is looked up once per device (with the
// device current) and kept in DeviceState::scratch_ptr, which is what every
// launch and copy uses.
constexpr size_t kNoAllocBytes = OSM_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

// Clears n 32-bit words (a kernel rather than a memset, so that a captured
// graph replays it as an ordinary kernel node).
__global__ void zero_u32(uint32_t* p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

struct DeviceState {
    std::once_flag once;
    int cus = 0;
    void* scratch_ptr = nullptr;  // device address of `scratch` (null if the lookup failed)
    hipMemPool_t pool = nullptr;
    bool pool_ok = false;
    std::mutex mu;  // guards the scratch and counter tables
    ScratchSlot slots[kScratchSlots] = {};
    int nslots = 0;
    ScratchSlot cslots[kScratchSlots] = {};  // zeroed counter arrays, per stream
    int ncslots = 0;
};
DeviceState g_dev[kMaxDevices];

DeviceState* device_state(int* dev_out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    DeviceState& s = g_dev[dev];
    std::call_once(s.once, [&s, dev]() {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            cus <= 0)
            cus = 256;
        s.cus = cus;
        void* sp = nullptr;
        if (hipGetSymbolAddress(&sp, HIP_SYMBOL(scratch)) == hipSuccess && sp) s.scratch_ptr = sp;
        // A library-owned stream-ordered pool keeps split-V scratch cheap to
        // allocate and free on any stream without touching the device's
        // default pool settings.
        hipMemPoolProps props = {};
        props.allocType = hipMemAllocationTypePinned;
        props.handleTypes = hipMemHandleTypeNone;
        props.location.type = hipMemLocationTypeDevice;
        props.location.id = dev;
        if (hipMemPoolCreate(&s.pool, &props) == hipSuccess) {
            uint64_t keep = UINT64_MAX;
            (void)hipMemPoolSetAttribute(s.pool, hipMemPoolAttrReleaseThreshold, &keep);
            s.pool_ok = true;
        }
        (void)hipGetLastError();
    });
    if (dev_out) *dev_out = dev;
    return &s;
}

// The scratch and counter tables are guarded by the device's mutex, and a
// call that uses a stream's buffers holds it from acquiring them until its
// last launch has been enqueued (`lk`, locked by the first acquire): calls
// from several host threads on one stream then enqueue their kernels whole,
// one call after another, so no call's launches land between another's on
// the same buffers, and a buffer is replaced (its old copy freed in stream
// order) only between calls.

// Slot of `stream` in `tab`, creating it if the table has room; null if full.
ScratchSlot* find_slot(ScratchSlot* tab, int* n, hipStream_t stream) {
    for (int i = 0; i < *n; ++i)
        if (tab[i].stream == stream) return &tab[i];
    if (*n >= kScratchSlots) return nullptr;
    ScratchSlot* slot = &tab[(*n)++];
    *slot = ScratchSlot{stream, nullptr, 0};
    return slot;
}

// Scratch of at least `bytes` for work enqueued on `stream`.  A stream's
// buffer grows by a stream-ordered allocation from the library pool (the old
// one is freed in stream order behind the work already enqueued) and is kept
// until osm_stream_release or the end of the process.  Once the table is
// full, a call gets a buffer of its own (*temp = true) that it frees in
// stream order after its launches.
int acquire_scratch(DeviceState* ds, std::unique_lock<std::mutex>& lk, hipStream_t stream,
                    size_t bytes, void** out, bool* temp) {
    if (!ds->pool_ok) return OSM_ENOMEM;
    if (!lk.owns_lock()) lk.lock();
    ScratchSlot* slot = find_slot(ds->slots, &ds->nslots, stream);
    *temp = slot == nullptr;
    if (slot && slot->bytes >= bytes) {
        *out = slot->ptr;
        return OSM_OK;
    }
    size_t want = bytes;
    if (slot) {
        want = bytes > 2 * slot->bytes ? bytes : 2 * slot->bytes;
        want = want > kScratchMin ? want : kScratchMin;
    }
    void* p = nullptr;
    if (hipMallocFromPoolAsync(&p, want, ds->pool, stream) != hipSuccess || !p) {
        (void)hipGetLastError();
        return OSM_ENOMEM;
    }
    if (slot) {
        if (slot->ptr) (void)hipFreeAsync(slot->ptr, stream);
        slot->ptr = p;
        slot->bytes = want;
    }
    *out = p;
    return OSM_OK;
}

// A zeroed array of at least `count` 32-bit counters for work enqueued on
// `stream`; the kernels that use it leave it zeroed.  A stream's array grows
// by a stream-ordered allocation, cleared in stream order by a fill kernel
// (not a memset, so that a call captured into a graph records a kernel
// node); once the table is full, a call gets an array of its own
// (*temp = true) to free after its launches.  Locking as acquire_scratch.
int acquire_counters(DeviceState* ds, std::unique_lock<std::mutex>& lk, hipStream_t stream,
                     size_t count, uint32_t** out, bool* temp) {
    if (!ds->pool_ok) return OSM_ENOMEM;
    if (!lk.owns_lock()) lk.lock();
    ScratchSlot* slot = find_slot(ds->cslots, &ds->ncslots, stream);
    *temp = slot == nullptr;
    const size_t bytes = count * 4;
    if (slot && slot->bytes >= bytes) {
        *out = static_cast<uint32_t*>(slot->ptr);
        return OSM_OK;
    }
    size_t want = bytes;
    if (slot) want = bytes > 2 * slot->bytes ? bytes : 2 * slot->bytes;
    void* p = nullptr;
    if (hipMallocFromPoolAsync(&p, want, ds->pool, stream) != hipSuccess || !p) {
        (void)hipGetLastError();
        return OSM_ENOMEM;
    }
    const int64_t words = (int64_t)(want / 4);
    hipLaunchKernelGGL(zero_u32, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, stream,
                       static_cast<uint32_t*>(p), words);
    if (hipGetLastError() != hipSuccess) {
        (void)hipFreeAsync(p, stream);
        return OSM_EHIP;
    }
    if (slot) {
        if (slot->ptr) (void)hipFreeAsync(slot->ptr, stream);
        slot->ptr = p;
        slot->bytes = want;
    }
    *out = static_cast<uint32_t*>(p);
    return OSM_OK;
}

// Drops `stream`'s slot from `tab` (its buffer freed in stream order).
hipError_t release_slot(ScratchSlot* tab, int* n, hipStream_t stream) {
    hipError_t e = hipSuccess;
    for (int i = 0; i < *n; ++i) {
        if (tab[i].stream != stream) continue;
        if (tab[i].ptr) e = hipFreeAsync(tab[i].ptr, stream);
        tab[i] = tab[*n - 1];
        --*n;
        break;
    }
    return e;
}

// ------------------------------------------------------------- validation
bool overlaps(const void* a, size_t abytes, const void* b, size_t bbytes) {
    uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    return a0 < b0 + bbytes && b0 < a0 + abytes;
}

bool aligned(const void* p, size_t a) { return ((uintptr_t)p % a) == 0; }

// Sizes, dtype and byte count of an N x V batch; false on any violation.
bool check_shape(int64_t N, int64_t V, int dtype, size_t* bytes) {
    if (N < 0 || N > kMaxDim || V < 1 || V > kMaxDim) return false;
    if (dtype != OSM_F32 && dtype != OSM_BF16) return false;
    // N, V < 2^31 and element size <= 4: the product is below 2^64
    *bytes = (size_t)N * (size_t)V * elem_size(dtype);
    return true;
}

int hip_status(hipError_t e) { return e == hipSuccess ? OSM_OK : OSM_EHIP; }

// ---------------------------------------------------------------- planning
struct Plan {
    int kernel;
    int64_t param;
};

// vec: x and y are congruent modulo 16 bytes (else rows are taken an element at
// a time).
Plan choose(int64_t N, int64_t V, int dtype, int cus, bool vec = true) {
    const int64_t E = elems_per_vec(dtype);
    const int64_t nv = (V + E - 1) / E;  // 16-byte vectors per row
    // Short rows: a lane group per row, sized so each lane has ~2-4 vectors.
    if (nv <= 16) return {OSM_KERNEL_ROWS, 4};
    if (nv <= 32) return {OSM_KERNEL_ROWS, 8};
    if (nv <= 64) return {OSM_KERNEL_ROWS, 16};
    // The longer of them with few rows, which leave most of the chip idle, take
    // a workgroup each (us, a wavefront a row -> this; binary32 64 x 1500 4.06 ->
    // 3.30, 400 x 1000 3.64 -> 3.37, 200 x 4096 6.5 -> 3.4, but 400 x 600 3.04 ->
    // 3.20; bfloat16 64 x 2000 4.4 -> 3.0, 200 x 8192 8.2 -> 3.8), then two
    // wavefronts (binary32 800 x 4096 6.9 -> 4.9, but 1024 x 2000 5.08 -> 5.14).
    // Larger batches keep a wavefront, but for bfloat16 rows of 513 to 768
    // vectors in batches of eight rows a CU and more (4000 x 5000 18.8 -> 15.6,
    // 32768 x 5000 139 -> 115; 3000 x 2400 6.9 -> 7.7).  Between four and eight
    // rows a CU two wavefronts gain at some lengths and lose at others (1500 x
    // 5000 9.2 -> 8.3, 1500 x 6144 8.5 -> 8.6, 1800 x 6144 8.6 -> 9.1).
    const int64_t c = cus;
    if (nv <= 128) {  // bfloat16: 200 x 1000 4.4 -> 3.0, but 512 x 600 3.40 -> 3.55
        if (dtype != OSM_F32 && nv > 96 && N <= 2 * c) return {OSM_KERNEL_ROWS, 128};
        return {OSM_KERNEL_ROWS, 32};
    }
    if (nv <= 1024) {
        if (N <= (nv > 200 ? 2 * c : nv > 160 ? c : 0)) return {OSM_KERNEL_ROWS, 256};
        if (nv > 512 && N <= 4 * c && N > 2 * c) return {OSM_KERNEL_ROWS, 128};
        if (dtype != OSM_F32 && nv > 512 && nv <= 768 && N >= 8 * c) return {OSM_KERNEL_ROWS, 128};
        return {OSM_KERNEL_ROWS, 64};
    }
    // Long rows but too few of them to fill the chip: split each row, into
    // about four chunks per CU in all, six for the smallest batches (at 10
    // rows of 10^6: 19.5 us with six against 22.5 with four; at 64 or 256
    // rows four is as fast or faster).
    //
    // A workgroup per row is faster for rows of up to 20480 elements, and for
    // up to 57344 (24576 in bfloat16, which brings twice the arithmetic per
    // byte to one CU) once three CUs in eight have a row (us, a workgroup per
    // row against the split: 64 x 16384 binary32 5.1 / 6.1, 200 x 32000 11.3 /
    // 15.1, 300 x 20481 bfloat16 9.2 / 11.2). Longer rows need half of the CUs
    // busy, three quarters for the longest bfloat16 ones (130 x 100000 binary32
    // 24.1 / 28.5, but 96 x 66001 16.1 / 15.4; bfloat16 130 x 50257 10.5 / 12.6,
    // but 96 x 32000 8.5 / 7.8 and 160 x 100000 21.3 / 18.8); no second round
    // of rows that only some CUs take (300 x 57344 bfloat16 19.4 / 17.3, but
    // 511 x 57344 25.0 / 32.5); and a second pass that still finds most of the
    // row in cache (150 x 150001 binary32 50.9 / 47.1).
    const int64_t want_blocks = (N <= 16 ? 6 : 4) * (int64_t)cus;
    const bool f32 = dtype == OSM_F32;
    const bool busy = f32 || V <= 57344 ? 2 * N >= cus : 4 * N >= 3 * (int64_t)cus;
    const bool even = N <= cus || 5 * N >= 8 * (int64_t)cus;
    bool rows = V <= 20480 || (V <= (f32 ? 57344 : 24576) && 8 * N >= 3 * (int64_t)cus) ||
                (V <= 131072 && busy && even);
    // With half to five eighths of the CUs busy, binary32 rows of 48 K to 64 K
    // elements lose more at some lengths than they gain at others (rows / split: 128 x 50000 16.7 / 12.8, x 50257 16.1 / 14.2, x 53000 14.4 /
    // 14.9, x 57344 15.2 / 13.1; 160 x 50000 18.4 / 16.5, x 53000 16.8 / 17.5, x
    // 57344 18.8 / 17.3; but 112 x 50000 11.6 / 13.0, 192 x 57344 20.4 / 23.7).
    if (f32 && V > 49152 && V <= 65536 && 2 * N >= cus && 8 * N <= 5 * (int64_t)cus) rows = false;
    // An element at a time a row is bound by the accesses a CU can make, not by
    // memory, and the split's many workgroups are faster down to 16384 elements
    // until every CU has a row of more than 6144 vectors' length (x and y apart by
    // 3 elements, rows / split: bfloat16 64 x 16384 19.2 / 8.8, 192 x 32000 33.7 /
    // 15.4, 410 x 40000 54.2 / 43.1; binary32 96 x 57344 39.1 / 20.1, 300 x 24576
    // 34.9 / 23.9; but 256 x 32000 26.2 / 28.0, bfloat16 410 x 57344 47.7 / 58.8).
    if (!vec) rows = V < 16384 || (rows && nv > 6144 && N >= cus);
    if (N < 2 * (int64_t)cus && rows && nv > 2048 && nv <= 6144) return {OSM_KERNEL_ROWS, 512};
    if (N < 2 * (int64_t)cus && !rows) {
        int64_t S = (want_blocks + N - 1) / N;
        int64_t s_cap = (V + 4095) / 4096;  // keep chunks >= 4096 elements
        if (S > s_cap) S = s_cap;
        if (S >= 2) return {OSM_KERNEL_SPLIT, S};
    }
    if (nv <= 2048) return {OSM_KERNEL_ROWS, 256};
    if (nv <= 4096) return {OSM_KERNEL_ROWS, 512};
    return {OSM_KERNEL_ROWS, 1024};
}

// Row-resident mode: the first (block, 16-byte vectors per lane) shape that
// holds the row's vectors; false if none does.  Smaller workgroups come
// first: with 16 vectors per lane (4 wavefronts per SIMD) a CU then holds two
// or four rows at once, so one row's loads overlap another's reduction.
struct ResShape {
    int block, r;
};
bool choose_resident(int64_t V, int dtype, int64_t block_req, ResShape* out) {
    const int64_t need = V / elems_per_vec(dtype);  // at least the row's whole vectors
    static const ResShape shapes[] = {{256, 4}, {256, 8}, {256, 16}, {512, 16}, {1024, 16}};
    for (const ResShape& c : shapes) {
        if (block_req && c.block != block_req) continue;
        if (need <= (int64_t)c.block * c.r) {
            *out = c;
            return true;
        }
    }
    return false;
}

bool team_ok(int64_t t) {
    return t == 4 || t == 8 || t == 16 || t == 32 || t == 64 || t == 128 || t == 256 ||
           t == 512 || t == 1024;
}

int run_softmax(const void* x, void* y, int64_t N, int64_t V, int dtype, int mode, int kernel,
                int64_t param, hipStream_t stream) {
    size_t bytes = 0;
    if (!check_shape(N, V, dtype, &bytes)) return OSM_EINVAL;
    if (mode != OSM_NAIVE && mode != OSM_SAFE && mode != OSM_ONLINE && mode != OSM_RESIDENT)
        return OSM_EINVAL;
    if (kernel != OSM_KERNEL_AUTO && kernel != OSM_KERNEL_ROWS && kernel != OSM_KERNEL_SPLIT)
        return OSM_EINVAL;
    if (mode == OSM_RESIDENT) {
        if (kernel == OSM_KERNEL_SPLIT ||
            (kernel == OSM_KERNEL_ROWS && param != 256 && param != 512 && param != 1024))
            return OSM_EINVAL;
    } else {
        if (kernel == OSM_KERNEL_ROWS && !team_ok(param)) return OSM_EINVAL;
        if (kernel == OSM_KERNEL_SPLIT && (param < 1 || param > kMaxDim)) return OSM_EINVAL;
    }
    if (N == 0) return OSM_OK;
    if (!x || !y) return OSM_EINVAL;
    const size_t es = elem_size(dtype);
    if (!aligned(x, es) || !aligned(y, es)) return OSM_EINVAL;
    if (overlaps(x, bytes, y, bytes)) return OSM_EINVAL;
    const bool vec = (((uintptr_t)x - (uintptr_t)y) % 16) == 0;
    if (mode == OSM_RESIDENT) {
        ResShape rs;
        if (!choose_resident(V, dtype, kernel == OSM_KERNEL_ROWS ? param : 0, &rs))
            return OSM_EUNSUPPORTED;
        return hip_status(
            osm::launch_softmax_resident(x, y, N, V, dtype, rs.block, rs.r, vec, stream));
    }

    int dev = 0;
    DeviceState* ds = device_state(&dev);
    if (!ds) return OSM_EHIP;
    Plan p = kernel == OSM_KERNEL_AUTO ? choose(N, V, dtype, ds->cus, vec) : Plan{kernel, param};

    if (p.kernel == OSM_KERNEL_ROWS)
        return hip_status(osm::launch_softmax_rows(x, y, N, V, dtype, mode, (int)p.param, vec,
                                                   stream));

    // split-V: chunk = ceil(V / S) rounded up to whole 16-byte vectors
    const int64_t E = elems_per_vec(dtype);
    int64_t S = p.param;
    if (S > V) S = V;
    int64_t chunk = (V + S - 1) / S;
    chunk = (chunk + E - 1) / E * E;
    S = (V + chunk - 1) / chunk;  // drop chunks that would start past the row
    if (N * S > kMaxDim) return OSM_EINVAL;
    void* part = nullptr;
    bool temp = false;
    std::unique_lock<std::mutex> lk(ds->mu, std::defer_lock);  // held until the launches are in
    const int st = acquire_scratch(ds, lk, stream, (size_t)N * (size_t)S * 8, &part, &temp);
    if (st != OSM_OK) return st;
    hipError_t e = osm::launch_softmax_split(x, y, part, N, V, dtype, mode, S, chunk, vec,
                                             stream);
    hipError_t f = temp ? hipFreeAsync(part, stream) : hipSuccess;
    if (e != hipSuccess) return OSM_EHIP;
    return hip_status(f);
}

// Top-k plans.  Rows that the registers hold (topk_held.hpp) take a wavefront
// or a workgroup each; only longer ones are streamed or split.

// Streamed rows: one wavefront per row once the batch alone can give every
// SIMD several wavefronts, or when rows are short (up to 1536 elements: a
// wavefront streams them in a step or two, and more wavefronts per row only
// add the barrier and the cross-wavefront merge); a small batch of long rows
// is split into chunks (a workgroup each, at most two workgroups per CU in
// all, at least two chunks a row: every chunk pays a fixed selection cost, so
// more, shorter chunks stop paying off early, and a third workgroup on a few
// CUs slows their chunks, which the rows then wait for: 10 x 4e6 top-5 took
// 34.5 us in 510 workgroups against 41.8 in 520); otherwise a workgroup (four
// wavefronts) per row.
//
// The chunk count is also capped so that a row's S * K partial keys fit one
// batch of a wavefront's merge (512 keys), and chunks keep at least `min_chunk`
// elements.  The cap is low for K > 15: the whole workgroup merges more keys as
// well, and longer chunks no longer fit in registers (10 x 10^6 binary32, this
// plan / 34 / 51 chunks: top-15 16.5 / 16.4 / 17.8 us, top-30 25.8 / 18.1 / 17.9,
// top-50 34.9 / 19.6 / 18.7, top-64 44.7 / 27.4 / 31.7; bfloat16 top-30 14.1 /
// 15.2 / 16.3).
Plan choose_topk_stream(int64_t N, int64_t V, int K, int cus, int64_t min_chunk = 4096) {
    if (N >= 4 * (int64_t)cus || V <= 1536) return {OSM_KERNEL_ROWS, 64};
    if (N < 2 * (int64_t)cus && V >= 8192) {
        int64_t S = (2 * (int64_t)cus) / N;
        if (S < 2) S = 2;
        int64_t s_cap = V / min_chunk;
        if (S > s_cap) S = s_cap;
        const int64_t k_cap = 512 / K;
        if (S > k_cap) S = k_cap;
        if (S >= 2) return {OSM_KERNEL_SPLIT, S};
    }
    return {OSM_KERNEL_ROWS, 256};
}

// Rows of nv 16-byte vectors, by the measured crossings (us, one device):
//  * up to 1024 vectors a wavefront holds a row.  It is the faster one for
//    large batches (16000 x 4000 bfloat16 top-5: 25.6 against 38.4 with a
//    workgroup per row; 4000 x 1000 binary32 6.4 against 8.0); for batches
//    under four rows a CU, rows past 1536 elements take a workgroup
//    (300 x 2000 binary32 top-5: 4.4 against 5.1);
//  * up to 8192 vectors a workgroup of four (to 4096 vectors) or eight
//    wavefronts does, against streaming the row by one wavefront (4000 x 10000
//    binary32 top-5 / top-50: 28.2 / 29.7 against 31.0 / 37.2; 4000 x 32000
//    bfloat16 43.3 / 46.7 against 52.4 / 67.8; 16000 x 32000 binary32 292 / 328
//    against 303 / 330; 4000 x 25000 top-5 / top-30 63.5 / 63.8 against 63.9 /
//    66.3) and against splitting it (64 x 32000 binary32 8.3 / 9.9 against
//    9.8 / 11.4).  Large batches of bfloat16 rows past 4096 vectors
//    stream (4000 x 50000 top-5: 69.1 against 73.9: half the bytes for the same
//    arithmetic, which a held row does not overlap with its loads), and so do, at
//    large K, binary32 rows of 13 to 15 vectors a lane that load 16 (top-5 /
//    top-30 / top-64, streamed against held: 4000 x 27000 68.5 / 70.5 / 77.3
//    against 69.0 / 74.7 / 84.9, x 30000 75.3 / 77.1 / 84.3 against 75.4 / 78.6 /
//    88.7; but 2100 x 27000, a few rows into another round of streams, 47.1 /
//    49.2 / 57.0 against 40.6 / 43.9 / 51.4, and 1024 x 27000 22.3 / 29.4 / 39.0
//    against 21.0 / 22.9 / 25.8).  A few rows past 4096 vectors at small K split
//    (1 x 65000 bfloat16 top-5: 6.9 against 8.0; top-50 9.9 against 9.3);
//  * longer rows are streamed or split, the chunks with at least 2048 vectors
//    (16 x 128256 bfloat16 top-5: 9.4 in 8 chunks, 12.4 in 31), or 1024 for a
//    few rows (1 x 128256 bfloat16 top-5: 8.2 in 7 chunks, 7.1 in 31);
//  * a batch of so many rows that a workgroup each would pass what one launch
//    takes (2^24 rows and more: 275 GB of the shortest such rows) keeps a
//    wavefront a row.
Plan choose_topk(int64_t N, int64_t V, int dtype, int K, int cus) {
    const int64_t E = elems_per_vec(dtype), nv = V / E;
    const bool many = N >= 4 * (int64_t)cus;
    if (V <= 1536 || (many && nv <= 1024) || N * 256 > kMaxThreads) return {OSM_KERNEL_ROWS, 64};
    if (nv <= 4096) return {OSM_KERNEL_ROWS, 256};
    const bool stream = dtype == OSM_F32 ? K > 20 && nv > 6656 && nv <= 7800 && N >= 11 * (int64_t)cus
                                         : N >= 8 * (int64_t)cus;
    if (nv <= 8192 && (many ? !stream : N >= 16 || K > 8)) return {OSM_KERNEL_ROWS, 256};
    return choose_topk_stream(N, V, K, cus, (N <= 8 ? 1024 : 2048) * E);
}

// One top-k pass of variant `var` over x (already validated).  noalloc: the
// split path's partials and row counters go to the device's fixed scratch
// array instead of the stream's pool buffers.
int launch_topk_pass(const void* x, float* vals, int32_t* idx, int64_t N, int64_t V, int K,
                     int dtype, int var, int kernel, int64_t param, DeviceState* ds,
                     hipStream_t stream, bool noalloc = false) {
    // (the safe variant reads its rows twice and is always streamed)
    Plan p = kernel != OSM_KERNEL_AUTO ? Plan{kernel, param}
             : var == osm::TK_SAFE     ? choose_topk_stream(N, V, K, ds->cus)
                                       : choose_topk(N, V, dtype, K, ds->cus);
    osm::TopkLaunch a{x, vals, idx, nullptr, N, V, K, 1, 1, V, ds->cus, stream};
    if (p.kernel == OSM_KERNEL_ROWS) {
        a.waves_per_row = (int)(p.param / 64);
        return hip_status(osm::launch_topk(a, dtype, var));
    }
    // split: chunk = ceil(V / S) rounded up to whole 16-byte vectors
    const int64_t E = elems_per_vec(dtype);
    int64_t S = p.param;
    if (S > V) S = V;
    int64_t chunk = (V + S - 1) / S;
    chunk = (chunk + E - 1) / E * E;
    S = (V + chunk - 1) / chunk;  // drop chunks that would start past the row
    if (N * S > kMaxDim) return OSM_EINVAL;
    if (S == 1) {  // one chunk is the whole row
        a.waves_per_row = 4;
        return hip_status(osm::launch_topk(a, dtype, var));
    }
    a.S = S;
    a.chunk = chunk;
    if (noalloc) {
        // partials first, then N row counters (256-byte aligned), cleared by a
        // fill kernel in stream order before the split kernel
        const size_t pb = (osm::topk_part_bytes(N, S, K) + 255) / 256 * 256;
        if (pb + (size_t)N * 4 > kNoAllocBytes) return OSM_ESCRATCH;
        if (!ds->scratch_ptr) return OSM_EHIP;
        a.part = ds->scratch_ptr;
        a.ctr = reinterpret_cast<uint32_t*>(static_cast<char*>(ds->scratch_ptr) + pb);
        const int64_t blocks = (N + 255) / 256;
        hipLaunchKernelGGL(zero_u32, dim3((unsigned)blocks), dim3(256), 0, stream, a.ctr, N);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return OSM_EHIP;
        return hip_status(osm::launch_topk(a, dtype, var));
    }
    void* part = nullptr;
    bool temp = false;
    std::unique_lock<std::mutex> lk(ds->mu, std::defer_lock);  // held until the launch is in
    int st = acquire_scratch(ds, lk, stream, osm::topk_part_bytes(N, S, K), &part, &temp);
    if (st != OSM_OK) return st;
    a.part = part;
    // per-row chunk counters: each row's last chunk merges it in the same kernel
    bool ctemp = false;
    st = acquire_counters(ds, lk, stream, (size_t)N, &a.ctr, &ctemp);
    if (st != OSM_OK) {
        if (temp) (void)hipFreeAsync(part, stream);
        return st;
    }
    hipError_t e = osm::launch_topk(a, dtype, var);
    hipError_t f = temp ? hipFreeAsync(part, stream) : hipSuccess;
    hipError_t g = ctemp ? hipFreeAsync(a.ctr, stream) : hipSuccess;
    if (e != hipSuccess) return OSM_EHIP;
    if (f != hipSuccess) return hip_status(f);
    return hip_status(g);
}

bool topk_algo_ok(int algo) {
    return algo == OSM_TOPK_ONLINE_FUSED || algo == OSM_TOPK_SAFE_FUSED ||
           algo == OSM_TOPK_SAFE_UNFUSED || algo == OSM_TOPK_ONLINE_UNFUSED ||
           algo == OSM_TOPK_VALUES;
}

int run_topk(const void* x, void* y, float* vals, int32_t* idx, int64_t N, int64_t V, int K,
             int dtype, int algo, int kernel, int64_t param, hipStream_t stream,
             bool noalloc = false) {
    size_t bytes = 0;
    if (!check_shape(N, V, dtype, &bytes)) return OSM_EINVAL;
    if (K < 1 || K > OSM_TOPK_KMAX || (int64_t)K > V) return OSM_EINVAL;
    if (!topk_algo_ok(algo)) return OSM_EINVAL;
    const bool unfused = algo == OSM_TOPK_SAFE_UNFUSED || algo == OSM_TOPK_ONLINE_UNFUSED;
    if (kernel == OSM_KERNEL_ROWS) {
        // the two-wavefront shape exists for the one-pass variant only
        const bool two_ok = algo == OSM_TOPK_ONLINE_FUSED;
        if (!(param == 64 || (param == 128 && two_ok) || param == 256)) return OSM_EINVAL;
    } else if (kernel == OSM_KERNEL_SPLIT) {
        if (param < 1 || param > kMaxDim || N * (param < V ? param : V) > kMaxDim)
            return OSM_EINVAL;
    } else if (kernel != OSM_KERNEL_AUTO) {
        return OSM_EINVAL;
    }
    if (N == 0) return OSM_OK;
    if (!x || !vals || !idx || (unfused && !y)) return OSM_EINVAL;
    const size_t es = elem_size(dtype);
    if (!aligned(x, es) || !aligned(vals, 4) || !aligned(idx, 4)) return OSM_EINVAL;
    const size_t ob = (size_t)N * (size_t)K * 4;
    if (overlaps(x, bytes, vals, ob) || overlaps(x, bytes, idx, ob) || overlaps(vals, ob, idx, ob))
        return OSM_EINVAL;
    if (unfused && (!aligned(y, es) || overlaps(y, bytes, x, bytes) ||
                    overlaps(y, bytes, vals, ob) || overlaps(y, bytes, idx, ob)))
        return OSM_EINVAL;
    DeviceState* ds = device_state(nullptr);
    if (!ds) return OSM_EHIP;
    switch (algo) {
        case OSM_TOPK_ONLINE_FUSED:
            return launch_topk_pass(x, vals, idx, N, V, K, dtype, osm::TK_ONLINE, kernel, param,
                                    ds, stream, noalloc);
        case OSM_TOPK_SAFE_FUSED:
            return launch_topk_pass(x, vals, idx, N, V, K, dtype, osm::TK_SAFE, kernel, param, ds,
                                    stream);
        case OSM_TOPK_VALUES:
            return launch_topk_pass(x, vals, idx, N, V, K, dtype, osm::TK_VALUES, kernel, param,
                                    ds, stream);
        default: {
            // softmax into y (Alg. 2 or Alg. 3), then a separate top-k over y
            const int mode = algo == OSM_TOPK_SAFE_UNFUSED ? OSM_SAFE : OSM_ONLINE;
            int st = run_softmax(x, y, N, V, dtype, mode, OSM_KERNEL_AUTO, 0, stream);
            if (st != OSM_OK) return st;
            return launch_topk_pass(y, vals, idx, N, V, K, dtype, osm::TK_VALUES, kernel, param,
                                    ds, stream);
        }
    }
}

// ---------------------------------------------------------------- projection
constexpr int64_t kProjTile = 128;     // tile edge of the largest grids
constexpr int64_t kProjMaxH = 1 << 20;  // 32-bit load offsets within a tile

// Arguments shared by the projection entry points; OSM_OK if valid.
int check_proj(const void* h, const void* w, int64_t N, int64_t H, int64_t V) {
    // the tile grid is one-dimensional: (N / 128) * (V / 128) workgroups < 2^31
    // (the tiles with shorter edges take a single strip of up to 64 rows)
    if (N < 0 || N > 65535 * kProjTile || V < 1 || V > kMaxDim || H < 8 || H > kProjMaxH ||
        H % 8 != 0 ||
        ((N + kProjTile - 1) / kProjTile) * ((V + kProjTile - 1) / kProjTile) > (kMaxDim - 7))
        return OSM_EINVAL;
    if (N == 0) return OSM_OK;
    if (!h || !w || !aligned(h, 16) || !aligned(w, 16)) return OSM_EINVAL;
    return OSM_OK;
}

int run_proj_logits(const void* h, const void* w, float* out, int64_t N, int64_t H, int64_t V,
                    hipStream_t stream) {
    int st = check_proj(h, w, N, H, V);
    if (st != OSM_OK || N == 0) return st;
    if (!out || !aligned(out, 4)) return OSM_EINVAL;
    const size_t ob = (size_t)N * (size_t)V * 4, hb = (size_t)N * (size_t)H * 2,
                 wb = (size_t)V * (size_t)H * 2;
    if (overlaps(out, ob, h, hb) || overlaps(out, ob, w, wb)) return OSM_EINVAL;
    DeviceState* ds = device_state(nullptr);
    if (!ds) return OSM_EHIP;
    return hip_status(osm::launch_proj_logits(h, w, out, N, H, V, ds->cus, stream));
}

int run_proj_topk(const void* h, const void* w, float* vals, int32_t* idx, int64_t N, int64_t H,
                  int64_t V, int K, hipStream_t stream) {
    int st = check_proj(h, w, N, H, V);
    if (st != OSM_OK) return st;
    if (K < 1 || K > OSM_PROJ_KMAX || (int64_t)K > V) return OSM_EINVAL;
    if (N == 0) return OSM_OK;
    if (!vals || !idx || !aligned(vals, 4) || !aligned(idx, 4)) return OSM_EINVAL;
    const size_t ob = (size_t)N * (size_t)K * 4, hb = (size_t)N * (size_t)H * 2,
                 wb = (size_t)V * (size_t)H * 2;
    if (overlaps(vals, ob, idx, ob) || overlaps(vals, ob, h, hb) || overlaps(vals, ob, w, wb) ||
        overlaps(idx, ob, h, hb) || overlaps(idx, ob, w, wb))
        return OSM_EINVAL;
    DeviceState* ds = device_state(nullptr);
    if (!ds) return OSM_EHIP;
    const osm::ProjTopkShape p = osm::proj_topk_shape(N, H, V, K, ds->cus);
    void* part = nullptr;
    bool temp = false;
    std::unique_lock<std::mutex> lk(ds->mu, std::defer_lock);  // held until the launches are in
    st = acquire_scratch(ds, lk, stream, osm::proj_topk_part_bytes(N, p.S, p.parts, K), &part,
                         &temp);
    if (st != OSM_OK) return st;
    hipError_t e =
        osm::launch_proj_topk(h, w, vals, idx, part, N, H, V, K, p, stream);
    hipError_t f = temp ? hipFreeAsync(part, stream) : hipSuccess;
    if (e != hipSuccess) return OSM_EHIP;
    return hip_status(f);
}

}  // namespace

extern "C" {

int softmax_fwd(const void* x, void* y, int64_t N, int64_t V, int dtype, int mode,
                hipStream_t stream) {
    return run_softmax(x, y, N, V, dtype, mode, OSM_KERNEL_AUTO, 0, stream);
}

int softmax_fwd_ex(const void* x, void* y, int64_t N, int64_t V, int dtype, int mode, int kernel,
                   int64_t param, hipStream_t stream) {
    return run_softmax(x, y, N, V, dtype, mode, kernel, param, stream);
}

int softmax_topk(const float* x, float* vals, int32_t* idx, int64_t N, int64_t V, int K,
                 hipStream_t stream) {
    return run_topk(x, nullptr, vals, idx, N, V, K, OSM_F32, OSM_TOPK_ONLINE_FUSED,
                    OSM_KERNEL_AUTO, 0, stream);
}

int softmax_topk_dt(const void* x, float* vals, int32_t* idx, int64_t N, int64_t V, int K,
                    int dtype, hipStream_t stream) {
    return run_topk(x, nullptr, vals, idx, N, V, K, dtype, OSM_TOPK_ONLINE_FUSED,
                    OSM_KERNEL_AUTO, 0, stream);
}

int softmax_topk_ex(const void* x, float* vals, int32_t* idx, int64_t N, int64_t V, int K,
                    int dtype, int kernel, int64_t param, hipStream_t stream) {
    return run_topk(x, nullptr, vals, idx, N, V, K, dtype, OSM_TOPK_ONLINE_FUSED, kernel, param,
                    stream);
}

int softmax_topk_ex_noalloc(const void* x, float* vals, int32_t* idx, int64_t N, int64_t V,
                            int K, int dtype, int kernel, int64_t param, hipStream_t stream) {
    return run_topk(x, nullptr, vals, idx, N, V, K, dtype, OSM_TOPK_ONLINE_FUSED, kernel, param,
                    stream, true);
}

int softmax_topk_algo(const void* x, void* y, float* vals, int32_t* idx, int64_t N, int64_t V,
                      int K, int dtype, int algo, int kernel, int64_t param, hipStream_t stream) {
    return run_topk(x, y, vals, idx, N, V, K, dtype, algo, kernel, param, stream);
}

int topk_fwd(const void* x, float* vals, int32_t* idx, int64_t N, int64_t V, int K, int dtype,
             hipStream_t stream) {
    return run_topk(x, nullptr, vals, idx, N, V, K, dtype, OSM_TOPK_VALUES, OSM_KERNEL_AUTO, 0,
                    stream);
}

int osm_topk_plan(int64_t N, int64_t V, int dtype, int K, int* kernel, int64_t* param) {
    size_t bytes = 0;
    if (!check_shape(N, V, dtype, &bytes)) return OSM_EINVAL;
    if (K < 1 || K > OSM_TOPK_KMAX || (int64_t)K > V) return OSM_EINVAL;
    if (!kernel || !param) return OSM_EINVAL;
    DeviceState* ds = device_state(nullptr);
    Plan p = choose_topk(N > 0 ? N : 1, V, dtype, K, ds ? ds->cus : 256);
    *kernel = p.kernel;
    *param = p.param;
    return OSM_OK;
}

int osm_ref_stream(int op, const void* x, void* y, int64_t bytes, hipStream_t stream) {
    if ((op != 0 && op != 1) || bytes < 0 || bytes % 16 != 0) return OSM_EINVAL;
    if (bytes == 0) return OSM_OK;
    if (!x || !y || !aligned(x, 16) || !aligned(y, 16)) return OSM_EINVAL;
    if (op == 1 && overlaps(x, (size_t)bytes, y, (size_t)bytes)) return OSM_EINVAL;
    DeviceState* ds = device_state(nullptr);
    if (!ds) return OSM_EHIP;
    return hip_status(osm::launch_ref_stream(op, x, y, bytes / 16, ds->cus, stream));
}

int proj_fwd(const void* h, const void* w, float* logits, int64_t N, int64_t H, int64_t V,
             hipStream_t stream) {
    return run_proj_logits(h, w, logits, N, H, V, stream);
}

int proj_softmax_topk(const void* h, const void* w, float* vals, int32_t* idx, int64_t N,
                      int64_t H, int64_t V, int K, hipStream_t stream) {
    return run_proj_topk(h, w, vals, idx, N, H, V, K, stream);
}

int osm_stream_release(hipStream_t stream) {
    DeviceState* ds = device_state(nullptr);
    if (!ds) return OSM_EHIP;
    std::lock_guard<std::mutex> guard(ds->mu);
    const hipError_t e = release_slot(ds->slots, &ds->nslots, stream);
    const hipError_t f = release_slot(ds->cslots, &ds->ncslots, stream);
    if (e != hipSuccess || f != hipSuccess) {
        (void)hipGetLastError();
        return OSM_EHIP;
    }
    return OSM_OK;
}

int osm_plan(int64_t N, int64_t V, int dtype, int mode, int* kernel, int64_t* param) {
    size_t bytes = 0;
    if (!check_shape(N, V, dtype, &bytes)) return OSM_EINVAL;
    if (mode != OSM_NAIVE && mode != OSM_SAFE && mode != OSM_ONLINE && mode != OSM_RESIDENT)
        return OSM_EINVAL;
    if (!kernel || !param) return OSM_EINVAL;
    if (mode == OSM_RESIDENT) {
        ResShape rs;
        if (!choose_resident(V, dtype, 0, &rs)) return OSM_EUNSUPPORTED;
        *kernel = OSM_KERNEL_ROWS;
        *param = rs.block;
        return OSM_OK;
    }
    DeviceState* ds = device_state(nullptr);
    Plan p = choose(N > 0 ? N : 1, V, dtype, ds ? ds->cus : 256);
    *kernel = p.kernel;
    *param = p.param;
    return OSM_OK;
}

const char* osm_status_string(int status) {
    switch (status) {
        case OSM_OK: return "success";
        case OSM_EINVAL: return "invalid argument";
        case OSM_EUNSUPPORTED: return "unsupported configuration";
        case OSM_EHIP: return "HIP error while enqueuing work";
        case OSM_ENOMEM: return "scratch allocation failed";
        case OSM_ESCRATCH: return "needs more than the fixed no-allocation scratch";
        default: return "unknown status";
    }
}

}  // extern "C"
