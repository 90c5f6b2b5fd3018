// Layer ingest: unpack one layer payload (concatenated KV_L2TD layer slices
// of the matched chunk objects, Section 3.3) and scatter it into the paged
// pool through the block table.
//
// Both sides keep one head's d-element row per token, so the scatter is a
// copy of 16-byte pieces with remapped addresses: the payload holds the rows
// of a chunk token-major ([K|V][token][head][dim]), the pool holds them per
// (page, head) block ([slot][dim]).  Two launch shapes:
//  - alone on the GPU (the single-layer entry point, the first layer of a
//    run): one piece per thread in payload order, so every wavefront reads
//    1 KiB of the payload contiguously and writes four 256-byte rows, and
//    many short wavefronts keep the most bytes in flight;
//  - beside the attention kernel of an earlier layer, where one ingest
//    wavefront per SIMD runs at the lowest issue priority: a thread takes
//    8 slots x one 16-byte column of one (page, head) block and moves its K
//    rows, then its V rows (8 loads in flight, one page lookup per 256 bytes
//    moved, a shift decode of the thread's block and column).
// The gather (pool -> payload or whole chunk objects, the offload direction)
// numbers pieces the same way, reversed.  The suffix append writes the new
// tokens' K/V rows behind the prefix through the same block table.
#include "common.hpp"

namespace oc {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;

// 8 slots x one 16-byte column of one (page, head) block, K then V.  With
// POW2 (d/8, page size, KV heads and a chunk size of at least 8 all powers of
// two) the decode is shifts and masks and the 8 tokens sit in one chunk.
// Every group of 8 slots lies wholly inside or wholly past the prefix when
// the chunk size is a multiple of 8; only other chunk sizes reach the
// per-token bounds checks.
template <bool POW2>
__global__ __launch_bounds__(kThreads, 8) void kv_ingest_rows_kernel(IngestArgs a, int64_t n_rows8) {
    const int64_t u = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (u >= n_rows8) return;
    const int d = a.d, G = a.G, nkv = a.n_kv;
    int c, s8, h;
    int64_t q, T0;
    if (POW2) {
        const int lg_s8 = a.lg_ps - 3;                   // page_size / 8 groups per page
        c = (int)(u & (a.d8 - 1));
        s8 = (int)((u >> a.lg_d8) & ((1 << lg_s8) - 1));
        h = (int)((u >> (a.lg_d8 + lg_s8)) & (nkv - 1));
        q = u >> (a.lg_d8 + lg_s8 + a.lg_nkv);
        T0 = (q << a.lg_ps) + s8 * 8;
    } else {
        c = (int)(u % a.d8);
        int64_t rest = u / a.d8;
        s8 = (int)(rest % (a.Ps / 8));
        rest /= a.Ps / 8;
        h = (int)(rest % nkv);
        q = rest / nkv;
        T0 = q * a.Ps + s8 * 8;                          // first token of the 8
    }
    const int64_t left = a.num_tokens - T0;
    if (left <= 0) return;                               // slots past the prefix
    const int64_t D = (int64_t)nkv * d;
    const int64_t page = a.pages[q];
    uint16_t *kdst = a.pool_k + ((page * nkv + h) * a.Ps + s8 * 8) * (int64_t)d + c * 8;
    const int64_t col = (int64_t)h * d + c * 8;
    const int64_t vstep = (int64_t)G * D;                // K row -> V row of a token
    // non-temporal: the payload is read once and the pool rows are not read
    // again until that layer's attention, so keep both out of the L2 that the
    // running attention uses for its K/V tiles
    u32x4 r[8];
    if (POW2 || (G % 8 == 0)) {
        // the 8 tokens sit in one chunk, one payload row apart, all inside
        // the prefix (it is a whole number of chunks)
        const int64_t j = POW2 ? T0 >> a.lg_g : T0 / G;
        const uint16_t *src = a.staging + j * a.chunk_stride + (T0 - j * G) * D + col;
#pragma unroll
        for (int kv = 0; kv < 2; ++kv) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                r[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src + kv * vstep + i * D));
#pragma unroll
            for (int i = 0; i < 8; ++i)
                __builtin_nontemporal_store(r[i], reinterpret_cast<u32x4 *>(kdst + kv * a.region + i * d));
        }
        return;
    }
    // chunk sizes that are not a multiple of 8: the 8 tokens may span two
    // chunks and run past the prefix
    const int valid = left < 8 ? (int)left : 8;
    int64_t src[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int64_t T = T0 + i, j = T / G;
        src[i] = j * a.chunk_stride + (T - j * G) * D + col;
    }
#pragma unroll
    for (int kv = 0; kv < 2; ++kv) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (i < valid)
                r[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(a.staging + src[i] + kv * vstep));
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (i < valid) __builtin_nontemporal_store(r[i], reinterpret_cast<u32x4 *>(kdst + kv * a.region + i * d));
    }
}

// Piece e of a payload numbered in payload order ([chunk][K|V][token][head]
// [16-byte column]; from chunk blockIdx.z on) -> its element offsets in the
// staging (from `staging`) and in the pool (from `pool_k`), both including the
// layer step of blockIdx.y.  With POW2 every divisor (d/8, KV heads, chunk size, page size)
// is a power of two and the decode is shifts and masks.
template <bool POW2>
__device__ inline void src_order_piece(const IngestArgs &a, int64_t e, int64_t &stage, int64_t &pool) {
    const int64_t slice_pieces = 2LL * a.G * a.n_kv * a.d8;   // 16-byte pieces per chunk slice
    int c, h, t, kv;
    int64_t j;
    if (POW2) {
        c = (int)(e & (a.d8 - 1));
        h = (int)((e >> a.lg_d8) & (a.n_kv - 1));
        t = (int)((e >> (a.lg_d8 + a.lg_nkv)) & (a.G - 1));
        kv = (int)((e >> (a.lg_d8 + a.lg_nkv + a.lg_g)) & 1);
        j = e >> (a.lg_d8 + a.lg_nkv + a.lg_g + 1);
    } else {
        int64_t r = e / a.d8;
        c = (int)(e - r * a.d8);
        int64_t r2 = r / a.n_kv;
        h = (int)(r - r2 * a.n_kv);
        int64_t r3 = r2 / a.G;
        t = (int)(r2 - r3 * a.G);
        j = r3 >> 1;
        kv = (int)(r3 & 1);
    }
    const int64_t jz = j + blockIdx.z;
    const int64_t T = a.token0 + jz * a.G + t;
    int64_t q, slot;
    if (POW2) {
        q = T >> a.lg_ps;
        slot = T & (a.Ps - 1);
    } else {
        q = T / a.Ps;
        slot = T - q * a.Ps;
    }
    const int64_t page = a.pages[q];
    stage = blockIdx.y * a.layer_step_staging + jz * a.chunk_stride + (e - j * slice_pieces) * 8;
    pool = blockIdx.y * a.layer_step_pool + kv * a.region + ((page * a.n_kv + h) * a.Ps + slot) * (int64_t)a.d +
           c * 8;
}

// Ingest, one 16-byte piece per thread in payload order: every wavefront
// reads 1 KiB of the payload contiguously and writes 256-byte rows into the
// (page, head) blocks.  Many short wavefronts keep the most bytes in flight.
// Every byte is read once and written once, so both sides bypass the L2's
// normal retention (non-temporal): about 2.5 % faster alone than plain
// accesses at the 8b-64k layer.
// For whole chunk objects blockIdx.y is the layer.
template <bool POW2>
__global__ __launch_bounds__(kThreads) void kv_ingest_src_kernel(IngestArgs a, int64_t n_pieces) {
    const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (e >= n_pieces) return;
    int64_t stage, pool;
    src_order_piece<POW2>(a, e, stage, pool);
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(a.staging + stage));
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(a.pool_k + pool));
}

// Gather (pool -> layer payload or whole chunk objects, the offload
// direction): the same numbering, so every wavefront writes 1 KiB of the
// output contiguously and reads 256-byte pool rows; non-temporal on both
// sides like the ingest (about 7 % faster than plain accesses over the
// chunk objects of the 64K prefix).
template <bool POW2>
__global__ __launch_bounds__(kThreads) void kv_gather_src_kernel(IngestArgs a, uint16_t *out, int64_t n_pieces) {
    const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (e >= n_pieces) return;
    int64_t stage, pool;
    src_order_piece<POW2>(a, e, stage, pool);
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(a.pool_k + pool));
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(out + stage));
}

// Suffix append: token i of k_new / v_new ([T_s][n_kv][d]; blockIdx.y picks
// K or V) goes to logical position token0 + i through the block table.
// Piece e of the 16-byte pieces of one tensor; with POW2 (d/8, KV heads and
// page size powers of two) the decode is shifts and masks.
template <bool POW2, class Args>
__device__ inline void append_piece(const Args &a, uint32_t e, int kv) {
    uint32_t c, h, i;
    int64_t q, slot;
    if (POW2) {
        c = e & (a.d8 - 1);
        h = (e >> a.lg_d8) & (a.n_kv - 1);
        i = e >> (a.lg_d8 + a.lg_nkv);
        const int64_t T = a.token0 + i;
        q = T >> a.lg_ps;
        slot = T & (a.Ps - 1);
    } else {
        const uint32_t r = e / (uint32_t)a.d8;
        c = e - r * a.d8;
        i = r / (uint32_t)a.n_kv;
        h = r - i * a.n_kv;
        const int64_t T = a.token0 + i;
        q = T / a.Ps;
        slot = T - q * a.Ps;
    }
    const uint16_t *src = (kv ? a.v_new : a.k_new) + (int64_t)e * 8;
    const u32x4 v = *reinterpret_cast<const u32x4 *>(src);
    const int64_t page = a.pages[q];
    uint16_t *dst = a.pool_k + kv * a.region + ((page * a.n_kv + h) * a.Ps + slot) * (int64_t)a.d + c * 8;
    *reinterpret_cast<u32x4 *>(dst) = v;
}

// One layer's suffix is a few MiB, so this is launch and latency bound (4 MiB
// read and written at 512 tokens: 3.0 us per launch back to back, 3.4 with
// 64-bit divisions in the decode).
template <bool POW2>
__global__ __launch_bounds__(kThreads) void kv_append_kernel(AppendArgs a, uint32_t n_pieces) {
    const uint32_t e = blockIdx.x * kThreads + threadIdx.x;
    if (e < n_pieces) append_piece<POW2>(a, e, (int)blockIdx.y);
}

// The appends of several requests to one layer in one launch: a workgroup
// belongs to the last request whose first workgroup it has reached.
struct AppendBatch {
    int32_t n;
    uint32_t first_wg[MAX_APPEND_BATCH], n_pieces[MAX_APPEND_BATCH];
    AppendArgs req[MAX_APPEND_BATCH];
};
template <bool POW2>
__global__ __launch_bounds__(kThreads) void kv_append_batch_kernel(AppendBatch batch) {
    // parameters straight from the kernel-argument segment: indexing the
    // by-value copy would place it in scratch memory
    typedef const __attribute__((address_space(4))) AppendBatch *batch_ptr;
    const batch_ptr bp = (batch_ptr)__builtin_amdgcn_kernarg_segment_ptr();
    int r = 0;
    for (int i = 1; i < bp->n; ++i) r += blockIdx.x >= bp->first_wg[i];
    const uint32_t e = (blockIdx.x - bp->first_wg[r]) * kThreads + threadIdx.x;
    if (e < bp->n_pieces[r]) append_piece<POW2>(bp->req[r], e, (int)blockIdx.y);
}

static bool pow2(int64_t x) { return x > 0 && (x & (x - 1)) == 0; }
static int lg(int64_t x) {
    int r = 0;
    while ((1LL << r) < x) ++r;
    return r;
}

// Fills the derived fields and the defaults of a single layer payload;
// returns whether the shift decode applies.
static bool prepare(IngestArgs &a) {
    if (a.chunk_stride == 0) a.chunk_stride = 2LL * a.G * a.n_kv * a.d;
    if (a.n_layers == 0) a.n_layers = 1;
    a.d8 = a.d / 8;
    a.region = (int64_t)(a.pool_v - a.pool_k);
    const bool p2 = pow2(a.d8) && pow2(a.Ps) && pow2(a.n_kv) && pow2(a.G);
    a.lg_d8 = lg(a.d8);
    a.lg_ps = lg(a.Ps);
    a.lg_nkv = lg(a.n_kv);
    a.lg_g = lg(a.G);
    return p2;
}

// An ingest workgroup next to the attention reserves LDS (the kernel itself uses
// none) so that one of them, one wavefront per SIMD, shares a CU with each
// attention workgroup: more than half of what that leaves free, in the units
// that LDS is handed out in, and never more than that, which would keep every
// ingest waiting for CUs the attention does not hold.
size_t ingest_reservation(size_t beside_lds) {
    const size_t held = (beside_lds + LDS_GRANULE - 1) / LDS_GRANULE, all = CU_LDS_BYTES / LDS_GRANULE;
    return beside_lds > 0 && held < all ? ((all - held) / 2 + 1) * LDS_GRANULE : 0;
}

int ingest_registers(bool pow2) {
    hipFuncAttributes a{};
    const void *f = reinterpret_cast<const void *>(pow2 ? &kv_ingest_rows_kernel<true> : &kv_ingest_rows_kernel<false>);
    return hipFuncGetAttributes(&a, f) == hipSuccess ? a.numRegs : -1;
}

hipError_t launch_ingest(IngestArgs a, int64_t n_pages_used, hipStream_t s, size_t beside_lds) {
    if (n_pages_used == 0) return hipSuccess;
    const bool p2 = prepare(a);
    if (beside_lds > 0 && a.token0 == 0) {
        const int64_t n = n_pages_used * a.n_kv * (a.Ps / 8) * a.d8;
        const dim3 grid((unsigned)((n + kThreads - 1) / kThreads));
        const size_t lds = ingest_reservation(beside_lds);
        if (p2 && a.Ps >= 8 && a.G >= 8)
            hipLaunchKernelGGL(kv_ingest_rows_kernel<true>, grid, dim3(kThreads), lds, s, a, n);
        else
            hipLaunchKernelGGL(kv_ingest_rows_kernel<false>, grid, dim3(kThreads), lds, s, a, n);
    } else {
        const int64_t n = a.num_tokens * 2 * a.n_kv * a.d8;   // 16-byte pieces of the payload
        const dim3 grid((unsigned)((n + kThreads - 1) / kThreads));
        if (p2) hipLaunchKernelGGL(kv_ingest_src_kernel<true>, grid, dim3(kThreads), 0, s, a, n);
        else hipLaunchKernelGGL(kv_ingest_src_kernel<false>, grid, dim3(kThreads), 0, s, a, n);
    }
    return hipGetLastError();
}

// Grid over `pieces` 16-byte pieces of one layer.  Whole chunk objects go
// object by object, so that the workgroups running at a time read (or write)
// one stretch of memory instead of one layer's slice of many objects (64
// objects of 64 tokens, 32 layers: ingest 5.25 -> 5.64 TB/s, a 64 MiB gather
// 24.4 -> 22.4 us); `n` is then the pieces of one slice.  Short slices that
// are no whole number of workgroups keep one run of pieces per layer.
static dim3 payload_grid(const IngestArgs &a, int64_t &n) {
    const int64_t chunks = a.num_tokens / a.G, slice = 2LL * a.G * a.n_kv * a.d8;
    if (a.n_layers > 1 && chunks <= 65535 && (slice % kThreads == 0 || slice >= 16 * kThreads)) {
        n = slice;
        return dim3((unsigned)((n + kThreads - 1) / kThreads), (unsigned)a.n_layers, (unsigned)chunks);
    }
    n = a.num_tokens * 2 * a.n_kv * a.d8;
    return dim3((unsigned)((n + kThreads - 1) / kThreads), (unsigned)a.n_layers);
}

hipError_t launch_chunks_ingest(IngestArgs a, hipStream_t s) {
    if (a.num_tokens == 0) return hipSuccess;
    const bool p2 = prepare(a);
    int64_t n;
    const dim3 grid = payload_grid(a, n);
    if (p2) hipLaunchKernelGGL(kv_ingest_src_kernel<true>, grid, dim3(kThreads), 0, s, a, n);
    else hipLaunchKernelGGL(kv_ingest_src_kernel<false>, grid, dim3(kThreads), 0, s, a, n);
    return hipGetLastError();
}

hipError_t launch_gather(IngestArgs a, uint16_t *out, hipStream_t s) {
    if (a.num_tokens == 0) return hipSuccess;
    const bool p2 = prepare(a);
    int64_t n;
    const dim3 grid = payload_grid(a, n);
    if (p2) hipLaunchKernelGGL(kv_gather_src_kernel<true>, grid, dim3(kThreads), 0, s, a, out, n);
    else hipLaunchKernelGGL(kv_gather_src_kernel<false>, grid, dim3(kThreads), 0, s, a, out, n);
    return hipGetLastError();
}

// Fills the derived fields; returns whether the shift decode applies.
static bool prepare(AppendArgs &a) {
    a.d8 = a.d / 8;
    a.region = (int64_t)(a.pool_v - a.pool_k);
    a.lg_d8 = lg(a.d8);
    a.lg_nkv = lg(a.n_kv);
    a.lg_ps = lg(a.Ps);
    return pow2(a.d8) && pow2(a.n_kv) && pow2(a.Ps);
}

// 16-byte pieces of K (and of V); the callers' checks keep it below 2^32
static uint32_t append_pieces(const AppendArgs &a) { return (uint32_t)(a.num_tokens * a.n_kv * a.d8); }

hipError_t launch_append(AppendArgs a, hipStream_t s) {
    if (a.num_tokens == 0) return hipSuccess;
    const bool p2 = prepare(a);
    const uint32_t n = append_pieces(a);
    const dim3 grid((unsigned)(((int64_t)n + kThreads - 1) / kThreads), 2);
    if (p2) hipLaunchKernelGGL(kv_append_kernel<true>, grid, dim3(kThreads), 0, s, a, n);
    else hipLaunchKernelGGL(kv_append_kernel<false>, grid, dim3(kThreads), 0, s, a, n);
    return hipGetLastError();
}

hipError_t launch_append_batch(const AppendArgs *a, int n, hipStream_t s) {
    if (n < 1 || n > MAX_APPEND_BATCH) return hipErrorInvalidValue;
    AppendBatch batch{};
    bool p2 = true;
    int64_t grid = 0;
    for (int i = 0; i < n; ++i) {
        if (a[i].num_tokens == 0) continue;
        AppendArgs &r = batch.req[batch.n];
        r = a[i];
        p2 = prepare(r) && p2;
        batch.first_wg[batch.n] = (uint32_t)grid;
        batch.n_pieces[batch.n] = append_pieces(r);
        grid += ((int64_t)batch.n_pieces[batch.n] + kThreads - 1) / kThreads;
        ++batch.n;
    }
    if (grid == 0) return hipSuccess;
    if (grid * kThreads > OC_MAX_GRID_ITEMS) return hipErrorInvalidConfiguration;
    if (p2) hipLaunchKernelGGL(kv_append_batch_kernel<true>, dim3((unsigned)grid, 2), dim3(kThreads), 0, s, batch);
    else hipLaunchKernelGGL(kv_append_batch_kernel<false>, dim3((unsigned)grid, 2), dim3(kThreads), 0, s, batch);
    return hipGetLastError();
}

}  // namespace oc
