// Rest-of-layer compute window: what a transformer layer runs on the miss
// tokens besides the attention (the C_l of eq. (3); every layer has the same
// projections and feed-forward network, Section 3.6).  Four bf16 GEMMs with
// fp32 accumulation (O, gate|up, down, next layer's QKV): on few rows the
// library's own kernels, which stream the weights, else rocBLAS, with the SiLU
// gating as a kernel of its own.
#include <rocblas/rocblas.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <utility>

#include "common.hpp"
#include "split_workspace.hpp"

namespace oc {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x8 __attribute__((ext_vector_type(8)));

// act[t][c] = silu(gu[t][c]) * gu[t][F + c], 8 columns per thread, fp32 math,
// rounded to bf16 (nearest even).
__global__ __launch_bounds__(256) void silu_mul_kernel(const uint16_t *gu, uint16_t *act, int64_t F8, int64_t n) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n) return;
    const int64_t t = e / F8, c = e - t * F8;
    const uint16_t *grow = gu + t * 16 * F8 + c * 8;
    const u32x4 gb = *reinterpret_cast<const u32x4 *>(grow);
    const u32x4 ub = *reinterpret_cast<const u32x4 *>(grow + 8 * F8);
    f32x8 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float g0 = __uint_as_float(gb[i] << 16), g1 = __uint_as_float(gb[i] & 0xFFFF0000u);
        const float u0 = __uint_as_float(ub[i] << 16), u1 = __uint_as_float(ub[i] & 0xFFFF0000u);
        r[2 * i] = g0 / (1.f + __expf(-g0)) * u0;
        r[2 * i + 1] = g1 / (1.f + __expf(-g1)) * u1;
    }
    *reinterpret_cast<u32x4 *>(act + t * 8 * F8 + c * 8) = __builtin_bit_cast(u32x4, __builtin_convertvector(r, bf16x8));
}

// Per (device, stream): a rocBLAS handle and the few-row GEMM's workspaces for
// split partials.  The first eager call on the stream makes the handle and the
// eager calls' workspace, whichever of them its row count needs; they live until
// the process ends, or until forget_blas_stream() for streams the library owns.
// hipStreamPerThread is one handle for a queue per host thread, whose calls may
// overlap: it gets no workspace, and products that would need one go to the
// GEMM library.
struct StreamState {
    rocblas_handle handle = nullptr;
    SplitWorkspace ws;
};
static std::mutex g_blas_mu;
static std::map<std::pair<int, hipStream_t>, StreamState> g_blas;
static int g_workspaces = 0;

// In relaxed mode: a plain allocation would end this stream's capture, and fail
// beside another thread's.
static void *allocate_workspace() {
    void *p = nullptr;
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    if (hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess) {
        if (hipMalloc(&p, GEMM_WORKSPACE_BYTES) != hipSuccess) p = nullptr;
        (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
    if (!p) (void)hipGetLastError();
    return p;
}

// the stream's handle, and where the call's split partials go
struct CallState {
    rocblas_handle handle = nullptr;
    SplitWorkspace *ws = nullptr;           // NULL: nowhere
    bool capturing = false;
    unsigned long long capture = 0;

    void *workspace() const {
        if (!ws) return nullptr;
        return capturing ? ws->get_captured(g_workspaces, capture, allocate_workspace)
                         : ws->get(g_workspaces, allocate_workspace);
    }
};

static int stream_state(hipStream_t s, CallState *out) {
    int dev = 0;
    OC_HIP(hipGetDevice(&dev));
    StreamState *st = &g_blas[std::make_pair(dev, s)];
    if (!st->handle && rocblas_create_handle(&st->handle) != rocblas_status_success) {
        st->handle = nullptr;
        return fail(OC_EHIP, "rocblas_create_handle failed");
    }
    if (rocblas_set_stream(st->handle, s) != rocblas_status_success) return fail(OC_EHIP, "rocblas_set_stream failed");
    out->handle = st->handle;
    if (s == hipStreamPerThread) return OC_OK;
    out->ws = &st->ws;
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamGetCaptureInfo(s, &status, &out->capture) != hipSuccess) {
        (void)hipGetLastError();      // the null stream while another captures: the launches report it
        out->ws = nullptr;
    } else if (status != hipStreamCaptureStatusNone) {
        out->capturing = true;
    } else {
        (void)out->workspace();
    }
    return OC_OK;
}

void forget_blas_stream(hipStream_t s) {
    std::lock_guard<std::mutex> g(g_blas_mu);
    for (auto it = g_blas.begin(); it != g_blas.end();) {
        if (it->first.second == s) {
            if (it->second.handle) rocblas_destroy_handle(it->second.handle);
            it->second.ws.give_back(g_workspaces, [](void *p) { (void)hipFree(p); });
            it = g_blas.erase(it);
        } else {
            ++it;
        }
    }
}

// Y[M][N] = X[M][K] . W[K][N], all row-major bf16: column-major rocBLAS sees
// Y^T = W^T . X^T with no transposes.
static int gemm(rocblas_handle h, const uint16_t *X, const uint16_t *W, uint16_t *Y, int64_t M, int64_t K, int64_t N) {
    const float alpha = 1.f, beta = 0.f;
    rocblas_status st = rocblas_gemm_ex(h, rocblas_operation_none, rocblas_operation_none, (rocblas_int)N,
                                        (rocblas_int)M, (rocblas_int)K, &alpha, W, rocblas_datatype_bf16_r,
                                        (rocblas_int)N, X, rocblas_datatype_bf16_r, (rocblas_int)K, &beta, Y,
                                        rocblas_datatype_bf16_r, (rocblas_int)N, Y, rocblas_datatype_bf16_r,
                                        (rocblas_int)N, rocblas_datatype_f32_r, rocblas_gemm_algo_standard, 0, 0);
    if (st != rocblas_status_success)
        return fail(OC_EHIP, std::string("rocblas_gemm_ex: ") + rocblas_status_to_string(st));
    return OC_OK;
}

// Rows are independent, so long inputs go through the chain in row blocks
// that keep every matrix handed to the GEMM library under 1 GiB.
int launch_rest_of_layer(const LayerArgs &a, hipStream_t s) {
    if (a.T == 0) return OC_OK;
    std::lock_guard<std::mutex> g(g_blas_mu);
    CallState call;
    int rc = stream_state(s, &call);
    if (rc) return rc;
    const int64_t widest = std::max(std::max(2 * a.F, a.H), a.NQKV);
    const int64_t rb = std::max<int64_t>(1, (INT64_C(1) << 29) / widest);
    // one product of the chain on m rows; with `act`, the gating as well
    auto product = [&](const uint16_t *x, const uint16_t *w, uint16_t *y, uint16_t *act, int64_t m, int64_t K,
                       int64_t N) -> int {
        // the fused gating writes act while x is still being read: where a
        // caller lets act take x's memory (o is done with after this product),
        // the gating follows the product
        const bool apart = !act || act + m * (N / 2) <= x || x + m * K <= act;
        if (apart && gemm_rows_applies(m, K, N, true)) {
            void *const ws = gemm_rows_splits(m, K, N) > 1 ? call.workspace() : nullptr;
            if (gemm_rows_applies(m, K, N, ws != nullptr)) {
                OC_HIP(launch_gemm_rows(x, w, y, act, ws, m, K, N, s));
                return OC_OK;
            }
        }
        const int r = gemm(call.handle, x, w, y, m, K, N);
        if (r) return r;
        if (act) {
            const int64_t n = m * (N / 16);
            hipLaunchKernelGGL(silu_mul_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, y, act,
                               (int64_t)(N / 16), n);
            OC_HIP(hipGetLastError());
        }
        return OC_OK;
    };
    for (int64_t r0 = 0; r0 < a.T; r0 += rb) {
        const int64_t m = std::min(rb, a.T - r0);
        const uint16_t *x = a.attn_out + r0 * a.H;
        uint16_t *o = a.o + r0 * a.H, *gu = a.gu + r0 * 2 * a.F, *act = a.act + r0 * a.F;
        uint16_t *hh = a.h + r0 * a.H, *qkv = a.qkv + r0 * a.NQKV;
        if ((rc = product(x, a.w_o, o, nullptr, m, a.H, a.H))) return rc;
        if ((rc = product(o, a.w_gu, gu, act, m, a.H, 2 * a.F))) return rc;
        if ((rc = product(act, a.w_down, hh, nullptr, m, a.F, a.H))) return rc;
        if ((rc = product(hh, a.w_qkv, qkv, nullptr, m, a.H, a.NQKV))) return rc;
    }
    return OC_OK;
}

LayerArgs layer_args(const oc_layout &l, const oc_layer_weights &w, int32_t layer, const void *attn_out,
                     int64_t tokens, const oc_layer_buffers &b) {
    LayerArgs a{};
    a.T = tokens;
    a.H = (int64_t)l.num_q_heads * l.head_dim;
    a.F = w.ffn_dim;
    a.NQKV = (int64_t)(l.num_q_heads + 2 * l.num_kv_heads) * l.head_dim;
    a.attn_out = static_cast<const uint16_t *>(attn_out);
    a.w_o = static_cast<const uint16_t *>(w.w_o) + layer * a.H * a.H;
    a.w_gu = static_cast<const uint16_t *>(w.w_gate_up) + layer * a.H * 2 * a.F;
    a.w_down = static_cast<const uint16_t *>(w.w_down) + layer * a.F * a.H;
    a.w_qkv = static_cast<const uint16_t *>(w.w_qkv) + layer * a.H * a.NQKV;
    a.o = static_cast<uint16_t *>(b.o);
    a.gu = static_cast<uint16_t *>(b.gate_up);
    a.act = static_cast<uint16_t *>(b.act);
    a.h = static_cast<uint16_t *>(b.h);
    a.qkv = static_cast<uint16_t *>(b.qkv);
    return a;
}

int check_layer_weights(const oc_layout &l, const oc_layer_weights *w) {
    if (!w) return fail(OC_EINVAL, "layer weights are NULL");
    if (w->ffn_dim < 8 || w->ffn_dim % 8) return fail(OC_ESHAPE, "ffn_dim must be a positive multiple of 8");
    if (!w->w_o || !w->w_gate_up || !w->w_down || !w->w_qkv) return fail(OC_EINVAL, "NULL layer weight");
    if (!aligned(w->w_o, 16) || !aligned(w->w_gate_up, 16) || !aligned(w->w_down, 16) || !aligned(w->w_qkv, 16))
        return fail(OC_EALIGN, "layer weights must be 16-byte aligned");
    const int64_t H = (int64_t)l.num_q_heads * l.head_dim;
    if (H * 2 * w->ffn_dim > INT32_MAX || (int64_t)(l.num_q_heads + 2 * l.num_kv_heads) * l.head_dim > INT32_MAX)
        return fail(OC_ERANGE, "layer too wide");
    return OC_OK;
}

int check_layer_buffers(const oc_layer_buffers *b) {
    if (!b) return fail(OC_EINVAL, "layer buffers are NULL");
    if (!b->o || !b->gate_up || !b->act || !b->h || !b->qkv) return fail(OC_EINVAL, "NULL layer buffer");
    if (!aligned(b->o, 16) || !aligned(b->gate_up, 16) || !aligned(b->act, 16) || !aligned(b->h, 16) ||
        !aligned(b->qkv, 16))
        return fail(OC_EALIGN, "layer buffers must be 16-byte aligned");
    return OC_OK;
}

size_t layer_buffer_bytes(const oc_layout &l, int32_t ffn_dim, int64_t tokens, size_t off[5]) {
    const int64_t H = (int64_t)l.num_q_heads * l.head_dim;
    const int64_t NQKV = (int64_t)(l.num_q_heads + 2 * l.num_kv_heads) * l.head_dim;
    const int64_t cols[5] = {H, 2LL * ffn_dim, ffn_dim, H, NQKV};
    size_t total = 0;
    for (int i = 0; i < 5; ++i) {
        off[i] = total;
        total += ((size_t)tokens * cols[i] * 2 + 255) / 256 * 256;
    }
    return total;
}

}  // namespace oc
