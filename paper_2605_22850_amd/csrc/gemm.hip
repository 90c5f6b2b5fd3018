// Y[M][N] = X[M][K] . W[K][N] for few rows (bf16 in and out, fp32
// accumulation): the projections and the feed-forward network of the layer
// around the attention, on the miss tokens only.
//
// With so few rows these products stream the weights: what bounds them is
// that every byte of W is read once, at the HBM rate, by enough workgroups.
// A workgroup owns 32 to 256 rows x 128 columns and one contiguous range of
// K.  Steps of 64 k are copied straight into LDS (global -> LDS, NS steps in
// the ring): the W rows as they lie in memory ([k][n], transposed by the
// operand reads as the attention does with V), the X rows XOR-swizzled like
// the attention's K.  Where N / 128 column tiles leave CUs idle, K is split
// over workgroups (down: 32 tiles but 14336 k); the partial tiles are written
// in accumulator order, one coalesced 1 KiB store per instruction, and
// gemm_reduce_kernel adds them in split order.  The SiLU gating is part of
// the gate|up product's epilogue: its tiles pair 16 gate columns with the same
// 16 up columns, so one lane ends up with both.
//
// Up to 32 rows W streams at 4.9-5.1 TB/s (gate|up: 235 MB in 46.5-48 us).
// With more rows the copies of X through the same path add to it (52 us at
// 64 rows, 62 at 128): more steps in the ring, other wavefront grids, 8
// wavefronts and different k orders per workgroup changed that by 3 % at
// most, and the copies alone, without any MFMA, take 61.8 us at 128 rows.
#include <algorithm>

#include "mfma_tiles.hpp"

namespace oc {

constexpr int BK = 64;              // k per step
constexpr int GEMM_BN = 128;        // columns per workgroup
constexpr int GEMM_WGS = 256;       // workgroups to aim at, one per CU

struct GemmParams {
    const uint16_t *x, *w;
    uint16_t *y;
    uint16_t *act;         // GLU: silu(gate) * up, [M][N/2]
    float *part;           // split partials, [m tile][n tile][split][BM*BN]
    int32_t M, N, K;
    int32_t m_tiles, n_tiles, n_split, steps_per_split;
};

// Wavefront grid of a workgroup: WM x WN wavefronts, each with MW x NW tiles
// of 32 rows x 32 columns.
template <int WM, int WN, int MW, int NW>
struct GemmShape {
    static constexpr int WAVES = WM * WN, THREADS = WAVES * 64;
    static constexpr int BM = 32 * MW * WM, BN = 32 * NW * WN;
    static constexpr int W_STEP = BK * BN, X_STEP = BM * BK;             // elements per step
    static constexpr int STEP = W_STEP + X_STEP;
    static constexpr int W_CPW = W_STEP * 2 / 1024 / WAVES;              // 1 KiB copies per wavefront
    static constexpr int X_CPW = X_STEP * 2 / 1024 / WAVES;
    static_assert(W_CPW * WAVES * 512 == W_STEP && X_CPW * WAVES * 512 == X_STEP, "copies do not cover the step");
    static constexpr int TILE = BM * BN;                                 // floats of one partial tile
};

// First of four consecutive columns that accumulator group vq of tile `et` of
// a BN-column tile holds.  GLU tiles hold BN/2 gate columns and the same BN/2
// up columns, 16 of each per 32-column tile: vq 0, 1 gate, 2, 3 up.
__device__ inline int tile_col(int et, int vq, int half) { return et * 32 + vq * 8 + half * 4; }

__device__ inline float silu_mul(float g, float u) { return g / (1.f + __expf(-g)) * u; }

// Store the gate and up columns and the gated product of one lane's pair.
__device__ inline void store_glu(const GemmParams &p, int m, int col, f32x4 g, f32x4 u) {
    const bf16x4 gb = __builtin_convertvector(g, bf16x4), ub = __builtin_convertvector(u, bf16x4);
    const int64_t F = p.N / 2;
    uint16_t *row = p.y + (int64_t)m * p.N + col;
    *reinterpret_cast<bf16x4 *>(row) = gb;
    *reinterpret_cast<bf16x4 *>(row + F) = ub;
    f32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = silu_mul((float)gb[i], (float)ub[i]);     // of the rounded values
    *reinterpret_cast<bf16x4 *>(p.act + (int64_t)m * F + col) = __builtin_convertvector(r, bf16x4);
}

template <class Sh, int WM, int WN, int MW, int NW, int NS, bool GLU>
__device__ __forceinline__ void gemm_rows(const GemmParams &p) {
    constexpr int BN = Sh::BN;
    constexpr int PER = Sh::W_CPW + Sh::X_CPW;          // copies per wavefront per step
    extern __shared__ __align__(1024) uint16_t lds[];   // [NS][W step, X step]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;

    // workgroup w runs on XCD w % 8: the row tiles of one (column tile, split)
    // follow one another on one XCD and share its W range in that L2, and
    // each XCD keeps to few splits, so its part of X stays in that L2 too
    const int local = (int)blockIdx.x >> 3;
    const int group = (local / p.m_tiles) * 8 + ((int)blockIdx.x & 7);
    if (group >= p.n_tiles * p.n_split) return;
    const int mt = local % p.m_tiles;
    const int split = group % p.n_split, nt = group / p.n_split;

    const int n_steps = p.K / BK;
    const int s0 = split * p.steps_per_split;
    int n = n_steps - s0;
    if (n > p.steps_per_split) n = p.steps_per_split;
    if (n < 0) n = 0;

    // Per-lane parts of the copy addresses (bytes).  Chunk q of a W step is
    // 512 / BN rows of k; chunk q of an X step is 8 rows of m.
    constexpr int WROWS = 512 / BN, WCOLS = BN / 8;
    uint32_t wl[Sh::W_CPW], xl[Sh::X_CPW];
#pragma unroll
    for (int u = 0; u < Sh::W_CPW; ++u) {
        const int r = (u * Sh::WAVES + wave) * WROWS + lane / WCOLS;
        const int c = (lane % WCOLS) ^ v_swz<BN>(r);          // 16-byte column of the tile
        int64_t e;
        if (GLU) {   // 32-column tiles of 16 gate then 16 up columns
            const int et = c >> 2, pc = c & 3;
            e = (int64_t)nt * (BN / 2) + et * 16 + (pc & 1) * 8 + (pc >> 1) * (int64_t)(p.N / 2);
        } else {
            e = (int64_t)nt * BN + c * 8;
        }
        wl[u] = (uint32_t)(((int64_t)r * p.N + e) * 2);
    }
#pragma unroll
    for (int u = 0; u < Sh::X_CPW; ++u) {
        const int r = (u * Sh::WAVES + wave) * 8 + lane / 8;
        const int c = (lane % 8) ^ (r & 7);
        int m = mt * Sh::BM + r;
        if (m > p.M - 1) m = p.M - 1;                         // rows past the last repeat it (not stored)
        xl[u] = (uint32_t)((m - mt * Sh::BM) * p.K + c * 8) * 2;
    }
    const uint16_t *wb = p.w + (int64_t)s0 * BK * p.N;
    const uint16_t *xb = p.x + (int64_t)mt * Sh::BM * p.K + (int64_t)s0 * BK;
    auto issue = [&](int s) {
        uint16_t *wt = lds + (s % NS) * Sh::STEP, *xt = wt + Sh::W_STEP;
        const uint16_t *ws = wb + (int64_t)s * BK * p.N, *xs = xb + s * BK;
#pragma unroll
        for (int u = 0; u < Sh::W_CPW; ++u) dma16(ws, wl[u], wt + (u * Sh::WAVES + wave) * 512);
#pragma unroll
        for (int u = 0; u < Sh::X_CPW; ++u) dma16(xs, xl[u], xt + (u * Sh::WAVES + wave) * 512);
    };

    const int wm = wave % WM, wn = wave / WM;
    f32x16 acc[MW][NW];
#pragma unroll
    for (int i = 0; i < MW; ++i)
#pragma unroll
        for (int t = 0; t < NW; ++t) acc[i][t] = f32x16{};
    int voff[BN / 32];
#pragma unroll
    for (int et = 0; et < BN / 32; ++et) voff[et] = vt_offset<BN>(lane, et);

#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
        if (s < n) issue(s);
    for (int s = 0; s < n; ++s) {
        // step s has landed once at most the NS - 2 later ones are in flight;
        // its buffer's previous reader finished before the barrier
        if (s + NS - 2 < n) wait_vmcnt<(NS - 2) * PER>();
        else wait_vmcnt<0>();
        lds_barrier();
        if (s + NS - 1 < n) issue(s + NS - 1);
        const uint16_t *wt = lds + (s % NS) * Sh::STEP, *xt = wt + Sh::W_STEP;
        // operands of the next 16 k are read beside the MFMAs of these (a
        // scheduling fence keeps that order)
        bf16x8 xf[2][MW], wf[2][NW];
        auto load = [&](int k16) {
#pragma unroll
            for (int t = 0; t < NW; ++t) wf[k16 & 1][t] = load_vt<BN>(wt, voff, k16 * (BN / 32) + wn * NW + t);
#pragma unroll
            for (int i = 0; i < MW; ++i)
                xf[k16 & 1][i] =
                    *reinterpret_cast<const bf16x8 *>(&xt[k_lds<BK>((wm * MW + i) * 32 + col, k16 * 2 + half)]);
        };
        load(0);
#pragma unroll
        for (int k16 = 0; k16 < BK / 16; ++k16) {
            if (k16 + 1 < BK / 16) load(k16 + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < NW; ++t)
#pragma unroll
                for (int i = 0; i < MW; ++i)
                    acc[i][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[k16 & 1][t], xf[k16 & 1][i], acc[i][t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    float *const pt = p.part + ((int64_t)(mt * p.n_tiles + nt) * p.n_split + split) * Sh::TILE;
#pragma unroll
    for (int i = 0; i < MW; ++i) {
        const int m = mt * Sh::BM + (wm * MW + i) * 32 + col;
        if (m >= p.M) break;
#pragma unroll
        for (int t = 0; t < NW; ++t) {
            const int et = wn * NW + t;
            f32x4 a[4];
#pragma unroll
            for (int vq = 0; vq < 4; ++vq)
                a[vq] = f32x4{acc[i][t][vq * 4], acc[i][t][vq * 4 + 1], acc[i][t][vq * 4 + 2], acc[i][t][vq * 4 + 3]};
            if (p.n_split > 1) {
                // accumulator order: [wave][row tile][column tile][vq][lane] groups of four floats
#pragma unroll
                for (int vq = 0; vq < 4; ++vq)
                    *reinterpret_cast<f32x4 *>(pt + ((((wave * MW + i) * NW + t) * 4 + vq) * 64 + lane) * 4) = a[vq];
            } else if constexpr (GLU) {
#pragma unroll
                for (int vq = 0; vq < 2; ++vq)
                    store_glu(p, m, nt * (BN / 2) + et * 16 + vq * 8 + half * 4, a[vq], a[vq + 2]);
            } else {
#pragma unroll
                for (int vq = 0; vq < 4; ++vq)
                    *reinterpret_cast<bf16x4 *>(p.y + (int64_t)m * p.N + nt * BN + tile_col(et, vq, half)) =
                        __builtin_convertvector(a[vq], bf16x4);
            }
        }
    }
}

template <int WM, int WN, int MW, int NW, int NS, bool GLU>
__global__ __launch_bounds__(WM *WN * 64) void gemm_rows_kernel(GemmParams p) {
    gemm_rows<GemmShape<WM, WN, MW, NW>, WM, WN, MW, NW, NS, GLU>(p);
}

// Add the splits of each tile and store it: one thread per group of four
// columns (GLU: per gate group, with its up group), all splits' loads in
// flight together.
template <int WM, int WN, int MW, int NW, bool GLU>
__global__ __launch_bounds__(256) void gemm_reduce_kernel(GemmParams p) {
    using Sh = GemmShape<WM, WN, MW, NW>;
    constexpr int BN = Sh::BN;
    constexpr int GROUPS = Sh::TILE / 4 / (GLU ? 2 : 1);        // per tile
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int tile = (int)(e / GROUPS);
    int r = (int)(e % GROUPS);
    const int lane = r & 63, half = lane >> 5;
    r >>= 6;
    const int vq = GLU ? r & 1 : r & 3;
    r >>= GLU ? 1 : 2;
    const int t = r % NW, i = r / NW % MW, wave = r / NW / MW;
    const int et = wave / WM * NW + t;
    const int mt = tile / p.n_tiles, nt = tile - mt * p.n_tiles;
    const int m = mt * Sh::BM + (wave % WM * MW + i) * 32 + (lane & 31);
    if (mt >= p.m_tiles || m >= p.M) return;
    const float *pt = p.part + (int64_t)tile * p.n_split * Sh::TILE;
    const int o = ((((wave * MW + i) * NW + t) * 4 + vq) * 64 + lane) * 4;
    f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f};
    constexpr int GS = 8;
    for (int s0 = 0; s0 < p.n_split; s0 += GS) {
        f32x4 va[GS], vb[GS];
#pragma unroll
        for (int k = 0; k < GS; ++k)
            if (s0 + k < p.n_split) {
                const float *ps = pt + (int64_t)(s0 + k) * Sh::TILE + o;
                va[k] = *reinterpret_cast<const f32x4 *>(ps);
                if (GLU) vb[k] = *reinterpret_cast<const f32x4 *>(ps + 2 * 64 * 4);
            }
#pragma unroll
        for (int k = 0; k < GS; ++k)
            if (s0 + k < p.n_split) {
                a += va[k];
                if (GLU) b += vb[k];
            }
    }
    if constexpr (GLU) {
        store_glu(p, m, nt * (BN / 2) + et * 16 + vq * 8 + half * 4, a, b);
    } else {
        *reinterpret_cast<bf16x4 *>(p.y + (int64_t)m * p.N + nt * BN + tile_col(et, vq, half)) =
            __builtin_convertvector(a, bf16x4);
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// Row tile for M rows (32, 64, 128 or 256): the smallest that holds them; past
// 256 rows, tiles of 128 where they waste fewer padded rows than tiles of 256.
static int rows_per_tile(int64_t M) {
    if (M <= 32) return 32;
    if (M <= 64) return 64;
    if (M <= 128) return 128;
    return (M + 127) / 128 % 2 && M > 256 ? 128 : 256;
}

// Tiles of one product and the ranges its K is split into.
struct RowsPlan {
    int64_t bm, m_tiles, n_tiles, n_split, steps_per_split;
};
static RowsPlan plan_rows(int64_t M, int64_t K, int64_t N) {
    RowsPlan r;
    r.bm = rows_per_tile(M);
    r.m_tiles = (M + r.bm - 1) / r.bm;
    r.n_tiles = N / GEMM_BN;
    // one workgroup per CU; at least four steps each, so that the ring fills;
    // within the workspace
    const int64_t tiles = r.m_tiles * r.n_tiles, steps = K / BK;
    int64_t split = std::min<int64_t>(GEMM_WGS / tiles, steps / 4);
    split = std::min<int64_t>(split, (int64_t)GEMM_WORKSPACE_BYTES / (tiles * r.bm * GEMM_BN * 4));
    if (split < 1) split = 1;
    r.steps_per_split = (steps + split - 1) / split;
    r.n_split = (steps + r.steps_per_split - 1) / r.steps_per_split;
    return r;
}

template <int WM, int WN, int MW, int NW, int NS, bool GLU>
static hipError_t launch_shape(GemmParams p, const RowsPlan &r, hipStream_t s) {
    using Sh = GemmShape<WM, WN, MW, NW>;
    static_assert(Sh::BN == GEMM_BN, "column tile");
    constexpr size_t lds = (size_t)NS * Sh::STEP * 2;
    static_assert(lds <= CU_LDS_BYTES, "ring larger than the LDS");
    if (r.bm != Sh::BM || (r.n_split > 1 && !p.part)) return hipErrorInvalidValue;
    p.m_tiles = (int32_t)r.m_tiles;
    p.n_tiles = (int32_t)r.n_tiles;
    p.n_split = (int32_t)r.n_split;
    p.steps_per_split = (int32_t)r.steps_per_split;
    const int64_t tiles = r.m_tiles * r.n_tiles;
    const hipError_t e = allow_dynamic_lds<&gemm_rows_kernel<WM, WN, MW, NW, NS, GLU>>((int)lds);
    if (e != hipSuccess) return e;
    const int64_t grid = 8LL * ((p.n_tiles * p.n_split + 7) / 8) * p.m_tiles;
    hipLaunchKernelGGL((gemm_rows_kernel<WM, WN, MW, NW, NS, GLU>), dim3((unsigned)grid), dim3(Sh::THREADS), lds, s, p);
    if (p.n_split > 1) {
        const int64_t items = tiles * (Sh::TILE / 4 / (GLU ? 2 : 1));
        hipLaunchKernelGGL((gemm_reduce_kernel<WM, WN, MW, NW, GLU>), dim3((unsigned)(items / 256)), dim3(256), 0, s, p);
    }
    return hipGetLastError();
}

template <bool GLU>
static hipError_t launch_glu(const GemmParams &p, const RowsPlan &r, hipStream_t s) {
    switch (r.bm) {
        case 32: return launch_shape<1, 4, 1, 1, 4, GLU>(p, r, s);
        case 64: return launch_shape<1, 4, 2, 1, 3, GLU>(p, r, s);
        case 128: return launch_shape<2, 2, 2, 2, 4, GLU>(p, r, s);
        default: return launch_shape<2, 4, 4, 1, 3, GLU>(p, r, s);
    }
}

// Where these kernels take a product from the GEMM library, which does not
// split K here.  The figures are us per product gained over the library's
// (gate|up: over its product and the gating kernel), inside a whole layer whose
// weights come from HBM, for layers of H/F 2048/5632, 2048/8192, 3584/18944,
// 4096/14336, 5120/13824 and 8192/28672:
//  - up to 64 rows, column tiles that fit the CUs in one go: O 4 to 28, down 12
//    to 108, QKV 4 to 29; gate|up -5 to 17 (-5 at 32 and 64 rows of N 27648,
//    the library's own tile sizes).  More column tiles than CUs leave a second
//    round nearly empty: gate|up of N 37888 loses 21 to 24 (of 156 to 215 for
//    the layer), of N 57344 32 to 44 (of 374 to 486);
//  - to 512 rows where the tiles fill at most half the CUs, so that K is split
//    and the library leaves CUs idle: down 8 to 131, but for N 3584, K 18944 at
//    257 to 384 rows (-7 to -18); O -6 to 40, QKV -5 to 38.  257 to 384 rows are
//    three tiles of 128 and 385 to 512 two of 256, so a product can be the
//    library's in the first range and ours in the second: QKV of N 6144, K
//    4096 would gain -3 to 0 in the first and gains -2 to 14 in the second,
//    down of N 8192 -12 to -67 and 51 to 67, O of N 8192 0 to 5 and -6 to -3;
//  - gate|up past 64 rows: X moves through each CU once per column tile, which
//    costs more than the fused gating saves (N 28672: -17 at 192 rows, -58 at
//    512); past 512 rows all products: O -35 to 4, down -190 to 46.
// Without a workspace a product whose K would be split is the library's.
bool gemm_rows_applies(int64_t M, int64_t K, int64_t N, bool has_workspace) {
    if (M < 1 || K < BK || K % BK || N % GEMM_BN || N < GEMM_BN) return false;
    // 32-bit offsets within a step's rows of W and a row tile of X
    if ((int64_t)BK * N * 2 >= INT32_MAX || 256 * K * 2 >= INT32_MAX) return false;
    const RowsPlan r = plan_rows(M, K, N);
    if (M > 512 || r.m_tiles * r.n_tiles * (M > 64 ? 2 : 1) > GEMM_WGS) return false;
    return has_workspace || r.n_split == 1;
}

int64_t gemm_rows_splits(int64_t M, int64_t K, int64_t N) { return plan_rows(M, K, N).n_split; }

hipError_t launch_gemm_rows(const uint16_t *x, const uint16_t *w, uint16_t *y, uint16_t *act, void *ws, int64_t M,
                            int64_t K, int64_t N, hipStream_t s) {
    GemmParams p{};
    p.x = x;
    p.w = w;
    p.y = y;
    p.act = act;
    p.part = static_cast<float *>(ws);
    p.M = (int32_t)M;
    p.N = (int32_t)N;
    p.K = (int32_t)K;
    const RowsPlan r = plan_rows(M, K, N);
    return act ? launch_glu<true>(p, r, s) : launch_glu<false>(p, r, s);
}

}  // namespace oc
