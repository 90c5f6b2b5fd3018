// Suffix-prefill GQA attention over a paged cached prefix plus the new
// suffix tokens (the per-layer compute C_l of eq. (3)).
//
// Work split: for each KV head g the query rows are the (suffix token, query
// head of g's group) pairs, token-major, so one 32-row MFMA block shares
// tokens across the group's heads (GQA packing).  A workgroup of 8
// wavefronts owns 8 x 32 rows and one contiguous range of 64-key blocks; key
// ranges are split over workgroups (split-KV) so long prefixes fill the chip,
// and a combine kernel merges the splits by log-sum-exp.  Workgroups that read
// the same K/V pages (same KV head and split) are dispatched back to back onto
// the same XCD, so their re-reads hit that XCD's L2.
//
// Per 64-key block: the K and V rows of four pages ([slot][dim] pool blocks,
// or for the suffix the k_new / v_new rows themselves) are copied straight
// into token-major LDS tiles by the global->LDS load path, two blocks in
// flight, a barrier per phase.  The tiles' 16-byte columns are XOR-swizzled
// by row so the operand reads are free of bank conflicts.  Each wavefront
// computes S^T = K Q^T for its 32 queries with bf16 MFMA 32x32x16 (fp32
// accumulate), runs the online softmax with one query column per lane (the
// two half-waves combine their maxima with a lane swap; the running maximum
// is only raised -- and O rescaled -- when a block's maximum exceeds it by more
// than 2^8), converts P to bf16 and accumulates O^T += V^T P.  The V^T operand
// (eight consecutive keys of one dimension per lane) comes from two
// transposing LDS reads of the token-major V tile.  The K tile's rows are fed
// to the MFMA in an order (bits 2 and 3 of the row swapped) that leaves each
// half-wave holding eight consecutive keys of P, matching those eight keys of
// the V operand.
#include <math.h>

#include <algorithm>
#include <cmath>

#include "mfma_tiles.hpp"

namespace oc {

constexpr int PAGE = 16;          // tokens per pool page (attention requires page_size 16)
constexpr int KB = 64;            // keys per block = 4 pages
constexpr int WAVES = 8;          // two per SIMD: one's softmax overlaps the other's MFMAs
constexpr int QB = 1;             // 32-row query blocks per wavefront
constexpr int WAVE_ROWS = 32 * QB;
constexpr int TILE_ROWS = WAVES * WAVE_ROWS;
constexpr int THREADS = WAVES * 64;
constexpr int TARGET_WGS = 256;   // one workgroup per CU
#ifndef OC_BATCH_ROUNDS
#define OC_BATCH_ROUNDS 2
#endif
constexpr int BATCH_ROUNDS = OC_BATCH_ROUNDS;   // workgroups per CU a batched launch may queue
constexpr float RESCALE_SLACK = 8.0f;   // log2 units the running max may lag
constexpr int LOOKAHEAD = 3;              // MFMAs an operand read runs ahead of its use

struct KParams {
    const uint16_t *q;
    const uint16_t *pool_k, *pool_v;
    const int32_t *pages;
    const uint16_t *k_new, *v_new;   // suffix rows [Ts][nkv][D]
    float *o_part, *ml_part;
    uint16_t *out;
    int64_t Tp, Ts, rows, rows_pad, n_pre_pages, n_suf_pages, n_blocks, blocks_per_split;
    int nq, nkv, grp, m_tiles, n_split, n_groups;
    float scale_log2;
};

// One launch serves up to MAX_ATTN_BATCH requests of one layer: workgroup w
// belongs to the last request whose first workgroup it has reached (and a
// block of the split merge, likewise, to the last whose first block it has
// reached; a request without splits has none).
struct KBatch {
    int32_t n;
    int32_t first_wg[MAX_ATTN_BATCH];
    int32_t first_cb[MAX_ATTN_BATCH];
    KParams req[MAX_ATTN_BATCH];
};

// value of the lane 32 positions away (the other half of the wavefront)
__device__ inline float half_swap_max(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float half_swap_sum(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Zero n rows of an LDS tile with one wavefront, 16 bytes per lane and store.
// (Two bytes took some 0.5 us of a 7 us call: 20 + 6 tokens, d = 128, 6.6 -> 6.1.
// The 256-row kernel clears with 256 lanes and two bytes: this way its loop ran
// 0.1 to 0.3 % slower.)
template <int D>
__device__ __forceinline__ void clear_rows(uint16_t *rows, int n, int lane) {
    uint32_t z = 0;
    asm volatile("" : "+v"(z));      // made here: the compiler would keep four registers of zeros through the loop
    for (int i = lane; i < n * (D / 8); i += 64) *reinterpret_cast<u32x4 *>(rows + i * 8) = u32x4{z, z, z, z};
}

// Whether all row tiles of a (KV head, split) group get consecutive slots on
// one XCD (workgroup w runs on XCD w % 8), so that their K/V re-reads hit that
// XCD's L2, or the tiles are dealt out to the XCDs one by one.
//  - A multiple of 8 groups loads the XCDs evenly: by XCD.
//  - 256-row tiles, any other count: dealt.  They re-read little, and XCDs that
//    hold a group less idle (by XCD 0.95 to 1.82 times as long, 1.11 on
//    average, over 87 shapes of 4 to 122 groups).
//  - Tiles of 32 and 64 rows: by XCD where there is a group for every XCD and
//    the busiest XCD's workgroups all run at once on its 32 CUs (0.60 to 1.05
//    times as long as dealt, 0.94 on average, over 123 shapes of 9 to 108
//    groups) or the XCDs are within 1/15 of even (0.48 to 1.12, 0.91 on average,
//    over 36 shapes of 15 to 100 groups).  Otherwise the uneven XCDs cost more
//    than their L2 gives (0.95 to 1.87, 1.28 on average, over 232 shapes), and
//    with fewer groups than XCDs some would idle (1.0 to 6.3).
__host__ __device__ inline bool tiles_by_xcd(int m_tiles, int n_groups, bool small_tiles) {
    if ((n_groups & 7) == 0) return true;
    const int per_xcd = (n_groups + 7) / 8;           // groups of the busiest XCD
    return small_tiles && n_groups > 8 &&
           ((int64_t)per_xcd * m_tiles <= 32 || 2 * (int64_t)n_groups >= 15 * (int64_t)per_xcd);
}

// Workgroup wg of a launch -> its (KV head, split) group and row tile; false
// past the last.  Either way the last row tile comes first: under the causal
// mask later rows see more suffix keys, and dispatching the longest tiles
// first keeps them out of the tail.
__host__ __device__ inline bool tile_of(int wg, int m_tiles, int n_groups, bool small_tiles, int &gamma, int &mt) {
    if (!tiles_by_xcd(m_tiles, n_groups, small_tiles)) {
        gamma = wg % n_groups;
        mt = m_tiles - 1 - wg / n_groups;
        return mt >= 0;
    }
    const int xcd = wg & 7, local = wg >> 3;
    gamma = (local / m_tiles) * 8 + xcd;
    mt = m_tiles - 1 - local % m_tiles;
    return gamma < n_groups;
}

// tile row r of a 32-key MFMA tile reads physical key perm(r): bits 2 and 3 swapped
__device__ inline int key_perm(int r) { return (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1); }

// Per-wavefront running state of the online softmax for its 32 query rows.
template <int D>
struct WaveState {
    f32x16 o[D / 32];    // O^T: 32 dims x 32 rows per tile, fp32
    f32x16 s[2];         // scores of the current block, one 32-key half each
    bf16x8 p[2][2];      // P of the last softmaxed block as the PV operand: [half][8-key group]
    float m, l;          // running maximum (log2 units) and sum of this lane's row
};

// The first LOOKAHEAD V^T fragments of a PV pass, read ahead of the barrier
// that opens the matrix phase (the V tile of the previous block is already
// readable there), so the phase starts without waiting on LDS.
template <int D>
__device__ __forceinline__ void prefetch_vt(const uint16_t *V, const int (&voff)[D / 32], bf16x8 (&pre)[LOOKAHEAD]) {
#pragma unroll
    for (int n = 0; n < LOOKAHEAD; ++n) pre[n] = load_vt<D>(V, voff, n);
}

// Matrix phase of a wavefront: O^T += V^T P for the previous block (PV:
// 16 MFMAs at d = 128, each V^T fragment from two transposing LDS reads),
// then S^T = K Q^T for the current block (S: 16 MFMAs, K fragments from the
// swizzled tile, the two 32-key halves alternating so that consecutive MFMAs
// are independent).  Written as one flat sequence whose operand reads run
// LOOKAHEAD MFMAs ahead (with PV, the first LOOKAHEAD come preloaded, see
// prefetch_vt); a scheduling fence after every MFMA keeps that order (left
// alone, the compiler hoists every read to the top and runs out of VGPRs).
template <int D, bool PV, bool S>
__device__ __forceinline__ void matrix_phase(WaveState<D> &w, const uint16_t *V, const int (&voff)[D / 32],
                                             const uint16_t *K, const bf16x8 (&qop)[D / 16], int krow, int half,
                                             const bf16x8 (&pre)[LOOKAHEAD]) {
    constexpr int NET = D / 32, NDS = D / 16;
    constexpr int NPV = PV ? 4 * NET : 0;
    constexpr int N = NPV + (S ? 2 * NDS : 0);
    static_assert(!PV || NPV >= LOOKAHEAD, "prefetched fragments must all be V^T fragments");
    auto load = [&](int n) -> bf16x8 {
        if (n < NPV) return load_vt<D>(V, voff, n);
        const int n2 = n - NPV, ds = n2 >> 1, kt = n2 & 1;
        return *reinterpret_cast<const bf16x8 *>(&K[k_lds<D>(kt * 32 + krow, ds * 2 + half)]);
    };
    bf16x8 f[N];
    // the wavefront in its matrix phase issues ahead of its SIMD partner's
    // softmax: the MFMA pipe is the longer of the two (about 3 % per layer)
    __builtin_amdgcn_s_setprio(2);
#pragma unroll
    for (int n = 0; n < LOOKAHEAD && n < N; ++n) f[n] = PV ? pre[n] : load(n);
#pragma unroll
    for (int n = 0; n < N; ++n) {
        if (n + LOOKAHEAD < N) f[n + LOOKAHEAD] = load(n + LOOKAHEAD);
        if (n < NPV) {
            const int et = n % NET, g4 = n / NET;
            w.o[et] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[n], w.p[g4 >> 1][g4 & 1], w.o[et], 0, 0, 0);
        } else {
            const int n2 = n - NPV, ds = n2 >> 1, kt = n2 & 1;
            w.s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[n], qop[ds], ds == 0 ? f32x16{} : w.s[kt], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_setprio(1);
}

// Softmax phase of a wavefront for one block: the block maximum (one lane
// swap between the half-waves), the lazy raise of the running maximum (O and
// l rescaled only when the block maximum exceeds it by more than
// 2^RESCALE_SLACK), then P = 2^(s*scale*log2(e) - m) as bf16 and the row sums
// of that rounded P.
template <int D>
__device__ __forceinline__ void softmax_phase(WaveState<D> &w, float scale_log2) {
    float mx[2] = {-__builtin_inff(), -__builtin_inff()};   // two partial maxima
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int i2 = 0; i2 < 16; ++i2) mx[i2 & 1] = fmaxf(mx[i2 & 1], w.s[kt][i2]);
    const float mblk = half_swap_max(fmaxf(mx[0], mx[1])) * scale_log2;
    if (__any(mblk > w.m + RESCALE_SLACK)) {
        const float m_new = fmaxf(w.m, mblk);
        const float alpha = __builtin_amdgcn_exp2f(w.m - (m_new == -__builtin_inff() ? 0.f : m_new));
        w.m = m_new;
        w.l *= alpha;
#pragma unroll
        for (int et = 0; et < D / 32; ++et) w.o[et] *= alpha;
    }
    const float m_use = w.m == -__builtin_inff() ? 0.f : w.m;
    // row sums of the rounded P (the values the PV product uses), two bf16
    // pairs per dot instruction, two partial sums
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 ones = {(__bf16)1.f, (__bf16)1.f};
    float lsum[2] = {0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            f32x8 pv;
#pragma unroll
            for (int i2 = 0; i2 < 8; ++i2)
                pv[i2] = __builtin_amdgcn_exp2f(fmaf(w.s[kt][hf * 8 + i2], scale_log2, -m_use));
            const bf16x8 pp = __builtin_convertvector(pv, bf16x8);
            w.p[kt][hf] = pp;
            lsum[0] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pp, pp, 0, 1), ones, lsum[0], false);
            lsum[1] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pp, pp, 2, 3), ones, lsum[1], false);
            lsum[0] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pp, pp, 4, 5), ones, lsum[0], false);
            lsum[1] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pp, pp, 6, 7), ones, lsum[1], false);
        }
    w.l += lsum[0] + lsum[1];
}

template <int D>
__global__ __launch_bounds__(THREADS) void attn_fwd_kernel(KBatch batch) {
    // read the request's parameters straight from the kernel-argument segment
    // (scalar loads at a uniform offset; indexing the by-value copy would
    // place it in scratch memory)
    typedef const __attribute__((address_space(4))) KBatch *kbatch_ptr;
    // every wavefront issues ahead of the ingest wavefronts that may share
    // its SIMD (they keep the lowest priority); the matrix phase goes one
    // level higher still
    __builtin_amdgcn_s_setprio(1);
    const kbatch_ptr bp = (kbatch_ptr)__builtin_amdgcn_kernarg_segment_ptr();
    int req = 0;
    for (int i = 1; i < bp->n; ++i) req += (int)blockIdx.x >= bp->first_wg[i];
    const __attribute__((address_space(4))) KParams &p = bp->req[req];
    const int wg = (int)blockIdx.x - bp->first_wg[req];
    // Every parameter is read once into a register here: read through `p`
    // inside the loop, each use would be reloaded from the argument segment
    // after every inline-assembly statement (they clobber memory), each reload
    // a scalar load that the next LDS wait must also wait for.  Token, page,
    // block and row counts fit 32 bits (the host limits prefix + suffix to
    // 2^30 tokens and rows to 2^30).
    const int m_tiles = p.m_tiles, n_groups = p.n_groups, n_split = p.n_split;
    const int grp = p.grp, nq = p.nq, nkv = p.nkv;
    const int rows = (int)p.rows, Tp = (int)p.Tp, Ts = (int)p.Ts, n_pre_pages = (int)p.n_pre_pages;
    const int n_blocks = (int)p.n_blocks, blocks_per_split = (int)p.blocks_per_split;
    const int64_t rows_pad = p.rows_pad;
    const float scale_log2 = p.scale_log2;
    const uint16_t *const q_in = p.q;
    const uint16_t *const pool_k = p.pool_k, *const pool_v = p.pool_v;
    const uint16_t *const k_new = p.k_new, *const v_new = p.v_new;
    uint16_t *const out_ptr = p.out;
    float *const o_part = p.o_part, *const ml_part = p.ml_part;
    const __attribute__((address_space(4))) int32_t *pages_c =
        (const __attribute__((address_space(4))) int32_t *)p.pages;
    constexpr int TILE = KB * D;                   // elements of one K (or V) tile
    constexpr int CHUNKS = TILE * 2 / 1024;        // 1 KiB DMA chunks per tile
    constexpr int CPW = CHUNKS / WAVES;            // chunks per wavefront per tile
    constexpr int KROWS = 512 / D;                 // K rows per chunk
    constexpr int CPP = D / 32;                    // chunks per page (K and V alike)
    constexpr int NDMA = 2 * CPW;                  // DMA instructions per wavefront per block
    // buffers: the current block, the previous one (its V is read in this
    // block's phase B), and two blocks whose copies are in flight
    constexpr int NBUF = 4;
    static_assert(CPW >= 1 && CHUNKS % WAVES == 0, "tile does not divide");
    extern __shared__ __align__(1024) uint16_t lds[];   // [NBUF][K tile, V tile]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;

    int gamma, mt;
    if (!tile_of(wg, m_tiles, n_groups, false, gamma, mt)) return;
    const int g = gamma / n_split, split = gamma - g * n_split;

    const int row = mt * TILE_ROWS + wave * WAVE_ROWS + col;
    const bool row_ok = row < rows;
    const int tok = row_ok ? row / grp : 0;
    bf16x8 qop[D / 16];
    {
        const int head = g * grp + (row_ok ? row % grp : 0);
        const uint16_t *qr = q_in + ((int64_t)tok * nq + head) * D + half * 8;
#pragma unroll
        for (int ds = 0; ds < D / 16; ++ds) {
            u32x4 v = row_ok ? *reinterpret_cast<const u32x4 *>(qr + ds * 16) : u32x4{0, 0, 0, 0};
            qop[ds] = __builtin_bit_cast(bf16x8, v);
        }
    }

    const int b0 = split * blocks_per_split;
    int b1 = b0 + blocks_per_split;
    if (b1 > n_blocks) b1 = n_blocks;
    {   // causal clip: no row of this tile sees suffix keys past its last token
        int row_hi = (mt + 1) * TILE_ROWS - 1;
        if (row_hi > rows - 1) row_hi = rows - 1;
        const int last_page = n_pre_pages + (row_hi / grp) / PAGE;
        if (b1 > last_page / 4 + 1) b1 = last_page / 4 + 1;
    }
    const int full_pre_pages = Tp / PAGE;
    const int64_t head_block = (int64_t)PAGE * D;      // elements of one (page, head) block

    // ---- global -> LDS copy of one 64-key block (4 pages) ----
    // Both tiles are token-major ([key][dim]) with 16-byte columns XOR-swizzled
    // by key row (K for the S reads, V for the transposing PV reads); each
    // lane fetches the global piece that belongs at its fixed LDS position.
    // Every 1 KiB chunk comes from a single page; a wavefront copies CPW
    // chunks of each tile.  The base pointers stay in registers, and the page
    // ids of a block are loaded (scalar loads through the constant address
    // space) one block ahead of its copy, so no copy waits on a lookup.
    auto load_pids = [&](int b, int32_t (&pid)[CPW]) {
#pragma unroll
        for (int u = 0; u < CPW; ++u) {
            const int v = b * 4 + (u * WAVES + wave) / CPP;
            pid[u] = v < n_pre_pages ? pages_c[v] : 0;
        }
    };
    // per-lane parts of the copy addresses (bytes), fixed for the whole loop:
    // chunk u of a wavefront covers key rows rr[u] + [0, KROWS) of its page
    uint32_t klane[CPW], vlane[CPW];
    int rr[CPW];
#pragma unroll
    for (int u = 0; u < CPW; ++u) {
        const unsigned q = (unsigned)(u * WAVES + wave);
        const int r = (int)(q % CPP) * KROWS + lane / (D / 8);   // key row within the page
        const int ck = (lane % (D / 8)) ^ (r & (D / 8 - 1));
        const int cv = (lane % (D / 8)) ^ v_swz<D>(r);
        rr[u] = r;
        klane[u] = (uint32_t)(r * D + ck * 8) * 2;
        vlane[u] = (uint32_t)(r * D + cv * 8) * 2;
    }
    const uint32_t page_bytes = (uint32_t)(nkv * head_block * 2);     // one page of K (or V)
    const int n_fast_pages = nkv * head_block * 2 <= 0xFFFFFFFFLL ? n_pre_pages : 0;
    const unsigned char *const kg = reinterpret_cast<const unsigned char *>(pool_k + g * head_block);
    const int64_t kv_step = (pool_v - pool_k) * 2;
    auto issue_block = [&](int b, int buf, const int32_t (&pid)[CPW]) {
        uint16_t *kt_lds = lds + buf * 2 * TILE;
        uint16_t *vt_lds = kt_lds + TILE;
        if (b * 4 + 4 <= n_fast_pages) {     // all prefix: one 32 x 32 -> 64-bit product per page
#pragma unroll
            for (int u = 0; u < CPW; ++u) {
                const int q = u * WAVES + wave;
                const unsigned char *kp = kg + (uint64_t)(uint32_t)pid[u] * page_bytes;
                dma16(kp, klane[u], kt_lds + q * 512);
                dma16(kp + kv_step, vlane[u], vt_lds + q * 512);
            }
            return;
        }
#pragma unroll
        for (int u = 0; u < CPW; ++u) {
            const int q = u * WAVES + wave;                   // chunk index, uniform per wavefront
            const int v = b * 4 + q / CPP;                    // page of the key sequence
            if (v < n_pre_pages) {
                const int64_t blk = ((int64_t)pid[u] * nkv + g) * head_block;
                dma16(pool_k + blk, klane[u], kt_lds + q * 512);
                dma16(pool_v + blk, vlane[u], vt_lds + q * 512);
            } else {
                // suffix token; rows past the last one repeat it (finite, and masked)
                int T = (v - n_pre_pages) * PAGE + rr[u];
                if (T > Ts - 1) T = Ts - 1;
                // below 2^31: the host limits T_s * n_kv * d * 2 bytes
                const uint32_t rw = ((uint32_t)(T * nkv + g) * D - (uint32_t)rr[u] * D) * 2;
                dma16(k_new, rw + klane[u], kt_lds + q * 512);
                dma16(v_new, rw + vlane[u], vt_lds + q * 512);
            }
        }
    };

    WaveState<D> w;
#pragma unroll
    for (int et = 0; et < D / 32; ++et) w.o[et] = f32x16{};
    w.m = -__builtin_inff();
    w.l = 0.f;
    const int krow = key_perm(col);
    int voff[D / 32];
#pragma unroll
    for (int et = 0; et < D / 32; ++et) voff[et] = vt_offset<D>(lane, et);

    // Mask of one block: keys [0, pe) of the block are prefix keys, suffix
    // keys start at ps, and a row sees suffix key k (block position) when
    // k - ps <= its token.  Branch-free bitwise select of the score or -inf
    // (a short-circuit form was compiled into divergent branches that
    // dropped the kept value).
    // (The limits are shifted by this half-wave's key offset so that each
    // comparison is against a constant: no per-lane key index stays live.)
    auto mask_block = [&](int b) {
        const int sh = 8 * half;
        const int pe = Tp - b * KB - sh;
        const int ps = n_pre_pages * PAGE - b * KB - sh;
        const int lim = tok + ps;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int i2 = 0; i2 < 16; ++i2) {
                const int kin = kt * 32 + (i2 < 8 ? i2 : 8 + i2);   // key in the block, less 8*half
                const uint32_t keep = 0u - (uint32_t)((kin < pe) | ((kin >= ps) & (kin <= lim)));
                w.s[kt][i2] = __uint_as_float((__float_as_uint(w.s[kt][i2]) & keep) | (0xff800000u & ~keep));
            }
    };
    // Q operands are in registers before the key loop starts (a wait the
    // compiler sees, so it places none of its own inside the loop)
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    const int nb = b1 > b0 ? b1 - b0 : 0;
    int32_t pid[CPW];
    if (nb > 0) {
        load_pids(b0, pid);
        issue_block(b0, 0, pid);
    }
    if (nb > 1) {
        load_pids(b0 + 1, pid);
        issue_block(b0 + 1, 1, pid);
    }
    if (nb > 2) load_pids(b0 + 2, pid);
    // Ping-pong schedule.  Each wavefront alternates a matrix phase (PV of
    // block j-1, S of block j) and a softmax phase (block j); wavefronts 4-7
    // (the second wavefront of every SIMD) run the same sequence one phase
    // later than wavefronts 0-3, so on every SIMD one wavefront's MFMAs run
    // beside the other's softmax.  A workgroup barrier ends every phase.
    //
    // A wavefront issues its tile copies (scalar address work and vector
    // memory instructions, some 400 cycles) at the start of a softmax phase:
    // there they run in the shadow of the partner's MFMAs, while in a matrix
    // phase the MFMA pipe would wait for them.  Block j+2's copies are thus
    // issued in phase 2j by wavefronts 4-7 and in phase 2j+1 by wavefronts
    // 0-3, into the buffer of block j-2, whose last reads (wavefronts 4-7's PV)
    // ended with phase 2j-1; each wavefront waits for its own copies before
    // the barrier that opens phase 2j+4, where the tile becomes readable.
    // (65536 + 512 tokens, one layer: 507 us with both groups' copies at the
    // barrier that opens a block, 490 like this; 553 with wavefronts 4-7's in
    // their matrix phase; a fifth buffer with the copies one block further
    // ahead changes nothing.)
    const bool first = (wave >> 2) == 0;
    auto tile_k = [&](int j) -> const uint16_t * { return lds + (j % NBUF) * 2 * TILE; };
    auto tile_v = [&](int j) -> const uint16_t * { return lds + (j % NBUF) * 2 * TILE + TILE; };
    auto refill = [&](int j) {
        if (j + 2 < nb) issue_block(b0 + j + 2, (j + 2) % NBUF, pid);
        if (j + 3 < nb) load_pids(b0 + j + 3, pid);
    };
    // The barrier that ends a matrix phase waits for the phase's tile reads
    // (lds_barrier); the one that ends a softmax phase does not: the V^T
    // fragments prefetched there may arrive after it, they are waited for
    // where the matrix phase uses them.
    auto softmax_end = [] { asm volatile("s_barrier" ::: "memory"); };
    // this wavefront's copies of block j are in; the barrier that follows,
    // the start of phase 2j, makes the tile readable
    auto await_block = [&](int j) {
        if (j + 1 < nb) wait_vmcnt<NDMA>();
        else wait_vmcnt<0>();
    };
    // Wavefronts 4-7, in phase 2j: in the last, partial prefix page the slots
    // past Tp may hold anything; zero them so masked keys contribute exactly
    // nothing (the V tile is first read after the next barrier).
    auto zero_stale = [&](int j) {
        const int b = b0 + j;
        if (j < nb && (b + 1) * 4 > full_pre_pages && b * 4 <= full_pre_pages && full_pre_pages < n_pre_pages) {
            uint16_t *V = lds + (j % NBUF) * 2 * TILE + TILE;
            const int pg = full_pre_pages - b * 4, k0 = Tp % PAGE;
            for (int idx = tid - THREADS / 2; idx < D * (PAGE - k0); idx += THREADS / 2) V[(pg * PAGE + k0) * D + idx] = 0;
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
    };
    // A block needs the mask only if it holds slots of the prefix's partial
    // last page, or suffix keys that some row of this wavefront does not see
    // yet (the wavefront's rows start at token tok_min).
    const int tok_min = (mt * TILE_ROWS + wave * WAVE_ROWS) / grp;
    auto softmax_block = [&](int j) {
        const int b = b0 + j;
        if ((b + 1) * 4 > full_pre_pages) {
            const int ps = n_pre_pages * PAGE - b * KB, pe = Tp - b * KB;
            const bool partial_prefix = ps > 0 && pe < (ps < KB ? ps : KB);
            const bool unseen_suffix = ps < KB && KB - 1 - ps > tok_min;
            if (partial_prefix || unseen_suffix) mask_block(b);
        }
        softmax_phase<D>(w, scale_log2);
    };
    // Each group runs its own copy of the loop (one straight path each, so
    // the accumulators keep their registers); both execute the same barriers.
    if (nb > 0) {
        bf16x8 pre[LOOKAHEAD];
        await_block(0);
        lds_barrier();
        if (first) {
            matrix_phase<D, false, true>(w, nullptr, voff, tile_k(0), qop, krow, half, pre);
            lds_barrier();
            refill(0);
            softmax_block(0);
            for (int j = 1; j < nb; ++j) {
                prefetch_vt<D>(tile_v(j - 1), voff, pre);
                await_block(j);
                softmax_end();
                matrix_phase<D, true, true>(w, tile_v(j - 1), voff, tile_k(j), qop, krow, half, pre);
                lds_barrier();
                refill(j);
                softmax_block(j);
            }
            prefetch_vt<D>(tile_v(nb - 1), voff, pre);
            softmax_end();
            matrix_phase<D, true, false>(w, tile_v(nb - 1), voff, nullptr, qop, krow, half, pre);
            lds_barrier();
        } else {
            refill(0);
            zero_stale(0);
            lds_barrier();
            matrix_phase<D, false, true>(w, nullptr, voff, tile_k(0), qop, krow, half, pre);
            for (int j = 1; j < nb; ++j) {
                await_block(j);
                lds_barrier();
                refill(j);
                zero_stale(j);
                softmax_block(j - 1);
                prefetch_vt<D>(tile_v(j - 1), voff, pre);
                softmax_end();
                matrix_phase<D, true, true>(w, tile_v(j - 1), voff, tile_k(j), qop, krow, half, pre);
            }
            lds_barrier();
            softmax_block(nb - 1);
            prefetch_vt<D>(tile_v(nb - 1), voff, pre);
            softmax_end();
            matrix_phase<D, true, false>(w, tile_v(nb - 1), voff, nullptr, qop, krow, half, pre);
        }
    }

    const float l_tot = half_swap_sum(w.l);
    if (!row_ok) return;
    if (n_split == 1) {
        const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
        const int head = g * grp + row % grp;
        uint16_t *orow = out_ptr + ((int64_t)tok * nq + head) * D;
#pragma unroll
        for (int et = 0; et < D / 32; ++et)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
                f32x4 o4 = {w.o[et][vq * 4 + 0], w.o[et][vq * 4 + 1], w.o[et][vq * 4 + 2], w.o[et][vq * 4 + 3]};
                *reinterpret_cast<bf16x4 *>(orow + et * 32 + vq * 8 + half * 4) = __builtin_convertvector(o4 * inv, bf16x4);
            }
    } else {
        const int64_t prow = ((int64_t)split * nkv + g) * rows_pad + row;
        float *orow = o_part + prow * D;
#pragma unroll
        for (int et = 0; et < D / 32; ++et)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
                f32x4 o4 = {w.o[et][vq * 4 + 0], w.o[et][vq * 4 + 1], w.o[et][vq * 4 + 2], w.o[et][vq * 4 + 3]};
                *reinterpret_cast<f32x4 *>(orow + et * 32 + vq * 8 + half * 4) = o4;
            }
        if (half == 0) {
            ml_part[prow * 2 + 0] = w.m;
            ml_part[prow * 2 + 1] = l_tot;
        }
    }
}

// ---------------------------------------------------------------------------
// Few query rows: the wavefronts of a workgroup share one row tile and split
// the keys among themselves.
//
// With few rows per KV head the kernel above pads its 256-row tile, and to
// fill the CUs it splits the keys over so many workgroups that writing and
// merging the fp32 partials costs more than the attention.  Here a workgroup
// owns 32*QB rows and each of its NW wavefronts takes every NW-th unit of 32
// keys, with a private ring of NB units in LDS: no barrier until the end, the
// copies of a unit wait only for that wavefront's own reads.  A wavefront
// refills its K buffer once S is computed and its V buffer after the PV
// product.  The wavefronts' (m, l, O) are merged through LDS, so only NW times
// fewer key ranges, if any, go through global partials.
//
// Two tiles: 32 rows (Q in registers), and 64 rows, where each copied unit
// feeds twice the MFMAs (at d = 128 Q is then read from LDS: in registers it
// would spill beside O).  One query row streams a 32K prefix at 4.4 TB/s; with
// more rows the copies bound the 32-row tile (0.19 us per unit and CU at
// d = 128, from L2) and the copies and MFMAs together the 64-row tile (0.27).
// One layer on its own, us, 256-row tiles -> these (32 query / 8 KV heads, d
// 128): 250 + 128 tokens 20.6 -> 8.4, 1024 + 128 24.8 -> 11.3, 4096 + 128
// 28.1 -> 22.5, 32763 + 1 41.6 -> 30.4, 1024 + 512 33.4 -> 21.9.  Past some
// 500 rows over 8K keys the 256-row tiles are the faster ones (65536 + 512:
// 502 against 599).
// ---------------------------------------------------------------------------
constexpr int UNIT = 32;          // keys per unit: two pages
constexpr int NW = 8;             // wavefronts of a workgroup

template <int D, int QB>
struct WaysShape {
    static constexpr int ROWS = 32 * QB;
    static constexpr int TILE = UNIT * D;                       // elements of one K (or V) unit
    static constexpr int ND = TILE * 2 / 1024;                  // 1 KiB copies per K (or V) unit
    static constexpr int CPP = ND / 2;                          // copies per page
    static constexpr int KROWS = 512 / D;                       // key rows per copy
    static constexpr int RING = 2 * TILE * 2;                   // bytes per wavefront: a K and a V unit, ...
    static_assert(RING == 32 * D * 4, "... later the wavefront's O of 32 rows");
    static constexpr bool QLDS = QB * D > 128;                  // Q stays in LDS where it would spill
    static constexpr int Q_BYTES = QLDS ? ROWS * D * 2 : 0;
    static constexpr int LDS = NW * RING + Q_BYTES + NW * ROWS * 8;   // rings, Q, (m, l) per wavefront and row
};

template <int D, int QB>
__global__ __launch_bounds__(NW * 64) void attn_ways_kernel(KParams p) {
    using Sh = WaysShape<D, QB>;
    constexpr int ND = Sh::ND, CPP = Sh::CPP, TILE = Sh::TILE, NET = D / 32, NDS = D / 16;
    extern __shared__ __align__(1024) uint16_t lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    // ahead of ingest wavefronts on the same SIMD, as the kernel above (no
    // difference in a run's time was measured: they meet at L2, not at issue)
    __builtin_amdgcn_s_setprio(1);

    int gamma, mt;
    if (!tile_of((int)blockIdx.x, p.m_tiles, p.n_groups, true, gamma, mt)) return;
    const int g = gamma / p.n_split, split = gamma - g * p.n_split;
    const int rows = (int)p.rows, Tp = (int)p.Tp, Ts = (int)p.Ts, n_pre_pages = (int)p.n_pre_pages;
    const int grp = p.grp, nq = p.nq, nkv = p.nkv;
    const float scale_log2 = p.scale_log2;
    const __attribute__((address_space(4))) int32_t *pages_c =
        (const __attribute__((address_space(4))) int32_t *)p.pages;

    // this split's units, clipped to what the tile's last row sees
    int u0 = split * (int)p.blocks_per_split, u1 = u0 + (int)p.blocks_per_split;
    {
        int row_hi = (mt + 1) * Sh::ROWS - 1;
        if (row_hi > rows - 1) row_hi = rows - 1;
        const int last_page = n_pre_pages + row_hi / grp / PAGE;
        const int n_units = last_page / 2 + 1;
        if (u1 > n_units) u1 = n_units;
    }
    const int n = u1 > u0 + wave ? (u1 - u0 - wave + NW - 1) / NW : 0;     // units of this wavefront
    auto unit = [&](int j) { return u0 + wave + j * NW; };

    uint16_t *const ring = lds + wave * (Sh::RING / 2);
    // Per-lane parts of the copy addresses (bytes): copy c of a page covers its
    // key rows c * KROWS + rr0.  V's swizzle is the same in each (one offset,
    // the rest in the scalar base); K's is not at d = 128.
    const int rr0 = lane / (D / 8);
    uint32_t klane[CPP];
#pragma unroll
    for (int c = 0; c < CPP; ++c)
        klane[c] = (uint32_t)(rr0 * D + ((lane % (D / 8)) ^ ((c * Sh::KROWS + rr0) & (D / 8 - 1))) * 8) * 2;
    const uint32_t vlane = (uint32_t)(rr0 * D + ((lane % (D / 8)) ^ v_swz<D>(rr0)) * 8) * 2;
    auto load_pids = [&](int j, int32_t (&pid)[2]) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int v = unit(j) * 2 + h;
            pid[h] = v < n_pre_pages ? pages_c[v] : 0;
        }
    };
    // copy one unit's K (or V) rows: two pages of the pool, or suffix rows
    auto issue = [&](int j, const int32_t (&pid)[2], bool is_k, uint16_t *dst) {
        const uint16_t *const pool = is_k ? p.pool_k : p.pool_v, *const dense = is_k ? p.k_new : p.v_new;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int v = unit(j) * 2 + h;
            if (v < n_pre_pages) {
                const uint16_t *base = pool + ((int64_t)pid[h] * nkv + g) * (PAGE * D);
#pragma unroll
                for (int c = 0; c < CPP; ++c)
                    dma16(base + c * Sh::KROWS * D, is_k ? klane[c] : vlane, dst + (h * CPP + c) * 512);
            } else {
#pragma unroll
                for (int c = 0; c < CPP; ++c) {
                    // suffix token; rows past the last one repeat it (masked)
                    int T = (v - n_pre_pages) * PAGE + c * Sh::KROWS + rr0;
                    if (T > Ts - 1) T = Ts - 1;
                    const uint32_t rw = ((uint32_t)(T * nkv + g) * D - (uint32_t)rr0 * D) * 2;
                    dma16(dense, rw + (is_k ? klane[c] : vlane), dst + (h * CPP + c) * 512);
                }
            }
        }
    };
    uint16_t *const K = ring, *const V = ring + TILE;
    uint16_t *const q_lds = lds + NW * Sh::RING / 2;
    float2 *const ml = reinterpret_cast<float2 *>(reinterpret_cast<unsigned char *>(lds) + NW * Sh::RING + Sh::Q_BYTES);

    // Q: to LDS (swizzled as K), or each lane's row to registers
    bf16x8 qop[Sh::QLDS ? 1 : QB][NDS];
    int tok[QB];
    const int tok0 = mt * Sh::ROWS / grp;
    if constexpr (Sh::QLDS) {
        const uint16_t *qbase = p.q + ((int64_t)tok0 * nq + g * grp) * D;
#pragma unroll
        for (int u = 0; u < Sh::Q_BYTES / 1024 / NW; ++u) {
            const int c = u * NW + wave;
            const int r = c * Sh::KROWS + lane / (D / 8);
            int row = mt * Sh::ROWS + r;
            if (row > rows - 1) row = rows - 1;                  // rows past the last repeat it (not stored)
            const uint32_t e = (uint32_t)((row / grp - tok0) * nq + row % grp) * D +
                               ((lane % (D / 8)) ^ (r & (D / 8 - 1))) * 8;
            dma16(qbase, e * 2, q_lds + c * 512);
        }
    }
    int32_t pid[2];
    if (n > 0) {
        load_pids(0, pid);
        issue(0, pid, true, K);
        issue(0, pid, false, V);
    }
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int row = mt * Sh::ROWS + qb * 32 + col;
        const bool ok = row < rows;
        tok[qb] = ok ? row / grp : 0;
        if constexpr (!Sh::QLDS) {
            const uint16_t *qr = p.q + ((int64_t)tok[qb] * nq + g * grp + (ok ? row % grp : 0)) * D + half * 8;
#pragma unroll
            for (int ds = 0; ds < NDS; ++ds)
                qop[qb][ds] = ok ? *reinterpret_cast<const bf16x8 *>(qr + ds * 16) : bf16x8{};
        }
    }
    int voff[NET];
#pragma unroll
    for (int et = 0; et < NET; ++et) voff[et] = vt_offset<D>(lane, et);
    // LDS offsets of the S operands' first pieces; the piece of ds differs by XOR
    // with ds * 16.  With Q in LDS they are made opaque in every round, so that
    // the other pieces' offsets are computed and not kept: 243 -> 223 VGPRs, which
    // leaves registers for one ingest wavefront per SIMD beside the attention's
    // two (18400 + 63 tokens, 64 query heads, device-staged 907 -> 860 us over ten
    // layers, 12208 + 83 with 32 query heads 631 -> 604; the attention alone is
    // unchanged).
    int k_at = k_lds<D>(key_perm(col), half), q_at = k_lds<D>(col, half);

    f32x16 o[QB][NET];
    float m[QB], l[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        m[qb] = -__builtin_inff();
        l[qb] = 0.f;
#pragma unroll
        for (int et = 0; et < NET; ++et) o[qb][et] = f32x16{};
    }
    const int full_pre_pages = Tp / PAGE;
    // Q has arrived: a wait the compiler sees, so that it places none of its
    // own (for every copy in flight) inside the loop.  It waits for the first
    // unit too, which the loop needs next.
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    if constexpr (Sh::QLDS) lds_barrier();

    for (int j = 0; j < n; ++j) {
        const int u = unit(j);
        const bool refill = j + 1 < n;
        if (refill) load_pids(j + 1, pid);
        wait_vmcnt<ND>();                 // K of this unit has landed: at most its V is in flight
        f32x16 s[QB];
        {
            bf16x8 kf[NDS], qf[QB][NDS];
            if constexpr (Sh::QLDS) asm volatile("" : "+v"(k_at), "+v"(q_at));
            auto load = [&](int ds) {
                kf[ds] = *reinterpret_cast<const bf16x8 *>(&K[k_at ^ (ds * 16)]);
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
                    if constexpr (Sh::QLDS)
                        qf[qb][ds] = *reinterpret_cast<const bf16x8 *>(&q_lds[qb * 32 * D + (q_at ^ (ds * 16))]);
                    else
                        qf[qb][ds] = qop[qb][ds];
            };
            constexpr int AHEAD = Sh::QLDS ? 2 : NDS;      // operands read ahead of their use
#pragma unroll
            for (int ds = 0; ds < AHEAD; ++ds) load(ds);
#pragma unroll
            for (int ds = 0; ds < NDS; ++ds) {
                if (ds + AHEAD < NDS) load(ds + AHEAD);
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
                    s[qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ds], qf[qb][ds], ds == 0 ? f32x16{} : s[qb], 0, 0, 0);
                if constexpr (Sh::QLDS) __builtin_amdgcn_sched_barrier(0);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // K is read: its buffer may be refilled
        if (refill) issue(j + 1, pid, true, K);

        if ((u + 1) * 2 > full_pre_pages) {     // the prefix's partial last page, or suffix keys
            const int ps = n_pre_pages * PAGE - u * UNIT, pe = Tp - u * UNIT;
            const bool partial_prefix = ps > 0 && pe < (ps < UNIT ? ps : UNIT);
            const bool unseen_suffix = ps < UNIT && UNIT - 1 - ps > tok0;
            if (partial_prefix || unseen_suffix) {
                const int sh = 8 * half;
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int kin = i < 8 ? i : 8 + i;                    // key in the unit, less 8*half
                        const uint32_t keep =
                            0u - (uint32_t)((kin < pe - sh) | ((kin >= ps - sh) & (kin <= tok[qb] + ps - sh)));
                        s[qb][i] = __uint_as_float((__float_as_uint(s[qb][i]) & keep) | (0xff800000u & ~keep));
                    }
            }
        }
        // online softmax, as softmax_phase: the running maximum is raised, and
        // O rescaled, only when a unit's maximum exceeds it by 2^RESCALE_SLACK
        bf16x8 pp[QB][2];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            float mx[2] = {-__builtin_inff(), -__builtin_inff()};
#pragma unroll
            for (int i = 0; i < 16; ++i) mx[i & 1] = fmaxf(mx[i & 1], s[qb][i]);
            const float mu = half_swap_max(fmaxf(mx[0], mx[1])) * scale_log2;
            if (__any(mu > m[qb] + RESCALE_SLACK)) {
                const float mn = fmaxf(m[qb], mu);
                const float alpha = __builtin_amdgcn_exp2f(m[qb] - (mn == -__builtin_inff() ? 0.f : mn));
                m[qb] = mn;
                l[qb] *= alpha;
#pragma unroll
                for (int et = 0; et < NET; ++et) o[qb][et] *= alpha;
            }
            const float m_use = m[qb] == -__builtin_inff() ? 0.f : m[qb];
            typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
            const bf16x2 ones = {(__bf16)1.f, (__bf16)1.f};
            float ls[2] = {0.f, 0.f};
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                f32x8 e;
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    e[i] = __builtin_amdgcn_exp2f(fmaf(s[qb][hf * 8 + i], scale_log2, -m_use));
                const bf16x8 b = __builtin_convertvector(e, bf16x8);
                pp[qb][hf] = b;
                ls[0] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 0, 1), ones, ls[0], false);
                ls[1] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 2, 3), ones, ls[1], false);
                ls[0] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 4, 5), ones, ls[0], false);
                ls[1] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 6, 7), ones, ls[1], false);
            }
            l[qb] += ls[0] + ls[1];
        }
        if (refill) wait_vmcnt<ND>();     // V has landed
        else wait_vmcnt<0>();
        if ((u + 1) * 2 > full_pre_pages && u * 2 <= full_pre_pages && full_pre_pages < n_pre_pages) {
            // zero the partial prefix page's slots past Tp, which may hold
            // anything: masked keys then contribute exactly nothing
            const int pg = full_pre_pages - u * 2, k0 = Tp % PAGE;
            clear_rows<D>(V + (pg * PAGE + k0) * D, PAGE - k0, lane);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
        {
            bf16x8 vf[2 * NET];
            constexpr int AHEAD = Sh::QLDS ? 3 : 2 * NET;
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) vf[i] = load_vt<D>(V, voff, i);
#pragma unroll
            for (int i = 0; i < 2 * NET; ++i) {
                if (i + AHEAD < 2 * NET) vf[i + AHEAD] = load_vt<D>(V, voff, i + AHEAD);
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
                    o[qb][i % NET] =
                        __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[i], pp[qb][i / NET], o[qb][i % NET], 0, 0, 0);
                if constexpr (Sh::QLDS) __builtin_amdgcn_sched_barrier(0);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // V is read
        if (refill) issue(j + 1, pid, false, V);
    }

    // ---- merge the wavefronts, 32 rows at a time ----
    // Row r's 16-byte chunks are stored XOR r, so that neither the writes (one
    // row per lane) nor the reads (one chunk per lane) meet on a bank.
    constexpr int CH = D / 4;                                   // chunks of four floats per row
    float *const mine = reinterpret_cast<float *>(ring);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const float lt = half_swap_sum(l[qb]);
        if (half == 0) ml[wave * Sh::ROWS + qb * 32 + col] = float2{m[qb], lt};
    }
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        if (qb > 0) __syncthreads();                            // the last rows have been read
#pragma unroll
        for (int et = 0; et < NET; ++et)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
                const f32x4 a = {o[qb][et][vq * 4], o[qb][et][vq * 4 + 1], o[qb][et][vq * 4 + 2], o[qb][et][vq * 4 + 3]};
                const int ch = et * 8 + vq * 2 + half;
                *reinterpret_cast<f32x4 *>(mine + col * D + ((ch ^ col) & (CH - 1)) * 4) = a;
            }
        __syncthreads();
        for (int i = tid; i < 32 * CH; i += NW * 64) {
            const int r = i / CH, ch = i % CH;
            const int row = mt * Sh::ROWS + qb * 32 + r;
            if (row >= rows) break;
            float2 w[NW];
            float M = -__builtin_inff();
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                w[k] = ml[k * Sh::ROWS + qb * 32 + r];
                M = fmaxf(M, w[k].x);
            }
            const float Mu = M == -__builtin_inff() ? 0.f : M;
            float L = 0.f;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                const float e = __builtin_amdgcn_exp2f(w[k].x - Mu);
                L += e * w[k].y;
                acc += e * *reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(lds) + k * (Sh::RING / 4) +
                                                           r * D + ((ch ^ r) & (CH - 1)) * 4);
            }
            if (p.n_split == 1) {
                const float inv = L > 0.f ? 1.f / L : 0.f;
                uint16_t *orow = p.out + ((int64_t)(row / grp) * nq + g * grp + row % grp) * D;
                *reinterpret_cast<bf16x4 *>(orow + ch * 4) = __builtin_convertvector(acc * inv, bf16x4);
            } else {
                const int64_t prow = ((int64_t)split * nkv + g) * p.rows_pad + row;
                *reinterpret_cast<f32x4 *>(p.o_part + prow * D + ch * 4) = acc;
                if (ch == 0) *reinterpret_cast<float2 *>(p.ml_part + prow * 2) = float2{M, L};
            }
        }
    }
}

template <int D>
constexpr size_t attn_lds_bytes() { return (size_t)4 * 2 * KB * D * 2; }

// Merge the splits of each row: weights 2^(m_s - M), normalised by the
// matching sum of l_s; bf16 out.  Block `blk` of a request's merge covers
// RPB of its (KV head, row) pairs.
template <int D>
__device__ __forceinline__ void combine_block(const float *ml_part, const float *o_part, uint16_t *out, int nkv,
                                              int64_t rows, int64_t rows_pad, int n_split, int grp, int nq,
                                              int64_t blk) {
    constexpr int TPR = D / 4;                 // threads per row, 4 floats each
    constexpr int RPB = 256 / TPR;             // rows per block
    const int64_t gr = blk * RPB + threadIdx.x / TPR;   // over nkv * rows
    const int c4 = threadIdx.x % TPR;
    if (gr >= (int64_t)nkv * rows) return;
    const int g = (int)(gr / rows);
    const int64_t row = gr - (int64_t)g * rows;
    // One pass over the splits, eight at a time: a group's (m, l) pairs and
    // partial rows are independent loads issued together, so the merge waits
    // on memory once per group rather than once for the maxima and again
    // for the sums; the running maximum rescales what earlier groups added.
    const int64_t split_stride = (int64_t)nkv * rows_pad;
    const int64_t prow0 = (int64_t)g * rows_pad + row;
    constexpr int GS = 8;
    float M = -__builtin_inff(), L = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < n_split; s0 += GS) {
        float2 ml[GS];
        f32x4 o[GS];
#pragma unroll
        for (int i = 0; i < GS; ++i) {
            if (s0 + i < n_split) {
                const int64_t prow = prow0 + (int64_t)(s0 + i) * split_stride;
                ml[i] = *reinterpret_cast<const float2 *>(ml_part + prow * 2);
                o[i] = *reinterpret_cast<const f32x4 *>(o_part + prow * D + c4 * 4);
            }
        }
        float Mg = M;
#pragma unroll
        for (int i = 0; i < GS; ++i)
            if (s0 + i < n_split) Mg = fmaxf(Mg, ml[i].x);
        const float Mu = Mg == -__builtin_inff() ? 0.f : Mg;
        const float r = __builtin_amdgcn_exp2f(M - Mu);     // 0 while nothing has been added
        L *= r;
        acc *= r;
#pragma unroll
        for (int i = 0; i < GS; ++i) {
            if (s0 + i < n_split) {
                const float w = __builtin_amdgcn_exp2f(ml[i].x - Mu);
                L += w * ml[i].y;
                acc += w * o[i];
            }
        }
        M = Mg;
    }
    const float inv = L > 0.f ? 1.f / L : 0.f;
    const int64_t tok = row / grp;
    const int head = g * grp + (int)(row % grp);
    *reinterpret_cast<bf16x4 *>(out + (tok * nq + head) * D + c4 * 4) = __builtin_convertvector(acc * inv, bf16x4);
}

// The merge of one request, with its parameters alone as the kernel
// arguments (a lone request's launch stays short).
template <int D>
__global__ __launch_bounds__(256) void attn_combine_kernel(KParams p) {
    combine_block<D>(p.ml_part, p.o_part, p.out, p.nkv, p.rows, p.rows_pad, p.n_split, p.grp, p.nq, blockIdx.x);
}

// The merges of every request of a batch that has splits, in one launch.
template <int D>
__global__ __launch_bounds__(256) void attn_combine_batch_kernel(KBatch batch) {
    // parameters straight from the kernel-argument segment, as in the
    // attention kernel
    typedef const __attribute__((address_space(4))) KBatch *kbatch_ptr;
    const kbatch_ptr bp = (kbatch_ptr)__builtin_amdgcn_kernarg_segment_ptr();
    int req = 0;
    for (int i = 1; i < bp->n; ++i) req += (int)blockIdx.x >= bp->first_cb[i];
    const __attribute__((address_space(4))) KParams &p = bp->req[req];
    combine_block<D>(p.ml_part, p.o_part, p.out, p.nkv, p.rows, p.rows_pad, p.n_split, p.grp, p.nq,
                     (int64_t)blockIdx.x - bp->first_cb[req]);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Tiles and key blocks of one request; the split count is set apart.
static AttnPlan plan_shape(const oc_layout &lay, int64_t Tp, int64_t Ts, int tile_rows) {
    AttnPlan p{};
    p.Tp = Tp;
    p.Ts = Ts;
    p.nq = lay.num_q_heads;
    p.nkv = lay.num_kv_heads;
    p.grp = p.nq / p.nkv;
    p.d = lay.head_dim;
    p.rows = Ts * p.grp;
    p.tile_rows = tile_rows;
    p.m_tiles = (int)((p.rows + p.tile_rows - 1) / p.tile_rows);
    p.n_pre_pages = (Tp + PAGE - 1) / PAGE;
    p.n_suf_pages = (Ts + PAGE - 1) / PAGE;
    const int pages_per_block = (tile_rows == TILE_ROWS ? KB : UNIT) / PAGE;
    p.n_blocks = (p.n_pre_pages + p.n_suf_pages + pages_per_block - 1) / pages_per_block;
    return p;
}

// Split the keys into ns ranges, then size the workspace.
static void plan_splits(AttnPlan &p, int64_t ns) {
    if (ns > p.n_blocks) ns = p.n_blocks;
    if (ns < 1) ns = 1;
    p.blocks_per_split = (p.n_blocks + ns - 1) / ns;
    p.n_split = (int)((p.n_blocks + p.blocks_per_split - 1) / p.blocks_per_split);
    const int64_t rows_pad = (int64_t)p.m_tiles * p.tile_rows;
    size_t off = 0;
    p.off_o = off;
    if (p.n_split > 1) off = round_up(off + (size_t)p.n_split * p.nkv * rows_pad * p.d * 4, 256);
    p.off_ml = off;
    if (p.n_split > 1) off = round_up(off + (size_t)p.n_split * p.nkv * rows_pad * 2 * 4, 256);
    p.total = off > 256 ? off : 256;   // never 0: a size of 0 reports an unsupported shape
}

// Estimated time (us) of one request's attention under a plan: the rule that
// picks the row tile and the split count.  Fitted to 192 shapes (n_q/n_kv/d of
// 32/8/128, 64/8/128, 4/1/128, 32/4/64, 8/8/64, 4/2/64; prefixes of 100 to
// 50000 tokens, suffixes of 1 to 1600) with up to 40 plans each: over them the
// plan it picks is 1 % slower than the best one measured, on average.  Over 500
// other shapes (prefixes of 1 to 65536 tokens, suffixes of 1 to 3584) it takes
// 0.70 times as long as 256-row tiles alone did before there were others; it
// loses 2 to 7 % on three of them (64/8/128 with 21449 + 17 tokens: 38.3 us,
// 35.8), where the merge of many splits costs less than estimated.
struct PlanCost {
    double block128, block64;   // one key block of one workgroup, at d = 128 and 64
    double round;               // the least time of one block per wavefront
    double start, spread;       // launch, first copies, epilogue; extra when every CU holds a workgroup
    double wave;                // each further workgroup per CU
};
static const PlanCost COST_32 = {0.182, 0.112, 0.63, 4.2, 3.2, 1.4}, COST_64 = {0.259, 0.167, 1.38, 5.6, 3.5, 3.8},
                      COST_256 = {1.45, 1.15, 0.88, 6.2, 1.6, 1.0};

static double plan_cost(const AttnPlan &p) {
    const PlanCost &k = p.tile_rows == 32 ? COST_32 : p.tile_rows == 64 ? COST_64 : COST_256;
    const double tiles = (double)p.nkv * p.m_tiles, wgs = tiles * p.n_split, bps = (double)p.blocks_per_split;
    // average share of the key blocks a row tile sees under the causal mask
    const double pages = (double)(p.n_pre_pages + p.n_suf_pages);
    const double seen = p.m_tiles > 1 ? (p.n_pre_pages + 0.5 * (p.n_suf_pages + 1)) / pages : 1.0;
    const double per_cu = wgs / TARGET_WGS;
    const double block = p.d == 128 ? k.block128 : k.block64;
    double body = block * bps;
    if (per_cu > 1) body *= seen * std::max(1.0, std::min(std::ceil(per_cu), per_cu + 0.55));
    body = std::max(body, k.round * (p.tile_rows == TILE_ROWS ? 1.0 : std::ceil(bps / NW)));
    // all inputs and the output once at 5 TB/s
    const double hbm = 4.0 * p.d * ((double)p.nq * p.Ts + (double)p.nkv * (p.Tp + p.Ts)) / 5e6;
    body = std::sqrt(body * body + hbm * hbm);
    double t = k.start + k.spread * std::min(per_cu, 1.0) + body;
    if (per_cu > 1) t += k.wave * (std::ceil(per_cu) - 1);
    // the merge's launch, and its partials written and read
    if (p.n_split > 1) t += 2.4 + 0.556e-6 * p.n_split * p.nkv * p.rows * p.d * 4;
    return t;
}

// One request alone.  256-row tiles with the keys split so that they fill the
// CUs; or another tile or split count where the estimate says that it is at
// least 4 % faster.  The workspace asked for is always that of the first plan
// (a caller may hold one of that size), so a plan that needs more is left.
int plan_attention(const oc_layout &lay, int64_t Tp, int64_t Ts, AttnPlan *pl) {
    AttnPlan best = plan_shape(lay, Tp, Ts, TILE_ROWS);
    const int64_t fill = (TARGET_WGS + (int64_t)best.nkv * best.m_tiles - 1) / ((int64_t)best.nkv * best.m_tiles);
    plan_splits(best, fill);
    const size_t ws_bytes = best.total;
    double least = 0.96 * plan_cost(best);
    for (const int tile : {32, 64, TILE_ROWS}) {
        // the 64-row tile copies its Q rows with 32-bit offsets from its first token's
        if (tile == 64 && (int64_t)65 * lay.num_q_heads * lay.head_dim * 2 > INT32_MAX) continue;
        AttnPlan p = plan_shape(lay, Tp, Ts, tile);
        const int64_t tiles = (int64_t)p.nkv * p.m_tiles;
        if (tiles > 4 * TARGET_WGS && tile != TILE_ROWS) continue;     // long suffixes: whole 256-row tiles
        for (const int ns : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 24, 32, 48, 64, 96, 128}) {
            if (ns > 1 && (ns > p.n_blocks || ns * tiles > 2 * TARGET_WGS)) break;
            if (tile == TILE_ROWS && ns > fill) break;
            plan_splits(p, ns);
            if (p.total > ws_bytes) continue;
            const double t = plan_cost(p);
            if (t < least) {
                least = t;
                best = p;
            }
        }
    }
    best.total = ws_bytes;
    *pl = best;
    return OC_OK;
}

// Several requests in one launch: every workgroup gets at most `budget` key
// blocks, the smallest budget that keeps the launch within BATCH_ROUNDS
// workgroups per CU (or one range per tile, if there are more tiles), so the
// dispatcher can even out long and short prefixes as CUs free up.
int plan_attention_batch(const oc_layout &lay, const int64_t *Tp, const int64_t *Ts, int n, AttnPlan *plans) {
    int64_t tiles = 0, work = 0, longest = 1;
    for (int i = 0; i < n; ++i) {
        plans[i] = plan_shape(lay, Tp[i], Ts[i], TILE_ROWS);
        const int64_t t = (int64_t)plans[i].nkv * plans[i].m_tiles;
        tiles += t;
        work += t * plans[i].n_blocks;
        longest = std::max<int64_t>(longest, plans[i].n_blocks);
    }
    auto wgs_for = [&](int64_t budget) {
        int64_t w = 0;
        for (int i = 0; i < n; ++i)
            w += (int64_t)plans[i].nkv * plans[i].m_tiles * ((plans[i].n_blocks + budget - 1) / budget);
        return w;
    };
    const int64_t cap = std::max<int64_t>((int64_t)TARGET_WGS * BATCH_ROUNDS, tiles);
    int64_t budget = std::max<int64_t>(1, (work + cap - 1) / cap);
    while (budget < longest && wgs_for(budget) > cap) ++budget;
    for (int i = 0; i < n; ++i) plan_splits(plans[i], (plans[i].n_blocks + budget - 1) / budget);
    return OC_OK;
}

int attention_registers(const AttnPlan &p) {
    const void *f = reinterpret_cast<const void *>(
        p.tile_rows == 32   ? (p.d == 128 ? &attn_ways_kernel<128, 1> : &attn_ways_kernel<64, 1>)
        : p.tile_rows == 64 ? (p.d == 128 ? &attn_ways_kernel<128, 2> : &attn_ways_kernel<64, 2>)
                            : nullptr);
    if (!f) f = reinterpret_cast<const void *>(p.d == 128 ? &attn_fwd_kernel<128> : &attn_fwd_kernel<64>);
    hipFuncAttributes a{};
    return hipFuncGetAttributes(&a, f) == hipSuccess ? a.numRegs : -1;
}

int64_t attention_grid(const AttnPlan &p) {
    const int64_t groups = (int64_t)p.nkv * p.n_split;
    if (groups <= INT32_MAX && tiles_by_xcd(p.m_tiles, (int)groups, p.tile_rows != TILE_ROWS))
        return (groups + 7) / 8 * 8 * p.m_tiles;
    return (groups * p.m_tiles + 7) / 8 * 8;
}

bool attention_tile(int wg, const AttnPlan &p, int *group, int *row_tile) {
    return tile_of(wg, p.m_tiles, p.nkv * p.n_split, p.tile_rows != TILE_ROWS, *group, *row_tile);
}

// a dispatch holds at most 2^32 - 1 work-items along x
int64_t attention_max_grid() { return OC_MAX_GRID_ITEMS / THREADS; }

size_t attention_lds_bytes(const AttnPlan &p) {
    if (p.tile_rows == 32) return p.d == 128 ? WaysShape<128, 1>::LDS : WaysShape<64, 1>::LDS;
    if (p.tile_rows == 64) return p.d == 128 ? WaysShape<128, 2>::LDS : WaysShape<64, 2>::LDS;
    return p.d == 128 ? attn_lds_bytes<128>() : attn_lds_bytes<64>();
}

int check_attention_shape(const oc_layout &l, int64_t Tp, int64_t Ts, AttnPlan *plan) {
    if (l.head_dim != 64 && l.head_dim != 128) return fail(OC_ESHAPE, "attention supports head_dim 64 or 128");
    if (l.page_size != PAGE) return fail(OC_ESHAPE, "attention supports page_size 16");
    if (Tp < 0 || Ts < 1) return fail(OC_EINVAL, "attention needs prefix_tokens >= 0 and suffix_tokens >= 1");
    // the suffix rows are copied to LDS with 32-bit byte offsets from k_new / v_new
    if (Ts * l.num_kv_heads * l.head_dim * 2 > INT32_MAX)
        return fail(OC_ERANGE, "suffix K/V of more than 2^31 bytes (suffix_tokens * n_kv * d * 2)");
    // key positions, query rows and their tokens are 32-bit in the kernels
    if (Tp + Ts > (int64_t)1 << 30) return fail(OC_ERANGE, "prefix + suffix tokens exceed 2^30");
    const int64_t grp = l.num_q_heads / l.num_kv_heads;
    if (Ts * grp > (int64_t)1 << 30) return fail(OC_ERANGE, "suffix_tokens * (n_q / n_kv) exceeds 2^30");
    AttnPlan p;
    if (!plan) plan = &p;
    plan_attention(l, Tp, Ts, plan);
    if (attention_grid(*plan) > attention_max_grid())
        return fail(OC_ERANGE, "attention grid of more than " + std::to_string(attention_max_grid()) + " workgroups");
    // the split merge runs d/4 work-items per (KV head, row)
    if ((int64_t)plan->nkv * plan->rows * (plan->d / 4) > OC_MAX_GRID_ITEMS)
        return fail(OC_ERANGE, "split merge grid exceeds 2^32 work-items");
    return OC_OK;
}

template <int D>
static KParams make_params(const AttnPlan &pl, const AttnArgs &a) {
    KParams p{};
    p.q = a.q;
    p.pool_k = a.pool_k;
    p.pool_v = a.pool_v;
    p.pages = a.pages;
    p.k_new = a.k_new;
    p.v_new = a.v_new;
    p.o_part = reinterpret_cast<float *>(a.ws + pl.off_o);
    p.ml_part = reinterpret_cast<float *>(a.ws + pl.off_ml);
    p.out = a.out;
    p.Tp = pl.Tp;
    p.Ts = pl.Ts;
    p.rows = pl.rows;
    p.rows_pad = (int64_t)pl.m_tiles * pl.tile_rows;
    p.n_pre_pages = pl.n_pre_pages;
    p.n_suf_pages = pl.n_suf_pages;
    p.n_blocks = pl.n_blocks;
    p.blocks_per_split = pl.blocks_per_split;
    p.nq = pl.nq;
    p.nkv = pl.nkv;
    p.grp = pl.grp;
    p.m_tiles = pl.m_tiles;
    p.n_split = pl.n_split;
    p.n_groups = pl.nkv * pl.n_split;
    p.scale_log2 = (float)(1.4426950408889634 / sqrt((double)D));
    return p;
}

template <int D>
static hipError_t launch_d(const AttnPlan *pl, const AttnArgs *a, int n, hipStream_t s) {
    // requests with the longest workgroups first: the dispatcher then fills
    // the tail of the launch with short ones
    int order[MAX_ATTN_BATCH];
    for (int i = 0; i < n; ++i) order[i] = i;
    std::stable_sort(order, order + n, [&](int x, int y) { return pl[x].blocks_per_split > pl[y].blocks_per_split; });
    KBatch batch{};
    batch.n = n;
    int64_t grid = 0;
    for (int k = 0; k < n; ++k) {
        const int i = order[k];
        batch.req[k] = make_params<D>(pl[i], a[i]);
        batch.first_wg[k] = (int32_t)grid;
        grid += attention_grid(pl[i]);
    }
    if (grid > attention_max_grid()) return hipErrorInvalidConfiguration;
    const hipError_t e = allow_dynamic_lds<&attn_fwd_kernel<D>>((int)attn_lds_bytes<D>());
    if (e != hipSuccess) return e;
    if (grid > 0) hipLaunchKernelGGL(attn_fwd_kernel<D>, dim3((unsigned)grid), dim3(THREADS), attn_lds_bytes<D>(), s, batch);
    // the split merge of every request that has splits, in one launch
    constexpr int RPB = 256 / (D / 4);
    int64_t cblocks[MAX_ATTN_BATCH], ctotal = 0;
    for (int k = 0; k < n; ++k) {
        cblocks[k] = batch.req[k].n_split > 1 ? ((int64_t)batch.req[k].nkv * batch.req[k].rows + RPB - 1) / RPB : 0;
        batch.first_cb[k] = (int32_t)std::min<int64_t>(ctotal, INT32_MAX);
        ctotal += cblocks[k];
    }
    const int with_splits = (int)std::count_if(cblocks, cblocks + n, [](int64_t c) { return c > 0; });
    if (with_splits > 1 && ctotal * 256 <= OC_MAX_GRID_ITEMS) {
        hipLaunchKernelGGL(attn_combine_batch_kernel<D>, dim3((unsigned)ctotal), dim3(256), 0, s, batch);
    } else {
        // one request with splits, or too many rows for one dispatch: one
        // merge per request (each fits, as the shape checks require)
        for (int k = 0; k < n; ++k)
            if (cblocks[k])
                hipLaunchKernelGGL(attn_combine_kernel<D>, dim3((unsigned)cblocks[k]), dim3(256), 0, s,
                                   batch.req[k]);
    }
    return hipGetLastError();
}

template <int D, int QB>
static hipError_t launch_ways(const AttnPlan &pl, const AttnArgs &a, hipStream_t s) {
    using Sh = WaysShape<D, QB>;
    static_assert(Sh::LDS <= (int)CU_LDS_BYTES, "rings larger than the LDS");
    const KParams p = make_params<D>(pl, a);
    const hipError_t e = allow_dynamic_lds<&attn_ways_kernel<D, QB>>(Sh::LDS);
    if (e != hipSuccess) return e;
    const int64_t grid = attention_grid(pl);
    static_assert(NW * 64 == THREADS, "the grid's limit is shared");
    if (grid > attention_max_grid()) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((attn_ways_kernel<D, QB>), dim3((unsigned)grid), dim3(NW * 64), Sh::LDS, s, p);
    if (p.n_split > 1) {
        constexpr int RPB = 256 / (D / 4);
        const int64_t blocks = ((int64_t)p.nkv * p.rows + RPB - 1) / RPB;
        hipLaunchKernelGGL(attn_combine_kernel<D>, dim3((unsigned)blocks), dim3(256), 0, s, p);
    }
    return hipGetLastError();
}

hipError_t launch_attention(const AttnPlan &pl, const AttnArgs &a, hipStream_t s) {
    if (pl.tile_rows == 32) return pl.d == 128 ? launch_ways<128, 1>(pl, a, s) : launch_ways<64, 1>(pl, a, s);
    if (pl.tile_rows == 64) return pl.d == 128 ? launch_ways<128, 2>(pl, a, s) : launch_ways<64, 2>(pl, a, s);
    if (pl.d == 128) return launch_d<128>(&pl, &a, 1, s);
    return launch_d<64>(&pl, &a, 1, s);
}

hipError_t launch_attention_batch(const AttnPlan *pl, const AttnArgs *a, int n, hipStream_t s) {
    if (n < 1 || n > MAX_ATTN_BATCH) return hipErrorInvalidValue;
    if (pl[0].d == 128) return launch_d<128>(pl, a, n, s);
    return launch_d<64>(pl, a, n, s);
}

}  // namespace oc
