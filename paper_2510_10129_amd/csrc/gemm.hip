// bf16 MFMA GEMMs of the recompute path: C[M,N] = A[M,K] * B[N,K]^T with fp32
// accumulation, where A holds the (few) recomputed rows and B a weight matrix
// stored [out][in].  Four fused epilogues:
//   QKV     bias + rotary embedding at the token's global position, q to the
//           query buffer, k/v scattered into the KV cache rows idx[i]
//   OPROJ   + residual (gathered hidden row) -> fp32 residual stream
//   GATE_UP B tile = 64 gate rows + 64 up rows; writes silu(gate)*up
//   DOWN    + residual stream -> bf16 layer output
//
// Tiling: one workgroup of WAVES_M x WAVES_N waves computes a BM x BN tile.  Operands
// go from global memory straight into LDS (16-byte global->LDS loads, no register
// staging), XOR-swizzled so that the 16-byte fragment reads are conflict-free on the
// 64-bank LDS.  Six K loops:
//   ping-pong (K % 128 == 0; gemm_pingpong_kernel, the 256x256 tile) two LDS buffers of
//          64 columns filled half tile by half tile, four phases per 64 columns, the two
//          waves of a SIMD alternating between fragment reads and MFMAs.
//   duo    (K % 128 == 0; gemm_duo_kernel, 256x128 and 128x128 where K is not short) K tiles of
//          64 columns, 64x64 waves in two groups, a whole K tile per turn.
//   ring16 (K % 128 == 0; gemm_ring16_kernel, 128x128 where K is short) slices of 32 columns
//          in a ring of four LDS slots; a slice is requested three slices (96 columns of
//          MFMA work) before it is read, which hides the L2/fabric latency that a
//          two-stage pipeline exposes; one barrier per slice, waits by explicit vmcnt;
//          v_mfma_f32_16x16x32_bf16 (one k-step per slice) with hand-written fragment
//          reads and hand-counted lgkmcnt waits.
//   thin   (any K % 64 == 0; gemm_thin_kernel, 64x128 tiles) for few rows: six slots of 64
//          columns, so that the weight stream keeps five of them on the way.
//   ring   (gemm_ring_kernel) the same ring with v_mfma_f32_32x32x16_bf16 and
//          compiler-scheduled fragment reads; kept as a cross-check behind
//          cc_debug_set_launch.
//   staged (any K % 64 == 0; gemm_nt_kernel) two stages of 64 columns, one barrier
//          per stage, 32x32x16 MFMAs.
// The accumulators are written back through LDS so that every global store is
// 16 or 32 contiguous bytes per lane along the row; those of the ping-pong loop, but for QKV and for
// shares of a grid with many rows past M, from the registers, 16 bytes a lane.
#include "cc_internal.h"
#include "launch_plan.h"
#include <algorithm>
#include <type_traits>

namespace {

struct BSingle {
    const bf16_t* B;
    int ldb, N;
    template <int BN>
    __device__ __forceinline__ const bf16_t* row(int bn, int r) const {
        int n = bn * BN + r;
        n = n < N ? n : N - 1;
        return B + (int64_t)n * ldb;
    }
    // ring loop: tile rows [half*BN/2, (half+1)*BN/2) start at base() and there are
    // rows_left() valid rows from there (rows past the end are clamped by the caller)
    template <int BN>
    __device__ __forceinline__ const bf16_t* base(int bn, int half) const {
        int n0 = bn * BN + half * (BN / 2);
        n0 = n0 < N ? n0 : N - 1;
        return B + (int64_t)n0 * ldb;
    }
    template <int BN>
    __device__ __forceinline__ int rows_left(int bn, int half) const {
        const int l = N - bn * BN - half * (BN / 2);
        return l < 1 ? 1 : l;
    }
};

// rows [0, BN/2) of the tile come from B0 (gate), rows [BN/2, BN) from B1 (up)
struct BDual {
    const bf16_t* B0;
    const bf16_t* B1;
    int ldb, f;
    template <int BN>
    __device__ __forceinline__ const bf16_t* row(int bn, int r) const {
        constexpr int H = BN / 2;
        int n = bn * H + (r < H ? r : r - H);
        n = n < f ? n : f - 1;
        return (r < H ? B0 : B1) + (int64_t)n * ldb;
    }
    template <int BN>
    __device__ __forceinline__ const bf16_t* base(int bn, int half) const {
        int n0 = bn * (BN / 2);
        n0 = n0 < f ? n0 : f - 1;
        return (half ? B1 : B0) + (int64_t)n0 * ldb;
    }
    template <int BN>
    __device__ __forceinline__ int rows_left(int bn, int half) const {
        const int l = f - bn * (BN / 2);
        return l < 1 ? 1 : l;
    }
};

__device__ __forceinline__ void store_bf16x8(bf16_t* dst, const float* v) {
    bf16x8 o;
#pragma unroll
    for (int u = 0; u < 8; ++u) o[u] = (bf16_t)v[u];
    *reinterpret_cast<bf16x8*>(dst) = o;
}

// Two quads of bf16 columns per lane, as the matrix instruction with its operands exchanged leaves them (lane L
// has columns 4 (L/16) .. + 3 of two 16-column tiles j): lanes of odd 16-lane rows trade tile 0 for tile 1 with the row
// below, after which each has 8 columns in a row, from column 16 (L/16 % 2) + 8 (L/32) on.
__device__ __forceinline__ bf16x8 eight_columns(const f32x4& t0, const f32x4& t1) {
    union { bf16_t h[4]; uint32_t u[2]; } a, b;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        a.h[v] = (bf16_t)t0[v];
        b.h[v] = (bf16_t)t1[v];
    }
    union { bf16x8 v; uint32_t u[4]; } o;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const auto sw = __builtin_amdgcn_permlane16_swap(a.u[k], b.u[k], false, false);
        o.u[k] = sw[0];
        o.u[2 + k] = sw[1];
    }
    return o.v;
}

// What an epilogue does with 8 columns of a staged fp32 row (column c of it at c ^ swz).  `pre` loads what it needs from
// memory besides, by the row's key (a load of its own), so that a kernel can ask for both early; ASKS_BY_KEY: `pre` loads at an
// address that the key gives.  COLS: tile columns that
// make one output column.  A tile's threads are dealt over BN / COLS columns: with gate and up dealt over all BN, the
// half at the up columns had nothing to do and each row cost twice its passes (gate/up of 3404 rows and d = 2048
// 199.0 -> 182.9 us, d = 4096 593.4 -> 571.6; 883 rows 175.9 -> 167.3; 8192 rows 1332.7 -> 1282.2).
// DIRECT: the ping-pong loop stores from its accumulators.  `two` takes a lane's quads of columns c and c + 16 of a row (c with
// the lane's own 4 (L/16)), for which `ask` has loaded what it needs, every lane of the wave with it (`on`: the row exists).
// A lane turns both columns of its rotary pairs: with a lane per 8 columns either side read the other's sums and the same 64
// bytes of rotary pairs again (us, before -> after: 8192 rows, d = 4096 323.3 -> 308.2, d = 2048 118.0 -> 108.2; 3404 rows
// 162.7 -> 156.7 and 59.5 -> 52.9; 883 rows, d = 4096 63.1 -> 60.6; 237 rows, d = 256 8.2 -> 7.4).
struct EpiQKV {
    static constexpr int COLS = 2;                         // the two columns of a rotary pair (of a head of V: c and c + d_h/2)
    static constexpr bool ASKS_BY_KEY = false;
    static constexpr bool DIRECT = false;                  // a column's rotary partner is in another wave
    const int32_t* idx;
    const bf16_t* bias;
    const float2* rope;
    int H_q, H_kv, d_h, N;
    bf16_t* q_out;
    bf16_t* K;
    bf16_t* V;
    int64_t st, sh;
    // the rotary pairs are not asked for early: 64 bytes a lane from rows far apart, 1 us more for thin tiles of a short K
    struct Pre {
        int pos;
    };
    __device__ __forceinline__ int key(int m) const { return idx[m]; }
    template <int BN>
    __device__ __forceinline__ Pre pre(int, int, int, int pos) const { return {pos}; }
    // cc counts pairs: 8 columns of a head's first half and the 8 they are rotated with
    template <int BN>
    __device__ __forceinline__ void operator()(int m, int bn, int cc, const float* crow, int swz, const Pre& pr) const {
        const int half = d_h >> 1, hd = cc / half, j = cc - hd * half;
        const int lo = hd * d_h + j, n = bn * BN + lo;     // a tile holds whole heads
        if (n >= N) return;
        const int head = n / d_h;
        float v[8], p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            v[u] = crow[(lo ^ swz) + u];
            p[u] = crow[((lo + half) ^ swz) + u];
        }
        if (bias) {
            const bf16x8 b = *reinterpret_cast<const bf16x8*>(bias + n), b2 = *reinterpret_cast<const bf16x8*>(bias + n + half);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                v[u] += (float)b[u];
                p[u] += (float)b2[u];
            }
        }
        if (head < H_q + H_kv) {
            const float2* cs = rope + (int64_t)pr.pos * half + j;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float2 t = cs[u];
                const float x = v[u];
                v[u] = x * t.x - p[u] * t.y;
                p[u] = p[u] * t.x + x * t.y;
            }
        }
        bf16_t* dst;
        if (head < H_q)
            dst = q_out + (int64_t)m * H_q * d_h + n;
        else if (head < H_q + H_kv)
            dst = K + (int64_t)pr.pos * st + (int64_t)(head - H_q) * sh + j;
        else
            dst = V + (int64_t)pr.pos * st + (int64_t)(head - H_q - H_kv) * sh + j;
        store_bf16x8(dst, v);
        store_bf16x8(dst + half, p);
    }
    template <int BN>
    __device__ __forceinline__ void operator()(int m, int bn, int cc, const float* crow, int swz) const {
        operator()<BN>(m, bn, cc, crow, swz, pre<BN>(m, bn, cc, key(m)));
    }
};

struct EpiOProj {
    static constexpr int COLS = 1;
    static constexpr bool ASKS_BY_KEY = true;
    static constexpr bool DIRECT = true;
    const bf16_t* hidden;
    const int32_t* gather_idx;
    int d;
    float* y;
    struct Pre {
        bf16x8 x;
    };
    __device__ __forceinline__ int key(int m) const { return gather_idx ? gather_idx[m] : m; }
    template <int BN>
    __device__ __forceinline__ Pre pre(int, int bn, int cc, int src) const {
        Pre p;
        const int n = bn * BN + cc;
        if (n >= d) return p;
        p.x = *reinterpret_cast<const bf16x8*>(hidden + (int64_t)src * d + n);
        return p;
    }
    template <int BN>
    __device__ __forceinline__ void operator()(int m, int bn, int cc, const float* crow, int swz) const {
        operator()<BN>(m, bn, cc, crow, swz, pre<BN>(m, bn, cc, key(m)));
    }
    template <int BN>
    __device__ __forceinline__ void operator()(int m, int bn, int cc, const float* crow, int swz, const Pre& p) const {
        const int n = bn * BN + cc;
        if (n >= d) return;
        const bf16x8 x = p.x;
        const float* cr = crow + (cc ^ swz);
        f32x4 a, b;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            a[u] = cr[u] + (float)x[u];
            b[u] = cr[4 + u] + (float)x[4 + u];
        }
        f32x4* dst = reinterpret_cast<f32x4*>(y + (int64_t)m * d + n);
        dst[0] = a;
        dst[1] = b;
    }
    struct Two {
        bf16x4 x[2];
    };
    template <int BN>
    __device__ __forceinline__ Two ask(int, int bn, int c, int src) const {
        Two t;
        const int n = bn * BN + c;
#pragma unroll
        for (int j = 0; j < 2; ++j) t.x[j] = *reinterpret_cast<const bf16x4*>(hidden + (int64_t)src * d + min(n + 16 * j, d - 4));
        return t;
    }
    template <int BN>
    __device__ __forceinline__ void two(int m, int bn, int c, int, const f32x4 (&t)[2], const Two& p, bool on) const {
        const int n = bn * BN + c;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            f32x4 a;
#pragma unroll
            for (int u = 0; u < 4; ++u) a[u] = t[j][u] + (float)p.x[j][u];
            if (on && n + 16 * j < d) *reinterpret_cast<f32x4*>(y + (int64_t)m * d + n + 16 * j) = a;
        }
    }
};

struct EpiGateUp {
    int f;
    bf16_t* act;
    static constexpr int COLS = 2;                         // a gate and an up column
    static constexpr bool ASKS_BY_KEY = false;
    static constexpr bool DIRECT = true;
    struct Pre {};
    __device__ __forceinline__ int key(int) const { return 0; }
    template <int BN>
    __device__ __forceinline__ Pre pre(int, int, int, int) const { return {}; }
    template <int BN>
    __device__ __forceinline__ void operator()(int m, int bn, int cc, const float* crow, int swz, const Pre& = {}) const {
        constexpr int H = BN / 2;
        const int n = bn * H + cc;                         // cc < H
        if (n >= f) return;
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            float g = crow[(cc ^ swz) + u], up = crow[((cc + H) ^ swz) + u];
            v[u] = g / (1.0f + __expf(-g)) * up;
        }
        store_bf16x8(act + (int64_t)m * f + n, v);
    }
    template <int BN>
    __device__ __forceinline__ void two(int m, int bn, int c, int fk, const f32x4 (&g)[2], const f32x4 (&up)[2], bool on) const {
        f32x4 t[2];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int u = 0; u < 4; ++u) t[j][u] = g[j][u] / (1.0f + __expf(-g[j][u])) * up[j][u];
        const bf16x8 o = eight_columns(t[0], t[1]);
        const int n = bn * (BN / 2) + c - 4 * fk + (fk & 1) * 16 + (fk >> 1) * 8;
        if (on && n < f) *reinterpret_cast<bf16x8*>(act + (int64_t)m * f + n) = o;
    }
};

struct EpiDown {
    static constexpr int COLS = 1;
    static constexpr bool ASKS_BY_KEY = false;
    static constexpr bool DIRECT = true;
    const float* y;
    int d;
    bf16_t* out;
    struct Pre {
        f32x4 a, b;
    };
    __device__ __forceinline__ int key(int) const { return 0; }
    template <int BN>
    __device__ __forceinline__ Pre pre(int m, int bn, int cc, int) const {
        Pre p;
        const int n = bn * BN + cc;
        if (n >= d) return p;
        const f32x4* r = reinterpret_cast<const f32x4*>(y + (int64_t)m * d + n);
        p.a = r[0];
        p.b = r[1];
        return p;
    }
    template <int BN>
    __device__ __forceinline__ void operator()(int m, int bn, int cc, const float* crow, int swz) const {
        operator()<BN>(m, bn, cc, crow, swz, pre<BN>(m, bn, cc, key(m)));
    }
    template <int BN>
    __device__ __forceinline__ void operator()(int m, int bn, int cc, const float* crow, int swz, const Pre& p) const {
        const int n = bn * BN + cc;
        if (n >= d) return;
        const f32x4 a = p.a, b = p.b;
        const float* cr = crow + (cc ^ swz);
        float v[8];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            v[u] = cr[u] + a[u];
            v[4 + u] = cr[4 + u] + b[u];
        }
        store_bf16x8(out + (int64_t)m * d + n, v);
    }
    struct Two {
        f32x4 x[2];
    };
    template <int BN>
    __device__ __forceinline__ Two ask(int m, int bn, int c, int) const {
        Two t;
        const int n = bn * BN + c;
#pragma unroll
        for (int j = 0; j < 2; ++j) t.x[j] = *reinterpret_cast<const f32x4*>(y + (int64_t)m * d + min(n + 16 * j, d - 4));
        return t;
    }
    template <int BN>
    __device__ __forceinline__ void two(int m, int bn, int c, int fk, const f32x4 (&t)[2], const Two& p, bool on) const {
        const bf16x8 o = eight_columns(t[0] + p.x[0], t[1] + p.x[1]);
        const int n = bn * BN + c - 4 * fk + (fk & 1) * 16 + (fk >> 1) * 8;
        if (on && n < d) *reinterpret_cast<bf16x8*>(out + (int64_t)m * d + n) = o;
    }
};

// Split-K: workgroup row blockIdx.y computes the products over its share of K: `K` columns, the first
// k_more rows one unit of UNIT columns more.  Returns the share's columns.
template <int UNIT>
__device__ __forceinline__ int k_share(int K, int k_more, int64_t* first_byte) {
    const int y = blockIdx.y;
    *first_byte = ((int64_t)y * K + min(y, k_more) * UNIT) * 2;
    return K + (y < k_more ? UNIT : 0);
}
// It leaves its fp32 tile in a workspace [share][tile slot][ROWS][BN] (slot = the tile's index
// within the launch); splitk_finish_kernel adds the shares and applies the launch's own
// epilogue functor.
template <int ROWS>
struct EpiPartial {
    static constexpr int COLS = 1;
    static constexpr bool ASKS_BY_KEY = false;
    static constexpr bool DIRECT = true;
    float* ws;
    int64_t share_stride;     // floats per share: slots * ROWS * BN
    int slot, m0;             // set by the kernel: this workgroup's slot and first row
    struct Pre {};
    __device__ __forceinline__ int key(int) const { return 0; }
    template <int BN>
    __device__ __forceinline__ Pre pre(int, int, int, int) const { return {}; }
    template <int BN>
    __device__ __forceinline__ void operator()(int m, int bn, int cc, const float* crow, int swz, const Pre& = {}) const {
        float* dst = ws + blockIdx.y * share_stride + (int64_t)slot * (ROWS * BN) + (m - m0) * BN + cc;
        const f32x4* cr = reinterpret_cast<const f32x4*>(crow + (cc ^ swz));
        reinterpret_cast<f32x4*>(dst)[0] = cr[0];
        reinterpret_cast<f32x4*>(dst)[1] = cr[1];
    }
    struct Two {};
    template <int BN>
    __device__ __forceinline__ Two ask(int, int, int, int) const { return {}; }
    template <int BN>
    __device__ __forceinline__ void two(int m, int, int c, int, const f32x4 (&t)[2], const Two&, bool on) const {
        float* dst = ws + blockIdx.y * share_stride + (int64_t)slot * (ROWS * BN) + (m - m0) * BN + c;
        if (!on) return;
        reinterpret_cast<f32x4*>(dst)[0] = t[0];
        reinterpret_cast<f32x4*>(dst)[4] = t[1];
    }
};
template <class Epi>
__device__ __forceinline__ Epi epi_for_tile(const Epi& e, int, int) { return e; }
template <int ROWS>
__device__ __forceinline__ EpiPartial<ROWS> epi_for_tile(const EpiPartial<ROWS>& e, int slot, int m0) {
    EpiPartial<ROWS> r = e;
    r.slot = slot;
    r.m0 = m0;
    return r;
}

__device__ __forceinline__ void tile_of_seq(int vb, int tiles_m, int tiles_n, int GM, int* bm, int* bn);

// One workgroup per 2048 / BN rows of one tile slot: sums the shares of each 8-column chunk into an
// LDS row, then every thread calls the functor on its chunk (functors may read other chunks of the
// row: the RoPE partner, the up half of a gate/up tile).  The loads of four shares are issued
// together; the shares are added in ascending order.
template <int SLOT_ROWS, int BN, class Epi>
__global__ __launch_bounds__(256) void splitk_finish_kernel(const float* __restrict__ ws, int64_t share_stride,
                                                            int n_shares, int M, int BM, int vb0, int tiles_m,
                                                            int tiles_n, int GM, Epi epi) {
    constexpr int TPR = BN / 8, ROWS = 256 / TPR;
    __shared__ __align__(16) float stage[ROWS][BN];
    const int r = threadIdx.x / TPR, cc = (threadIdx.x % TPR) * 8;
    int bm, bn;
    tile_of_seq(vb0 + blockIdx.x, tiles_m, tiles_n, GM, &bm, &bn);
    const int row = blockIdx.y * ROWS + r, m = bm * BM + row;
    const bool on = row < BM && m < M;
    // the epilogue's rows and columns: of a gate/up tile half as many
    constexpr int TPE = TPR / Epi::COLS;
    const int re = threadIdx.x / TPE, ce = (threadIdx.x % TPE) * 8, row_e = blockIdx.y * ROWS + re, m_e = bm * BM + row_e;
    const bool on_e = re < ROWS && row_e < BM && m_e < M;
    typename Epi::Pre pre;
    if (on_e) pre = epi.template pre<BN>(m_e, bn, ce, epi.key(m_e));
    if (on) {
        const float* src = ws + (int64_t)blockIdx.x * (SLOT_ROWS * BN) + row * BN + cc;
        f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f};
        int sp = 0;
        for (; sp + 4 <= n_shares; sp += 4) {
            f32x4 x[4][2];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const f32x4* p = reinterpret_cast<const f32x4*>(src + (sp + u) * share_stride);
                x[u][0] = p[0];
                x[u][1] = p[1];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                a += x[u][0];
                b += x[u][1];
            }
        }
        for (; sp < n_shares; ++sp) {
            const f32x4* p = reinterpret_cast<const f32x4*>(src + sp * share_stride);
            a += p[0];
            b += p[1];
        }
        *reinterpret_cast<f32x4*>(&stage[r][cc]) = a;
        *reinterpret_cast<f32x4*>(&stage[r][cc + 4]) = b;
    }
    __syncthreads();
    if (on_e) epi.template operator()<BN>(m_e, bn, ce, stage[re], 0, pre);
}

// Consecutive workgroup ids go round-robin to the 8 XCDs (each with its own
// L2).  Every XCD gets one contiguous range of the tile sequence, and the
// sequence walks bands of GM row-tiles column by column, so the workgroups that
// run together on an XCD form a GM x (32/GM) block of tiles: they share GM
// tiles of A and 32/GM tiles of B through that L2.
// tile `vb` of the sequence (bands of GM row-tiles, column by column)
__device__ __forceinline__ void tile_of_seq(int vb, int tiles_m, int tiles_n, int GM, int* bm, int* bn) {
    if (tiles_m == 1) {                       // the divisions take 0.1 us each
        *bm = 0;
        *bn = vb;
        return;
    }
    const int band = GM * tiles_n;
    const int b = GM >= tiles_m ? 0 : vb / band, rb = vb - b * band;
    const int gm = min(GM, tiles_m - b * GM);
    *bn = rb / gm;
    *bm = b * GM + rb - *bn * gm;
}
// workgroup `bid` of a launch over tiles vb0 .. vb0 + nb - 1 of the sequence; returns its tile's index
__device__ __forceinline__ int tile_of_block(int bid, int nb, int vb0, int tiles_m, int tiles_n, int GM,
                                             int* bm, int* bn) {
    const int q = nb >> 3, r = nb & 7;
    const int x = bid & 7, local = bid >> 3;
    const int vb = vb0 + x * q + (x < r ? x : r) + local;
    tile_of_seq(vb, tiles_m, tiles_n, GM, bm, bn);
    return vb;
}
__device__ __forceinline__ void tile_of_block(int bid, int tiles_m, int tiles_n, int GM, int* bm,
                                              int* bn) {
    (void)tile_of_block(bid, tiles_m * tiles_n, 0, tiles_m, tiles_n, GM, bm, bn);
}

// 16 bytes per lane straight from global memory into LDS (no VGPR staging, no
// LDS store instruction).  The LDS destination is wave-uniform: lane L lands at
// lds_base + 16*L.  Completion is tracked by vmcnt like any vector load.
__device__ __forceinline__ void dma16(const bf16_t* gsrc, bf16_t* lds_wave_base) {
    __builtin_amdgcn_global_load_lds(
        (const void __attribute__((address_space(1)))*)gsrc,
        (void __attribute__((address_space(3)))*)lds_wave_base, 16, 0, 0);
}

// The same with an immediate offset, added to both the LDS and the global address: loads
// that share a wave base need no rewrite of M0 between them.
template <int OFF>
__device__ __forceinline__ void dma16_at(const char* gsrc_minus_off, bf16_t* lds_wave_base) {
    static_assert(OFF >= 0 && OFF < 4096, "the instruction offset is 13 bits signed; a larger value wraps silently");
    __builtin_amdgcn_global_load_lds(
        (const void __attribute__((address_space(1)))*)gsrc_minus_off,
        (void __attribute__((address_space(3)))*)lds_wave_base, 16, OFF, 0);
}
// The same for lines that no other workgroup reads: kept out of the caches behind it.
template <int OFF>
__device__ __forceinline__ void dma16_stream_at(const char* gsrc_minus_off, bf16_t* lds_wave_base) {
    static_assert(OFF >= 0 && OFF < 4096, "the instruction offset is 13 bits signed; a larger value wraps silently");
    __builtin_amdgcn_global_load_lds(
        (const void __attribute__((address_space(1)))*)gsrc_minus_off,
        (void __attribute__((address_space(3)))*)lds_wave_base, 16, OFF, 2 /* nt */);
}
template <int N, int I = 0, class F>
__device__ __forceinline__ void unrolled(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        unrolled<N, I + 1>(f);
    }
}

// Workgroup barrier without the memory fence of __syncthreads() (that fence waits for
// every outstanding global->LDS load; the ring loop waits only for the slice it needs,
// with wait_vm_lds0 just before).  The empty asm statements keep the compiler from
// moving LDS accesses across the barrier.
__device__ __forceinline__ void wg_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// s_waitcnt: at most N vector-memory operations outstanding, no LDS operation.
template <int N>
__device__ __forceinline__ void wait_vm_lds0() {
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4));
}

// Accumulators -> LDS (fp32, RG rows at a time) -> fused store.  `stage` must
// hold RG * (BN + 4) floats and no wave may still be reading operands from it.
template <int BM, int BN, int WAVES_M, int WAVES_N, int RG, class Epi>
__device__ __forceinline__ void store_tile(f32x16 (&acc)[BM / WAVES_M / 32][BN / WAVES_N / 32],
                                           float* stage, int m0, int bn, int M, const Epi& epi) {
    constexpr int NT = WAVES_M * WAVES_N * 64;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int TM = WM / 32, TN = WN / 32;
    constexpr int LDS_LD = BN + 4;
    constexpr int TPR = BN / Epi::COLS / 8;   // threads per staged row
    constexpr int RPP = NT / TPR;         // rows per pass
    static_assert(RG == 32 || RG == 16, "row group");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm0 = (wave % WAVES_M) * WM, wn0 = (wave / WAVES_M) * WN;
    const int frow = lane & 31, fk = lane >> 5;
#pragma unroll
    for (int rg = 0; rg < BM / RG; ++rg) {
        if (rg) __syncthreads();
        // register v of a 32x32 accumulator tile holds tile row 8*(v>>2) + 4*fk + (v&3):
        // the rows of this group are those of one accumulator tile (or of its half `sub`)
        constexpr int VPG = 16 * RG / 32;                 // accumulator registers per row group
        const int sub = (rg * RG % 32) / RG;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int tr = wm0 + i * 32;                  // first row of this accumulator tile
            if (tr / 32 == rg * RG / 32) {                // wave-uniform
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int vv = 0; vv < VPG; ++vv) {
                        const int v = sub * VPG + vv;
                        const int r = 8 * (v >> 2) + 4 * fk + (v & 3) - sub * RG;
                        stage[r * LDS_LD + wn0 + j * 32 + frow] = acc[i][j][v];
                    }
            }
        }
        __syncthreads();
        const int cc = (tid % TPR) * 8;
        for (int r = tid / TPR; r < RG; r += RPP) {
            int m = m0 + rg * RG + r;
            if (m < M) epi.template operator()<BN>(m, bn, cc, stage + r * LDS_LD, 0);
        }
    }
}

// Ring-loop epilogue.  After the K loop the four ring slots are free; each holds
// one RG-row group of the tile as fp32 [RG][BN] (RG = 32 where a slot is large enough,
// else 16: half an accumulator tile), so a tile leaves in phases of four groups with two
// barriers per phase, and a thread's functor calls of a phase are independent (their
// global loads overlap).  Column c of staged row r sits at c ^ 32*((r>>2)&1): the two
// half-waves of an accumulator store (rows r and r+4) then hit disjoint banks, and
// 8-column chunks stay contiguous for the functors.
template <int BM, int BN, int WAVES_M, int WAVES_N, int RG, class Epi>
__device__ __forceinline__ void store_tile_ring(f32x16 (&acc)[BM / WAVES_M / 32][BN / WAVES_N / 32],
                                                float* s0, float* s1, float* s2, float* s3, int m0,
                                                int bn, int M, const Epi& epi) {
    constexpr int NT = WAVES_M * WAVES_N * 64;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int TM = WM / 32, TN = WN / 32;
    constexpr int GPW = 4 / WAVES_M;      // staged groups per wave and phase
    constexpr int VPG = RG / 2;           // accumulator registers per group and tile
    constexpr int BPP = GPW * RG / 32;    // accumulator row blocks per wave and phase
    constexpr int PHASES = TM / BPP;
    constexpr int TPR = BN / Epi::COLS / 8;   // threads per staged row
    constexpr int RPP = NT / TPR;         // rows per pass
    static_assert(RG == 32 || RG == 16, "row group");
    static_assert(4 % WAVES_M == 0 && GPW * RG % 32 == 0 && TM % BPP == 0 && 4 * RG % RPP == 0, "epilogue shape");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WAVES_M, wn0 = (wave / WAVES_M) * WN;
    const int frow = lane & 31, fk = lane >> 5;
    auto stage = [&](int q) -> float* { return q == 0 ? s0 : q == 1 ? s1 : q == 2 ? s2 : s3; };
#pragma unroll
    for (int p = 0; p < PHASES; ++p) {
        if (p) __syncthreads();
        // register v of a 32x32 accumulator tile holds tile row 8*(v>>2) + 4*fk + (v&3): rows
        // 0..15 are registers 0..7, rows 16..31 registers 8..15; (row>>2)&1 == fk
#pragma unroll
        for (int g = 0; g < GPW; ++g) {
            const int i = p * BPP + g * RG / 32;  // accumulator row block
            const int sub = (g * RG % 32) / RG;   // which half of it (RG = 16)
            float* st = stage(wm * GPW + g);      // slot q holds wave-row q / GPW, group q % GPW
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int vv = 0; vv < VPG; ++vv) {
                    const int v = sub * VPG + vv;
                    const int r = 8 * (v >> 2) + 4 * fk + (v & 3) - sub * RG;
                    st[r * BN + ((wn0 + j * 32 + frow) ^ (fk << 5))] = acc[i][j][v];
                }
        }
        __syncthreads();
        const int cc = (tid % TPR) * 8;
#pragma unroll
        for (int k = 0; k < 4 * RG / RPP; ++k) {
            const int rr = tid / TPR + k * RPP, q = rr / RG, r = rr % RG;
            const int m = m0 + (q / GPW) * WM + p * BPP * 32 + (q % GPW) * RG + r;   // slot q's first tile row, and r
            if (m < M) epi.template operator()<BN>(m, bn, cc, stage(q) + r * BN, ((r >> 2) & 1) << 5);
        }
    }
}

// ---------------------------------------------------------------- staged loop
constexpr int BK = 64;
constexpr int CPR = BK / 8;   // 16-byte chunks per tile row

template <int BM, int BN, int WAVES_M, int WAVES_N, class BSrc, class Epi>
__global__ __launch_bounds__(WAVES_M* WAVES_N * 64) void gemm_nt_kernel(
    const bf16_t* __restrict__ A, int lda, int M, int K, int tiles_m, int tiles_n, int GM, BSrc bsrc,
    Epi epi) {
    constexpr int NW = WAVES_M * WAVES_N;
    constexpr int NT = NW * 64;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int TM = WM / 32, TN = WN / 32;
    constexpr int A_CH = BM * CPR / NT, B_CH = BN * CPR / NT;   // DMA instructions per wave and tile
    static_assert(BM * CPR % NT == 0 && BN * CPR % NT == 0, "tile/threads");
    static_assert(WM % 32 == 0 && WN % 32 == 0, "wave tile");
    static_assert(32 * (BN + 4) * 4 <= (BM + BN) * BK * 2, "epilogue stage fits in one pipeline stage");

    // Two pipeline stages as separate arrays, so that a DMA into one stage is
    // known not to alias the fragment reads of the other.
    __shared__ __align__(16) bf16_t st0[(BM + BN) * BK];
    __shared__ __align__(16) bf16_t st1[(BM + BN) * BK];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm0 = (wave % WAVES_M) * WM, wn0 = (wave / WAVES_M) * WN;
    int bm, bn;
    tile_of_block(blockIdx.x, tiles_m, tiles_n, GM, &bm, &bn);
    const int m0 = bm * BM;

    // One DMA instruction moves 8 tile rows (8 x 128 B).  Lane L fills physical
    // chunk slot L%8 of row L/8; the XOR swizzle (slot = chunk ^ ((row>>1)&7),
    // conflict-free on the 64-bank LDS for 16-byte fragment reads) is applied by
    // choosing which global chunk the lane fetches.
    const bf16_t* ag[A_CH];
    const bf16_t* bg[B_CH];
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
        int r = (i * NW + wave) * 8 + (lane >> 3);
        int c = (lane & 7) ^ ((r >> 1) & 7);
        int m = m0 + r;
        m = m < M ? m : M - 1;
        ag[i] = A + (int64_t)m * lda + c * 8;
    }
#pragma unroll
    for (int i = 0; i < B_CH; ++i) {
        int r = (i * NW + wave) * 8 + (lane >> 3);
        int c = (lane & 7) ^ ((r >> 1) & 7);
        bg[i] = bsrc.template row<BN>(bn, r) + c * 8;
    }
    auto dma_tile = [&](bf16_t* stage, int kt) {
        const int k0 = kt * BK;
#pragma unroll
        for (int i = 0; i < A_CH; ++i) dma16(ag[i] + k0, stage + (i * NW + wave) * 8 * BK);
#pragma unroll
        for (int i = 0; i < B_CH; ++i) dma16(bg[i] + k0, stage + BM * BK + (i * NW + wave) * 8 * BK);
        // keep the loads at the top of the iteration: the compiler would otherwise sink
        // them below the MFMAs, next to the barrier that waits for them
        __builtin_amdgcn_sched_barrier(0);
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    const int frow = lane & 31, fk = lane >> 5;
    const int fsw = (frow >> 1) & 7;      // rows of a fragment differ by multiples of 32
    auto compute = [&](const bf16_t* stage) {
        const bf16_t* as = stage;
        const bf16_t* bs = stage + BM * BK;
        bf16x8 af[2][TM], bfr[2][TN];
        auto load_frags = [&](int ks, int fb) {
            const int sl = ((ks * 2 + fk) ^ fsw) << 3;
#pragma unroll
            for (int i = 0; i < TM; ++i)
                af[fb][i] = *reinterpret_cast<const bf16x8*>(as + (wm0 + i * 32 + frow) * BK + sl);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                bfr[fb][j] = *reinterpret_cast<const bf16x8*>(bs + (wn0 + j * 32 + frow) * BK + sl);
        };
        load_frags(0, 0);
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            if (ks + 1 < BK / 16) load_frags(ks + 1, (ks + 1) & 1);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[ks & 1][i], bfr[ks & 1][j],
                                                                        acc[i][j], 0, 0, 0);
        }
        // issue order: the first k-step's fragments, then every MFMA followed by one
        // fragment read of the next k-step, so LDS latency hides behind the matrix pipe
        constexpr int NF = TM + TN, NM = TM * TN;
        __builtin_amdgcn_sched_group_barrier(0x100, NF, 0);
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks)
#pragma unroll
            for (int mm = 0; mm < NM; ++mm) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (ks + 1 < BK / 16 && mm < NF) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
    };

    // K loop: while tile kt is multiplied out of one stage, the DMA engine fills
    // the other with tile kt+1; the barrier at the end of the iteration waits for
    // both (vmcnt for the DMA, every wave done reading).
    const int KT = K / BK;
    dma_tile(st0, 0);
    __syncthreads();
    int kt = 0;
    for (; kt + 2 <= KT; kt += 2) {
        dma_tile(st1, kt + 1);
        compute(st0);
        __syncthreads();
        if (kt + 2 < KT) dma_tile(st0, kt + 2);
        compute(st1);
        __syncthreads();
    }
    if (kt < KT) {
        compute(st0);
        __syncthreads();
    }
    store_tile<BM, BN, WAVES_M, WAVES_N, 32>(acc, reinterpret_cast<float*>(st0), m0, bn, M, epi);
}

// ------------------------------------------------------------------ ring loop
constexpr int BKS = CC_GEMM_SLICE;   // K columns per slice
constexpr int NS = 4;                // ring slots
static_assert(BKS * NS == CC_GEMM_GROUP, "a group is one ring of slices");

template <int BM, int BN, int WAVES_M, int WAVES_N, class BSrc, class Epi>
__global__ __launch_bounds__(WAVES_M* WAVES_N * 64) void gemm_ring_kernel(
    const bf16_t* __restrict__ A, int lda, int M, int K, int k_more, int tiles_m, int tiles_n, int GM, int nb, int vb0,
    BSrc bsrc, Epi epi) {
    constexpr int NW = WAVES_M * WAVES_N;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int TM = WM / 32, TN = WN / 32;
    // DMA instructions per wave and slice
    constexpr int A_I = BM / 16 / NW, B_I = BN / 16 / NW;
    constexpr int DPS = A_I + B_I;
    constexpr int SL = NW * DPS * 16 * BKS;
    // rows of a staged fp32 group: 32 if that fits in one slot and a wave's row blocks pair up, else 16
    constexpr int RG = (32 * BN * 4 <= SL * 2 && TM % (4 / WAVES_M) == 0) ? 32 : 16;
    static_assert(BM % (16 * NW) == 0 && BN % (16 * NW) == 0 && BN % 32 == 0, "tile/waves");
    static_assert(WM % 32 == 0 && WN % 32 == 0, "wave tile");
    static_assert(RG * BN * 4 <= SL * 2, "an fp32 row group fits in one slot");
    static_assert(DPS * (NS - 1) < 64, "vmcnt range");

    // One array per ring slot: the compiler then knows that a DMA into one slot
    // does not alias the fragment reads of another and adds no waits of its own.
    __shared__ __align__(16) bf16_t sl0[SL];
    __shared__ __align__(16) bf16_t sl1[SL];
    __shared__ __align__(16) bf16_t sl2[SL];
    __shared__ __align__(16) bf16_t sl3[SL];
    auto slot = [&](int i) -> bf16_t* { return i == 0 ? sl0 : i == 1 ? sl1 : i == 2 ? sl2 : sl3; };

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm0 = (wave % WAVES_M) * WM, wn0 = (wave / WAVES_M) * WN;
    int bm, bn;
    const int vb = tile_of_block(blockIdx.x, nb, vb0, tiles_m, tiles_n, GM, &bm, &bn);   // this launch covers tiles vb0 .. vb0 + nb - 1
    const int m0 = bm * BM;

    // One DMA instruction moves 16 slice rows (16 x 64 B).  Lane L fills physical
    // chunk slot L%4 of row L/4 and fetches the logical chunk slot ^ ((row>>2)&3):
    // a 16-byte fragment read of 16 consecutive rows then touches every bank once.
    // Wave w loads its A pieces (16 rows each) and B rows w*16*B_I .. of the tile, and a slot
    // holds them wave by wave ([wave][A rows | B rows], DPS KB each): the DPS loads of a wave
    // and slice share one LDS base and differ in their immediate offset only.
    // Global addresses are a wave-uniform base (advanced along K in scalar
    // registers) plus a loop-invariant 32-bit lane offset.
    uint32_t ao[A_I], bo[B_I];
    const int a_rows = M - m0;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
#pragma unroll
    for (int i = 0; i < A_I; ++i) {
        int r = (wave_u * A_I + i) * 16 + (lane >> 2);
        const int c = (lane & 3) ^ ((r >> 2) & 3);
        r = r < a_rows ? r : a_rows - 1;
        ao[i] = (uint32_t)((r * lda + c * 8) * 2);
    }
    // B rows: the rows of one wave lie in one half of the tile (BN/2 is a multiple of
    // 16*B_I); each half has its own base (the gate and the up matrix of a fused gate/up tile,
    // or simply row BN/2 of the same matrix).
    static_assert((BN / 2) % (16 * B_I) == 0, "a wave's B rows stay in one half");
    const bool hi_half = wave_u * B_I * 16 >= BN / 2;          // wave-uniform
#pragma unroll
    for (int i = 0; i < B_I; ++i) {
        int r = (wave_u * B_I + i) * 16 - (hi_half ? BN / 2 : 0) + (lane >> 2);   // row within the half
        const int c = (lane & 3) ^ ((r >> 2) & 3);             // same swizzle as for the tile row
        const int left = bsrc.template rows_left<BN>(bn, hi_half ? 1 : 0);
        r = r < left ? r : left - 1;
        bo[i] = (uint32_t)((r * bsrc.ldb + c * 8) * 2);
    }
    int64_t kz;                        // this workgroup row's share of K
    K = k_share<BKS * NS>(K, k_more, &kz);
    const char* abase = reinterpret_cast<const char*>(A + (int64_t)m0 * lda) + kz;
    const char* bbase = reinterpret_cast<const char*>(bsrc.template base<BN>(bn, hi_half ? 1 : 0)) + kz;
    const int wbase = wave_u * DPS * 16 * BKS;
    auto scalar_ptr = [](const char* p) -> const char* {   // keeps the base in scalar registers
        const uint64_t u = reinterpret_cast<uint64_t>(p);
        const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
        const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
        return reinterpret_cast<const char*>((hi << 32) | lo);
    };
    auto dma_slice = [&](bf16_t* s, int sidx) {
        const int64_t kb = (int64_t)sidx * (BKS * 2);
        unrolled<A_I>([&](auto i) {
            const char* ab = scalar_ptr(abase + kb - i.value * 1024);   // the immediate adds it back
            asm volatile("" : "+v"(ao[i.value]));   // keeps the offset a 32-bit register operand of the load
            dma16_at<i.value * 1024>(ab + ao[i.value], s + wbase);
        });
        unrolled<B_I>([&](auto i) {
            const char* bb = scalar_ptr(bbase + kb - (A_I + i.value) * 1024);
            asm volatile("" : "+v"(bo[i.value]));
            dma16_at<(A_I + i.value) * 1024>(bb + bo[i.value], s + wbase);
        });
    };
    // element offset in a slot of tile row r of A (is_b = 0) or B (is_b = 1)
    auto row_at = [](int r, int is_b) {
        constexpr int per_b = 16 * B_I;
        if (is_b) return ((r / per_b) * DPS * 16 + A_I * 16 + r % per_b) * BKS;
        constexpr int per_a = 16 * A_I;
        return (r / per_a * DPS * 16 + r % per_a) * BKS;
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    const int frow = lane & 31, fk = lane >> 5;
    const int fsw = (frow >> 2) & 3;      // rows of a fragment differ by multiples of 32
    bf16x8 af[2][TM], bfr[2][TN];
    auto load_frags = [&](const bf16_t* s, int ks, int fb) {
        const int sl = ((ks * 2 + fk) ^ fsw) << 3;
#pragma unroll
        for (int i = 0; i < TM; ++i)
            af[fb][i] = *reinterpret_cast<const bf16x8*>(s + row_at(wm0 + i * 32 + frow, 0) + sl);
#pragma unroll
        for (int j = 0; j < TN; ++j)
            bfr[fb][j] = *reinterpret_cast<const bf16x8*>(s + row_at(wn0 + j * 32 + frow, 1) + sl);
    };
    auto mfmas = [&](int fb) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[fb][i], bfr[fb][j], acc[i][j], 0, 0, 0);
    };
    constexpr int NF = TM + TN, NM = TM * TN;
    auto pin_interleave = [&]() {   // issue order: every MFMA followed by one fragment read
#pragma unroll
        for (int mm = 0; mm < NM; ++mm) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if (mm < NF) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
    };

    // The two 16-column k-steps of a slice alternate between two fragment
    // register sets, and the stream of k-steps runs on across slice boundaries:
    // the MFMAs of a slice's second k-step are issued after the barrier that opens
    // the next slice, so they cover the latency of its first fragment reads.
    // At a boundary a wave waits until its own loads of the next slice have landed
    // (vmcnt: only the younger slices may be outstanding) and its fragment reads
    // of the current slice have returned; after the barrier the slot just read is
    // free everywhere and is refilled with the slice NS ahead.
    const int KS = K / BKS;            // K % (BKS * NS) == 0, KS >= NS
#pragma unroll
    for (int j = 0; j < NS; ++j) dma_slice(slot(j), j);
    wait_vm_lds0<DPS * (NS - 1)>();
    wg_barrier();
    load_frags(slot(0), 0, 0);
    int s0 = 0;
    for (; s0 + 2 * NS <= KS; s0 += NS) {
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            load_frags(slot(j), 1, 1);
            mfmas(0);
            pin_interleave();
            wait_vm_lds0<DPS * (NS - 2)>();
            wg_barrier();
            dma_slice(slot(j), s0 + j + NS);
            __builtin_amdgcn_sched_barrier(0);
            load_frags(slot((j + 1) % NS), 0, 0);
            mfmas(1);
            pin_interleave();
        }
    }
    // the last NS slices are in flight or landed: no refills
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        load_frags(slot(j), 1, 1);
        mfmas(0);
        pin_interleave();
        if (j + 1 < NS) {
            if (j == 0) wait_vm_lds0<DPS * (NS - 2)>();
            else if (j == 1) wait_vm_lds0<DPS * (NS - 3)>();
            else wait_vm_lds0<0>();
            wg_barrier();
            __builtin_amdgcn_sched_barrier(0);
            load_frags(slot(j + 1), 0, 0);
            mfmas(1);
            pin_interleave();
        } else {
            mfmas(1);
        }
    }
    __syncthreads();   // every wave has finished reading the ring
    store_tile_ring<BM, BN, WAVES_M, WAVES_N, RG>(acc, reinterpret_cast<float*>(sl0), reinterpret_cast<float*>(sl1),
                                              reinterpret_cast<float*>(sl2), reinterpret_cast<float*>(sl3),
                                              m0, bn, M, epi_for_tile(epi, vb - vb0, m0));
}

// The same ring with 16x16x32 MFMAs and hand-written fragment reads.
template <int BM, int BN, int WAVES_M, int WAVES_N, class BSrc, class Epi>
__global__ __launch_bounds__(WAVES_M* WAVES_N * 64) void gemm_ring16_kernel(
    const bf16_t* __restrict__ A, int lda, int M, int K, int k_more, int tiles_m, int tiles_n, int GM, int nb, int vb0,
    BSrc bsrc, Epi epi) {
    constexpr int NW = WAVES_M * WAVES_N;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int TM = WM / 32;
    constexpr int UM = WM / 16, UN = WN / 16;       // 16x16 accumulator tiles per wave
    // DMA instructions per wave and slice
    constexpr int A_I = BM / 16 / NW, B_I = BN / 16 / NW;
    constexpr int DPS = A_I + B_I;
    constexpr int SL = NW * DPS * 16 * BKS;
    // rows of a staged fp32 group: 32 if that fits in one slot and a wave's row blocks pair up, else 16
    constexpr int RG = (32 * BN * 4 <= SL * 2 && TM % (4 / WAVES_M) == 0) ? 32 : 16;
    static_assert(BM % (16 * NW) == 0 && BN % (16 * NW) == 0 && BN % 32 == 0, "tile/waves");
    static_assert(WM % 32 == 0 && WN % 32 == 0, "wave tile");
    static_assert(RG * BN * 4 <= SL * 2, "an fp32 row group fits in one slot");
    static_assert(DPS * (NS - 1) < 64, "vmcnt range");

    // One array: the fragment reads of this loop are written by hand, so the compiler has no
    // LDS reads to order against the global -> LDS loads.
    __shared__ __align__(16) bf16_t ring[NS * SL];
    auto slot = [&](int i) -> bf16_t* { return ring + i * SL; };

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm0 = (wave % WAVES_M) * WM, wn0 = (wave / WAVES_M) * WN;
    int bm, bn;
    const int vb = tile_of_block(blockIdx.x, nb, vb0, tiles_m, tiles_n, GM, &bm, &bn);   // this launch covers tiles vb0 .. vb0 + nb - 1
    const int m0 = bm * BM;

    // One DMA instruction moves 16 slice rows (16 x 64 B).  Lane L fills physical
    // chunk slot L%4 of row L/4 and fetches the logical chunk slot ^ ((row>>1)&3).  The
    // fragment read of this loop (lane = row L%16, chunk L/16 of 16 consecutive rows) runs at
    // the full LDS rate with this swizzle and at half of it with slot ^ ((row>>2)&3), with
    // slot ^ (row&3) or without one (measured with a read-only kernel on this part; the
    // bank-conflict counter of the loop agrees: half of the active LDS cycles before).
    // Wave w loads its A pieces (16 rows each) and B rows w*16*B_I .. of the tile, and a slot
    // holds them wave by wave ([wave][A rows | B rows], DPS KB each): the DPS loads of a wave
    // and slice share one LDS base and differ in their immediate offset only.
    // Global addresses are a wave-uniform base (advanced along K in scalar
    // registers) plus a loop-invariant 32-bit lane offset.
    uint32_t ao[A_I], bo[B_I];
    const int a_rows = M - m0;
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
#pragma unroll
    for (int i = 0; i < A_I; ++i) {
        int r = (wave_u * A_I + i) * 16 + (lane >> 2);
        const int c = (lane & 3) ^ ((r >> 1) & 3);
        r = r < a_rows ? r : a_rows - 1;
        ao[i] = (uint32_t)((r * lda + c * 8) * 2);
    }
    // B rows: the rows of one wave lie in one half of the tile (BN/2 is a multiple of
    // 16*B_I); each half has its own base (the gate and the up matrix of a fused gate/up tile,
    // or simply row BN/2 of the same matrix).
    static_assert((BN / 2) % (16 * B_I) == 0, "a wave's B rows stay in one half");
    const bool hi_half = wave_u * B_I * 16 >= BN / 2;          // wave-uniform
#pragma unroll
    for (int i = 0; i < B_I; ++i) {
        int r = (wave_u * B_I + i) * 16 - (hi_half ? BN / 2 : 0) + (lane >> 2);   // row within the half
        const int c = (lane & 3) ^ ((r >> 1) & 3);             // same swizzle as for the tile row
        const int left = bsrc.template rows_left<BN>(bn, hi_half ? 1 : 0);
        r = r < left ? r : left - 1;
        bo[i] = (uint32_t)((r * bsrc.ldb + c * 8) * 2);
    }
    int64_t kz;                        // this workgroup row's share of K
    K = k_share<BKS * NS>(K, k_more, &kz);
    const char* abase = reinterpret_cast<const char*>(A + (int64_t)m0 * lda) + kz;
    const char* bbase = reinterpret_cast<const char*>(bsrc.template base<BN>(bn, hi_half ? 1 : 0)) + kz;
    const int wbase = wave_u * DPS * 16 * BKS;
    auto scalar_ptr = [](const char* p) -> const char* {   // keeps the base in scalar registers
        const uint64_t u = reinterpret_cast<uint64_t>(p);
        const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
        const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
        return reinterpret_cast<const char*>((hi << 32) | lo);
    };
    auto dma_one = [&](bf16_t* s, int sidx, auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value;
        const int64_t kb = (int64_t)sidx * (BKS * 2);
        if constexpr (i < A_I) {
            const char* ab = scalar_ptr(abase + kb - i * 1024);   // the immediate adds it back
            asm volatile("" : "+v"(ao[i]));   // keeps the offset a 32-bit register operand of the load
            dma16_at<i * 1024>(ab + ao[i], s + wbase);
        } else {
            const char* bb = scalar_ptr(bbase + kb - i * 1024);
            asm volatile("" : "+v"(bo[i - A_I]));
            dma16_at<i * 1024>(bb + bo[i - A_I], s + wbase);
        }
    };
    auto dma_slice = [&](bf16_t* s, int sidx) __attribute__((always_inline)) {
        unrolled<DPS>([&](auto i) __attribute__((always_inline)) { dma_one(s, sidx, i); });
    };
    // element offset in a slot of tile row r of A (is_b = 0) or B (is_b = 1)
    auto row_at = [](int r, int is_b) {
        constexpr int per_b = 16 * B_I;
        if (is_b) return ((r / per_b) * DPS * 16 + A_I * 16 + r % per_b) * BKS;
        constexpr int per_a = 16 * A_I;
        return (r / per_a * DPS * 16 + r % per_a) * BKS;
    };

    // ---- 16x16x32 MFMAs: one k-step per slice.  Lane L holds row (column) L%16 and the eight k
    //      values of 16-byte chunk L/16 of the slice row; an accumulator tile is f32x4 with
    //      row 4*(L/16) + v, column L%16 ----
    static_assert(UM % 2 == 0 && UM >= 4 && UN >= 2, "fragment ring");
    static_assert(WM % (16 * A_I) == 0 && WN % (16 * B_I) == 0, "fragment offsets are lane-independent");
    static_assert(DPS <= 2 * UN, "one load per MFMA of a block's first part at most");
    f32x4 acc[UM][UN];
#pragma unroll
    for (int i = 0; i < UM; ++i)
#pragma unroll
        for (int j = 0; j < UN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int frow = lane & 15, fk = lane >> 4;
    const int fsw = (lane >> 1) & 3;
    const int sl = (fk ^ fsw) << 3;
    // A fragments cycle through four registers (two rows ahead of the MFMAs), B fragments of a
    // slice stay for the slice and alternate between two sets from slice to slice
    bf16x8 ar[4], bq[2][UN];
    // byte offset of fragment i (16 rows) from the lane's address of fragment 0
    constexpr auto delta = [](int i, int per, int dps) { return 2 * BKS * (((16 * i) / per) * dps * 16 + (16 * i) % per); };
    const uint32_t ring_base = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)ring;
    const uint32_t a_lane = ring_base + 2 * (row_at(wm0 + frow, 0) + sl), b_lane = ring_base + 2 * (row_at(wn0 + frow, 1) + sl);
    // slots 0, 1 and 2, 3 share an address register each: the offset field of an LDS read is 16 bits
    static_assert(NS == 4, "slot pairs");
    const uint32_t a_addr[2] = {a_lane, a_lane + 2 * 2 * SL}, b_addr[2] = {b_lane, b_lane + 2 * 2 * SL};
    auto read_a = [&](auto jc, auto ic) __attribute__((always_inline)) -> bf16x8 {
        constexpr int j = decltype(jc)::value, i = decltype(ic)::value;
        bf16x8 v;
        constexpr int off = (j & 1) * 2 * SL + delta(i, 16 * A_I, DPS);
        static_assert(off < 65536, "ds offset field");
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(a_addr[j >> 1]), "n"(off));
        return v;
    };
    auto read_b = [&](auto jc, auto ic) __attribute__((always_inline)) -> bf16x8 {
        constexpr int j = decltype(jc)::value, i = decltype(ic)::value;
        constexpr int off = (j & 1) * 2 * SL + delta(i, 16 * B_I, DPS);
        static_assert(off < 65536, "ds offset field");
        bf16x8 v;
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(b_addr[j >> 1]), "n"(off));
        return v;
    };
    // One slice (slot j), straight-line code: [the last two fragment rows of the previous slice,
    // between their MFMAs the first reads of this slice and the refill of the slot freed at the
    // previous barrier], rows 0 .. UM-3 (the A fragment two rows ahead is requested before each
    // row's MFMAs), wait, barrier.  The compiler does not know that a hand-written read fills
    // its registers later: every read is issued and waited for inside this block, and none is
    // in flight at its end.  Reads return in issue order (A0 B0 .. B(UN-1) A1 A2 ...): when a
    // row's MFMAs need their operands, exactly two younger reads may still be out.
    auto block = [&](auto jc, auto firstc, auto dmac, auto vmc, int sidx) __attribute__((always_inline)) {
        constexpr int j = decltype(jc)::value, bb = j & 1;
        constexpr bool first = decltype(firstc)::value, with_dma = decltype(dmac)::value;
        constexpr int VM = decltype(vmc)::value;
        // A fragment i of this slice lives in ar[(i + RO) % 4]; with UM % 4 == 2 the slices of odd
        // slots start two registers on, so that the previous slice's last two stay clear of the
        // first two of this one
        constexpr int RO = (UM % 4) * (j & 1) % 4, RP = (UM % 4) * ((j + NS - 1) & 1) % 4;
        unrolled<2 * UN>([&](auto mc) __attribute__((always_inline)) {
            constexpr int m = decltype(mc)::value, i = UM - 2 + m / UN, n = m % UN;
            if constexpr (!first) acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar[(i + RP) % 4], bq[bb ^ 1][n], acc[i][n], 0, 0, 0);
            if constexpr (m == 0) ar[RO % 4] = read_a(jc, std::integral_constant<int, 0>{});
            else if constexpr (m <= UN) bq[bb][m - 1] = read_b(jc, std::integral_constant<int, m - 1>{});
            else if constexpr (m == UN + 1) ar[(1 + RO) % 4] = read_a(jc, std::integral_constant<int, 1>{});
            if constexpr (with_dma && m < DPS) dma_one(slot((j + NS - 1) % NS), sidx, mc);
            if constexpr (!first) __builtin_amdgcn_sched_barrier(0);
        });
        unrolled<UM - 2>([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value;
            ar[(i + 2 + RO) % 4] = read_a(jc, std::integral_constant<int, i + 2>{});
            asm volatile("s_waitcnt lgkmcnt(2)" : "+v"(ar[(i + RO) % 4]));
            if constexpr (i == 0) {
#pragma unroll
                for (int n = 0; n < UN; ++n) asm volatile("" : "+v"(bq[bb][n]));
            }
            unrolled<UN>([&](auto nc) __attribute__((always_inline)) {
                constexpr int n = decltype(nc)::value;
                acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar[(i + RO) % 4], bq[bb][n], acc[i][n], 0, 0, 0);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        // this wave's loads of the next slice have landed (at most VM younger ones may be out) and
        // its last two A fragments have arrived; after the barrier slot j is free everywhere
        asm volatile("s_waitcnt vmcnt(%2) lgkmcnt(0)" : "+v"(ar[(UM - 2 + RO) % 4]), "+v"(ar[(UM - 1 + RO) % 4]) : "n"(VM));
        wg_barrier();
    };
    using T = std::true_type;
    using F = std::false_type;
#define CC_IC(x) std::integral_constant<int, (x)>{}
    const int KS = K / BKS;            // K % (BKS * NS) == 0, KS >= NS
#pragma unroll
    for (int j = 0; j < NS; ++j) dma_slice(slot(j), j);
    wait_vm_lds0<DPS * (NS - 1)>();
    wg_barrier();
    constexpr int VS = DPS * (NS - 2);
    block(CC_IC(0), T{}, F{}, CC_IC(VS), 0);
    int t = 1;
    for (; t + 3 + NS <= KS; t += NS) {      // slices t .. t+3 in slots 1, 2, 3, 0; each refills the slot before its own
        block(CC_IC(1), F{}, T{}, CC_IC(VS), t - 1 + NS);
        block(CC_IC(2), F{}, T{}, CC_IC(VS), t + NS);
        block(CC_IC(3), F{}, T{}, CC_IC(VS), t + 1 + NS);
        block(CC_IC(0), F{}, T{}, CC_IC(VS), t + 2 + NS);
    }
    // t == KS - NS + 1: the last three slices, every load has been issued
    block(CC_IC(1), F{}, F{}, CC_IC(DPS), 0);
    block(CC_IC(2), F{}, F{}, CC_IC(0), 0);
    block(CC_IC(3), F{}, F{}, CC_IC(0), 0);
#undef CC_IC
    // rows UM-2, UM-1 of the last slice (slot NS-1)
    unrolled<2 * UN>([&](auto mc) __attribute__((always_inline)) {
        constexpr int m = decltype(mc)::value, i = UM - 2 + m / UN, n = m % UN;
        constexpr int RL = (UM % 4) * ((NS - 1) & 1) % 4;
        acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar[(i + RL) % 4], bq[1][n], acc[i][n], 0, 0, 0);
    });
    __syncthreads();   // every wave has finished reading the ring

    // ---- epilogue: the four slots take one RG-row group each as fp32 [RG][BN] (RG = 32: two
    //      accumulator tiles, where a slot is large enough and a wave's 32-row blocks pair up; else
    //      16: one), a wave's rows leave in phases of 4 / WAVES_M groups.  Column c of staged row r
    //      sits at c ^ 16*((r>>2)&3): the four 16-lane groups of an accumulator store (rows 4 apart)
    //      hit disjoint banks, and 8-column chunks stay contiguous for the functors ----
    {
        constexpr int NT = NW * 64;
        constexpr int GPW = 4 / WAVES_M;          // staged groups per wave and phase
        constexpr int RGS = (32 * BN * 4 <= SL * 2 && TM % GPW == 0) ? 32 : 16;
        constexpr int TPG = RGS / 16;             // accumulator tiles per group
        constexpr int PHASES = UM / (GPW * TPG);
        constexpr int TPR = BN / Epi::COLS / 8, RPP = NT / TPR;
        static_assert(RGS * BN * 4 <= SL * 2 && 4 % WAVES_M == 0 && UM % (GPW * TPG) == 0 && 4 * RGS % RPP == 0, "epilogue shape");
        const int wm = wave % WAVES_M;
        auto stage = [&](int q) -> float* { return reinterpret_cast<float*>(ring + q * SL); };
        const auto e2 = epi_for_tile(epi, vb - vb0, m0);
#pragma unroll
        for (int p = 0; p < PHASES; ++p) {
            if (p) __syncthreads();
#pragma unroll
            for (int g = 0; g < GPW; ++g) {
                float* st = stage(wm * GPW + g);      // slot q holds wave-row q / GPW, group q % GPW
#pragma unroll
                for (int hh = 0; hh < TPG; ++hh) {    // the 16-row accumulator tiles of the group
                    const int i = (p * GPW + g) * TPG + hh;
#pragma unroll
                    for (int jj = 0; jj < UN; ++jj)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int r = 16 * hh + 4 * fk + v;
                            st[r * BN + ((wn0 + jj * 16 + frow) ^ (fk << 4))] = acc[i][jj][v];
                        }
                }
            }
            __syncthreads();
            const int cc = (tid % TPR) * 8;
#pragma unroll
            for (int k = 0; k < 4 * RGS / RPP; ++k) {
                const int rr = tid / TPR + k * RPP, q = rr / RGS, r = rr % RGS;
                const int m = m0 + (q / GPW) * WM + (p * GPW + q % GPW) * RGS + r;   // slot q's first tile row, and r
                if (m < M) e2.template operator()<BN>(m, bn, cc, stage(q) + r * BN, ((r >> 2) & 3) << 4);
            }
        }
    }
}

// ------------------------------------------------------------- ping-pong loop
template <int IMM>
__device__ __forceinline__ bf16x8 lds_read16(uint32_t addr) {
    static_assert(IMM >= 0 && IMM < 65536, "ds offset field");
    bf16x8 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(IMM));
    return v;
}

// The 256x256 tile with the two waves of every SIMD half a phase apart.
//
// What bounds it: the matrix pipe at the clock that the power limit leaves (full rounds run at
// 1.40 PFLOP/s).  The ring loop above keeps its eight waves in step: every wave reads fragments,
// issues loads and multiplies at the same time, a slice row is half a cache line, and a slice
// took 1300 clocks for 1024 of matrix pipe.  Here
//   - a K tile is 64 columns, so a row is one whole 128-byte line and a load moves 8 of them;
//   - the tile is cut in halves, A0, A1 (128 rows each) and B0, B1 (128 columns each), and a K
//     tile is four phases, one per quadrant of C: (A0,B0) (A0,B1) (A1,B1) (A1,B0).  A phase has
//     a memory part (fragment reads, two loads) and a compute part (16 MFMAs, 256 clocks of the
//     pipe), a barrier behind each.  Waves 4..7 run one barrier behind waves 0..3, and wave w
//     and w + 4 share a SIMD: one multiplies while the other reads;
//   - a wave owns 64 x 32 of every quadrant, so it reads 8 + 4 + 8 + 4 fragments per K tile, B0
//     of the next tile in the last phase (a second register set) to even the phases out.
// LDS: two buffers of one K tile (2 x 64 KB), filled half tile by half tile.  The half read in
// phase p is refilled two phases later (both groups have read it by then) and the refill is
// waited for five phases after its issue:
//   phase   reads      loads          waited for before the first barrier (5 younger halves out)
//   1       A0(t)      A1(t+1)        B1(t)
//   2       B1(t)      B0(t+2)        A1(t)
//   3       A1(t)      A0(t+2)        B0(t+1)
//   4       B0(t+1)    B1(t+2)        A0(t+1)
// A wave waits for its own loads before the first barrier of phase p; both groups have passed
// such a barrier before either reads in phase p + 1.
// Slot swizzle: 16-byte chunk c of row r sits at c ^ ((r>>1)&7), free of bank conflicts for the
// fragment read (lane = row L%16, chunk L/16 of 16 rows).
// Against the ring loop with this tile (same sums, same bits), microseconds: M = 3404, d = 4096,
// f = 14336: gate/up 727 -> 642, down 331 -> 290, O 114 -> 107; M = 13363, d = 8192, f = 28672:
// gate/up 10370 -> 9050, down 5480 -> 4450, QKV 1990 -> 1720, O 1520 -> 1260.  Raising the
// wave's priority around the MFMAs, waiting for the reads after the barrier instead of before it,
// and issuing the loads before the reads: each within 1 %.
// Epilogue: with the operands of the MFMAs exchanged a lane holds four columns of one row and stores them from its registers;
// through LDS the tile was written a word at a time behind two barriers a half (M = 8192, before -> after: O 239.6 -> 229.9
// us for d = 4096, 210.7 -> 200.7 for 3584, 77.5 -> 72.4 for 2048, gate/up 1352.7 -> 1339.1, 1604.7 -> 1591.1, 421.8 -> 417.0;
// down the same, and 5 % more with 8-byte stores, which is why lanes trade columns first).
template <bool DIRECT, class BSrc, class Epi>
__device__ __forceinline__ void pingpong(
    const bf16_t* __restrict__ A, int lda, int M, int K, int k_more, int tiles_m, int tiles_n, int GM, int nb, int vb0,
    const BSrc& bsrc, const Epi& epi) {
    constexpr int H = 128, BM = 2 * H, BN = 2 * H;
    constexpr int UM = 4, UN = 2;                      // 16x16 accumulator tiles of a wave in one quadrant
    constexpr int LPH = 2;                             // loads of a wave per half tile
    constexpr int ROWB = 128;                          // bytes of a K tile's row
    constexpr int HALF = H * ROWB, BUF = 4 * HALF;     // a buffer is A0 | A1 | B0 | B1
    static_assert(2 * BUF >= H * BN * 4, "half of the fp32 tile fits for the epilogue");
    __shared__ __align__(16) char smem[2 * BUF];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 2, wc = wave & 3;           // wave row = group
    int bm, bn;
    const int vb = tile_of_block(blockIdx.x, nb, vb0, tiles_m, tiles_n, GM, &bm, &bn);
    const int m0 = bm * BM;
    int64_t kz;                                        // this workgroup row's share of K
    K = k_share<CC_GEMM_GROUP>(K, k_more, &kz);

    // ---- global -> LDS: a wave moves rows 16 wave .. 16 wave + 15 of every half, 8 per load; lane L
    //      fills slot L%8 of row L/8.  Wave-uniform bases advance along K in scalar registers. ----
    uint32_t ao[2][LPH], bo[2][LPH];
    const int a_rows = M - m0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int left = bsrc.template rows_left<BN>(bn, h);
#pragma unroll
        for (int i = 0; i < LPH; ++i) {
            const int rl = (wave * LPH + i) * 8 + (lane >> 3);
            const int c = (lane & 7) ^ ((rl >> 1) & 7);
            const int ra = min(h * H + rl, a_rows - 1), rb = min(rl, left - 1);   // rows past the end repeat the last
            ao[h][i] = (uint32_t)((ra * lda + c * 8) * 2);
            bo[h][i] = (uint32_t)((rb * bsrc.ldb + c * 8) * 2);
        }
    }
    const char* const abase = reinterpret_cast<const char*>(A + (int64_t)m0 * lda) + kz;
    const char* const bbase[2] = {reinterpret_cast<const char*>(bsrc.template base<BN>(bn, 0)) + kz,
                                  reinterpret_cast<const char*>(bsrc.template base<BN>(bn, 1)) + kz};
    auto scalar_ptr = [](const char* p) -> const char* {   // keeps the base in scalar registers
        const uint64_t u = reinterpret_cast<uint64_t>(p);
        const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
        const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
        return reinterpret_cast<const char*>((hi << 32) | lo);
    };
    auto load_half = [&](const char* base, uint32_t (&off)[LPH], int lds_at, int kt) __attribute__((always_inline)) {
        unrolled<LPH>([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value;
            const char* g = scalar_ptr(base + (int64_t)kt * ROWB - i * 1024);   // the immediate adds it back
            asm volatile("" : "+v"(off[i]));   // keeps the offset a 32-bit register operand of the load
            dma16_at<i * 1024>(g + off[i], reinterpret_cast<bf16_t*>(smem + lds_at + wave * LPH * 1024));
        });
    };
    auto load_a = [&](int h, int buf, int kt) __attribute__((always_inline)) { load_half(abase, ao[h], buf * BUF + h * HALF, kt); };
    auto load_b = [&](int h, int buf, int kt) __attribute__((always_inline)) { load_half(bbase[h], bo[h], buf * BUF + (2 + h) * HALF, kt); };

    f32x4 acc[2][2][UM][UN];                           // [row half][column half]
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int i = 0; i < UM; ++i)
#pragma unroll
            for (int j = 0; j < UN; ++j) acc[x >> 1][x & 1][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int frow = lane & 15, fk = lane >> 4;
    const int fsw = (frow >> 1) & 7;
    const uint32_t smem_base = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)smem;
    uint32_t a_addr[2][2], b_addr[2][2];               // [buffer][k-step of 32 columns]
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const uint32_t at = smem_base + b * BUF + frow * ROWB + ((fk + 4 * ks) ^ fsw) * 16;
            a_addr[b][ks] = at + wr * (H / 2) * ROWB;
            b_addr[b][ks] = at + 2 * HALF + wc * (H / 4) * ROWB;
        }
    bf16x8 af[2][UM], b0[2][2][UN], b1[2][UN];         // [k-step][16-row tile]; B0 of two K tiles
    auto read_a = [&](auto bufc, auto hc) __attribute__((always_inline)) {
        constexpr int buf = decltype(bufc)::value, h = decltype(hc)::value;
        unrolled<2 * UM>([&](auto xc) __attribute__((always_inline)) {
            constexpr int x = decltype(xc)::value, ks = x / UM, i = x % UM;
            af[ks][i] = lds_read16<h * HALF + i * 16 * ROWB>(a_addr[buf][ks]);
        });
    };
    auto read_b = [&](auto bufc, auto hc, bf16x8 (&dst)[2][UN]) __attribute__((always_inline)) {
        constexpr int buf = decltype(bufc)::value, h = decltype(hc)::value;
        unrolled<2 * UN>([&](auto xc) __attribute__((always_inline)) {
            constexpr int x = decltype(xc)::value, ks = x / UN, i = x % UN;
            dst[ks][i] = lds_read16<h * HALF + i * 16 * ROWB>(b_addr[buf][ks]);
        });
    };
    // orders the uses of hand-read fragments behind the wait in front of this
    auto arrived_a = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < 2 * UM; ++x) asm volatile("" : "+v"(af[x / UM][x % UM]));
    };
    auto arrived_b = [&](bf16x8 (&dst)[2][UN]) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < 2 * UN; ++x) asm volatile("" : "+v"(dst[x / UN][x % UN]));
    };
    // end of a memory part: at most VM of this wave's loads are out, its reads have returned
    auto wait_bar = [&](auto vmc) __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(decltype(vmc)::value));
        wg_barrier();
    };
    auto compute = [&](f32x4 (&c)[UM][UN], bf16x8 (&b)[2][UN]) __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < UM; ++i)
#pragma unroll
                for (int j = 0; j < UN; ++j)
                    c[i][j] = DIRECT ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[ks][j], af[ks][i], c[i][j], 0, 0, 0)
                                     : __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[ks][i], b[ks][j], c[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        wg_barrier();
    };
#define CC_IC(x) std::integral_constant<int, (x)>{}
    // One K tile; `left` = K tiles after this one whose loads are still to be issued or waited for
    // (2: steady state, 1: the last but one, 0: the last).
    auto k_tile = [&](auto bufc, auto leftc, int kt) __attribute__((always_inline)) {
        constexpr int buf = decltype(bufc)::value, left = decltype(leftc)::value;
        read_a(bufc, CC_IC(0));
        if constexpr (left > 0) load_a(1, buf ^ 1, kt + 1);
        wait_bar(CC_IC(left > 0 ? 5 * LPH : LPH));
        arrived_a();
        arrived_b(b0[buf]);
        compute(acc[0][0], b0[buf]);

        read_b(bufc, CC_IC(1), b1);
        if constexpr (left > 1) load_b(0, buf, kt + 2);
        wait_bar(CC_IC(left > 1 ? 5 * LPH : left > 0 ? 4 * LPH : 0));
        arrived_b(b1);
        compute(acc[0][1], b1);

        read_a(bufc, CC_IC(1));
        if constexpr (left > 1) load_a(0, buf, kt + 2);
        wait_bar(CC_IC(left > 1 ? 5 * LPH : left > 0 ? 3 * LPH : 0));
        arrived_a();
        compute(acc[1][1], b1);

        if constexpr (left > 0) read_b(CC_IC(buf ^ 1), CC_IC(0), b0[buf ^ 1]);
        if constexpr (left > 1) load_b(1, buf, kt + 2);
        wait_bar(CC_IC(left > 1 ? 5 * LPH : left > 0 ? 2 * LPH : 0));
        if constexpr (left > 0) arrived_b(b0[buf ^ 1]);
        compute(acc[1][0], b0[buf]);
    };
    const int KT = K / 64;                             // even and >= 2 (K % 128 == 0)
    load_b(0, 0, 0);
    load_a(0, 0, 0);
    load_b(1, 0, 0);
    load_a(1, 0, 0);
    load_b(0, 1, 1);
    load_a(0, 1, 1);
    load_b(1, 1, 1);
    wait_bar(CC_IC(5 * LPH));                          // B0(0) and A0(0) are in place
    read_b(CC_IC(0), CC_IC(0), b0[0]);
    asm volatile("s_waitcnt lgkmcnt(0)");
    arrived_b(b0[0]);
    if (wr) wg_barrier();                              // the second group runs one barrier behind
    int kt = 0;
    for (; kt + 2 < KT; kt += 2) {
        k_tile(CC_IC(0), CC_IC(2), kt);
        k_tile(CC_IC(1), CC_IC(2), kt + 1);
    }
    k_tile(CC_IC(0), CC_IC(1), kt);
    k_tile(CC_IC(1), CC_IC(0), kt + 1);
    if (!wr) wg_barrier();
#undef CC_IC

    const auto e2 = epi_for_tile(epi, vb - vb0, m0);
    if constexpr (DIRECT) {
        // ---- epilogue from the registers (lane L has columns 4 (L/16) .. + 3 of row L%16 of a 16x16 tile): no pass through
        //      LDS and no barrier, so the waves that are done store while the others still multiply ----
        const int cl = wc * (H / 4) + 4 * fk;
        auto row = [&](int ha, int i) __attribute__((always_inline)) { return m0 + ha * H + wr * (H / 2) + i * 16 + frow; };
        if constexpr (Epi::COLS == 2) {                // B0 and B1 hold the two columns of an output column
#pragma unroll
            for (int x = 0; x < 2 * UM; ++x) {
                const int ha = x / UM, i = x % UM, m = row(ha, i);
                e2.template two<BN>(m, bn, cl, fk, acc[ha][0][i], acc[ha][1][i], m < M);
            }
        } else {
            int key[2][UM];
#pragma unroll
            for (int x = 0; x < 2 * UM; ++x) key[x / UM][x % UM] = e2.key(min(row(x / UM, x % UM), M - 1));
#pragma unroll
            for (int ha = 0; ha < 2; ++ha) {
                typename Epi::Two p[UM][2];
#pragma unroll
                for (int x = 0; x < 2 * UM; ++x)
                    p[x >> 1][x & 1] = e2.template ask<BN>(min(row(ha, x >> 1), M - 1), bn, (x & 1) * H + cl, key[ha][x >> 1]);
#pragma unroll
                for (int x = 0; x < 2 * UM; ++x) {
                    const int i = x >> 1, hb = x & 1, m = row(ha, i);
                    e2.template two<BN>(m, bn, hb * H + cl, fk, acc[ha][hb][i], p[i][hb], m < M);
                }
            }
        }
        return;
    }
    // ---- epilogue: one row half at a time through LDS as fp32 [H][BN], column c of row r at
    //      c ^ 16*((r>>2)&3) (the four 16-lane groups of an accumulator store hit disjoint banks) ----
    constexpr int TPR = BN / Epi::COLS / 8, RPP = 512 / TPR;       // threads per row, rows per pass
    float* stage = reinterpret_cast<float*>(smem);
    const int cc = (tid % TPR) * 8;
#pragma unroll
    for (int ha = 0; ha < 2; ++ha) {
        __syncthreads();
#pragma unroll
        for (int hb = 0; hb < 2; ++hb)
#pragma unroll
            for (int i = 0; i < UM; ++i)
#pragma unroll
                for (int j = 0; j < UN; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int r = wr * (H / 2) + i * 16 + 4 * fk + v;
                        const int c = hb * H + wc * (H / 4) + j * 16 + frow;
                        stage[r * BN + (c ^ (fk << 4))] = acc[ha][hb][i][j][v];
                    }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < H / RPP; ++k) {
            const int r = tid / TPR + k * RPP;
            const int m = m0 + ha * H + r;
            if (m < M) e2.template operator()<BN>(m, bn, cc, stage + r * BN, ((r >> 2) & 3) << 4);
        }
    }
}

template <class BSrc, class Epi>
__global__ __launch_bounds__(512, 2) void gemm_pingpong_kernel(
    const bf16_t* __restrict__ A, int lda, int M, int K, int k_more, int tiles_m, int tiles_n, int GM, int nb, int vb0,
    BSrc bsrc, Epi epi) {
    pingpong<Epi::DIRECT>(A, lda, M, K, k_more, tiles_m, tiles_n, GM, nb, vb0, bsrc, epi);
}
// Shares of K with the operands as QKV has them and the sums through LDS.  Row tiles that end past M read their last row again
// and again; as the second operand of the MFMAs such rows cost power, and with it clocks, even where nothing is stored
// (65 rows, d = 8192, down in 8 shares: 93.5 us this way, 123 from the accumulators, 120.6 with the stores left out).
template <class BSrc, class Epi>
__global__ __launch_bounds__(512, 2) void gemm_pingpong_parts_kernel(
    const bf16_t* __restrict__ A, int lda, int M, int K, int k_more, int tiles_m, int tiles_n, int GM, int nb, int vb0,
    BSrc bsrc, Epi epi) {
    pingpong<false>(A, lda, M, K, k_more, tiles_m, tiles_n, GM, nb, vb0, bsrc, epi);
}

// ------------------------------------------------------------------ duo loop
// 256x128 and 128x128 tiles, whole K tiles of 64 columns, eight waves of 64x64 in two groups half a step
// apart as in the ping-pong loop: one group multiplies a K tile (32 MFMAs, 512 clocks of the pipe) while the
// other reads the fragments of its next one and asks for the one after.  A wave of 64x64 reads 16 fragments for
// 32 MFMAs.  256x128: the groups are the upper and the lower 128 rows and share B.  128x128: the groups
// take the even and the odd K tiles (each holds sums of the whole tile, added at the end), for a 64x32
// wave would read half as much again per MFMA.
//
// What bounds it: the arrival of its K tiles.  With every load in the same column 128x128 takes 0.27 us per K tile, with real
// addresses 0.56 (57 KB/us a CU).  It is neither the L2's rate (150 KB/us a CU in a kernel of nothing but loads that hit) nor the
// lines that the L2 does not hold: QKV of 1025 rows, d = 4096 (256x128) finds 75 % of its requests there and takes 12 of its 46 KB/us
// a CU from behind it, QKV and O of 1787 rows, d = 3584 find 81 and 77 %, with the matrix pipes busy in 0.68, 0.56 and 0.48 of the
// CUs' busy clocks.  The L2 asked ahead by a ninth wave changed nothing.  A wave's loads go between its fragment
// reads: eight in a row wait for one another (16 clocks each for every wave that issues them), which the reads
// behind them then wait for too (128x128 0.36 us per K tile instead of 0.27, all in the same column).
// LDS: 256x128 three slots of A0 | A1 | B (48 KB), 128x128 five of A | B (32 KB); a K tile is asked for
// four half steps before it is read (the second group's half of a shared B three).
// Against the ring loop with the same tile, event us of 2.5 more than the kernel's: M = 883, d = 4096: O (128x128)
// 59.8 -> 44.0, QKV (256x128) 79.9 -> 63 (256x256 tiles in 2 and 4 shares, which such calls took before: 55.9, 69.2);  M = 1523, d = 3584:
// QKV 80.8 -> 61, O 79 -> 62 (256x128);  M = 3404, N = 2048,
// K = 256 (432 tiles of 128x128, two on a CU in the ring loop) 14.5 -> 19, where the ring loop stays.
template <int BM, class BSrc, class Epi>
__global__ __launch_bounds__(512, 2) void gemm_duo_kernel(
    const bf16_t* __restrict__ A, int lda, int M, int K, int k_more, int tiles_m, int tiles_n, int GM, int nb, int vb0,
    BSrc bsrc, Epi epi) {
    constexpr int BN = 128, KG = 256 / BM;             // waves of 64x64; groups along K
    static_assert(BM == 128 || BM == 256, "eight waves");
    constexpr int AR = BM / 128;                       // 128-row regions of A in a K tile
    constexpr int ROWB = 128, REG = 128 * ROWB;        // bytes of a K tile's row and of a region
    constexpr int SLOT = (AR + 1) * REG, NSLOT = KG == 2 ? 5 : 3;
    constexpr int LA = 4, LB = KG == 2 ? 4 : 2, L = LA + LB;        // loads of a wave and K tile, 8 rows each
    static_assert(BM * BN * 4 <= NSLOT * SLOT, "the fp32 tile fits for the epilogue");
    __shared__ __align__(16) char smem[NSLOT * SLOT];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave >> 2, w = wave & 3;
    int bm, bn;
    const int vb = tile_of_block(blockIdx.x, nb, vb0, tiles_m, tiles_n, GM, &bm, &bn);
    const int m0 = bm * BM;
    int64_t kz;                                        // this workgroup row's share of K
    K = k_share<CC_GEMM_GROUP>(K, k_more, &kz);
    const int ar = AR == 2 ? grp : 0;                  // this group's region of A

    // ---- global -> LDS: wave w of a group moves rows 32 w .. of the group's A region and rows 32 w .. of B (of a
    //      K tile that both groups read, the eight waves 16 rows each); lane L fills slot L%8 of row L/8.
    //      Wave-uniform bases advance along K in scalar registers. ----
    uint32_t ao[LA], bo[LB];
    const int ra0 = w * 32, rb0 = (KG == 2 ? w : wave) * 8 * LB;
    const int bh = rb0 / (BN / 2);                     // half of the tile that the wave's B rows lie in
    const int a_rows = M - m0, left = bsrc.template rows_left<BN>(bn, bh);
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int r = ra0 + i * 8 + (lane >> 3);
        ao[i] = (uint32_t)((min(ar * 128 + r, a_rows - 1) * lda + ((lane & 7) ^ ((r >> 1) & 7)) * 8) * 2);   // rows past the end repeat the last
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int r = rb0 + i * 8 + (lane >> 3);
        bo[i] = (uint32_t)((min(r - bh * (BN / 2), left - 1) * bsrc.ldb + ((lane & 7) ^ ((r >> 1) & 7)) * 8) * 2);
    }
    const char* const abase = reinterpret_cast<const char*>(A + (int64_t)m0 * lda) + kz;
    const char* const bbase = reinterpret_cast<const char*>(bsrc.template base<BN>(bn, bh)) + kz;
    auto scalar_ptr = [](const char* p) -> const char* {   // keeps the base in scalar registers
        const uint64_t u = reinterpret_cast<uint64_t>(p);
        const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
        const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
        return reinterpret_cast<const char*>((hi << 32) | lo);
    };
    // load i of K tile kt into a slot: B's first
    auto load_one = [&](auto ic, int kt, int slot) __attribute__((always_inline)) {
        constexpr int x = decltype(ic)::value;
        if constexpr (x < LB) {
            const char* g = scalar_ptr(bbase + (int64_t)kt * ROWB - x * 1024);   // the immediate adds it back
            asm volatile("" : "+v"(bo[x]));   // keeps the offset a 32-bit register operand of the load
            dma16_at<x * 1024>(g + bo[x], reinterpret_cast<bf16_t*>(smem + slot * SLOT + AR * REG + rb0 * ROWB));
        } else {
            constexpr int i = x - LB;
            const char* g = scalar_ptr(abase + (int64_t)kt * ROWB - i * 1024);
            asm volatile("" : "+v"(ao[i]));
            dma16_at<i * 1024>(g + ao[i], reinterpret_cast<bf16_t*>(smem + slot * SLOT + ar * REG + ra0 * ROWB));
        }
    };

    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int frow = lane & 15, fk = lane >> 4;
    const int fsw = (frow >> 1) & 7;
    const uint32_t smem_base = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)smem;
    uint32_t a_addr[2], b_addr[2];                     // [k-step of 32 columns], in slot 0
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const uint32_t at = smem_base + frow * ROWB + ((fk + 4 * ks) ^ fsw) * 16;
        a_addr[ks] = at + ar * REG + (w & 1) * 64 * ROWB;
        b_addr[ks] = at + AR * REG + (w >> 1) * 64 * ROWB;
    }
    bf16x8 af[2][4], bf[2][4];

    // The K tiles of this group are KG n + (KG == 2 ? grp : 0), n < NT, in slots by their index modulo NSLOT.
    const int k0 = KG == 2 ? grp : 0, NT = K / 64 / KG;             // K % 128 == 0
    int rd = k0, wrs = KG == 2 ? (grp ? 0 : 4) : 2;                 // slots of tiles n and n + 2
    using yes = std::integral_constant<int, 1>;
    using no = std::integral_constant<int, 0>;
    // One K tile: 16 fragment reads with the loads of tile n + 2 between them, barrier, 32 MFMAs, barrier.
    auto k_tile = [&](auto loadc, int n) __attribute__((always_inline)) {
        constexpr bool LOAD = decltype(loadc)::value;
        const uint32_t at = rd * SLOT;
        const uint32_t a0 = a_addr[0] + at, a1 = a_addr[1] + at, b0 = b_addr[0] + at, b1 = b_addr[1] + at;
        unrolled<8>([&](auto xc) __attribute__((always_inline)) {
            constexpr int x = decltype(xc)::value, ks = x >> 2, y = (x & 1) * 2;
            if constexpr ((x & 2) == 0) {
                bf[ks][y] = lds_read16<y * 16 * ROWB>(ks ? b1 : b0);
                bf[ks][y + 1] = lds_read16<(y + 1) * 16 * ROWB>(ks ? b1 : b0);
            } else {
                af[ks][y] = lds_read16<y * 16 * ROWB>(ks ? a1 : a0);
                af[ks][y + 1] = lds_read16<(y + 1) * 16 * ROWB>(ks ? a1 : a0);
            }
            if constexpr (LOAD && x < L) {
                __builtin_amdgcn_sched_barrier(0);
                load_one(xc, KG * (n + 2) + k0, wrs);
                __builtin_amdgcn_sched_barrier(0);
            }
        });
        // where the groups share B: this wave's part of tile n + 1 has landed (the other group reads it next)
        if constexpr (KG == 1 && LOAD) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(L + LA));
        else if constexpr (KG == 1) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)");
        else asm volatile("s_waitcnt lgkmcnt(0)");
#pragma unroll
        for (int x = 0; x < 8; ++x) asm volatile("" : "+v"(af[x >> 2][x & 3]), "+v"(bf[x >> 2][x & 3]));
        wg_barrier();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[ks][i], bf[ks][j], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (LOAD) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(L));      // tile n + 1 has landed
        else asm volatile("s_waitcnt vmcnt(0)");
        wg_barrier();
        rd = rd + KG >= NSLOT ? rd + KG - NSLOT : rd + KG;
        wrs = wrs + KG >= NSLOT ? wrs + KG - NSLOT : wrs + KG;
    };
    unrolled<L>([&](auto x) __attribute__((always_inline)) { load_one(x, k0, rd); });
    if (NT > 1) {
        unrolled<L>([&](auto x) __attribute__((always_inline)) { load_one(x, KG + k0, rd + KG); });
        asm volatile("s_waitcnt vmcnt(%0)" : : "n"(L));
    } else {
        asm volatile("s_waitcnt vmcnt(0)");
    }
    wg_barrier();                                      // the first K tile of either group is in place
    if (grp) wg_barrier();                             // the second group runs one barrier behind
    int n = 0;
    for (; n + 2 < NT; ++n) k_tile(yes{}, n);
    for (; n < NT; ++n) k_tile(no{}, n);
    if (!grp) wg_barrier();

    // ---- epilogue through LDS as fp32 [BM][BN], column c of row r at c ^ 16*((r>>2)&3) (the four 16-lane
    //      groups of an accumulator store hit disjoint banks); with two groups along K the second
    //      leaves its sums there and the first adds them to its own ----
    __syncthreads();
    float* stage = reinterpret_cast<float*>(smem);
    auto each = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = ar * 128 + (w & 1) * 64 + i * 16 + 4 * fk + v;
                    const int c = (w >> 1) * 64 + j * 16 + frow;
                    f(stage[r * BN + (c ^ (fk << 4))], acc[i][j][v]);
                }
    };
    if (KG == 1 || grp == 1) each([](float& at, float v) __attribute__((always_inline)) { at = v; });
    __syncthreads();
    if constexpr (KG == 2) {
        if (grp == 0) each([](float& at, float v) __attribute__((always_inline)) { at = v + at; });
        __syncthreads();
    }
    constexpr int TPR = BN / Epi::COLS / 8, RPP = 512 / TPR;       // threads per row, rows per pass
    const auto e2 = epi_for_tile(epi, vb - vb0, m0);
    const int cc = (tid % TPR) * 8;
#pragma unroll
    for (int k = 0; k < BM / RPP; ++k) {
        const int r = tid / TPR + k * RPP;
        const int m = m0 + r;
        if (m < M) e2.template operator()<BN>(m, bn, cc, stage + r * BN, ((r >> 2) & 3) << 4);
    }
}

// ------------------------------------------------------------------ thin tiles
// 64x128 tiles for few rows, where a call reads a whole weight matrix for one or two row tiles.
//
// What bounds it: the weight stream from HBM, so bytes in flight count and matrix work does not.
// The 256-row tiles above pad 64 rows to 256: three quarters of the MFMAs, of the A loads and of
// the LDS reads are for rows that do not exist, and with 96 KB a K tile the ring holds little of B.
// Here a slice is 64 columns (whole 128-byte lines, 8 KB of A + 16 KB of B) and six slots (144 KB
// of LDS, one workgroup per CU) keep five slices = 80 KB of weights per CU on the way.  Four waves
// of 64x32; one barrier per slice; any K % 64 == 0.  Column tile bn starts bn slices into K and
// wraps round: rows of a weight matrix are a power of two bytes apart as often as not, and
// workgroups that walk K in step then ask the same few memory channels at any one time (a layer of
// 64 rows, d = 4096: 176 us in step, 164 rotated).  With one row tile every line of B is read once and,
// where the plan says so, is not kept in the caches (nt): 7.1 TB/s instead of 6.0 in a kernel of nothing but loads, gate/up below 46 -> 41.4;
// with more row tiles the others find it there (M = 128, O 19.3 us, 21.1 with nt).  The loads of a slice lie
// between its fragment reads and MFMAs, in a loop without conditions (the last five slices are a loop of
// their own): O and QKV at 16 rows 16.6 -> 16.2 and 17.7 -> 17.1.
// Swizzle and fragment layout as in the ping-pong loop.
// M = 64, d = 4096, f = 14336, event microseconds with the finishing pass, weights cold (870 MB of others
// between two reads), 256-row tiles and these: gate/up 65 -> 41 (6.1 TB/s of weights without the events' 2.5 us), down 41 -> 28,
// QKV 26 -> 20, O 24 -> 18.  Slices of 128 columns in three slots: the same within 2 % over these shapes, gate/up
// slower by a fifth at 64 rows.
// Launch bounds: 512 threads where 256 are launched, so that a wave has 256 registers.  With 512 of them the compiler kept the
// sums in accumulation registers and, in a loop without conditions, moved 20 of them to vector registers and back in every
// slice, between the MFMAs (140 instructions a slice, now 81).  M = 1 without shares, d = 4096: QKV 31.2 us in the loop
// with conditions, 33.3 so, 26.3 now; 768 rows, N = 2880, K = 7744: 104.7, 110.0, 83.7; d = 576, 512 rows, gate/up 11.1, 10.0, 9.1.
constexpr int THIN_M = CC_THIN_M, THIN_N = CC_THIN_N, THIN_SLOTS = 6;
template <class BSrc, class Epi>
__global__ __launch_bounds__(512, 2) void gemm_thin_kernel(const bf16_t* __restrict__ A, int lda, int M, int K, int k_more,
                                                           int tiles_m, int tiles_n, int GM, int nb, int stream,
                                                           BSrc bsrc, Epi epi) {
    constexpr int BM = THIN_M, BN = THIN_N, D = THIN_SLOTS, ROWB = 128;
    constexpr int A_L = 2, B_L = 4, LPS = A_L + B_L;   // loads of a wave and slice (8 rows each)
    constexpr int SLOT = (BM + BN) * ROWB;
    static_assert(BM * BN * 4 <= D * SLOT && LPS * (D - 2) < 64, "epilogue space, vmcnt range");
    __shared__ __align__(16) char smem[D * SLOT];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int bm, bn;
    const int vb = tile_of_block(blockIdx.x, nb, 0, tiles_m, tiles_n, GM, &bm, &bn);
    const int m0 = bm * BM;
    int64_t kz;                                        // this workgroup row's share of K
    K = k_share<64>(K, k_more, &kz);

    // ---- global -> LDS: wave w moves rows 16w .. of A and 32w .. of B; lane L fills slot L%8 of row L/8 ----
    uint32_t ao[A_L], bo[B_L];
    const int hb = wave >> 1;                          // half of the tile that the wave's B rows lie in
    const int left = bsrc.template rows_left<BN>(bn, hb);
#pragma unroll
    for (int i = 0; i < A_L; ++i) {
        const int r = wave * 16 + i * 8 + (lane >> 3);
        ao[i] = (uint32_t)((min(r, M - m0 - 1) * lda + ((lane & 7) ^ ((r >> 1) & 7)) * 8) * 2);
    }
#pragma unroll
    for (int i = 0; i < B_L; ++i) {
        const int r = wave * 32 + i * 8 + (lane >> 3);
        bo[i] = (uint32_t)((min(r - hb * (BN / 2), left - 1) * bsrc.ldb + ((lane & 7) ^ ((r >> 1) & 7)) * 8) * 2);
    }
    const char* const abase = reinterpret_cast<const char*>(A + (int64_t)m0 * lda) + kz;
    const char* const bbase = reinterpret_cast<const char*>(bsrc.template base<BN>(bn, hb)) + kz;
    auto scalar_ptr = [](const char* p) -> const char* {   // keeps the base in scalar registers
        const uint64_t u = reinterpret_cast<uint64_t>(p);
        const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
        const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
        return reinterpret_cast<const char*>((hi << 32) | lo);
    };
    const int KT = K / 64, rot = bn < KT ? bn : bn % KT;
    // load i of slice n: B's first
    auto load_one = [&](auto xc, auto streamc, int n, int slot) __attribute__((always_inline)) {
        constexpr int x = decltype(xc)::value;
        const int t = n + rot < KT ? n + rot : n + rot - KT;
        if constexpr (x < B_L) {
            const char* g = scalar_ptr(bbase + (int64_t)t * ROWB - x * 1024);   // the immediate adds it back
            bf16_t* at = reinterpret_cast<bf16_t*>(smem + slot * SLOT + BM * ROWB + wave * B_L * 1024);
            asm volatile("" : "+v"(bo[x]));
            if constexpr (decltype(streamc)::value) dma16_stream_at<x * 1024>(g + bo[x], at);
            else dma16_at<x * 1024>(g + bo[x], at);
        } else {
            constexpr int i = x - B_L;
            const char* g = scalar_ptr(abase + (int64_t)t * ROWB - i * 1024);
            asm volatile("" : "+v"(ao[i]));
            dma16_at<i * 1024>(g + ao[i], reinterpret_cast<bf16_t*>(smem + slot * SLOT + wave * A_L * 1024));
        }
    };

    f32x4 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int frow = lane & 15, fk = lane >> 4;
    const int fsw = (frow >> 1) & 7;
    const uint32_t smem_base = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)smem;
    uint32_t a_addr[2], b_addr[2];                     // [k-step of 32 columns]
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        a_addr[ks] = smem_base + frow * ROWB + ((fk + 4 * ks) ^ fsw) * 16;
        b_addr[ks] = a_addr[ks] + (BM + wave * 32) * ROWB;
    }
    const auto e2 = epi_for_tile(epi, vb, m0);
    constexpr int TPR = BN / Epi::COLS / 8, RPP = 256 / TPR;       // threads per row, rows per pass
    const int cc = (tid % TPR) * 8;
    typename std::remove_const_t<decltype(e2)>::Pre pre[BM / RPP];
    // What the epilogue needs from memory is asked for ahead of the first slices (loads return in order).  Behind them the compiler,
    // which cannot count the loads that a short K leaves out, waited for every slice before it asked and, with one row
    // tile, again before the first and in the last ones (O by gathered rows, cold: 64 rows, d = 512 10.0 -> 8.8 us, 512 rows,
    // d = 1024 12.3 -> 12.0; one row, d = 4096 26.7 -> 25.4; all of it behind the K loop 9.3, 13.1, 25.7).
    int key[BM / RPP];
#pragma unroll
    for (int k = 0; k < BM / RPP; ++k) key[k] = e2.key(min(m0 + tid / TPR + k * RPP, M - 1));
    if constexpr (Epi::ASKS_BY_KEY)                    // one wait for all keys, then all loads by them
#pragma unroll
        for (int k = 0; k < BM / RPP; ++k) asm volatile("" : "+v"(key[k]));
#pragma unroll
    for (int k = 0; k < BM / RPP; ++k) pre[k] = e2.template pre<BN>(min(m0 + tid / TPR + k * RPP, M - 1), bn, cc, key[k]);
    auto k_loop = [&](auto streamc) __attribute__((always_inline)) {
        int rd = 0, wrs = D - 1;                       // slots of slice t and of slice t + D - 1
        // One slice, with at most `younger` slices' loads out when it is read.  The loads of slice t + D - 1 go
        // between the fragment reads and between the MFMAs: a wave's loads in a row wait for one another
        // (64 clocks each with four waves at it), and nothing behind them starts meanwhile.
        auto slice = [&](auto loadc, auto youngerc, int t) __attribute__((always_inline)) {
            constexpr bool LOAD = decltype(loadc)::value;
            asm volatile("s_waitcnt vmcnt(%0)" : : "n"(decltype(youngerc)::value * LPS));
            wg_barrier();                              // for every wave; and slot wrs (slice t - 1) has been read
            auto load = [&](auto xc) __attribute__((always_inline)) {
                if constexpr (LOAD) {
                    __builtin_amdgcn_sched_barrier(0);
                    load_one(xc, streamc, t + D - 1, wrs);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            bf16x8 af[2][4], bf[2][2];
            const uint32_t at = rd * SLOT;
            unrolled<2>([&](auto kc) __attribute__((always_inline)) {
                constexpr int ks = decltype(kc)::value;
                const uint32_t a = a_addr[ks] + at, b = b_addr[ks] + at;
                unrolled<2>([&](auto ic) __attribute__((always_inline)) { bf[ks][ic.value] = lds_read16<ic.value * 16 * ROWB>(b); });
                unrolled<4>([&](auto ic) __attribute__((always_inline)) { af[ks][ic.value] = lds_read16<ic.value * 16 * ROWB>(a); });
                load(std::integral_constant<int, ks>{});
            });
            unrolled<2>([&](auto kc) __attribute__((always_inline)) {
                constexpr int ks = decltype(kc)::value;
                if constexpr (ks == 0) asm volatile("s_waitcnt lgkmcnt(6)");
                else asm volatile("s_waitcnt lgkmcnt(0)");
#pragma unroll
                for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(af[ks][i]));
#pragma unroll
                for (int j = 0; j < 2; ++j) asm volatile("" : "+v"(bf[ks][j]));
                unrolled<2>([&](auto hc) __attribute__((always_inline)) {
                    constexpr int hh = decltype(hc)::value;
#pragma unroll
                    for (int i = 2 * hh; i < 2 * hh + 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[ks][i], bf[ks][j], acc[i][j], 0, 0, 0);
                    load(std::integral_constant<int, 2 + 2 * ks + hh>{});
                });
            });
            wrs = rd;
            rd = rd + 1 == D ? 0 : rd + 1;
        };
        static_assert(LPS == 6, "places of the loads");
        unrolled<D - 1>([&](auto tc) __attribute__((always_inline)) {
            if (tc.value < KT) unrolled<LPS>([&](auto xc) __attribute__((always_inline)) { load_one(xc, streamc, tc.value, tc.value); });
        });
        int t = 0;
        for (; t + D - 1 < KT; ++t) slice(std::true_type{}, std::integral_constant<int, D - 2>{}, t);
        // the last D - 1 slices (or all of a shorter K): nothing left to load
        unrolled<D - 1>([&](auto jc) __attribute__((always_inline)) {
            constexpr int after = D - 2 - decltype(jc)::value;
            if (KT > after) slice(std::false_type{}, std::integral_constant<int, after>{}, t);
        });
    };
    if (stream) k_loop(std::true_type{});
    else k_loop(std::false_type{});

    // ---- epilogue through LDS as fp32 [BM][BN], column c of row r at c ^ 16*((r>>2)&3) ----
    __syncthreads();
    float* stage = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = i * 16 + 4 * fk + v, c = wave * 32 + j * 16 + frow;
                stage[r * BN + (c ^ (fk << 4))] = acc[i][j][v];
            }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < BM / RPP; ++k) {
        const int r = tid / TPR + k * RPP;
        const int m = m0 + r;
        if (m < M) e2.template operator()<BN>(m, bn, cc, stage + r * BN, ((r >> 2) & 3) << 4, pre[k]);
    }
}

// cc_plan_gemm picks the tile shape and the shares of K: a grid runs as a whole number of "rounds" of
// workgroups, so the shape is chosen per launch to minimise rounds x tile cost.
template <class BSrc, class Epi>
void launch_gemm(const bf16_t* A, int lda, int M, int N_tiles_cols, int K, int ldb, int gm_big,
                 BSrc bsrc, Epi epi, float* ws, int64_t ws_floats, const cc_launch_override& ovr,
                 hipStream_t s) {
    const int n_cu = cc_device_cus();
    const cc_gemm_plan plan = cc_plan_gemm(n_cu, M, N_tiles_cols, K, lda, ldb, ws != nullptr, ws_floats, ovr);
    const char pick = plan.tile;
    const bool ring = plan.ring, mfma16 = !ovr.gemm_mfma32;
    const int S = plan.shares;
    if (pick == 't') {
        const int tiles_m = (M + THIN_M - 1) / THIN_M, tiles_n = (N_tiles_cols + THIN_N - 1) / THIN_N;
        const int GM = std::min(ovr.gemm_gm > 0 ? ovr.gemm_gm : 4, tiles_m);
        const int nt = tiles_m * tiles_n;
        if (S == 1) {
            hipLaunchKernelGGL((gemm_thin_kernel<BSrc, Epi>), dim3(nt), dim3(256), 0, s, A, lda, M, K, 0, tiles_m, tiles_n,
                               GM, nt, plan.stream, bsrc, epi);
        } else {
            constexpr int SLOT = THIN_M * THIN_N;
            EpiPartial<THIN_M> pe{ws, (int64_t)nt * SLOT, 0, 0};
            hipLaunchKernelGGL((gemm_thin_kernel<BSrc, EpiPartial<THIN_M>>), dim3(nt, S), dim3(256), 0, s, A, lda, M,
                               K / 64 / S * 64, K / 64 % S, tiles_m, tiles_n, GM, nt, plan.stream, bsrc, pe);
            hipLaunchKernelGGL((splitk_finish_kernel<THIN_M, THIN_N, Epi>), dim3(nt, THIN_M * THIN_N / 2048), dim3(256), 0, s,
                               ws, (int64_t)nt * SLOT, S, M, THIN_M, 0, tiles_m, tiles_n, GM, epi);
        }
        return;
    }
    const int bm = pick == 's' ? 128 : 256, bn = pick == 'b' ? 256 : 128;
    const int tiles_m = (M + bm - 1) / bm, tiles_n = (N_tiles_cols + bn - 1) / bn;
    int GM = pick == 's' ? 2 * gm_big : gm_big;
    if (ovr.gemm_gm > 0) GM = ovr.gemm_gm;
    GM = GM < 1 ? 1 : (GM > tiles_m ? tiles_m : GM);
    const int n_tiles = tiles_m * tiles_n, groups = K / CC_GEMM_GROUP;     // groups: where the ring loops apply, all of K
#define CC_LAUNCH(KERN, BM_, BN_, WM_, WN_, EPI_T, EPI_V, NB_, VB0_, GY_)                              \
    hipLaunchKernelGGL((KERN<BM_, BN_, WM_, WN_, BSrc, EPI_T>), dim3(NB_, GY_), dim3(WM_ * WN_ * 64), 0, s, A, \
                       lda, M, groups / (GY_) * CC_GEMM_GROUP, groups % (GY_), tiles_m, tiles_n, GM, NB_, VB0_, bsrc, EPI_V)
#define CC_LAUNCH_PP(KERN, EPI_T, EPI_V, NB_, VB0_, GY_)                                                \
    hipLaunchKernelGGL((KERN<BSrc, EPI_T>), dim3(NB_, GY_), dim3(512), 0, s, A, lda, M,    \
                       groups / (GY_) * CC_GEMM_GROUP, groups % (GY_), tiles_m, tiles_n, GM, NB_, VB0_, bsrc, EPI_V)
#define CC_LAUNCH_DUO(BM_, EPI_T, EPI_V, NB_, VB0_, GY_)                                                    \
    hipLaunchKernelGGL((gemm_duo_kernel<BM_, BSrc, EPI_T>), dim3(NB_, GY_), dim3(512), 0, s, A, lda, M,  \
                       groups / (GY_) * CC_GEMM_GROUP, groups % (GY_), tiles_m, tiles_n, GM, NB_, VB0_, bsrc, EPI_V)
#define CC_LAUNCH_NT(BM_, BN_, WM_, WN_)                                                                    \
    hipLaunchKernelGGL((gemm_nt_kernel<BM_, BN_, WM_, WN_, BSrc, Epi>), dim3(n_tiles), dim3(WM_ * WN_ * 64), 0, \
                       s, A, lda, M, K, tiles_m, tiles_n, GM, bsrc, epi)
    if (S > 1 && pick == 'h') {
        const int rem = n_tiles % n_cu == 0 ? n_cu : n_tiles % n_cu, full = n_tiles - rem;
        EpiPartial<256> pe{ws, (int64_t)rem * 32768, 0, 0};
        if (full) CC_LAUNCH_DUO(256, Epi, epi, full, 0, 1);
        CC_LAUNCH_DUO(256, EpiPartial<256>, pe, rem, full, S);
        hipLaunchKernelGGL((splitk_finish_kernel<256, 128, Epi>), dim3(rem, 16), dim3(256), 0, s, ws, (int64_t)rem * 32768, S,
                           M, bm, full, tiles_m, tiles_n, GM, epi);
    } else if (S > 1) {
        const int rem = n_tiles % n_cu == 0 ? n_cu : n_tiles % n_cu, full = n_tiles - rem;
        EpiPartial<256> pe{ws, (int64_t)rem * 65536, 0, 0};
        if (mfma16) {
            if (full) CC_LAUNCH_PP(gemm_pingpong_kernel, Epi, epi, full, 0, 1);
            if (plan.staged_parts) CC_LAUNCH_PP(gemm_pingpong_parts_kernel, EpiPartial<256>, pe, rem, full, S);
            else CC_LAUNCH_PP(gemm_pingpong_kernel, EpiPartial<256>, pe, rem, full, S);
        } else {
            if (full) CC_LAUNCH(gemm_ring_kernel, 256, 256, 2, 4, Epi, epi, full, 0, 1);
            CC_LAUNCH(gemm_ring_kernel, 256, 256, 2, 4, EpiPartial<256>, pe, rem, full, S);
        }
        hipLaunchKernelGGL((splitk_finish_kernel<256, 256, Epi>), dim3(rem, (bm + 7) / 8), dim3(256), 0, s, ws,
                           (int64_t)rem * 65536, S, M, bm, full, tiles_m, tiles_n, GM, epi);
    } else if (pick == 'b') {
        if (ring && mfma16) CC_LAUNCH_PP(gemm_pingpong_kernel, Epi, epi, n_tiles, 0, 1);
        else if (ring) CC_LAUNCH(gemm_ring_kernel, 256, 256, 2, 4, Epi, epi, n_tiles, 0, 1);
        else CC_LAUNCH_NT(256, 256, 2, 4);
    } else if (pick == 'h') {
        CC_LAUNCH_DUO(256, Epi, epi, n_tiles, 0, 1);
    } else {
        if (mfma16 && plan.duo) CC_LAUNCH_DUO(128, Epi, epi, n_tiles, 0, 1);
        else if (ring && mfma16) CC_LAUNCH(gemm_ring16_kernel, 128, 128, 2, 2, Epi, epi, n_tiles, 0, 1);
        else if (ring) CC_LAUNCH(gemm_ring_kernel, 128, 128, 2, 2, Epi, epi, n_tiles, 0, 1);
        else CC_LAUNCH_NT(128, 128, 2, 2);
    }
#undef CC_LAUNCH
#undef CC_LAUNCH_NT
#undef CC_LAUNCH_DUO
#undef CC_LAUNCH_PP
}

}  // namespace

void cc_launch_qkv(const bf16_t* xn, int M, const int32_t* idx, const bf16_t* w_qkv,
                   const bf16_t* b_qkv, const cc_model_desc& m, const float2* rope,
                   const cc_kv_layer& kv, bf16_t* q_out, float* ws, int64_t ws_floats,
                   const cc_launch_override& ovr, hipStream_t s) {
    if (M <= 0) return;
    const int N = (m.H_q + 2 * m.H_kv) * m.d_h;
    BSingle b{w_qkv, m.d, N};
    EpiQKV e{idx, b_qkv, rope, m.H_q, m.H_kv, m.d_h, N, q_out,
             (bf16_t*)kv.K, (bf16_t*)kv.V, kv.stride_token, kv.stride_head};
    launch_gemm(xn, m.d, M, N, m.d, m.d, 4, b, e, ws, ws_floats, ovr, s);
}

void cc_launch_oproj(const bf16_t* o, int M, const bf16_t* w_o, const bf16_t* hidden,
                     const int32_t* gather_idx, const cc_model_desc& m, float* y, float* ws,
                     int64_t ws_floats, const cc_launch_override& ovr, hipStream_t s) {
    if (M <= 0) return;
    const int K = m.H_q * m.d_h;
    BSingle b{w_o, K, m.d};
    EpiOProj e{hidden, gather_idx, m.d, y};
    launch_gemm(o, K, M, m.d, K, K, 4, b, e, ws, ws_floats, ovr, s);
}

void cc_launch_gate_up(const bf16_t* mn, int M, const bf16_t* w_gate, const bf16_t* w_up,
                       const cc_model_desc& m, bf16_t* act, float* ws, int64_t ws_floats,
                       const cc_launch_override& ovr, hipStream_t s) {
    if (M <= 0) return;
    BDual b{w_gate, w_up, m.d, m.f};
    EpiGateUp e{m.f, act};
    // each 128-column tile holds 64 gate + 64 up columns: 2*f tile columns in total
    launch_gemm(mn, m.d, M, 2 * m.f, m.d, m.d, 4, b, e, ws, ws_floats, ovr, s);
}

void cc_launch_down(const bf16_t* act, int M, const bf16_t* w_down, const float* y,
                    const cc_model_desc& m, bf16_t* out, float* ws, int64_t ws_floats,
                    const cc_launch_override& ovr, hipStream_t s) {
    if (M <= 0) return;
    BSingle b{w_down, m.f, m.d};
    EpiDown e{y, m.d, out};
    launch_gemm(act, m.f, M, m.d, m.f, m.f, 8, b, e, ws, ws_floats, ovr, s);
}
