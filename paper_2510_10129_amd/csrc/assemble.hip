// Online assembly of one layer's global KV cache from per-chunk caches
// (Section 4.1 of the paper): one copy of the shared prefix, every chunk's own
// rows appended, keys re-numbered from chunk-local to global positions by one
// more rotary rotation (rotations by p and by delta compose to p + delta).
// Pure data movement plus 2 multiply-adds per key element: bound by HBM.
//
// A wave owns a.rows consecutive destination rows of one segment, their keys (grid row 0)
// or their values (grid row 1).  A lane owns one unit of a row: of a key row one 16-byte piece
// of the low half of a head and the matching piece of the high half (the two members of every
// rotary pair meet in one lane; its (cos, sin) of the segment's position shift are loaded once and kept
// in registers), of a value row 16 bytes.  Rows of fewer than 64 units share a wave.  Loads of eight
// rows a lane are issued before their stores.
// Bytes in flight bound it; with keys and values of 16 rows in one wave and a row's units alone across
// its lanes a small model's request was a few waves deep in latency: H_kv = 2, d_h = 64, 1072 rows
// 14.5 -> 6.2 us by events (2.5 of it theirs); H_kv = 8, d_h = 128, 66k rows 111 -> 94 (5.9 TB/s), 10 us of it the second
// launch that 66 segments took, 5 the rows of a wave (cc_asm_rows).
#include "cc_internal.h"

namespace {

__device__ __forceinline__ bf16x8 zero8() {
    bf16x8 z;
#pragma unroll
    for (int u = 0; u < 8; ++u) z[u] = (bf16_t)0.0f;
    return z;
}

template <int D_H>
__global__ __launch_bounds__(256) void assemble_kernel(cc_asm_args a, const float2* __restrict__ rope,
                                                       int H_kv, int64_t src_st, int64_t src_sh,
                                                       bf16_t* __restrict__ Kd, bf16_t* __restrict__ Vd,
                                                       int64_t dst_st, int64_t dst_sh) {
    constexpr int HALF = D_H / 2;
    constexpr int UPH = HALF / 8;          // (lo, hi) 16-byte pairs per head
    constexpr int CPH = D_H / 8;           // 16-byte chunks per head
    constexpr int RU = 8;                  // rows in flight
    const int lane = threadIdx.x & 63;
    const int blk = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (blk >= a.n_blocks) return;
    int s = 0;                             // last segment whose first block is <= blk
    for (int lo = 0, hi = a.n_seg - 1; lo <= hi;) {
        const int mid = (lo + hi) >> 1;
        if (a.seg[mid].blk0 <= blk) { s = mid; lo = mid + 1; } else { hi = mid - 1; }
    }
    const cc_asm_seg sg = a.seg[s];
    const int r0 = (blk - sg.blk0) * a.rows;
    const int r1 = min(sg.len, r0 + a.rows);
    const bool zero = sg.K == nullptr;
    const int units = H_kv * (blockIdx.y ? CPH : UPH);
    const int rpw = units < 64 ? 64 / units : 1;      // rows side by side in the wave
    const int lr = units < 64 ? lane / units : 0;     // this lane's row of them
    if (lr >= rpw) return;
    const int u0 = lane - lr * units;
    const int step = RU * rpw;

    if (blockIdx.y == 0) {
        for (int u = u0; u < units; u += 64) {
            const int h = u / UPH, j0 = (u - h * UPH) * 8;
            float2 cs[8];
            if (sg.delta != 0) {
#pragma unroll
                for (int e = 0; e < 8; ++e) cs[e] = rope[(int64_t)sg.delta * HALF + j0 + e];
            }
            const bf16_t* src = sg.K + (int64_t)h * src_sh + j0;
            bf16_t* dst = Kd + (int64_t)sg.dst * dst_st + (int64_t)h * dst_sh + j0;
            for (int r = r0 + lr; r < r1; r += step) {
                bf16x8 lo[RU], hi[RU];
#pragma unroll
                for (int i = 0; i < RU; ++i) {
                    const int rr = min(r + i * rpw, r1 - 1);       // rows past the end repeat the last one
                    if (zero) {
                        lo[i] = zero8();
                        hi[i] = zero8();
                    } else {
                        lo[i] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(src + (int64_t)rr * src_st));
                        hi[i] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(src + (int64_t)rr * src_st + HALF));
                    }
                }
#pragma unroll
                for (int i = 0; i < RU; ++i) {
                    if (r + i * rpw >= r1) break;
                    bf16x8 ol = lo[i], oh = hi[i];
                    if (sg.delta != 0) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const float x = (float)lo[i][e], y = (float)hi[i][e];
                            ol[e] = (bf16_t)(x * cs[e].x - y * cs[e].y);
                            oh[e] = (bf16_t)(y * cs[e].x + x * cs[e].y);
                        }
                    }
                    bf16_t* d = dst + (int64_t)(r + i * rpw) * dst_st;
                    __builtin_nontemporal_store(ol, reinterpret_cast<bf16x8*>(d));
                    __builtin_nontemporal_store(oh, reinterpret_cast<bf16x8*>(d + HALF));
                }
            }
        }
    } else {
        for (int c = u0; c < units; c += 64) {
            const int h = c / CPH, e0 = (c - h * CPH) * 8;
            const bf16_t* src = sg.V + (int64_t)h * src_sh + e0;
            bf16_t* dst = Vd + (int64_t)sg.dst * dst_st + (int64_t)h * dst_sh + e0;
            for (int r = r0 + lr; r < r1; r += step) {
                bf16x8 v[RU];
#pragma unroll
                for (int i = 0; i < RU; ++i) {
                    const int rr = min(r + i * rpw, r1 - 1);
                    v[i] = zero ? zero8()
                                : __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(src + (int64_t)rr * src_st));
                }
#pragma unroll
                for (int i = 0; i < RU; ++i) {
                    if (r + i * rpw >= r1) break;
                    __builtin_nontemporal_store(v[i], reinterpret_cast<bf16x8*>(dst + (int64_t)(r + i * rpw) * dst_st));
                }
            }
        }
    }
}

}  // namespace

void cc_launch_assemble(const cc_asm_args& a, const float2* rope, const cc_model_desc& m,
                        int64_t src_st, int64_t src_sh, const cc_kv_layer& dst, hipStream_t s) {
    if (a.n_blocks <= 0) return;
    dim3 grid((a.n_blocks + 3) / 4, 2), block(256);
    if (m.d_h == 128)
        hipLaunchKernelGGL(assemble_kernel<128>, grid, block, 0, s, a, rope, m.H_kv, src_st, src_sh,
                           (bf16_t*)dst.K, (bf16_t*)dst.V, dst.stride_token, dst.stride_head);
    else
        hipLaunchKernelGGL(assemble_kernel<64>, grid, block, 0, s, a, rope, m.H_kv, src_st, src_sh,
                           (bf16_t*)dst.K, (bf16_t*)dst.V, dst.stride_token, dst.stride_head);
}
