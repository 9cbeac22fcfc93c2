// Token selection on the device: importance scores, top-k candidates with
// lowest-index tie-break, sliding-window grouping and compaction
// (Sections 4.2 and 4.3 of the paper).
#include "cc_internal.h"
#include "launch_plan.h"

// Order-preserving 32-bit key of a score: a larger score has a larger key.
__device__ __forceinline__ uint32_t score_key(float s) {
    const uint32_t u = __float_as_uint(s + 0.0f);   // -0 -> +0
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);   // negative: all bits flipped; else the sign bit set
}

// Wave-wide steps in the vector ALU (data-parallel primitives: a row shift moves a value N lanes up within 16 lanes,
// the two row broadcasts hand lane 15 of a row to the next row, lane 31 to the upper half), a few clocks each
// where a lane exchange through LDS takes over a hundred.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp(uint32_t old, uint32_t x) {       // lanes without a source get `old`
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)x, CTRL, ROWS, 0xF, false);
}
// inclusive scan over the wave; F(old, x): the identity of the operation is passed
template <class F>
__device__ __forceinline__ uint32_t wave_scan(uint32_t x, uint32_t identity, F&& f) {
    x = f(x, dpp<0x111, 0xF>(identity, x));
    x = f(x, dpp<0x112, 0xF>(identity, x));
    x = f(x, dpp<0x114, 0xF>(identity, x));
    x = f(x, dpp<0x118, 0xF>(identity, x));
    x = f(x, dpp<0x142, 0xA>(identity, x));
    x = f(x, dpp<0x143, 0xC>(identity, x));
    return x;
}
__device__ __forceinline__ uint32_t wave_scan_add(uint32_t x) {
    return wave_scan(x, 0u, [](uint32_t a, uint32_t b) __attribute__((always_inline)) { return a + b; });
}
__device__ __forceinline__ uint32_t lane_value(uint32_t x, int lane) { return (uint32_t)__builtin_amdgcn_readlane((int)x, lane); }
__device__ __forceinline__ uint32_t wave_min(uint32_t x) {
    return lane_value(wave_scan(x, 0xFFFFFFFFu, [](uint32_t a, uint32_t b) __attribute__((always_inline)) { return min(a, b); }), 63);
}
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
    return lane_value(wave_scan(x, 0u, [](uint32_t a, uint32_t b) __attribute__((always_inline)) { return max(a, b); }), 63);
}

// Smallest and largest key of a score kernel's 64 columns (lanes whose column does not exist pass
// ok = false), for the digits of the selection.
__device__ __forceinline__ void write_key_range(float acc, bool ok, uint2* dst) {
    const uint32_t mn = wave_min(ok ? score_key(acc) : 0xFFFFFFFFu), mx = wave_max(ok ? score_key(acc) : 0u);
    if ((threadIdx.x & 63) == 0) *dst = make_uint2(mn, mx);
}

// ----------------------------------------------------------------------------
// Importance score per chunk token: sum of the query->chunk attention block
// over its query rows (Section 4.2).  Every column has ONE fp32 accumulator
// and its rows are added in ascending order, so the result is the same bit
// pattern on every run and on any host that adds in that order.
//
// The adds are cheap; the kernel lives on bytes in flight.  A workgroup of four
// waves owns 64 columns.  Rows are taken 64 at a time: wave w issues the loads
// of rows 16w .. 16w+15 of the chunk together (lane = column, 256 contiguous
// bytes per row and wave) and parks them in LDS; wave 0 then walks the 64
// rows of its column in order.  32 KB of LDS per workgroup: five workgroups per
// CU.  The loads of the next chunk are in flight before this chunk is parked, and
// two LDS buffers let the waves go on while the sums of this one are taken.
// ----------------------------------------------------------------------------
#define CS_ROWS 64
#define CS_RPW (CS_ROWS / 4)   // rows per wave and chunk
__global__ __launch_bounds__(256) void colsum_kernel(const float* __restrict__ attn, int Q_a, int T,
                                                     int64_t ld, float* __restrict__ score,
                                                     uint2* __restrict__ key_range) {
    __shared__ float tile[2][CS_ROWS][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t = blockIdx.x * 64 + lane;
    const bool col_ok = t < T;
    const float* p = attn + (col_ok ? t : 0);
    float acc = 0.0f;
    const int n_chunks = (Q_a + CS_ROWS - 1) / CS_ROWS;
    // the loads of chunk c + 1 are issued before chunk c is parked: two chunks of loads in flight
    float va[CS_RPW], vb[CS_RPW];
    auto load_chunk = [&](float (&v)[CS_RPW], int c) {
        const int q0 = c * CS_ROWS + wave * CS_RPW;
#pragma unroll
        for (int u = 0; u < CS_RPW; ++u) {      // rows past the end re-read the last row and are not summed
            const int q = min(q0 + u, Q_a - 1);
            v[u] = __builtin_nontemporal_load(p + (int64_t)q * ld);
        }
    };
    auto park_and_sum = [&](const float (&v)[CS_RPW], int c) {
        float (*buf)[64] = tile[c & 1];
#pragma unroll
        for (int u = 0; u < CS_RPW; ++u) buf[wave * CS_RPW + u][lane] = v[u];
        // the buffer written now was last read two chunks ago; one barrier per chunk
        // orders both that reuse and this hand-over
        __syncthreads();
        if (wave == 0) {
            const int rows = min(CS_ROWS, Q_a - c * CS_ROWS);
            int r = 0;
            for (; r + 8 <= rows; r += 8) {
                float x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = buf[r + u][lane];
#pragma unroll
                for (int u = 0; u < 8; ++u) acc = acc + x[u];
            }
            for (; r < rows; ++r) acc = acc + buf[r][lane];
        }
    };
    load_chunk(va, 0);
    for (int c = 0; c < n_chunks; c += 2) {
        if (c + 1 < n_chunks) load_chunk(vb, c + 1);
        park_and_sum(va, c);
        if (c + 1 < n_chunks) {
            if (c + 2 < n_chunks) load_chunk(va, c + 2);
            park_and_sum(vb, c + 1);
        }
    }
    if (wave == 0 && col_ok) score[t] = acc;
    if (wave == 0 && key_range) write_key_range(acc, col_ok, key_range + blockIdx.x);
}

void cc_launch_colsum(const float* attn, int Q_a, int T, int64_t ld, float* score, uint2* key_range, hipStream_t s) {
    hipLaunchKernelGGL(colsum_kernel, dim3((T + 63) / 64), dim3(256), 0, s, attn, Q_a, T, ld, score, key_range);
}

// ----------------------------------------------------------------------------
// Importance scores straight from the auxiliary model's batched last-layer
// attention (Section 4.2): batch element c holds the attention of `chunk c +
// query`, [head][query row][key column]; the query -> chunk block starts at
// column col0 and is len columns wide.  Heads are averaged (the attention maps
// of Section 3 are head averages), then the query rows are summed:
//     a(q, j) = (sum over heads, ascending, of A[h][q][col0 + j]) * (1 / H)
//     s(t0 + j) = sum over q, ascending, of a(q, j)
// all in fp32 with one accumulator each, so the result has one bit pattern.
// Same scheme as the column sum above with more loads in flight (a request has
// only T / 64 workgroups): sixteen waves own 64 columns of one batch element,
// wave w forms a(q, .) for four of every 64 query rows (the loads of four rows
// x eight heads are issued together), parks them in LDS, and wave 0 adds the 64
// parked values of its column in order.
// ----------------------------------------------------------------------------
#define BS_WAVES 16
#define BS_RPW (CS_ROWS / BS_WAVES)
__global__ __launch_bounds__(64 * BS_WAVES) void block_scores_kernel(cc_blk_args a, int H, int Q_a, float inv_h,
                                                                     float* __restrict__ score,
                                                                     uint2* __restrict__ key_range) {
    __shared__ float tile[2][CS_ROWS][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int blk = blockIdx.x;
    int lo = 0, hi = a.n_seg - 1, sidx = 0;
    while (lo <= hi) {                      // last segment whose first workgroup is <= blk
        const int mid = (lo + hi) >> 1;
        if (a.seg[mid].blk0 <= blk) { sidx = mid; lo = mid + 1; } else { hi = mid - 1; }
    }
    const cc_blk_seg sg = a.seg[sidx];
    const int j = (blk - sg.blk0) * 64 + lane;
    const bool col_ok = j < sg.len;
    const float* p = sg.attn + sg.col0 + (col_ok ? j : 0);
    float acc = 0.0f;
    const int n_groups = (Q_a + CS_ROWS - 1) / CS_ROWS;
    for (int c = 0; c < n_groups; ++c) {
        const int q0 = c * CS_ROWS + wave * BS_RPW;
        float (*buf)[64] = tile[c & 1];
        const float* pq[BS_RPW];
        float m[BS_RPW];
#pragma unroll
        for (int u = 0; u < BS_RPW; ++u) {      // rows past the end re-read the last row and are not summed
            pq[u] = p + (int64_t)min(q0 + u, Q_a - 1) * sg.stride_row;
            m[u] = 0.0f;
        }
        for (int h0 = 0; h0 < H; h0 += 8) {
            float v[BS_RPW][8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {       // heads past the end re-read the last head and are not added
                const int64_t ho = (int64_t)min(h0 + i, H - 1) * sg.stride_head;
#pragma unroll
                for (int u = 0; u < BS_RPW; ++u) v[u][i] = __builtin_nontemporal_load(pq[u] + ho);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int u = 0; u < BS_RPW; ++u) m[u] = h0 + i < H ? m[u] + v[u][i] : m[u];
        }
#pragma unroll
        for (int u = 0; u < BS_RPW; ++u) buf[wave * BS_RPW + u][lane] = m[u] * inv_h;
        // the buffer written now was last read two groups ago; one barrier per group
        // orders both that reuse and this hand-over
        __syncthreads();
        if (wave == 0) {
            const int rows = min(CS_ROWS, Q_a - c * CS_ROWS);
            int r = 0;
            for (; r + 8 <= rows; r += 8) {
                float x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = buf[r + u][lane];
#pragma unroll
                for (int u = 0; u < 8; ++u) acc = acc + x[u];
            }
            for (; r < rows; ++r) acc = acc + buf[r][lane];
        }
    }
    if (wave == 0 && col_ok) score[sg.t0 + j] = acc;
    if (wave == 0 && key_range) write_key_range(acc, col_ok, key_range + blk);
}

void cc_launch_block_scores(const cc_blk_args& a, int H, int Q_a, float* score, uint2* key_range, hipStream_t s) {
    if (a.n_blocks <= 0) return;
    hipLaunchKernelGGL(block_scores_kernel, dim3(a.n_blocks), dim3(64 * BS_WAVES), 0, s, a, H, Q_a, 1.0f / (float)H, score,
                       key_range);
}

// ----------------------------------------------------------------------------
// Top-k + grouping + compaction in one workgroup of 16 waves.
//
// What bounds it: one compute unit, for its latencies (a barrier, a load, a chain of lane exchanges), a dozen of
// them in a row, its vector instructions (16 waves of which four share a SIMD) and the fetch of its
// instructions, which it runs once: unrolled over a thread's keys the same steps took twice as long.  So
// every score is loaded once, 16 bytes a lane and all of a thread's loads together, its order-preserving 32-bit key
// (a larger score has a larger key) stays in LDS where only its thread reads it, loops are rolled, scans and
// reductions run in the vector ALU, and a bitmap is written and judged by threads that own some bits of it.
// The k-th largest key is found by histograms of 2048 equal bins: the first over the range of the keys, so that
// the bin of the k-th key holds a few dozen of them, then over that bin, until it holds at most SEL_LIST keys,
// all of them are taken, or it is one key wide.  The keys of a bin of which some are taken are ranked against
// each other (equal keys by token, the lowest first); more than SEL_LIST equal keys by ballots and a scan
// over per-word counts.
// Candidates, passing window starts and chosen tokens are bitmaps in LDS.  For windows up to 64 tokens a thread
// judges the 16 starts of a quarter word (the first window's count, then a token in and a token out), then
// spreads a word's passing starts over their windows by doubling shifts; longer windows are tested per token with
// popcounts over the words they span.
// Against a radix search over the keys' digits with the scores read twice (event us, k = T / 5, window 16): T = 1024
// 11.0 -> 6.9, 4096 12.4 -> 7.5, 16384 19.7 -> 12.1, 20480 22.4 -> 13.8; 16384 equal scores 30 -> 20, a zero beside scores within
// an octave 27 -> 20.5.  Clocks at 16384: load 2700, key range 1500, histogram and bin 5500, candidates 4100, list 500,
// windows 2700, scan 600, indices 4500.
// ----------------------------------------------------------------------------
#define SEL_THREADS 1024
#define SEL_WAVES 16
#define SEL_TCAP CC_SEL_ONE_MAX
#define SEL_ROWS (SEL_TCAP / (4 * SEL_THREADS))   // rows of 4096 tokens, four consecutive ones a thread
#define SEL_WORDS (SEL_TCAP / 64 + 20)   // bitmap words incl. zero padding past T + window
#define SEL_BINS 2048
#define SEL_BATCH 8                      // loads of a thread that are out together, in passes over more than SEL_TCAP scores
#define SEL_LIST 64                      // keys of the threshold bin that are ranked against each other
static_assert(SEL_TCAP % (4 * SEL_THREADS) == 0 && SEL_TCAP / 64 <= SEL_THREADS && SEL_LIST <= 64,
              "whole rows of keys; a word a thread; a listed key a lane");

// popcount of bits [b0, b1) of a zero-padded bitmap
__device__ __forceinline__ int window_popc(const uint64_t* bm, int b0, int b1) {
    int w0 = b0 >> 6, w1 = (b1 - 1) >> 6;
    int cnt = 0;
    for (int wi = w0; wi <= w1; ++wi) {
        uint64_t word = bm[wi];
        if (wi == w0) word &= ~0ULL << (b0 & 63);
        if (wi == w1) {
            int e = b1 & 63;
            if (e) word &= (1ULL << e) - 1ULL;
        }
        cnt += __popcll(word);
    }
    return cnt;
}

// In-place exclusive prefix sum of v[0 .. n) by the whole workgroup; returns the total.
// wave_tot: SEL_WAVES words of LDS.  Ends with a barrier.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t* v, int n, uint32_t* wave_tot) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t run = 0;
    for (int base = 0; base < n; base += SEL_THREADS) {
        const int i = base + tid;
        const uint32_t c = i < n ? v[i] : 0u;
        const uint32_t inc = wave_scan_add(c);
        if (lane == 63) wave_tot[wave] = inc;
        __syncthreads();
        const uint32_t wt = wave_scan_add(lane < SEL_WAVES ? wave_tot[lane] : 0u);     // in every wave
        const uint32_t before = run + (wave ? lane_value(wt, wave - 1) : 0u);
        if (i < n) v[i] = before + inc - c;
        run += lane_value(wt, SEL_WAVES - 1);
        __syncthreads();
    }
    return run;
}

// Adds one digit to a thread's run of equal digits; a run that ends goes to the histogram with
// one LDS atomic (same-address atomics serialise, and the scores of a request sit in a few
// binades: measured against one atomic per key, merging runs is a fifth faster).
__device__ __forceinline__ void run_add(uint32_t* hist, uint32_t dgt, uint32_t& run_d, uint32_t& run_n) {
    if (run_n && dgt == run_d) {
        ++run_n;
    } else {
        if (run_n) atomicAdd(&hist[run_d], run_n);
        run_d = dgt;
        run_n = 1;
    }
}

// The bin b of the krem-th largest of `total` entries of a histogram of SEL_BINS bins: the entries in bins above b are
// fewer than krem, those and bin b's are not.  Returns b, krem minus the entries above b, and the bin's
// count through sh[0..2].  Thread t holds bins 2t, 2t+1; prefix sums, entry total - krem from below.  Ends with a barrier.
__device__ __forceinline__ void pick_bin(const uint32_t* hist, uint32_t total, uint32_t krem, uint32_t* wave_tot, uint32_t* sh) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint2 h = reinterpret_cast<const uint2*>(hist)[tid];
    const uint32_t inc = wave_scan_add(h.x + h.y);
    if (lane == 63) wave_tot[wave] = inc;
    __syncthreads();
    const uint32_t wt = wave_scan_add(lane < SEL_WAVES ? wave_tot[lane] : 0u);         // in every wave
    const uint32_t end = inc + (wave ? lane_value(wt, wave - 1) : 0u), mid = end - h.y, begin = mid - h.x;
    const uint32_t r = total - krem;                  // 0 <= r < total
    if (begin <= r && r < end) {
        const bool hi = r >= mid;
        sh[0] = (uint32_t)(2 * tid + (hi ? 1 : 0));
        sh[1] = (hi ? end : mid) - r;                 // krem - (total - the entries up to this bin)
        sh[2] = hi ? h.y : h.x;
    }
    __syncthreads();
}

struct SelLds {
    u32x4 key[SEL_ROWS][SEL_THREADS];
    uint64_t cand[SEL_WORDS];
    uint64_t pass[SEL_WORDS];
    uint32_t word_n[SEL_TCAP / 64];
    uint32_t hist[SEL_BINS];
    uint32_t list_t[SEL_LIST], list_key[SEL_LIST];
    uint32_t wave_tot[SEL_WAVES], mn[SEL_WAVES], mx[SEL_WAVES];
    uint32_t sh[3], list_n;
};

// n_host (may be NULL): a second place for the count, in host memory.
__global__ __launch_bounds__(SEL_THREADS) void select_kernel(
    const float* __restrict__ score, int T, int k, int window, int tau, int grouping,
    int idx_offset, int n_tail, int32_t* __restrict__ idx_out, int32_t* __restrict__ n_out, int32_t* __restrict__ n_host) {
    __shared__ SelLds L;
    uint64_t* const cand = L.cand;
    uint64_t* const pass = L.pass;
    uint64_t* const marked = cand;      // the chosen-token bitmap takes the candidates' place once the windows are judged
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_words = (T + 63) >> 6, n_rows = (T + 4 * SEL_THREADS - 1) / (4 * SEL_THREADS);
    const bool all = k >= T, none = k <= 0;

    // ---- keys: row j, thread tid: tokens 4096 j + 4 tid .. + 3 (past the end: the last token's key) ----
    uint32_t mn = 0xFFFFFFFFu, mx = 0;
    {
        f32x4 v[SEL_ROWS];
#pragma unroll
        for (int j = 0; j < SEL_ROWS; ++j) {
            const int t = 4 * (j * SEL_THREADS + tid);
            if (t + 3 < T) {
                v[j] = *reinterpret_cast<const f32x4*>(score + t);
            } else if (j < n_rows) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[j][e] = score[min(t + e, T - 1)];
            }
        }
        L.hist[tid] = 0;
        L.hist[tid + SEL_THREADS] = 0;
        // the bitmaps are read up to `window` bits past T: clear the words behind the rows
        if (tid < 20) cand[64 * n_rows + tid] = pass[64 * n_rows + tid] = 0;
        if (tid == 0) L.list_n = 0;
#pragma unroll
        for (int j = 0; j < SEL_ROWS; ++j)
            if (j < n_rows) {
                u32x4 q;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    q[e] = score_key(v[j][e]);
                    mn = min(mn, q[e]);
                    mx = max(mx, q[e]);
                }
                L.key[j][tid] = q;                  // read by this thread alone
            }
    }

    uint32_t base = 0, krem = 0, in_bin = 0;        // threshold bin: first key, keys taken of it, keys in it
    int shift = 0;                                  // its width: 2^shift keys
    if (!all && !none) {
        mn = wave_min(mn);
        mx = wave_max(mx);
        if (lane == 0) {
            L.mn[wave] = mn;
            L.mx[wave] = mx;
        }
        __syncthreads();
        mn = wave_min(L.mn[lane & (SEL_WAVES - 1)]);
        mx = wave_max(L.mx[lane & (SEL_WAVES - 1)]);
        base = mn;
        krem = (uint32_t)k;
        in_bin = (uint32_t)T;
        const int bits = mx == mn ? 0 : 32 - __clz((int)(mx - mn));
        shift = bits > 11 ? bits - 11 : 0;
        uint32_t last = mx - mn;                    // the bin's last key, from its base
#pragma unroll 1
        for (;;) {
#pragma unroll 1
            for (int j = 0; j < n_rows; ++j) {
                const u32x4 q = L.key[j][tid];
                const int n_ok = T - 4 * (j * SEL_THREADS + tid);
                uint32_t bin[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {       // a key below the bin wraps round past its width
                    const uint32_t low = q[e] - base;
                    bin[e] = e < n_ok && low <= last ? low >> shift : SEL_BINS;
                }
                // equal scores share a bin, and adds to one address go one after the other
                if (bin[0] == bin[1] && bin[0] == bin[2] && bin[0] == bin[3]) {
                    if (bin[0] < SEL_BINS) atomicAdd(&L.hist[bin[0]], 4u);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (bin[e] < SEL_BINS) atomicAdd(&L.hist[bin[e]], 1u);
                }
            }
            __syncthreads();
            pick_bin(L.hist, in_bin, krem, L.wave_tot, L.sh);
            base += L.sh[0] << shift;
            krem = L.sh[1];
            in_bin = L.sh[2];
            if (in_bin <= SEL_LIST || shift == 0 || krem == in_bin) break;
            last = (1u << shift) - 1u;
            shift = shift > 11 ? shift - 11 : 0;
            L.hist[tid] = 0;
            L.hist[tid + SEL_THREADS] = 0;
            __syncthreads();
        }
    }

    // ---- candidates: the keys above the bin, those in it that are taken.  A thread has four bits of the bitmap,
    //      two threads write a byte ----
    const bool whole = krem == in_bin;              // all of the bin
    const bool listed = !whole && in_bin <= SEL_LIST;
#pragma unroll 1
    for (int j = 0; j < n_rows; ++j) {
        const u32x4 q = L.key[j][tid];
        const int t = 4 * (j * SEL_THREADS + tid);
        uint32_t gt = 0, eq = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t above = q[e] < base ? 0u : (q[e] - base) >> shift;
            gt |= (uint32_t)(above > 0) << e;
            eq |= (uint32_t)(q[e] >= base && above == 0) << e;
        }
        const uint32_t ok = T - t >= 4 ? 15u : T - t <= 0 ? 0u : (1u << (T - t)) - 1u;
        eq &= ok;
        uint32_t bits = none ? 0u : all ? ok : (gt & ok) | (whole ? eq : 0u);
        const uint32_t other = dpp<0xB1, 0xF>(0u, bits);         // quad permutation 1 0 3 2: the neighbour's
        if (!(lane & 1)) reinterpret_cast<uint8_t*>(cand)[(j * SEL_THREADS + tid) >> 1] = (uint8_t)(bits | other << 4);
        if (listed) {
            for (; eq; eq &= eq - 1) {
                const int e = __ffs((int)eq) - 1;
                const uint32_t at = atomicAdd(&L.list_n, 1u);
                L.list_t[at] = (uint32_t)(t + e);
                L.list_key[at] = e == 0 ? q[0] : e == 1 ? q[1] : e == 2 ? q[2] : q[3];
            }
        }
    }
    __syncthreads();
    if (listed) {
        if (wave == 0) {                            // the list holds in_bin keys, one a lane
            const uint32_t my_key = L.list_key[lane], my_t = L.list_t[lane];
            uint32_t rank = 0;
            for (int i = 0; i < (int)in_bin; ++i) {
                const uint32_t key = lane_value(my_key, i), t = lane_value(my_t, i);
                rank += key > my_key || (key == my_key && t < my_t);
            }
            if (lane < (int)in_bin && rank < krem)
                atomicOr(reinterpret_cast<unsigned long long*>(&cand[my_t >> 6]), 1ULL << (my_t & 63));
        }
        __syncthreads();
    } else if (!whole) {                            // equal keys: the first krem tokens
        const uint32_t* keys = reinterpret_cast<const uint32_t*>(L.key);      // in token order
        for (int i = wave; i < n_words; i += SEL_WAVES) {
            const uint64_t be = __ballot(64 * i + lane < T && keys[64 * i + lane] == base);
            if (lane == 0) L.word_n[i] = (uint32_t)__popcll(be);
        }
        __syncthreads();
        (void)block_exclusive_scan(L.word_n, n_words, L.wave_tot);
        for (int i = wave; i < n_words; i += SEL_WAVES) {
            const uint64_t be = __ballot(64 * i + lane < T && keys[64 * i + lane] == base);
            const uint32_t before = L.word_n[i] + (uint32_t)__popcll(be & ((1ULL << lane) - 1ULL));
            const uint64_t take = __ballot((be >> lane & 1ULL) && before < krem);
            if (lane == 0) cand[i] |= take;
        }
        __syncthreads();
    }

    // ---- windows that start at a candidate and hold >= tau candidates; a token is chosen when
    //      some passing window covers it ----
    if (grouping && window <= 64) {
        // a thread judges 16 starts: the count of the first one's window, then one token in and one out
        const uint32_t* c32 = reinterpret_cast<const uint32_t*>(cand);
#pragma unroll 1
        for (int g = tid; g < 4 * n_words; g += SEL_THREADS) {
            const uint32_t a0 = c32[g >> 1], a1 = c32[(g >> 1) + 1], a2 = c32[(g >> 1) + 2];   // past the last word: zeros
            const int off = 16 * (g & 1);
            const uint64_t w = __builtin_amdgcn_alignbit(a1, a0, off) | (uint64_t)__builtin_amdgcn_alignbit(a2, a1, off) << 32;
            const uint64_t next = a2 >> off;                                                   // tokens 64 .. of w
            const uint32_t in = (uint32_t)(window == 64 ? next : w >> window | next << 1 << (63 - window));
            int cnt = __popcll(window == 64 ? w : w & ((1ULL << window) - 1ULL));
            uint32_t ok = 0;
#pragma unroll
            for (int s = 0; s < 16; ++s) {
                ok |= (uint32_t)(cnt >= tau) << s;
                cnt += (int)(in >> s & 1u) - (int)((uint32_t)w >> s & 1u);
            }
            reinterpret_cast<uint16_t*>(pass)[g] = (uint16_t)(ok & (uint32_t)w);
        }
        __syncthreads();
        if (tid < n_words) {
            // bits (lo, hi) = tokens 64(i-1) .. 64i+63; OR of the shifts by 0 .. window-1, by doubling
            uint64_t lo = tid ? pass[tid - 1] : 0ULL, hi = pass[tid];
            for (int covered = 1; covered < window;) {
                const int st = min(covered, window - covered);  // 1 <= st <= 32
                hi |= (hi << st) | (lo >> (64 - st));
                lo |= lo << st;
                covered += st;
            }
            if (tid == n_words - 1 && (T & 63)) hi &= (1ULL << (T & 63)) - 1ULL;   // windows are cut at T
            marked[tid] = hi;
        }
    } else if (grouping) {
        for (int i = wave; i < n_words; i += SEL_WAVES) {
            const int t = 64 * i + lane;                        // bits past T are zero
            const uint64_t b = __ballot((cand[i] >> lane & 1ULL) && window_popc(cand, t, t + window) >= tau);
            if (lane == 0) pass[i] = b;
        }
        __syncthreads();
        for (int i = wave; i < n_words; i += SEL_WAVES) {
            const int t = 64 * i + lane;
            const uint64_t b = __ballot(t < T && window_popc(pass, max(t - window + 1, 0), t + 1) > 0);
            if (lane == 0) marked[i] = b;
        }
        __syncthreads();
    }                                   // without grouping the candidates are the chosen tokens

    // ---- place of every word's first token: scan of the popcounts of a wave's 64 words (a thread has the word that it
    //      has just written), and the waves' totals ----
    const uint32_t c = tid < n_words ? (uint32_t)__popcll(marked[tid]) : 0u;
    const uint32_t inc = wave_scan_add(c);
    if (tid < n_words) L.word_n[tid] = inc - c;
    if (lane == 63) L.wave_tot[wave] = inc;
    __syncthreads();
    const uint32_t wt = wave_scan_add(lane < SEL_WAVES ? L.wave_tot[lane] : 0u);
    const uint32_t n_sel = lane_value(wt, SEL_WAVES - 1);

    // ---- compaction: a wave writes the indices of its words ----
#pragma unroll 1
    for (int i = wave; i < n_words; i += SEL_WAVES) {
        const uint64_t word = marked[i];
        const uint32_t at = L.word_n[i] + (i >= 64 ? lane_value(wt, (i >> 6) - 1) : 0u);
        if (word >> lane & 1ULL)
            idx_out[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(word >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)word, 0u))] =
                idx_offset + 64 * i + lane;
    }
    for (int j = tid; j < n_tail; j += SEL_THREADS) idx_out[n_sel + j] = idx_offset + T + j;
    if (tid == 0) {
        *n_out = (int32_t)n_sel + n_tail;
        if (n_host) *n_host = (int32_t)n_sel + n_tail;
    }
}

// ----------------------------------------------------------------------------
// The same selection by several workgroups, SEL_TILE tokens each, in four short launches (long
// requests: one compute unit then is what the selection waits for, and the leading digits of a
// request's scores take a few dozen values, so that its histogram atomics serialise).
//   hist    every workgroup finds the range of all keys from the score kernel's per-block ranges and
//           histograms its keys over 2048 equal bins of that range: the bin of the threshold holds a
//           few dozen keys instead of a fifth of them, and few keys of a wave share a bin.
//   cand    every workgroup adds the histograms up, finds the threshold bin, writes its keys above
//           the bin as candidate words and lists its keys in the bin (ascending tokens).
//   mark    every workgroup resolves the whole list (radix passes over the bits below the bin; of equal
//           keys the lowest tokens, by their place in the list), sets the candidates of its tile and of
//           1024 tokens around it, judges the windows and writes its chosen words and their count.
//   write   every workgroup adds up the counts before it and writes its indices.
// The list is short where the scores spread over the range: softmax sums of a request put a few dozen of
// 65536 keys in a bin.  One score far below the others (a masked column's zero) stretches the range to 2^30
// keys, a bin to a sixteenth of an octave; scores within an octave then crowd into it, and scores that
// mostly agree always do.  With more than SELM_LIST keys every mark workgroup takes the digits below the bin, and
// the equal keys before its tile, from all scores instead of the list.
// Against one workgroup of the radix search (sum of the launches, k = T / 5, window 16): T = 65536: 51 -> 23 us, 131072:
// 94 -> 24, and 21.8 at 65536 with scans in the vector ALU; what is left are four launches' latencies and, per launch, three or four loads that wait for one another.
// Crowded, one workgroup / that in the mark launch / now: T = 65536, a zero beside scores within an octave
// 82 / 96 / 48, all equal 88 / 103 / 32, five values 90 / 104 / 50;  T = 131072: 122 / 136 / 61, 167 / 183 / 39, 171 / 185 / 71.
// ----------------------------------------------------------------------------
#define SELM_TILE CC_SEL_TILE
#define SELM_LIST 8192
#define SELM_PAD 16                      // words of 64 tokens on either side of a tile that its windows see
#define SELM_WORDS (SELM_TILE / 64)
#define SELM_LOC (SELM_WORDS + 2 * SELM_PAD)

struct SelRange {
    uint32_t lo;
    int shift;                           // bin of a key: (key - lo) >> shift, < 2048
};
// Range of all keys (wave_mn, wave_mx: SEL_WAVES words of LDS each).  Ends with a barrier.
__device__ __forceinline__ SelRange key_range_of(const uint2* __restrict__ range, int n, uint32_t* wave_mn, uint32_t* wave_mx) {
    const int tid = threadIdx.x, lane = tid & 63;
    uint32_t mn = 0xFFFFFFFFu, mx = 0;
    for (int i = tid; i < n; i += SEL_THREADS) {
        const uint2 r = range[i];
        mn = min(mn, r.x);
        mx = max(mx, r.y);
    }
    for (int off = 32; off > 0; off >>= 1) {
        mn = min(mn, (uint32_t)__shfl_xor((int)mn, off));
        mx = max(mx, (uint32_t)__shfl_xor((int)mx, off));
    }
    if (lane == 0) {
        wave_mn[tid >> 6] = mn;
        wave_mx[tid >> 6] = mx;
    }
    __syncthreads();
    for (int w = 0; w < SEL_WAVES; ++w) {
        mn = min(mn, wave_mn[w]);
        mx = max(mx, wave_mx[w]);
    }
    const int bits = 32 - __clz((int)(mx - mn));
    SelRange r = {mn, bits > 11 ? bits - 11 : 0};
    return r;
}
__device__ __forceinline__ uint32_t bin_of(uint32_t key, SelRange r) { return min((key - r.lo) >> r.shift, 2047u); }

// workspace layout: cc_sel_ws in cc_internal.h
__global__ __launch_bounds__(SEL_THREADS) void select_hist_kernel(const float* __restrict__ score, int T,
                                                                  const uint2* __restrict__ range, int n_range,
                                                                  cc_sel_ws ws) {
    __shared__ uint32_t hist[SEL_BINS], mn[SEL_WAVES], mx[SEL_WAVES];
    const int tid = threadIdx.x;
    float v[SELM_TILE / SEL_THREADS];
#pragma unroll
    for (int j = 0; j < SELM_TILE / SEL_THREADS; ++j) {
        const int t = blockIdx.x * SELM_TILE + j * SEL_THREADS + tid;
        v[j] = t < T ? score[t] : 0.0f;
    }
    hist[tid] = 0;
    hist[tid + SEL_THREADS] = 0;
    const SelRange r = key_range_of(range, n_range, mn, mx);
#pragma unroll
    for (int j = 0; j < SELM_TILE / SEL_THREADS; ++j) {
        const int t = blockIdx.x * SELM_TILE + j * SEL_THREADS + tid;
        if (t < T) atomicAdd(&hist[bin_of(score_key(v[j]), r)], 1u);
    }
    __syncthreads();
    ws->hist[blockIdx.x][tid] = hist[2 * tid] | hist[2 * tid + 1] << 16;      // a count is at most SELM_TILE
}

__global__ __launch_bounds__(SEL_THREADS) void select_cand_kernel(const float* __restrict__ score, int T, int k,
                                                                  const uint2* __restrict__ range, int n_range,
                                                                  cc_sel_ws ws) {
    constexpr int KPT = SELM_TILE / SEL_THREADS;
    __shared__ __align__(16) uint32_t hist[SEL_BINS];
    __shared__ uint32_t mn[SEL_WAVES], mx[SEL_WAVES], wave_tot[SEL_WAVES], sh[3], eq_n[SELM_WORDS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, G = gridDim.x;
    const uint64_t lane_lt = (1ULL << lane) - 1ULL;
    const int n_words = (T + 63) >> 6;
    const bool all = k >= T, none = k <= 0;
    float v[KPT];
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        const int t = blockIdx.x * SELM_TILE + j * SEL_THREADS + tid;
        v[j] = t < T ? score[t] : 0.0f;
    }
    uint32_t h0 = 0, h1 = 0;
#pragma unroll 8
    for (int g = 0; g < G; ++g) {
        const uint32_t h = ws->hist[g][tid];
        h0 += h & 0xFFFFu;
        h1 += h >> 16;
    }
    hist[2 * tid] = h0;
    hist[2 * tid + 1] = h1;
    if (tid < 3) sh[tid] = 0;
    const SelRange r = key_range_of(range, n_range, mn, mx);
    if (!all && !none) pick_bin(hist, (uint32_t)T, (uint32_t)k, wave_tot, sh);
    const uint32_t b0 = sh[0];
    uint64_t be[KPT];
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        const int t = blockIdx.x * SELM_TILE + j * SEL_THREADS + tid;
        const uint32_t b = bin_of(score_key(v[j]), r);
        const uint64_t bg = __ballot(t < T && !none && (all || b > b0));
        be[j] = __ballot(t < T && !none && !all && b == b0);
        const int wl = j * SEL_WAVES + wave, wi = blockIdx.x * SELM_WORDS + wl;
        if (lane == 0) {
            if (wi < n_words) ws->cand[wi] = bg;
            eq_n[wl] = (uint32_t)__popcll(be[j]);
        }
    }
    __syncthreads();
    // place of a word's first listed key: exclusive scan over the tile's 64 words, in every wave
    static_assert(SELM_WORDS == 64, "one word a lane");
    const uint32_t c = eq_n[lane];
    uint32_t inc = c;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_up(inc, off);
        if (lane >= off) inc += o;
    }
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        const uint32_t at = __shfl(inc - c, j * SEL_WAVES + wave);
        if (be[j] >> lane & 1)
            ws->list[blockIdx.x][at + (uint32_t)__popcll(be[j] & lane_lt)] = (uint16_t)(j * SEL_THREADS + tid);
    }
    if (tid == 63) ws->list_n[blockIdx.x] = inc;
    if (blockIdx.x == 0 && tid == 0) {
        ws->base = r.lo + (b0 << r.shift);
        ws->shift = r.shift;
        ws->krem = sh[1];
        ws->bin_count = sh[2];               // 0: nothing to resolve
    }
}

struct SelMarkLds {
    uint32_t t[SELM_LIST], low[SELM_LIST], eq[SELM_LIST];
    uint32_t hist[SEL_BINS], pre[CC_SEL_TILES + 1], wave_tot[SEL_WAVES], sh[3];
    uint64_t cand[SELM_LOC + 20], pass[SELM_LOC + 20];
};

// f(token, key) for every score, thread tid taking tokens 4 tid .., 4 (tid + 1024) .. (score 16-byte aligned): eight
// 16-byte loads a thread are out together.
template <class F>
__device__ __forceinline__ void for_all_scores(const float* __restrict__ score, int T, F&& f) {
    const int n4 = T >> 2;
    for (int base = 0; base < n4; base += SEL_THREADS * SEL_BATCH) {
        f32x4 v[SEL_BATCH];
#pragma unroll
        for (int j = 0; j < SEL_BATCH; ++j) {
            const int i = base + j * SEL_THREADS + (int)threadIdx.x;
            if (i < n4) v[j] = reinterpret_cast<const f32x4*>(score)[i];
        }
#pragma unroll
        for (int j = 0; j < SEL_BATCH; ++j) {
            const int i = base + j * SEL_THREADS + (int)threadIdx.x;
            if (i < n4) {
#pragma unroll
                for (int e = 0; e < 4; ++e) f(4 * i + e, score_key(v[j][e]));
            }
        }
    }
    if ((int)threadIdx.x < (T & 3)) f(4 * n4 + (int)threadIdx.x, score_key(score[4 * n4 + threadIdx.x]));
}

// Candidates of the local words among the keys of a threshold bin [base, base + 2^shift) that holds
// `in_bin` keys of which the krem largest are taken, from all scores: radix passes over the bits below
// the bin, then of equal keys the lowest tokens, ranked by a count of those before the local words.
// Ends with a barrier.
__device__ __forceinline__ void mark_crowded(SelMarkLds& L, const float* __restrict__ score, int T, int wb,
                                             uint32_t base, int shift, uint32_t krem, uint32_t in_bin) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t width = 1u << shift;                          // shift <= 21
    uint32_t ties = in_bin, kth = 0, mask = 0;
    for (int hi = shift; hi > 0;) {
        const int lo = hi > 11 ? hi - 11 : 0;
        const uint32_t dmask = (1u << (hi - lo)) - 1u;
        for (int i = tid; i < SEL_BINS; i += SEL_THREADS) L.hist[i] = 0;
        __syncthreads();
        uint32_t run_d = 0, run_n = 0;
        for_all_scores(score, T, [&](int, uint32_t key) __attribute__((always_inline)) {
            const uint32_t low = key - base;                     // a key below the bin wraps round past its width
            if (low < width && (low & mask) == kth) run_add(L.hist, (low >> lo) & dmask, run_d, run_n);
        });
        if (run_n) atomicAdd(&L.hist[run_d], run_n);
        __syncthreads();
        pick_bin(L.hist, ties, krem, L.wave_tot, L.sh);
        kth |= L.sh[0] << lo;
        mask |= dmask << lo;
        krem = L.sh[1];
        ties = L.sh[2];
        hi = lo;
    }
    const uint32_t thr = base + kth;                             // the threshold key: krem of its `ties` tokens are taken
    const bool rank = krem < ties;
    uint32_t before = 0;                                         // its tokens before the local words
    if (rank && wb > 0) {
        uint32_t n = 0;
        for_all_scores(score, 64 * wb, [&](int, uint32_t key) __attribute__((always_inline)) { n += key == thr; });
        for (int off = 32; off > 0; off >>= 1) n += (uint32_t)__shfl_xor((int)n, off);
        if (lane == 0) L.wave_tot[wave] = n;
        __syncthreads();
        for (int w = 0; w < SEL_WAVES; ++w) before += L.wave_tot[w];
        __syncthreads();
    }
    constexpr int WPW = SELM_LOC / SEL_WAVES;                    // local words of a wave
    static_assert(SELM_LOC % SEL_WAVES == 0, "whole waves of local words");
    uint64_t gt[WPW], eq[WPW];
#pragma unroll
    for (int j = 0; j < WPW; ++j) {
        const int i = j * SEL_WAVES + wave, t = 64 * (wb + i) + lane;
        const bool ok = t >= 0 && t < T;
        const uint32_t key = ok ? score_key(score[t]) : 0u;
        gt[j] = __ballot(ok && key - base < width && key > thr);
        eq[j] = __ballot(ok && key == thr);
        if (lane == 0) L.eq[i] = (uint32_t)__popcll(eq[j]);
    }
    __syncthreads();
    if (rank) (void)block_exclusive_scan(L.eq, SELM_LOC, L.wave_tot);
#pragma unroll
    for (int j = 0; j < WPW; ++j) {
        const int i = j * SEL_WAVES + wave;
        const uint32_t at = before + L.eq[i] + (uint32_t)__popcll(eq[j] & ((1ULL << lane) - 1ULL));
        const uint64_t take = __ballot((eq[j] >> lane & 1ULL) && (!rank || at < krem));
        if (lane == 0) L.cand[i] |= gt[j] | take;
    }
    __syncthreads();
}

__global__ __launch_bounds__(SEL_THREADS) void select_mark_kernel(
    const float* __restrict__ score, int T, int window, int tau, int grouping, cc_sel_ws ws) {
    __shared__ SelMarkLds L;
    const uint32_t in_bin = ws->bin_count;
    const bool crowded = in_bin > SELM_LIST;                     // the same for every workgroup
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, G = gridDim.x;
    const int n_words = (T + 63) >> 6;
    const int wb = (int)blockIdx.x * SELM_WORDS - SELM_PAD;      // word of the bitmaps' first local word
    for (int i = tid; i < SELM_LOC + 20; i += SEL_THREADS) {
        const int wi = wb + i;
        L.cand[i] = i < SELM_LOC && wi >= 0 && wi < n_words ? ws->cand[wi] : 0ULL;
        L.pass[i] = 0ULL;
    }
    if (!crowded) {
        // ---- the list: place of every tile's first key, then the keys ----
        if (wave == 0) {
            const uint32_t c = lane < G ? ws->list_n[lane] : 0u;
            uint32_t inc = c;
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t o = __shfl_up(inc, off);
                if (lane >= off) inc += o;
            }
            if (lane <= CC_SEL_TILES) L.pre[lane] = inc - c;
        }
        __syncthreads();
        const int n_list = min((int)L.pre[G], SELM_LIST);            // G <= CC_SEL_TILES: lane G holds the total
        const uint32_t base = ws->base;
        for (int i = tid; i < n_list; i += SEL_THREADS) {
            int g = 0;
            for (int step = CC_SEL_TILES / 2; step > 0; step >>= 1)
                if (g + step < G && (int)L.pre[g + step] <= i) g += step;
            const uint32_t t = (uint32_t)g * SELM_TILE + ws->list[g][i - (int)L.pre[g]];
            L.t[i] = t;
            L.low[i] = score_key(score[t]) - base;
        }
        __syncthreads();
        if (n_list > 0) {
            // the bits below the bin, at most 21: 11 (or all of them), then the rest
            uint32_t krem = ws->krem, ties = in_bin, kth = 0, mask = 0;
            for (int hi = ws->shift; hi > 0;) {
                const int lo = hi > 11 ? hi - 11 : 0;
                const uint32_t dmask = (1u << (hi - lo)) - 1u;
                for (int i = tid; i < SEL_BINS; i += SEL_THREADS) L.hist[i] = 0;
                __syncthreads();
                for (int i = tid; i < n_list; i += SEL_THREADS)
                    if ((L.low[i] & mask) == kth) atomicAdd(&L.hist[(L.low[i] >> lo) & dmask], 1u);
                __syncthreads();
                pick_bin(L.hist, ties, krem, L.wave_tot, L.sh);
                kth |= L.sh[0] << lo;
                mask |= dmask << lo;
                krem = L.sh[1];
                ties = L.sh[2];
                hi = lo;
            }
            const bool rank = krem < ties;       // of `ties` equal keys the first krem of the list
            if (rank) {
                for (int i = tid; i < n_list; i += SEL_THREADS) L.eq[i] = L.low[i] == kth;
                __syncthreads();
                (void)block_exclusive_scan(L.eq, n_list, L.wave_tot);
            }
            for (int i = tid; i < n_list; i += SEL_THREADS) {
                const int wi = (int)(L.t[i] >> 6) - wb;
                if (wi >= 0 && wi < SELM_LOC && (L.low[i] > kth || (L.low[i] == kth && (!rank || L.eq[i] < krem))))
                    atomicOr(reinterpret_cast<unsigned long long*>(&L.cand[wi]), 1ULL << (L.t[i] & 63));
            }
            __syncthreads();
        }
    } else {
        mark_crowded(L, score, T, wb, ws->base, ws->shift, ws->krem, in_bin);
    }
    // ---- windows, as in the one-workgroup selection, on local words ----
    uint64_t* const marked = L.cand;
    constexpr int W1 = SELM_PAD + SELM_WORDS;                    // starts are judged in words [0, W1)
    if (grouping && window <= 64) {
        const uint64_t wmask = window == 64 ? ~0ULL : (1ULL << window) - 1ULL;
        const uint32_t m0 = (uint32_t)wmask, m1 = (uint32_t)(wmask >> 32);
        const uint32_t* c32 = reinterpret_cast<const uint32_t*>(L.cand);
        for (int i = wave; i < W1; i += SEL_WAVES) {
            const uint32_t* wp = c32 + 2 * i + (lane >> 5);
            const uint32_t w0 = wp[0], w1 = wp[1], w2 = wp[2];
            const uint32_t sh5 = lane & 31;
            const uint32_t v0 = __builtin_amdgcn_alignbit(w1, w0, sh5), v1 = __builtin_amdgcn_alignbit(w2, w1, sh5);
            const uint64_t b = __ballot((v0 & 1u) && __popc(v0 & m0) + __popc(v1 & m1) >= tau);
            if (lane == 0) L.pass[i] = b;
        }
        __syncthreads();
        if (tid < SELM_WORDS) {
            const int i = SELM_PAD + tid;
            uint64_t lo = L.pass[i - 1], hi = L.pass[i];
            for (int covered = 1; covered < window;) {
                const int st = min(covered, window - covered);
                hi |= (hi << st) | (lo >> (64 - st));
                lo |= lo << st;
                covered += st;
            }
            marked[i] = hi;
        }
    } else if (grouping) {
        for (int i = wave; i < W1; i += SEL_WAVES) {
            const int t = 64 * i + lane;
            const uint64_t b = __ballot((L.cand[i] >> lane & 1ULL) && window_popc(L.cand, t, t + window) >= tau);
            if (lane == 0) L.pass[i] = b;
        }
        __syncthreads();
        for (int i = SELM_PAD + wave; i < W1; i += SEL_WAVES) {
            const int t = 64 * i + lane;                         // window <= 1024 = 64 * SELM_PAD: t - window + 1 > 0
            const uint64_t b = __ballot(window_popc(L.pass, t - window + 1, t + 1) > 0);
            if (lane == 0) marked[i] = b;
        }
    }
    __syncthreads();
    if (wave == 0) {
        const int wi = wb + SELM_PAD + lane;
        uint64_t m = wi < n_words ? marked[SELM_PAD + lane] : 0ULL;
        if (wi == n_words - 1 && (T & 63)) m &= (1ULL << (T & 63)) - 1ULL;       // windows are cut at T
        if (wi < n_words) ws->marked[wi] = m;
        uint32_t n = (uint32_t)__popcll(m);
        for (int off = 32; off > 0; off >>= 1) n += (uint32_t)__shfl_xor((int)n, off);
        if (lane == 0) ws->marked_n[blockIdx.x] = n;
    }
}

__global__ __launch_bounds__(256) void select_write_kernel(int T, int idx_offset, int n_tail, int32_t* __restrict__ idx_out,
                                                           int32_t* __restrict__ n_out, int32_t* __restrict__ n_host,
                                                           cc_sel_ws ws) {
    __shared__ uint64_t words[SELM_WORDS];
    __shared__ uint32_t first[SELM_WORDS];
    const int tid = threadIdx.x, lane = tid & 63, G = gridDim.x;
    const int n_words = (T + 63) >> 6;
    uint32_t c = lane < G ? ws->marked_n[lane] : 0u;
    uint32_t before = lane < (int)blockIdx.x ? c : 0u;
    for (int off = 32; off > 0; off >>= 1) {
        c += (uint32_t)__shfl_xor((int)c, off);
        before += (uint32_t)__shfl_xor((int)before, off);
    }
    const uint32_t n_sel = c;
    if (tid < SELM_WORDS) {
        const int wi = (int)blockIdx.x * SELM_WORDS + lane;
        const uint64_t w = wi < n_words ? ws->marked[wi] : 0ULL;
        const uint32_t p = (uint32_t)__popcll(w);
        uint32_t inc = p;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t o = __shfl_up(inc, off);
            if (lane >= off) inc += o;
        }
        words[lane] = w;
        first[lane] = before + inc - p;
    }
    __syncthreads();
    // a thread writes the indices of a 16-token quarter of a word
    const uint64_t word = words[tid >> 2];
    const int sb = 16 * (tid & 3);
    uint32_t sub = (uint32_t)(word >> sb) & 0xFFFFu;
    uint32_t pos = first[tid >> 2] + (uint32_t)__popcll(word & ((1ULL << sb) - 1ULL));
    const int t0 = idx_offset + (int)blockIdx.x * SELM_TILE + 64 * (tid >> 2) + sb;
    while (sub) {
        const int b = __ffs((int)sub) - 1;
        sub &= sub - 1;
        idx_out[pos++] = t0 + b;
    }
    for (int j = blockIdx.x * 256 + tid; j < n_tail; j += G * 256) idx_out[n_sel + j] = idx_offset + T + j;
    if (blockIdx.x == 0 && tid == 0) {
        *n_out = (int32_t)n_sel + n_tail;
        if (n_host) *n_host = (int32_t)n_sel + n_tail;
    }
}

void cc_launch_select(const float* score, int T, int k, int window, int tau, int grouping,
                      int idx_offset, int n_tail, int32_t* idx_out, int32_t* n_out, int32_t* n_host, const uint2* key_range,
                      int n_range, cc_sel_ws ws, hipStream_t s) {
    if (!cc_select_uses_ranges(T)) {
        hipLaunchKernelGGL(select_kernel, dim3(1), dim3(SEL_THREADS), 0, s, score, T, k, window, tau,
                           grouping, idx_offset, n_tail, idx_out, n_out, n_host);
        return;
    }
    const dim3 grid((T + SELM_TILE - 1) / SELM_TILE), block(SEL_THREADS);
    hipLaunchKernelGGL(select_hist_kernel, grid, block, 0, s, score, T, key_range, n_range, ws);
    hipLaunchKernelGGL(select_cand_kernel, grid, block, 0, s, score, T, k, key_range, n_range, ws);
    hipLaunchKernelGGL(select_mark_kernel, grid, block, 0, s, score, T, window, tau, grouping, ws);
    hipLaunchKernelGGL(select_write_kernel, grid, dim3(256), 0, s, T, idx_offset, n_tail, idx_out, n_out, n_host, ws);
}

// ----------------------------------------------------------------------------
// idx check: strictly ascending (or merely in range when strict == 0), each in
// [lo, hi).  flag receives the number of violations.
// ----------------------------------------------------------------------------
__global__ void check_idx_kernel(const int32_t* __restrict__ idx, int M, int lo, int hi, int strict,
                                 int32_t* __restrict__ flag) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= M) return;
    int v = idx[i];
    bool bad = v < lo || v >= hi;
    if (strict && i > 0 && idx[i - 1] >= v) bad = true;
    if (bad) atomicAdd(flag, 1);
}

void cc_launch_check_idx(const int32_t* idx, int M, int lo, int hi, int strict, int32_t* flag,
                         hipStream_t s) {
    if (M <= 0) return;
    hipLaunchKernelGGL(check_idx_kernel, dim3((M + 255) / 256), dim3(256), 0, s, idx, M, lo, hi,
                       strict, flag);
}
