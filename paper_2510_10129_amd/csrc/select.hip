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

// Smallest and largest key of a score kernel's 64 columns (lanes whose column does not exist pass
// ok = false), for the digits of the selection.
__device__ __forceinline__ void write_key_range(float acc, bool ok, uint2* dst) {
    uint32_t mn = ok ? score_key(acc) : 0xFFFFFFFFu, mx = ok ? score_key(acc) : 0u;
    for (int off = 32; off > 0; off >>= 1) {
        mn = min(mn, (uint32_t)__shfl_xor((int)mn, off));
        mx = max(mx, (uint32_t)__shfl_xor((int)mx, off));
    }
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
// Top-k + grouping + compaction in one workgroup of 16 waves.  One compute unit
// executes all of it, so the work per token is kept to two passes over the
// scores and everything after them runs per 64-token bitmap word.
//
// Scores become order-preserving 32-bit keys; the k-th largest key is found by a
// most-significant-digit-first radix search over 11 + 11 + 10 bits (LDS
// histogram, then the bin of the k-th key by a suffix sum over the bins).
//   scan 1  histogram of the first digit of every key.  The scores of a request
//           sit in a few binades, so neighbouring keys mostly share the digit: a
//           thread merges runs of equal digits among its own keys and adds a run
//           with one LDS atomic (same-address atomics serialise).
//   scan 2  keys above the threshold digit are candidates (one ballot per word);
//           keys of the threshold digit go, with their token index, into a list in
//           LDS.  The two remaining digits are resolved on that list, and the
//           list entries at or above the threshold set their candidate bits.
// A list that would not fit (more than SEL_LIST keys share the threshold digit)
// or a threshold value of which only some keys are taken (equal scores: the lowest
// indices win, ranked with wave ballots and a scan over per-word counts) takes the
// general path: the remaining digits and the candidates from further passes over
// the scores.
// Candidates, passing window starts and chosen tokens are bitmaps in LDS.  For
// windows up to 64 tokens a thread owns a bitmap word: it tests the windows that
// start at the word's candidates with shifts and popcounts, spreads passing
// starts over their windows by doubling shifts, and writes the indices of a
// 16-token quarter of a word from its set bits; longer windows are tested per
// token with popcounts over the words they span.
// ----------------------------------------------------------------------------
#define SEL_THREADS 1024
#define SEL_WAVES 16
#define SEL_TCAP CC_SEL_ONE_MAX
#define SEL_WORDS (SEL_TCAP / 64 + 20)   // bitmap words incl. zero padding past T + window
#define SEL_BINS 2048
#define SEL_BATCH 8                      // keys a thread loads together
#define SEL_LIST 12288                   // keys of the threshold digit that the LDS list holds

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
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t run = 0;
    for (int base = 0; base < n; base += SEL_THREADS) {
        const int i = base + tid;
        const uint32_t c = i < n ? v[i] : 0u;
        uint32_t inc = c;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t o = __shfl_up(inc, off);
            if (lane >= off) inc += o;
        }
        if (lane == 63) wave_tot[wave] = inc;
        __syncthreads();
        // lanes 0..15 of every wave hold the sixteen totals; inclusive prefix over them by shuffles
        uint32_t wt = lane < SEL_WAVES ? wave_tot[lane] : 0u;
        for (int off = 1; off < SEL_WAVES; off <<= 1) {
            const uint32_t o = __shfl_up(wt, off);
            if (lane >= off) wt += o;
        }
        const uint32_t before = run + (wave ? __shfl(wt, wave - 1) : 0u);
        const uint32_t total = __shfl(wt, SEL_WAVES - 1);
        if (i < n) v[i] = before + inc - c;
        run += total;
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

// Histogram (nb = dmask + 1 bins, zeroed here) of digit (key >> shift) & dmask over the keys
// with (key & mask) == prefix.  Thread tid takes tokens tid, tid + 1024, ...; the loads of the
// next batch are issued before the current one is processed.  Ends with a barrier.
__device__ __forceinline__ void hist_of_scores(const float* __restrict__ score, int T, uint32_t prefix,
                                               uint32_t mask, int shift, uint32_t dmask, uint32_t* hist) {
    const int tid = threadIdx.x;
    for (int i = tid; i <= (int)dmask; i += SEL_THREADS) hist[i] = 0;
    __syncthreads();
    constexpr int STEP = SEL_THREADS * SEL_BATCH;
    float cur[SEL_BATCH], nxt[SEL_BATCH];
#pragma unroll
    for (int j = 0; j < SEL_BATCH; ++j) {
        const int t = j * SEL_THREADS + tid;
        cur[j] = t < T ? score[t] : 0.0f;
        nxt[j] = 0.0f;
    }
    uint32_t run_d = 0, run_n = 0;
    for (int base = 0; base < T; base += STEP) {
        if (base + STEP < T) {
#pragma unroll
            for (int j = 0; j < SEL_BATCH; ++j) {
                const int t = base + STEP + j * SEL_THREADS + tid;
                nxt[j] = t < T ? score[t] : 0.0f;
            }
        }
#pragma unroll
        for (int j = 0; j < SEL_BATCH; ++j) {
            const int t = base + j * SEL_THREADS + tid;
            const uint32_t key = score_key(cur[j]);
            if (t < T && (key & mask) == prefix) run_add(hist, (key >> shift) & dmask, run_d, run_n);
        }
#pragma unroll
        for (int j = 0; j < SEL_BATCH; ++j) cur[j] = nxt[j];
    }
    if (run_n) atomicAdd(&hist[run_d], run_n);
    __syncthreads();
}

// The bin b of the krem-th largest entry of a histogram of nb (1024 or 2048) bins: the largest b
// with (entries in bins above b) < krem <= (those + bin b).  Returns b, krem minus the entries
// above b, and the bin's count through sh[0..2].  Thread t holds bins 2t, 2t+1 (nb = 2048) or
// bin t; suffix sums by wave shuffles, then over the waves' totals.  Ends with a barrier.
__device__ __forceinline__ void pick_bin(const uint32_t* hist, int nb, uint32_t krem, uint32_t* wave_tot,
                                         uint32_t* sh) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = nb / SEL_THREADS;
    const uint32_t h0 = hist[tid * per], h1 = per == 2 ? hist[tid * per + 1] : 0u;
    const uint32_t mine = h0 + h1;
    uint32_t inc = mine;                              // this thread's bins .. end of the wave
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_down(inc, off);
        if (lane + off < 64) inc += o;
    }
    if (lane == 0) wave_tot[wave] = inc;
    __syncthreads();
    // lanes 0..15 of every wave hold the sixteen totals; suffix sums over them by shuffles
    uint32_t wt = lane < SEL_WAVES ? wave_tot[lane] : 0u;
    for (int off = 1; off < SEL_WAVES; off <<= 1) {
        const uint32_t o = __shfl_down(wt, off);
        if (lane + off < SEL_WAVES) wt += o;
    }
    // entries in bins above this thread's: the rest of its wave, then the waves above
    uint32_t above = inc - mine + (wave + 1 < SEL_WAVES ? __shfl(wt, wave + 1) : 0u);
    if (per == 2) {                                   // the upper of the two bins first
        if (above < krem && krem <= above + h1) {
            sh[0] = (uint32_t)(tid * 2 + 1);
            sh[1] = krem - above;
            sh[2] = h1;
        }
        above += h1;
    }
    if (above < krem && krem <= above + h0) {
        sh[0] = (uint32_t)(tid * per);
        sh[1] = krem - above;
        sh[2] = h0;
    }
    __syncthreads();
}

struct SelLds {
    uint64_t cand[SEL_WORDS];
    uint64_t pass[SEL_WORDS];
    uint32_t word_prefix[SEL_TCAP / 64 + 1];
    uint32_t hist[SEL_BINS];
    uint32_t list_t[SEL_LIST];       // token index and low 21 key bits of the keys of the threshold digit
    uint32_t list_low[SEL_LIST];
    uint32_t wave_tot[SEL_WAVES];
    uint32_t sh[3];
    uint32_t sh_list_n;
};

__global__ __launch_bounds__(SEL_THREADS) void select_kernel(
    const float* __restrict__ score, int T, int k, int window, int tau, int grouping,
    int idx_offset, int n_tail, int32_t* __restrict__ idx_out, int32_t* __restrict__ n_out) {
    __shared__ SelLds L;
    uint64_t* const cand = L.cand;
    uint64_t* const pass = L.pass;
    uint64_t* const marked = cand;      // the chosen-token bitmap takes the candidates' place once the windows are judged
    uint32_t* const word_prefix = L.word_prefix;
    uint32_t* const hist = L.hist;
    uint32_t* const list_t = L.list_t;
    uint32_t* const list_low = L.list_low;
    uint32_t* const wave_tot = L.wave_tot;
    uint32_t* const sh = L.sh;
    uint32_t& sh_list_n = L.sh_list_n;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const uint64_t lane_lt = (1ULL << lane) - 1ULL;
    const int n_words = (T + 63) >> 6;

    // the bitmaps are read up to `window` bits past T: clear the words that the phases below
    // do not write
    for (int i = n_words + tid; i < n_words + 20 && i < SEL_WORDS; i += SEL_THREADS) {
        cand[i] = 0;
        pass[i] = 0;
    }
    if (tid == 0) sh_list_n = 0;

    // ---- threshold key: the k-th largest (0 < k < T) ----
    uint32_t kth = 0, krem = 0;
    bool rank_ties = false, have_cand = false;
    const bool all = k >= T, none = k <= 0;
    if (!all && !none) {
        // scan 1: first digit (bits 31..21)
        hist_of_scores(score, T, 0u, 0u, 21, 2047u, hist);
        pick_bin(hist, 2048, (uint32_t)k, wave_tot, sh);
        const uint32_t b0 = sh[0];
        krem = sh[1];
        uint32_t bin_count = sh[2];
        uint32_t prefix = b0 << 21, mask = 2047u << 21;
        if (bin_count <= SEL_LIST) {
            // scan 2: candidates above the threshold digit; the keys of that digit into the list
            constexpr int STEP = SEL_THREADS * SEL_BATCH;
            float cur[SEL_BATCH], nxt[SEL_BATCH];
#pragma unroll
            for (int j = 0; j < SEL_BATCH; ++j) {
                const int t = j * SEL_THREADS + tid;
                cur[j] = t < T ? score[t] : 0.0f;
                nxt[j] = 0.0f;
            }
            for (int base = 0; base < T; base += STEP) {
                if (base + STEP < T) {
#pragma unroll
                    for (int j = 0; j < SEL_BATCH; ++j) {
                        const int t = base + STEP + j * SEL_THREADS + tid;
                        nxt[j] = t < T ? score[t] : 0.0f;
                    }
                }
#pragma unroll
                for (int j = 0; j < SEL_BATCH; ++j) {
                    const int r0 = base + j * SEL_THREADS;       // first token of this row of the batch
                    if (r0 < T) {                                // workgroup-uniform
                        const int t = r0 + tid;
                        const uint32_t key = score_key(cur[j]);
                        const uint32_t dgt = key >> 21;
                        const bool gt = t < T && dgt > b0, eq = t < T && dgt == b0;
                        const uint64_t bg = __ballot(gt), be = __ballot(eq);
                        if (lane == 0 && (r0 >> 6) + wave < n_words) cand[(r0 >> 6) + wave] = bg;
                        if (be) {
                            uint32_t at = 0;
                            if (lane == 0) at = atomicAdd(&sh_list_n, (uint32_t)__popcll(be));
                            at = __shfl(at, 0) + (uint32_t)__popcll(be & lane_lt);
                            if (eq) {
                                list_t[at] = (uint32_t)t;
                                list_low[at] = key & 0x1FFFFFu;
                            }
                        }
                    }
                }
#pragma unroll
                for (int j = 0; j < SEL_BATCH; ++j) cur[j] = nxt[j];
            }
            __syncthreads();
            const int n_list = (int)sh_list_n;                   // == bin_count
            // second and third digit (bits 20..10, 9..0) on the list
            uint32_t lprefix = 0, lmask = 0;
#pragma unroll 1
            for (int p = 1; p < 3; ++p) {
                const int shift = p == 1 ? 10 : 0;
                const uint32_t dmask = p == 1 ? 2047u : 1023u;
                for (int i = tid; i <= (int)dmask; i += SEL_THREADS) hist[i] = 0;
                __syncthreads();
                uint32_t run_d = 0, run_n = 0;
                for (int i = tid; i < n_list; i += SEL_THREADS) {
                    const uint32_t low = list_low[i];
                    if ((low & lmask) == lprefix) run_add(hist, (low >> shift) & dmask, run_d, run_n);
                }
                if (run_n) atomicAdd(&hist[run_d], run_n);
                __syncthreads();
                pick_bin(hist, (int)dmask + 1, krem, wave_tot, sh);
                lprefix |= sh[0] << shift;
                lmask |= dmask << shift;
                krem = sh[1];
                bin_count = sh[2];
            }
            kth = prefix | lprefix;
            // bin_count keys equal the threshold and krem of them are candidates
            rank_ties = krem < bin_count;
            if (!rank_ties) {
                for (int i = tid; i < n_list; i += SEL_THREADS)
                    if (list_low[i] >= lprefix) {
                        const uint32_t t = list_t[i];
                        atomicOr(reinterpret_cast<unsigned long long*>(&cand[t >> 6]), 1ULL << (t & 63));
                    }
                have_cand = true;
            }
        } else {
            // general path: the other two digits from passes over all scores
#pragma unroll 1
            for (int p = 1; p < 3; ++p) {
                const int shift = p == 1 ? 10 : 0;
                const uint32_t dmask = p == 1 ? 2047u : 1023u;
                hist_of_scores(score, T, prefix, mask, shift, dmask, hist);
                pick_bin(hist, (int)dmask + 1, krem, wave_tot, sh);
                prefix |= sh[0] << shift;
                mask |= dmask << shift;
                krem = sh[1];
                bin_count = sh[2];
            }
            kth = prefix;
            rank_ties = krem < bin_count;
        }
    }

    // ---- candidate bitmap, general path: word (r0 >> 6) + wave is written by wave `wave` ----
    if (!have_cand) {
        if (rank_ties) {
            // threshold keys per word, exclusive scan over the words = rank of a word's first one
            for (int base = 0; base < T; base += SEL_THREADS) {
                const int t = base + tid;
                const bool eq = t < T && score_key(score[t]) == kth;
                const uint64_t be = __ballot(eq);
                if (lane == 0 && (base >> 6) + wave < n_words) word_prefix[(base >> 6) + wave] = (uint32_t)__popcll(be);
            }
            __syncthreads();
            (void)block_exclusive_scan(word_prefix, n_words, wave_tot);
        }
        for (int base = 0; base < T; base += SEL_THREADS * SEL_BATCH) {
            float sv[SEL_BATCH];
#pragma unroll
            for (int j = 0; j < SEL_BATCH; ++j) {
                const int t = base + j * SEL_THREADS + tid;
                sv[j] = t < T ? score[t] : 0.0f;
            }
#pragma unroll
            for (int j = 0; j < SEL_BATCH; ++j) {
                const int r0 = base + j * SEL_THREADS;
                if (r0 < T) {                                // workgroup-uniform
                    const int t = r0 + tid;
                    const int wi = (r0 >> 6) + wave;
                    const uint32_t key = score_key(sv[j]);
                    const bool eq = t < T && !all && !none && key == kth;
                    bool take = t < T && (all || (!none && key > kth));
                    if (rank_ties) {
                        const uint64_t be = __ballot(eq);
                        const uint32_t before = wi < n_words ? word_prefix[wi] : 0u;
                        if (eq && before + (uint32_t)__popcll(be & lane_lt) < krem) take = true;
                    } else if (eq) {
                        take = true;
                    }
                    const uint64_t bc = __ballot(take);
                    if (lane == 0 && wi < n_words) cand[wi] = bc;
                }
            }
        }
    }
    __syncthreads();

    // ---- windows that start at a candidate and hold >= tau candidates; a token is chosen when
    //      some passing window covers it ----
    if (grouping && window <= 64) {
        const uint64_t wmask = window == 64 ? ~0ULL : (1ULL << window) - 1ULL;
        // a wave takes a word, lane = token: the window's tokens are bits lane .. lane + window - 1
        // of the 128 bits (word i, word i + 1), fetched as two 32-bit funnel shifts
        const uint32_t m0 = (uint32_t)wmask, m1 = (uint32_t)(wmask >> 32);
        const uint32_t* c32 = reinterpret_cast<const uint32_t*>(cand);
        for (int i = wave; i < n_words; i += SEL_WAVES) {
            const uint32_t* wp = c32 + 2 * i + (lane >> 5);      // word n_words is zero padding
            const uint32_t w0 = wp[0], w1 = wp[1], w2 = wp[2];
            const uint32_t sh5 = lane & 31;
            const uint32_t v0 = __builtin_amdgcn_alignbit(w1, w0, sh5), v1 = __builtin_amdgcn_alignbit(w2, w1, sh5);
            const int cnt = __popc(v0 & m0) + __popc(v1 & m1);
            const uint64_t b = __ballot((v0 & 1u) && cnt >= tau);
            if (lane == 0) pass[i] = b;
        }
        __syncthreads();
        for (int i = tid; i < n_words; i += SEL_THREADS) {
            // bits (lo, hi) = tokens 64(i-1) .. 64i+63; OR of the shifts by 0 .. window-1, by doubling
            uint64_t lo = i ? pass[i - 1] : 0ULL, hi = pass[i];
            for (int covered = 1; covered < window;) {
                const int st = min(covered, window - covered);  // 1 <= st <= 32
                hi |= (hi << st) | (lo >> (64 - st));
                lo |= lo << st;
                covered += st;
            }
            if (i == n_words - 1 && (T & 63)) hi &= (1ULL << (T & 63)) - 1ULL;   // windows are cut at T
            marked[i] = hi;
        }
    } else if (grouping) {
        for (int base = 0; base < T; base += SEL_THREADS) {
            int t = base + tid;
            bool ok = false;
            if (t < T && ((cand[t >> 6] >> (t & 63)) & 1ULL))
                ok = window_popc(cand, t, t + window) >= tau;   // bits past T are zero
            uint64_t b = __ballot(ok);
            if (lane == 0 && (base >> 6) + wave < n_words) pass[(base >> 6) + wave] = b;
        }
        __syncthreads();
        for (int base = 0; base < T; base += SEL_THREADS) {
            int t = base + tid;
            bool ok = false;
            if (t < T) {
                int b0 = t - window + 1;
                ok = window_popc(pass, b0 < 0 ? 0 : b0, t + 1) > 0;
            }
            uint64_t b = __ballot(ok);
            if (lane == 0 && (base >> 6) + wave < n_words) marked[(base >> 6) + wave] = b;
        }
    }                                   // without grouping the candidates are the chosen tokens
    __syncthreads();

    // ---- exclusive scan of per-word popcounts ----
    for (int i = tid; i < n_words; i += SEL_THREADS) word_prefix[i] = (uint32_t)__popcll(marked[i]);
    __syncthreads();
    const uint32_t n_sel = block_exclusive_scan(word_prefix, n_words, wave_tot);

    // ---- compaction: a thread writes the indices of a 16-token quarter of a word ----
    for (int q = tid; q < 4 * n_words; q += SEL_THREADS) {
        const uint64_t word = marked[q >> 2];
        const int sb = 16 * (q & 3);
        uint32_t sub = (uint32_t)(word >> sb) & 0xFFFFu;
        uint32_t pos = word_prefix[q >> 2] + (uint32_t)__popcll(word & ((1ULL << sb) - 1ULL));
        const int t0 = idx_offset + 64 * (q >> 2) + sb;
        while (sub) {
            const int b = __ffs((int)sub) - 1;
            sub &= sub - 1;
            idx_out[pos++] = t0 + b;
        }
    }
    for (int j = tid; j < n_tail; j += SEL_THREADS) idx_out[n_sel + j] = idx_offset + T + j;
    if (tid == 0) *n_out = (int32_t)n_sel + n_tail;
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
// Against one workgroup (sum of the launches, k = T / 5, window 16): T = 65536: 51 -> 23 us, 131072: 94 -> 24;
// what is left are four launches' latencies and, per launch, three or four loads that wait for one another.
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
    __shared__ uint32_t hist[SEL_BINS], mn[SEL_WAVES], mx[SEL_WAVES], wave_tot[SEL_WAVES], sh[3], eq_n[SELM_WORDS];
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
    if (!all && !none) pick_bin(hist, SEL_BINS, (uint32_t)k, wave_tot, sh);
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
        pick_bin(L.hist, SEL_BINS, krem, L.wave_tot, L.sh);
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
                pick_bin(L.hist, SEL_BINS, krem, L.wave_tot, L.sh);
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
                                                           int32_t* __restrict__ n_out, cc_sel_ws ws) {
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
    if (blockIdx.x == 0 && tid == 0) *n_out = (int32_t)n_sel + n_tail;
}

void cc_launch_select(const float* score, int T, int k, int window, int tau, int grouping,
                      int idx_offset, int n_tail, int32_t* idx_out, int32_t* n_out, const uint2* key_range,
                      int n_range, cc_sel_ws ws, hipStream_t s) {
    if (!cc_select_uses_ranges(T)) {
        hipLaunchKernelGGL(select_kernel, dim3(1), dim3(SEL_THREADS), 0, s, score, T, k, window, tau,
                           grouping, idx_offset, n_tail, idx_out, n_out);
        return;
    }
    const dim3 grid((T + SELM_TILE - 1) / SELM_TILE), block(SEL_THREADS);
    hipLaunchKernelGGL(select_hist_kernel, grid, block, 0, s, score, T, key_range, n_range, ws);
    hipLaunchKernelGGL(select_cand_kernel, grid, block, 0, s, score, T, k, key_range, n_range, ws);
    hipLaunchKernelGGL(select_mark_kernel, grid, block, 0, s, score, T, window, tau, grouping, ws);
    hipLaunchKernelGGL(select_write_kernel, grid, dim3(256), 0, s, T, idx_offset, n_tail, idx_out, n_out, ws);
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
