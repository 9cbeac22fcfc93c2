// Sparse-query causal GQA attention over the updated KV cache: recomputed row i
// (global position idx[i]) attends to every cache slot j <= idx[i].  This is
// the kernel Section 5.6 of the paper describes as flash attention with sparse
// query indices; the design below is for gfx950.
//
// Work split: the (recomputed token, query head of the group) pairs of one kv
// head form one flat column sequence c = i*g + h (g = H_q/H_kv); a workgroup of
// eight waves owns 256 consecutive columns, a wave 32 of them on the N side of
// the MFMA tile, so a K/V tile read from LDS serves the whole query group and
// no column is padding when g does not divide 32.
//
// Each wave computes S^T = K Q^T (keys on the MFMA row side, query rows on the
// column side).  In the 32x32 accumulator layout a lane then owns ONE query row
// and 16 keys per tile, so the online-softmax maximum and sum are in-lane
// reductions plus one exchange with lane^32, the rescale factor is a per-lane
// scalar, and the probabilities are already laid out as the B operand of
// O^T = V^T P^T: no shuffle between the two contractions.
//
// Two wave groups alternate between the matrix pipe and the vector ALU.  Per
// 64-key tile a wave issues 32 MFMAs and about as many cycles of exponentials,
// sums and conversions, one after the other; two independent waves on a SIMD
// drift into the same phase (both contend for the matrix pipe, then both for
// the vector ALU) and each pipe idles half of the time.  Here the two waves of a
// SIMD belong to the same workgroup, one to group A and one to group B, and
// the workgroup barrier separates phases: while A runs the softmax of tile t, B
// runs P V of tile t-1 and Q K^T of tile t, and the other way round in the next
// phase.  A wave issues its global -> LDS loads in its softmax phase, one after every
// second group of four exponentials (group A the V tiles, group B the K tiles): the four of
// them back to back at the end of the matrix phase queue up behind each other and lengthen
// the phase that the matrix pipe is busy in.  The form of the load decides: scalar base plus
// 32-bit lane offset and one LDS base for the four.  With 64-bit vector addresses and the LDS
// base rewritten between them the same placement ran 18 % slower.  At 64k context, 64 query
// heads and M = 13363: 12.05 -> 11.72 ms; M = 16576 at 16k: 2.05 -> 1.99 ms.
//
// K and V tiles (64 keys) go from the cache straight into LDS with 16-byte
// global->LDS loads, row-major as they are stored, three stages of K, four of V.  K
// fragments are plain 16-byte LDS reads; the V^T fragments (contraction index =
// key) come from the row-major V tile through the transposing LDS read
// ds_read_b64_tr_b16, so V is never transposed in registers.  Both tiles are
// XOR-swizzled (by choosing which global chunk a lane fetches) so that the
// fragment reads spread over the 64 LDS banks.
//
// Causality with sorted idx: the key loop of a workgroup ends at the position
// of its last row; the per-row mask only bites between the positions of the
// first and last row of the tile.  Workgroups are issued longest-first and
// workgroup id modulo H_kv picks the kv head, so the workgroups resident on
// one XCD walk the same K/V stream through that XCD's L2.
#include "cc_internal.h"
#include "launch_plan.h"
#include <algorithm>
#include <type_traits>

namespace {

constexpr int BN_KEYS = 64;

// 16 bytes per lane from global memory straight into LDS.  The LDS address is
// wave base (M0) + OFF + 16 * lane and OFF is also added to the global address.
// Rewriting M0 between loads is expensive while MFMAs are in flight (measured:
// several hundred cycles per rewrite with two MFMA-bound waves on a SIMD), so
// the loads of one tile and tensor share one base and differ in OFF only.
template <int OFF>
__device__ __forceinline__ void dma16(const bf16_t* gsrc_minus_off, bf16_t* lds_wave_base) {
    static_assert(OFF >= 0 && OFF < 4096, "the instruction offset is 13 bits signed; a larger value wraps silently");
    __builtin_amdgcn_global_load_lds(
        (const void __attribute__((address_space(1)))*)gsrc_minus_off,
        (void __attribute__((address_space(3)))*)lds_wave_base, 16, OFF, 0);
}
// LDS reads whose place in the instruction stream is fixed by the source order (the
// compiler's scheduler, short of registers, would issue every read right before its use).
// The waits for them are written by hand: LDS operations of a wave return in order, so
// "at most N outstanding" after N younger reads means this one has arrived.
// Transposing LDS read: within each group of 16 lanes, lane i receives, as element e, element (i % 4) of
// the 8-byte row addressed by lane (i / 4 + 4 e).
template <int IMM>
__device__ __forceinline__ bf16x4 lds_read_tr_at(uint32_t addr) {
    bf16x4 v;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(IMM));
    return v;
}
template <int IMM>
__device__ __forceinline__ bf16x8 lds_read_b128_at(uint32_t addr) {
    bf16x8 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(IMM));
    return v;
}
template <int N>
__device__ __forceinline__ void lds_wait_all_but(bf16x8& x) {
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(x) : "n"(N));
}

template <int NI, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < NI) {
        f(std::integral_constant<int, I>{});
        static_for<NI, I + 1>(f);
    }
}

constexpr int LDS_TILES = 7;              // K tile t lives in stage t % 3, V tile t in stage 3 + t % 4

// Group (0: A, 1: B) and slot of this wave.  The two waves that share a SIMD must land in different
// groups: the SIMD id comes from the hardware id register (HW_ID bits 5:4), the first
// wave to register on a SIMD joins group A (0), the second group B (1).  Should the
// eight waves not sit two per SIMD, the split falls back to wave index order (correct,
// but the phases of a SIMD's waves then no longer alternate).
__device__ __forceinline__ void wave_role(int* simd_waves, int* group_waves, int& grp, int& widx) {
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid < 4) simd_waves[tid] = 0;
    if (tid < 2) group_waves[tid] = 0;
    __syncthreads();
    int a = 0, b = 0;
    if (lane == 0) {
        const int simd = __builtin_amdgcn_s_getreg(((2 - 1) << 11) | (4 << 6) | 4);
        a = atomicAdd(&simd_waves[simd & 3], 1) & 1;
        b = atomicAdd(&group_waves[a], 1);
    }
    grp = __builtin_amdgcn_readfirstlane(a);
    widx = __builtin_amdgcn_readfirstlane(b);
    __syncthreads();
    if (group_waves[0] != 4) {
        const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
        grp = w >> 2;
        widx = w & 3;
    }
}

// last position that the 256 columns of row tile rt see (rows are sorted)
__device__ __forceinline__ int last_key(const int32_t* idx, int M, int g, int rt) {
    return idx[min(M - 1, (rt * 256 + 255) / g)];
}

// Key tiles ta .. ta + n_tiles - 1 (n_tiles >= 1) of the 256 columns of row tile rt and kv head kvh.
// PIECE and slot >= 0: the sums stay unnormalised and go to part's slot.  Off: type
// of the lane offsets of the global -> LDS loads.  Can be called again by the same
// workgroup: every wave's reads of LDS lie before its last barrier, and a wave only loads
// into rows that it has loaded (and waited for) itself.
template <int D_H, bool PIECE, class Off>
__device__ __forceinline__ void attend(
    const bf16_t* __restrict__ q, int M, const int32_t* __restrict__ idx, int H_q, int g,
    const bf16_t* __restrict__ Kc, const bf16_t* __restrict__ Vc, int64_t st, int64_t sh, int N,
    bf16_t* __restrict__ o, float scale_log2, float* __restrict__ part, bf16_t* smem, int grp, int widx,
    int kvh, int rt, int ta, int n_tiles, int slot) {
    constexpr int KS = D_H / 16;          // k-steps of the QK^T contraction
    constexpr int DT = D_H / 32;          // 32-row tiles of O^T
    constexpr int CPRW = D_H / 8;         // 16-byte chunks per cache row
    constexpr int RPI = 64 / CPRW;        // rows moved by one global->LDS instruction
    constexpr int NI = BN_KEYS / RPI / 4; // such instructions per wave, tile and tensor

    constexpr int TILE = BN_KEYS * D_H;   // elements of one K or V tile
    auto k_stage = [&](int t) __attribute__((always_inline)) { return smem + (t % 3) * TILE; };
    auto v_stage = [&](int t) __attribute__((always_inline)) { return smem + (3 + t % 4) * TILE; };

    const int lane = threadIdx.x & 63;
    const int wave = widx;                              // role in the cooperative tile loads
    const int qr = lane & 31, hf = lane >> 5;
    const int col_in = (grp * 4 + widx) * 32 + qr;      // column within the row tile
    const int col = rt * 256 + col_in;                  // flat (token, head) column
    const int mi = col / g, hg = col - mi * g;
    const bool valid = mi < M;
    const int limit = valid ? idx[mi] : -1;
    const int j_a = ta * BN_KEYS;                       // first key of this piece

    // wave-wide largest limit (tiles beyond it are skipped by this wave) and smallest
    // limit of a valid row (tiles that end at or below it need no mask)
    int wave_limit = limit;
    for (int off = 32; off > 0; off >>= 1) wave_limit = max(wave_limit, __shfl_xor(wave_limit, off));
    int wave_min = valid ? limit : 0x7fffffff;
    for (int off = 32; off > 0; off >>= 1) wave_min = min(wave_min, __shfl_xor(wave_min, off));

    // ---- Q fragments (B operand of S^T = K Q^T): lane = query row, 8 d's per k-step ----
    bf16x8 qf[KS];
    {
        const bf16_t* qp = q + ((int64_t)(valid ? mi : 0) * H_q + kvh * g + hg) * D_H + 8 * hf;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (valid) {
                qf[ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 16);
            } else {
#pragma unroll
                for (int u = 0; u < 8; ++u) qf[ks][u] = (bf16_t)0.0f;
            }
        }
    }

    // ---- global -> LDS: instruction i of this wave moves the RPI logical rows
    //      (i*4 + wave)*RPI ..; lane L fills physical chunk L % CPRW of row L / CPRW and
    //      fetches the logical chunk that the swizzle maps there.  In LDS the rows of one
    //      wave's NI instructions are adjacent (physical row rho(r) below), so they are
    //      reached from one base with immediate offsets of 1 KB ----
    //   K rows: chunk c sits at slot c ^ kswz(row)           (16-byte fragment reads)
    //   V rows: the 64-byte group dt sits at group dt ^ vswz(row)  (transposing 8-byte reads)
    // The swizzles use row bits that the instruction index does not touch, so one lane
    // offset per tensor serves every instruction.
    auto kswz = [](int r) { return D_H == 128 ? (r & 15) : ((r >> 1) & 7); };
    auto vswz = [](int r) { return D_H == 128 ? (r & 3) : ((r >> 1) & 1); };
    constexpr auto rho = [](int r) constexpr { return (((r / RPI) % 4) * NI + r / (4 * RPI)) * RPI + r % RPI; };
    static_assert((4 * RPI) % 16 == 0 && NI * 1024 <= 4096, "row bits of the swizzle / immediate offset range");
    const bf16_t* kbase = Kc + (int64_t)kvh * sh;
    const bf16_t* vbase = Vc + (int64_t)kvh * sh;
    const int l_row = lane / CPRW, l_p = lane % CPRW;
    const int r0 = wave * RPI + l_row;                 // logical row of instruction 0
    const int k_col = (l_p ^ kswz(r0)) * 8;
    const int v_col = ((((l_p >> 2) ^ vswz(r0)) << 2) | (l_p & 3)) * 8;
    const int wave_slot = wave * NI * RPI * D_H;
    // Group A loads V tiles, group B K tiles: a wave-uniform base per tile (scalar registers) plus
    // 32-bit lane offsets that are the same for every tile; from the tile on that reaches past the
    // cache (only a workgroup's last one can) rows past N-1 are clamped (they are masked anyway).
    const char* const lbase = reinterpret_cast<const char*>(grp == 0 ? vbase : kbase);
    const int l_col = grp == 0 ? v_col : k_col;
    Off loff[NI];
    auto set_loff = [&](int rmax) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NI; ++i) loff[i] = ((Off)min(r0 + i * 4 * RPI, rmax) * (Off)st + (Off)l_col) * 2;
    };
    set_loff(BN_KEYS);
    auto tile_at = [&](int t) __attribute__((always_inline)) -> const char* {
        const int j0 = j_a + t * BN_KEYS;
        if (j0 + BN_KEYS > N) set_loff(N - 1 - j0);
        return lbase + (int64_t)j0 * st * 2;
    };
    auto scalar_ptr = [](const char* p) -> const char* {   // keeps the base in scalar registers
        const uint64_t u = reinterpret_cast<uint64_t>(p);
        const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
        const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
        return reinterpret_cast<const char*>((hi << 32) | lo);
    };
    auto load_part = [&](const char* tile, bf16_t* stage, auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value;
        const char* b = scalar_ptr(tile - i * 1024);           // the immediate adds it back
        asm volatile("" : "+v"(loff[i]));   // keeps the (32-bit) offset a register operand of the load
        dma16<i * 1024>(reinterpret_cast<const bf16_t*>(b + loff[i]), stage + wave_slot);
    };
    auto load_tile = [&](const char* tile, bf16_t* stage) __attribute__((always_inline)) {
        static_for<NI>([&](auto i) __attribute__((always_inline)) { load_part(tile, stage, i); });
    };

    // ---- fragment addresses: LDS byte addresses in the stage this wave reads next (they
    //      move on after every matrix phase); key block and half are immediate offsets ----
    const uint32_t smem_base = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)smem;
    // K: logical row kt*32 + qr (physical rho(qr) + 8 kt), logical chunk 2 ks + hf
    const int k_sw = kswz(qr);
    uint32_t kaddr[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        kaddr[ks] = smem_base + 2 * (rho(qr) * D_H + (((ks * 2 + hf) ^ k_sw) << 3));
    // V^T through the transposing read: lane s of a 16-lane group addresses key
    // (4 hf + s/4) and the 4 d's starting at 16*(group%2) + 4*(s%4); the lane then
    // holds 4 consecutive keys of column d = 32 dt + lane%32.  Key 16 ss + 8 e + v_key sits
    // in physical row rho(16 ss + 8 e) + rho(v_key) (the two parts use different row bits).
    const int s16 = lane & 15, dsub = (lane >> 4) & 1;
    const int v_key = 4 * hf + (s16 >> 2);
    const int v_sw = vswz(v_key);
    const int v_lane = (2 * dsub + ((s16 & 3) >> 1)) * 8 + (s16 & 1) * 4;
    uint32_t vaddr[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
        vaddr[dt] = smem_base + 2 * (3 * TILE + rho(v_key) * D_H + v_lane + ((dt ^ v_sw) << 5));

    f32x16 acc_o[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc_o[dt][v] = 0.0f;
    float m_run = -INFINITY, l_run = 0.0f;
    f32x16 s[2];       // S^T tile: 64 keys x 32 query rows
    bf16x8 pf[4];      // its probabilities as B operand of the second contraction

    // `load`: the four loads of this wave's next tile go between the exponentials, evenly apart
    auto softmax = [&](int j0, auto load) __attribute__((always_inline)) {
        // ---- causal mask (only in tiles that reach past the wave's first row),
        //      online softmax in base 2 with the 1/sqrt(d_h) scale folded into the exponent ----
        if (j0 + BN_KEYS - 1 > wave_min) {
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    int key = j0 + kt * 32 + 8 * (v >> 2) + 4 * hf + (v & 3);
                    if (key > limit) s[kt][v] = -INFINITY;
                }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int v = 0; v < 16; ++v) mx = fmaxf(mx, s[kt][v]);
        {   // the other half-wave's maximum of the same query row: lanes i and i + 32 exchange by a
            // register swap (no LDS round trip)
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
            mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * scale_log2;
        }
        // The reference point m_run of the exponent is only moved when a row's maximum
        // grew by more than 2^8: until then probabilities up to 256 are accumulated
        // (harmless in fp32 / bf16, and the final division by the row sum cancels it),
        // which keeps the 64-element rescale of O out of most tiles.
        const bool grow = mx > m_run + 8.0f;
        if (__any(grow)) {
            const float m_new = grow ? mx : m_run;
            const float alpha = __builtin_amdgcn_exp2f(m_run - (m_new == -INFINITY ? 0.0f : m_new));
            l_run *= alpha;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc_o[dt][v] *= alpha;
            m_run = m_new;
        }
        const float m_use = m_run == -INFINITY ? 0.0f : m_run;
        float psum = 0.0f;
        // four scores at a time: exponentials, their sum and their bf16 pair conversions are
        // finished before the next four start (keeps only four probabilities live)
        static_for<8>([&](auto chunk) __attribute__((always_inline)) {
            constexpr int c = decltype(chunk)::value;
            constexpr int kt = c >> 2, v0 = (c & 3) * 4;
            if constexpr (c * NI % 8 == 0) {
                __builtin_amdgcn_sched_barrier(0);
                load(std::integral_constant<int, c * NI / 8>{});
                __builtin_amdgcn_sched_barrier(0);
            }
            float pv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) pv[u] = __builtin_amdgcn_exp2f(fmaf(s[kt][v0 + u], scale_log2, -m_use));
            psum += (pv[0] + pv[1]) + (pv[2] + pv[3]);
            typedef float f32x2 __attribute__((ext_vector_type(2)));
            typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));
            bf16x2 lo = __builtin_convertvector(f32x2{pv[0], pv[1]}, bf16x2);
            bf16x2 hi = __builtin_convertvector(f32x2{pv[2], pv[3]}, bf16x2);
            asm volatile("" : "+v"(lo), "+v"(hi));   // converted here, not gathered at the end
            bf16x8& dst = pf[kt * 2 + (v0 >> 3)];
            dst[(v0 & 7) + 0] = lo[0];
            dst[(v0 & 7) + 1] = lo[1];
            dst[(v0 & 7) + 2] = hi[0];
            dst[(v0 & 7) + 3] = hi[1];
            });
        l_run += psum;
    };
    // End of a phase: all of this wave's global -> LDS loads but the newest tile's
    // (`pending`) have landed, then the workgroup barrier.  The tile
    // reads are written by hand, so no compiler-made wait is needed around the barrier.
    auto phase_end = [&](bool pending) __attribute__((always_inline)) {
        if (pending) __builtin_amdgcn_s_waitcnt((NI & 0xF) | ((NI >> 4) << 14) | (0x7 << 4) | (0xF << 8));
        else __builtin_amdgcn_s_waitcnt((0x7 << 4) | (0xF << 8));
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // Matrix phase of one wave: O^T += V^T P^T for the V tile at vaddr (with_pv), then
    // S^T = K Q^T for the K tile at kaddr.  The other wave of the SIMD is in
    // its softmax, so this wave alone has to keep the matrix pipe fed: the LDS reads of MFMA
    // j + PD are issued before MFMA j.  P V: MFMA j = (ss, dt) = (j / DT, j % DT), DT
    // independent accumulation chains; A slots 0..3 <- keys 16ss+4hf.., 4..7 <- keys
    // 16ss+8+4hf..  Scores: MFMA n = (ks, kt) = (n / 2, n % 2), two chains.
    constexpr int PD = 4;
    auto matrix_phase = [&](auto with_pv) __attribute__((always_inline)) {
        constexpr int NPV = decltype(with_pv)::value ? 4 * DT : 0, NQK = 2 * KS, NALL = NPV + NQK;
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        bf16x8 opnd[NALL];
        // Order of the MFMAs when both contractions run: two of P V, two of Q K^T, and so on, so
        // that an MFMA follows the one whose accumulator it continues four issue slots later, not
        // two (the score tile has only two accumulation chains; back to back they wait for each
        // other's result).
        constexpr auto is_pv = [](int j) constexpr { return NPV != 0 && (j & 3) < 2; };
        constexpr auto pv_of = [](int j) constexpr { return (j >> 2) * 2 + (j & 3); };
        constexpr auto qk_of = [](int j) constexpr { return NPV != 0 ? (j >> 2) * 2 + (j & 3) - 2 : j; };
        static_assert(NPV == 0 || NPV == NQK, "the interleaved order pairs the two contractions one to one");
        // reads of the operands j+1 .. last (a P V operand is two reads)
        constexpr auto reads_after = [](int j, int last) constexpr {
            int n = 0;
            for (int i = j + 1; i <= last; ++i) n += (NPV != 0 && (i & 3) < 2) ? 2 : 1;
            return n;
        };
        auto issue = [&](auto jc) __attribute__((always_inline)) {
            constexpr int j = decltype(jc)::value;
            if constexpr (j < NALL) {
                if constexpr (is_pv(j)) {
                    constexpr int p = pv_of(j), ss = p / DT, dt = p % DT;
                    constexpr int at = 2 * rho(16 * ss) * D_H;
                    constexpr int at8 = 2 * rho(16 * ss + 8) * D_H;
                    const bf16x4 a0 = lds_read_tr_at<at>(vaddr[dt]);
                    const bf16x4 a1 = lds_read_tr_at<at8>(vaddr[dt]);
                    opnd[j] = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
                } else {
                    constexpr int n = qk_of(j), ks = n / 2, kt = n % 2;
                    opnd[j] = lds_read_b128_at<2 * kt * 8 * D_H>(kaddr[ks]);
                }
            }
        };
        static_for<PD>(issue);
        static_for<NALL>([&](auto jc) __attribute__((always_inline)) {
            constexpr int j = decltype(jc)::value;
            issue(std::integral_constant<int, j + PD>{});
            constexpr int last = j + PD < NALL ? j + PD : NALL - 1;
            lds_wait_all_but<reads_after(j, last)>(opnd[j]);
            if constexpr (is_pv(j)) {
                constexpr int p = pv_of(j), ss = p / DT, dt = p % DT;
                acc_o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(opnd[j], pf[ss], acc_o[dt], 0, 0, 0);
            } else {
                constexpr int n = qk_of(j), ks = n / 2, kt = n % 2;
                s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(opnd[j], qf[ks], ks == 0 ? zero : s[kt], 0, 0, 0);
            }
        });
    };

    // ---- phases.  P0: A scores(0).  P(2t+1): A softmax(t) | B values(t-1), scores(t).
    //      P(2t+2): A values(t), scores(t+1) | B softmax(t).  A wave issues its loads in its
    //      softmax phase, between the exponentials.  Group A loads V(t+2) in P(2t+1) into the
    //      stage of V(t-2), which group B left in P(2t-1); first read in P(2t+6).  Group A lets
    //      only its newest tile stay in flight at the end of P(2t+1): V(t+1) has landed, and is
    //      first read in P(2t+4).  Group B loads K(t+3) in P(2t+2) into the stage of K(t), which it
    //      left in P(2t+1); at the end of P(2t+2) K(t+2) has landed, first read in P(2t+4).
    //      Every wave passes 2 n_tiles + 3 barriers; tiles past a wave's own last key only cost it
    //      the barriers and its loads.  The scores of tile my_tiles (computed from whatever its
    //      stage holds) are never used.
    const int my_tiles = wave_limit < 0 ? 0 : max(0, min(wave_limit / BN_KEYS + 1 - ta, n_tiles));
    using yes = std::integral_constant<int, 1>;
    using no = std::integral_constant<int, 0>;
    int k_at = 0, v_at = 0;           // stages the address registers point at
    auto advance = [&](bool also_v) __attribute__((always_inline)) {
        const int kd = k_at == 2 ? -4 * TILE : 2 * TILE;
        k_at = k_at == 2 ? 0 : k_at + 1;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kaddr[ks] += kd;
        if (also_v) {
            const int vd = v_at == 3 ? -6 * TILE : 2 * TILE;
            v_at = v_at == 3 ? 0 : v_at + 1;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) vaddr[dt] += vd;
        }
    };
    if (grp == 0) {
        load_tile(tile_at(0), v_stage(0));
        if (n_tiles > 1) load_tile(tile_at(1), v_stage(1));
        phase_end(n_tiles > 1);                            // K(0), V(0) are in place
        if (my_tiles > 0) {                                // P0
            matrix_phase(no{});
            advance(false);
        }
        phase_end(n_tiles > 1);
        for (int t = 0; t < n_tiles; ++t) {
            const char* next = tile_at(min(t + 2, n_tiles - 1));   // past the end: the last tile again, unused
            if (t < my_tiles)
                softmax(j_a + t * BN_KEYS, [&](auto i) __attribute__((always_inline)) { load_part(next, v_stage(t + 2), i); });
            else
                load_tile(next, v_stage(t + 2));
            phase_end(true);                               // V(t), V(t+1) have landed
            if (t < my_tiles) {
                matrix_phase(yes{});
                advance(true);
            }
            phase_end(true);
        }
        phase_end(false);
    } else {
        load_tile(tile_at(0), k_stage(0));
        if (n_tiles > 1) load_tile(tile_at(1), k_stage(1));
        if (n_tiles > 2) load_tile(tile_at(2), k_stage(2));
        if (n_tiles > 2) __builtin_amdgcn_s_waitcnt(((2 * NI) & 0xF) | (((2 * NI) >> 4) << 14) | (0x7 << 4) | (0xF << 8));
        phase_end(n_tiles > 1);                            // K(0), V(0) are in place
        phase_end(true);                                   // P0
        if (my_tiles > 0) {                                // P1
            matrix_phase(no{});
            advance(false);
        }
        phase_end(n_tiles > 2);                            // K(1) has landed
        for (int t = 0; t < n_tiles; ++t) {
            const char* next = tile_at(min(t + 3, n_tiles - 1));   // past the end: the last tile again, unused
            if (t < my_tiles)
                softmax(j_a + t * BN_KEYS, [&](auto i) __attribute__((always_inline)) { load_part(next, k_stage(t), i); });
            else
                load_tile(next, k_stage(t));
            phase_end(true);                               // K(t+2) has landed
            if (t < my_tiles) {
                matrix_phase(yes{});
                advance(true);
            }
            phase_end(true);
        }
    }

    __builtin_amdgcn_s_waitcnt((0x7 << 4) | (0xF << 8));   // the unused loads of the last tiles have landed

    // ---- normalise and write: lane holds 4 consecutive d per (dt, v/4) ----
    float l_tot = l_run + __shfl_xor(l_run, 32);
    if (!valid) return;
    if (!PIECE || slot < 0) {
        const float inv = 1.0f / l_tot;
        bf16_t* op = o + ((int64_t)mi * H_q + kvh * g + hg) * D_H;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
                bf16x4 w;
#pragma unroll
                for (int u = 0; u < 4; ++u) w[u] = (bf16_t)(acc_o[dt][vq * 4 + u] * inv);
                *reinterpret_cast<bf16x4*>(op + dt * 32 + 8 * vq + 4 * hf) = w;
            }
    } else {
        // as the registers lie, so that every store is one contiguous KB: [wave][D_H / 8][lane] four
        // unnormalised sums, then [lane] the exponent's reference point and the row sum
        float* pp = part + (int64_t)slot * 256 * (D_H + 4) + (grp * 4 + widx) * 32 * (D_H + 4);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
                f32x4 w;
#pragma unroll
                for (int u = 0; u < 4; ++u) w[u] = acc_o[dt][vq * 4 + u];
                *reinterpret_cast<f32x4*>(pp + (dt * 4 + vq) * 256 + lane * 4) = w;
            }
        *reinterpret_cast<float2*>(pp + 32 * D_H + lane * 2) = make_float2(m_run, l_tot);
    }
}

// One block of 256 columns per workgroup, longest first.  Off: 64 bits only for token strides that
// a 32-bit lane offset cannot hold.
#define CC_ATTN_ARGS                                                                                        \
    const bf16_t *__restrict__ q, int M, const int32_t *__restrict__ idx, int H_q, int H_kv,                \
        const bf16_t *__restrict__ Kc, const bf16_t *__restrict__ Vc, int64_t st, int64_t sh, int N,        \
        bf16_t *__restrict__ o, int n_row_tiles, float scale_log2
template <int D_H, class Off>
__device__ __forceinline__ void attend_block(CC_ATTN_ARGS) {
    __shared__ __align__(16) bf16_t smem[LDS_TILES * BN_KEYS * D_H];
    __shared__ int simd_waves[4], group_waves[2];
    int grp, widx;
    wave_role(simd_waves, group_waves, grp, widx);
    const int g = H_q / H_kv, kvh = blockIdx.x % H_kv, rt = n_row_tiles - 1 - blockIdx.x / H_kv;
    attend<D_H, false, Off>(q, M, idx, H_q, g, Kc, Vc, st, sh, N, o, scale_log2, nullptr, smem, grp, widx, kvh, rt, 0,
                            last_key(idx, M, g, rt) / BN_KEYS + 1, -1);
}
template <int D_H>
__global__ __launch_bounds__(512, 1) void sparse_attn_kernel(CC_ATTN_ARGS) {
    attend_block<D_H, uint32_t>(q, M, idx, H_q, H_kv, Kc, Vc, st, sh, N, o, n_row_tiles, scale_log2);
}
template <int D_H>
__global__ __launch_bounds__(512, 1) void wide_stride_attn_kernel(CC_ATTN_ARGS) {
    attend_block<D_H, uint64_t>(q, M, idx, H_q, H_kv, Kc, Vc, st, sh, N, o, n_row_tiles, scale_log2);
}

// Even grid.  A block costs as many key tiles as its last row can see, so a grid of a few hundred
// blocks ends unevenly: its makespan is the longest block or one more round.  Here every workgroup (one
// per CU) takes the same number of units of one long sequence: the blocks of kv head 0 by row
// tile, those of head 1, ...; a block of L key tiles is L + EVEN_START units long, the first of
// them for what a block costs besides its tiles (query loads, first tiles, output).  A range
// covers some whole blocks and, at its ends, pieces of two; the pieces go to slots 2 w and 2 w + 1
// of range w (a piece of the block that the range starts in, of a later one) and
// attn_merge_kernel combines the pieces of a block.  Consecutive ranges run on one XCD, so that its
// L2 serves one kv head when H_kv = 8.
constexpr int EVEN_START = CC_ATTN_EVEN_START;          // 3 and 5 units measured: 5 is 1 % of the layer faster
constexpr int EVEN_MAX_TILES = CC_ATTN_EVEN_MAX_TILES;
// table: [n_row_tiles + 2] the first unit of every row tile within a head, their sum, units per range
template <int D_H>
__global__ __launch_bounds__(512, 1) void even_attn_kernel(CC_ATTN_ARGS, int per_min, float* __restrict__ part,
                                                           int* __restrict__ table) {
    __shared__ __align__(16) bf16_t smem[LDS_TILES * BN_KEYS * D_H];
    __shared__ int simd_waves[4], group_waves[2], wave_units[8];
    __shared__ int pre[EVEN_MAX_TILES + 1];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int g = H_q / H_kv;
    int grp, widx;
    wave_role(simd_waves, group_waves, grp, widx);

    // first unit of every row tile: exclusive scan, two row tiles a thread
    int len[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
        len[i] = 2 * tid + i < n_row_tiles ? last_key(idx, M, g, 2 * tid + i) / BN_KEYS + 1 + EVEN_START : 0;
    int inc = len[0] + len[1];
    for (int off = 1; off < 64; off <<= 1) {
        const int v = __shfl_up(inc, off);
        if (lane >= off) inc += v;
    }
    if (lane == 63) wave_units[w] = inc;
    __syncthreads();
    int base = inc - len[0] - len[1];
    for (int i = 0; i < w; ++i) base += wave_units[i];
    pre[2 * tid] = base;
    pre[2 * tid + 1] = base + len[0];
    if (tid == 511) pre[EVEN_MAX_TILES] = base + len[0] + len[1];
    __syncthreads();
    const int head_units = __builtin_amdgcn_readfirstlane(pre[n_row_tiles]);   // tiles past the last have no units
    const int total = head_units * H_kv, n_wg = gridDim.x;
    const int per = max(per_min, (total + n_wg - 1) / n_wg);
    if (blockIdx.x == 0) {
        for (int t = tid; t <= n_row_tiles; t += 512) table[t] = pre[t];
        if (tid == 0) table[n_row_tiles + 1] = per;
    }
    // workgroup ids go round-robin to the 8 XCDs: each gets consecutive ranges
    const int x = blockIdx.x & 7, xq = n_wg >> 3, xr = n_wg & 7;
    const int range = x * xq + min(x, xr) + (int)(blockIdx.x >> 3);
    int u = range * per, stop = min(u + per, total);     // units of the whole sequence, then of head kvh
    if (u < total) {
        int kvh = u / head_units;
        u -= kvh * head_units;
        stop -= kvh * head_units;
        int rt = 0;                                      // last row tile whose first unit is <= u
        for (int hi = n_row_tiles - 1; rt < hi;) {
            const int mid = (rt + hi + 1) >> 1;
            if (pre[mid] <= u) rt = mid; else hi = mid - 1;
        }
        rt = __builtin_amdgcn_readfirstlane(rt);
        for (int later = 0; u < stop; later = 1) {
            const int b0 = __builtin_amdgcn_readfirstlane(pre[rt]), b1 = __builtin_amdgcn_readfirstlane(pre[rt + 1]);
            const int ta = max(0, u - b0 - EVEN_START), te = min(b1, stop) - b0 - EVEN_START;
            if (te > ta) {
                const bool whole = ta == 0 && te == b1 - b0 - EVEN_START;
                attend<D_H, true, uint32_t>(q, M, idx, H_q, g, Kc, Vc, st, sh, N, o, scale_log2, part, smem, grp, widx,
                                            kvh, rt, ta, te - ta, whole ? -1 : 2 * range + later);
            }
            u = b1;
            if (++rt == n_row_tiles) {
                rt = 0;
                ++kvh;
                u = 0;
                stop -= head_units;
            }
        }
    }
}

// Whole blocks cut S ways: workgroup (block, s) takes the s-th of S equal runs of the block's key tiles
// and leaves its piece in slot block * S + s; attn_merge_kernel combines them.
template <int D_H, class Off>
__device__ __forceinline__ void attend_cut(CC_ATTN_ARGS, float* __restrict__ part) {
    __shared__ __align__(16) bf16_t smem[LDS_TILES * BN_KEYS * D_H];
    __shared__ int simd_waves[4], group_waves[2];
    int grp, widx;
    wave_role(simd_waves, group_waves, grp, widx);
    const int g = H_q / H_kv, kvh = blockIdx.x % H_kv, rt = n_row_tiles - 1 - blockIdx.x / H_kv, S = gridDim.y;
    const int L = last_key(idx, M, g, rt) / BN_KEYS + 1, per = (L + S - 1) / S;
    const int ta = blockIdx.y * per, n = min(per, L - ta);
    const int slot = (kvh * n_row_tiles + rt) * S + blockIdx.y;
    if (n <= 0) {                                        // a short block: no keys for this piece
        float* pp = part + (int64_t)slot * 256 * (D_H + 4) + (threadIdx.x >> 6) * 32 * (D_H + 4);
        *reinterpret_cast<float2*>(pp + 32 * D_H + (threadIdx.x & 63) * 2) = make_float2(-INFINITY, 0.0f);
        return;
    }
    attend<D_H, true, Off>(q, M, idx, H_q, g, Kc, Vc, st, sh, N, o, scale_log2, part, smem, grp, widx, kvh, rt, ta, n, slot);
}
template <int D_H>
__global__ __launch_bounds__(512, 1) void cut_attn_kernel(CC_ATTN_ARGS, float* __restrict__ part) {
    attend_cut<D_H, uint32_t>(q, M, idx, H_q, H_kv, Kc, Vc, st, sh, N, o, n_row_tiles, scale_log2, part);
}

template <int D_H>
__global__ __launch_bounds__(512, 1) void wide_stride_cut_attn_kernel(CC_ATTN_ARGS, float* __restrict__ part) {
    attend_cut<D_H, uint64_t>(q, M, idx, H_q, H_kv, Kc, Vc, st, sh, N, o, n_row_tiles, scale_log2, part);
}

// Combines the pieces of the blocks that an even grid (S = 0) or a cut one (S pieces) has left:
// o = sum_s 2^(m_s - m) O_s / sum_s 2^(m_s - m) l_s with m = max m_s, pieces in the order of their keys.
// Workgroup (block, 32 of its columns = one wave of the attention kernel, 32 of their d's); a
// thread holds the same elements as the lane that wrote them, four of a column.  Up to eight pieces at
// a time, so that their loads are out together.  Workgroup id modulo H_kv is the kv head, as in the attention
// kernels, so that a piece is read through the L2 that it was written to: with the heads one after
// the other 64 blocks of 3 pieces took 34 us in both launches, so 25 (64 query heads of 8, N = 850,
// M = 256).  32 d's a workgroup instead of all: 1 to 2 us of a few blocks' merge.
template <int D_H>
__global__ __launch_bounds__(256) void attn_merge_kernel(const float* __restrict__ part, const int* __restrict__ table,
                                                         int S, int M, int H_q, int H_kv, int n_row_tiles,
                                                         bf16_t* __restrict__ o) {
    const int g = H_q / H_kv, kvh = blockIdx.x % H_kv, rt = blockIdx.x / H_kv;
    int w0 = 0, w1 = S - 1, per = 1, first = 0;
    if (S == 0) {                                        // even grid: the ranges that hold the block's key tiles
        per = table[n_row_tiles + 1];
        const int head = kvh * table[n_row_tiles], end = head + table[rt + 1];
        first = head + table[rt];
        w0 = (first + EVEN_START) / per;
        w1 = (end - 1) / per;
        if (w0 == w1) return;
    }
    const int lane = threadIdx.x & 63, v0 = blockIdx.z * 4 + (threadIdx.x >> 6);     // 16-byte group of a column
    const int col = rt * 256 + blockIdx.y * 32 + (lane & 31), mi = col / g, hg = col - mi * g;
    if (mi >= M) return;
    float m = -INFINITY, l = 0.0f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    auto take = [&](auto nc, int wb) __attribute__((always_inline)) {
        constexpr int NP = decltype(nc)::value;
        f32x4 v[NP];
        float2 ml[NP];
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int w = min(wb + k, w1);               // past the end: the last piece again, with weight 0
            const int slot = S ? (kvh * n_row_tiles + rt) * S + w : 2 * w + (w * per < first ? 1 : 0);
            const float* pp = part + (int64_t)slot * 256 * (D_H + 4) + blockIdx.y * 32 * (D_H + 4);
            ml[k] = *reinterpret_cast<const float2*>(pp + 32 * D_H + lane * 2);
            v[k] = *reinterpret_cast<const f32x4*>(pp + v0 * 256 + lane * 4);
        }
        float mn = m;
#pragma unroll
        for (int k = 0; k < NP; ++k) mn = fmaxf(mn, ml[k].x);
        const float ref = mn == -INFINITY ? 0.0f : mn;   // no key of this column so far
        const float keep = __builtin_amdgcn_exp2f(m - ref);
        l *= keep;
        acc *= keep;
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            // a piece without keys of this column: a cut grid's empty piece leaves no sums at all
            const bool on = wb + k <= w1 && ml[k].x != -INFINITY;
            const float f = on ? __builtin_amdgcn_exp2f(ml[k].x - ref) : 0.0f;
            l += ml[k].y * f;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] += on ? v[k][e] * f : 0.0f;
        }
        m = mn;
    };
    for (int wb = w0; wb <= w1;) {
        const int left = w1 - wb + 1;
        if (left > 4) take(std::integral_constant<int, 8>{}, wb), wb += 8;
        else if (left > 2) take(std::integral_constant<int, 4>{}, wb), wb += 4;
        else take(std::integral_constant<int, 2>{}, wb), wb += 2;
    }
    const float inv = l > 0.0f ? 1.0f / l : 0.0f;
    bf16_t* op = o + ((int64_t)mi * H_q + kvh * g + hg) * D_H + 4 * (lane >> 5);
    bf16x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = (bf16_t)(acc[e] * inv);
    *reinterpret_cast<bf16x4*>(op + 8 * v0) = r;
}

}  // namespace

int cc_attn_piece_workgroups(const cc_model_desc& m, int64_t M, int64_t N) {
    return cc_plan_attn_workgroups(cc_device_cus(), (M * (m.H_q / m.H_kv) + 255) / 256 * m.H_kv, (N + BN_KEYS - 1) / BN_KEYS);
}

void cc_launch_attention(const bf16_t* q, int M, const int32_t* idx, const cc_model_desc& m,
                         const cc_kv_layer& kv, bf16_t* o, float* part, int slots, int* table,
                         const cc_launch_override& ovr, hipStream_t s) {
    if (M <= 0) return;
    const int g = m.H_q / m.H_kv;
    const int n_row_tiles = (int)(((int64_t)M * g + 255) / 256);   // 256 (token, head) columns each
    const float scale_log2 = 1.4426950408889634f / sqrtf((float)m.d_h);
    const int n_wg = n_row_tiles * m.H_kv;
    const int t_max = (kv.N + BN_KEYS - 1) / BN_KEYS;
#define CC_ATTN_LAUNCH(KERN, GRID, ...)                                                                       \
    do {                                                                                                      \
        if (m.d_h == 128)                                                                                     \
            hipLaunchKernelGGL(KERN<128>, dim3(GRID), dim3(512), 0, s, q, M, idx, m.H_q, m.H_kv,              \
                               (const bf16_t*)kv.K, (const bf16_t*)kv.V, kv.stride_token, kv.stride_head,     \
                               kv.N, o, n_row_tiles, scale_log2, ##__VA_ARGS__);                              \
        else                                                                                                  \
            hipLaunchKernelGGL(KERN<64>, dim3(GRID), dim3(512), 0, s, q, M, idx, m.H_q, m.H_kv,               \
                               (const bf16_t*)kv.K, (const bf16_t*)kv.V, kv.stride_token, kv.stride_head,     \
                               kv.N, o, n_row_tiles, scale_log2, ##__VA_ARGS__);                              \
    } while (0)
    // 64 rows of a tile, 2 bytes an element, in an unsigned 32-bit lane offset
    const bool wide = kv.stride_token >= (1ll << 32) / (2 * (BN_KEYS + 1));
    const cc_attn_plan p = cc_plan_attention(cc_device_cus(), n_row_tiles, m.H_kv, m.d_h, t_max, slots, wide, ovr.attn_splits);
    if (p.kind == CC_ATTN_EVEN) {
        CC_ATTN_LAUNCH(even_attn_kernel, p.ranges, p.per_min, part, table);
    } else if (p.kind == CC_ATTN_CUT) {
        const dim3 cg(n_wg, p.pieces);
        if (wide) CC_ATTN_LAUNCH(wide_stride_cut_attn_kernel, cg, part);
        else CC_ATTN_LAUNCH(cut_attn_kernel, cg, part);
    } else if (wide) {
        CC_ATTN_LAUNCH(wide_stride_attn_kernel, n_wg);
    } else {
        CC_ATTN_LAUNCH(sparse_attn_kernel, n_wg);
    }
    if (p.kind != CC_ATTN_WHOLE) {
        const int S = p.kind == CC_ATTN_CUT ? p.pieces : 0;
        const dim3 mg(n_wg, 8, m.d_h / 32);
        if (m.d_h == 128)
            hipLaunchKernelGGL(attn_merge_kernel<128>, mg, dim3(256), 0, s, part, table, S, M, m.H_q, m.H_kv, n_row_tiles, o);
        else
            hipLaunchKernelGGL(attn_merge_kernel<64>, mg, dim3(256), 0, s, part, table, S, M, m.H_q, m.H_kv, n_row_tiles, o);
    }
#undef CC_ATTN_LAUNCH
}
