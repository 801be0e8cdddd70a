// Flash-attention forward, gfx950, d = 128 and 64: the whole query tiles of a launch in pairs, 512 rows a workgroup.
//
// The kernel of attn_fwd_sp.hip gives a wavefront 32 query rows, so every operand fragment that it reads from LDS feeds one
// MFMA, and every K/V tile that a CU fetches serves 256 rows.  Both cost power, which bounds long sweeps on this data (an
// MFMA-only loop runs at 1 750 TFLOP/s, with the softmax arithmetic 1 550, with the operand reads 1 380, with half of them 1 460).  Here a
// wavefront owns 64 rows: 128 registers of O, 64 of Q and 32 of scores or packed probabilities leave no room to overlap
// the softmax of one tile with the products of another inside a wavefront.  The overlap is between the two
// wavefronts of a SIMD instead: wavefronts 0-3 and 4-7 of a workgroup run in opposite phases,
//
//     matrix phase of step t:  O += V_{t-1} P_{t-1}, S_t = K_t Q^T      (32 keys; 32 MFMAs at d = 128, 1 024 cycles)
//     softmax phase:           P_t = exp2(S_t c - reference)            (about 600 cycles of the VALU)
//
// with a barrier at the end of each, so that one of the two feeds the matrix pipe at any time (raised priority there: without
// it 1 % slower, zeros 6 %).  The four-slot rings of K and V tiles are filled two steps ahead.  4 heads x 65 536, d = 128: 6 620 ->
// 6 070 us = 1 450 TFLOP/s (on zeros 4 336 -> 3 968), d = 64 4 020 -> 3 840; with one block of 32 rows per wavefront in the
// same phases 6 900, so single tiles and key ranges stay with the other kernel's code.
//
// A launch starts with n_wide wide items, pairs of consecutive tiles of a head, taken like any items; the
// others follow in the same workgroups (sp_items): the last tile of each head of an odd number of tiles that wide items cover,
// then whatever lies behind the wide items.  How many are wide: attn_internal.h, wide_plan.  A row gets the bits it has in a
// single tile: same reference, same order of sums.  Rows that need the second sweep get it there, too: a wide item
// hands back a tile with such a row, and the workgroup makes the running-max sweep of that tile later, for the rows that the wide
// item has found; if it has collected sixteen, it takes no more wide items than it has claimed and sweeps those as single tiles.
// Wavefronts without such a row only fetch for that sweep (fetch_for_sweep).  us, without pairs -> with pairs: 24 x 9 600 with every row
// swept twice 1 774 -> 1 729, with one row in 160 1 882 -> 1 571 (2 293 and 2 381 with the first sweep of a tile given back repeated as
// well; 1 867 for the latter with all wavefronts computing in the second; another box, 1 866 and 1 939 without pairs).  24 x 16 384
// on 570 keys with one row in 500 174 -> 184: in short sweeps items of 128 rows, which such launches have without pairs, are swept again
// less often than tiles of 256.
#ifndef PDA_SP_DEVICE_ONLY
#define PDA_SP_DEVICE_ONLY
#endif
#include "attn_fwd_sp.hip"

namespace pda {

template <int D>
struct Wide {
    static constexpr int KEYS = 32;                    // keys of a step
    static constexpr int TILE = KEYS * D * 2;          // 8 KB or 4 KB
    static constexpr int RING = 4;                     // tile buffers per tensor
    static constexpr int AHEAD = 2;                    // V tile t + AHEAD and K tile t + 1 + AHEAD are fetched in step t
    static constexpr int ROWS = 512;                   // query rows of a workgroup
};

// The kernel's arguments, read where they are needed: kept in scalar registers from the start they would be spilled into
// lanes of vector registers, of which the main loop has none to spare.
typedef const AttnParams __attribute__((address_space(4))) KernelArgs;
__device__ __forceinline__ KernelArgs& args_here() {
    auto x = (KernelArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(x));
    return *x;
}

// The part of a wavefront in sp_items' second sweep of a tile given back of which none of its rows needs it: its chunks of every
// tile of K and V, and the barriers of that sweep, in the same order.  A sweep in which half of the wavefronts compute nothing is shorter.
template <int D>
__device__ __forceinline__ void fetch_for_sweep(KernelArgs& p, int tile, int wave) {
    constexpr int BN = 64, G = D / 8, NBUF = sp_buffers(D, 8), TILE = BN * D * 2, CPW = TILE / 1024 / 8, RPC = 1024 / (D * 2);
    static_assert(NBUF == 4, "the ring of sp_items with eight wavefronts");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const unsigned dma_base = (unsigned)(uintptr_t)(LDS_PTR(const void))smem + wave * 1024;
    const int bh = tile / p.tiles_per_head, b = bh / p.Hg, h = bh - b * p.Hg, n_v = (int)p.n_v, nt = (n_v + BN - 1) / BN, l = fresh_lane();
    const __bf16* kp = p.k + (int64_t)b * p.kv_bs + (int64_t)h * p.kv_hs;
    const __bf16* vp = p.v + (int64_t)b * p.kv_bs + (int64_t)h * p.kv_hs;
    auto issue = [&](bool is_k, int buf, int t) __attribute__((always_inline)) {
        const __bf16* src = (is_k ? kp : vp) + (int64_t)t * BN * D;
        const int last = n_v - t * BN - 1;                     // hidden keys are never read
#pragma unroll
        for (int j = 0; j < CPW; ++j) {
            const int row = wave * RPC + l / G + j * (8 * RPC);
            const unsigned at = (((l % G) ^ (is_k ? swz_k<D>(row) : swz_v<D>(row))) * 16);
            lds_dma16(src, (unsigned)(row < last ? row : last) * (D * 2) + at, dma_base + ((is_k ? 0 : NBUF) + buf) * TILE + j * 8192);
        }
    };
    auto barrier = [&]() __attribute__((always_inline)) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    for (int t = 0; t < NBUF && t < nt; ++t) issue(true, t, t);
    for (int t = 0; t < NBUF - 2 && t < nt; ++t) issue(false, t, t);
    wait_vmcnt<0>();
    barrier();                                                 // Q and the first tiles are there
    barrier();                                                 // the first scores are
    for (int t = 0; t < nt - 1; ++t) {
        if (t + NBUF < nt) issue(true, t % NBUF, t + NBUF);
        if (t + NBUF - 2 < nt) issue(false, (t + NBUF - 2) % NBUF, t + NBUF - 2);
        if (nt - t > 4) wait_vmcnt<4 * CPW>();                 // K tile t + 2 and V tile t, as there
        else if (nt - t == 4) wait_vmcnt<3 * CPW>();
        else if (nt - t == 3) wait_vmcnt<2 * CPW>();
        else wait_vmcnt<0>();
        barrier();
    }
    barrier();                                                 // the sweep is over
}

template <int D, bool BASE2, bool OUT16>
__global__ __launch_bounds__(512, 2) void attn_fwd_wide_kernel(const AttnParams) {
    constexpr int KEYS = Wide<D>::KEYS, TILE = Wide<D>::TILE, R = Wide<D>::RING, P = Wide<D>::AHEAD;
    constexpr int G = D / 8, NKK = D / 16, NDB = D / 32;
    constexpr int K_BASE = 0, V_BASE = R * TILE;
    constexpr int RPC = 1024 / (D * 2);                // rows of a 1 KB chunk
    constexpr int LPI = D == 128 ? 2 : 1;              // loads of a wavefront per step: a chunk of K and one of V, or one of either
    constexpr int kStores = 2 * ((OUT16 ? 2 : 4) * NDB + 1);      // stores of a wavefront's results
    constexpr int kRedoMax = 16;

    extern __shared__ __attribute__((aligned(256))) unsigned char wide_smem[];      // aligned to a row: blocks are XORed into addresses
    __shared__ int w_next;
    __shared__ int w_flag[8];
    __shared__ int w_redo[kRedoMax];
    __shared__ unsigned w_rows[kRedoMax][8];           // of a tile given back: the rows that need the second sweep, 32 each

    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const bool second = wave >= 4;                     // the group of wavefronts that runs a phase behind
    const unsigned lds0 = (unsigned)(uintptr_t)(LDS_PTR(const void))wide_smem;
    int item = (int)blockIdx.x, n_redo = 0;
    float c;
    int n_v, n_wide;
    bool direct;
    {
        KernelArgs& p = args_here();
        c = BASE2 ? 1.0f : p.scale_log2e;
        n_v = (int)p.n_v;
        n_wide = p.n_wide;
        direct = p.n_items - p.n_wide <= (int)gridDim.x;
    }
    const int nt = (n_v + KEYS - 1) / KEYS;

    auto barrier = [&]() __attribute__((always_inline)) {          // keeps the phases apart
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    auto lds_done = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };

    if (item < n_wide) {
        const int lane = fresh_lane(), li = lane & 31, lh = lane >> 5;
        const int cw = D == 128 ? wave : wave & 3;             // d = 64: wavefronts 0-3 fetch K, 4-7 V
        const int crow = cw * RPC + lane / G;
        const unsigned ld_k = crow * (D * 2) + (((lane % G) ^ swz_k<D>(crow)) * 16);
        const unsigned ld_v = crow * (D * 2) + (((lane % G) ^ swz_v<D>(crow)) * 16);
        const unsigned dma_base = lds0 + cw * 1024;
        // operand addresses of buffer 0 and block 0; blocks are XORed in, buffers are immediates
        unsigned k_at = lds0 + K_BASE + li * (D * 2) + ((lh ^ swz_k<D>(li)) * 16);
        const int t16 = lane & 15, v_key_in = 4 * lh + (t16 >> 2);
        unsigned v_at = lds0 + V_BASE + v_key_in * (D * 2) + (((2 * (li >> 4) + ((t16 & 3) >> 1)) ^ swz_v<D>(v_key_in)) * 16) + (t16 & 1) * 8;
        asm volatile("" : "+v"(k_at), "+v"(v_at));
        auto block = [](unsigned at, auto n) __attribute__((always_inline)) {
            unsigned r = at;
            if constexpr (decltype(n)::value != 0) asm volatile("v_xor_b32 %0, %1, %2" : "=v"(r) : "n"(decltype(n)::value), "v"(at));
            return r;
        };
        auto k_frag = [&](unsigned at, auto off, auto kk) __attribute__((always_inline)) {
            return *(LDS_PTR(const bf16x8))((LDS_PTR(const unsigned char))(uintptr_t)block(at, std::integral_constant<int, decltype(kk)::value * 32>{}) + decltype(off)::value);
        };
        auto v_frag = [&](unsigned at, auto off, auto db) __attribute__((always_inline)) {
            LDS_PTR(const unsigned char) x = (LDS_PTR(const unsigned char))(uintptr_t)block(at, std::integral_constant<int, decltype(db)::value * 64>{}) + decltype(off)::value;
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))x);
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))(x + 8 * (D * 2)));
            return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        };

        const __bf16* kp = nullptr;
        const __bf16* vp = nullptr;
        bf16x8 qf[2][NKK];
        // this wavefront's chunk of a tile; rows beyond the last valid key: that key again
        auto issue = [&](const __bf16* base, bool is_v, int buf, int tile) __attribute__((always_inline)) {
            if (D == 64 && is_v != second) return;
            const __bf16* src = base + (int64_t)tile * (KEYS * D);
            const unsigned lds = dma_base + (is_v ? V_BASE : K_BASE) + buf * TILE;
            const int last = n_v - tile * KEYS - 1;
            if (last >= KEYS - 1) {
                lds_dma16(src, is_v ? ld_v : ld_k, lds);
            } else {
                const int l = fresh_lane(), row = cw * RPC + l / G;
                lds_dma16(src, (unsigned)(row < last ? row : last) * (D * 2) + (((l % G) ^ (is_v ? swz_v<D>(row) : swz_k<D>(row))) * 16), lds);
            }
        };
        auto place = [&](KernelArgs& p, int it, int& b, int& h, int64_t& row0) __attribute__((always_inline)) {
            const int pairs_per_head = p.tiles_per_head >> 1, bh = it / pairs_per_head;
            b = bh / p.Hg;
            h = bh - b * p.Hg;
            row0 = (int64_t)(it - bh * pairs_per_head) * Wide<D>::ROWS + wave * 64;
        };
        // Q rows of 32-row block i of item `it`: 64 bytes of 16 rows per load, put in order by arrange_q
        auto load_q = [&](auto i_c, KernelArgs& p, int b, int h, int64_t row0) __attribute__((always_inline)) {
            constexpr int i = decltype(i_c)::value;
            const int l = fresh_lane();
            const int64_t first = row0 + 32 * i < p.Sq ? row0 + 32 * i : p.Sq - 1;         // rows beyond the last one: the last one again
            const int last = (int)(p.Sq - 1 - first < 31 ? p.Sq - 1 - first : 31);
            const char* src = reinterpret_cast<const char*>(p.q + (int64_t)b * p.q_bs + (int64_t)h * p.q_hs + first * D);
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int row = (l & 15) + 16 * r;
                const unsigned off = (unsigned)((row < last ? row : last) * (D * 2) + ((l >> 4) & 1) * 32 + (l >> 5) * 16);
#pragma unroll
                for (int kk = r; kk < NKK; kk += 2) qf[i][kk] = *reinterpret_cast<const bf16x8*>(src + off + (kk & ~1) * 32);
            }
        };
        // Makes `it` the item to come.  First its K tiles and half of its Q (all that finds registers beside the last
        // matrix phase of the item before), then, when nobody reads V any more, its V tiles and the rest.
        auto begin = [&](int it) __attribute__((always_inline)) {
            KernelArgs& p = args_here();
            int b, h;
            int64_t row0;
            place(p, it, b, h, row0);
            kp = p.k + (int64_t)b * p.kv_bs + (int64_t)h * p.kv_hs;
            vp = p.v + (int64_t)b * p.kv_bs + (int64_t)h * p.kv_hs;
            load_q(std::integral_constant<int, 0>{}, p, b, h, row0);
#pragma unroll
            for (int j = 0; j <= P; ++j) issue(kp, false, j, j);
        };
        auto begin_rest = [&](int it) __attribute__((always_inline)) {
            KernelArgs& p = args_here();
            int b, h;
            int64_t row0;
            place(p, it, b, h, row0);
            load_q(std::integral_constant<int, 1>{}, p, b, h, row0);
#pragma unroll
            for (int j = 0; j < P; ++j) issue(vp, true, j, j);
        };
        auto arrange_q = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int kk = 0; kk < NKK; kk += 2) {
                    u32x4 x = __builtin_bit_cast(u32x4, qf[i][kk]), y = __builtin_bit_cast(u32x4, qf[i][kk + 1]);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const auto r = __builtin_amdgcn_permlane16_swap(x[j], y[j], false, false);
                        x[j] = r[0];
                        y[j] = r[1];
                    }
                    qf[i][kk] = __builtin_bit_cast(bf16x8, x);
                    qf[i][kk + 1] = __builtin_bit_cast(bf16x8, y);
                }
        };

        begin(item);
        begin_rest(item);
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
        while (item < n_wide && n_redo + 2 <= kRedoMax) {
            float neg_mc[2], l_run[2] = {0.f, 0.f}, ls0[2] = {0.f, 0.f}, ls1[2] = {0.f, 0.f};
            f32x16 o[2][NDB], s[2];
            unsigned pk[2][2][4];
            bf16x8 frag[4];
            float zero_o = 0.f;
            asm volatile("" : "+v"(zero_o));
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int db = 0; db < NDB; ++db)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[i][db][r] = zero_o;
            const f32x16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
            // the loads of Q and the first tiles precede the stores of the item before
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int kk = 0; kk < NKK; ++kk) asm volatile("" : "+v"(qf[i][kk]));
            wait_vmcnt<kStores>();
            arrange_q();
            barrier();

            // ---- reference: the row max over the first 64 keys
            {
                float m[2] = {-INFINITY, -INFINITY};
                static_for<0, 2>([&](auto j) {
                    constexpr int off = K_BASE + (1 - decltype(j)::value) * TILE;
                    static_for<0, NKK>([&](auto kk) {
                        const bf16x8 a = k_frag(k_at, std::integral_constant<int, off>{}, kk);
#pragma unroll
                        for (int i = 0; i < 2; ++i) s[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[i][decltype(kk)::value], decltype(kk)::value == 0 ? zero : s[i], 0, 0, 0);
                    });
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int r = 0; r < 16; ++r) m[i] = fmaxf(m[i], s[i][r]);
                });
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    neg_mc[i] = -(pair_max(m[i]) * c);
                    asm volatile("" : "+v"(neg_mc[i]));          // one register: not the positive value as well, for the lse
                }
            }
            if (second) barrier();

            constexpr std::false_type no{};
            constexpr std::true_type yes{};
            constexpr std::integral_constant<int, 0> I0{};
            constexpr std::integral_constant<int, 1> I1{};
            constexpr std::integral_constant<int, 2> I2{};
            constexpr std::integral_constant<int, 3> I3{};
            // ---- fragments of the matrix phase behind step t: PV(t) from V at v_off, then QK(t+1) from K at k_off
            constexpr int N_PV = 2 * NDB, N_FR = N_PV + NKK, PF = 3;
            auto load_frag = [&](auto idx, unsigned ka, unsigned va, auto k_off, auto v_off, auto last) __attribute__((always_inline)) {
                constexpr int i = decltype(idx)::value;
                if constexpr (i < N_PV)
                    frag[i % 4] = v_frag(va, std::integral_constant<int, decltype(v_off)::value + (i / NDB) * 16 * (D * 2)>{}, std::integral_constant<int, i % NDB>{});
                else if constexpr (i < N_FR && !decltype(last)::value)
                    frag[i % 4] = k_frag(ka, k_off, std::integral_constant<int, i - N_PV>{});
            };
            auto matrix_head = [&](unsigned ka, unsigned va, auto k_off, auto v_off, auto last) __attribute__((always_inline)) {
                static_for<0, PF>([&](auto i) {
                    load_frag(i, ka, va, k_off, v_off, last);
                    __builtin_amdgcn_sched_barrier(0);
                });
            };
            // Base 2: the scores start from minus the reference, not from zero.  There are registers for that only as P dies:
            // the first block's are set in the second half of PV, the second block's during the first two products
            // of the first block.  Ordinary moves, each anchored by an empty statement: a VALU write needs two wait states before
            // an MFMA that reads the register, and the compiler inserts none behind a move written in assembly.
            auto seed = [&](auto b_c, auto lo, auto hi) __attribute__((always_inline)) {
                static_for<decltype(lo)::value, decltype(hi)::value>([&](auto r) {
                    float x = neg_mc[decltype(b_c)::value];
                    asm volatile("" : "+v"(x));
                    s[decltype(b_c)::value][decltype(r)::value] = x;
                });
            };
            auto pv_mfma = [&](auto idx, auto b_c) __attribute__((always_inline)) {
                constexpr int i = decltype(idx)::value, b = decltype(b_c)::value;
                const u32x4 pv = {pk[b][i / NDB][0], pk[b][i / NDB][1], pk[b][i / NDB][2], pk[b][i / NDB][3]};
                o[b][i % NDB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[i % 4], __builtin_bit_cast(bf16x8, pv), o[b][i % NDB], 0, 0, 0);
            };
            auto qk_mfma = [&](auto idx, auto b_c, auto seeded) __attribute__((always_inline)) {
                constexpr int i = decltype(idx)::value, b = decltype(b_c)::value;
                s[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[i % 4], qf[b][i - N_PV], i == N_PV && !decltype(seeded)::value ? zero : s[b], 0, 0, 0);
            };
            auto matrix_phase = [&](unsigned ka, unsigned va, auto k_off, auto v_off, auto last, auto seeded) __attribute__((always_inline)) {
                constexpr bool LAST = decltype(last)::value, SEEDED = decltype(seeded)::value;
                auto fetch = [&](auto idx) __attribute__((always_inline)) {
                    load_frag(std::integral_constant<int, decltype(idx)::value + PF>{}, ka, va, k_off, v_off, last);
                    __builtin_amdgcn_sched_barrier(0);
                };
                __builtin_amdgcn_s_setprio(1);
                static_for<0, N_PV>([&](auto idx) {
                    constexpr int i = decltype(idx)::value;
                    pv_mfma(idx, I0);
                    fetch(idx);
                    if constexpr (SEEDED && i >= NDB) seed(I0, std::integral_constant<int, (i - NDB) * 16 / NDB>{}, std::integral_constant<int, (i - NDB + 1) * 16 / NDB>{});
                    pv_mfma(idx, I1);
                    __builtin_amdgcn_sched_barrier(0);
                });
                if constexpr (!LAST) {
                    constexpr std::integral_constant<int, N_PV> K0{};
                    constexpr std::integral_constant<int, N_PV + 1> K1{};
                    if constexpr (SEEDED) {
                        qk_mfma(K0, I0, seeded);
                        fetch(K0);
                        seed(I1, I0, std::integral_constant<int, 8>{});
                        __builtin_amdgcn_sched_barrier(0);
                        qk_mfma(K1, I0, seeded);
                        seed(I1, std::integral_constant<int, 8>{}, std::integral_constant<int, 16>{});
                        __builtin_amdgcn_sched_barrier(0);
                        qk_mfma(K0, I1, seeded);
                        fetch(K1);                   // takes the place of the first fragment
                        qk_mfma(K1, I1, seeded);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    static_for<N_PV + (SEEDED ? 2 : 0), N_FR>([&](auto idx) {
                        qk_mfma(idx, I0, seeded);
                        fetch(idx);
                        qk_mfma(idx, I1, seeded);
                        __builtin_amdgcn_sched_barrier(0);
                    });
                }
                __builtin_amdgcn_s_setprio(0);
            };
            // FIRST: a step of the first 64 keys (base 2: their scores are not seeded with the reference)
            auto softmax = [&](auto first) __attribute__((always_inline)) {
#pragma unroll
                for (int r = 0; r < 16; r += 2)
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        float x = s[b][r], y = s[b][r + 1];
                        if constexpr (!BASE2) {
                            x = __builtin_fmaf(x, c, neg_mc[b]);
                            y = __builtin_fmaf(y, c, neg_mc[b]);
                        } else if constexpr (decltype(first)::value) {
                            x += neg_mc[b];
                            y += neg_mc[b];
                        }
                        x = __builtin_amdgcn_exp2f(x);
                        y = __builtin_amdgcn_exp2f(y);
                        ls0[b] += x;
                        ls1[b] += y;
                        pk[b][r / 8][(r % 8) / 2] = pack_bf16(x, y);
                    }
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(pk[b][u][j]));
            };
            auto fold_sum = [&]() __attribute__((always_inline)) {           // the sums of 64 keys
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    l_run[b] += ls0[b] + ls1[b];
                    ls0[b] = ls1[b] = 0.f;
                }
            };
            const __bf16* k_dma = kp + (1 + P) * KEYS * D;
            const __bf16* v_dma = vp + P * KEYS * D;
            // step t, t % 4 == TB, whose fetches are whole tiles; NTH: 0, 1 the steps of the first 64 keys, 2 any other
            auto step = [&](auto tb_c, auto nth) __attribute__((always_inline)) {
                constexpr int TB = decltype(tb_c)::value, NTH = decltype(nth)::value;
                constexpr std::integral_constant<int, ((TB + 1) % R) * TILE> k_off{};
                constexpr std::integral_constant<int, (TB % R) * TILE> v_off{};
                if (D == 128 || !second) lds_dma16_at<K_BASE + ((TB + 1 + P) % R) * TILE>(k_dma, ld_k, dma_base);
                if (D == 128 || second) lds_dma16_at<V_BASE + ((TB + P) % R) * TILE>(v_dma, ld_v, dma_base);
                k_dma += KEYS * D;
                v_dma += KEYS * D;
                softmax(std::integral_constant<bool, NTH < 2>{});
                if constexpr (TB & 1) fold_sum();
                matrix_head(k_at, v_at, k_off, v_off, no);
                wait_vmcnt<LPI * (P - 1)>();             // K tile t+2, V tile t+1
                barrier();
                matrix_phase(k_at, v_at, k_off, v_off, no, std::integral_constant<bool, BASE2 && (NTH > 0)>{});
                barrier();
            };
            int t = 0;
            const int whole = n_v / KEYS;
            if constexpr (BASE2) {
                step(I0, I0);
                step(I1, I1);
                step(I2, I2);
                step(I3, I2);
                t = 4;
            }
            for (; t + 4 + P < whole; t += 4) {
                step(I0, I2);
                step(I1, I2);
                step(I2, I2);
                step(I3, I2);
            }
            // the last few steps: ragged tiles, nothing fetched beyond the end, operand addresses moved to the buffers
            int claimed = 0;
            for (; t < nt - 1; ++t) {
                const bool more_k = t + 1 + P < nt, more_v = t + P < nt;
                if (more_k) issue(kp, false, (t + 1 + P) % R, t + 1 + P);
                if (more_v) issue(vp, true, (t + P) % R, t + P);
                if (t == nt - 3 && !direct && wave == 0 && fresh_lane() == 0) {
                    int lane0 = 0;
                    asm volatile("" : "+v"(lane0));
                    claimed = __hip_atomic_fetch_add((GLOBAL_PTR(int))args_here().counter + lane0, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                softmax(no);
                if (t & 1) fold_sum();
                const unsigned ka = k_at + ((t + 1) % R) * TILE, va = v_at + (t % R) * TILE;
                matrix_head(ka, va, I0, I0, no);
                if (more_k) wait_vmcnt<LPI * (P - 1)>(); else wait_vmcnt<0>();
                if (t == nt - 2 && !direct && wave == 0 && fresh_lane() == 0) {
                    w_next = (int)gridDim.x + claimed;
                    lds_done();
                }
                barrier();
                matrix_phase(ka, va, I0, I0, no, std::integral_constant<bool, BASE2>{});
                barrier();
            }
            asm volatile("" :: "v"(claimed));
            // last step: hidden keys, no further scores
            if (nt * KEYS > n_v) {
                const int hidden = n_v - (nt - 1) * KEYS - 4 * (fresh_lane() >> 5);      // key 4 lh + x is hidden if x >= this
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if ((r >> 2) * 8 + (r & 3) >= hidden) s[0][r] = s[1][r] = -INFINITY;
            }
            softmax(no);
            fold_sum();
            asm volatile("" : "+v"(l_run[0]), "+v"(l_run[1]));         // (otherwise the sums would be taken behind the matrix phase)
            {
                const unsigned va = v_at + (t % R) * TILE;
                matrix_head(0, va, I0, I0, yes);
                barrier();
                const int now = item;
                item = direct ? 0x7fffffff : __builtin_amdgcn_readfirstlane(w_next);
                if (item < n_wide) begin(item);          // Q is used up, and nobody reads K any more
                matrix_phase(0, va, I0, I0, yes, no);
                if (!second) barrier();

                // ---- rows whose sum or accumulators left the safe range: their tiles are swept again by the other items' code
                unsigned bad_rows[2];                      // of this wavefront's two blocks
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    float x = 0.f;
#pragma unroll
                    for (int db = 0; db < NDB; ++db)
#pragma unroll
                        for (int r = 0; r < 16; ++r) x = __builtin_fmaf(o[i][db][r], 0.0f, x);
                    const bool bad = !(pair_sum(l_run[i]) < 1.8446744e19f) || !(x == 0.f);
                    const uint64_t lanes = __builtin_amdgcn_ballot_w64(bad);      // lanes l and l + 32 hold one row
                    bad_rows[i] = (unsigned)lanes | (unsigned)(lanes >> 32);
                }
                if (fresh_lane() == 0) w_flag[wave] = (bad_rows[0] | bad_rows[1]) != 0;
                lds_done();
                barrier();                                 // and every wavefront is done with V
                int bad_tile[2] = {0, 0};
#pragma unroll
                for (int w = 0; w < 8; ++w) bad_tile[w / 4] |= w_flag[w];
                KernelArgs& p = args_here();
                int b, h;
                int64_t row0;
                place(p, now, b, h, row0);
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (__builtin_amdgcn_readfirstlane(bad_tile[i])) {
                        if (wave == 0 && fresh_lane() == 0) w_redo[n_redo] = (b * p.Hg + h) * p.tiles_per_head + (int)((row0 - wave * 64) / kTileRows) + i;
                        if (wave / 4 == i && fresh_lane() == 0) {
                            w_rows[n_redo][wave % 4 * 2] = bad_rows[0];
                            w_rows[n_redo][wave % 4 * 2 + 1] = bad_rows[1];
                        }
                        ++n_redo;
                    }
                if (item < n_wide) begin_rest(item);

                // ---- normalise and store, 64 bytes of 16 rows per store; rows beyond Sq fall to the bounds check
                const int l = fresh_lane(), l16 = l & 15, r16 = (l >> 4) & 1, half = l >> 5;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int64_t first = row0 + 32 * i, left = p.Sq - first;
                    const int rows = left < 0 ? 0 : (left < 32 ? (int)left : 32);
                    const float l_tot = pair_sum(l_run[i]), inv = 1.0f / l_tot;
                    constexpr int row_bytes = D * (OUT16 ? 2 : 4);
                    char* out = reinterpret_cast<char*>(p.out) + ((int64_t)b * p.o_bs + (int64_t)h * p.o_hs + first * D) * (OUT16 ? 2 : 4);
                    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(out, 0, rows * row_bytes, kRawBuffer);
                    const int base = l16 * row_bytes + r16 * 32 + half * 16;
                    auto store = [&](const u32x4 (&v2)[2], int at) __attribute__((always_inline)) {
                        __builtin_amdgcn_raw_buffer_store_b128(v2[0], rsrc, base + at, 0, 0);
                        __builtin_amdgcn_raw_buffer_store_b128(v2[1], rsrc, base + 16 * row_bytes + at, 0, 0);
                    };
#pragma unroll
                    for (int db = 0; db < NDB; ++db) {
                        if constexpr (!OUT16) {
#pragma unroll
                            for (int m = 0; m < 2; ++m) {
                                u32x4 y[2];
#pragma unroll
                                for (int j = 0; j < 4; ++j) {
                                    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(o[i][db][8 * m + j] * inv),
                                                                                    __float_as_uint(o[i][db][8 * m + 4 + j] * inv), false, false);
                                    y[0][j] = r[0];
                                    y[1][j] = r[1];
                                }
                                store(y, db * 128 + m * 64);
                            }
                        } else {
                            u32x4 y[2], z[2];
#pragma unroll
                            for (int m = 0; m < 2; ++m)          // 16 columns: the halves exchange their inner 4
#pragma unroll
                                for (int j = 0; j < 2; ++j) {
                                    const unsigned a0 = pack_bf16(o[i][db][8 * m + 2 * j] * inv, o[i][db][8 * m + 2 * j + 1] * inv);
                                    const unsigned a1 = pack_bf16(o[i][db][8 * m + 4 + 2 * j] * inv, o[i][db][8 * m + 5 + 2 * j] * inv);
                                    const auto r = __builtin_amdgcn_permlane32_swap(a0, a1, false, false);
                                    z[m][j] = r[0];
                                    z[m][2 + j] = r[1];
                                }
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                const auto r = __builtin_amdgcn_permlane16_swap(z[0][j], z[1][j], false, false);
                                y[0][j] = r[0];
                                y[1][j] = r[1];
                            }
                            store(y, db * 64);
                        }
                    }
                    const auto lse_rsrc = __builtin_amdgcn_make_buffer_rsrc(p.lse + (int64_t)b * p.l_bs + (int64_t)h * p.l_hs + first, 0, rows * 4, kRawBuffer);
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(-neg_mc[i] * 0.6931471805599453f + __logf(l_tot)), lse_rsrc,
                                                          half == 0 ? (l & 31) * 4 : 1 << 30, 0, 0);
                }
            }
        }
    }

    // ---- the other units of the launch; first the tiles given back, and the wide items of a workgroup whose list was full
    __builtin_amdgcn_s_waitcnt(kWaitVm0);                      // no load into LDS and no store of a tile given back is under way
    lds_done();
    barrier();                                                 // w_redo and w_rows are written, LDS is free
    bool swept = true;                                         // the tiles of the list lack the running-max sweep only
    for (bool more = true; more;) {
        KernelArgs& p = args_here();
        int wave_here = wave;                                  // opaque: scalar registers would be taken up from here on by what is formed from it
        asm volatile("" : "+s"(wave_here));
        int unit, end = 0x7fffffff;
        unsigned again = 0;
        if (n_redo > 0) {
            unit = p.n_items + __builtin_amdgcn_readfirstlane(w_redo[--n_redo]);
            again = __builtin_amdgcn_readfirstlane(w_rows[n_redo][wave_here]);
        } else if (item < n_wide) {
            if (wave == 0 && fresh_lane() == 0) {
                const int pairs_per_head = p.tiles_per_head >> 1, bh = item / pairs_per_head;
                w_redo[0] = bh * p.tiles_per_head + 2 * (item - bh * pairs_per_head);
                w_redo[1] = w_redo[0] + 1;
                w_next = direct ? 0x7fffffff : (int)gridDim.x + __hip_atomic_fetch_add((GLOBAL_PTR(int))p.counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            lds_done();
            barrier();
            n_redo = 2;
            swept = false;
            item = __builtin_amdgcn_readfirstlane(w_next);
            continue;
        } else {
            more = swept = false;
            unit = item < 0x7fffffff - n_wide ? item + n_wide : item;
            end = p.n_items;
        }
        if (swept && again == 0) fetch_for_sweep<D>(p, unit - p.n_items, wave_here);
        else sp_items<D, 8, BASE2, OUT16, true>(p, unit, end, direct || more, wave_here, swept, again);
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
        lds_done();
        barrier();
    }
    if (!direct && wave == 0 && fresh_lane() == 0) reset_counter(args_here());
}

template <int D, bool BASE2, bool OUT16>
static hipError_t launch_wide(const AttnParams& p, int n_cu, hipStream_t st) {
    auto kern = attn_fwd_wide_kernel<D, BASE2, OUT16>;
    constexpr int smem = 2 * sp_buffers(D, 8) * 64 * D * 2, alone = 96 * 1024, lds = smem > alone ? smem : alone;
    static_assert(2 * Wide<D>::RING * Wide<D>::TILE <= smem, "the other items need more");
    static KernelSetup setup;
    hipError_t e = setup.ensure(reinterpret_cast<const void*>(kern), lds, nullptr);
    if (e != hipSuccess) return e;
    const int items = p.n_items - p.n_wide;
    hipLaunchKernelGGL(kern, dim3((unsigned)(items < n_cu ? items : n_cu)), dim3(512), lds, st, p);
    return hipGetLastError();
}

// Head dimension 64 is compiled by attn_fwd_wide_d64.hip, which includes this file with PDA_SP_HEAD_DIM 64.
template <int D>
static hipError_t launch_wide_form(const AttnParams& p, int n_cu, hipStream_t st) {
    if (p.out_bf16) return launch_wide<D, false, true>(p, n_cu, st);
    return p.base2 ? launch_wide<D, true, false>(p, n_cu, st) : launch_wide<D, false, false>(p, n_cu, st);
}
#ifndef PDA_SP_HEAD_DIM
hipError_t launch_attn_wide_d64(const AttnParams& p, int n_cu, hipStream_t st);

hipError_t launch_attn_wide(const AttnParams& p, int D, int n_cu, hipStream_t st) {
    return D == 64 ? launch_attn_wide_d64(p, n_cu, st) : launch_wide_form<128>(p, n_cu, st);
}
#else
hipError_t launch_attn_wide_d64(const AttnParams& p, int n_cu, hipStream_t st) { return launch_wide_form<64>(p, n_cu, st); }
#endif

}  // namespace pda
