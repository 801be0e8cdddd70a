// Flash-attention forward for launches of few query rows, gfx950, d = 128 and 64 (which launches: attn_internal.h,
// rows_form).
//
// The software-pipelined kernel needs the keys of such a launch cut into ranges to fill the chip, a partial result of
// every range in memory and a second launch that merges them; at 2 x 1 024 rows, d = 64, that was 13.6 us, of which 3 us
// for the merge and most of the rest one wavefront per SIMD walking eight key tiles.  Here a workgroup finishes 32 query
// rows: its KS wavefronts share the keys among them, sweep their shares independently of each other (own LDS tiles, own
// waits, no barrier until the end) and add up their partial results in LDS.  One launch, and nothing in the workspace.
//
// MFMA formulation, operand order and LDS swizzle are those of attn_fwd_sp.hip; tiles of 32 keys, one of K and one of V per
// wavefront: K tile t+1 travels under the softmax and PV of tile t, V tile t+1 under the next QK and softmax.  The
// reference is a running max.  It follows the max over the first eighth of a share, from there on it moves when the max grew by more
// than 2^8: the largest weight of a row is exact, and its rounding to bf16 no part of the error, if it is the reference, and ranges
// of 512 keys and more with the max of 64 as reference have that at most as often (relative error in the 2-norm, 8 x 1 024 on 5 120,
// d = 128, cut in ranges 1.625e-3, reference from 32 keys 1.638e-3, now 1.606e-3; 4 x 1 024: 1.615, 1.635, 1.605).  It starts from the lowest finite value, not from
// -inf: keys that score -inf then weigh 0 also where they are the first of a share (-inf - -inf would make the row NaN).
//
// What bounds it: nothing is saturated.  Every workgroup streams all keys of its head into LDS, 4 d bytes per key.  One block of rows:
// up to 110 GB/s per CU, of the 64 bytes a clock that the vector cache can deliver (a round of workgroups costs 3 us (start, sum,
// stores) and 5.3 us per 1 024 keys at d = 128, half of that at d = 64), against 2 us of MFMA time for 32 rows and 1 024 keys at d = 128.
// Two blocks of 32 rows (NR = 2), each K and V fragment feeding two MFMAs: a round on 2 048 keys takes 25 us, 42 GB/s per CU; in
// three such rounds (24 x 2 048, d = 128, 78 us at 2.2 GHz) the matrix pipe is busy 29 % of the time, the VALU port 40 %, LDS
// 22 %, and wavefronts wait 38 % of theirs: each of them does the products, the softmax and the products of a tile one after the
// other, and there are two per SIMD.  Q is read from LDS beside K there at d = 128 (in registers, 23 of them spilled and a tile
// took 2.4 us instead of 1.2).  When two blocks pay: attn_internal.h, rows_blocks.  KS = 8: two wavefronts per SIMD; d = 64 needs 70 KB of
// LDS, so two workgroups share a CU (16 wavefronts of 32 rows, one workgroup per CU: 8 x 2 048 rows 16.3 -> 20.0 us).
#include <hip/hip_runtime.h>
#include <float.h>
#include <stdint.h>
#include "attn_internal.h"
#include "attn_device.h"

namespace pda {

constexpr int kRows = 32;            // query rows of a block: a workgroup has NR of them
constexpr int kKeys = 32;            // keys of a tile
static_assert(kRows == kKeys, "a wavefront's partial result takes the place of its two tiles");

// LDS of a workgroup: per wavefront a tile of K and one of V (later its partial O in fp32), the rows of Q, and the reference
// and sum of every row and wavefront.
constexpr int rows_smem(int d, int ks, int nr) { return ks * 2 * kKeys * d * 2 + nr * kRows * d * 2 + 2 * ks * kRows * 4; }

template <int D, int KS, int NR>
__global__ __launch_bounds__(64 * KS, 2) void attn_rows_kernel(const AttnParams p) {
    static_assert(D == 128 || D == 64, "head dimension");
    constexpr int G = D / 8;              // 16-byte granules per bf16 row
    constexpr int NKK = D / 16, NDB = D / 32;
    constexpr int TILE = kKeys * D * 2;   // 8 KB or 4 KB
    constexpr int CPT = TILE / 1024;      // DMA chunks of 1 KB per tile
    constexpr int RPC = 1024 / (D * 2);   // rows per chunk
    constexpr int M = NR * kRows;         // query rows of the workgroup
    constexpr int Q_BASE = KS * 2 * TILE, ST_BASE = Q_BASE + NR * TILE;

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 31, lh = lane >> 5;
    const unsigned lds0 = (unsigned)(uintptr_t)(LDS_PTR(const void))smem;

    // Workgroups are dealt to the 8 XCDs round robin; each XCD gets a consecutive range of row blocks, so that few heads
    // pass through its L2.
    const int per = (int)gridDim.x >> 3, extra = (int)gridDim.x & 7, xcd = (int)blockIdx.x & 7;
    const int block = xcd * per + (xcd < extra ? xcd : extra) + ((int)blockIdx.x >> 3);
    const int blocks_per_head = (int)((p.Sq + M - 1) / M);
    const int bh = block / blocks_per_head, heads = p.Hg * p.n_groups;
    const int b = bh / heads, h = bh - b * heads;
    const int64_t row0 = (int64_t)(block - bh * blocks_per_head) * M;
    const int rows = (int)(p.Sq - row0 < M ? p.Sq - row0 : M);
    const char* qp = reinterpret_cast<const char*>(p.q + (int64_t)b * p.q_bs + (int64_t)h * p.q_hs + row0 * D);
    const char* kp = reinterpret_cast<const char*>(p.k + (int64_t)b * p.kv_bs + (int64_t)h * p.kv_hs);
    const char* vp = reinterpret_cast<const char*>(p.v + (int64_t)b * p.kv_bs + (int64_t)h * p.kv_hs);

    // this wavefront's key tiles: none if there are fewer tiles than wavefronts
    const int nt = (int)((p.n_v + kKeys - 1) / kKeys);
    const int t0 = (int)((int64_t)nt * wave / KS), t1 = (int)((int64_t)nt * (wave + 1) / KS);

    // ---- loads into LDS: chunk j of a tile holds rows j RPC .. j RPC + RPC-1, lane -> row lane / G of them, granule position lane % G
    const unsigned lds_k = lds0 + wave * (2 * TILE), lds_v = lds_k + TILE;
    auto granule = [&](int row, bool is_v) __attribute__((always_inline)) {
        return (unsigned)(((lane % G) ^ (is_v ? swz_v<D>(row) : swz_k<D>(row))) * 16);
    };
    unsigned ld_k[CPT], ld_v[CPT];
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
        const int row = j * RPC + lane / G;
        ld_k[j] = row * (D * 2) + granule(row, false);
        ld_v[j] = row * (D * 2) + granule(row, true);
    }
    auto issue = [&](const char* base, bool is_v, unsigned lds, int tile) __attribute__((always_inline)) {
        const char* src = base + (int64_t)tile * TILE;
        const int64_t left = p.n_v - (int64_t)tile * kKeys;
        if (left >= kKeys) {
#pragma unroll
            for (int j = 0; j < CPT; ++j) lds_dma16(src, is_v ? ld_v[j] : ld_k[j], lds + j * 1024);
        } else {                                      // rows clamped to the last valid key: hidden keys are never read
#pragma unroll
            for (int j = 0; j < CPT; ++j) {
                const int row = j * RPC + lane / G;
                lds_dma16(src, (unsigned)(row < (int)left ? row : (int)left - 1) * (D * 2) + granule(row, is_v), lds + j * 1024);
            }
        }
    };
    for (int j = wave; j < NR * CPT; j += KS) {
        const int row = j * RPC + lane / G;
        lds_dma16(qp, (unsigned)(row < rows ? row : rows - 1) * (D * 2) + granule(row, false), lds0 + Q_BASE + j * 1024);
    }
    if (t0 < t1) {
        issue(kp, false, lds_k, t0);
        issue(vp, true, lds_v, t0);
        wait_vmcnt<2 * CPT>();                        // the chunks of Q came first
    } else {
        wait_vmcnt<0>();
    }
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    // ---- operand reads
    auto k_off = [&](int kk) __attribute__((always_inline)) { return li * (D * 2) + (((2 * kk + lh) ^ swz_k<D>(li)) * 16); };
    auto q_frag = [&](int i, int kk) __attribute__((always_inline)) { return *(LDS_PTR(const bf16x8))((LDS_PTR(const unsigned char))smem + Q_BASE + i * TILE + k_off(kk)); };
    bf16x8 qf[NKK];                                   // one block: in registers; two blocks: read with K, there is no room for both
    if constexpr (NR == 1)
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) qf[kk] = q_frag(0, kk);
    LDS_PTR(const unsigned char) my_k = (LDS_PTR(const unsigned char))smem + wave * (2 * TILE);
    LDS_PTR(const unsigned char) my_v = my_k + TILE;
    const int t16 = lane & 15, v_key_in = 4 * lh + (t16 >> 2);
    auto v_frag = [&](int db, int u) __attribute__((always_inline)) {
        const int g = (db * 4 + 2 * (li >> 4) + ((t16 & 3) >> 1)) ^ swz_v<D>(v_key_in);
        LDS_PTR(const unsigned char) at = my_v + (u * 16 + v_key_in) * (D * 2) + g * 16 + (t16 & 1) * 8;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))at);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))(at + 8 * (D * 2)));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto reads_done = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };

    // ---- sweep over the wavefront's keys
    const float c = p.scale_log2e;
    float mc[NR], l_run[NR];                          // reference in exp2 units; the lane's share of the sum
    f32x16 o_acc[NR][NDB];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        mc[i] = -FLT_MAX;
        l_run[i] = 0.f;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) o_acc[i][db][r] = 0.f;
    }

    auto tile = [&](int t, float slack) __attribute__((always_inline)) {       // slack: how far the max may grow without moving it
        wait_vmcnt<CPT>();                            // K tile t is in; V tile t, issued after it, perhaps not
        f32x16 s[NR];
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) {
            const f32x16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
            const bf16x8 a = *(LDS_PTR(const bf16x8))(my_k + k_off(kk));
#pragma unroll
            for (int i = 0; i < NR; ++i)
                s[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, NR == 1 ? qf[kk] : q_frag(i, kk), kk == 0 ? zero : s[i], 0, 0, 0);
        }
        reads_done();
        const bool more = t + 1 < t1;
        if (more) issue(kp, false, lds_k, t + 1);
        if ((int64_t)(t + 1) * kKeys > p.n_v) {
            const int hidden = (int)(p.n_v - (int64_t)t * kKeys) - 4 * lh;      // key 4 lh + x is hidden if x >= this
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if ((r >> 2) * 8 + (r & 3) >= hidden)
#pragma unroll
                    for (int i = 0; i < NR; ++i) s[i][r] = -INFINITY;
        }
        u32x4 pk[NR][2];
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            float m0 = s[i][0], m1 = s[i][1];
#pragma unroll
            for (int r = 2; r < 16; r += 2) {
                m0 = fmaxf(m0, s[i][r]);
                m1 = fmaxf(m1, s[i][r + 1]);
            }
            const float mxc = pair_max(fmaxf(m0, m1)) * c;
            const float mc_new = (mxc - mc[i] > slack) ? mxc : mc[i];
            const float alpha = __builtin_amdgcn_exp2f(mc[i] - mc_new);          // 1 if unmoved, 0 on the first tile
            if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
                for (int db = 0; db < NDB; ++db)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o_acc[i][db][r] *= alpha;
            }
            mc[i] = mc_new;
            float sum0 = 0.f, sum1 = 0.f;
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const float x = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i][r], c, -mc_new));
                const float y = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i][r + 1], c, -mc_new));
                sum0 += x;
                sum1 += y;
                pk[i][r / 8][(r % 8) / 2] = pack_bf16(x, y);
            }
            l_run[i] = __builtin_fmaf(l_run[i], alpha, sum0 + sum1);
        }
        if (more) wait_vmcnt<CPT>();                  // V tile t is in; K tile t+1, issued after it, perhaps not
        else wait_vmcnt<0>();
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int db = 0; db < NDB; ++db) {
                const bf16x8 a = v_frag(db, u);
#pragma unroll
                for (int i = 0; i < NR; ++i)
                    o_acc[i][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8, pk[i][u]), o_acc[i][db], 0, 0, 0);
            }
        reads_done();
        if (more) issue(vp, true, lds_v, t + 1);
    };
    int t = t0;
    if (t1 - t0 > 11)                                 // (a loop of its own: with a varying limit in one, every tile takes 1 to 3 % longer)
        for (const int settled = t0 + (t1 - t0 + 4) / 8; t < settled; ++t) tile(t, 0.f);
    for (; t < t1; ++t) tile(t, 8.f);

    // ---- block by block: partial results into LDS, O where the wavefront's tiles were, 16-byte granules XORed with the row;
    // their sum on a common reference goes out, 16 bytes (8 of bf16) per lane
    constexpr int G4 = D / 4;             // 16-byte granules per fp32 row
    LDS_PTR(unsigned char) part = (LDS_PTR(unsigned char))smem;
    LDS_PTR(float) st_m = (LDS_PTR(float))((LDS_PTR(unsigned char))smem + ST_BASE);
    LDS_PTR(float) st_l = st_m + KS * kRows;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        if (i > 0) {
            if (i * kRows >= rows) break;
            __syncthreads();              // the block before has been read
        }
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const f32x4 x = {o_acc[i][db][4 * a], o_acc[i][db][4 * a + 1], o_acc[i][db][4 * a + 2], o_acc[i][db][4 * a + 3]};
                const int g = (db * 8 + 2 * a + lh) ^ (li % G4);
                *(LDS_PTR(f32x4))(part + wave * (2 * TILE) + li * (D * 4) + g * 16) = x;
            }
        const float l_tot = pair_sum(l_run[i]);
        if (lh == 0) {
            st_m[wave * kRows + li] = l_tot == 0.f ? -INFINITY : mc[i];        // -inf: no keys, or none above -inf
            st_l[wave * kRows + li] = l_tot;
        }
        __syncthreads();
#pragma unroll
        for (int n = tid; n < kRows * G4; n += 64 * KS) {
            const int r = n / G4, g = n % G4, row = i * kRows + r;
            float f[KS], big = -INFINITY, tot = 0.f;
#pragma unroll
            for (int w = 0; w < KS; ++w) {
                f[w] = st_m[w * kRows + r];
                big = fmaxf(big, f[w]);
            }
#pragma unroll
            for (int w = 0; w < KS; ++w) {
                f[w] = __builtin_amdgcn_exp2f(f[w] - big);                    // 0 for a wavefront without keys
                tot = __builtin_fmaf(f[w], st_l[w * kRows + r], tot);
            }
            const float inv = 1.0f / tot;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < KS; ++w) {       // normalised one by one: their plain sum may leave fp32 where the result does not
                const f32x4 x = *(LDS_PTR(const f32x4))(part + w * (2 * TILE) + r * (D * 4) + ((g ^ (r % G4)) * 16));
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] = __builtin_fmaf(f[w] * inv, x[e], acc[e]);
            }
            if (row < rows) {
                const int64_t at = (int64_t)b * p.o_bs + (int64_t)h * p.o_hs + (row0 + row) * D + g * 4;
                if (p.out_bf16)
                    *reinterpret_cast<u32x2*>(reinterpret_cast<__bf16*>(p.out) + at) =
                        u32x2{pack_bf16(acc[0], acc[1]), pack_bf16(acc[2], acc[3])};
                else
                    *reinterpret_cast<f32x4*>(p.out + at) = acc;
                if (g == 0) {                // ln of the mantissa only: the error of the logarithm grows with its value
                    int e;
                    const float f = frexpf(tot, &e);
                    p.lse[(int64_t)b * p.l_bs + (int64_t)h * p.l_hs + row0 + row] =
                        __builtin_fmaf((float)e, 0.6931471805599453f, __builtin_fmaf(big, 0.6931471805599453f, __logf(f)));
                }
            }
        }
    }
}

template <int D, int NR>
static hipError_t launch_rows(const AttnParams& p, int BH, hipStream_t st) {
    constexpr int KS = 8, smem = rows_smem(D, KS, NR);
    auto kern = attn_rows_kernel<D, KS, NR>;
    static KernelSetup setup;
    hipError_t e = setup.ensure(reinterpret_cast<const void*>(kern), smem, nullptr);
    if (e != hipSuccess) return e;
    const int64_t blocks = (p.Sq + NR * kRows - 1) / (NR * kRows) * BH * p.n_groups;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(64 * KS), smem, st, p);
    return hipGetLastError();
}

hipError_t launch_attn_rows(const AttnParams& p, int BH, int D, int n_cu, hipStream_t st) {
    const bool two = rows_blocks((p.Sq + kRows - 1) / kRows * BH * p.n_groups, p.n_v, D, n_cu) == 2;
    if (D == 128) return two ? launch_rows<128, 2>(p, BH, st) : launch_rows<128, 1>(p, BH, st);
    return two ? launch_rows<64, 2>(p, BH, st) : launch_rows<64, 1>(p, BH, st);
}

}  // namespace pda
