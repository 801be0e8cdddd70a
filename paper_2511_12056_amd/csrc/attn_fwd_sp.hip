// Flash-attention forward, software-pipelined schedule for gfx950, d = 128 and 64, 64-key tiles.
// A workgroup of NW wavefronts sweeps 32 NW query rows: eight wavefronts (256 rows, one workgroup per
// CU) or four (128 rows, two per CU); either way two wavefronts share a SIMD.  A wavefront owns 32 rows
// of them.  Two such sub-tiles in one wavefront per SIMD, each K/V fragment feeding two MFMAs,
// were slower: a single wavefront leaves the latencies at the iteration boundary exposed.  (With two wavefronts per SIMD in
// opposite phases they are faster where there are pairs of whole tiles: attn_fwd_wide.hip.)
//
// MFMA formulation and LDS tile layout are those of attn_fwd.hip (S^T = K Q^T, O^T = V^T P^T on
// v_mfma_f32_32x32x16_bf16, one query per lane, XOR-swizzled 16-byte granules).  Schedule: on
// this hardware the matrix pipe is fed through the VALU issue port (an MFMA holds it for 8 of its
// 32 cycles, a plain VALU op for ~4, a transcendental for ~8), and the softmax of a tile needs
// about as much port time as the tile's MFMAs need matrix-pipe time.  Each wavefront therefore
// runs one instruction stream per key tile t that interleaves three independent pieces of work:
//
//     matrix pipe:   PV(t-1)  (O += V_{t-1} P_{t-1})   then   QK(t+1)  (S_{t+1} = K_{t+1} Q^T)
//     VALU:          softmax(t):  S_t -> running max / sum, P_t (bf16)
//     LDS reads:     MFMA operand fragments, issued PF slots ahead of their use
//
// written slot by slot in issue order (a scheduling barrier after every slot keeps that order).
//
// Softmax reference.  The value of softmax does not depend on the reference that is subtracted
// before the exponential, only overflow and underflow do, and fp32 (and bf16, which shares its
// exponent range) leaves a wide margin.  The item is therefore first swept with a FIXED reference per
// row, the max of the row's scores in the first key tile: no max pass, no rescaling of O, weights
// may exceed 1.  If a row's sum ends up beyond 2^64 (some later score lay that far above the
// first tile, or the input held non-finite values), or an output accumulator is not finite (large
// weights times large V entries), the workgroup sweeps the item again with the
// usual running max, where the reference moves only when the max grew by more than 2^8 and O is
// rescaled after the stream in a rare wave-uniform branch; the rows in question take their result
// from that sweep, the others keep theirs.  The row sum is taken with plain fp32
// adds on the unrounded probabilities; the dot-product instructions (v_dot2c_f32_bf16), which
// would sum two rounded ones at a time, occupy the matrix pipe and stall the MFMA stream.
//
// K/V tiles go from global memory straight into LDS (global_load_lds_dwordx4), NBUF buffers per tensor
// (four; two for d = 128 with four wavefronts, so that two workgroups fit the CU's LDS); the main loop is
// unrolled four times so that every buffer offset is an immediate, and runs as long as all tiles that a
// group of four fetches are whole.  What is left goes through one iteration whose operand bases are moved
// instead; it knows the ragged tile, hidden keys and that nothing is fetched beyond the last tile.  The last
// tile has no further scores to compute and carries its own PV.  With one form of iteration for all of it
// (branches in every copy, scores of a tile beyond the end, PV of the last tile by itself) the last three
// iterations of a sweep took 0.3, 0.5 and 1.8 us longer than the others (d = 128, two workgroups per CU), and
// every copy of the loop body was 452 instructions, branches included, instead of 247: 24 x 16 384 on 570
// keys 166 -> 161 us, 24 x 9 600 -1.7 %, 3 x 67 576 -1.1 %, d = 64, 6 x 67 576 -2.7 %.  At the top of iteration t a
// wavefront issues its share of K tile t+NBUF (over K tile t) and V tile t+NBUF-2 (over V tile t-2),
// both last read in iteration t-1; before the barrier that closes the iteration it waits for K tile
// t+2 and V tile t, which iteration t+1 reads: with four buffers all but its two newest batches.
//
// Between items: the next one is claimed in the last iteration but one; its Q fragments and first K tiles are
// fetched under the last iteration, which computes no scores and so needs neither the registers of Q nor the
// buffers of K (before that, together with the stores: 24 x 16 384 on 570 keys 156.7 -> 155.5 us, on 192 keys
// 102 -> 98, 26 x 10 100 on 866 keys 145 -> 143, 24 x 9 600 920 -> 917); its V tiles follow with the stores.
// All CUs pass through it at about the same time: 192 KB of Q and results per CU in 9 us are 5.5 TB/s, so what
// is left of it is mostly HBM time.  Q and the results move in 64-byte pieces, and a sweep does not wait for
// the stores before it (with the claim under the last PV: 24 x 16 384 on 570 keys 174 -> 166 us, 24 x 4 797 in
// bf16 268 -> 261, 24 x 9 600 921 -> 913).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "attn_internal.h"
#include "attn_device.h"

namespace pda {

constexpr int kTileRows = 256;       // query rows of a tile of the launch plan
constexpr int kRawBuffer = 0x00027000;   // buffer descriptor of untyped data (bounds-checked by bytes)
constexpr int kWaitVm0 = 0x0f70;     // s_waitcnt vmcnt(0), the other counters not waited for

// LDS tile buffers per tensor (see the top of the file): four, or two where two workgroups of d = 128
// share a CU's 160 KB.
constexpr int sp_buffers(int d, int n_waves) { return d == 128 && n_waves < 8 ? 2 : 4; }

// Same with the LDS address given as wave-uniform base + compile-time offset.
template <int LDS_OFF>
__device__ __forceinline__ void lds_dma16_at(const void* sbase, unsigned voff, unsigned lds_base) {
    asm volatile("s_add_u32 m0, %0, %1\n\ts_mov_b64 vcc, %3\n\tglobal_load_lds_dwordx4 %2, vcc"
                 :
                 : "s"(lds_base), "n"(LDS_OFF), "v"(voff), "s"(sbase)
                 : "memory", "scc", "m0", "vcc");
}

// The last workgroup to leave puts both counters back to zero for the next launch that uses this
// workspace (launches sharing a workspace are ordered on one stream).  Every workgroup has made
// its last fetch before it counts itself out, so nobody fetches after the reset.
template <class Args>
__device__ __forceinline__ void reset_counter(const Args& p) {
    __threadfence();
    if (atomicAdd(p.counter + 1, 1) == (int)gridDim.x - 1) {
        __hip_atomic_store(p.counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(p.counter + 1, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// The lane's index in its wavefront, in a register that the compiler cannot trace back to an earlier one.
__device__ __forceinline__ int fresh_lane() {
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}

enum class Iter { MAIN, FIRST, TAIL, LAST };      // forms of an iteration of the sweep

// BASE2: the scores are already in units of log2 (the caller folded scale*log2(e) into Q), so the
// weights are 2^(q.k) and the first sweep needs no arithmetic before the exponential at all: the
// score accumulators start from minus the row's reference instead of from zero.
//
// Works off the units of a launch from `item` on (claiming the following ones unless `direct`) until one is not below
// n_items.  AFTER_WIDE: behind the wide items of attn_fwd_wide.hip, which number and leave out units as described there; if
// `swept`, `item` is a single unit that has had its first sweep, of which this wavefront's rows `again` need the second one.
template <int D, int NW, bool BASE2, bool OUT16, bool AFTER_WIDE, class Args>
__device__ __forceinline__ void sp_items(const Args& p, int item, const int n_items, const bool direct, const int wave_in, const bool swept,
                                         const unsigned again) {
    static_assert(D == 128 || D == 64, "head dimension");
    static_assert(NW == 8 || NW == 4, "wavefronts per workgroup");
    constexpr int BN = 64;
    constexpr int M = 32 * NW;            // query rows of an item
    constexpr int SUB = kTileRows / M;    // items per query tile (and key range)
    constexpr int G = D / 8;              // 16-byte granules per row: 16 (d = 128) or 8
    constexpr int NKB = BN / 32;          // 2
    constexpr int NKK = D / 16;           // 8 or 4
    constexpr int NDB = D / 32;           // 4 or 2
    constexpr int TILE = BN * D * 2;      // 16 KB or 8 KB
    constexpr int NBUF = sp_buffers(D, NW);
    constexpr int K_BASE = 0, V_BASE = NBUF * TILE;       // LDS byte offsets
    constexpr int CHUNKS = TILE / 1024;   // DMA chunks of 1 KB per tile: 16 or 8
    constexpr int CPW = CHUNKS / NW;      // per wavefront: 2 (eight wavefronts) or 4 for d = 128, 1 or 2 for d = 64
    constexpr int RPC = 1024 / (D * 2);   // rows per chunk: 4 or 8
    constexpr int kStores = (OUT16 ? 2 : 4) * NDB + 1;    // an item's results take at least this many stores
    static_assert(CPW >= 1, "every wavefront fetches at least one chunk of a tile");

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ int next_item;
    __shared__ int redo_flag[NW];

    // (after wide items from a fresh lane index: formed from the thread's, all that follows would be ahead of those items)
    const int tid = AFTER_WIDE ? fresh_lane() : threadIdx.x;
    const int lane = tid & 63;
    const int wave = AFTER_WIDE ? wave_in : __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 31, lh = lane >> 5;
    // Values formed from the lane index outside the sweep's main path (tail rows, masks, Q rows, store
    // addresses) start from a copy that the compiler cannot trace back: it would otherwise form them
    // once, ahead of the item loop, and carry them in registers that the sweep has no room for.
    auto opaque = [](int x) { asm volatile("" : "+v"(x)); return x; };
    // The one lane that claims items for the workgroup.  (Not by threadIdx.x, which would be a register more to carry:
    // the d = 128 forms have none to spare, and one that spills gives the kernel a private segment.)
    auto leader = [&]() __attribute__((always_inline)) { return wave == 0 && lane == 0; };
    const int64_t Sq = p.Sq;
    const unsigned lds0 = (unsigned)(uintptr_t)(LDS_PTR(const void))smem;

    // Persistent workgroups (one per CU, or two of four wavefronts) take work items in index order: workgroup i starts with item
    // i and fetches the following ones from a device counter.  The chip's XCDs run at persistently
    // different speeds (several percent apart under the power limit) and the hardware deals the
    // workgroups of a grid to them round robin, so a grid with one workgroup per item would end with
    // the slowest XCD while the others idle.  A launch with no more items than workgroups does not
    // touch the counter.

    // ---- work item -> (query tile, head, key range), inside the group of heads blockIdx.y.  Items [0, n_full) are whole tiles; then the
    // cut tiles' key ranges, range-major, so that the items in flight at any time sweep the same keys.
    int tile, part, b, h, q_tile, sub;
    auto decode = [&](int it) __attribute__((always_inline)) {
        sub = SUB == 1 ? 0 : it % SUB;
        it /= SUB;
        tile = it;
        part = 0;
        if (AFTER_WIDE && it >= p.n_items) {
            tile = it - p.n_items;                    // a tile that a wide item has given back
        } else if (AFTER_WIDE && it < 2 * p.n_wide + p.n_odd) {
            tile = (it - 2 * p.n_wide + 1) * p.tiles_per_head - 1;      // the last tile of a head of wide items
        } else if (it >= p.n_full) {
            const int idx = it - p.n_full;
            part = idx / p.n_cut;
            tile = p.n_full + (idx - part * p.n_cut);
        }
        const int bh = tile / p.tiles_per_head;
        q_tile = tile - bh * p.tiles_per_head;
        b = bh / p.Hg;
        h = bh - b * p.Hg + (int)blockIdx.y * p.Hg;
    };

    // ---- tile DMA: wavefront w fetches the 1 KB chunks w, w+NW, ... of a tile (4 key rows each).
    // Lane -> (row, granule to fetch): row j * NW * RPC + wave * RPC + lane / G of chunk j, granule
    // position lane % G.
    auto granule_off = [&](int l, int j, bool is_k) __attribute__((always_inline)) {     // byte offset of the lane's granule inside its row
        const int row = wave * RPC + l / G + j * (NW * RPC);
        return (unsigned)(((l % G) ^ (is_k ? swz_k<D>(row) : swz_v<D>(row))) * 16);
    };
    const __bf16* kp = nullptr;                       // the item's keys and values: n_v >= 1 of them in nt tiles
    const __bf16* vp = nullptr;
    int n_v = 1, nt = 1;
    unsigned ld_k[CPW], ld_v[CPW];                    // per-lane offsets of the wavefront's chunks
#pragma unroll
    for (int j = 0; j < CPW; ++j) {
        const unsigned row_off = (unsigned)(wave * RPC + lane / G + j * (NW * RPC)) * (D * 2);
        ld_k[j] = row_off + granule_off(lane, j, true);
        ld_v[j] = row_off + granule_off(lane, j, false);
    }
    const unsigned dma_base = lds0 + wave * 1024;
    const __bf16* k_dma = nullptr;                    // main loop: K tile t+NBUF and V tile t+NBUF-2 of the coming iteration
    const __bf16* v_dma = nullptr;
    // this wavefront's share (chunks 0..CPW-1) of a tile of K or V, tile < nt
    auto issue_tile = [&](const __bf16* base, bool is_k, unsigned lds_tile, int tile) __attribute__((always_inline)) {
        const __bf16* src = base + (int64_t)tile * BN * D;
        const int rows = n_v - tile * BN;
        if (rows >= BN) {                             // whole tile valid
#pragma unroll
            for (int j = 0; j < CPW; ++j) lds_dma16(src, is_k ? ld_k[j] : ld_v[j], dma_base + lds_tile + j * (NW * 1024));
        } else {                                      // rows clamped to the last valid key: hidden keys are never read
            const int l = opaque(lane);
#pragma unroll
            for (int j = 0; j < CPW; ++j) {
                const int row = wave * RPC + l / G + j * (NW * RPC);
                lds_dma16(src, (unsigned)(row < rows ? row : rows - 1) * (D * 2) + granule_off(l, j, is_k), dma_base + lds_tile + j * (NW * 1024));
            }
        }
    };
    // the tiles an item starts with: K 0..NBUF-1 and V 0..NBUF-3 (every wavefront is done with those buffers)
    auto issue_first_k = [&]() __attribute__((always_inline)) {
        issue_tile(kp, true, K_BASE + 0 * TILE, 0);
        if (nt > 1) issue_tile(kp, true, K_BASE + 1 * TILE, 1);
        if constexpr (NBUF == 4) {
            if (nt > 2) issue_tile(kp, true, K_BASE + 2 * TILE, 2);
            if (nt > 3) issue_tile(kp, true, K_BASE + 3 * TILE, 3);
        }
    };
    auto issue_first_v = [&]() __attribute__((always_inline)) {
        if constexpr (NBUF == 4) {
            issue_tile(vp, false, V_BASE + 0 * TILE, 0);
            if (nt > 1) issue_tile(vp, false, V_BASE + 1 * TILE, 1);
        }
    };

    // ---- Q operand fragments, resident for the whole sweep.  A fragment holds 16 bytes of each of 32 rows
    // in either half of the wavefront; loaded as such, an instruction would touch 32 bytes in each of 32 rows.
    // A pair (kk, kk + 1) is loaded as 64 bytes of each of 16 rows instead, rows 0-15 and then 16-31.
    bf16x8 qf[NKK];
    // Makes `it` the item to come: its key range [kv0, kv1) (tile aligned; all keys, or range `part` of a
    // cut tile), its Q fragments and first K tiles on their way (issue_first_v is left to the caller).
    auto begin_item = [&](int it) __attribute__((always_inline)) {
        decode(it);
        int64_t kv0 = 0, kv1 = p.n_v;
        if (p.split > 1 && tile >= p.n_full) {
            kv0 = p.part_off[part];
            kv1 = p.part_off[part + 1];
        }
        const __bf16* __restrict__ qp = p.q + (int64_t)b * p.q_bs + (int64_t)h * p.q_hs;
        kp = p.k + (int64_t)b * p.kv_bs + (int64_t)h * p.kv_hs + kv0 * D;
        vp = p.v + (int64_t)b * p.kv_bs + (int64_t)h * p.kv_hs + kv0 * D;
        n_v = (int)(kv1 - kv0);
        nt = (n_v + BN - 1) / BN;
        const int l = opaque(lane);
        int64_t row0 = (int64_t)q_tile * kTileRows + sub * M + wave * 32;      // rows beyond the last one: the last one again
        row0 = row0 < Sq ? row0 : Sq - 1;
        const int last = (int)(Sq - 1 - row0 < 31 ? Sq - 1 - row0 : 31);
        // scalar base and 32-bit offset: 64-bit addresses per lane were two registers too many (base 2, four wavefronts)
        const char* src = reinterpret_cast<const char*>(qp + row0 * D);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int row = (l & 15) + 16 * r;
            const unsigned off = (unsigned)((row < last ? row : last) * (D * 2) + ((l >> 4) & 1) * 32 + (l >> 5) * 16);
#pragma unroll
            for (int kk = r; kk < NKK; kk += 2) qf[kk] = *reinterpret_cast<const bf16x8*>(src + off + (kk & ~1) * 32);
        }
        issue_first_k();
    };
    // Once the loads have arrived: 16-lane rows of each pair trade places, which puts the fragments into MFMA order.
    auto arrange_q = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < NKK; kk += 2) {
            u32x4 x = __builtin_bit_cast(u32x4, qf[kk]), y = __builtin_bit_cast(u32x4, qf[kk + 1]);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const auto r = __builtin_amdgcn_permlane16_swap(x[j], y[j], false, false);
                x[j] = r[0];
                y[j] = r[1];
            }
            qf[kk] = __builtin_bit_cast(bf16x8, x);
            qf[kk + 1] = __builtin_bit_cast(bf16x8, y);
        }
    };

    // ---- per-lane LDS operand addresses (loop invariant; buffer and block offsets are immediates)
    // K operand: row kb*32+li, granule (2kk+lh) ^ swz_k(li)
    LDS_PTR(const unsigned char) k_ptr[NKK];
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) k_ptr[kk] = (LDS_PTR(const unsigned char))smem + (K_BASE + li * (D * 2) + (((2 * kk + lh) ^ swz_k<D>(li)) * 16));
    // V^T operand through the transposing read: within a 16-lane block, lane t supplies the address
    // of 4 consecutive columns (t%4) of key row (t/4) and receives column t of those 4 rows.
    const int t16 = lane & 15;
    const int v_key_in = 4 * lh + (t16 >> 2);                  // key inside a 16-key group (first 4-key read)
    LDS_PTR(const unsigned char) v_ptr[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
        const int g = (db * 4 + 2 * (li >> 4) + ((t16 & 3) >> 1)) ^ swz_v<D>(v_key_in);
        v_ptr[db] = (LDS_PTR(const unsigned char))smem + (V_BASE + v_key_in * (D * 2) + g * 16 + (t16 & 1) * 8);
    }
    // 16 keys of the 32 columns of block db, from byte offset off of the V tile on
    auto v_frag = [&](int db, int off) __attribute__((always_inline)) {
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))(v_ptr[db] + off));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))(v_ptr[db] + off + 8 * (D * 2)));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };

    // The item after this one, claimed by one lane, and whether its Q and K are on their way.
    int next = n_items;
    bool begun = false;
    auto claim = [&]() __attribute__((always_inline)) {
        int lane0 = 0;                   // a lane's own address: for a uniform one the compiler would broadcast the answer at once
        asm volatile("" : "+v"(lane0));
        return __hip_atomic_fetch_add((GLOBAL_PTR(int))p.counter + lane0, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto publish = [&](int claimed) __attribute__((always_inline)) { next_item = (int)gridDim.x + claimed + (AFTER_WIDE ? p.n_wide : 0); };
    float mc_run, l_run;     // reference max in exp2 units (max * scale * log2 e), lane's share of the running sum
    f32x16 o_acc[NDB];
    f32x16 nref;                         // BASE2, first sweep: minus the row's reference, as an accumulator seed
    f32x16 s_a[NKB], s_b[NKB];           // scores of two consecutive tiles, alternating roles
    // Packed bf16 P (MFMA operand order).  One buffer serves two consecutive tiles: group (kb,u) of
    // tile t-1 is consumed by the PV MFMAs of slots (d/32)(2kb+u) .. +d/32-1, before the softmax of tile t writes it.
    unsigned p_io[NKB][2][4];
    const float c = BASE2 ? 1.0f : p.scale_log2e;   // > 0 (the host substitutes a tiny positive value for scale 0)

    auto mask_tail = [&](f32x16 (&s)[NKB], int t) __attribute__((always_inline)) {
        const int hidden = n_v - t * BN - 4 * (opaque(lane) >> 5);      // key 4 lh + x is hidden if x >= this
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if (kb * 32 + (r >> 2) * 8 + (r & 3) >= hidden) {
                    s[kb][r] = -INFINITY;
                }
            }
    };
    // The operand bases normally point at buffer 0; a tail moves them to the buffer it reads.
    int k_at = 0, v_at = 0;
    auto move_k = [&](int off) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) k_ptr[kk] += off - k_at;
        k_at = off;
    };
    auto move_v = [&](int off) __attribute__((always_inline)) {
#pragma unroll
        for (int db = 0; db < NDB; ++db) v_ptr[db] += off - v_at;
        v_at = off;
    };
    // rescales O if some lane moved its reference (rare after the first tiles)
    auto rescale = [&](float alpha) __attribute__((always_inline)) {
        if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) o_acc[db][r] *= alpha;
        }
    };
    auto barrier = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
    };

    // One sweep over the item's keys.  SAFE = false (first attempt): the reference of a row is the
    // max of its scores in the first key tile and never moves, so the loop carries no max pass and
    // no rescaling; probabilities may exceed 1.  That is exact as long as nothing overflows, which
    // the caller of the sweep checks on the row sums.  SAFE = true: running max with lazy updates.
    auto sweep = [&](auto safe_c) __attribute__((always_inline)) {
        constexpr bool SAFE = decltype(safe_c)::value;
        // opaque operand bases: each buffer and block offset stays the immediate of its read instead of
        // becoming a further address that is carried through the loop
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) asm volatile("" : "+v"(k_ptr[kk]));
#pragma unroll
        for (int db = 0; db < NDB; ++db) asm volatile("" : "+v"(v_ptr[db]));
        mc_run = -INFINITY;
        l_run = 0.f;
        // (an opaque zero: the compiler would keep a register vector of constant zeros for all items)
        float zero_o = 0.f;
        asm volatile("" : "+v"(zero_o));
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) o_acc[db][r] = zero_o;
        k_dma = kp + (1 + NBUF) * BN * D;
        v_dma = vp + (NBUF - 1) * BN * D;
        // The Q fragments (resident for both sweeps) and the item's first tiles have arrived.  They were
        // requested before the previous item's stores, which need not have reached memory.
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) asm volatile("" : "+v"(qf[kk]));
        if constexpr (SAFE) wait_vmcnt<0>(); else { wait_vmcnt<kStores>(); arrange_q(); }
        barrier();

        // ---- S_0 = K_0 Q^T (not overlapped with anything)
        {
            const f32x16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int kk = 0; kk < NKK; ++kk)
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb) {
                    const bf16x8 a = *(LDS_PTR(const bf16x8))(k_ptr[kk] + kb * 32 * (D * 2));
                    s_a[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[kk], kk == 0 ? zero : s_a[kb], 0, 0, 0);
                }
            if (BN > n_v) mask_tail(s_a, 0);
            if constexpr (!SAFE) {
                // fixed reference: the row max over the first key tile (key 0 is always valid)
                float m0 = s_a[0][0], m1 = s_a[0][1];
#pragma unroll
                for (int e = 2; e < 32; e += 2) {
                    m0 = fmaxf(m0, s_a[e / 16][e % 16]);
                    m1 = fmaxf(m1, s_a[(e + 1) / 16][(e + 1) % 16]);
                }
                mc_run = pair_max(fmaxf(m0, m1)) * c;
                if constexpr (BASE2) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) nref[r] = -mc_run;
#pragma unroll
                    for (int e = 0; e < 32; ++e) s_a[e / 16][e % 16] -= mc_run;
                }
            }
        }
        barrier();           // K tile 0 is overwritten by the first DMA of the loop

        int claimed = 0;
        // One iteration; TB = t % 4 fixes every LDS buffer offset at compile time.
        //   s_c: scores of tile t (in, overwritten by its probabilities)   s_n: scores of tile t+1 (out)
        // Slot i (0..N_FR-1; N_FR = 32 for d = 128, 16 for d = 64) = the MFMAs fed by operand fragment
        // i (first the PV fragments, then as many QK fragments), the LDS reads of fragment i+PF, and slice i
        // of the softmax VALU work: slices 0-3 the row max, 4-5 the reference / rescale factors, the others
        // the 32 exponentials with their packing to bf16 and the row sum.
        //   MAIN:  every tile it fetches is whole: running scalar tile pointers, fixed per-lane offsets, LDS
        //          destinations as immediates, no hidden keys
        //   FIRST: t = 0, no PV yet (its slots hold softmax work only)
        //   TAIL:  any t with a tile t+1; operand bases moved to the tiles it reads (TB is not used)
        //   LAST:  t = nt-1 >= 1: no scores are left to compute, PV(t) takes the place of QK(t+1)
        auto iteration = [&](auto tb_c, auto kind_c, int t, f32x16 (&s_c)[NKB], f32x16 (&s_n)[NKB]) {
            constexpr int TB = decltype(tb_c)::value;
            constexpr Iter KIND = decltype(kind_c)::value;
            constexpr bool FIRST = KIND == Iter::FIRST, LAST = KIND == Iter::LAST, MOVED = KIND == Iter::TAIL || LAST;
            constexpr int KN = MOVED ? 0 : (TB + 1) % NBUF;           // buffer of K tile t+1
            constexpr int VP = MOVED ? 0 : (TB + 3) % NBUF;           // buffer of V tile t-1
            // DMA of this iteration: K tile t+NBUF over K tile t, V tile t+NBUF-2 over V tile t-2 (both last
            // read in iteration t-1).
            if constexpr (KIND == Iter::MAIN) {
                constexpr int KD = TB % NBUF, VD = (TB + NBUF - 2) % NBUF;
                static_for<0, CPW>([&](auto jc) {
                    constexpr int j = decltype(jc)::value;
                    lds_dma16_at<K_BASE + KD * TILE + j * (NW * 1024)>(k_dma, ld_k[j], dma_base);
                });
                static_for<0, CPW>([&](auto jc) {
                    constexpr int j = decltype(jc)::value;
                    lds_dma16_at<V_BASE + VD * TILE + j * (NW * 1024)>(v_dma, ld_v[j], dma_base);
                });
                k_dma += BN * D;
                v_dma += BN * D;
            } else {
                if (!LAST && t + NBUF < nt) issue_tile(kp, true, K_BASE + (t % NBUF) * TILE, t + NBUF);
                if (!LAST && t + NBUF - 2 < nt) issue_tile(vp, false, V_BASE + ((t + NBUF - 2) % NBUF) * TILE, t + NBUF - 2);
            }
            // The next item is claimed in the last iteration but one, where the answer has an iteration to arrive.
            if constexpr (KIND == Iter::TAIL && !SAFE)
                if (t == nt - 2 && !direct && leader()) claimed = claim();
            if constexpr (KIND == Iter::TAIL) move_k(((t + 1) % NBUF) * TILE);
            if constexpr (MOVED) move_v(((t - 1) % NBUF) * TILE);
            constexpr int N_PV = NKB * 2 * NDB, N_QK = NKK * NKB, N_FR = N_PV + N_QK;
            constexpr int PF = 3, RING = 4;
            static_assert(N_FR == 32 || N_FR == 16, "slot plan below is written for 64-key tiles and d = 128 or 64");
            static_assert(N_PV == N_QK, "PV fragments of the last tile take the slots of QK fragments");
            bf16x8 frag[RING];

            auto load_frag = [&](auto idx) {
                constexpr int i = decltype(idx)::value;
                if constexpr (i < N_PV && FIRST) {
                } else if constexpr (i < N_PV) {
                    constexpr int kb = i / (2 * NDB), u = (i / NDB) % 2, db = i % NDB;
                    constexpr int off0 = VP * TILE + (kb * 32 + u * 16) * (D * 2);
                    frag[i % RING] = v_frag(db, off0);
                } else if constexpr (i < N_FR && LAST) {
                    constexpr int n = i - N_PV, kb = n / (2 * NDB), u = (n / NDB) % 2, db = n % NDB;
                    constexpr int off0 = (kb * 32 + u * 16) * (D * 2);
                    frag[i % RING] = v_frag(db, off0);
                } else if constexpr (i < N_FR) {
                    constexpr int j = i - N_PV, kk = j / 2, kb = j % 2;
                    frag[i % RING] = *(LDS_PTR(const bf16x8))(k_ptr[kk] + (KN * TILE + kb * 32 * (D * 2)));
                }
            };
            auto do_mfma = [&](auto idx) {
                constexpr int i = decltype(idx)::value;
                if constexpr (i < N_PV && FIRST) {
                } else if constexpr (i < N_PV || LAST) {
                    constexpr int n = i % N_PV, kb = n / (2 * NDB), u = (n / NDB) % 2, db = n % NDB;
                    const u32x4 pv = {p_io[kb][u][0], p_io[kb][u][1], p_io[kb][u][2], p_io[kb][u][3]};
                    o_acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[i % RING], __builtin_bit_cast(bf16x8, pv), o_acc[db], 0, 0, 0);
                } else {
                    constexpr int j = i - N_PV, kk = j / 2, kb = j % 2;
                    if constexpr (kk == 0) {
                        const f32x16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
                        s_n[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[i % RING], qf[kk], (BASE2 && !SAFE) ? nref : zero, 0, 0, 0);
                    } else {
                        s_n[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[i % RING], qf[kk], s_n[kb], 0, 0, 0);
                    }
                }
            };

            // Softmax of tile t, slice by slice (anchored with empty asm statements: pure arithmetic
            // would otherwise drift out of the slot it is written in).
            float mx = s_c[0][0], mx2 = s_c[0][1];
            float mc_new = SAFE ? 0.f : mc_run, alpha = 1.f, lsum = 0.f, lsum2 = 0.f;
            // Elements of the lane's 32 scores handled by exponential slot k (0..NX-1): [e_lo(k), e_lo(k+1)).
            // The work on an element is spread over consecutive slots so that no instruction needs a
            // result produced in its own slot: slot k-1 forms z = s*c - m, slot k takes exp2(z), slot k+1
            // adds it to the row sum and, once both halves of a pair exist, packs the pair to bf16.
            // SAFE: slots 0-3 row max, 4-5 reference and rescale factor, 6.. exponentials.  Otherwise the
            // exponentials start at slot 3 (not earlier: the packed pair q of this tile may replace that of
            // the previous tile only after the PV MFMAs of its group, which come d/32 slots per group in
            // the first half of the slots, have read it).
            // LAST: the exponentials end early enough for PV(t), whose group g of 8 weights comes d/32 slots per
            // group into the second half.
            constexpr int X0 = SAFE ? 6 : 3;
            constexpr int NX = !LAST ? N_FR - X0 : N_FR == 32 ? (SAFE ? 20 : 23) : (SAFE ? 4 : 9);
            auto e_lo = [](int k) constexpr { return k <= 0 ? 0 : (k >= NX ? 32 : k * 32 / NX); };
            static_assert([](auto lo) constexpr {
                for (int k = 0; k < NX; ++k)
                    for (int e = lo(k); e < lo(k + 1); ++e) {
                        const int packed = X0 + k + 1, g = e / 8;           // slot that packs element e of group g
                        if (e % 2 && packed < NDB * g + NDB - 1) return false;                  // PV(t-1) has read the group
                        if (LAST && packed >= N_PV + NDB * g) return false;                     // PV(t) has not
                    }
                return true;
            }(e_lo), "slots of the exponentials");
            auto fma_of = [&](auto kc) {
                constexpr int k = decltype(kc)::value;
                if constexpr (BASE2 && !SAFE) return;             // the MFMA output already is s - reference
                static_for<e_lo(k), e_lo(k + 1)>([&](auto ec) {
                    constexpr int e = decltype(ec)::value;
                    float z = __builtin_fmaf(s_c[e / 16][e % 16], c, -mc_new);
                    asm volatile("" : "+v"(z));
                    s_c[e / 16][e % 16] = z;
                });
            };
            auto exp_of = [&](auto kc) {
                constexpr int k = decltype(kc)::value;
                static_for<e_lo(k), e_lo(k + 1)>([&](auto ec) {
                    constexpr int e = decltype(ec)::value;
                    float pe = __builtin_amdgcn_exp2f(s_c[e / 16][e % 16]);
                    asm volatile("" : "+v"(pe));
                    s_c[e / 16][e % 16] = pe;
                });
            };
            auto sum_pack_of = [&](auto kc) {
                constexpr int k = decltype(kc)::value;
                static_for<e_lo(k), e_lo(k + 1)>([&](auto ec) {
                    constexpr int e = decltype(ec)::value;
                    // row sum with plain adds, two chains (the dot-product instructions would take two
                    // values at a time, but they occupy the matrix pipe and stall the MFMA stream)
                    if constexpr (e % 2 == 0) {
                        lsum += s_c[e / 16][e % 16];
                        asm volatile("" : "+v"(lsum));
                    } else {
                        lsum2 += s_c[e / 16][e % 16];
                        asm volatile("" : "+v"(lsum2));
                        constexpr int q = e / 2, kb = q / 8, u = (q % 8) / 4, j = q % 4;   // pair q = elements 2q, 2q+1
                        unsigned pk = pack_bf16(s_c[kb][8 * u + 2 * j], s_c[kb][8 * u + 2 * j + 1]);
                        asm volatile("" : "+v"(pk));
                        p_io[kb][u][j] = pk;
                    }
                });
            };
            auto valu_slice = [&](auto idx) {
                constexpr int i = decltype(idx)::value;
                if constexpr (SAFE && i < 4) {                          // row max over the lane's 32 scores, two chains
#pragma unroll
                    for (int e = 8 * i; e < 8 * i + 8; e += 4) {
                        mx = fmaxf(fmaxf(mx, s_c[e / 16][e % 16]), s_c[(e + 2) / 16][(e + 2) % 16]);
                        mx2 = fmaxf(fmaxf(mx2, s_c[(e + 1) / 16][(e + 1) % 16]), s_c[(e + 3) / 16][(e + 3) % 16]);
                    }
                } else if constexpr (SAFE && i == 4) {
                    // Move the reference only if the max grew by more than 2^8 (or there is none yet:
                    // -inf gives an infinite difference; a fully hidden tile gives -inf and no move).
                    const float mxc = pair_max(fmaxf(mx, mx2)) * c;
                    mc_new = (mxc - mc_run > 8.0f) ? mxc : mc_run;
                } else if constexpr (SAFE && i == 5) {
                    alpha = __builtin_amdgcn_exp2f(mc_run - mc_new);      // 1 if unmoved, 0 on the first tile
                    fma_of(std::integral_constant<int, 0>{});
                } else if constexpr (!SAFE && i == X0 - 1) {
                    fma_of(std::integral_constant<int, 0>{});
                } else if constexpr (i >= X0) {                         // 32 exponentials over NX slots
                    constexpr int k = i - X0;
                    exp_of(std::integral_constant<int, k>{});
                    fma_of(std::integral_constant<int, k + 1>{});
                    sum_pack_of(std::integral_constant<int, k - 1>{});
                }
            };

            // ================= interleaved region: softmax(t) | PV(t-1), QK(t+1) =================
            // in this order: grouped by base address instead, the second MFMA would wait for six reads
            static_for<0, PF>([&](auto i) {
                load_frag(i);
                __builtin_amdgcn_sched_barrier(0);
            });
            static_for<0, N_FR>([&](auto idx) {
                constexpr int i = decltype(idx)::value;
                // LAST: the fragments from here on are read from V tile t
                if constexpr (LAST && i == (NBUF == 2 ? N_PV : N_PV - PF)) move_v((t % NBUF) * TILE);
                if constexpr (LAST && i == N_PV) {
                    if constexpr (SAFE) rescale(alpha);
                    if constexpr (NBUF == 2) {      // V tile t was fetched in this iteration, then what the next item starts with
                        if (begun && next < n_items) wait_vmcnt<NKK + CPW>();
                        else wait_vmcnt<0>();
                        barrier();
                        static_for<0, PF>([&](auto j) { load_frag(std::integral_constant<int, N_PV + decltype(j)::value>{}); });
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                do_mfma(idx);
                if constexpr (!(LAST && NBUF == 2 && i < N_PV && i + PF >= N_PV)) load_frag(std::integral_constant<int, i + PF>{});
                __builtin_amdgcn_sched_barrier(0);       // the reads go first: they are on the path of slot i + PF
                valu_slice(idx);
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (X0 + NX == N_FR) sum_pack_of(std::integral_constant<int, NX - 1>{});
            if constexpr (SAFE) {
                l_run = __builtin_fmaf(l_run, alpha, lsum + lsum2);
                mc_run = mc_new;
            } else {
                l_run += lsum + lsum2;
            }
            // =====================================================================================

            if constexpr (LAST) return;
            if constexpr (SAFE) rescale(alpha);       // once PV(t-1) is in
            if constexpr (KIND != Iter::MAIN)
                if ((t + 2) * BN > n_v) mask_tail(s_n, t + 1);     // S_{t+1} holds hidden keys

            // Iteration t+1 reads K tile t+2 and V tile t; the last one, t+1 = nt-1, V tiles t and t+1.  With four
            // buffers, what this iteration and the previous one issued may still be in flight (two batches of K and
            // V, in a tail fewer); with two, this iteration issued just the tiles that are wanted.  In the first
            // iteration of four-buffer sweeps all of them came with the item's first tiles.
            if constexpr (NBUF == 2 || KIND == Iter::MAIN) {
                wait_vmcnt<NBUF == 4 ? 4 * CPW : 0>();
            } else if constexpr (KIND == Iter::TAIL) {
                if (nt - t > 4) wait_vmcnt<4 * CPW>();
                else if (nt - t == 4) wait_vmcnt<3 * CPW>();
                else if (nt - t == 3) wait_vmcnt<2 * CPW>();
                else wait_vmcnt<0>();
            }
            if constexpr (KIND == Iter::TAIL && !SAFE)
                if (t == nt - 2 && !direct && leader()) publish(claimed);
            barrier();
        };

        // Tiles 0 .. nt-1: the first and the last peeled off, groups of four (buffer offsets are immediates and the
        // score / probability registers alternate roles without copies) as long as all tiles they fetch are whole,
        // and what is left one at a time.
        auto pin_o = [&]() {       // keeps the zeroed accumulators in registers (a constant would be copied at every exit)
#pragma unroll
            for (int db = 0; db < NDB; ++db) asm volatile("" : "+v"(o_acc[db]));
        };
        auto run = [&](auto tb_c, auto kind_c, int t, f32x16 (&s_c)[NKB], f32x16 (&s_n)[NKB]) __attribute__((always_inline)) {
            iteration(tb_c, kind_c, t, s_c, s_n);
        };
        constexpr std::integral_constant<Iter, Iter::MAIN> MAIN{};
        constexpr std::integral_constant<int, 0> B0{};
        constexpr std::integral_constant<int, 1> B1{};
        constexpr std::integral_constant<int, 2> B2{};
        constexpr std::integral_constant<int, 3> B3{};
        pin_o();
        run(B0, std::integral_constant<Iter, Iter::FIRST>{}, 0, s_a, s_b);
        pin_o();
        int t = 1;
        for (const int whole = n_v / BN; t + NBUF + 4 <= whole; t += 4) {
            run(B1, MAIN, t, s_b, s_a);
            run(B2, MAIN, t + 1, s_a, s_b);
            run(B3, MAIN, t + 2, s_b, s_a);
            run(B0, MAIN, t + 3, s_a, s_b);
        }
        for (; t < nt - 1; ++t) {
            run(B0, std::integral_constant<Iter, Iter::TAIL>{}, t, s_b, s_a);
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) s_b[kb] = s_a[kb];
        }
        asm volatile("" :: "v"(claimed));        // its register is not in flight beyond the tail
        const bool single = nt == 1;
        if constexpr (NBUF == 2)
            if (!single) issue_tile(vp, false, V_BASE + (t % NBUF) * TILE, t);
        begun = !SAFE && !direct && nt >= 3;
        if constexpr (!SAFE) {
            // No scores are left to compute: the registers of Q and the buffers of K are free for the next item.
            if (begun) {
                next = __builtin_amdgcn_readfirstlane(next_item);
                if (next < n_items) begin_item(next);
            } else if (!direct && leader()) {
                publish(claim());
            }
        }
        if (!single) {
            run(B0, std::integral_constant<Iter, Iter::LAST>{}, t, s_b, s_a);
        } else {                    // a single tile: its PV alone
#pragma unroll
            for (int i = 0; i < NKB * 2 * NDB; ++i) {
                const int kb = i / (2 * NDB), u = (i / NDB) % 2, db = i % NDB;
                const bf16x8 av = v_frag(db, (kb * 32 + u * 16) * (D * 2));
                const u32x4 pv = {p_io[kb][u][0], p_io[kb][u][1], p_io[kb][u][2], p_io[kb][u][3]};
                o_acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, __builtin_bit_cast(bf16x8, pv), o_acc[db], 0, 0, 0);
            }
        }
        move_k(0);
        move_v(0);
    };

    // ---- where the results of `item` go: part 0 writes the tile's rows of out/lse; later parts write
    // rows 0..255 of their partial slot.  With a bf16 `out` the merge pass needs fp32 partials of ALL
    // parts of a cut tile, part 0 included.
    float* __restrict__ op;
    float* __restrict__ lp;
    __bf16* __restrict__ oph;
    int64_t row_sub, q_row0;                           // row_sub: subtracted from the global row on store
    bool store_bf16;
    auto locate = [&]() __attribute__((always_inline)) {
        decode(item);
        const bool cut = p.split > 1 && tile >= p.n_full;
        const bool to_ws = part > 0 || (cut && OUT16);
        store_bf16 = OUT16 && !to_ws;
        if (!to_ws) {
            op = p.out + (OUT16 ? 0 : (int64_t)b * p.o_bs + (int64_t)h * p.o_hs);
            lp = p.lse + (int64_t)b * p.l_bs + (int64_t)h * p.l_hs;
            row_sub = 0;
        } else {
            const int64_t slot = (int)blockIdx.y * p.group_slots + (OUT16 ? (tile - p.n_full) * p.split + part
                                                                          : (tile - p.n_full) * (p.split - 1) + (part - 1));
            op = p.part_out + slot * (kTileRows * D);
            lp = p.part_lse + slot * kTileRows;
            row_sub = (int64_t)q_tile * kTileRows;
        }
        oph = reinterpret_cast<__bf16*>(p.out) + (int64_t)b * p.o_bs + (int64_t)h * p.o_hs;
        q_row0 = (int64_t)q_tile * kTileRows + sub * M + wave * 32;
    };
    // ---- epilogue: normalise, write out and lse (rows of the lanes in `mask`).  A lane holds 16-byte pieces
    // of one row; stored as such, an instruction would write 32 bytes in each of 32 rows.  Neighbouring pieces
    // trade places between the 16-lane rows (and, for bf16, the halves) of the wavefront first, so that an
    // instruction writes 64 bytes in each of 16 rows.  Buffer stores: rows beyond Sq and rows outside the mask
    // fall to the bounds check, so no path has fewer than kStores stores and the next sweep can wait for the loads
    // that precede them without waiting for all of the stores.  That takes more than equal branches: of two
    // alternatives the compiler makes two conditional blocks, counts the path through neither, and then waits for all
    // stores but one in front of the first use of Q.  So bf16 results and the fp32 partials of a cut tile share their
    // first 2 NDB stores, with selected contents, and only what fp32 has beyond them is conditional.
    auto store_results = [&](uint64_t mask) __attribute__((always_inline)) {
        const int l = opaque(lane), l16 = l & 15, r16 = (l >> 4) & 1, half = l >> 5;
        const float l_tot = pair_sum(l_run);
        const float inv = 1.0f / l_tot;
        const int64_t left = Sq - q_row0;
        const int rows = left < 0 ? 0 : (left < 32 ? (int)left : 32);
        constexpr int kOutside = 1 << 30;
        const unsigned m32 = (unsigned)mask;
        const bool ok0 = (m32 >> l16) & 1, ok1 = (m32 >> (16 + l16)) & 1;
        const bool bf16 = OUT16 && store_bf16;
        const int row_bytes = D * (bf16 ? 2 : 4);
        char* first = bf16 ? reinterpret_cast<char*>(oph + q_row0 * D) : reinterpret_cast<char*>(op + (q_row0 - row_sub) * D);
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(first, 0, rows * row_bytes, kRawBuffer);
        const int base = l16 * row_bytes + r16 * 32 + half * 16;
        const int off0 = ok0 ? base : kOutside, off1 = ok1 ? base + 16 * row_bytes : kOutside;
        auto store = [&](const u32x4 (&x)[2], int at) __attribute__((always_inline)) {       // 64 bytes of rows 0-15, of rows 16-31
            __builtin_amdgcn_raw_buffer_store_b128(x[0], rsrc, off0 + at, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b128(x[1], rsrc, off1 + at, 0, 0);
        };
        auto fp32 = [&](int db, int m, u32x4 (&x)[2]) __attribute__((always_inline)) {        // 16 of the 32 columns of block db
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(o_acc[db][8 * m + j] * inv),
                                                                __float_as_uint(o_acc[db][8 * m + 4 + j] * inv), false, false);
                x[0][j] = r[0];
                x[1][j] = r[1];
            }
        };
        if constexpr (!OUT16) {
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    u32x4 x[2];
                    fp32(db, m, x);
                    store(x, db * 128 + m * 64);
                }
        } else {
#pragma unroll
            for (int db = 0; db < NDB; ++db) {
                u32x4 x[2], z[2];
                fp32(db, 0, x);
#pragma unroll
                for (int m = 0; m < 2; ++m)          // 16 columns: the halves exchange their inner 4
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const unsigned a = pack_bf16(o_acc[db][8 * m + 2 * j] * inv, o_acc[db][8 * m + 2 * j + 1] * inv);
                        const unsigned b = pack_bf16(o_acc[db][8 * m + 4 + 2 * j] * inv, o_acc[db][8 * m + 5 + 2 * j] * inv);
                        const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
                        z[m][j] = r[0];
                        z[m][2 + j] = r[1];
                    }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const auto r = __builtin_amdgcn_permlane16_swap(z[0][j], z[1][j], false, false);
                    x[0][j] = bf16 ? r[0] : x[0][j];
                    x[1][j] = bf16 ? r[1] : x[1][j];
                }
                store(x, db * (bf16 ? 64 : 128));
            }
            if (!bf16)
#pragma unroll
                for (int db = 0; db < NDB; ++db) {
                    u32x4 x[2];
                    fp32(db, 1, x);
                    store(x, db * 128 + 64);
                }
        }
        const auto lse_rsrc = __builtin_amdgcn_make_buffer_rsrc(lp + (q_row0 - row_sub), 0, rows * 4, kRawBuffer);
        const bool ok = half == 0 && ((m32 >> (l & 31)) & 1);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(mc_run * 0.6931471805599453f + __logf(l_tot)), lse_rsrc,
                                              ok ? (l & 31) * 4 : kOutside, 0, 0);
    };

    if (item < n_items) {
        begin_item(item);
        issue_first_v();
    }
    __builtin_amdgcn_s_waitcnt(kWaitVm0);     // no stores follow the first item's loads
    while (item < n_items) {
    // The next item is claimed as late as possible (the order of the items balances the end of the
    // launch): one iteration before the last, in which its Q and first K tiles travel; V follows with the stores.
    // Sweeps of one or two tiles claim it in the last one and begin it with the stores.
    uint64_t store_mask = ~0ull;                      // lanes whose results are still to be stored
    auto second_sweep = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
        arrange_q();
        sweep(std::true_type{});
        // Q is fetched anew from here.  The compiler does not know it and would keep the old fragments through the
        // last iteration above, up to six registers more than there are.
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) asm volatile("" : "=v"(qf[kk]));
        barrier();                                   // as above, before the next item's tiles are fetched
    };
    int any = 0;
    if (!AFTER_WIDE || !swept) {
        sweep(std::false_type{});
        // A row whose sum left the safe range (a later score exceeded the first tile's max by more
        // than ~2^64, or non-finite input) or whose accumulators are not finite takes its result from a
        // second sweep with the running max (weights <= 2^8 there).  The workgroup sweeps together, but
        // the other rows keep the result of the first sweep: what a row gets depends on that row alone,
        // not on the rows that happen to share its workgroup, whose number depends on the launch.
        bool bad = p.redo_always != 0;               // test switch: every row takes the second sweep
        bad |= !(pair_sum(l_run) < 1.8446744e19f);
        // Weights of up to 2^64 times large finite V entries can overflow the accumulators while the
        // row sum stays in range: inf * 0 and NaN * 0 are NaN, any finite value * 0 is 0.
        float t = 0.f;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) t = __builtin_fmaf(o_acc[db][r], 0.0f, t);
        bad |= !(t == 0.f);
        uint64_t redo = __builtin_amdgcn_ballot_w64(bad);
        redo |= redo << 32 | redo >> 32;             // lanes l and l + 32 hold one row
        if (lane == 0) redo_flag[wave] = redo != 0 ? 1 : 0;
        barrier();                                   // flags are written, and every wavefront is done with the LDS tiles
#pragma unroll
        for (int w = 0; w < NW; ++w) any |= redo_flag[w];
        if (!begun && !direct) next = __builtin_amdgcn_readfirstlane(next_item);
        if (__builtin_expect(__builtin_amdgcn_readfirstlane(any), 0)) {
            locate();
            store_results(~redo);
            store_mask = redo;
            begin_item(item);                        // again: the next one may have taken its place
            issue_first_v();
            if constexpr (!AFTER_WIDE) second_sweep();
        }
    } else {
        store_mask = (uint64_t)again << 32 | again;
        any = 1;
    }
    if constexpr (AFTER_WIDE)
        if (__builtin_expect(__builtin_amdgcn_readfirstlane(any), 0)) second_sweep();      // one copy of it for both ways
    locate();
    if (next < n_items) {
        if (!begun) begin_item(next);
        issue_first_v();
    }
    store_results(store_mask);
    item = next;
    }   // next work item

    if (!AFTER_WIDE && !direct && leader()) reset_counter(p);
}

template <int D, int NW, bool BASE2, bool OUT16>
__global__ __launch_bounds__(64 * NW, 2) void attn_fwd_sp_kernel(const AttnParams p) {
    sp_items<D, NW, BASE2, OUT16, false>(p, (int)blockIdx.x, p.n_items, p.n_items <= (int)gridDim.x, 0, false, 0);
}

#ifndef PDA_SP_DEVICE_ONLY
// Folds the key-range partials of the cut tiles into out/lse (in place): per row,
// L = ln sum_p exp(lse_p), out = sum_p exp(lse_p - L) out_p.  One group of d/4 lanes (half or a
// quarter of a wavefront) per row, so a row's lse is read by all its lanes before one of them
// overwrites it.  Latency bound: N is the number of parts (or the largest one the kernel takes), so that
// the loads of all parts are in flight together (whole calls, one part after the other in a loop -> now: 300
// rows x 40 000 keys, 16 parts, 43.8 -> 40.7 us; 1 x 2 048, d = 128, 4 parts, 18.9 -> 18.0; 2 x 1 024, d = 64,
// 2 parts, 14.4 -> 13.8).
template <int D, int N>
__global__ __launch_bounds__(256) void tail_merge_kernel(const AttnParams p) {
    constexpr int M = 256, LPR = D / 4, RPB = 256 / LPR;      // lanes per row, rows per workgroup
    const int tile = p.n_full + blockIdx.x / (M / RPB);
    const int r_in = (blockIdx.x % (M / RPB)) * RPB + (threadIdx.x / LPR);
    const int c4 = threadIdx.x % LPR;
    const int bh = tile / p.tiles_per_head;
    const int q_tile = tile - bh * p.tiles_per_head;
    const int b = bh / p.Hg, h = bh - b * p.Hg + (int)blockIdx.y * p.Hg;
    const int64_t row = (int64_t)q_tile * M + r_in;
    if (row >= p.Sq) return;
    float* lp = p.lse + (int64_t)b * p.l_bs + (int64_t)h * p.l_hs + row;
    const float* op = p.out + (int64_t)b * p.o_bs + (int64_t)h * p.o_hs + row * D;      // fp32 out only
    // fp32 out: part 0 sits in out/lse and parts 1.. in the workspace; bf16 out: all parts in the workspace
    const int n = N <= 6 ? N : p.split;
    const int n_ws = p.out_bf16 ? n : n - 1;
    const int64_t slot0 = (int)blockIdx.y * p.group_slots + (tile - p.n_full) * n_ws;
    float l[N];
    f32x4 x[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int part = j < n ? j : n - 1;
        const bool in_out = part == 0 && !p.out_bf16;
        const int64_t slot = slot0 + (p.out_bf16 ? part : part - 1);
        const float* xs = in_out ? op : p.part_out + (slot * M + r_in) * D;
        l[j] = *(in_out ? lp : p.part_lse + slot * M + r_in);
        x[j] = reinterpret_cast<const f32x4*>(xs)[c4];
    }
    // one pass with a running reference (the parts of a cut tile are never empty: lse is finite)
    float m = -INFINITY, tot = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < N; ++j) {
        if (j >= n) continue;
        const float m_new = fmaxf(m, l[j]);
        const float a_old = __expf(m - m_new);          // 0 on the first part
        const float w = __expf(l[j] - m_new);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = acc[e] * a_old + w * x[j][e];
        tot = tot * a_old + w;
        m = m_new;
    }
    const float inv = 1.0f / tot;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] *= inv;
    if (p.out_bf16) {
        __bf16* oh = reinterpret_cast<__bf16*>(p.out) + (int64_t)b * p.o_bs + (int64_t)h * p.o_hs + row * D;
        reinterpret_cast<u32x2*>(oh)[c4] = u32x2{pack_bf16(acc[0], acc[1]), pack_bf16(acc[2], acc[3])};
    } else {
        reinterpret_cast<f32x4*>(const_cast<float*>(op))[c4] = acc;
    }
    if (c4 == 0) *lp = m + __logf(tot);
}

template <int D>
static hipError_t launch_tail_merge(const AttnParams& p, hipStream_t st) {
    const dim3 grid((unsigned)(p.n_cut * (kTileRows / (1024 / D))), (unsigned)p.n_groups);
    switch (p.split) {
        case 2: hipLaunchKernelGGL((tail_merge_kernel<D, 2>), grid, dim3(256), 0, st, p); break;
        case 3: hipLaunchKernelGGL((tail_merge_kernel<D, 3>), grid, dim3(256), 0, st, p); break;
        case 4: hipLaunchKernelGGL((tail_merge_kernel<D, 4>), grid, dim3(256), 0, st, p); break;
        case 5: hipLaunchKernelGGL((tail_merge_kernel<D, 5>), grid, dim3(256), 0, st, p); break;
        case 6: hipLaunchKernelGGL((tail_merge_kernel<D, 6>), grid, dim3(256), 0, st, p); break;
        case 7: case 8: hipLaunchKernelGGL((tail_merge_kernel<D, 8>), grid, dim3(256), 0, st, p); break;
        default: hipLaunchKernelGGL((tail_merge_kernel<D, kMaxSplit>), grid, dim3(256), 0, st, p); break;
    }
    return hipGetLastError();
}

// Launches the items of `p` (already planned) as workgroups of NW wavefronts.
template <int D, int NW, bool BASE2, bool OUT16>
static hipError_t launch_items(AttnParams p, int64_t items, int n_cu, hipStream_t st) {
    auto kern = attn_fwd_sp_kernel<D, NW, BASE2, OUT16>;
    constexpr int smem = 2 * sp_buffers(D, NW) * 64 * D * 2;       // 128 KB (d = 128, 8 wavefronts) or 64 KB
    constexpr int alone = 96 * 1024;                               // keeps a second workgroup off the CU
    static KernelSetup setup;
    hipError_t e = setup.ensure(reinterpret_cast<const void*>(kern), smem > alone ? smem : alone, nullptr);
    if (e != hipSuccess) return e;
    items *= kTileRows / (32 * NW);
    p.n_items = (int)items;
    // two workgroups of four wavefronts share a CU, unless there are not enough of them to fill every CU
    const int64_t slots = (int64_t)n_cu * (NW == 8 ? 1 : 2);
    const int lds = NW < 8 && items * p.n_groups <= n_cu ? alone : smem;
    // several groups: one workgroup per item (they fit the chip at once), no chains and no counter
    if (p.n_groups > 1 && items * p.n_groups > slots) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kern, dim3((unsigned)(items < slots ? items : slots), (unsigned)p.n_groups), dim3(64 * NW), lds, st, p);
    return hipGetLastError();
}

template <int D, bool BASE2, bool OUT16>
static hipError_t launch_sp(AttnParams p, int BH, float* ws, int64_t ws_slots, hipStream_t st) {
    int n_cu = 0;
    {
        hipError_t e = device_cu_count(&n_cu);
        if (e != hipSuccess) return e;
    }
    const TailPlan t = plan_tail(p.Sq, BH, p.n_v, n_cu);
    if (rows_form(t, p.Sq, BH, p.n_v, D, n_cu) && !p.redo_always) return launch_attn_rows(p, BH, D, n_cu, st);
    p.group_slots = (int)tail_slots(t, p.out_bf16 != 0);
    const int64_t slots = (int64_t)p.group_slots * p.n_groups;
    if (ws == nullptr || slots > ws_slots) return hipErrorInvalidValue;
    // no key range may be empty or start off a 64-key boundary
    if (t.split > 1) {
        if (t.split > kMaxSplit || t.part_off[0] != 0 || t.part_off[t.split] != p.n_v) return hipErrorInvalidValue;
        for (int j = 0; j < t.split; ++j)
            if (t.part_off[j + 1] <= t.part_off[j] || t.part_off[j] % 64 != 0) return hipErrorInvalidValue;
    }
    p.tiles_per_head = t.tiles_per_head;
    p.split = t.split;
    p.n_cut = (int)t.n_cut;
    p.n_full = (int)(t.n_tiles - t.n_cut);
    for (int j = 0; j <= kMaxSplit; ++j) p.part_off[j] = t.part_off[j];
    p.part_out = slots ? ws : nullptr;
    p.part_lse = slots ? ws + slots * (kTileRows * D) : nullptr;
    p.counter = reinterpret_cast<int*>(ws + ws_slots * kSlotFloats);     // two ints behind the slots, zero between launches
    const int64_t items = p.n_full + t.n_cut * t.split;
    hipError_t e;
    const WidePlan wide = p.n_groups > 1 || p.redo_always || !wide_pays(t, p.n_v, D, BASE2, n_cu) ? WidePlan{0, 0} : wide_plan(t, p.n_v, n_cu);
    if (wide.items > 0) {
        p.n_wide = wide.items;
        p.n_odd = wide.odd_heads;
        p.n_items = (int)items;
        e = launch_attn_wide(p, D, n_cu, st);
    } else if (sp_wavefronts(t, p.n_v, D, n_cu) == 4) {
        e = launch_items<D, 4, BASE2, OUT16>(p, items, n_cu, st);
    } else {
        e = launch_items<D, 8, BASE2, OUT16>(p, items, n_cu, st);
    }
    if (e != hipSuccess || t.split <= 1) return e;
    return launch_tail_merge<D>(p, st);
}

// Head dimension 64 is compiled by attn_fwd_sp_d64.hip, which includes this file with
// PDA_SP_HEAD_DIM 64: the two sets of kernels then build side by side.
template <int D>
static hipError_t launch_sp_form(const AttnParams& p, int BH, float* ws, int64_t ws_slots, hipStream_t st) {
    if (p.out_bf16) return p.base2 ? hipErrorInvalidValue : launch_sp<D, false, true>(p, BH, ws, ws_slots, st);
    return p.base2 ? launch_sp<D, true, false>(p, BH, ws, ws_slots, st) : launch_sp<D, false, false>(p, BH, ws, ws_slots, st);
}

#ifndef PDA_SP_HEAD_DIM
hipError_t launch_attn_fwd_sp_d64(const AttnParams& p, int BH, float* ws, int64_t ws_slots, hipStream_t st);

hipError_t launch_attn_fwd_sp(const AttnParams& p, int BH, int D, float* ws, int64_t ws_slots, hipStream_t st) {
    return D == 64 ? launch_attn_fwd_sp_d64(p, BH, ws, ws_slots, st) : launch_sp_form<128>(p, BH, ws, ws_slots, st);
}
#else
hipError_t launch_attn_fwd_sp_d64(const AttnParams& p, int BH, float* ws, int64_t ws_slots, hipStream_t st) {
    return launch_sp_form<64>(p, BH, ws, ws_slots, st);
}
#endif
#endif   // PDA_SP_DEVICE_ONLY

}  // namespace pda
