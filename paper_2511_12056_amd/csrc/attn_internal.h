// Internal declarations shared by the translation units of libpipedit_attn (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <vector>

namespace pda {

// One-time, per-device launch setup of a kernel that needs more than the default dynamic LDS size:
// sets the attribute on the current device the first time the kernel is launched there and
// returns that device's CU count through n_cu.  One instance per kernel (function-local static).
struct KernelSetup {
    static constexpr int MAX_DEV = 64;
    std::atomic<int> cu[MAX_DEV] = {};
    hipError_t ensure(const void* kern, int smem_bytes, int* n_cu) {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        const bool cached = dev >= 0 && dev < MAX_DEV;
        int v = cached ? cu[dev].load(std::memory_order_acquire) : 0;
        if (v == 0) {   // two threads may both get here: setting the attribute twice is harmless
            if ((e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem_bytes)) != hipSuccess) return e;
            if ((e = hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
            if (cached) cu[dev].store(v, std::memory_order_release);
        }
        if (n_cu) *n_cu = v;
        return hipSuccess;
    }
};

// One attention launch over Hg heads of B batches.  Strides are in elements; a head group of a
// compact [B,H,S,d] tensor is addressed by offsetting the base pointers and keeping the full
// tensor's batch stride.
struct AttnParams {
    const __bf16* q;
    const __bf16* k;
    const __bf16* v;
    float* out;
    float* lse;
    int64_t Sq;
    int64_t n_v;            // number of valid keys (kv_valid_len)
    int64_t q_bs, q_hs;     // q batch / head stride
    int64_t kv_bs, kv_hs;   // k and v batch / head stride
    int64_t o_bs, o_hs;     // out batch / head stride
    int64_t l_bs, l_hs;     // lse batch / head stride
    int Hg;                 // heads of a group
    int n_groups;           // groups of Hg heads, one after the other, each with the same plan: grid.y (1: the launch is one group)
    int group_slots;        // workspace slots of a group
    float scale;            // softmax scale
    float scale_log2e;      // scale * log2(e)
    // Work items of the software-pipelined kernel, taken in index order by persistent workgroups.
    // Units [0, n_full) are whole 256-row query tiles (tile = unit; head = tile / tiles_per_head).
    // Every later tile is cut into `split` key ranges [part_off[j], part_off[j+1]), one unit each
    // (unit = n_full + part * n_cut + cut tile), so that the end of the launch is made of short ones.
    // With workgroups of eight wavefronts an item is a unit; with four, items 2u and 2u + 1 are the
    // upper and the lower 128 rows of unit u.
    // part 0 writes out/lse, parts >= 1 write normalised partials to part_out/part_lse, which a
    // merge pass folds into out/lse.  split <= 1: no cut.
    int tiles_per_head;
    int n_full;
    int split;
    int64_t part_off[17];   // first key of each range (multiples of 64); part_off[split] = n_v
    float* part_out;        // [(tile - n_full) * (split - 1) + part - 1][256][d]
    float* part_lse;        // [(tile - n_full) * (split - 1) + part - 1][256]
    int n_cut;              // number of cut tiles (the last n_cut of a group)
    int n_items;            // n_full + n_cut * split per group, twice that with four wavefronts (set by the launch)
    int n_wide;             // leading items that are pairs of whole tiles (attn_fwd_wide.hip); 0: none
    int n_odd;              // heads whose last, single tile is left out of those pairs
    int* counter;           // two ints, zero between launches: items taken beyond each workgroup's first, workgroups that have finished
    int out_bf16;           // software-pipelined kernel: `out` points to bf16 elements (same element strides)
    int base2;              // scores are already in log2 units: weights 2^(q.k), scale_log2e == 1
    int redo_always;        // software-pipelined kernel: sweep every item a second time with the running max (testing aid)
};

// Tail plan of the software-pipelined kernel (256-row query tiles; persistent workgroups, one per CU
// or two that take half a tile each, taking items in order).  Whole tiles are long items (a 119 056-key sweep takes
// 3 ms), the XCDs run at different speeds, and a launch ends when the last item does; so the
// `rem` = n_tiles mod n_cu tiles that do not fill a round of whole tiles are cut into `split` key
// ranges, short items that the workgroups pick up as they run out of whole tiles.  Measured on
// the device: about three part items per CU balance the end of a long launch; every part pays a
// prologue, a partial store and its share of the merge, so parts are kept at 100 key tiles or more
// (50 where that gives no more than 4 ranges).  Rule:
//     split = round(3 * n_cu / rem), at least 2, at most the smallest of
//             16, max(nt / 100, min(nt / 50, 4)) (nt = key tiles of a whole sweep), n_v / 512,
//             1 + (9 * n_cu / 4) / rem   (workspace: the parts beyond the first must fit),
//     lowered until the last range is not empty; uncut if that leaves less than 2 or rem = 0.
// Where the parts are short and the CUs become free together, parts run in rounds like tiles do,
// and ONE round of parts is best: split = floor(n_cu / rem) under the same caps except the one on
// the part length.  That is the plan of a launch with fewer tiles than CUs (one head of a short
// clip, the unit PipeSP pipelines, would otherwise leave CUs without work for its whole duration;
// measured: 38 tiles of 150 key tiles, split 6: 0.081 ms instead of 0.181 ms) and of sweeps of
// under 200 key tiles whose left-over tiles fill at most half the machine (measured: 10 heads x
// 9 600 tokens, rem = 124: 0.502 / 0.428 / 0.451 / 0.442 ms for split 1 / 2 / 3 / 4).
// Where the left-over tiles fill more than half the machine and at most three rounds of whole
// tiles precede them, no equal cut within the workspace balances the end (210 left-over tiles in
// 3 ranges are 630 parts: 2.5 rounds, which end when 3 would).  Such tiles are cut UNEQUALLY: a
// long first range of a fraction A of the keys, taken by rem CUs, and split-1 short ranges, which
// the other n_cu - rem CUs work off meanwhile, k each: k = ceil(rem (split-1) / (n_cu - rem)),
// A = k / (k + split - 1) (both kinds of CU then finish together), split = 4 after one round of
// whole tiles, else 3, within the workspace cap and with short ranges of at least 1024 keys
// (measured, one head at S = 119 056 = 256 + 210 tiles: 5.78 -> 5.47 ms; 5 x 36 000: 2.64 -> 2.55).
// After four or more rounds of whole tiles the CUs do not become free together, items are handed
// out as CUs ask for them, and what is left idle at the end is about half of the items started
// last.  There the ranges (2 to 6 of them) get DECREASING sizes, each 5/8 of the one before, range
// 0 first: the items started last are the shortest (measured, 3-head group at S = 119 056, five
// ranges of 41 / 26 / 16 / 10 / 6 % instead of 20 % each: 16.53 -> 16.43 ms; 6 heads, three
// ranges of 50 / 31 / 19 %: 32.98 -> 32.85 ms); kept equal if the last range would fall under
// 50 key tiles.
// A pure function of (Sq, number of (batch, head) pairs, valid keys, CU count): the cut tiles are
// the last n_cut of the launch's n_tiles tiles in (batch, head, query tile) order.
constexpr int kMaxSplit = 16;
struct TailPlan {
    int tiles_per_head;
    int64_t n_tiles;
    int64_t n_cut;          // 0 if no tile is cut
    int split;              // 1 if no tile is cut
    int64_t part_off[kMaxSplit + 1];   // range j of a cut tile = keys [part_off[j], part_off[j+1]); multiples of 64 up to
                                       // part_off[split] = n_v; entries beyond split are n_v as well
};
inline int64_t max_extra_slots(int n_cu) { return (int64_t)n_cu * 9 / 4; }
inline int64_t part_keys_for(int64_t n_v, int s) { return ((n_v + s - 1) / s + 63) / 64 * 64; }
inline TailPlan plan_tail(int64_t Sq, int BH, int64_t n_v, int n_cu) {
    TailPlan t{};
    t.tiles_per_head = (int)((Sq + 255) / 256);
    t.n_tiles = (int64_t)t.tiles_per_head * BH;
    t.split = 1;
    const int64_t rem = t.n_tiles % n_cu;
    bool one_round = false;
    if (rem) {
        const int64_t nt = (n_v + 63) / 64;
        // One round of parts (n_cu / rem ranges per tile) where the parts are short and start together:
        // a launch of fewer tiles than CUs, or sweeps of under 200 key tiles whose left-over tiles
        // fill at most half the machine.  Otherwise about three rounds of parts, round(3 n_cu / rem),
        // of at least 100 key tiles each (at least 50 where that gives no more than 4 ranges).
        one_round = t.n_tiles < n_cu || (nt < 200 && 2 * rem <= n_cu);
        int64_t s_max = kMaxSplit;
        if (!one_round) {
            int64_t by_len = nt / 50 < 4 ? nt / 50 : 4;
            if (nt / 100 > by_len) by_len = nt / 100;
            if (by_len < s_max) s_max = by_len;
        }
        if (n_v / 512 < s_max) s_max = n_v / 512;
        if (1 + max_extra_slots(n_cu) / rem < s_max) s_max = 1 + max_extra_slots(n_cu) / rem;
        int64_t s = one_round ? n_cu / rem : (6 * (int64_t)n_cu + rem) / (2 * rem);
        if (s < 2 && !one_round) s = 2;
        if (s > s_max) s = s_max;
        while (s >= 2 && (s - 1) * part_keys_for(n_v, (int)s) >= n_v) --s;   // the last range must not be empty
        if (s >= 2) t.split = (int)s;
    }
    for (int j = 0; j <= kMaxSplit; ++j) t.part_off[j] = n_v;
    if (t.split > 1) {
        t.n_cut = rem;
        const int64_t pk = part_keys_for(n_v, t.split);
        for (int j = 0; j < t.split; ++j) t.part_off[j] = j * pk;
        // decreasing ranges after four or more rounds of whole tiles: weights 8^(s-1-j) 5^j
        if (!one_round && t.n_tiles >= 4 * (int64_t)n_cu && t.split <= 6) {
            int64_t w[6], total = 0, cum = 0, off[7];
            for (int j = 0; j < t.split; ++j) {
                w[j] = 1;
                for (int i = 0; i < t.split - 1 - j; ++i) w[j] *= 8;
                for (int i = 0; i < j; ++i) w[j] *= 5;
                total += w[j];
            }
            off[0] = 0;
            for (int j = 1; j < t.split; ++j) { cum += w[j - 1]; off[j] = n_v * cum / total / 64 * 64; }
            off[t.split] = n_v;
            bool ok = n_v - off[t.split - 1] >= 3200;
            for (int j = 0; j < t.split; ++j) ok = ok && off[j + 1] > off[j];
            if (ok) for (int j = 0; j < t.split; ++j) t.part_off[j] = off[j];
        }
    }
    // unequal cut: many left-over tiles after at most three rounds of whole tiles
    if (rem && 2 * rem > n_cu && t.n_tiles < 4 * (int64_t)n_cu && t.n_tiles > n_cu) {
        int64_t s = t.n_tiles < 2 * (int64_t)n_cu ? 4 : 3;
        if (1 + max_extra_slots(n_cu) / rem < s) s = 1 + max_extra_slots(n_cu) / rem;
        for (; s >= 2; --s) {
            const int64_t k = (rem * (s - 1) + (n_cu - rem) - 1) / (n_cu - rem);
            const int64_t first = ((n_v * k / (k + s - 1) + n_v / 100) / 64 + 1) * 64;
            if (first >= n_v) continue;
            const int64_t part = ((n_v - first + (s - 2)) / (s - 1) + 63) / 64 * 64;
            if (part < 1024 || first + (s - 2) * part >= n_v) continue;    // short ranges too short, or the last one empty
            t.split = (int)s;
            t.n_cut = rem;
            for (int j = 0; j <= kMaxSplit; ++j) t.part_off[j] = j == 0 ? 0 : (j < s ? first + (j - 1) * part : n_v);
            break;
        }
    }
    return t;
}
// Wavefronts per workgroup of a launch with plan `t` and no pairs of tiles (wide_plan, wide_pays below): eight (256 rows, one
// workgroup per CU) or four (128 rows, half a tile; two per CU).  The results are the same bits; only the time differs (us,
// eight -> four).  Eight is the rule: a K/V tile in LDS serves twice the rows, half the global -> LDS
// traffic (3 heads x 67 576, d = 128: 5 530 -> 6 120; 10 x 9 600: 419 -> 471).  Four
//  * where even the halves of the items do not fill every CU: twice the CUs work on the launch, one
//    wavefront per SIMD (112 shapes of 1 to 128 tiles, 64 to 119 056 keys: none slower beyond the noise;
//    1 head x 1 024 on 119 056, d = 128: 149 -> 107);
//  * for short sweeps (up to 24 key tiles) in more than four rounds of tiles: two workgroups share a CU
//    and one computes while the other loads or stores, and the last round is spread more evenly.  Pairs have taken over most of
//    these launches.  What is left is fewer keys than pairs need (24 x 40 000, d = 128, on 128 keys 197 -> 186, on 200
//    231 -> 219; 26 x 10 100 on 200 80.2 -> 77.4; 24 x 16 384 on 220 the same, but on 192, six full rounds, 91.8 -> 98.9), base 2 at
//    d = 64 where pairs do not pay (193 x 1 900 on 1 000 145 -> 132; 26 x 10 100 on 866 93.0 -> 89.4, on 1 400 122 -> 122;
//    24 x 16 384 on 800 to 1 536 within 1 %), and variant 3, which has no pairs.  Not
//      - in exactly four rounds, at d = 64 not in four to six rounds whose last is more than half full;
//      - with too few key tiles to hide the second workgroup's start behind: at d = 64, where a tile
//        takes half the time, under eight (24 x 16 384 on 192 keys: 56.9 -> 63.7), at d = 128 under four
//        unless there are six rounds (88 x 4 096 on 64 keys: 86 -> 87);
//      - under eight tiles per head (four with up to four key tiles), where K and V of a head are fetched
//        for few rows (1 126 x 256, d = 128, on 1 529 keys: 286 -> 315).
inline int sp_wavefronts(const TailPlan& t, int64_t n_v, int d, int n_cu) {
    const int64_t items = t.n_tiles - t.n_cut + t.n_cut * t.split, key_tiles = (n_v + 63) / 64;
    if (2 * items <= n_cu) return 4;
    if (key_tiles > 24 || t.tiles_per_head < (key_tiles > 4 ? 8 : 4) || t.n_tiles <= 4 * (int64_t)n_cu) return 8;
    const bool six_rounds = t.n_tiles >= 6 * (int64_t)n_cu;
    if (d == 128) return six_rounds || key_tiles >= 4 ? 4 : 8;
    const int64_t rem = t.n_tiles % n_cu;
    return key_tiles >= 8 && (six_rounds || (rem > 0 && 2 * rem <= n_cu)) ? 4 : 8;
}
// Leading items of a launch with plan `t` that are pairs of whole tiles of one head, 512 rows a workgroup (attn_fwd_wide.hip),
// and the heads among those with an odd number of tiles that they cover but for the last tile.  A CU works off a pair in 1.83
// times (d = 128; 1.9 at d = 64) what it needs for a tile, so pairs are taken wherever each CU has two whole tiles to
// do: of `full` whole tiles, n_cu - rem CUs have full / n_cu and rem have one more.  That is worth most where the last round is
// partly full and uncut: those CUs have one pair instead of two tiles (us, eight or four wavefronts a tile -> pairs first,
// d = 128 / d = 64):
//   long sweeps:  3 x 119 056 16 430 -> 15 140 (five rounds, four of them in pairs); 24 x 9 600 927 -> 879 / 574 -> 558;
//                 24 x 5 000 289 -> 247 / 180 -> 158 (1.88 rounds, uncut)
//   short ones:   24 x 16 384 on 1 536 keys 292 -> 271 / 177 -> 162, on 570 154 -> 150 / 100 -> 86, on 224 110 -> 102 / 67 -> 55;
//                 48 x 4 800 on 400 92 -> 76 / 61 -> 52; 400 x 301 on 700 99 -> 86 / 68 -> 60
// Of 64 shapes (1 to 12 rounds, 224 to 119 056 keys, fp32 and bf16 results, and base 2 at d = 128) none is slower; base 2 at
// d = 64: wide_pays.  Below 224 keys the first steps of a sweep would not find the whole tiles they fetch.
// (With rows that need the second sweep: attn_fwd_wide.hip.)
constexpr int64_t kWideKeys = 224;
struct WidePlan { int items, odd_heads; };
inline WidePlan wide_plan(const TailPlan& t, int64_t n_v, int n_cu) {
    const int64_t full = t.n_tiles - t.n_cut, pairs = t.tiles_per_head / 2;
    if (n_v < kWideKeys || full < n_cu || pairs == 0) return {0, 0};
    const int64_t rounds = full / n_cu, rem = full % n_cu;
    const int64_t have = full / t.tiles_per_head * pairs + full % t.tiles_per_head / 2;
    int64_t n = (n_cu - rem) * (rounds / 2) + rem * ((rounds + 1) / 2);
    if (n > have) n = have;
    return {(int)n, t.tiles_per_head % 2 ? (int)(n / pairs) : 0};
}
// Do the pairs pay?  At d = 64 with scores in base 2 (no scale left to apply, so the single tiles of attn_fwd_sp.hip have the least
// to do beside the products) only for short sweeps: the phases of a pair, seeded scores among them, take 1 to 4 % longer, what
// pairs save is between items and in the last round (us, without -> with pairs: 24 x 9 600 on 3 000 keys 192 -> 188, on 9 600
// 517 -> 524, 24 x 6 400 on 65 536 2 200 -> 2 293; 24 x 5 000, under two rounds, on 9 600 287 -> 286, on 32 768 894 -> 900; 19 x
// 24 087, seven rounds, on 512 99 -> 96, 24 x 26 708 on 768 163 -> 160, 19 x 24 087 on 1 024 149 -> 152, on 65 536 6 456 -> 6 696).
inline bool wide_pays(const TailPlan& t, int64_t n_v, int d, bool base2, int n_cu) {
    if (d != 64 || !base2) return true;
    if (t.n_tiles < 2 * (int64_t)n_cu) return n_v <= 9600;
    return n_v <= (t.n_tiles <= 4 * (int64_t)n_cu ? 3072 : 768);
}
// Does a launch with plan `t` (of one group, if several share it) take the kernel for few query rows (attn_rows.hip: its
// wavefronts share the keys) instead of cut tiles and their merge?  Only launches in which every tile is cut: rows of whole
// tiles keep the bits of a sweep in one pass.  The time of that kernel goes by rounds of its workgroups (one per CU, at d = 64
// two) and by the keys; the cut form hardly grows with the keys as long as CUs are free, but starts at 12 to 16 us.  So
// the line lies at a number of keys that grows with the blocks of 32 rows up to the end of a round and falls behind it (us,
// cut -> rows; of about 750 shapes of 1 to 1 024 blocks on 1 024 to 12 288 keys those that the rule takes are not slower, but for a few
// blocks more than two rounds on 1 025 to 1 152 keys at d = 128: 17 x 1 024 on 1 152 29.1 -> 31.7, 22 x 1 024 on 1 100 33.9 -> 31.0.  The
// reference of shares of twelve tiles and more has since cost up to 3 %, no line moved):
//   d = 64:  2 x 1 024 rows on 1 024 keys (64 blocks) 14.0 -> 7.0, on 4 096 16.1 -> 15.8, on 5 120 17.6 -> 18.4;
//            1 x 256 on 3 072 14.1 -> 12.6, on 4 096 13.8 -> 15.0; 8 x 1 024 on 6 144 27.4 -> 23.0, on 12 288 39.1 -> 42.7;
//            16 x 1 024 on 4 096 30.8 -> 28.3, on 6 144 38.9 -> 40.5; 18 x 1 024 on 2 048 24.6 -> 21.9, on 3 072 29.1 -> 29.9
//   d = 128: 1 x 1 024 on 1 024 15.9 -> 10.1, on 2 048 16.5 -> 13.9, on 3 072 17.3 -> 18.0; 4 x 1 024 on 5 120
//            31.6 -> 26.5; 8 x 1 024 on 2 048 24.1 -> 15.8, on 8 192 48.4 -> 48.4; 9 x 1 024 on 1 024 20.5 -> 15.4, on 4 096
//            39.1 -> 38.7; 16 x 1 024 on 2 048 37.6 -> 26.4, on 6 144 64.7 -> 64.0; 17 x 1 024 on 1 024 29.9 -> 29.2, on 1 536
//            33.7 -> 37.0; 32 x 1 024 on 1 536 46.9 -> 43.6, on 2 048 52.6 -> 53.4
inline bool rows_form(const TailPlan& t, int64_t Sq, int BH, int64_t n_v, int d, int n_cu) {
    if (t.split <= 1 || t.n_cut != t.n_tiles) return false;
    const int64_t blocks = (Sq + 31) / 32 * BH, round = n_cu;
    if (blocks > 4 * round) return false;
    if (d == 64) {
        if (blocks > 2 * round) return n_v <= (blocks <= 3 * round ? 2048 : 1536);
        if (n_v <= 3072) return true;
        return 4 * blocks >= round && n_v <= (8 * blocks >= 3 * round && blocks <= round ? 6144 : 4096);
    }
    if (blocks > 2 * round) return n_v <= (2 * blocks >= 7 * round ? 1536 : 1152);
    if (blocks > round) return n_v <= 4096;
    return n_v <= (2 * blocks >= round ? 5120 : 4 * blocks >= round ? 3072 : 2048);
}
// Blocks of 32 rows in a workgroup of that kernel, for a launch of `blocks` (of all groups that share it); same bits.  Two halve the
// keys that a CU streams for a row, but a wavefront then needs 1.7 times as long for a tile, so at d = 128 they pay as soon as there
// is more than one round (us, one -> two: 9 x 1 024 on 2 048 keys 28.5 -> 22.6, 16 x 1 024 31.8 -> 26.4, 32 x 1 024 65.7 -> 53.4; 8 x
// 1 024 16.7 -> 22.9), at d = 64, where two workgroups share a CU, for a nearly full second round of few keys (16 x 1 024 on
// 1 024 13.4 -> 11.2, on 1 536 16.5 -> 14.4, on 2 048 17.7 -> 18.0; 24 x 1 024 on 1 024 16.1 -> 21.4).
inline int rows_blocks(int64_t blocks, int64_t n_v, int d, int n_cu) {
    if (d == 128) return blocks > n_cu ? 2 : 1;
    return 2 * blocks >= 3 * (int64_t)n_cu && blocks <= 2 * (int64_t)n_cu && n_v <= 1536 ? 2 : 1;
}
// Head groups of a pipeline that share a launch: `left` groups of BH (batch, head) pairs each remain.
// A group of at most half an item per CU (the four-wavefront rule above: its half items are alone on a CU or leave
// CUs without work) cannot fill the chip, and its launch, merge, event and hand-off cost the host more than the GPU.
// As many such groups as give each CU one item go out as one launch, two workgroups per CU, each group with the plan
// and so the bits it has alone; their hand-off waits for that one launch.  24 x 2 048, d = 128, head by head (8 tiles
// in 4 ranges = 32 items a group, batches of eight): 680 -> 151 us, host time.  Above half an item per CU a group
// goes out alone: two of them would not fit the chip at once.
inline int batch_of_groups(int64_t Sq, int BH, int64_t n_v, int n_cu, int left) {
    if (n_v <= 0 || left < 2) return 1;
    const TailPlan t = plan_tail(Sq, BH, n_v, n_cu);
    const int64_t items = t.n_tiles + t.n_cut * (t.split - 1);
    if (2 * items > n_cu) return 1;
    const int64_t fit = n_cu / items;
    return (int)(fit < left ? fit : left);
}
// The launches of a pipeline over head groups of the given sizes (B batches): `groups` groups of hg heads each from
// head h0 on.  One group each if their times are wanted (`alone`), otherwise runs of equal groups in batches.
// Every size is looked at twice, the plan of a run made once: 65 535 groups are allowed.
struct PipelineStep { int h0, hg, groups; };
template <class Sizes>
std::vector<PipelineStep> pipeline_steps(const Sizes& sizes, int B, int64_t Sq, int64_t n_v, int n_cu, bool alone) {
    std::vector<PipelineStep> steps;
    const int n = (int)sizes.size();
    for (int g = 0, h0 = 0; g < n;) {
        const int hg = sizes[g];
        int end = g + 1;
        while (end < n && sizes[end] == hg) ++end;
        const int fit = alone ? 1 : batch_of_groups(Sq, B * hg, n_v, n_cu, end - g);
        for (; g < end; g += steps.back().groups) {
            steps.push_back({h0, hg, fit < end - g ? fit : end - g});
            h0 += hg * steps.back().groups;
        }
    }
    return steps;
}
// Steps whose launches take the kernel for few query rows need neither workgroups all at once nor workspace, so consecutive ones can go
// out as one launch of up to three rounds (six blocks of 32 rows per CU).  That saves the host's part of a step (launch,
// event, wait and hand-off: 20 us, of which the wait on the drain stream takes 8), and it fills the CUs: a step is as many groups as the
// cut form fills them with (batch_of_groups), with this kernel often half of that (us, head by head, apart -> joined: d = 128,
// 24 x 1 536 116 -> 92, 24 x 2 048 140 -> 109, 48 x 1 024 on 2 048 122 -> 107; d = 64, 24 x 3 072 238 -> 139, 24 x 4 096 328 -> 198; where
// one step holds all groups, 24 x 1 024, no difference).
// The line, 2 048 keys at d = 128 and 4 096 at d = 64, is not where joining stops paying: 24 x 2 304 164 -> 133, 24 x 3 072
// 294 -> 199, 24 x 5 120 811 -> 439, d = 64 24 x 4 608 590 -> 259, 24 x 6 144 657 -> 388, no shape of 12, 24 and 48 heads slower.  It
// bounds how long the hand-offs of a joined launch, which all wait for its end, are held back (three rounds of 25 us).
inline std::vector<PipelineStep> join_steps(const std::vector<PipelineStep>& steps, int B, int64_t Sq, int64_t n_v, int d, int n_cu, bool alone) {
    std::vector<PipelineStep> out;
    for (const PipelineStep& s : steps) {
        if (!alone && !out.empty() && out.back().hg == s.hg && n_v * d <= 2048 * 128) {
            PipelineStep& last = out.back();
            const int BH = B * s.hg;
            const int64_t blocks = (Sq + 31) / 32 * BH;
            if ((last.groups + s.groups) * blocks <= 6 * (int64_t)n_cu && rows_form(plan_tail(Sq, BH, n_v, n_cu), Sq, BH, n_v, d, n_cu)) {
                last.groups += s.groups;
                continue;
            }
        }
        out.push_back(s);
    }
    return out;
}
// One workspace slot holds one key-range partial of a cut tile: 256 x 128 values + 256 lse.
// A workspace of n slots is n * kSlotFloats floats followed by kCounterFloats floats that hold the
// kernel's two work counters (zero whenever no launch is running on it).
constexpr size_t kSlotFloats = 256 * 128 + 256;
constexpr size_t kCounterFloats = 64;
// Slots a launch needs: parts 1.. of every cut tile (part 0 goes to out/lse), or all parts when
// out is bf16 (the merge pass then needs part 0 in fp32 as well).
inline int64_t tail_slots(const TailPlan& t, bool out_bf16) {
    return t.split > 1 ? t.n_cut * (out_bf16 ? t.split : t.split - 1) : 0;
}
// Largest slot count any launch can need on a device with n_cu compute units.
inline int64_t max_tail_slots(int n_cu, bool out_bf16) {
    return max_extra_slots(n_cu) + (out_bf16 ? n_cu - 1 : 0);
}

// Enqueue the forward kernel for B*Hg = BH (batch, head) pairs.  variant selects a tiling (0 = the
// software-pipelined kernel; 1, 2 = reference tilings; 3 = 0 with its running-max sweep forced on
// every item).  ws / ws_slots: device workspace for the key-range partials of the
// software-pipelined kernel and its capacity in slots of kSlotFloats floats; a launch that needs
// more returns hipErrorInvalidValue (the caller sizes it with plan_tail / tail_slots).
hipError_t launch_attn_fwd(const AttnParams& p, int BH, int D, int variant, float* ws, int64_t ws_slots, hipStream_t st);

// Software-pipelined kernel for d = 128 and 64 (attn_fwd_sp.hip); p.n_v >= 1, p.scale_log2e > 0.
hipError_t launch_attn_fwd_sp(const AttnParams& p, int BH, int D, float* ws, int64_t ws_slots, hipStream_t st);

// Software-pipelined kernel with p.n_wide > 0 wide items in front (attn_fwd_wide.hip); all of p but the grid is set.
hipError_t launch_attn_wide(const AttnParams& p, int D, int n_cu, hipStream_t st);

// Kernel for launches of few query rows (attn_rows.hip).
hipError_t launch_attn_rows(const AttnParams& p, int BH, int D, int n_cu, hipStream_t st);

// Does this (d, variant, valid key count) take the software-pipelined kernel (and so possibly a workspace)?
inline bool uses_sp_kernel(int D, int variant, int64_t n_v) { return (D == 128 || D == 64) && n_v > 0 && (variant == 0 || variant == 3); }

// CU count of the current device (cached per device).
hipError_t device_cu_count(int* n_cu);

struct MergeParams {
    const float* part[16];
    const float* lse[16];
    float* out;
    float* lse_out;         // nullable
    int64_t rows;
    int n;
};
hipError_t launch_merge(const MergeParams& p, int d, hipStream_t st);

// Copy n floats (n % 4 == 0, 16-byte aligned) on a stream: the hand-off op of the head-chunk pipeline.
hipError_t launch_copy_f32(const float* src, float* dst, int64_t n, hipStream_t st);

// Algorithm 1 steps 10-13 in one pass: hidden[r, i*h + j, :] = chunk[j][r, i, :].
struct PostParams {
    const float* chunk[64];  // h device pointers
    float* hidden;           // [rows, n*h, D]
    int64_t rows;
    int64_t row_stride4;     // distance between rows of a chunk, in float4s
    int h, n, D4;            // D4 = D / 4
};
hipError_t launch_postprocess(const PostParams& p, hipStream_t st);

// Hand-off of hg heads [hg, S, d] (global heads h0.. of H = n*h) into a token-major [S, H, d]
// buffer; arrival != 0 places head i*h+j at slot j*n+i (PipeSP's arrival order), else at i*h+j.
hipError_t launch_scatter_heads(const float* src, float* dst, int64_t S, int d, int hg, int H, int h0,
                                int h, int n, int arrival, hipStream_t st);

// Token-major fp32 [B,S,H,d] -> head-major bf16 [B,H,S,d] (d = 64 or 128), optional unit-RMS vectors,
// every element times premul before the rounding.
hipError_t launch_pack(const float* x, void* y, int B, int64_t S, int H, int d, int unit_rms, float premul, hipStream_t st);

// MFMA rate probes (probe.hip): n_cu workgroups x 8 wavefronts, each wavefront issues about 8*iters
// MFMAs (32x32x16 bf16) on fragments read from src (n_frag 16-byte fragments); mix 0 = MFMAs only,
// 1..3 = with the other instruction classes of the attention loop added; sink: >= 512 floats.
hipError_t launch_mfma_rate(const void* src, int64_t n_frag, int64_t iters, int n_cu, int mix, float* sink, hipStream_t st);

}  // namespace pda
