// Tree attention for gfx950 (Sec. 2.2 of arXiv 2409.10644): every node of the candidate tree attends
// to the prefix KV cache and to its own ancestors under the topology-aware mask.
//
// bf16 path.  One workgroup of 4 wavefronts (two workgroups per compute unit) owns one (sequence, head, key split).  The tree's
// queries are cut into blocks of 32 rows; a wavefront keeps one block of Q in registers for the whole sweep.  K/V
// tiles stream from HBM straight into a ring of LDS stages (global_load_lds, 16 bytes per lane, no registers
// in between), several tiles ahead of the one being computed, so every K/V byte leaves HBM once and is used by
// all queries.  The LDS image of a tile is XOR-swizzled at 16-byte granularity, which makes both read patterns
// below bank-conflict free without padding (direct-to-LDS loads can only write 1 KiB contiguous per instruction).
// Scores are computed transposed, S^T = K * Q^T, with v_mfma_f32_32x32x16_bf16: the accumulator then holds,
// per lane, 16 keys of ONE query, so the online-softmax reductions are in-lane plus one half-wave swap,
// and the exponentiated scores are already in the register layout of the B operand of O^T += V^T * P^T.
// V^T operands come from the row-major V tile through the LDS transpose load (ds_read_b64_tr_b16).
// Wavefronts that share a query block split each tile's keys (key groups) and are merged through LDS at the
// end; key splits across workgroups write partial results, which the workgroup of the (sequence, head) that arrives
// last folds at the end of the same kernel (a small second kernel when the splits do not share one die's L2).
// The tree's own keys are extra tiles whose scores are masked with the packed bitmask slice.
//
// fp32 path: the same operation on the fp32 matrix instructions, see tree_attn_f32_kernel.
#include <math.h>
#include <stdlib.h>

#include <atomic>
#include <type_traits>

#include "mcsd_internal.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((ext_vector_type(8))) short s16x8_t;

struct AttnParams {
    const void *q, *kt, *vt, *kp, *vp;
    void *out;
    const int64_t *seq_base;
    const int32_t *lens;
    const uint64_t *mask_bits;
    int32_t mask_words;
    int32_t B, H, n;  // H: workgroup units per sequence (bf16 sweep: kv heads x chunks of query heads; fp32: query heads)
    int32_t Hq, Hkv;  // query heads, key/value heads (Hq = grp * Hkv)
    int32_t grp;      // query heads that share one key/value head
    int32_t hpw;      // query heads one workgroup of the bf16 sweep serves (they share its K/V stream)
    int32_t bph;      // 32-row query blocks per query head in a workgroup (1, 2 or 4); QBP = bph * hpw
    int32_t chunks;   // grp / hpw: workgroup units per key/value head
    uint32_t mul_chunks, shift_chunks;   // its reciprocal (see fast_div), and that of tps
    uint32_t mul_tps, shift_tps;
    int32_t log2_bph;
    int32_t pair_cus; // > 0: compute units; the grid has more workgroups than that and no separate tree workgroup (see the kernel)
    int32_t xcc;      // accelerator dies the hardware deals workgroup ids to round-robin (>= 1)
    int32_t fold;     // 1: the workgroup of a (sequence, unit) that finishes last folds the partial results itself
    int32_t tree_last; // 1 (no separate tree workgroup, no pairing): the last split that has keys takes the tree's keys, else split 0
    unsigned long long *ctr;   // fold == 1: arrival counter of unit u at ctr[u * CTR_STRIDE], zero before and after every launch
    const uint32_t *ws_tag;    // fold == 1: first word of the workspace, WS_TAG once prepared
    int32_t QT;       // fp32 path: tiles of 16 query rows
    int32_t row0;     // first query row: rows row0 .. n-1 are computed (keys are always all n tree nodes)
    int32_t max_prefix;
    int64_t node_stride, head_stride;
    float c;          // softmax_scale * log2(e)
    float k_scale, v_scale;   // fp8 prefix cache: value = stored * scale
    int32_t S;        // key splits of the prefix
    int32_t G;        // workgroups per (b,h): S, plus one for the tree's own keys when the bf16 sweep splits the prefix
    int32_t tps;      // tiles per split (bf16 sweep): split s owns tiles [s*tps, (s+1)*tps) of every sequence
    int32_t SP;       // partial results per (b,h) (== G)
    int32_t part_f32; // bf16 sweep: partial O as fp32, not bf16 (see PART_F32_KEYS)
    float *part_o;    // [B*H][SP][n][D]; the bf16 sweep keeps its partial O there as bf16 unless part_f32
    float *part_m;    // [B*H][SP][n]   reference maximum of the raw scores
    float *part_l;    // [B*H][SP][n]   sum of exp2((s - m) * c)
};

// Workspace of a call with split keys: [tag word, 256 bytes] [arrival counters, 64 KiB] [part_m] [part_l] [part_o].
// mcsd_workspace_init writes the tag and zeroes the counters; every launch leaves them as it found them.
constexpr uint32_t WS_TAG = 0x4d435344u;
constexpr size_t WS_HEADER = 256, WS_CTR_BYTES = 64 * 1024;
// One arrival counter per 128-byte line: atomics on one line are served one after the other (~85 ns each on this
// machine), so counters of different (sequence, unit) pairs that share a line would queue behind each other.
constexpr int CTR_STRIDE = 16;                          // in 8-byte counters
constexpr int FOLD_MAX_PARTIALS = 16;     // the in-kernel fold keeps one weight per partial result in registers
// Partial O of the bf16 sweep travel as bf16, half the bytes to store and fold, except for prefix bounds below this one: those
// are split for latency alone, and an unsplit sequence is rounded once, from fp32.  With fp32 partial results a split one is
// too.  Up to PART_F32_MAX partial results (what the fold holds at once); more only come from the caller's own plan.
constexpr int PART_F32_KEYS = 512, PART_F32_MAX = 7;
constexpr long PART_F32_BYTES = 16l << 20;  // all of a call's, as much as bf16 ones take when they fill the chip

// What a value row beyond the last one is read as.  Its weight is zero whatever stands there, but zero times an infinity is
// not; a key row may be any (its score is replaced).  Four lanes read 64 contiguous bytes: the same 16 would take four times
// as long.
__device__ __align__(64) const unsigned char zeros[128] = {};

struct AttnPlan {
    int bph, hpw, chunks;  // bf16: query blocks per head, heads per workgroup, units per kv head (see AttnParams)
    int units;             // workgroup units per sequence: kv heads x chunks (bf16), query heads (fp32)
    int QBP;   // query blocks of 32 rows, rounded up to 1, 2 or 4 (bf16 path)
    int T;     // keys per tile
    int QT;    // tiles of 16 query rows (fp32 path), 1 on the bf16 path
    int S;     // key splits of the prefix
    int G;     // workgroups per (b,h): S, or S + 1 when the bf16 sweep gives the tree's own keys a workgroup of their own
    int NS;    // LDS stages of the bf16 sweep
    int xcc;   // dies the workgroup ids are dealt to (1 when unknown: no renumbering)
    int pair_cus;  // see AttnParams
    int tree_last; // see AttnParams
    long grid_units; // (sequence, unit) slots of the grid: B * units, rounded up to a multiple of the dies where that lets the fold run in the kernel
    int fold;  // 1: folded inside the sweep kernel through the L2 its workgroups share
    int part_f32;  // see AttnParams
    int cus;       // compute units the plan is made for
};

constexpr int MCSD_CUS = 256;             // of the whole chip: what a plan is made for where there is no device to ask

__host__ __device__ inline int tile_keys_bf16(int QBP) { return QBP == 1 ? 128 : 64; }   // == SweepCfg::T

// Compute units and accelerator dies of the current device (asked once per device; concurrent first calls store
// the same values).
void device_shape(int &n_cus, int &n_xcc)
{
    static std::atomic<int> cus_of_device[64];
    n_cus = -1;
    n_xcc = 0;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return;
    n_cus = cus_of_device[dev].load(std::memory_order_relaxed);
    if (n_cus == 0) {
        int v = 0;
        n_cus = hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0 ? v : -1;
        cus_of_device[dev].store(n_cus, std::memory_order_relaxed);
    }
    n_xcc = mcsd_xcc_count(dev);
}

// How the bf16 sweep cuts the keys of a (sequence, unit): S splits, and who takes the tree's own keys (1: a workgroup of its
// own, 2: the first split, 3: the last).  The candidates are the S that give every split keys; each is priced in tiles of
// time and the cheapest taken: a workgroup's tiles follow one another at one memory latency each (1.03 us per 64 keys of 128
// dimensions, 0.7 us of 64), partial results cost their exchange and fold (`fold_us`), two workgroups on a compute unit slow
// each other down almost by their sum, and a grid beyond the residents costs its remainder.
// Measured on 3900 shapes of at most one unit per compute unit (1-64 sequences of up to eight times different lengths, 4-64 heads
// of 64 or 128 with 1-8 of them sharing keys, bf16 and fp8, 64-32768 keys, 1-120 rows; every S up to 15 with every place for the
// tree's keys): within 2.2 % of the best of the measured ones on average, one in a hundred 26 % off.  Two workgroups per compute unit
// and at least 256 keys per split lost 11 %; prefixes of fewer than PART_F32_KEYS keys, whose partial results are fp32, would
// lose 11 % unsplit, up to 49 %.  Prices fitted to a sweep that requests two tiles at once (0.88 and 0.62 us, dearer folds)
// were 2.1 % off, on other calls: 2 x 64 heads over 32, 728 keys, 44 rows 12.9 us with these and 16.1 with those; 5 x 4 heads, 552
// keys, 14 rows 8.0 and 6.5.  They cut finer, so that a member of a ragged batch that fits one split here exchanged partial
// results in bf16, a second rounding (1.2 times the error): not worth it.
struct SplitChoice { int S, tree; };
SplitChoice choose_splits(int cus, int d, int QBP, bool f8, int B, long bh, int tiles, int tree_tiles, int tree_forced)
{
    struct Memo { int cus, d, QBP, f8, B, tiles, tree_tiles, forced; long bh; SplitChoice c; };
    static thread_local Memo memo = {0, 0, 0, 0, 0, 0, 0, 0, 0, {1, 2}}; // a decoding loop asks for the same shape again and again
    if (memo.cus == cus && memo.d == d && memo.QBP == QBP && memo.f8 == (int)f8 && memo.B == B && memo.bh == bh && memo.tiles == tiles &&
        memo.tree_tiles == tree_tiles && memo.forced == tree_forced)
        return memo.c;
    static const float fold_us[10] = {0.f, 0.f, 1.4f, 1.85f, 2.4f, 2.5f, 3.15f, 3.2f, 4.7f, 6.3f};   // by partial results
    const float tile_us = (d == 128 ? (QBP == 1 ? 1.6f : QBP == 2 ? 1.03f : 1.15f) : (QBP == 1 ? 1.f : QBP == 2 ? 0.7f : 0.74f)) *
                          (f8 ? 0.8f : 1.f);
    const bool part_f32 = tiles * tile_keys_bf16(QBP) < PART_F32_KEYS;
    const float fold_scale = (d == 64 ? 0.55f : 1.f) * (QBP == 4 ? 1.75f : QBP == 1 ? 1.35f : part_f32 ? 1.5f : 1.f);
    const int per_cu = d == 128 && QBP == 1 ? 1 : 2;                     // resident workgroups (LDS)
    SplitChoice best = {1, tree_forced ? tree_forced : 2};
    if (bh > cus) {
        // The chip is full without splits.  Halves even out ragged batches where two workgroups fit a compute unit.
        if (per_cu == 2 && bh < 2 * cus && tiles >= 8) best.S = 2;
    } else {
        float best_us = 1e30f;
        for (int S = 1; S <= 15 && S <= (tiles > 1 ? tiles : 1) && (S == 1 || bh * S <= 2 * cus); ++S) {
            const int tps = tiles > S ? (tiles + S - 1) / S : 1;
            if (S > 1 && (tiles + tps - 1) / tps != S) continue;         // some split would have no keys
            const int last = tiles - (S - 1) * tps;
            for (int tree = 1; tree <= 3; ++tree) {
                if (tree_forced && tree != tree_forced && S > 1) continue;
                if (S == 1 && tree != 2) continue;
                if (tree == 1 && bh * (S + 1) > (long)cus * per_cu) continue;
                const int parts = S + (tree == 1);
                // One block of 128 columns fills a compute unit's LDS, and what is beyond the residents waits for one of them to end: where two
                // splits are resident no more are made (11 x 8 heads, 6433 keys, 10 rows 53.9 -> 45.7 us; unsplit, 5 x 32 heads of 835-6687
                // keys 73.0 -> 76.1).  Up to nine tiles what is left would give the tree's keys a workgroup, and short members a second
                // partial result with it.
                if (per_cu == 1 && 2 * bh <= cus && tiles > 9 && bh * parts > cus) continue;
                if (S > 1 && part_f32 && (parts > PART_F32_MAX || (long)bh * parts * QBP * 32 * d * 4 > PART_F32_BYTES)) continue;
                const int most = S == 1 ? tiles + tree_tiles
                                 : tree == 1 ? (tps > tree_tiles ? tps : tree_tiles)
                                 : tree == 2 ? tps + tree_tiles : (tps > last + tree_tiles ? tps : last + tree_tiles);
                const float all = (float)(tiles + tree_tiles), load = (float)bh * parts / cus;   // workgroups per compute unit
                float us;
                if (load <= 1.f) us = tile_us * most;
                else if (load <= per_cu) us = 0.94f * tile_us * (most + 0.8f * all / parts);
                else {
                    const float even = all * bh / cus, two = (float)most * per_cu;
                    if (S == 1) us = 0.9f * tile_us * two * (float)(int)(load / per_cu + 0.999f);
                    else us = tile_us * ((tree == 3 ? 0.88f : 0.98f) * (two > even ? two : even) + (tree == 3 ? 0.5f : 0.3f) * most);
                }
                if (tree == 3 && B > 1 && bh * S > cus) us *= 1.08f;     // (not ordered by length: 8 x 32 heads, 500-4000 keys 54 us ordered, 62 not)
                if (tree == 2 && S > 1 && bh * S > cus) us += 1.85f;     // the ordering by length itself
                if (parts > 1) us += fold_us[parts < 9 ? parts : 9] * fold_scale;
                if (us < best_us) { best_us = us; best = {S, tree}; }
            }
        }
    }
    memo = {cus, d, QBP, (int)f8, B, tiles, tree_tiles, tree_forced, bh, best};
    return best;
}

AttnPlan make_plan(int dtype, int B, int Hq, int Hkv, int d, int n_rows, int n_keys, int max_prefix,
                   bool f8 = false, const mcsd_attention_tuning_t *tune = nullptr)
{
    AttnPlan pl;
    const int grp = Hq / Hkv;
    if (dtype == MCSD_BF16) {
        const int qb = (n_rows + 31) / 32;
        pl.bph = qb <= 1 ? 1 : (qb == 2 ? 2 : 4);
        // the fp8 ring is sized for 64-key tiles: a single query block of one head runs as two, the second one empty
        if (f8 && pl.bph == 1 && grp % 2 != 0) pl.bph = 2;
        // grouped-query attention: as many query heads of one kv head as fit the workgroup's four query blocks
        // share its K/V stream (so those bytes leave HBM once for all of them)
        pl.hpw = 1;
        for (int c = 4 / pl.bph; c > 1; c >>= 1)
            if (grp % c == 0) { pl.hpw = c; break; }
        pl.QBP = pl.bph * pl.hpw;
        pl.chunks = grp / pl.hpw;
        pl.units = Hkv * pl.chunks;
        pl.T = tile_keys_bf16(pl.QBP);
        pl.QT = 1;
    } else {
        pl.bph = pl.hpw = 1;
        pl.chunks = grp;
        pl.units = Hq;
        pl.QBP = 1;
        pl.T = 16;
        pl.QT = (n_rows + 15) / 16;
    }
    const long bh = (long)B * pl.units;
    long tiles_max = (max_prefix + pl.T - 1) / pl.T;
    if (dtype == MCSD_F32) tiles_max += (n_rows + pl.T - 1) / pl.T;      // (the tree's own keys are blocks like the prefix's)
    // Key splits.  bf16: see choose_splits; a separate workgroup for the tree's keys costs one more partial result.
    // fp32: one workgroup per compute unit while that takes splitting (more only add partial results: 12 heads of 64, 1024
    // keys, 60 nodes: 9.2 us with 192 workgroups, 10.4 with 384), else as many as fit (4 per compute unit at d = 64, 2 at
    // 128), which evens out ragged batches; at least five 16-key blocks per split.
    int n_cus, n_xcc;
    device_shape(n_cus, n_xcc);
    const int cus = n_cus > 0 ? n_cus : MCSD_CUS;
    long S;
    int tree = 2;
    const int tree_forced = tune && dtype == MCSD_BF16 ? tune->tree_keys : 0;
    if (dtype == MCSD_F32) {
        const long u = (bh + 7) / 8 * 8 * pl.QT;            // (a die's slots are whole (sequence, head) pairs, see grid_units)
        S = u <= cus ? cus / u : (d == 64 ? (4 * cus - 1 + u) / u : 2 * cus / u);
        if (S > tiles_max / 5) S = tiles_max / 5;
        if (S < 1) S = 1;
        if (S > 64) S = 64;
    } else {
        const SplitChoice c = choose_splits(cus, d, pl.QBP, f8, B, bh, (int)tiles_max, (n_keys + pl.T - 1) / pl.T, tree_forced);
        S = c.S;
        tree = c.tree;
    }
    if (tune && tune->key_splits >= 1 && tune->key_splits <= 64) {       // the caller's choice
        S = tune->key_splits;
        // with that many, the tree's keys in a workgroup of their own while all workgroups are resident at once
        if (dtype == MCSD_BF16) tree = tree_forced ? tree_forced : bh * (S + 1) <= 2 * cus ? 1 : 2;
    }
    pl.NS = f8 ? 4 : 2;                                     // LDS stages (bf16: see below)
    pl.S = (int)S;
    pl.cus = cus;
    pl.G = (dtype == MCSD_BF16 && S > 1 && tree == 1) ? (int)S + 1 : (int)S;
    pl.tree_last = dtype == MCSD_BF16 && S > 1 && tree == 3;
    // Ragged grids larger than the chip are ordered by length inside the kernel (see there)
    pl.pair_cus = 0;
    if (dtype == MCSD_BF16 && pl.G == pl.S && (long)B * pl.S <= 256 && n_cus > 0 && bh * pl.S > n_cus &&
        !(tune && tune->natural_order) && !pl.tree_last)
        pl.pair_cus = n_cus;
    // bf16 tiles: two stages and two workgroups per compute unit.  Four stages (64-key tiles only: a 128-key tile is
    // 64 KB) exist for measurement: on launches that have a compute unit per workgroup anyway three tiles in flight
    // instead of one were expected to help and do not (cfg2: 7.5 against 6.2 us until the partial results are stored;
    // a bare ring of direct-to-LDS loads needs ~5 us for 128 KB per workgroup on 128 compute units at any depth: a
    // cold burst of this size is bound by the memory system's ramp-up, not by the bytes a compute unit has in flight).
    if (tune && !f8 && tune->stages == 4 && dtype == MCSD_BF16 && pl.QBP != 1) pl.NS = 4;
    pl.part_f32 = dtype == MCSD_BF16 && S > 1 && tiles_max * pl.T < PART_F32_KEYS && pl.G <= PART_F32_MAX && (f8 || pl.NS == 2);
    pl.xcc = n_xcc > 0 ? n_xcc : 8;        // unknown: the renumbering is then only a guess that may help locality
    // The fold runs inside the sweep when all workgroups of one (sequence, unit) share a die's L2: the dealing of
    // workgroup ids to dies is known, and the kernel's numbering keeps a unit's workgroups at one id modulo dies.
    // A number of (sequence, unit) pairs that is no multiple of the dies is rounded up: the workgroups of the slots
    // beyond the last pair leave at once, and every real pair's workgroups still share a die.
    pl.grid_units = bh;
    bool same_die = n_xcc == 1;
    if (n_xcc > 1 && pl.pair_cus == 0) {
        same_die = true;
        if (pl.S > 1 || pl.QT > 1) pl.grid_units = (bh + n_xcc - 1) / n_xcc * n_xcc;
        else same_die = bh % n_xcc == 0;
    }
    if (pl.pair_cus > 0) same_die = n_xcc == 1 || (n_xcc > 1 && pl.units % n_xcc == 0 && pl.pair_cus % n_xcc == 0);
    if (pl.xcc & (pl.xcc - 1)) same_die = false;           // (the kernel renumbers by shifts)
    pl.fold = pl.S > 1 && same_die && (dtype == MCSD_F32 || pl.G <= FOLD_MAX_PARTIALS) &&
              (size_t)bh * pl.QT * CTR_STRIDE * sizeof(unsigned long long) <= WS_CTR_BYTES && !(tune && tune->fold == 1);
    return pl;
}

__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Swap the upper 32 lanes of one value with the lower 32 lanes of the other; with both arguments equal the
// pair (r0, r1) holds {own, partner} in some order on every lane, so max / sum across halves is r0 op r1.
__device__ inline float half_swap_max(float v)
{
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float half_swap_sum(float v)
{
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ inline s16x4_t lds_read_tr16(const unsigned char *p)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4_t __attribute__((address_space(3))) *)(p));
}
// 8-bit variant.  Within 16 lanes, lane i receives byte i%8 of the 8-byte words addressed by lanes 2e + i/8,
// e = 0..7 (checked on the hardware): lanes 2e and 2e+1 point at the two halves of a 16-byte piece of the row for
// slot e, and lane i ends up with column i of that piece from all eight rows.
typedef __attribute__((ext_vector_type(2))) int i32x2_t;
__device__ inline i32x2_t lds_read_tr8(const unsigned char *p)
{
    return __builtin_amdgcn_ds_read_tr8_b64_v2i32((i32x2_t __attribute__((address_space(3))) *)(p));
}

// ---------------------------------------------------------------------------------------------------
// bf16 / MFMA kernel
// ---------------------------------------------------------------------------------------------------
// F8: the prefix K/V cache holds fp8 (e4m3) elements; a ring stage is then a raw fp8 tile (half the bytes, twice
// the stages) that the operand reads convert to bf16 on their way into the matrix cores.
template <int D, int QBP, int NS_, bool F8 = false>
struct SweepCfg {
    static constexpr int WAVES = 4;
    static constexpr int KG = 4 / QBP;                 // key groups: wavefronts that share a query block and split the keys
    static constexpr int KPW = QBP == 4 ? 2 : 1;       // 32-key blocks per wavefront per tile
    static constexpr int THREADS = WAVES * 64;
    static constexpr int T = 32 * KG * KPW;            // keys per tile (64, 64, 128 for QBP = 4, 2, 1)
    static constexpr int RB = D * 2;                   // bytes per bf16 K/V row (tree tiles)
    static constexpr int RBP = F8 ? D : D * 2;         // bytes per prefix K/V row (ring stages)
    static constexpr int CPR = RBP / 16;               // 16-byte chunks per prefix row
    static constexpr int RPI = 64 / CPR;               // rows covered by one direct-to-LDS instruction (1 KiB)
    static constexpr int TILE_K = T * RBP;             // bytes of the K half of a ring stage; V follows
    static constexpr int TILE = 2 * TILE_K;
    static constexpr int BTILE_K = T * RB;             // the same for a bf16 tile (the tree's own; beside fp8 stages its halves take one each)
    static constexpr int BCPR = RB / 16;
    static constexpr int NI = T / RPI / WAVES;         // direct-to-LDS instructions per wavefront for K (same for V)
    static constexpr int DPT = 2 * NI;                 // ... per tile
    static constexpr int NS = NS_;                     // LDS stages: one being computed, NS - 1 being filled
    static constexpr int KS = D / 16;                  // k-steps of S^T = K Q^T
    static constexpr int CB = D / 32;                  // 32-row blocks of O^T
    static constexpr int XCHG = (KG - 1) * QBP * 32 * D * 4;   // LDS bytes in which key groups hand over their outputs; maxima and denominators follow
    static constexpr int RING = NS * TILE;
    // Two stages: behind the ring, and where two workgroups' share of a compute unit (80 KB) ends before, over its last halves,
    // lie Q and the first two mask words of every row until they have been read; the first HALVES_FIRST halves of the first two
    // tiles are requested beside them.
    static constexpr int Q_BYTES = QBP * 32 * RB, MASK_BYTES = QBP * 32 * 16;
    static constexpr int LDS_BYTES = NS > 2 ? (RING > XCHG + 1040 ? RING : XCHG + 1040)
                                   : D == 64 || QBP == 1 ? RING + Q_BYTES + MASK_BYTES : 80 * 1024;
    static constexpr int MASK_AT = LDS_BYTES - MASK_BYTES, Q_AT = MASK_AT - Q_BYTES;
    static constexpr int HALVES_FIRST = Q_AT / TILE_K < 4 ? Q_AT / TILE_K : 4;
    static constexpr int PAIR_AT = NS == 2 ? MASK_AT + MASK_BYTES - 2048 : 0;                       // the table that orders ragged grids
    static_assert(NI >= 1 && (NS - 2) * DPT < 64 && LDS_BYTES <= 160 * 1024 && XCHG + 1040 <= LDS_BYTES, "tile does not map onto the workgroup");
    static_assert(NS > 2 || HALVES_FIRST >= 2, "the first tile is requested beside Q");
    static_assert(!F8 || D == 128, "fp8 tiles are laid out for 128-byte rows");
    static_assert(!F8 || (BTILE_K == TILE && BTILE_K / 1024 / WAVES == DPT), "half a tree tile is a slot of the ring");
};

// XOR swizzle of the 16-byte chunk index inside row r.  With it, 16 consecutive rows read at the same logical
// chunk (K operand loads) and 4 consecutive rows read at 4 consecutive chunks (V transpose loads) both hit 16
// different 16-byte bank groups.
template <int D>
__device__ inline int swz(int r)
{
    return D == 128 ? (((r & 3) << 2) | ((r >> 2) & 3)) : ((((r >> 1) & 1) << 2) | ((r >> 2) & 3));
}

// The same for fp8 tiles (128-byte rows, 8 chunks): bijective on row bits 1-3, so 16 consecutive rows read at one
// chunk with 16-byte loads (K operands) hit 16 different bank groups together with the row's parity, and the rows
// {0..3, 8..11} + 4g read at two neighbouring chunks by the transpose loads (V operands) do as well.
__device__ inline int swz8(int r)
{
    return ((r >> 2) & 1) | (((r >> 1) & 1) << 1) | (((r >> 3) & 1) << 2);
}

// 8 fp8 (e4m3, OCP) values in two dwords -> 8 bf16, exact.
__device__ inline bf16x8_t fp8x8_to_bf16(unsigned lo, unsigned hi)
{
    typedef __attribute__((ext_vector_type(4))) unsigned u4;
    u4 w;
    w[0] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, false));
    w[1] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, true));
    w[2] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, false));
    w[3] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, true));
    return __builtin_bit_cast(bf16x8_t, w);
}

// Log2-domain slack of the running reference maximum: the accumulators are rescaled only when a block's maximum
// exceeds the reference by more than this, so exponentiated scores stay below 2^RESCALE_SLACK.  The result is
// exact: numerator and denominator always share the same reference.
constexpr float RESCALE_SLACK = 6.f;

// Per-lane LDS offsets of the two operand read patterns inside a stage (computed once).
struct LaneAddr {
    int k;   // K operand: row (kg*32 + ln), chunk g ^ swz; XOR ks*32 selects the k-step
    int v;   // V^T operand: row (kg*32 + 4g + j/4), chunk/sub of this lane; XOR ct*16 and an immediate select the rest
    int k8;  // the same inside an fp8 tile: row (kg*32 + ln), chunk g ^ swz8; XOR kp*32 selects the pair of k-steps
    int v8;  // fp8 V^T operand (8-bit transpose load): row of this lane's key slot, chunk (ln/16) ^ swz8, half ln & 1
};

// State of one 32-query block held by a wavefront.
template <int D>
struct QBlock {
    bf16x8_t q[D / 16];        // Q as B operands: lane holds Q[row][ks*16 + 8g .. +8]
    f32x16_t o[D / 32];        // O^T accumulators
    float m_ref, l_run;        // reference maximum (raw score units), per-lane part of the denominator
};

// Exponentials of one pair of scores: p = exp2(s*c - mc), added to the denominator and packed as bf16 into P^T
// (kept as dwords: pb[r/8] is one B operand).  The empty asm keeps the pair where it is written, between two MFMAs.
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4_t;
// SCALED: the packed values carry the factor vs (the scale of an fp8 V tile); the denominator does not.
template <bool SCALED = false>
__device__ inline void softmax_exp2(const f32x16_t &sacc, int r, float c, float mc, float &psum, u32x4_t *pb, float vs = 1.f)
{
    const float p0 = fast_exp2(fmaf(sacc[r], c, -mc)), p1 = fast_exp2(fmaf(sacc[r + 1], c, -mc));
    psum += p0 + p1;
    bf16x2_t pk;
    pk[0] = (__bf16)(SCALED ? p0 * vs : p0);
    pk[1] = (__bf16)(SCALED ? p1 * vs : p1);
    unsigned u = __builtin_bit_cast(unsigned, pk);
    asm volatile("" : "+v"(u));
    pb[r / 8][(r % 8) / 2] = u;
}

// One tile: the wavefront's KPW blocks of 32 keys against its 32 queries.  With two blocks the instruction stream
// is laid out so that the matrix pipe and the vector ALU overlap inside the wavefront:
//     QK_0, QK_1 | block maxima, rare rescale | exp(0) | PV_0 with exp(1) in its shadow | PV_1
// Operand reads are issued ahead of their use.  MODE 0: all keys visible; MODE 1: bit k of bits[u] says whether
// key k of block u is visible to this lane's query; MODE 2: the one or the other, as `masked` (uniform) says.
// F8K: the kernel serves an fp8 prefix cache: the reference maximum is kept in log2 units (tiles of different
// scale share it) and P carries the V scale `vs` of the tile.  F8T: this stage is a raw fp8 tile.
// `values` is called when the scores are under way and before the first value is read.
struct NothingToDo { __device__ void operator()() const {} };
template <int D, int QBP, int NS, int MODE, bool F8K = false, bool F8T = false, typename Values = NothingToDo>
__device__ __forceinline__ void attn_tile(const unsigned char *stage, const LaneAddr la, QBlock<D> &qs, float c, int g,
                                          const uint32_t *bits, float vs = 1.f, const unsigned char *vstage = nullptr,
                                          bool masked = false, Values values = Values())
{
    using C = SweepCfg<D, QBP, NS, F8K>;
    constexpr int U = C::KPW;
    constexpr int ROWB = F8T ? C::RBP : C::RB;             // bytes per row of this stage
    constexpr int VOFF = F8T ? C::TILE_K : C::BTILE_K;     // where its V half starts
    // K rows of the blocks (A operands of S^T = K Q^T); block u sits 32*u rows below the lane's base row
    bf16x8_t kf[U][C::KS];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if constexpr (F8T) {
            // one 16-byte read = the lane's share of two k-steps (see the column order in the kernel)
#pragma unroll
            for (int kp = 0; kp < C::KS / 2; ++kp) {
                const uint4 raw = *(const uint4 *)(stage + (la.k8 ^ (kp * 32)) + u * 32 * ROWB);
                kf[u][2 * kp] = fp8x8_to_bf16(raw.x, raw.y);
                kf[u][2 * kp + 1] = fp8x8_to_bf16(raw.z, raw.w);
            }
        } else {
#pragma unroll
            for (int ks = 0; ks < C::KS; ++ks)
                kf[u][ks] = *(const bf16x8_t *)(stage + (la.k ^ ((F8K ? 4 * (ks >> 1) + (ks & 1) : 2 * ks) * 16)) + u * 32 * ROWB);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // S^T[key][query] : lane (query = ln, half g) gets keys 8*(r/4) + 4*g + r%4, r = 0..15
    f32x16_t sacc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        // The wavefront's runs of matrix instructions are issued at raised priority: the other wavefront of the SIMD,
        // busy with its soft-max, then does not delay them (measured: 2-3 % on the long sweeps; the opposite
        // assignment costs as much).
        if (u == 0) __builtin_amdgcn_s_setprio(2);
        sacc[u] = (f32x16_t){0};
#pragma unroll
        for (int ks = 0; ks < C::KS; ++ks) sacc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[u][ks], qs.q[ks], sacc[u], 0, 0, 0);
    }
    __builtin_amdgcn_s_setprio(0);
    values();
    // V^T fragments via the LDS transpose load, issued ahead of their use: block 0's during the softmax, block 1's
    // before the first PV MFMA.  The reads of one k-step pair (ks2, e4) sit 16*ks2 + 8*e4 rows below the lane's
    // base row; the chunk select is cb*4 ^ e4*2.
    const unsigned char *vst = vstage ? vstage : stage + VOFF;   // (null or not at compile time)
    bf16x8_t vf[U][2][C::CB];
    auto read_v = [&](int u) {
#pragma unroll
        for (int ks2 = 0; ks2 < 2; ++ks2)
#pragma unroll
            for (int cb = 0; cb < C::CB; ++cb) {
                if constexpr (F8T) {
                    // one 8-bit transpose load: the 8 key slots of this lane's column (slot e = key 8(e/4) + 4g + e%4)
                    const i32x2_t t = lds_read_tr8(vst + (la.v8 ^ ((cb * 2) * 16)) + (u * 32 + ks2 * 16) * ROWB);
                    vf[u][ks2][cb] = fp8x8_to_bf16((unsigned)t[0], (unsigned)t[1]);
                } else {
                    const s16x4_t lo = lds_read_tr16(vst + (la.v ^ (((cb * 4) ^ 0) * 16)) + (u * 32 + ks2 * 16) * ROWB);
                    const s16x4_t hi = lds_read_tr16(vst + (la.v ^ (((cb * 4) ^ 2) * 16)) + (u * 32 + ks2 * 16 + 8) * ROWB);
                    vf[u][ks2][cb] = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                }
            }
    };
    read_v(0);
    // masking, maximum over the tile's blocks, rare rescale of the accumulators
    float mx = -INFINITY;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (MODE == 1 || (MODE == 2 && masked)) {
            // Bits at constant places, spread over the register and blended: two instructions per score.  (Comparing and selecting
            // took four, one of them a wait for the condition: 0.1-0.3 us of a call of a tile or two.)
            const uint32_t own = bits[u] >> (4 * g);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const uint32_t seen = (uint32_t)__builtin_amdgcn_sbfe((int)own, 8 * (r / 4) + r % 4, 1);       // all ones or zero
                sacc[u][r] = __uint_as_float((__float_as_uint(sacc[u][r]) & seen) | (0xff800000u & ~seen));
            }
        }
        mx = fmaxf(fmaxf(mx, sacc[u][0]), sacc[u][1]);
#pragma unroll
        for (int r = 2; r < 16; r += 2) mx = fmaxf(fmaxf(mx, sacc[u][r]), sacc[u][r + 1]);
    }
    mx = half_swap_max(mx);
    if (F8K) mx *= c;                                       // log2 units from here on (c > 0)
    const float cm = F8K ? 1.f : c;                         // what turns a difference of reference maxima into log2 units
    // rescale only when the maximum outgrows the reference by more than the slack (first tile: -inf)
    const bool grow = (mx - qs.m_ref) * cm > RESCALE_SLACK;
    if (__builtin_amdgcn_ballot_w64(grow) != 0) {
        const float m_new = grow ? mx : qs.m_ref;
        const float alpha = m_new == qs.m_ref ? 1.f : fast_exp2((qs.m_ref - m_new) * cm);   // -inf reference: exp2(-inf) = 0
        qs.m_ref = m_new;
        qs.l_run *= alpha;
#pragma unroll
        for (int cb = 0; cb < C::CB; ++cb)
#pragma unroll
            for (int r = 0; r < 16; ++r) qs.o[cb][r] *= alpha;
    }
    const float mc = (qs.m_ref == -INFINITY ? 0.f : qs.m_ref) * cm;
    u32x4_t pb[U][2];
    float psum = 0.f;
    // With one block per wavefront the exponentials of its second half of keys (registers 8..15, the operand of the
    // second k-step pair) run in the shadow of the first half's PV MFMAs.
#pragma unroll
    for (int r = 0; r < (U == 1 ? 8 : 16); r += 2) softmax_exp2<F8K>(sacc[0], r, c, mc, psum, pb[0], vs);
    __builtin_amdgcn_sched_barrier(0);
    // O^T[c][query] += V^T[c][key] * P^T[key][query]
    if (U == 1) {
#pragma unroll
        for (int cb = 0; cb < C::CB; ++cb) {
            qs.o[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[0][0][cb], __builtin_bit_cast(bf16x8_t, pb[0][0]), qs.o[cb], 0, 0, 0);
            if (C::CB == 4) softmax_exp2<F8K>(sacc[0], 8 + 2 * cb, c, mc, psum, pb[0], vs);
            else { softmax_exp2<F8K>(sacc[0], 8 + 4 * cb, c, mc, psum, pb[0], vs); softmax_exp2<F8K>(sacc[0], 10 + 4 * cb, c, mc, psum, pb[0], vs); }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int cb = 0; cb < C::CB; ++cb)
            qs.o[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[0][1][cb], __builtin_bit_cast(bf16x8_t, pb[0][1]), qs.o[cb], 0, 0, 0);
        qs.l_run += psum;
        return;
    }
    if (U == 2) {
        read_v(1);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(2);
#pragma unroll
        for (int i = 0; i < 2 * C::CB; ++i) {
            const int ks2 = i / C::CB, cb = i % C::CB;
            qs.o[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[0][ks2][cb], __builtin_bit_cast(bf16x8_t, pb[0][ks2]), qs.o[cb], 0, 0, 0);
            if (C::CB == 4) softmax_exp2<F8K>(sacc[U - 1], 2 * i, c, mc, psum, pb[U - 1], vs);
            else { softmax_exp2<F8K>(sacc[U - 1], 4 * i, c, mc, psum, pb[U - 1], vs); softmax_exp2<F8K>(sacc[U - 1], 4 * i + 2, c, mc, psum, pb[U - 1], vs); }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int ks2 = 0; ks2 < 2; ++ks2)
#pragma unroll
        for (int cb = 0; cb < C::CB; ++cb)
            qs.o[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[U - 1][ks2][cb], __builtin_bit_cast(bf16x8_t, pb[U - 1][ks2]), qs.o[cb], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    qs.l_run += psum;
}

// What a workgroup of the sweep needs before it can ask for its first key comes as the kernel's leading scalar arguments,
// which the hardware preloads into registers (see the build's kernarg-preload option), and its place in the grid follows
// without integer division (some 50 dependent instructions each): multiplication by a reciprocal that the host rounded up,
// floor(a / d) = a * mul >> (31 + shift) for 0 <= a < 2^31 with shift = ceil(log2 d), mul = ceil(2^(31 + shift) / d).
// Measured, start of a workgroup to its prefix length known: 1.45 us without.
struct FastDiv { uint32_t mul, shift; };
inline FastDiv fast_div_of(uint32_t d)
{
    FastDiv f = {0, 0};
    while ((1ull << f.shift) < d) ++f.shift;
    f.mul = (uint32_t)(((1ull << (31 + f.shift)) + d - 1) / d);
    return f;
}
__device__ __forceinline__ int fast_div(int a, uint32_t mul, uint32_t shift) { return (int)(((uint64_t)(uint32_t)a * mul) >> (31 + shift)); }
// `how`: bits 0-4 shift of G, 5-9 shift of H, 10-13 log2 of the dies, and flags
constexpr uint32_t HOW_RENUMBER = 1u << 14, HOW_PAIR = 1u << 15;
__device__ __forceinline__ uint32_t how_shift_G(uint32_t how) { return how & 31u; }
__device__ __forceinline__ uint32_t how_shift_H(uint32_t how) { return (how >> 5) & 31u; }
__device__ __forceinline__ uint32_t how_xcc(uint32_t how) { return (how >> 10) & 15u; }

// The fold of the partial results of one query block by one wavefront of the workgroup that arrived last (see the
// end of the sweep kernel): rows = the wavefront's 32 queries (lane ln, half g), columns = the 32-column blocks
// kg, kg + KG, ..  ro / rm / rl describe the unit's partial O (fragment order), maxima and denominators and end after
// the last partial result in use: a load beyond it returns zero without touching memory, so nothing below branches
// on the number of partial results and all loads of a round are in flight together.
// A round: NSLOT partial results x the lane's two 16-byte chunks (jp = 0, 1: eight bf16 each = its float4 positions
// j = 2 jp, 2 jp + 1) of a column block.  The rounds of a column block are (first group), [(second group)]: an
// accumulator lives across the groups and its result is stored after every round (with two groups the first store
// of a position is overwritten by the complete one: same lane, same address, program order).  The loads of the next
// round are issued before this one is added up (two register buffers); a round beyond the last loads from beyond the
// end, i.e. nothing, and is not added up.
// PF32: the partial O are fp32.  A round is then one half of a column block (the same 16-byte chunks, four columns each), and
// all partial results are one group.
// Partial results are added in slot order whoever arrived last, so the result is reproducible.
// Nothing here may spill: a workgroup's scratch memory is cold at this point, every first touch a trip to HBM (a
// variant that spilled its weights took 9.7 us for five partial results, against 3).
template <int D, int QBP, int KG, int NSLOT, bool PF32 = false>
__device__ __attribute__((always_inline)) inline void fold_partials(const __amdgpu_buffer_rsrc_t ro, const __amdgpu_buffer_rsrc_t rm,
                                     const __amdgpu_buffer_rsrc_t rl, const int n_active, const int kg, const int g,
                                     const int ln, const float cm, __bf16 *orow, f32x4_t *wlds)
{
    constexpr int CB = D / 32;
    constexpr int NW = NSLOT == 8 ? FOLD_MAX_PARTIALS : NSLOT;      // partial results this variant can hold
    constexpr int SLOT_BYTES = QBP * 32 * D * (PF32 ? 4 : 2);
    static_assert(!PF32 || NSLOT <= PART_F32_MAX, "one group");
    float wgt[NW], lw[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        wgt[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rm, (i * QBP * 32 + ln) * 4, 0, 1));
        lw[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rl, (i * QBP * 32 + ln) * 4, 0, 1));
    }
    const int ngrp = NSLOT == 8 && n_active > NSLOT ? 2 : 1;
    const int rounds = ((CB - kg + KG - 1) / KG) * (PF32 ? 2 : ngrp);
    typedef u32x4_t Round[NSLOT][2];
    auto issue = [&](Round &buf, int r) {
        const int grp = r % ngrp, cb = kg + (PF32 ? r >> 1 : r / ngrp) * KG;
        int off = PF32 ? ((cb * 8 + (r & 1) * 4 + g) * 32 + ln) * 16 : ((cb * 4 + g) * 32 + ln) * 16 + grp * NSLOT * SLOT_BYTES;
        if (r >= rounds) off = 0x40000000;                          // (uniform select) beyond every workspace
#pragma unroll
        for (int i = 0; i < NSLOT; ++i)
#pragma unroll
            for (int jp = 0; jp < 2; ++jp) buf[i][jp] = __builtin_amdgcn_raw_buffer_load_b128(ro, off + jp * 1024 + i * SLOT_BYTES, 0, 1);
    };
    Round bufA, bufB;
    issue(bufA, 0);
    float M = -INFINITY;
#pragma unroll
    for (int i = 0; i < NW; ++i) M = fmaxf(M, i < n_active ? wgt[i] : -INFINITY);
    float den = 0.f;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        // 0 for a split that saw no visible key, and beyond the partial results in use
        wgt[i] = i < n_active ? fast_exp2((wgt[i] - M) * cm) : 0.f;
        den = fmaf(wgt[i], lw[i], den);
    }
    const float inv = 1.f / den;
    // Two groups: a round picks its group at run time, and registers cannot be indexed at run time, so the weights
    // go through LDS (the ring is free by now), written and read back by the same lane.
    if constexpr (NSLOT == 8) {
#pragma unroll
        for (int q4 = 0; q4 < NW / 4; ++q4)
            wlds[q4 * 256] = (f32x4_t){wgt[4 * q4], wgt[4 * q4 + 1], wgt[4 * q4 + 2], wgt[4 * q4 + 3]};
    }
    f32x4_t acc[4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    auto add_up = [&](Round &buf, int r) {
        if constexpr (PF32) {
            const int cb = kg + (r >> 1) * KG;
#pragma unroll
            for (int jp = 0; jp < 2; ++jp) {
                f32x4_t a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < NSLOT; ++i) a += wgt[i] * __builtin_bit_cast(f32x4_t, buf[i][jp]);        // slot order
                bf16x4_t v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = (__bf16)(a[e] * inv);
                *(bf16x4_t *)(orow + cb * 32 + 16 * (r & 1) + 8 * jp + 4 * g) = v;
            }
            return;
        }
        const int grp = r % ngrp, cb = kg + (r / ngrp) * KG;
        float w[NSLOT];
        if constexpr (NSLOT == 8) {
            const f32x4_t wa = wlds[(2 * grp) * 256], wb = wlds[(2 * grp + 1) * 256];
#pragma unroll
            for (int i = 0; i < 4; ++i) { w[i] = wa[i]; w[4 + i] = wb[i]; }
        } else {
#pragma unroll
            for (int i = 0; i < NSLOT; ++i) w[i] = wgt[i];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {                               // the lane's float4 position j of this column block
            if (grp == 0) acc[j] = (f32x4_t){0.f, 0.f, 0.f, 0.f};   // a new position starts from zero (a select)
#pragma unroll
            for (int i = 0; i < NSLOT; ++i) {                       // slot order
                const unsigned d0 = buf[i][j >> 1][2 * (j & 1)], d1 = buf[i][j >> 1][2 * (j & 1) + 1];   // four bf16: exact as fp32 bit patterns
                const u32x4_t bits = {d0 << 16, d0 & 0xffff0000u, d1 << 16, d1 & 0xffff0000u};
                acc[j] += w[i] * __builtin_bit_cast(f32x4_t, bits);
            }
            bf16x4_t v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (__bf16)(acc[j][e] * inv);
            *(bf16x4_t *)(orow + cb * 32 + 8 * j + 4 * g) = v;
        }
    };
#pragma unroll 1
    for (int r = 0; r < rounds; r += 2) {
        issue(bufB, r + 1);
        __builtin_amdgcn_sched_barrier(0);
        add_up(bufA, r);
        __builtin_amdgcn_sched_barrier(0);
        issue(bufA, r + 2);
        __builtin_amdgcn_sched_barrier(0);
        if (r + 1 < rounds) add_up(bufB, r + 1);                    // (uniform)
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Whether there is a kernel for grids of long and short workgroups in pairs.  Not for four query blocks, where a second loop
// does not fit the registers (40 of them spilled), nor for split keys (16 x 16 heads, 851-3407 keys: 53.4 us without, 56.1 with
// it), nor where a workgroup has the compute unit to itself anyway.  What it serves by the plan's own choice: unsplit grids of more
// units than compute units and at most twice as many, that is twice as many (16 sequences of 32 heads) for prefixes of eight tiles
// and more, which are halved between, and any number for shorter ones.  16 sequences of 512-4096 keys, 32 heads, 60 nodes, 20
// draws of the lengths: 7-16 % faster with it for 17, 1-2 % slower for the 3 whose longest pair has two long members.
template <int D, int QBP, int NS, bool F8>
constexpr bool has_ragged_kernel() { return NS == 2 && !F8 && QBP != 4 && !(D == 128 && QBP == 1); }

// PF32: partial O as fp32 (see PART_F32_KEYS).  RAGGED: a grid of such pairs.
template <int D, int QBP, int NS, bool F8, bool PF32, bool RAGGED>
__device__ __forceinline__ void sweep(const int32_t *lens, const int64_t *seq_base, const uint32_t per_die, const int32_t G, const uint32_t mul_G,
                                      const int32_t H, const uint32_t mul_H, const int32_t BH, const uint32_t how, const int32_t max_prefix,
                                      const int32_t tps, const AttnParams &p)
{
    using C = SweepCfg<D, QBP, NS, F8>;
    __shared__ __attribute__((aligned(1024))) unsigned char ring[C::LDS_BYTES];

    // Workgroup ids are dealt round-robin to the accelerator dies (p.xcc of them, each with its own L2): renumber so
    // that the key splits of one (sequence, head), which read the same Q, tree K/V and mask rows, write neighbouring
    // partial results and fold them through that L2, share one die.
    int wg = blockIdx.x;
    if (how & HOW_RENUMBER) wg = (wg & ((1 << how_xcc(how)) - 1)) * per_die + (wg >> how_xcc(how));
    int bhi = fast_div(wg, mul_G, how_shift_G(how));
    int s = wg - bhi * G;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // the same in all lanes: keep it in a scalar register
    // The rest of the argument block is needed here, before the loads below leave: scalar loads come back in any order, so a
    // wait for one is a wait for all.
    asm("" : "+s"(bhi) : "s"(p.q), "s"(p.kt), "s"(p.vt), "s"(p.kp), "s"(p.vp), "s"(p.mask_bits), "s"(p.mask_words), "s"(p.n), "s"(p.Hq),
        "s"(p.Hkv), "s"(p.grp), "s"(p.hpw), "s"(p.bph), "s"(p.chunks), "s"(p.mul_chunks), "s"(p.shift_chunks), "s"(p.log2_bph),
        "s"(p.S), "s"(p.tree_last), "s"(p.row0), "s"(p.node_stride), "s"(p.head_stride), "s"(p.mul_tps), "s"(p.shift_tps));
    // Two tiles' halves are kept under way by a workgroup that will have its compute unit to itself: one query block of 128
    // columns always (its stages fill the LDS), the long one of a pair while the short one is at least a fifth shorter.
    bool alone = NS == 2 && !PF32 && D == 128 && QBP == 1;
    if (how & HOW_PAIR) {
        const int total = gridDim.x;
        // More workgroups than compute units.  Up to two per compute unit they are all resident at once, and on this
        // machine workgroups i and i + #CUs of such a grid land on the same compute unit (measured; nothing but
        // speed depends on it): that pair gets a long and a short piece of work, so that every compute unit has
        // about the same number of keys to stream however ragged the batch is.  With more than two per compute unit
        // the hardware hands out workgroups in id order as slots free up: longest first.  The pieces are the
        // (sequence, key split) classes, p.H equal items each, ranked by their number of tiles here (B * S <= 256).
        typedef __attribute__((address_space(3))) int32_t lds_int;
        lds_int *const s_work = (lds_int *)(ring + C::PAIR_AT), *const s_cls_at = s_work + 256;
        const int n_cls = p.B * p.S;
        if (tid < n_cls) {
            const int Lt = p.lens[tid / p.S], sp = tid % p.S;
            const int Lc = Lt < 0 ? 0 : (Lt > p.max_prefix ? p.max_prefix : Lt);
            const int tl = (Lc + C::T - 1) / C::T - sp * p.tps;
            s_work[tid] = (tl < 0 ? 0 : (tl > p.tps ? p.tps : tl)) + (sp == 0 ? (p.n + C::T - 1) / C::T : 0);
        }
        __syncthreads();
        if (tid < n_cls) {
            int rank = 0;
            for (int o = 0; o < n_cls; ++o) rank += (s_work[o] > s_work[tid]) || (s_work[o] == s_work[tid] && o < tid);
            s_cls_at[rank] = tid;
        }
        __syncthreads();
        // rank i with rank total-1-i, in groups of p.xcc ids so that a rank keeps its id modulo the number of dies
        // (every key split of a (sequence, unit) then runs on the die of unit % dies)
        int r = wg, r_other = total;                                             // longest first
        if (total <= 2 * p.pair_cus) {
            const int w2 = wg >= p.pair_cus ? wg - p.pair_cus : wg, cnt = total - p.pair_cus;
            const int second = (cnt % p.xcc == 0) ? p.pair_cus + (cnt / p.xcc - 1 - w2 / p.xcc) * p.xcc + w2 % p.xcc : total - 1 - w2;
            if (wg >= p.pair_cus) r = second;
            else if (wg < cnt) r_other = second;
        }
        const int rank = fast_div(r, mul_H, how_shift_H(how));
        const int cls = __builtin_amdgcn_readfirstlane(s_cls_at[rank]);
        if (RAGGED && wg < p.pair_cus) {
            const int others = r_other < total ? s_work[s_cls_at[fast_div(r_other, mul_H, how_shift_H(how))]] : 0;
            alone = __builtin_amdgcn_readfirstlane(4 * s_work[cls]) > 5 * __builtin_amdgcn_readfirstlane(others);
        }
        __syncthreads();                                     // (the first loads land there)
        s = cls % p.S;
        // Units that stream the same keys for different query heads are neighbours: give them one die, and so one L2 (a die's
        // share of a class is then H / dies neighbours; ids modulo the dies stay what they were for every split of a unit).
        int unit = r - rank * H;
        const int xb = how_xcc(how);
        if (p.chunks > 1 && (H & ((1 << xb) - 1)) == 0) unit = (unit & ((1 << xb) - 1)) * (H >> xb) + (unit >> xb);
        bhi = (cls / p.S) * H + unit;
    }
    bhi = __builtin_amdgcn_readfirstlane(bhi);              // (uniform, and the compiler has to know)
    s = __builtin_amdgcn_readfirstlane(s);
    if (bhi >= BH) return;                                   // a slot of a grid rounded up to whole dies
    const int b = fast_div(bhi, mul_H, how_shift_H(how)), h = bhi - b * H;

    const int g = lane >> 5, ln = lane & 31;
    const int qb = wave % QBP, kg = wave / QBP;

    int L = lens[b];
    int64_t seq_at = seq_base[b];
    __builtin_amdgcn_sched_barrier(0);
    const int64_t bh = bhi;                                  // workgroup unit: indexes the partial results
    const int kvh = fast_div(h, p.mul_chunks, p.shift_chunks); // key/value head of this unit
    const int hq = kvh * p.grp + (h - kvh * p.chunks) * p.hpw + (qb >> p.log2_bph);   // query head of this wavefront's block
    const int64_t bh_kv = (int64_t)b * p.Hkv + kvh, bh_q = (int64_t)b * p.Hq + hq;
    const __bf16 *q = (const __bf16 *)p.q + bh_q * p.node_stride * D;
    const __bf16 *kt = (const __bf16 *)p.kt + bh_kv * p.node_stride * D;
    const __bf16 *vt = (const __bf16 *)p.vt + bh_kv * p.node_stride * D;
    // Query block of this wavefront; mask row of this lane's query.  A padded row (beyond the last) is the last one again, unwritten.
    QBlock<D> qs;
    const int qrow = p.row0 + (qb & (p.bph - 1)) * 32 + ln, qclamped = min(qrow, p.n - 1);
    uint64_t mrow[2] = {0, 0};
    if constexpr (NS == 2) {
        // Through LDS, in the layout of the keys: every row comes once and whole, where each wavefront of a query block would
        // fetch it for itself in pieces of 32 bytes, and the compiler, which knows nothing of the tiles' loads and would wait
        // for all of them where Q is first used, has nothing to wait for.  (Q in registers and two tiles requested at once:
        // 14.2 us where this takes 13.7, and nothing gained where a workgroup has one tile.)
        const int hq0 = kvh * p.grp + (h - kvh * p.chunks) * p.hpw;
#pragma unroll
        for (int j = 0; j < C::Q_BYTES / 1024 / C::WAVES; ++j) {
            const int piece = j * C::WAVES + wave, r = piece * (1024 / C::RB) + lane / C::BCPR, qbr = piece * (1024 / C::RB) >> 5;
            const int node = min(p.row0 + (qbr & (p.bph - 1)) * 32 + (r & 31), p.n - 1);
            const int64_t row = ((int64_t)b * p.Hq + hq0 + (qbr >> p.log2_bph)) * p.node_stride + node;
            load_to_lds16_at((const unsigned char *)p.q + row * C::RB + ((lane % C::BCPR) ^ swz<D>(r)) * 16, ring + C::Q_AT + piece * 1024);
        }
        // (rows are as long as the full mask's, which may have more words than the at most 128 columns in use)
#pragma unroll
        for (int j = 0; j * C::WAVES < C::MASK_BYTES / 256; ++j) {
            const int piece = j * C::WAVES + wave, i = piece * 64 + lane;                    // dword i % 4 of row i / 4
            const int64_t at = (int64_t)min(p.row0 + (i >> 2), p.n - 1) * p.mask_words * 2 + min(i & 3, p.mask_words * 2 - 1);
            if (C::MASK_BYTES / 256 % C::WAVES == 0 || piece < C::MASK_BYTES / 256)
                load_to_lds4_at((const uint32_t *)p.mask_bits + at, ring + C::MASK_AT + piece * 256);
        }
    } else {
#pragma unroll
        for (int ks = 0; ks < C::KS; ++ks) {
            // Columns of k-step ks in lane half g: 16 ks + 8 g .. +7.  With an fp8 prefix cache the halves trade places
            // with the k-step's parity, 32 (ks/2) + 16 g + 8 (ks%2) .. +7, so that a lane's columns of two consecutive
            // k-steps are 16 consecutive bytes of an fp8 row (one conflict-free 16-byte LDS read); the contraction is
            // over all columns either way.
            const int col = F8 ? (ks >> 1) * 32 + g * 16 + (ks & 1) * 8 : ks * 16 + g * 8;
            qs.q[ks] = *(const bf16x8_t *)(q + (int64_t)qclamped * D + col);
        }
        // (rows are as long as the full mask's, which may have more words than the at most 128 columns in use)
        mrow[0] = p.mask_bits[(int64_t)qclamped * p.mask_words];
        mrow[1] = p.mask_bits[(int64_t)qclamped * p.mask_words + (p.mask_words > 1)];
    }
    asm volatile("" ::: "memory");                          // (requested here, not where they are first used)
#pragma unroll
    for (int cb = 0; cb < C::CB; ++cb) qs.o[cb] = (f32x16_t){0};
    qs.m_ref = -INFINITY;
    qs.l_run = 0.f;

    // operand read offsets of this lane inside a stage; its first key block starts at row kg * KPW * 32
    LaneAddr la;
    {
        const int krow = kg * C::KPW * 32 + ln;
        la.k = krow * C::RB + (((F8 ? 2 * g : g) ^ swz<D>(krow)) * 16);     // bf16 chunk of (k-step 0, half g)
        const int j = ln & 15, grp = ln >> 4, jr = j >> 2;
        const int vrow = kg * C::KPW * 32 + 4 * g + jr;               // + 32*u + 16*ks2 + 8*e4 by immediate
        const int lchunk = grp * 2 + ((j & 3) >> 1);                   // + 4*cb
        // swz(vrow + 32*u + 16*ks2 + 8*e4) = swz(vrow) ^ (e4 << 1): the e4 part is folded into the compile-time XOR
        la.v = vrow * C::RB + ((lchunk ^ swz<D>(vrow)) * 16) + (j & 1) * 8;
        la.k8 = la.v8 = 0;
        if constexpr (F8) {
            la.k8 = krow * C::RBP + ((g ^ swz8(krow)) * 16);
            const int e = j >> 1;                                        // key slot this lane addresses
            const int row8 = kg * C::KPW * 32 + 8 * (e >> 2) + 4 * g + (e & 3);
            la.v8 = row8 * C::RBP + ((grp ^ swz8(row8)) * 16) + (j & 1) * 8;
        }
    }
    // Lane's source offset inside a tile for instruction 0: row wave * RPI + lane / CPR, logical chunk (lane % CPR) ^ swz(row);
    // instruction i covers the rows i * WAVES * RPI further down, whose swizzle is the same.
    constexpr int STEP = C::WAVES * C::RPI;
    const int row0 = wave * C::RPI + lane / C::CPR;
    const uint32_t goff = (uint32_t)(row0 * C::RBP + (((lane % C::CPR) ^ (F8 ? swz8(row0) : swz<D>(row0))) * 16));
    uint32_t goffs[C::NI];                                  // (registers rather than scalar additions per load: 1.5 % of the long sweeps)
#pragma unroll
    for (int i = 0; i < C::NI; ++i) {
        goffs[i] = goff + (uint32_t)(i * STEP * C::RBP);
        asm volatile("" : "+v"(goffs[i]));
    }
    static_assert(STEP % (F8 || D == 128 ? 16 : 8) == 0, "the swizzle repeats");
    asm volatile("" : "+v"(la.k), "+v"(la.v));
    asm volatile("" : "+s"(L), "+s"(seq_at));               // (keeps everything above where it is)
    L = L < 0 ? 0 : (L > max_prefix ? max_prefix : L);
    const int tiles_b = (int)((unsigned)(L + C::T - 1) / C::T);   // (tps is fixed per call: short sequences use fewer splits)
    const bool sep = G > p.S;                               // the tree's own keys have a workgroup of their own
    const int np = fast_div(tiles_b + tps - 1, p.mul_tps, p.shift_tps);   // prefix splits that have keys for this sequence (<= S)
    const bool tree_wg = sep ? s == p.S : s == (p.tree_last ? max(np, 1) - 1 : 0);
    const int t0 = (sep && tree_wg) ? tiles_b : min(s * tps, tiles_b), t1 = min(t0 + tps, tiles_b);
    const int n_tree_tiles = tree_wg ? (p.n + C::T - 1) / C::T : 0;
    const int n_pre = t1 - t0;
    if (n_pre + n_tree_tiles == 0) return;                  // this split has no keys (the program's end waits for Q and the masks)
    const int n_active = sep ? np + 1 : max(1, np);         // partial results of this sequence: slots 0 .. n_active-1
    const int slot_id = (sep && tree_wg) ? np : s;
    // leading tiles of this split that are full (only the sequence's last tile can be ragged)
    const int n_hot = (n_pre > 0 && t1 * C::T > L) ? n_pre - 1 : n_pre;

    const int64_t pre0 = seq_at + (int64_t)kvh * p.head_stride;     // in elements: 2 bytes each, 1 when fp8
    const unsigned char *kp = (const unsigned char *)p.kp + pre0 * (F8 ? 1 : 2);
    const unsigned char *vp = (const unsigned char *)p.vp + pre0 * (F8 ? 1 : 2);
    // softmax scale of a prefix tile and the factor its V values carry; the tree's own tiles use p.c and 1
    const float c_pre = F8 ? p.c * p.k_scale : p.c, vs_pre = F8 ? p.v_scale : 1.f;

    uint32_t all_keys[C::KPW];
#pragma unroll
    for (int u = 0; u < C::KPW; ++u) all_keys[u] = 0xffffffffu;

    // ---- keys: HBM -> LDS directly, NS - 1 tiles ahead of the compute ----
    // Every workgroup walks its full tiles in a rotated order (soft-max does not care): workgroups that start
    // together would otherwise sweep their equally aligned K/V streams in lock-step and crowd the same
    // memory channels.  `nxt` is the full tile the next request fetches.
    // Workgroups that stream the same keys for different query heads keep step instead: the second finds them in L2
    // (16 sequences of 512-4096 keys, 32 query heads over 8: 69 -> 65 us).
    const unsigned turn = p.chunks == 1 ? (unsigned)wg : (unsigned)((int)bh_kv * G + s);
    int nxt = (int)(((turn * 37u) & 127u) * (unsigned)n_hot >> 7);
    const unsigned char *ksrc = kp + (int64_t)t0 * C::TILE_K, *vsrc = vp + (int64_t)t0 * C::TILE_K;
    // (uniform tile base + 32-bit lane offset: a load takes its base from scalar registers)
    const unsigned char *kbase = ksrc + (int64_t)nxt * C::TILE_K, *vbase = vsrc + (int64_t)nxt * C::TILE_K;
    const bool read_once = p.chunks == 1;                   // no other workgroup streams these keys (uniform)
    constexpr std::integral_constant<int, 0> KEYS;
    constexpr std::integral_constant<int, 1> VALUES;
    constexpr std::integral_constant<int, 2> BOTH;
    auto issue_full = [&](unsigned char *stage, auto half) __attribute__((always_inline)) {      // (the values come last)
        constexpr int HALF = decltype(half)::value, PER = HALF == 2 ? 2 : 1;
        stage += wave * 1024;
        if (read_once) {
#pragma unroll
            for (int i = 0; i < PER * C::NI; ++i) {
                const int w = HALF == 2 ? (i & 1) : HALF, j = i / PER;
                load_to_lds16<true>(w ? vbase : kbase, goffs[j], stage + w * C::TILE_K + j * C::WAVES * 1024);
            }
        } else {
#pragma unroll
            for (int i = 0; i < PER * C::NI; ++i) {
                const int w = HALF == 2 ? (i & 1) : HALF, j = i / PER;
                load_to_lds16<false>(w ? vbase : kbase, goffs[j], stage + w * C::TILE_K + j * C::WAVES * 1024);
            }
        }
        if constexpr (HALF == 0) return;
        nxt = nxt + 1 == n_hot ? 0 : nxt + 1;
        kbase = ksrc + (int64_t)nxt * C::TILE_K;
        vbase = vsrc + (int64_t)nxt * C::TILE_K;
    };
    // behind the full tiles: the ragged last prefix tile, if it is here, and the tree's own tiles, if they are
    const int n_tail = n_pre - n_hot, n_all = n_hot + n_tail + n_tree_tiles;
    const int tail_rows = L - (t1 - 1) * C::T;
    // Tile i of those: which keys of this wavefront's blocks exist (ragged tile) or are ancestors of its queries (tree)
    auto rest_bits = [&](int i, uint32_t (&bits)[C::KPW]) {
#pragma unroll
        for (int u = 0; u < C::KPW; ++u) {
            const int key0 = (kg * C::KPW + u) * 32;        // first key of this block inside the tile
            if (i < 0) {                                    // (a full tile)
                bits[u] = 0xffffffffu;
            } else if (RAGGED) {                            // (without branches: with them four registers spill, 102 -> 106 us)
                const int left = tail_rows - key0;
                const uint32_t exist = left >= 32 ? 0xffffffffu : (left <= 0 ? 0u : ((1u << left) - 1u));
                const int col = max(i - n_tail, 0) * C::T + key0;
                const uint64_t word = (col >> 6) ? (p.mask_words > 1 ? mrow[1] : 0) : mrow[0];
                const uint32_t tree = i < n_tail ? 0u : 0xffffffffu;
                bits[u] = ((uint32_t)(word >> (col & 63)) & tree) | (exist & ~tree);
            } else if (i < n_tail) {
                const int left = tail_rows - key0;          // keys of the block that exist
                bits[u] = left >= 32 ? 0xffffffffu : (left <= 0 ? 0u : ((1u << left) - 1u));
            } else {
                const int col = (i - n_tail) * C::T + key0;
                bits[u] = (uint32_t)(((col >> 6) ? (p.mask_words > 1 ? mrow[1] : 0) : mrow[0]) >> (col & 63));
            }
        }
    };
    if constexpr (NS == 2) {
        // The tiles that are not full come the same way, a key beyond the last one as that one again (masked out), a value as
        // zeros: through registers behind the last full tile each of them cost its whole latency once more, 1.7 us.  Both halves in
        // one go, keys first, share their offsets: made anew for the values they cost short calls 0.1-0.2 us.  (For 128 columns only
        // behind the first two tiles: there, and in the kernel for pairs, which has no registers for it, halves by themselves.)
        auto issue_rest = [&](int i, unsigned char *stage, auto half) __attribute__((always_inline)) {
            constexpr int HALF = decltype(half)::value;
            const bool tail = i < n_tail;
            const unsigned char *ks = tail ? kp + (int64_t)(t1 - 1) * C::TILE_K : (const unsigned char *)kt + (int64_t)(i - n_tail) * C::TILE_K;
            const unsigned char *vs = tail ? vp + (int64_t)(t1 - 1) * C::TILE_K : (const unsigned char *)vt + (int64_t)(i - n_tail) * C::TILE_K;
            const int last = (tail ? tail_rows : p.n - (i - n_tail) * C::T) - 1;
            stage += wave * 1024;
            const unsigned char *no_row = zeros + (lane & 3) * 16;
            uint32_t off[C::NI];
#pragma unroll
            for (int j = 0; j < C::NI; ++j) off[j] = goff + (uint32_t)((j * STEP - max(row0 + j * STEP - last, 0)) * C::RBP);
            if (HALF != 1) {
#pragma unroll
                for (int j = 0; j < C::NI; ++j) load_to_lds16<false>(ks, off[j], stage + j * C::WAVES * 1024);
            }
            if (HALF != 0) {
#pragma unroll
                for (int j = 0; j < C::NI; ++j)
                    load_to_lds16_at(row0 + j * STEP > last ? no_row : vs + off[j], stage + C::TILE_K + j * C::WAVES * 1024);
            }
        };
        // This wavefront's reads of the half tile that is asked for next are done, and what it has waited for has landed; now everyone's.
        auto meet = []() __attribute__((always_inline)) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
        };
        auto issue = [&](int i, unsigned char *stage, auto half) __attribute__((always_inline)) {
            if (i < n_hot) issue_full(stage, half);
            else issue_rest(i - n_hot, stage, half);
        };
        // A short call is one or two tiles per workgroup, and what it takes is their way from memory: the first tile waits for its
        // keys alone, with the values and what fits of the second tile already under way behind them.  32 heads of 128 columns:
        // one sequence of 1024 keys 5.5 % of a whole step, of 2000 keys under 120 nodes 17.1 -> 16.8 us; four of 700 under 14
        // nodes 14.8 -> 13.7 (waiting for the whole first tile, with the second behind it: 13.7 too, but 1.5 % of the step).
        auto issue_first = [&](int i, unsigned char *stage) __attribute__((always_inline)) {         // (one of the first two tiles)
            if (D == 64 && i >= n_hot) issue_rest(i - n_hot, stage, BOTH);
            else {
                issue(i, stage, KEYS);
                issue(i, stage, VALUES);
            }
        };
        issue_first(0, ring);                                // (behind Q: requested ahead of Q it costs 2 %)
        if (n_all > 1) {
            if constexpr (C::HALVES_FIRST == 3) issue(1, ring + C::TILE, KEYS);
            if constexpr (C::HALVES_FIRST > 3) issue_first(1, ring + C::TILE);
            MCSD_WAIT_VMCNT((C::HALVES_FIRST - 1) * C::NI);
        } else {
            MCSD_WAIT_VMCNT(C::NI);
        }
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        {
            const unsigned char *qr = ring + C::Q_AT + (qb * 32 + ln) * C::RB;
#pragma unroll
            for (int ks = 0; ks < C::KS; ++ks) qs.q[ks] = *(const bf16x8_t *)(qr + (((2 * ks + g) ^ swz<D>(ln)) * 16));
            const uint64_t *mr = (const uint64_t *)(ring + C::MASK_AT) + ((qb & (p.bph - 1)) * 32 + ln) * 2;
            mrow[0] = mr[0];
            mrow[1] = mr[1];
            uint32_t bits[C::KPW];
            rest_bits(-n_hot, bits);
            attn_tile<D, QBP, NS, 2, false, false>(ring, la, qs, p.c, g, bits, 1.f, nullptr, n_hot == 0, [&]() __attribute__((always_inline)) {
                if (n_all > 1) MCSD_WAIT_VMCNT((C::HALVES_FIRST - 2) * C::NI);
                else MCSD_WAIT_VMCNT(0);
                meet();                                      // (Q has been read, too)
                if (n_all > 1) {                             // the rest of the second tile, partly where Q was, and the third's keys
                    if constexpr (C::HALVES_FIRST == 3) issue(1, ring + C::TILE, VALUES);
                    if constexpr (C::HALVES_FIRST == 2) issue(1, ring + C::TILE, BOTH);
                    if (alone && n_all > 2) issue(2, ring, KEYS);
                }
            });
        }
        // The workgroup that shares its compute unit asks for a tile when the tile before has landed and waits for all of it: the
        // other one's loads are under way meanwhile, and where memory is the limit more requests cost 1-2 % (8 x 32 heads of 16384
        // keys: 345 us so, 355 with the loop for one that is alone; 16 x 32 of 2300: 97.7, 98.9).  The one that is alone asks for
        // a half as soon as its place is free, two barriers and waits per tile, and never waits for the last two: 16 sequences of
        // 1000-4000 keys, 16 heads, one query block 68.9 -> 59.9 us; of 512-4096 keys, 32 heads, 60 nodes 113.7 -> 106.  (A ring of
        // five halves with one barrier per tile: 60.5, 106.7, and 355 above, for the reads' addresses are then made for every tile.)
        int it = 1;
        auto full = [&](unsigned char *stage, unsigned char *other) __attribute__((always_inline)) {
            MCSD_WAIT_VMCNT(2 * C::NI);
            meet();
            issue_full(other, VALUES);
            attn_tile<D, QBP, NS, 0, false, false>(stage, la, qs, p.c, g, all_keys, 1.f, nullptr, false, [&]() __attribute__((always_inline)) {
                MCSD_WAIT_VMCNT(2 * C::NI);
                meet();
                issue_full(stage, KEYS);
            });
        };
        bool ahead = alone && n_all > 2;                     // the keys of the tile after this one have been requested
        auto arrived = [&]() __attribute__((always_inline)) {
            MCSD_WAIT_VMCNT(0);
            meet();
        };
        if (alone) {
            for (; it + 3 < n_hot; it += 2) {
                full(ring + C::TILE, ring);
                full(ring, ring + C::TILE);
            }
        } else {
            for (; it + 2 < n_hot; it += 2) {
                arrived();
                issue_full(ring, BOTH);
                attn_tile<D, QBP, NS, 0, false, false>(ring + C::TILE, la, qs, p.c, g, all_keys);
                arrived();
                issue_full(ring + C::TILE, BOTH);
                attn_tile<D, QBP, NS, 0, false, false>(ring, la, qs, p.c, g, all_keys);
            }
        }
        auto rest = [&](int i, unsigned char *stage, unsigned char *other) __attribute__((always_inline)) {
            arrived();
            if (i + 1 < n_all) {
                if constexpr (!RAGGED && !(D == 128 && QBP == 1)) issue(i + 1, other, BOTH);     // (never `ahead`)
                else {
                    if (!ahead) issue(i + 1, other, KEYS);
                    issue(i + 1, other, VALUES);
                }
            }
            ahead = false;
            uint32_t bits[C::KPW];
            rest_bits(i - n_hot, bits);
            attn_tile<D, QBP, NS, 2, false, false>(stage, la, qs, p.c, g, bits, 1.f, nullptr, i >= n_hot);
        };
        while (it < n_all) {
            rest(it, ring + C::TILE, ring);
            if (__builtin_expect(it + 1 >= n_all, 0)) break;
            rest(it + 1, ring, ring + C::TILE);
            it += 2;
        }
        static_assert(!F8, "fp8 tiles use the ring below");
    } else {
        // A ring of NS stages keeps NS-1 slots in flight: fp8 tiles (half the bytes); bf16 tiles only on request (it
        // needs a compute unit's LDS per workgroup and measured slower, see make_plan).  Slot x lives in stage x % NS and is
        // DPT loads per wavefront: a full tile, the ragged one, or of the tree's own tiles a whole one (bf16) or, beside an
        // fp8 prefix, its K or its V half.  A step waits until exactly the slots requested after its own are still
        // outstanding: NS-2 of them in the steady state, fewer at the end.
        constexpr int TS = F8 ? 2 : 1;                       // slots of a tree tile
        const int n8 = n_hot + n_tail, n_slots = n8 + TS * n_tree_tiles;
        auto stage_of = [&](int x) { return ring + (x & (NS - 1)) * C::TILE; };
        auto issue_rest = [&](int x) {                       // a slot behind the full tiles
            unsigned char *stage = stage_of(x) + wave * 1024;
            if (F8 && x >= n8) {
                const int t = (x - n8) >> 1, last = p.n - t * C::T - 1;
                const unsigned char *src = (const unsigned char *)(((x - n8) & 1) ? vt : kt) + (int64_t)t * C::BTILE_K;
#pragma unroll
                for (int j = 0; j < C::DPT; ++j) {           // 1 KiB of bf16 rows per instruction
                    const int r = (j * C::WAVES + wave) * (1024 / C::RB) + lane / C::BCPR;
                    load_to_lds16<false>(src, (uint32_t)(min(r, last) * C::RB + (((lane % C::BCPR) ^ swz<D>(r)) * 16)), stage + j * C::WAVES * 1024);
                }
                return;
            }
            const bool tail = x < n8;
            const unsigned char *ks = tail ? kp + (int64_t)(t1 - 1) * C::TILE_K : (const unsigned char *)kt + (int64_t)(x - n8) * C::TILE_K;
            const unsigned char *vs = tail ? vp + (int64_t)(t1 - 1) * C::TILE_K : (const unsigned char *)vt + (int64_t)(x - n8) * C::TILE_K;
            const int last = (tail ? tail_rows : p.n - (x - n8) * C::T) - 1;
            int l = lane;
            asm volatile("" : "+v"(l));
            const unsigned char *no_row = zeros + (l & 3) * 16;
#pragma unroll
            for (int j = 0; j < C::NI; ++j) {
                const uint32_t off = goff + (uint32_t)((j * STEP - max(row0 + j * STEP - last, 0)) * C::RBP);
                load_to_lds16<false>(ks, off, stage + j * C::WAVES * 1024);
                if constexpr (F8) load_to_lds16<false>(vs, off, stage + C::TILE_K + j * C::WAVES * 1024);   // (the format has no infinity)
                else load_to_lds16_at(row0 + j * STEP > last ? no_row : vs + j * STEP * C::RBP + goff, stage + C::TILE_K + j * C::WAVES * 1024);
            }
        };
        auto issue = [&](int x) {
            if (x < n_hot) issue_full(stage_of(x), BOTH);
            else if (x < n_slots) issue_rest(x);
        };
        auto arrived = [&](int later) {                      // all but `later` slots, and everywhere; the slot before is free again
            if (later >= 2) MCSD_WAIT_VMCNT(2 * C::DPT);
            else if (later == 1) MCSD_WAIT_VMCNT(C::DPT);
            else MCSD_WAIT_VMCNT(0);
            __builtin_amdgcn_s_barrier();
        };
        auto step = [&](auto stage, int it) {
            constexpr int ST = decltype(stage)::value;
            arrived(min(n_slots - it - 1, NS - 2));
            if (it + NS - 1 < n_hot) issue_full(ring + (ST + NS - 1) % NS * C::TILE, BOTH);
            else if (it + NS - 1 < n_slots) issue_rest(it + NS - 1);
            attn_tile<D, QBP, NS, 0, F8, F8>(ring + ST * C::TILE, la, qs, c_pre, g, all_keys, vs_pre);
        };
        static_assert(NS == 4, "the step sequence below is unrolled for four stages");
        // Q and the mask row must have arrived before the first direct-to-LDS load is issued: the steps wait with a non-zero
        // count, and the compiler, which does not see those loads, would otherwise place its own wait for Q at the first
        // MFMA inside the loop, where it would also wait for the tiles in flight.  (Waiting behind the first loads: 1-4 % more.)
        MCSD_WAIT_VMCNT(0);
        issue(0);
        issue(1);
        issue(2);
        for (int it = 0; it < n_hot; it += 4) {
            step(std::integral_constant<int, 0>(), it);
            if (it + 1 < n_hot) step(std::integral_constant<int, 1 % NS>(), it + 1);
            if (it + 2 < n_hot) step(std::integral_constant<int, 2 % NS>(), it + 2);
            if (it + 3 < n_hot) step(std::integral_constant<int, 3 % NS>(), it + 3);
        }
        if (n_tail) {
            arrived(min(n_slots - n_hot - 1, NS - 2));
            issue(n_hot + NS - 1);
            uint32_t bits[C::KPW];
            rest_bits(0, bits);
            attn_tile<D, QBP, NS, 1, F8, F8>(stage_of(n_hot), la, qs, c_pre, g, bits, vs_pre);
        }
        for (int t = 0; t < n_tree_tiles; ++t) {
            // requested so far: NS - 1 slots from the first tree slot on, or (second fp8 tile) up to this tile's own last
            const int x = n8 + TS * t, have = min(n_slots, TS == 2 && t == 1 ? x + TS : x + NS - 1);
            arrived(have - x - TS);
            issue(x + NS - 1);
            if (F8 && p.n - t * C::T < C::T) {               // (uniform) the values behind the last row: zeros after all
                // (as addresses of their own for every lane, like above, they cost a small call 4 %: eight loads per slot)
                for (int r = p.n - t * C::T + tid / C::BCPR; r < C::T; r += C::THREADS / C::BCPR)
                    *(uint4 *)(stage_of(x + 1) + r * C::RB + (tid % C::BCPR) * 16) = make_uint4(0, 0, 0, 0);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
            }
            uint32_t bits[C::KPW];
            rest_bits(n_tail + t, bits);
            attn_tile<D, QBP, NS, 1, F8, false>(stage_of(x), la, qs, p.c, g, bits, 1.f, F8 ? stage_of(x + 1) : nullptr);
        }
    }
    __syncthreads();

    // ---- merge the key groups of each query block through LDS ----
    // A wavefront's output is CB * 4 pieces (16 bytes per lane: four columns of one query); key group kg ends up with pieces
    // kg * PP .. of all groups.  Every group hands over the pieces that are not its own, so all wavefronts merge and store
    // (one of them merging everything: 0.65 us for two groups, 0.9 us for four).
    constexpr int PP = C::CB * 4 / C::KG;
    float l_tot = half_swap_sum(qs.l_run);
    const float cm = F8 ? 1.f : p.c;                           // reference maxima are in log2 units already with fp8 tiles
    f32x4_t acc[PP];
    const auto piece = [&](int x) {
        f32x4_t v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = qs.o[x >> 2][4 * (x & 3) + e];
        return v;
    };
    if constexpr (C::KG == 1) {
#pragma unroll
        for (int x = 0; x < PP; ++x) acc[x] = piece(x);
    } else {
        float *ml = (float *)(ring + C::XCHG);                  // [key group][query block][m: 32, l: 32]
        // pieces for owner o from the key group that is number r among the others
        auto at = [&](int o, int r, int x) { return (f32x4_t *)(ring + ((((o * (C::KG - 1) + r) * QBP + qb) * PP + x) * 64 + lane) * 16); };
#pragma unroll
        for (int o = 0; o < C::KG; ++o) {
            if (o == kg) {
#pragma unroll
                for (int x = 0; x < PP; ++x) acc[x] = piece(o * PP + x);
            } else {
#pragma unroll
                for (int x = 0; x < PP; ++x) *at(o, kg < o ? kg : kg - 1, x) = piece(o * PP + x);
            }
        }
        if (g == 0) {
            ml[(kg * QBP + qb) * 64 + ln] = qs.m_ref;
            ml[(kg * QBP + qb) * 64 + 32 + ln] = l_tot;
        }
        __syncthreads();
        float m[C::KG], l[C::KG], M = -INFINITY;
#pragma unroll
        for (int k = 0; k < C::KG; ++k) {
            m[k] = ml[(k * QBP + qb) * 64 + ln];
            l[k] = ml[(k * QBP + qb) * 64 + 32 + ln];
            M = fmaxf(M, m[k]);
        }
        const float Mf = M == -INFINITY ? 0.f : M;              // (nobody has seen a key: every weight is exp2(-inf) = 0)
        l_tot = 0.f;
#pragma unroll
        for (int k = 0; k < C::KG; ++k) l_tot = fmaf(l[k], fast_exp2((m[k] - Mf) * cm), l_tot);
        const float own = fast_exp2((qs.m_ref - Mf) * cm);
#pragma unroll
        for (int x = 0; x < PP; ++x) acc[x] *= own;
#pragma unroll
        for (int r = 0; r < C::KG - 1; ++r) {
            const float w = fast_exp2((ml[((r < kg ? r : r + 1) * QBP + qb) * 64 + ln] - Mf) * cm);
#pragma unroll
            for (int x = 0; x < PP; ++x) acc[x] += *at(kg, r, x) * w;
        }
        qs.m_ref = M;
    }
    if (n_active == 1) {                                   // the only split of this sequence: no exchange needed
        if (qrow >= p.n) return;
        const float inv = 1.f / l_tot;
        __bf16 *o = (__bf16 *)p.out + (bh_q * p.node_stride + qrow) * D;
#pragma unroll
        for (int x = 0; x < PP; ++x) {
            bf16x4_t v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (__bf16)(acc[x][e] * inv);
            const int y = kg * PP + x;
            *(bf16x4_t *)(o + (y >> 2) * 32 + 8 * (y & 3) + 4 * g) = v;
        }
        return;
    }

    // ---- key splits: every split writes (O, m, l) in register-fragment order (fully coalesced) ----
    if (qrow < p.n) {                                      // padded query rows are never read back
        // O goes out rounded to bf16, the precision the output itself has (one more rounding of 2^-9 relative to the
        // partial's own magnitude; maxima and denominators stay fp32): half the bytes to write, acknowledge and fold.
        // A lane's 16-byte chunk is two pieces.  Short prefixes: fp32, a chunk per piece.
        const int64_t slot0 = (bh * p.SP + slot_id) * (int64_t)(QBP * 32 * D) + qb * 32 * D;
        if constexpr (PF32) {
            float *po = p.part_o + slot0;
#pragma unroll
            for (int x = 0; x < PP; ++x) *(f32x4_t *)(po + (((kg * PP + x) * 2 + g) * 32 + ln) * 4) = acc[x];
        } else {
            __bf16 *po = (__bf16 *)p.part_o + slot0;
#pragma unroll
            for (int x2 = 0; x2 < PP / 2; ++x2) {
                bf16x8_t v;
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = (__bf16)acc[2 * x2 + (e >> 2)][e & 3];
                *(bf16x8_t *)(po + (((kg * (PP / 2) + x2) * 2 + g) * 32 + ln) * 8) = v;
            }
        }
        if (kg == 0 && g == 0) {
            const int64_t prow = (bh * p.SP + slot_id) * (QBP * 32) + qb * 32 + ln;
            p.part_m[prow] = qs.m_ref;
            p.part_l[prow] = l_tot;
        }
    }
    if (!p.fold) return;                                   // a second kernel folds
    // Requested here, so that its latency is the stores' own: ahead of the merge above, the wait for it came right behind it
    // and held up every workgroup (32 layers of 1024 keys: 352.2 -> 350.9 us).
    const uint32_t ws_tag = __hip_atomic_load(p.ws_tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);

    // ---- fold inside this kernel: the workgroup of this (sequence, unit) that arrives last does it ----
    // All workgroups of the unit run on one die (see the numbering above), so their partial results meet in that
    // die's L2: a store is there once it is acknowledged (the vector L1 writes through), and the loads below go past
    // the L1.  Nobody waits for anybody: a workgroup counts itself in and leaves unless it is the last.  The
    // counter also records, per die, how many of the arrivals ran there, so a launch that was not dealt to the
    // dies as the host established shows up here and poisons the output instead of folding stale data.
    auto store_nan = [&]() {
        if (kg != 0 || qrow >= p.n) return;
        __bf16 *o = (__bf16 *)p.out + (bh_q * p.node_stride + qrow) * D;
        bf16x4_t v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (__bf16)__builtin_nanf("");
#pragma unroll
        for (int cb = 0; cb < C::CB; ++cb)
#pragma unroll
            for (int j = 0; j < 4; ++j) *(bf16x4_t *)(o + cb * 32 + 8 * j + 4 * g) = v;
    };
    if (ws_tag != WS_TAG) {                                // workspace never prepared: its counters mean nothing
        store_nan();
        return;
    }
    unsigned long long &s_prev = *(unsigned long long *)(ring + C::LDS_BYTES - 16);
    unsigned die;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(die));
    die &= 7u;
    // This wavefront's partial stores have reached the L2 once the vector-memory counter is back at zero.  (A release
    // fence of workgroup scope does not wait for it: within a workgroup the shared L1 already orders them.)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0)
        s_prev = __hip_atomic_fetch_add(p.ctr + bh * CTR_STRIDE, 1ull + (1ull << (8 + 7 * die)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const unsigned long long prev = s_prev;
    if ((int)(prev & 0xffu) + 1 != n_active) return;       // someone else arrives later
    asm volatile("" ::: "memory");                         // (the loads below go past the L1: nothing to invalidate)
    if (tid == 0) __hip_atomic_store(p.ctr + bh * CTR_STRIDE, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // as it was found
    if ((int)((prev >> (8 + 7 * die)) & 0x7fu) + 1 != n_active) {   // an arrival from another die
        store_nan();
        return;
    }
    if (qrow >= p.n) return;
    // Every wavefront folds its query block's rows for its share of the columns (32-column blocks kg, kg + KG, ..),
    // all partial results read back in slot order, its own included: the result does not depend on who came last.
    // Loads go through buffer descriptors that end after the last partial result in use (see fold_partials).
    constexpr int part_bytes = QBP * 32 * D * (PF32 ? 4 : 2);
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
        (void *)((char *)p.part_o + (bh * p.SP) * (int64_t)part_bytes + qb * (part_bytes / QBP)), 0, n_active * part_bytes, 0x00027000);
    const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(p.part_m + bh * p.SP * (QBP * 32) + qb * 32), 0, (int)(n_active * QBP * 32 * 4), 0x00027000);
    const __amdgpu_buffer_rsrc_t rl = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(p.part_l + bh * p.SP * (QBP * 32) + qb * 32), 0, (int)(n_active * QBP * 32 * 4), 0x00027000);
    __bf16 *orow = (__bf16 *)p.out + (bh_q * p.node_stride + qrow) * D;
    // as few slots per round as hold the partial results: a load beyond the end still costs its turn in the L1
    if (n_active <= 3) fold_partials<D, QBP, C::KG, 3, PF32>(ro, rm, rl, n_active, kg, g, ln, cm, orow, (f32x4_t *)ring + tid);
    else if (n_active <= 5) fold_partials<D, QBP, C::KG, 5, PF32>(ro, rm, rl, n_active, kg, g, ln, cm, orow, (f32x4_t *)ring + tid);
    else if (PF32 || n_active <= 7) fold_partials<D, QBP, C::KG, 7, PF32>(ro, rm, rl, n_active, kg, g, ln, cm, orow, (f32x4_t *)ring + tid);
    else fold_partials<D, QBP, C::KG, PF32 ? 7 : 8, PF32>(ro, rm, rl, n_active, kg, g, ln, cm, orow, (f32x4_t *)ring + tid);
}

#define SWEEP_KERNEL(NAME, PF32, RAGGED)                                                                                                 \
    template <int D, int QBP, int NS, bool F8 = false>                                                                              \
    __global__ __launch_bounds__((SweepCfg<D, QBP, NS, F8>::THREADS)) __attribute__((amdgpu_waves_per_eu(2, 2)))                    \
    void NAME(const int32_t *lens, const int64_t *seq_base, const uint32_t per_die, const int32_t G, const uint32_t mul_G,          \
              const int32_t H, const uint32_t mul_H, const int32_t BH, const uint32_t how, const int32_t max_prefix,                \
              const int32_t tps, const AttnParams p)                                                                                \
    {                                                                                                                               \
        sweep<D, QBP, NS, F8, PF32, RAGGED>(lens, seq_base, per_die, G, mul_G, H, mul_H, BH, how, max_prefix, tps, p);              \
    }
SWEEP_KERNEL(tree_attn_bf16_kernel, false, false)
// (a kernel of its own: as a branch the second set of folds cost calls that do not use it up to 1 %, 32 layers of 1024 keys 352 -> 357 us)
SWEEP_KERNEL(tree_attn_bf16_short_kernel, true, false)
// (a kernel of its own, too: the second loop costs 50 registers, and calls that never take it 0.1 us: that step 334 -> 336 us)
SWEEP_KERNEL(tree_attn_bf16_ragged_kernel, false, true)
#undef SWEEP_KERNEL

// Folds the partial results of the key splits of the bf16 sweep.  One thread per 4 output columns of one query;
// fragment order makes the loads of a wavefront contiguous.  Partials are folded in split order.
template <int D, int QBP>
__global__ __launch_bounds__(256) void tree_attn_merge_bf16_kernel(const AttnParams p, int T)
{
    constexpr int POS = D * 8;                                // float4 positions per (b, h, query block)
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int pos = (int)(idx % POS);
    const int qb = (int)((idx / POS) % QBP);
    const int64_t bh = idx / ((int64_t)POS * QBP);
    if (bh >= (int64_t)p.B * p.H) return;
    const int ln = pos & 31, g = (pos >> 5) & 1, f = pos >> 6;
    const int lrow = qb * 32 + ln;                            // row of the partial results
    const int row = p.row0 + (qb % p.bph) * 32 + ln;          // tree node
    if (row >= p.n) return;
    const int unit = (int)(bh % p.H);
    const int64_t bh_q = (bh / p.H) * p.Hq + (unit / p.chunks) * p.grp + (unit % p.chunks) * p.hpw + qb / p.bph;
    int L = p.lens[bh / p.H];
    L = L < 0 ? 0 : (L > p.max_prefix ? p.max_prefix : L);
    const int tiles_b = (L + T - 1) / T;
    const int np = (tiles_b + p.tps - 1) / p.tps;
    const int n_active = p.G > p.S ? np + 1 : max(1, np);
    if (n_active == 1) return;                                // the sweep wrote this sequence's output itself
    // eight partials at a time, all loads issued before the first use; folded in slot order
    float M = -INFINITY, den = 0.f;
    f32x4_t num = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < n_active; s0 += 8) {
        float m[8], l[8];
        f32x4_t o[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            m[i] = -INFINITY;
            l[i] = 0.f;
            o[i] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
            if (s0 + i < n_active) {
                const int64_t prow = (bh * p.SP + s0 + i) * (QBP * 32) + lrow;
                m[i] = p.part_m[prow];
                l[i] = p.part_l[prow];
                const int64_t slot0 = (bh * p.SP + s0 + i) * (int64_t)(QBP * 32 * D) + qb * 32 * D;
                if (p.part_f32) {
                    o[i] = *(const f32x4_t *)(p.part_o + slot0 + ((f * 2 + g) * 32 + ln) * 4);
                } else {
                    const bf16x4_t ob = *(const bf16x4_t *)((const __bf16 *)p.part_o + slot0 + ((((f >> 2) * 2 + ((f >> 1) & 1)) * 2 + g) * 32 + ln) * 8 + (f & 1) * 4);
                    o[i] = (f32x4_t){(float)ob[0], (float)ob[1], (float)ob[2], (float)ob[3]};
                }
            }
        }
        float Mn = M;
#pragma unroll
        for (int i = 0; i < 8; ++i) Mn = fmaxf(Mn, m[i]);
        if (Mn == -INFINITY) continue;                        // nothing visible so far
        const float a = fast_exp2((M - Mn) * p.c);            // exp2(-inf) = 0 on the first group
        den *= a;
        num *= a;
        M = Mn;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float w = fast_exp2((m[i] - M) * p.c);      // 0 for a split that saw no visible key
            den = fmaf(w, l[i], den);
            num += w * o[i];
        }
    }
    const f32x4_t r = num / den;
    bf16x4_t v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (__bf16)r[e];
    const int c = (f / 4) * 32 + 8 * (f % 4) + 4 * g;
    *(bf16x4_t *)((__bf16 *)p.out + (bh_q * p.node_stride + row) * D + c) = v;
}

// ---------------------------------------------------------------------------------------------------
// fp32 / MFMA kernel
// ---------------------------------------------------------------------------------------------------
// One workgroup of 4 wavefronts owns one (sequence, head, tile of 16 query rows, key split); its wavefronts take the split's
// 16-key blocks in turn and never meet before the end.  v_mfma_f32_16x16x4_f32 is fp32 in and out with fused multiply-adds,
// at twice the vector ALU's rate.  As in the bf16 sweep scores are computed transposed, so a lane holds 4 keys of one query
// and the exponentials are the B operand of O^T += V^T P^T as they stand.  Nothing of K or V is shared between
// wavefronts, so neither goes through LDS: the contraction's column order and the output's row order are chosen such that
// a lane's operands are 16-byte pieces of rows (K: columns 16 t + 4 g ..; V: columns i D/16 .., whole rows per 16 lanes),
// loaded one block ahead.  The query tiles of a (sequence, head) read the same keys at about the same time from one die's
// L2; cutting the queries instead of the keys leaves few partial results to fold (16 rows each).
// Bound: 16 KB per wavefront in flight against the latency of the memory system (about 30 GB/s per compute unit); at 120
// nodes x 1000 keys x 64 heads the matrix cores are 43 % busy.  Measured against the vector ALU kernel and its fold kernel
// that this replaced, us per call: 14 nodes, 4 heads of 64, 128 keys 19.0 -> 6.0; 81 nodes, 2 x 16 heads of 128, 329 keys
// 459 -> 17; 80 nodes, 2 x 8 heads of 64, 1205 keys 150 -> 12; 82 nodes, 6 x 32 heads of 128, 120 keys 803 -> 40.
constexpr int F32_ROWS = 16, F32_KEYS = 16;

typedef __attribute__((address_space(1))) f32x4_t global_f32x4_t;   // (told apart from LDS: a choice of two addresses loses that)

template <int D>
struct F32Block {
    f32x4_t k[D / 16];          // K[key i][16 t + 4 g ..], i = lane % 16, g = lane / 16
    f32x4_t v[4][D / 64];       // V[key 4 g + r][i D/16 + 4 j ..]
};

// Maximum / sum over the four lanes that hold one query (lanes i, i + 16, i + 32, i + 48).
__device__ inline float quarter_max(float v)
{
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return half_swap_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ inline float quarter_sum(float v)
{
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return half_swap_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// Keys of one (sequence, head) in 16-key blocks: the prefix's, then the tree's.  Split s owns blocks s * bps ..
struct F32Keys {
    int L, n_pre, n_blk, bps, n_active;
    __device__ F32Keys(const AttnParams &p, int b)
    {
        L = p.lens[b];
        L = L < 0 ? 0 : (L > p.max_prefix ? p.max_prefix : L);
        n_pre = (L + F32_KEYS - 1) / F32_KEYS;
        n_blk = n_pre + (p.n + F32_KEYS - 1) / F32_KEYS;
        bps = (n_blk + p.S - 1) / p.S;
        n_active = (n_blk + bps - 1) / bps;              // splits that have keys
    }
};

// Output columns of lane (i, g)'s accumulators [e]: (4 g + e) D/16 .. + D/16 - 1, of query i.  acc[e] / den to out or NaN.
template <int D>
__device__ inline void f32_store(float *out, const float (&acc)[D / 16], float scale)
{
#pragma unroll
    for (int j = 0; j < D / 64; ++j) {
        f32x4_t v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[4 * j + e] * scale;
        *(f32x4_t *)(out + 4 * j) = v;
    }
}

// Folds the partial results of one query tile for output rows e of the accumulators: out += all splits in order.  A partial
// is [e][lane][D/16] floats, its maxima and denominators 16 + 16 floats of a 128-byte line of their own.  THROUGH_L2: read
// past the L1 (written by other workgroups of this launch, see the end of the bf16 sweep).
template <int D, bool THROUGH_L2>
__device__ inline void f32_fold(const float *po, const float *pml, int n_active, int e, int lane, float c, float (&acc)[D / 16], float &den)
{
    constexpr int W = D / 16, PART = 4 * 64 * W;
    const int i = lane & 15;
    const auto ro = __builtin_amdgcn_make_buffer_rsrc((void *)po, 0, n_active * PART * 4, 0x00027000);
    const auto rm = __builtin_amdgcn_make_buffer_rsrc((void *)pml, 0, n_active * 128, 0x00027000);
    constexpr int AUX = THROUGH_L2 ? 1 : 0;
    float M = -INFINITY;
    den = 0.f;
#pragma unroll
    for (int k = 0; k < W; ++k) acc[k] = 0.f;
    constexpr int R = 4;                                     // partial results in flight; beyond the last one loads return zero
    for (int s0 = 0; s0 < n_active; s0 += R) {
        float m[R], l[R];
        f32x4_t o[R][D / 64];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            m[r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rm, (s0 + r) * 128 + i * 4, 0, AUX));
            l[r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rm, (s0 + r) * 128 + 64 + i * 4, 0, AUX));
#pragma unroll
            for (int j = 0; j < D / 64; ++j)
                o[r][j] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(ro, (((s0 + r) * 4 + e) * 64 + lane) * W * 4 + j * 16, 0, AUX));
        }
        float Mn = M;
#pragma unroll
        for (int r = 0; r < R; ++r) Mn = fmaxf(Mn, s0 + r < n_active ? m[r] : -INFINITY);
        if (Mn == -INFINITY) continue;                       // (per query) nothing visible so far
        const float a = fast_exp2((M - Mn) * c);             // exp2(-inf) = 0 in the first round
        M = Mn;
        den *= a;
#pragma unroll
        for (int k = 0; k < W; ++k) acc[k] *= a;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float w = s0 + r < n_active ? fast_exp2((m[r] - M) * c) : 0.f;
            den = fmaf(w, l[r], den);
#pragma unroll
            for (int k = 0; k < W; ++k) acc[k] = fmaf(w, o[r][k / 4][k % 4], acc[k]);
        }
    }
}

template <int D>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void tree_attn_f32_kernel(const AttnParams p)
{
    constexpr int W = D / 16, KT = D / 16, PART = 4 * 64 * W;
    __shared__ __attribute__((aligned(16))) float s_o[4][4][64][W];      // [wavefront][e][lane][column]
    __shared__ float s_m[4][16], s_l[4][16];
    // ids are dealt round-robin to the dies: the workgroups of one (sequence, head) share one
    const int total = gridDim.x;
    int wg = blockIdx.x;
    if (p.xcc > 1 && total % p.xcc == 0) wg = (wg % p.xcc) * (total / p.xcc) + wg / p.xcc;
    const int tile = wg % p.QT, s = (wg / p.QT) % p.S, bhi = wg / (p.QT * p.S);
    if (bhi >= p.B * p.H) return;                            // a slot of a grid rounded up to whole dies
    const int h = bhi % p.H, b = bhi / p.H;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4;
    const int64_t bh = bhi;
    const int kvh = h / p.grp;
    const int qrow = p.row0 + tile * F32_ROWS + i;
    const bool mine = qrow < p.n;

    // query tile, as B operands: Q[query i][16 t + 4 g ..]; rows beyond the tree repeat the first one and are never stored
    f32x4_t q[KT];
    const float *qp = (const float *)p.q + (bh * p.node_stride + (mine ? qrow : p.row0)) * D + 4 * g;
#pragma unroll
    for (int t = 0; t < KT; ++t) q[t] = *(const f32x4_t *)(qp + 16 * t);
    uint64_t mrow[2] = {0, 0};
    {
        const uint64_t *mb = p.mask_bits + (int64_t)(mine ? qrow : p.row0) * p.mask_words;
        mrow[0] = mb[0];
        if (p.mask_words > 1) mrow[1] = mb[1];
    }
    const F32Keys ks(p, b);
    const int blk0 = s * ks.bps, blk1 = min(blk0 + ks.bps, ks.n_blk);
    if (blk0 >= blk1) return;                                // this split has no keys
    const uint32_t ws_tag = p.fold ? p.ws_tag[0] : WS_TAG;
    const int64_t pre0 = p.seq_base[b] + (int64_t)kvh * p.head_stride, tree0 = ((int64_t)b * p.Hkv + kvh) * p.node_stride * D;
    const float *kp = (const float *)p.kp + pre0, *vp = (const float *)p.vp + pre0;
    const float *kt = (const float *)p.kt + tree0, *vt = (const float *)p.vt + tree0;

    f32x4_t o[W];                                            // O^T: [cb], rows 4 g + e are columns (4 g + e) W + cb
#pragma unroll
    for (int cb = 0; cb < W; ++cb) o[cb] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    float m_ref = -INFINITY, l_run = 0.f;

    auto load = [&](F32Block<D> &x, int blk) {
        const bool pre = blk < ks.n_pre;                     // (uniform)
        const int key0 = (pre ? blk : blk - ks.n_pre) * F32_KEYS, last = (pre ? ks.L : p.n) - 1;
        const float *kb = pre ? kp : kt, *vb = pre ? vp : vt;
        const float *kr = kb + (int64_t)min(key0 + i, last) * D + 4 * g;      // keys beyond the last repeat it, masked below; values: zeros
#pragma unroll
        for (int t = 0; t < KT; ++t) x.k[t] = *(const f32x4_t *)(kr + 16 * t);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int key = key0 + 4 * g + r;
            const global_f32x4_t *vr = key > last ? (const global_f32x4_t *)zeros + (lane & 3) : (const global_f32x4_t *)(vb + (int64_t)key * D + i * W);
#pragma unroll
            for (int j = 0; j < D / 64; ++j) x.v[r][j] = vr[j];
        }
    };
    auto compute = [&](const F32Block<D> &x, int blk) {
        f32x4_t sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) sc = __builtin_amdgcn_mfma_f32_16x16x4f32(x.k[t][e], q[t][e], sc, 0, 0, 0);
        const bool pre = blk < ks.n_pre;
        const int key0 = (pre ? blk : blk - ks.n_pre) * F32_KEYS;
        if (!pre || key0 + F32_KEYS > ks.L) {                // (uniform) bit k: key k of the block is visible to this lane's query
            const int left = ks.L - key0;
            const uint32_t bits = pre ? (1u << left) - 1u : (uint32_t)((key0 >> 6 ? mrow[1] : mrow[0]) >> (key0 & 63));
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (!((bits >> (4 * g + r)) & 1u)) sc[r] = -INFINITY;
        }
        const float mx = quarter_max(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])));
        // the accumulators are rescaled only when the maximum outgrows the reference by more than the slack (exact either way)
        const bool grow = (mx - m_ref) * p.c > RESCALE_SLACK;
        if (__builtin_amdgcn_ballot_w64(grow) != 0) {
            const float m_new = grow ? mx : m_ref;
            const float alpha = m_new == m_ref ? 1.f : exp2f((m_ref - m_new) * p.c);
            m_ref = m_new;
            l_run *= alpha;
#pragma unroll
            for (int cb = 0; cb < W; ++cb) o[cb] *= alpha;
        }
        const float mc = (m_ref == -INFINITY ? 0.f : m_ref) * p.c;
        float pr[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            pr[r] = exp2f(fmaf(sc[r], p.c, -mc));
            l_run += pr[r];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int cb = 0; cb < W; ++cb) o[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.v[r][cb / 4][cb % 4], pr[r], o[cb], 0, 0, 0);
    };
    {
        // this wavefront's blocks: every fourth one; the next is loaded while one is computed (a load beyond the last repeats it)
        F32Block<D> x0, x1;
        int blk = blk0 + wave;
        if (blk < blk1) {
            load(x0, blk);
            while (true) {
                load(x1, min(blk + 4, blk1 - 1));
                __builtin_amdgcn_sched_barrier(0);
                compute(x0, blk);
                blk += 4;
                if (blk >= blk1) break;
                load(x0, min(blk + 4, blk1 - 1));
                __builtin_amdgcn_sched_barrier(0);
                compute(x1, blk);
                blk += 4;
                if (blk >= blk1) break;
            }
        }
    }

    // ---- merge the four wavefronts: each adds up one accumulator row e of all of them ----
    const float l_tot = quarter_sum(l_run);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < W / 4; ++j)
            *(f32x4_t *)&s_o[wave][e][lane][4 * j] = (f32x4_t){o[4 * j][e], o[4 * j + 1][e], o[4 * j + 2][e], o[4 * j + 3][e]};
    if (g == 0) { s_m[wave][i] = m_ref; s_l[wave][i] = l_tot; }
    __syncthreads();
    float acc[W], M = -INFINITY, den = 0.f;
#pragma unroll
    for (int k = 0; k < W; ++k) acc[k] = 0.f;
#pragma unroll
    for (int v = 0; v < 4; ++v) M = fmaxf(M, s_m[v][i]);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const float w = M == -INFINITY ? 0.f : exp2f((s_m[v][i] - M) * p.c);
        den = fmaf(w, s_l[v][i], den);
#pragma unroll
        for (int k = 0; k < W; ++k) acc[k] = fmaf(w, s_o[v][wave][lane][k], acc[k]);
    }
    float *out = (float *)p.out + (bh * p.node_stride + qrow) * D + (4 * g + wave) * W;
    if (ks.n_active == 1) {                                  // the only split of this sequence: no exchange needed
        if (mine) f32_store<D>(out, acc, 1.f / den);
        return;
    }

    // ---- key splits: partial results in fragment order; the workgroup that arrives last folds (protocol: bf16 sweep) ----
    const int64_t unit = bh * p.QT + tile;
    f32_store<D>(p.part_o + ((unit * p.S + s) * 4 + wave) * 64 * W + lane * W, acc, 1.f);
    float *ml = p.part_m + (unit * p.S + s) * 32;
    if (wave == 0 && g == 0) { ml[i] = M; ml[16 + i] = den; }
    if (!p.fold) return;                                     // a second kernel folds
    const float nan[4] = {__builtin_nanf(""), __builtin_nanf(""), __builtin_nanf(""), __builtin_nanf("")};
    auto store_nan = [&]() {
        if (!mine) return;
#pragma unroll
        for (int j = 0; j < W / 4; ++j) f32_store<64>(out + 4 * j, nan, 1.f);
    };
    if (ws_tag != WS_TAG) {                                  // workspace never prepared: its counters mean nothing
        store_nan();
        return;
    }
    __shared__ unsigned long long s_prev;
    unsigned die;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(die));
    die &= 7u;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // this wavefront's partial result has reached the L2
    __syncthreads();
    if (tid == 0)
        s_prev = __hip_atomic_fetch_add(p.ctr + unit * CTR_STRIDE, 1ull + (1ull << (8 + 7 * die)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const unsigned long long prev = s_prev;
    if ((int)(prev & 0xffu) + 1 != ks.n_active) return;      // someone else arrives later
    if (tid == 0) __hip_atomic_store(p.ctr + unit * CTR_STRIDE, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // as it was found
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    if ((int)((prev >> (8 + 7 * die)) & 0x7fu) + 1 != ks.n_active) {         // an arrival from another die
        store_nan();
        return;
    }
    f32_fold<D, true>(p.part_o + unit * p.S * PART, p.part_m + unit * p.S * 32, ks.n_active, wave, lane, p.c, acc, den);
    if (mine) f32_store<D>(out, acc, 1.f / den);
}

// The same fold as a kernel of its own, for splits that do not share one die's L2: a workgroup per query tile.
template <int D>
__global__ __launch_bounds__(256) void tree_attn_merge_f32_kernel(const AttnParams p)
{
    constexpr int W = D / 16, PART = 4 * 64 * W;
    const int64_t unit = blockIdx.x, bh = unit / p.QT;
    const int tile = (int)(unit % p.QT), b = (int)(bh / p.H);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const F32Keys ks(p, b);
    if (ks.n_active == 1) return;                            // the sweep wrote this sequence's output itself
    const int qrow = p.row0 + tile * F32_ROWS + (lane & 15);
    float acc[W], den;
    f32_fold<D, false>(p.part_o + unit * p.S * PART, p.part_m + unit * p.S * 32, ks.n_active, wave, lane, p.c, acc, den);
    if (qrow < p.n) f32_store<D>((float *)p.out + (bh * p.node_stride + qrow) * D + (4 * (lane >> 4) + wave) * W, acc, 1.f / den);
}


size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// workspace: [tag] [counters] [part_m] [part_l] [part_o]; nothing when the keys are not split
size_t partial_rows(const AttnPlan &pl, int dtype, int B)
{
    // per workgroup unit and split; whole query blocks of 32 (bf16) or 16 (fp32) rows, in register-fragment order
    return (size_t)B * pl.units * pl.G * (dtype == MCSD_BF16 ? (size_t)pl.QBP * 32 : (size_t)pl.QT * F32_ROWS);
}

size_t workspace_bytes_for(const AttnPlan &pl, int dtype, int B, int d)
{
    if (pl.S == 1) return 0;
    const size_t rows = partial_rows(pl, dtype, B);
    return WS_HEADER + WS_CTR_BYTES + 2 * align256(rows * sizeof(float)) + align256(rows * d * (dtype == MCSD_BF16 && !pl.part_f32 ? 2 : sizeof(float)));
}

// Prepares a workspace: tag word, zero counters.  One thread per 16 bytes of the header and counter area.
__global__ __launch_bounds__(256) void workspace_init_kernel(uint4 *ws)
{
    const unsigned i = blockIdx.x * 256 + threadIdx.x;
    if (i < (WS_HEADER + WS_CTR_BYTES) / 16) ws[i] = make_uint4(i == 0 ? WS_TAG : 0u, 0u, 0u, 0u);
}

template <int D, int QBP, int NS, bool F8 = false>
void launch_sweep(const AttnParams &p, const AttnPlan &pl, hipStream_t st)
{
    const uint32_t total = (uint32_t)((size_t)pl.G * pl.grid_units);
    const FastDiv g = fast_div_of(pl.G), h = fast_div_of(p.H);
    uint32_t log2_xcc = 0;
    while ((2 << log2_xcc) <= p.xcc) ++log2_xcc;
    uint32_t how = g.shift | h.shift << 5 | log2_xcc << 10;
    if (pl.G > 1 && p.pair_cus == 0 && p.xcc > 1 && total % p.xcc == 0 && (1 << log2_xcc) == p.xcc) how |= HOW_RENUMBER;
    if (p.pair_cus > 0) how |= HOW_PAIR;
    auto kernel = tree_attn_bf16_kernel<D, QBP, NS, F8>;
    if constexpr (F8 || NS == 2)
        if (pl.part_f32) kernel = tree_attn_bf16_short_kernel<D, QBP, NS, F8>;
    if constexpr (has_ragged_kernel<D, QBP, NS, F8>())
        if (pl.S == 1 && p.pair_cus > 0 && total <= 2u * p.pair_cus) kernel = tree_attn_bf16_ragged_kernel<D, QBP, NS, F8>;
    mcsd_launch(MCSD_KERNEL_ATTN_SWEEP, kernel, dim3(total), dim3(SweepCfg<D, QBP, NS, F8>::THREADS), st,
                p.lens, p.seq_base, total >> log2_xcc, (int32_t)pl.G, g.mul, p.H, h.mul, (int32_t)(p.B * p.H), how, p.max_prefix, p.tps, p);
}

template <int D, int QBP>
void launch_merge(const AttnParams &p, const AttnPlan &pl, hipStream_t st)
{
    const size_t threads = (size_t)p.B * p.H * QBP * D * 8;
    mcsd_launch(MCSD_KERNEL_ATTN_MERGE, tree_attn_merge_bf16_kernel<D, QBP>, dim3((unsigned)((threads + 255) / 256)), dim3(256), st, p, pl.T);
}

template <int D>
hipError_t launch_bf16(const AttnParams &p, const AttnPlan &pl, hipStream_t st)
{
    if (pl.QBP == 1) launch_sweep<D, 1, 2>(p, pl, st);
    else if (pl.QBP == 2) { if (pl.NS == 4) launch_sweep<D, 2, 4>(p, pl, st); else launch_sweep<D, 2, 2>(p, pl, st); }
    else { if (pl.NS == 4) launch_sweep<D, 4, 4>(p, pl, st); else launch_sweep<D, 4, 2>(p, pl, st); }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || pl.S == 1 || pl.fold) return e;
    if (pl.QBP == 1) launch_merge<D, 1>(p, pl, st);
    else if (pl.QBP == 2) launch_merge<D, 2>(p, pl, st);
    else launch_merge<D, 4>(p, pl, st);
    return hipGetLastError();
}

// fp8 prefix cache (d = 128): four-stage ring; reference maxima reach the fold in log2 units
hipError_t launch_fp8kv(const AttnParams &p, const AttnPlan &pl, hipStream_t st)
{
    if (pl.QBP == 2) launch_sweep<128, 2, 4, true>(p, pl, st);
    else launch_sweep<128, 4, 4, true>(p, pl, st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || pl.S == 1 || pl.fold) return e;
    AttnParams pm = p;
    pm.c = 1.f;
    if (pl.QBP == 2) launch_merge<128, 2>(pm, pl, st);
    else launch_merge<128, 4>(pm, pl, st);
    return hipGetLastError();
}

template <int D>
hipError_t launch_f32(const AttnParams &p, const AttnPlan &pl, hipStream_t st)
{
    mcsd_launch(MCSD_KERNEL_ATTN_SWEEP, tree_attn_f32_kernel<D>, dim3((unsigned)((size_t)pl.S * pl.QT * pl.grid_units)), dim3(256), st, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || pl.S == 1 || pl.fold) return e;
    mcsd_launch(MCSD_KERNEL_ATTN_MERGE, tree_attn_merge_f32_kernel<D>, dim3((unsigned)((size_t)p.B * p.H * pl.QT)), dim3(256), st, p);
    return hipGetLastError();
}

size_t workspace_query(const mcsd_attention_tuning_t *tune, bool f8, int32_t B, int32_t H_q, int32_t H_kv, int32_t d,
                       int32_t n_nodes, int32_t row_begin, int32_t max_prefix)
{
    if (B < 1 || H_q < 1 || H_kv < 1 || H_q % H_kv != 0 || (d != 64 && d != 128) || n_nodes < 1 ||
        n_nodes > MCSD_ATTN_MAX_NODES || max_prefix < 0 || row_begin < 0 || row_begin >= n_nodes || (f8 && d != 128))
        return 0;
    size_t wa = 0;
    if (tune && tune->key_splits >= 1) {
        wa = workspace_bytes_for(make_plan(MCSD_BF16, B, H_q, H_kv, d, n_nodes - row_begin, n_nodes, max_prefix, f8, tune), MCSD_BF16, B, d);
    } else {
        // What any choice of splits may need, for this number of rows or fewer and this prefix or a shorter one: a workspace
        // sized for the largest call serves the smaller ones, whose splits may be more.
        for (int rows = n_nodes - row_begin; rows > 0; rows = rows > 64 ? 64 : rows > 32 ? 32 : 0) {
            AttnPlan a = make_plan(MCSD_BF16, B, H_q, H_kv, d, rows, n_nodes, max_prefix, f8, tune);
            const long bh = (long)B * a.units, tiles = ((long)max_prefix + a.T - 1) / a.T;
            long most = bh > a.cus ? a.G : 2 * a.cus / bh;
            if (most > tiles + 1) most = tiles + 1;
            if (most > 16) most = 16;
            if (tiles < 2 || most < 1) most = 1;
            a.G = (int)most;
            a.S = most > 1 ? 2 : 1;
            a.part_f32 = 0;
            const size_t w = workspace_bytes_for(a, MCSD_BF16, B, d);
            if (w > wa) wa = w;
            // a short prefix: fewer partial results, each twice the bytes
            const long part = bh * a.QBP * 32 * d * 4, few = (PART_F32_KEYS - 1) / a.T < tiles ? (PART_F32_KEYS - 1) / a.T : tiles;
            if (most > few + 1) most = few + 1;
            if (most > PART_F32_MAX) most = PART_F32_MAX;
            if (most * part > PART_F32_BYTES) most = PART_F32_BYTES / part;
            if (few < 2 || most < 2) continue;
            a.G = (int)most;
            a.part_f32 = 1;
            const size_t w32 = workspace_bytes_for(a, MCSD_BF16, B, d);
            if (w32 > wa) wa = w32;
        }
    }
    if (f8) return wa;
    // the larger of the two dtypes' needs, so one buffer serves both; fp32: for every number of query tiles up to this one
    // (fewer tiles mean more splits: 9 x 32 heads of 64, 243 keys: none with 6 tiles, 3.7 MB with 1) and this prefix, whose
    // splits are at least a shorter one's
    for (int rows = n_nodes - row_begin; rows > 0; rows = tune && tune->key_splits >= 1 ? 0 : (rows - 1) / F32_ROWS * F32_ROWS) {
        const AttnPlan f = make_plan(MCSD_F32, B, H_q, H_kv, d, rows, n_nodes, max_prefix, false, tune);
        const size_t w = workspace_bytes_for(f, MCSD_F32, B, d);
        if (w > wa) wa = w;
    }
    return wa;
}

int attention_call(const mcsd_attention_tuning_t *tune, const mcsd_mask_view_t *mask, mcsd_dtype_t dtype, bool f8,
                   float k_scale, float v_scale, int32_t B,
                   int32_t H_q, int32_t H_kv, int32_t d, int32_t row_begin, const void *q, const void *k_tree,
                   const void *v_tree, int64_t node_stride, const void *k_prefix, const void *v_prefix,
                   const int64_t *seq_base_dev, const int32_t *prefix_lens_dev, int64_t head_stride, int32_t max_prefix,
                   float softmax_scale, void *out, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    const int32_t H = H_q;
    if (H_kv < 1 || H_q < 1 || H_q % H_kv != 0) return MCSD_EINVAL;
    if (!mask || !mask->bits_dev || !q || !k_tree || !v_tree || !out || !seq_base_dev || !prefix_lens_dev)
        return MCSD_EINVAL;
    if (dtype != MCSD_F32 && dtype != MCSD_BF16) return MCSD_EINVAL;
    if (B < 1 || H < 1 || B > 65535 || H > 65535 || max_prefix < 0) return MCSD_EINVAL;
    if (max_prefix > 0 && (!k_prefix || !v_prefix)) return MCSD_EINVAL;
    if (tune && (tune->key_splits < 0 || tune->key_splits > 64 || tune->fold < 0 || tune->fold > 1 ||
                 tune->tree_keys < 0 || tune->tree_keys > 3 ||
                 (tune->stages != 0 && tune->stages != 2 && tune->stages != 4)))
        return MCSD_EINVAL;
    const int32_t n = mask->n_nodes;
    if (n < 1 || node_stride < n || head_stride < 0) return MCSD_EINVAL;
    if (row_begin < 0 || row_begin >= n) return MCSD_EINVAL;
    if (!(softmax_scale > 0.f) || !isfinite(softmax_scale)) return MCSD_EINVAL;
    if (d != 64 && d != 128) return MCSD_EUNSUPPORTED;
    if (n > MCSD_ATTN_MAX_NODES) return MCSD_EUNSUPPORTED;
    if (f8 && (d != 128 || dtype != MCSD_BF16)) return MCSD_EUNSUPPORTED;
    if (f8 && (!(k_scale > 0.f) || !isfinite(k_scale) || !isfinite(v_scale))) return MCSD_EINVAL;
    const uintptr_t align = (uintptr_t)q | (uintptr_t)k_tree | (uintptr_t)v_tree | (uintptr_t)out |
                            (uintptr_t)k_prefix | (uintptr_t)v_prefix;
    if (align & 15) return MCSD_EINVAL;
    if (((node_stride * d) & 7) || (head_stride & (f8 ? 15 : 7))) return MCSD_EINVAL;   // 16-byte rows and heads

    const AttnPlan pl = make_plan(dtype, B, H_q, H_kv, d, n - row_begin, n, max_prefix, f8, tune);
    if ((int64_t)pl.G * pl.QT * pl.grid_units > 0x7fffffff) return MCSD_EUNSUPPORTED;           // one-dimensional grid
    const size_t need = workspace_bytes_for(pl, dtype, B, d);
    if (need > 0 && (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 255))) return MCSD_EWORKSPACE;

    AttnParams p;
    p.q = q; p.kt = k_tree; p.vt = v_tree; p.kp = k_prefix; p.vp = v_prefix; p.out = out;
    p.seq_base = seq_base_dev; p.lens = prefix_lens_dev;
    p.mask_bits = mask->bits_dev; p.mask_words = mask->words_per_row;
    p.B = B; p.H = pl.units; p.n = n; p.row0 = row_begin; p.max_prefix = max_prefix;
    p.Hq = H_q; p.Hkv = H_kv; p.grp = H_q / H_kv; p.hpw = pl.hpw; p.bph = pl.bph; p.chunks = pl.chunks;
    p.log2_bph = pl.bph == 4 ? 2 : pl.bph - 1;
    const FastDiv chunks = fast_div_of(pl.chunks);
    p.mul_chunks = chunks.mul; p.shift_chunks = chunks.shift;
    p.node_stride = node_stride; p.head_stride = head_stride;
    p.c = softmax_scale * 1.4426950408889634f;
    p.k_scale = f8 ? k_scale : 1.f;
    p.v_scale = f8 ? v_scale : 1.f;
    p.S = pl.S; p.G = pl.G; p.SP = pl.G; p.QT = pl.QT;
    p.pair_cus = pl.pair_cus;
    p.tree_last = pl.tree_last;
    p.xcc = pl.xcc;
    p.fold = pl.fold;
    p.part_f32 = pl.part_f32;
    p.tps = (int32_t)((((int64_t)max_prefix + pl.T - 1) / pl.T + pl.S - 1) / pl.S);
    if (p.tps < 1) p.tps = 1;
    const FastDiv tps = fast_div_of(p.tps);
    p.mul_tps = tps.mul; p.shift_tps = tps.shift;
    char *w = (char *)workspace;
    p.part_o = p.part_m = p.part_l = nullptr;
    p.ctr = nullptr;
    p.ws_tag = nullptr;
    if (pl.S > 1) {
        const size_t rows = partial_rows(pl, dtype, B);
        p.ws_tag = (const uint32_t *)w;
        p.ctr = (unsigned long long *)(w + WS_HEADER);
        w += WS_HEADER + WS_CTR_BYTES;
        p.part_m = (float *)w;
        w += align256(rows * sizeof(float));
        p.part_l = (float *)w;
        w += align256(rows * sizeof(float));
        p.part_o = (float *)w;
    }
    hipStream_t st = (hipStream_t)hip_stream;
    hipError_t e;
    if (f8) e = launch_fp8kv(p, pl, st);
    else if (dtype == MCSD_BF16) e = d == 128 ? launch_bf16<128>(p, pl, st) : launch_bf16<64>(p, pl, st);
    else e = d == 128 ? launch_f32<128>(p, pl, st) : launch_f32<64>(p, pl, st);
    return mcsd_hip_status(e);
}

}  // namespace

// ---------------------------------------------------------------------------------------------------
// Entry point that allocates nothing: the workspace is a file-scope device array.  Each GPU the library runs on
// holds its own copy at its own address; the array's name is a host-side stand-in only, so the device address is
// asked for once per device with hipGetSymbolAddress and that pointer, never the name, is what the kernels get.
// ---------------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[MCSD_STATIC_SCRATCH_BYTES];

namespace {
std::atomic<void *> g_scratch_of_device[64];        // device address of `scratch`, null until the first call there
std::atomic<int> g_scratch_prepared[64];            // 1 once the tag word has been written on that device

// Device address of this device's copy of `scratch`; the first call on a device also enqueues the fill kernel that
// writes the workspace tag (the counters start as zeros like all of the array, and every launch leaves them zero).
int static_scratch(hipStream_t st, void **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MCSD_EHIP;
    void *ptr = g_scratch_of_device[dev].load(std::memory_order_acquire);
    if (!ptr) {
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return MCSD_EHIP;
        }
        g_scratch_of_device[dev].store(ptr, std::memory_order_release);
    }
    if (g_scratch_prepared[dev].load(std::memory_order_acquire) == 0) {
        const unsigned n16 = (unsigned)((WS_HEADER + WS_CTR_BYTES) / 16);
        hipLaunchKernelGGL(workspace_init_kernel, dim3((n16 + 255) / 256), dim3(256), 0, st, (uint4 *)ptr);
        if (hipGetLastError() != hipSuccess) return MCSD_EHIP;
        g_scratch_prepared[dev].store(1, std::memory_order_release);
    }
    *out = ptr;
    return MCSD_OK;
}
}  // namespace

extern "C" int mcsd_tree_attention_static(const mcsd_mask_view_t *mask, mcsd_dtype_t dtype, int32_t B, int32_t H,
                                          int32_t d, const void *q, const void *k_tree, const void *v_tree,
                                          int64_t node_stride, const void *k_prefix, const void *v_prefix,
                                          const int64_t *seq_base_dev, const int32_t *prefix_lens_dev,
                                          int64_t head_stride, int32_t max_prefix, float softmax_scale, void *out,
                                          void *hip_stream)
{
    if (!mask || B < 1 || H < 1 || max_prefix < 0 || (d != 64 && d != 128) || mask->n_nodes < 1 ||
        mask->n_nodes > MCSD_ATTN_MAX_NODES || (dtype != MCSD_F32 && dtype != MCSD_BF16))
        return attention_call(nullptr, mask, dtype, false, 1.f, 1.f, B, H, H, d, 0, q, k_tree, v_tree, node_stride, k_prefix,
                              v_prefix, seq_base_dev, prefix_lens_dev, head_stride, max_prefix, softmax_scale, out, nullptr,
                              0, hip_stream);          // (reports the argument error; nothing is launched)
    // the shape's need against the array's size, before anything is enqueued
    const AttnPlan pl = make_plan(dtype, B, H, H, d, mask->n_nodes, mask->n_nodes, max_prefix);
    if (workspace_bytes_for(pl, dtype, B, d) > (size_t)MCSD_STATIC_SCRATCH_BYTES) return MCSD_EUNSUPPORTED;
    void *ws = nullptr;
    const int rc = static_scratch((hipStream_t)hip_stream, &ws);
    if (rc != MCSD_OK) return rc;
    return attention_call(nullptr, mask, dtype, false, 1.f, 1.f, B, H, H, d, 0, q, k_tree, v_tree, node_stride, k_prefix,
                          v_prefix, seq_base_dev, prefix_lens_dev, head_stride, max_prefix, softmax_scale, out, ws,
                          (size_t)MCSD_STATIC_SCRATCH_BYTES, hip_stream);
}

extern "C" int mcsd_workspace_init(void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!workspace && workspace_bytes > 0) return MCSD_EINVAL;
    if ((uintptr_t)workspace & 255) return MCSD_EINVAL;
    if (workspace_bytes < WS_HEADER + WS_CTR_BYTES) return MCSD_OK;    // too small to serve a call that needs one
    const unsigned n16 = (unsigned)((WS_HEADER + WS_CTR_BYTES) / 16);
    hipLaunchKernelGGL(workspace_init_kernel, dim3((n16 + 255) / 256), dim3(256), 0, (hipStream_t)hip_stream, (uint4 *)workspace);
    return mcsd_hip_status(hipGetLastError());
}

extern "C" size_t mcsd_tree_attention_gqa_workspace(int32_t B, int32_t H_q, int32_t H_kv, int32_t d, int32_t n_nodes,
                                                    int32_t row_begin, int32_t max_prefix)
{
    return workspace_query(nullptr, false, B, H_q, H_kv, d, n_nodes, row_begin, max_prefix);
}

extern "C" size_t mcsd_tree_attention_rows_workspace(int32_t B, int32_t H, int32_t d, int32_t n_nodes,
                                                     int32_t row_begin, int32_t max_prefix)
{
    return workspace_query(nullptr, false, B, H, H, d, n_nodes, row_begin, max_prefix);
}

extern "C" size_t mcsd_tree_attention_workspace(int32_t B, int32_t H, int32_t d, int32_t n_nodes, int32_t max_prefix)
{
    return workspace_query(nullptr, false, B, H, H, d, n_nodes, 0, max_prefix);
}

extern "C" size_t mcsd_tree_attention_fp8kv_workspace(int32_t B, int32_t H_q, int32_t H_kv, int32_t n_nodes,
                                                      int32_t row_begin, int32_t max_prefix)
{
    return workspace_query(nullptr, true, B, H_q, H_kv, 128, n_nodes, row_begin, max_prefix);
}

extern "C" size_t mcsd_tree_attention_tuned_workspace(const mcsd_attention_tuning_t *tuning, int32_t prefix_fp8, int32_t B,
                                                      int32_t H_q, int32_t H_kv, int32_t d, int32_t n_nodes,
                                                      int32_t row_begin, int32_t max_prefix)
{
    if (tuning && (tuning->key_splits < 0 || tuning->key_splits > 64)) return 0;
    return workspace_query(tuning, prefix_fp8 != 0, B, H_q, H_kv, d, n_nodes, row_begin, max_prefix);
}

extern "C" int mcsd_tree_attention_plan(const mcsd_attention_tuning_t *tuning, mcsd_dtype_t dtype, int32_t prefix_fp8,
                                        int32_t B, int32_t H_q, int32_t H_kv, int32_t d, int32_t n_nodes, int32_t row_begin,
                                        int32_t max_prefix, mcsd_attention_plan_t *out)
{
    if (!out || B < 1 || H_q < 1 || H_kv < 1 || H_q % H_kv != 0 || (d != 64 && d != 128) || n_nodes < 1 ||
        n_nodes > MCSD_ATTN_MAX_NODES || max_prefix < 0 || row_begin < 0 || row_begin >= n_nodes ||
        (dtype != MCSD_F32 && dtype != MCSD_BF16) || (prefix_fp8 && (d != 128 || dtype != MCSD_BF16)))
        return MCSD_EINVAL;
    if (tuning && (tuning->key_splits < 0 || tuning->key_splits > 64 || tuning->fold < 0 || tuning->fold > 1 ||
                   tuning->tree_keys < 0 || tuning->tree_keys > 3 ||
                   (tuning->stages != 0 && tuning->stages != 2 && tuning->stages != 4)))
        return MCSD_EINVAL;
    const AttnPlan pl = make_plan(dtype, B, H_q, H_kv, d, n_nodes - row_begin, n_nodes, max_prefix, prefix_fp8 != 0, tuning);
    out->mfma_path = dtype == MCSD_BF16;
    out->query_blocks = pl.QBP;
    out->key_splits = pl.S;
    out->workgroups = (int32_t)((int64_t)pl.G * pl.QT * pl.grid_units);
    out->stages = dtype == MCSD_BF16 ? pl.NS : 0;
    out->fold_in_kernel = pl.fold;
    out->ordered_by_length = pl.pair_cus > 0;
    return MCSD_OK;
}

extern "C" int mcsd_tree_attention(const mcsd_mask_view_t *mask, mcsd_dtype_t dtype, int32_t B, int32_t H, int32_t d,
                                   const void *q, const void *k_tree, const void *v_tree, int64_t node_stride,
                                   const void *k_prefix, const void *v_prefix, const int64_t *seq_base_dev,
                                   const int32_t *prefix_lens_dev, int64_t head_stride, int32_t max_prefix,
                                   float softmax_scale, void *out, void *workspace, size_t workspace_bytes,
                                   void *hip_stream)
{
    return attention_call(nullptr, mask, dtype, false, 1.f, 1.f, B, H, H, d, 0, q, k_tree, v_tree, node_stride, k_prefix,
                          v_prefix, seq_base_dev, prefix_lens_dev, head_stride, max_prefix, softmax_scale, out, workspace,
                          workspace_bytes, hip_stream);
}

extern "C" int mcsd_tree_attention_rows(const mcsd_mask_view_t *mask, mcsd_dtype_t dtype, int32_t B, int32_t H,
                                        int32_t d, int32_t row_begin, const void *q, const void *k_tree,
                                        const void *v_tree, int64_t node_stride, const void *k_prefix,
                                        const void *v_prefix, const int64_t *seq_base_dev,
                                        const int32_t *prefix_lens_dev, int64_t head_stride, int32_t max_prefix,
                                        float softmax_scale, void *out, void *workspace, size_t workspace_bytes,
                                        void *hip_stream)
{
    return attention_call(nullptr, mask, dtype, false, 1.f, 1.f, B, H, H, d, row_begin, q, k_tree, v_tree, node_stride,
                          k_prefix, v_prefix, seq_base_dev, prefix_lens_dev, head_stride, max_prefix, softmax_scale, out,
                          workspace, workspace_bytes, hip_stream);
}

extern "C" int mcsd_tree_attention_gqa(const mcsd_mask_view_t *mask, mcsd_dtype_t dtype, int32_t B, int32_t H_q,
                                       int32_t H_kv, int32_t d, int32_t row_begin, const void *q, const void *k_tree,
                                       const void *v_tree, int64_t node_stride, const void *k_prefix,
                                       const void *v_prefix, const int64_t *seq_base_dev,
                                       const int32_t *prefix_lens_dev, int64_t head_stride, int32_t max_prefix,
                                       float softmax_scale, void *out, void *workspace, size_t workspace_bytes,
                                       void *hip_stream)
{
    return attention_call(nullptr, mask, dtype, false, 1.f, 1.f, B, H_q, H_kv, d, row_begin, q, k_tree, v_tree,
                          node_stride, k_prefix, v_prefix, seq_base_dev, prefix_lens_dev, head_stride, max_prefix,
                          softmax_scale, out, workspace, workspace_bytes, hip_stream);
}

extern "C" int mcsd_tree_attention_fp8kv(const mcsd_mask_view_t *mask, int32_t B, int32_t H_q, int32_t H_kv,
                                         int32_t row_begin, const void *q, const void *k_tree, const void *v_tree,
                                         int64_t node_stride, const void *k_prefix_fp8, const void *v_prefix_fp8,
                                         float k_scale, float v_scale, const int64_t *seq_base_dev,
                                         const int32_t *prefix_lens_dev, int64_t head_stride, int32_t max_prefix,
                                         float softmax_scale, void *out, void *workspace, size_t workspace_bytes,
                                         void *hip_stream)
{
    return attention_call(nullptr, mask, MCSD_BF16, true, k_scale, v_scale, B, H_q, H_kv, 128, row_begin, q, k_tree,
                          v_tree, node_stride, k_prefix_fp8, v_prefix_fp8, seq_base_dev, prefix_lens_dev, head_stride,
                          max_prefix, softmax_scale, out, workspace, workspace_bytes, hip_stream);
}

extern "C" int mcsd_tree_attention_tuned(const mcsd_attention_tuning_t *tuning, const mcsd_mask_view_t *mask,
                                         mcsd_dtype_t dtype, int32_t prefix_fp8, float k_scale, float v_scale, int32_t B,
                                         int32_t H_q, int32_t H_kv, int32_t d, int32_t row_begin, const void *q,
                                         const void *k_tree, const void *v_tree, int64_t node_stride,
                                         const void *k_prefix, const void *v_prefix, const int64_t *seq_base_dev,
                                         const int32_t *prefix_lens_dev, int64_t head_stride, int32_t max_prefix,
                                         float softmax_scale, void *out, void *workspace, size_t workspace_bytes,
                                         void *hip_stream)
{
    return attention_call(tuning, mask, dtype, prefix_fp8 != 0, k_scale, v_scale, B, H_q, H_kv, d, row_begin, q, k_tree,
                          v_tree, node_stride, k_prefix, v_prefix, seq_base_dev, prefix_lens_dev, head_stride, max_prefix,
                          softmax_scale, out, workspace, workspace_bytes, hip_stream);
}
