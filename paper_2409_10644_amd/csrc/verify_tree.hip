// Multi-candidate verification for gfx950 (Sec. 2.1, Sec. 3.1 and Fig. 1 steps 4-6 of arXiv 2409.10644):
// recursive rejection sampling down the candidate tree, longest-path selection for target-initialised
// trees, and sampling of the new token(s).
//
// A walk (one tree, or one level-1 subtree of a target-initialised one) is latency: a chain of row fetches, vocabulary sums
// and accept tests.  Sums over the vocabulary follow the balanced binary tree over the zero-padded index space that the
// header specifies; all arithmetic is binary64 with explicit fma, so results equal the oracle's recursion bit for bit.
//
// verify_walk_team_kernel: several workgroups share a walk, each holding an aligned power-of-two chunk of the vocabulary
// (4096 to 16384 entries) in registers, so the rows arrive through as many compute units as share the walk and no row is
// read twice; they exchange one partial sum per rejection round.  A context visited after its first rejection costs a row
// fetch (0.5-1 us) and 1.5-2 us a round.  Measured, rows in the last-level cache, us per call before (one workgroup per
// walk; vocabularies above 32768 streamed from memory every round) and after: 1 walk of 32000 entries 11.5 -> 7.1, 128 of
// 32000 25 -> 21, 64 (8 sequences, target-initialised) 19.8 -> 16, 16 of 131072 171 -> 17, 1 of 34347 66 -> 8.8.
//
// verify_walk_fast_kernel: one workgroup per walk, for vocabularies up to 32768 when there are more walks than the chip
// has room for teams.  Lane t owns the 32 CONSECUTIVE elements 32 t .. 32 t + 31: an aligned subtree of the sum tree, so
// a sum is 31 in-lane additions, one 6-level butterfly over the wavefront's 64 lanes and a 4-level tree over the 16
// wavefront sums (one barrier per rejection round).  The residual r <- max(r - S q, 0) lives in registers as
// binary64 and is updated in place; the draft row is parked in LDS.  Rows are fetched with coalesced 16-byte loads
// and handed to their owner lanes through LDS (a wavefront's 2048 elements stay inside the wavefront, so the
// hand-over needs no barrier); the LDS image is XOR-swizzled so that both sides are free of bank conflicts.
// New tokens are drawn by the wavefronts independently (wavefront k takes draws k, k + 16, ..): the 16 wavefront
// sums, then the heap of the chosen wavefront's lane sums (kept in LDS from the butterfly's levels), then the 32
// elements of the chosen lane, recomputed from the rows and the history of sums.
//
// Compiled with -ffp-contract=off.
#include <atomic>
#include <chrono>

#include "mcsd_internal.h"
#include "team_protocol.h"

namespace {

constexpr int VT = 1024;                 // threads per workgroup

struct VerifyParams {
    McsdTreeDesc t;
    int32_t mode, B, V, n_nodes, n_new, R;
    const int32_t *tokens;
    const float *p, *q;
    int64_t pbs, qbs;
    const float *ua, *us;
    const int32_t *parent;               // of every tree node, -1 on level 1
    int32_t *cand_path;                  // [B][R][gamma]
    int32_t *cand_len;                   // [B][R]
    int32_t *cand_new;                   // [B][R][n_new]
    // target-initialised trees: where the longest walk goes, and with what the walks of a sequence find out who is last
    int32_t *out_path, *out_len, *out_new;
    unsigned long long *done;            // [B][R * workgroups per walk]
    unsigned long long launch_id;        // of this launch alone; never 0
};

// A result that workgroups on other dies read in the same launch: written through to where they see it.
__device__ inline void put(int32_t *at, int32_t v) { __hip_atomic_store(at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline int32_t get(const int32_t *at) { return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// max(d, 0) as one instruction.  d is never NaN here, and the sign of a zero result never reaches a decision
// (zeros only enter sums, products and comparisons with 0), so this equals "d > 0 ? d : 0" for every use below.
__device__ inline double pos_part(double d) { return __builtin_fmax(d, 0.0); }

// The rejections at a context: S before each round; for candidates without replacement also the sum of the shrunken
// draft row before each round and the token rejected in it (its draft mass is zero afterwards).
struct History {
    double s[MCSD_MAX_BRANCH + 1], sq[MCSD_MAX_BRANCH + 1];
    int x[MCSD_MAX_BRANCH + 1];
};

// One element of the distribution after `rounds` rejections, from its target value r and draft value qd.
// With replacement: r <- max(r - S q, 0) per round.  NOREP (candidates drawn without replacement): the draft row
// loses every rejected token, and with Sq the sum of what is left, r <- max(r Sq - S q', 0).
template <bool NOREP>
__device__ inline double residual_chain(const History &h, double r, double qd, int t, int rounds)
{
    for (int k = 0; k < rounds; ++k) {
        if (NOREP) {
            if (k > 0 && t == h.x[k - 1]) qd = 0.0;
            r = __dmul_rn(r, h.sq[k]);
        }
        const double d = __fma_rn(-h.s[k], qd, r);
        r = pos_part(d);
    }
    return r;
}

// Element t of the distribution after `rounds` rejections at a context with rows prow / qrow.
template <bool NOREP>
__device__ inline double residual_at(const History &h, const float *prow, const float *qrow, int rounds, int t)
{
    const double r = (double)prow[t];
    return rounds > 0 ? residual_chain<NOREP>(h, r, (double)qrow[t], t, rounds) : r;
}

// A double from another lane of the row through the data-parallel-primitive path of the vector ALU (no LDS).
template <int CTRL>
__device__ inline double dpp_f64(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// Sum over the 64 lanes in balanced-tree order (lane pairs, then pairs of pairs, ...); every lane gets the total.
// Partner lanes: l^1 and l^2 by quad permutation; then, since all lanes of a group of 4 (8) already hold the same
// value, the mirrored lane of the half row (row) stands in for l^4 (l^8); l^16 by swizzle; l^32 by the half-wave
// swap, whose two results are {own, partner} in an order that the commutative addition does not care about.
__device__ inline double wave_tree_sum(double v)
{
    v = __dadd_rn(v, dpp_f64<0xB1>(v));          // quad_perm [1,0,3,2]
    v = __dadd_rn(v, dpp_f64<0x4E>(v));          // quad_perm [2,3,0,1]
    v = __dadd_rn(v, dpp_f64<0x141>(v));         // row_half_mirror
    v = __dadd_rn(v, dpp_f64<0x140>(v));         // row_mirror
    {
        const int lo = __builtin_amdgcn_ds_swizzle(__double2loint(v), 0x401F);   // lane ^ 16 inside each 32
        const int hi = __builtin_amdgcn_ds_swizzle(__double2hiint(v), 0x401F);
        v = __dadd_rn(v, __hiloint2double(hi, lo));
    }
    {
        const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(v), (unsigned)__double2loint(v), false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(v), (unsigned)__double2hiint(v), false, false);
        v = __dadd_rn(__hiloint2double((int)hi[0], (int)lo[0]), __hiloint2double((int)hi[1], (int)lo[1]));
    }
    return v;
}

// Target-initialised trees: the level-1 subtree with the longest accepted path wins, lowest id on ties.  Every workgroup of
// a sequence calls this when its results are written; the one that finds all of them done copies the winner out, inside
// the same launch (a second kernel cost 4 us).  A workgroup marks itself done, and only then looks at the others' marks:
// the last to mark sees them all.  Two may, and then write the same values.  A mark is the launch's own id, so what the
// workspace held before does not matter, and the copier takes all marks back, so a replay of the same launch starts clean.
__device__ inline void select_longest(const VerifyParams &P, int b, int slot, int slots)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // this wavefront's results are where everyone sees them ...
    __syncthreads();                                        // ... and everyone's of the workgroup
    if (threadIdx.x >= 64) return;
    const int lane = threadIdx.x;
    unsigned long long *done = P.done + (int64_t)b * slots;
    if (lane == 0) __hip_atomic_store(&done[slot], P.launch_id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    bool all = true;
    for (int i = lane; i < slots; i += 64) all = all && __hip_atomic_load(&done[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == P.launch_id;
    if (__builtin_amdgcn_ballot_w64(!all) != 0) return;
    int key = -1;                                           // longest first, then lowest id (R <= 64)
    if (lane < P.R) key = get(P.cand_len + (int64_t)b * P.R + lane) * 64 + (63 - lane);
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        const int o = __shfl_xor(key, m, 64);
        key = o > key ? o : key;
    }
    const int best = 63 - (key & 63);
    const int64_t c = (int64_t)b * P.R + best;
    if (lane == 0) P.out_len[b] = key >> 6;
    if (lane < P.t.gamma) P.out_path[(int64_t)b * P.t.gamma + lane] = get(P.cand_path + c * P.t.gamma + lane);
    if (lane < P.n_new) P.out_new[(int64_t)b * P.n_new + lane] = get(P.cand_new + c * P.n_new + lane);
    for (int i = lane; i < slots; i += 64) __hip_atomic_store(&done[i], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What the walk needs to know about the tree's nodes, fetched at the start by one lane per node: two dependent trips to
// memory for the whole walk instead of two per context.
constexpr int NODE_CACHE = 256;          // trees of up to this many nodes; larger ones are read context by context
struct NodeCache {
    float u[NODE_CACHE], q[NODE_CACHE], p[NODE_CACHE];      // acceptance uniform, draft and target value of the node's token
    int x[NODE_CACHE];                                      // token
    unsigned kid[NODE_CACHE + 1];                           // of context c (node c - 1): first child, bit 31: accepted at once
};
struct NodeRegs { int x, par, prev; float u; bool mine; };

// Node tid's token and uniform are requested ...
__device__ inline NodeRegs node_request(const VerifyParams &P, const int32_t *tokens, const float *ua, int i)
{
    NodeRegs n{0, -1, -2, 0.f, false};
    // (level 1 of a target-initialised tree goes untested)
    n.mine = P.n_nodes <= NODE_CACHE && i < P.n_nodes && !(P.mode == MCSD_TARGET_INIT && i < P.t.off[1]);
    if (n.mine) {
        n.x = tokens[i];
        n.par = P.parent[i];
        if (i > 0) n.prev = P.parent[i - 1];
        n.u = ua[i];
    }
    return n;
}
// ... and its probabilities fetched.  With S = 1 the first child of a context passes or fails its test whatever happened
// before, so that test is made here, for all contexts at once.  The caller's barrier makes the cache visible.
__device__ inline void node_fetch(NodeCache &c, const VerifyParams &P, const float *p, const float *q, NodeRegs n, int i)
{
    if (!n.mine) return;
    const int x = n.x < 0 ? 0 : (n.x >= P.V ? P.V - 1 : n.x);   // ids outside 0..V-1 are clamped, never dereferenced
    const float qx = q[(int64_t)(n.par + 1) * P.V + x], px = p[(int64_t)(n.par + 1) * P.V + x];
    c.x[i] = x;
    c.u[i] = n.u;
    c.q[i] = qx;
    c.p[i] = px;
    if (n.prev != n.par) c.kid[n.par + 1] = (unsigned)i | (__dmul_rn((double)n.u, (double)qx) < (double)px ? 0x80000000u : 0u);
}

// ---------------------------------------------------------------------------------------------------
// Vocabularies up to FAST_V: rows held by the workgroup, 32 consecutive elements per lane
// ---------------------------------------------------------------------------------------------------
constexpr int EPL = 32;                  // consecutive vocabulary elements per lane
constexpr int FAST_V = VT * EPL;         // 32768
constexpr int NWAVE = VT / 64;           // 16
constexpr int WCHUNKS = 64 * EPL / 4;    // 16-byte chunks of a wavefront's 2048 elements

struct FastShared {
    float qrow[FAST_V];                  // the context's draft row; wavefront w owns [2048 w, 2048 w + 2048), swizzled
    double wsum[2][NWAVE];               // sums of the wavefronts' 2048-element subtrees, double-buffered over rounds
    double heapw[NWAVE][128];            // per wavefront: heap over its 64 lane sums (root 1, leaves 64..127), for sampling
    History hist;                        // of the current context
    NodeCache node;
    int path[MCSD_MAX_LEVELS];           // accepted nodes so far, written out at the end (a store in flight delays every later load)
};

// Position of chunk j (elements 4 j .. 4 j + 3 of the lane's 32) of lane l inside the wavefront's region, in 16-byte
// chunks.  The XOR makes the 16 lanes that LDS serves together hit 16 different 16-byte bank groups both when lanes
// read their own chunk j (lane stride 128 bytes) and when they write consecutive chunks of a row (see fast_load_row).
__device__ inline int fast_slot(int l, int j) { return l * 8 + (j ^ ((l >> 1) & 7)); }

// One row (V floats) from global memory into the wavefront's LDS region: coalesced 16-byte loads (lane i of load k
// fetches the wavefront's chunk 64 k + i), stored where the owner lane will look for it.  Elements beyond V are 0.
__device__ inline void fast_fetch_row(const VerifyParams &P, const float *row, float4 (&v)[8])
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));          // (offsets recomputed at every use instead of kept in registers for the whole walk)
    const int wave = t >> 6, lane = t & 63;
    if ((((uintptr_t)row & 15) | (P.V & 3)) == 0) {            // aligned rows: a chunk is inside V or outside as a whole
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int t0 = (wave * WCHUNKS + k * 64 + lane) * 4;
            v[k] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (t0 < P.V) v[k] = *(const float4 *)(row + t0);
        }
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int t0 = (wave * WCHUNKS + k * 64 + lane) * 4;
            v[k].x = t0 + 0 < P.V ? row[t0 + 0] : 0.f;
            v[k].y = t0 + 1 < P.V ? row[t0 + 1] : 0.f;
            v[k].z = t0 + 2 < P.V ? row[t0 + 2] : 0.f;
            v[k].w = t0 + 3 < P.V ? row[t0 + 3] : 0.f;
        }
    }
}
__device__ inline void fast_park_row(float4 *region, const float4 (&v)[8])
{
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));       // (LDS addresses recomputed here, a few integer operations, instead of spilled)
#pragma unroll
    for (int k = 0; k < 8; ++k) region[fast_slot(k * 8 + (lane >> 3), lane & 7)] = v[k];   // chunk 64 k + lane: owner lane, its chunk
}

// Sum of the lane's 32 elements in tree order (pairs, pairs of pairs, ...).
__device__ inline double lane_tree_sum(const double (&r)[EPL])
{
    double q[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) q[j] = __dadd_rn(__dadd_rn(r[4 * j], r[4 * j + 1]), __dadd_rn(r[4 * j + 2], r[4 * j + 3]));
    return __dadd_rn(__dadd_rn(__dadd_rn(q[0], q[1]), __dadd_rn(q[2], q[3])), __dadd_rn(__dadd_rn(q[4], q[5]), __dadd_rn(q[6], q[7])));
}

// The four tree levels over 16 values held by lanes 0..15 of every row of 16 lanes (partners l^1, l^2, then the
// mirrored lanes standing in for l^4 and l^8, as in wave_tree_sum).
__device__ inline double row16_tree_sum(double v)
{
    v = __dadd_rn(v, dpp_f64<0xB1>(v));
    v = __dadd_rn(v, dpp_f64<0x4E>(v));
    v = __dadd_rn(v, dpp_f64<0x141>(v));
    v = __dadd_rn(v, dpp_f64<0x140>(v));
    return v;
}

// Lane `src` (uniform) of a double.
__device__ inline double read_lane_f64(double v, int src)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), src), __builtin_amdgcn_readlane(__double2loint(v), src));
}

// One inverse-CDF draw from the terminal distribution by ONE wavefront (all 64 lanes call it; no barrier inside).
// wsum[buf] holds the wavefront sums and heapw the lane-sum heaps of that distribution; its elements are recomputed
// from the rows and the history (prow, qrow, rounds).  Returns the token in every lane.
template <bool NOREP>
__device__ int fast_sample(const FastShared &sh, const VerifyParams &P, int buf, const float *prow, const float *qrow,
                           int rounds, float u)
{
    const int lane = threadIdx.x & 63;
    // heap over the 16 wavefront sums, in registers: n[16 + w] = sum of wavefront w
    double n[32];
#pragma unroll
    for (int w = 0; w < NWAVE; ++w) n[16 + w] = sh.wsum[buf][w];
#pragma unroll
    for (int i = 15; i >= 1; --i) n[i] = __dadd_rn(n[2 * i], n[2 * i + 1]);
    double thr = __dmul_rn((double)u, n[1]);
    int node = 1;
#pragma unroll
    for (int lvl = 0; lvl < 4; ++lvl) {
        double left = 0.0;
#pragma unroll
        for (int j = 0; j < (1 << lvl); ++j)
            if (node == (1 << lvl) + j) left = n[2 * ((1 << lvl) + j)];      // (selects: registers cannot be indexed at run time)
        if (thr < left) {
            node = 2 * node;
        } else {
            thr = __dsub_rn(thr, left);
            node = 2 * node + 1;
        }
    }
    const int w = node - 16;
    node = 1;
    while (node < 64) {
        const double left = sh.heapw[w][2 * node];
        if (thr < left) {
            node = 2 * node;
        } else {
            thr = __dsub_rn(thr, left);
            node = 2 * node + 1;
        }
    }
    const int t0 = (w * 64 + (node - 64)) * EPL;          // first element of the chosen lane
    // its 32 elements, one per lane of this wavefront (lanes 32..63 hold zeros), and the levels of their sum tree
    const int te = t0 + lane;
    double lv[6];
    lv[0] = (lane < EPL && te < P.V) ? residual_at<NOREP>(sh.hist, prow, qrow, rounds, te) : 0.0;
    lv[1] = __dadd_rn(lv[0], dpp_f64<0xB1>(lv[0]));
    lv[2] = __dadd_rn(lv[1], dpp_f64<0x4E>(lv[1]));
    lv[3] = __dadd_rn(lv[2], dpp_f64<0x141>(lv[2]));
    lv[4] = __dadd_rn(lv[3], dpp_f64<0x140>(lv[3]));
    int lo = 0;
#pragma unroll
    for (int j = 5; j >= 1; --j) {                         // the node covers lanes lo .. lo + 2^j - 1
        const double left = read_lane_f64(lv[j - 1], lo);
        if (!(thr < left)) {
            thr = __dsub_rn(thr, left);
            lo += 1 << (j - 1);
        }
    }
    int t = t0 + lo;
    if (t < P.V && read_lane_f64(lv[0], lo) > 0.0) return t;
    // Reached a zero-weight index (last-bit rounding of the subtraction, or an all-zero distribution):
    // nearest positive-weight index below, else nearest above, else 0.
    int below = -1, above = 0x7fffffff;
    for (int e = lane; e < P.V; e += 64) {
        if (e == t) continue;
        if (residual_at<NOREP>(sh.hist, prow, qrow, rounds, e) > 0.0) {
            if (e < t) below = e > below ? e : below;
            else above = e < above ? e : above;
        }
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        const int ob = __shfl_xor(below, m, 64), oa = __shfl_xor(above, m, 64);
        below = ob > below ? ob : below;
        above = oa < above ? oa : above;
    }
    return below >= 0 ? below : (above != 0x7fffffff ? above : 0);
}

template <bool NOREP>
__global__ __launch_bounds__(VT) void verify_walk_fast_kernel(const VerifyParams P)
{
    __shared__ FastShared sh;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int root = blockIdx.x, b = blockIdx.y;
    const int32_t *tokens = P.tokens + (int64_t)b * P.n_nodes;
    const float *p = P.p + (int64_t)b * P.pbs;
    const float *q = P.q + (int64_t)b * P.qbs;
    const float *ua = P.ua + (int64_t)b * P.n_nodes;
    int32_t *path_out = P.cand_path + ((int64_t)b * P.R + root) * P.t.gamma;
    float4 *region = (float4 *)sh.qrow + wave * WCHUNKS;      // this wavefront's part of the parked row
    const bool cached = P.n_nodes <= NODE_CACHE;
    node_fetch(sh.node, P, p, q, node_request(P, tokens, ua, tid), tid);

    int cur = -1, level = 0, n_acc = 0;      // context: node id (-1 = end of the prefix) and its level
    if (P.mode == MCSD_TARGET_INIT) {         // level-1 node `root` is accepted untested
        cur = root;
        level = 1;
        n_acc = 1;
        if (tid == 0) sh.path[0] = root;
    }
    double r[EPL];                            // this lane's 32 elements of the current residual
    const float *term_p = nullptr, *term_q = nullptr;
    int term_rounds = 0;
    bool term_in_regs = false;                // r holds the terminal distribution (a residual with positive sum)
    int buf = 0;

    // the target row `prow` into r: fetched coalesced, handed to the owner lanes through this wavefront's LDS region
    auto row_to_regs = [&](const float4 (&pv)[8]) {
        fast_park_row(region, pv);
        int ln = lane;
        asm volatile("" : "+v"(ln));
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float4 v = region[fast_slot(ln, j)];
            r[4 * j] = (double)v.x; r[4 * j + 1] = (double)v.y; r[4 * j + 2] = (double)v.z; r[4 * j + 3] = (double)v.w;
        }
    };
    // sum of r over the vocabulary; with `heap` the levels of the wavefront's butterfly are kept for the sampler.
    // One barrier; wsum[buf] is written, the other buffer may still be read by slower wavefronts.
    auto total = [&](bool heap) {
        double v = lane_tree_sum(r);
        if (heap) sh.heapw[wave][64 + lane] = v;
        v = __dadd_rn(v, dpp_f64<0xB1>(v));
        if (heap && (lane & 1) == 0) sh.heapw[wave][32 + (lane >> 1)] = v;
        v = __dadd_rn(v, dpp_f64<0x4E>(v));
        if (heap && (lane & 3) == 0) sh.heapw[wave][16 + (lane >> 2)] = v;
        v = __dadd_rn(v, dpp_f64<0x141>(v));
        if (heap && (lane & 7) == 0) sh.heapw[wave][8 + (lane >> 3)] = v;
        v = __dadd_rn(v, dpp_f64<0x140>(v));
        if (heap && (lane & 15) == 0) sh.heapw[wave][4 + (lane >> 4)] = v;
        {
            const int lo = __builtin_amdgcn_ds_swizzle(__double2loint(v), 0x401F);   // lane ^ 16 inside each 32
            const int hi = __builtin_amdgcn_ds_swizzle(__double2hiint(v), 0x401F);
            v = __dadd_rn(v, __hiloint2double(hi, lo));
        }
        if (heap && (lane & 31) == 0) sh.heapw[wave][2 + (lane >> 5)] = v;
        {
            const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(v), (unsigned)__double2loint(v), false, false);
            const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(v), (unsigned)__double2hiint(v), false, false);
            v = __dadd_rn(__hiloint2double((int)hi[0], (int)lo[0]), __hiloint2double((int)hi[1], (int)lo[1]));
        }
        if (lane == 0) {
            sh.wsum[buf][wave] = v;
            if (heap) sh.heapw[wave][1] = v;
        }
        __syncthreads();
        return read_lane_f64(row16_tree_sum(sh.wsum[buf][lane & 15]), 0);
    };

    __syncthreads();                          // the node cache is visible
    // The walk is the same in all lanes and has to be scalar control flow; see verify_walk_team_kernel.
    while (true) {
        level = __builtin_amdgcn_readfirstlane(level);
        cur = __builtin_amdgcn_readfirstlane(cur);
        n_acc = __builtin_amdgcn_readfirstlane(n_acc);
        unsigned kid = 0;
        if (cached) {                         // contexts whose first candidate passes need nothing but that fact
            while (level < P.t.gamma) {
                kid = __builtin_amdgcn_readfirstlane(sh.node.kid[cur + 1]);
                if (!(kid >> 31)) break;
                cur = (int)(kid & 0x7fffffffu);
                if (tid == 0) sh.path[n_acc] = cur;
                n_acc += 1;
                level += 1;
            }
        }
        if (level >= P.t.gamma) break;
        const float *prow = p + (int64_t)(cur + 1) * P.V;
        const float *qrow = q + (int64_t)(cur + 1) * P.V;
        const int cnt = P.t.b[level];
        const int first = cached ? (int)kid : (cur < 0 ? 0 : P.t.off[level] + (cur - P.t.off[level - 1]) * cnt);
        // candidate `lane` of this context (in every wavefront): acceptance uniform, q(x) and the residual at x,
        // which is updated in place after every rejection
        double uc = 0.0, qc = 0.0, rc = 0.0;
        int xc = -1;
        auto candidates = [&]() {
            if (lane >= cnt) return;
            const int i = first + lane;
            if (cached) {
                xc = sh.node.x[i];
                uc = (double)sh.node.u[i];
                qc = (double)sh.node.q[i];
                rc = (double)sh.node.p[i];
            } else {
                int x = tokens[i];
                x = x < 0 ? 0 : (x >= P.V ? P.V - 1 : x);   // ids outside 0..V-1 are clamped, never dereferenced
                float u = ua[i], qx = qrow[x], px = prow[x];
                asm volatile("" : "+v"(u), "+v"(qx), "+v"(px));      // (keeps the compiler from merging these loads with those above)
                xc = x;
                uc = (double)u;
                qc = (double)qx;
                rc = (double)px;
            }
        };
        int rounds = 0, accepted = -1;
        double S = 1.0, Sq = 1.0;                        // both rows are trusted to be normalised in round 0
        // accept test of candidate c, evaluated by its lane; the same answer in every wavefront
        auto accept = [&](int c) {
            const double rhs = NOREP ? __dmul_rn(rc, Sq) : rc;
            return __builtin_amdgcn_readlane((int)(__dmul_rn(uc, __dmul_rn(qc, S)) < rhs), c) != 0;
        };
        if (!cached) candidates();
        if (!cached && accept(0)) {
            accepted = first;
        } else {
            // First rejection at this context: from here on the residual is needed.  Both rows in flight at once
            // (one memory latency); the target row goes through the LDS region into r, then the draft row is parked
            // there.  The region is private to the wavefront, so none of this needs a barrier.
            {
                float4 pv[8], qv[8];
                fast_fetch_row(P, qrow, qv);
                fast_fetch_row(P, prow, pv);
                __builtin_amdgcn_sched_barrier(0);
                row_to_regs(pv);
                __builtin_amdgcn_sched_barrier(0);
                fast_park_row(region, qv);
            }
            candidates();                     // (after the rows: with them in flight there is no register to spare)
            for (int c = 0;;) {
                // candidate c was rejected: r <- max(r - S q, 0), S <- sum r
                const int xrej = NOREP ? __builtin_amdgcn_readlane(xc, c) : 0;
                const double qrej = NOREP ? read_lane_f64(qc, c) : 0.0;
                if (tid == 0) {
                    sh.hist.s[rounds] = S;
                    if (NOREP) { sh.hist.sq[rounds] = Sq; sh.hist.x[rounds] = xrej; }
                }
                buf ^= 1;
                // two chunks at a time, the next two read from LDS while these are updated
                float4 qv[2][2];
                qv[0][0] = region[fast_slot(lane, 0)];
                qv[0][1] = region[fast_slot(lane, 1)];
#pragma unroll
                for (int j0 = 0; j0 < 8; j0 += 2) {
                    if (j0 + 2 < 8) {
                        qv[(j0 / 2 + 1) & 1][0] = region[fast_slot(lane, j0 + 2)];
                        qv[(j0 / 2 + 1) & 1][1] = region[fast_slot(lane, j0 + 3)];
                    }
#pragma unroll
                    for (int jj = 0; jj < 2; ++jj) {
                        const float4 q4 = qv[(j0 / 2) & 1][jj];
                        const float qe[4] = {q4.x, q4.y, q4.z, q4.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int i = 4 * (j0 + jj) + e;
                            r[i] = pos_part(__fma_rn(-S, (double)qe[e], NOREP ? __dmul_rn(r[i], Sq) : r[i]));
                        }
                    }
                }
                if (NOREP) {
                    // the rejected token leaves the draft row: its owner lane clears its LDS copy, after this round's
                    // update has used it
                    if (tid == (xrej >> 5)) ((float *)&region[fast_slot(lane, (xrej & 31) >> 2)])[xrej & 3] = 0.f;
                }
                {
                    const double d = __fma_rn(-S, qc, NOREP ? __dmul_rn(rc, Sq) : rc);
                    rc = pos_part(d);
                }
                if (NOREP) {
                    Sq = __dsub_rn(Sq, qrej);
                    if (xc == xrej) qc = 0.0;             // also a later duplicate of the rejected token
                }
                rounds += 1;
                S = total(false);
                if (++c == cnt) break;
                if (accept(c)) { accepted = first + c; break; }
            }
        }
        if (accepted < 0) {
            term_p = prow; term_q = qrow;
            if (S > 0.0) { term_rounds = rounds; term_in_regs = true; }
            else { term_rounds = 0; term_in_regs = false; }   // vanished residual: the context's own target row
            break;
        }
        if (tid == 0) sh.path[n_acc] = accepted;
        n_acc += 1;
        cur = accepted;
        level += 1;
    }
    if (term_p == nullptr) {                  // every level accepted: bonus from the row after the last node
        term_p = p + (int64_t)(cur + 1) * P.V;
        term_q = term_p;                      // never read: rounds == 0
        term_rounds = 0;
        term_in_regs = false;
    }
    if (P.n_new > 0) {
        if (!term_in_regs) {                  // the terminal distribution is a target row: bring it into r
            float4 pv[8];
            fast_fetch_row(P, term_p, pv);
            row_to_regs(pv);
        }
        buf ^= 1;
        (void)total(true);                    // wavefront sums and lane-sum heaps of the terminal distribution; one barrier
        for (int k = wave; k < P.n_new; k += NWAVE) {       // wavefronts draw independently from here on
            const int t = fast_sample<NOREP>(sh, P, buf, term_p, term_q, term_rounds, P.us[(int64_t)b * P.n_new + k]);
            if (lane == 0) put(P.cand_new + ((int64_t)b * P.R + root) * P.n_new + k, t);
        }
    }
    if (wave == 0) {                          // (lane 0 wrote the path: no barrier needed)
        if (lane < P.t.gamma) put(path_out + lane, lane < n_acc ? sh.path[lane] : -1);
        if (lane == 0) put(P.cand_len + (int64_t)b * P.R + root, n_acc);
    }
    if (P.mode == MCSD_TARGET_INIT) select_longest(P, b, root, P.R);
}

// ---------------------------------------------------------------------------------------------------
// Teams: several workgroups share one walk, each holding one aligned power-of-two chunk of the vocabulary
// ---------------------------------------------------------------------------------------------------
// All workgroups of a team take the same decisions (they are functions of the same binary64 numbers), so the only thing
// they exchange is the sum of their chunk once per rejection round: an all-gather through a mailbox in device memory.
// Nothing depends on the others arriving: a workgroup that has waited TEAM_POLLS polls for a sum computes it from the
// two rows itself (the same tree, hence the same bits) and does not wait again, so every wait ends whatever else
// occupies the chip.
//
// A message is the sum in four 16-bit pieces, each in a 64-bit word of its own under the same 48-bit tag, so it needs no
// ordering against anything: the tag says which walk, which run and which step the sum is of (see team_protocol.h), and the
// value under a tag is always the same.  Nonces come from a host counter, one per walk.  The exit count grows by one per
// workgroup that leaves and so differs between two replays of one captured launch.  A mailbox that two launches happen to
// use at once only loses messages: the reader finds other tags and computes the sum itself.
constexpr int TEAM_POLLS = 64;
struct TeamMailbox {
    unsigned exits;
    unsigned pad[31];
    unsigned long long box[2][TEAM_MAX][TEAM_MAX][4];     // [step parity][reader][writer][piece]
};
__device__ __align__(128) TeamMailbox g_team[TEAM_MAILBOXES];

struct TeamParams {
    VerifyParams v;
    unsigned long long nonce;            // of walk 0
    int32_t C, log_c;                    // workgroups per team, a power of two
    int32_t log_xcc;                     // dies the workgroup ids are dealt to (a power of two); a team's ids agree modulo their number
    int32_t polls;                       // how often a sum is looked for; < 0: never (every sum computed here)
};

template <int EPL_, int NT>
struct TeamShared {
    float4 region[EPL_ == 16 ? NT * 4 : 1];                 // see team_load
    double wsum[2][NT / 64];             // sums of the wavefronts' parts of the chunk, double-buffered over rounds
    double csum[2][TEAM_MAX];            // sums of the team's chunks
    double lsum[NT];                     // the lanes' sums of the latest round, for sampling
    double S[2];
    History hist;                        // of the current context
    NodeCache node;
    int path[MCSD_MAX_LEVELS];           // accepted nodes so far, written out at the end (a store in flight delays every later load)
    float us[64];                        // sampling uniforms
    double thr[64];                      // sampling: what is left of draw k's threshold inside its lane
    int at[64];                          // ... wavefront * 64 + lane, -1 when another workgroup owns it
};

// Four floats at any 4-byte aligned address.
struct __attribute__((packed, aligned(4))) Float4u { float x, y, z, w; };

// Floats t .. t + 3 of a row (V >= 4).  The load itself is unconditional, from an address inside the row, so that a lane's
// loads are in flight together; the few lanes at the row's end shift or clear afterwards (team_edge).
__device__ inline float4 team_load4(const float *row, int t, int V)
{
    const Float4u f = *(const Float4u *)(row + (t < V - 4 ? t : V - 4));
    return make_float4(f.x, f.y, f.z, f.w);
}
__device__ inline float4 team_edge(float4 v, int t, int V)
{
    const int over = t - (V - 4);                           // > 0: the piece starts `over` floats after what was loaded
    if (over > 0) {
        v.x = over == 1 ? v.y : (over == 2 ? v.z : (over == 3 ? v.w : 0.f));
        v.y = over == 1 ? v.z : (over == 2 ? v.w : 0.f);
        v.z = over == 1 ? v.w : 0.f;
        v.w = 0.f;
    }
    return v;
}

// The lane's N consecutive elements base + lane * N .. of a row, base = the wavefront's first.  N = 8: a lane's 32 bytes
// straight from memory.  N = 16: fetched coalesced (16 bytes per lane, 1 KiB contiguous per instruction; 64 bytes per lane
// would pull every line through the L1 four times) and handed to the owner lanes through the wavefront's LDS region; the XOR
// makes both sides free of bank conflicts.  First the requests ...
template <int N>
__device__ inline void team_request(const float *row, int base, int V, float4 (&f)[N / 4])
{
    int lane = threadIdx.x & 63;
    if constexpr (N == 16) asm volatile("" : "+v"(lane));  // (addresses recomputed here instead of kept, and spilled, all along)
    const int first = base + (N == 8 ? lane * 8 : lane * 4);
#pragma unroll
    for (int j = 0; j < N / 4; ++j) f[j] = team_load4(row, first + j * (N == 8 ? 4 : 256), V);
}
// ... then, when they have arrived, the values.
template <int N>
__device__ inline void team_take(float4 (&f)[N / 4], int base, int V, float (&v)[N], float4 *region)
{
    int lane = threadIdx.x & 63;
    if constexpr (N == 16) asm volatile("" : "+v"(lane));
    const int first = base + (N == 8 ? lane * 8 : lane * 4);
    if (base + 64 * N > V) {                                // (uniform) the wavefront reaches beyond the row
#pragma unroll
        for (int j = 0; j < N / 4; ++j) f[j] = team_edge(f[j], first + j * (N == 8 ? 4 : 256), V);
    }
    if constexpr (N == 16) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int l = j * 16 + (lane >> 2);             // owner of 16-byte unit 64 j + lane
            region[4 * l + ((lane & 3) ^ ((l >> 2) & 3))] = f[j];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) f[j] = region[4 * lane + (j ^ ((lane >> 2) & 3))];
    }
#pragma unroll
    for (int j = 0; j < N / 4; ++j) { v[4 * j] = f[j].x; v[4 * j + 1] = f[j].y; v[4 * j + 2] = f[j].z; v[4 * j + 3] = f[j].w; }
}

// Which of 2^K values the threshold falls into; thr becomes what is left of it.  Value i sits in lane i, or with QUAD in all
// lanes of quad i.  lvl[j] holds in every lane the sum over its aligned group of 2^j values.
template <int K, bool QUAD = false>
__device__ inline int lane_descend(double v, double &thr)
{
    constexpr int S = QUAD ? 2 : 0;                         // lanes per value, as a power of two
    double lvl[K];
    lvl[0] = v;
#pragma unroll
    for (int j = 1; j < K; ++j) {
        const double x = lvl[j - 1];
        const int d = j - 1 + S;                            // partner: lane ^ 2^d (see wave_tree_sum)
        double o;
        if (d == 0) o = dpp_f64<0xB1>(x);
        else if (d == 1) o = dpp_f64<0x4E>(x);
        else if (d == 2) o = dpp_f64<0x141>(x);
        else if (d == 3) o = dpp_f64<0x140>(x);
        else o = __hiloint2double(__builtin_amdgcn_ds_swizzle(__double2hiint(x), 0x401F), __builtin_amdgcn_ds_swizzle(__double2loint(x), 0x401F));
        lvl[j] = __dadd_rn(x, o);
    }
    static_assert(K - 2 + S <= 4, "lane ^ 32 has no case above");
    int lo = 0;
#pragma unroll
    for (int j = K; j >= 1; --j) {                         // the node covers values lo .. lo + 2^j - 1
        const double left = read_lane_f64(lvl[j - 1], lo << S);
        const bool right = __builtin_amdgcn_readfirstlane((int)!(thr < left)) != 0;
        if (right) {
            thr = __dsub_rn(thr, left);
            lo += 1 << (j - 1);
        }
    }
    return lo;
}

// In-lane: which of the lane's N elements the threshold falls into.  Halves are selected, never indexed: registers
// cannot be indexed at run time.
template <int N>
__device__ inline int reg_descend(const double (&r)[N], double thr, double &val)
{
    double x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = r[i];
    int at = 0;
#pragma unroll
    for (int h = N / 2; h >= 1; h >>= 1) {
        double s[N / 2];                                    // the tree over the first half of what is left
#pragma unroll
        for (int i = 0; i < h; ++i) s[i] = x[i];
#pragma unroll
        for (int w = h / 2; w >= 1; w >>= 1)
#pragma unroll
            for (int i = 0; i < w; ++i) s[i] = __dadd_rn(s[2 * i], s[2 * i + 1]);
        const bool right = !(thr < s[0]);
        if (right) thr = __dsub_rn(thr, s[0]);
        at += right ? h : 0;
#pragma unroll
        for (int i = 0; i < h; ++i) x[i] = right ? x[h + i] : x[i];
    }
    val = x[0];
    return at;
}

// The sum of elements base .. base + chunk - 1 of the distribution (prow, qrow, rounds), computed by one wavefront from
// memory: what a workgroup does for a sum that did not arrive.
template <bool NOREP>
__device__ inline double chunk_sum_alone(const History &h, int V, const float *prow, const float *qrow, int rounds,
                                                            int base, int chunk)
{
    const int lane = threadIdx.x & 63;
    double blocks = 0.0;                                    // lane i: sum of the chunk's i-th block of 256 elements
#pragma unroll 1
    for (int k = 0; k < chunk / 256; ++k) {
        double e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int t = base + k * 256 + lane * 4 + i;
            e[i] = t < V ? residual_at<NOREP>(h, prow, qrow, rounds, t) : 0.0;
        }
        const double s = wave_tree_sum(__dadd_rn(__dadd_rn(e[0], e[1]), __dadd_rn(e[2], e[3])));
        if (lane == k) blocks = s;
    }
    return wave_tree_sum(blocks);
}

// NT lanes with EPL_ consecutive elements each: a chunk of EPL_ * NT elements, residual (binary64) and draft values in
// registers.  One launch serves any number of teams; with more workgroups than the chip holds the hardware starts them
// in id order, a team's ids lie close together, and a workgroup whose partners are late falls back to its own sums.
template <bool NOREP, int EPL_, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void verify_walk_team_kernel(const TeamParams T)
{
    constexpr int NWV = NT / 64, CHUNK = EPL_ * NT;
    __shared__ TeamShared<EPL_, NT> sh;
    const VerifyParams &P = T.v;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroup ids are dealt round-robin to the dies: ids of a team agree modulo their number, so the mailbox stays in
    // one die's L2
    const int group = blockIdx.x >> (T.log_xcc + T.log_c), die = blockIdx.x & ((1 << T.log_xcc) - 1);
    const int walk = (group << T.log_xcc) + die, member = (blockIdx.x >> T.log_xcc) & (T.C - 1);
    if (walk >= P.B * P.R) return;
    const int b = P.R == 1 ? walk : walk / P.R, root = walk - b * P.R;
    const int t_wave = member * CHUNK + wave * 64 * EPL_, t_lane = t_wave + lane * EPL_;   // first element of the wavefront, of the lane
    float4 *region = EPL_ == 16 ? sh.region + wave * 256 : nullptr;
    const int32_t *tokens = P.tokens + (int64_t)b * P.n_nodes;
    const float *p = P.p + (int64_t)b * P.pbs;
    const float *q = P.q + (int64_t)b * P.qbs;
    const float *ua = P.ua + (int64_t)b * P.n_nodes;
    int32_t *path_out = P.cand_path + (int64_t)walk * P.t.gamma;
    TeamMailbox &mail = g_team[(T.nonce + walk) % TEAM_MAILBOXES];

    // Requested together at the start: the mailbox's exit count, the rows of the first context (small chunks only: a
    // large one would delay what follows) and token, uniform, q(x) and p(x) of every candidate of the tree, two dependent
    // trips to memory for the whole walk.
    const bool target = P.mode == MCSD_TARGET_INIT;
    const bool cached = P.n_nodes <= NODE_CACHE;
    unsigned epoch = 0;
    if (wave == 0) epoch = __hip_atomic_load(&mail.exits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    constexpr bool AHEAD = CHUNK <= 4096;
    double r[EPL_];                           // this lane's elements of the current residual, at first the target row
    float qv[EPL_];                           // ... and of the draft row of that context
    int cur = target ? root : -1;             // context: node id (-1 = end of the prefix)
    int rows_of = -2;                         // context whose rows r and qv hold, untouched
    float4 pf[EPL_ / 4], qf[EPL_ / 4];
    auto take_rows = [&](bool both) {
        float pv[EPL_];
        team_take<EPL_>(pf, t_wave, P.V, pv, region);
        if (both) team_take<EPL_>(qf, t_wave, P.V, qv, region);
#pragma unroll
        for (int i = 0; i < EPL_; ++i) r[i] = (double)pv[i];
    };
    const NodeRegs mine = node_request(P, tokens, ua, tid);
    const bool ahead = AHEAD && P.t.gamma > (target ? 1 : 0);
    if (ahead) {
        team_request<EPL_>(p + (int64_t)(cur + 1) * P.V, t_wave, P.V, pf);
        team_request<EPL_>(q + (int64_t)(cur + 1) * P.V, t_wave, P.V, qf);
    }
    node_fetch(sh.node, P, p, q, mine, tid);
    static_assert(NODE_CACHE <= NT, "one lane per cached node");
    if (tid < P.n_new) sh.us[tid] = P.us[(int64_t)b * P.n_new + tid];
    if (ahead) {
        take_rows(true);
        rows_of = cur;
    }
    int level = 0, n_acc = 0;
    if (target) {                             // level-1 node `root` is accepted untested
        level = 1;
        n_acc = 1;
        if (tid == 0) sh.path[0] = root;
    }
    double S_term = 0.0;                      // sum of the terminal distribution
    int buf = 0;
    unsigned step = 0;
    bool alone = false;                       // this workgroup has waited in vain once
    const float *term_p = nullptr, *term_q = nullptr;
    int term_rounds = 0;
    bool term_in_regs = false;

    // The sum of r over the vocabulary, after `rounds` rejections at the context with rows prow / qrow.
    auto total = [&](const float *prow, const float *qrow, int rounds) -> double {
        double v[EPL_];
#pragma unroll
        for (int i = 0; i < EPL_; ++i) v[i] = r[i];
#pragma unroll
        for (int w = EPL_ / 2; w >= 1; w >>= 1)
#pragma unroll
            for (int i = 0; i < w; ++i) v[i] = __dadd_rn(v[2 * i], v[2 * i + 1]);
        sh.lsum[tid] = v[0];
        const double ws = wave_tree_sum(v[0]);
        buf ^= 1;
        if (lane == 0) sh.wsum[buf][wave] = ws;
        __syncthreads();
        double c = 0.0;
        if (T.C == 1 || wave == 0) {
            c = sh.wsum[buf][lane & (NWV - 1)];
            c = __dadd_rn(c, dpp_f64<0xB1>(c));
            c = __dadd_rn(c, dpp_f64<0x4E>(c));
            c = __dadd_rn(c, dpp_f64<0x141>(c));
            if constexpr (NWV >= 16) c = __dadd_rn(c, dpp_f64<0x140>(c));
        }
        if (T.C == 1) return read_lane_f64(c, 0);     // (uniform by construction, and the compiler has to know: the walk is scalar)
        if (wave == 0) {
            // lane 4 m + k: piece k of the message to, then from member m
            const int m = lane >> 2, k = lane & 3;
            const unsigned long long tag = team_tag(epoch, T.nonce + walk, step);
            unsigned long long(*box)[TEAM_MAX][4] = mail.box[team_box(step)];
            const unsigned half = (unsigned)(k & 2 ? __double2hiint(c) : __double2loint(c)), piece = k & 1 ? half >> 16 : half & 0xffffu;
            unsigned long long w = tag | piece;
            if (m < T.C) __hip_atomic_store(&box[m][member][k], w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const bool other = m < T.C && m != member;
            unsigned long long missing;
            for (int polls = __builtin_amdgcn_readfirstlane(alone ? 0 : T.polls);; --polls) {
                if (other) w = T.polls >= 0 ? __hip_atomic_load(&box[member][m][k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : ~tag;
                missing = __builtin_amdgcn_ballot_w64(other && !team_carries(w, tag));
                if (missing == 0 || __builtin_amdgcn_readfirstlane(polls) <= 0) break;
            }
            step += 1;
            unsigned half_lo = (unsigned)w & 0xffffu;
            const int w0 = __builtin_amdgcn_update_dpp(0, (int)half_lo, 0x00, 0xF, 0xF, false), w1 = __builtin_amdgcn_update_dpp(0, (int)half_lo, 0x55, 0xF, 0xF, false);
            const int w2 = __builtin_amdgcn_update_dpp(0, (int)half_lo, 0xAA, 0xF, 0xF, false), w3 = __builtin_amdgcn_update_dpp(0, (int)half_lo, 0xFF, 0xF, 0xF, false);
            double s = m < T.C ? __hiloint2double(w2 | w3 << 16, w0 | w1 << 16) : 0.0;
            while (missing) {
                alone = true;
                const int mm = __builtin_ctzll(missing) >> 2;
                missing &= ~(0xfull << (4 * mm));
                const double a = chunk_sum_alone<NOREP>(sh.hist, P.V, prow, qrow, rounds, mm * CHUNK, CHUNK);
                if (m == mm) s = a;
            }
            if (k == 0) sh.csum[buf][m] = s;
            s = __dadd_rn(s, dpp_f64<0x141>(s));        // the tree over the 16 quads
            s = __dadd_rn(s, dpp_f64<0x140>(s));
            {
                const int lo = __builtin_amdgcn_ds_swizzle(__double2loint(s), 0x401F), hi = __builtin_amdgcn_ds_swizzle(__double2hiint(s), 0x401F);
                s = __dadd_rn(s, __hiloint2double(hi, lo));
            }
            {
                const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(s), (unsigned)__double2loint(s), false, false);
                const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(s), (unsigned)__double2hiint(s), false, false);
                s = __dadd_rn(__hiloint2double((int)hi[0], (int)lo[0]), __hiloint2double((int)hi[1], (int)lo[1]));
            }
            if (lane == 0) sh.S[buf] = s;
        }
        __syncthreads();
        return read_lane_f64(sh.S[buf], 0);
    };

    __syncthreads();                          // the cached candidates are visible
    // The walk is the same in all lanes and has to be scalar control flow (tree description from scalar loads, no
    // execution masks); the compiler loses sight of that where a lane-dependent branch joins, hence the readfirstlanes.
    while (true) {
        level = __builtin_amdgcn_readfirstlane(level);
        cur = __builtin_amdgcn_readfirstlane(cur);
        n_acc = __builtin_amdgcn_readfirstlane(n_acc);
        unsigned kid = 0;
        if (cached) {                         // contexts whose first candidate passes need nothing but that fact
            while (level < P.t.gamma) {
                kid = __builtin_amdgcn_readfirstlane(sh.node.kid[cur + 1]);
                if (!(kid >> 31)) break;
                cur = (int)(kid & 0x7fffffffu);
                if (tid == 0) sh.path[n_acc] = cur;
                n_acc += 1;
                level += 1;
            }
        }
        if (level >= P.t.gamma) break;
        const float *prow = p + (int64_t)(cur + 1) * P.V;
        const float *qrow = q + (int64_t)(cur + 1) * P.V;
        const int cnt = P.t.b[level];
        const int first = cached ? (int)kid : (cur < 0 ? 0 : P.t.off[level] + (cur - P.t.off[level - 1]) * cnt);
        // candidate `lane` of this context (in every wavefront): acceptance uniform, q(x) and the residual at x,
        // which is updated in place after every rejection
        double uc = 0.0, qc = 0.0, rc = 0.0;
        int xc = -1;
        if (lane < cnt) {
            const int i = first + lane;
            if (cached) {
                xc = sh.node.x[i];
                uc = (double)sh.node.u[i];
                qc = (double)sh.node.q[i];
                rc = (double)sh.node.p[i];
            } else {
                int x = tokens[i];
                x = x < 0 ? 0 : (x >= P.V ? P.V - 1 : x);
                float u = ua[i], qx = qrow[x], px = prow[x];
                asm volatile("" : "+v"(u), "+v"(qx), "+v"(px));      // (keeps the compiler from merging these loads with those above)
                xc = x;
                uc = (double)u;
                qc = (double)qx;
                rc = (double)px;
            }
        }
        int rounds = 0, accepted = -1;
        double S = 1.0, Sq = 1.0;                        // both rows are trusted to be normalised in round 0
        // accept test of candidate c, evaluated by its lane; the same answer in every wavefront
        auto accept = [&](int c) {
            const double rhs = NOREP ? __dmul_rn(rc, Sq) : rc;
            return __builtin_amdgcn_readlane((int)(__dmul_rn(uc, __dmul_rn(qc, S)) < rhs), c) != 0;
        };
        if (!cached && accept(0)) {
            accepted = first;
        } else {
            if (!AHEAD || __builtin_amdgcn_readfirstlane(rows_of) != cur) {
                team_request<EPL_>(prow, t_wave, P.V, pf);
                team_request<EPL_>(qrow, t_wave, P.V, qf);
                take_rows(true);
            }
            rows_of = -2;
            for (int c = 0;;) {
                // candidate c was rejected: r <- max(r - S q, 0), S <- sum r
                const int xrej = NOREP ? __builtin_amdgcn_readlane(xc, c) : 0;
                const double qrej = NOREP ? read_lane_f64(qc, c) : 0.0;
                if (tid == 0) {
                    sh.hist.s[rounds] = S;
                    if (NOREP) { sh.hist.sq[rounds] = Sq; sh.hist.x[rounds] = xrej; }
                }
                if constexpr (EPL_ == 16) {   // (the conversions below stay in the loop: 32 registers fewer)
#pragma unroll
                    for (int i = 0; i < EPL_; ++i) asm volatile("" : "+v"(qv[i]));
                }
#pragma unroll
                for (int i = 0; i < EPL_; ++i)
                    r[i] = pos_part(__fma_rn(-S, (double)qv[i], NOREP ? __dmul_rn(r[i], Sq) : r[i]));
                if (NOREP) {                  // the rejected token leaves the draft row after this round's update has used it
#pragma unroll
                    for (int i = 0; i < EPL_; ++i)
                        if (xrej - t_lane == i) qv[i] = 0.f;
                }
                {
                    const double d = __fma_rn(-S, qc, NOREP ? __dmul_rn(rc, Sq) : rc);
                    rc = pos_part(d);
                }
                if (NOREP) {
                    Sq = __dsub_rn(Sq, qrej);
                    if (xc == xrej) qc = 0.0;             // also a later duplicate of the rejected token
                }
                rounds += 1;
                S = total(prow, qrow, rounds);
                if (++c == cnt) break;
                if (accept(c)) { accepted = first + c; break; }
            }
        }
        if (accepted < 0) {
            term_p = prow; term_q = qrow;
            if (S > 0.0) { term_rounds = rounds; term_in_regs = true; S_term = S; }
            else { term_rounds = 0; term_in_regs = false; }   // vanished residual: the context's own target row
            break;
        }
        if (tid == 0) sh.path[n_acc] = accepted;
        cur = accepted;
        n_acc += 1;
        level += 1;
    }
    if (term_p == nullptr) {                  // every level accepted: bonus from the row after the last node
        term_p = p + (int64_t)(cur + 1) * P.V;
        term_q = term_p;                      // never read: rounds == 0
    }
    if (P.n_new > 0) {
        if (!term_in_regs) {                  // the terminal distribution is a target row: bring it into r
            team_request<EPL_>(term_p, t_wave, P.V, pf);
            take_rows(false);
            S_term = total(term_p, term_q, 0);
        }
        // Wavefront k places draws k, k + NWV, ..: chunk, wavefront and lane; a draw in another chunk is its owner's
        // (a single draw is placed by every wavefront for itself, which saves the hand-over)
        const bool single = P.n_new == 1;
        int at1 = -1;
        double thr1 = 0.0;
        for (int k = single ? 0 : wave; k < P.n_new; k += NWV) {
            double thr = __dmul_rn((double)sh.us[k], S_term);
            int at = -1;
            if (T.C == 1 || lane_descend<4, true>(sh.csum[buf][lane >> 2], thr) == member) {
                constexpr int KW = NWV == 8 ? 3 : 4;
                const int w = lane_descend<KW>(sh.wsum[buf][lane & (NWV - 1)], thr);
                const int l = lane_descend<6>(sh.lsum[w * 64 + lane], thr);
                at = w * 64 + l;
            }
            at1 = at;
            thr1 = thr;
            if (!single && lane == 0) { sh.at[k] = at; sh.thr[k] = thr; }
        }
        if (!single) __syncthreads();
        for (int k = 0; k < P.n_new; ++k) {
            const int at = single ? at1 : __builtin_amdgcn_readfirstlane(sh.at[k]);
            if (at < 0 || (at >> 6) != wave) continue;
            double val;
            int t = t_lane + reg_descend<EPL_>(r, single ? thr1 : sh.thr[k], val);      // every lane for itself; lane `at` is meant
            t = __builtin_amdgcn_readlane(t, at & 63);
            if (!(t < P.V && read_lane_f64(val, at & 63) > 0.0)) {
                // Reached a zero-weight index (last-bit rounding of the subtraction, or an all-zero distribution):
                // nearest positive-weight index below, else nearest above, else 0.
                int below = -1, above = 0x7fffffff;
                for (int e = lane; e < P.V; e += 64) {
                    if (e == t) continue;
                    if (residual_at<NOREP>(sh.hist, term_p, term_q, term_rounds, e) > 0.0) {
                        if (e < t) below = e > below ? e : below;
                        else above = e < above ? e : above;
                    }
                }
#pragma unroll
                for (int m = 1; m < 64; m <<= 1) {
                    const int ob = __shfl_xor(below, m, 64), oa = __shfl_xor(above, m, 64);
                    below = ob > below ? ob : below;
                    above = oa < above ? oa : above;
                }
                t = below >= 0 ? below : (above != 0x7fffffff ? above : 0);
            }
            if (lane == 0) put(P.cand_new + (int64_t)walk * P.n_new + k, t);
        }
    }
    if (member == 0 && wave == 0) {           // (lane 0 wrote the path: no barrier needed)
        if (lane < P.t.gamma) put(path_out + lane, lane < n_acc ? sh.path[lane] : -1);
        if (lane == 0) put(P.cand_len + walk, n_acc);
    }
    if (target) select_longest(P, b, root * T.C + member, P.R * T.C);
    if (T.C > 1 && tid == 0) (void)__hip_atomic_fetch_add(&mail.exits, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

extern "C" size_t mcsd_verify_tree_workspace(const mcsd_mask_view_t *mask, mcsd_mode_t mode, int32_t B, int32_t n_new)
{
    if (!mask || mode != MCSD_TARGET_INIT || B < 1 || n_new < 0 || mask->gamma < 1) return 0;
    const size_t R = (size_t)mask->branching_host[0];
    return align256(sizeof(int32_t) * B * R * mask->gamma) + align256(sizeof(int32_t) * B * R) +
           align256(sizeof(int32_t) * B * R * (n_new > 0 ? n_new : 1)) + align256(sizeof(unsigned long long) * B * R * TEAM_MAX);
}

namespace {
// One number per walk ever launched: the nonces of the teams' messages and, with a part of its own for every process, the id
// of a launch.
std::atomic<unsigned long long> g_team_nonce{0};
const unsigned long long g_process_part = (unsigned long long)std::chrono::system_clock::now().time_since_epoch().count() << 40;

// Chunk of the vocabulary a team's workgroup holds; 0: one workgroup of the fast kernel per walk.  Up to 16384 entries one
// workgroup does it all (an exchange costs about as much as it saves there).  Beyond, the smallest chunk that leaves every
// workgroup a compute unit of its own, at least 4096 entries, at most 16 workgroups per team.  Vocabularies up to 32768 go
// to the fast kernel when even two workgroups per walk would not fit (200 walks: 25 us against 30).
int team_chunk(int V, long walks, int team)
{
    if (V < 4) return 0;                                    // (rows shorter than one load)
    int space = 4096;
    while (space < V) space <<= 1;
    int chunk = space / TEAM_MAX < 4096 ? 4096 : space / TEAM_MAX;
    if (team > 0) {
        while (chunk < 16384 && space / chunk > team) chunk <<= 1;
        return chunk;
    }
    if (space <= 16384) return space;
    while (chunk < 16384 && walks * (space / chunk) > 256) chunk <<= 1;
    return space == FAST_V && walks * (space / chunk) > 256 ? 0 : chunk;
}

void launch_walk(VerifyParams &P, bool norep, const mcsd_verify_tuning_t *tune, int device, hipStream_t st)
{
    const long walks = (long)P.B * P.R;
    const unsigned long long nonce = g_team_nonce.fetch_add((unsigned long long)walks, std::memory_order_relaxed);
    P.launch_id = g_process_part | (nonce & 0xffffffffffull);
    if (P.launch_id == 0) P.launch_id = 1;
    const int chunk = team_chunk(P.V, walks, tune ? tune->team : 0);
    if (chunk == 0) {
        mcsd_launch(MCSD_KERNEL_VERIFY_WALK, norep ? verify_walk_fast_kernel<true> : verify_walk_fast_kernel<false>, dim3(P.R, P.B), dim3(VT), st, P);
        return;
    }
    TeamParams T;
    T.v = P;
    T.C = 1;
    while (T.C * chunk < P.V) T.C <<= 1;
    T.nonce = nonce;
    T.polls = tune && tune->polls != 0 ? tune->polls : TEAM_POLLS;
    const int xcc = T.C > 1 ? mcsd_xcc_count(device) : 1;
    T.log_c = __builtin_ctz(T.C);
    T.log_xcc = xcc > 1 ? __builtin_ctz(xcc) : 0;
    const long dies = 1l << T.log_xcc, groups = (walks - 1) / dies;             // whole groups of `dies` teams before the last
    const dim3 grid((unsigned)(groups * dies * T.C + (T.C - 1) * dies + (walks - 1) % dies + 1));
    if (chunk == 4096) mcsd_launch(MCSD_KERNEL_VERIFY_WALK, norep ? verify_walk_team_kernel<true, 8, 512> : verify_walk_team_kernel<false, 8, 512>, grid, dim3(512), st, T);
    else if (chunk == 8192) mcsd_launch(MCSD_KERNEL_VERIFY_WALK, norep ? verify_walk_team_kernel<true, 8, 1024> : verify_walk_team_kernel<false, 8, 1024>, grid, dim3(1024), st, T);
    else mcsd_launch(MCSD_KERNEL_VERIFY_WALK, norep ? verify_walk_team_kernel<true, 16, 1024> : verify_walk_team_kernel<false, 16, 1024>, grid, dim3(1024), st, T);
}
}  // namespace

extern "C" int mcsd_verify_tree(const mcsd_mask_view_t *mask, mcsd_mode_t mode, int32_t B, int32_t V,
                                const int32_t *tokens, const float *p_target, const float *q_draft,
                                int64_t p_batch_stride, int64_t q_batch_stride, const float *u_accept,
                                const float *u_sample, int32_t n_new, int32_t *out_path, int32_t *out_accept_len,
                                int32_t *out_new_tokens, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return mcsd_verify_tree_sampling(mask, mode, MCSD_WITH_REPLACEMENT, B, V, tokens, p_target, q_draft, p_batch_stride,
                                     q_batch_stride, u_accept, u_sample, n_new, out_path, out_accept_len,
                                     out_new_tokens, workspace, workspace_bytes, hip_stream);
}

extern "C" int mcsd_verify_tree_sampling(const mcsd_mask_view_t *mask, mcsd_mode_t mode, mcsd_sampling_t sampling,
                                         int32_t B, int32_t V, const int32_t *tokens, const float *p_target,
                                         const float *q_draft, int64_t p_batch_stride, int64_t q_batch_stride,
                                         const float *u_accept, const float *u_sample, int32_t n_new,
                                         int32_t *out_path, int32_t *out_accept_len, int32_t *out_new_tokens,
                                         void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return mcsd_verify_tree_tuned(nullptr, mask, mode, sampling, B, V, tokens, p_target, q_draft, p_batch_stride, q_batch_stride,
                                  u_accept, u_sample, n_new, out_path, out_accept_len, out_new_tokens, workspace,
                                  workspace_bytes, hip_stream);
}

extern "C" int mcsd_verify_tree_tuned(const mcsd_verify_tuning_t *tuning, const mcsd_mask_view_t *mask, mcsd_mode_t mode,
                                      mcsd_sampling_t sampling, int32_t B, int32_t V, const int32_t *tokens,
                                      const float *p_target, const float *q_draft, int64_t p_batch_stride,
                                      int64_t q_batch_stride, const float *u_accept, const float *u_sample,
                                      int32_t n_new, int32_t *out_path, int32_t *out_accept_len,
                                      int32_t *out_new_tokens, void *workspace, size_t workspace_bytes,
                                      void *hip_stream)
{
    if (tuning && (tuning->team < 0 || tuning->team > TEAM_MAX || tuning->polls < -1 || tuning->polls > 1 << 16)) return MCSD_EINVAL;
    if (sampling != MCSD_WITH_REPLACEMENT && sampling != MCSD_WITHOUT_REPLACEMENT) return MCSD_EINVAL;
    const bool norep = sampling == MCSD_WITHOUT_REPLACEMENT;
    if (!mask || !tokens || !p_target || !u_accept || !out_path || !out_accept_len) return MCSD_EINVAL;
    if (mode != MCSD_DRAFT_INIT && mode != MCSD_TARGET_INIT) return MCSD_EINVAL;
    if (B < 1 || B > 65535 || V < 1 || n_new < 0 || n_new > 64) return MCSD_EINVAL;
    if (n_new > 0 && (!u_sample || !out_new_tokens)) return MCSD_EINVAL;
    if (mask->gamma < 1 || mask->gamma > MCSD_MAX_LEVELS) return MCSD_EINVAL;
    // draft rows are needed whenever some context has children to test
    const bool has_tests = mode == MCSD_DRAFT_INIT ? true : mask->gamma > 1;
    if (has_tests && !q_draft) return MCSD_EINVAL;
    if (V > MCSD_MAX_VOCAB) return MCSD_EUNSUPPORTED;
    if (p_batch_stride < (int64_t)(1 + mask->n_nodes) * V) return MCSD_EINVAL;
    if (has_tests && q_batch_stride < (int64_t)(1 + mask->level_off_host[mask->gamma - 1]) * V) return MCSD_EINVAL;

    VerifyParams P;
    P.t.gamma = mask->gamma;
    for (int l = 0; l < mask->gamma; ++l) P.t.b[l] = mask->branching_host[l];
    for (int l = 0; l <= mask->gamma; ++l) P.t.off[l] = mask->level_off_host[l];
    P.mode = mode; P.B = B; P.V = V; P.n_nodes = mask->n_nodes; P.n_new = n_new;
    P.R = mode == MCSD_TARGET_INIT ? mask->branching_host[0] : 1;
    P.tokens = tokens; P.p = p_target; P.q = q_draft ? q_draft : p_target;
    P.pbs = p_batch_stride; P.qbs = q_batch_stride;
    P.ua = u_accept; P.us = u_sample;
    P.parent = mask->parent_dev;
    hipStream_t st = (hipStream_t)hip_stream;
    P.out_path = P.out_len = P.out_new = nullptr;
    P.done = nullptr;
    if (mode == MCSD_DRAFT_INIT) {
        if (!mask->parent_dev) return MCSD_EINVAL;          // a mask built without a device
        P.cand_path = out_path; P.cand_len = out_accept_len; P.cand_new = out_new_tokens;
        launch_walk(P, norep, tuning, mask->device, st);
        return mcsd_hip_status(hipGetLastError());
    }
    const size_t need = mcsd_verify_tree_workspace(mask, mode, B, n_new);
    if (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 255)) return MCSD_EWORKSPACE;
    if (!mask->parent_dev) return MCSD_EINVAL;
    const size_t R = (size_t)P.R;
    char *w = (char *)workspace;
    P.cand_path = (int32_t *)w;
    w += align256(sizeof(int32_t) * B * R * mask->gamma);
    P.cand_len = (int32_t *)w;
    w += align256(sizeof(int32_t) * B * R);
    P.cand_new = (int32_t *)w;
    w += align256(sizeof(int32_t) * B * R * (n_new > 0 ? n_new : 1));
    P.done = (unsigned long long *)w;
    P.out_path = out_path; P.out_len = out_accept_len; P.out_new = out_new_tokens;
    launch_walk(P, norep, tuning, mask->device, st);
    return mcsd_hip_status(hipGetLastError());
}
