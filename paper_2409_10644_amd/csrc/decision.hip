// Early-stop decision models (Sec. 3.3): after a draft-generation turn a small MLP predicts, per candidate
// sequence, the probability that the target model accepts it; the tree stops growing when every sequence is
// predicted below the threshold (caption of Fig. 2).
//
//   decision_distribution_kernel  type 2: Concat(Topk(y), Ent(y)) of one draft distribution y per workgroup (the
//                                 row is read once into registers, or streamed when it is too long), then
//                                 the MLP
//   decision_hidden_kernel        type 1: the MLP on the draft model's hidden states, four rows per workgroup
//   early_stop_kernel             stop[b] = every sequence of tree b below the threshold
//
// Type 2 is bound by reading each 128 kB vocabulary row once; type 1 by streaming the layers' weights through
// a compute unit.  Topk values are selected, not computed, so they are exact; the entropy uses the hardware fp32
// logarithm with binary64 sums, the networks fp32 multiply-adds with tree-combined partial sums: the probabilities
// stay within ~1e-6 of a binary64 evaluation.
#include "mcsd_internal.h"

namespace {

constexpr int DT = 512;              // lanes per workgroup
constexpr int NW = DT / 64;          // wavefronts per workgroup
typedef float nt_f32x4_t __attribute__((ext_vector_type(4)));
constexpr int REG_F4 = 16;           // float4 a lane holds when the whole row fits in registers (V <= 32768)
constexpr int CAND_REG = 1024;       // candidates for the top-k kept in LDS: row in registers ...
constexpr int CAND_MEM = 8192;       // ... row streamed (any V up to MCSD_MAX_VOCAB)
constexpr int K = MCSD_DECISION_MAX_K;

struct MlpDesc {
    int32_t n_layers;
    int32_t width[4];
    const float *w[3];
    const float *b[3];
};

// A value from another lane through the data-parallel-primitive path of the vector ALU (no LDS round trip).
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// Sum over the 64 lanes, result in every lane.  Partner lanes: l^1 and l^2 by quad permutation; the mirrored lane of
// the half row (row) stands in for l^4 (l^8) because groups of 4 (8) already agree; l^16 by swizzle; l^32 by the
// half-wave swap, which returns {own, partner} in an order a commutative operation ignores.
__device__ __forceinline__ double wave_sum(double v)
{
    v += dpp_f64<0xB1>(v);
    v += dpp_f64<0x4E>(v);
    v += dpp_f64<0x141>(v);
    v += dpp_f64<0x140>(v);
    {
        const int lo = __builtin_amdgcn_ds_swizzle(__double2loint(v), 0x401F);
        const int hi = __builtin_amdgcn_ds_swizzle(__double2hiint(v), 0x401F);
        v += __hiloint2double(hi, lo);
    }
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(v), (unsigned)__double2loint(v), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(v), (unsigned)__double2hiint(v), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}

// The same for N independent fp32 values at once, level by level, so the N chains overlap.
template <int N>
__device__ __forceinline__ void wave_sum_f32_n(float (&v)[N])
{
    float t[N];
#pragma unroll
    for (int i = 0; i < N; ++i) t[i] = dpp_f32<0xB1>(v[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += t[i];
#pragma unroll
    for (int i = 0; i < N; ++i) t[i] = dpp_f32<0x4E>(v[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += t[i];
#pragma unroll
    for (int i = 0; i < N; ++i) t[i] = dpp_f32<0x141>(v[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += t[i];
#pragma unroll
    for (int i = 0; i < N; ++i) t[i] = dpp_f32<0x140>(v[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += t[i];
#pragma unroll
    for (int i = 0; i < N; ++i) t[i] = __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v[i]), 0x401F));
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] += t[i];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const auto s = __builtin_amdgcn_permlane32_swap((unsigned)__float_as_int(v[i]), (unsigned)__float_as_int(v[i]), false, false);
        v[i] = __int_as_float((int)s[0]) + __int_as_float((int)s[1]);
    }
}

// Order-preserving map of a float to an unsigned key (larger value = larger key); 0 is below the key of every
// number, -inf included, and marks an absent value.
__device__ __forceinline__ unsigned order_key(float v)
{
    const unsigned b = __float_as_uint(v);
    return (b >> 31) ? ~b : b | 0x80000000u;
}
__device__ __forceinline__ float key_value(unsigned key)
{
    return __uint_as_float((key >> 31) ? key & 0x7fffffffu : ~key);
}

// Key of the k-th largest of the wave's two values per lane (0 if there are fewer than k): the key is built from
// the top bit down, keeping a bit whenever at least k keys are still at or above the candidate.  32 steps of two
// compares and two population counts, no data moves between lanes.
__device__ __forceinline__ unsigned wave_kth_key(unsigned ka, unsigned kb, int k)
{
    unsigned t = 0;
#pragma unroll 4
    for (int bit = 31; bit >= 0; --bit) {
        const unsigned c = t | (1u << bit);
        const int n = __popcll(__ballot(ka >= c)) + __popcll(__ballot(kb >= c));
        if (n >= k) t = c;
    }
    return t;
}

// One layer for R rows at once: out[r][j] = act(b[j] + sum_i W[j][i] * in(r, i)), fp32 multiply-adds.
// Narrow layers (<= 64 inputs, >= 64 outputs): a lane per output unit.  Otherwise a wavefront takes four output
// units per step, lanes over the inputs (coalesced weight reads), and the per-lane partial sums are combined as a
// balanced tree.  Weight loads are issued in batches ahead of their use.  Ends with a barrier.
template <int R, typename In, int PITCH>
__device__ __forceinline__ void mlp_layer(In in, int n_in, const float *W, const float *b, int n_out,
                                          float (*out)[PITCH], bool relu, int tid)
{
    const int lane = tid & 63, wave = tid >> 6;
    if (n_in <= 64 && n_out >= 64) {
        for (int j = tid; j < n_out; j += DT) {
            float s[R];
            const float bj = b[j];
#pragma unroll
            for (int r = 0; r < R; ++r) s[r] = bj;
            const float *wr = W + (size_t)j * n_in;
            for (int i0 = 0; i0 < n_in; i0 += 16) {
                float w[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) w[u] = wr[min(i0 + u, n_in - 1)];
#pragma unroll
                for (int u = 0; u < 16; ++u)
                    if (i0 + u < n_in) {
#pragma unroll
                        for (int r = 0; r < R; ++r) s[r] = fmaf(w[u], in(r, i0 + u), s[r]);
                    }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) out[r][j] = (relu && s[r] < 0.0f) ? 0.0f : s[r];
        }
    } else {
        constexpr int JB = 4;
        for (int j0 = wave * JB; j0 < n_out; j0 += NW * JB) {
            float s[JB * R];
#pragma unroll
            for (int q = 0; q < JB * R; ++q) s[q] = 0.0f;
            for (int i0 = lane; i0 < n_in; i0 += 128) {
                float w[2][JB];
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int jj = 0; jj < JB; ++jj)
                        w[u][jj] = W[(size_t)min(j0 + jj, n_out - 1) * n_in + min(i0 + 64 * u, n_in - 1)];
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    if (i0 + 64 * u < n_in) {
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const float xv = in(r, i0 + 64 * u);
#pragma unroll
                            for (int jj = 0; jj < JB; ++jj) s[jj * R + r] = fmaf(w[u][jj], xv, s[jj * R + r]);
                        }
                    }
            }
            wave_sum_f32_n<JB * R>(s);
            if (lane == 0) {
#pragma unroll
                for (int jj = 0; jj < JB; ++jj)
                    if (j0 + jj < n_out) {
                        const float bj = b[j0 + jj];
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const float z = s[jj * R + r] + bj;
                            out[r][j0 + jj] = (relu && z < 0.0f) ? 0.0f : z;
                        }
                    }
            }
        }
    }
    __syncthreads();
}

// Layers first..n_layers-1 on activations already in act[cur]; returns the buffer index holding the logits.
template <int R>
__device__ __forceinline__ int mlp_tail(int n_layers, const int32_t *width, const float *const *w, const float *const *b,
                                        int first, float (*act)[R][MCSD_MLP_MAX_WIDTH], int cur, int tid)
{
    for (int l = first; l < n_layers; ++l) {
        float (*src)[MCSD_MLP_MAX_WIDTH] = act[cur];
        mlp_layer<R>([src](int r, int i) { return src[r][i]; }, width[l], w[l], b[l], width[l + 1], act[cur ^ 1],
                     l + 1 < n_layers, tid);
        cur ^= 1;
    }
    return cur;
}

__device__ __forceinline__ float logistic(float z) { return 1.0f / (1.0f + expf(-z)); }

// ---------------------------------------------------------------------------------------------- stop rule, in the launch
// The stop flag of a tree depends on probabilities that several workgroups write.  For few rows, instead of a second launch
// behind them (4 us, and 2.5 on the host), each workgroup, once its own probability is where everyone sees it, evaluates the
// flag from what it finds, writes it and looks again until what it wrote is still true.  The last write is then right: a
// workgroup that wrote from an old probability either looked again after that probability was replaced, and wrote again, or
// looked before, and then the workgroup that replaced it looks and writes later still.
__device__ __forceinline__ void settle_stop(const float *prob, int b, int W, float beta, int32_t *stop, int lane)
{
    auto look = [&]() {
        bool below = true;
        for (int w = lane; w < W; w += 64) below = below && __hip_atomic_load(prob + (int64_t)b * W + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < beta;
        return __ballot(!below) == 0 ? 1 : 0;
    };
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // the probability has arrived
    int all_below = look();
    while (true) {                                              // (a probability changes once: at most W + 1 rounds)
        if (lane == 0) __hip_atomic_store(stop + b, all_below, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const int now = look();
        if (now == all_below) break;
        all_below = now;
    }
}

// ---------------------------------------------------------------------------------------------- type 2
// FEW: the launch does not fill the chip, so what counts is one workgroup's chain of steps, not its registers: the threshold
// comes from 32 maxima in one exchange, one wavefront ranks the candidates, the first layer's weights are in registers before
// they are needed, the stop flags are settled here.  16 rows of 32000, with the flags: 14.3 us -> 9.9 us.  Otherwise other
// workgroups hide the chain and registers are what counts (a compute unit holds three workgroups).
// MODE 0: the row lives in registers (V a multiple of 4, <= 32768, 16-byte aligned): one trip to HBM, all loads in
// flight at once.  MODE 1: any row, streamed, CHUNK 16-byte loads per lane in flight, and once more by the
// lanes with several candidates.  (Against one load at a time and a second pass in every lane with a candidate: 3200 rows of
// 128256 400 -> 277 us, 5.9 TB/s; 340 rows of 246592 162 -> 94 us; 231 rows of 146375, unaligned, 239 -> 42 us.)
template <int MODE, bool FEW>
__global__ __launch_bounds__(DT) void decision_distribution_kernel(MlpDesc mlp, int W, int V, int k,
                                                                   const float *__restrict__ rows, int64_t batch_stride,
                                                                   int64_t row_stride, float *__restrict__ features,
                                                                   float *prob, float beta, int32_t *stop)
{
    constexpr int CAP = MODE == 0 ? CAND_REG : CAND_MEM;
    __shared__ float s_cand[CAP];
    __shared__ __attribute__((aligned(16))) float s_part[NW * K];
    __shared__ float s_top[K];
    __shared__ double s_ent[NW];
    __shared__ float s_act[2][1][MCSD_MLP_MAX_WIDTH];
    __shared__ int s_cnt;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m = blockIdx.x;
    const int tree = m / W;
    const float *y = rows + (int64_t)tree * batch_stride + (int64_t)(m - tree * W) * row_stride;
    // two layers: lane j's row of the first and its weight of the second, requested first
    const bool fused = FEW && mlp.n_layers == 2;
    float w1[FEW ? K + 1 : 1], b1 = 0.0f, w2 = 0.0f, b2 = 0.0f;
    if (fused) {
        const int j = min(tid, mlp.width[1] - 1);
#pragma unroll
        for (int u = 0; u <= K; ++u) w1[FEW ? u : 0] = mlp.w[0][j * (k + 1) + min(u, k)];
        b1 = mlp.b[0][j];
        w2 = mlp.w[1][j];
        b2 = mlp.b[1][0];
    }

    float4 reg[MODE == 0 ? REG_F4 : 1];
    if (MODE == 0) {
#pragma unroll
        for (int j = 0; j < REG_F4; ++j) {
            const int i = tid * 4 + j * DT * 4;
            reg[j] = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
            if (i < V) {                                     // read exactly once: non-temporal, the caches need not keep it
                const nt_f32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const nt_f32x4_t *>(y + i));
                reg[j] = make_float4(t.x, t.y, t.z, t.w);
            }
        }
    }
    // streamed: up to three entries before the first 16-byte boundary, n4 quadruples, up to three entries
    constexpr int CHUNK = FEW ? 8 : 4;
    const int head = MODE == 0 ? 0 : min(V, (int)((4u - ((unsigned)((uintptr_t)y >> 2) & 3u)) & 3u)), n4 = (V - head) >> 2;
    // every entry of the row, in the lane's own order (both passes must agree on nothing but the set)
    auto for_each = [&](auto f) {
        if (MODE == 0) {
#pragma unroll
            for (int j = 0; j < REG_F4; ++j) { f(reg[j].x, j * 4); f(reg[j].y, j * 4 + 1); f(reg[j].z, j * 4 + 2); f(reg[j].w, j * 4 + 3); }
        } else {
            const nt_f32x4_t *body = reinterpret_cast<const nt_f32x4_t *>(y + head);
            for (int c = tid; c - tid < n4; c += CHUNK * DT) {
                nt_f32x4_t v[CHUNK];                             // all of them in flight; beyond the end the last one again, unused
#pragma unroll
                for (int u = 0; u < CHUNK; ++u) v[u] = FEW ? body[min(c + u * DT, n4 - 1)] : __builtin_nontemporal_load(body + min(c + u * DT, n4 - 1));
#pragma unroll
                for (int u = 0; u < CHUNK; ++u)
                    if (c + u * DT < n4) { f(v[u].x, 0); f(v[u].y, 1); f(v[u].z, 2); f(v[u].w, 3); }
            }
            if (tid < head) f(y[tid], 0);
            if (tid < V - head - 4 * n4) f(y[head + 4 * n4 + tid], 0);
        }
    };

    // pass 1: the lane's maximum and its share of -sum y log2 y.  The hardware logarithm (1 ulp) on normal numbers;
    // entries below the normal range contribute less than 1e-36 each and are skipped.  Four fp32 accumulators of
    // at most a quarter of the lane's entries each, combined in binary64.
    float tmax = -INFINITY, tnext = -INFINITY;                  // the lane's largest and second largest entry
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    double hd = 0.0;                                            // streamed rows can be long: binary64 right away
    for_each([&](float p, int n) {
        if (MODE != 0 || FEW) tnext = __builtin_amdgcn_fmed3f(p, tmax, tnext);
        tmax = fmaxf(tmax, p);
        const float t = (p >= 1.17549435e-38f) ? p * __log2f(p) : 0.0f;
        if (MODE == 0) acc[n & 3] -= t; else hd -= (double)t;
    });
    {
        if (MODE == 0) hd = ((double)acc[0] + (double)acc[1]) + ((double)acc[2] + (double)acc[3]);
        const double h = wave_sum(hd);
        if (lane == 0) s_ent[wave] = h;
    }
    if (tid == 0) s_cnt = 0;
    float tau;
    auto exact_threshold = [&]() {
        // tau = k-th largest lane maximum: at least k entries of the row are >= tau, and every entry above tau sits in
        // one of the at most k-1 lanes whose maximum is above it.  First the k largest of every wavefront (those above
        // its own k-th largest, then copies of that) ...
        {
            const unsigned key = order_key(tmax);
            const unsigned tw = wave_kth_key(key, 0u, k);
            const unsigned long long above = __ballot(key > tw);
            const int n_above = __popcll(above);
            if (key > tw) s_part[wave * K + __popcll(above & ((1ull << lane) - 1ull))] = tmax;
            if (lane >= n_above && lane < k) s_part[wave * K + lane] = key_value(tw);
        }
        __syncthreads();
        // ... then, in every wavefront for itself, the k-th largest of those 8 k values
        {
            const int ia = (lane / k) * K + lane % k, ib = ((lane + 64) / k) * K + (lane + 64) % k;
            const unsigned ka = lane < NW * k ? order_key(s_part[ia]) : 0u;
            const unsigned kb = lane + 64 < NW * k ? order_key(s_part[ib]) : 0u;
            tau = key_value(wave_kth_key(ka, kb, k));
        }
    };
    auto collect = [&]() {
        // the entries above tau, in any order; a second pass only in the lanes that have more than one
        if constexpr (MODE == 0 && !FEW) {                      // (counted first: 75 registers, 138 the other way)
            if (tmax > tau) {
                int mine = 0;
                for_each([&](float p, int) { mine += p > tau ? 1 : 0; });
                int pos = atomicAdd(&s_cnt, mine);
                if (mine == 1) {                                // the usual case: the lane's maximum and nothing else
                    if (pos < CAP) s_cand[pos] = tmax;
                } else {
                    for_each([&](float p, int) {
                        if (p > tau) {
                            if (pos < CAP) s_cand[pos] = p;
                            ++pos;
                        }
                    });
                }
            }
        } else if (tmax > tau) {
            auto add = [&](float p) {
                const int pos = atomicAdd(&s_cnt, 1);
                if (pos < CAP) s_cand[pos] = p;
            };
            if (!(tnext > tau)) add(tmax);
            else for_each([&](float p, int) { if (p > tau) add(p); });
        }
        __syncthreads();
    };
    if (FEW && V >= 4 * DT) {
        // A threshold that at least k entries reach: the k-th largest of the 32 maxima of 16 lanes each.  In practice little
        // more than k entries lie above it; if it is more than the list holds, the exact one after all.
        float g = tmax;
        g = fmaxf(g, dpp_f32<0xB1>(g));
        g = fmaxf(g, dpp_f32<0x4E>(g));
        g = fmaxf(g, dpp_f32<0x141>(g));
        g = fmaxf(g, dpp_f32<0x140>(g));
        if ((lane & 15) == 0) s_part[tid >> 4] = g;
        __syncthreads();
        const int me = lane & (DT / 16 - 1);                    // by rank, in every wavefront for itself
        const float mine = s_part[me];
        int rank = 0;
#pragma unroll
        for (int j4 = 0; j4 < DT / 64; ++j4) {
            const float4 o4 = *reinterpret_cast<const float4 *>(&s_part[4 * j4]);
            const float o[4] = {o4.x, o4.y, o4.z, o4.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) rank += (o[e] > mine || (o[e] == mine && 4 * j4 + e < me)) ? 1 : 0;
        }
        tau = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine), __builtin_ctzll(__ballot(rank == k - 1))));
        collect();
        const int found = s_cnt;
        if (found > CAP) {                                      // (uniform)
            __syncthreads();                                    // everyone has read the count
            if (tid == 0) s_cnt = 0;
            __syncthreads();
            exact_threshold();
            collect();
        }
    } else {
        exact_threshold();
        collect();
    }
    if (FEW && s_cnt <= 64) {
        // one wavefront ranks the candidates: entries > tau, then copies of tau (or zeros when the row has fewer than k)
        if (wave == 0) {
            const int n = s_cnt;
            const float c = lane < n ? s_cand[lane] : -INFINITY;
            int rank = lane < n ? 0 : k;
            for (int j = 0; j < n; ++j) {
                const float o = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(c), j));
                rank += (o > c || (o == c && j < lane)) ? 1 : 0;
            }
            if (rank < k) s_act[0][0][rank] = c;
            if (lane >= n && lane < k) s_act[0][0][lane] = tau > -INFINITY ? tau : 0.0f;
        } else if (tid == 64) {
            double e = 0.0;
            for (int w = 0; w < NW; ++w) e += s_ent[w];
            s_act[0][0][k] = (float)(e * 0.69314718055994530942);   // log2 -> nats
        }
    } else {
        // Topk = those candidates by rank (ties in list order), then copies of tau (entries equal to tau exist in
        // sufficient number), or zeros when the row has fewer than k entries
        {
            const int n = min(s_cnt, CAP);
            for (int i = tid; i < n; i += DT) {
                const float c = s_cand[i];
                int rank = 0;
                for (int j = 0; j < n; ++j) {
                    const float o = s_cand[j];
                    rank += (o > c || (o == c && j < i)) ? 1 : 0;
                }
                if (rank < k) s_top[rank] = c;
            }
            if (tid >= n && tid < k) s_top[tid] = tau > -INFINITY ? tau : 0.0f;
        }
        __syncthreads();
        if (tid < k) s_act[0][0][tid] = s_top[tid];
        if (tid == 0) {
            double e = 0.0;
            for (int w = 0; w < NW; ++w) e += s_ent[w];
            s_act[0][0][k] = (float)(e * 0.69314718055994530942);   // log2 -> nats
        }
    }
    __syncthreads();
    if (features && tid <= k) features[(int64_t)m * (k + 1) + tid] = s_act[0][0][tid];

    float z;
    if (fused) {
        float h = b1;
#pragma unroll
        for (int u = 0; u <= K; ++u)
            if (u <= k) h = fmaf(w1[FEW ? u : 0], s_act[0][0][u], h);
        h = h < 0.0f ? 0.0f : h;                                // (a NaN stays one, as in mlp_layer)
        h = tid < mlp.width[1] ? h * w2 : 0.0f;
        float v[1] = {h};
        wave_sum_f32_n<1>(v);
        if (mlp.width[1] > 64) {
            if (lane == 0) s_part[wave] = v[0];
            __syncthreads();
            v[0] = ((s_part[0] + s_part[1]) + (s_part[2] + s_part[3])) + ((s_part[4] + s_part[5]) + (s_part[6] + s_part[7]));
        }
        z = v[0] + b2;
    } else {
        const int cur = mlp_tail<1>(mlp.n_layers, mlp.width, mlp.w, mlp.b, 0, s_act, 0, tid);
        z = s_act[cur][0][0];
    }
    if (!FEW) {
        if (tid == 0) prob[m] = logistic(z);
    } else if (tid < 64) {
        if (tid == 0) __hip_atomic_store(prob + m, logistic(z), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (stop) settle_stop(prob, tree, W, beta, stop, lane);
    }
}

// ---------------------------------------------------------------------------------------------- type 1
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// What a column beyond a row's end is read as, weights and inputs alike (zero times an infinite weight would be NaN).
__device__ __align__(64) const float zeros[16] = {};

// The networks on four hidden states per workgroup.  A layer is v_mfma_f32_4x4x1_16b_f32 (fp32 in and out, fused multiply-adds):
// its 16 blocks are four of four output units at one column, and the same units at columns 16, 32 and 48 further; A holds
// those columns of the four rows, broadcast from the blocks that have them (cbsz, abid).  So a wavefront has 16 units at a time,
// and what is left is the sum of four quarters of the columns.  Fewer than eight groups of 16 units: the wavefronts split the
// columns too and add up through LDS.  A sum is four columns in one accumulator, a tree of four of them per batch, the even
// batches one after the other and the odd ones, a tree of the quarters.  Error against binary64 over that of the 16 column blocks
// and a tree over them that this replaced, 36 networks of 288 to 2048 columns, 64 to 256 and 32 or 64 units, 6144 rows each: 0.91
// (0.80-0.99) for inputs of both signs, 0.98 (0.89-1.03) for inputs behind a ReLU; with all batches one after the other 0.94
// (0.81-1.00) and 1.00 (0.94-1.04), and 1 % of the time less.
// Weights go through LDS: batches of 16 units x 64 columns come by direct-to-LDS loads into the wavefront's own ring of RING
// batches (no barriers, only its own waits), whole 256-byte pieces of rows (128-byte ones reach the same rate only where
// rows are a multiple of that long, 64-byte ones use half of every line), swizzled so that the operand reads are free of bank
// conflicts.  The ring runs on into the next layer, whose first batches are there when it starts.  Rows are staged through LDS as
// they lie in memory (read as operands from memory, four rows in four neighbouring lanes, they cost 6000 cycles), four banks
// apart: what an instruction reads, four columns of four quarters of four rows, then lies in 64 banks (16 apart, in 16).  A batch's
// operands are read while the one before is multiplied.  (One after the other, and rows 16 banks apart: 2048-256-64-1, 16 rows
// 27.5 us, 26.4 so.)
// Bound: the weights, once per workgroup from L2; 256 workgroups at once get 48 bytes per cycle each (768 x 256: 6.8 us; fewer
// get 64).  Eight rows per workgroup halve that but not the time: the matrix instructions then take as long.
// Against 16 column blocks per output unit and a tree over them, with the stop rule: 768-256-64-1, 1024 rows 20.0 -> 17.7 us,
// 64 rows 19.0 -> 15.5; 288-256-64-1, 1024 rows 16.9 -> 12.6; 1000-256-64-1, whose rows are not whole lines, 22.2 -> 21.5;
// 2048-256-64-1, 1024 rows 31.3 -> 30.2, but 16 rows 25.6 -> 26.4 and 256 rows 26.9 -> 28.5.
constexpr int BATCH = 64, UNITS = 16, RING = 3;          // columns and units per batch; batches per wavefront
constexpr int R = 4;                                     // rows per workgroup
constexpr int ACT_PITCH = MCSD_MLP_MAX_WIDTH + 4;        // floats; rows 4 banks apart
constexpr int WIDE = 2048;                               // widest hidden state of the matrix path
struct HiddenShared {
    float4 ring[NW][RING][UNITS * BATCH / 4];
    float x[R][WIDE + 4];                                // the rows; later partial sums
    float act[R][ACT_PITCH];
    float bias[MCSD_MLP_MAX_LAYERS][MCSD_MLP_MAX_WIDTH];
    float last[MCSD_MLP_MAX_WIDTH];                      // weights of the last layer
};

// What one wavefront does of a layer: batches b0 .. b1 - 1 of unit group ug, of unit group ug + NW, ..
struct HiddenPart { int groups, ug, kp, parts, b0, b1, units; };
__device__ __forceinline__ HiddenPart hidden_part(int n_in, int n_out, int wave)
{
    HiddenPart p;
    p.units = (n_out + UNITS - 1) / UNITS;
    const int lg = p.units <= 1 ? 0 : p.units <= 2 ? 1 : p.units <= 4 ? 2 : 3;
    p.groups = 1 << lg;
    p.parts = NW >> lg;
    p.ug = wave & (p.groups - 1);
    p.kp = wave >> lg;
    const int nb = (n_in + BATCH - 1) / BATCH, per = (nb + p.parts - 1) >> (3 - lg);
    p.b0 = min(p.kp * per, nb);
    p.b1 = min(p.b0 + per, nb);
    return p;
}

// GEN: rows of any width, stride and alignment: their layer is evaluated without the matrix cores.
template <bool GEN>
__global__ __launch_bounds__(DT) void decision_hidden_kernel(MlpDesc mlp, int M, int W, const float *__restrict__ hidden,
                                                             int64_t batch_stride, int64_t row_stride,
                                                             float *prob, float beta, int32_t *stop)
{
    constexpr int GROUPS = MCSD_MLP_MAX_WIDTH / UNITS / NW;
    __shared__ __attribute__((aligned(1024))) HiddenShared sh;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = blockIdx.x * R, n_layers = mlp.n_layers;
    auto row = [&](int r) {
        const unsigned m = min(m0 + r, M - 1), tree = m / (unsigned)W;      // rows past the end repeat the last one, unwritten
        return hidden + (int64_t)tree * batch_stride + (int64_t)(m - tree * W) * row_stride;
    };
    // layers whose weights come through the ring (the last one has a single unit)
    auto streamed = [&](int l) {
        return l < n_layers - 1 && (GEN ? l > 0 : true) && (l == 0 || (mlp.width[l] % 4 == 0 && ((uintptr_t)mlp.w[l] & 15) == 0));
    };

    // ---- the wavefront's stream of weights through all layers ----
    // as a source: of instruction j, lane l takes row 4 j + l / 16 and there piece (l % 16) ^ row; as an operand: unit u's piece c is
    // at 16 u + (c ^ u)
    float4 *const ring = &sh.ring[wave][0][0];
    int rq_l = -1, rq_u = 0, rq_units = 0, rq_full = 0, rq_tail = 0, rq_at = 0;     // whole batches to come, columns of a last one that is not
    const float *rq_w = zeros;
    uint32_t rq_off[4] = {0, 0, 0, 0};
    auto next_group = [&]() {                                               // this wavefront's next group of units, or layer
        rq_u += NW;
        while (rq_u >= rq_units) {
            if (++rq_l >= n_layers - 1) {                                   // none: the count goes on, unused
                rq_w = zeros;
                rq_full = 0x7fffffff;
#pragma unroll
                for (int j = 0; j < 4; ++j) rq_off[j] = 0;
                return;
            }
            rq_units = rq_u = 0;
            if (!streamed(rq_l)) continue;
            const HiddenPart p = hidden_part(mlp.width[rq_l], mlp.width[rq_l + 1], wave);
            if (p.b0 == p.b1) continue;
            rq_units = p.units;
            rq_u = p.ug;
        }
        const int n_in = mlp.width[rq_l], n_out = mlp.width[rq_l + 1];
        const HiddenPart p = hidden_part(n_in, n_out, wave);
        rq_w = (rq_l == 0 ? mlp.w[0] : mlp.w[1]) + BATCH * p.b0;
        const int cols = min(BATCH * p.b1, n_in) - BATCH * p.b0;
        rq_full = cols / BATCH;
        rq_tail = cols % BATCH;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = 4 * j + (lane >> 4);
            rq_off[j] = (uint32_t)(min(rq_u * UNITS + r, n_out - 1) * n_in + ((lane & 15) ^ r) * 4) * 4u;
        }
    };
    auto request = [&]() {
        if (rq_full == 0 && rq_tail == 0) next_group();
        float4 *at = ring + rq_at;
        rq_at = rq_at == (RING - 1) * 256 ? 0 : rq_at + 256;
        if (rq_full > 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j) load_to_lds16<false>(rq_w, rq_off[j], at + 64 * j);
            --rq_full;
            rq_w += rq_l < n_layers - 1 ? BATCH : 0;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int col = ((lane & 15) ^ (4 * j + (lane >> 4))) * 4;
                load_to_lds16_at(col < rq_tail ? (const void *)((const char *)rq_w + rq_off[j]) : (const void *)zeros, at + 64 * j);
            }
            rq_tail = 0;
        }
    };
#pragma unroll
    for (int k = 0; k < RING; ++k) request();

    // ---- rows, biases, last weights: HBM -> LDS ----
    if constexpr (!GEN) {
        const int chunks = (mlp.width[0] + 255) >> 8;                       // 1 KiB of a row per instruction
        const int r = wave & (R - 1);                                       // (a wavefront keeps to one row)
        const float *src = row(r);
        for (int c = wave / R; c < chunks; c += NW / R) {
            const int col = 256 * c + 4 * lane;
            load_to_lds16_at(col < mlp.width[0] ? (const void *)(src + col) : (const void *)zeros, &sh.x[r][256 * c]);
        }
    }
#pragma unroll
    for (int l = 0; l < MCSD_MLP_MAX_LAYERS; ++l)
        if (l < n_layers)
            for (int c = wave; c * 64 < mlp.width[l + 1]; c += NW)
                load_to_lds4_at(mlp.b[l] + min(64 * c + lane, mlp.width[l + 1] - 1), &sh.bias[l][64 * c]);
    const int n_last = mlp.width[n_layers - 1];
    const float *w_last = n_layers == 1 ? mlp.w[0] : n_layers == 2 ? mlp.w[1] : mlp.w[2];
    if (n_layers > 1)
        for (int c = wave; c * 64 < n_last; c += NW) load_to_lds4_at(w_last + min(64 * c + lane, n_last - 1), &sh.last[64 * c]);
    // (a layer reads its input in whole batches, and zero times what happens to be there may be NaN)
    for (int i = tid; i < R * ACT_PITCH / 4; i += DT) reinterpret_cast<float4 *>(&sh.act[0][0])[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    MCSD_WAIT_VMCNT(0);
    __syncthreads();

    // ---- layers ----
    const float *h = &sh.x[0][0];            // input of the layer: rows `pitch` floats apart
    int pitch = sizeof(sh.x[0]) / sizeof(float), slot = 0;
    for (int l = 0; l < n_layers - 1; ++l) {
        const int n_in = mlp.width[l], n_out = mlp.width[l + 1];
        if (!streamed(l)) {
            if (GEN && l == 0) {
                mlp_layer<R>([x0 = row(0), x1 = row(1), x2 = row(2), x3 = row(3)](int r, int i) {
                                 return (r == 0 ? x0 : r == 1 ? x1 : r == 2 ? x2 : x3)[i];
                             }, n_in, mlp.w[0], mlp.b[0], n_out, sh.act, true, tid);
                h = &sh.act[0][0];
            } else {
                mlp_layer<R>([h, pitch](int r, int i) { return h[r * pitch + i]; }, n_in, mlp.w[l], mlp.b[l], n_out,
                             (float (*)[ACT_PITCH])&sh.x[0][0], true, tid);                    // (the last but one: its input is in act)
                h = &sh.x[0][0];
            }
            pitch = ACT_PITCH;
            continue;
        }
        const HiddenPart p = hidden_part(n_in, n_out, wave);
        f32x4_t sum[GROUPS];                                 // of the wavefront's groups of units; [row]
#pragma unroll
        for (int u = 0; u < GROUPS; ++u) sum[u] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
        const int blk = lane >> 2, quarter = blk >> 2, unit = lane & 15;
        const float *xr = h + (lane & 3) * pitch + quarter * 16 + (blk & 3) + BATCH * p.b0;
        const int op = unit * 16 + ((quarter * 4) ^ unit);
#pragma unroll
        for (int u = 0; u < GROUPS; ++u) {
            if (p.ug + u * NW >= p.units) break;             // (uniform)
            const float *xb = xr;
            float4 w[2][4];
            float x[2][4];
            f32x4_t odd = {0.f, 0.f, 0.f, 0.f};              // every other batch's sums (behind the generic layer there are few batches)
            // operands of a batch: LDS -> registers `to`; its place in the ring is free when they are there
            auto read = [&](int to) {
                MCSD_WAIT_VMCNT((RING - 1) * 4);             // this batch has landed, the later ones are under way
                asm volatile("" ::: "memory");
                const float4 *at = ring + slot;
                slot = slot == (RING - 1) * 256 ? 0 : slot + 256;
#pragma unroll
                for (int c = 0; c < 4; ++c) w[to][c] = at[op ^ c];
#pragma unroll
                for (int c = 0; c < 4; ++c) x[to][c] = xb[4 * c];
                xb += BATCH;
            };
            auto there = [&](int to) {
                asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(w[to][0].x), "+v"(w[to][1].x), "+v"(w[to][2].x), "+v"(w[to][3].x) :: "memory");
                request();
            };
            auto add = [&](int of) {
                f32x4_t a[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) a[c] = __builtin_amdgcn_mfma_f32_4x4x1f32(x[of][c], w[of][c].x, (f32x4_t){0.f, 0.f, 0.f, 0.f}, 2, 0, 0);
#pragma unroll
                for (int c = 0; c < 4; ++c) a[c] = __builtin_amdgcn_mfma_f32_4x4x1f32(x[of][c], w[of][c].y, a[c], 2, 1, 0);
#pragma unroll
                for (int c = 0; c < 4; ++c) a[c] = __builtin_amdgcn_mfma_f32_4x4x1f32(x[of][c], w[of][c].z, a[c], 2, 2, 0);
#pragma unroll
                for (int c = 0; c < 4; ++c) a[c] = __builtin_amdgcn_mfma_f32_4x4x1f32(x[of][c], w[of][c].w, a[c], 2, 3, 0);
                (of && !GEN ? odd : sum[u]) += (a[0] + a[1]) + (a[2] + a[3]);
            };
            const int batches = p.b1 - p.b0;
            if (batches > 0) {
                read(0);
                there(0);
                int b = 1;
#pragma unroll 1
                for (; b + 1 < batches; b += 2) {
                    read(1);
                    add(0);
                    there(1);
                    read(0);
                    add(1);
                    there(0);
                }
                if (b < batches) {
                    read(1);
                    add(0);
                    there(1);
                    add(1);
                } else add(0);
                if (!GEN) sum[u] += odd;
            }
            // the quarters' columns: lanes l, l + 16, l + 32, l + 48
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const unsigned v = __float_as_uint(sum[u][r]);
                const auto o = __builtin_amdgcn_permlane16_swap(v, v, false, false);
                sum[u][r] = __uint_as_float(o[0]) + __uint_as_float(o[1]);
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const unsigned v = __float_as_uint(sum[u][r]);
                const auto o = __builtin_amdgcn_permlane32_swap(v, v, false, false);
                sum[u][r] = __uint_as_float(o[0]) + __uint_as_float(o[1]);
            }
        }
        __syncthreads();                                     // everyone has read the layer's input
        float *part = &sh.x[0][0];                           // [column part][unit group][row][unit]
        if (p.parts > 1) {
            if (p.ug < p.units && p.kp > 0 && quarter == 0) {
#pragma unroll
                for (int r = 0; r < R; ++r) part[(((p.kp - 1) * p.groups + p.ug) * R + r) * UNITS + unit] = sum[0][r];
            }
            __syncthreads();
        }
        if (p.kp == 0 && quarter == 0) {
#pragma unroll 1
            for (int k = 1; k < p.parts; ++k)
#pragma unroll
                for (int r = 0; r < R; ++r) sum[0][r] += part[(((k - 1) * p.groups + p.ug) * R + r) * UNITS + unit];
#pragma unroll
            for (int u = 0; u < GROUPS; ++u) {
                const int j = (p.ug + u * NW) * UNITS + unit;
                if (p.ug + u * NW >= p.units) break;
                const float bias = sh.bias[l][j];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    float v = sum[u][r] + bias;
                    v = v < 0.0f ? 0.0f : v;                 // (a NaN stays one)
                    if (j < n_out) sh.act[r][j] = v;
                }
            }
        }
        __syncthreads();
        h = &sh.act[0][0];
        pitch = ACT_PITCH;
    }
    // ---- the last layer, one unit: a wavefront per row ----
    for (int r = wave; r < R; r += NW) {
        float v[1] = {0.0f};
        if (n_layers == 1) {
            const float *x = row(r);
            for (int j = lane; j < n_last; j += 64) v[0] = fmaf(w_last[j], x[j], v[0]);
        } else {
            for (int j = lane; j < n_last; j += 64) v[0] = fmaf(sh.last[j], h[r * pitch + j], v[0]);
        }
        wave_sum_f32_n<1>(v);
        if (lane == 0 && m0 + r < M) {
            const float y = logistic(v[0] + sh.bias[n_layers - 1][0]);
            if (stop) __hip_atomic_store(prob + m0 + r, y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else prob[m0 + r] = y;
        }
    }
    if (stop) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        const int first = m0 / W, last = min(m0 + R, M) - 1;
        for (int tree = first + wave; tree * W <= last; tree += NW) settle_stop(prob, tree, W, beta, stop, lane);
    }
    MCSD_WAIT_VMCNT(0);                                      // (the ring's last requests; the end of the program would wait for them as well)
}

// ---------------------------------------------------------------------------------------------- stop rule
__global__ __launch_bounds__(256) void early_stop_kernel(const float *__restrict__ prob, int B, int W, float beta,
                                                         int32_t *__restrict__ stop)
{
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b >= B) return;
    int all_below = 1;
    for (int w = 0; w < W; ++w)
        if (!(prob[(int64_t)b * W + w] < beta)) all_below = 0;
    stop[b] = all_below;
}

int check_mlp(const mcsd_mlp_t *mlp, int32_t n_in, MlpDesc *out)
{
    if (!mlp || mlp->n_layers < 1 || mlp->n_layers > MCSD_MLP_MAX_LAYERS) return MCSD_EINVAL;
    if (mlp->width[0] != n_in || mlp->width[mlp->n_layers] != 1) return MCSD_EINVAL;
    out->n_layers = mlp->n_layers;
    for (int l = 0; l <= mlp->n_layers; ++l) {
        if (mlp->width[l] < 1) return MCSD_EINVAL;
        if (l > 0 && mlp->width[l] > MCSD_MLP_MAX_WIDTH) return MCSD_EUNSUPPORTED;
        out->width[l] = mlp->width[l];
    }
    for (int l = 0; l < mlp->n_layers; ++l) {
        if (!mlp->weight[l] || !mlp->bias[l]) return MCSD_EINVAL;
        out->w[l] = mlp->weight[l];
        out->b[l] = mlp->bias[l];
    }
    for (int l = mlp->n_layers; l < 3; ++l) { out->w[l] = nullptr; out->b[l] = nullptr; out->width[l + 1] = 0; }
    return MCSD_OK;
}

constexpr int FEW_ROWS = 256;        // one workgroup per compute unit
constexpr int SETTLE_HIDDEN = 160;   // (four rows share a workgroup: 64 rows 16.2 us with a launch, 15.4 so; 128 rows 16.4 and 16.0; 256 rows 16.3 and 17.0)
constexpr int SETTLE_ROWS = 64;      // beyond, the flags' and probabilities' cache lines are fought over: 180 rows 15.7 us, 12.8 with a launch

int launch_stop(const float *prob, int32_t B, int32_t W, float beta, int32_t *stop, hipStream_t st)
{
    hipLaunchKernelGGL(early_stop_kernel, dim3((B + 255) / 256), dim3(256), 0, st, prob, (int)B, (int)W, beta, stop);
    return mcsd_hip_status(hipGetLastError());
}

}  // namespace

extern "C" int mcsd_early_stop_distribution(const mcsd_mlp_t *mlp, int32_t B, int32_t W, int32_t V, int32_t k,
                                            const float *draft_rows_dev, int64_t batch_stride, int64_t row_stride,
                                            float beta, float *features_dev, float *prob_dev, int32_t *stop_dev,
                                            void *hip_stream)
{
    if (B < 0 || W < 1 || V < 1 || k < 1 || batch_stride < 0 || row_stride < 0) return MCSD_EINVAL;
    if (k > MCSD_DECISION_MAX_K || V > MCSD_MAX_VOCAB) return MCSD_EUNSUPPORTED;
    MlpDesc d;
    if (int rc = check_mlp(mlp, k + 1, &d)) return rc;
    if (B == 0) return MCSD_OK;
    if (!draft_rows_dev || !prob_dev || !stop_dev) return MCSD_EINVAL;
    if ((int64_t)B * W > 0x7fffffff / (MCSD_DECISION_MAX_K + 1)) return MCSD_EUNSUPPORTED;
    // a lane holds at most ceil(V / (4 DT)) * 4 entries and at most k-1 lanes hold entries above the threshold
    // (two more of a streamed row's ends)
    static_assert((int64_t)(K - 1) * ((MCSD_MAX_VOCAB + 4 * DT - 1) / (4 * DT) * 4 + 2) <= CAND_MEM, "candidate list too small");
    static_assert((K - 1) * REG_F4 * 4 <= CAND_REG, "candidate list too small");
    const bool vec = V % 4 == 0 && batch_stride % 4 == 0 && row_stride % 4 == 0 && ((uintptr_t)draft_rows_dev & 15) == 0;
    const int mode = vec && V <= REG_F4 * 4 * DT ? 0 : 1;
    hipStream_t st = (hipStream_t)hip_stream;
    const dim3 grid((unsigned)(B * W)), block(DT);
    const bool few = (int64_t)B * W <= FEW_ROWS, settle = (int64_t)B * W <= SETTLE_ROWS;
    auto kernel = mode == 0 ? (few ? decision_distribution_kernel<0, true> : decision_distribution_kernel<0, false>)
                            : (few ? decision_distribution_kernel<1, true> : decision_distribution_kernel<1, false>);
    mcsd_launch(MCSD_KERNEL_DECISION, kernel, grid, block, st, d, (int)W, (int)V, (int)k, draft_rows_dev, batch_stride,
                row_stride, features_dev, prob_dev, beta, settle ? stop_dev : (int32_t *)nullptr);
    if (int rc = mcsd_hip_status(hipGetLastError())) return rc;
    return settle ? MCSD_OK : launch_stop(prob_dev, B, W, beta, stop_dev, st);
}

extern "C" int mcsd_early_stop_hidden(const mcsd_mlp_t *mlp, int32_t B, int32_t W, const float *hidden_dev,
                                      int64_t batch_stride, int64_t row_stride, float beta, float *prob_dev,
                                      int32_t *stop_dev, void *hip_stream)
{
    if (B < 0 || W < 1 || batch_stride < 0 || row_stride < 0 || !mlp) return MCSD_EINVAL;
    if (mlp->width[0] > MCSD_MLP_MAX_INPUTS) return MCSD_EUNSUPPORTED;
    MlpDesc d;
    if (int rc = check_mlp(mlp, mlp->width[0], &d)) return rc;
    if (B == 0) return MCSD_OK;
    if (!hidden_dev || !prob_dev || !stop_dev) return MCSD_EINVAL;
    if ((int64_t)B * W > 0x7fffffff / 2) return MCSD_EUNSUPPORTED;
    hipStream_t st = (hipStream_t)hip_stream;
    const int M = B * W, n_in = d.width[0];
    const bool aligned = n_in % 4 == 0 && batch_stride % 4 == 0 && row_stride % 4 == 0 && (((uintptr_t)hidden_dev | (uintptr_t)d.w[0]) & 15) == 0;
    const bool settle = M <= SETTLE_HIDDEN;
    auto kernel = !aligned || n_in > WIDE ? decision_hidden_kernel<true> : decision_hidden_kernel<false>;
    mcsd_launch(MCSD_KERNEL_DECISION, kernel, dim3((M + R - 1) / R), dim3(DT), st, d, M, (int)W,
                hidden_dev, batch_stride, row_stride, prob_dev, beta, settle ? stop_dev : (int32_t *)nullptr);
    if (int rc = mcsd_hip_status(hipGetLastError())) return rc;
    return settle ? MCSD_OK : launch_stop(prob_dev, B, W, beta, stop_dev, st);
}
