// Stages 1 and 2 in one pass (Algorithm 1 steps 1-2): the gating decision of every token and the
// GPU-to-GPU traffic matrix D^(1) it implies, without reading the indices back from memory.
//
// For rows of at most 8 logits a lane holds a whole row, so the lane that picks a row's k experts
// also knows the row's source GPU and replica index: it bumps the destination's bin in an LDS
// histogram of the workgroup (which owns a slice of one (matrix, source GPU) pair's tokens) right
// after the pick.  HBM traffic is the logits once, plus the indices once if the caller wants them;
// the separate stage 2 would read them again.  The picks are made by the same comparisons as stage 1
// (strict '>' in ascending expert index, winners replaced by -inf), so both outputs are bit-identical
// to the two separate calls.
// Rows of 9..32 logits with k <= 8 are spread over the lanes by whole-row loads and an exchange, and picked from a list.
// Rows of 33..256 logits with k <= 8 have a one-pass kernel too, for callers that do not want the indices: the
// insertion kernel of stage 1 with the same addition - once the lanes of a row hold its winners, lane j looks up
// the destination of winner j and bumps its bin.  A workgroup walks a few hundred consecutive tokens of one pair
// so that its G counts are a small share of the logits it read.  When the indices are wanted the two stages run
// back to back instead: 4 194 304 rows of 256 logits, top-8, take 0.70 ms in one pass without and 0.71 in two kernels with the
// indices, and the index stores cost the one-pass kernel 0.08 ms more (its workgroups live eight times longer than stage 1's,
// which ends the launch on a longer tail).  Other shapes always run the two stages.
//
// Short-lived workgroups of one or a few rounds of 512 tokens stream best, so a pair's tokens are cut
// into many slices; each slice leaves its G counts in the workspace with plain stores and a second,
// small kernel sums a pair's slices and scales by the payload.
#include "common.h"
#include "count_reduce.h"
#include "topk_core.h"

namespace rs {

typedef float rt_f32x4 __attribute__((ext_vector_type(4)));
typedef int rt_i32x2 __attribute__((ext_vector_type(2)));

constexpr int kRtThreads = 256;
constexpr int kRtThreadsWhole = 1024; // rows of at most 8 logits: see rt_whole
constexpr int kRtThreadsTwo = 512;    // rows of 9..32 logits: see rt_list_splits
// rows per thread with their loads in flight together: 64 bytes of logits and more
constexpr int rt_unroll(int vpl) { return vpl <= 16 ? 2 : 1; }
constexpr int rt_round(int vpl) { return kRtThreads * rt_unroll(vpl); }   // tokens per workgroup and round
constexpr int rt_vpl(int E) { return E <= 4 ? 4 : E <= 8 ? 8 : E <= 16 ? 16 : 32; }
constexpr int kRtTableMax = 8192;     // placement entries staged in LDS

struct RtArgs {
    const float *logits;
    const int32_t *expert_gpu;
    int32_t *topk_idx;       // may be null: the picks are only counted
    int64_t *D1;
    uint32_t *partial;       // [pairs][splits][G] counts when a pair has several slices
    int64_t tokens_per_gpu;
    int64_t payload;
    int32_t E, k, R, rmask;  // rmask >= 0 when R is a power of two
    int32_t G, splits;
    int32_t copies, lanes_per_period;
    int32_t bin_stride;      // words between histogram copies: odd, so that a bin's copies lie in different LDS banks
    int32_t table_in_lds;
    int32_t wide_idx;        // bytes topk_idx is aligned to: 4, 8 or 16 (or more)
};

// D1[pair][d] = payload * sum of the pair's slice counts
__global__ __launch_bounds__(256) void rt_reduce_kernel(const uint32_t *__restrict__ partial, int64_t *__restrict__ D1, int64_t n, int G,
                                                        int splits, int64_t payload)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t pair = i / G;
        const int d = (int)(i - pair * G);
        const uint32_t *src = partial + pair * splits * G + d;
        uint64_t cnt = 0;
        int p = 0;
        for (; p + 8 <= splits; p += 8) {                    // eight independent loads in flight
            uint32_t x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = src[(int64_t)(p + u) * G];
#pragma unroll
            for (int u = 0; u < 8; ++u) cnt += x[u];
        }
        for (; p < splits; ++p) cnt += src[(int64_t)p * G];
        D1[i] = (int64_t)cnt * payload;
    }
}

int launch_count_reduce(const uint32_t *partial, int64_t *D1, int64_t n, int G, int splits, int64_t payload, hipStream_t st)
{
    const int64_t blocks = (n + 255) / 256 > 65536 ? 65536 : (n + 255) / 256;
    hipLaunchKernelGGL(rt_reduce_kernel, dim3((unsigned)blocks), dim3(256), 0, st, partial, D1, n, G, splits, payload);
    return launch_status();
}

template <int VPL, bool VEC4>
__device__ __forceinline__ void rt_load_row(const RtArgs &a, int64_t row, bool live, float (&v)[VPL])
{
    if constexpr (VEC4) {
#pragma unroll
        for (int c = 0; c < VPL / 4; ++c) {
            rt_f32x4 x = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
            if (live && 4 * c < a.E) x = __builtin_nontemporal_load(reinterpret_cast<const rt_f32x4 *>(a.logits + row * a.E + 4 * c));
            v[4 * c + 0] = x.x; v[4 * c + 1] = x.y; v[4 * c + 2] = x.z; v[4 * c + 3] = x.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < VPL; ++j) v[j] = (live && j < a.E) ? a.logits[row * a.E + j] : -INFINITY;
    }
}

template <int VPL, int L, int J>
__device__ __forceinline__ void rt_insert(const float (&v)[VPL], int E, int (&lst)[L], unsigned &bits)
{
    if constexpr (J < VPL) {
        if constexpr (J % 4 == 0 && J > VPL / 2 && J >= L) {             // E > VPL / 2
            if (J >= E) return;                     // uniform
        }
        const unsigned c = __float_as_uint(v[J] + 0.0f);
        bits |= c;
        list_insert<L, (J < L ? J : L)>(lst, make_ikey<~((unsigned)VPL - 1u) | (unsigned)J>(c, ~((unsigned)VPL - 1u)));
        rt_insert<VPL, L, J + 1>(v, E, lst, bits);
    }
}

// picks of one row, largest first, lowest index on ties; counts each pick's destination GPU.  With k = 2 the two
// winners come back in `pair` and the caller stores them once all its rows are picked: a store between two rows
// made the second row's table lookups wait for it (memory operations of a wavefront complete in order).
template <int VPL>
__device__ __forceinline__ void rt_pick_row(const RtArgs &a, const int32_t *table, unsigned *bins, int64_t row, int64_t t_local,
                                            float (&v)[VPL], rt_i32x2 &pair)
{
    const int rho = a.rmask >= 0 ? (int)(t_local & a.rmask) : (int)(t_local % a.R);
    int keep0 = 0;
    for (int sel = 0; sel < a.k; ++sel) {
        float bv = -INFINITY;
        int bi = INT_MAX;
#pragma unroll
        for (int j = 0; j < VPL; ++j) {
            const bool better = v[j] > bv;
            bv = better ? v[j] : bv;
            bi = better ? j : bi;
        }
#pragma unroll
        for (int j = 0; j < VPL; ++j) v[j] = (j == bi) ? -INFINITY : v[j];
        if ((unsigned)bi < (unsigned)a.E) {
            const int32_t d = table[bi * a.R + rho];
            if ((unsigned)d < (unsigned)a.G) atomicAdd(&bins[d], 1u);
        }
        if (a.k == 2) {                                       // both winners leave in one 8-byte store, issued by the caller
            if (sel == 0) keep0 = bi;
            else { pair.x = keep0; pair.y = bi; }
        } else if (a.topk_idx) {
            a.topk_idx[row * a.k + sel] = bi;
        }
    }
}

// 64 rows of 9..32 logits (tokens first .. first + 63 of a pair, those below hi) into the lanes, a whole row each.  A lane reading
// its own row 16 bytes at a time touches 64 lines per load and gets an eighth of each (32 logits: 0.26 ms instead of 0.084 for
// 402 MB), so the LPR = VPL / 4 lanes of a group read LPR rows together, one whole row per load, and exchange: out[c] of lane q
// is what lane c read in load q, a transposition by log2(LPR) exchange steps.  Lane p * LPR + q ends with row q * (64 / LPR) + p.
template <int VPL>
__device__ __forceinline__ int rt_list_row(int lane) { constexpr int LPR = VPL / 4; return (lane % LPR) * (64 / LPR) + lane / LPR; }

template <int D>
__device__ __forceinline__ float xor_lane(float f)
{
    int v = __float_as_int(f);
    if constexpr (D == 1) v = __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);
    else if constexpr (D == 2) v = __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);
    else {                                                               // lane ^ 7, then ^ 3
        v = __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true);
        v = __builtin_amdgcn_update_dpp(0, v, 0x1B, 0xF, 0xF, true);
    }
    return __int_as_float(v);
}

template <int VPL, int D>
__device__ __forceinline__ void rt_exchange(float (&v)[VPL], int q)
{
    constexpr int LPR = VPL / 4;
    const bool up = (q & D) != 0;
#pragma unroll
    for (int i = 0; i < LPR; ++i)
        if ((i & D) == 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float a = v[4 * i + e], b = v[4 * (i + D) + e];
                const float got = xor_lane<D>(up ? a : b);
                v[4 * i + e] = up ? got : a;
                v[4 * (i + D) + e] = up ? b : got;
            }
        }
}

template <int VPL>
__device__ __forceinline__ void rt_load_rows(const RtArgs &a, int64_t row0, int64_t first, int64_t hi, int lane, float (&v)[VPL])
{
    constexpr int LPR = VPL / 4;
    const int p = lane / LPR, q = lane % LPR;
#pragma unroll
    for (int i = 0; i < LPR; ++i) {
        const int64_t t = first + i * (64 / LPR) + p;
        rt_f32x4 x = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};   // logits that do not exist, as in row_load
        if (t < hi && 4 * q < a.E) x = __builtin_nontemporal_load(reinterpret_cast<const rt_f32x4 *>(a.logits + (row0 + t) * a.E + 4 * q));
        v[4 * i + 0] = x.x; v[4 * i + 1] = x.y; v[4 * i + 2] = x.z; v[4 * i + 3] = x.w;
    }
}
template <int VPL>
__device__ __forceinline__ void rt_rows_to_lanes(float (&v)[VPL], int lane)
{
    const int q = lane % (VPL / 4);
    rt_exchange<VPL, 1>(v, q);
    rt_exchange<VPL, 2>(v, q);
    if constexpr (VPL == 32) rt_exchange<VPL, 4>(v, q);
}

// Picks of one row of 9..32 logits, largest first, lowest index on ties: win[0..k).  The list form of topk_core.h with the whole
// row in one lane: the lane's L >= k + 1 largest keys are the row's winners and its best loser, so nothing is merged and only
// neighbours that share a cut value which the cut took something from send the lane to the full comparisons.  16 logits, top-4:
// 140 instructions a row where the rounds take 320 (and 60 where four lanes share a row, but each of those serves 16 rows, not 64).
template <int VPL, int L>
__device__ __forceinline__ void rt_pick_list(const RtArgs &a, const float (&v)[VPL], int (&win)[L - 1])
{
    constexpr unsigned MASK = (unsigned)VPL - 1u;
    if constexpr (L == 2) {                         // the largest logit alone: compared as it is
        float bv = -INFINITY;
        int bi = INT_MAX;
#pragma unroll
        for (int j = 0; j < VPL; ++j) {
            const bool better = v[j] > bv;
            bv = better ? v[j] : bv;
            bi = better ? j : bi;
        }
        win[0] = bi;
        return;
    }
    int lst[L];
    unsigned bits = 0;
    rt_insert<VPL, L, 0>(v, a.E, lst, bits);
    unsigned close = 0xFFFFFFFFu;
#pragma unroll
    for (int j = 1; j < L; ++j)
        if (j <= a.k) close = min_xor_dist(close, (unsigned)lst[j], (unsigned)lst[j - 1]);
#pragma unroll
    for (int j = 0; j < L - 1; ++j) win[j] = (int)key_index<MASK>((unsigned)lst[j]);
    if (close < MASK && (bits & MASK) != 0u) {
        float x[VPL];
#pragma unroll
        for (int j = 0; j < VPL; ++j) x[j] = v[j];
#pragma unroll
        for (int sel = 0; sel < L - 1; ++sel) {
            if (sel >= a.k) break;
            float bv = -INFINITY;
            int bi = INT_MAX;
#pragma unroll
            for (int j = 0; j < VPL; ++j) {
                const bool better = x[j] > bv;
                bv = better ? x[j] : bv;
                bi = better ? j : bi;
            }
#pragma unroll
            for (int j = 0; j < VPL; ++j) x[j] = (j == bi) ? -INFINITY : x[j];
            win[sel] = bi;
        }
    }
}

// the row's indices, in the widest pieces that k and the array's alignment allow
template <int KM>
__device__ __forceinline__ void rt_store_row(const RtArgs &a, int64_t row, const int (&win)[KM])
{
    int32_t *dst = a.topk_idx + row * a.k;
    if (a.wide_idx >= 16 && (a.k & 3) == 0) {
#pragma unroll
        for (int j = 0; j + 4 <= KM; j += 4)
            if (j < a.k) {
                i32x4 x;
                x.x = win[j]; x.y = win[j + 1]; x.z = win[j + 2]; x.w = win[j + 3];
                __builtin_nontemporal_store(x, reinterpret_cast<i32x4 *>(dst + j));
            }
    } else if (a.wide_idx >= 8 && (a.k & 1) == 0) {
#pragma unroll
        for (int j = 0; j + 2 <= KM; j += 2)
            if (j < a.k) {
                i32x2 x;
                x.x = win[j]; x.y = win[j + 1];
                __builtin_nontemporal_store(x, reinterpret_cast<i32x2 *>(dst + j));
            }
    } else {
#pragma unroll
        for (int j = 0; j < KM; ++j)
            if (j < a.k) __builtin_nontemporal_store(win[j], dst + j);
    }
}

// L = 0: rows of at most 8 logits, picked in rounds.  L > 0: rows of 9..32 logits and k < L, picked from a list.
// THREADS: kRtThreads, or more where a workgroup's tokens are several of its rounds (kRtThreadsWhole for L = 0, kRtThreadsTwo otherwise).
template <int VPL, int L, bool VEC4, bool TABLE_LDS, int THREADS>
__global__ __launch_bounds__(THREADS) void route_traffic_kernel(RtArgs a)
{
    constexpr int kRtUnroll = rt_unroll(VPL), kRtRound = THREADS * kRtUnroll;
    extern __shared__ unsigned rt_lds[];
    // [copies][G] counters; lanes that share a replica index - every lanes_per_period-th lane - would pile
    // onto the bins of the popular experts, so neighbouring periods count in different copies
    unsigned *all_bins = rt_lds;
    unsigned *bins = all_bins + (size_t)((threadIdx.x / a.lanes_per_period) & (a.copies - 1)) * a.bin_stride;
    int32_t *lds_table = reinterpret_cast<int32_t *>(rt_lds + (size_t)a.copies * a.bin_stride);
    const int64_t pair = blockIdx.x / a.splits;              // b*G + s
    const int part = blockIdx.x % a.splits;

    // the pair's tokens are dealt to its workgroups in rounds of kRtRound, so the workgroups of a
    // pair, which are dispatched together, sweep one contiguous window of the logits side by side
    const int64_t hi = a.tokens_per_gpu;
    const int64_t row0 = pair * a.tokens_per_gpu;
    const int64_t round = (int64_t)a.splits * kRtRound;
    const int lane = threadIdx.x & 63;
    const int wave0 = threadIdx.x & ~63;
    int64_t t = (int64_t)part * kRtRound + (L > 0 ? wave0 + rt_list_row<VPL>(lane) : (int)threadIdx.x);
    const int64_t t_wave = (int64_t)part * kRtRound + wave0;            // L > 0: first token of the wavefront's 64
    float v[kRtUnroll][VPL];
    // the first round's logits are requested before the histogram is set up, so that clearing it and
    // fetching the placement table do not delay them
#pragma unroll
    for (int u = 0; u < kRtUnroll; ++u) {
        const int64_t tu = t + (int64_t)u * THREADS;
        if constexpr (L > 0) rt_load_rows<VPL>(a, row0, t_wave + (int64_t)u * THREADS, hi, lane, v[u]);
        else rt_load_row<VPL, VEC4>(a, row0 + tu, tu < hi, v[u]);
    }

    for (int i = threadIdx.x; i < a.bin_stride * a.copies; i += THREADS) all_bins[i] = 0;
    if (TABLE_LDS)
        for (int i = threadIdx.x; i < a.E * a.R; i += THREADS) lds_table[i] = a.expert_gpu[i];
    __syncthreads();

    if constexpr (L > 0) {
        const int32_t *table;
        if constexpr (TABLE_LDS) table = lds_table; else table = a.expert_gpu;
        for (int64_t tw = t_wave; tw < hi; tw += round) {               // wavefront-uniform: the exchanges take all lanes
            int win[kRtUnroll][L - 1];
#pragma unroll
            for (int u = 0; u < kRtUnroll; ++u) {
                const int64_t tu = t + (int64_t)u * THREADS;
                rt_rows_to_lanes<VPL>(v[u], lane);
                if (tu < hi) {
                    rt_pick_list<VPL, L>(a, v[u], win[u]);
                    const int rho = a.rmask >= 0 ? (int)(tu & a.rmask) : (int)((uint32_t)tu % (uint32_t)a.R);   // fewer than 2^31 tokens
#pragma unroll
                    for (int j = 0; j < L - 1; ++j)
                        if (j < a.k && (unsigned)win[u][j] < (unsigned)a.E) {
                            const int32_t d = table[win[u][j] * a.R + rho];
                            if ((unsigned)d < (unsigned)a.G) atomicAdd(&bins[d], 1u);
                        }
                }
            }
#pragma unroll
            for (int u = 0; u < kRtUnroll; ++u) {
                const int64_t tu = t + (int64_t)u * THREADS;
                if (tu < hi) rt_store_row<L - 1>(a, row0 + tu, win[u]);
            }
            t += round;
            if (tw + round >= hi) break;
#pragma unroll
            for (int u = 0; u < kRtUnroll; ++u) rt_load_rows<VPL>(a, row0, tw + round + (int64_t)u * THREADS, hi, lane, v[u]);
        }
    }
    while (L == 0 && t < hi) {
        rt_i32x2 pairs[kRtUnroll];
#pragma unroll
        for (int u = 0; u < kRtUnroll; ++u) {
            const int64_t tu = t + (int64_t)u * THREADS;
            pairs[u].x = 0; pairs[u].y = 0;
            // two calls, so that the table is read with LDS instructions where it is in LDS: through one pointer
            // that may be either, every lookup waited for all of the wavefront's memory traffic
            if (tu < hi) {
                if (TABLE_LDS) rt_pick_row<VPL>(a, lds_table, bins, row0 + tu, tu, v[u], pairs[u]);
                else rt_pick_row<VPL>(a, a.expert_gpu, bins, row0 + tu, tu, v[u], pairs[u]);
            }
        }
        if (a.topk_idx && a.k == 2) {
#pragma unroll
            for (int u = 0; u < kRtUnroll; ++u) {
                const int64_t tu = t + (int64_t)u * THREADS;
                if (tu < hi) __builtin_nontemporal_store(pairs[u], reinterpret_cast<rt_i32x2 *>(a.topk_idx + (row0 + tu) * 2));
            }
        }
        t += round;
        if (t >= hi) break;
#pragma unroll
        for (int u = 0; u < kRtUnroll; ++u) {
            const int64_t tu = t + (int64_t)u * THREADS;
            rt_load_row<VPL, VEC4>(a, row0 + tu, tu < hi, v[u]);
        }
    }
    __syncthreads();

    int64_t *dst = a.D1 + pair * a.G;
    for (int i = threadIdx.x; i < a.G; i += THREADS) {
        unsigned cnt = 0;
        for (int c = 0; c < a.copies; ++c) cnt += all_bins[(size_t)c * a.bin_stride + i];
        if (a.splits == 1) dst[i] = (int64_t)cnt * a.payload;    // sole owner of the pair
        else a.partial[((int64_t)pair * a.splits + part) * a.G + i] = cnt;
    }
}

template <int VPL, int L, int THREADS>
static int launch_route_traffic_t(const RtArgs &a, int64_t pairs, size_t lds, hipStream_t st)
{
    const bool vec4 = (a.E % 4 == 0) && (reinterpret_cast<uintptr_t>(a.logits) % 16 == 0);
    const dim3 grid((unsigned)(pairs * a.splits));
    if (vec4 && a.table_in_lds) hipLaunchKernelGGL((route_traffic_kernel<VPL, L, true, true, THREADS>), grid, dim3(THREADS), lds, st, a);
    else if (vec4) hipLaunchKernelGGL((route_traffic_kernel<VPL, L, true, false, THREADS>), grid, dim3(THREADS), lds, st, a);
    else if constexpr (L == 0) {
        if (a.table_in_lds) hipLaunchKernelGGL((route_traffic_kernel<VPL, L, false, true, THREADS>), grid, dim3(THREADS), lds, st, a);
        else hipLaunchKernelGGL((route_traffic_kernel<VPL, L, false, false, THREADS>), grid, dim3(THREADS), lds, st, a);
    }
    return launch_status();
}

// An uncut pair of more than one round takes 1024 threads instead of 256 while the chip has room for its wavefronts: up to 256 pairs (a CU
// holds two such workgroups) always - 256 GPUs x 2048 tokens, 8 logits: top-2 8.0 -> 4.8 us, top-8 22.7 -> 15.1 - and up to 512 from three rounds on
// (512 GPUs, top-2: 1024 tokens 5.9 / 6.2, 2048 tokens 10.5 / 9.5, 4096 tokens 19.0 / 15.8); 1024 pairs lose (4096 tokens: 26.9 / 33.1).
static bool rt_whole(int64_t tokens, int64_t pairs, int64_t splits, int round)
{
    return splits == 1 && tokens > round && (pairs <= 256 || (pairs <= 512 && tokens > 2 * round));
}

template <int VPL, int L>
static int launch_route_traffic(const RtArgs &a, int64_t pairs, int64_t slice, size_t lds, hipStream_t st)
{
    if constexpr (L == 0) {
        if (rt_whole(a.tokens_per_gpu, pairs, a.splits, rt_round(VPL))) return launch_route_traffic_t<VPL, L, kRtThreadsWhole>(a, pairs, lds, st);
    } else {
        if ((a.splits == 1 ? a.tokens_per_gpu : slice) > rt_round(VPL)) return launch_route_traffic_t<VPL, L, kRtThreadsTwo>(a, pairs, lds, st);
    }
    return launch_route_traffic_t<VPL, L, kRtThreads>(a, pairs, lds, st);
}

// ---------------------------------------------------------------------------------------------- rows of 33..256 logits
struct RwArgs {
    const float *logits;
    const int32_t *expert_gpu;
    int64_t *D1;
    uint32_t *partial;       // [pairs][splits][G] counts when a pair has several slices
    int64_t tokens_per_gpu;
    int64_t payload;
    int32_t E, k, R, rmask;  // rmask >= 0 when R is a power of two
    int32_t G, splits;
    int32_t iters;           // row groups (of 4 * 64/LANES tokens) a workgroup walks
    int32_t table_in_lds;
};

template <int LANES, int VPL, int L, int WAVES, bool FULL, bool TABLE_LDS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WAVES, 8))) void route_traffic_insert_kernel(RwArgs a)
{
    extern __shared__ unsigned rw_lds[];
    constexpr int RPW = 64 / LANES;                 // rows per wavefront
    constexpr int RPB = 4 * RPW;                    // rows per workgroup and iteration
    constexpr unsigned MASK = (unsigned)(LANES * VPL) - 1u;
    unsigned *bins = rw_lds;                        // [G] destination counts of this workgroup's tokens
    int32_t *lds_table = reinterpret_cast<int32_t *>(rw_lds + a.G);
    const int64_t pair = blockIdx.x / a.splits;     // b*G + s
    const int part = blockIdx.x % a.splits;
    const int lane = threadIdx.x & 63;
    const int q = lane % LANES;

    for (int i = threadIdx.x; i < a.G; i += 256) bins[i] = 0;
    if (TABLE_LDS)
        for (int i = threadIdx.x; i < a.E * a.R; i += 256) lds_table[i] = a.expert_gpu[i];
    __syncthreads();
    const int32_t *table;
    if constexpr (TABLE_LDS) table = lds_table; else table = a.expert_gpu;   // one definite kind of memory per instantiation

    const int64_t t_lo = (int64_t)part * a.iters * RPB;
    const float *pair_logits = a.logits + pair * a.tokens_per_gpu * a.E;
    const int64_t t_first = t_lo + (threadIdx.x >> 6) * RPW + lane / LANES;     // this lane's token in the first row group
    auto clamp_token = [&](int64_t t) { return t < a.tokens_per_gpu ? t : a.tokens_per_gpu - 1; };
    float4 x[VPL / 4];
    row_load<LANES, VPL, FULL>(pair_logits + clamp_token(t_first) * a.E, a.E, q, x);
    for (int it = 0; it < a.iters; ++it) {
        if (t_lo + (int64_t)it * RPB >= a.tokens_per_gpu) break;                 // workgroup-uniform
        const int64_t t = t_first + (int64_t)it * RPB;                           // token inside the pair
        const bool live = t < a.tokens_per_gpu;
        const int rho = a.rmask >= 0 ? (int)(t & a.rmask) : (int)(t % a.R);
        auto count = [&](int e) {
            if ((unsigned)e < (unsigned)a.E) {
                const int32_t d = table[e * a.R + rho];
                if ((unsigned)d < (unsigned)a.G) atomicAdd(&bins[d], 1u);
            }
        };
        int keys[VPL], own[L];
        unsigned bits;
        lane_keys<LANES, VPL>(x, q, keys, bits);
        // the next row group's logits are on the way while this one's keys are worked on
        if (it + 1 < a.iters) row_load<LANES, VPL, FULL>(pair_logits + clamp_token(t + RPB) * a.E, a.E, q, x);
        list_of_keys<LANES, VPL, L, FULL>(keys, a.E, own);
        unsigned u[8];
        const bool bad = row_best<LANES, VPL, L, 8>(own, bits, a.k, u);
        if (__ballot(live && bad) == 0ull) {
#pragma unroll
            for (int r = 0; r < (8 + LANES - 1) / LANES; ++r) {          // winners q, q+LANES, ... are counted by this lane
                unsigned sel = 0;
#pragma unroll
                for (int j = 0; j < 8; ++j) sel = (j == q + r * LANES) ? u[j] : sel;
                if (live && q + r * LANES < a.k) count((int)key_index<MASK>(sel));
            }
        } else {
            // rare: the wavefront's rows are read again and picked by full comparisons
            row_exact<LANES, VPL>(pair_logits + t * a.E, live, a.E, a.k, q, [&](int sel, int bi) {
                if (live && q == sel % LANES) count(bi);
            });
        }
    }
    __syncthreads();
    int64_t *dst = a.D1 + pair * a.G;
    for (int i = threadIdx.x; i < a.G; i += 256) {
        if (a.splits == 1) dst[i] = (int64_t)bins[i] * a.payload;      // sole owner of the pair
        else a.partial[((int64_t)pair * a.splits + part) * a.G + i] = bins[i];
    }
}

// Row groups per workgroup: at least 64 rows (32 of more than 128 logits), and so many tokens that the G counts a workgroup leaves behind are
// under a hundredth of the logits it read, or under a two-hundredth where that still leaves 2048 workgroups (64 GPUs x 4096 tokens of 128
// logits, top-2: 28.3 -> 26.4 us; where it leaves 256 of them, 256 GPUs x 1024 tokens of 64 logits, top-8: 23.2 -> 28.7).  No more than 128
// slices a pair: one thread of the second kernel sums a count over all of them (16 GPUs x 16384 tokens of 256 logits: 512 slices 62 us,
// 128 slices 54; 4 GPUs: 35 and 22).
constexpr int kRwMaxSplits = 128;
// `longer`: the longer slices in any case, for a caller whose workspace holds no more.
static int rw_iters(int64_t tokens_per_gpu, int64_t G, int64_t pairs, int E, int rows_per_group, bool longer)
{
    const int64_t least = E <= 128 ? 64 : 32;
    int64_t rows = rows_per_group;
    auto splits = [&](int64_t r) { return (tokens_per_gpu + r - 1) / r; };
    while ((rows < least || rows * E < 128 * G || splits(rows) > kRwMaxSplits) && rows < tokens_per_gpu) rows *= 2;
    if (rows * E < 256 * G && (longer || pairs * splits(2 * rows) >= 2048)) rows *= 2;
    // slices of one length: three thousand tokens are two slices of 1536, not one of 2048 and the rest
    const int64_t groups = (tokens_per_gpu + rows_per_group - 1) / rows_per_group;
    return (int)((groups + splits(rows) - 1) / splits(rows));
}

template <int LANES, int VPL, int L, int WAVES>
static int launch_route_traffic_insert(RwArgs a, int64_t pairs, hipStream_t st)
{
    const size_t lds = sizeof(unsigned) * (size_t)a.G + (a.table_in_lds ? sizeof(int32_t) * (size_t)a.E * a.R : 0);
    const dim3 grid((unsigned)(pairs * a.splits));
    const bool full = a.E == LANES * VPL;
#define RW_LAUNCH(FULL_, TAB_) hipLaunchKernelGGL((route_traffic_insert_kernel<LANES, VPL, L, WAVES, FULL_, TAB_>), grid, dim3(256), lds, st, a)
    if (full && a.table_in_lds) RW_LAUNCH(true, true);
    else if (full) RW_LAUNCH(true, false);
    else if (a.table_in_lds) RW_LAUNCH(false, true);
    else RW_LAUNCH(false, false);
#undef RW_LAUNCH
    return launch_status();
}

// Lanes per row of the one-pass kernel: 16 logits per lane up to 128, as in stage 1, and 32 above, where stage 1 takes 16 lanes of 16: a
// workgroup here lives long enough to have its next rows' loads in flight (64 GPUs x 16384 tokens of 256 logits, top-2 / top-8: 167 / 174 us,
// 178 / 186 by 16 lanes; 512 GPUs x 256 tokens: 24.4 / 33.9 and 27.6 / 33.0).
static int rw_lanes(int E) { return E <= 64 ? 4 : 8; }

// shape of the one-pass kernel for rows of 33..256 logits; false: the two stages run back to back
static bool rw_shape(const float *logits, int32_t E, int32_t k, int64_t G, int *lanes)
{
    const bool vec4 = (E % 4 == 0) && (reinterpret_cast<uintptr_t>(logits) % 16 == 0);
    if (!vec4 || E <= 32 || E > 256 || k > 8) return false;
    if (4 * G > 16 * 1024) return false;            // the destination counts of a workgroup live in LDS
    *lanes = rw_lanes(E);
    return true;
}

}  // namespace rs

namespace rs {
// the workspace holds the counts of `splits` slices per pair (one slice needs none)
static bool rt_ws_holds(const void *ws, size_t ws_bytes, int64_t pairs, int64_t splits, int64_t G)
{
    return splits <= 1 || (ws && reinterpret_cast<uintptr_t>(ws) % 4 == 0 && ws_bytes >= sizeof(uint32_t) * (size_t)(pairs * splits * G));
}

static bool rt_may_stay_whole(int64_t tokens_per_gpu, int64_t pairs, int round) { return pairs <= 64 && tokens_per_gpu <= 4 * round; }

// slices per pair, rows of at most 8 logits: one round of tokens per slice while that keeps the slice counts (4*G bytes per slice)
// a small fraction of the logits, more rounds per slice for large G
static int64_t rt_splits(int64_t tokens_per_gpu, int64_t G, int64_t pairs, int E, int k)
{
    const int kRtRound = rt_round(rt_vpl(E));
    const int64_t rounds = (8 * G + kRtRound - 1) / kRtRound;
    const int64_t slice = kRtRound * (rounds < 1 ? 1 : rounds);
    int64_t splits = (tokens_per_gpu + slice - 1) / slice;
    if (splits < 1) splits = 1;
    // Few pairs of few tokens leave the chip idle either way: a workgroup of 1024 threads takes a pair of up to 2048 tokens in one of its
    // rounds and the launch that sums slice counts is saved, as long as the picks of one round are not the longer part (16 GPUs, 8
    // logits, us cut / uncut: 2048 tokens top-2 5.2 / 4.1, top-4 6.5 / 5.7, top-8 8.4 / 10.2; 1024 tokens top-8 8.1 / 6.3).
    if (rt_may_stay_whole(tokens_per_gpu, pairs, kRtRound) && tokens_per_gpu * k <= 8192) return 1;
    while (splits > 1 && pairs * splits > 0x7FFFFFFFll) splits = (splits + 1) / 2;
    return splits;
}

// Slices per pair, rows of 9..32 logits, and the tokens of a slice: one round of 256 threads, more where the slice counts would be more than
// a sixty-fourth of the logits.  Two rounds are one round of 512 threads: a pair that is no longer is not cut, which saves the second kernel.
static int64_t rt_list_splits(int64_t tokens_per_gpu, int64_t G, int E, int64_t *slice_out)
{
    const int round = rt_round(rt_vpl(E));
    const int64_t rounds = (64 * G / E + round - 1) / round;
    const int64_t slice = round * (rounds < 1 ? 1 : rounds);
    const int64_t splits = (tokens_per_gpu + slice - 1) / slice;
    *slice_out = slice;
    return splits < 1 || tokens_per_gpu <= 2 * round ? 1 : splits;
}
}  // namespace rs

extern "C" size_t railsched_route_traffic_workspace_bytes(int32_t batch, int64_t tokens_per_gpu, int32_t E, int32_t k,
                                                          const railsched_topo_t *h_topo)
{
    using namespace rs;
    if (check_topo(h_topo) != RAILSCHED_OK || batch < 0 || tokens_per_gpu < 0 || E < 1 || k < 1) return 0;
    const int64_t G = (int64_t)h_topo->nodes * h_topo->rails;
    const int64_t pairs = (int64_t)batch * G;
    if (E > 8) {
        // the larger of what the one-pass kernel for 33..256 logits and the two-stage path would need
        size_t need = railsched_traffic_matrix_workspace_bytes(batch, tokens_per_gpu, k, h_topo);
        const int rpg = 4 * (64 / rw_lanes(E));
        if (E <= 32 && k <= 8 && pairs > 0) {
            int64_t slice;
            const int64_t splits = rt_list_splits(tokens_per_gpu, G, E, &slice);
            const size_t one = splits > 1 ? align_up(sizeof(uint32_t) * (size_t)(pairs * splits * G), 256) : 256;
            need = one > need ? one : need;
        }
        if (E > 32 && E <= 256 && k <= 8 && pairs > 0 && 4 * G <= 16 * 1024) {
            const int64_t rb = (int64_t)rw_iters(tokens_per_gpu, G, pairs, E, rpg, false) * rpg;
            const int64_t splits = (tokens_per_gpu + rb - 1) / rb;
            const size_t one = splits > 1 ? align_up(sizeof(uint32_t) * (size_t)(pairs * splits * G), 256) : 256;
            need = one > need ? one : need;
        }
        return need;
    }
    if (pairs == 0) return 256;
    const int64_t splits = rt_splits(tokens_per_gpu, G, pairs, E, k);
    return splits > 1 ? align_up(sizeof(uint32_t) * (size_t)(pairs * splits * G), 256) : 256;
}

extern "C" int railsched_route_traffic(const float *logits, int32_t batch, int64_t tokens_per_gpu, int32_t E, int32_t k,
                                       const int32_t *expert_gpu, int32_t R, int64_t payload_bytes,
                                       const railsched_topo_t *h_topo, int32_t *topk_idx, int64_t *D1, void *ws,
                                       size_t ws_bytes, void *stream)
{
    using namespace rs;
    if (int rc = check_topo(h_topo)) return rc;
    if (batch < 0 || tokens_per_gpu < 0 || E < 1 || k < 1 || k > E || R < 1 || payload_bytes < 0) return RAILSCHED_ERR_INVALID_ARG;
    if (E > kMaxExperts) return RAILSCHED_ERR_UNSUPPORTED;
    const int64_t G = (int64_t)h_topo->nodes * h_topo->rails;
    if (tokens_per_gpu > (int64_t(1) << 31) / k) return RAILSCHED_ERR_UNSUPPORTED;   // 32-bit bin counters
    if (batch == 0) return RAILSCHED_OK;
    if (!D1 || !expert_gpu || (!logits && tokens_per_gpu > 0)) return RAILSCHED_ERR_NULL_PTR;
    const int64_t pairs = (int64_t)batch * G;
    const int64_t rows = pairs * tokens_per_gpu;

    int lanes = 0;
    if (E > 8 && rows > 0 && !topk_idx && rw_shape(logits, E, k, G, &lanes)) {
        // the indices are not wanted: one pass (with them, the two stages below are the faster way on this chip)
        RwArgs a;
        a.logits = logits; a.expert_gpu = expert_gpu; a.D1 = D1;
        a.tokens_per_gpu = tokens_per_gpu; a.payload = payload_bytes;
        a.E = E; a.k = k; a.R = R; a.rmask = is_pow2(R) ? R - 1 : -1;
        a.G = (int32_t)G;
        const int rpg = 4 * (64 / lanes);
        auto slices = [&](bool longer) {
            a.iters = rw_iters(tokens_per_gpu, G, pairs, E, rpg, longer);
            const int64_t rb = (int64_t)a.iters * rpg;
            return (tokens_per_gpu + rb - 1) / rb;
        };
        int64_t splits = slices(false);
        if (!rt_ws_holds(ws, ws_bytes, pairs, splits, G)) splits = slices(true);
        if (pairs * splits > 0x7FFFFFFFll) return RAILSCHED_ERR_UNSUPPORTED;
        if (!rt_ws_holds(ws, ws_bytes, pairs, splits, G)) return RAILSCHED_ERR_WORKSPACE;
        a.splits = (int32_t)splits;
        a.partial = static_cast<uint32_t *>(ws);
        a.table_in_lds = ((int64_t)E * R <= kRtTableMax && 4 * (G + (int64_t)E * R) <= 16 * 1024) ? 1 : 0;
        hipStream_t st = static_cast<hipStream_t>(stream);
        int rc;
        if (E <= 64) rc = launch_route_traffic_insert<4, 16, 8, 5>(a, pairs, st);
        else if (E <= 128) rc = launch_route_traffic_insert<8, 16, 6, 6>(a, pairs, st);
        else rc = launch_route_traffic_insert<8, 32, 6, 4>(a, pairs, st);
        if (rc) return rc;
        if (splits > 1) return launch_count_reduce(a.partial, D1, pairs * G, (int)G, (int)splits, payload_bytes, st);
        return RAILSCHED_OK;
    }
    int64_t slice = 0;
    const int64_t list_splits = E > 8 && E <= 32 ? rt_list_splits(tokens_per_gpu, G, E, &slice) : 1;
    // rows of 9..32 logits: one pass when the indices are wanted, k fits the lists, whole float4s load, and the workspace (if any
    // is needed) holds the slice counts.  3.1 M rows, both stages back to back against this: 16 logits top-4 80 -> 50 us, top-2 62 -> 49;
    // 32 logits top-4 145 -> 84, top-8 232 -> 110; 20 logits top-1 85 -> 73.
    const bool list = E > 8 && E <= 32 && k <= 8 && topk_idx && rows > 0 && E % 4 == 0 && reinterpret_cast<uintptr_t>(logits) % 16 == 0 &&
                      pairs * list_splits <= 0x7FFFFFFFll && G <= 8192 && rt_ws_holds(ws, ws_bytes, pairs, list_splits, G);
    if (E > 8 && !list) {
        // other shapes: the two stages run one after the other through the index array
        if (!topk_idx && rows > 0) return RAILSCHED_ERR_NULL_PTR;
        if (int rc = railsched_route_topk(logits, rows, E, k, topk_idx, stream)) return rc;
        return railsched_traffic_matrix(topk_idx, batch, tokens_per_gpu, k, expert_gpu, E, R, payload_bytes, h_topo, D1, ws, ws_bytes, stream);
    }
    hipStream_t st = static_cast<hipStream_t>(stream);

    RtArgs a;
    a.logits = logits; a.expert_gpu = expert_gpu; a.topk_idx = topk_idx; a.D1 = D1;
    a.tokens_per_gpu = tokens_per_gpu; a.payload = payload_bytes;
    a.E = E; a.k = k; a.R = R; a.rmask = is_pow2(R) ? R - 1 : -1;
    a.G = (int32_t)G;
    a.copies = 1;
    while (a.copies < 8 && (int64_t)a.copies * 2 * (G | 1) <= 8192) a.copies *= 2;
    a.lanes_per_period = R <= 64 ? R : 1;                    // a lane holds one token, so rho repeats every R lanes
    a.bin_stride = (int32_t)(a.copies > 1 ? (G | 1) : G);
    a.table_in_lds = ((int64_t)E * R <= kRtTableMax && 4 * (a.copies * (int64_t)a.bin_stride + (int64_t)E * R) <= 64 * 1024) ? 1 : 0;

    const uintptr_t at = reinterpret_cast<uintptr_t>(topk_idx);
    a.wide_idx = at % 16 == 0 ? 16 : at % 8 == 0 ? 8 : 4;
    int64_t splits = list ? list_splits : rt_splits(tokens_per_gpu, G, pairs, E, k);
    // a pair that may stay whole does so for a caller without room for its slices
    if (!list && !rt_ws_holds(ws, ws_bytes, pairs, splits, G) && rt_may_stay_whole(tokens_per_gpu, pairs, rt_round(rt_vpl(E)))) splits = 1;
    if (pairs * splits > 0x7FFFFFFFll) return RAILSCHED_ERR_UNSUPPORTED;
    if (!rt_ws_holds(ws, ws_bytes, pairs, splits, G)) return RAILSCHED_ERR_WORKSPACE;
    a.splits = (int32_t)splits;
    a.partial = static_cast<uint32_t *>(ws);
    const size_t lds = sizeof(unsigned) * (size_t)a.bin_stride * a.copies + (a.table_in_lds ? sizeof(int32_t) * (size_t)E * R : 0);
    const int rc = E <= 4 ? launch_route_traffic<4, 0>(a, pairs, slice, lds, st) : E <= 8 ? launch_route_traffic<8, 0>(a, pairs, slice, lds, st)
                 : E <= 16 ? (k == 1 ? launch_route_traffic<16, 2>(a, pairs, slice, lds, st) : k <= 4 ? launch_route_traffic<16, 5>(a, pairs, slice, lds, st) : launch_route_traffic<16, 9>(a, pairs, slice, lds, st))
                           : (k == 1 ? launch_route_traffic<32, 2>(a, pairs, slice, lds, st) : k <= 4 ? launch_route_traffic<32, 5>(a, pairs, slice, lds, st) : launch_route_traffic<32, 9>(a, pairs, slice, lds, st));
    if (rc) return rc;
    if (splits > 1) return launch_count_reduce(a.partial, D1, pairs * G, (int)G, (int)splits, payload_bytes, st);
    return RAILSCHED_OK;
}
