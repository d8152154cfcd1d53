// Device-side pieces of stage 3 (Section 5.1 "Flow Splitting and Atomicity"; Algorithm 2 steps 1-2) shared by
// the stage-3 kernels and by the one-call scheduler of small batches.
#pragma once

#include "common.h"

namespace rs {

struct CsArgs {
    const int64_t *D1;
    int64_t *chunk_off;
    uint32_t *chunk_w, *chunk_flow, *perm;
    int64_t capacity;
    int64_t *cnt_all, *cnt_full;
    uint32_t *full_start;        // [n_inst][NF] full chunks of the instance before flow f
    uint16_t *tails_before;      // [n_inst][NF] tails before flow f (at most NF <= 16384); canonical start of the flow = the two together
    uint2 *entries;              // [n_entries] (instance, flow) at every 2^s-th record, where the record fill starts its searches (fill_entry_shift)
    int64_t n_entries;           // 0: none, the fill searches
    unsigned *tickets;           // when set, the counters that the fill's last workgroups draw further tiles on
    int64_t *sums;               // when set, [workgroups of the scan] chunks of the instances of each
    int64_t C;
    uint64_t cinv;       // (2^64 - 1) / C
    uint32_t ginv;       // 2^32 / G, rounded up (G > 1)
    int32_t cshift;      // >= 0 when C is a power of two
    int32_t M, N, G, NF, intra;
    int32_t n_inst;
    int32_t nmask;       // N - 1 when N is a power of two, else -1
    uint8_t *rail;       // when set, the fill also writes the rails of every instance's leading run (see cs_fill_kernel)
    int32_t gmask, nshift;   // G - 1 and log2 N when G / N are powers of two, else -1
    int64_t *clear;      // when set, the counts' kernel clears clear[inst * N ..  + N - 1] (the receive loads that the instances then add to)
    int64_t *run_end;    // when set, run_end[inst * N] receives the length of every instance's leading run of full chunks
};

__device__ __forceinline__ void split_bytes(const CsArgs &a, int64_t B, uint32_t &q, uint32_t &r)
{
    if (B < 0) B = 0;
    if (a.cshift >= 0) {
        q = (uint32_t)(B >> a.cshift);
        r = (uint32_t)(B & (a.C - 1));
    } else {
        const uint64_t qq = (uint64_t)B / (uint64_t)a.C;
        q = (uint32_t)qq;
        r = (uint32_t)((uint64_t)B - qq * (uint64_t)a.C);
    }
}

// bytes of flow f of instance (b, k); 0 for destinations inside node k unless intra-node traffic is kept
__device__ __forceinline__ int64_t flow_bytes(const CsArgs &a, const int64_t *rows, int k, int f)
{
    if (!a.intra) {
        const int node = (a.gmask >= 0 && a.nshift >= 0) ? ((f & a.gmask) >> a.nshift) : (f % a.G) / a.N;   // of the destination
        if (node == k) return 0;
    }
    return rows[f];
}

// The flows f0, f0 + step, ... (V of them) of instance (b, k), 0 behind the last flow and for destinations inside node k unless intra-node traffic is kept.
// Without branches, so that all loads are in flight together: what does not count is read and dropped.
template <int V>
__device__ __forceinline__ void load_flows(const CsArgs &a, const int64_t *rows, int k, int f0, int step, int64_t (&bytes)[V])
{
#pragma unroll
    for (int j = 0; j < V; ++j) {
        const int f = f0 + step * j;
        bytes[j] = rows[f < a.NF ? f : a.NF - 1];
    }
#pragma unroll
    for (int j = 0; j < V; ++j) {
        const unsigned f = (unsigned)(f0 + step * j);
        // f / G by the reciprocal is exact: f and G are at most 2^14, so what rounding up adds stays below one part in G
        const unsigned dst = f - (a.G > 1 ? __umulhi(f, a.ginv) : f) * (unsigned)a.G;
        const bool inside = !a.intra && dst - (unsigned)(k * a.N) < (unsigned)a.N;
        bytes[j] = (int)f < a.NF && !inside ? bytes[j] : 0;
    }
}

template <int V>
__device__ __forceinline__ void split_flows(const CsArgs &a, const int64_t (&bytes)[V], uint32_t (&q)[V], uint32_t (&r)[V])
{
    if (a.cshift >= 0) {
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const int64_t B = bytes[j] < 0 ? 0 : bytes[j];
            q[j] = (uint32_t)(B >> a.cshift);
            r[j] = (uint32_t)B & (uint32_t)(a.C - 1);
        }
    } else {
#pragma unroll
        for (int j = 0; j < V; ++j) {
            // with the reciprocal rounded down the quotient comes out right or one too small
            const uint64_t B = bytes[j] < 0 ? 0 : (uint64_t)bytes[j];
            uint64_t qq = __umul64hi(B, a.cinv);
            uint64_t rr = B - qq * (uint64_t)a.C;
            if (rr >= (uint64_t)a.C) { rr -= (uint64_t)a.C; ++qq; }
            q[j] = (uint32_t)qq;
            r[j] = (uint32_t)rr;
        }
    }
}

// v of the lane the DPP control points at, 0 where there is none (or where row_mask switches the row off)
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ unsigned dpp_or_zero(unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, false);
}

// Exclusive prefix sum over the 64 lanes (and the total), all in the vector ALU: four shifted adds inside the
// rows of 16 lanes, then lane 15 of rows 0 and 2 into rows 1 and 3, then lane 31 into rows 2 and 3.
__device__ __forceinline__ unsigned wave_exscan(unsigned v, unsigned &total)
{
    unsigned inc = v;
    inc += dpp_or_zero<0x111, 0xF>(inc);            // row_shr:1
    inc += dpp_or_zero<0x112, 0xF>(inc);            // row_shr:2
    inc += dpp_or_zero<0x114, 0xF>(inc);            // row_shr:4
    inc += dpp_or_zero<0x118, 0xF>(inc);            // row_shr:8
    inc += dpp_or_zero<0x142, 0xA>(inc);            // row_bcast15 into rows 1 and 3
    inc += dpp_or_zero<0x143, 0xC>(inc);            // row_bcast31 into rows 2 and 3
    total = (unsigned)__builtin_amdgcn_readlane((int)inc, 63);
    return inc - v;
}

// Ordering point between LDS accesses of the lanes of ONE wavefront, whatever the others of the workgroup are at: waiting
// for the wavefront's own LDS operations is enough (LDS executes a wavefront's operations in order) and
// the asm statement keeps the compiler from moving LDS accesses across it.
__device__ __forceinline__ void lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Maximum over the lanes before the caller's, and `first` (a lower bound of all) for lane 0.
__device__ __forceinline__ unsigned wave_max_before(unsigned inc, unsigned first)
{
    inc = max(inc, (unsigned)__builtin_amdgcn_update_dpp(0, (int)inc, 0x111, 0xF, 0xF, false));   // row_shr:1
    inc = max(inc, (unsigned)__builtin_amdgcn_update_dpp(0, (int)inc, 0x112, 0xF, 0xF, false));   // row_shr:2
    inc = max(inc, (unsigned)__builtin_amdgcn_update_dpp(0, (int)inc, 0x114, 0xF, 0xF, false));   // row_shr:4
    inc = max(inc, (unsigned)__builtin_amdgcn_update_dpp(0, (int)inc, 0x118, 0xF, 0xF, false));   // row_shr:8
    inc = max(inc, (unsigned)__builtin_amdgcn_update_dpp(0, (int)inc, 0x142, 0xA, 0xF, false));   // row_bcast15 into rows 1 and 3
    inc = max(inc, (unsigned)__builtin_amdgcn_update_dpp(0, (int)inc, 0x143, 0xC, 0xF, false));   // row_bcast31 into rows 2 and 3
    return (unsigned)__builtin_amdgcn_update_dpp((int)first, (int)inc, 0x138, 0xF, 0xF, false);   // wave_shr:1; lane 0 keeps `first`
}

// Flows of the 256 positions first .. first + 255, four per lane, for a wavefront that knows the flow j_lo of position `first` or of one
// before it (the same in all lanes): every flow that starts in the window, or between j_lo and it, leaves its number where it
// starts (the largest wins: the ones before it are empty) and a running maximum carries them on.  No search: a window costs a few
// LDS round trips whatever the flows' lengths.  mark[256] is this wavefront's scratch, 16-byte aligned.  Positions beyond `last` (of
// the last lanes) get the flow of `last`.  Returns the flow of `last`.
__device__ __forceinline__ int window_flows(const uint32_t *fs, int nf, int j_lo, uint32_t first, uint32_t last, unsigned *mark, uint32_t (&fl)[4])
{
    const int lane = threadIdx.x & 63;
    *reinterpret_cast<uint4 *>(mark + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
    lds_sync();
    for (int f = j_lo + 1 + lane;; f += 64) {
        const uint32_t s = f < nf ? fs[f] : 0xFFFFFFFFu;
        const bool in = s <= last;
        if (in) atomicMax(&mark[s > first ? s - first : 0u], (unsigned)f);
        if (__ballot(!in) != 0ull) break;           // starts ascend: nothing further on starts at or before `last`
    }
    lds_sync();
    const uint4 m = *reinterpret_cast<const uint4 *>(mark + 4 * lane);
    const unsigned m1 = max(m.x, m.y), m2 = max(m1, m.z), m3 = max(m2, m.w);
    const unsigned left = wave_max_before(max(m3, (unsigned)j_lo), (unsigned)j_lo);
    fl[0] = max(left, m.x); fl[1] = max(left, m1); fl[2] = max(left, m2); fl[3] = max(left, m3);
    return __builtin_amdgcn_readlane((int)fl[3], 63);
}

constexpr int kTailLoads = 4;       // flows per thread and round of the flow scans: their loads are in flight together

// LDS words tail_sort_block needs beside rem[NF], hist[] and the two index arrays
template <int T> constexpr int tail_hist_words() { return 256 * (T / 64); }
constexpr int kTailShared = 64 + 2 + 16;
// Tails whose places are counted (one pass over the others in LDS, no histogram) instead of sorted for: what a wavefront by itself counts in one
// round, or a quarter of a thousand for several.  Flows up to which even the empty ones are counted along, without gathering the tails first.
// One wavefront each, 3840 instances of 256 tails of 16 differing bits: 56 us counted, 16 sorted.
// Workgroups, whole schedule, us along / gathered first: 4 instances of 64 flows 13.9 / 14.4, 80 of 64 16.8 / 17.6; 20 of 128, all tails 17.1 / 16.7, a third of them
// 16.9 / 14.9; 600 of 256, a third 25.3 / 19.7.
template <int T> constexpr int rank_tails() { return T == 64 ? 64 : 256; }
template <int T> constexpr int rank_flows() { return T == 64 ? 96 : 64; }

// Tails (B mod C > 0) of the flows of one instance, sorted by weight descending, ties in canonical (flow) order:
// stable LSD radix sort by one workgroup of T threads in LDS, 8-bit digits over the span of key bits that differ at all.
// A wavefront owns a contiguous share of the order and a histogram of its own, so ranks inside a share need no workgroup
// barrier (ballot matching in batches of 64); a pass has four.  rem[NF] receives every flow's tail bytes,
// hist[tail_hist_words<T>()] and sh[kTailShared] are scratch, idx_a/idx_b[NF] are ping-pong arrays of flow ids; returns the
// array that holds the sorted ids and their number in nt.  Latency bound: one wavefront took 32 us for the 4096 flows of a
// 512-GPU instance, a workgroup of 1024 takes 6.  Callers: the one-call scheduler's instances, and in stage 3 those of up to 256 flows and of more than 8192.
// stage() is called once with the first flows' loads in flight, for what the caller has to fetch as well.
template <int T, typename F>
__device__ __forceinline__ unsigned short *tail_sort_block(const CsArgs &a, const int64_t *rows, int k, unsigned *rem, unsigned *hist,
                                                           unsigned short *idx_a, unsigned short *idx_b, unsigned *sh, int &nt_out, F stage)
{
    constexpr int W = T / 64, U = kTailLoads;
    static_assert(U * W <= 64, "one lane per (round, wavefront)");
    unsigned *sh_cnt = sh, *sh_bits = sh + 64, *sh_tot = sh + 66;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned long long lt = (1ull << lane) - 1ull;
    int nt = 0;
    if (a.NF <= rank_flows<T>()) {
        // few flows: a tail's place is the number of tails that go before it, counted over all flows by the P neighbouring threads of its own
        constexpr int R = T == 64 ? 2 : 1, P = T >= 512 ? T / 256 : 1;   // rounds of loads, threads per flow
        const int quads = (a.NF + 3) >> 2;
        int64_t bytes[R];
#pragma unroll
        for (int u = 0; u < R; ++u) bytes[u] = u * T + tid < a.NF ? flow_bytes(a, rows, k, u * T + tid) : 0;
        stage();
        unsigned tails = 0;
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int f = u * T + tid;
            uint32_t q = 0, r = 0;
            split_bytes(a, bytes[u], q, r);
            if (f < 4 * quads) rem[f] = r;                               // nothing behind the last flow: zeros
            tails += (unsigned)__popcll(__ballot(r != 0));
        }
        if (lane == 0) sh_cnt[wave] = tails;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < (W < 4 ? W : 4); ++w) nt += (int)sh_cnt[w];  // 256 flows are in four wavefronts
        for (int base = 0; base < a.NF; base += T / P) {
            const int f = base + tid / P;
            const unsigned w = f < a.NF ? rem[f] : 0u;
            unsigned rank = 0;
            if (w)
                for (int g = tid % P; g < quads; g += P) {
                    const uint4 o = *reinterpret_cast<const uint4 *>(rem + 4 * g);
                    const int j = 4 * g;
                    rank += (o.x > w || (o.x == w && j + 0 < f)) ? 1u : 0u;
                    rank += (o.y > w || (o.y == w && j + 1 < f)) ? 1u : 0u;
                    rank += (o.z > w || (o.z == w && j + 2 < f)) ? 1u : 0u;
                    rank += (o.w > w || (o.w == w && j + 3 < f)) ? 1u : 0u;
                }
#pragma unroll
            for (int d = 1; d < P; d <<= 1) rank += (unsigned)__shfl_xor((int)rank, d);
            if (w && tid % P == 0) idx_b[rank] = (unsigned short)f;
        }
        __syncthreads();
        nt_out = nt;
        return idx_b;
    }
    if (tid == 0) { sh_bits[0] = 0u; sh_bits[1] = 0xFFFFFFFFu; }
    // tails in canonical order; which key bits differ at all between them
    unsigned any1 = 0u, all1 = 0xFFFFFFFFu;
    for (int f0 = 0; f0 < a.NF; f0 += U * T) {
        int64_t bytes[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int f = f0 + u * T + tid;
            bytes[u] = f < a.NF ? flow_bytes(a, rows, k, f) : 0;
        }
        if (f0 == 0) stage();
        unsigned r[U];
        unsigned long long m[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int f = f0 + u * T + tid;
            uint32_t q = 0;
            split_bytes(a, bytes[u], q, r[u]);
            if (f < a.NF) rem[f] = r[u];
            m[u] = __ballot(r[u] != 0);
            if (r[u]) { any1 |= r[u]; all1 &= r[u]; }
            if (lane == 0) sh_cnt[u * W + wave] = (unsigned)__popcll(m[u]);
        }
        __syncthreads();
        unsigned total;
        const unsigned before = wave_exscan(lane < U * W ? sh_cnt[lane] : 0u, total);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned at = (unsigned)nt + (unsigned)__shfl((int)before, u * W + wave);
            if (r[u]) idx_a[at + __popcll(m[u] & lt)] = (unsigned short)(f0 + u * T + tid);
        }
        nt += (int)total;
        __syncthreads();                            // sh_cnt has been read
    }
    nt_out = nt;
    if (nt <= rank_tails<T>()) {
        // few tails: a tail's place is the number of tails that go before it.  Keys side by side in hist, read four at a time;
        // with T / 256 threads per tail each counts a share of them.
        constexpr int P = T >= 256 ? T / 256 : 1, STEP = T >= 256 ? 256 : T;
        const int quads = (nt + 3) >> 2;
        for (int i = tid; i < 4 * quads; i += T) hist[i] = i < nt ? rem[idx_a[i]] : 0u;   // a tail is at least one byte
        if constexpr (P > 1) { if (tid < 256) hist[256 + tid] = 0u; }
        __syncthreads();
        const int part = tid / 256;
        for (int i = tid % 256; i < nt; i += STEP) {
            const unsigned w = hist[i];
            unsigned rank = 0;
            for (int g = part; g < quads; g += P) {
                const uint4 o = *reinterpret_cast<const uint4 *>(hist + 4 * g);
                const int j = 4 * g;
                rank += (o.x > w || (o.x == w && j + 0 < i)) ? 1u : 0u;
                rank += (o.y > w || (o.y == w && j + 1 < i)) ? 1u : 0u;
                rank += (o.z > w || (o.z == w && j + 2 < i)) ? 1u : 0u;
                rank += (o.w > w || (o.w == w && j + 3 < i)) ? 1u : 0u;
            }
            if constexpr (P > 1) atomicAdd(&hist[256 + i], rank);
            else idx_b[rank] = idx_a[i];
        }
        __syncthreads();
        if constexpr (P > 1) {
            if (tid < nt) idx_b[hist[256 + tid]] = idx_a[tid];
            __syncthreads();
        }
        return idx_b;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) { any1 |= (unsigned)__shfl_xor((int)any1, d); all1 &= (unsigned)__shfl_xor((int)all1, d); }
    if (lane == 0) { atomicOr(&sh_bits[0], any1); atomicAnd(&sh_bits[1], all1); }
    __syncthreads();
    // bits that are equal in every key cannot change the order: sort on the span of differing bits only
    // (token payloads make tails multiples of some power of two, so the span is usually one digit wide)
    const unsigned diff = sh_bits[0] ^ sh_bits[1];
    const int lo_bit = diff ? __ffs((int)diff) - 1 : 0;
    const int n_pass = (nt > 1 && diff) ? (32 - __clz((int)diff) - lo_bit + 7) / 8 : 0;
    const int share = ((nt + W - 1) / W + 63) & ~63;                     // of one wavefront, whole batches
    const int i_lo = wave * share, i_hi = i_lo + share < nt ? i_lo + share : nt;
    unsigned *mine = hist + wave * 256;

    for (int pass = 0; pass < n_pass; ++pass) {
        const int shift = lo_bit + 8 * pass;
        for (int i = lane; i < 256; i += 64) mine[i] = 0;
        lds_sync();
        for (int i = i_lo + lane; i < i_hi; i += 64) atomicAdd(&mine[255u - ((rem[idx_a[i]] >> shift) & 255u)], 1u);
        __syncthreads();
        {   // exclusive scan over (digit, wavefront): four consecutive entries per thread
            unsigned h[4], sum = 0, tot;
#pragma unroll
            for (int j = 0; j < 4; ++j) { const int e = 4 * tid + j; h[j] = hist[(e % W) * 256 + e / W]; sum += h[j]; }
            unsigned ex = wave_exscan(sum, tot);
            if (lane == 0) sh_tot[wave] = tot;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < W; ++w) ex += w < wave ? sh_tot[w] : 0u;
#pragma unroll
            for (int j = 0; j < 4; ++j) { const int e = 4 * tid + j; hist[(e % W) * 256 + e / W] = ex; ex += h[j]; }
        }
        __syncthreads();
        for (int i0 = i_lo; i0 < i_hi; i0 += 64) {                       // batches in order keep the sort stable
            const int i = i0 + lane;
            const bool act = i < i_hi;
            const unsigned short f = act ? idx_a[i] : 0;
            const unsigned d = act ? 255u - ((rem[f] >> shift) & 255u) : 0u;
            unsigned long long peers = __ballot(act);
#pragma unroll
            for (int bit = 0; bit < 8; ++bit) {
                const bool one = (d >> bit) & 1u;
                const unsigned long long bm = __ballot(act && one);
                peers &= one ? bm : ~bm;
            }
            const unsigned base = act ? mine[d] : 0u;
            if (act) idx_b[base + __popcll(peers & lt)] = f;
            lds_sync();
            if (act && (peers >> lane) == 1ull) mine[d] = base + __popcll(peers);   // highest lane of the peer set
            lds_sync();
        }
        __syncthreads();
        unsigned short *t = idx_a; idx_a = idx_b; idx_b = t;
    }

    return idx_a;
}

// Host side of stage 3, shared by railsched_chunk_sort and the one-call scheduler (defined in chunk_sort.hip):
// validates, lays the workspace out and launches count, scan, tail sort and fill.  With `rail` set the fill also
// writes rail[i] = i mod N for the first n_full - n_full mod N positions of every instance - the greedy
// allocation of a leading run of equal weights from empty rails (Algorithm 2 step 3) in closed form.
// run_end, if given, receives those runs' lengths n_full at run_end[inst * N], where stage 4's serial kernels look for them.
// *args_out, if given, receives the argument block (workspace pointers included).
int cs_run(const int64_t *D1, int32_t batch, const railsched_topo_t *h_topo, int64_t *chunk_off, uint32_t *chunk_w,
           uint32_t *chunk_flow, uint32_t *perm, int64_t capacity, uint8_t *rail, int64_t *run_end, void *ws, size_t ws_bytes, hipStream_t st,
           CsArgs *args_out);

}  // namespace rs
