// Stage 3: flow splitting into fixed-size chunks and the per-node descending sort
// (Section 5.1 "Flow Splitting and Atomicity"; Algorithm 2 steps 1-2).
//
// The sorted order has structure the kernels use instead of sorting every chunk: a flow of B bytes
// gives floor(B/C) chunks of exactly C bytes and at most one tail of B mod C < C bytes.  Under
// "weight descending, ties in canonical order" all full chunks therefore come first, in canonical
// order (their positions follow from an exclusive scan of floor(B/C) over the instance's flows), and
// only the tails - at most one per flow, N*G per instance - need a real sort.  The tails of one
// instance are sorted by one workgroup with a stable LSD radix sort held in LDS (8-bit digits,
// ranks inside a 64-element batch from ballot matching).  Every chunk record is written to HBM
// exactly once.
//
// An instance (matrix b, node k) owns the N consecutive rows k*N..k*N+N-1 of D1[b]; read as one
// array of N*G entries its index is exactly the canonical flow id n*G + dst.
#include "common.h"
#include "chunk_core.h"

namespace rs {

// Record fill.  us of the whole call by 128 / 256 / 512 / 1024 threads a workgroup: 4096 instances, 480 M records of 13 bytes 1147 / 1118 / 1122 / 1100..1150, one
// matrix of 3.9 G records of 9 bytes 5820 / 5510 / 5400 / 5450.  Neighbouring tiles on one XCD: a bare writer of 13 bytes a record with one read in front of its stores
// 5.6 TB/s when tiles go round robin over the XCDs, 5.8 / 6.0 / 6.1 when an XCD has 64 / 128 / 512 KiB of an array in a row.
constexpr int kFillThreads = 512;
constexpr int kFillGranule = 7;     // log2 of the neighbouring tiles that the workgroups of one XCD write: 1 MiB of an array
constexpr int64_t kFillTiles = 1 << 22;   // most tiles of one launch: 2^31 threads

// ---- A: per-instance chunk counts and the two exclusive scans over its flows -----------------
// One workgroup of T threads per instance, T * kTailLoads flows per round.  Latency bound (a few dependent trips to memory and
// barriers): with one wavefront per instance the 4096 flows of a 512-GPU instance took 31 us, 7 now.
template <int T>
__global__ __launch_bounds__(T) void cs_count_kernel(CsArgs a)
{
    constexpr int W = T / 64, U = kTailLoads;
    static_assert(U * W <= 64, "one lane per (round, wavefront)");
    __shared__ unsigned sh_q[64], sh_c[64];
    __shared__ int64_t sh_n[W];
    const int inst = blockIdx.x;
    const int b = inst / a.M, k = inst % a.M;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t *rows = a.D1 + ((int64_t)b * a.G + (int64_t)k * a.N) * a.G;
    uint32_t *fs = a.full_start + (int64_t)inst * a.NF;
    uint16_t *tb = a.tails_before + (int64_t)inst * a.NF;
    const unsigned long long lt = (1ull << lane) - 1ull;
    unsigned carry_q = 0, carry_c = 0;
    int64_t n_full = 0;
    for (int f0 = 0; f0 < a.NF; f0 += U * T) {
        int64_t bytes[U];                           // all of a round's loads in flight before the scans, which chain
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int f = f0 + u * T + tid;
            bytes[u] = f < a.NF ? flow_bytes(a, rows, k, f) : 0;
        }
        unsigned eq[U], ec[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            uint32_t q = 0, r = 0;
            split_bytes(a, bytes[u], q, r);
            unsigned tq;
            eq[u] = wave_exscan(q, tq);
            const unsigned long long tails = __ballot(r != 0);
            const unsigned tc = (unsigned)__popcll(tails);
            ec[u] = (unsigned)__popcll(tails & lt);
            if constexpr (W == 1) {                 // a wavefront by itself carries its totals along
                const int f = f0 + u * T + tid;
                if (f < a.NF) { fs[f] = carry_q + eq[u]; tb[f] = (uint16_t)(carry_c + ec[u]); }
                carry_q += tq; carry_c += tc;
            } else if (lane == 0) {
                sh_q[u * W + wave] = tq; sh_c[u * W + wave] = tc;
            }
            n_full += q;
        }
        if constexpr (W == 1) continue;
        __syncthreads();
        unsigned total_q, total_c;
        const unsigned bq = wave_exscan(lane < U * W ? sh_q[lane] : 0u, total_q);
        const unsigned bc = wave_exscan(lane < U * W ? sh_c[lane] : 0u, total_c);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int f = f0 + u * T + tid;
            const unsigned oq = carry_q + (unsigned)__shfl((int)bq, u * W + wave) + eq[u];
            const unsigned oc = carry_c + (unsigned)__shfl((int)bc, u * W + wave) + ec[u];
            if (f < a.NF) { fs[f] = oq; tb[f] = (uint16_t)oc; }
        }
        carry_q += total_q; carry_c += total_c;
        __syncthreads();                            // the totals have been read
    }
    // exact 64-bit total
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) n_full += __shfl_xor(n_full, d);
    if constexpr (W > 1) {
        if (lane == 0) sh_n[wave] = n_full;
        __syncthreads();
    }
    if (tid == 0) {
        for (int w = 1; w < W; ++w) n_full += sh_n[w];
        a.cnt_all[inst] = n_full + carry_c; a.cnt_full[inst] = n_full;
        if (a.run_end) a.run_end[(int64_t)inst * a.N] = n_full;
    }
}

// Threads per instance of the flow kernels (count, tail sort): four flows each up to 256 flows; then as many as shorten the one
// instance a CU has, or, with more than four instances per CU, as few as let them overlap (tail sort of 4096 instances of
// 2048 flows: 57 us with one wavefront, 37 with 256 threads, 106 with 1024; 3904 of 4096: 364, 157, 213)
static int flow_threads(int64_t n_inst, int64_t NF)
{
    if (NF <= 256) return 64;
    if (NF <= 1024 || n_inst > 1024) return 256;
    return 1024;
}

// ---- B: chunk_off = exclusive scan of instance sizes --------------------------------------------
__global__ __launch_bounds__(1024) void cs_scan_kernel(CsArgs a)
{
    constexpr int PER = 4;                            // consecutive instances per thread and round
    __shared__ int64_t sh_a[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int64_t carry = 0;                                // the same in every thread
    for (int base = 0; base < a.n_inst; base += 1024 * PER) {
        int64_t va[PER], sa = 0;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int i = base + tid * PER + u;
            va[u] = i < a.n_inst ? a.cnt_all[i] : 0;
            sa += va[u];
        }
        int64_t ia = sa;                              // inclusive scan of the thread sums inside the wavefront
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int64_t xa = __shfl_up(ia, d);
            if (lane >= d) ia += xa;
        }
        __syncthreads();                              // the round before is done with sh_a
        if (lane == 63) sh_a[wave] = ia;
        __syncthreads();
        int64_t before = 0, total = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const int64_t xa = sh_a[w];
            if (w < wave) before += xa;
            total += xa;
        }
        int64_t oa = carry + before + ia - sa;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int i = base + tid * PER + u;
            if (i < a.n_inst) a.chunk_off[i] = oa;
            oa += va[u];
        }
        carry += total;
    }
    if (tid == 0) a.chunk_off[a.n_inst] = carry;
}

// ---- C: tails of one instance: stable descending radix sort in LDS, one workgroup per instance; beside it the entries of the fill ----
// Every 2^s-th record's instance and flow (NF where it is a tail), for the fill's wavefronts to start from: the smallest s from kEntryShift on for which
// the room behind the workspace's other arrays is enough (two bytes a flow, so about four flows lie between two entries at most, on average).
// One for every wavefront of the fill where there is room: 61 layers of 512 GPUs, 220 M records, 933 us the call with an entry every 256 records, 952 with
// one every 512, 975 every 1024 (the scan from an entry to the window is as long as the window's own).
constexpr int kEntryShift = 8;
__host__ __device__ __forceinline__ int fill_entry_shift(int64_t total, int64_t n_entries)
{
    int s = kEntryShift;
    while (((total - 1) >> s) >= n_entries) ++s;
    return s;
}

// Entries u .. u + 63, one per lane.  The first and the last lane's instance and flow are searched for by the whole wavefront, the others' by
// each lane between the two (a lane by itself from the start: a dozen dependent trips to memory).
__device__ __forceinline__ void fill_entries(const CsArgs &a, int64_t u)
{
    const int lane = threadIdx.x & 63;
    const int64_t total = a.chunk_off[a.n_inst];
    if (total > a.capacity || total == 0) return;
    const int s = fill_entry_shift(total, a.n_entries);
    const int64_t end = (total - 1) >> s;                                // last entry
    if (u > end) return;
    const int64_t u_last = u + 63 < end ? u + 63 : end;
    const int i_lo = wave_last_le<int64_t>(a.chunk_off, a.n_inst, u << s), i_hi = wave_last_le<int64_t>(a.chunk_off, a.n_inst, u_last << s);
    const int64_t mine = u + lane < u_last ? u + lane : u_last;          // lanes behind the last entry repeat it
    const int inst = i_lo + (i_hi > i_lo ? last_le<int64_t>(a.chunk_off + i_lo, i_hi - i_lo + 1, mine << s) : 0);
    const int64_t p = (mine << s) - a.chunk_off[inst];
    const bool full = p < a.cnt_full[inst];
    const uint32_t *fs = a.full_start + (int64_t)inst * a.NF;
    int j_lo = 0, j_hi = a.NF - 1;
    if (i_lo == i_hi) {                                                  // flow starts ascend: all lanes' flows lie between these two
        const uint32_t p0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p), p1 = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)p, 63);
        j_lo = wave_last_le<uint32_t>(fs, a.NF, p0);
        j_hi = wave_last_le<uint32_t>(fs, a.NF, p1);
    }
    const int j = full ? j_lo + last_le<uint32_t>(fs + j_lo, j_hi - j_lo + 1, (uint32_t)p) : a.NF;
    a.entries[mine] = make_uint2((unsigned)inst, (unsigned)j);
}

template <int T>
__global__ __launch_bounds__(T) void cs_tail_kernel(CsArgs a, unsigned entry_blocks)
{
    extern __shared__ __align__(16) unsigned cs_lds[];
    __shared__ unsigned sh[kTailShared];
    if (blockIdx.x < entry_blocks) {
        fill_entries(a, ((int64_t)blockIdx.x * T + threadIdx.x) & ~(int64_t)63);
        return;
    }
    unsigned *hist = cs_lds;                                             // [tail_hist_words<T>()], read 16 bytes at a time
    unsigned *rem = hist + tail_hist_words<T>();                         // [NF] tail bytes per flow
    unsigned short *idx_a = reinterpret_cast<unsigned short *>(rem + a.NF);    // [NF] flow ids, ping
    unsigned short *idx_b = idx_a + a.NF;                                      // [NF] pong
    if (a.chunk_off[a.n_inst] > a.capacity) return;                      // record arrays too small: leave them alone

    const int inst = (int)(blockIdx.x - entry_blocks);
    const int b = inst / a.M, k = inst % a.M;
    const int64_t *rows = a.D1 + ((int64_t)b * a.G + (int64_t)k * a.N) * a.G;

    int nt = 0;
    const unsigned short *sorted = tail_sort_block<T, T == 64>(a, rows, k, rem, hist, idx_a, idx_b, sh, nt, [] {});

    const uint32_t n_full = (uint32_t)a.cnt_full[inst];
    const int64_t out0 = a.chunk_off[inst] + a.cnt_full[inst];
    const uint32_t *fs = a.full_start + (int64_t)inst * a.NF;
    const uint16_t *tb = a.tails_before + (int64_t)inst * a.NF;
    constexpr int U = 4;                                                 // the flows' starts are fetched for four tails at a time
    for (int i0 = threadIdx.x; i0 < nt; i0 += U * T) {
        int f[U];
        uint32_t pm[U];
#pragma unroll
        for (int u = 0; u < U; ++u) f[u] = i0 + u * T < nt ? sorted[i0 + u * T] : sorted[i0];
        if (a.perm) {
            // the tail is its flow's last chunk: the full chunks up to the next flow and the tails before it come first
#pragma unroll
            for (int u = 0; u < U; ++u) pm[u] = (f[u] + 1 < a.NF ? fs[f[u] + 1] : n_full) + tb[f[u]];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * T;
            if (i >= nt) break;
            a.chunk_w[out0 + i] = rem[f[u]];
            a.chunk_flow[out0 + i] = (uint32_t)f[u];
            if (a.perm) a.perm[out0 + i] = pm[u];
        }
    }
}

template <int T>
static int launch_cs_tail(const CsArgs &a, hipStream_t st)
{
    const size_t lds = sizeof(unsigned) * (size_t)(a.NF + tail_hist_words<T>()) + 2 * sizeof(unsigned short) * (size_t)a.NF;
    if (lds > 48 * 1024) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(cs_tail_kernel<T>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds) != hipSuccess)
            return RAILSCHED_ERR_HIP;
    }
    int64_t entries = (a.capacity >> kEntryShift) + 1;
    entries = entries < a.n_entries ? entries : a.n_entries;
    const unsigned entry_blocks = (unsigned)((entries + T - 1) / T);
    hipLaunchKernelGGL(cs_tail_kernel<T>, dim3(entry_blocks + (unsigned)a.n_inst), dim3(T), lds, st, a, entry_blocks);
    return launch_status();
}

// ---- D: full chunks ---------------------------------------------------------------------------
// Write bound: 9 to 13 bytes a record.  A workgroup writes one tile of 4 T records at a multiple of that and exits, a wavefront its own kilobyte of
// every array, on a 1 KiB boundary, with streaming stores.  What a writer reaches of the chip's 6.9 TB/s hangs on how many bytes wait behind
// how long a chain of reads, and on what lies side by side in time: bare writers of 13 bytes a record, TB/s: no reads 6.1, two dependent trips in front
// of the stores 5.2, the same with neighbouring tiles on one XCD 5.5, with streaming stores too 6.0; two and four tiles a workgroup are
// slower throughout (5.2, 5.1).  So a wavefront makes two trips (its entry; then its instance's bounds and the flow starts from the entry's flow on), no
// barrier, and finds the flows of its records from the starts that fall among them, as window_flows does.
// Measured, as contiguous runs of tiles per workgroup with their flow starts staged in LDS / now: 4096 instances of 117 K records 1295 / 990 us (4.8 / 6.3 TB/s),
// one matrix of 3.9 G records without perm 6720 / 5310 (5.3 / 6.7), 3904 instances of 57 K in flows of 14: 611 / 500.
template <int T>
__global__ __launch_bounds__(T) void cs_fill_kernel(CsArgs a, int vec_ok, int kshift, int64_t tile0)
{
    constexpr int kWindow = 256;
    __shared__ __align__(16) unsigned marks[T / 64][kWindow];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const unsigned b = blockIdx.x;
    const int64_t tile = tile0 + ((int64_t)(b >> (3 + kshift)) << (3 + kshift)) + ((b & 7u) << kshift) + ((b >> 3) & ((1u << kshift) - 1u));
    const int64_t w0 = tile * (T * 4) + wave * kWindow;                  // this wavefront's first record
    const int64_t total = a.chunk_off[a.n_inst];
    if (total > a.capacity || w0 >= total) return;
    const uint2 entry = a.entries[w0 >> fill_entry_shift(total, a.n_entries)];
    int inst = __builtin_amdgcn_readfirstlane((int)entry.x), j0 = __builtin_amdgcn_readfirstlane((int)entry.y);
    unsigned *mark = marks[wave];
    const uint32_t cw = (uint32_t)a.C;

    int64_t out0 = a.chunk_off[inst], out1 = a.chunk_off[inst + 1];
    while (out1 <= w0) {                                                 // the entry lies before the window, in another instance
        const int i = inst + 1 + lane < a.n_inst ? inst + 1 + lane : a.n_inst;
        inst += __popcll(__ballot(a.chunk_off[i] <= w0));                // chunk_off[n_inst] = total > w0
        j0 = 0;
        out0 = a.chunk_off[inst]; out1 = a.chunk_off[inst + 1];
    }
    while (true) {                                                       // the instances that have records in the window: one, but where one ends
        const uint32_t n_full = (uint32_t)a.cnt_full[inst];
        const int64_t first = w0 - out0;                                 // instance position of the window's first record; negative where the instance starts in it
        if (n_full != 0 && first < (int64_t)n_full) {
            const uint32_t last = first + kWindow <= (int64_t)n_full ? (uint32_t)(first + kWindow - 1) : n_full - 1u;
            const uint32_t *fs = a.full_start + (int64_t)inst * a.NF;
            const uint16_t *tb = a.tails_before + (int64_t)inst * a.NF;
            *reinterpret_cast<uint4 *>(mark + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
            lds_sync();
            unsigned base = 0;                                           // flow << 16 | tails before it: both ascend together
            for (int f = j0 + lane;; f += 64) {
                const bool is = f < a.NF;
                const uint32_t s = is ? fs[f] : 0xFFFFFFFFu;
                const unsigned v = (unsigned)f << 16 | (is ? (unsigned)tb[f] : 0u);
                const bool in = s <= last, before = in && (int64_t)s <= first;
                const int n = __popcll(__ballot(before));
                if (n) base = (unsigned)__builtin_amdgcn_readlane((int)v, n - 1);
                if (in && !before) atomicMax(&mark[(uint32_t)((int64_t)s - first)], v);
                if (__ballot(!in) != 0ull) break;
            }
            lds_sync();
            const uint4 m = *reinterpret_cast<const uint4 *>(mark + 4 * lane);
            const unsigned m1 = max(m.x, m.y), m2 = max(m1, m.z), m3 = max(m2, m.w);
            const unsigned left = wave_max_before(max(m3, base), base);
            const unsigned v[4] = {max(left, m.x), max(left, m1), max(left, m2), max(left, m3)};
            const int64_t p = first + 4 * lane;
            const uint32_t lead = n_full - n_full % (uint32_t)a.N;       // positions below it go round robin (a.rail)
            const int64_t at = w0 + 4 * lane;
            uint32_t rr = 0;
            if (a.rail) {
                uint32_t r = a.nmask >= 0 ? ((uint32_t)p & (uint32_t)a.nmask) : (uint32_t)p % (uint32_t)a.N;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    rr |= r << (8 * e);
                    r = (r + 1 == (uint32_t)a.N) ? 0u : r + 1;
                }
            }
            if (vec_ok && p >= 0 && p + 4 <= (int64_t)n_full) {
                const uint32_t q = (uint32_t)p;
                __builtin_nontemporal_store(u32x4{cw, cw, cw, cw}, reinterpret_cast<u32x4 *>(a.chunk_w + at));
                __builtin_nontemporal_store(u32x4{v[0] >> 16, v[1] >> 16, v[2] >> 16, v[3] >> 16}, reinterpret_cast<u32x4 *>(a.chunk_flow + at));
                if (a.perm)
                    __builtin_nontemporal_store(u32x4{q + (v[0] & 0xFFFFu), q + 1 + (v[1] & 0xFFFFu), q + 2 + (v[2] & 0xFFFFu), q + 3 + (v[3] & 0xFFFFu)},
                                                reinterpret_cast<u32x4 *>(a.perm + at));
                if (a.rail) {
                    if (q + 4 <= lead) {
                        __builtin_nontemporal_store(rr, reinterpret_cast<uint32_t *>(a.rail + at));
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) if (q + e < lead) a.rail[at + e] = (uint8_t)(rr >> (8 * e));
                    }
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (p + e < 0 || p + e >= (int64_t)n_full) continue;
                    const uint32_t q = (uint32_t)(p + e);
                    a.chunk_w[at + e] = cw;
                    a.chunk_flow[at + e] = v[e] >> 16;
                    if (a.perm) a.perm[at + e] = q + (v[e] & 0xFFFFu);
                    if (a.rail && q < lead) a.rail[at + e] = (uint8_t)(q % (uint32_t)a.N);
                }
            }
        }
        if (out1 >= w0 + kWindow || out1 >= total) return;
        do { ++inst; out0 = out1; out1 = a.chunk_off[inst + 1]; } while (out1 == out0);
        j0 = 0;
    }
}

static void ws_layout(int64_t n_inst, int64_t NF, size_t off[6])
{
    const size_t flows = (size_t)(n_inst * NF);
    size_t o = 0;
    off[0] = o; o += align_up(sizeof(int64_t) * (size_t)n_inst, 256);          // cnt_all
    off[1] = o; o += align_up(sizeof(int64_t) * (size_t)n_inst, 256);          // cnt_full
    off[2] = o; o += align_up(sizeof(uint32_t) * flows, 256);                  // full_start
    off[3] = o; o += align_up(sizeof(uint16_t) * flows, 256);                  // tails_before
    off[4] = o;                                                                // entries of the fill: two bytes a flow and 8 an instance, 256 or more
    off[5] = off[2] + align_up(sizeof(int64_t) * (size_t)(n_inst + 1), 256) + 2 * align_up(sizeof(uint32_t) * flows, 256);
}

// pointers into the workspace, and what the kernels derive from the topology
static void fill_args(CsArgs &a, const railsched_topo_t *h_topo, int64_t n_inst, void *ws)
{
    const int64_t M = h_topo->nodes, N = h_topo->rails, G = M * N, NF = N * G;
    size_t off[6];
    ws_layout(n_inst, NF, off);
    char *w8 = static_cast<char *>(ws);
    a.cnt_all = reinterpret_cast<int64_t *>(w8 + off[0]);
    a.cnt_full = reinterpret_cast<int64_t *>(w8 + off[1]);
    a.full_start = reinterpret_cast<uint32_t *>(w8 + off[2]);
    a.tails_before = reinterpret_cast<uint16_t *>(w8 + off[3]);
    a.entries = reinterpret_cast<uint2 *>(w8 + off[4]);
    a.n_entries = (int64_t)((off[5] - off[4]) / sizeof(uint2));
    a.C = h_topo->chunk_bytes;
    a.cshift = is_pow2(a.C) ? ilog2(a.C) : -1;
    a.M = (int32_t)M; a.N = (int32_t)N; a.G = (int32_t)G; a.NF = (int32_t)NF; a.intra = h_topo->include_intra_node;
    a.n_inst = (int32_t)n_inst;
    a.nmask = is_pow2(N) ? (int32_t)N - 1 : -1;
    a.gmask = is_pow2(G) ? (int32_t)G - 1 : -1;
    a.nshift = is_pow2(N) ? ilog2(N) : -1;
}

// entry points for the one-call scheduler (schedule.hip)
void cs_fill_args(CsArgs &a, const railsched_topo_t *h_topo, int64_t n_inst, void *ws) { fill_args(a, h_topo, n_inst, ws); }
void launch_cs_count(const CsArgs &a, hipStream_t st)
{
    const int T = flow_threads(a.n_inst, a.NF);
    const dim3 grid((unsigned)a.n_inst);
    if (T == 64) hipLaunchKernelGGL(cs_count_kernel<64>, grid, dim3(64), 0, st, a);
    else if (T == 256) hipLaunchKernelGGL(cs_count_kernel<256>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(cs_count_kernel<1024>, grid, dim3(1024), 0, st, a);
}

}  // namespace rs

extern "C" size_t railsched_chunk_sort_workspace_bytes(int32_t batch, const railsched_topo_t *h_topo)
{
    using namespace rs;
    if (check_topo(h_topo) != RAILSCHED_OK || batch < 0) return 0;
    const int64_t G = (int64_t)h_topo->nodes * h_topo->rails;
    size_t off[6];
    ws_layout((int64_t)batch * h_topo->nodes, (int64_t)h_topo->rails * G, off);
    return off[5] ? off[5] : 256;
}

namespace rs {
int cs_run(const int64_t *D1, int32_t batch, const railsched_topo_t *h_topo, int64_t *chunk_off, uint32_t *chunk_w,
           uint32_t *chunk_flow, uint32_t *perm, int64_t capacity, uint8_t *rail, int64_t *run_end, void *ws, size_t ws_bytes,
           hipStream_t st, CsArgs *args_out)
{
    if (int rc = check_topo(h_topo)) return rc;
    if (batch < 0 || capacity < 0) return RAILSCHED_ERR_INVALID_ARG;
    const int64_t M = h_topo->nodes, N = h_topo->rails, G = M * N, NF = N * G;
    if (NF > kMaxFlows) return RAILSCHED_ERR_UNSUPPORTED;
    const int64_t n_inst = (int64_t)batch * M;
    if (n_inst > 0x7FFFFFFFll) return RAILSCHED_ERR_UNSUPPORTED;
    if (!chunk_off) return RAILSCHED_ERR_NULL_PTR;
    if (n_inst > 0 && !D1) return RAILSCHED_ERR_NULL_PTR;
    if (chunk_w && !chunk_flow) return RAILSCHED_ERR_NULL_PTR;
    size_t off[6];
    ws_layout(n_inst, NF, off);
    if (!ws || ws_bytes < off[5] || reinterpret_cast<uintptr_t>(ws) % 256) return RAILSCHED_ERR_WORKSPACE;
    CsArgs a;
    a.D1 = D1; a.chunk_off = chunk_off; a.chunk_w = chunk_w; a.chunk_flow = chunk_flow; a.perm = perm;
    a.capacity = capacity;
    a.rail = rail;
    a.run_end = run_end;
    fill_args(a, h_topo, n_inst, ws);
    if (args_out) *args_out = a;

    if (n_inst > 0) {
        launch_cs_count(a, st);
        if (int rc = launch_status()) return rc;
    }
    hipLaunchKernelGGL(cs_scan_kernel, dim3(1), dim3(1024), 0, st, a);
    if (int rc = launch_status()) return rc;
    if (!chunk_w || n_inst == 0) return RAILSCHED_OK;

    const int T = flow_threads(n_inst, NF);
    if (int rc = T == 64 ? launch_cs_tail<64>(a, st) : T == 256 ? launch_cs_tail<256>(a, st) : launch_cs_tail<1024>(a, st)) return rc;
    const int vec_ok = (reinterpret_cast<uintptr_t>(chunk_w) % 16 == 0 && reinterpret_cast<uintptr_t>(chunk_flow) % 16 == 0 &&
                        reinterpret_cast<uintptr_t>(perm) % 16 == 0 && reinterpret_cast<uintptr_t>(rail) % 4 == 0) ? 1 : 0;
    int kshift = 0;
    const int64_t tiles = (capacity + kFillThreads * 4 - 1) / (kFillThreads * 4);
    while (kshift < kFillGranule && (tiles >> (kshift + 6)) > 0) ++kshift;
    const int64_t group = (int64_t)8 << kshift;
    for (int64_t tile0 = 0; tile0 < tiles; tile0 += kFillTiles) {
        const int64_t n = tiles - tile0 < kFillTiles ? tiles - tile0 : kFillTiles;
        hipLaunchKernelGGL(cs_fill_kernel<kFillThreads>, dim3((unsigned)((n + group - 1) / group * group)), dim3(kFillThreads), 0, st, a, vec_ok, kshift, tile0);
    }
    return launch_status();
}
}  // namespace rs

extern "C" int railsched_chunk_sort(const int64_t *D1, int32_t batch, const railsched_topo_t *h_topo,
                                    int64_t *chunk_off, uint32_t *chunk_w, uint32_t *chunk_flow, uint32_t *perm,
                                    int64_t capacity, void *ws, size_t ws_bytes, void *stream)
{
    return rs::cs_run(D1, batch, h_topo, chunk_off, chunk_w, chunk_flow, perm, capacity, nullptr, nullptr, ws, ws_bytes,
                      static_cast<hipStream_t>(stream), nullptr);
}
