// Stage 3: flow splitting into fixed-size chunks and the per-node descending sort
// (Section 5.1 "Flow Splitting and Atomicity"; Algorithm 2 steps 1-2).
//
// The sorted order has structure the kernels use instead of sorting every chunk: a flow of B bytes
// gives floor(B/C) chunks of exactly C bytes and at most one tail of B mod C < C bytes.  Under
// "weight descending, ties in canonical order" all full chunks therefore come first, in canonical
// order (their positions follow from an exclusive scan of floor(B/C) over the instance's flows), and
// only the tails - at most one per flow, N*G per instance - need a real sort.  The tails of one
// instance are sorted by one workgroup with a stable LSD radix sort, held in registers up to 8192 flows (8-bit digits,
// ranks inside a 64-element batch from ballot matching).  Every chunk record is written to HBM
// exactly once.
//
// An instance (matrix b, node k) owns the N consecutive rows k*N..k*N+N-1 of D1[b]; read as one
// array of N*G entries its index is exactly the canonical flow id n*G + dst.
#include "common.h"
#include "chunk_core.h"

namespace rs {

// Record fill.  us of the whole call by 128 / 256 / 512 / 1024 threads a workgroup (a workgroup's room is free when its last wavefront is done, and a window in a stretch
// of flows without full chunks takes long): 61 layers of 512 GPUs, 220 M records 955 / 788 / 815 / -, as routed 1.1 Zipf - / 730 / 805 / -; 4096 instances, 480 M records 1147 / 1118 / 1122 /
// 1100..1150, one matrix of 3.9 G records 5820 / 5510 / 5400 / 5450 (boxes and placements differ by 8 %).  Neighbouring tiles on one XCD: a bare writer of 13 bytes
// a record with one read in front of its stores 5.6 TB/s when tiles go round robin over the XCDs, 5.8 / 6.0 / 6.05 when an XCD has 256 / 512 / 1024 KiB of an array in a row.
constexpr int kFillThreads = 256;
constexpr int kFillWindow = 256;    // records of one wavefront
constexpr int kFillTile = kFillThreads / 64 * kFillWindow;
constexpr int kFillGranule = 8;     // log2 of the neighbouring tiles that the workgroups of one XCD write: 1 MiB of an array
// Workgroups of the launch: a tile each for all records there is room for, because a wavefront that exits behind its stores is what writes fastest, up to a limit, because one that finds
// nothing to do costs 0.21 ns (the chip starts a wavefront every 0.053 ns) and the host does not know how much of the room is used.  The limit is 2^15 (7 us in all, what the other
// launches of a call cost) and one more for every 16 flows, 13 ps a flow beside the 10 to 25 that the rest of the call takes (for every 32, the fill of 3.86 G records of 32 768 instances
// of 2048 flows took 10.4 ms for 9.2).  What lies behind it goes to the last workgroups
// by tickets, so that what is being written stays close together: to as many as the chip holds, or half of them with perm, whose larger records fill the way to memory with fewer
// (1024 / 2048, with perm 3.6 G records of 1024 GPUs 7050 / 7560, without 6400 / 4875).  us, chunk_sort, all tiles launched / 2^15 and tickets / 2^15 workgroups that go
// round: 226 M records of 512 GPUs 597 / 626 / 640, 489 M of 256 GPUs 1045 / 1087 / 1200, 3.7 G of 1024 GPUs without perm 4620 / 5040 / 5500; the other way round, 8.6 M records of
// 64 GPUs and room for 8.6 M / 430 M / 3.4 G 33 / 117 / 740 when all tiles are launched, 33 / 37 / 37 so.  The 5 to 18 % stay however the rest is cut: tickets of two and four tiles, 8 to
// 64 counters, the next tile's instance fetched ahead, flow starts through the scalar cache, two windows side by side, waves of 2 to 64 windows launched for all of them.
constexpr int64_t kFillTiles = 1 << 15, kFillTileFlows = 16, kFillTilesMost = 1 << 22;   // 2^22: the launch stays within 2^30 threads
constexpr unsigned kFillRounds = 2048, kFillRoundsPerm = 1024;
// Counters of tickets and the words from one to the next, a cache line.  A line takes 16 ns an addition: eight counters 7.4 ms for the 3.7 G records.  A batch of few flows has no room for
// them; all its workgroups go round.
constexpr int kFillCounters = 16, kTicketStep = 32;
constexpr int kFillInstWaves = 1 << 18;   // most wavefronts that look for instances of few full chunks

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
    if (a.clear && tid < a.N) a.clear[(int64_t)inst * a.N + tid] = 0;
    for (int f0 = 0; f0 < a.NF; f0 += U * T) {
        int64_t bytes[U];                           // all of a round's loads in flight before the scans, which chain
        uint32_t qs[U], rs[U];
        load_flows<U>(a, rows, k, f0 + tid, T, bytes);
        split_flows<U>(a, bytes, qs, rs);
        unsigned eq[U], ec[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t q = qs[u], r = rs[u];
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

// Threads per instance of the count: four flows each up to 256 flows; then as many as shorten the one instance a CU has, or, with more
// than four instances per CU, as few as let them overlap.
static int flow_threads(int64_t n_inst, int64_t NF)
{
    if (NF <= 256) return 64;
    if (NF <= 1024 || n_inst > 1024) return 256;
    return 1024;
}

// ---- B: chunk_off = exclusive scan of instance sizes; the entries of the record fill ----
// Entries: instance and flow (NF where it is a tail) of every 2^s-th record, for the fill's wavefronts to start from: the smallest s from kEntryShift on
// for which the room behind the workspace's other arrays is enough (two bytes a flow, so about four flows lie between two entries at most, on average).
// One for every wavefront of the fill where there is room: 61 layers of 512 GPUs, 220 M records, 933 us the call with an entry every 256 records, 952 with
// one every 512, 975 every 1024 (the scan from an entry to the window is as long as the window's own).
constexpr int kEntryShift = 8;
constexpr int kSearchFlows = 1024;  // flows of an instance, and
constexpr int64_t kSearchRecords = 1 << 21;   // room for records, up to which there are no entries
constexpr int kSmallFlows = 256;    // flows of an instance that one wavefront sorts the tails of
__host__ __device__ __forceinline__ int fill_entry_shift(int64_t total, int64_t n_entries)
{
    int s = kEntryShift;
    while (((total - 1) >> s) >= n_entries) ++s;
    return s;
}

// The entries that fall among the full chunks of an instance's flows: mostly none or one a flow, more than a few by the whole wavefront.
template <typename P, int T>
__device__ __forceinline__ void flow_entries(const CsArgs &a, int inst, uint32_t n_full, int64_t out0, int s, int tid)
{
    constexpr int U = 8;                            // flows per thread whose starts are in flight together
    const int lane = tid & 63;
    const P up = ((P)1 << s) - 1, off = (P)out0 & up;
    uint2 *entries = a.entries + (out0 >> s);
    const uint32_t *fs = a.full_start + (int64_t)inst * a.NF;
    for (int f0 = 0; f0 < a.NF; f0 += U * T) {
        uint32_t lo[U], hi[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int f = f0 + u * T + tid;
            lo[u] = f < a.NF ? fs[f] : n_full;
            hi[u] = f + 1 < a.NF ? fs[f + 1] : n_full;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned flow = (unsigned)(f0 + u * T + tid);
            P e = (off + lo[u] + up) >> s;
            const P end = lo[u] < hi[u] ? ((off + hi[u] - 1) >> s) + 1 : e;
            if (e < end) entries[e] = make_uint2((unsigned)inst, flow);
            if (__ballot(end - e > 1) == 0ull) continue;
            unsigned long long many = __ballot(end - e > 5);
            if (end - e <= 5)
                for (++e; e < end; ++e) entries[e] = make_uint2((unsigned)inst, flow);
            while (many) {
                const int l = __builtin_ctzll(many);
                many &= many - 1;
                const P from = __shfl(e, l), to = __shfl(end, l);
                const unsigned of = (unsigned)__shfl((int)flow, l);
                for (P x = from + 1 + lane; x < to; x += 64) entries[x] = make_uint2((unsigned)inst, of);
            }
        }
    }
}

// All entries of one instance, by T threads, of which the caller is number tid.
template <int T>
__device__ __forceinline__ void instance_entries(const CsArgs &a, int inst, int64_t out0, int64_t n_all, int64_t n_full, int s, int tid)
{
    if (n_all == 0) return;
    if (n_full >> 32) {                             // more than an instance may have: flow starts do not fit, but every entry names an instance
        for (int64_t e = ((out0 - 1) >> s) + 1 + tid; (e << s) < out0 + n_all; e += T) a.entries[e] = make_uint2((unsigned)inst, 0u);
        return;
    }
    // in 32 bits where positions, counted from the entry before the instance's first record, fit
    if (s < 31 && n_full < (int64_t)1 << 31) flow_entries<uint32_t, T>(a, inst, (uint32_t)n_full, out0, s, tid);
    else flow_entries<uint64_t, T>(a, inst, (uint32_t)n_full, out0, s, tid);
    for (int64_t e = ((out0 + n_full - 1) >> s) + 1 + tid; (e << s) < out0 + n_all; e += T)   // among its tails
        a.entries[e] = make_uint2((unsigned)inst, (unsigned)a.NF);
}

// Every workgroup takes a few consecutive instances and adds up all counts by itself, or, of more than kScanAlone instances, the sums that a launch before left,
// one for the instances of each workgroup: what all workgroups read together grows with workgroups times instances otherwise.  us, count query alone / whole call, by
// counts / by sums: 16 000 instances of 2 flows 16.7 / 17.5 and 31.0 / 31.5, 32 000 27 / 23 and 48 / 45, 131 072 165 / 60 and 260 / 155, 1 M 1249 / 359 and 1657 / 764, 4.2 M of
// 64 flows 5170 / 1530 and 11 000 / 7520.  A workgroup writes its instances' offsets and entries, those of instances of few flows by a wavefront each: 16 000 instances of 64 flows
// 18 us by a wavefront, 36 by all threads (20 by one workgroup without entries); 3904 of 4096 flows 40 and 26.
constexpr int kScanThreads = 256, kScanBlocks = 2048;
constexpr int64_t kScanAlone = 16384;   // at least kScanBlocks: the sums lie where entries of 8 bytes an instance would

// the instances of workgroup b of the scan: first(b) .. first(b + 1) - 1
__device__ __forceinline__ int scan_first(const CsArgs &a, unsigned b) { return (int)((int64_t)a.n_inst * b / gridDim.x); }

__global__ __launch_bounds__(kScanThreads) void cs_sums_kernel(CsArgs a)
{
    constexpr int W = kScanThreads / 64;
    __shared__ int64_t sh[W];
    const int tid = threadIdx.x, i1 = scan_first(a, blockIdx.x + 1);
    int64_t sum = 0;
#pragma unroll 4
    for (int i = scan_first(a, blockIdx.x) + tid; i < i1; i += kScanThreads) sum += a.cnt_all[i];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d);
    if ((tid & 63) == 0) sh[tid >> 6] = sum;
    __syncthreads();
    if (tid != 0) return;
    for (int w = 1; w < W; ++w) sum += sh[w];
    a.sums[blockIdx.x] = sum;
}

__global__ __launch_bounds__(kScanThreads) void cs_scan_kernel(CsArgs a)
{
    constexpr int W = kScanThreads / 64, U = 16;
    __shared__ int64_t sh[2][W];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i0 = scan_first(a, blockIdx.x), i1 = scan_first(a, blockIdx.x + 1);
    // the counts of its instances, 64 at a time; the first ones are on their way while all are added up
    auto count = [&](const int64_t *of, int base) { return base + lane < i1 ? of[base + lane] : 0; };
    int64_t n_all = count(a.cnt_all, i0), n_full = count(a.cnt_full, i0);
    int64_t before = 0, total = 0;
    const int64_t *of = a.sums ? a.sums : a.cnt_all;
    const int n = a.sums ? (int)gridDim.x : a.n_inst, n0 = a.sums ? (int)blockIdx.x : i0;
    for (int base = 0; base < n; base += U * kScanThreads) {
        int64_t c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = base + u * kScanThreads + tid;
            c[u] = of[i < n ? i : n - 1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = base + u * kScanThreads + tid;
            total += i < n ? c[u] : 0;
            before += i < n0 ? c[u] : 0;
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) { before += __shfl_xor(before, d); total += __shfl_xor(total, d); }
    if (lane == 0) { sh[0][wave] = before; sh[1][wave] = total; }
    __syncthreads();
    before = 0; total = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) { before += sh[0][w]; total += sh[1][w]; }
    if (blockIdx.x == gridDim.x - 1 && tid == 0) a.chunk_off[a.n_inst] = total;
    if (a.tickets && blockIdx.x == 0 && tid < kFillCounters) a.tickets[tid * kTicketStep] = 0u;
    const bool entries = a.n_entries != 0 && total <= a.capacity && total > 0;
    const int s = entries ? fill_entry_shift(total, a.n_entries) : 0;
    for (int base = i0; base < i1; base += 64) {                         // the same in every wavefront
        if (base > i0) { n_all = count(a.cnt_all, base); n_full = count(a.cnt_full, base); }
        int64_t inc = n_all;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int64_t o = __shfl_up(inc, d);
            if (lane >= d) inc += o;
        }
        const int64_t out0 = before + inc - n_all;
        if (wave == 0 && base + lane < i1) a.chunk_off[base + lane] = out0;
        before += __shfl(inc, 63);
        if (!entries) continue;
        if (a.NF <= kSmallFlows)
            for (int l = wave; l < 64 && base + l < i1; l += W)
                instance_entries<64>(a, base + l, __shfl(out0, l), __shfl(n_all, l), __shfl(n_full, l), s, lane);
        else
            for (int l = 0; l < 64 && base + l < i1; ++l)
                instance_entries<kScanThreads>(a, base + l, __shfl(out0, l), __shfl(n_all, l), __shfl(n_full, l), s, tid);
    }
}

// ---- C: tails of one instance: stable descending radix sort, one workgroup per instance ----
// Up to kRegisterFlows flows: T threads, V flows per thread, which stay in its registers: a wavefront owns 64 V consecutive flows, 64 at a time.  A pass
// (8 bits of the key; nearly always the only one, since tails are multiples of the token payload and only the span of bits that
// differ at all counts) ranks a wavefront's elements among its own by ballots, batch after batch, the count of a digit so far in LDS; the scan of the
// counts over (digit, wavefront) makes that the place; then the elements change places through LDS, one word each, keys first, then flows, at last
// the canonical positions, which are read in flow order.  LDS is four bytes a flow and a kilobyte a wavefront: twice the
// workgroups on a CU of a sort that keeps flow ids and tail bytes in LDS, and no gathers from memory.
template <int T> constexpr size_t tail_lds(int64_t NF) { return sizeof(unsigned) * (size_t)(NF + 4 + 256 * (T / 64)); }

// at[j] = place of element j (key[j], act bit) among all active elements by bits shift .. shift + bits - 1 of the keys, descending, stable.  `mine` is this
// wavefront's histogram, hist all of them; the wavefront has elements in its first `batches` batches only.
template <int T, int V>
__device__ __forceinline__ void tail_places(const unsigned (&key)[V], const bool (&act)[V], unsigned (&at)[V], int batches, int shift, int bits, unsigned *hist,
                                            unsigned *sh_tot)
{
    constexpr int W = T / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned long long lt = (1ull << lane) - 1ull;
    unsigned *mine = hist + wave * 256;
    *reinterpret_cast<uint4 *>(mine + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int j = 0; j < V; ++j) {                                        // batches in order keep the sort stable
        if (j >= batches) break;
        const unsigned d = 255u - ((key[j] >> shift) & 255u);
        unsigned long long peers = __ballot(act[j]);
        for (int bit = 0; bit < bits; bit += 2) {   // one bit too many changes nothing: it is the same in all keys
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                const bool one = (d >> (bit + o)) & 1u;
                const unsigned long long bm = __ballot(one), x = one ? 0ull : ~0ull;
                peers &= bm ^ x;
            }
        }
        asm volatile("" ::: "memory");              // LDS executes a wavefront's accesses in order
        const unsigned before = mine[d];
        at[j] = before + (unsigned)__popcll(peers & lt);
        if (act[j] && (peers >> lane) == 1ull) mine[d] = before + (unsigned)__popcll(peers);   // highest lane of the peer set
        __builtin_amdgcn_sched_barrier(0);          // the batches' masks would take twice the registers side by side
    }
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
    asm volatile("" : "+s"(shift));                 // the digits anew: kept from above they and their addresses would take V registers more
#pragma unroll
    for (int j = 0; j < V; ++j) if (j < batches) at[j] += mine[255u - ((key[j] >> shift) & 255u)];
}

// Bits that differ at all between the tails of a workgroup, from every thread's any1 and all1; one barrier.
template <int T>
__device__ __forceinline__ unsigned tail_bits(unsigned any1, unsigned all1, unsigned *sh_bits)
{
    constexpr int W = T / 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) { any1 |= (unsigned)__shfl_xor((int)any1, d); all1 &= (unsigned)__shfl_xor((int)all1, d); }
    if (lane == 0) { sh_bits[wave] = any1; sh_bits[W + wave] = all1; }
    __syncthreads();
    any1 = 0u; all1 = 0xFFFFFFFFu;
#pragma unroll
    for (int w = 0; w < W; ++w) { any1 |= sh_bits[w]; all1 &= sh_bits[W + w]; }
    return (unsigned)__builtin_amdgcn_readfirstlane((int)(any1 ^ all1));
}

// Tails whose places are counted, one pass over the others in LDS, instead of sorted for (4000 instances of 224 tails of 512 flows 51 us counted, 35 sorted).
template <int T> constexpr int few_tails() { return T >= 512 ? 256 : 128; }

// The tails of an instance at most half of whose flows have one: brought together in LDS (where to is what tails_before says), then counted or sorted.
template <int T, int V>
__device__ __forceinline__ void write_few_tails(const CsArgs &a, int inst, int nt, int64_t n_full, const int64_t *rows, int k, unsigned *lds, unsigned *sh)
{
    constexpr int W = T / 64, C = (V + 1) / 2;
    unsigned *hist = lds, *stage = lds + 256 * W, *ids = stage + ((a.NF + 1) / 2 + 3) / 4 * 4;
    unsigned *sh_bits = sh, *sh_tot = sh + 2 * W;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t out0 = a.chunk_off[inst] + n_full;
    const uint32_t *fs = a.full_start + (int64_t)inst * a.NF;
    const uint16_t *tb = a.tails_before + (int64_t)inst * a.NF;
    unsigned any1 = 0u, all1 = 0xFFFFFFFFu;
    {
        int64_t bytes[V];
        uint32_t q[V], r[V];
        unsigned to[V];
#pragma unroll
        for (int j = 0; j < V; ++j) { const int f = j * T + tid; to[j] = tb[f < a.NF ? f : a.NF - 1]; }
        load_flows<V>(a, rows, k, tid, T, bytes);
        split_flows<V>(a, bytes, q, r);
#pragma unroll
        for (int j = 0; j < V; ++j) {
            if (r[j] == 0) continue;
            stage[to[j]] = r[j];
            ids[to[j]] = (unsigned)(j * T + tid);
            any1 |= r[j]; all1 &= r[j];
        }
    }
    auto put = [&](int64_t i, unsigned w, unsigned f) {
        a.chunk_w[i] = w;
        a.chunk_flow[i] = f;
        if (a.perm) a.perm[i] = ((int)f + 1 < a.NF ? fs[f + 1] : (uint32_t)n_full) + tb[f];
    };
    if (nt <= few_tails<T>()) {
        constexpr int P = T >= 1024 ? 4 : T >= 512 ? 2 : 1;              // threads a tail
        const int quads = (nt + 3) >> 2, i = tid / P;
        if (tid < 4 * quads - nt) stage[nt + tid] = 0u;                  // behind the last: a tail is at least one byte
        __syncthreads();
        const unsigned w = i < nt ? stage[i] : 0u;
        unsigned rank = 0;
        if (w)
            for (int g = tid % P; g < quads; g += P) {
                const uint4 o = *reinterpret_cast<const uint4 *>(stage + 4 * g);
                const int j = 4 * g;
                rank += (o.x > w || (o.x == w && j + 0 < i)) ? 1u : 0u;
                rank += (o.y > w || (o.y == w && j + 1 < i)) ? 1u : 0u;
                rank += (o.z > w || (o.z == w && j + 2 < i)) ? 1u : 0u;
                rank += (o.w > w || (o.w == w && j + 3 < i)) ? 1u : 0u;
            }
#pragma unroll
        for (int d = 1; d < P; d <<= 1) rank += (unsigned)__shfl_xor((int)rank, d);
        if (w && tid % P == 0) put(out0 + rank, w, ids[i]);
        return;
    }
    const unsigned diff = tail_bits<T>(any1, all1, sh_bits);
    const int lo_bit = diff ? __builtin_ctz(diff) : 0;
    const int span = diff ? 32 - __builtin_clz(diff) - lo_bit : 0;
    const int share = (nt + 64 * W - 1) / (64 * W), i0 = wave * 64 * share + lane;   // batches of a wavefront
    unsigned key[C], id[C], at[C];
    bool act[C];
    auto take = [&] {
#pragma unroll
        for (int j = 0; j < C; ++j) {
            const int i = i0 + 64 * j;
            act[j] = j < share && i < nt;
            key[j] = act[j] ? stage[i] : 0u;
            id[j] = act[j] ? ids[i] : 0u;
        }
        __syncthreads();
    };
    take();
    for (int done = 0; done < span; done += 8) {
        tail_places<T, C>(key, act, at, share, lo_bit + done, span - done < 8 ? span - done : 8, hist, sh_tot);
#pragma unroll
        for (int j = 0; j < C; ++j) if (act[j]) { stage[at[j]] = key[j]; ids[at[j]] = id[j]; }
        __syncthreads();
        take();
    }
#pragma unroll
    for (int j = 0; j < C; ++j) if (act[j]) put(out0 + i0 + 64 * j, key[j], id[j]);
}

template <int T, int V>
__device__ __forceinline__ void write_tails(const CsArgs &a, int inst, unsigned *lds, unsigned *sh)
{
    constexpr int W = T / 64;
    unsigned *hist = lds, *stage = lds + 256 * W;
    unsigned *sh_bits = sh, *sh_tot = sh + 2 * W;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = inst / a.M, k = inst % a.M;
    const int64_t *rows = a.D1 + ((int64_t)b * a.G + (int64_t)k * a.N) * a.G;
    const int64_t n_full = a.cnt_full[inst];
    const int nt = (int)(a.cnt_all[inst] - n_full);
    if (nt == 0) return;
    if (2 * nt <= a.NF) {
        write_few_tails<T, V>(a, inst, nt, n_full, rows, k, lds, sh);
        return;
    }
    const int64_t out0 = a.chunk_off[inst] + n_full;
    const uint32_t *fs = a.full_start + (int64_t)inst * a.NF;
    const uint16_t *tb = a.tails_before + (int64_t)inst * a.NF;
    const int i0 = wave * 64 * V + lane;            // this thread's elements: i0, i0 + 64, ...
    const int batches = (a.NF - wave * 64 * V + 63) / 64;   // of this wavefront, V and more: all
    unsigned key[V], at[V];
    bool act[V];
    unsigned any1 = 0u, all1 = 0xFFFFFFFFu;         // which key bits differ at all
    {
        int64_t bytes[V];
        uint32_t q[V];
        load_flows<V>(a, rows, k, i0, 64, bytes);
        split_flows<V>(a, bytes, q, key);
#pragma unroll
        for (int j = 0; j < V; ++j) {
            act[j] = key[j] != 0u;
            any1 |= key[j];
            all1 &= act[j] ? key[j] : 0xFFFFFFFFu;
        }
    }
    const unsigned diff = tail_bits<T>(any1, all1, sh_bits);
    const int lo_bit = diff ? __builtin_ctz(diff) : 0;
    const int span = diff ? 32 - __builtin_clz(diff) - lo_bit : 0;
    tail_places<T, V>(key, act, at, batches, lo_bit, span < 8 ? span : 8, hist, sh_tot);
    // a tail is its flow's last chunk: the full chunks up to the next flow and the tails before it come first
    if (span <= 8) {
        auto through = [&](auto value, uint32_t *to) {
#pragma unroll
            for (int j = 0; j < V; ++j) if (act[j]) stage[at[j]] = value(j);
            __syncthreads();
#pragma unroll
            for (int j = 0; j < V; ++j) if (i0 + 64 * j < nt) to[out0 + i0 + 64 * j] = stage[i0 + 64 * j];
        };
        through([&](int j) { return key[j]; }, a.chunk_w);
        uint32_t pm[V];
        if (a.perm) {
#pragma unroll
            for (int j = 0; j < V; ++j) {
                const int f = i0 + 64 * j;
                pm[j] = act[j] ? (f + 1 < a.NF ? fs[f + 1] : (uint32_t)n_full) + tb[f] : 0u;
            }
        }
        __syncthreads();
        through([&](int j) { return (unsigned)(i0 + 64 * j); }, a.chunk_flow);
        if (a.perm) {
            __syncthreads();
            through([&](int j) { return pm[j]; }, a.perm);
        }
        return;
    }
    unsigned id[V];
#pragma unroll
    for (int j = 0; j < V; ++j) id[j] = (unsigned)(i0 + 64 * j);
    for (int done = 8;; done += 8) {
        // the elements in the order of the bits so far, then the next ones
        auto swap = [&](unsigned (&x)[V]) {
#pragma unroll
            for (int j = 0; j < V; ++j) if (act[j]) stage[at[j]] = x[j];
            __syncthreads();
#pragma unroll
            for (int j = 0; j < V; ++j) if (i0 + 64 * j < nt) x[j] = stage[i0 + 64 * j];
            __syncthreads();
        };
        swap(key);
        swap(id);
        if (done >= span) break;
#pragma unroll
        for (int j = 0; j < V; ++j) act[j] = i0 + 64 * j < nt;           // flows without a tail have left
        tail_places<T, V>(key, act, at, (nt - wave * 64 * V + 63) / 64, lo_bit + done, span - done < 8 ? span - done : 8, hist, sh_tot);
    }
#pragma unroll
    for (int j = 0; j < V; ++j) {
        const int64_t i = out0 + i0 + 64 * j;
        if (i0 + 64 * j >= nt) continue;
        a.chunk_w[i] = key[j];
        a.chunk_flow[i] = id[j];
        if (a.perm) a.perm[i] = ((int)id[j] + 1 < a.NF ? fs[id[j] + 1] : (uint32_t)n_full) + tb[id[j]];
    }
}

// V = 4 fits 64 registers, that is eight wavefronts on a SIMD.  us, 3904 instances of 4096 flows, 3074 tails of 64 values: by 256 threads with ids and tail bytes in LDS
// 159, eight flows a thread 152, four 104 (its traffic 57); whole stage, LDS / registers: all tails of 16 bits, 4000 instances of 1024 flows 66 / 55, 3600 of 2700 136 / 136,
// 3904 of 4096 247 / 206, 3600 of 7680 666 / 504, 850 of 5440 123 / 108; a tenth of them 48 / 36, 88 / 88, 117 / 120, 367 / 251, 75 / 62; 30 in a thousand
// 40 / 31, 75 / 65, 112 / 88, 367 / 200, 62 / 50 (45, 143, 164, 356, 93 when all flows went through the passes).  3600 instances of 2700 flows and 1700 of 1088 of which half have tails
// are what loses: 113 / 122, 37 / 40.
template <int T, int V>
__global__ __launch_bounds__(T, V <= 4 ? 8 : 1) void cs_tail_kernel(CsArgs a)
{
    extern __shared__ __align__(16) unsigned cs_lds[];
    __shared__ unsigned sh[3 * T / 64];
    if (a.chunk_off[a.n_inst] > a.capacity) return;                      // record arrays too small: leave them alone
    write_tails<T, V>(a, blockIdx.x, cs_lds, sh);
}

// The sort of chunk_core.h, with flow ids and tail bytes in LDS: up to kSmallFlows flows by a wavefront, which counts the tails before each instead of sorting where they
// are few, and beyond kRegisterFlows: sixteen flows a thread spill.  us of the whole stage, sixteen a thread / LDS, 256 instances of 16384 flows: all tails 112 / 80, a tenth 77 / 45,
// 3 in a hundred 73 / 41; 520 of 8320 flows 166 / 128, 150 / 73, 140 / 64.  Canonical positions picked out in memory instead of LDS: 107 for the 80, but 1903 / 2076 the
// other way round for 9001 instances of 9001 flows, two workgroups of 256 threads on a CU, and 41 / 45 for the 3 in a hundred.
template <int T>
__global__ __launch_bounds__(T) void cs_tail_lds_kernel(CsArgs a)
{
    extern __shared__ __align__(16) unsigned cs_lds[];
    __shared__ unsigned sh[kTailShared];
    unsigned *hist = cs_lds;                                             // [tail_hist_words<T>()], read 16 bytes at a time
    unsigned *rem = hist + tail_hist_words<T>();                         // [NF] tail bytes per flow
    unsigned short *idx_a = reinterpret_cast<unsigned short *>(rem + a.NF);    // [NF] flow ids, ping
    unsigned short *idx_b = idx_a + a.NF;                                      // [NF] pong
    if (a.chunk_off[a.n_inst] > a.capacity) return;                      // record arrays too small: leave them alone

    const int inst = blockIdx.x;
    const int b = inst / a.M, k = inst % a.M;
    const int64_t *rows = a.D1 + ((int64_t)b * a.G + (int64_t)k * a.N) * a.G;

    int nt = 0;
    const unsigned short *sorted = tail_sort_block<T>(a, rows, k, rem, hist, idx_a, idx_b, sh, nt, [] {});

    const int64_t out0 = a.chunk_off[inst] + a.cnt_full[inst];
    const uint32_t n_full = (uint32_t)a.cnt_full[inst];
    const uint32_t *fs = a.full_start + (int64_t)inst * a.NF;
    const uint16_t *tb = a.tails_before + (int64_t)inst * a.NF;
    auto canonical = [&](int f) { return (f + 1 < a.NF ? fs[f + 1] : n_full) + tb[f]; };
    const bool through = T == 1024 && a.perm && 4 * nt > a.NF;           // canonical positions read in flow order and picked out in LDS
    for (int i = threadIdx.x; i < nt; i += T) {
        const int f = sorted[i];
        a.chunk_w[out0 + i] = rem[f];
        a.chunk_flow[out0 + i] = (uint32_t)f;
        if (!through && a.perm) a.perm[out0 + i] = canonical(f);
    }
    if (!through) return;
    __syncthreads();
    for (int f = threadIdx.x; f < a.NF; f += T) rem[f] = canonical(f);
    __syncthreads();
    for (int i = threadIdx.x; i < nt; i += T) a.perm[out0 + i] = rem[sorted[i]];
}

static int launch_tail_kernel(void (*kernel)(CsArgs), int T, size_t lds, const CsArgs &a, hipStream_t st)
{
    if (lds > 48 * 1024) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) return RAILSCHED_ERR_HIP;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)a.n_inst), dim3((unsigned)T), lds, st, a);
    return launch_status();
}

template <int T, int V>
static int launch_cs_tail(const CsArgs &a, hipStream_t st) { return launch_tail_kernel(cs_tail_kernel<T, V>, T, tail_lds<T>(a.NF), a, st); }

template <int T>
static int launch_cs_tail_lds(const CsArgs &a, hipStream_t st)
{
    return launch_tail_kernel(cs_tail_lds_kernel<T>, T, sizeof(unsigned) * (size_t)(a.NF + tail_hist_words<T>()) + 2 * sizeof(unsigned short) * (size_t)a.NF, a, st);
}

constexpr int kRegisterFlows = 8192;
// Threads for four flows each: a wavefront without flows waits at every barrier and holds its room (1590 instances of 1080 flows 45 us by 512 threads, 40 by 320; 1200 of 2700 66
// by 1024, 58 by 768).
static int launch_tails(const CsArgs &a, hipStream_t st)
{
    if (a.NF <= kSmallFlows) return launch_cs_tail_lds<64>(a, st);
    if (a.NF > kRegisterFlows) return flow_threads(a.n_inst, a.NF) == 256 ? launch_cs_tail_lds<256>(a, st) : launch_cs_tail_lds<1024>(a, st);
    return a.NF <= 512 ? launch_cs_tail<256, 2>(a, st) : a.NF <= 1024 ? launch_cs_tail<256, 4>(a, st) : a.NF <= 1280 ? launch_cs_tail<320, 4>(a, st)
         : a.NF <= 1536 ? launch_cs_tail<384, 4>(a, st) : a.NF <= 2048 ? launch_cs_tail<512, 4>(a, st) : a.NF <= 3072 ? launch_cs_tail<768, 4>(a, st)
         : a.NF <= 4096 ? launch_cs_tail<1024, 4>(a, st) : launch_cs_tail<1024, 8>(a, st);
}

// ---- D: full chunks ---------------------------------------------------------------------------
// Write bound: 9 to 13 bytes a record.  A workgroup writes one tile of 1024 records at a multiple of that and exits, a wavefront its own kilobyte of
// every array, on a 1 KiB boundary, with streaming stores.  What a writer reaches of the chip's 6.9 TB/s hangs on how many bytes wait behind
// how long a chain of reads, and on what lies side by side in time: bare writers of 13 bytes a record, TB/s: no reads 6.1, two dependent trips in front
// of the stores 5.2, the same with neighbouring tiles on one XCD 5.5, with streaming stores too 6.0; two and four tiles a workgroup are
// slower throughout (5.2, 5.1), and so are two and four windows behind one chain of reads (226 M records of 512 GPUs, whole stage 600 us by one, 613, 625).  A wavefront
// makes four trips (the number of records; its entry; its instance's bounds; the flow starts from the entry's flow on), the first three through the scalar cache,
// no barrier, and finds the flows of its records from the starts that fall among them, as window_flows does.
// Measured, as contiguous runs of tiles per workgroup with their flow starts staged in LDS / now: 4096 instances of 117 K records 1295 / 990 us (4.8 / 6.3 TB/s),
// 3904 instances of 57 K in flows of 14: 611 / 515 (5.3).
// Windows write the instances of kFillWindow full chunks and more.  Of these at most two have records in one: the one that holds the window's first record, and the one that
// holds the record behind it.  The instances of fewer have a wavefront of their own (16 000 instances of two flows, 2000 records in all: 480 us when windows
// went from instance to instance, 37 now; 1335 matrices of 24 GPUs, 12 500 records 95 and 20).

// v of lane l, the same in all lanes
__device__ __forceinline__ int64_t shfl_i64(int64_t v, int l)
{
    return (int64_t)((uint64_t)(unsigned)__builtin_amdgcn_readlane((int)((uint64_t)v >> 32), l) << 32 | (unsigned)__builtin_amdgcn_readlane((int)v, l));
}

// p[i] through the scalar cache, i the same in all lanes, for what no workgroup of the launch writes: the compiler by itself takes a vector load once there are
// stores in front (61 layers of 512 GPUs 743 us for 630)
template <typename T>
__device__ __forceinline__ T scalar_load(const T *p, int64_t i) { return ((const __attribute__((address_space(4))) T *)p)[i]; }

// Full chunks of an instance (out0: its first record, n_full of them, at least one, fewer than 2^32) among the records w0 .. w0 + 255, w0 a multiple of 4.  j0: a flow that starts at
// the first of them or before.  mark: 256 words of LDS for the calling wavefront, 16-byte aligned.  U: flow starts a lane has in flight, after one by itself where U = 2.
template <int U>
__device__ __forceinline__ void fill_part(const CsArgs &a, int vec_ok, unsigned *mark, int64_t w0, int inst, int64_t out0, uint32_t n_full, int j0)
{
    const int lane = threadIdx.x & 63;
    const uint32_t cw = (uint32_t)a.C;
    const int64_t first = w0 - out0;                                     // instance position of the window's first record; negative where the instance starts in it
    const uint32_t last = first + kFillWindow <= (int64_t)n_full ? (uint32_t)(first + kFillWindow - 1) : n_full - 1u;
    const uint32_t *fs = a.full_start + (int64_t)inst * a.NF;
    const uint16_t *tb = a.tails_before + (int64_t)inst * a.NF;
    *reinterpret_cast<uint4 *>(mark + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
    lds_sync();
    unsigned base = 0;                                                   // flow << 16 | tails before it: both ascend together
    auto take = [&](int f, uint32_t s, unsigned tails) {                 // 64 flow starts; false when the window's end is among them
        const unsigned v = (unsigned)f << 16 | tails;
        const bool in = s <= last, before = in && (int64_t)s <= first;
        const int n = __popcll(__ballot(before));
        if (n) base = (unsigned)__builtin_amdgcn_readlane((int)v, n - 1);
        // of flows that start at one place only the last can hold it: the others are empty
        const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)s, 0x130, 0xF, 0xF, false);   // wave_shl:1
        if (in && !before && (s != next || lane == 63)) atomicMax(&mark[(uint32_t)((int64_t)s - first)], v);
        return __ballot(!in) == 0ull;
    };
    bool on = true;
    int f0 = j0;
    if constexpr (U == 2) {
        const int f = j0 + lane;
        on = take(f, f < a.NF ? fs[f] : 0xFFFFFFFFu, f < a.NF ? (unsigned)tb[f] : 0u);
        f0 += 64;
    }
    // Many flows of no full chunk: two loads in flight (273 instances of 5616 flows, nearly all tails: 36 us one by one, 23 so, 18 by four, but mostly one more
    // is enough: 224 M records of 61 layers as routed, 1.1 Zipf, whole stage 725 us by four, 708 by two)
    for (; on; f0 += 64 * U) {
        uint32_t s[U];
        unsigned tails[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int fu = f0 + 64 * u + lane, fc = fu < a.NF ? fu : a.NF - 1;
            s[u] = fs[fc];
            tails[u] = tb[fc];
            if (fu >= a.NF) s[u] = 0xFFFFFFFFu;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) if (on) on = take(f0 + 64 * u + lane, s[u], tails[u]);
    }
    lds_sync();
    const uint4 m = *reinterpret_cast<const uint4 *>(mark + 4 * lane);
    const unsigned m1 = max(m.x, m.y), m2 = max(m1, m.z), m3 = max(m2, m.w);
    const unsigned left = wave_max_before(max(m3, base), base);
    const unsigned v[4] = {max(left, m.x), max(left, m1), max(left, m2), max(left, m3)};
    const int64_t p = first + 4 * lane;
    const uint32_t lead = n_full - n_full % (uint32_t)a.N;               // positions below it go round robin (a.rail)
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

// Instance that holds record w, and a flow of it that starts before w's or is w's; its bounds and full chunks.
__device__ __forceinline__ void find_instance(const CsArgs &a, int64_t w, int64_t total, int &inst, int &j0, int64_t &out0, int64_t &out1, int64_t &n_full)
{
    j0 = 0;
    if (a.n_entries == 0) {
        inst = wave_last_le<int64_t>(a.chunk_off, a.n_inst, w);
    } else {
        const uint64_t entry = scalar_load(reinterpret_cast<const uint64_t *>(a.entries), w >> fill_entry_shift(total, a.n_entries));
        inst = (int)(uint32_t)entry;
        j0 = (int)(entry >> 32);
    }
    while (true) {
        out0 = scalar_load(a.chunk_off, inst);
        out1 = scalar_load(a.chunk_off, inst + 1);
        n_full = scalar_load(a.cnt_full, inst);
        if (out1 > w) return;
        const int i = inst + 1 + (threadIdx.x & 63) < a.n_inst ? inst + 1 + (threadIdx.x & 63) : a.n_inst;
        inst += __popcll(__ballot(a.chunk_off[i] <= w));                 // the entry lies before w, in another instance; chunk_off[n_inst] = total > w
        j0 = 0;
    }
}

__device__ __forceinline__ bool fill_windows_write(int64_t n_full) { return n_full >= kFillWindow && n_full <= 0xFFFFFFFFll; }

// The records w0 .. w0 + 255 of instances of kFillWindow full chunks and more; w0, a multiple of 256, is below `total`.
__device__ __forceinline__ void fill_window(const CsArgs &a, int vec_ok, unsigned *mark, int64_t w0, int64_t total)
{
    const int64_t w1 = w0 + kFillWindow;
    int inst, j0;
    int64_t out0, out1, n_full;
    find_instance(a, w0, total, inst, j0, out0, out1, n_full);
    if (fill_windows_write(n_full) && w0 < out0 + n_full) fill_part<2>(a, vec_ok, mark, w0, inst, out0, (uint32_t)n_full, j0);
    if (out1 >= w1 || w1 >= total) return;
    find_instance(a, w1, total, inst, j0, out0, out1, n_full);                   // such an instance that starts behind w0 goes on behind the window
    if (out0 >= w1) return;
    if (fill_windows_write(n_full)) fill_part<2>(a, vec_ok, mark, w0, inst, out0, (uint32_t)n_full, 0);
}

// The first inst_blocks workgroups write the instances of few full chunks, the others the windows.  Workgroup b, which the hardware deals to XCD b mod 8: every XCD takes 2^kshift
// neighbouring tiles in a row.
template <bool BEYOND>
__global__ __launch_bounds__(kFillThreads) void cs_fill_kernel(CsArgs a, int vec_ok, int kshift, unsigned inst_blocks)
{
    __shared__ __align__(16) unsigned marks[kFillThreads / 64][kFillWindow];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    unsigned *mark = marks[wave];
    const int64_t total = scalar_load(a.chunk_off, a.n_inst);
    if (total > a.capacity) return;
    if (blockIdx.x < inst_blocks) {
        const int64_t waves = (int64_t)inst_blocks * (kFillThreads / 64), w = (int64_t)blockIdx.x * (kFillThreads / 64) + wave;
        const int i0 = (int)(a.n_inst * w / waves), i1 = (int)(a.n_inst * (w + 1) / waves);
        for (int base = i0; base < i1; base += 64) {
            const int i = base + lane < i1 ? base + lane : i0;
            const int64_t off = a.chunk_off[i], full = a.cnt_full[i];
            unsigned long long few = __ballot(base + lane < i1 && full > 0 && full < kFillWindow);
            while (few) {
                const int l = __builtin_ctzll(few);
                few &= few - 1;
                const int64_t out0 = shfl_i64(off, l);
                const uint32_t n_full = (uint32_t)shfl_i64(full, l);
                for (int64_t w0 = out0 & ~(int64_t)3; w0 < out0 + n_full; w0 += kFillWindow)   // one round, or two
                    fill_part<4>(a, vec_ok, mark, w0, base + l, out0, n_full, 0);
            }
        }
        return;
    }
    const unsigned b = blockIdx.x - inst_blocks, blocks = gridDim.x - inst_blocks, in_granule = (1u << kshift) - 1u;
    auto window_of = [&](unsigned v) {
        const int64_t tile = ((int64_t)(v >> (3 + kshift)) << (3 + kshift)) + ((v & 7u) << kshift) + ((v >> 3) & in_granule);
        return tile * kFillTile + wave * kFillWindow;
    };
    int64_t w0 = window_of(b);
    if (w0 < total) fill_window(a, vec_ok, mark, w0, total);
    if (!BEYOND || (int64_t)blocks * kFillTile >= total || (a.tickets && b + (a.perm ? kFillRoundsPerm : kFillRounds) < blocks)) return;
    // Tiles behind the launch's: workgroup b draws on counter b mod kFillCounters, so that it stays with its XCD's.  The next ticket is on its way while a tile is written.
    __shared__ unsigned sh_ticket[2];
    const unsigned x = b & (kFillCounters - 1);
    auto draw = [&] {
        return a.tickets && threadIdx.x == 0 ? __hip_atomic_fetch_add(a.tickets + x * kTicketStep, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    };
    unsigned ticket = draw();
    int64_t v = b;
    for (int k = 0;; k ^= 1) {                                           // the slot before is still being read
        if (a.tickets) {
            if (threadIdx.x == 0) sh_ticket[k] = ticket;
            lds_sync();
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            v = (int64_t)blocks + (int64_t)kFillCounters * (unsigned)__builtin_amdgcn_readfirstlane((int)sh_ticket[k]) + x;
        } else {
            v += blocks;
        }
        if ((v >> (3 + kshift) << (3 + kshift)) * kFillTile >= total) return;   // the same in all wavefronts
        ticket = draw();
        w0 = window_of((unsigned)v);
        if (w0 < total) fill_window(a, vec_ok, mark, w0, total);
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
    a.tickets = nullptr;
    a.sums = nullptr;
    a.C = h_topo->chunk_bytes;
    a.cinv = ~0ull / (uint64_t)a.C;
    a.ginv = G > 1 ? (uint32_t)(((1ull << 32) + (uint64_t)G - 1) / (uint64_t)G) : 0u;
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
    a.clear = nullptr;
    fill_args(a, h_topo, n_inst, ws);
    if (n_inst > kScanAlone) {
        a.n_entries -= kScanBlocks;
        a.sums = reinterpret_cast<int64_t *>(a.entries + a.n_entries);
    }
    // Few records of instances of few flows are written as fast by wavefronts that search for their instance and go through its flows (scan / fill in us
    // with entries and without, 1672 instances of 152 flows 7.2 / 9.4, 4.3 / 10.0; 1457 of 775 flows 10.7 / 3.2, 5.0 / 3.5); a count query needs none.
    if (!chunk_w || (NF <= kSearchFlows && capacity <= kSearchRecords)) a.n_entries = 0;
    int64_t tiles = capacity / kFillTile + 1, most = kFillTiles + n_inst * NF / kFillTileFlows;
    if (most > kFillTilesMost) most = kFillTilesMost;
    const bool beyond = tiles > most;
    if (beyond) tiles = most;
    if (beyond && chunk_w && a.n_entries >= 2 * kFillCounters * kTicketStep) {   // at the end of the entries' room; few flows have too little
        a.n_entries -= kFillCounters * kTicketStep / 2;
        a.tickets = reinterpret_cast<unsigned *>(a.entries + a.n_entries);
    }
    if (args_out) *args_out = a;

    if (n_inst > 0) {
        launch_cs_count(a, st);
        if (int rc = launch_status()) return rc;
    }
    const int64_t scan_wants = a.n_entries ? n_inst : (n_inst + 63) / 64;       // workgroups: offsets alone are 64 lanes' work
    const int64_t scan_blocks = scan_wants < 1 ? 1 : scan_wants > kScanBlocks ? kScanBlocks : scan_wants;
    if (a.sums) {
        hipLaunchKernelGGL(cs_sums_kernel, dim3((unsigned)scan_blocks), dim3(kScanThreads), 0, st, a);
        if (int rc = launch_status()) return rc;
    }
    hipLaunchKernelGGL(cs_scan_kernel, dim3((unsigned)scan_blocks), dim3(kScanThreads), 0, st, a);
    if (int rc = launch_status()) return rc;
    if (!chunk_w || n_inst == 0) return RAILSCHED_OK;

    const int vec_ok = (reinterpret_cast<uintptr_t>(chunk_w) % 16 == 0 && reinterpret_cast<uintptr_t>(chunk_flow) % 16 == 0 &&
                        reinterpret_cast<uintptr_t>(perm) % 16 == 0 && reinterpret_cast<uintptr_t>(rail) % 4 == 0) ? 1 : 0;
    if (int rc = launch_tails(a, st)) return rc;
    int kshift = 0;
    while (kshift < kFillGranule && (tiles >> (kshift + 6)) > 0) ++kshift;
    const int64_t group = (int64_t)8 << kshift;
    const int64_t inst_waves = n_inst < kFillInstWaves ? n_inst : kFillInstWaves;
    const int64_t inst_blocks = (inst_waves + kFillThreads / 64 * 8 - 1) / (kFillThreads / 64 * 8) * 8;   // a whole number of rounds over the XCDs
    const dim3 grid((unsigned)((tiles + group - 1) / group * group + inst_blocks));
    hipLaunchKernelGGL(beyond ? cs_fill_kernel<true> : cs_fill_kernel<false>, grid, dim3(kFillThreads), 0, st, a, vec_ok, kshift, (unsigned)inst_blocks);
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
