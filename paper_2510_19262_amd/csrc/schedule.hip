// Stages 3-5 in one call (Algorithm 2 steps 1-3 and 6; Section 4.1 load matrices): chunk split and sort, LPT
// allocation, send/receive loads and statistics.  Outputs are those of railsched_chunk_sort, railsched_lpt_spray
// and railsched_eval run one after the other, bit for bit.
//
// Large batches run the kernels of the three stages, minus what stage 3 already knows: every instance starts with
// a run of n_full chunks of weight C, whose allocation from empty rails is round robin (rail = i mod N, the closed
// form behind Theorem 4's premise of equal granularity).  So the fill kernel writes those rails with the records,
// stage 4's streaming scan for the leading runs is skipped (its serial kernels start behind them), and stage 5 gets
// the leading runs' receive loads flow by flow in closed form and reads only the few chunks behind them - 13 bytes
// of HBM traffic per chunk in all instead of 27.  Small ones - up to 1024 instances of up to 64 K chunks on average, the
// shape of one training step's MoE layers - are bound by the latency of nine dependent launches, so they take
// three: the per-instance counts (stage 3's count kernel), then ONE workgroup per instance that does everything
// the instance needs, then the per-matrix reduction of stage 5.  Inside the workgroup all wavefronts sort the
// tails; then wavefront 0 runs the serial LPT chain on them - weights and rails in LDS, the chain being what bounds the
// time - while the other wavefronts write the full-chunk records, the round-robin rails of the leading run (closed
// form: from empty rails a run of one weight is rail = i mod N) and the receive loads those imply.  The average is all
// the host knows; an instance far longer than it leaves the rest of its full chunks to further workgroups of the launch.
#include "chunk_core.h"
#include "eval_core.h"
#include "lpt_core.h"

#include <mutex>

namespace rs {

// Workspace of railsched_schedule_static: one array per GPU, part of the library's device image, so the call needs no
// allocation.  The name below is only a handle for host code; the array's device address is asked for once per device
// (static_scratch) and that address is what kernels and every other use get.
static __device__ __align__(256) unsigned char scratch[RAILSCHED_STATIC_SCRATCH_BYTES];

constexpr int kScratchDevices = 64;
static void *g_scratch_ptr[kScratchDevices];       // device address of `scratch` on each GPU, once known
static std::mutex g_scratch_mutex;

// address of the current device's copy of `scratch`; nullptr if the runtime refuses
static void *static_scratch()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kScratchDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;   // this device is the current one
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}

void launch_cs_count(const CsArgs &a, hipStream_t st);          // chunk_sort.hip
int lpt_serial_after_leading_runs(const int64_t *chunk_off, const uint32_t *chunk_w, int64_t n_inst, int N, uint8_t *rail,
                                  int64_t *S, int64_t capacity, hipStream_t st);   // lpt_spray.hip
void cs_fill_args(CsArgs &a, const railsched_topo_t *h_topo, int64_t n_inst, void *ws);   // chunk_sort.hip

constexpr int kSlThreads = 256;         // closed-form receive loads of large batches
constexpr int kSsRun = 24;              // late chunks per run of one weight from which the chain goes run by run (lpt_runs_body)
constexpr int kSsLateAlone = 128;       // late chunks up to which the chain's wavefront also finishes them, beside the others' records
constexpr int kSsMaxInst = 1024;        // instances whose counts one workgroup adds up
// N*G of an instance held in LDS, 19 bytes a flow and 8 a GPU: 82 KB of a CU's 160 at 4096 flows of 8 rails, 111 of one.  No limit of speed: up to 6000
// fit for any N, 8192 from 16 rails on, and 5120 of 8 rails (80 nodes, 4.9 M chunks) take 87 us by one workgroup each, 146 by the separate kernels.
constexpr int kSsMaxFlows = 4096;
constexpr int kSsWideFlows = 1024;      // N*G above which an instance's workgroup has 1024 threads instead of 512: 16 flows a thread of the sort at most
// Instances of more than 2048 flows: one workgroup per CU, one round of them.  512 of 4096 flows and 61 K chunks even / skewed 145 / 241 us, by the separate
// kernels 209 / 224; 256 78 / 118 and 147 / 160.
constexpr int kSsMaxInstWide = 256;
// Full chunks an instance's workgroup writes itself; what a longer one has over is spread over further workgroups (ss_help).  us without / with that and
// by the separate kernels: 64 nodes x 8 rails, transposed Zipf 1.1, 3.9 M chunks, 751 K of them one instance's 187 / 79 / 134; 32 x 8, 15.1 M, 466 K
// 146 / 92 / 114; 16 x 8, 0.9 M, 214 K 97 / 36 / 53; even instances of 61 K on 64 x 8 75.6 / 76.9 / 124, of 57 K on 16 x 8 42 / 36 / 53.
constexpr int64_t kSsOwn = 8192;
constexpr int64_t kSsOwnWide = 32768;   // where thousands of tails are scheduled meanwhile
constexpr int64_t kSsOwnBusy = 65536;   // where no CU is idle
constexpr uint32_t kSsHelpTile = 4096;  // full chunks in a tile of those it leaves over
// Chunks per instance (capacity / instances) up to which one workgroup an instance, with helpers, is faster than the separate kernels.  us even / skewed,
// against the separate kernels: 256 instances of 4096 flows and 120 K chunks 156 / 170 against 195 / 205, 248 K 266 / 310 against 255 / 262; 1024 of 2048
// flows and 59 K 214 / 226 against 269 / 275, 117 K 541 / 540 against 372 / 372; 800 of 512 flows and 53 K 141 / 158 against 160 / 160.
constexpr int64_t kSsMaxAvg = 131072, kSsMaxAvgBusy = 65536;

struct SsArgs {
    uint8_t *rail;
    int64_t *S;
    int64_t *partial;       // stage 5 workspace: [batch][M][G + 1]; one workgroup per instance leaves only the largest weight there, behind the sums
    int64_t *R;             // receive loads of the matrices, cleared: the instances' workgroups add theirs up
    int64_t own;            // full chunks from which an instance leaves its records to the helping workgroups
    int32_t helpers;        // how many of them there are
    int32_t vec_ok;
    int32_t nshift, gmask;  // >= 0 when N / G are powers of two
};

__device__ __forceinline__ int ss_dst_node(const CsArgs &a, const SsArgs &x, uint32_t flow)   // flow = n*G + dst -> dst / N
{
    if (x.gmask >= 0 && x.nshift >= 0) return (int)((flow & (uint32_t)x.gmask) >> x.nshift);
    return (int)((flow % (uint32_t)a.G) / (uint32_t)a.N);
}

// Receive loads of the leading run (positions below `lead`, rails i mod N) into bins[G], in closed form.  The flows of one source
// GPU to the N GPUs of one node are neighbours in canonical order, so their full chunks are one range of positions:
// NF / N ranges of N rails each, dealt to the threads t, t + T, ... (per flow, as before, it was N times the atomics).
__device__ __forceinline__ void add_leading_run(const CsArgs &a, const SsArgs &x, const uint32_t *fs, uint32_t n_full, uint32_t lead,
                                                unsigned long long *bins, int t, int T)
{
    const int N = a.N, ranges = a.NF / N;
    const uint32_t cw = (uint32_t)a.C;
    for (int i = t; i < ranges; i += T) {
        const uint32_t s = fs[i * N];
        uint32_t e = i + 1 < ranges ? fs[(i + 1) * N] : n_full;
        e = e < lead ? e : lead;
        if (s >= e) continue;
        const int node = i % a.M;
        for (int n = 0; n < N; ++n) {
            // positions i < v with i mod N == n number (v + N - 1 - n) / N
            const uint32_t up = (uint32_t)(N - 1 - n);
            const uint32_t c = x.nshift >= 0 ? ((e + up) >> x.nshift) - ((s + up) >> x.nshift) : (e + up) / (uint32_t)N - (s + up) / (uint32_t)N;
            if (c) atomicAdd(&bins[node * N + n], (unsigned long long)c * (unsigned long long)cw);
        }
    }
}

// LDS words of hist, which the late chunks' weights take over once the tails are sorted
template <int T>
__host__ __device__ constexpr int ss_hist_words(int NF) { return tail_hist_words<T>() > NF + 128 ? tail_hist_words<T>() : (NF + 128 + 3) / 4 * 4; }
// LDS words of rem, where the wavefronts that write records then mark flow starts
template <int T>
__host__ __device__ constexpr int ss_rem_words(int NF) { return 256 * (T / 64 - 1) > NF ? 256 * (T / 64 - 1) : (NF + 3) / 4 * 4; }

// Records of the full chunks p_lo .. p_hi - 1 of one instance, and the rails of those in the leading run (below `skip`), by the wavefronts 1 .. of
// a workgroup that has the instance's flow starts in LDS.  marks: 256 words for each of them.
template <int kSsThreads>
__device__ __forceinline__ void fill_full(const CsArgs &a, const SsArgs &x, const unsigned *st_fs, const unsigned short *st_tb, unsigned *marks, int64_t out0,
                                          uint32_t skip, uint32_t p_lo, uint32_t p_hi)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t = (int)threadIdx.x - 64, N = a.N;
    constexpr int T = kSsThreads - 64;
    const uint32_t cw = (uint32_t)a.C;
    if (!x.vec_ok) {
        for (uint32_t p = p_lo + t; p < p_hi; p += T) {
            const int j = last_le<uint32_t>(st_fs, a.NF, p);
            a.chunk_w[out0 + p] = cw;
            a.chunk_flow[out0 + p] = (uint32_t)j;
            if (a.perm) a.perm[out0 + p] = p + st_tb[j];
            if (p < skip) x.rail[out0 + p] = (uint8_t)(p % (uint32_t)N);
        }
        return;
    }
    const uint32_t head = (uint32_t)((4 - ((out0 + p_lo) & 3)) & 3);      // scalar positions before the first aligned group
    const uint32_t pa = p_hi - p_lo < head ? p_hi : p_lo + head;
    const uint32_t groups = (p_hi - pa) / 4;
    const uint32_t pb = pa + groups * 4;
    // A wavefront streams a contiguous share of the groups, 64 at a time: shares and steps end where the global group index is
    // a multiple of 64, so the 64 lanes store one whole kilobyte on a 1 KiB boundary of each record array.
    constexpr int kFill = kSsThreads / 64 - 1;
    const uint32_t G0 = (uint32_t)(((out0 + pa) >> 2) & 63);             // global group index of group 0, mod 64
    auto share = [&](int w) {
        if (w <= 0) return 0u;
        if (w >= kFill) return groups;
        const uint32_t cut = ((G0 + (uint32_t)((uint64_t)groups * w / kFill)) & ~63u);
        return cut > G0 ? cut - G0 : 0u;
    };
    const uint32_t g0 = share(wave - 1), g1 = share(wave);
    unsigned *mark = marks + (wave - 1) * 256;
    int j_lo = g0 < g1 ? last_le<uint32_t>(st_fs, a.NF, pa + 4 * g0) : 0;
    uint32_t cnt = 0;
    for (uint32_t gb = g0; gb < g1; gb += cnt) {
        cnt = 64u - ((G0 + gb) & 63u);
        cnt = cnt < g1 - gb ? cnt : g1 - gb;
        const uint32_t p = pa + 4 * (gb + lane);
        uint32_t fl[4], pm[4], rr = 0;
        j_lo = window_flows(st_fs, a.NF, j_lo, pa + 4 * gb, pa + 4 * (gb + cnt) - 1, mark, fl);
        if ((uint32_t)lane >= cnt) continue;
        uint32_t r = x.nshift >= 0 ? (p & ((1u << x.nshift) - 1u)) : p % (uint32_t)N;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (a.perm) pm[e] = p + e + st_tb[fl[e]];
            rr |= r << (8 * e);
            r = (r + 1 == (uint32_t)N) ? 0u : r + 1;
        }
        *reinterpret_cast<uint4 *>(a.chunk_w + out0 + p) = make_uint4(cw, cw, cw, cw);
        *reinterpret_cast<uint4 *>(a.chunk_flow + out0 + p) = make_uint4(fl[0], fl[1], fl[2], fl[3]);
        if (a.perm) *reinterpret_cast<uint4 *>(a.perm + out0 + p) = make_uint4(pm[0], pm[1], pm[2], pm[3]);
        if (p + 4 <= skip) {
            *reinterpret_cast<uint32_t *>(x.rail + out0 + p) = rr;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) if (p + e < skip) x.rail[out0 + p + e] = (uint8_t)(rr >> (8 * e));
        }
    }
    const uint32_t n_edge = (pa - p_lo) + (p_hi - pb);                    // at most 6 positions outside the aligned groups
    if ((uint32_t)t < n_edge) {
        const uint32_t p = (uint32_t)t < pa - p_lo ? p_lo + (uint32_t)t : pb + ((uint32_t)t - (pa - p_lo));
        const int j = last_le<uint32_t>(st_fs, a.NF, p);
        a.chunk_w[out0 + p] = cw;
        a.chunk_flow[out0 + p] = (uint32_t)j;
        if (a.perm) a.perm[out0 + p] = p + st_tb[j];
        if (p < skip) x.rail[out0 + p] = (uint8_t)(p % (uint32_t)N);
    }
}

// Full chunks that an instance's own workgroup writes: x.own of them and up to a 1 KiB boundary of the record arrays.
__device__ __forceinline__ uint32_t ss_own_end(const SsArgs &x, int64_t out0, uint32_t n_full)
{
    const int64_t end = ((out0 + x.own + 255) & ~(int64_t)255) - out0;
    return end < (int64_t)n_full ? (uint32_t)end : n_full;
}

// What concerns an instance is the same in all lanes and is read out of its lane into scalar registers: with it in vector registers the kernel took 88 of
// them, not 72, and a CU two workgroups of 512 instead of three (800 instances of 256 flows: 38.8 us, now 36.0).
__device__ __forceinline__ uint32_t lane_u32(uint32_t v, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); }
__device__ __forceinline__ int64_t lane_i64(int64_t v, int l) { return (int64_t)((uint64_t)lane_u32((uint32_t)((uint64_t)v >> 32), l) << 32 | lane_u32((uint32_t)v, l)); }

// The workgroups behind the instances' write what the long instances leave over, in tiles of kSsHelpTile chunks, every one a run of consecutive
// tiles.  Which instances are long is known here only: the host sees the sum of their chunks at most (capacity), and the counts' kernel has just
// ended.  They read the counts, 64 instances at a time, and end at once when there is nothing over (or no room for the records).
template <int kSsThreads>
__device__ __forceinline__ void ss_help(const CsArgs &a, const SsArgs &x, unsigned *lds)
{
    const int tid = threadIdx.x, lane = tid & 63;
    unsigned *st_fs = lds, *marks = lds + (a.NF + 1 + (a.NF + 1) / 2 + 3) / 4 * 4;
    unsigned short *st_tb = reinterpret_cast<unsigned short *>(st_fs + a.NF + 1);
    // tiles of instance base + lane, its first record and its full chunks; `before` counts the records of the instances before `base`
    auto tiles_of = [&](int base, int64_t before, int64_t &out0, uint32_t &n_full, unsigned &tiles) {
        const int i = base + lane;
        const int64_t c = i < a.n_inst ? a.cnt_all[i] : 0;
        n_full = i < a.n_inst ? (uint32_t)a.cnt_full[i] : 0u;
        int64_t inc = c;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int64_t o = __shfl_up(inc, d);
            inc += lane >= d ? o : 0;
        }
        out0 = before + inc - c;
        tiles = (n_full - ss_own_end(x, out0, n_full) + kSsHelpTile - 1) / kSsHelpTile;
        return before + lane_i64(inc, 63);          // records up to base + 64
    };
    bool over = false;
#pragma unroll
    for (int u = 0; u < kSsMaxInst / kSsThreads; ++u) {                  // all loads in flight together: mostly this is all there is to do
        const int i = u * kSsThreads + tid;
        over |= i < a.n_inst && a.cnt_full[i] > x.own;
    }
    if (!__syncthreads_or(over)) return;
    int64_t out0, records = 0;
    uint32_t n_full;
    unsigned tiles, all = 0, sum;
    for (int base = 0; base < a.n_inst; base += 64) {
        records = tiles_of(base, records, out0, n_full, tiles);
        wave_exscan(tiles, sum);
        all += sum;
    }
    if (all == 0 || records > a.capacity) return;
    const unsigned h = blockIdx.x - (unsigned)a.n_inst, H = gridDim.x - (unsigned)a.n_inst;
    unsigned u = (unsigned)((uint64_t)all * h / H);
    const unsigned u1 = (unsigned)((uint64_t)all * (h + 1) / H);
    unsigned seen = 0;                              // tiles before `base`
    records = 0;
    for (int base = 0; base < a.n_inst && u < u1; base += 64) {          // the same in all wavefronts
        records = tiles_of(base, records, out0, n_full, tiles);
        const unsigned first = seen + wave_exscan(tiles, sum);           // first tile of this lane's instance
        seen += sum;
        while (u < u1 && u < seen) {
            const int l = 63 - __clzll((long long)__ballot(tiles != 0 && first <= u));
            const int inst = base + l;
            const int64_t o = lane_i64(out0, l);
            const uint32_t nf = lane_u32(n_full, l);
            const unsigned t0 = lane_u32(first, l), tn = lane_u32(tiles, l);
            const unsigned to = t0 + tn < u1 ? t0 + tn : u1;             // this workgroup's tiles of the instance: u .. to - 1
            __syncthreads();                                             // the instance before is done with the starts
            const uint32_t *fs = a.full_start + (int64_t)inst * a.NF;
            const uint16_t *tb = a.tails_before + (int64_t)inst * a.NF;
            for (int i = tid; i < a.NF; i += kSsThreads) { st_fs[i] = fs[i]; st_tb[i] = tb[i]; }
            if (tid == 0) st_fs[a.NF] = 0xFFFFFFFFu;
            __syncthreads();
            const uint32_t own = ss_own_end(x, o, nf);
            const uint32_t p_lo = own + (u - t0) * kSsHelpTile;
            const uint32_t left = nf - p_lo, run = (to - u) * kSsHelpTile;
            if (tid >= 64) fill_full<kSsThreads>(a, x, st_fs, st_tb, marks, o, nf - nf % (uint32_t)a.N, p_lo, p_lo + (left < run ? left : run));
            u = to;
        }
    }
}

template <int GW, int kSsThreads>
__global__ __launch_bounds__(kSsThreads) void ss_instance_kernel(CsArgs a, SsArgs x)
{
    extern __shared__ __align__(16) unsigned long long ss_lds64[];
    __shared__ int64_t sh_red[2][kSsThreads / 64];
    __shared__ unsigned sh_runs;
    __shared__ unsigned sh_sort[kTailShared];
    // LDS: hist / late_w | rem[NF] / marks | bins[G] u64 | st_fs[NF+1] | st_tb[NF] idx_a[NF] idx_b[NF] u16 | late_rail[NF+64] u8
    unsigned *hist = reinterpret_cast<unsigned *>(ss_lds64);             // read 16 bytes at a time
    unsigned *late_w = hist;
    unsigned *rem = hist + ss_hist_words<kSsThreads>(a.NF);              // later the record writers' marks, 16-byte aligned
    unsigned long long *bins = reinterpret_cast<unsigned long long *>(rem + ss_rem_words<kSsThreads>(a.NF));
    unsigned *st_fs = reinterpret_cast<unsigned *>(bins + a.G);
    unsigned short *st_tb = reinterpret_cast<unsigned short *>(st_fs + a.NF + 1);
    unsigned short *idx_a = st_tb + a.NF;
    unsigned short *idx_b = idx_a + a.NF;
    uint8_t *late_rail = reinterpret_cast<uint8_t *>(idx_b + a.NF);

    if ((int)blockIdx.x >= a.n_inst) {
        // with arguments read anew: those of the instances' path, kept for both, would not fit its scalar registers (75 of them parked in vector lanes, 10 so)
        typedef const __attribute__((address_space(4))) uint64_t *Words;
        constexpr size_t A = sizeof(CsArgs) / 8, X = sizeof(SsArgs) / 8;
        static_assert(sizeof(CsArgs) % 8 == 0 && sizeof(SsArgs) % 8 == 0 && alignof(SsArgs) == 8, "both are whole words, one behind the other");
        Words args = (Words)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(args));
        uint64_t words[A + X];
#pragma unroll
        for (size_t i = 0; i < A + X; ++i) words[i] = args[i];
        CsArgs ha;
        SsArgs hx;
        __builtin_memcpy(&ha, words, sizeof(CsArgs));
        __builtin_memcpy(&hx, words + A, sizeof(SsArgs));
        ss_help<kSsThreads>(ha, hx, hist);
        return;
    }
    const int inst = blockIdx.x;
    const int b = inst / a.M, k = inst % a.M;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int N = a.N;

    // ---- the tails; while their flows are on the way, the offsets (chunks of the instances before this one, and of all) and this
    // instance's flow starts
    int64_t before = 0, total = 0;
    uint32_t n_full = 0;
    int nt = 0;
    const int64_t *rows = a.D1 + ((int64_t)b * a.G + (int64_t)k * a.N) * a.G;
    const unsigned short *sorted = tail_sort_block<kSsThreads>(a, rows, k, rem, hist, idx_a, idx_b, sh_sort, nt, [&] {
        for (int i = tid; i < a.n_inst; i += kSsThreads) {
            const int64_t c = a.cnt_all[i];
            total += c;
            before += i < inst ? c : 0;
        }
        n_full = (uint32_t)a.cnt_full[inst];
        const uint32_t *fs = a.full_start + (int64_t)inst * a.NF;
        const uint16_t *tb = a.tails_before + (int64_t)inst * a.NF;
        for (int i = tid; i < a.NF; i += kSsThreads) { st_fs[i] = fs[i]; st_tb[i] = tb[i]; }
        for (int i = tid; i < a.G; i += kSsThreads) bins[i] = 0;
        if (tid == 0) { st_fs[a.NF] = 0xFFFFFFFFu; sh_runs = 0; }        // nothing starts behind the last flow
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) { before += __shfl_xor(before, d); total += __shfl_xor(total, d); }
        if (lane == 0) { sh_red[0][wave] = before; sh_red[1][wave] = total; }
    });                                                                  // its barriers cover the above
    before = 0; total = 0;
#pragma unroll
    for (int w = 0; w < kSsThreads / 64; ++w) { before += sh_red[0][w]; total += sh_red[1][w]; }
    const int64_t out0 = before;
    if (tid == 0) {
        a.chunk_off[inst] = out0;
        if (inst == a.n_inst - 1) a.chunk_off[a.n_inst] = total;
    }
    if (total > a.capacity) {                                            // record arrays too small: leave them alone, mark the loads
        if (tid < N) x.S[(int64_t)inst * N + tid] = -1;
        return;
    }

    // leading run: the full chunks (weight C) up to a multiple of N go round robin from empty rails
    const uint32_t cw = (uint32_t)a.C;
    const uint32_t skip = n_full - n_full % (uint32_t)N;
    const uint32_t late_full = n_full - skip;                            // full chunks left to the chain (< N)

    const int n_late = (int)late_full + nt;
    {   // the late chunks' weights, and how many runs of one weight they are
        unsigned starts = 0, total_starts;
        for (int i = tid; i < nt; i += kSsThreads) {
            const unsigned w = rem[sorted[i]];
            late_w[late_full + i] = w;
            starts += (i == 0 || rem[sorted[i - 1]] != w) ? 1u : 0u;
        }
        if (tid < (int)late_full) late_w[tid] = cw;
        if (tid < 64) late_w[n_late + tid] = 0;
        wave_exscan(starts, total_starts);
        if (lane == 0 && total_starts) atomicAdd(&sh_runs, total_starts);
    }
    // rails of the late chunks to memory, and their bytes to the receive bins
    auto finish_late = [&](int first, int step) {
        for (int i = first; i < n_late; i += step) {
            const unsigned r = late_rail[i];
            x.rail[out0 + skip + i] = (uint8_t)r;
            const uint32_t f = i < (int)late_full ? (uint32_t)last_le<uint32_t>(st_fs, a.NF, skip + i) : (uint32_t)sorted[i - late_full];
            atomicAdd(&bins[ss_dst_node(a, x, f) * N + r], (unsigned long long)late_w[i]);
        }
    };
    __syncthreads();
    if (wave == 0) {
        // ---- the serial chain over [late full chunks | sorted tails]; the others write the records
        __builtin_amdgcn_s_setprio(3);              // it is what the workgroup waits for
        const unsigned long long base = (unsigned long long)cw * (unsigned long long)(skip / (uint32_t)N);
        int64_t *S_row = x.S + (int64_t)inst * N;
        bool runs = false;
        if constexpr (GW <= 16) {
            runs = n_late >= kSsRun * (int)(sh_runs + 1u);
            if (runs) lpt_runs_body<GW>(late_w, late_rail, n_late, base, N, S_row);
        }
        if (!runs) lpt_wide_body<GW, true>(late_w, late_rail, n_late, base, N, S_row, late_w);
        __builtin_amdgcn_s_setprio(0);
        if (n_late <= kSsLateAlone) { lds_sync(); finish_late(lane, 64); }
    } else {
        // ---- full chunks: records, rails of the leading run, receive loads of the leading run
        const int t = tid - 64;
        constexpr int T = kSsThreads - 64;
        const int64_t tail0 = out0 + n_full;
        for (int i = t; i < nt; i += T) {
            const int f = sorted[i];
            a.chunk_w[tail0 + i] = late_w[late_full + i];
            a.chunk_flow[tail0 + i] = (uint32_t)f;
            // the tail is its flow's last chunk: the full chunks up to the next flow and the tails before it come first
            if (a.perm) a.perm[tail0 + i] = (f + 1 < a.NF ? st_fs[f + 1] : n_full) + st_tb[f];
        }
        fill_full<kSsThreads>(a, x, st_fs, st_tb, rem, out0, skip, 0u, ss_own_end(x, out0, n_full));
        add_leading_run(a, x, st_fs, n_full, skip, bins, t, T);
    }
    __syncthreads();
    if (n_late > kSsLateAlone) {
        finish_late(tid, kSsThreads);
        __syncthreads();
    }
    // Into R straight away: integers, in any order.  By slots that one workgroup a matrix then sums, whole call: 64 instances of 512 GPUs 55.9 us, 51.3 so;
    // 2 x 128 of 512 GPUs 46 / 38; 32 of 256 39.4 / 37.6; 4 of 16 GPUs and 800 of 32 the same.
    for (int i = tid; i < a.G; i += kSsThreads)
        if (const unsigned long long v = bins[i]) atomicAdd(reinterpret_cast<unsigned long long *>(x.R + (int64_t)b * a.G + i), v);
    if (tid == 0) x.partial[(int64_t)inst * (a.G + 1) + a.G] = n_full ? (int64_t)cw : nt ? (int64_t)late_w[0] : 0;   // no full chunk: the first tail is the largest
}

// ---------------------------------------------------------------------------------------------- large batches
// Receive loads of one instance into its workspace slot [G + 1]: the leading run (positions below
// n_full - n_full mod N, rails i mod N) flow by flow in closed form, the chunks behind it from their records.
__global__ __launch_bounds__(kSlThreads) void sl_recv_kernel(CsArgs a, SsArgs x)
{
    extern __shared__ unsigned long long sl_bins[];
    if (a.chunk_off[a.n_inst] > a.capacity) return;                      // the record arrays hold nothing
    const int inst = blockIdx.x, tid = threadIdx.x, N = a.N;
    for (int i = tid; i < a.G; i += kSlThreads) sl_bins[i] = 0;
    __syncthreads();
    const uint32_t n_full = (uint32_t)a.cnt_full[inst], n_all = (uint32_t)a.cnt_all[inst];
    const uint32_t lead = n_full - n_full % (uint32_t)N;
    const int64_t out0 = a.chunk_off[inst];
    const uint32_t *fs = a.full_start + (int64_t)inst * a.NF;
    add_leading_run(a, x, fs, n_full, lead, sl_bins, tid, kSlThreads);
    constexpr int U = 4;                                                 // records per thread and round, their loads in flight together (3904 instances of 3500: 75 -> 59 us)
    const int n_late = (int)(n_all - lead);                              // fewer than N full chunks and one tail per flow
    const int64_t late0 = out0 + lead;
    for (int i0 = tid; i0 < n_late; i0 += U * kSlThreads) {
        uint32_t w[U], f[U], r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = late0 + (i0 + u * kSlThreads < n_late ? i0 + u * kSlThreads : i0);
            w[u] = a.chunk_w[i]; f[u] = a.chunk_flow[i]; r[u] = x.rail[i];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int node = ss_dst_node(a, x, f[u]);
            if (i0 + u * kSlThreads < n_late && node < a.M && r[u] < (uint32_t)N) atomicAdd(&sl_bins[node * N + r[u]], (unsigned long long)w[u]);
        }
    }
    __syncthreads();
    int64_t *slot = x.partial + (int64_t)inst * (a.G + 1);
    for (int i = tid; i < a.G; i += kSlThreads) slot[i] = (int64_t)sl_bins[i];
    if (tid == 0) slot[a.G] = n_all ? (int64_t)a.chunk_w[out0] : 0;      // records are sorted: the first is the largest
}

template <int GW, int T>
static int launch_ss_t(const CsArgs &a, const SsArgs &x, hipStream_t st)
{
    const size_t lds = sizeof(unsigned long long) * (size_t)a.G + sizeof(unsigned) * (size_t)(a.NF + 1 + ss_rem_words<T>(a.NF) + ss_hist_words<T>(a.NF)) +
                       3 * sizeof(unsigned short) * (size_t)a.NF + (size_t)a.NF + 64 + 16;
    if (lds > 48 * 1024) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(ss_instance_kernel<GW, T>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds) != hipSuccess)
            return RAILSCHED_ERR_HIP;
    }
    hipLaunchKernelGGL((ss_instance_kernel<GW, T>), dim3((unsigned)(a.n_inst + x.helpers)), dim3(T), lds, st, a, x);
    return launch_status();
}

template <int GW>
static int launch_ss(const CsArgs &a, const SsArgs &x, hipStream_t st)
{
    // More instances than fit the chip together: half the threads each, so that more of them overlap (72 registers: three workgroups of 512 a CU, one of
    // 1024).  us by half / all of them: 288 instances of 2048 flows 69 / 111, 1024 of them 124 / 217; 1024 of 1024 flows and 2.4 K chunks 54 / 73, 800
    // of 256 and 0.5 K 31 / 36.  With many chunks per flow or instance the record writers want the threads: 800 of 256 flows and 22.6 K 70 / 66, 600 of 256 and
    // 1.6 K 30 / 30, 6.1 K 36 / 34, 22.6 K 60 / 51; 560 of 512 and 7.2 K 37 / 40, 26.5 K 61 / 55.
    if (a.NF > kSsWideFlows) return a.n_inst > 256 ? launch_ss_t<GW, 512>(a, x, st) : launch_ss_t<GW, 1024>(a, x, st);
    const bool half = a.n_inst > 512 && a.capacity <= a.n_inst * (a.n_inst > 768 ? (int64_t)16384 : 16 * (int64_t)a.NF);
    return half ? launch_ss_t<GW, 256>(a, x, st) : launch_ss_t<GW, 512>(a, x, st);
}

}  // namespace rs

namespace rs {
// stage 5 part of the workspace: stage 5's own slots, or one slot of G + 1 sums per instance, whichever is larger
static size_t sched_eval_bytes(int32_t batch, const railsched_topo_t *h_topo)
{
    const size_t e = railsched_eval_workspace_bytes(batch, h_topo);
    const size_t G = (size_t)h_topo->nodes * h_topo->rails;
    const size_t per_inst = align_up(sizeof(int64_t) * (size_t)batch * h_topo->nodes * (G + 1), 256);
    return e > per_inst ? e : per_inst;
}
}  // namespace rs

extern "C" size_t railsched_schedule_workspace_bytes(int32_t batch, const railsched_topo_t *h_topo)
{
    const size_t s = railsched_chunk_sort_workspace_bytes(batch, h_topo);
    const size_t e = railsched_eval_workspace_bytes(batch, h_topo);
    return (s && e) ? s + rs::sched_eval_bytes(batch, h_topo) : 0;     // both are multiples of 256
}

namespace rs {
// Stages 3-5 with the workspace already checked: ws holds railsched_schedule_workspace_bytes(batch, topo) bytes, 256-byte aligned.
static int schedule_run(const int64_t *D1, int32_t batch, const railsched_topo_t *h_topo, int64_t *chunk_off, uint32_t *chunk_w,
                        uint32_t *chunk_flow, uint32_t *perm, int64_t capacity, uint8_t *rail, int64_t *S, int64_t *R, int64_t *stats,
                        void *ws, hipStream_t st)
{
    const int64_t M = h_topo->nodes, N = h_topo->rails, G = M * N, NF = N * G;
    const int64_t n_inst = (int64_t)batch * M;
    const size_t ws_sort = railsched_chunk_sort_workspace_bytes(batch, h_topo);
    char *w8 = static_cast<char *>(ws);

    const int GW = N <= 4 ? 4 : N <= 8 ? 8 : N <= 16 ? 16 : N <= 32 ? 32 : 64;
    const unsigned w_limit = GW == 4 ? WideLimit<4>::value : GW == 8 ? WideLimit<8>::value : GW == 16 ? WideLimit<16>::value
                           : GW == 32 ? WideLimit<32>::value : WideLimit<64>::value;
    const bool small = n_inst <= (NF <= 2048 ? kSsMaxInst : kSsMaxInstWide) && NF <= kSsMaxFlows && capacity <= n_inst * (n_inst <= 256 ? kSsMaxAvg : kSsMaxAvgBusy) &&
                       (uint64_t)h_topo->chunk_bytes <= (uint64_t)w_limit;
    SsArgs x;
    x.rail = rail; x.S = S; x.partial = reinterpret_cast<int64_t *>(w8 + ws_sort);
    x.R = nullptr;
    x.vec_ok = 0; x.own = 0; x.helpers = 0;
    x.nshift = is_pow2(N) ? ilog2(N) : -1;
    x.gmask = is_pow2(G) ? (int32_t)G - 1 : -1;
    EvArgs e;
    e.chunk_off = chunk_off; e.chunk_w = chunk_w; e.chunk_flow = chunk_flow; e.rail = rail; e.S = S;
    e.R = R; e.stats = stats; e.partial = x.partial;
    e.M = (int32_t)M; e.N = (int32_t)N; e.G = (int32_t)G; e.slices = (int32_t)M;   // one slot per instance
    e.nshift = x.nshift; e.gmask = x.gmask; e.wide_ok = 0; e.copies = 1;
    e.capacity = capacity; e.n_inst = (int32_t)n_inst;

    if (!small) {
        CsArgs a;
        if (int rc = cs_run(D1, batch, h_topo, chunk_off, chunk_w, chunk_flow, perm, capacity, rail, S, w8, ws_sort, st, &a)) return rc;
        if (int rc = lpt_serial_after_leading_runs(chunk_off, chunk_w, n_inst, (int)N, rail, S, capacity, st)) return rc;
        const size_t lds = sizeof(unsigned long long) * (size_t)G;
        if (lds > 48 * 1024) {
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(sl_recv_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)lds) != hipSuccess)
                return RAILSCHED_ERR_HIP;
        }
        hipLaunchKernelGGL(sl_recv_kernel, dim3((unsigned)n_inst), dim3(kSlThreads), lds, st, a, x);
        if (int rc = launch_status()) return rc;
        return launch_eval_reduce(e, batch, st);
    }

    CsArgs a;
    a.D1 = D1; a.chunk_off = chunk_off; a.chunk_w = chunk_w; a.chunk_flow = chunk_flow; a.perm = perm;
    a.capacity = capacity;
    a.rail = nullptr; a.run_end = nullptr;          // unused by the count kernel
    cs_fill_args(a, h_topo, n_inst, w8);
    x.R = a.clear = R;
    launch_cs_count(a, st);
    if (int rc = launch_status()) return rc;

    x.vec_ok = (reinterpret_cast<uintptr_t>(chunk_w) % 16 == 0 && reinterpret_cast<uintptr_t>(chunk_flow) % 16 == 0 &&
                reinterpret_cast<uintptr_t>(perm) % 16 == 0 && reinterpret_cast<uintptr_t>(rail) % 4 == 0) ? 1 : 0;
    // One instance may hold as many chunks as there are records.  Up to 256 instances, or 128 of more than kSsWideFlows flows, which take a CU each, leave
    // CUs idle, and sharing starts early; beyond that an instance of the mean length writes all its records itself (960 instances of 29 K chunks: 101 us,
    // 129 when they shared theirs) and helpers come last.  64 / 256 of them, 1024 instances of 2048 flows, 59 K chunks each: even 213 / 214, skewed 337 / 226;
    // 960 of 1024 flows 174 / 174 and 290 / 199.  Beyond 2048 flows helpers would wait for a CU as long as the rest: only what one round holds, or 64.
    const bool wide = NF > kSsWideFlows, idle = n_inst <= (wide ? 128 : 256);
    x.own = !idle ? kSsOwnBusy : wide ? kSsOwnWide : kSsOwn;
    const int64_t room = NF <= 2048 || idle ? 256 : n_inst <= 192 ? 256 - n_inst : 64;
    const int64_t over = (capacity - x.own + kSsHelpTile - 1) / kSsHelpTile;
    x.helpers = (int32_t)(over <= 0 ? 0 : over < room ? over : room);
    int rc = GW == 4 ? launch_ss<4>(a, x, st) : GW == 8 ? launch_ss<8>(a, x, st) : GW == 16 ? launch_ss<16>(a, x, st)
           : GW == 32 ? launch_ss<32>(a, x, st) : launch_ss<64>(a, x, st);
    if (rc) return rc;
    return launch_eval_reduce(e, batch, st, true);
}

// arguments of railsched_schedule apart from the workspace: 0 and *nothing_to_do = false when the kernels should run
static int schedule_check(const int64_t *D1, int32_t batch, const railsched_topo_t *h_topo, int64_t *chunk_off, uint32_t *chunk_w,
                          uint32_t *chunk_flow, int64_t capacity, uint8_t *rail, int64_t *S, int64_t *R, int64_t *stats,
                          bool *nothing_to_do)
{
    *nothing_to_do = false;
    if (int rc = check_topo(h_topo)) return rc;
    if (batch < 0 || capacity < 0) return RAILSCHED_ERR_INVALID_ARG;
    if (batch > 65535) return RAILSCHED_ERR_UNSUPPORTED;
    const int64_t M = h_topo->nodes, N = h_topo->rails, G = M * N, NF = N * G;
    if (NF > kMaxFlows) return RAILSCHED_ERR_UNSUPPORTED;
    if ((int64_t)batch * M > 0x7FFFFFFFll / 64) return RAILSCHED_ERR_UNSUPPORTED;
    if (batch == 0) { *nothing_to_do = true; return RAILSCHED_OK; }
    if (!D1 || !chunk_off || !chunk_w || !chunk_flow || !rail || !S || !R || !stats) return RAILSCHED_ERR_NULL_PTR;
    return RAILSCHED_OK;
}
}  // namespace rs

extern "C" int railsched_schedule(const int64_t *D1, int32_t batch, const railsched_topo_t *h_topo, int64_t *chunk_off,
                                  uint32_t *chunk_w, uint32_t *chunk_flow, uint32_t *perm, int64_t capacity, uint8_t *rail,
                                  int64_t *S, int64_t *R, int64_t *stats, void *ws, size_t ws_bytes, void *stream)
{
    using namespace rs;
    bool nothing = false;
    if (int rc = schedule_check(D1, batch, h_topo, chunk_off, chunk_w, chunk_flow, capacity, rail, S, R, stats, &nothing)) return rc;
    if (nothing) return RAILSCHED_OK;
    if (!ws || ws_bytes < railsched_schedule_workspace_bytes(batch, h_topo) || reinterpret_cast<uintptr_t>(ws) % 256)
        return RAILSCHED_ERR_WORKSPACE;
    return schedule_run(D1, batch, h_topo, chunk_off, chunk_w, chunk_flow, perm, capacity, rail, S, R, stats, ws,
                        static_cast<hipStream_t>(stream));
}

extern "C" int railsched_schedule_static(const int64_t *D1, int32_t batch, const railsched_topo_t *h_topo, int64_t *chunk_off,
                                         uint32_t *chunk_w, uint32_t *chunk_flow, uint32_t *perm, int64_t capacity, uint8_t *rail,
                                         int64_t *S, int64_t *R, int64_t *stats, void *stream)
{
    using namespace rs;
    bool nothing = false;
    if (int rc = schedule_check(D1, batch, h_topo, chunk_off, chunk_w, chunk_flow, capacity, rail, S, R, stats, &nothing)) return rc;
    if (nothing) return RAILSCHED_OK;
    const size_t need = railsched_schedule_workspace_bytes(batch, h_topo);
    if (need == 0 || need > (size_t)RAILSCHED_STATIC_SCRATCH_BYTES) return RAILSCHED_ERR_SCRATCH;
    void *ws = static_scratch();
    if (!ws) return RAILSCHED_ERR_HIP;
    // every word of the workspace that a kernel reads was written earlier in the same call (counts and scans by the count
    // and scan kernels, one slot of receive loads per instance or slice), so what the last call left needs no clearing
    return schedule_run(D1, batch, h_topo, chunk_off, chunk_w, chunk_flow, perm, capacity, rail, S, R, stats, ws,
                        static_cast<hipStream_t>(stream));
}
