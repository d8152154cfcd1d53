// Extensions around the five core stages:
//  * railsched_transpose_matrix: traffic of the second all-to-all of an MoE layer (Algorithm 1 step 4:
//    expert outputs return to the token owners), i.e. every traffic matrix transposed;
//  * railsched_assign_policy: the path-selection schemes the paper compares against (Sections 1, 2.2,
//    6.1), reduced to arithmetic on the same chunk records: which rail would each chunk take.
#include "chunk_core.h"

namespace rs {

// ------------------------------------------------------------------------------------ transpose
constexpr int kTrTile = 32;

__global__ __launch_bounds__(256) void transpose_kernel(const int64_t *__restrict__ in, int64_t *__restrict__ out, int G, int tiles)
{
    __shared__ int64_t tile[kTrTile][kTrTile + 1];
    const int64_t b = blockIdx.x / ((int64_t)tiles * tiles);
    const int t = (int)(blockIdx.x % ((int64_t)tiles * tiles));
    const int ty = t / tiles, tx = t % tiles;
    const int64_t base = b * (int64_t)G * G;
    const int lx = threadIdx.x % kTrTile, ly = threadIdx.x / kTrTile;       // 32 x 8 threads
    for (int j = ly; j < kTrTile; j += 8) {
        const int r = ty * kTrTile + j, c = tx * kTrTile + lx;
        if (r < G && c < G) tile[j][lx] = in[base + (int64_t)r * G + c];
    }
    __syncthreads();
    for (int j = ly; j < kTrTile; j += 8) {
        const int r = tx * kTrTile + j, c = ty * kTrTile + lx;              // transposed block, rows written contiguously
        if (r < G && c < G) out[base + (int64_t)r * G + c] = tile[lx][j];
    }
}

// ------------------------------------------------------------------------------------ comparison schemes
constexpr int kPolThreads = 256;
constexpr int kPolTile = 8192;      // chunk positions per workgroup iteration
constexpr int kPolStage = 1024;     // instance boundaries staged in LDS per tile
constexpr int kPolSlots = 8;        // instances of a tile whose rail loads are accumulated in LDS
constexpr int kPolBlocks = 2048;

struct PolArgs {
    const int64_t *chunk_off;
    const uint32_t *chunk_w, *chunk_flow;
    uint8_t *rail;
    int64_t *S;
    uint64_t seed;
    int32_t n_inst, N, G, NF, policy;
    int32_t nmask, gshift;          // >= 0 when N / G are powers of two
    int32_t wide_ok;
    int64_t capacity;               // records the per-chunk arrays hold
};

__device__ __forceinline__ uint64_t mix64(uint64_t z)                   // splitmix64 finaliser
{
    z ^= z >> 30; z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27; z *= 0x94D049BB133111EBull;
    z ^= z >> 31;
    return z;
}

__device__ __forceinline__ uint32_t mod_n(const PolArgs &a, uint64_t x)
{
    return a.nmask >= 0 ? (uint32_t)x & (uint32_t)a.nmask : (uint32_t)(x % (uint64_t)a.N);
}

__device__ __forceinline__ uint32_t policy_rail(const PolArgs &a, int64_t inst, int64_t pos_global, int64_t pos_in_inst, uint32_t flow)
{
    switch (a.policy) {
        case 0: return a.gshift >= 0 ? flow >> a.gshift : flow / (uint32_t)a.G;                                  // NIC-direct
        case 1: return mod_n(a, mix64(a.seed + 0x9E3779B97F4A7C15ull * ((uint64_t)inst * (uint64_t)a.NF + flow + 1)));   // flow hash
        case 2: return mod_n(a, mix64(a.seed + 0x9E3779B97F4A7C15ull * ((uint64_t)pos_global + 1)));             // random spray
        default: return mod_n(a, (uint64_t)pos_in_inst);                                                        // round robin
    }
}

// S = 0 before the sums; -1 throughout when there are more chunks than the record arrays hold (the policy kernel
// then touches nothing)
__global__ void policy_init_kernel(PolArgs a, int64_t n)
{
    const int64_t v = a.chunk_off[a.n_inst] > a.capacity ? -1 : 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) a.S[i] = v;
}

// Streaming over all chunk positions, four per thread at multiples of four.  Send loads go to LDS bins
// for the first kPolSlots instances a tile touches (a tile rarely touches more) and from there, or
// directly for the rest, to S with integer atomics (S is zeroed first; integer sums are order-free).
__global__ __launch_bounds__(kPolThreads) void policy_kernel(PolArgs a)
{
    __shared__ int64_t s_off[kPolStage + 1];
    __shared__ unsigned long long bins[kPolSlots][kMaxRails];
    const int64_t total = a.chunk_off[a.n_inst];
    if (total > a.capacity) return;
    for (int64_t t0 = (int64_t)blockIdx.x * kPolTile; t0 < total; t0 += (int64_t)gridDim.x * kPolTile) {
        const int64_t t1 = t0 + kPolTile < total ? t0 + kPolTile : total;
        const int inst_lo = wave_last_le<int64_t>(a.chunk_off, a.n_inst, t0);
        const int inst_hi = wave_last_le<int64_t>(a.chunk_off, a.n_inst, t1 - 1);
        const int cnt = inst_hi - inst_lo + 1;
        const bool staged = cnt <= kPolStage;
        __syncthreads();                                   // previous tile is done with the LDS
        if (staged)
            for (int i = threadIdx.x; i <= cnt; i += kPolThreads) s_off[i] = a.chunk_off[inst_lo + i];
        for (int i = threadIdx.x; i < kPolSlots * kMaxRails; i += kPolThreads) (&bins[0][0])[i] = 0ull;
        __syncthreads();
        // one sweep for instance boundaries staged in LDS and one for boundaries read from memory (through a pointer that
        // may be either, every lookup is a flat load, which waits for all of the wavefront's memory traffic);
        // offs[i] = start of instance inst_lo + i
        auto sweep = [&](const int64_t *offs, int n_offs) {
            for (int64_t p = t0 + (int64_t)threadIdx.x * 4; p < t1; p += (int64_t)kPolThreads * 4) {
                uint32_t w[4], fl[4];
                const bool full = p + 4 <= total;
                if (full && a.wide_ok) {
                    const uint4 v = *reinterpret_cast<const uint4 *>(a.chunk_w + p);
                    const uint4 f = *reinterpret_cast<const uint4 *>(a.chunk_flow + p);
                    w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
                    fl[0] = f.x; fl[1] = f.y; fl[2] = f.z; fl[3] = f.w;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        w[e] = (p + e < total) ? a.chunk_w[p + e] : 0u;
                        fl[e] = (p + e < total) ? a.chunk_flow[p + e] : 0u;
                    }
                }
                int li = last_le<int64_t>(offs, n_offs, p);
                uint32_t packed = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (p + e >= total) break;
                    int64_t nxt = offs[li + 1];
                    while (p + e >= nxt) { ++li; nxt = offs[li + 1]; }
                    const int64_t b = offs[li];
                    const uint32_t r = policy_rail(a, inst_lo + li, p + e, p + e - b, fl[e]);
                    packed |= r << (8 * e);
                    if (r < (uint32_t)a.N) {
                        if (li < kPolSlots) atomicAdd(&bins[li][r], (unsigned long long)w[e]);
                        else atomicAdd(reinterpret_cast<unsigned long long *>(a.S + (int64_t)(inst_lo + li) * a.N + r), (unsigned long long)w[e]);
                    }
                }
                if (full && a.wide_ok) {
                    *reinterpret_cast<uint32_t *>(a.rail + p) = packed;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) if (p + e < total) a.rail[p + e] = (uint8_t)(packed >> (8 * e));
                }
            }
        };
        if (staged) sweep(s_off, cnt);
        else sweep(a.chunk_off + inst_lo, a.n_inst - inst_lo);
        __syncthreads();
        for (int i = threadIdx.x; i < kPolSlots * a.N; i += kPolThreads) {
            const int li = i / a.N, r = i % a.N;
            const unsigned long long v = bins[li][r];
            if (v && li < cnt) atomicAdd(reinterpret_cast<unsigned long long *>(a.S + (int64_t)(inst_lo + li) * a.N + r), v);
        }
    }
}

// ------------------------------------------------------------------------------------ port round robin
// Algorithm 2 step 4.  port[i] = (how many earlier chunks of the same instance went to the same rail) mod P.
// Instances are cut into as many tiles as kPortTile chunks each would be; they start at multiples of 16 of the record index, the first up to 15
// chunks early, and the last takes up to 15 chunks more; (1) tile offsets per instance, (2) per-tile per-rail counts, (3) per instance an exclusive scan of the counts over its tiles, (4) per tile the running
// counts.  Both tile kernels give a wavefront a tile.
//   packed (N <= 16, P a power of two up to 128, rail and port 16-byte aligned): a lane takes 16 consecutive chunks per 16-byte load
//     and keeps the N counts as bytes of one or two 64-bit registers; P <= 128 leaves a byte room for a start below P and 16
//     increments, and all sums modulo P come out right in wider fields.  Steps of 1024 chunks whose rails go round and round need no
//     counting.  120 M chunks, N = 8, P = 8: 32 us for the counts and 50 for the ports, 40 and 70 where everything is counted
//   by ballot (everything else): 64 chunks at a time, lanes with the same rail find each other by ballot matching, rank = running
//     count + number of lower lanes with that rail: 130 us for the counts and 200 for the ports of the same chunks.
constexpr int kPortTile = 4096;
constexpr int kPortWaves = 4;
// Most workgroups of a tile kernel: a tile a wavefront and exit up to 256 M chunks (2048 that go on: 86 us for the whole call on those 120 M chunks, 80 so; 991 M 725 / 620;
// four consecutive tiles a wavefront with one search 95 / 829).
constexpr int kPortBlocks = 16384;

struct PortArgs {
    const int64_t *chunk_off;
    const uint8_t *rail;
    uint8_t *port;
    int64_t *tile_off;          // [n_inst + 1]
    uint32_t *cnt;              // [tiles][N]: counts, then exclusive prefixes inside the instance
    int64_t max_tiles;
    int64_t capacity;           // records rail and port hold
    int32_t n_inst, N, P, pmask, rail_bits;
    int32_t nmask;              // N - 1 when N is a power of two up to 16, else -1
};

// first position of an instance's first tile
__device__ __forceinline__ int64_t port_base(int64_t off) { return off & ~int64_t(15); }

// 16-bit fields of the rails' byte counts: out[j] holds rails 2j and 2j + 1
template <int NW>
__device__ __forceinline__ void port_widen(const unsigned long long (&c)[NW], unsigned (&out)[4 * NW])
{
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const unsigned lo = (unsigned)c[w], hi = (unsigned)(c[w] >> 32);
        out[4 * w + 0] = (lo & 0xFFu) | ((lo << 8) & 0xFF0000u);
        out[4 * w + 1] = ((lo >> 16) & 0xFFu) | ((lo >> 8) & 0xFF0000u);
        out[4 * w + 2] = (hi & 0xFFu) | ((hi << 8) & 0xFF0000u);
        out[4 * w + 3] = ((hi >> 16) & 0xFFu) | ((hi >> 8) & 0xFF0000u);
    }
}

// The rails of a leading run, and of any run of one weight from level loads, go round and round.  A lane whose 16 chunks do (N a power of two up to 16: every
// rail 16 / N times, whichever comes first) needs no counting.
__device__ __forceinline__ bool port_cyclic(const uint4 &x, unsigned nmask)
{
    const unsigned all = nmask * 0x01010101u, r0 = x.x & 0xFFu;
    auto want = [&](unsigned d) { return (0x03020100u + ((r0 + 4u * d) & nmask) * 0x01010101u) & all; };
    return x.x == want(0) && x.y == want(1) && x.z == want(2) && x.w == want(3);
}

// Ports of 16 such chunks: run[r] = earlier chunks of rail r modulo P, a byte each; element j goes to rail (r0 + j) mod N and is that rail's (j / N)-th here.
template <int NW>
__device__ __forceinline__ void port_cyclic_out(const unsigned long long (&run)[NW], unsigned r0, int N, unsigned pm, uint32_t (&out)[4])
{
    unsigned e[4];                                  // the bytes of run, round and round
    e[0] = (unsigned)run[0]; e[1] = (unsigned)(run[0] >> 32);
    if constexpr (NW == 2) { e[2] = (unsigned)run[1]; e[3] = (unsigned)(run[1] >> 32); }
    if (N < 8) {
        if (N == 1) e[0] = (e[0] & 0xFFu) * 0x01010101u;
        if (N == 2) e[0] = (e[0] & 0xFFFFu) * 0x00010001u;
        e[1] = e[0];
    }
    if (N <= 8) { e[2] = e[0]; e[3] = e[1]; }
    const unsigned k = r0 >> 2;
    const unsigned a0 = k & 1 ? e[1] : e[0], a1 = k & 1 ? e[2] : e[1], a2 = k & 1 ? e[3] : e[2], a3 = k & 1 ? e[0] : e[3];
    const unsigned b0 = k & 2 ? a2 : a0, b1 = k & 2 ? a3 : a1, b2 = k & 2 ? a0 : a2, b3 = k & 2 ? a1 : a3;
    // turns before element 4 d + e, a byte each: bytes stay below 128 + 16
    const unsigned t0 = N == 1 ? 0x03020100u : N == 2 ? 0x01010000u : 0u, td = N == 1 ? 4u : N == 2 ? 2u : N == 4 ? 1u : 0u;
    const unsigned t2 = N == 8 ? 0x01010101u : 2u * td * 0x01010101u, t1 = td * 0x01010101u, p4 = pm * 0x01010101u;
    out[0] = (__builtin_amdgcn_alignbyte(b1, b0, r0 & 3u) + t0) & p4;
    out[1] = (__builtin_amdgcn_alignbyte(b2, b1, r0 & 3u) + t0 + t1) & p4;
    out[2] = (__builtin_amdgcn_alignbyte(b3, b2, r0 & 3u) + t0 + t2) & p4;
    out[3] = (__builtin_amdgcn_alignbyte(b0, b3, r0 & 3u) + t0 + t2 + t1) & p4;
}

// NW: 64-bit registers of byte counters (8 rails each)
template <bool ASSIGN, int NW>
__global__ __launch_bounds__(64 * kPortWaves) void port_packed_kernel(PortArgs a)
{
    constexpr int STEPS = kPortTile / 1024 + 1;     // 16-byte loads per lane and tile, all in flight together; the last for the last tile's up to 15 chunks more
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (a.chunk_off[a.n_inst] > a.capacity) return;                 // more chunks than rail and port hold: touch neither
    int64_t n_tiles = a.tile_off[a.n_inst];
    if (n_tiles > a.max_tiles) n_tiles = a.max_tiles;               // workspace sized for fewer chunks: never write past it
    for (int64_t u = (int64_t)blockIdx.x * kPortWaves + wv; u < n_tiles; u += (int64_t)gridDim.x * kPortWaves) {
        const int inst = wave_last_le<int64_t>(a.tile_off, a.n_inst, u);
        const int64_t lo = a.chunk_off[inst];
        const int64_t beg = port_base(lo) + (u - a.tile_off[inst]) * kPortTile;
        const int64_t hi = u + 1 == a.tile_off[inst + 1] ? a.chunk_off[inst + 1] : beg + kPortTile;   // this tile's end
        uint4 x[STEPS];
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            const int64_t i = beg + s * 1024 + lane * 16;
            x[s] = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);       // no rail
            if (i >= lo && i + 16 <= hi) {
                x[s] = *reinterpret_cast<const uint4 *>(a.rail + i);
            } else if (i < hi && i + 16 > lo) {                     // the instance's first or last chunks
                uint32_t w[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    w[q] = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int64_t p = i + 4 * q + e;
                        const uint32_t r = (p >= lo && p < hi) ? a.rail[p] : 0xFFu;
                        w[q] |= r << (8 * e);
                    }
                }
                x[s] = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
        uint32_t *c = a.cnt + u * a.N;
        if constexpr (!ASSIGN) {
            unsigned long long ctr[NW] = {};                        // at most 80 per byte
            unsigned turns = 0;                                     // steps that go round and round: 1024 / N of every rail
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                if (beg + s * 1024 >= hi) break;                    // wavefront-uniform: an instance's last tile may be short, a small instance has no other
                if (a.nmask >= 0 && __ballot(!port_cyclic(x[s], (unsigned)a.nmask)) == 0ull) { ++turns; continue; }
                const uint32_t w[4] = {x[s].x, x[s].y, x[s].z, x[s].w};
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const uint32_t r = (w[j >> 2] >> (8 * (j & 3))) & 0xFFu;
                    const unsigned long long one = (r < (uint32_t)a.N ? 1ull : 0ull) << ((r & 7u) * 8u);
#pragma unroll
                    for (int q = 0; q < NW; ++q) ctr[q] += (NW == 1 || (r >> 3) == (uint32_t)q) ? one : 0ull;
                }
            }
            if (turns * 1024u == (unsigned)(hi - beg)) {            // nothing else in the tile
                if (lane < a.N) c[lane] = turns * (1024u / (unsigned)a.N);
                continue;
            }
            unsigned f[4 * NW];
            port_widen<NW>(ctr, f);                                 // at most 4111 per field, summed over the lanes
#pragma unroll
            for (int q = 0; q < 4 * NW; ++q) {
                unsigned v = f[q];
#pragma unroll
                for (int d = 32; d >= 1; d >>= 1) v += (unsigned)__shfl_xor((int)v, d);
                if (lane == 2 * q && lane < a.N) c[lane] = (v & 0xFFFFu) + turns * (1024u / (unsigned)a.N);
                if (lane == 2 * q + 1 && lane < a.N) c[lane] = (v >> 16) + turns * (1024u / (unsigned)a.N);
            }
        } else {
            // A 64-bit shift by the last register a wavefront has goes wrong when others share its SIMD: 88 registers, amount in v87, and one chunk of
            // sixteen got a wrong port in one tile of twenty.  Taking the last register of the granule, v95 of 96 and five wavefronts a SIMD up to 8 rails, v103 of 104 and
            // four beyond, keeps the shifts below under it (by 32-bit halves instead, without such shifts: 850 us for three stages and ports of 120 M chunks, 820 so).
            if constexpr (NW == 1) asm volatile("; v95 is not used" ::: "v95");
            else asm volatile("; v103 is not used" ::: "v103");
            const unsigned pm = (unsigned)a.P - 1u, pm2 = pm | (pm << 16);
            const unsigned per_lane = a.nmask >= 0 ? 16u / (unsigned)a.N : 0u;          // of every rail, where rails go round and round
            unsigned start[4 * NW];                                 // counts before the step modulo P, 16-bit fields
#pragma unroll
            for (int q = 0; q < 4 * NW; ++q) {
                const unsigned b0 = 2 * q < a.N ? c[2 * q] : 0u, b1 = 2 * q + 1 < a.N ? c[2 * q + 1] : 0u;
                start[q] = (b0 & pm) | ((b1 & pm) << 16);
            }
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                if (beg + s * 1024 >= hi) break;
                const uint32_t w[4] = {x[s].x, x[s].y, x[s].z, x[s].w};
                unsigned f[4 * NW];
                const bool cyclic = a.nmask >= 0 && __ballot(!port_cyclic(x[s], (unsigned)a.nmask)) == 0ull;
                if (cyclic) {
                    const unsigned mine = (unsigned)lane * per_lane, total = 64u * per_lane;
#pragma unroll
                    for (int q = 0; q < 4 * NW; ++q) {
                        f[q] = (start[q] + (mine | mine << 16)) & pm2;
                        start[q] = (start[q] + (total | total << 16)) & pm2;
                    }
                } else {
                    unsigned long long ctr[NW] = {};
#pragma unroll
                    for (int j = 0; j < 16; ++j) {
                        const uint32_t r = (w[j >> 2] >> (8 * (j & 3))) & 0xFFu;
                        const unsigned long long one = (r < (uint32_t)a.N ? 1ull : 0ull) << ((r & 7u) * 8u);
#pragma unroll
                        for (int q = 0; q < NW; ++q) ctr[q] += (NW == 1 || (r >> 3) == (uint32_t)q) ? one : 0ull;
                    }
                    port_widen<NW>(ctr, f);
#pragma unroll
                    for (int q = 0; q < 4 * NW; ++q) {
                        unsigned total;
                        const unsigned before = wave_exscan(f[q], total);       // at most 1024 per field
                        f[q] = (start[q] + before) & pm2;
                        start[q] = (start[q] + total) & pm2;
                    }
                }
                unsigned long long run[NW];                         // the lane's counts modulo P, a byte each
#pragma unroll
                for (int q = 0; q < NW; ++q) {
                    const unsigned l = (f[4 * q] & 0xFFu) | ((f[4 * q] >> 8) & 0xFF00u) | ((f[4 * q + 1] & 0xFFu) << 16) | ((f[4 * q + 1] & 0xFF0000u) << 8);
                    const unsigned h = (f[4 * q + 2] & 0xFFu) | ((f[4 * q + 2] >> 8) & 0xFF00u) | ((f[4 * q + 3] & 0xFFu) << 16) | ((f[4 * q + 3] & 0xFF0000u) << 8);
                    run[q] = (unsigned long long)l | ((unsigned long long)h << 32);
                }
                uint32_t out[4] = {0, 0, 0, 0};
                if (cyclic) {
                    port_cyclic_out<NW>(run, w[0] & 0xFFu, a.N, pm, out);
                } else {
#pragma unroll
                    for (int j = 0; j < 16; ++j) {
                        const uint32_t r = (w[j >> 2] >> (8 * (j & 3))) & 0xFFu;
                        const bool ok = r < (uint32_t)a.N;
                        const unsigned sh = (r & 7u) * 8u;
                        const unsigned long long one = (ok ? 1ull : 0ull) << sh;
                        unsigned long long cur = run[0];
                        if constexpr (NW == 2) cur = (r >> 3) == 1u ? run[1] : run[0];
                        const uint32_t port = ok ? (uint32_t)(cur >> sh) & pm : 0u;
                        out[j >> 2] |= port << (8 * (j & 3));
#pragma unroll
                        for (int q = 0; q < NW; ++q) run[q] += (NW == 1 || (r >> 3) == (uint32_t)q) ? one : 0ull;
                    }
                }
                const int64_t i = beg + s * 1024 + lane * 16;
                if (i >= lo && i + 16 <= hi) {
                    __builtin_nontemporal_store(u32x4{out[0], out[1], out[2], out[3]}, reinterpret_cast<u32x4 *>(a.port + i));
                } else if (i < hi && i + 16 > lo) {
#pragma unroll
                    for (int j = 0; j < 16; ++j) {
                        const int64_t p = i + j;
                        if (p >= lo && p < hi) a.port[p] = (uint8_t)(out[j >> 2] >> (8 * (j & 3)));
                    }
                }
            }
        }
    }
}

__global__ __launch_bounds__(1024) void port_tiles_kernel(PortArgs a)
{
    __shared__ int64_t sh[1024];
    __shared__ int64_t carry;
    const int tid = threadIdx.x;
    if (tid == 0) carry = 0;
    __syncthreads();
    for (int base = 0; base < a.n_inst; base += 1024) {
        const int i = base + tid;
        int64_t v = 0;
        if (i < a.n_inst) {
            const int64_t lo = a.chunk_off[i], hi = a.chunk_off[i + 1];
            v = (hi - lo + kPortTile - 1) / kPortTile;
        }
        sh[tid] = v;
        __syncthreads();
        for (int d = 1; d < 1024; d <<= 1) {
            const int64_t x = tid >= d ? sh[tid - d] : 0;
            __syncthreads();
            sh[tid] += x;
            __syncthreads();
        }
        if (i < a.n_inst) a.tile_off[i] = carry + sh[tid] - v;
        __syncthreads();
        if (tid == 1023) carry += sh[1023];
        __syncthreads();
    }
    if (tid == 0) a.tile_off[a.n_inst] = carry;
}

template <bool ASSIGN>
__global__ __launch_bounds__(64 * kPortWaves) void port_tile_kernel(PortArgs a)
{
    __shared__ unsigned run[kPortWaves][kMaxRails];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const unsigned long long lt = (1ull << lane) - 1ull;
    if (a.chunk_off[a.n_inst] > a.capacity) return;                 // more chunks than rail and port hold: touch neither
    int64_t n_tiles = a.tile_off[a.n_inst];
    if (n_tiles > a.max_tiles) n_tiles = a.max_tiles;               // workspace sized for fewer chunks: never write past it
    unsigned *mine = run[wv];
    for (int64_t u = (int64_t)blockIdx.x * kPortWaves + wv; u < n_tiles; u += (int64_t)gridDim.x * kPortWaves) {
        const int inst = wave_last_le<int64_t>(a.tile_off, a.n_inst, u);
        const int64_t from = port_base(a.chunk_off[inst]) + (u - a.tile_off[inst]) * kPortTile;
        const int64_t beg = from > a.chunk_off[inst] ? from : a.chunk_off[inst];
        const int64_t end = u + 1 == a.tile_off[inst + 1] ? a.chunk_off[inst + 1] : from + kPortTile;
        uint32_t *c = a.cnt + u * a.N;
        if (lane < a.N) mine[lane] = ASSIGN ? c[lane] : 0u;
        __builtin_amdgcn_wave_barrier();
        for (int64_t i0 = beg; i0 < end; i0 += 64) {
            const int64_t i = i0 + lane;
            const bool act = i < end;
            const unsigned r = act ? a.rail[i] : 0u;
            const bool ok = act && r < (unsigned)a.N;
            if (!ASSIGN) {
                if (ok) atomicAdd(&mine[r], 1u);
            } else {
                unsigned long long peers = __ballot(ok);
                for (int bit = 0; bit < a.rail_bits; ++bit) {
                    const bool one = (r >> bit) & 1u;
                    const unsigned long long bm = __ballot(ok && one);
                    peers &= one ? bm : ~bm;
                }
                const unsigned base = ok ? mine[r] : 0u;
                const unsigned rank = base + (unsigned)__popcll(peers & lt);
                if (act) a.port[i] = ok ? (uint8_t)(a.pmask >= 0 ? (rank & (unsigned)a.pmask) : (rank % (unsigned)a.P)) : (uint8_t)0;
                __builtin_amdgcn_wave_barrier();
                if (ok && (peers >> lane) == 1ull) mine[r] = base + (unsigned)__popcll(peers);   // highest lane of the peer set
                __builtin_amdgcn_wave_barrier();
            }
        }
        if (!ASSIGN) {
            __builtin_amdgcn_wave_barrier();
            if (lane < a.N) c[lane] = mine[lane];
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// exclusive scan of the per-tile counts over the tiles of one instance; lane = rail
__global__ __launch_bounds__(64) void port_scan_kernel(PortArgs a)
{
    const int inst = blockIdx.x, lane = threadIdx.x;
    int64_t t0 = a.tile_off[inst], t1 = a.tile_off[inst + 1];
    if (t1 > a.max_tiles) t1 = a.max_tiles;
    if (lane >= a.N) return;
    unsigned running = 0;
    for (; t0 + 16 <= t1; t0 += 16) {                               // sixteen loads in flight: an instance may have thousands of tiles
        unsigned v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = a.cnt[(t0 + u) * a.N + lane];
#pragma unroll
        for (int u = 0; u < 16; ++u) { a.cnt[(t0 + u) * a.N + lane] = running; running += v[u]; }
    }
    for (; t0 < t1; ++t0) {
        const unsigned v = a.cnt[t0 * a.N + lane];
        a.cnt[t0 * a.N + lane] = running;
        running += v;
    }
}

// most tiles an instance list of `capacity` chunks is cut into
static int64_t port_max_tiles(int64_t capacity, int64_t n_inst) { return capacity / kPortTile + n_inst + 1; }

static void port_ws_layout(int64_t n_inst, int64_t max_tiles, int N, size_t off[3])
{
    size_t o = 0;
    off[0] = o; o += align_up(sizeof(int64_t) * (size_t)(n_inst + 1), 256);
    off[1] = o; o += align_up(sizeof(uint32_t) * (size_t)max_tiles * (size_t)N, 256);
    off[2] = o;
}

}  // namespace rs

extern "C" int railsched_transpose_matrix(const int64_t *D1, int32_t batch, const railsched_topo_t *h_topo, int64_t *D1T,
                                          void *stream)
{
    using namespace rs;
    if (int rc = check_topo(h_topo)) return rc;
    if (batch < 0) return RAILSCHED_ERR_INVALID_ARG;
    if (batch == 0) return RAILSCHED_OK;
    if (!D1 || !D1T) return RAILSCHED_ERR_NULL_PTR;
    if (D1 == D1T) return RAILSCHED_ERR_INVALID_ARG;     // not in place
    const int G = h_topo->nodes * h_topo->rails;
    const int tiles = (G + kTrTile - 1) / kTrTile;
    const int64_t blocks = (int64_t)batch * tiles * tiles;
    if (blocks > 0x7FFFFFFFll) return RAILSCHED_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(transpose_kernel, dim3((unsigned)blocks), dim3(256), 0, static_cast<hipStream_t>(stream), D1, D1T, G, tiles);
    return launch_status();
}

extern "C" int railsched_assign_policy(int32_t policy, uint64_t seed, const int64_t *chunk_off, const uint32_t *chunk_w,
                                       const uint32_t *chunk_flow, int32_t batch, const railsched_topo_t *h_topo,
                                       int64_t capacity, uint8_t *rail, int64_t *S, void *stream)
{
    using namespace rs;
    if (int rc = check_topo(h_topo)) return rc;
    if (batch < 0 || policy < 0 || policy > 3 || capacity < 0) return RAILSCHED_ERR_INVALID_ARG;
    const int64_t n_inst = (int64_t)batch * h_topo->nodes;
    if (n_inst > 0x7FFFFFFFll / 64) return RAILSCHED_ERR_UNSUPPORTED;
    if (n_inst == 0) return RAILSCHED_OK;
    if (!chunk_off || !S || (capacity > 0 && (!chunk_w || !chunk_flow || !rail))) return RAILSCHED_ERR_NULL_PTR;
    hipStream_t st = static_cast<hipStream_t>(stream);
    PolArgs a;
    a.capacity = capacity;
    a.chunk_off = chunk_off; a.chunk_w = chunk_w; a.chunk_flow = chunk_flow; a.rail = rail; a.S = S; a.seed = seed;
    a.n_inst = (int32_t)n_inst; a.N = h_topo->rails; a.G = h_topo->nodes * h_topo->rails; a.NF = a.N * a.G; a.policy = policy;
    a.nmask = is_pow2(a.N) ? a.N - 1 : -1;
    a.gshift = is_pow2(a.G) ? ilog2(a.G) : -1;
    a.wide_ok = (reinterpret_cast<uintptr_t>(chunk_w) % 16 == 0 && reinterpret_cast<uintptr_t>(chunk_flow) % 16 == 0 &&
                 reinterpret_cast<uintptr_t>(rail) % 4 == 0) ? 1 : 0;
    const int64_t n = n_inst * a.N;
    hipLaunchKernelGGL(policy_init_kernel, dim3((unsigned)((n + 255) / 256 > 1024 ? 1024 : (n + 255) / 256)), dim3(256), 0, st, a, n);
    if (int rc = launch_status()) return rc;
    hipLaunchKernelGGL(policy_kernel, dim3(kPolBlocks), dim3(kPolThreads), 0, st, a);
    return launch_status();
}

extern "C" size_t railsched_port_round_robin_workspace_bytes(int32_t batch, const railsched_topo_t *h_topo, int64_t capacity)
{
    using namespace rs;
    if (check_topo(h_topo) != RAILSCHED_OK || batch < 0 || capacity < 0) return 0;
    const int64_t n_inst = (int64_t)batch * h_topo->nodes;
    size_t off[3];
    port_ws_layout(n_inst, port_max_tiles(capacity, n_inst), h_topo->rails, off);
    return off[2];
}

extern "C" int railsched_port_round_robin(const int64_t *chunk_off, const uint8_t *rail, int32_t batch,
                                          const railsched_topo_t *h_topo, int32_t ports, int64_t capacity, uint8_t *port,
                                          void *ws, size_t ws_bytes, void *stream)
{
    using namespace rs;
    if (int rc = check_topo(h_topo)) return rc;
    if (batch < 0 || capacity < 0 || ports < 1) return RAILSCHED_ERR_INVALID_ARG;
    if (ports > 256) return RAILSCHED_ERR_UNSUPPORTED;
    const int64_t n_inst = (int64_t)batch * h_topo->nodes;
    if (n_inst > 0x7FFFFFFFll / 64) return RAILSCHED_ERR_UNSUPPORTED;
    if (n_inst == 0) return RAILSCHED_OK;
    if (!chunk_off || (capacity > 0 && (!rail || !port))) return RAILSCHED_ERR_NULL_PTR;
    const int64_t max_tiles = port_max_tiles(capacity, n_inst);
    size_t off[3];
    port_ws_layout(n_inst, max_tiles, h_topo->rails, off);
    if (!ws || ws_bytes < off[2] || reinterpret_cast<uintptr_t>(ws) % 256) return RAILSCHED_ERR_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    PortArgs a;
    a.chunk_off = chunk_off; a.rail = rail; a.port = port;
    a.tile_off = reinterpret_cast<int64_t *>(static_cast<char *>(ws) + off[0]);
    a.cnt = reinterpret_cast<uint32_t *>(static_cast<char *>(ws) + off[1]);
    a.max_tiles = max_tiles; a.capacity = capacity;
    a.n_inst = (int32_t)n_inst; a.N = h_topo->rails; a.P = ports; a.pmask = is_pow2(ports) ? ports - 1 : -1;
    a.rail_bits = a.N > 1 ? ilog2(a.N - 1) + 1 : 0;
    a.nmask = a.N <= 16 && is_pow2(a.N) ? a.N - 1 : -1;
    hipLaunchKernelGGL(port_tiles_kernel, dim3(1), dim3(1024), 0, st, a);
    if (int rc = launch_status()) return rc;
    // a few hundred chunks are all first and last ones of their instances, which the packed kernels take byte by byte (161 chunks: 12 us, 9 by ballot)
    const bool packed = capacity >= 1024 && a.N <= 16 && is_pow2(ports) && ports <= 128 && reinterpret_cast<uintptr_t>(rail) % 16 == 0 &&
                        reinterpret_cast<uintptr_t>(port) % 16 == 0;
    auto tiles = [&](auto by_ballot, auto one, auto two) {
        const int64_t want = (max_tiles + kPortWaves - 1) / kPortWaves;
        hipLaunchKernelGGL(packed ? (a.N <= 8 ? one : two) : by_ballot, dim3((unsigned)(want < kPortBlocks ? want : kPortBlocks)), dim3(64 * kPortWaves), 0, st, a);
        return launch_status();
    };
    if (int rc = tiles(port_tile_kernel<false>, port_packed_kernel<false, 1>, port_packed_kernel<false, 2>)) return rc;
    hipLaunchKernelGGL(port_scan_kernel, dim3((unsigned)n_inst), dim3(64), 0, st, a);
    if (int rc = launch_status()) return rc;
    return tiles(port_tile_kernel<true>, port_packed_kernel<true, 1>, port_packed_kernel<true, 2>);
}
