// Device-side pieces of the gating decision (Algorithm 1 step 1; Top-K of Section 6.3) shared by stage 1 and by the
// one-pass routing call: streaming loads and stores, the (value, index) argmax of the exact path, and the sorted
// per-lane key lists of the insertion kernels.
#pragma once

#include "common.h"

#include <cfloat>
#include <climits>

namespace rs {

// Logits are read once and indices written once: streaming (non-temporal) accesses keep them from
// displacing anything useful in the caches.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 load_stream4(const float *p)
{
    const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store_stream2(int32_t *p, int a, int b)
{
    i32x2 v; v.x = a; v.y = b;
    __builtin_nontemporal_store(v, reinterpret_cast<i32x2 *>(p));
}

template <int LANES, int VPL, bool VEC4>
__device__ __forceinline__ int slot_index(int q, int j)
{
    if constexpr (VEC4) return 4 * (q + LANES * (j >> 2)) + (j & 3);   // lane holds whole float4s, interleaved over lanes
    else return q + LANES * j;                                         // element-interleaved
}

template <int OFF>
__device__ __forceinline__ void argmax_step(float &bv, int &bi)
{
    const float ov = xlane<OFF>(bv);
    const int oi = xlane<OFF>(bi);
    const bool take = (ov > bv) || (ov == bv && oi < bi);
    bv = take ? ov : bv;
    bi = take ? oi : bi;
}

template <int LANES>
__device__ __forceinline__ void group_argmax(float &bv, int &bi)
{
    if constexpr (LANES >= 2) argmax_step<1>(bv, bi);
    if constexpr (LANES >= 4) argmax_step<2>(bv, bi);
    if constexpr (LANES >= 8) argmax_step<4>(bv, bi);
    if constexpr (LANES >= 16) argmax_step<8>(bv, bi);
    if constexpr (LANES >= 32) argmax_step<16>(bv, bi);
    if constexpr (LANES >= 64) argmax_step<32>(bv, bi);
}

// largest value / smallest index of a group of LANES lanes, in all of them
template <int LANES>
__device__ __forceinline__ float group_max(float v)
{
    if constexpr (LANES >= 2) v = fmaxf(v, xlane<1>(v));
    if constexpr (LANES >= 4) v = fmaxf(v, xlane<2>(v));
    if constexpr (LANES >= 8) v = fmaxf(v, xlane<4>(v));
    if constexpr (LANES >= 16) v = fmaxf(v, xlane<8>(v));
    return v;
}
template <int LANES>
__device__ __forceinline__ int group_min(int v)
{
    if constexpr (LANES >= 2) v = min(v, xlane<1>(v));
    if constexpr (LANES >= 4) v = min(v, xlane<2>(v));
    if constexpr (LANES >= 8) v = min(v, xlane<4>(v));
    if constexpr (LANES >= 16) v = min(v, xlane<8>(v));
    return v;
}

// ---------------------------------------------------------------------------------------------
// Insertion kernels for rows of 33..1024 logits and k <= KM (8 or 16): no rounds and no sorting networks.
//
// Keys are signed integers.  The order-preserving integer image of a logit keeps its upper bits and takes
// MASK - (expert index) into its low IDXBITS bits, so every key of a row is different, larger keys are larger cut values
// and, between equal cut values, lower expert indices, and the index comes back with one AND.  Four instructions per logit.
// The cut loses nothing when the bits it drops are zero in the whole row - logits that a gate computed in bf16 (16 zero
// bits) or any other short format - and then key order IS the exact order, ties included.  Otherwise the index bits are
// not trusted to order two logits of the same cut value: such rows are found and redone exactly, see below.
// A lane keeps the L largest keys it has seen as a descending list in registers.  Inserting x into a >= b >= c...
// is one instruction per entry: the new i-th entry is the median of (old entry i-1, old entry i, x), the new head
// max(head, x).  Then the LANES lanes of a row merge pairwise, log2(LANES) times, each keeping the KM largest of
// its own and its partner's list (max(a[i], b[KM-1-i]) is that set as a bitonic sequence; log2(KM) exchange layers sort
// it); both partners end with the same list, so finally every lane of the row holds the row's KM largest keys.
// The result is exact unless (a) the cut lost something and two neighbours among the k winners and the best loser share a
// cut value, or (b) a lane's whole list ended up among the winners, so that a key it dropped might have belonged there too.
// (A dropped key that shares the k-th winner's cut value is below the lane's last entry, which then shares it as well,
// and so does the best loser.)  A wavefront with such a row re-reads its rows and picks by full (value, index) comparisons.
// 4 194 304 rows of 64 logits from a bf16 gate, top-6, where most wavefronts hold a tie: 0.39 ms when every tie took the full
// comparisons, 0.21 now.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ int imed3(int a, int b, int c)
{
    int r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// x into the descending list a[0..HAVE) (a[0..L) once it is full)
template <int L, int HAVE>
__device__ __forceinline__ void list_insert(int (&a)[L], int x)
{
    if constexpr (HAVE == 0) {
        a[0] = x;
    } else {
        if constexpr (HAVE < L) a[HAVE] = min(a[HAVE - 1], x);
#pragma unroll
        for (int i = (HAVE < L ? HAVE - 1 : L - 1); i >= 1; --i) a[i] = imed3(a[i - 1], a[i], x);   // old a[i-1]: bottom first
        a[0] = max(a[0], x);
    }
}

// a bitonic sequence of N (a power of two) into descending order
template <int N>
__device__ __forceinline__ void bitonic_desc(int (&a)[N])
{
#pragma unroll
    for (int d = N / 2; d >= 1; d /= 2)
#pragma unroll
        for (int i = 0; i < N; ++i)
            if ((i & d) == 0) {
                const int hi = max(a[i], a[i + d]), lo = min(a[i], a[i + d]);
                a[i] = hi; a[i + d] = lo;
            }
}

template <int OFF>
__device__ __forceinline__ int from_partner(int v)
{
    constexpr int CTRL = OFF == 1 ? 0xB1 : OFF == 2 ? 0x4E : OFF == 4 ? 0x141 : 0x140;
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}

constexpr int kNoKey = INT_MIN;                     // below the key of every logit

// the KM largest of this lane's and its partner's descending lists of LEN entries (entries LEN..KM-1 count as lowest);
// both partners end with the same list
template <int OFF, int LEN, int KM>
__device__ __forceinline__ void merge_lists(const int (&a)[LEN], int (&out)[KM])
{
    static_assert(OFF == 1 || OFF == 2 || OFF == 4 || OFF == 8, "exchanges inside a row of 16 lanes");
    static_assert(LEN <= KM, "lists of at most KM keys");
#pragma unroll
    for (int i = 0; i < KM; ++i) {
        const bool own = i < LEN, theirs = KM - 1 - i < LEN;
        if (own && theirs) out[i] = max(a[i], from_partner<OFF>(a[KM - 1 - i]));   // folds into one v_max_i32 with a DPP operand
        else if (own) out[i] = a[i];                                  // the partner has nothing to set against it
        else if (theirs) out[i] = from_partner<OFF>(a[KM - 1 - i]);  // nor this lane against the partner's
        else out[i] = kNoKey;
    }
    bitonic_desc<KM>(out);
}

// key of a logit whose bits (-0 made +0) are c: lane_field has ones above the index bits and the lane's share of the index
// inside them; SLOT (a constant) likewise with the slot's share; the two never have an index bit in common.
template <unsigned SLOT>
__device__ __forceinline__ int make_ikey(unsigned c, unsigned lane_field)
{
    const unsigned sign = (unsigned)((int)c >> 31);
    const unsigned ord = __builtin_amdgcn_bitop3_b32(c, sign, 0x7FFFFFFFu, 0x78);       // c ^ (sign & 0x7FFFFFFF): monotone
    return (int)__builtin_amdgcn_bitop3_b32(ord, lane_field, SLOT, 0x91);               // (ord & lane & slot) | ~(lane | slot)
}
// expert index of a key
template <unsigned MASK>
__device__ __forceinline__ unsigned key_index(unsigned u) { return ~u & MASK; }

// float4s that no lane of the row has (E < LANES * VPL; E > LANES * VPL / 2) are left out: 132 logits in 8 lanes are 20 places a lane, not 32
template <int LANES, int VPL, int L, unsigned MASK, bool FULL, int C, int J>
__device__ __forceinline__ void insert_loaded(const float4 (&x)[VPL / 4], unsigned lane_field, int E, int (&lst)[L], unsigned &bits)
{
    if constexpr (C < VPL / 4) {
        if constexpr (!FULL && J == 0 && C >= VPL / 8) {
            if (4 * LANES * C >= E) return;         // uniform
        }
        constexpr unsigned SLOT = ~MASK | (unsigned)(4 * LANES * C + J);
        const float v = J == 0 ? x[C].x : J == 1 ? x[C].y : J == 2 ? x[C].z : x[C].w;
        const unsigned c = __float_as_uint(v + 0.0f);
        bits |= c;
        list_insert<L, (4 * C + J < L ? 4 * C + J : L)>(lst, make_ikey<SLOT>(c, lane_field));
        if constexpr (J == 3 && VPL >= 32) __builtin_amdgcn_sched_barrier(0);   // keys of later logits made early would only take registers
        insert_loaded<LANES, VPL, L, MASK, FULL, (J == 3 ? C + 1 : C), (J == 3 ? 0 : J + 1)>(x, lane_field, E, lst, bits);
    }
}

// smallest of (a ^ b) - 1 and m: zero-based distance of two keys' bit patterns, all-ones when they are the same key
__device__ __forceinline__ unsigned min_xor_dist(unsigned m, unsigned a, unsigned b)
{
    return min(m, (a ^ b) - 1u);
}

// This lane's VPL logits of the row at `row_logits` (LANES lanes per row, float4s interleaved over the lanes).
// FULL: E == LANES * VPL, every load is in range.
// Logits that do not exist (E < LANES * VPL) read as -infinity: a cut value of its own below every finite one, with zeros in the bits that
// the cut drops, so neither the order of the keys nor the union of the bits needs to know of them.
template <int LANES, int VPL, bool FULL>
__device__ __forceinline__ void row_load(const float *__restrict__ row_logits, int E, int q, float4 (&x)[VPL / 4])
{
#pragma unroll
    for (int c = 0; c < VPL / 4; ++c) {
        const int e0 = 4 * (q + LANES * c);
        if constexpr (FULL) x[c] = load_stream4(row_logits + e0);
        else x[c] = e0 < E ? load_stream4(row_logits + e0) : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
    }
}

// The L largest keys among this lane's logits, descending.  The logits are not needed afterwards.  bits: the union of their bit patterns.
template <int LANES, int VPL, int L, bool FULL>
__device__ __forceinline__ void lane_best(const float4 (&x)[VPL / 4], int E, int q, int (&own)[L], unsigned &bits)
{
    constexpr unsigned MASK = (unsigned)(LANES * VPL) - 1u;   // expert index bits of a key
    static_assert(VPL % 4 == 0 && VPL >= 8 && LANES >= 2 && LANES <= 16 && L >= 4 && L <= VPL / 2, "shape");
    bits = 0;
    insert_loaded<LANES, VPL, L, MASK, FULL, 0, 0>(x, ~MASK | (unsigned)(4 * q), E, own, bits);
}

// The same in two halves, so that a kernel that walks over rows can ask for its next logits between them: the keys take the logits' registers,
// and the list is made while the loads are on the way.
template <int LANES, int VPL, unsigned MASK, int C, int J>
__device__ __forceinline__ void make_keys(const float4 (&x)[VPL / 4], unsigned lane_field, int (&keys)[VPL], unsigned &bits)
{
    if constexpr (C < VPL / 4) {
        constexpr unsigned SLOT = ~MASK | (unsigned)(4 * LANES * C + J);
        const float v = J == 0 ? x[C].x : J == 1 ? x[C].y : J == 2 ? x[C].z : x[C].w;
        const unsigned c = __float_as_uint(v + 0.0f);
        bits |= c;
        keys[4 * C + J] = make_ikey<SLOT>(c, lane_field);
        make_keys<LANES, VPL, MASK, (J == 3 ? C + 1 : C), (J == 3 ? 0 : J + 1)>(x, lane_field, keys, bits);
    }
}
template <int LANES, int VPL>
__device__ __forceinline__ void lane_keys(const float4 (&x)[VPL / 4], int q, int (&keys)[VPL], unsigned &bits)
{
    constexpr unsigned MASK = (unsigned)(LANES * VPL) - 1u;
    bits = 0;
    make_keys<LANES, VPL, MASK, 0, 0>(x, ~MASK | (unsigned)(4 * q), keys, bits);
}
template <int LANES, int VPL, int L, bool FULL, int I = 0>
__device__ __forceinline__ void list_of_keys(const int (&keys)[VPL], int E, int (&own)[L])
{
    if constexpr (I < VPL) {
        if constexpr (!FULL && I % 4 == 0 && I >= VPL / 2) {
            if (LANES * I >= E) return;             // uniform; as in insert_loaded
        }
        list_insert<L, (I < L ? I : L)>(own, keys[I]);
        list_of_keys<LANES, VPL, L, FULL, I + 1>(keys, E, own);
    }
}

// The KM largest keys of the row from the lists of its LANES lanes, as bit patterns in u[0..KM), the same in all lanes of the
// row.  Returns true when the result cannot be trusted (see above): the caller then picks the row's winners by full comparisons.
template <int LANES, int VPL, int L, int KM>
__device__ __forceinline__ bool row_best(const int (&own)[L], unsigned bits, int k, unsigned (&u)[KM])
{
    constexpr unsigned MASK = (unsigned)(LANES * VPL) - 1u;
    int lst[KM];
    merge_lists<1, L, KM>(own, lst);
    if constexpr (LANES >= 4) { int t[KM]; merge_lists<2, KM, KM>(lst, t);
#pragma unroll
        for (int i = 0; i < KM; ++i) lst[i] = t[i]; }
    if constexpr (LANES >= 8) { int t[KM]; merge_lists<4, KM, KM>(lst, t);
#pragma unroll
        for (int i = 0; i < KM; ++i) lst[i] = t[i]; }
    if constexpr (LANES >= 16) { int t[KM]; merge_lists<8, KM, KM>(lst, t);
#pragma unroll
        for (int i = 0; i < KM; ++i) lst[i] = t[i]; }

    // lst[j] = j-th largest key of the row (if no lane dropped one of them), the same in all its lanes
#pragma unroll
    for (int j = 0; j < KM; ++j) u[j] = (unsigned)lst[j];
    int kth = lst[KM - 1];
    unsigned close = 0xFFFFFFFFu;                   // (a ^ b) - 1 < MASK: a and b are different keys of one cut value
#pragma unroll
    for (int j = 1; j < KM; ++j) {
        if (j <= k) close = min_xor_dist(close, u[j], u[j - 1]);     // neighbours among the winners and the best loser (k is uniform)
        if (j == k) kth = lst[j - 1];
    }
    if (k == KM) {                                  // the best loser is not in the list: this lane's keys against the last winner
#pragma unroll
        for (int i = 0; i < L; ++i) close = min_xor_dist(close, (unsigned)own[i], u[KM - 1]);
    }
    bool bad = close < MASK;
    if (__ballot(bad) != 0ull) {                    // did the cut lose anything in this row?
        bits |= (unsigned)from_partner<1>((int)bits);
        if constexpr (LANES >= 4) bits |= (unsigned)from_partner<2>((int)bits);
        if constexpr (LANES >= 8) bits |= (unsigned)from_partner<4>((int)bits);
        if constexpr (LANES >= 16) bits |= (unsigned)from_partner<8>((int)bits);
        bad = bad && (bits & MASK) != 0u;
    }
    return bad || own[L - 1] >= kth;                // ... or every key this lane kept is a winner
}

// expert indices of the row's k winners to topk_idx[row][0..k); streaming stores (4 194 304 rows of 64 logits, top-6: 0.209 ms, plain 0.227),
// but not of single indices, a sixteenth of a line per row and more (262 144 x 256 top-1: 46 us streaming, 43 plain).  Those have a branch of
// their own: two stores to one address under one condition become one store, and a plain one
template <int LANES, unsigned MASK, int KM>
__device__ __forceinline__ void store_best(int32_t *__restrict__ topk_idx, int64_t row, int k, int q, bool live, int wide_store,
                                           const unsigned (&u)[KM])
{
    if (KM == 8 && wide_store && k == 8) {          // one lane stores the row's eight indices: two 16-byte stores
        if (live && q == 0) {
            i32x4 lo, hi;
            lo.x = (int)key_index<MASK>(u[0]); lo.y = (int)key_index<MASK>(u[1]); lo.z = (int)key_index<MASK>(u[2]); lo.w = (int)key_index<MASK>(u[3]);
            hi.x = (int)key_index<MASK>(u[4]); hi.y = (int)key_index<MASK>(u[5]); hi.z = (int)key_index<MASK>(u[6]); hi.w = (int)key_index<MASK>(u[7]);
            i32x4 *dst = reinterpret_cast<i32x4 *>(topk_idx + row * 8);
            __builtin_nontemporal_store(lo, dst);
            __builtin_nontemporal_store(hi, dst + 1);
        }
    } else if (k == 1) {
        if (live && q == 0) topk_idx[row] = (int)key_index<MASK>(u[0]);
    } else {
#pragma unroll
        for (int r = 0; r < (KM + LANES - 1) / LANES; ++r) {         // winners q, q+LANES, ... of this lane
            unsigned sel = 0;
#pragma unroll
            for (int j = r * LANES; j < KM && j < (r + 1) * LANES; ++j) sel = (j == q + r * LANES) ? u[j] : sel;
            if (live && q + r * LANES < k) __builtin_nontemporal_store((int)key_index<MASK>(sel), topk_idx + row * k + q + r * LANES);
        }
    }
}

// The k winners of the row by full (value, index) comparisons, one round each: emit(j, expert) is called in every lane
// of the row for j = 0 .. k-1.  Lanes of rows that do not exist (live == false) load nothing and take part in the exchanges.
template <int LANES, int VPL, typename F>
__device__ __forceinline__ void row_exact(const float *__restrict__ row_logits, bool live, int E, int k, int q, F emit)
{
    float v[VPL];
#pragma unroll
    for (int c = 0; c < VPL / 4; ++c) {
        const int e0 = 4 * (q + LANES * c);
        const float4 cur = (live && e0 < E) ? load_stream4(row_logits + e0) : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
        v[4 * c + 0] = cur.x; v[4 * c + 1] = cur.y; v[4 * c + 2] = cur.z; v[4 * c + 3] = cur.w;
    }
    for (int sel = 0; sel < k; ++sel) {
        // the row's largest value first, then the lowest index that holds it: no branches (one such wavefront is what a small launch waits
        // for: 2048 x 512 top-8 10.0 -> 6.9 us, 8192 x 64 top-8 6.0 -> 5.0), and places inside the lane (constants)
        // while scanning and removing - expert indices of all VPL places would be kept in registers
        float bv = v[0];
#pragma unroll
        for (int j = 1; j < VPL; ++j) bv = fmaxf(bv, v[j]);
        bv = group_max<LANES>(bv);
        int bj = VPL;
#pragma unroll
        for (int j = VPL - 1; j >= 0; --j) bj = v[j] == bv ? j : bj;
        const int mine = bj < VPL && bv > -INFINITY ? 4 * (q + LANES * (bj >> 2)) + (bj & 3) : INT_MAX;
        const int bi = group_min<LANES>(mine);
        const int gone = bi == mine ? bj : VPL;     // only the winner's lane loses an entry
#pragma unroll
        for (int j = 0; j < VPL; ++j) v[j] = (j == gone) ? -INFINITY : v[j];
        emit(sel, bi);
    }
}

}  // namespace rs
