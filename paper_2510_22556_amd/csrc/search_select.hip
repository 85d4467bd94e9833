// Budget-driven block-size search and selection (Alg. 2; Eqs. topk,
// implicit_budget, rk, gk_star, final_selection).
//
// row_rank_kernel, topb_kernel  one workgroup per problem: the min(B,T)-th best score of
//                 the row, ties resolved by ascending index (rows of up to 16 384 tokens,
//                 and longer ones whose better tokens are listed, of not too many segments;
//                 the others).
//                 Result: (ordered key v, index cut c); token t is in T_topB iff
//                 key(t) > v or (key(t) == v and t <= c).  Its last phase counts
//                 the Top-B tokens of every segment: the implicit budgets b_k.
// heavy_list_kernel one workgroup per problem: segments with b_k >= 2 are recorded (only
//                 they need a search; b_k == 1 means g_k* = 1, b_k == 0 means g_k* = 0).
// search_kernel   wavefronts stride over a problem's records: Score_base of a segment, then
//                 the candidates largest first.
// seg_prefix_kernel one workgroup per problem: prefix sum of b_k (output offsets); the
//                 segments that retain anything are appended to one of two lists for
//                 the call: token-level ones (g_k* = 1) and the others.
// select_light_kernel sixteen lanes per token-level segment: its Top-B tokens in order.
// select_kernel   wavefronts stride over the other list: T_k(g_k*) written in
//                 ascending order at the segment's offset.
// A record carries everything its consumer needs (segment bounds, budget, block size,
// output offset), so a consumer starts with one 32-byte load; the order of the records
// does not matter.
//
// All quantities that decide an integer (block sums Phi, Score_k(g), Score_base,
// tau * Score_base) are fp64 and have the bits of the sum in ascending token order,
// one addition at a time: where no partial sum can round (sums_are_exact) they are
// formed in any order and as differences of prefix sums, elsewhere in that order.
// Rankings use (value descending, index ascending).
#include "sablock_internal.h"

#include <algorithm>
#include <cstdlib>

namespace sablock {
namespace {

// one unit of work of search_kernel / select_kernel
struct __attribute__((aligned(32))) SegRec {
    int32_t p, k;        // problem, segment
    int32_t a, b;        // token range of the segment
    int32_t bk;          // implicit budget b_k
    int32_t g;           // select: block size g_k*;  search: ordered key of the Top-B threshold
    int32_t pos;         // select: offset of the segment's tokens in the problem's idx_out row;  search: index cut
    int32_t out;         // search that also selects: offset of the segment's tokens in the problem's idx_out row
};

// LDS of a select wavefront: tokens whose scores are staged (CAPT), blocks whose Phi / class are kept (CAPB).
// Two sizes: the small one keeps many wavefronts resident for the bulk of the segments; longer segments go to a
// second list that is served by the same kernel with the large one.
constexpr int CAPB = 256, CAPT = 2 * CAPB;
constexpr int CAPB_LONG = 2048, CAPT_LONG = 2 * CAPB_LONG;
// Tokens of a segment whose prefix sums fit the LDS of a search wavefront (5 KiB); longer ones are searched from memory
// (search_streamed).
constexpr int PRE_TOKENS = 639;
constexpr int MAX_G = 64;           // largest candidate block size

// Wavefront reductions without LDS round trips: four DPP steps inside each row of 16 lanes (lane ^ 1, lane ^ 2,
// mirror inside 8, mirror inside 16: together they pair every lane with every other lane of its row), then lane 15 of
// rows 0 and 2 joins the row behind it and lane 31 the upper half, so lane 63 holds the result, which is read as a
// scalar: it is wave-uniform.
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_MIRROR = 0x140, DPP_BCAST15 = 0x142, DPP_BCAST31 = 0x143;
template <int CTRL>
__device__ inline int dpp_i(int v) { return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true); }     // every lane has a source
template <int CTRL, int ROWS>
__device__ inline int dpp_rows_i(int old, int v) { return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xf, false); }
template <int CTRL>
__device__ inline double dpp_d(double v) { return __hiloint2double(dpp_i<CTRL>(__double2hiint(v)), dpp_i<CTRL>(__double2loint(v))); }
template <int CTRL, int ROWS>
__device__ inline double dpp_rows_d(double old, double v)
{
    return __hiloint2double(dpp_rows_i<CTRL, ROWS>(__double2hiint(old), __double2hiint(v)),
                            dpp_rows_i<CTRL, ROWS>(__double2loint(old), __double2loint(v)));
}
__device__ inline double readlane_d(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane), __builtin_amdgcn_readlane(__double2loint(v), lane));
}
__device__ inline double shfl_d(double v, int lane)
{
    return __hiloint2double(__shfl(__double2hiint(v), lane), __shfl(__double2loint(v), lane));
}

__device__ inline int wave_sum_i(int v)
{
    v += dpp_i<DPP_XOR1>(v);
    v += dpp_i<DPP_XOR2>(v);
    v += dpp_i<DPP_HALF_MIRROR>(v);
    v += dpp_i<DPP_MIRROR>(v);
    v += dpp_rows_i<DPP_BCAST15, 0xa>(0, v);
    v += dpp_rows_i<DPP_BCAST31, 0xc>(0, v);
    return __builtin_amdgcn_readlane(v, 63);
}
template <typename V>
__device__ inline V wave_max_32(V v)                           // int or uint32_t
{
    v = max(v, (V)dpp_i<DPP_XOR1>((int)v));
    v = max(v, (V)dpp_i<DPP_XOR2>((int)v));
    v = max(v, (V)dpp_i<DPP_HALF_MIRROR>((int)v));
    v = max(v, (V)dpp_i<DPP_MIRROR>((int)v));
    v = max(v, (V)dpp_rows_i<DPP_BCAST15, 0xa>((int)v, (int)v));
    v = max(v, (V)dpp_rows_i<DPP_BCAST31, 0xc>((int)v, (int)v));
    return (V)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ inline int wave_max_i(int v) { return wave_max_32<int>(v); }
__device__ inline uint32_t wave_max_u(uint32_t v) { return wave_max_32<uint32_t>(v); }
__device__ inline uint64_t wave_max_u64(uint64_t v)
{
    const uint32_t hi = wave_max_u((uint32_t)(v >> 32)), lo = wave_max_u((uint32_t)(v >> 32) == hi ? (uint32_t)v : 0u);
    return ((uint64_t)hi << 32) | lo;
}
__device__ inline double wave_max_d(double v)
{
    v = fmax(v, dpp_d<DPP_XOR1>(v));
    v = fmax(v, dpp_d<DPP_XOR2>(v));
    v = fmax(v, dpp_d<DPP_HALF_MIRROR>(v));
    v = fmax(v, dpp_d<DPP_MIRROR>(v));
    v = fmax(v, dpp_rows_d<DPP_BCAST15, 0xa>(v, v));
    v = fmax(v, dpp_rows_d<DPP_BCAST31, 0xc>(v, v));
    return readlane_d(v, 63);
}
// only for sums that do not round (the order differs from an ascending one)
__device__ inline double wave_sum_d(double v)
{
    v += dpp_d<DPP_XOR1>(v);
    v += dpp_d<DPP_XOR2>(v);
    v += dpp_d<DPP_HALF_MIRROR>(v);
    v += dpp_d<DPP_MIRROR>(v);
    v += dpp_rows_d<DPP_BCAST15, 0xa>(0.0, v);
    v += dpp_rows_d<DPP_BCAST31, 0xc>(0.0, v);
    return readlane_d(v, 63);
}
// Inclusive prefix sums over the wavefront: shifts by 1, 2, 4 and 8 lanes inside a row of 16 (a lane without a source
// adds zero), then the two steps across rows
__device__ inline uint32_t wave_scan_u(uint32_t v)
{
    v += (uint32_t)dpp_rows_i<0x111, 0xf>(0, (int)v);
    v += (uint32_t)dpp_rows_i<0x112, 0xf>(0, (int)v);
    v += (uint32_t)dpp_rows_i<0x114, 0xf>(0, (int)v);
    v += (uint32_t)dpp_rows_i<0x118, 0xf>(0, (int)v);
    v += (uint32_t)dpp_rows_i<DPP_BCAST15, 0xa>(0, (int)v);
    v += (uint32_t)dpp_rows_i<DPP_BCAST31, 0xc>(0, (int)v);
    return v;
}
__device__ inline double wave_scan_d(double v)                 // exact sums only, as wave_sum_d
{
    v += dpp_rows_d<0x111, 0xf>(0.0, v);
    v += dpp_rows_d<0x112, 0xf>(0.0, v);
    v += dpp_rows_d<0x114, 0xf>(0.0, v);
    v += dpp_rows_d<0x118, 0xf>(0.0, v);
    v += dpp_rows_d<DPP_BCAST15, 0xa>(0.0, v);
    v += dpp_rows_d<DPP_BCAST31, 0xc>(0.0, v);
    return v;
}
// lanes below this one whose bit is set
__device__ inline int lanes_below(unsigned long long m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// best (value descending, index ascending) of the lanes' (value, index) pairs
__device__ inline bool pair_better(double op, int om, double bp, int bm) { return op > bp || (op == bp && om < bm); }
template <int CTRL>
__device__ inline void argmax_step(double &bp, int &bm)
{
    const int olo = dpp_i<CTRL>(__double2loint(bp)), ohi = dpp_i<CTRL>(__double2hiint(bp)), om = dpp_i<CTRL>(bm);
    const double op = __hiloint2double(ohi, olo);
    if (pair_better(op, om, bp, bm)) { bp = op; bm = om; }
}
__device__ inline void wave_argmax(double &bp, int &bm)
{
    argmax_step<DPP_XOR1>(bp, bm);
    argmax_step<DPP_XOR2>(bp, bm);
    argmax_step<DPP_HALF_MIRROR>(bp, bm);
    argmax_step<DPP_MIRROR>(bp, bm);
    const int lo = __double2loint(bp), hi = __double2hiint(bp);
    double rp = __hiloint2double(__builtin_amdgcn_readlane(hi, 0), __builtin_amdgcn_readlane(lo, 0));
    int rm = __builtin_amdgcn_readlane(bm, 0);
#pragma unroll
    for (int r = 16; r < 64; r += 16) {
        const double op = __hiloint2double(__builtin_amdgcn_readlane(hi, r), __builtin_amdgcn_readlane(lo, r));
        const int om = __builtin_amdgcn_readlane(bm, r);
        if (pair_better(op, om, rp, rm)) { rp = op; rm = om; }
    }
    bp = rp;
    bm = rm;
}

// acc += v[j] for every set bit j of mask, ascending; mask and acc are wave-uniform
__device__ inline double add_in_order(double acc, unsigned long long mask, float v)
{
    while (mask) {
        const int j = __builtin_ctzll(mask);                 // wave-uniform, so the value comes by v_readlane
        acc += (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), j));
        mask &= mask - 1;
    }
    return acc;
}

// ------------------------------------------------------------------ Top-B
constexpr int TB_THREADS = 1024;
constexpr int TB_WAVES = TB_THREADS / 64;
constexpr int TB_REG = 16;                         // values of a row that a thread holds at a time
constexpr int TB_ROUND = TB_THREADS * TB_REG;      // ... and the workgroup: 16 384
constexpr int TB_BINS = 4096;
constexpr int TB_RANKED = 1024;                    // entries of one bin that are ranked one against another
constexpr int TB_BUDGET_MAX = 16384;               // budgets of the one-call form
constexpr int TB_OFFS = 4096;                      // segment offsets and counters of a sequence kept in LDS:
constexpr int TB_OFFS_MAX = 16384;                 // the launch picks 4 096, 8 192 or 16 384 entries

__device__ inline bool in_topb(float v, int t, uint32_t thr_key, int thr_cut)
{
    const uint32_t key = ordered_key(v);
    return key > thr_key || (key == thr_key && t <= thr_cut);
}

// the float that a key stands for (of the two zeros, +0)
__device__ inline float float_of_key(uint32_t key)
{
    return __uint_as_float((key & 0x80000000u) ? key ^ 0x80000000u : ~key);
}

// segment of token t: the k with seg_off[k] <= t < seg_off[k+1], 0 <= k < K
__device__ inline int segment_of(const int32_t *off, int K, int t)
{
    int lo = 0, hi = K;                       // invariant: off[lo] <= t < off[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (off[mid] <= t) lo = mid; else hi = mid;
    }
    return lo;
}

// A row of T scores as 16-byte vectors: `head` scalars in front of the first aligned one, nvec vectors, a tail of
// at most three scalars.  The scalars are dealt out to the first threads, one each (`extra`, -1: none).
struct RowView {
    const float *sp;
    const float4 *vp;
    int head, nvec, extra;
    __device__ inline RowView(const float *sp_, int T, int tid) : sp(sp_)
    {
        head = min(T, (int)(((16u - (uint32_t)((uintptr_t)sp & 15u)) & 15u) >> 2));
        nvec = (T - head) >> 2;
        vp = reinterpret_cast<const float4 *>(sp + head);
        const int tail0 = head + 4 * nvec;
        extra = tid < head ? tid : tid >= 4 && tid - 4 < T - tail0 ? tail0 + tid - 4 : -1;
    }
    __device__ inline int token(int i) const { return head + 4 * i; }
};

// f(t, s_tilde[t]) for every token of a row, in no particular order
template <int NTH = TB_THREADS, typename F>
__device__ inline void scan_row(const RowView &r, int tid, F &&f)
{
    for (int i0 = tid; i0 < r.nvec; i0 += 4 * NTH) {
        float4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = r.vp[min(i0 + j * NTH, r.nvec - 1)];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = i0 + j * NTH;
            if (i < r.nvec) {
                const int t = r.token(i);
                f(t, v[j].x); f(t + 1, v[j].y); f(t + 2, v[j].z); f(t + 3, v[j].w);
            }
        }
    }
    if (r.extra >= 0) f(r.extra, r.sp[r.extra]);
}

struct TopbShared {
    uint32_t kmax[TB_WAVES], kmin[TB_WAVES];
    uint32_t w[TB_WAVES];
    uint32_t found[3];             // bin, entries in front of it, entries in it
    int n;                         // length of the token list
    int n_bin, n_rec;
    uint32_t thr;
    int cut;
};

// Bin that holds the entry of rank r (1-based, counted from bin 0) of hist[0 .. TB_BINS): (bin, entries in front,
// entries in it).  Every thread has read its bins when the first of the two barriers is passed.
__device__ inline void find_bin(const uint32_t *hist, uint32_t r, TopbShared &sh, uint32_t &bin, uint32_t &above, uint32_t &count)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint4 c = reinterpret_cast<const uint4 *>(hist)[tid];
    const uint32_t mine = c.x + c.y + c.z + c.w, incl = wave_scan_u(mine);
    if (lane == 63) sh.w[wave] = incl;
    __syncthreads();
    uint32_t before = incl - mine;
#pragma unroll
    for (int w = 0; w < TB_WAVES; ++w) before += w < wave ? sh.w[w] : 0u;
    if (before < r && r <= before + mine) {
        uint32_t b = 4 * tid, n = c.x;
        if (before + n < r) { before += n; ++b; n = c.y; }
        if (before + n < r) { before += n; ++b; n = c.z; }
        if (before + n < r) { before += n; ++b; n = c.w; }
        sh.found[0] = b; sh.found[1] = before; sh.found[2] = n;
    }
    __syncthreads();
    bin = sh.found[0]; above = sh.found[1]; count = sh.found[2];
}

// Histogram of the workgroup's keys (N per thread, bit e of `valid`: key e counts) over TB_BINS bins of equal width
// that span exactly the keys there are, bin 0 the largest.  The span is what keeps the LDS atomics apart: scores of a
// row crowd into a few bins of a fixed digit of the key.  At least one key must be valid; ends with a barrier.
template <int N>
__device__ inline void span_histogram(const uint32_t (&key)[N], uint32_t valid, uint32_t *hist, TopbShared &sh, uint32_t &top, int &shift)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t mx = 0u, mn = 0xFFFFFFFFu;
#pragma unroll
    for (int e = 0; e < N; ++e)
        if ((valid >> e) & 1u) { mx = max(mx, key[e]); mn = min(mn, key[e]); }
    mx = wave_max_u(mx);
    mn = ~wave_max_u(~mn);
    if (lane == 0) { sh.kmax[wave] = mx; sh.kmin[wave] = mn; }
    reinterpret_cast<uint4 *>(hist)[tid] = make_uint4(0, 0, 0, 0);
    static_assert(TB_BINS == 4 * TB_THREADS, "four bins per thread");
    __syncthreads();
    mx = 0u; mn = 0xFFFFFFFFu;
#pragma unroll
    for (int w = 0; w < TB_WAVES; ++w) { mx = max(mx, sh.kmax[w]); mn = min(mn, sh.kmin[w]); }
    const uint32_t range = mx - mn;
    shift = range < TB_BINS ? 0 : 20 - __builtin_clz(range);
    top = mx;
#pragma unroll
    for (int e = 0; e < N; ++e)
        if ((valid >> e) & 1u) atomicAdd(&hist[(mx - key[e]) >> shift], 1u);
    __syncthreads();
}

// Key and index cut of the k-th best of the workgroup's (key, token) pairs, value descending, token ascending, 1 <= k
// <= their number: the histogram gives its bin, the entries of the bin (usually a handful) are ranked one against
// another.  false when the bin holds more than TB_RANKED of them.
template <int N, typename TOK>
__device__ inline bool kth_best(const uint32_t (&key)[N], uint32_t valid, TOK tok, int k, int T, uint32_t *hist, TopbShared &sh,
                                uint32_t &thr, int &cut)
{
    const int tid = threadIdx.x;
    uint32_t top, bin, above, count;
    int shift;
    if (tid == 0) sh.n_bin = 0;
    span_histogram<N>(key, valid, hist, sh, top, shift);
    find_bin(hist, (uint32_t)k, sh, bin, above, count);
    if (count > (uint32_t)TB_RANKED) return false;
    uint2 *ent = reinterpret_cast<uint2 *>(hist);              // the histogram has been read by everyone
#pragma unroll
    for (int e = 0; e < N; ++e)
        if (((valid >> e) & 1u) && (top - key[e]) >> shift == bin) ent[atomicAdd(&sh.n_bin, 1)] = make_uint2(key[e], (uint32_t)tok(e));
    __syncthreads();
    if (tid < (int)count) {
        const uint2 me = ent[tid];
        int rank = 0, gt = 0, eq = 0;
        for (int j = 0; j < (int)count; ++j) {
            const uint2 o = ent[j];
            gt += o.x > me.x;
            eq += o.x == me.x;
            rank += o.x > me.x || (o.x == me.x && o.y < me.y);
        }
        const int krem = k - (int)above;
        if (rank == krem - 1) {
            sh.thr = me.x;
            sh.cut = krem - gt == eq ? T - 1 : (int)me.y;      // all ties inside: no cut
        }
    }
    __syncthreads();
    thr = sh.thr;
    cut = sh.cut;
    return true;
}

// Appends the tokens t0[j] + 0 .. 3 of the vectors v[j] that `take` to the workgroup's list: one LDS atomic per
// wavefront.  Tokens behind the list's end are counted but not stored.
template <int J, typename F>
__device__ inline void append_tokens(const float4 (&v)[J], const int (&t0)[J], F take, int32_t *list, int cap, TopbShared &sh)
{
    unsigned long long m[4 * J];
    int total = 0;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        m[4 * j] = __ballot(take(t0[j], v[j].x));
        m[4 * j + 1] = __ballot(take(t0[j] + 1, v[j].y));
        m[4 * j + 2] = __ballot(take(t0[j] + 2, v[j].z));
        m[4 * j + 3] = __ballot(take(t0[j] + 3, v[j].w));
    }
#pragma unroll
    for (int e = 0; e < 4 * J; ++e) total += __popcll(m[e]);
    if (total == 0) return;
    const int lane = threadIdx.x & 63;
    int base = 0;
    if (lane == 0) base = atomicAdd(&sh.n, total);
    base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
    for (int e = 0; e < 4 * J; ++e) {
        if (m[e] == 0) continue;
        const int pos = base + lanes_below(m[e]);
        if (((m[e] >> lane) & 1ull) && pos < cap) list[pos] = t0[e >> 2] + (e & 3);
        base += __popcll(m[e]);
    }
}

// A lower bound of the k-th best score of a row, from a sample of TB_ROUND of its values (512 pieces of 128 bytes,
// evenly spaced): the edge of the bin that holds the sample's `rank`-th best, where `rank` lies so far behind the share
// of the k best that falls into a sample that they are all above it (see topb_rank).  A bound that is wrong all the
// same is noticed by the count of what lies above it.
__device__ inline float sample_bound(const RowView &r, int rank, uint32_t *hist, TopbShared &sh)
{
    if (rank >= TB_ROUND) return -INFINITY;
    const int tid = threadIdx.x, pieces = r.nvec >> 3;         // 511 or more (then one is read twice)
    float4 v[TB_REG / 4];
#pragma unroll
    for (int j = 0; j < TB_REG / 4; ++j) {
        const int c = (j * TB_THREADS + tid) >> 3;
        v[j] = r.vp[(int)(((int64_t)c * pieces) >> 9) * 8 + (tid & 7)];
    }
    uint32_t key[TB_REG];
#pragma unroll
    for (int j = 0; j < TB_REG / 4; ++j) {
        key[4 * j] = ordered_key(v[j].x); key[4 * j + 1] = ordered_key(v[j].y);
        key[4 * j + 2] = ordered_key(v[j].z); key[4 * j + 3] = ordered_key(v[j].w);
    }
    uint32_t top, bin, above, count;
    int shift;
    span_histogram<TB_REG>(key, 0xFFFFu, hist, sh, top, shift);
    find_bin(hist, (uint32_t)rank, sh, bin, above, count);
    const uint64_t down = (((uint64_t)bin + 1) << shift) - 1;  // the bin's smallest key is `down` below the largest
    return down >= top ? -INFINITY : float_of_key(top - (uint32_t)down);
}

// tokens [a, b) of the row's vectors (multiples of the round only at a) whose score reaches `bound`, to the list; one that
// is not a number too, as its key may be above the bound's
__device__ inline void collect_above(const RowView &r, int i_begin, int i_end, float bound, int32_t *list, int cap, TopbShared &sh)
{
    const int tid = threadIdx.x;
    constexpr int J = TB_REG / 4;
    float4 nxt[J];
    auto fetch = [&](int i0) {
#pragma unroll
        for (int j = 0; j < J; ++j) nxt[j] = r.vp[min(i0 + j * TB_THREADS + tid, r.nvec - 1)];
    };
    fetch(i_begin);
    for (int i0 = i_begin; i0 < i_end; i0 += J * TB_THREADS) {
        float4 v[J];
        int t0[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int i = i0 + j * TB_THREADS + tid;
            v[j] = nxt[j];
            t0[j] = i < i_end ? r.token(i) : -4;
        }
        if (i0 + J * TB_THREADS < i_end) fetch(i0 + J * TB_THREADS);
        append_tokens<J>(v, t0, [&](int t, float x) { return t >= 0 && !(x < bound); }, list, cap, sh);
    }
}

// one scalar token per thread (or none)
__device__ inline void append_extra(const RowView &r, bool take, int32_t *list, int cap, TopbShared &sh)
{
    if (take) { const int pos = atomicAdd(&sh.n, 1); if (pos < cap) list[pos] = r.extra; }
}

// ------------------------------------------------------------------ one segment, one block size
struct WaveScratch {
    double *phi;        // block sums
    uint8_t *cls;       // block classes: 0 not taken, 1 taken whole, 2 cut to its best tokens
    int capb;           // blocks that fit
};

// Phi of block m of segment [a,b) with block size g: ascending fp64 sum.  `val(t)` yields s_tilde of token t
// (from the wave's LDS copy of the segment when it fits, else from global memory).
template <typename V>
__device__ inline double block_sum(V val, int a, int b, int g, int m)
{
    const int lo = a + m * g, hi = min(lo + g, b);
    double phi = 0.0;
    for (int t = lo; t < hi; ++t) phi += (double)val(t);
    return phi;
}

// number of blocks ranked before block m
__device__ inline int block_rank(int nb, int m, double phi_m, const double *phi_lds)
{
    int r = 0;
#pragma unroll 4
    for (int o = 0; o < nb; ++o) {
        const double po = phi_lds[o];
        r += (po > phi_m || (po == phi_m && o < m)) ? 1 : 0;
    }
    return r;
}

// ranks of the block walk of Alg. 2 without the short last block's own place in the order: how many blocks are taken
// whole, and how many tokens they hold.  q: blocks ranked before the short last one (`ts` < g tokens; unused else)
__device__ inline void whole_blocks(int nb, int g, int ts, int c, int r, int q, int &rstar, int &nwhole)
{
    if (ts == g) {
        rstar = min(nb, c);
        nwhole = rstar * g;
        return;
    }
    if (q < c) {
        if (ts <= r) { rstar = c + 1; nwhole = c * g + ts; } else { rstar = c; nwhole = c * g - g + ts; }
    } else if (q == c) {
        if (ts <= r) { rstar = c + 1; nwhole = c * g + ts; } else { rstar = c; nwhole = c * g; }
    } else {
        rstar = c; nwhole = c * g;
    }
    rstar = min(rstar, nb);
}

// order-preserving signed key of a float (the two zeros: callers pass no -0)
__device__ inline int key_of(float x) { const int b = __float_as_int(x); return b ^ ((b >> 31) & 0x7fffffff); }
constexpr int NO_KEY = (int)0x80000000;
__device__ inline uint64_t ordered_key_d(double x)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x == 0.0 ? 0.0 : x);       // the zeros rank as equal
    return (u >> 63) ? ~u : u | (1ull << 63);
}

// The best `rem` (value descending, index ascending; what is not a number by its bits) of the sz <= 64 scores that lanes
// 0 .. sz - 1 hold; adds their sum to `score`.
constexpr int FEW_TOKENS = 4;              // up to so many are picked one by one, more by their ranks
__device__ inline unsigned long long best_tokens(float v, int sz, int rem, double &score)
{
    const int lane = threadIdx.x & 63;
    v += 0.f;                                                  // no -0
    int key = lane < sz ? max(key_of(v), NO_KEY + 1) : NO_KEY;
    if (rem <= FEW_TOKENS) {
        unsigned long long taken = 0;
#pragma nounroll
        for (int j = 0; j < rem; ++j) {
            const int l = __builtin_ctzll(__ballot(key == wave_max_i(key)));
            taken |= 1ull << l;
            score += (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
            if (lane == l) key = NO_KEY;
        }
        return taken;
    }
    int rk = 0;
#pragma nounroll
    for (int j = 0; j < sz; ++j) {
        const int o = __builtin_amdgcn_readlane(key, j);
        rk += (o > key || (o == key && j < lane)) ? 1 : 0;
    }
    const bool tk = lane < sz && rk < rem;
    score += wave_sum_d(tk ? (double)v : 0.0);
    return __ballot(tk);
}

// ------------------------------------------------------------------ one segment of any length, one block size
// Where the blocks of a segment do not fit LDS, a lane forms the sum of its block in every pass over the blocks (in
// ascending order, as block_sum), and the blocks that are taken are found as everything above a (sum, index) pair: the
// k-th best by digits of eight bits fitted to the sums there are, the last 64 candidates ranked one against another.  Two
// or three passes over the segment for scores in no particular order, however long it is; ranking every block against
// every other took up to 9 s for one segment of 65 536 tokens.
constexpr int ST_BINS = 256, ST_RANKED = 64;
struct StreamScratch {
    uint32_t hist[ST_BINS];
    uint64_t key[ST_RANKED];
    int32_t m[ST_RANKED];
};
static_assert(sizeof(StreamScratch) <= 8 * CAPB, "lies where the block sums of a segment that fits would");
// block m is taken whole when the key of its sum is above `key`, or equal to it and m <= cut; mp: the block of which the
// tokens plo + j with bit j of pmask are taken (-1: none)
struct StreamFill {
    uint64_t key;
    int cut, mp, plo;
    unsigned long long pmask;
    __device__ inline bool whole(uint64_t k, int m) const { return k > key || (k == key && m <= cut); }
};

// Sum of block m, loads in flight; zero behind the last block
template <typename V>
__device__ inline double stream_sum(V val, int a, int b, int g, int m)
{
    const int lo = a + m * g, n = min(g, b - lo);
    double phi = 0.0;
#pragma nounroll
    for (int j0 = 0; j0 < g; j0 += 8) {
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = val(min(lo + min(j0 + j, g - 1), b - 1));
#pragma unroll
        for (int j = 0; j < 8; ++j) phi += j0 + j < n ? (double)v[j] : 0.0;
    }
    return phi;
}

// The blocks of T_k(g); phi(m): sum of block m of nb, any m below nb rounded up to 64.  `part` += the sum of the cut
// block's tokens.
template <typename P, typename V>
__device__ inline StreamFill stream_select(P phi, V val, int a, int b, int g, int bk, StreamScratch &sc, double &part)
{
    const int lane = threadIdx.x & 63, nb = (b - a + g - 1) / g, mt = nb - 1, ts = b - a - mt * g;
    StreamFill f{0, nb, -1, 0, 0};                             // everything
    uint64_t hi = 0, lo = ~0ull;                               // the k-th best key lies in [lo, hi]
    int q = 0;
    {
        const uint64_t kt = ordered_key_d(phi(mt));
#pragma nounroll
        for (int m0 = 0; m0 < nb; m0 += 64) {
            const int m = m0 + lane;
            const uint64_t k = ordered_key_d(phi(m));
            if (m < nb) {
                hi = max(hi, k);
                lo = min(lo, k);
                q += m < mt && k >= kt ? 1 : 0;                // an equal sum ranks first
            }
        }
        hi = wave_max_u64(hi);
        lo = ~wave_max_u64(~lo);
        q = wave_sum_i(q);
    }
    int rstar, nwhole;
    whole_blocks(nb, g, ts, bk / g, bk % g, q, rstar, nwhole);
    if (rstar >= nb) return f;
    const int rem = bk - nwhole;
    int k_rem = rstar + (rem > 0 ? 1 : 0);                     // the cut block is the next one
    for (;;) {
        const uint64_t range = hi - lo;
        const int shift = range < ST_BINS ? 0 : 56 - __builtin_clzll(range);
        reinterpret_cast<uint4 *>(sc.hist)[lane] = make_uint4(0, 0, 0, 0);
        static_assert(ST_BINS == 4 * 64, "four bins per lane");
        __builtin_amdgcn_wave_barrier();
#pragma nounroll
        for (int m0 = 0; m0 < nb; m0 += 64) {
            const int m = m0 + lane;
            const uint64_t k = ordered_key_d(phi(m));
            if (m < nb && k >= lo && k <= hi) atomicAdd(&sc.hist[(int)((hi - k) >> shift)], 1u);
        }
        __builtin_amdgcn_wave_barrier();
        const uint4 c = reinterpret_cast<const uint4 *>(sc.hist)[lane];
        __builtin_amdgcn_wave_barrier();                       // read before the next round's zeros
        const int mine = (int)(c.x + c.y + c.z + c.w), incl = (int)wave_scan_u((uint32_t)mine);
        int bin = 4 * lane, above = incl - mine, count = (int)c.x;
        const int src = __builtin_ctzll(__ballot(above < k_rem && k_rem <= incl));
        if (above + count < k_rem) { above += count; ++bin; count = (int)c.y; }
        if (above + count < k_rem) { above += count; ++bin; count = (int)c.z; }
        if (above + count < k_rem) { above += count; ++bin; count = (int)c.w; }
        bin = __builtin_amdgcn_readlane(bin, src);
        count = __builtin_amdgcn_readlane(count, src);
        k_rem -= __builtin_amdgcn_readlane(above, src);
        hi -= (uint64_t)bin << shift;
        const uint64_t width = (1ull << shift) - 1;
        if (hi - lo > width) lo = hi - width;
        if (rem == 0 && k_rem == count) {                      // the whole bin is inside
            f.key = lo;
            return f;
        }
        if (shift == 0) {                                      // equal sums: lowest indices first
            f.key = hi;
#pragma nounroll
            for (int m0 = 0; m0 < nb; m0 += 64) {
                const int m = m0 + lane;
                const unsigned long long eq = __ballot(m < nb && ordered_key_d(phi(m)) == hi);
                const int c0 = __popcll(eq);
                if (k_rem <= c0) {
                    f.cut = m0 + __builtin_ctzll(__ballot(((eq >> lane) & 1ull) && lanes_below(eq) == k_rem - 1));
                    break;
                }
                k_rem -= c0;
            }
            break;
        }
        if (count <= ST_RANKED) {
            int at = 0;
#pragma nounroll
            for (int m0 = 0; m0 < nb; m0 += 64) {
                const int m = m0 + lane;
                const uint64_t k = ordered_key_d(phi(m));
                const bool in = m < nb && k >= lo && k <= hi;
                const unsigned long long bal = __ballot(in);
                if (in) {
                    sc.key[at + lanes_below(bal)] = k;
                    sc.m[at + lanes_below(bal)] = m;
                }
                at += __popcll(bal);
            }
            __builtin_amdgcn_wave_barrier();
            const uint64_t me = sc.key[min(lane, count - 1)];
            const int m = sc.m[min(lane, count - 1)];
            int rank = 0;
#pragma nounroll
            for (int j = 0; j < count; ++j) {
                const uint64_t o = sc.key[j];
                rank += o > me || (o == me && j < lane) ? 1 : 0;
            }
            const int l = __builtin_ctzll(__ballot(lane < count && rank == k_rem - 1));
            f.key = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(me >> 32), l) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)me, l);
            f.cut = __builtin_amdgcn_readlane(m, l);
            __builtin_amdgcn_wave_barrier();
            break;
        }
    }
    if (rem > 0) {
        f.mp = f.cut--;
        f.plo = a + f.mp * g;
        const int sz = min(g, b - f.plo);
        f.pmask = best_tokens(val(f.plo + min(lane, sz - 1)), sz, rem, part);
    }
    return f;
}

// emit(c0, mask of the tokens c0 + lane that are taken, value) in ascending order; 64 tokens without a taken one may be
// left out
template <typename P, typename V, typename F>
__device__ inline void stream_walk(P phi, V val, int a, int b, int g, const StreamFill &f, F &&emit)
{
    const int lane = threadIdx.x & 63, nb = (b - a + g - 1) / g;
#pragma nounroll
    for (int m0 = 0; m0 < nb; m0 += 64) {
        const int m = m0 + lane;
        const unsigned long long any = __ballot(m < nb && (f.whole(ordered_key_d(phi(m)), m) || m == f.mp));
        if (any == 0) continue;
        const int first = a + m0 * g;
        float nxt = val(min(first + lane, b - 1));             // one chunk ahead
#pragma nounroll
        for (int c0 = 0; c0 < 64 * g && first + c0 < b; c0 += 64) {
            const int t = first + c0 + lane, mm = (c0 + lane) / g;
            const float v = nxt;
            nxt = val(min(t + 64, b - 1));
            const bool take = t < b && ((any >> mm) & 1ull) && (m0 + mm != f.mp || ((f.pmask >> (t - f.plo)) & 1ull));
            const unsigned long long mask = __ballot(take);
            if (mask) emit(first + c0, mask, v);
        }
    }
}

// T_k(g) for segment [a,b) with implicit budget bk (Alg. 2's inner loop).  Calls
// emit(c0, taken_mask, value) for the 64-token chunks with a taken token in ascending order; lane l
// of the chunk starting at token c0 holds the value of token c0 + l.
// Requires 1 <= g <= MAX_G, g <= min(b - a, bk); all arguments wave-uniform.
template <typename V, typename F>
__device__ inline void segment_fill(V val, int a, int b, int g, int bk, WaveScratch ws, F &&emit)
{
    const int lane = threadIdx.x & 63;
    const int len = b - a;
    const int nb = (len + g - 1) / g;
    const int ts = len - (nb - 1) * g;                 // size of the last block, 1..g
    const int mt = nb - 1;
    if (nb > ws.capb) {
        auto phi = [&](int m) { return stream_sum(val, a, b, g, m); };
        double part = 0.0;
        const StreamFill f = stream_select(phi, val, a, b, g, bk, *reinterpret_cast<StreamScratch *>(ws.phi), part);
        stream_walk(phi, val, a, b, g, f, emit);
        return;
    }

    // a sum that is not a number ranks with the infinite ones, so that every place in the order has one block
    for (int m = lane; m < nb; m += 64) {
        const double phi = block_sum(val, a, b, g, m);
        ws.phi[m] = phi == phi ? phi : INFINITY;
    }
    __builtin_amdgcn_wave_barrier();
    // blocks taken whole: the first rstar in rank order; all blocks have g tokens except a short last one,
    // whose rank q decides how many blocks fit
    int rstar, nwhole, q = 0;
    if (ts != g) {
        const double phi_t = ws.phi[mt];
        int cnt = 0;
        for (int o = lane; o < mt; o += 64) cnt += (ws.phi[o] >= phi_t) ? 1 : 0;       // o < mt: an equal sum ranks first
        q = wave_sum_i(cnt);
    }
    const int c = bk / g;
    whole_blocks(nb, g, ts, c, bk - c * g, q, rstar, nwhole);
    const int rem = bk - nwhole;                         // tokens to take from the block ranked rstar

    // classify blocks; remember the cut block
    int mp_local = -1;
    const int picks = rstar + (rem > 0 ? 1 : 0);           // blocks to single out when rstar < nb
    if (rstar < nb && (picks <= 8 || picks * 512 <= nb * nb)) {
        // few blocks are taken: pick them one by one, best first (sum descending, index ascending), instead of
        // ranking every block against every other
        for (int m = lane; m < nb; m += 64) ws.cls[m] = 0;
        __builtin_amdgcn_wave_barrier();
        for (int sel = 0; sel < picks; ++sel) {
            double bp = -INFINITY;
            int bm = 0x7fffffff;
            for (int m = lane; m < nb; m += 64) {
                const double pm = ws.phi[m];
                if (ws.cls[m] == 0 && (pm > bp || (pm == bp && m < bm))) { bp = pm; bm = m; }
            }
            wave_argmax(bp, bm);
            if (lane == 0) ws.cls[bm] = sel < rstar ? 1 : 2;
            if (sel == rstar) mp_local = bm;
            __builtin_amdgcn_wave_barrier();
        }
    } else {
        for (int m = lane; m < nb; m += 64) {
            int rk = (rstar >= nb) ? 0 : block_rank(nb, m, ws.phi[m], ws.phi);
            uint8_t c = (rk < rstar) ? 1 : ((rk == rstar && rem > 0) ? 2 : 0);
            ws.cls[m] = c;
            if (c == 2) mp_local = m;
        }
        __builtin_amdgcn_wave_barrier();
    }
    const int mp = wave_max_i(mp_local);

    // inside the cut block: its best rem tokens
    unsigned long long pmask = 0;
    int plo = 0;
    if (mp >= 0) {
        plo = a + mp * g;
        const int sz = min(g, b - plo);
        double sum = 0.0;
        pmask = best_tokens(val(plo + min(lane, sz - 1)), sz, rem, sum);
    }

    for (int c0 = a; c0 < b; c0 += 64) {
        const int t = c0 + lane;
        const bool live = t < b;
        float v = 0.f;
        bool take = false;
        if (live) {
            v = val(t);
            const int c = ws.cls[(t - a) / g];
            take = (c == 1) || (c == 2 && ((pmask >> (t - plo)) & 1ull));
        }
        emit(c0, __ballot(take), v);
    }
    __builtin_amdgcn_wave_barrier();
}

// ------------------------------------------------------------------ sums that cannot round
// The scores of a segment are fp32 values, summed in fp64.  Every value and every partial sum is a multiple of the
// last bit of the smallest nonzero one, and the sum of n of them stays below n times twice the power of two of the
// largest, so as long as
//     exponent range + 24 bits of mantissa + ceil(log2 n) <= 53
// no partial sum rounds in ANY order: prefix sums by lane shuffles, differences of prefixes and sums over arbitrary
// subsets then equal the ordered sums bit for bit.  Segments whose scores span more (23 powers of two at 64 tokens, 17
// at 4 095) take ordered sums.
// biggest: the largest |score| of a segment; smallest: the smallest nonzero one as its bits doubled, less one; total:
// the sum (not finite when a score is not); n >= 2
__device__ inline void note_size(float v, float &biggest, uint32_t &smallest)
{
    biggest = fmaxf(biggest, fabsf(v));
    smallest = min(smallest, (__float_as_uint(v) << 1) - 1u);  // zero becomes the largest value
}
__device__ inline bool sums_are_exact(float biggest, uint32_t smallest, double total, int n)
{
    const int hi = max(wave_max_i(__float_as_int(biggest)) >> 23, 1), lo = max((int)((~wave_max_u(~smallest) + 1u) >> 24), 1);
    return hi - lo <= 29 - (32 - __builtin_clz(n - 1)) && fabs(total) < INFINITY;
}

// Lane of the largest x (lowest lane among equal ones) whose key, of x rounded to fp32, is not NO_KEY: one 32-bit
// reduction, and an fp64 one only where several x round to the same fp32 value.
__device__ inline int best_lane(double x, int key)
{
    const int mk = wave_max_i(key);
    unsigned long long m = __ballot(key == mk);
    if (m & (m - 1)) {
        const double mx = wave_max_d(key == mk ? x : -INFINITY);
        m = __ballot(key == mk && x == mx);
    }
    return __builtin_ctzll(m);
}

// T_k(g) of a segment of n tokens whose sums are exact; pre[x], 0 <= x <= n, is the sum of its first x scores.  Returns
// Score_k(g).  Up to 64 blocks: one per lane, the blocks taken whole are the bits of `blocks`.  More: block lane + 64 i
// is taken whole when bit i of the lane's `whole` is set.  Tokens plo + j of the cut block (plo < 0: none) are taken
// when bit j of pmask is set.  inv: see CandList.
struct Fill {
    unsigned long long blocks, pmask;
    uint32_t whole;
    int plo;
};
constexpr int FEW_PICKS = 16;              // of more than 64 blocks, so many are picked one by one, more by bisection of their sums

__device__ inline double fill_prefix(const double *pre, int n, int g, int inv, int bk, Fill &f)
{
    const int lane = threadIdx.x & 63;
    const int nb = ((n + g - 1) * inv) >> CAND_INV_BITS, ts = n - (nb - 1) * g;
    const int c = (bk * inv) >> CAND_INV_BITS, r = bk - c * g;
    int rstar, nwhole, q = 0;
    double score = 0.0;
    f.plo = -1;
    f.pmask = 0;
    int rem;
    if (nb <= 64) {
        const int x0 = min(lane * g, n), x1 = min(x0 + g, n);
        const double phi = pre[x1] - pre[x0];
        if (ts != g) {
            const double pt = readlane_d(phi, nb - 1);
            q = __popcll(__ballot(lane < nb - 1 && phi >= pt));     // an equal sum ranks first
        }
        whole_blocks(nb, g, ts, c, r, q, rstar, nwhole);
        if (rstar >= nb) {
            f.blocks = ~0ull;
            return pre[n];
        }
        rem = bk - nwhole;
        int key = lane < nb ? key_of((float)phi) : NO_KEY;
        f.blocks = 0;
        // pick the blocks one by one, best first (sum descending, index ascending); the last pick is the cut block
        const int picks = rstar + (rem > 0 ? 1 : 0);
#pragma nounroll
        for (int sel = 0; sel < picks; ++sel) {
            const int m = best_lane(phi, key);
            if (sel < rstar) {
                f.blocks |= 1ull << m;
                score += readlane_d(phi, m);
                if (lane == m) key = NO_KEY;
            } else {
                f.plo = m * g;
            }
        }
    } else {
        auto phi = [&](int m) { return pre[min(m * g + g, n)] - pre[m * g]; };
        if (ts != g) {
            const double pt = phi(nb - 1);
            int cnt = 0;
#pragma nounroll
            for (int m = lane; m < nb - 1; m += 64) cnt += phi(m) >= pt ? 1 : 0;
            q = wave_sum_i(cnt);
        }
        whole_blocks(nb, g, ts, c, r, q, rstar, nwhole);
        f.whole = 0;
        if (rstar >= nb) {
            f.whole = ~0u;
            return pre[n];
        }
        rem = bk - nwhole;
        int one_by_one = rstar;
        if (rstar > FEW_PICKS) {
            one_by_one = 0;
            // the largest key with at least rstar blocks at or above it, by bisection
            uint64_t lo = 0, hi = ~0ull;                       // count(>= lo) >= rstar
#pragma nounroll
            while (lo < hi) {
                const uint64_t mid = lo + ((hi - lo) >> 1) + 1;
                int cnt = 0;
#pragma nounroll
                for (int m = lane; m < nb; m += 64) cnt += ordered_key_d(phi(m)) >= mid ? 1 : 0;
                if (wave_sum_i(cnt) >= rstar) lo = mid; else hi = mid - 1;
            }
            int gt = 0;
#pragma nounroll
            for (int m = lane; m < nb; m += 64) gt += ordered_key_d(phi(m)) > lo ? 1 : 0;
            int ties = rstar - wave_sum_i(gt);                 // ties at the threshold: lowest indices first
            double part = 0.0;
#pragma nounroll
            for (int i = 0; i < (nb + 63) / 64; ++i) {
                const int m = lane + 64 * i;
                const double x = m < nb ? phi(m) : 0.0;
                const uint64_t key = ordered_key_d(x);
                const unsigned long long eq = __ballot(m < nb && key == lo);
                const bool take = m < nb && (key > lo || (key == lo && lanes_below(eq) < ties));
                ties -= min(ties, (int)__popcll(eq));
                if (take) { f.whole |= 1u << i; part += x; }
            }
            score = wave_sum_d(part);
        }
        const int picks = one_by_one + (rem > 0 ? 1 : 0);
#pragma nounroll
        for (int sel = 0; sel < picks; ++sel) {
            double mx = -INFINITY;
            int bm = 0x7fffffff;
#pragma nounroll
            for (int m = lane, i = 0; m < nb; m += 64, ++i) {
                const double x = phi(m);
                if (!((f.whole >> i) & 1u) && x > mx) { mx = x; bm = m; }
            }
            const double all = wave_max_d(mx);
            bm = -wave_max_i(mx == all ? -bm : -0x7fffffff);
            if (sel < one_by_one) {
                score += all;
                if (lane == (bm & 63)) f.whole |= 1u << (bm >> 6);
            } else {
                f.plo = bm * g;
            }
        }
    }
    if (rem > 0) {
        const int sz = min(g, n - f.plo), t = f.plo + min(lane, sz - 1);
        f.pmask = best_tokens((float)(pre[t + 1] - pre[t]), sz, rem, score);     // the scores themselves, exactly
    }
    return score;
}

// What a wavefront needs to know of its problem and call
struct SearchCtx {
    const float *sp;           // the problem's scores
    int32_t *block_size;       // its row
    int32_t *out;              // its idx_out row
    int budget;
    float tau;
    int cand_g, cand_inv, n_cand;          // lane c: candidate c (the wavefront's copy of CandList)
    __device__ inline SearchCtx(const float *s_tilde, int T, int p, int32_t *bs, int max_segments, int32_t *idx, int budget_, float tau_,
                                const CandList &cand)
        : sp(s_tilde + (int64_t)p * T), block_size(bs + (int64_t)p * max_segments), out(idx ? idx + (int64_t)p * budget_ : nullptr),
          budget(budget_), tau(tau_), cand_g(cand.g[threadIdx.x & (MAX_CAND - 1)]), cand_inv(cand.inv[threadIdx.x & (MAX_CAND - 1)]),
          n_cand(cand.n)
    {
    }
    // R_k(g) >= tau  <=>  Score_k(g) >= tau * Score_base.  tau is widened here each time: two vector registers less.
    __device__ inline double need(double base) const
    {
        float t = tau;
        asm volatile("" : "+s"(t));
        return (double)t * base;
    }
};

// appends the tokens c0 + lane of mask m, ascending, at `pos` of the problem's idx_out row
__device__ inline void put_tokens(const SearchCtx &x, int &pos, int c0, unsigned long long m)
{
    const int lane = threadIdx.x & 63, jo = pos + lanes_below(m);
    if (((m >> lane) & 1ull) && jo < x.budget) x.out[jo] = c0 + lane;
    pos += __popcll(m);
}
// T_k(1) = T_topB & S_k (b_k is the implicit budget); J loads in flight
template <int J>
__device__ inline void put_topb(const SearchCtx &x, const SegRec &r)
{
    const int lane = threadIdx.x & 63;
    int pos = r.out;
#pragma nounroll
    for (int c0 = r.a; c0 < r.b; c0 += 64 * J) {
        float v[J];
#pragma unroll
        for (int j = 0; j < J; ++j) v[j] = x.sp[min(c0 + 64 * j + lane, r.b - 1)];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int t = c0 + 64 * j + lane;
            put_tokens(x, pos, c0 + 64 * j, __ballot(t < r.b && in_topb(v[j], t, (uint32_t)r.g, r.pos)));
        }
    }
}

// A segment's scores as search_exact takes them, behind its end those of its last token: up to 64 tokens one per lane, up
// to 128 two; of longer segments nothing is needed.
__device__ inline float2 first_scores(const float *sp, const SegRec &r)
{
    const int lane = threadIdx.x & 63, last = r.b - 1;
    if (r.b - r.a <= 64) return make_float2(sp[min(r.a + lane, last)], 0.f);
    return make_float2(sp[min(r.a + 2 * lane, last)], sp[min(r.a + 2 * lane + 1, last)]);
}

// The search of one segment by one wavefront: Score_base, then the candidates largest first, g_k* and (EMIT) T_k(g_k*) in
// ascending order at the record's `out`.  false, and nothing written, when its sums may round.  pre: LDS for n + 1 (at
// least 129) prefix sums; v: first_scores of the segment.
//
// What bounds this is the length of the wavefront's instruction stream, so a segment's scores are turned into prefix sums
// once, where a block's sum is one subtraction for every candidate.
template <bool EMIT>
__device__ inline bool search_exact(const SearchCtx &x, const SegRec &r, float2 v, double *pre)
{
    const int lane = threadIdx.x & 63;
    const int a = r.a, n = r.b - a, bk = r.bk, gcap = min(n, bk);                // G_k: g <= min(|S_k|, b_k, g_max)
    const float *sp = x.sp;
    // ---- Score_base, prefix sums (R tokens per lane and round of 64 R), sizes of the scores
    double base, total;
    float big = 0.f;
    uint32_t small = ~0u;
    const float thr = r.g ? float_of_key((uint32_t)r.g) : -INFINITY;             // key 0: everything is inside
    auto top = [&](float v, int t) { return v > thr || (v == thr && a + t <= r.pos); };    // finite scores: as in_topb
    if (n <= 64) {
        const float w = lane < n ? v.x : 0.f;
        note_size(w, big, small);
        base = top(w, lane) && lane < n ? (double)w : 0.0;
        const double s = wave_scan_d((double)w);
        if (lane == 0) pre[0] = 0.0;
        pre[lane + 1] = s;
        total = readlane_d(s, 63);
    } else if (n <= 128) {
        const int t0 = 2 * lane;
        const float w0 = t0 < n ? v.x : 0.f, w1 = t0 + 1 < n ? v.y : 0.f;
        note_size(w0, big, small);
        note_size(w1, big, small);
        base = (top(w0, t0) && t0 < n ? (double)w0 : 0.0) + (top(w1, t0 + 1) && t0 + 1 < n ? (double)w1 : 0.0);
        const double sum = (double)w0 + (double)w1, s = wave_scan_d(sum);
        if (lane == 0) pre[0] = 0.0;
        pre[t0 + 1] = s - (double)w1;
        pre[t0 + 2] = s;
        total = readlane_d(s, 63);
    } else {
        base = total = 0.0;
#pragma nounroll
        for (int c0 = 0; c0 <= n; c0 += 512) {                 // pre[n] included
            const int t0 = c0 + 8 * lane;
            float w[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) w[j] = sp[min(a + t0 + j, r.b - 1)];
            double sum = 0.0;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (t0 + j >= n) w[j] = 0.f;
                note_size(w[j], big, small);
                sum += (double)w[j];
                base += t0 + j < n && top(w[j], t0 + j) ? (double)w[j] : 0.0;
            }
            const double s = total + wave_scan_d(sum);
            double y = s - sum;
            if (t0 <= n) {
#pragma unroll
                for (int j = 0; j < 8; ++j) { pre[t0 + j] = y; y += (double)w[j]; }
            }
            total = readlane_d(s, 63);
        }
    }
    __builtin_amdgcn_wave_barrier();
    if (!sums_are_exact(big, small, total, n)) return false;

    // R_k(g) >= tau  <=>  Score_k(g) >= tau * Score_base; g_k* is the first accepted, largest first (Eq. gk_star)
    const double need = x.need(wave_sum_d(base));
    int gstar = 0, inv = 0;
    Fill f;
#pragma nounroll
    for (int c = x.n_cand - 1; c >= 0; --c) {
        const int g = __builtin_amdgcn_readlane(x.cand_g, c);
        if (g > gcap) continue;
        if (g == 1) { gstar = 1; break; }                      // token level: the unconditional last resort
        inv = __builtin_amdgcn_readlane(x.cand_inv, c);
        if (fill_prefix(pre, n, g, inv, bk, f) >= need) { gstar = g; break; }
    }
    if (lane == 0) x.block_size[r.k] = gstar;
    if (EMIT && gstar == 1) put_topb<1>(x, r);
    if (EMIT && gstar > 1) {
        int pos = r.out;
        const bool few = n <= 64 * gstar;
#pragma nounroll
        for (int c0 = 0; c0 < n; c0 += 64) {
            const int t = c0 + lane, m = (t * inv) >> CAND_INV_BITS, j = t - f.plo;
            bool tk;
            if (few) tk = (f.blocks >> m) & 1ull;
            else tk = ((uint32_t)__shfl((int)f.whole, m & 63) >> (m >> 6)) & 1u;
            put_tokens(x, pos, a + c0, __ballot(t < n && (tk || (f.plo >= 0 && j >= 0 && j < 64 && ((f.pmask >> j) & 1ull)))));
        }
    }
    __builtin_amdgcn_wave_barrier();                           // `pre` is reused by the next segment
    return true;
}

// The search of a segment of any length, from memory (it stays in the L2 cache): what search_exact does, for segments
// whose prefix sums do not fit LDS, and where sums may round with ordered ones.  kept: LDS for n_kept block sums.  Bound by
// the latency of one wavefront's loads.  Top-B and search, 8 rows of 32 736 tokens: segments of 800 54 us, of 4 000 168 us
// (529 and 3 909 with prefix sums of 4 095 tokens in the LDS of the Top-B workgroup, a few segments at a time); of 131 040,
// mean length 64, sums that may round: 55 us (1 317); one segment of 16 384 among short ones: 270 us (896 ms).
template <bool EMIT>
__device__ inline void search_streamed(const SearchCtx &x, const SegRec &r, StreamScratch &sc, double *kept, int n_kept)
{
    const int lane = threadIdx.x & 63, a = r.a, b = r.b, n = b - a, gcap = min(n, r.bk);
    const float *sp = x.sp;
    auto val = [&](int t) { return sp[t]; };
    double base = 0.0, total = 0.0;
    float big = 0.f;
    uint32_t small = ~0u;
#pragma nounroll
    for (int c0 = a; c0 < b; c0 += 512) {
        float w[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) w[j] = sp[min(c0 + 64 * j + lane, b - 1)];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int t = c0 + 64 * j + lane;
            if (t >= b) w[j] = 0.f;
            note_size(w[j], big, small);
            total += (double)w[j];
            base += t < b && in_topb(w[j], t, (uint32_t)r.g, r.pos) ? (double)w[j] : 0.0;
        }
    }
    const bool exact = sums_are_exact(big, small, wave_sum_d(total), n);
    if (exact) base = wave_sum_d(base);
    else {
        base = 0.0;
        float nxt = sp[min(a + lane, b - 1)];
#pragma nounroll
        for (int c0 = a; c0 < b; c0 += 64) {
            const int t = c0 + lane;
            const float v = nxt;
            nxt = sp[min(t + 64, b - 1)];
            base = add_in_order(base, __ballot(t < b && in_topb(v, t, (uint32_t)r.g, r.pos)), v);
        }
    }
    const double need = x.need(base);
    int gstar = 0;
#pragma nounroll
    for (int c = x.n_cand - 1; c >= 0; --c) {
        const int g = __builtin_amdgcn_readlane(x.cand_g, c);
        if (g > gcap) continue;
        if (g == 1) { gstar = 1; break; }
        const int nb = (n + g - 1) / g;
        const bool keep = nb <= n_kept;
        if (keep) {
#pragma nounroll
            for (int m = lane; m < nb; m += 64) kept[m] = stream_sum(val, a, b, g, m);
            __builtin_amdgcn_wave_barrier();
        }
        auto phi = [&](int m) { return keep ? kept[min(m, nb - 1)] : stream_sum(val, a, b, g, m); };
        double score = 0.0;
        const StreamFill f = stream_select(phi, val, a, b, g, r.bk, sc, score);
        int pos = r.out;
        bool writing = false;                                  // the accepted candidate: its tokens
        for (;;) {
            if (exact && !writing) {
                double sum = 0.0;
#pragma nounroll
                for (int m = lane; m < nb; m += 64) {
                    const double p = phi(m);
                    sum += f.whole(ordered_key_d(p), m) ? p : 0.0;
                }
                score += wave_sum_d(sum);
            } else {
                if (!writing) score = 0.0;
                stream_walk(phi, val, a, b, g, f, [&](int c0, unsigned long long m, float v) {
                    if (EMIT && writing) put_tokens(x, pos, c0, m);
                    else score = add_in_order(score, m, v);
                });
            }
            if (writing || !(score >= need)) break;
            gstar = g;
            if (!EMIT) break;
            writing = true;
        }
        __builtin_amdgcn_wave_barrier();                       // `kept` is filled anew by the next candidate
        if (gstar) break;
    }
    if (lane == 0) x.block_size[r.k] = gstar;
    if (EMIT && gstar == 1) put_topb<8>(x, r);
}

// What the search that also selects needs of the Top-B kernel (see topb_kernel<true, ..>)
struct PlanArgs {
    SegRec *list;                // [P][capacity] records
    int32_t *counts;             // [P]
    int capacity;
    int32_t *idx_out, *n_sel_out;
};

// ---- several workgroups per row (few problems in a call, long rows: one workgroup per row would be bound by the
// latency of its own loads).  Grid of slices: every workgroup forms the row's bound from the same sample and
// collects its slice's tokens above it.
__global__ void __launch_bounds__(TB_THREADS)
topb_collect_kernel(Dims d, const float *s_tilde, int sample_rank, int pre_cap, uint2 *pre_list, int32_t *pre_cnt)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t sh_dyn[];   // histogram, then the list
    __shared__ TopbShared sh;
    uint32_t *hist = sh_dyn;
    int32_t *list = reinterpret_cast<int32_t *>(sh_dyn + TB_BINS);
    const int p = grid_problem(d), sl = grid_part(d), n_slices = grid_parts(d), tid = threadIdx.x;
    const RowView r(s_tilde + (int64_t)p * d.T, d.T, tid);
    if (tid == 0) sh.n = 0;
    const float bound = r.nvec > TB_ROUND / 4 ? sample_bound(r, sample_rank, hist, sh) : -INFINITY;
    __syncthreads();
    const int per = (r.nvec + n_slices - 1) / n_slices;
    const int i0 = min(sl * per, r.nvec), i1 = min(i0 + per, r.nvec);
    if (i0 < i1) collect_above(r, i0, i1, bound, list, pre_cap, sh);
    if (sl == 0) append_extra(r, r.extra >= 0 && !(r.sp[max(r.extra, 0)] < bound), list, pre_cap, sh);
    __syncthreads();
    const int64_t o = (int64_t)p * n_slices + sl;
    for (int i = tid; i < min(sh.n, pre_cap); i += TB_THREADS) pre_list[o * pre_cap + i] = make_uint2(ordered_key(r.sp[list[i]]), (uint32_t)list[i]);
    if (tid == 0) pre_cnt[o] = sh.n;
}

// ------------------------------------------------------------------ Top-B of a row that a workgroup holds in registers
constexpr int RR_KEYS = 16;                        // scores per thread of a row, and of a list
constexpr int RUN = 4;                             // segments per thread where there are more of them than threads
constexpr int RR_RANKED = 64;                      // entries of one bin that are ranked one against another

template <int NTH> struct RowShared {
    uint32_t most[NTH / 64], least[NTH / 64], w[NTH / 64];
    uint32_t found[3];                             // bin, entries in front of it, entries in it
    int n_bin, n_long, long_at;
    uint32_t thr;
    int cut;
};

// adds to a counter in LDS, a lane at a time; few lanes: the compiler's own form scans the wavefront first, and is forty instructions
__device__ inline int lds_add(int *counter, int v)
{
    int r;
    asm volatile("ds_add_rtn_u32 %0, %1, %2\n\ts_waitcnt lgkmcnt(0)" : "=&v"(r) : "v"((uint32_t)(uintptr_t)(__attribute__((address_space(3))) int *)counter), "v"(v) : "memory");
    return r;
}

// sum of the wavefronts' totals in front of this one; `mine` is the lane's inclusive sum.  One barrier.
template <int NTH>
__device__ inline uint32_t waves_before(uint32_t mine, RowShared<NTH> &sh)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 63) sh.w[wave] = mine;
    __syncthreads();
    uint32_t before = 0;
#pragma unroll
    for (int w = 0; w < NTH / 64 - 1; ++w) before += w < wave ? sh.w[w] : 0u;
    return before;
}

// The scores that a workgroup looks at: held in registers (thread i: entries i + e * NTH of n), ...
template <int NTH, int N, bool TOK> struct HeldScores {
    uint32_t key[N];
    int tok[TOK ? N : 1];
    int n;
    template <typename F>
    __device__ __forceinline__ void each(F &&f) const       // f(key, token), for what this thread holds
    {
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const int i = (int)threadIdx.x + e * NTH;
            if (e * NTH < n && i < n) {            // the first is uniform
                if constexpr (TOK) f(key[e], tok[e]);
                else f(key[e], i);
            }
        }
    }
};
// ... or read from the row each time
template <int NTH> struct RowScores {
    RowView r;
    template <typename F>
    __device__ __forceinline__ void each(F &&f) const
    {
        scan_row<NTH>(r, threadIdx.x, [&](int t, float x) __attribute__((always_inline)) { f(ordered_key(x), t); });
    }
};

// Key and index cut of the k-th best of the scores, 1 <= k <= their number: a histogram over the span of the keys gives the
// k-th one's bin; a bin of few entries is ranked, one of many is the next span.  sp, T: the row, T - 1 the cut that cuts nothing.
template <int NTH, typename S>
__device__ __forceinline__ void row_kth_best(const S &sc, const float *sp, int T, int k, uint32_t *hist, RowShared<NTH> &sh, uint32_t &thr, int &cut)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t most = 0u, least = 0xFFFFFFFFu;
    sc.each([&](uint32_t key, int) { most = max(most, key); least = min(least, key); });
    most = wave_max_u(most);
    least = ~wave_max_u(~least);
    if (lane == 0) { sh.most[wave] = most; sh.least[wave] = least; }
    if (tid == 0) sh.n_bin = 0;
    reinterpret_cast<uint4 *>(hist)[tid] = make_uint4(0, 0, 0, 0);         // four bins per thread
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NTH / 64; ++w) { most = max(most, sh.most[w]); least = min(least, sh.least[w]); }
    constexpr int BITS = NTH == 1024 ? 12 : NTH == 512 ? 11 : 10;
    static_assert(4 * NTH == 1 << BITS, "bins");
    uint32_t count;
#pragma nounroll
    for (bool again = false;; again = true) {
        if (again) {                               // everyone has read its bins
            reinterpret_cast<uint4 *>(hist)[tid] = make_uint4(0, 0, 0, 0);
            __syncthreads();
        }
        const uint32_t range = most - least;
        const int shift = max(0, 32 - BITS - __builtin_clz(range | 1u));
        sc.each([&](uint32_t key, int) {
            const uint32_t down = most - key;      // wraps above `most`
            if (down <= range) atomicAdd(&hist[down >> shift], 1u);
        });
        __syncthreads();
        const uint4 c = reinterpret_cast<const uint4 *>(hist)[tid];
        const uint32_t mine = c.x + c.y + c.z + c.w, incl = wave_scan_u(mine);
        uint32_t before = waves_before<NTH>(incl, sh) + incl - mine;
        if (before < (uint32_t)k && (uint32_t)k <= before + mine) {
            uint32_t b = 4 * tid, n = c.x;
            if (before + n < (uint32_t)k) { before += n; ++b; n = c.y; }
            if (before + n < (uint32_t)k) { before += n; ++b; n = c.z; }
            if (before + n < (uint32_t)k) { before += n; ++b; n = c.w; }
            sh.found[0] = b; sh.found[1] = before; sh.found[2] = n;
        }
        __syncthreads();
        k -= (int)sh.found[1];
        count = sh.found[2];
        const uint32_t top = most - (sh.found[0] << shift), low = top - ((1u << shift) - 1u);       // of the bin; low wraps below key 0
        least = low > top ? least : max(least, low);
        most = top;
        if (count <= (uint32_t)RR_RANKED || most == least) break;
    }
    if (count <= (uint32_t)RR_RANKED) {
        uint2 *ent = reinterpret_cast<uint2 *>(hist);          // everyone has read its bins
        sc.each([&](uint32_t key, int t) { if (key <= most && key >= least) ent[lds_add(&sh.n_bin, 1)] = make_uint2(key, (uint32_t)t); });
        __syncthreads();
        if (tid < (int)count) {
            const uint2 me = ent[tid];
            int rank = 0, gt = 0, eq = 0;
#pragma nounroll
            for (int j0 = 0; j0 < (int)count; j0 += 4) {
                uint2 o[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) o[j] = ent[min(j0 + j, (int)count - 1)];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int there = j0 + j < (int)count, above = there & (o[j].x > me.x), same = there & (o[j].x == me.x);
                    gt += above;
                    eq += same;
                    rank += above | (same & (o[j].y < me.y));
                }
            }
            if (rank == k - 1) {
                sh.thr = me.x;
                sh.cut = k - gt == eq ? T - 1 : (int)me.y;     // all ties inside: no cut
            }
        }
        __syncthreads();
        thr = sh.thr;
        cut = sh.cut;
        return;
    }
    // more ties than are ranked: k of `count`, lowest indices first
    thr = most;
    cut = T - 1;
    if (k == (int)count) return;
#pragma nounroll
    for (int c0 = 0; c0 < T; c0 += NTH) {
        const int t = c0 + tid;
        const bool tie = t < T && ordered_key(sp[t]) == thr;
        const unsigned long long bal = __ballot(tie);
        if (lane == 0) sh.most[wave] = (uint32_t)__popcll(bal);
        __syncthreads();
        int before = 0, total = 0;
        for (int w = 0; w < NTH / 64; ++w) { const int c = (int)sh.most[w]; if (w < wave) before += c; total += c; }
        if (tie && before + lanes_below(bal) + 1 == k) sh.cut = t;
        __syncthreads();
        if (k <= total) { cut = sh.cut; return; }
        k -= total;
    }
}

// Tokens at or above a row's bound, collected by several workgroups per row
struct Candidates {
    const uint2 *entries;        // [P][n_slices][cap]: key, token
    const int32_t *counts;       // [P][n_slices], more than cap when some were dropped
    int n_slices, cap;
};


// LDS of row_rank_kernel: the histogram; per segment its first token, its Top-B tokens and one of them; and (not LISTED) a bit per token where a segment begins, with the
// number of them in front of each word
constexpr int RR_LDS_MOST = 150 * 1024;
struct RowLds {
    int cnt, one, off, bits, before, bytes;
    __host__ __device__ RowLds(bool listed, int nth, int T, int K)
    {
        const int words = listed ? 0 : (T + 31) / 32, seg = 4 * ((K + 4) & ~3);
        cnt = 16 * nth;
        one = cnt + seg;
        off = one + seg;
        bits = off + seg;
        before = bits + 4 * words;
        bytes = (before + 4 * words + 15) & ~15;
    }
};

// grid (P).  What topb_kernel does, 0 < k = B < T, for rows of up to N * NTH tokens (LISTED: for longer ones, of which
// other workgroups have listed the tokens above a bound; a list that is none, of fewer than k or more than there is room for,
// leaves the row to be read again and again).
//
// What bounds it: the latency of its steps and the instructions of its threads (one costs a compute unit 4 cycles per
// wavefront and SIMD).  So a row gets as many threads as hold it with 16 scores each, and what a row has no tokens for is
// jumped over; a token finds its segment by counting bits, and a segment with one token remembers it, so that the tokens
// need no second look.  The kernel alone, 2 rows of 2 032 tokens 11.1 -> 7.2 us, 8 rows of 8 160 14.8 -> 10.4 against 1 024 threads
// that list the tokens and look each segment up by halves; 8 rows of 131 040 from eight lists each 15.9 -> 12.6.
template <bool PLAN, int NTH, bool LISTED, int N = RR_KEYS>
__global__ void __launch_bounds__(NTH, 4)
row_rank_kernel(Dims d, const float *s_tilde, int k, int32_t *thr_out, SegView sv, int32_t *seg_budget, int32_t *block_size, PlanArgs pa,
                Candidates cd, int most_segments)
{
    extern __shared__ __attribute__((aligned(16))) char sh_row[];
    __shared__ __attribute__((aligned(16))) RowShared<NTH> sh;
    const int p = blockIdx.x, T = d.T, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const RowLds lds(LISTED, NTH, T, most_segments);
    uint32_t *hist = reinterpret_cast<uint32_t *>(sh_row);
    int32_t *cnt = reinterpret_cast<int32_t *>(sh_row + lds.cnt), *one = reinterpret_cast<int32_t *>(sh_row + lds.one);
    int32_t *off = reinterpret_cast<int32_t *>(sh_row + lds.off);
    uint32_t *bits = reinterpret_cast<uint32_t *>(sh_row + lds.bits), *before = reinterpret_cast<uint32_t *>(sh_row + lds.before);
    const float *sp = s_tilde + (int64_t)p * T;
    const int seq = seq_of_problem(d, p);
    const int32_t *seg_off = sv.seg_off + sv.seq_ptr[seq];
    const int K = seg_budget ? sv.seq_ptr[seq + 1] - sv.seq_ptr[seq] - 1 : -1;
    const int64_t row = (int64_t)p * sv.max_segments;

    int32_t o[4];                                  // the first offsets, on their way with the scores
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = K >= 0 ? seg_off[min(tid + i * NTH, K)] : 0;        // K < 0: there may be no offsets
    HeldScores<NTH, N, LISTED> held;
    held.n = T;
    const int words = LISTED ? 0 : (T + 31) / 32;
    if constexpr (LISTED) {
        // the lists one behind another
        const int n = lane < cd.n_slices ? cd.counts[(int64_t)p * cd.n_slices + lane] : 0;
        const int upto = (int)wave_scan_u((uint32_t)n);
        held.n = __any(n > cd.cap) ? 0 : __builtin_amdgcn_readlane(upto, 63);
        if (held.n < k || held.n > N * NTH) held.n = 0;
#pragma unroll
        for (int e = 0; e < N; ++e) {
            if (e * NTH < held.n) {
                const int i = tid + e * NTH;
                int slice = 0, first = 0;          // of the entry
#pragma nounroll
                for (int sl = 0; sl < cd.n_slices - 1; ++sl) {
                    const int end = __builtin_amdgcn_readlane(upto, sl);
                    if (end <= i) { slice = sl + 1; first = end; }
                }
                if (i < held.n) {
                    const uint2 c = cd.entries[((int64_t)p * cd.n_slices + slice) * cd.cap + (i - first)];
                    held.key[e] = c.x;
                    held.tok[e] = (int)c.y;
                }
            }
        }
    } else {
        float v[N];
#pragma unroll
        for (int e = 0; e < N; ++e)
            if (e * NTH < T) v[e] = sp[min(tid + e * NTH, T - 1)];
#pragma nounroll
        for (int w = tid; w < words; w += NTH) bits[w] = 0u;
#pragma unroll
        for (int e = 0; e < N; ++e)
            if (e * NTH < T) held.key[e] = ordered_key(v[e]);
    }
    if (tid == 0) sh.n_long = sh.long_at = 0;
    if (!LISTED) __syncthreads();                  // the bits are clear
#pragma nounroll
    for (int j0 = tid; j0 <= K; j0 += 4 * NTH) {
        if (j0 >= 4 * NTH)
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = seg_off[min(j0 + i * NTH, K)];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (j0 + i * NTH <= K) {
                off[j0 + i * NTH] = o[i];
                cnt[j0 + i * NTH] = 0;
                if (!LISTED && o[i] < T) atomicOr(&bits[o[i] >> 5], 1u << (o[i] & 31));
            }
    }
    uint32_t thr;
    int cut;
    const RowScores<NTH> all{RowView(sp, T, tid)};
    const bool whole_row = LISTED && held.n == 0;
    if (whole_row) row_kth_best<NTH>(all, sp, T, k, hist, sh, thr, cut);
    else row_kth_best<NTH>(held, sp, T, k, hist, sh, thr, cut);
    if (tid == 0) { thr_out[2 * p] = (int32_t)thr; thr_out[2 * p + 1] = cut; }
    if (!seg_budget) return;

    // ---- implicit budgets: every Top-B token adds one to its segment, the last one that begins at or in front of it
    if (!LISTED) {
        static_assert(N <= 32, "a word per thread is enough");
        const uint32_t mine = tid < words ? (uint32_t)__popc(bits[tid]) : 0u, incl = wave_scan_u(mine);
        const uint32_t b = waves_before<NTH>(incl, sh) + incl - mine;
        if (tid < words) before[tid] = b;
        __syncthreads();
    }
    const int half = K > 1 ? 1 << (31 - __builtin_clz(K - 1)) : 0;
    auto add = [&](const int (&t)[4], const bool (&in)[4]) __attribute__((always_inline)) {      // four at a time, for their latency
        int sg[4];
        if (LISTED) {
#pragma unroll
            for (int i = 0; i < 4; ++i) sg[i] = 0;
#pragma nounroll
            for (int step = half; step > 0; step >>= 1) {
                int at[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) at[i] = off[min(sg[i] + step, K)];
#pragma unroll
                for (int i = 0; i < 4; ++i) sg[i] += (sg[i] + step < K) & (at[i] <= t[i]) ? step : 0;
            }
        } else {
            uint32_t b[4], n[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { const int w = min(t[i], T - 1) >> 5; b[i] = bits[w]; n[i] = before[w]; }
#pragma unroll
            for (int i = 0; i < 4; ++i) sg[i] = max((int)(n[i] + (uint32_t)__popc(b[i] & (0xFFFFFFFFu >> (31 - (t[i] & 31))))) - 1, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (in[i]) {
                atomicAdd(&cnt[sg[i]], 1);
                one[sg[i]] = t[i];                 // the one there is, where there is one
            }
    };
    if (whole_row) {
        all.each([&](uint32_t key, int t) {
            const int tt[4] = {t, t, t, t};
            const bool in[4] = {key > thr || (key == thr && t <= cut), false, false, false};
            add(tt, in);
        });
    } else {
#pragma unroll
        for (int e0 = 0; e0 < N; e0 += 4) {
            if (e0 * NTH < held.n) {               // uniform
                int t[4];
                bool in[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int j = tid + (e0 + i) * NTH;
                    t[i] = j;
                    if constexpr (LISTED) t[i] = j < held.n ? held.tok[e0 + i] : 0;
                    const uint32_t key = j < held.n ? held.key[e0 + i] : 0u;
                    in[i] = (j < held.n) & ((key > thr) | ((key == thr) & (t[i] <= cut)));
                }
                add(t, in);
            }
        }
    }
    __syncthreads();
    if (PLAN) {
        // ---- the search begins with the longest segments, as their search takes longest: how many are there?  (As a rule none.)
        bool longer = false;
#pragma nounroll
        for (int j = tid; j < K; j += NTH) longer |= off[j + 1] - off[j] > PRE_TOKENS && cnt[j] >= 2;
        if (__any(longer)) {
#pragma nounroll
            for (int j = tid; j < K; j += NTH)
                if (off[j + 1] - off[j] > PRE_TOKENS && cnt[j] >= 2) lds_add(&sh.n_long, 1);
        }
    }
#pragma nounroll
    for (int j = tid; j < sv.max_segments; j += NTH) {
        const int c = j < K ? cnt[j] : 0;
        seg_budget[row + j] = c;
        block_size[row + j] = PLAN && c == 1 ? 1 : 0;          // the others: written by the search
    }
    if (!PLAN) return;
    // ---- the exclusive prefix of the budgets is the place of a segment's tokens in the problem's idx row: a single token goes
    // there straight away, segments of more to the search's list.  A run of segments per thread; in the upper half of the sums
    // the segments of more that are not the longest
    SegRec *recs = pa.list + (int64_t)p * pa.capacity;
    int32_t *out = pa.idx_out + (int64_t)p * k;
    const int per = K <= NTH ? 1 : RUN;
    uint32_t run = 0;
#pragma nounroll
    for (int j0 = 0; j0 < K; j0 += per * NTH) {
        int c[RUN], a[RUN + 1];
        uint32_t mine = 0;
        const int j = j0 + per * tid;
#pragma unroll
        for (int i = 0; i < RUN; ++i)
            if (i < per) {
                c[i] = j + i < K ? cnt[j + i] : 0;
                a[i] = off[min(j + i, K)];
                a[i + 1] = off[min(j + i + 1, K)];
                mine += (uint32_t)c[i] + (c[i] >= 2 && a[i + 1] - a[i] <= PRE_TOKENS ? 0x10000u : 0u);
            }
        const uint32_t incl = wave_scan_u(mine);
        __syncthreads();                                       // (the first time: n_long is complete; later: the totals have been read)
        if (lane == 63) sh.w[wave] = incl;
        __syncthreads();
        uint32_t pos = run + incl - mine;
#pragma unroll
        for (int w = 0; w < NTH / 64; ++w) {
            const uint32_t x = sh.w[w];
            pos += w < wave ? x : 0u;
            run += x;
        }
#pragma unroll
        for (int i = 0; i < RUN; ++i)
            if (i < per) {
                if (c[i] == 1) out[pos & 0xFFFFu] = one[j + i];
                if (c[i] >= 2) {
                    const bool first = a[i + 1] - a[i] > PRE_TOKENS;
                    const int at = first ? lds_add(&sh.long_at, 1) : sh.n_long + (int)(pos >> 16);
                    SegRec r;
                    r.p = p; r.k = j + i; r.a = a[i]; r.b = a[i + 1]; r.bk = c[i]; r.g = (int32_t)thr; r.pos = cut; r.out = (int)(pos & 0xFFFFu);
                    recs[at] = r;
                    if (!first) pos += 0x10000u;
                }
                pos += (uint32_t)c[i];
            }
    }
    if (tid == 0) {
        pa.n_sel_out[p] = k;                                   // k = B < T here, so there is nothing to pad
        pa.counts[p] = K > 0 ? sh.n_long + (int)(run >> 16) : 0;
    }
}

// grid (P).  Selection of the k-th best score, k = min(B, T), as (ordered key v, index cut c), and, with seg_budget
// != NULL, the implicit budgets (Eq. implicit_budget).
//
// What bounds it: LDS atomics, if every score is counted (a histogram of 12 key bits puts a fifth of a row into one bin),
// and two reads of the row; so only a sample is counted, in bins fitted to it, and the row is read once.  256 rows of
// 131 040: 77 -> 46 us (134 MB, 2.9 TB/s with the sample); 1 024 rows of 65 472: 402 -> 111 us.
//
// A row of up to TB_ROUND tokens (those of many segments, see row_rank_for) is held in registers and its k-th best found there
// (kth_best).  Of a longer row a sample gives a lower bound first, ONE pass over the row lists the tokens that reach it (somewhat more than k), and the
// k-th best is found among those.  E * 1024 tokens fit the list; when they do not (many equal scores, a sample that
// misled), three histogram passes over the row (11 + 11 + 10 bits) and one to cut the ties by ascending index decide.
//
// PLAN (the search that also selects; the host launches it only when 0 < B < T, B fits the list and every sequence has
// fewer than `offs_cap` segments): the same workgroup goes on to the exclusive prefix of b_k (each segment's offset in
// the problem's idx_out row), writes n_sel, the token of every segment with b_k == 1 (g_k* = 1) straight to its place,
// and records the segments with b_k >= 2 for the search, with their output offset.
//
// TWO: two workgroups share a CU, which calls with more rows than CUs gain from although 64 registers spill three (Top-B
// and search, 1 024 rows of 65 472: 505 us, 529 with one per CU; 512 rows of 8 160: 112 and 116).  With fewer rows a
// workgroup has its CU to itself and up to 128 registers (256 rows of 131 040: 110 and 112).
template <bool PLAN, int E, bool TWO>
__global__ void __launch_bounds__(TB_THREADS, TWO ? 8 : 4)
topb_kernel(Dims d, const float *s_tilde, int budget, int32_t *thr_out, SegView sv, int32_t *seg_budget,
            int32_t *block_size, PlanArgs pa, Candidates cd, int offs_cap, int sample_rank)
{
    constexpr int CAP = E * TB_THREADS;          // tokens the list holds
    extern __shared__ __attribute__((aligned(16))) uint32_t sh_dyn[];   // histogram [TB_BINS] and list [CAP]; later offsets and counters [2][offs_cap]
    __shared__ TopbShared sh;
    uint32_t *hist = sh_dyn;
    int32_t *list = reinterpret_cast<int32_t *>(sh_dyn + TB_BINS);
    int32_t *sh_off = reinterpret_cast<int32_t *>(sh_dyn), *sh_cnt = sh_off + offs_cap;
    const int p = blockIdx.x, T = d.T;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const RowView r(s_tilde + (int64_t)p * T, T, tid);
    const int k = min(budget, T);
    const int64_t row = (int64_t)p * sv.max_segments;

    uint32_t thr = 0u;                           // k >= T: everything is inside, key 0 is below every score's key
    int cut = T - 1;
    int hit[E];                                  // this thread's share of T_topB (-1: none)
    bool have_hits = false;
    if (tid == 0) sh.n = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) hit[e] = -1;
    auto hits_from_list = [&]() {
        __syncthreads();
        const int n = min(sh.n, CAP);
#pragma unroll
        for (int e = 0; e < E; ++e) hit[e] = tid + e * TB_THREADS < n ? list[tid + e * TB_THREADS] : -1;
        have_hits = true;
    };
    if (k <= 0) {
        thr = 0xFFFFFFFFu;                       // nothing is inside
        cut = -1;
    } else if (k < T) {
        const bool sliced = PLAN && cd.n_slices > 0;
        bool found = false;
        if (!sliced && r.nvec <= TB_ROUND / 4) {
            // ---- the whole row in registers
            constexpr int J = TB_REG / 4;
            float4 v[J];
            int t0[J];
            uint32_t valid = 0;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int i = j * TB_THREADS + tid;
                v[j] = r.nvec > 0 ? r.vp[min(i, r.nvec - 1)] : make_float4(0.f, 0.f, 0.f, 0.f);
                t0[j] = i < r.nvec ? r.token(i) : -4;
                if (i < r.nvec) valid |= 15u << (4 * j);
            }
            const float ve = r.extra >= 0 ? r.sp[r.extra] : 0.f;
            if (r.extra >= 0) valid |= 1u << TB_REG;
            uint32_t key[TB_REG + 1];
#pragma unroll
            for (int j = 0; j < J; ++j) {
                key[4 * j] = ordered_key(v[j].x); key[4 * j + 1] = ordered_key(v[j].y);
                key[4 * j + 2] = ordered_key(v[j].z); key[4 * j + 3] = ordered_key(v[j].w);
            }
            key[TB_REG] = ordered_key(ve);
            found = kth_best<TB_REG + 1>(key, valid, [&](int e) { return e == TB_REG ? r.extra : t0[e >> 2] + (e & 3); }, k, T, hist,
                                         sh, thr, cut);
            if (found && k <= CAP && seg_budget) {
                append_tokens<J>(v, t0, [&](int t, float x) { return t >= 0 && in_topb(x, t, thr, cut); }, list, CAP, sh);
                append_extra(r, r.extra >= 0 && in_topb(ve, r.extra, thr, cut), list, CAP, sh);
                hits_from_list();                // exactly k of them
            }
        } else if (k <= CAP) {
            // ---- the tokens that reach a lower bound of the k-th best
            if (sliced) {
                int base = 0;
                for (int sl = 0; sl < cd.n_slices; ++sl) {
                    const int64_t o = (int64_t)p * cd.n_slices + sl;
                    const int n = cd.counts[o];
                    if (n > cd.cap || base + n > CAP) { base = CAP + 1; break; }
                    for (int i = tid; i < n; i += TB_THREADS) list[base + i] = (int)cd.entries[o * cd.cap + i].y;
                    base += n;
                }
                if (tid == 0) sh.n = base;
            } else {
                const float bound = sample_bound(r, sample_rank, hist, sh);
                __syncthreads();                 // the list's length is zero
                collect_above(r, 0, r.nvec, bound, list, CAP, sh);
                append_extra(r, r.extra >= 0 && !(r.sp[max(r.extra, 0)] < bound), list, CAP, sh);
            }
            __syncthreads();
            const int n = sh.n;
            if (n >= k && n <= CAP) {
                uint32_t key[E], valid = 0;
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int i = tid + e * TB_THREADS;
                    key[e] = 0u;
                    if (i < n) { key[e] = ordered_key(r.sp[list[i]]); valid |= 1u << e; }
                }
                found = kth_best<E>(key, valid, [&](int e) { return list[tid + e * TB_THREADS]; }, k, T, hist, sh, thr, cut);
                if (found) {
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        const int t = (valid >> e) & 1u ? list[tid + e * TB_THREADS] : -1;
                        if (((valid >> e) & 1u) && (key[e] > thr || (key[e] == thr && t <= cut))) hit[e] = t;
                    }
                    have_hits = true;
                }
            }
        }
        if (!found) {
            // ---- three histogram passes over the row
            uint32_t prefix = 0, mask = 0, krem = (uint32_t)k, n_eq = 0;
            const int shifts[3] = {21, 10, 0};
            const int bits[3] = {11, 11, 10};
            for (int pass = 0; pass < 3; ++pass) {
                const uint32_t last = (1u << bits[pass]) - 1u;
                const int shift = shifts[pass];
                __syncthreads();
                reinterpret_cast<uint4 *>(hist)[tid] = make_uint4(0, 0, 0, 0);
                __syncthreads();
                scan_row(r, tid, [&](int, float x) {
                    const uint32_t key = ordered_key(x);
                    if ((key & mask) == prefix) atomicAdd(&hist[last - ((key >> shift) & last)], 1u);    // bin 0: the largest
                });
                __syncthreads();
                uint32_t bin, above, count;
                find_bin(hist, krem, sh, bin, above, count);
                krem -= above;
                n_eq = count;
                prefix |= (last - bin) << shift;
                mask |= last << shift;
            }
            // prefix is the key of the k-th best score; krem of its n_eq ties are inside, lowest indices first
            thr = prefix;
            cut = T - 1;
            if (krem < n_eq) {
                int seen = 0;
                for (int c0 = 0; c0 < T; c0 += TB_THREADS) {
                    const int t = c0 + tid;
                    const bool tie = t < T && ordered_key(r.sp[t]) == prefix;
                    const unsigned long long bal = __ballot(tie);
                    __syncthreads();
                    if (lane == 0) sh.w[wave] = __popcll(bal);
                    __syncthreads();
                    int before = 0, total = 0;
                    for (int w = 0; w < TB_WAVES; ++w) { const int c = sh.w[w]; if (w < wave) before += c; total += c; }
                    const bool last = seen + total >= (int)krem;
                    if (last && tie && seen + before + lanes_below(bal) + 1 == (int)krem) sh.cut = t;
                    __syncthreads();
                    if (last) { cut = sh.cut; break; }
                    seen += total;
                }
            }
            if (k <= CAP && seg_budget) {
                __syncthreads();
                if (tid == 0) sh.n = 0;
                __syncthreads();
                scan_row(r, tid, [&](int t, float x) {
                    if (in_topb(x, t, thr, cut)) list[atomicAdd(&sh.n, 1)] = t;                          // exactly k of them
                });
                hits_from_list();
            }
        }
    }
    if (tid == 0) { thr_out[2 * p] = (int32_t)thr; thr_out[2 * p + 1] = cut; }
    if (!seg_budget) return;

    // ---- implicit budgets: every Top-B token adds one to its segment
    const int seq = seq_of_problem(d, p);
    const int32_t *off = sv.seg_off + sv.seq_ptr[seq];
    const int K = sv.seq_ptr[seq + 1] - sv.seq_ptr[seq] - 1;
    const bool counted = have_hits && K + 1 <= offs_cap;       // in LDS; always so with PLAN
    if (!counted) {
        for (int j = tid; j < sv.max_segments; j += TB_THREADS) {
            seg_budget[row + j] = k >= T && k > 0 && j < K ? off[j + 1] - off[j] : 0;
            block_size[row + j] = 0;
        }
        if (k <= 0 || k >= T) return;
        __syncthreads();                       // the clearing stores of all wavefronts before the first atomic
        if (have_hits) {
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (hit[e] >= 0) atomicAdd(&seg_budget[row + segment_of(off, K, hit[e])], 1);
        } else {
            scan_row(r, tid, [&](int t, float x) {
                if (in_topb(x, t, thr, cut)) atomicAdd(&seg_budget[row + segment_of(off, K, t)], 1);
            });
        }
        return;
    }
    __syncthreads();                           // the list has been read by everyone
    for (int j = tid; j <= K; j += TB_THREADS) { sh_off[j] = off[j]; sh_cnt[j] = 0; }
    if (tid == 0) sh.n_rec = 0;
    __syncthreads();
    int seg[E];
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (hit[e] >= 0) { seg[e] = segment_of(sh_off, K, hit[e]); atomicAdd(&sh_cnt[seg[e]], 1); }
    __syncthreads();
    for (int j = tid; j < sv.max_segments; j += TB_THREADS) {
        const int c = j < K ? sh_cnt[j] : 0;
        seg_budget[row + j] = c;
        block_size[row + j] = PLAN && c == 1 ? 1 : 0;          // the others: written by the search
    }
    if (!PLAN) return;
    // exclusive prefix of the counters in place (K + 1 entries: b_k = pos[k + 1] - pos[k]); offs_cap / 1024
    // consecutive entries per thread, wavefront scan, then the sixteen wavefront totals
    __syncthreads();
    {
        constexpr int PER_MAX = TB_OFFS_MAX / TB_THREADS;
        const int per = offs_cap / TB_THREADS;
        const int j0 = per * tid;
        int c[PER_MAX], tot = 0;
#pragma unroll
        for (int i = 0; i < PER_MAX; ++i) { c[i] = (i < per && j0 + i < K) ? sh_cnt[j0 + i] : 0; tot += c[i]; }
        const int incl = (int)wave_scan_u((uint32_t)tot);
        if (lane == 63) sh.w[wave] = incl;
        __syncthreads();
        int run = incl - tot;
#pragma unroll
        for (int w = 0; w < TB_WAVES; ++w) run += w < wave ? (int)sh.w[w] : 0;
#pragma unroll
        for (int i = 0; i < PER_MAX; ++i) { if (i < per && j0 + i <= K) sh_cnt[j0 + i] = run; run += c[i]; }
    }
    __syncthreads();
    int32_t *out = pa.idx_out + (int64_t)p * budget;
    if (tid == 0) pa.n_sel_out[p] = k;                         // k = B < T here, so there is nothing to pad
    // the token of every single-token segment goes straight to its place
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (hit[e] >= 0 && sh_cnt[seg[e] + 1] - sh_cnt[seg[e]] == 1) out[sh_cnt[seg[e]]] = hit[e];
    // the others to the search's list, with their output offset; the longest ones first, as their search takes longest
    SegRec *recs = pa.list + (int64_t)p * pa.capacity;
    for (int pass = 0; pass < 2; ++pass) {
        for (int sg = tid; sg < K; sg += TB_THREADS) {
            const int bk = sh_cnt[sg + 1] - sh_cnt[sg];
            if (bk < 2 || (sh_off[sg + 1] - sh_off[sg] > PRE_TOKENS) != (pass == 0)) continue;
            SegRec rec;
            rec.p = p; rec.k = sg; rec.a = sh_off[sg]; rec.b = sh_off[sg + 1]; rec.bk = bk; rec.g = (int32_t)thr; rec.pos = cut;
            rec.out = sh_cnt[sg];
            recs[atomicAdd(&sh.n_rec, 1)] = rec;
        }
        __syncthreads();
    }
    if (tid == 0) pa.counts[p] = sh.n_rec;
}

// ------------------------------------------------------------------ search
// One workgroup per problem: g_k* = 1 where b_k == 1 (the rows are zero elsewhere), and the segments with b_k >= 2 are
// recorded for the search (by topb_kernel itself when the search also selects).
constexpr int LIST_THREADS = 1024;         // threads of the per-problem list-building kernels: segments handled per step

__global__ void __launch_bounds__(LIST_THREADS)
heavy_list_kernel(Dims d, SegView sv, const int32_t *thr, const int32_t *seg_budget, int32_t *block_size, SegRec *list,
                  int32_t *counts, int capacity)
{
    __shared__ int n_rec;
    const int p = blockIdx.x, tid = threadIdx.x;
    const int seq = seq_of_problem(d, p);
    const int32_t *off = sv.seg_off + sv.seq_ptr[seq];
    const int K = sv.seq_ptr[seq + 1] - sv.seq_ptr[seq] - 1;
    const int64_t row = (int64_t)p * sv.max_segments;
    SegRec *recs = list + (int64_t)p * capacity;
    if (tid == 0) n_rec = 0;
    __syncthreads();
    for (int pass = 0; pass < 2; ++pass) {                     // the longest ones first, as their search takes longest
        for (int k = tid; k < K; k += LIST_THREADS) {
            const int bk = seg_budget[row + k];
            if (pass == 0 && bk == 1) block_size[row + k] = 1;
            if (bk < 2 || (off[k + 1] - off[k] > PRE_TOKENS) != (pass == 0)) continue;
            SegRec r;
            r.p = p; r.k = k; r.a = off[k]; r.b = off[k + 1]; r.bk = bk; r.g = thr[2 * p]; r.pos = thr[2 * p + 1]; r.out = 0;
            recs[atomicAdd(&n_rec, 1)] = r;
        }
        __syncthreads();
    }
    if (tid == 0) counts[p] = n_rec;
}

// One wavefront per workgroup; the wavefronts of a problem (grid.x) stride over its records.  EMIT: see search_exact; no
// select pass over the segment is then needed.  24 wavefronts per CU (80 registers) are all that fit without spills, and
// as fast as 28 with them (256 rows of 131 040 tokens, Top-B and search: 115.7 and 122.2 us).
constexpr int SLICE_BYTES = 8 * (PRE_TOKENS + 1);
static_assert(17 * CAPB + CAPT / 8 <= SLICE_BYTES, "ordered sums: CAPT scores (fp32), block sums (fp64), block classes, taken tokens");
constexpr int STREAM_KEPT = (SLICE_BYTES - (int)sizeof(StreamScratch)) / 8;      // block sums of a segment searched from memory

template <bool EMIT>
__global__ void __launch_bounds__(64, 6)
search_kernel(Dims d, const float *s_tilde, int32_t max_segments, CandList cand, float tau, const SegRec *list,
              const int32_t *counts, int capacity, int32_t *block_size, int budget, int32_t *idx_out)
{
    __shared__ __attribute__((aligned(16))) char slice[SLICE_BYTES];
    const int p = grid_problem(d), stride = grid_parts(d), lane = threadIdx.x;
    const SegRec *recs = list + (int64_t)p * capacity;
    const SearchCtx x(s_tilde, d.T, p, block_size, max_segments, EMIT ? idx_out : nullptr, budget, tau, cand);
    const float *sp = x.sp;

    int i = grid_part(d);                                      // < capacity: the grid is no wider than the list can get
    SegRec nxt = recs[i];                                      // fetched together with the list's length
    const int n_rec = min(counts[p], capacity);
    if (i >= n_rec) return;
    float2 v_nxt = first_scores(sp, nxt);
    for (bool more = true; more; i += stride) {
        const SegRec r = nxt;
        const float2 v0 = v_nxt;
        more = i + stride < n_rec;
        if (more) {                                            // the next record and its scores, under this one's work
            nxt = recs[i + stride];
            v_nxt = first_scores(sp, nxt);
        }
        const int a = r.a, b = r.b, n = b - a;
        if (n <= PRE_TOKENS && search_exact<EMIT>(x, r, v0, reinterpret_cast<double *>(slice))) continue;

        if (n > CAPT) {
            search_streamed<EMIT>(x, r, *reinterpret_cast<StreamScratch *>(slice), reinterpret_cast<double *>(slice + sizeof(StreamScratch)),
                                  STREAM_KEPT);
            __builtin_amdgcn_wave_barrier();                   // the slice is reused by the next segment
            continue;
        }

        // ---- ordered sums, from LDS
        float *lv = reinterpret_cast<float *>(slice);
        WaveScratch ws{reinterpret_cast<double *>(slice + 8 * CAPB), reinterpret_cast<uint8_t *>(slice + 16 * CAPB), CAPB};
        unsigned long long *taken = reinterpret_cast<unsigned long long *>(slice + 17 * CAPB);      // of the candidate just tried
        const int gcap = min(n, r.bk);
        double sum = 0.0;
#pragma nounroll
        for (int c0 = a; c0 < b; c0 += 64) {
            const int t = c0 + lane;
            const float v = t < b ? sp[t] : 0.f;
            if (t < b) lv[t - a] = v;
            sum = add_in_order(sum, __ballot(t < b && in_topb(v, t, (uint32_t)r.g, r.pos)), v);
        }
        __builtin_amdgcn_wave_barrier();
        const double need = x.need(sum);
        int gstar = 0;
#pragma nounroll
        for (int c = cand.n - 1; c >= 0; --c) {
            const int g = __builtin_amdgcn_readlane(x.cand_g, c);
            if (g > gcap) continue;
            if (g == 1) { gstar = 1; break; }
            double score = 0.0;
            segment_fill([&](int t) { return lv[t - a]; }, a, b, g, r.bk, ws, [&](int c0, unsigned long long m, float v) {
                score = add_in_order(score, m, v);
                if (EMIT && lane == 0) taken[(c0 - a) >> 6] = m;
            });
            if (score >= need) { gstar = g; break; }
        }
        if (lane == 0) x.block_size[r.k] = gstar;
        if (EMIT && gstar == 1) put_topb<1>(x, r);
        if (EMIT && gstar > 1) {
            int pos = r.out;
#pragma nounroll
            for (int c0 = a; c0 < b; c0 += 64) put_tokens(x, pos, c0, taken[(c0 - a) >> 6]);
        }
        __builtin_amdgcn_wave_barrier();                       // the slice is reused by the next segment
    }
}

// ------------------------------------------------------------------ select
__global__ void reset_counters_kernel(int32_t *counters)
{
    if (threadIdx.x < 3) counters[threadIdx.x] = 0;
}

// One workgroup per problem: exclusive prefix of b_k over its segments (where each segment's tokens go in the
// problem's idx_out row), n_sel, the -1 padding of idx_out.  The segments that retain anything are appended to
// one of the call's three select lists: token-level ones (g_k* = 1) to `light`, the others to `full` or, when
// longer than CAPT tokens, to `full_long`.  counters[0..2] are the lengths of light / full / full_long.
__global__ void __launch_bounds__(LIST_THREADS)
seg_prefix_kernel(Dims d, SegView sv, const int32_t *seg_budget, const int32_t *block_size, int budget,
                  SegRec *light, SegRec *full, SegRec *full_long, int32_t *counters, int capacity, int32_t *idx_out,
                  int32_t *n_sel_out)
{
    __shared__ int sh_w[LIST_THREADS / 64], sh_l[LIST_THREADS / 64], sh_f[LIST_THREADS / 64], sh_x[LIST_THREADS / 64];
    __shared__ int sh_base[3];
    const int p = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int seq = seq_of_problem(d, p);
    const int32_t *off = sv.seg_off + sv.seq_ptr[seq];
    const int K = sv.seq_ptr[seq + 1] - sv.seq_ptr[seq] - 1;
    const int64_t row = (int64_t)p * sv.max_segments;
    const unsigned long long lt = (1ull << lane) - 1ull;
    int carry = 0;
    for (int c0 = 0; c0 < K; c0 += LIST_THREADS) {
        const int k = c0 + tid;
        const int v = (k < K) ? seg_budget[row + k] : 0;
        const int g = (k < K) ? block_size[row + k] : 0;
        const int sa = k < K ? off[k] : 0, sb = k < K ? off[k + 1] : 0;
        const bool is_light = v > 0 && g == 1;
        const bool is_full = v > 0 && g > 1 && sb - sa <= CAPT, is_long = v > 0 && g > 1 && sb - sa > CAPT;
        const unsigned long long bl = __ballot(is_light), bf = __ballot(is_full), bx = __ballot(is_long);
        int incl = v;
        for (int o = 1; o < 64; o <<= 1) { int x = __shfl_up(incl, o); if (lane >= o) incl += x; }
        if (lane == 63) sh_w[wave] = incl;
        if (lane == 0) { sh_l[wave] = __popcll(bl); sh_f[wave] = __popcll(bf); sh_x[wave] = __popcll(bx); }
        __syncthreads();
        int before = 0, total = 0, before_l = 0, total_l = 0, before_f = 0, total_f = 0, before_x = 0, total_x = 0;
        for (int w = 0; w < LIST_THREADS / 64; ++w) {
            if (w < wave) { before += sh_w[w]; before_l += sh_l[w]; before_f += sh_f[w]; before_x += sh_x[w]; }
            total += sh_w[w]; total_l += sh_l[w]; total_f += sh_f[w]; total_x += sh_x[w];
        }
        if (tid == 0 && total_l > 0) sh_base[0] = atomicAdd(&counters[0], total_l);
        if (tid == 1 && total_f > 0) sh_base[1] = atomicAdd(&counters[1], total_f);
        if (tid == 2 && total_x > 0) sh_base[2] = atomicAdd(&counters[2], total_x);
        __syncthreads();
        if (is_light || is_full || is_long) {
            const int slot = is_light ? sh_base[0] + before_l + __popcll(bl & lt)
                           : is_full ? sh_base[1] + before_f + __popcll(bf & lt)
                                     : sh_base[2] + before_x + __popcll(bx & lt);
            if (slot < capacity) {
                SegRec r;
                r.p = p; r.k = k; r.a = sa; r.b = sb; r.bk = v; r.g = g; r.pos = carry + before + incl - v; r.out = 0;
                (is_light ? light : is_full ? full : full_long)[slot] = r;
            }
        }
        carry += total;
    }
    const int n = min(carry, budget);
    if (tid == 0) n_sel_out[p] = n;
    for (int j = n + tid; j < budget; j += LIST_THREADS) idx_out[(int64_t)p * budget + j] = -1;
}

// Token-level segments, sixteen lanes each (most retaining segments hold one or two Top-B tokens, so a wavefront
// per segment would mostly idle): T_k(1) = T_topB & S_k when b_k is the implicit budget, written in ascending
// order.  A segment whose b_k is something else (a caller's own budgets) is passed on to one of the full lists.
constexpr int LIGHT_GROUP = 16;

__global__ void __launch_bounds__(256)
select_light_kernel(Dims d, const float *s_tilde, const int32_t *thr, const SegRec *light, SegRec *full,
                    SegRec *full_long, int32_t *counters, int capacity, int budget, int32_t *idx_out)
{
    const int sub = threadIdx.x & (LIGHT_GROUP - 1);
    const int j = blockIdx.x * (256 / LIGHT_GROUP) + threadIdx.x / LIGHT_GROUP;       // < capacity rounded up
    const int n_list = min(counters[0], capacity);
    if (j >= n_list) return;
    const SegRec r = light[j];
    const int p = r.p, a = r.a, b = r.b;
    const int bk = min(r.bk, b - a);
    const float *sp = s_tilde + (int64_t)p * d.T;
    int32_t *out = idx_out + (int64_t)p * budget;
    const uint32_t thr_key = (uint32_t)thr[2 * p];
    const int thr_cut = thr[2 * p + 1];
    const int shift = (threadIdx.x & 63) & ~(LIGHT_GROUP - 1);                          // first lane of this group
    int cnt = 0;
    // groups of one wavefront may run different trip counts: ballots are taken over the lanes still in the loop
    for (int c0 = a; c0 < b; c0 += LIGHT_GROUP) {
        const int t = c0 + sub;
        const bool in = t < b && in_topb(sp[t < b ? t : a], t, thr_key, thr_cut);
        const uint32_t gm = (uint32_t)(__ballot(in) >> shift) & ((1u << LIGHT_GROUP) - 1u);
        const int slot = cnt + __popc(gm & ((1u << sub) - 1u));
        if (in && slot < bk && r.pos + slot < budget) out[r.pos + slot] = t;
        cnt += __popc(gm);
    }
    if (cnt != bk && sub == 0) {
        const bool lng = b - a > CAPT;
        const int slot = atomicAdd(&counters[lng ? 2 : 1], 1);
        if (slot < capacity) (lng ? full_long : full)[slot] = r;
    }
}

// T_k(g_k*) of one listed segment, written in ascending order from its offset in idx_out
template <int CT, int CB>
__device__ inline void select_segment(const Dims &d, const float *s_tilde, const int32_t *thr, const SegRec &r,
                                      int budget, int32_t *idx_out, double (&sh_phi)[CB], float (&sh_val)[CT],
                                      uint8_t (&sh_cls)[CB])
{
    const int lane = threadIdx.x & 63;
    const int p = r.p, a = r.a, b = r.b;
    const int bk = min(r.bk, b - a);
    int g = r.g;
    if (bk <= 0 || g <= 0) return;
    g = min(min(g, MAX_G), bk);
    const float *sp = s_tilde + (int64_t)p * d.T;
    int32_t *out = idx_out + (int64_t)p * budget;
    int pos = r.pos;
    const unsigned long long lt = (1ull << lane) - 1ull;
    auto put = [&](int c0, unsigned long long m, float) {
        const int j = pos + __popcll(m & lt);
        if (((m >> lane) & 1ull) && j < budget) out[j] = c0 + lane;
        pos += __popcll(m);
    };
    if (g == 1) {
        // T_k(1) = T_topB & S_k whenever b_k is the implicit budget; otherwise rank the tokens
        const uint32_t thr_key = (uint32_t)thr[2 * p];
        const int thr_cut = thr[2 * p + 1];
        if (b - a <= 64) {
            const int t = a + lane;
            const unsigned long long m = __ballot(t < b && in_topb(sp[t < b ? t : a], t, thr_key, thr_cut));
            if (__popcll(m) == bk) { put(a, m, 0.f); return; }
        } else {
            int cnt = 0;
            for (int c0 = a; c0 < b; c0 += 64) {
                const int t = c0 + lane;
                cnt += (t < b && in_topb(sp[t], t, thr_key, thr_cut)) ? 1 : 0;
            }
            if (wave_sum_i(cnt) == bk) {
                for (int c0 = a; c0 < b; c0 += 64) {
                    const int t = c0 + lane;
                    put(c0, __ballot(t < b && in_topb(sp[t], t, thr_key, thr_cut)), 0.f);
                }
                return;
            }
        }
    }
    WaveScratch ws{sh_phi, sh_cls, CB};
    if (b - a <= CT) {
        float *lv = sh_val;
        for (int t = a + lane; t < b; t += 64) lv[t - a] = sp[t];
        __builtin_amdgcn_wave_barrier();
        auto val = [lv, a](int t) { return lv[t - a]; };
        segment_fill(val, a, b, g, bk, ws, put);
    } else {
        auto val = [sp](int t) { return sp[t]; };
        segment_fill(val, a, b, g, bk, ws, put);
    }
}

// one wavefront per workgroup, striding over the call's select list
constexpr int SELECT_WGS = 32768;

template <int CT, int CB>
__global__ void __launch_bounds__(64)
select_kernel(Dims d, const float *s_tilde, const int32_t *thr, const SegRec *list, const int32_t *counter,
              int capacity, int budget, int32_t *idx_out)
{
    __shared__ __attribute__((aligned(16))) double sh_phi[CB];
    __shared__ float sh_val[CT];
    __shared__ uint8_t sh_cls[CB];
    int j = blockIdx.x;                                     // < capacity: the grid is no larger than the list can get
    SegRec r = list[j];                                     // fetched together with the list length
    const int n_list = min(*counter, capacity);
    for (; j < n_list; j += gridDim.x, r = list[min(j, capacity - 1)]) {
        select_segment<CT, CB>(d, s_tilde, thr, r, budget, idx_out, sh_phi, sh_val, sh_cls);
        __builtin_amdgcn_wave_barrier();                    // the LDS slices are reused by the next segment
    }
}

}  // namespace

// ---- launches of the Top-B kernel
// Rank in a sample of TB_ROUND scores of the row behind which the bound is taken: the share of the k best that falls into
// the sample has mean k * TB_ROUND / T and, for scores in no particular order, a standard deviation below the root of
// that; six of them and a constant for small shares leave room for scores that keep together.
static int topb_rank(const Dims &d, int k)
{
    const double share = (double)k * TB_ROUND / std::max(d.T, 1);
    return (int)std::min<double>(TB_ROUND, share + 6.0 * sqrt(share) + 16.0);
}
// Tokens the list must hold (thousands, one of 4, 8, 16, 32): the k best, and of a sampled row what lies above the bound
static int topb_list_k(const Dims &d, int32_t budget)
{
    const int k = std::min(budget, d.T);
    double n = k;
    if (d.T > TB_ROUND) n = std::min<double>(d.T, 1.2 * topb_rank(d, k) * d.T / TB_ROUND + 256.0);
    return n <= 4 * TB_THREADS ? 4 : n <= 8 * TB_THREADS ? 8 : n <= 16 * TB_THREADS ? 16 : 32;
}
static int topb_offs_cap(int32_t max_segments)
{
    return max_segments + 1 <= TB_OFFS ? TB_OFFS : max_segments + 1 <= 2 * TB_OFFS ? 2 * TB_OFFS : TB_OFFS_MAX;
}

template <bool PLAN, int E, bool TWO>
static hipError_t run_topb(const Dims &d, const float *s_tilde, int32_t budget, int32_t *thr, const SegView &sv, int32_t *seg_budget,
                           int32_t *block_size, const PlanArgs &pa, const Candidates &cd,
                           hipStream_t st)
{
    const int offs_cap = PLAN || seg_budget ? topb_offs_cap(sv.max_segments) : 0;
    const size_t lds = std::max((size_t)(TB_BINS + E * TB_THREADS) * 4, (size_t)offs_cap * 8);
    constexpr size_t lds_most = std::max((size_t)(TB_BINS + E * TB_THREADS) * 4, (size_t)TB_OFFS_MAX * 8);
    if (lds > 64 * 1024) {
        static thread_local PerDeviceOnce attr_once;
        if (attr_once.needed()) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(topb_kernel<PLAN, E, TWO>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_most);
            if (e != hipSuccess) return e;
            attr_once.done();
        }
    }
    hipLaunchKernelGGL((topb_kernel<PLAN, E, TWO>), dim3(d.P), dim3(TB_THREADS), lds, st, d, s_tilde, budget, thr, sv, seg_budget,
                       block_size, pa, cd, offs_cap, topb_rank(d, std::min(budget, d.T)));
    return hipGetLastError();
}

// ---- launches of row_rank_kernel: rows of up to 16 384 tokens and listed ones, but for all or nothing inside and too many segments
static int most_segments(const Dims &d, const SegView &sv)
{
    int n = 0;
    for (int s = 0; s < d.n_seq; ++s) n = std::max(n, sv.seq_ptr[s + 1] - sv.seq_ptr[s] - 1);
    return n;
}
// Where segments have hardly two tokens, the bits of neighbours meet in the same words and three words of LDS per segment cost more than
// topb_kernel's two or none; and rows that are more than the compute units have to leave room for two workgroups on each.  Search and
// selection of 8, 256 and 1 024 rows: 8 160 tokens of mean length 1.3, 22.6, 31.2 and 97.7 us, topb_kernel 20.3, 30.7 and 77.7; of 2, 19.4, 34.2
// and 95.9, topb_kernel 20.1, 36.0 and 105.7; 1 024 of 16 000 of mean length 2, 137 and 98, of 3, 116 and 119; 2 000 tokens, whatever their
// segments, a tenth to a third less.  Listed rows of as many segments as fit: 8 of 131 040 tokens and 9 360 segments, 30.3 and 32.6.
static bool row_rank_for(bool listed, int nth, const Dims &d, int32_t budget, int segments)
{
    if (budget <= 0 || budget >= d.T) return false;
    const int bytes = RowLds(listed, nth, d.T, std::min(segments, 65535)).bytes;
    if (listed) return bytes <= RR_LDS_MOST;
    const bool two = d.P > d.cus;
    return bytes <= (two ? RR_LDS_MOST / 2 : RR_LDS_MOST) && segments <= std::max(2048, two ? d.T / 4 * 3 : d.T / 2);
}

template <bool PLAN, int NTH, bool LISTED, int N = RR_KEYS>
static hipError_t run_row_rank(const Dims &d, const float *s_tilde, int32_t budget, int32_t *thr, const SegView &sv, int32_t *seg_budget,
                               int32_t *block_size, const PlanArgs &pa, const Candidates &cd, int segments, hipStream_t st)
{
    static thread_local PerDeviceOnce attr_once;
    if (attr_once.needed()) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(row_rank_kernel<PLAN, NTH, LISTED, N>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, RR_LDS_MOST);
        if (e != hipSuccess) return e;
        attr_once.done();
    }
    hipLaunchKernelGGL((row_rank_kernel<PLAN, NTH, LISTED, N>), dim3(d.P), dim3(NTH), RowLds(LISTED, NTH, d.T, segments).bytes, st, d,
                       s_tilde, budget, thr, sv, seg_budget, block_size, pa, cd, segments);
    return hipGetLastError();
}

template <bool PLAN>
static hipError_t run_topb(const Dims &d, const float *s_tilde, int32_t budget, int32_t *thr, const SegView &sv, int32_t *seg_budget,
                           int32_t *block_size, const PlanArgs &pa, const Candidates &cd, hipStream_t st)
{
    // (more rows than CUs, of more than 8 192 tokens: half the threads with twice the scores, so that two workgroups share a CU;
    // 1 024 rows of 16 000 tokens, 992 retained, Top-B and search 220 us, with 1 024 threads 244)
    const bool two = d.P > d.cus;
    const int nth = d.T <= 256 * RR_KEYS ? 256 : d.T <= 512 * RR_KEYS || two ? 512 : 1024, segments = most_segments(d, sv);
    if (d.T <= 1024 * RR_KEYS && row_rank_for(false, nth, d, budget, segments)) {
        const auto run = nth == 256 ? run_row_rank<PLAN, 256, false> : nth == 1024 ? run_row_rank<PLAN, 1024, false> :
                         d.T <= 512 * RR_KEYS ? run_row_rank<PLAN, 512, false> : run_row_rank<PLAN, 512, false, 2 * RR_KEYS>;
        return run(d, s_tilde, budget, thr, sv, seg_budget, block_size, pa, Candidates{}, segments, st);
    }
    switch (topb_list_k(d, budget)) {
    case 4: return (two ? run_topb<PLAN, 4, true> : run_topb<PLAN, 4, false>)(d, s_tilde, budget, thr, sv, seg_budget, block_size, pa, cd, st);
    case 8: return (two ? run_topb<PLAN, 8, true> : run_topb<PLAN, 8, false>)(d, s_tilde, budget, thr, sv, seg_budget, block_size, pa, cd, st);
    case 16: return run_topb<PLAN, 16, false>(d, s_tilde, budget, thr, sv, seg_budget, block_size, pa, cd, st);
    default: return run_topb<PLAN, 32, false>(d, s_tilde, budget, thr, sv, seg_budget, block_size, pa, cd, st);
    }
}

hipError_t launch_topb(const Dims &d, const float *s_tilde, int32_t budget, int32_t *thr, hipStream_t st)
{
    if (d.P <= 0) return hipSuccess;
    return run_topb<false>(d, s_tilde, budget, thr, SegView{}, nullptr, nullptr, PlanArgs{}, Candidates{}, st);
}

// upper bound of a problem's records: a recorded segment holds at least two of the |T_topB| tokens
static int max_heavy_segments(const Dims &d, int32_t max_segments, int32_t budget)
{
    const int k = budget < d.T ? budget : d.T;
    return std::max(0, std::min(k / 2, (int)max_segments));
}

size_t search_ws_bytes(const Dims &d, int32_t max_segments, int32_t budget)
{
    const size_t cap = (size_t)d.P * max_heavy_segments(d, max_segments, budget);
    return 2 * align256((size_t)d.P * 2 * 4) + align256((cap > 0 ? cap : 1) * sizeof(SegRec));
}

struct SearchWs {
    int32_t *thr, *counts;
    SegRec *list;
    SearchWs(const Dims &d, void *ws)
    {
        char *w = static_cast<char *>(ws);
        thr = reinterpret_cast<int32_t *>(w);
        counts = reinterpret_cast<int32_t *>(w + align256((size_t)d.P * 2 * 4));
        list = reinterpret_cast<SegRec *>(w + 2 * align256((size_t)d.P * 2 * 4));
    }
};

template <bool EMIT>
static void run_search(const Dims &d, const float *s_tilde, const SegView &sv, const CandList &cand, float tau, const SearchWs &w, int cap,
                       int32_t *block_size, int32_t budget, int32_t *idx_out, hipStream_t st)
{
    // wavefronts per problem: one per possible record up to 128 per CU (24 are resident at once), striding over the records
    unsigned gx = (unsigned)std::max<int64_t>(1, std::min<int64_t>(cap, (int64_t)d.cus * 128 / d.P));
    // ... an odd number of them: segments are the same for all problems of a sequence and stand in the same order in their lists,
    // and an XCD, which gets every eighth workgroup, would else get the same eighth of them of every problem (1 024 rows of 16 000
    // tokens, 4 000 retained, Top-B and search: 894 us with 32 wavefronts per problem, 574 with 31)
    if (gx > 1 && gx < (unsigned)cap) gx -= 1 - gx % 2;
    Dims o = d;
    const dim3 grid = parts_grid(o, gx);
    hipLaunchKernelGGL(search_kernel<EMIT>, grid, dim3(64), 0, st, o, s_tilde, sv.max_segments, cand, tau, w.list,
                       w.counts, cap, block_size, budget, idx_out);
}

hipError_t launch_search(const Dims &d, const float *s_tilde, const SegView &sv, const CandList &cand,
                         int32_t budget, float tau, int32_t *seg_budget, int32_t *block_size, int32_t *topb_out,
                         void *ws, hipStream_t st)
{
    if (d.P <= 0 || sv.max_segments <= 0) return hipSuccess;
    const int cap = max_heavy_segments(d, sv.max_segments, budget);
    const SearchWs w(d, ws);
    int32_t *thr = topb_out ? topb_out : w.thr;
    hipError_t e = run_topb<false>(d, s_tilde, budget, thr, sv, seg_budget, block_size, PlanArgs{}, Candidates{}, st);
    if (e != hipSuccess) return e;
    if (budget > 0 && d.T > 0) {
        hipLaunchKernelGGL(heavy_list_kernel, dim3(d.P), dim3(LIST_THREADS), 0, st, d, sv, thr, seg_budget, block_size, w.list,
                           w.counts, cap);
        if (cap > 0) run_search<false>(d, s_tilde, sv, cand, tau, w, cap, block_size, 0, nullptr, st);
    }
    return hipGetLastError();
}

constexpr int LONG_WGS = 8192;             // workgroups of the kernel that selects from the list of long segments

// upper bound of the select lists: a listed segment retains at least one token of its problem's budget
static size_t max_active_segments(const Dims &d, int32_t max_segments, int32_t budget)
{
    const int a = budget < max_segments ? budget : max_segments;
    return (size_t)d.P * (size_t)(a > 0 ? a : 0);
}

size_t select_ws_bytes(const Dims &d, int32_t max_segments, int32_t budget)
{
    const size_t cap = max_active_segments(d, max_segments, budget);
    return align256((size_t)d.P * 2 * 4) + align256(12) + 3 * align256((cap > 0 ? cap : 1) * sizeof(SegRec));
}

hipError_t launch_select(const Dims &d, const float *s_tilde, const SegView &sv, const int32_t *seg_budget,
                         const int32_t *block_size, const int32_t *topb, int32_t budget, int32_t *idx_out,
                         int32_t *n_sel_out, void *ws, hipStream_t st)
{
    if (d.P <= 0) return hipSuccess;
    const size_t cap = max_active_segments(d, sv.max_segments, budget);
    const size_t list_bytes = align256((cap > 0 ? cap : 1) * sizeof(SegRec));
    char *w = static_cast<char *>(ws);
    int32_t *thr_ws = reinterpret_cast<int32_t *>(w);
    w += align256((size_t)d.P * 2 * 4);
    int32_t *counters = reinterpret_cast<int32_t *>(w);
    w += align256(12);
    SegRec *light = reinterpret_cast<SegRec *>(w);
    SegRec *full = reinterpret_cast<SegRec *>(w + list_bytes);
    SegRec *full_long = reinterpret_cast<SegRec *>(w + 2 * list_bytes);
    const int32_t *thr = topb;
    if (!thr) {
        hipError_t e = launch_topb(d, s_tilde, budget, thr_ws, st);
        if (e != hipSuccess) return e;
        thr = thr_ws;
    }
    hipLaunchKernelGGL(reset_counters_kernel, dim3(1), dim3(64), 0, st, counters);
    hipLaunchKernelGGL(seg_prefix_kernel, dim3(d.P), dim3(LIST_THREADS), 0, st, d, sv, seg_budget, block_size, budget,
                       light, full, full_long, counters, (int)cap, idx_out, n_sel_out);
    if (cap > 0) {
        const unsigned per_wg = 256 / LIGHT_GROUP;
        hipLaunchKernelGGL(select_light_kernel, dim3((unsigned)((cap + per_wg - 1) / per_wg)), dim3(256), 0, st, d,
                           s_tilde, thr, light, full, full_long, counters, (int)cap, budget, idx_out);
        hipLaunchKernelGGL((select_kernel<CAPT, CAPB>), dim3((unsigned)(cap < SELECT_WGS ? cap : SELECT_WGS)), dim3(64), 0,
                           st, d, s_tilde, thr, full, counters + 1, (int)cap, budget, idx_out);
        hipLaunchKernelGGL((select_kernel<CAPT_LONG, CAPB_LONG>), dim3((unsigned)(cap < LONG_WGS ? cap : LONG_WGS)), dim3(64),
                           0, st, d, s_tilde, thr, full_long, counters + 2, (int)cap, budget, idx_out);
    }
    return hipGetLastError();
}

// ---- search and select in one sequence (same results as launch_search followed by launch_select)
bool search_select_fused(const Dims &d, const SegView &sv, int32_t budget)
{
    return budget > 0 && budget < d.T && budget <= TB_BUDGET_MAX && sv.max_segments + 1 <= TB_OFFS_MAX;
}

// Workgroups per row that collect the tokens above the row's bound in the one-call form: with few problems in a call (a
// layer at a time) one workgroup per long row would leave most of the chip idle.  1: the per-row kernel scans its row.
static int topb_slices(const Dims &d, int32_t budget)
{
    if (budget <= 0 || budget >= d.T || topb_list_k(d, budget) > 8 || d.T <= TB_ROUND) return 1;
    if (const int v = d.tune.topb_slices; v >= 1) return (int64_t)v * 4096 <= d.T ? v : 1;
    // a slice is one round of loads; a kernel of its own (5 us) for them pays when it saves the per-row kernel four rounds
    // or more (both calls together, 8 rows: 32 752 tokens 26.7 us in one kernel, 27.1 in two; 65 520: 32.5, 29.0; 32
    // rows of 131 056: 43.0, 35.7)
    const int s = (d.T + TB_ROUND - 1) / TB_ROUND;
    return s >= 4 && (int64_t)s * d.P <= d.cus ? std::min(s, 64) : 1;
}
static size_t sliced_bytes(const Dims &d, int32_t budget)
{
    const size_t n = (size_t)d.P * topb_slices(d, budget);
    return align256(n * 4) + align256(n * topb_list_k(d, budget) * TB_THREADS * sizeof(uint2));
}

// The slices' lists lie behind the larger of the search and select layouts.
static size_t sliced_offset(const Dims &d, int32_t max_segments, int32_t budget)
{
    return std::max(search_ws_bytes(d, max_segments, budget), select_ws_bytes(d, max_segments, budget));
}
size_t search_select_ws_bytes(const Dims &d, int32_t max_segments, int32_t budget)
{
    return sliced_offset(d, max_segments, budget) + (topb_slices(d, budget) > 1 ? sliced_bytes(d, budget) : 0);
}

hipError_t launch_search_select(const Dims &d, const float *s_tilde, const SegView &sv, const CandList &cand,
                                int32_t budget, float tau, int32_t *seg_budget, int32_t *block_size, int32_t *topb_out,
                                int32_t *idx_out, int32_t *n_sel_out, void *ws, hipStream_t st)
{
    if (d.P <= 0) return hipSuccess;
    if (!search_select_fused(d, sv, budget)) {
        hipError_t e = launch_search(d, s_tilde, sv, cand, budget, tau, seg_budget, block_size, topb_out, ws, st);
        if (e != hipSuccess) return e;
        // the select lists reuse the workspace of the search's records, which are consumed by then; the Top-B state
        // sits in front of both layouts
        const int32_t *thr = topb_out ? topb_out : static_cast<const int32_t *>(ws);
        return launch_select(d, s_tilde, sv, seg_budget, block_size, thr, budget, idx_out, n_sel_out, ws, st);
    }
    const int cap = max_heavy_segments(d, sv.max_segments, budget);
    const SearchWs w(d, ws);
    int32_t *thr = topb_out ? topb_out : w.thr;
    const PlanArgs pa{w.list, w.counts, cap, idx_out, n_sel_out};
    Candidates cd{};
    if (const int n_slices = topb_slices(d, budget); n_slices > 1) {
        char *x = static_cast<char *>(ws) + sliced_offset(d, sv.max_segments, budget);
        int32_t *counts = reinterpret_cast<int32_t *>(x);
        uint2 *entries = reinterpret_cast<uint2 *>(x + align256((size_t)d.P * n_slices * 4));
        const int pre_cap = topb_list_k(d, budget) * TB_THREADS;
        Dims o = d;
        const dim3 grid = parts_grid(o, n_slices);
        hipLaunchKernelGGL(topb_collect_kernel, grid, dim3(TB_THREADS), (size_t)(TB_BINS + pre_cap) * 4, st, o, s_tilde,
                           topb_rank(d, budget), pre_cap, entries, counts);
        cd = Candidates{entries, counts, n_slices, pre_cap};
    }
    // threads of the listed rows' kernel: for a thread's share of the lists, or of the segments where they are more (8 rows of 131 040
    // tokens: 512 and 1 024 threads 50.9 and 51.2 us with 1 092 segments, 31.7 and 31.2 with 2 184, 30.8 and 28.7 with 6 552)
    const int segments = most_segments(d, sv), nth = segments <= 2048 ? 512 : 1024;
    const auto ranked = nth == 512 ? run_row_rank<true, 512, true> : run_row_rank<true, 1024, true, RR_KEYS / 2>;
    hipError_t e = cd.n_slices > 0 && row_rank_for(true, nth, d, budget, segments)
                       ? ranked(d, s_tilde, budget, thr, sv, seg_budget, block_size, pa, cd, segments, st)
                       : run_topb<true>(d, s_tilde, budget, thr, sv, seg_budget, block_size, pa, cd, st);
    if (e != hipSuccess) return e;
    if (cap > 0) run_search<true>(d, s_tilde, sv, cand, tau, w, cap, block_size, budget, idx_out, st);
    return hipGetLastError();
}

}  // namespace sablock
