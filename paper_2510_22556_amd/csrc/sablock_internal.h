// Internal declarations shared by the host ABI layer and the kernel files.
#pragma once

#include <hip/hip_runtime.h>
#include <algorithm>
#include <stdint.h>
#include <stddef.h>

#include "../../include/sablock.h"

namespace sablock {

// Host-validated view of one call; passed to kernels by value.
struct Dims {
    int32_t n_seq, n_layers, Hq, Hkv, G, D, L, W, T, M;   // M = G * W rows of the window-query matrix
    int32_t P;                                            // problems = n_seq * n_layers * Hkv
    int32_t dtype;
    int32_t cus;                                          // compute units the launch plans assume (never 0)
    int32_t local;                                        // a problem's workgroups share an XCD, see grid_problem
    uint32_t inv_heads, inv_seq;                          // ceil(2^32 / Hkv), ceil(2^32 / (n_layers * Hkv)); 0 for a divisor of 1
    sablock_tuning tune;                                  // the caller's launch parameters, validated (0 = plan)
    int64_t qs[4], ks[4], vs[4];
};

constexpr int MAX_SEQ = 64;
constexpr int MAX_CAND = 16;

struct SegView {
    const int32_t *seg_off;      // device, CSR
    int32_t seq_ptr[MAX_SEQ + 1];  // host copy of the CSR pointers, travels in the kernel arguments
    int32_t max_segments;
};

constexpr int MAX_DELIM = 64;

struct DelimSet {                  // delimiter token ids, by value in the kernel arguments
    int32_t n;
    int32_t id[MAX_DELIM];
};

struct SeqPtr {                    // host CSR pointers of the segment offsets, by value in the kernel arguments
    int32_t ptr[MAX_SEQ + 1];
};

constexpr int MAX_SLICES = 128;    // slices of all sequences of a sliced segmentation call
struct SlicePlaces {               // place of each slice's offsets, by value in the kernel arguments; the end of the last one behind them
    int32_t at[MAX_SLICES + 1];
};

// candidate block sizes; x / g = (x * inv) >> CAND_INV_BITS for 0 <= x < 4 160 (inv = ceil(2^19 / g), g <= 64)
constexpr int CAND_INV_BITS = 19;
struct CandList {
    int32_t n;
    int32_t g[MAX_CAND], inv[MAX_CAND];
};

// x / n for 0 <= x, n < 65 536 with inv = ceil(2^32 / n), 0 for n = 1 (x * inv exceeds x 2^32 / n by less than x, and x is
// below 2^32 / n, so the integer part of the quotient is right).  Every workgroup starts with the place of its problem, and three divisions by
// numbers that the compiler does not know are a hundred instructions, fetched cold.
__host__ __device__ inline uint32_t inverse_of(uint32_t n) { return n > 1 ? (uint32_t)(((1ull << 32) + n - 1) / n) : 0u; }
__host__ __device__ inline int32_t quotient(int32_t x, uint32_t inv) { return inv ? (int32_t)(((uint64_t)(uint32_t)x * inv) >> 32) : x; }
__host__ __device__ inline int32_t seq_of_problem(const Dims &d, int32_t p) { return quotient(p, d.inv_seq); }
__host__ __device__ inline int32_t head_of_problem(const Dims &d, int32_t p) { return p - quotient(p, d.inv_heads) * d.Hkv; }
__host__ __device__ inline int32_t layer_of_problem(const Dims &d, int32_t p)
{
    return quotient(p, d.inv_heads) - seq_of_problem(d, p) * d.n_layers;
}

// Grids over (parts, problems).  Workgroups go round the 8 XCDs, each of which has an L2
// cache of 4 MiB; where what the steps hand on to each other (12 bytes per key) fits these caches, the problems come first, so that
// with 8 problems, a layer of most models, every step finds what the one before it wrote in its own XCD's cache.  With more data
// nothing is left of it, and neighbouring workgroups had better read neighbouring memory.  The whole path against parts first, G = 4, W =
// 32: 8 problems of 8 192 keys 46.6 -> 43.0 us, of 131 072 137.9 -> 134.0; 9, 12, 20 and 28 of 20 011 1.00, 0.97, 0.97 and 0.96 of the time;
// at the line, 16 of 131 072 229 -> 232, 64 of 20 011 184 -> 178 (147 shapes of 1 to 120 problems: 0.91 to 1.02).
// A grid's second axis has 65 535 places: problems always fit it (make_dims), parts that do not come first.  Clears d.local for them:
// the kernel gets the same d.
constexpr unsigned GRID_Y_MOST = 65535;
__host__ inline dim3 parts_grid(Dims &d, unsigned parts, unsigned z = 1)
{
    if (parts > GRID_Y_MOST) d.local = 0;
    return d.local ? dim3(d.P, parts, z) : dim3(parts, d.P, z);
}
__device__ __forceinline__ int grid_problem(const Dims &d) { return d.local ? blockIdx.x : blockIdx.y; }
__device__ __forceinline__ int grid_part(const Dims &d) { return d.local ? blockIdx.y : blockIdx.x; }
__device__ __forceinline__ int grid_parts(const Dims &d) { return d.local ? gridDim.y : gridDim.x; }

__host__ __device__ inline int64_t k_problem_offset(const Dims &d, int32_t p)
{
    return seq_of_problem(d, p) * d.ks[0] + layer_of_problem(d, p) * d.ks[1] + head_of_problem(d, p) * d.ks[2];
}
__host__ __device__ inline int64_t v_problem_offset(const Dims &d, int32_t p)
{
    return seq_of_problem(d, p) * d.vs[0] + layer_of_problem(d, p) * d.vs[1] + head_of_problem(d, p) * d.vs[2];
}
// offset of window-query row (h_local, i) of problem p
__host__ __device__ inline int64_t q_row_offset(const Dims &d, int32_t p, int32_t h_local, int32_t i)
{
    return seq_of_problem(d, p) * d.qs[0] + layer_of_problem(d, p) * d.qs[1] +
           (int64_t)(head_of_problem(d, p) * d.G + h_local) * d.qs[2] + (int64_t)i * d.qs[3];
}

// order-preserving map float -> uint32 (larger float <=> larger key; -0.0 and +0.0 share a key, as they compare equal)
__host__ __device__ inline uint32_t ordered_key(float f)
{
    uint32_t u;
#if defined(__HIP_DEVICE_COMPILE__)
    u = __float_as_uint(f);
#else
    __builtin_memcpy(&u, &f, 4);
#endif
    if (u == 0x80000000u) u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Keys per workgroup: a problem's L keys in chunks of `len`, the last one what is left.  A workgroup costs its keys and `fixed`
// keys' time besides (prologue, epilogue); `slots` of them run at a time.  Equal chunks in whole rounds of workgroups, or, where
// those leave places idle, larger ones whose remainders the idle places take (96 problems on 256: two and a shorter one); then
// the workgroups start chunk by chunk (by_chunk), all problems' first ones first.  At most `most` keys each, and `wgs`
// workgroups in all where one round needs no more.  Where one round does, more of them have to gain a ninth or to have chunks of
// `from_one` keys; where several do, chunks are not cut below `shortest`.
struct ChunkPlan { int len, n; bool by_chunk; };
inline ChunkPlan plan_chunks(int64_t P, int64_t L, int64_t slots, int step, int fixed, int64_t most, int64_t wgs, int shortest, int from_one,
                             bool remainders)
{
    auto up = [&](int64_t keys) { return (keys + step - 1) / step * step; };
    int64_t best = 0, best_len = up(L);
    bool by_chunk = false;
    auto offer = [&](int64_t cost, int64_t len, bool rest) {
        if (best == 0 || cost < best) { best = cost; best_len = len; by_chunk = rest; }
    };
    const int64_t least = (L + most - 1) / most, first = std::max<int64_t>(1, (least * P + slots - 1) / slots);
    int64_t one = 0, one_len = 0;
    for (int64_t r = first; r < first + 8; ++r) {              // r rounds of equal chunks
        const int64_t n = r * slots / P, len = std::min(up((L + n - 1) / n), most);
        if (r > first && (P * n > wgs || (first > 1 && len < shortest))) break;
        offer((P * ((L + len - 1) / len) + slots - 1) / slots * (len + fixed), len, false);
        if (r == 1) { one = best; one_len = len; }
        if (len == step) break;
    }
    const int64_t ideal = P * L / slots + fixed;
    // where they would gain a twelfth or more (a tenth where whole rows fit one round), and with remainders of a quarter or more: with most
    // places taken the memory is as busy as it gets (128 rows, 30 011 keys on 256 places: 112 problems in two chunks 302 us, in two and a sixth
    // 315; 56 in four 185, in four and two fifths 171)
    const int64_t equal = best;
    if (remainders && equal * 100 > ideal * 108)
        for (int64_t n = std::max<int64_t>(2, least); n <= 6 && P * n <= wgs; ++n) {     // n - 1 chunks and the remainder of each
            const int64_t from = up((L + n - 1) / n), to = std::min(up((L + n - 2) / (n - 1)) - step, most), by = std::max<int64_t>(step, up((to - from) / 16));
            for (int64_t len = from + by; len <= to; len += by) {
                if (4 * (L - (n - 1) * len) < len || len < shortest) continue;
                const int64_t big = len + fixed, small = L - (n - 1) * len + fixed, q = P * (n - 1) / slots, late = P * (n - 1) % slots;
                // `late` places have q + 1 chunks, the others q and a chunk's time for remainders; what is over comes on top
                const int64_t per = big / small, early = slots - late, room = late ? early * per : 0, over = std::max<int64_t>(0, P - room);
                // a few places that take remainders one behind the other need some to spare (128 rows, 109 problems of 22 569 keys in two chunks
                // 235 us, in two and a quarter, room for 114 remainders, 266; 64 rows of heads of 64, 106 of 21 609, room for 132, 147 and 134)
                if (n > 2 && over == 0 && room * 100 <= P * (100 + 6 * (per - 1) * (per - 1))) continue;
                const int64_t cost = (late ? q + 1 : q) * big + (over + slots - 1) / slots * small;
                if (cost * 108 < equal * 100 && (one_len < L || cost * 100 < one * 90)) offer(cost, len, true);
            }
        }
    if (one > 0 && !by_chunk && best * 100 >= one * 89 && best_len < from_one) best_len = one_len;
    return {(int)best_len, (int)((L + best_len - 1) / best_len), by_chunk};
}

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// ---- kernel launchers (each returns the hipError_t of its launches) ----

// generic (any shape/dtype) scoring; row statistics go through ws
size_t score_generic_ws_bytes(const Dims &d);
hipError_t launch_score_generic(const Dims &d, const void *q, const void *k, const float *row_lse, float eps,
                                float *s_out, float *ent_out, void *ws, hipStream_t st);

// MFMA scoring for bf16 (which shapes: score_mfma_supported)
bool score_mfma_supported(const Dims &d);
size_t score_mfma_ws_bytes(const Dims &d);
hipError_t launch_score_mfma(const Dims &d, const void *q, const void *k, const float *row_lse, float eps,
                             float *s_out, float *ent_out, void *ws, hipStream_t st);

// measurement aid: K streamed through the scoring kernels' load ring with no arithmetic
bool stream_probe_supported(const Dims &d);
hipError_t launch_stream_probe(const Dims &d, const void *k, int read_lds, float *s_out, float *e_out, void *sink,
                               hipStream_t st);

// head mean over all query heads of a layer (one score row per layer)
bool score_all_heads_supported(const Dims &d);
size_t score_all_heads_ws_bytes(const Dims &d);
hipError_t launch_score_all_heads(const Dims &d, const void *q, const void *k, const float *row_lse, float eps,
                                  float *s_out, float *ent_out, void *ws, hipStream_t st);

hipError_t launch_refine(const Dims &d, const float *s, const float *ent, const SegView &sv,
                         sablock_hparams hp, float *s_tilde, float *omega, hipStream_t st);

// Top-B threshold per problem: thr[p] = {ordered key of the B-th best score, index cut among its ties}
hipError_t launch_topb(const Dims &d, const float *s_tilde, int32_t budget, int32_t *thr, hipStream_t st);

size_t search_ws_bytes(const Dims &d, int32_t max_segments, int32_t budget);
hipError_t launch_search(const Dims &d, const float *s_tilde, const SegView &sv, const CandList &cand,
                         int32_t budget, float tau, int32_t *seg_budget, int32_t *block_size, int32_t *topb_out,
                         void *ws, hipStream_t st);

size_t select_ws_bytes(const Dims &d, int32_t max_segments, int32_t budget);
hipError_t launch_select(const Dims &d, const float *s_tilde, const SegView &sv, const int32_t *seg_budget,
                         const int32_t *block_size, const int32_t *topb, int32_t budget, int32_t *idx_out,
                         int32_t *n_sel_out, void *ws, hipStream_t st);

// search and select in one sequence: same results as launch_search followed by launch_select; when the Top-B
// tokens and the segment counters of a problem fit on chip (search_select_fused) the Top-B kernel also plans the
// output rows and the search kernel writes the selected tokens, so no select kernel runs
bool search_select_fused(const Dims &d, const SegView &sv, int32_t budget);
size_t search_select_ws_bytes(const Dims &d, int32_t max_segments, int32_t budget);
hipError_t launch_search_select(const Dims &d, const float *s_tilde, const SegView &sv, const CandList &cand,
                                int32_t budget, float tau, int32_t *seg_budget, int32_t *block_size, int32_t *topb_out,
                                int32_t *idx_out, int32_t *n_sel_out, void *ws, hipStream_t st);

hipError_t launch_compact(const Dims &d, const void *k, const void *v, const int32_t *idx,
                          const int32_t *n_sel, int32_t budget, int32_t append_window,
                          void *k_out, void *v_out, int32_t shared_rows, hipStream_t st);

// punctuation-based segmentation (the step before the path)
hipError_t launch_segment_count(const int32_t *tok, int64_t stride, int32_t n_seq, int32_t T, const DelimSet &ds,
                                int32_t *seg_count, hipStream_t st);
hipError_t launch_segment_offsets(const int32_t *tok, int64_t stride, int32_t n_seq, int32_t T, const DelimSet &ds,
                                  const SeqPtr &sp, int32_t *seg_off, hipStream_t st);
// the same by slices of 16 384 tokens (segment_slices of them per sequence), whose counts the caller fetches in between
int segment_slices(int32_t T);
hipError_t launch_segment_slice_count(const int32_t *tok, int64_t stride, int32_t n_seq, int32_t T, const DelimSet &ds,
                                      int32_t *count, hipStream_t st);
hipError_t launch_segment_slice_offsets(const int32_t *tok, int64_t stride, int32_t n_seq, int32_t T, const DelimSet &ds,
                                        const SlicePlaces &sp, int32_t *seg_off, hipStream_t st);
hipError_t launch_segment_check(const int32_t *seg_off, int32_t n_seq, int32_t T, const SeqPtr &sp, int32_t *bad,
                                hipStream_t st);

// Opt-ins that hold per device (dynamic LDS above 64 KiB for a kernel) are made once per host thread and device:
//     static thread_local PerDeviceOnce once;  if (once.needed()) { ...; once.done(); }
// A thread that switches devices simply makes them again.
struct PerDeviceOnce {
    int done_dev = -1, cur = -1;
    bool needed()
    {
        if (hipGetDevice(&cur) != hipSuccess) cur = -1;
        return cur < 0 || cur != done_dev;
    }
    void done() { done_dev = cur; }
};

// row statistics of the scoring step by the attention kernel's first product alone, a lane per window query, for 129 .. 256
// window-query rows per KV head and for G = 4 with W = 32; on request (tuning.stats_per_key = 2): stats [P][row_stats_chunks][G * W][2] = (reference in the log2 domain, sum)
bool row_stats_supported(const Dims &d);
int row_stats_chunks(const Dims &d);
hipError_t launch_row_stats(const Dims &d, const void *q, const void *k, float *stats, hipStream_t st);

// attention of the window queries over all keys, with the rows' log-sum-exp (the producer of sablock_score's row_lse)
bool window_attention_supported(const Dims &d);
size_t window_attention_ws_bytes(const Dims &d);
hipError_t launch_window_attention(const Dims &d, const void *q, const void *k, const void *v, float *out, float *lse,
                                   void *ws, hipStream_t st);

// decode-time attention over a cache (the step after the path); d.L = rows of the cache buffers
bool decode_supported(const Dims &d);
size_t decode_ws_bytes(const Dims &d);
hipError_t launch_decode(const Dims &d, const void *q, const void *k, const void *v, const int32_t *n_sel,
                         int32_t budget, float *out, void *ws, hipStream_t st);

}  // namespace sablock
