// Window scoring for any shape and element type (Sec. 3.2, Eqs. barA, st, Dk).
//
// The path for fp32 inputs and for shapes that the bf16 matrix kernels do not cover.  The contraction runs on the fp32
// matrix instructions (products and sums in fp32, twice the rate of the vector pipe), bf16 inputs widened exactly.
//
// A window is padded to WP = 8, 16, 32 or 64 queries and the rows head * WP + query are cut into tiles of 32, so a tile
// holds several heads, one, or half of one; padding rows have zero queries and an infinite log-sum-exp, so they add exact
// zeros.  A wavefront works on 32 keys at a time, which it loads straight into registers (the two halves of the wavefront
// take alternate groups of four elements: any order of the contraction's index is as good, as long as both operands
// follow it); the queries come from LDS, four steps per 16-byte read.
//
// Pass 1 (skipped when the caller supplies row_lse): scores transposed, a lane per row, running (max, sum exp) of its
// scaled logits over the visible keys of a chunk.  Pass 2: a lane per key; probabilities exp2(x - lse), head mean,
// column sum s_t and the per-token entropy term.  The chunk partials are folded in pass 2's prologue while that is little,
// else by a kernel of their own.
//
// What bounds it: the fp32 matrix pipe where a problem has many rows (128 rows of 128 elements, 32 problems of 8 200 fp32
// keys: 111 + 136 us for the two passes = 77 and 63 TFLOP/s of 157; 943 us on the vector pipe, eight rows at a time from
// LDS), the key stream where it has few (32 rows, 80 problems of 13 000: 148 + 139 us, 3.6 TB/s), latency in the smallest
// calls (2 problems of 2 048: 5.5 + 6.6 us; 44 on the vector pipe in three kernels).
#include "sablock_internal.h"

#include <algorithm>

namespace sablock {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int NT = 256;                // threads per workgroup
constexpr int NW = NT / 64;
constexpr int KEYS = 32;               // keys of a wavefront
constexpr int QPAD = 4;                // floats behind a query row in LDS: consecutive rows start four banks apart
constexpr size_t Q_LDS = 64 * 1024;    // queries held in LDS at a time
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

struct GenArgs {
    Dims d;
    const void *q, *k;
    int n_tiles;           // 32-row tiles per problem
    int stage_tiles;       // of them held in LDS at a time (pass 2)
    int chunk_len, n_chunks;           // keys per workgroup of pass 1, a multiple of NW * KEYS
    float c1;              // log2(e) / sqrt(D)
    float eps;
    float *partial;        // [P][n_chunks][M][2] (max, sum exp2), log2 domain; the padding has no entries
    const float *merged;   // the same with pc chunks
    int pc;
    const float *lse;      // optional [P][G * W], natural log
    float *s_out, *e_out;
};

__device__ inline floatx4 load4(const float *p) { return *reinterpret_cast<const floatx4 *>(p); }
__device__ inline floatx4 load4(const uint16_t *p)             // bf16 bit patterns
{
    const uint2 u = *reinterpret_cast<const uint2 *>(p);
    return floatx4{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u)};
}

// row of a 32 x 32 result tile that accumulator register i of lane half hf holds
__device__ inline int tile_row(int i, int hf) { return 8 * (i >> 2) + 4 * hf + (i & 3); }

// this lane's share of a key row: elements 8 s + 4 hf .. + 3
template <typename T, int KS>
__device__ inline void load_key(floatx4 (&kf)[KS], const T *row, int hf, int ns)
{
#pragma unroll
    for (int s = 0; s < KS; ++s)
        if (s < ns) kf[s] = load4(row + 8 * s + 4 * hf);
}

// rows 32 j0 .. 32 (j0 + n) - 1 of the problem's padded window-query matrix to LDS
template <typename T, int WP>
__device__ inline void stage_queries(const GenArgs &a, int p, int j0, int n, float *q_lds)
{
    const Dims &d = a.d;
    const int per_row = d.D / 4, stride = d.D + QPAD;
    const T *q = static_cast<const T *>(a.q);
    for (int e = threadIdx.x; e < 32 * n * per_row; e += NT) {
        const int rr = e / per_row, c = e - rr * per_row, R = 32 * j0 + rr, h = R / WP, i = R % WP;
        floatx4 v = {0.f, 0.f, 0.f, 0.f};
        if (h < d.G && i < d.W) v = load4(q + q_row_offset(d, p, h, i) + 4 * c);
        *reinterpret_cast<floatx4 *>(q_lds + rr * stride + 4 * c) = v;
    }
}

// 32 x 32 products of the keys in registers with the query tile at qt.  KEY_ROWS: keys are the rows of the result.
template <bool KEY_ROWS, int KS>
__device__ inline floatx16 products(const floatx4 (&kf)[KS], const float *qt, int stride, int n, int hf, int ns)
{
    floatx16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    const float *row = qt + n * stride + 4 * hf;
#pragma unroll
    for (int s = 0; s < KS; ++s)
        if (s < ns) {
            const floatx4 qv = *reinterpret_cast<const floatx4 *>(row + 8 * s);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc = KEY_ROWS ? __builtin_amdgcn_mfma_f32_32x32x2f32(kf[s][j], qv[j], acc, 0, 0, 0)
                               : __builtin_amdgcn_mfma_f32_32x32x2f32(qv[j], kf[s][j], acc, 0, 0, 0);
        }
    return acc;
}

// (m, z) += (m2, z2): references in the log2 domain and sums relative to them; z = 0: nothing yet
__device__ inline void fold(float &m, float &z, float m2, float z2)
{
    const float mn = fmaxf(m, m2);
    z = (z > 0.f ? z * __builtin_amdgcn_exp2f(m - mn) : 0.f) + (z2 > 0.f ? z2 * __builtin_amdgcn_exp2f(m2 - mn) : 0.f);
    m = mn;
}
__device__ inline float other_half(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float((threadIdx.x & 32) ? r[0] : r[1]);
}

// ---------------------------------------------------------------- pass 1
// grid (n_chunks, n_tiles, P)
template <typename T, int KS, int WP>
__global__ void __launch_bounds__(NT)
score_generic_stats(GenArgs a)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const Dims &d = a.d;
    const int stride = d.D + QPAD, ns = d.D / 8;
    float *red = lds + 32 * stride;                            // [NW][32][2]
    const int chunk = blockIdx.x, J = blockIdx.y, p = blockIdx.z;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = lane & 31, hf = lane >> 5;
    const T *kp = static_cast<const T *>(a.k) + k_problem_offset(d, p);
    const int lo = chunk * a.chunk_len, hi = min(lo + a.chunk_len, d.L);
    constexpr bool PREFETCH = KS <= 16;                        // two key tiles fit the registers
    floatx4 kf[KS], nx[PREFETCH ? KS : 1];
    int t0 = lo + wave * KEYS;
    if (t0 < hi) load_key<T, KS>(kf, kp + (int64_t)min(t0 + n, d.L - 1) * d.ks[3], hf, ns);
    stage_queries<T, WP>(a, p, J, 1, lds);
    __syncthreads();

    const int last_seen = d.T + (32 * J + n) % WP;             // last key that this lane's row sees
    float m = -INFINITY, z = 0.f;
    for (; t0 < hi; t0 += NW * KEYS) {
        const int t1 = t0 + NW * KEYS;
        if constexpr (PREFETCH) {
            if (t1 < hi) load_key<T, KS>(nx, kp + (int64_t)min(t1 + n, d.L - 1) * d.ks[3], hf, ns);
        }
        floatx16 acc = products<true, KS>(kf, lds, stride, n, hf, ns);
        if (t0 + KEYS > d.T) {                                 // causal inside the window, end of the sequence
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int t = t0 + tile_row(i, hf);
                if (t >= d.L || t > last_seen) acc[i] = -INFINITY;
            }
        }
        float mx = acc[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, acc[i]);
        mx *= a.c1;
        if (mx > m) {
            z *= __builtin_amdgcn_exp2f(m - mx);
            m = mx;
        }
        if (m > -INFINITY) {
#pragma unroll
            for (int i = 0; i < 16; ++i) z += fmaxf(__builtin_amdgcn_exp2f(fmaf(acc[i], a.c1, -m)), 0.f);    // not a number: no part of the sum
        }
        if constexpr (PREFETCH) {
#pragma unroll
            for (int s = 0; s < KS; ++s) kf[s] = nx[s];
        } else if (t1 < hi) {
            load_key<T, KS>(kf, kp + (int64_t)min(t1 + n, d.L - 1) * d.ks[3], hf, ns);
        }
    }
    fold(m, z, other_half(m), other_half(z));
    if (hf == 0) { red[(wave * 32 + n) * 2] = m; red[(wave * 32 + n) * 2 + 1] = z; }
    __syncthreads();
    if (threadIdx.x < 32) {
        m = red[2 * n]; z = red[2 * n + 1];
        for (int w = 1; w < NW; ++w) fold(m, z, red[(w * 32 + n) * 2], red[(w * 32 + n) * 2 + 1]);
        const int h = (32 * J + n) / WP, i = (32 * J + n) % WP;
        if (h < d.G && i < d.W)
            *reinterpret_cast<float2 *>(a.partial + (((int64_t)p * a.n_chunks + chunk) * d.M + h * d.W + i) * 2) = make_float2(m, z);
    }
}

// one thread per (problem, row): the chunks' pairs to one
__global__ void __launch_bounds__(NT)
score_generic_combine(const float *partial, float *merged, int n_chunks, int rows, int n)
{
    const int g = blockIdx.x * NT + threadIdx.x;
    if (g >= n) return;
    const int p = g / rows, r = g - p * rows;
    float m = -INFINITY, z = 0.f;
#pragma unroll 8
    for (int c = 0; c < n_chunks; ++c) {
        const float2 e = *reinterpret_cast<const float2 *>(partial + (((int64_t)p * n_chunks + c) * rows + r) * 2);
        fold(m, z, e.x, e.y);
    }
    *reinterpret_cast<float2 *>(merged + (int64_t)g * 2) = make_float2(m, z);
}

// ---------------------------------------------------------------- pass 2
// grid (workgroups per problem, P); the wavefronts of a problem's workgroups stride over its tiles of 32 keys
template <typename T, int KS, int WP>
__global__ void __launch_bounds__(NT)
score_generic_columns(GenArgs a)
{
    constexpr int QB = WP == 64 ? 2 : 1;                       // tiles of one head
    constexpr int NS = WP >= 32 ? 16 * QB : WP / 2;            // head-mean values per lane
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const Dims &d = a.d;
    const int stride = d.D + QPAD, ns = d.D / 8, rows = 32 * a.n_tiles;
    float *lse2 = lds;                                         // [rows] log2-domain log-sum-exp + log2 G
    float *q_lds = lds + rows;
    const int p = blockIdx.y;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = lane & 31, hf = lane >> 5;
    const T *kp = static_cast<const T *>(a.k) + k_problem_offset(d, p);
    const int n_kt = (d.L + KEYS - 1) / KEYS, step = gridDim.x * NW;
    int kt = blockIdx.x * NW + wave;
    constexpr bool PREFETCH = KS <= 16;
    floatx4 kf[KS], nx[PREFETCH ? KS : 1];
    if (kt < n_kt) load_key<T, KS>(kf, kp + (int64_t)min(kt * KEYS + n, d.L - 1) * d.ks[3], hf, ns);

    const float log2_G = __builtin_amdgcn_logf((float)d.G);
    for (int R = threadIdx.x; R < rows; R += NT) {
        const int h = R / WP, i = R % WP;
        float m = INFINITY, z = 1.f;                           // padding row
        if (h < d.G && i < d.W) {
            if (a.lse) m = a.lse[(int64_t)p * d.M + h * d.W + i] * LOG2E;
            else {
                m = -INFINITY;
                z = 0.f;
#pragma unroll 8
                for (int c = 0; c < a.pc; ++c) {
                    const float2 e = *reinterpret_cast<const float2 *>(a.merged + (((int64_t)p * a.pc + c) * d.M + h * d.W + i) * 2);
                    fold(m, z, e.x, e.y);
                }
            }
        }
        lse2[R] = m + __builtin_amdgcn_logf(z) + log2_G;
    }
    const bool all_staged = a.stage_tiles >= a.n_tiles;
    if (all_staged) stage_queries<T, WP>(a, p, 0, a.n_tiles, q_lds);
    __syncthreads();

    float *out = (hf == 0 ? a.s_out : a.e_out) + (int64_t)p * d.L;
    for (int base = blockIdx.x * NW; base < n_kt; base += step, kt += step) {          // uniform over the workgroup
        const bool live = kt < n_kt;
        if constexpr (PREFETCH) {
            if (kt + step < n_kt) load_key<T, KS>(nx, kp + (int64_t)min((kt + step) * KEYS + n, d.L - 1) * d.ks[3], hf, ns);
        }
        const int t = kt * KEYS + n;
        const bool edge = (kt + 1) * KEYS > d.T;
        float ab[NS];
#pragma unroll
        for (int i = 0; i < NS; ++i) ab[i] = 0.f;
        for (int j0 = 0; j0 < a.n_tiles; j0 += a.stage_tiles) {
            const int j1 = min(j0 + a.stage_tiles, a.n_tiles);
            if (!all_staged) {
                __syncthreads();
                stage_queries<T, WP>(a, p, j0, j1 - j0, q_lds);
                __syncthreads();
            }
            if (!live) continue;
            for (int J = j0; J < j1; J += QB) {
#pragma unroll
                for (int b = 0; b < QB; ++b) {
                    const floatx16 acc = products<false, KS>(kf, q_lds + (J + b - j0) * 32 * stride, stride, n, hf, ns);
                    const float *ls = lse2 + 32 * (J + b) + 4 * hf;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int r = tile_row(i, hf);
                        float v = __builtin_amdgcn_exp2f(fmaf(acc[i], a.c1, -ls[8 * (i >> 2) + (i & 3)]));              // A / G
                        if (edge && !(t < d.L && t <= d.T + (WP >= 32 ? 32 * b + r : r % WP))) v = 0.f;                 // causal inside the window
                        ab[WP >= 32 ? 16 * b + i : i % (WP / 2)] += v;                                                  // Eq. barA
                    }
                }
            }
        }
        if (live) {
            float s = 0.f;
#pragma unroll
            for (int i = 0; i < NS; ++i) s += ab[i];
            s += other_half(s);                                                                                         // Eq. st
            const float inv_s = s > 0.f ? 1.0f / s : 0.f;
            float e = 0.f;
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                const float ah = ab[i] * inv_s;
                e = fmaf(ah, __builtin_amdgcn_logf(ah + a.eps), e);
            }
            e += other_half(e);
            if (t < d.L) out[t] = hf == 0 ? s : s > 0.f ? -LN2 * e : 0.f;                                                             // inner sum of Eq. Dk
        }
        if constexpr (PREFETCH) {
#pragma unroll
            for (int s = 0; s < KS; ++s) kf[s] = nx[s];
        } else if (kt + step < n_kt) {
            load_key<T, KS>(kf, kp + (int64_t)min((kt + step) * KEYS + n, d.L - 1) * d.ks[3], hf, ns);
        }
    }
}

// ---------------------------------------------------------------- launches
int padded_window(const Dims &d) { return d.W <= 8 ? 8 : d.W <= 16 ? 16 : d.W <= 32 ? 32 : 64; }
int row_tiles(const Dims &d)
{
    const int wp = padded_window(d);
    return wp == 64 ? 2 * d.G : (d.G * wp + 31) / 32;
}

// Workgroups that the registers let a compute unit hold (512 per lane and SIMD, one wavefront of each workgroup on each):
// statistics 104 and, widened from bf16, 124 up to 64 elements, 168 and 172 up to 128, 176 above; columns up to 168, 216
// and 216, with padded windows of 64 228, 276 and 280.  One round of them, so that none starts late: against three where
// two fit and two where one does, columns of 8 problems of 8 200 fp32 keys, 256 rows of 128 140 -> 108 us, statistics of
// 8 of 32 768 bf16 keys, 48 rows of 128 99 -> 67 us.
int stats_per_cu(const Dims &d) { return d.D <= 64 ? 4 : d.D <= 128 && d.dtype == SABLOCK_F32 ? 3 : 2; }
int columns_per_cu(const Dims &d) { return (d.D <= 64 ? 3 : 2) - (padded_window(d) == 64 ? 1 : 0); }

// Pass 1: a workgroup per row tile and chunk of keys, at most 64 chunks.
void plan_chunks(const Dims &d, int *chunk_len, int *n_chunks)
{
    const int64_t per_tile = std::max<int64_t>(1, (int64_t)stats_per_cu(d) * d.cus / ((int64_t)d.P * row_tiles(d)));
    const int64_t chunks = std::min<int64_t>(64, per_tile);
    const int unit = NW * KEYS;
    *chunk_len = (int)(((d.L + chunks - 1) / chunks + unit - 1) / unit) * unit;
    *n_chunks = (d.L + *chunk_len - 1) / *chunk_len;
}
// (max, sum) pairs that a workgroup of pass 2 folds itself: up to 16 per thread, under the loads of its first keys
bool folds_in_pass2(const Dims &d, int n_chunks) { return (int64_t)n_chunks * 32 * row_tiles(d) <= 16 * NT; }

template <typename T, int KS, int WP>
hipError_t launch(GenArgs &a, hipStream_t st)
{
    const Dims &d = a.d;
    const size_t tile_bytes = (size_t)32 * (d.D + QPAD) * 4;
    const int rows = 32 * a.n_tiles;
    constexpr int QB = WP == 64 ? 2 : 1;
    a.stage_tiles = std::min<int>(a.n_tiles, std::max<int>(QB, (int)(Q_LDS / tile_bytes) / QB * QB));
    const size_t lds2 = (size_t)rows * 4 + a.stage_tiles * tile_bytes;
    if (lds2 > 64 * 1024) {
        static thread_local PerDeviceOnce attr_once;
        if (attr_once.needed()) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(score_generic_columns<T, KS, WP>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
            if (e != hipSuccess) return e;
            attr_once.done();
        }
    }
    if (!a.lse) {
        hipLaunchKernelGGL((score_generic_stats<T, KS, WP>), dim3(a.n_chunks, a.n_tiles, d.P), dim3(NT), tile_bytes + NW * 32 * 2 * 4, st, a);
        if (!folds_in_pass2(d, a.n_chunks)) {
            float *merged = a.partial + (size_t)d.P * a.n_chunks * d.M * 2;
            const int n = d.P * d.M;
            hipLaunchKernelGGL(score_generic_combine, dim3((n + NT - 1) / NT), dim3(NT), 0, st, a.partial, merged, a.n_chunks, d.M, n);
            a.merged = merged;
            a.pc = 1;
        }
    }
    const int n_kt = (d.L + KEYS - 1) / KEYS;
    const int64_t all = (n_kt + NW - 1) / NW, room = std::max<int64_t>(1, (int64_t)columns_per_cu(d) * d.cus / d.P);
    // queries that do not fit LDS are staged again for a second turn: a few late workgroups cost less than that (8 problems
    // of 8 200 keys, 256 rows of 64: 65 workgroups each 52 us, 64 of them 62)
    const int64_t wgs = all <= room + (a.stage_tiles < a.n_tiles ? room / 16 : 0) ? all : room;
    hipLaunchKernelGGL((score_generic_columns<T, KS, WP>), dim3((unsigned)wgs, d.P), dim3(NT), lds2, st, a);
    return hipGetLastError();
}

template <typename T, int KS>
hipError_t by_window(GenArgs &a, hipStream_t st)
{
    switch (padded_window(a.d)) {
    case 8: return launch<T, KS, 8>(a, st);
    case 16: return launch<T, KS, 16>(a, st);
    case 32: return launch<T, KS, 32>(a, st);
    default: return launch<T, KS, 64>(a, st);
    }
}
template <typename T>
hipError_t by_dim(GenArgs &a, hipStream_t st)
{
    if (a.d.D <= 64) return by_window<T, 8>(a, st);
    if (a.d.D <= 128) return by_window<T, 16>(a, st);
    return by_window<T, 32>(a, st);
}

}  // namespace

size_t score_generic_ws_bytes(const Dims &d)
{
    int chunk_len, n_chunks;
    plan_chunks(d, &chunk_len, &n_chunks);
    return align256((size_t)d.P * (n_chunks + (folds_in_pass2(d, n_chunks) ? 0 : 1)) * d.M * 2 * 4);
}

hipError_t launch_score_generic(const Dims &d, const void *q, const void *k, const float *row_lse, float eps,
                                float *s_out, float *ent_out, void *ws, hipStream_t st)
{
    GenArgs a = {};
    a.d = d;
    a.q = q;
    a.k = k;
    a.n_tiles = row_tiles(d);
    plan_chunks(d, &a.chunk_len, &a.n_chunks);
    a.c1 = (float)(1.4426950408889634 / sqrt((double)d.D));
    a.eps = eps;
    a.partial = static_cast<float *>(ws);
    a.merged = a.partial;
    a.pc = a.n_chunks;
    a.lse = row_lse;
    a.s_out = s_out;
    a.e_out = ent_out;
    return d.dtype == SABLOCK_F32 ? by_dim<float>(a, st) : by_dim<uint16_t>(a, st);
}

}  // namespace sablock
