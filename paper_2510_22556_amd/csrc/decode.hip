// Decode-time attention of one new token over a KV cache (Sec. 2.1 Eq. 1 for a single query position), for the
// compacted cache the compression path produces and for the full cache it replaces.  GQA: the G query heads of
// a KV head share its rows.  The work is one read of K and V, so the kernel is a plain streaming one:
//
//   decode_kernel        grid (splits, P).  A row (D elements) is spread over LPR = D*elt/16 consecutive lanes,
//       16 bytes each, so every load instruction of a wavefront covers whole consecutive rows; the lane groups of a
//       workgroup stride over the rows of the split, two or four rows of K and of V in flight each.  Logits of a row: every
//       lane forms its share of all G products, and the sum over the row's lanes hands each lane ONE head (lane % S,
//       S = 2, 4 or 8), so that the exponentials of a row are formed once and not once per lane; the probabilities go
//       back to the row's lanes by DPP.  Probabilities are relative to a reference per head that the whole wavefront
//       shares: it is set AHEAD (log2 domain) above the largest logit so far and moves only when a logit passes it, so
//       the weighted sums of V are not rescaled row by row and no probability exceeds one.  The lane
//       groups of a wavefront are merged by lane exchanges, the wavefronts through LDS.  With one split the workgroup
//       writes the result itself, else (reference, denominator, numerator[D]) per (problem, split, head).
//   decode_merge_kernel  merges the splits and divides.
//
// What bounds it: the cache read, as long as the vector work of a row stays below the time of its bytes; a read of 4 KB
// (four rows of K and of V per wavefront instruction) takes about 100 vector instructions at G = 4.  The
// full cache of 32 layers x 8 heads x 131 072 rows: 2.65 -> 2.48 ms (6.9 TB/s; exponentials and rescaling in every lane of
// a row, 168 instructions, before); seven heads per group, 240 problems of 3 593 rows of 128 bytes: 94 -> 49 us.
#include "sablock_internal.h"

#include <utility>

namespace sablock {
namespace {

constexpr int unroll_of(int G) { return G <= 4 ? 4 : 2; }               // rows in flight per lane group
constexpr int WIDE = 512;                  // threads of the workgroups that take a problem's rows alone
constexpr float AHEAD = 8.f;               // 2^-8 of the numbers' range at its small end, nothing at its large one

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// 16 bytes that are read once: non-temporal
__device__ inline u32x4 load16(const char *p) { return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p)); }

// value of lane ^ M
template <int M>
__device__ inline float xor_lane(float x)
{
    const int v = __float_as_int(x);
    if constexpr (M == 1) return __int_as_float(__builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true));
    if constexpr (M == 2) return __int_as_float(__builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true));
    if constexpr (M == 4) {                                    // banks 0, 2 from four lanes up, banks 1, 3 from four lanes down
        const int a = __builtin_amdgcn_update_dpp(v, v, 0x104, 0xF, 0x5, false);
        return __int_as_float(__builtin_amdgcn_update_dpp(a, v, 0x114, 0xF, 0xA, false));
    }
    if constexpr (M == 8) return __int_as_float(__builtin_amdgcn_mov_dpp(v, 0x128, 0xF, 0xF, true));
    if constexpr (M == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
        return __uint_as_float((threadIdx.x & 16) ? r[0] : r[1]);
    }
    const auto r = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
    return __uint_as_float((threadIdx.x & 32) ? r[0] : r[1]);
}
// value of the lane with the same place in the groups of S = 4, whose place inside the four is H
template <int H>
__device__ inline float quad_bcast(float x)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), H * 0x55, 0xF, 0xF, true));
}

// x[0 .. N) summed over the LPR lanes of a row, lane l getting the entries l % S + S j, j < N / S, in x[j]
template <int S, int B, int N>
__device__ inline void scatter_sum(float (&x)[N])
{
    if constexpr (B < S) {
        constexpr int M = N / (2 * B) > 0 ? N / (2 * B) : 1;   // entries left
        const bool up = threadIdx.x & B;
#pragma unroll
        for (int i = 0; i < M; ++i) {
            const float own = up ? x[2 * i + 1] : x[2 * i], other = up ? x[2 * i] : x[2 * i + 1];
            x[i] = own + xor_lane<B>(other);
        }
        scatter_sum<S, 2 * B, N>(x);
    }
}
template <int S, int LPR, int HP, int N>
__device__ inline void row_sums(float (&x)[N])
{
    scatter_sum<S, 1, N>(x);
#pragma unroll
    for (int j = 0; j < HP; ++j) {
        if constexpr (S <= 1 && LPR > 1) x[j] += xor_lane<1>(x[j]);
        if constexpr (S <= 2 && LPR > 2) x[j] += xor_lane<2>(x[j]);
        if constexpr (S <= 4 && LPR > 4) x[j] += xor_lane<4>(x[j]);
        if constexpr (S <= 8 && LPR > 8) x[j] += xor_lane<8>(x[j]);
        if constexpr (LPR > 16) x[j] += xor_lane<16>(x[j]);
        if constexpr (LPR > 32) x[j] += xor_lane<32>(x[j]);
    }
}
// f(integral_constant<int, g>) for every g
template <int... g, typename F>
__device__ inline void for_each_head(std::integer_sequence<int, g...>, F &&f) { (f(std::integral_constant<int, g>{}), ...); }

// entry g of values that lie as row_sums leaves them, in every lane
template <int S, int g, int HP>
__device__ inline float entry(const float (&x)[HP])
{
    const float v = x[g / S];
    if constexpr (S == 1) return v;
    if constexpr (S == 2) {
        const float o = xor_lane<1>(v);
        return ((threadIdx.x & 1) != 0) == (g % 2 != 0) ? v : o;
    }
    if constexpr (S == 4) return quad_bcast<g % 4>(v);
    const float o = xor_lane<4>(v);                            // S == 8
    return quad_bcast<g % 4>(((threadIdx.x & 4) != 0) == (g % 8 >= 4) ? v : o);
}

template <bool BF16> struct Chunk;         // 16 bytes of a row
template <> struct Chunk<true> {
    static constexpr int N = 8;
    static __device__ inline float dot(const u32x4 &a, const u32x4 &b, float c)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t x = a[i], y = b[i];                 // (a bit cast of the vector's element itself takes element 0)
            c = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, x), __builtin_bit_cast(bf16x2, y), c, false);
        }
        return c;
    }
    static __device__ inline float get(const u32x4 &v, int e) { return __uint_as_float((e & 1) ? v[e >> 1] & 0xffff0000u : v[e >> 1] << 16); }
};
template <> struct Chunk<false> {
    static constexpr int N = 4;
    static __device__ inline float dot(const u32x4 &a, const u32x4 &b, float c)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) c = fmaf(__uint_as_float(a[i]), __uint_as_float(b[i]), c);
        return c;
    }
    static __device__ inline float get(const u32x4 &v, int e) { return __uint_as_float(v[e]); }
};

struct DecodeArgs {
    Dims d;                 // d.L = rows of the cache buffers
    const char *q, *k, *v;
    const int32_t *n_sel;   // nullable; rows [n_sel[p], budget) of problem p hold nothing
    int budget;
    int rows_per_split, n_splits;
    float qscale;           // log2(e) / sqrt(D)
    float *part;            // [P][n_splits][G][2 + D]
    float *out;             // [n_seq][n_layers][Hq][D]
};

template <int G, bool BF16, int LPR, int NT>
__global__ void __launch_bounds__(NT)
decode_kernel(DecodeArgs a)
{
    constexpr int GP = G == 1 ? 1 : G == 2 ? 2 : G <= 4 ? 4 : 8;             // heads, padded
    constexpr int S = GP < LPR ? GP : LPR, HP = GP / S;                      // heads over S lanes, HP each
    constexpr int E = Chunk<BF16>::N, ELT = BF16 ? 2 : 4, D = LPR * E;
    constexpr int UNROLL = unroll_of(G);
    constexpr int NWV = NT / 64, groups = NT / LPR, STRIDE = 2 + D;
    __shared__ float sh[NWV * G * STRIDE];
    const Dims &d = a.d;
    const int p = blockIdx.y, split = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = threadIdx.x / LPR, sub = threadIdx.x % LPR;
    const int r0 = split * a.rows_per_split, r1 = min(r0 + a.rows_per_split, d.L);
    const int hole_lo = a.n_sel ? a.n_sel[p] : d.L, hole_hi = a.n_sel ? a.budget : d.L;   // rows without content
    const int head0 = head_of_problem(d, p) * G;
    const int64_t qbase = ((int64_t)(seq_of_problem(d, p) * d.n_layers + layer_of_problem(d, p)) * d.Hq + head0) * D;

    u32x4 q[G];
#pragma unroll
    for (int g = 0; g < G; ++g) q[g] = *reinterpret_cast<const u32x4 *>(a.q + (qbase + (int64_t)g * D) * ELT + sub * 16);
    float ref[HP], l[HP], acc[G][E];
#pragma unroll
    for (int j = 0; j < HP; ++j) { ref[j] = -INFINITY; l[j] = 0.f; }
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < E; ++e) acc[g][e] = 0.f;
    const char *kp = a.k + k_problem_offset(d, p) * ELT + (int64_t)sub * 16;
    const char *vp = a.v + v_problem_offset(d, p) * ELT + (int64_t)sub * 16;
    const int64_t kstep = d.ks[3] * ELT, vstep = d.vs[3] * ELT;

    // the wavefront's groups take the same number of steps (its exchanges span them)
    for (int rb = r0 + wave * (64 / LPR); rb < r1; rb += groups * UNROLL) {
        u32x4 kr[UNROLL], vr[UNROLL];
        bool live[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int r = rb + grp % (64 / LPR) + u * groups;
            live[u] = r < r1 && !(r >= hole_lo && r < hole_hi);
            const int rc = min(r, r1 - 1);                     // in bounds
            kr[u] = load16(kp + (int64_t)rc * kstep);
            vr[u] = load16(vp + (int64_t)rc * vstep);
        }
        // a row that is not live may hold anything, NaN and infinity too, and zero times those is NaN: its V counts as
        // zeros (its logit is replaced below).  Steps whose rows are all live skip this by a scalar test.
        const int last_row = rb + 64 / LPR - 1 + (UNROLL - 1) * groups;
        if (last_row >= r1 || (last_row >= hole_lo && rb < hole_hi)) {
#pragma unroll
            for (int u = 0; u < UNROLL; ++u)
                if (!live[u]) vr[u] = u32x4{0, 0, 0, 0};
        }
        float x[UNROLL][GP];
        float ahead = -INFINITY;
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
#pragma unroll
            for (int g = 0; g < GP; ++g) x[u][g] = g < G ? Chunk<BF16>::dot(q[g < G ? g : 0], kr[u], 0.f) : 0.f;
            row_sums<S, LPR, HP>(x[u]);
#pragma unroll
            for (int j = 0; j < HP; ++j) {
                x[u][j] = live[u] ? x[u][j] * a.qscale : -INFINITY;
                ahead = fmaxf(ahead, x[u][j] - ref[j]);        // +inf before the first live row, NaN (no maximum) while none is
            }
        }
        if (__ballot(ahead > 0.f) != 0ull) {
            // every head's reference to AHEAD above its largest logit among the wavefront's rows, or where it was
            float f[HP];
#pragma unroll
            for (int j = 0; j < HP; ++j) {
                float m = x[0][j];
#pragma unroll
                for (int u = 1; u < UNROLL; ++u) m = fmaxf(m, x[u][j]);
                if constexpr (S <= 1) m = fmaxf(m, xor_lane<1>(m));
                if constexpr (S <= 2) m = fmaxf(m, xor_lane<2>(m));
                if constexpr (S <= 4) m = fmaxf(m, xor_lane<4>(m));
                m = fmaxf(m, xor_lane<8>(m));
                m = fmaxf(m, xor_lane<16>(m));
                m = fmaxf(m, xor_lane<32>(m));
                m = m > ref[j] ? m + AHEAD : ref[j];
                f[j] = ref[j] > -INFINITY ? __builtin_amdgcn_exp2f(ref[j] - m) : 0.f;
                ref[j] = m;
                l[j] *= f[j];
            }
            for_each_head(std::make_integer_sequence<int, G>{}, [&](auto g) {
                const float fg = entry<S, g.value>(f);
#pragma unroll
                for (int e = 0; e < E; ++e) acc[g.value][e] *= fg;
            });
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            float pr[HP];
#pragma unroll
            for (int j = 0; j < HP; ++j) {
                pr[j] = x[u][j] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(x[u][j] - ref[j]);         // NaN stays NaN
                l[j] += pr[j];
            }
            float ve[E];
#pragma unroll
            for (int e = 0; e < E; ++e) ve[e] = Chunk<BF16>::get(vr[u], e);
            for_each_head(std::make_integer_sequence<int, G>{}, [&](auto g) {
                const float pg = entry<S, g.value>(pr);
#pragma unroll
                for (int e = 0; e < E; ++e) acc[g.value][e] = fmaf(pg, ve[e], acc[g.value][e]);
            });
        }
    }
    // merge the lane groups of the wavefront (they share the references) ...
    auto over_groups = [&](float v) {
        if constexpr (LPR <= 4) v += xor_lane<4>(v);
        if constexpr (LPR <= 8) v += xor_lane<8>(v);
        if constexpr (LPR <= 16) v += xor_lane<16>(v);
        if constexpr (LPR <= 32) v += xor_lane<32>(v);
        return v;
    };
#pragma unroll
    for (int j = 0; j < HP; ++j) l[j] = over_groups(l[j]);
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < E; ++e) acc[g][e] = over_groups(acc[g][e]);
    // ... and the wavefronts
    if (lane < LPR) {
#pragma unroll
        for (int j = 0; j < HP; ++j)
            if (lane < S && lane + S * j < G) {
                float *o = sh + (wave * G + lane + S * j) * STRIDE;
                o[0] = ref[j];
                o[1] = l[j];
            }
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int e = 0; e < E; ++e) sh[(wave * G + g) * STRIDE + 2 + lane * E + e] = acc[g][e];
    }
    __syncthreads();
    const bool last = a.n_splits == 1;
    float *po = a.part + ((int64_t)p * a.n_splits + split) * G * STRIDE;
    for (int i = threadIdx.x; i < G * D; i += NT) {
        const int g = i / D, c = i - g * D;
        float mx = -INFINITY;
#pragma unroll
        for (int w = 0; w < NWV; ++w) mx = fmaxf(mx, sh[(w * G + g) * STRIDE]);
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int w = 0; w < NWV; ++w) {
            const float *o = sh + (w * G + g) * STRIDE;
            const float f = mx > -INFINITY ? __builtin_amdgcn_exp2f(o[0] - mx) : 1.f;          // no row: zeros
            den += o[1] * f;
            num += o[2 + c] * f;
        }
        if (last) a.out[qbase + (int64_t)g * D + c] = den > 0.f ? num / den : 0.f;
        else {
            po[g * STRIDE + 2 + c] = num;
            if (c == 0) { po[g * STRIDE] = mx; po[g * STRIDE + 1] = den; }
        }
    }
}

// grid (G, P): the splits' weights first, one thread each, then their weighted sum, all loads independent
constexpr int MERGE_T = 256, MAX_SPLITS = MERGE_T;
__global__ void __launch_bounds__(MERGE_T)
decode_merge_kernel(DecodeArgs a)
{
    __shared__ float w_sh[MAX_SPLITS], red[2 * (MERGE_T / 64)], sum[MERGE_T];
    const Dims &d = a.d;
    const int g = blockIdx.x, p = blockIdx.y, D = d.D, stride = 2 + D, tid = threadIdx.x;
    const float *pp = a.part + ((int64_t)p * a.n_splits * d.G + g) * stride;
    const int64_t step = (int64_t)d.G * stride;
    float m = -INFINITY, z = 0.f;
    if (tid < a.n_splits) { m = pp[tid * step]; z = pp[tid * step + 1]; }
    float mx = m;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    if ((tid & 63) == 0) red[tid >> 6] = mx;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < MERGE_T / 64; ++w) mx = fmaxf(mx, red[w]);
    const float f = z == 0.f ? 0.f : __builtin_amdgcn_exp2f(m - mx);         // no row: nothing; NaN stays NaN
    w_sh[tid] = f;
    float den = z * f;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) den += __shfl_xor(den, o);
    if ((tid & 63) == 0) red[MERGE_T / 64 + (tid >> 6)] = den;
    __syncthreads();
    den = 0.f;
#pragma unroll
    for (int w = 0; w < MERGE_T / 64; ++w) den += red[MERGE_T / 64 + w];
    const int c = tid % D, part = tid / D, parts = MERGE_T / D;              // D is a power of two up to 256
    float num = 0.f;
#pragma unroll 8
    for (int s = part; s < a.n_splits; s += parts)
        num += pp[s * step + 2 + c] * w_sh[s];                 // a split without rows has written zeros
    sum[tid] = num;
    __syncthreads();
    if (part > 0) return;
    for (int i = 1; i < parts; ++i) num += sum[i * D + c];
    const int64_t o = ((int64_t)(seq_of_problem(d, p) * d.n_layers + layer_of_problem(d, p)) * d.Hq + head_of_problem(d, p) * d.G + g) * D;
    a.out[o + c] = den > 0.f ? num / den : 0.f;
}

// Splits of a problem's rows: eight workgroups per CU in all, 128 rows each at least.  One (a wide workgroup, no merge
// kernel) where the rows are so few that the merge would cost more than it saves (128 rows of 256 bytes: 7.1-7.4 us
// against 7.3-7.7), or half a CU's worth of problems and not too many rows (1 024 rows, 256 problems: 26.8 us against
// 32.5, 128 problems 19.2 against 20.5, 64 problems 18.5 against 13.4; 2 048 rows, 256 problems: 43.7 against 51.9).
struct DecodePlan { int n_splits; bool wide; };
DecodePlan decode_plan(const Dims &d)
{
    const int64_t chunks = (int64_t)d.L * (d.D * (d.dtype == SABLOCK_F32 ? 4 : 2) / 16);      // 16-byte pieces of K
    if (chunks <= 256 * 16 || (chunks <= 2048 * 16 && 2 * d.P >= d.cus)) return {1, true};
    int s = 1;
    while ((int64_t)d.P * s < 8 * d.cus && d.L / (s * 2) >= 128 && s * 2 <= MAX_SPLITS) s *= 2;
    return {s, false};
}

}  // namespace

bool decode_supported(const Dims &d)
{
    const int elt = d.dtype == SABLOCK_F32 ? 4 : 2;
    const int lpr = d.D * elt / 16;
    const bool pow2 = lpr >= 4 && lpr <= 64 && (lpr & (lpr - 1)) == 0 && lpr * 16 == d.D * elt;
    return pow2 && d.G >= 1 && d.G <= 8 && d.G * d.D <= 1024;
}

size_t decode_ws_bytes(const Dims &d)
{
    return align256((size_t)d.P * decode_plan(d).n_splits * d.G * (2 + d.D) * 4);
}

hipError_t launch_decode(const Dims &d, const void *q, const void *k, const void *v, const int32_t *n_sel,
                         int32_t budget, float *out, void *ws, hipStream_t st)
{
    if (d.P <= 0) return hipSuccess;
    const int elt = d.dtype == SABLOCK_F32 ? 4 : 2;
    const DecodePlan plan = decode_plan(d);
    DecodeArgs a;
    a.d = d;
    a.q = static_cast<const char *>(q);
    a.k = static_cast<const char *>(k);
    a.v = static_cast<const char *>(v);
    a.n_sel = n_sel;
    a.budget = budget;
    a.n_splits = plan.n_splits;
    a.rows_per_split = (d.L + a.n_splits - 1) / a.n_splits;
    const int lpr = d.D * elt / 16;
    a.qscale = (float)(1.4426950408889634 / sqrt((double)d.D));
    a.part = static_cast<float *>(ws);
    a.out = out;
    const bool bf = d.dtype == SABLOCK_BF16;
    // one instantiation per (G, dtype, lanes per row, threads)
    using Kern = void (*)(DecodeArgs);
    Kern fn = nullptr;
#define SABLOCK_DECODE_L(GV, BV, LV) \
    if constexpr (GV * LV * (BV ? 8 : 4) <= 1024) { \
        if (d.G == GV && bf == BV && lpr == LV) fn = plan.wide ? decode_kernel<GV, BV, LV, WIDE> : decode_kernel<GV, BV, LV, 256>; \
    }
#define SABLOCK_DECODE_G(GV)                                                                                         \
    SABLOCK_DECODE_L(GV, true, 4) SABLOCK_DECODE_L(GV, true, 8) SABLOCK_DECODE_L(GV, true, 16) SABLOCK_DECODE_L(GV, true, 32) \
    SABLOCK_DECODE_L(GV, false, 4) SABLOCK_DECODE_L(GV, false, 8) SABLOCK_DECODE_L(GV, false, 16)                    \
    SABLOCK_DECODE_L(GV, false, 32) SABLOCK_DECODE_L(GV, false, 64)
    SABLOCK_DECODE_G(1) SABLOCK_DECODE_G(2) SABLOCK_DECODE_G(3) SABLOCK_DECODE_G(4) SABLOCK_DECODE_G(5) SABLOCK_DECODE_G(6)
    SABLOCK_DECODE_G(7) SABLOCK_DECODE_G(8)
#undef SABLOCK_DECODE_G
#undef SABLOCK_DECODE_L
    if (!fn) return hipErrorInvalidValue;
    hipLaunchKernelGGL(fn, dim3(a.n_splits, d.P), dim3(plan.wide ? WIDE : 256), 0, st, a);
    if (a.n_splits > 1) hipLaunchKernelGGL(decode_merge_kernel, dim3(d.G, d.P), dim3(MERGE_T), 0, st, a);
    return hipGetLastError();
}

}  // namespace sablock
