// Punctuation-based segmentation of the compressible region (Sec. 3.1): a delimiter token closes the segment it
// belongs to, so a new segment starts after every delimiter that is not the region's last token.
//
// One 1024-thread workgroup per sequence; a wavefront takes 256 consecutive tokens per step, four per lane (16-byte
// loads, four steps in flight), and compares them with every delimiter, the hits of one token position of all lanes being
// one 64-bit mask: the tests cost the vector pipe one compare per token and delimiter, the rest is scalar work.  In the
// offsets kernel every wavefront owns a contiguous run of steps: it keeps their masks in LDS while it counts, and after
// one exchange of the sixteen counts writes its boundaries in order from the masks.
//
// A caller that fetches the counts between the two kernels anyway asks for them by slices of 16 384 tokens (one round of
// loads for a workgroup) and hands the slices' places back: neither kernel then walks more than its slice.  Four sequences
// of 65 472 tokens, both kernels and the wait between them: 38.4 -> 28.0 us, eight of 131 000
// 57.2 -> 33.3.
//
// What bounds it: the latency of one workgroup's loads and compares, and in kernels this short the fetch of their own
// instructions (eight steps in flight, i.e. twice the code, took 18.3 us where four take 14.5).  Four sequences of 65 472
// tokens, six delimiters: counts 39 -> 10.7 us, offsets 55 -> 14.5 us (scalar loads and a barrier per 4 096 tokens before);
// with the wait between them, which a copy of the counts made longer, 111 -> 38 us.
#include "sablock_internal.h"

#include <algorithm>

namespace sablock {
namespace {

constexpr int SG_THREADS = 1024;
constexpr int SG_WAVES = SG_THREADS / 64;
constexpr int SG_STEP = 256;               // tokens of a wavefront's step
constexpr int SG_FLY = 4;                  // steps whose loads are in flight together
constexpr int SG_SLICE = SG_WAVES * SG_FLY;               // steps of a slice: one round of a workgroup
constexpr int SG_KEEP = 60 * 1024;         // bytes of masks that the offsets kernel keeps in LDS

struct __attribute__((packed, aligned(4))) Tok4 { int32_t x, y, z, w; };        // rows start at any token

// tokens t .. t+3 of a row of T; -1 behind its end
__device__ inline Tok4 load_tokens(const int32_t *row, int t, int T)
{
    if (t + 4 <= T) return *reinterpret_cast<const Tok4 *>(row + t);
    Tok4 v = {-1, -1, -1, -1};
    if (t < T) v.x = row[t];
    if (t + 1 < T) v.y = row[t + 1];
    if (t + 2 < T) v.z = row[t + 2];
    return v;
}

// f(step, t of this lane, m) for the steps [r0, r1) of a wavefront; m[j] bit l: a boundary sits behind token t + j of lane
// l's t, i.e. that token is a delimiter and not the row's last.  A delimiter is fetched once for all steps in flight.
template <typename F>
__device__ inline void walk_steps(const int32_t *row, int r0, int r1, int T, const DelimSet &ds, F &&f)
{
    const int lane = threadIdx.x & 63;
    for (int r = r0; r < r1; r += SG_FLY) {
        Tok4 v[SG_FLY];
        unsigned long long m[SG_FLY][4] = {};
#pragma unroll
        for (int j = 0; j < SG_FLY; ++j) v[j] = load_tokens(row, (r + j) * SG_STEP + 4 * lane, r + j < r1 ? T : 0);
#pragma nounroll
        for (int i = 0; i < ds.n; ++i) {
            const int32_t id = ds.id[i];
#pragma unroll
            for (int j = 0; j < SG_FLY; ++j) {
                m[j][0] |= __ballot(v[j].x == id);
                m[j][1] |= __ballot(v[j].y == id);
                m[j][2] |= __ballot(v[j].z == id);
                m[j][3] |= __ballot(v[j].w == id);
            }
        }
#pragma unroll
        for (int j = 0; j < SG_FLY; ++j) {
            const int t = (r + j) * SG_STEP + 4 * lane;
            if (r + j >= r1) break;
            if ((r + j + 1) * SG_STEP >= T) {                  // uniform: the row's last step, where -1 may be an id too
#pragma unroll
                for (int e = 0; e < 4; ++e) m[j][e] &= __ballot(t + e < T - 1);
            }
            f(r + j, t, m[j]);
        }
    }
}

__device__ inline int count_bits(const unsigned long long (&m)[4])
{
    return __popcll(m[0]) + __popcll(m[1]) + __popcll(m[2]) + __popcll(m[3]);
}

// steps [r0, r1) of wavefront w: its contiguous part of [first, last)
__device__ inline void wave_steps(int first, int last, int &r0, int &r1)
{
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), per = (last - first + SG_WAVES - 1) / SG_WAVES;
    r0 = min(first + w * per, last);
    r1 = min(r0 + per, last);
}
__device__ __host__ inline int steps_of(int T) { return T / SG_STEP + (T % SG_STEP != 0); }

// sum of the wavefronts' values (wave-uniform) and of those before this one
__device__ inline int over_waves(int v, int *sh_w, int &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) sh_w[wave] = v;
    __syncthreads();
    int before = 0;
    total = 0;
    for (int w = 0; w < SG_WAVES; ++w) { const int c = sh_w[w]; if (w < wave) before += c; total += c; }
    return before;
}

// grid (n_seq): seg_count[s] = 1 + number of boundaries
__global__ void __launch_bounds__(SG_THREADS)
segment_count_kernel(const int32_t *tok, int64_t stride, int T, DelimSet ds, int32_t *seg_count)
{
    __shared__ int sh_w[SG_WAVES];
    int r0, r1, n = 0, total;
    wave_steps(0, steps_of(T), r0, r1);
    walk_steps(tok + (int64_t)blockIdx.x * stride, r0, r1, T, ds, [&](int, int, const unsigned long long (&m)[4]) { n += count_bits(m); });
    over_waves(n, sh_w, total);
    if (threadIdx.x == 0) seg_count[blockIdx.x] = total + 1;
}

// grid (slices, n_seq): count[s * slices + slice] = boundaries of the slice's SG_SLICE steps
__global__ void __launch_bounds__(SG_THREADS)
segment_slice_count_kernel(const int32_t *tok, int64_t stride, int T, DelimSet ds, int32_t *count)
{
    __shared__ int sh_w[SG_WAVES];
    const int first = blockIdx.x * SG_SLICE, last = min(first + SG_SLICE, steps_of(T));
    int r0, r1, n = 0, total;
    wave_steps(first, last, r0, r1);
    walk_steps(tok + (int64_t)blockIdx.y * stride, r0, r1, T, ds, [&](int, int, const unsigned long long (&m)[4]) { n += count_bits(m); });
    over_waves(n, sh_w, total);
    if (threadIdx.x == 0) count[blockIdx.y * gridDim.x + blockIdx.x] = total;
}

// grid (slices, n_seq): the slice's offsets, from place sp.at[s * slices + slice] of seg_off on, which holds the offset in
// front of the slice's first boundary; the first slice's is 0, and behind the last slice's comes T.  No boundary is written
// behind the place of the next slice.
__global__ void __launch_bounds__(SG_THREADS)
segment_slice_offsets_kernel(const int32_t *tok, int64_t stride, int T, DelimSet ds, SlicePlaces sp, int32_t *seg_off)
{
    __shared__ unsigned long long sh_m[SG_SLICE][4];
    __shared__ int sh_w[SG_WAVES];
    const int lane = threadIdx.x & 63, first = blockIdx.x * SG_SLICE, last = min(first + SG_SLICE, steps_of(T));
    const int at0 = sp.at[blockIdx.y * gridDim.x + blockIdx.x], at1 = sp.at[blockIdx.y * gridDim.x + blockIdx.x + 1];
    const bool ends = blockIdx.x == gridDim.x - 1;
    const int most = ends ? at1 - 2 : at1;                // place of the slice's last boundary (behind it: T, the next sequence)
    int r0, r1, n = 0, total;
    wave_steps(first, last, r0, r1);
    walk_steps(tok + (int64_t)blockIdx.y * stride, r0, r1, T, ds, [&](int r, int, const unsigned long long (&m)[4]) {
        n += count_bits(m);
        if (lane < 4) sh_m[r - first][lane] = lane == 0 ? m[0] : lane == 1 ? m[1] : lane == 2 ? m[2] : m[3];
    });
    int pos = at0 + 1 + over_waves(n, sh_w, total);
#pragma nounroll
    for (int r = r0; r < r1; ++r) {
        int at = pos;
#pragma unroll
        for (int j = 0; j < 4; ++j) at += __popcll(sh_m[r - first][j] & ((1ull << lane) - 1ull));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const unsigned long long m = sh_m[r - first][j];
            if ((m >> lane) & 1ull) { if (at <= most) seg_off[at] = r * SG_STEP + 4 * lane + j + 1; ++at; }
            pos += __popcll(m);
        }
    }
    if (threadIdx.x == 0) {
        if (blockIdx.x == 0) seg_off[at0] = 0;
        if (ends) seg_off[at1 - 1] = T;
    }
}

// grid (slices, n_seq): offsets 0, t+1 for every boundary t in ascending order, T.  A workgroup counts the boundaries in
// front of its slice (cheap: no stores) and writes those of the slice: writing takes a workgroup longer than counting.
template <bool KEEP>
__global__ void __launch_bounds__(SG_THREADS)
segment_offsets_kernel(const int32_t *tok, int64_t stride, int T, DelimSet ds, SeqPtr sp, int32_t *seg_off)
{
    extern __shared__ unsigned long long sh_m[];          // [steps of a slice][4]
    __shared__ int sh_w[SG_WAVES], sh_f[SG_WAVES];
    const int s = blockIdx.y, lane = threadIdx.x & 63;
    const int32_t *row = tok + (int64_t)s * stride;
    int32_t *out = seg_off + sp.ptr[s];
    const int n_out = sp.ptr[s + 1] - sp.ptr[s];         // offsets this sequence may write (segments + 1)
    const int per = (steps_of(T) + (int)gridDim.x - 1) / (int)gridDim.x;
    const int first = min((int)blockIdx.x * per, steps_of(T)), last = min(first + per, steps_of(T));
    int r0, r1, in_front = 0, n = 0, total, total_front;
#pragma nounroll
    for (int part = 0; part < 2; ++part) {               // one copy of the code: a short kernel waits for its instructions
        wave_steps(part ? first : 0, part ? last : first, r0, r1);
        in_front = n;
        n = 0;
        walk_steps(row, r0, r1, T, ds, [&](int r, int, const unsigned long long (&m)[4]) {
            n += count_bits(m);
            if (KEEP && part && lane < 4) sh_m[4 * (r - first) + lane] = lane == 0 ? m[0] : lane == 1 ? m[1] : lane == 2 ? m[2] : m[3];
        });
    }
    over_waves(in_front, sh_f, total_front);
    int pos = 1 + total_front + over_waves(n, sh_w, total);        // next free slot
    auto put = [&](int, int t, const unsigned long long (&m)[4]) {
        int at = pos;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            at += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m[j] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[j], 0u));
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if ((m[j] >> lane) & 1ull) { if (at < n_out) out[at] = t + j + 1; ++at; }
        pos += count_bits(m);
    };
    if (KEEP) {
#pragma nounroll
        for (int r = r0; r < r1; ++r) {
            unsigned long long m[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const unsigned long long x = sh_m[4 * (r - first) + j];        // wave-uniform
                m[j] = (unsigned long long)__builtin_amdgcn_readfirstlane((uint32_t)(x >> 32)) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)x);
            }
            put(r, r * SG_STEP + 4 * lane, m);
        }
    } else {
        walk_steps(row, r0, r1, T, ds, put);
    }
    if (threadIdx.x == 0) {
        if (blockIdx.x == 0) out[0] = 0;
        if (blockIdx.x == gridDim.x - 1 && total_front + total + 1 < n_out) out[total_front + total + 1] = T;
    }
}

// grid (n_seq): bad[s] = number of offsets of sequence s that break "0 = off[0] < off[1] < ... < off[K] = T"
// (an entry counts when it is not above its predecessor; the first when it is not 0, the last also when it is not T)
__global__ void __launch_bounds__(SG_THREADS)
segment_check_kernel(const int32_t *seg_off, SeqPtr sp, int T, int32_t *bad)
{
    __shared__ int sh_w[SG_WAVES];
    const int s = blockIdx.x;
    const int32_t *off = seg_off + sp.ptr[s];
    const int n = sp.ptr[s + 1] - sp.ptr[s];              // offsets of this sequence, >= 2
    int mine = 0;
    for (int j = threadIdx.x; j < n; j += SG_THREADS) {
        const int v = off[j];
        bool ok = j == 0 ? v == 0 : v > off[j - 1];
        if (j == n - 1) ok = ok && v == T;
        mine += !ok;
    }
    for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o);
    int total;
    over_waves(mine, sh_w, total);
    if (threadIdx.x == 0) bad[s] = total;
}

}  // namespace

hipError_t launch_segment_check(const int32_t *seg_off, int32_t n_seq, int32_t T, const SeqPtr &sp, int32_t *bad,
                                hipStream_t st)
{
    if (n_seq <= 0) return hipSuccess;
    hipLaunchKernelGGL(segment_check_kernel, dim3(n_seq), dim3(SG_THREADS), 0, st, seg_off, sp, T, bad);
    return hipGetLastError();
}

int segment_slices(int32_t T) { return (steps_of(T) + SG_SLICE - 1) / SG_SLICE; }

hipError_t launch_segment_slice_count(const int32_t *tok, int64_t stride, int32_t n_seq, int32_t T, const DelimSet &ds,
                                      int32_t *count, hipStream_t st)
{
    hipLaunchKernelGGL(segment_slice_count_kernel, dim3(segment_slices(T), n_seq), dim3(SG_THREADS), 0, st, tok, stride, T, ds, count);
    return hipGetLastError();
}

hipError_t launch_segment_slice_offsets(const int32_t *tok, int64_t stride, int32_t n_seq, int32_t T, const DelimSet &ds,
                                        const SlicePlaces &sp, int32_t *seg_off, hipStream_t st)
{
    hipLaunchKernelGGL(segment_slice_offsets_kernel, dim3(segment_slices(T), n_seq), dim3(SG_THREADS), 0, st, tok, stride, T, ds, sp, seg_off);
    return hipGetLastError();
}

hipError_t launch_segment_count(const int32_t *tok, int64_t stride, int32_t n_seq, int32_t T, const DelimSet &ds,
                                int32_t *seg_count, hipStream_t st)
{
    if (n_seq <= 0) return hipSuccess;
    hipLaunchKernelGGL(segment_count_kernel, dim3(n_seq), dim3(SG_THREADS), 0, st, tok, stride, T, ds, seg_count);
    return hipGetLastError();
}

hipError_t launch_segment_offsets(const int32_t *tok, int64_t stride, int32_t n_seq, int32_t T, const DelimSet &ds,
                                  const SeqPtr &sp, int32_t *seg_off, hipStream_t st)
{
    if (n_seq <= 0) return hipSuccess;
    const int slices = std::max(1, std::min(8, T / 8192)), kept = (steps_of(T) + slices - 1) / slices * 32;    // bytes of masks
    const dim3 grid(slices, n_seq);
    if (kept <= SG_KEEP) hipLaunchKernelGGL(segment_offsets_kernel<true>, grid, dim3(SG_THREADS), kept, st, tok, stride, T, ds, sp, seg_off);
    else hipLaunchKernelGGL(segment_offsets_kernel<false>, grid, dim3(SG_THREADS), 0, st, tok, stride, T, ds, sp, seg_off);
    return hipGetLastError();
}

}  // namespace sablock
