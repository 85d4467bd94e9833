// MFMA window scoring (Sec. 3.2, Eqs. barA, st, Dk) for bf16.
//
// The window-query rows of a KV head (G query heads x W window queries) stay in
// accumulation registers as MFMA A operands, 16 rows per tile; keys are the B
// operand, 32 per wavefront iteration ("subtile"), two tiles of 16.  In the
// 16x16 accumulator layout a lane owns ONE key column of each key tile and four
// rows of each row tile (lane group lane / 16):
//   * the head mean (Eq. barA) is an in-lane add,
//   * the column sum (Eq. st) is in-lane adds plus two exchanges between the
//     four lane groups, and so is the entropy term (inner sum of Eq. Dk),
//   * the per-row softmax statistics are kept per lane and only reduced across
//     lanes once per workgroup.
// Each wavefront streams its own keys: global -> LDS with direct-to-LDS loads
// (16 bytes per lane, fully coalesced 256-byte key rows) into a private ring,
// LDS -> registers with an XOR swizzle so the 16-byte reads of different key
// rows do not collide on banks.  No workgroup barrier in the loops.
//
// Softmax over all keys needs each row's log-sum-exp before any column is
// final, so scoring is two kernels unless the caller supplies row_lse:
//   pass 1  per row and lane the sum of the exponentials;
//   pass 2  the chunk partials are combined into the row log-sum-exp in the
//           prologue; probabilities, head mean, column sum and entropy term follow
//           in registers.
// The log-sum-exp enters as the MFMA's C operand, less a power of two that all rows
// share (common_power) and that comes off the column sums in the end: in full, some 140
// in units of <q,k>, it would cost every product the bits that it is larger (128 rows,
// 40 000 keys, statistics without references: scores 8.5e-7 off their 64-bit values,
// 4.9e-7 less it; with references 3.3e-7).
// In both passes the row tiles rotate, in groups of two, through two sets of
// accumulators: a group is multiplied while the one before it is exponentiated,
// which overlaps the matrix pipe with the exp/log work inside one wavefront (one
// wavefront per SIMD).  One launch per pass covers every problem of the call.
//
// What bounds both passes is vector issue at the clock that the power budget leaves:
// of 3 930 (pass 1) and 4 450 cycles (pass 2) per subtile of 256 rows vector
// instructions take 2 650 and 3 220, the matrix pipe is busy for 2 048 beside them, the
// rest are waits, mostly for an instruction's turn; the clock is 1.88 GHz of 2.4.  With
// 128 rows the keys' stream (1.20 ms for 8.6 GB, 1.54 with the stores) is as near.
// `v_mfma_f32_16x16x32_bf16` needs less power than `v_mfma_f32_32x32x16_bf16`
// (registers alone, normal variates, sustained: 2.0 against 1.78 PFLOP/s; with the
// exponentials of pass 1, two wavefronts per SIMD: 738 against 866 ns per subtile of
// 128 rows and SIMD), and a lane's sums and C operands take half the registers, so
// that even 256 rows of a KV head keep theirs out of LDS.
#include "sablock_internal.h"

#include <algorithm>
#include <type_traits>

namespace sablock {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef const void __attribute__((address_space(1))) *gptr_t;
typedef void __attribute__((address_space(3))) *lptr_t;

constexpr int SUB = 32;                    // keys per wavefront iteration
constexpr int TILE = 16;                   // rows or keys of an MFMA tile
constexpr int ROW_BYTES = 256;             // D = 128 bf16
constexpr int BUF_BYTES = SUB * ROW_BYTES; // 8 KiB
constexpr int M_ROWS = 128;
constexpr int STREAMS = 4;                 // key streams per workgroup (subtile u of the chunk goes to stream u % 4)
constexpr int STRIDE = STREAMS * SUB;      // keys between consecutive subtiles of one stream
constexpr int NBUF = 4;                    // subtiles of a stream's ring
constexpr int WAVES = 4;
constexpr int RING_BYTES = NBUF * BUF_BYTES;

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;
constexpr float RESCALE_AT = 64.f;         // pass 1, careful: a row's reference moves when an exponent exceeds this
constexpr float COMMON_MOST = 100.f;       // pass 2, see common_power
constexpr float SUM_MOST = 0x1p100f, SUM_LEAST = 0x1p-60f;     // pass 1, fast: a row's sum outside says that exponentials may have over- or underflowed

struct ScoreArgs {
    Dims d;
    const uint16_t *q, *k;
    int chunk_len;         // keys per workgroup, multiple of STRIDE
    int n_chunks;          // workgroups per problem
    int by_chunk;          // grid (problems, n_chunks), else (n_chunks, problems)
    int pc;                // (reference, sum) pairs per row that pass 2 reads: n_chunks, or 1 once they are merged
    float c1;              // log2(e) / sqrt(D)
    float log2_G;          // log2 of the heads per KV head (the head mean is folded into the rows' log-sum-exp)
    float eps;
    float *partial;        // pass 1 out: [problem][chunk][G * W][2] (reference, sum), log2 domain
    const float *merged;   // pass 2 in: the same layout with pc chunks
    const float *lse;      // pass 2 in, optional: [P][G * W] natural-log sum-exp per row (NULL: use partial)
    float *s_out, *e_out;  // pass 2 out: [P][L]
    float *abar;           // pass 2 out of the all-head variant: head-group means [P][W / 4][L][4]
};

__device__ __forceinline__ uint32_t lds_addr(const void *p) { return (uint32_t)(uintptr_t)(lptr_t)p; }

// Where the rows of a problem's window-query matrix (row = head * W + window query) sit.  Position 16 J + 4 g + i is
// accumulator register i of lane group g of tile J.  For W = 8 a lane's registers are two queries of two heads, so
// that the head mean needs no other lane; else positions are rows.  The rows behind the problem's G * W (W = 8 and G
// odd) are padding: zero queries, never written by pass 1 and given an infinite log-sum-exp in pass 2, so they add
// exact zeros.
template <int NT_, int W> struct Rows {
    static constexpr int NT = NT_;                          // tiles
    static constexpr int MP = TILE * NT;                    // rows of the tiles (padding included)
    static constexpr int NG = (NT + 1) / 2;                 // groups of two tiles
    static constexpr int NS = W / 4;                        // head-mean values per lane and key tile
    static constexpr int PER_HEAD = W == 8 ? 1 : W / TILE;  // tiles of a head
    static_assert(NT >= 1 && NT <= 16 && (W == 8 || W == 16 || W == 32 || W == 64) && NT % PER_HEAD == 0, "unsupported shape");
    __device__ static int row_of(int pos)
    {
        return W == 8 ? 8 * (2 * (pos >> 4) + ((pos >> 1) & 1)) + 2 * ((pos >> 2) & 3) + (pos & 1) : pos;
    }
    __device__ static int query(int J, int g, int i) { return W == 8 ? 2 * g + (i & 1) : TILE * (J % PER_HEAD) + 4 * g + i; }
    __host__ __device__ static constexpr int slot(int J, int i) { return W == 8 ? i & 1 : 4 * (J % PER_HEAD) + i; }
    __host__ __device__ static constexpr bool first(int J, int i) { return W == 8 ? J == 0 && i < 2 : J < PER_HEAD; }   // of its slot
};

// Direct-to-LDS load of 32 key rows starting at t0: 8 instructions of 1 KiB (4 rows each); LDS slot
// (row, pos) receives 16-byte chunk pos ^ (row & 15) of the row.  The address is a wave-uniform 64-bit base
// (scalar registers) plus a per-lane 32-bit byte offset; M0 carries the LDS destination of each 1 KiB group.
__device__ __forceinline__ void dma_1k(uint32_t voff, const char *sbase, uint32_t lds_dst)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" : : "v"(voff), "s"(sbase), "s"(lds_dst) : "memory", "m0");
}

// subtile entirely inside [0, L): one of four precomputed lane offsets
//   lane_off[j & 3] = (lane / 16) * row_bytes + (((lane & 15) ^ (lane / 16) ^ 4 (j & 3)) << 4),
// so issuing costs no vector ALU work
__device__ __forceinline__ void issue_subtile_fast(const char *base, int64_t row_bytes, const uint32_t (&lane_off)[4], uint32_t buf_lds)
{
#pragma unroll
    for (int j = 0; j < 8; ++j) dma_1k(lane_off[j & 3], base + (int64_t)(4 * j) * row_bytes, buf_lds + j * 1024);
}

// The same for dense rows (row_bytes = 256): four rows are then 1 KiB apart in memory as in LDS, and the
// instruction's immediate offset is added to the global address and to the LDS address alike, so four loads share
// one scalar base and one M0 value; the subtile takes two of each instead of eight.
__device__ __forceinline__ void dma_4k(const uint32_t (&lane_off)[4], const char *sbase, uint32_t lds_dst)
{
    asm volatile("s_mov_b32 m0, %5\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %0, %4 nt\n\t"
                 "global_load_lds_dwordx4 %1, %4 offset:1024 nt\n\t"
                 "global_load_lds_dwordx4 %2, %4 offset:2048 nt\n\t"
                 "global_load_lds_dwordx4 %3, %4 offset:3072 nt"
                 : : "v"(lane_off[0]), "v"(lane_off[1]), "v"(lane_off[2]), "v"(lane_off[3]), "s"(sbase), "s"(lds_dst) : "memory", "m0");
}
__device__ __forceinline__ void issue_subtile_dense(const char *base, const uint32_t (&lane_off)[4], uint32_t buf_lds)
{
    dma_4k(lane_off, base, buf_lds);
    dma_4k(lane_off, base + 4096, buf_lds + 4096);
}

// subtile that crosses L: rows past L-1 read row L-1 instead (their results are masked later); t0 < L
__device__ __forceinline__ void issue_subtile_clamped(const char *base, int64_t row_bytes, int rows_valid, uint32_t buf_lds, int lane)
{
    const int r4 = lane >> 4, pos = lane & 15;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int row = 4 * j + r4;
        const uint32_t voff = (uint32_t)min(row, rows_valid - 1) * (uint32_t)row_bytes + (uint32_t)(((pos ^ row) & 15) << 4);
        dma_1k(voff, base, buf_lds + j * 1024);
    }
}

// wait until this wavefront's direct-to-LDS loads issued before the last `subtiles_after` subtiles have landed
// (8 loads per subtile; later stores only make the wait longer, never shorter)
__device__ __forceinline__ void wait_loads(int subtiles_after)
{
    if (subtiles_after >= 3) asm volatile("s_waitcnt vmcnt(24)" ::: "memory");
    else if (subtiles_after == 2) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
    else if (subtiles_after == 1) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

struct WaveWork {
    const uint16_t *kp;    // keys of the problem
    int p, chunk;
    int first, n_sub;      // this stream's subtiles: keys [first + u * STRIDE, +SUB), u < n_sub
};

__device__ __forceinline__ WaveWork wave_work(const ScoreArgs &a, int stream)
{
    stream = __builtin_amdgcn_readfirstlane(stream);         // wave-uniform: addresses below stay in scalar registers
    WaveWork w;
    w.p = a.by_chunk ? blockIdx.x : blockIdx.y;
    w.chunk = a.by_chunk ? blockIdx.y : blockIdx.x;
    w.kp = a.k + k_problem_offset(a.d, w.p);
    const int lo = w.chunk * a.chunk_len;
    const int hi = min(lo + a.chunk_len, a.d.L);
    w.first = lo + stream * SUB;
    const int span = hi - w.first;
    w.n_sub = span > 0 ? (span + STRIDE - 1) / STRIDE : 0;
    return w;
}

// subtiles of a stream none of whose keys is masked for any window query: [0, this)
__device__ __forceinline__ int plain_subtiles(const WaveWork &w, int T)
{
    return w.first + SUB <= T ? min(w.n_sub, (T - SUB - w.first) / STRIDE + 1) : 0;
}

// ------------------------------------------------------------------ shared pieces of both passes
// B operands of one subtile: kb[t][s] = K[key 16 t + lane % 16][(4 s + lane / 16) * 8 .. +8].  buf = the lane's place in the
// buffer, (lane % 16) * 256 + ((lane / 16 ^ lane % 16) << 4); chunk 4 s + g of the key sits at that address ^ (s << 6).
// Ordinary loads: the compiler spreads them and waits where they are used.  That they come after the buffer's
// direct-to-LDS loads, and before its next ones, is the caller's to see to (see KeyStream::next).
__device__ __forceinline__ void read_subtile(uint32_t buf, bf16x8 (&kb)[2][4])
{
    typedef const bf16x8 __attribute__((address_space(3))) *lds_vec;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        kb[0][s] = *(lds_vec)(uintptr_t)(buf ^ (uint32_t)(s << 6));
        kb[1][s] = *(lds_vec)(uintptr_t)((buf ^ (uint32_t)(s << 6)) + TILE * ROW_BYTES);
    }
}
// the operands are in their registers behind this point (ACC: accumulation registers)
template <bool ACC>
__device__ __forceinline__ void have_subtile(bf16x8 (&kb)[2][4])
{
    if (ACC) asm volatile("" : "+a"(kb[0][0]), "+a"(kb[0][1]), "+a"(kb[0][2]), "+a"(kb[0][3]), "+a"(kb[1][0]), "+a"(kb[1][1]), "+a"(kb[1][2]), "+a"(kb[1][3]) : : "memory");
    else asm volatile("" : "+v"(kb[0][0]), "+v"(kb[0][1]), "+v"(kb[0][2]), "+v"(kb[0][3]), "+v"(kb[1][0]), "+v"(kb[1][1]), "+v"(kb[1][2]), "+v"(kb[1][3]) : : "memory");
}
__device__ __forceinline__ uint32_t lane_read_offset(int lane)
{
    const int n = lane & 15, g = lane >> 4;
    return (uint32_t)(n * ROW_BYTES + ((g ^ n) << 4));
}

// Group j of the row tiles (tiles 2 j and 2 j + 1) times the two key tiles; c(J): C operand of tile J
template <int NT, int KS, typename C>
__device__ __forceinline__ void multiply(const bf16x8 (&qa)[NT][KS], const bf16x8 (&kb)[2][KS], int j, C c, floatx4 (&acc)[2][2])
{
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int t = 0; t < 2; ++t)
                if (2 * j + r < NT)
                    acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[2 * j + r][s], kb[t][s], s == 0 ? c(2 * j + r) : acc[r][t], 0, 0, 0);
}
__device__ __forceinline__ floatx4 no_operand(int) { return floatx4{}; }

// what makes a pending group add zeros
__device__ __forceinline__ void set_nothing(floatx4 (&acc)[2][2])
{
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[r][t][i] = -INFINITY;
}

// Per-wavefront stream of subtiles through a ring of NBUF LDS buffers.  Subtile u lives in buffer u % NBUF.  AHEAD: the
// kernels hold two subtiles in registers, and while one is worked on the next one is read from LDS.  next()
// sees that the subtile at hand has left its buffer, re-fills that with subtile u + NBUF, waits for subtile u + 1 and
// starts to read it: NBUF subtiles (32 KiB per wavefront) are in flight or landed at any time.  Else there
// is room for one subtile (pass 2 of more than 128 rows), which next() reads itself.
template <bool AHEAD_, bool ACC>
struct KeyStream {
    static constexpr bool AHEAD = AHEAD_;
    const uint16_t *kp;
    int64_t ks3;
    char *ring;
    uint32_t lane_addr0, ring_lds;
    uint32_t lane_off[4];
    int first, n_sub, L, lane;
    const char *ahead;                                         // keys of the next subtile to issue
    int64_t step;                                              // bytes between consecutive subtiles of this stream

    __device__ __forceinline__ void init(const uint16_t *kp_, int64_t ks3_, char *ring_, int first_, int n_sub_, int L_, int lane_)
    {
        kp = kp_; ks3 = ks3_; ring = ring_; first = first_; n_sub = n_sub_; L = L_; lane = lane_;
        ahead = reinterpret_cast<const char *>(kp) + (int64_t)first * ks3 * 2;
        step = (int64_t)STRIDE * ks3 * 2;
        const int r4 = lane >> 4, pos = lane & 15;
        ring_lds = __builtin_amdgcn_readfirstlane(lds_addr(ring));
        lane_addr0 = ring_lds + lane_read_offset(lane);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) lane_off[jj] = (uint32_t)(r4 * ks3 * 2) + (uint32_t)(((pos ^ r4 ^ (4 * jj)) & 15) << 4);
    }
    __device__ __forceinline__ void issue(int u)
    {
        const int t0 = first + u * STRIDE;                     // wave-uniform, < L
        const char *base = ahead;                              // subtiles are issued in order: a running address
        ahead += step;
        const uint32_t buf_lds = ring_lds + (u % NBUF) * BUF_BYTES;
        if (t0 + SUB <= L) {
            if (ks3 == ROW_BYTES / 2) issue_subtile_dense(base, lane_off, buf_lds);
            else issue_subtile_fast(base, ks3 * 2, lane_off, buf_lds);
        } else issue_subtile_clamped(base, ks3 * 2, L - t0, buf_lds, lane);
    }
    // the first subtiles, [from, to) of the ring
    __device__ __forceinline__ void issue_first(int from = 0, int to = NBUF)
    {
        for (int u = from; u < min(to, n_sub); ++u) issue(u);
    }
    // subtile 0 into kb, where the first next() expects it or (not AHEAD) LOOK asks for it
    template <bool LOOK = false>
    __device__ __forceinline__ void start(bf16x8 (&kb)[2][4])
    {
        if (!(AHEAD || LOOK) || n_sub == 0) return;
        wait_loads(min(NBUF, n_sub) - 1);
        read_subtile(lane_addr0, kb);
    }
    // AHEAD: subtile u is in `cur`; subtile u + 1, if there is one, into `nxt`.  Else: subtile u into `cur`.
    __device__ __forceinline__ void next(int u, bf16x8 (&cur)[2][4], bf16x8 (&nxt)[2][4])
    {
        if (!AHEAD) {
            wait_loads(min(NBUF - 1, n_sub - 1 - u));
            read_subtile(lane_addr0 + (u % NBUF) * BUF_BYTES, cur);
        }
        have_subtile<ACC>(cur);
        if (u + NBUF < n_sub) issue(u + NBUF);
        if (AHEAD && u + 1 < n_sub) {
            wait_loads(min(NBUF - 1, n_sub - 2 - u));
            read_subtile(lane_addr0 + ((u + 1) % NBUF) * BUF_BYTES, nxt);
        }
    }
};

// Keys of other lengths (64, 96 or 256 elements): no LDS staging.  A lane loads its own B operands (elements (4 s +
// lane / 16) * 8 .. +8 of keys lane % 16 and 16 + lane % 16: the four lane groups of a key read adjacent 16-byte pieces)
// straight into registers with ordinary loads, one subtile ahead.  Keys past the end of the sequence read key L - 1 (their
// results are masked later, as in the staged stream).  Same interface as KeyStream.
template <int KS>
struct KeyStreamDirect {
    static constexpr bool AHEAD = true;
    const uint16_t *kp;
    int64_t ks3;
    int first, n_sub, L, lane;

    __device__ __forceinline__ void init(const uint16_t *kp_, int64_t ks3_, char *, int first_, int n_sub_, int L_, int lane_)
    {
        kp = kp_; ks3 = ks3_; first = first_; n_sub = n_sub_; L = L_; lane = lane_;
    }
    __device__ __forceinline__ void load(int u, bf16x8 (&kb)[2][KS])
    {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int key = min(first + u * STRIDE + TILE * t + (lane & 15), L - 1);
            const uint16_t *row = kp + (int64_t)key * ks3 + (lane >> 4) * 8;
#pragma unroll
            for (int s = 0; s < KS; ++s) kb[t][s] = *reinterpret_cast<const bf16x8 *>(row + 32 * s);
        }
    }
    __device__ __forceinline__ void issue_first(int = 0, int = 0) {}
    template <bool = false>
    __device__ __forceinline__ void start(bf16x8 (&kb)[2][KS])
    {
        if (n_sub > 0) load(0, kb);
    }
    __device__ __forceinline__ void next(int u, bf16x8 (&)[2][KS], bf16x8 (&nxt)[2][KS])
    {
        if (u + 1 < n_sub) load(u + 1, nxt);
    }
};

template <int KS>
__device__ __forceinline__ void copy_subtile(bf16x8 (&to)[2][KS], const bf16x8 (&from)[2][KS])
{
    if (&to == &from) return;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int s = 0; s < KS; ++s) to[t][s] = from[t][s];
}

__device__ __forceinline__ void copy_group(floatx4 (&to)[2][2], const floatx4 (&from)[2][2])
{
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int t = 0; t < 2; ++t) to[r][t] = from[r][t];
}

// the key stream by k-steps of 32 elements per key: 4 (D = 128) staged through LDS; 2 (D = 64), 3 (D = 96) and 8 (D =
// 256, whose 512-byte rows would need a ring twice the LDS) direct.  The A operands of up to 128 rows leave accumulation
// registers for the keys.
template <int NT, int KS, bool AHEAD> struct StreamFor { using type = KeyStreamDirect<KS>; };
template <int NT, bool AHEAD> struct StreamFor<NT, 4, AHEAD> { using type = KeyStream<AHEAD, NT <= 8>; };

// A operands, in accumulation registers: a lane's rows are positions 16 J + lane % 16 (see Rows); padding rows hold some
// other row until pin_queries clears them.  Straight from memory:
template <int NT, int W, int KS>
__device__ __forceinline__ void load_queries(bf16x8 (&qa)[NT][KS], const ScoreArgs &a, int p, int lane)
{
    const uint16_t *q = a.q + q_row_offset(a.d, p, 0, 0) + (lane >> 4) * 8;
#pragma unroll
    for (int J = 0; J < NT; ++J) {
        const int r = min(Rows<NT, W>::row_of(TILE * J + (lane & 15)), a.d.G * W - 1);
        const uint16_t *row = q + (r / W) * a.d.qs[2] + (r % W) * a.d.qs[3];
#pragma unroll
        for (int s = 0; s < KS; ++s) qa[J][s] = *reinterpret_cast<const bf16x8 *>(row + 32 * s);
    }
}

// ... or, where the keys are staged (D = 128), once per workgroup through the last buffers of the wavefronts' rings: block b
// of 32 rows by wavefront b % 4, in the keys' own layout.  Four wavefronts that each load all the rows take 10 000 cycles
// for 128 of them, as much as two subtiles of keys.
template <int NT> struct QueryStage {
    static constexpr int BLOCKS = (NT + 1) / 2;
    static constexpr int BUFS = (BLOCKS + WAVES - 1) / WAVES;                  // buffers of a ring that hold queries at first
    __device__ static uint32_t buffer(uint32_t ring0_lds, int b)
    {
        return ring0_lds + (b % WAVES) * RING_BYTES + (NBUF - 1 - b / WAVES) * BUF_BYTES;
    }
    template <int W>
    __device__ __forceinline__ static void issue(const ScoreArgs &a, int p, uint32_t ring0_lds, int wave, int lane)
    {
        const uint16_t *q = a.q + q_row_offset(a.d, p, 0, 0);
#pragma unroll
        for (int i = 0; i < BUFS; ++i) {
            const int b = wave + WAVES * i;
            if (b >= BLOCKS) break;
            const uint32_t lds = buffer(ring0_lds, b);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int row = 4 * j + (lane >> 4), r = min(Rows<NT, W>::row_of(min(2 * TILE * b + row, TILE * NT - 1)), a.d.G * W - 1);
                const uint16_t *src = q + (r / W) * a.d.qs[2] + (r % W) * a.d.qs[3] + (((lane ^ row) & 15) << 3);
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(lds + j * 1024) : "memory", "m0");
            }
        }
    }
    // behind a barrier that says that all blocks have landed; the buffers are free behind another one
    __device__ __forceinline__ static void read(bf16x8 (&qa)[NT][4], uint32_t ring0_lds, int lane)
    {
        typedef const bf16x8 __attribute__((address_space(3))) *lds_vec;
#pragma unroll
        for (int J = 0; J < NT; ++J)
#pragma unroll
            for (int s = 0; s < 4; ++s)
                qa[J][s] = *(lds_vec)(uintptr_t)((buffer(ring0_lds, J / 2) + (J & 1) * TILE * ROW_BYTES + lane_read_offset(lane)) ^ (uint32_t)(s << 6));
    }
};

// all LDS traffic of this wavefront done, then the workgroup barrier (global loads stay in flight)
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int NT, int W, int KS>
__device__ __forceinline__ void pin_queries(bf16x8 (&qa)[NT][KS], const ScoreArgs &a, int lane)
{
    if (W == 8 && Rows<NT, W>::row_of(TILE * (NT - 1) + (lane & 15)) >= a.d.G * W) {       // only the last tile can hold padding
#pragma unroll
        for (int s = 0; s < KS; ++s) qa[NT - 1][s] = bf16x8{};
    }
#pragma unroll
    for (int J = 0; J < NT; ++J)
#pragma unroll
        for (int s = 0; s < KS; ++s) asm volatile("" : "+a"(qa[J][s]));
}

// ------------------------------------------------------------------ pass 1
// Row statistics: per window-query row a reference and the sum z of exp2(c1 * <q,k> - ref) over the keys, kept per lane
// (its keys) until the end.
//
// More than 128 rows are walked without references at first: a sum of positive terms is as accurate as its terms
// whatever their size, as long as none overflows and those that underflow do not count.  Both can be told from the
// row's sum: no logit that it holds exceeds SUM_MOST, and what was flushed to zero (below 2^-126 each) is nothing beside
// SUM_LEAST.  Logits of unbiased keys lie within some tens of powers of two around 1; of a model whose keys carry a bias
// they need not.  A wavefront that finds a row outside, as a rule after its first sixteen subtiles, begins again with
// references: the row maxima over its first sixteen keys, negated the MFMA's C operands, so acc = <q,k> - reference.  Those
// cost an LDS read per tile and subtile (all registers are taken by 256 rows).  Where even then a sum is outside (a
// logit 100 powers of two above the first subtile's, or a stream that begins inside the window) it walks once more, through
// stats_careful, whose references move: any finite logits are handled.
//
// Up to 128 rows, and heads of other lengths, have references from the start, in registers: the exponent of a peak is smaller
// and rounds to less.  Scores against 64 bits with references and without, means over 48 heads of 128 elements, 64 keys
// scaled by four: 1 024 keys, (G, W) = (1, 8) 5.5e-7 and 7.8e-7, (4, 32) 3.3e-7 and 6.1e-7; 40 000 keys 8.2e-7 and 9.7e-7,
// 6.3e-7 and 9.2e-7; normal variates, 4 000 keys, (4, 32) 2.1e-7 and 3.4e-7.  They cost a product of sixteen keys per stream:
// a call on 8 problems of 8 192 keys, two subtiles to a stream, takes 0.5 us more of 49, 256 problems of 131 072 keys
// take no more (3.21 ms without, 3.18 with).

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));       // every lane has a source
}
// maximum and sum over the 16 lanes of a lane group: lane ^ 1, lane ^ 2, mirror inside 8, mirror inside 16
__device__ __forceinline__ float group_max(float v)
{
    // the maximum of two, a number where one is not: one instruction, where fmaxf takes another per operand
    auto larger = [](float x, float y) { return __builtin_amdgcn_fmed3f(x, y, INFINITY); };
    v = larger(v, dpp_f<0xB1>(v));
    v = larger(v, dpp_f<0x4E>(v));
    v = larger(v, dpp_f<0x141>(v));
    return larger(v, dpp_f<0x140>(v));
}
__device__ __forceinline__ float group_sum(float v)
{
    v += dpp_f<0xB1>(v);
    v += dpp_f<0x4E>(v);
    v += dpp_f<0x141>(v);
    return v + dpp_f<0x140>(v);
}

// Careful body: the subtile in kb, whose first key is t0, against all row tiles.  A row's state sits in LDS: state[pos / 2] =
// (cr, z) of two rows, z the sum over all lanes.  Three times as slow as the other walks: the tiles' loop is not unrolled and
// takes its queries from memory, for less code.
template <int NT, int W, int KS>
__device__ __forceinline__ void stats_careful(const ScoreArgs &a, int p, const bf16x8 (&kb)[2][KS], floatx4 *state, bool first, int t0, int n, int g)
{
    const float c1 = a.c1, inv_c1 = 1.0f / c1;
    const uint16_t *q = a.q + q_row_offset(a.d, p, 0, 0) + g * 8;
#pragma nounroll
    for (int J = 0; J < NT; ++J) {
        const int r = min(Rows<NT, W>::row_of(TILE * J + n), a.d.G * W - 1);                 // a padding row's results are not used
        const uint16_t *row = q + (r / W) * a.d.qs[2] + (r % W) * a.d.qs[3];
        floatx4 *st = state + (TILE * J + 4 * g) / 2;
        const floatx4 s0 = first ? floatx4{} : st[0], s1 = first ? floatx4{} : st[1];
        floatx4 cr = {s0[0], s0[2], s1[0], s1[2]}, z = {s0[1], s0[3], s1[1], s1[3]}, v[2] = {cr, cr};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const bf16x8 qa = *reinterpret_cast<const bf16x8 *>(row + 32 * s);
#pragma unroll
            for (int t = 0; t < 2; ++t) v[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa, kb[t][s], v[t], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
                v[t][i] = t0 + TILE * t + n <= a.d.T + Rows<NT, W>::query(J, g, i) ? v[t][i] * c1 : -INFINITY;       // causal inside the window
            const float rm = group_max(fmaxf(v[0][i], v[1][i]));
            const bool move = first ? rm > -INFINITY : rm > RESCALE_AT;
            const float cshift = move ? rm * inv_c1 : 0.f;      // change of the C operand
            const float shift = cshift * c1;                    // and the matching change of the exponent
            z[i] = (first ? 0.f : z[i] * __builtin_amdgcn_exp2f(-shift)) +
                   group_sum(__builtin_amdgcn_exp2f(v[0][i] - shift) + __builtin_amdgcn_exp2f(v[1][i] - shift));
            cr[i] -= cshift;
        }
        if (n == 0) {
            st[0] = floatx4{cr[0], z[0], cr[1], z[1]};
            st[1] = floatx4{cr[2], z[2], cr[3], z[3]};
        }
    }
    __builtin_amdgcn_wave_barrier();                            // written before the next subtile's reads
}

// adds the exponentials of group j; W: with the causal mask inside the window of so many queries (key T + q is the last that
// query q sees, and the last of all for the last one), 0: none is masked; t: the lane's key in the first key tile
template <int W, int NT>
__device__ __forceinline__ void stats_add(const floatx4 (&acc)[2][2], int j, floatx4 (&z)[NT], float c1, int t, int g, int T)
{
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (2 * j + r >= NT) continue;
                const float e = __builtin_amdgcn_exp2f(acc[r][kt][i] * c1);
                if constexpr (W == 0) z[2 * j + r][i] += e;
                else z[2 * j + r][i] += t + TILE * kt <= T + Rows<NT, W>::query(2 * j + r, g, i) ? e : 0.f;
            }
}

// Fast body of one subtile: group j is multiplied into acc[(j + PAR) & 1] while the group before it is exponentiated from
// the other set, at first the last group of the subtile before.  The last group is left waiting.
template <int PAR, int NT, int KS, typename C>
__device__ __forceinline__ void stats_fast(const bf16x8 (&qa)[NT][KS], const bf16x8 (&kb)[2][KS], floatx4 (&acc)[2][2][2],
                                           C c, floatx4 (&z)[NT], float c1)
{
    constexpr int NG = (NT + 1) / 2;
#pragma unroll
    for (int j = 0; j < NG; ++j) {
        multiply(qa, kb, j, c, acc[(j + PAR) & 1]);
        stats_add<0>(acc[(j + PAR + 1) & 1], j > 0 ? j - 1 : NG - 1, z, c1, 0, 0, 0);
        // above 192 rows products, multiplications, exponentials and additions by turns: in the compiler's own order the matrix pipe
        // waits (1 024 problems of 65 536 keys, 256 rows: 4.58 ms in its own, 4.43 in this; fewer rows: the same)
#pragma unroll
        for (int i = 0; i < (NT <= 12 ? 0 : 2 * j + 1 < NT ? 4 : 2); ++i) {
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);   // MFMA
            __builtin_amdgcn_sched_group_barrier(0x2, 4, 0);   // VALU
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x400, 4, 0); // transcendental
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x2, 4, 0);
            __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        }
    }
    // the sums as they are here: keeps the compiler from moving this subtile's exponentials behind the next one's loads
    // (where a step is one subtile there is nothing behind it)
#pragma unroll
    for (int J = 0; J < NT; ++J)
        if (NT <= 8) asm volatile("" : "+v"(z[J]));
}

// the lane, formed where it is used: what follows from it is not kept in registers through the loops in front
__device__ __forceinline__ int lane_again()
{
    int lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    return lane;
}

// whether the first walk has references already, and they have room in registers
template <int NT, int KS> constexpr bool refs_first() { return KS != 4 || NT <= 8; }

// One walk over the stream, whose first subtiles are on their way, to the rows' states.  REF: with references, kept in refs[MP].
// True (in some lane): a sum is outside what it can tell, the states are void; then the subtiles on their way may be any.
template <bool REF, int NT, int W, int KS, typename Stream>
__device__ __forceinline__ bool stats_walk(const ScoreArgs &a, const WaveWork &w, Stream &ks, const bf16x8 (&qa)[NT][KS],
                                           floatx4 *state, float *refs, int n_plain, int lane)
{
    using R = Rows<NT, W>;
    constexpr int NG = R::NG;
    constexpr bool ONE = !Stream::AHEAD && NG % 2 == 0;        // a step is one subtile, and nothing changes places
    // so is it here, and what changes places is copied: for less code, or because two subtiles of more than 192 rows spill
    constexpr bool SHORT = !ONE && ((REF && !refs_first<NT, KS>()) || NT > 12);
    const int T = a.d.T;
    int n = lane & 15, g = lane >> 4;
    bf16x8 ka[2][KS], ahead[2][KS];
    auto &kb = Stream::AHEAD ? ahead : ka;
    ks.template start<REF>(ka);
    floatx4 cr[NT];                                            // in registers where there is room for them
    if (REF) {
#pragma unroll
        for (int J = 0; J < NT; ++J) {
            floatx4 first = {}, ref;
            if (n_plain > 0)
#pragma unroll
                for (int s = 0; s < KS; ++s) first = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[J][s], ka[0][s], first, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float rm = group_max(first[i]);
                ref[i] = fabsf(rm) < INFINITY ? -rm : 0.f;
            }
            if (refs_first<NT, KS>()) cr[J] = ref;
            else if (n == 0) *reinterpret_cast<floatx4 *>(refs + TILE * J + 4 * g) = ref;
        }
        __builtin_amdgcn_wave_barrier();                       // written before the first subtile's reads
    }
    auto c = [&](int J) __attribute__((always_inline)) {
        return !REF ? floatx4{} : refs_first<NT, KS>() ? cr[J] : *reinterpret_cast<const floatx4 *>(refs + TILE * J + 4 * g);
    };
    // in two levels: beside one large term, small ones that are added to it one by one are lost, sixteen subtiles of
    // them together are not (rows with a peak of 2^26 times the rest, 131 072 keys: sums 5e-5 off without)
    floatx4 z[NT], zo[NT];
#pragma unroll
    for (int J = 0; J < NT; ++J) z[J] = zo[J] = floatx4{};
    auto level = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int J = 0; J < NT; ++J) {
            zo[J] += z[J];
            z[J] = floatx4{};
        }
    };
    auto outside = [&](float &least) __attribute__((always_inline)) {
        float most = 0.f;
        least = INFINITY;
#pragma unroll
        for (int J = 0; J < NT; ++J)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                least = fminf(least, zo[J][i]);
                most = fmaxf(most, zo[J][i]);
            }
        return most > SUM_MOST;
    };
    floatx4 acc[2][2][2];
    set_nothing(acc[0]);
    set_nothing(acc[1]);
    int u = 0;
    float least;
    // Without references the first sixteen subtiles of a long stream by themselves: whether they are outside is not asked in the
    // loop, where it costs the compiler's order of it (statistics of 256 problems of 131 072 keys: 1.35 ms, asked there 1.38), nor
    // at all where few subtiles follow (8 problems of 131 072 keys, 32 subtiles to a stream: the call 145.7 us, without 144.6)
    for (int end = REF || n_plain < 48 ? n_plain : 16;; end = n_plain) {
        for (; u + (ONE || SHORT ? 0 : 1) < end; u += ONE || SHORT ? 1 : 2) {
            ks.next(u, ka, kb);
            stats_fast<0>(qa, ka, acc, c, z, a.c1);
            if (SHORT) {
                copy_subtile(ka, kb);
                if (NG & 1) copy_group(acc[1], acc[0]);
            } else if (!ONE) {                                 // the operands, and with an odd number of groups the accumulators, change places
                ks.next(u + 1, kb, ka);
                stats_fast<NG & 1>(qa, kb, acc, c, z, a.c1);
            }
            if ((u & 15) >= 14) level();
        }
        if (end == n_plain) break;
        if (__any(outside(least) || least < SUM_LEAST)) return true;
    }
    if (!ONE && !SHORT && u < n_plain) {
        ks.next(u++, ka, kb);
        stats_fast<0>(qa, ka, acc, c, z, a.c1);
        stats_add<0>(acc[(NG & 1) ^ 1], NG - 1, z, a.c1, 0, 0, 0);
        copy_subtile(ka, kb);
    } else {
        stats_add<0>(acc[1], NG - 1, z, a.c1, 0, 0, 0);
    }
    lane = lane_again();
    n = lane & 15, g = lane >> 4;
    // the subtiles with masked keys
    for (; u < w.n_sub; ++u) {
        ks.next(u, ka, kb);
#pragma unroll
        for (int j = 0; j < NG; ++j) {
            multiply(qa, ka, j, c, acc[j & 1]);
            stats_add<W>(acc[j & 1], j, z, a.c1, w.first + u * STRIDE + n, g, T);
        }
        copy_subtile(ka, kb);
    }
    level();
    // per row: the lane group's 16 sums together
#pragma unroll
    for (int J = 0; J < NT; ++J) {
#pragma unroll
        for (int i = 0; i < 4; ++i) zo[J][i] = group_sum(zo[J][i]);
        const floatx4 ref = c(J);
        if (n == 0) {
            floatx4 *st = state + (TILE * J + 4 * g) / 2;
            st[0] = floatx4{ref[0], zo[J][0], ref[1], zo[J][1]};
            st[1] = floatx4{ref[2], zo[J][2], ref[3], zo[J][3]};
        }
    }
    bool again = outside(least);
    if (w.first <= T) again |= least < SUM_LEAST;
    else                                                       // inside the window: of the rows that see the stream's first key
        for (int pos = lane; pos < R::MP; pos += 64)
            again |= w.first <= T + R::row_of(pos) % W && reinterpret_cast<const float *>(state)[2 * pos + 1] < SUM_LEAST;
    return again;
}

template <int NT, int W, int KS>
__global__ void __launch_bounds__(WAVES * 64)
score_mfma_stats(ScoreArgs a)
{
    using R = Rows<NT, W>;
    constexpr int MP = R::MP;
    extern __shared__ __attribute__((aligned(8192))) char lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const Dims &d = a.d;
    char *ring = lds + wave * RING_BYTES;
    floatx4 *wg_state = reinterpret_cast<floatx4 *>(lds + WAVES * RING_BYTES);     // [WAVES][MP / 2], see stats_careful
    floatx4 *state = wg_state + wave * (MP / 2);
    float *refs = reinterpret_cast<float *>(wg_state + WAVES * (MP / 2)) + wave * MP;     // see stats_walk
    const WaveWork w = wave_work(a, wave);

    // queries before keys, as loads return in order; both are in flight together
    bf16x8 qa[NT][KS];
    using Stream = typename StreamFor<NT, KS, NT <= 8>::type;
    Stream ks;
    ks.init(w.kp, d.ks[3], ring, w.first, w.n_sub, d.L, lane);
    if constexpr (KS == 4) {
        using Q = QueryStage<NT>;
        const uint32_t ring0 = __builtin_amdgcn_readfirstlane(lds_addr(lds));
        Q::template issue<W>(a, w.p, ring0, wave, lane);
        ks.issue_first(0, NBUF - Q::BUFS);
        wait_loads(min(NBUF - Q::BUFS, w.n_sub));              // the queries; the keys stay in flight
        lds_barrier();
        Q::read(qa, ring0, lane);
        pin_queries<NT, W>(qa, a, lane);
        lds_barrier();
        ks.issue_first(NBUF - Q::BUFS, NBUF);
    } else {
        load_queries<NT, W>(qa, a, w.p, lane);
        pin_queries<NT, W>(qa, a, lane);
    }

    const int n_plain = plain_subtiles(w, d.T);
    if (__builtin_expect(__any(stats_walk<refs_first<NT, KS>(), NT, W, KS>(a, w, ks, qa, state, refs, n_plain, lane)), 0)) {
        auto restart = [&]() __attribute__((always_inline)) {
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");        // what is on its way to the ring or from it
            ks.init(w.kp, d.ks[3], ring, w.first, w.n_sub, d.L, lane_again());
            ks.issue_first();
        };
        restart();
        bool careful = refs_first<NT, KS>() || n_plain == 0;
        if constexpr (!refs_first<NT, KS>())
            if (!careful) {
                careful = __any(stats_walk<true, NT, W, KS>(a, w, ks, qa, state, refs, n_plain, lane));
                if (careful) restart();
            }
        if (careful) {
            bf16x8 ka[2][KS], kb[2][KS];
            ks.start(ka);
            for (int u = 0; u < w.n_sub; ++u) {
                ks.next(u, ka, kb);
                stats_careful<NT, W>(a, w.p, ka, state, u == 0, w.first + u * STRIDE, n, g);
                copy_subtile(ka, kb);
            }
        }
    }

    // ---- the four wavefronts' (reference, sum) pairs together
    __syncthreads();
    const int row = R::row_of(threadIdx.x), M = d.G * W;
    if (threadIdx.x < MP && row < M) {
        float ref[WAVES], sum[WAVES], m = -INFINITY, zz = 0.f;
#pragma unroll
        for (int wv = 0; wv < WAVES; ++wv) {
            const float *e = reinterpret_cast<const float *>(wg_state + wv * (MP / 2)) + threadIdx.x * 2;
            ref[wv] = -e[0] * a.c1;                            // log2 domain
            sum[wv] = e[1];
            if (sum[wv] > 0.f) m = fmaxf(m, ref[wv]);
        }
#pragma unroll
        for (int wv = 0; wv < WAVES; ++wv)
            if (sum[wv] > 0.f) zz += sum[wv] * __builtin_amdgcn_exp2f(ref[wv] - m);
        float *o = a.partial + (((int64_t)w.p * a.n_chunks + w.chunk) * M + row) * 2;
        o[0] = m;
        o[1] = zz;
    }
}
template <int NT> constexpr int stats_lds() { return WAVES * RING_BYTES + WAVES * TILE * NT * 3 * 4; }   // rings + the rows' state and references

// ------------------------------------------------------------------ pass 2
// Folds the (reference, sum) pairs c0, c0 + step, ... < n of one row (`stride` floats apart) into (m, z).  The pairs
// are read sixteen at a time, all loads in flight: what this costs a workgroup is their latency, not their bytes.
constexpr int FOLD_BATCH = 16;
__device__ __forceinline__ void fold_load(float2 (&e)[FOLD_BATCH], const float *pp, int64_t stride, int c, int step, int n)
{
#pragma unroll
    for (int j = 0; j < FOLD_BATCH; ++j) e[j] = *reinterpret_cast<const float2 *>(pp + (int64_t)min(c + j * step, n - 1) * stride);
}
__device__ __forceinline__ void fold_add(float2 (&e)[FOLD_BATCH], int c, int step, int n, float &m, float &z)
{
    float mn = m;
#pragma unroll
    for (int j = 0; j < FOLD_BATCH; ++j) {
        if (c + j * step >= n) e[j].y = 0.f;
        if (e[j].y > 0.f) mn = fmaxf(mn, e[j].x);
    }
    if (z > 0.f) z *= __builtin_amdgcn_exp2f(m - mn);
#pragma unroll
    for (int j = 0; j < FOLD_BATCH; ++j)
        if (e[j].y > 0.f) z += e[j].y * __builtin_amdgcn_exp2f(e[j].x - mn);
    m = mn;
}
__device__ __forceinline__ void fold_pairs(const float *pp, int64_t stride, int c0, int step, int n, float &m, float &z)
{
    m = -INFINITY;
    z = 0.f;
    for (int c = c0; c < n; c += step * FOLD_BATCH) {
        float2 e[FOLD_BATCH];
        fold_load(e, pp, stride, c, step, n);
        fold_add(e, c, step, n, m, z);
    }
}

// A row's log-sum-exp in the log2 domain plus log2 of the heads that the mean is over, into lse2[position]; +inf for
// padding.  Given by the caller, or folded from the chunk partials of pass 1 by several threads per row.  256 threads;
// meanwhile() runs when the first loads are on their way; ends without a barrier behind the last stores.
template <int NT, int W, typename F>
__device__ __forceinline__ void fold_rows(const ScoreArgs &a, int p, float log2_heads, float *lse2, float2 *comb, F &&meanwhile)
{
    constexpr int PER = NT <= 1 ? 16 : NT <= 2 ? 32 : NT <= 4 ? 64 : NT <= 8 ? 128 : 256, PARTS = 256 / PER;
    const int M = a.d.G * W, pos = threadIdx.x % PER, part = threadIdx.x / PER;
    const int r = Rows<NT, W>::row_of(pos);
    const bool real = pos < Rows<NT, W>::MP && r < M;
    float m = -INFINITY, z = 0.f;
    if (a.lse) {
        if (real && part == 0) { m = a.lse[(int64_t)p * M + r]; z = 1.f; }
        meanwhile();
        m *= LOG2E;
    } else {
        const float *pp = a.merged + ((int64_t)p * a.pc * M + min(r, M - 1)) * 2;
        float2 e[FOLD_BATCH];
        if (real && part < a.pc) fold_load(e, pp, M * 2, part, PARTS, a.pc);
        meanwhile();
        if (real && part < a.pc) fold_add(e, part, PARTS, a.pc, m, z);
        for (int c = part + PARTS * FOLD_BATCH; real && c < a.pc; c += PARTS * FOLD_BATCH) {
            fold_load(e, pp, M * 2, c, PARTS, a.pc);
            fold_add(e, c, PARTS, a.pc, m, z);
        }
    }
    if (PARTS > 1) {
        comb[threadIdx.x] = make_float2(m, z);
        __syncthreads();
        if (part != 0) return;
        float2 e[PARTS];
        m = -INFINITY;
#pragma unroll
        for (int j = 0; j < PARTS; ++j) { e[j] = comb[j * PER + pos]; m = fmaxf(m, e[j].x); }
        z = 0.f;
#pragma unroll
        for (int j = 0; j < PARTS; ++j)
            if (e[j].y > 0.f) z += e[j].y * __builtin_amdgcn_exp2f(e[j].x - m);
    }
    if (pos < Rows<NT, W>::MP) lse2[pos] = real ? m + __builtin_amdgcn_logf(z) + log2_heads : INFINITY;
}

// Adds group j's probabilities (acc = <q,k> - lse2 / c1, so exp2(c1 * acc) = A / heads) to the head means; t: the lane's key
// in the first key tile
template <int NT, int W, bool EDGE>
__device__ __forceinline__ void columns_add(const floatx4 (&acc)[2][2], int j, float (&ab)[2][W / 4], float c1, int t, int g, int T, int L)
{
    using R = Rows<NT, W>;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int J = 2 * j + r, key = t + TILE * kt;
                if (J >= NT) continue;
                float v = __builtin_amdgcn_exp2f(acc[r][kt][i] * c1);
                if (EDGE && !(key < L && key <= T + R::query(J, g, i))) v = 0.f;          // causal inside the window
                float &to = ab[kt][R::slot(J, i)];
                to = R::first(J, i) ? v : to + v;                                         // Eq. barA
            }
}

// Sums of two values over the four lane groups: lanes of the even groups get the first value's, the others the second's.
// permlane16_swap exchanges the odd groups of its first operand with the even groups of its second, permlane32_swap the
// upper half of the first with the lower half of the second.
__device__ __forceinline__ float sum_groups(float x0, float x1)
{
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x0), __float_as_uint(x1), false, false);
    const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// smallest value of the four lane groups that hold a key's rows; numbers before what is none
__device__ __forceinline__ float min_groups(float v)
{
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fminf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fminf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// The power of two that the probabilities of all rows are taken by (see above), from the smallest of the rows' log-sum-exps:
// no C operand is then larger than without it.  Never negative, as the exponentials flush to zero what lies below 2^-126 in
// any case: at -100 that were all probabilities below 2^-26.  At most 2^100, so that the sums over the rows stay finite
// (8 192 keys, 128 rows, all logits 60 above zero: scores 1.7e-6 off, 4.0e-6 with at most 2^32).
__device__ __forceinline__ float common_power(float least) { return fminf(fmaxf(rintf(least), 0.f), COMMON_MOST); }

// Column sums (Eq. st, lanes 0 .. 31: one of the subtile's 32 keys each) and entropy terms (inner sum of Eq. Dk, lanes 32
// .. 63) from the lane's head means, which are to be taken `scale` times
template <int NS>
__device__ __forceinline__ float columns_finish(const float (&ab)[2][NS], float scale, float eps, int lane)
{
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int i = 0; i < NS; ++i) { s0 += ab[0][i]; s1 += ab[1][i]; }
    const float s = sum_groups(s0, s1);
    const float inv = s > 0.f ? __builtin_amdgcn_rcpf(s) : 0.f;
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(inv), __float_as_uint(inv), false, false);
    const float inv0 = __uint_as_float(b[0]), inv1 = __uint_as_float(b[1]);                // of the two keys of this lane
    // sum_i Ahat_i log2(Ahat_i + eps) with Ahat_i = Abar_i / s: the division of the weights is applied once, to the sum
    float e0 = 0.f, e1 = 0.f;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
        e0 = fmaf(ab[0][i], __builtin_amdgcn_logf(fmaf(ab[0][i], inv0, eps)), e0);
        e1 = fmaf(ab[1][i], __builtin_amdgcn_logf(fmaf(ab[1][i], inv1, eps)), e1);
    }
    const float ent = -LN2 * inv * sum_groups(e0, e1);
    return lane < 32 ? s * scale : ent;
}

// Column sums and entropy terms.  STORE: instead of them, write the head-group mean Abar[query][key] itself (for the mean
// over ALL heads of a layer, which is formed across KV heads afterwards), layout [problem][W / 4][L][4]: consecutive
// window queries of a key per store.
//
// Results are stored one iteration late, at the top of the next iteration, so that the multiply/exponentiate section of
// an iteration is a single straight-line region.  The subtiles before the window (no mask) and the ones that touch the
// window or the end of the sequence run in two consecutive loops, which keeps the masked body out of the hot loop.
template <int NT, int W, bool STORE, int KS>
__global__ void __launch_bounds__(WAVES * 64)
score_mfma_columns(ScoreArgs a)
{
    using R = Rows<NT, W>;
    constexpr int NG = R::NG, NS = R::NS;
    extern __shared__ __attribute__((aligned(8192))) char lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const Dims &d = a.d;
    char *ring = lds + wave * RING_BYTES;
    float2 *comb = reinterpret_cast<float2 *>(lds + WAVES * RING_BYTES);     // [256] combine scratch
    float *lse2 = reinterpret_cast<float *>(comb + 256);                     // [MP] see fold_rows
    const WaveWork w = wave_work(a, wave);

    // queries and the first of the fold's loads before the keys, as loads return in order; all are in flight together
    bf16x8 qa[NT][KS];
    using Stream = typename StreamFor<NT, KS, NT <= 8>::type;
    Stream ks;
    ks.init(w.kp, d.ks[3], ring, w.first, w.n_sub, d.L, lane);
    if constexpr (KS == 4) {
        using Q = QueryStage<NT>;
        const uint32_t ring0 = __builtin_amdgcn_readfirstlane(lds_addr(lds));
        Q::template issue<W>(a, w.p, ring0, wave, lane);
        fold_rows<NT, W>(a, w.p, a.log2_G, lse2, comb, [&]() __attribute__((always_inline)) { ks.issue_first(0, NBUF - Q::BUFS); });
        wait_loads(min(NBUF - Q::BUFS, w.n_sub));
        lds_barrier();
        Q::read(qa, ring0, lane);
        pin_queries<NT, W>(qa, a, lane);
        lds_barrier();
        ks.issue_first(NBUF - Q::BUFS, NBUF);
    } else {
        load_queries<NT, W>(qa, a, w.p, lane);
        fold_rows<NT, W>(a, w.p, a.log2_G, lse2, comb, []() {});
        pin_queries<NT, W>(qa, a, lane);
        __syncthreads();
    }
    bf16x8 ka[2][KS], ahead[2][KS];
    auto &kb = Stream::AHEAD ? ahead : ka;
    ks.start(ka);

    floatx4 cinit[NT], acc[2][2][2];
    float least = INFINITY;
#pragma unroll
    for (int J = 0; J < NT; ++J) {
        cinit[J] = *reinterpret_cast<const floatx4 *>(lse2 + TILE * J + 4 * g);
#pragma unroll
        for (int i = 0; i < 4; ++i) least = fminf(least, cinit[J][i]);
    }
    const float common = common_power(min_groups(least));
    const float scale = __builtin_amdgcn_exp2f(-common), inv_c1 = 1.0f / a.c1;
#pragma unroll
    for (int J = 0; J < NT; ++J) {
#pragma unroll
        for (int i = 0; i < 4; ++i) cinit[J][i] = (common - cinit[J][i]) * inv_c1;
    }
    set_nothing(acc[0]);                                       // the "previous subtile" of iteration 0 is a no-op
    set_nothing(acc[1]);
    float ab[2][NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) ab[0][i] = ab[1][i] = 0.f;
    float *out = (lane < 32 ? a.s_out : a.e_out) + (int64_t)w.p * d.L;

    float pending = 0.f;                                       // result of subtile pending_u
    int pending_u = -1;
    auto finish = [&](int u, bool edge) __attribute__((always_inline)) {                      // the head means of subtile u are complete
        if (!STORE) {
            pending = columns_finish<NS>(ab, scale, a.eps, lane);
            pending_u = u;
            return;
        }
        if (u < 0) return;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
            const int t = w.first + u * STRIDE + TILE * kt + n;
            if (edge && t >= d.L) continue;
            float *row = a.abar + (int64_t)w.p * (W / 4) * d.L * 4;
            if (W == 8) *reinterpret_cast<float2 *>(row + ((int64_t)(g >> 1) * d.L + t) * 4 + 2 * (g & 1)) = make_float2(ab[kt][0] * scale, ab[kt][1] * scale);
            else
#pragma unroll
                for (int J = 0; J < R::PER_HEAD; ++J)
                    *reinterpret_cast<float4 *>(row + ((int64_t)(4 * J + g) * d.L + t) * 4) =
                        make_float4(ab[kt][4 * J] * scale, ab[kt][4 * J + 1] * scale, ab[kt][4 * J + 2] * scale, ab[kt][4 * J + 3] * scale);
        }
    };
    auto put = [&](bool edge) __attribute__((always_inline)) {
        const int t = w.first + pending_u * STRIDE + (lane & 31);
        if (!STORE && pending_u >= 0 && (!edge || t < d.L)) out[t] = pending;
    };
    int u = 0;
    // one subtile: group j is multiplied into acc[(j + PAR) & 1] while the group before it is exponentiated
    auto subtile = [&](bf16x8 (&cur)[2][KS], bf16x8 (&nxt)[2][KS], auto par, auto edge_t) __attribute__((always_inline)) {
        constexpr int PAR = decltype(par)::value;
        constexpr bool EDGE = decltype(edge_t)::value;
        put(EDGE);
        ks.next(u, cur, nxt);
        const int t = w.first + u * STRIDE + n;
#pragma unroll
        for (int j = 0; j < NG; ++j) {
            multiply(qa, cur, j, [&](int J) { return cinit[J]; }, acc[(j + PAR) & 1]);
            if (j == 1) finish(u - 1, EDGE);                   // under this group's products
            columns_add<NT, W, EDGE>(acc[(j + PAR + 1) & 1], j > 0 ? j - 1 : NG - 1, ab, a.c1, j > 0 ? t : t - STRIDE, g, d.T, d.L);
            if (NG == 1) finish(u - 1, EDGE);
        }
        // the means as they are here: keeps the compiler from moving this subtile's exponentials behind the next one's loads
#pragma unroll
        for (int i = 0; i < NS; ++i) asm volatile("" : "+v"(ab[0][i]), "+v"(ab[1][i]));
        if (!STORE) asm volatile("" : "+v"(pending));
        ++u;
    };
    // two subtiles a step: the operands, and with an odd number of groups the accumulators, change places
    auto run = [&](int end, auto edge_t) __attribute__((always_inline)) {
        using std::integral_constant;
        while (u + 1 < end) {
            subtile(ka, kb, integral_constant<int, 0>{}, edge_t);
            subtile(kb, ka, integral_constant<int, NG & 1>{}, edge_t);
        }
        if (u < end) {
            subtile(ka, kb, integral_constant<int, 0>{}, edge_t);
            copy_subtile(ka, kb);
            if (NG & 1) copy_group(acc[1], acc[0]);
        }
    };
    run(plain_subtiles(w, d.T), std::false_type{});
    run(w.n_sub, std::true_type{});
    put(true);
    if (w.n_sub > 0) {
        columns_add<NT, W, true>(acc[1], NG - 1, ab, a.c1, w.first + (w.n_sub - 1) * STRIDE + n, g, d.T, d.L);
        finish(w.n_sub - 1, true);
        put(true);
    }
}
template <int NT> constexpr int columns_lds() { return WAVES * RING_BYTES + 256 * 8 + TILE * NT * 4; }   // rings + combine scratch + the rows' log-sum-exp

// ------------------------------------------------------------------ pass 2, all heads of a layer
// Head mean over all 32 heads of a layer with 8 KV heads (Eq. barA taken literally) without writing the
// per-KV-head means to memory.  A workgroup owns a chunk of keys of one (sequence, layer).  Wavefront w multiplies
// the keys of KV heads 2w and 2w+1 (two load streams interleaved in one ring) by those heads' 8 query heads (256
// accumulation registers of A operands) and adds exp2 over its 8 heads; the four partial sums of a subtile meet
// in LDS, where the wavefronts take turns (subtile u: wavefront u % 4) to add them and to form the column sum
// and the entropy term.  One barrier per subtile; it waits for LDS only, never for the loads in flight.
constexpr int LAYER_KV = 8;                   // KV heads of a layer this kernel is built for (two per wavefront)
constexpr int XCH_BYTES = 16 * 64 * 4;        // one wavefront's partial sums of a subtile, [4][64 lanes][4]
constexpr int LAYER_NT = 16;                  // row tiles of a wavefront: two KV heads of four heads
constexpr int PL_LDS = WAVES * RING_BYTES + 2 * 3 * XCH_BYTES + WAVES * LAYER_NT * TILE * 4;   // rings + exchange + C operands

// Two key streams of one wavefront as one sequence of half-steps: element e = 2u + s is subtile u of stream s and
// lives in ring buffer e % NBUF, refilled with element e + NBUF right after it is read.  Subtile u covers keys
// [first + u * SUB, +SUB): here all wavefronts of a workgroup walk the same keys.
struct PairStream {
    const uint16_t *kp0, *kp1;
    int64_t ks3;
    uint32_t lane_addr0, ring_lds;
    uint32_t lane_off[4];
    int first, n_el, L, lane;

    __device__ __forceinline__ void init(const uint16_t *k0, const uint16_t *k1, int64_t ks3_, char *ring, int first_, int n_sub, int L_, int lane_)
    {
        kp0 = k0; kp1 = k1; ks3 = ks3_; first = first_; n_el = 2 * n_sub; L = L_; lane = lane_;
        const int r4 = lane >> 4, pos = lane & 15;
        ring_lds = __builtin_amdgcn_readfirstlane(lds_addr(ring));
        lane_addr0 = ring_lds + lane_read_offset(lane);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) lane_off[jj] = (uint32_t)(r4 * ks3 * 2) + (uint32_t)(((pos ^ r4 ^ (4 * jj)) & 15) << 4);
    }
    __device__ __forceinline__ void issue(int e) const
    {
        const int t0 = first + (e >> 1) * SUB;                 // wave-uniform, < L
        const char *base = reinterpret_cast<const char *>((e & 1) ? kp1 : kp0) + (int64_t)t0 * ks3 * 2;
        const uint32_t buf_lds = ring_lds + (e % NBUF) * BUF_BYTES;
        if (t0 + SUB <= L) {
            if (ks3 == ROW_BYTES / 2) issue_subtile_dense(base, lane_off, buf_lds);
            else issue_subtile_fast(base, ks3 * 2, lane_off, buf_lds);
        } else issue_subtile_clamped(base, ks3 * 2, L - t0, buf_lds, lane);
    }
    // element 0 into kb
    __device__ __forceinline__ void start(bf16x8 (&kb)[2][4]) const
    {
#pragma unroll
        for (int e = 0; e < NBUF; ++e)
            if (e < n_el) issue(e);
        if (n_el == 0) return;
        wait_loads(min(NBUF, n_el) - 1);
        read_subtile(lane_addr0, kb);
    }
    // element e is in `cur`; element e + 1, if there is one, into `nxt`
    __device__ __forceinline__ void next(int e, bf16x8 (&cur)[2][4], bf16x8 (&nxt)[2][4]) const
    {
        have_subtile<false>(cur);
        if (e + NBUF < n_el) issue(e + NBUF);
        if (e + 1 < n_el) {
            wait_loads(min(NBUF - 1, n_el - 2 - e));
            read_subtile(lane_addr0 + ((e + 1) % NBUF) * BUF_BYTES, nxt);
        }
    }
};

// this lane's 16 partial sums into an exchange slot / the sum of `ab` and the three slots of a buffer
__device__ __forceinline__ void xch_write(uint32_t addr, const float (&ab)[2][8])
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float *x = ab[j >> 1] + 4 * (j & 1);
        const floatx4 v = {x[0], x[1], x[2], x[3]};
        asm volatile("ds_write_b128 %0, %1" : : "v"(addr + j * 1024), "v"(v) : "memory");
    }
}
__device__ __forceinline__ void xch_add(uint32_t addr, float (&ab)[2][8])
{
    typedef const floatx4 __attribute__((address_space(3))) *lds_vec;
    floatx4 v[3][4];
#pragma unroll
    for (int sl = 0; sl < 3; ++sl)
#pragma unroll
        for (int j = 0; j < 4; ++j) v[sl][j] = *(lds_vec)(uintptr_t)(addr + sl * XCH_BYTES + j * 1024);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int c = 0; c < 4; ++c) ab[j >> 1][4 * (j & 1) + c] += v[0][j][c] + v[1][j][c] + v[2][j][c];
}
struct LayerCtx {
    uint32_t xch_lds;      // exchange area
    int wave, lane, n, g;
    int lo;                // first key of the chunk
    float c1, scale, eps;
    int T, L;
    float *out;            // s (lanes 0 .. 31) or entropy term (lanes 32 .. 63) row of this (sequence, layer)
};

// the partial sums `ab` of subtile `up` are complete in every wavefront: hand them to wavefront up % 4 ...
__device__ __forceinline__ void layer_give(const LayerCtx &c, int up, const float (&ab)[2][8])
{
    const int fin = up & 3;
    if (c.wave != fin) xch_write(c.xch_lds + (uint32_t)(((up & 1) * 3 + ((c.wave - fin - 1) & 3)) * XCH_BYTES + c.lane * 16), ab);
}
// ... which, after the barrier, adds them up and stores the two results of its key
__device__ __forceinline__ void layer_take(const LayerCtx &c, int up, float (&ab)[2][8])
{
    if (c.wave != (up & 3)) return;
    xch_add(c.xch_lds + (uint32_t)((up & 1) * 3 * XCH_BYTES + c.lane * 16), ab);
    const float v = columns_finish<8>(ab, c.scale, c.eps, c.lane);
    const int t = c.lo + up * SUB + (c.lane & 31);
    if (t < c.L) c.out[t] = v;
}

// One subtile u: heads 0-3 (KV head 2w) then 4-7 (KV head 2w+1), a group of two tiles each, rotating through two sets of
// accumulators; head 7 of the previous subtile is exponentiated first, which completes that subtile's partial sums (handed
// over mid-way).
template <bool EDGE>
__device__ __forceinline__ void layer_body(const LayerCtx &c, const bf16x8 (&qa)[LAYER_NT][4], const PairStream &ps,
                                           const float *cm, bf16x8 (&ka)[2][4], bf16x8 (&kb)[2][4], floatx4 (&acc)[2][2][2],
                                           float (&ab)[2][8], int u)
{
    const int t_cur = c.lo + u * SUB + c.n, t_prev = t_cur - SUB;
    float abp[2][8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (j % 4 == 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(ab[0][i]), "+v"(ab[1][i]));
            if (j == 0) ps.next(2 * u, ka, kb);
            else ps.next(2 * u + 1, kb, ka);
        }
        // the C operands come from LDS: all registers are taken
        multiply(qa, j < 4 ? ka : kb, j, [&](int J) { return *reinterpret_cast<const floatx4 *>(cm + J * TILE); }, acc[j & 1]);
        columns_add<LAYER_NT, 32, EDGE>(acc[(j & 1) ^ 1], j > 0 ? j - 1 : 7, ab, c.c1, j > 0 ? t_cur : t_prev, c.g, c.T, c.L);
        if (j == 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) { abp[0][i] = ab[0][i]; abp[1][i] = ab[1][i]; }
            if (u > 0) layer_give(c, u - 1, abp);
        }
        if (j == 4 && u > 0) {                                 // u is uniform over the workgroup
            lds_barrier();
            layer_take(c, u - 1, abp);
        }
    }
}

__global__ void __launch_bounds__(WAVES * 64)
score_mfma_columns_layer(ScoreArgs a)
{
    extern __shared__ __attribute__((aligned(8192))) char lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const Dims &d = a.d;
    char *ring = lds + wave * RING_BYTES;
    char *xch = lds + WAVES * RING_BYTES;                                     // [2 buffers][3 slots][4][64 lanes][4]
    float *cmat = reinterpret_cast<float *>(xch + 2 * 3 * XCH_BYTES);         // [wave][16 tiles][16 rows] C operands
    const int sl = blockIdx.y, chunk = blockIdx.x;
    const int p_first = sl * LAYER_KV;                                        // the layer's first problem
    const int lo = chunk * a.chunk_len, hi = min(lo + a.chunk_len, d.L);
    const int n_sub = hi > lo ? (hi - lo + SUB - 1) / SUB : 0;                // the same for the four wavefronts

    PairStream ps;
    ps.init(a.k + k_problem_offset(d, p_first + 2 * wave), a.k + k_problem_offset(d, p_first + 2 * wave + 1), d.ks[3], ring, lo,
            n_sub, d.L, lane);
    bf16x8 ka[2][4], kb[2][4];
    ps.start(ka);

    // C operands: minus (row log-sum-exp + log2 of the number of heads - the part that all rows share) / c1.  Row R = kv * 128
    // + h * 32 + query; four rows per thread.
    float lse[4];
    {
        const float log2_heads = __builtin_amdgcn_logf((float)(d.G * LAYER_KV));
#pragma unroll
        for (int k4 = 0; k4 < 4; ++k4) {
            const int R = threadIdx.x + 256 * k4, kv = R >> 7, row = R & (M_ROWS - 1);
            float m = -INFINITY, zz = 0.f;
            if (a.lse) {
                m = a.lse[(int64_t)(p_first + kv) * M_ROWS + row] * LOG2E;
                zz = 1.f;
            } else {
                fold_pairs(a.merged + ((int64_t)(p_first + kv) * a.pc * M_ROWS + row) * 2, M_ROWS * 2, 0, 1, a.pc, m, zz);
            }
            lse[k4] = m + __builtin_amdgcn_logf(zz) + log2_heads;
        }
        const float least = min_groups(-group_max(-fminf(fminf(lse[0], lse[1]), fminf(lse[2], lse[3]))));
        if (lane == 0) cmat[wave] = least;                     // the same power for all heads: their probabilities are added
    }
    __syncthreads();
    const float common = common_power(fminf(fminf(cmat[0], cmat[1]), fminf(cmat[2], cmat[3])));
    __syncthreads();
#pragma unroll
    for (int k4 = 0; k4 < 4; ++k4) cmat[threadIdx.x + 256 * k4] = (common - lse[k4]) * (1.0f / a.c1);
    __syncthreads();

    LayerCtx c;
    c.xch_lds = __builtin_amdgcn_readfirstlane(lds_addr(xch));
    c.wave = wave; c.lane = lane; c.n = lane & 15; c.g = lane >> 4;
    c.lo = lo; c.c1 = a.c1; c.scale = __builtin_amdgcn_exp2f(-common); c.eps = a.eps; c.T = d.T; c.L = d.L;
    c.out = (lane < 32 ? a.s_out : a.e_out) + (int64_t)sl * d.L;

    bf16x8 qa[LAYER_NT][4];
#pragma unroll
    for (int J = 0; J < LAYER_NT; ++J) {
        const uint16_t *row = a.q + q_row_offset(d, p_first + 2 * wave + J / 8, (J % 8) / 2, TILE * (J % 2) + c.n) + c.g * 8;
#pragma unroll
        for (int s = 0; s < 4; ++s) qa[J][s] = *reinterpret_cast<const bf16x8 *>(row + 32 * s);
    }
    pin_queries<LAYER_NT, 32>(qa, a, lane);                    // all 256 accumulation registers

    const float *cm = cmat + wave * LAYER_NT * TILE + 4 * c.g;
    floatx4 acc[2][2][2];
    set_nothing(acc[0]);
    set_nothing(acc[1]);
    float ab[2][8];
#pragma unroll
    for (int i = 0; i < 8; ++i) ab[0][i] = ab[1][i] = 0.f;

    const int n_plain = lo + SUB <= d.T ? min(n_sub, (d.T - SUB - lo) / SUB + 1) : 0;
    int u = 0;
    for (; u < n_plain; ++u) layer_body<false>(c, qa, ps, cm, ka, kb, acc, ab, u);
    for (; u < n_sub; ++u) layer_body<true>(c, qa, ps, cm, ka, kb, acc, ab, u);
    if (n_sub > 0) {                                           // head 7 of the last subtile, then its hand-over
        columns_add<LAYER_NT, 32, true>(acc[1], 7, ab, c.c1, lo + (n_sub - 1) * SUB + c.n, c.g, c.T, c.L);
        layer_give(c, n_sub - 1, ab);
        lds_barrier();
        layer_take(c, n_sub - 1, ab);
    }
}

// Folds the chunk partials of pass 1 into one (reference, sum) pair per row, one wavefront per row, so that
// with many chunks per problem the workgroups of pass 2 do not each repeat the fold.
// partial [blocks][n_chunks][M][2] -> merged [blocks][M][2]; grid ceil(blocks * M / 4), 256 threads
__global__ void __launch_bounds__(256)
merge_partials_kernel(const float *partial, float *merged, int n_chunks, int M, int n_rows)
{
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= n_rows) return;
    const int blk = r / M, row = r - blk * M;
    const float *pp = partial + ((int64_t)blk * n_chunks * M + row) * 2;
    float m = -INFINITY, z = 0.f;
    for (int c = lane; c < n_chunks; c += 64) {
        const float2 e = *reinterpret_cast<const float2 *>(pp + (int64_t)c * M * 2);
        if (e.y > 0.f) {
            const float mn = fmaxf(m, e.x);
            z = z * __builtin_amdgcn_exp2f(m - mn) + e.y * __builtin_amdgcn_exp2f(e.x - mn);
            m = mn;
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        const float m2 = __shfl_xor(m, off), z2 = __shfl_xor(z, off);
        const float mn = fmaxf(m, m2);
        z = (z > 0.f ? z * __builtin_amdgcn_exp2f(m - mn) : 0.f) + (z2 > 0.f ? z2 * __builtin_amdgcn_exp2f(m2 - mn) : 0.f);
        m = mn;
    }
    if (lane == 0) {
        merged[(int64_t)r * 2] = m;
        merged[(int64_t)r * 2 + 1] = z;
    }
}

// enqueues the fold when pass 2 is to read merged pairs (a.pc == 1 with more than one chunk)
void launch_merge(const ScoreArgs &a, int blocks, int M, hipStream_t st)
{
    if (a.merged == a.partial) return;
    const int n_rows = blocks * M;
    hipLaunchKernelGGL(merge_partials_kernel, dim3((unsigned)((n_rows + 3) / 4)), dim3(256), 0, st,
                       a.partial, const_cast<float *>(a.merged), a.n_chunks, M, n_rows);
}

template <int NT, int W, bool STORE, int KS = 4>
hipError_t launch_shape(const ScoreArgs &a, dim3 grid, bool with_stats, hipStream_t st)
{
    static thread_local PerDeviceOnce attr_once;
    if (attr_once.needed()) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(score_mfma_stats<NT, W, KS>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, stats_lds<NT>());
        if (e != hipSuccess) return e;
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(score_mfma_columns<NT, W, STORE, KS>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, columns_lds<NT>());
        if (e != hipSuccess) return e;
        attr_once.done();
    }
    if (with_stats) {
        hipLaunchKernelGGL((score_mfma_stats<NT, W, KS>), grid, dim3(WAVES * 64), stats_lds<NT>(), st, a);
        launch_merge(a, a.d.P, a.d.G * W, st);
    }
    hipLaunchKernelGGL((score_mfma_columns<NT, W, STORE, KS>), grid, dim3(WAVES * 64), columns_lds<NT>(), st, a);
    return hipGetLastError();
}

// Mean over the KV heads of a layer of the head-group means, then column sum and entropy term (Eqs. barA with
// all H heads, st, inner sum of Dk): one thread per key.  grid (ceil(L / 256), n_seq * n_layers)
template <int W>
__global__ void __launch_bounds__(256)
abar_reduce_kernel(const float *abar, int Hkv, int L, float eps, float *s_out, float *e_out)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= L) return;
    const int sl = blockIdx.y;
    float ab[W];
#pragma unroll
    for (int i = 0; i < W; ++i) ab[i] = 0.f;
    for (int kv = 0; kv < Hkv; ++kv) {
        const float4 *src = reinterpret_cast<const float4 *>(abar) + ((int64_t)(sl * Hkv + kv) * (W / 4)) * L + t;
#pragma unroll
        for (int j = 0; j < W / 4; ++j) {
            const float4 v = src[(int64_t)j * L];
            ab[4 * j] += v.x; ab[4 * j + 1] += v.y; ab[4 * j + 2] += v.z; ab[4 * j + 3] += v.w;
        }
    }
    const float inv_h = 1.0f / (float)Hkv;
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < W; ++i) { ab[i] *= inv_h; s += ab[i]; }
    const float inv_s = s > 0.f ? 1.0f / s : 0.f;
    float e = 0.f;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const float ah = ab[i] * inv_s;
        e = fmaf(ah, __builtin_amdgcn_logf(ah + eps), e);
    }
    s_out[(int64_t)sl * L + t] = s;
    e_out[(int64_t)sl * L + t] = -LN2 * e;
}

// (tiles, window) pairs: up to 128 rows; of a window of 32 or 64, up to 256 (the second list)
#define SABLOCK_SHAPES_96(X) X(1, 8) X(2, 8) X(3, 8) X(4, 8) X(5, 8) X(6, 8) X(1, 16) X(2, 16) X(3, 16) X(4, 16) X(5, 16) X(6, 16) X(2, 32) X(4, 32) X(6, 32)
#define SABLOCK_SHAPES(X) SABLOCK_SHAPES_96(X) X(7, 8) X(8, 8) X(7, 16) X(8, 16) X(8, 32)
#define SABLOCK_SHAPES_W64(X) X(4, 64) X(8, 64)
#define SABLOCK_SHAPES_WIDE(X) X(10, 32) X(12, 32) X(14, 32) X(16, 32) X(12, 64) X(16, 64)

bool tile_shape(const Dims &d)
{
    return (d.W == 8 || d.W == 16 || d.W == 32 || d.W == 64) && d.G >= 1 && d.G * d.W <= M_ROWS;
}
int tiles_of(const Dims &d) { return d.W == 8 ? (d.G + 1) / 2 : d.G * d.W / TILE; }
// 129 .. 256 rows of a window of 32 or 64 queries (G = 5 .. 8 / G = 3, 4)
bool wide_shape(const Dims &d)
{
    return (d.W == 32 || d.W == 64) && d.G * d.W > M_ROWS && d.G * d.W <= 2 * M_ROWS;
}

struct Plan {
    int chunk_len;    // keys per workgroup
    int n_chunks;     // workgroups per problem
    bool by_chunk;    // see plan_chunks
    bool merge;       // fold the chunk partials in a kernel of its own between the passes
};

// Chunks per problem from which the separate fold pays.  Up to 32 a column workgroup folds them itself in one or two
// reads of sixteen pairs per thread (8 problems of 8 192 keys, 32 chunks: the fold kernel took 4.1 us, the column pass is
// no slower without it); a workgroup of the all-head column kernel folds the rows of eight KV heads and hands over earlier.
constexpr int MERGE_FROM = 33, MERGE_FROM_LAYER = 8;

Plan make_plan(const Dims &d, int merge_from = MERGE_FROM)
{
    // One launch per pass covers every problem.  A workgroup owns chunk_len consecutive keys of one problem, and
    // one workgroup fills a CU (registers and the load ring).  Prologue and epilogue, during which its CU loads nothing, take
    // some 6 us, as long as 640 keys.  The chunk partials stay within 4 MiB where one round of workgroups does.  Both passes,
    // 128 rows, 30 011 keys, against the nearest whole number of chunks per unit: 24 problems 113 -> 74 us, 96 383 -> 287, 144
    // 563 -> 432, 320 1 117 -> 883.
    constexpr int MAX_CHUNK = 131072, FIXED = 640;
    Plan pl;
    if (d.tune.score_chunk >= STRIDE) {
        pl.chunk_len = (d.tune.score_chunk / STRIDE) * STRIDE;
        pl.n_chunks = (d.L + pl.chunk_len - 1) / pl.chunk_len;
        pl.by_chunk = false;
    } else {
        // More rounds than one, 128 rows of heads of 128: 175 problems of 5 943 keys in four chunks each 129 us, in one 112; 196 of 15 374
        // in five 302, in one 290; 200 of 49 215 907 and 947; 8 rows, 212 of 24 863 433 and 455.  More than two: 368 of 2 105 in two 113, in one 106.
        const int from_one = d.D < 128 || d.G * d.W <= 32 ? 5 * FIXED : d.G * d.W <= 64 ? 7 * FIXED : 10 * FIXED;
        const ChunkPlan c = plan_chunks(d.P, d.L, d.cus, STRIDE, FIXED, MAX_CHUNK, (4 << 20) / (d.G * d.W * 2 * 4),
                                        d.D == 128 && tiles_of(d) > 4 && tiles_of(d) <= 8 ? 1600 : 0, from_one, true);
        pl.chunk_len = c.len;
        pl.n_chunks = c.n;
        pl.by_chunk = c.by_chunk;
    }
    pl.merge = pl.n_chunks >= merge_from;
    return pl;
}

// bytes of the chunk partials, and of their merged form behind them
size_t partial_bytes(const Dims &d, const Plan &pl) { return align256((size_t)d.P * pl.n_chunks * d.G * d.W * 2 * 4); }
size_t merged_bytes(const Dims &d) { return align256((size_t)d.P * d.G * d.W * 2 * 4); }

// pass-1 bookkeeping of both entry points: where the partials go and what pass 2 reads
void plan_partials(ScoreArgs &a, const Dims &d, const Plan &pl, void *ws)
{
    a.chunk_len = pl.chunk_len;
    a.n_chunks = pl.n_chunks;
    a.by_chunk = pl.by_chunk || d.local;
    a.partial = static_cast<float *>(ws);
    a.merged = a.partial;
    a.pc = pl.n_chunks;
    if (pl.merge) {
        a.merged = reinterpret_cast<float *>(static_cast<char *>(ws) + partial_bytes(d, pl));
        a.pc = 1;
    }
}

}  // namespace

bool score_mfma_supported(const Dims &d)
{
    if (d.dtype != SABLOCK_BF16) return false;
    if (d.D == 64 || d.D == 96) return tile_shape(d);                       // up to 128 rows
    if (d.D == 256) return tile_shape(d) && (d.G * d.W + 31) / 32 <= 3;     // up to 96 rows: more A operands of 8 k-steps do not fit the registers
    return d.D == 128 && (tile_shape(d) || wide_shape(d));
}

// pass 1 by the window-attention kernel's first product (csrc/window_attn.hip), on request
static bool stats_by_rows(const Dims &d) { return row_stats_supported(d) && d.tune.stats_per_key == 2; }
static size_t row_stats_bytes(const Dims &d) { return align256((size_t)d.P * row_stats_chunks(d) * d.G * d.W * 2 * 4); }

size_t score_mfma_ws_bytes(const Dims &d)
{
    const Plan pl = make_plan(d);
    size_t part = partial_bytes(d, pl);
    if (stats_by_rows(d)) part = std::max(part, row_stats_bytes(d));
    return part + merged_bytes(d);
}

hipError_t launch_score_mfma(const Dims &d, const void *q, const void *k, const float *row_lse, float eps,
                             float *s_out, float *ent_out, void *ws, hipStream_t st)
{
    const Plan pl = make_plan(d);
    ScoreArgs a;
    a.d = d;
    a.q = static_cast<const uint16_t *>(q);
    a.k = static_cast<const uint16_t *>(k);
    plan_partials(a, d, pl, ws);
    a.c1 = (float)(1.4426950408889634 / sqrt((double)d.D));
    a.log2_G = (float)log2((double)d.G);
    a.eps = eps;
    a.s_out = s_out;
    a.e_out = ent_out;
    a.lse = row_lse;
    a.abar = nullptr;
    bool with_stats = !row_lse;
    if (with_stats && stats_by_rows(d)) {
        // a lane per window query; the chunks of this pass are its own
        const int nc1 = row_stats_chunks(d);
        hipError_t e = launch_row_stats(d, q, k, a.partial, st);
        if (e != hipSuccess) return e;
        a.merged = a.partial;
        a.pc = nc1;
        if (nc1 >= MERGE_FROM) {
            float *merged = reinterpret_cast<float *>(static_cast<char *>(ws) + row_stats_bytes(d));
            const int n_rows = d.P * d.G * d.W;
            hipLaunchKernelGGL(merge_partials_kernel, dim3((unsigned)((n_rows + 3) / 4)), dim3(256), 0, st, a.partial, merged,
                               nc1, d.G * d.W, n_rows);
            a.merged = merged;
            a.pc = 1;
        }
        with_stats = false;
    }
    const dim3 grid = a.by_chunk ? dim3(d.P, pl.n_chunks) : dim3(pl.n_chunks, d.P);
    const int nt = tiles_of(d);
#define X(NTV, WV) if (nt == NTV && d.W == WV) return launch_shape<NTV, WV, false, 8>(a, grid, with_stats, st);
    if (d.D == 256) { SABLOCK_SHAPES_96(X) X(4, 64) }
#undef X
#define X(NTV, WV) if (nt == NTV && d.W == WV) return launch_shape<NTV, WV, false, 3>(a, grid, with_stats, st);
    if (d.D == 96) { SABLOCK_SHAPES(X) SABLOCK_SHAPES_W64(X) }
#undef X
#define X(NTV, WV) if (nt == NTV && d.W == WV) return launch_shape<NTV, WV, false, 2>(a, grid, with_stats, st);
    if (d.D == 64) { SABLOCK_SHAPES(X) SABLOCK_SHAPES_W64(X) }
#undef X
#define X(NTV, WV) if (nt == NTV && d.W == WV) return launch_shape<NTV, WV, false>(a, grid, with_stats, st);
    if (d.D == 128) { SABLOCK_SHAPES(X) SABLOCK_SHAPES_W64(X) SABLOCK_SHAPES_WIDE(X) }
#undef X
    return hipErrorInvalidValue;
}

namespace {

// ---- measurement aid: the scoring kernels' key stream without their arithmetic
// Same chunk plan, same workgroups, same direct-to-LDS ring and waits as score_mfma_columns; per subtile a
// wavefront either only waits for the subtile and refills its buffer (READ_LDS = false), or also reads the whole
// subtile from LDS into registers as the scoring kernels do (READ_LDS = true).  With STORES it also writes what the
// column pass writes, 4 bytes per key into each of two [P][L] rows, with that kernel's store pattern (lanes 0..31 a
// row of s_out, lanes 32..63 a row of e_out, once per subtile).  What this kernel takes is what the memory system
// delivers to the scoring kernels' access pattern: the yardstick their times are compared with.
template <bool READ_LDS, bool STORES>
__global__ void __launch_bounds__(WAVES * 64)
stream_probe_kernel(ScoreArgs a, uint32_t *sink)
{
    extern __shared__ __attribute__((aligned(8192))) char lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    char *ring = lds + __builtin_amdgcn_readfirstlane(wave) * RING_BYTES;
    const WaveWork w = wave_work(a, wave);
    KeyStream<false, false> ks;
    ks.init(w.kp, a.d.ks[3], ring, w.first, w.n_sub, a.d.L, lane);
    ks.issue_first();
    uint32_t x = 0;
    for (int u = 0; u < w.n_sub; ++u) {
        if (READ_LDS) {
            bf16x8 kb[2][4];
            wait_loads(min(NBUF - 1, w.n_sub - 1 - u));
            read_subtile(ks.lane_addr0 + (u % NBUF) * BUF_BYTES, kb);
            have_subtile<false>(kb);
            if (u + NBUF < w.n_sub) ks.issue(u + NBUF);
#pragma unroll
            for (int s = 0; s < 8; ++s) x ^= ((const uint32_t *)&kb[s >> 2][s & 3])[0] ^ ((const uint32_t *)&kb[s >> 2][s & 3])[3];
        } else {
            wait_loads(min(NBUF - 1, w.n_sub - 1 - u));
            x ^= *reinterpret_cast<const volatile uint32_t *>(ring + (u % NBUF) * BUF_BYTES + lane * 4);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (u + NBUF < w.n_sub) ks.issue(u + NBUF);
        }
        if (STORES) {
            const int t = w.first + u * STRIDE + (lane & 31);
            float *out = ((lane >> 5) == 0 ? a.s_out : a.e_out) + (int64_t)w.p * a.d.L;
            if (t < a.d.L) out[t] = __uint_as_float(x & 0x3fffffffu);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (x == 0x5ab10c4bu) *sink = x;                           // keeps the reads alive; practically never taken
}

}  // namespace

bool stream_probe_supported(const Dims &d) { return d.dtype == SABLOCK_BF16 && d.D == 128; }

hipError_t launch_stream_probe(const Dims &d, const void *k, int read_lds, float *s_out, float *e_out, void *sink, hipStream_t st)
{
    static thread_local PerDeviceOnce attr_once;
    if (attr_once.needed()) {
#define X(R, S) { hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(stream_probe_kernel<R, S>), \
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, WAVES * RING_BYTES); \
                  if (e != hipSuccess) return e; }
        X(false, false) X(false, true) X(true, false) X(true, true)
#undef X
        attr_once.done();
    }
    const Plan pl = make_plan(d);
    ScoreArgs a = {};
    a.d = d;
    a.k = static_cast<const uint16_t *>(k);
    a.chunk_len = pl.chunk_len;
    a.n_chunks = pl.n_chunks;
    a.by_chunk = pl.by_chunk || d.local;
    a.s_out = s_out;
    a.e_out = e_out;
    const dim3 grid = a.by_chunk ? dim3(d.P, pl.n_chunks) : dim3(pl.n_chunks, d.P);
    uint32_t *sk = static_cast<uint32_t *>(sink);
    const bool stores = s_out != nullptr;
#define X(R, S) if ((read_lds != 0) == R && stores == S) hipLaunchKernelGGL((stream_probe_kernel<R, S>), grid, dim3(WAVES * 64), WAVES * RING_BYTES, st, a, sk);
    X(false, false) X(false, true) X(true, false) X(true, true)
#undef X
    return hipGetLastError();
}

// ---- head mean over all query heads of a layer (Eq. barA, literal): shapes with up to 128 window-query rows
bool score_all_heads_supported(const Dims &d)
{
    return d.dtype == SABLOCK_BF16 && d.D == 128 && tile_shape(d) && d.W <= 32;
}

// the shape whose layers one workgroup can sum in registers and LDS (score_mfma_columns_layer)
static bool layer_kernel_shape(const Dims &d) { return d.G == 4 && d.W == 32 && d.Hkv == LAYER_KV; }

size_t score_all_heads_ws_bytes(const Dims &d)
{
    const Plan pl = make_plan(d, MERGE_FROM_LAYER);
    const size_t abar = layer_kernel_shape(d) ? 0 : align256((size_t)d.P * d.L * d.W * 4);
    return partial_bytes(d, pl) + merged_bytes(d) + abar;
}

hipError_t launch_score_all_heads(const Dims &d, const void *q, const void *k, const float *row_lse, float eps,
                                  float *s_out, float *ent_out, void *ws, hipStream_t st)
{
    const Plan pl = make_plan(d, MERGE_FROM_LAYER);
    ScoreArgs a;
    a.d = d;
    a.q = static_cast<const uint16_t *>(q);
    a.k = static_cast<const uint16_t *>(k);
    plan_partials(a, d, pl, ws);
    a.c1 = (float)(1.4426950408889634 / sqrt((double)d.D));
    a.log2_G = (float)log2((double)d.G);
    a.eps = eps;
    a.lse = row_lse;
    a.abar = nullptr;
    const dim3 grid = a.by_chunk ? dim3(d.P, pl.n_chunks) : dim3(pl.n_chunks, d.P);
    if (layer_kernel_shape(d)) {
        static thread_local PerDeviceOnce attr_once;
        if (attr_once.needed()) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(score_mfma_stats<8, 32, 4>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, stats_lds<8>());
            if (e != hipSuccess) return e;
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(score_mfma_columns_layer),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, PL_LDS);
            if (e != hipSuccess) return e;
            attr_once.done();
        }
        a.s_out = s_out;
        a.e_out = ent_out;
        if (!row_lse) {
            hipLaunchKernelGGL((score_mfma_stats<8, 32, 4>), grid, dim3(WAVES * 64), stats_lds<8>(), st, a);
            launch_merge(a, d.P, M_ROWS, st);
        }
        // pass 2 has its own decomposition: a workgroup walks a chunk of keys through all 8 KV heads of a layer, one
        // workgroup per CU; its prologue takes as long as some 96 keys
        constexpr int MAX_LAYER_CHUNK = 32768, FIXED = 96;
        const int64_t n_sl = (int64_t)d.n_seq * d.n_layers;
        const ChunkPlan c = plan_chunks(n_sl, d.L, d.cus, SUB, FIXED, MAX_LAYER_CHUNK, INT32_MAX, 0, INT32_MAX, false);
        ScoreArgs a2 = a;
        a2.chunk_len = c.len;
        a2.n_chunks = c.n;
        hipLaunchKernelGGL(score_mfma_columns_layer, dim3(a2.n_chunks, (unsigned)n_sl), dim3(WAVES * 64), PL_LDS, st, a2);
        return hipGetLastError();
    }
    // other shapes: every KV head's head-group means go to memory, a second kernel averages them over the KV heads
    a.s_out = nullptr;
    a.e_out = nullptr;
    a.abar = reinterpret_cast<float *>(static_cast<char *>(ws) + partial_bytes(d, pl) + merged_bytes(d));
    hipError_t e = hipErrorInvalidValue;
    const int nt = tiles_of(d);
#define X(NTV, WV) if (nt == NTV && d.W == WV) e = launch_shape<NTV, WV, true>(a, grid, !row_lse, st);
    SABLOCK_SHAPES(X)
#undef X
    if (e != hipSuccess) return e;
    dim3 rgrid((unsigned)((d.L + 255) / 256), (unsigned)(d.n_seq * d.n_layers));
#define X(WV) if (d.W == WV) hipLaunchKernelGGL(abar_reduce_kernel<WV>, rgrid, dim3(256), 0, st, a.abar, d.Hkv, d.L, eps, s_out, ent_out);
    X(8) X(16) X(32)
#undef X
    return hipGetLastError();
}

}  // namespace sablock
