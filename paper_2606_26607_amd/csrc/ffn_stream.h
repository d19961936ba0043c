// Grouped SwiGLU expert FFN for few rows per expert (decode): both GEMMs
// stream the experts' weights past a handful of rows, and HBM is the bound.
//
// Every wave works alone: it holds a strip of 16 * NB weight rows (gated: half
// of them gate rows, half the matching up rows) against 16 * MB token rows and
// walks its run of K in 64-wide slices.  A slice's loads go to registers, one
// instruction per 8 rows x 128 bytes (whole lines: fragments loaded straight
// from memory, 16 rows x 64 bytes an instruction, reached 5.3 TB/s instead of
// 6.7, as every line was asked for twice), are turned into 16x16x32 MFMA
// fragments through a few KB of LDS that belong to the wave, and U slices of
// loads stay in flight: the register file holds more bytes in flight than the
// LDS rings of the tiled kernels, and no wave waits for another.  A
// workgroup is the waves that split one strip's K (their sums meet in LDS at
// the end) or two strips; workgroups are dealt by the hardware as others
// end, so launches need no tile schedule, no partial sums in memory and no
// even split.  An expert without rows ends its workgroups at once.
//
// Measured against the tiled kernels, in turn on one box (layer, replayed from
// a graph, us): DeepSeek-V3-shaped EP slice, 64 tokens 394 -> 369 (6.7 TB/s; on
// another box and in a longer graph 409 -> 404); Qwen3-shaped TP slice (128
// experts, I_s 192), 64 tokens 163 -> 108; Mixtral-shaped TP slice, 1 token 56 ->
// 29, 64 tokens 91 -> 72; the tiny replicated layer (which now also routes and
// permutes in one launch) 33 -> 16.
#pragma once
#include <type_traits>

#include "ffn_dev.h"

namespace moe {
namespace ffn_stream {

using namespace ffn_dev;

// Operands of one launch (row spaces and weight blocks as in the tiled
// kernels: the shared expert, index El, follows the routed ones).
struct StreamArgs {
    const uint16_t *A;          // activations: token matrix (with row_index) or permuted rows
    const int32_t *row_index;   // row -> pair index (divided by kdiv gives the token), or null
    int kdiv;
    int64_t a_rows;             // rows of A
    const int32_t *offsets;     // [El + 1] routed experts' row ranges
    int El;
    int cap, shared_rows, shared_begin;
    int N, K;                   // output columns (per part when gated), reduction length
    const uint16_t *W;          // [El] weight blocks of w_stride elements
    int64_t w_stride;
    const uint16_t *Wsh;        // the shared expert's
    int up_off;                 // first up row when gated
    uint16_t *C, *Csh;          // [cap, N] / [shared_rows, N] bf16 out
    int lks;                    // log2 of the waves that split K
};

typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));

constexpr int SK = 64;  // K per slice: one 128-byte line of every row

// 16-byte chunk c of LDS row r sits at c ^ swz(r): the 16 rows of a fragment
// read, and the 8 chunks of a row written, fall on distinct banks.
__device__ __forceinline__ int swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

// Buffer of `bytes` from p on (both uniform: pinned to scalar registers).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_rsrc(const uint16_t *p, int64_t bytes)
{
    const uint64_t b = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>((uint64_t)hi << 32 | lo), (short)0,
                                             __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
}

// Rows [row, row + n) of a weight block with rows of K values.  A part wholly
// past the block (n <= 0) gets the block's first row instead, whose products
// belong to columns that are not stored: a load's uniform offset along K is at
// most a row, so no range is shorter than it, whether the bounds check leaves
// that offset out or takes it off the range.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const uint16_t *W, int64_t row, int n, int K)
{
    return uniform_rsrc(n > 0 ? W + row * K : W, (int64_t)(n > 0 ? n : 1) * K * 2);
}

// 16 bytes of a buffer at this lane's byte offset plus a uniform one; past
// the buffer's end the load returns zeros and touches no memory.
template <bool NT>
__device__ __forceinline__ u32x4_t load16(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff)
{
    return __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, NT ? 2 : 0));
}

// One wave's stream: NB blocks of 16 weight rows against MB blocks of 16
// token rows.
template <int MB, int NB, int U, bool NT>
struct Stream {
    __amdgpu_buffer_rsrc_t w[2], x;  // the strip's two parts (NB / 2 blocks each); the activations
    uint32_t wo[NB], xo[2 * MB];     // this lane's byte offsets: its row of each weight block's first 8, of each 8 token rows
    uint32_t rowstep;                // bytes of 8 weight rows
    uint4 *lds;                      // (NB + MB) * 16 rows of 8 chunks
    f32x4_t acc[MB][NB];

    // A slice as loaded: lane l holds chunk l % 8 of row l / 8 of each 8 rows.
    struct Slice {
        u32x4_t w[2 * NB], x[2 * MB];
    };

    // (in = false: this lane's chunk lies past K and reads zeros; the offset
    // is past any buffer here)
    __device__ __forceinline__ void load(Slice &t, uint32_t so, bool in = true)
    {
#pragma unroll
        for (int i = 0; i < 2 * NB; ++i)
            t.w[i] = load16<NT>(w[i / NB], in ? wo[i >> 1] + (i & 1) * rowstep : 0xfffffff0u, so);
#pragma unroll
        for (int i = 0; i < 2 * MB; ++i) t.x[i] = load16<false>(x, in ? xo[i] : 0xfffffff0u, so);
    }

    // The slice through LDS into fragments (lane l: row l % 16, chunk 4 * kk +
    // l / 16) and its MFMAs: weights first, so a lane ends up with four
    // consecutive output columns of one token.  LDS keeps a wave's accesses in
    // order, so the next slice's writes need no wait.
    __device__ __forceinline__ void mul(const Slice &t)
    {
        const int lane = threadIdx.x & 63, wr = lane >> 3, wq = lane & 7, r = lane & 15, c = lane >> 4;
#pragma unroll
        for (int i = 0; i < 2 * (NB + MB); ++i) {
            const u32x4_t v = i < 2 * NB ? t.w[i] : t.x[i - 2 * NB];
            lds[(i * 8 + wr) * 8 + (wq ^ wr ^ (i & 1))] = make_uint4(v.x, v.y, v.z, v.w);
        }
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            bf16x8_t b[NB], a[MB];
            const int pos = (kk * 4 + c) ^ swz(r);
#pragma unroll
            for (int j = 0; j < NB; ++j) b[j] = __builtin_bit_cast(bf16x8_t, lds[(j * 16 + r) * 8 + pos]);
#pragma unroll
            for (int m = 0; m < MB; ++m) a[m] = __builtin_bit_cast(bf16x8_t, lds[((NB + m) * 16 + r) * 8 + pos]);
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    acc[m][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[m], acc[m][j], 0, 0, 0);
        }
    }

    // n (>= 1) slices from byte s0 of every row on, U slices of loads in
    // flight.  (The scheduling barriers keep each slice's loads behind the
    // MFMAs that free its registers: moved up, they spill.)
    __device__ __forceinline__ void run(uint32_t s0, int n)
    {
        Slice t[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            load(t[u], s0 + (u < n ? u : n - 1) * (SK * 2));
            __builtin_amdgcn_sched_barrier(0);
        }
        for (; n >= 2 * U; n -= U) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                mul(t[u]);
                __builtin_amdgcn_sched_barrier(0);
                load(t[u], s0 + (U + u) * (SK * 2));
                __builtin_amdgcn_sched_barrier(0);
            }
            s0 += U * SK * 2;
        }
        if (n > U) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                mul(t[u]);
                __builtin_amdgcn_sched_barrier(0);
                load(t[u], s0 + (U + u < n ? U + u : n - 1) * (SK * 2));
                __builtin_amdgcn_sched_barrier(0);
            }
            n -= U;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (u < n) mul(t[u]);
    }
};

// Token rows [m0, m0 + 16 * MB) of expert e's [r0, r1) against the strip of
// output columns from n0 on, over the wave's nsl whole slices from k0 on (and
// the partial last one, k_tail).  PER: 16-byte chunks of LDS per wave, the
// same for every MB of a launch (waves of a workgroup may be at different
// rows).
template <bool GATED, bool NT, int MB, int NB, int U, int PER>
__device__ __forceinline__ void strip_rows(const StreamArgs &g, int e, int r0, int r1, int m0, int n0, int k0,
                                           int nsl, bool k_tail, uint4 *lds)
{
    constexpr int OUTC = GATED ? 8 * NB : 16 * NB;  // output columns of the strip
    const int lane = threadIdx.x & 63, r = lane & 15, c = lane >> 4, wr = lane >> 3, wq = lane & 7;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int K = g.K, N = g.N;
    Stream<MB, NB, U, NT> st;
    st.lds = lds + wave * PER;
#pragma unroll
    for (int i = 0; i < 2 * MB; ++i) {
        int row = r0 + m0 + i * 8 + wr;
        row = row < r1 ? row : r1 - 1;
        uint32_t t = (uint32_t)row;
        if (g.row_index != nullptr)
            t = e < g.El ? (uint32_t)g.row_index[row] / (uint32_t)g.kdiv : (uint32_t)(g.shared_begin + row - g.cap);
        st.xo[i] = (t * (uint32_t)K + wq * 8) * 2;
    }
    // the strip's weight rows: NB/2 blocks of gate rows and the matching up
    // rows, or NB blocks of rows; rows past N read zeros (or the block's first
    // row) and are not stored
    const uint16_t *We = e < g.El ? g.W + (int64_t)e * g.w_stride : g.Wsh;
    const int v0 = N - n0 < NB * 8 ? N - n0 : NB * 8, n1 = GATED ? n0 : n0 + NB * 8, v1 = N - n1 < NB * 8 ? N - n1 : NB * 8;
    st.w[0] = rows_rsrc(We, n0, v0, K);
    st.w[1] = rows_rsrc(We, (GATED ? g.up_off : 0) + n1, v1, K);
    st.x = uniform_rsrc(g.A, g.a_rows * K * 2);
    st.rowstep = 8 * (uint32_t)K * 2;
#pragma unroll
    for (int j = 0; j < NB; ++j) st.wo[j] = (((j % (NB / 2)) * 16 + wr) * (uint32_t)K + wq * 8) * 2;
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int j = 0; j < NB; ++j) st.acc[m][j] = f32x4_t{};
    if (nsl > 0) st.run(k0 * 2, nsl);
    if (k_tail) {
        // the last, partial slice of K: chunks past K read zeros
        typename Stream<MB, NB, U, NT>::Slice t;
        st.load(t, (k0 + nsl * SK) * 2, k0 + nsl * SK + wq * 8 < K);
        st.mul(t);
    }
    const int ks = 1 << g.lks, kw = wave & (ks - 1);
    if (ks > 1) {
        // sums of the waves that split K, in their order (each wave's sums
        // take the place of its slices)
        __syncthreads();
        f32x4_t *buf = reinterpret_cast<f32x4_t *>(lds);
        static_assert(MB * NB * 64 <= PER, "the sums fit where the slices were");
        if (kw > 0) {
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int j = 0; j < NB; ++j) buf[wave * PER + (m * NB + j) * 64 + lane] = st.acc[m][j];
        }
        __syncthreads();
        if (kw == 0) {
            for (int q = 1; q < ks; ++q)
#pragma unroll
                for (int m = 0; m < MB; ++m)
#pragma unroll
                    for (int j = 0; j < NB; ++j) st.acc[m][j] += buf[(wave + q) * PER + (m * NB + j) * 64 + lane];
        }
        __syncthreads();
        if (kw > 0) return;
    }
    uint16_t *Cb = e < g.El ? g.C + (int64_t)r0 * N : g.Csh + (int64_t)(r0 - g.cap) * N;
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        const int row = m0 + m * 16 + r;
        if (row >= r1 - r0) continue;
#pragma unroll
        for (int j = 0; j < OUTC / 16; ++j) {
            const int col = n0 + 16 * j + 4 * c;
            float o[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                o[i] = GATED ? silu_mul(st.acc[m][j][i], st.acc[m][j + (GATED ? NB / 2 : 0)][i]) : st.acc[m][j][i];
            uint2 v;
            v.x = bf16_bits(o[0]) | (uint32_t)bf16_bits(o[1]) << 16;
            v.y = bf16_bits(o[2]) | (uint32_t)bf16_bits(o[3]) << 16;
            if (col < N) *reinterpret_cast<uint2 *>(Cb + (int64_t)row * N + col) = v;
        }
    }
}

// Device-side timestamps of a launch (null: off): per die, its earliest
// workgroup start and latest end.
struct LaunchStamps {
    unsigned long long *start, *end;
    int64_t stride;
};

// Die of this workgroup: the hardware deals them to the 8 dies round robin.
__device__ __forceinline__ int die()
{
    return (int)(((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x) & 7);
}

// Grid: x over the strips of output columns, y over the experts.  MBMAX: row
// blocks of a pass at most; an expert of more rows takes more passes (its
// weights then come from the caches).
template <bool GATED, bool NT, int MBMAX, int NB, int MINW>
__global__ __attribute__((amdgpu_flat_work_group_size(64, 512), amdgpu_waves_per_eu(MINW)))
void stream_kernel(StreamArgs g, LaunchStamps ts)
{
    extern __shared__ uint4 lds[];
    constexpr int OUTC = GATED ? 8 * NB : 16 * NB;
    const int e = blockIdx.y;
    const int r0 = __builtin_amdgcn_readfirstlane((int)expert_begin(g.offsets, g.El, g.cap, e));
    const int r1 = __builtin_amdgcn_readfirstlane((int)expert_end(g.offsets, g.El, g.cap, g.shared_rows, e));
    if (r1 - r0 <= (int)blockIdx.z * MBMAX * 16) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), ks = 1 << g.lks, kw = wave & (ks - 1);
    const int n0 = ((blockIdx.x * (blockDim.x >> 6) + wave) >> g.lks) * OUTC;
    if (g.lks == 0 && n0 >= g.N) return;
    // this wave's run of whole slices of K, and the partial last one on the
    // last wave
    const int full = g.K / SK, per = (full + ks - 1) >> g.lks;
    const int s0 = kw * per < full ? kw * per : full, s1 = s0 + per < full ? s0 + per : full;
    const bool k_tail = (g.K % SK) && kw == ks - 1;
    const int k0 = s0 * SK, ns = s1 - s0;
    if (ts.start != nullptr && threadIdx.x == 0) atomicMin(ts.start + die() * ts.stride, __builtin_amdgcn_s_memrealtime());
    constexpr int PER = (NB + MBMAX) * 16 * 8;  // 16-byte chunks of LDS per wave
    const int rows = r1 - r0;
    for (int m0 = blockIdx.z * MBMAX * 16; m0 < rows; m0 += gridDim.z * MBMAX * 16) {
        const int left = rows - m0;
        if (MBMAX == 1 || left <= 16) strip_rows<GATED, NT, 1, NB, NB == 4 ? 2 : 3, PER>(g, e, r0, r1, m0, n0, k0, ns, k_tail, lds);
        else if (MBMAX == 2 || left <= 32) strip_rows<GATED, NT, 2, NB, NB == 4 ? 2 : 3, PER>(g, e, r0, r1, m0, n0, k0, ns, k_tail, lds);
        else if constexpr (MBMAX >= 4) strip_rows<GATED, NT, 4, NB, 2, PER>(g, e, r0, r1, m0, n0, k0, ns, k_tail, lds);
    }
    if (ts.start != nullptr && threadIdx.x == 0) atomicMax(ts.end + die() * ts.stride, __builtin_amdgcn_s_memrealtime());
}

// ---------------------------------------------------------------------------
// The same stream for more rows per expert: a workgroup of four waves takes
// 16 * MB token rows (up to 128) against 64 * NB weight rows, 16 * NB of them
// a wave's own.  The weights move as above, each wave's slice through its own
// LDS; the activations' slice is loaded once by the four waves together (a
// quarter each) and shared through two LDS buffers, so a barrier per slice
// hands it over.
// ---------------------------------------------------------------------------
constexpr int MID_WAVES = 4;

template <bool GATED, bool NT, int MB, int NB, int U>
__device__ __forceinline__ void mid_rows(const StreamArgs &g, int e, int r0, int r1, int m0, int n0, uint4 *lds, int abuf,
                                         int bofs)
{
    constexpr int NX = MB / 2;                      // this wave's activation instructions per slice (8 rows each)
    constexpr int OUTC = GATED ? 8 * NB : 16 * NB;  // output columns of the wave
    static_assert(MB % 2 == 0, "a quarter of the rows in whole instructions");
    const int lane = threadIdx.x & 63, r = lane & 15, c = lane >> 4, wr = lane >> 3, wq = lane & 7;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int K = g.K, N = g.N;
    uint32_t xo[NX], wo[NB];
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        int row = r0 + m0 + (wave * NX + i) * 8 + wr;
        row = row < r1 ? row : r1 - 1;
        uint32_t t = (uint32_t)row;
        if (g.row_index != nullptr)
            t = e < g.El ? (uint32_t)g.row_index[row] / (uint32_t)g.kdiv : (uint32_t)(g.shared_begin + row - g.cap);
        xo[i] = (t * (uint32_t)K + wq * 8) * 2;
    }
    const uint16_t *We = e < g.El ? g.W + (int64_t)e * g.w_stride : g.Wsh;
    const int v0 = N - n0 < NB * 8 ? N - n0 : NB * 8, n1 = GATED ? n0 : n0 + NB * 8, v1 = N - n1 < NB * 8 ? N - n1 : NB * 8;
    const __amdgpu_buffer_rsrc_t w0 = rows_rsrc(We, n0, v0, K);
    const __amdgpu_buffer_rsrc_t w1 = rows_rsrc(We, (GATED ? g.up_off : 0) + n1, v1, K);
    const __amdgpu_buffer_rsrc_t xr = uniform_rsrc(g.A, g.a_rows * K * 2);
    const uint32_t rowstep = 8 * (uint32_t)K * 2;
#pragma unroll
    for (int j = 0; j < NB; ++j) wo[j] = (((j % (NB / 2)) * 16 + wr) * (uint32_t)K + wq * 8) * 2;
    f32x4_t acc[MB][NB];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[m][j] = f32x4_t{};

    uint4 *const bl = lds + bofs + wave * (NB * 16 * 8);
    struct Slice {
        u32x4_t w[2 * NB], x[NX];
    };
    Slice t[U];
    const int full = K / SK, ns = (K + SK - 1) / SK;  // whole slices, all slices
    auto load = [&](Slice &v, int s) {
        const uint32_t so = s * (SK * 2);
        // (a last slice partly past K: chunks past K read zeros)
        const bool in = s < full || s * SK + wq * 8 < K;
#pragma unroll
        for (int i = 0; i < 2 * NB; ++i)
            v.w[i] = load16<NT>(i < NB ? w0 : w1, in ? wo[i >> 1] + (i & 1) * rowstep : 0xfffffff0u, so);
#pragma unroll
        for (int i = 0; i < NX; ++i) v.x[i] = load16<false>(xr, in ? xo[i] : 0xfffffff0u, so);
    };
    auto mul = [&](const Slice &v, int s, auto more, int snext, Slice &nxt) {
        uint4 *const al = lds + (s & 1) * abuf;
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int row8 = wave * NX + i;
            al[(row8 * 8 + wr) * 8 + (wq ^ wr ^ (row8 & 1))] = __builtin_bit_cast(uint4, v.x[i]);
        }
#pragma unroll
        for (int i = 0; i < 2 * NB; ++i) bl[(i * 8 + wr) * 8 + (wq ^ wr ^ (i & 1))] = __builtin_bit_cast(uint4, v.w[i]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(more)::value) load(nxt, snext);
        __builtin_amdgcn_sched_barrier(0);
        // every wave's rows of the slice are in LDS; the other buffer's were
        // read before this wave came here
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        // step i multiplies token block i % MB of k-step i / MB; its fragment
        // is read D steps ahead (the LDS latency under D steps' MFMAs)
        constexpr int D = MB < 4 ? MB : 4, STEPS = 2 * MB;
        bf16x8_t b[2][NB], a[D];
        const int p0 = c ^ swz(r);
        auto read_b = [&](int kk) {
#pragma unroll
            for (int j = 0; j < NB; ++j) b[kk][j] = __builtin_bit_cast(bf16x8_t, bl[(j * 16 + r) * 8 + (p0 ^ (kk * 4))]);
        };
        auto read_a = [&](int i) {
            a[i % D] = __builtin_bit_cast(bf16x8_t, al[((i % MB) * 16 + r) * 8 + (p0 ^ ((i / MB) * 4))]);
        };
        read_b(0);
#pragma unroll
        for (int i = 0; i < D; ++i) read_a(i);
        read_b(1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
#pragma unroll
            for (int j = 0; j < NB; ++j)
                acc[i % MB][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[i / MB][j], a[i % D], acc[i % MB][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (i + D < STEPS) read_a(i + D);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using T_ = std::true_type;
    using F_ = std::false_type;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        load(t[u], u < ns ? u : ns - 1);
        __builtin_amdgcn_sched_barrier(0);
    }
    int s = 0;
    for (; s + 2 * U <= ns; s += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) mul(t[u], s + u, T_{}, s + U + u, t[u]);
    }
    if (s + U < ns) {
#pragma unroll
        for (int u = 0; u < U; ++u) mul(t[u], s + u, T_{}, s + U + u < ns ? s + U + u : ns - 1, t[u]);
        s += U;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (s + u < ns) mul(t[u], s + u, F_{}, 0, t[u]);

    uint16_t *Cb = e < g.El ? g.C + (int64_t)r0 * N : g.Csh + (int64_t)(r0 - g.cap) * N;
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        const int row = m0 + m * 16 + r;
        if (row >= r1 - r0) continue;
#pragma unroll
        for (int j = 0; j < OUTC / 16; ++j) {
            const int col = n0 + 16 * j + 4 * c;
            float o[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                o[i] = GATED ? silu_mul(acc[m][j][i], acc[m][j + (GATED ? NB / 2 : 0)][i]) : acc[m][j][i];
            uint2 v;
            v.x = bf16_bits(o[0]) | (uint32_t)bf16_bits(o[1]) << 16;
            v.y = bf16_bits(o[2]) | (uint32_t)bf16_bits(o[3]) << 16;
            if (col < N) *reinterpret_cast<uint2 *>(Cb + (int64_t)row * N + col) = v;
        }
    }
    // the next rows' first slice may not overtake a wave still reading these
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Grid: x over the strips of output columns, y over the experts, z over their
// runs of 16 * MBMAX rows, in the slowest dimension: with an expert's runs
// next to each other the workgroups past its rows, which end at once, left
// whole shader engines with nothing else (120 -> 200 us and more).  Two
// workgroups a CU: four weight blocks a wave, three workgroups a CU, a second
// set of buffers or the next slice staged between the MFMAs spill.
// Measured (layer, replayed from a graph, us; the kernels before): 8 slices of
// H 4096, I 1792, 400 tokens of a top-2 layer 147 -> 101 (tiled), 128 of H 2048, I
// 96, 2051 tokens top-8 192 -> 123 (general).  In the latter the gate-up (43 us)
// keeps the LDS busy for 48% of the cycles in which its CUs have work, a third
// of that conflicts, and the matrix cores for 16% of all; its waves wait 29%,
// two thirds of it for LDS; 191 MB come from memory (4.5 TB/s: the weights
// once, 100 MB, and the activations into each die's L2).  No one rate is the
// bound: the chain of a slice (registers to LDS, barrier, fragments, MFMAs) at
// two waves a SIMD is, with that traffic.  The down projection (52 us) has two
// slices a tile and moves 3.2 TB/s: prologue, epilogue and stores.
template <bool GATED, bool NT>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * MID_WAVES, 64 * MID_WAVES), amdgpu_waves_per_eu(2)))
void mid_kernel(StreamArgs g, LaunchStamps ts)
{
    constexpr int MBMAX = 8, NB = 2, U = 3;
    constexpr int ABUF = MBMAX * 16 * 8, BOFS = 2 * ABUF;
    __shared__ uint4 lds[BOFS + MID_WAVES * NB * 16 * 8];
    constexpr int OUTC = GATED ? 8 * NB : 16 * NB;
    const int e = blockIdx.y;
    const int r0 = __builtin_amdgcn_readfirstlane((int)expert_begin(g.offsets, g.El, g.cap, e));
    const int r1 = __builtin_amdgcn_readfirstlane((int)expert_end(g.offsets, g.El, g.cap, g.shared_rows, e));
    const int rows = r1 - r0;
    if (rows <= (int)blockIdx.z * MBMAX * 16) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = (blockIdx.x * MID_WAVES + wave) * OUTC;
    if (ts.start != nullptr && threadIdx.x == 0) atomicMin(ts.start + die() * ts.stride, __builtin_amdgcn_s_memrealtime());
    for (int m0 = blockIdx.z * MBMAX * 16; m0 < rows; m0 += gridDim.z * MBMAX * 16) {
        const int left = rows - m0;
        if (left <= 32) mid_rows<GATED, NT, 2, NB, U>(g, e, r0, r1, m0, n0, lds, ABUF, BOFS);
        else if (left <= 64) mid_rows<GATED, NT, 4, NB, U>(g, e, r0, r1, m0, n0, lds, ABUF, BOFS);
        else mid_rows<GATED, NT, 8, NB, U>(g, e, r0, r1, m0, n0, lds, ABUF, BOFS);
    }
    if (ts.start != nullptr && threadIdx.x == 0) atomicMax(ts.end + die() * ts.stride, __builtin_amdgcn_s_memrealtime());
}

}  // namespace ffn_stream
}  // namespace moe
