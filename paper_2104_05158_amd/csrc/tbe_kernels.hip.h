// Device kernels of the table-batched embedding-bag library for gfx950 (CDNA4, wave64).
//
// Forward: Section 2 "Embedding operators" + Section 5.1 (all tables in one launch).
// Backward: Section 5.1 (gradient sorting by rows, on-chip aggregation, fused optimizer) and
// Section 5.2 (row-wise AdaGrad) of arxiv 2104.05158.
//
// Everything on this path is a gather / scan / sort bound by HBM bandwidth: no MFMA.  The lane
// mapping is the same everywhere: a row of D elements is covered by LPR = pow2ceil(D / EPL) lanes
// (EPL contiguous elements per lane, vector loads), and the 64 / LPR lane groups of a wavefront
// fetch different rows at the same time; sums across groups and across a row use xor-shuffles.
#pragma once

#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <type_traits>

#include "tbe_rules.h"

namespace tbe {

// ---- geometry constants shared by host and device (those of the launch rules are in tbe_rules.h) ----
constexpr int kFwdUnroll = 4;             // row loads in flight per lane group (8 costs occupancy and is slower)
constexpr int kChunk = 128;               // sorted positions per pair of partial-row slots
constexpr int kSpanUnit = 16;             // a span of the update kernel is a multiple of this many sorted positions
constexpr int kWinMax = 16;               // most bag windows a long run is cut into
constexpr int kWinBatch = 8;               // pieces a workgroup of window_runs_kernel claims at a time
constexpr int kBwdThreads = 256;          // 4 wavefronts = 4 chunks per workgroup
constexpr int kBwdUnroll = 4;             // gradient rows in flight per lane group (long runs)
constexpr int kShortRun = 4;              // runs up to this length are handled one per lane group
constexpr int kMaxDim = 512;
// dense hot rows: runs longer than the call's dense threshold are summed as (count matrix) x (gradient block)
constexpr int kDenseRows = 32;            // most runs per group: they share one pass over the table's gradient block
constexpr int kDenseSlice = 1024;         // bags per work unit = per count table in LDS = per partial row of a dense run
constexpr int kDenseThreads = 256;
constexpr int kDenseMinRun = 1024;        // no run of this length or less is ever treated as dense (> kLongRun)
constexpr int kZeroRowBytes = 4096;        // a row of zeros in the workspace (largest row: 512 x fp32 = 2 KiB)

struct TableMeta {      // 32 bytes, one per table, in the workspace head
    int64_t woff;       // first element of the table in the flat weight array
    uint32_t rbase;     // linear id of the table's row 0
    int32_t dim;        // D_t
    int32_t col;        // first output column
    uint32_t rows;
    uint32_t lanes;     // log2 lanes per row: forward (EPL elements per lane), 256 x backward (2 x 4 floats per lane)
    int32_t key_bits;   // ceil(log2 rows) (at least 1): the bits of the table's row index that the sort orders

    __host__ __device__ int lpr_fwd() const { return (int)(lanes & 0xffu); }
    __host__ __device__ int lpr_bwd() const { return (int)(lanes >> 8); }
};

struct Counters {       // workspace scalars
    int64_t num_unique;         // written by the run-length pass of every sort
    // Long runs (and, when they are cut by position, their pieces) queued by the update kernel.  Zero between
    // updates, also before a second update after one sort and every replay of a captured graph: the window kernel
    // hands the number of runs over to the fix-up kernel (long_todo) and clears it, the fix-up kernel clears the
    // number of pieces.  Each is cleared by one workgroup of a kernel in which no other reads it.
    uint32_t long_count;        // (these two are added to together, as one word of 64 bits)
    uint32_t win_pieces;
    uint32_t long_todo;
    uint32_t check_flags;       // written only by tbe_check_inputs
    uint32_t dense_runs;        // written by the plan kernels: dense runs / groups, windowed runs of this update
    uint32_t dense_groups;
    uint32_t win_runs;          // windowed runs of this update (window_plan_kernel writes win_pieces, too)
    int32_t sort_chunks;        // written by sort_plan_kernel, which clears sort_units and sort_ticket: chunks of the partition,
    int32_t sort_multi;         // tables of more chunks than sort_units_kernel adds up itself
    uint32_t sort_units;
    uint32_t pad1[20];          // (the claim counters below start a 128-byte line of their own)
    uint32_t sort_ticket;       // next unit of sort_local_kernel
    uint32_t pad2[31];
    // window_runs_kernel: next unclaimed piece of each L2 domain, one counter per 128-byte line
    // (cleared by the kernel's plan kernel)
    uint32_t win_next[8][32];
};

// ---------------------------------------------------------------- small helpers

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// a + (lower, upper half of v), halves in fp16, as one mixed-precision FMA: x * 1 + a is exactly a + x.  (Written as
// fmaf(float(h), 1, a) the multiplication is dropped first, and what is left takes a conversion and an addition.)
__device__ __forceinline__ float acc_lo(float a, uint32_t v)
{
    asm("v_fma_mix_f32 %0, %1, 1.0, %0 op_sel_hi:[1,0,0]" : "+v"(a) : "v"(v));
    return a;
}
__device__ __forceinline__ float acc_hi(float a, uint32_t v)
{
    asm("v_fma_mix_f32 %0, %1, 1.0, %0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(a) : "v"(v));
    return a;
}

// Row access in the storage type: Vec is the raw vector one lane loads (EPL elements); `add`
// converts to fp32 and accumulates.  Loads are kept raw until they are consumed so that many can
// be in flight with few registers.
template <typename WT, int EPL>
struct RowIO;

template <>
struct RowIO<float, 4> {
    using Vec = float4;
    __device__ static __forceinline__ Vec ldv(const float* p) { return *reinterpret_cast<const float4*>(p); }
    __device__ static __forceinline__ void add(float (&a)[4], const Vec v)
    {
        a[0] += v.x; a[1] += v.y; a[2] += v.z; a[3] += v.w;
    }
    __device__ static __forceinline__ void unpack(const Vec v, float (&f)[4])
    {
        f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
    }
    __device__ static __forceinline__ void store(float* p, const float (&f)[4])
    {
        *reinterpret_cast<float4*>(p) = make_float4(f[0], f[1], f[2], f[3]);
    }
};

template <>
struct RowIO<__half, 4> {
    using Vec = uint2;
    __device__ static __forceinline__ Vec ldv(const __half* p) { return *reinterpret_cast<const uint2*>(p); }
    __device__ static __forceinline__ void unpack(Vec v, float (&f)[4])
    {
        const float2 a = __half22float2(*reinterpret_cast<__half2*>(&v.x));
        const float2 b = __half22float2(*reinterpret_cast<__half2*>(&v.y));
        f[0] = a.x; f[1] = a.y; f[2] = b.x; f[3] = b.y;
    }
    __device__ static __forceinline__ void add(float (&a)[4], Vec v)
    {
        a[0] = acc_lo(a[0], v.x); a[1] = acc_hi(a[1], v.x);
        a[2] = acc_lo(a[2], v.y); a[3] = acc_hi(a[3], v.y);
    }
    __device__ static __forceinline__ void store(__half* p, const float (&f)[4])
    {
        uint2 v;
        *reinterpret_cast<__half2*>(&v.x) = __floats2half2_rn(f[0], f[1]);
        *reinterpret_cast<__half2*>(&v.y) = __floats2half2_rn(f[2], f[3]);
        *reinterpret_cast<uint2*>(p) = v;
    }
};

template <>
struct RowIO<__half, 8> {
    using Vec = uint4;
    __device__ static __forceinline__ Vec ldv(const __half* p) { return *reinterpret_cast<const uint4*>(p); }
    __device__ static __forceinline__ void add(float (&a)[8], Vec v)
    {
        a[0] = acc_lo(a[0], v.x); a[1] = acc_hi(a[1], v.x);
        a[2] = acc_lo(a[2], v.y); a[3] = acc_hi(a[3], v.y);
        a[4] = acc_lo(a[4], v.z); a[5] = acc_hi(a[5], v.z);
        a[6] = acc_lo(a[6], v.w); a[7] = acc_hi(a[7], v.w);
    }
};

// Rows of a table of at most kBufferBytes by 32-bit byte offsets from its first element: a load from kNoRow (or from
// a column of it) on reads nothing and gives zeros.
constexpr uint32_t kNoRow = 0xffff0000u;
constexpr uint64_t kBufferBytes = kNoRow;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_buffer(const void* table, uint64_t bytes)
{
    constexpr int kDataFormat32 = 4 << 15;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(table), 0, (int)(uint32_t)bytes, kDataFormat32);
}

template <typename Vec>
__device__ __forceinline__ Vec load_buffer(__amdgpu_buffer_rsrc_t table, uint32_t offset)
{
    if constexpr (sizeof(Vec) == 16)
        return __builtin_bit_cast(Vec, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(table, offset, 0, 0));
    else
        return __builtin_bit_cast(Vec, (u32x2)__builtin_amdgcn_raw_buffer_load_b64(table, offset, 0, 0));
}

// ---------------------------------------------------------------- read-rate probe
//
// Streams n16 16-byte words through the chip `passes` times and discards them: the denominator for the
// gather kernels (what plain coalesced reads reach on the machine at hand, from HBM or, for a buffer that fits
// the memory-side cache, from there).  Four loads in flight per thread; an opaque copy of the pointer per pass
// keeps the passes from being merged; the sink is written only for one xor value in 2^32 (a vector store).
__global__ __launch_bounds__(256) void probe_read_kernel(const uint4* p, size_t n16, int passes, uint32_t* sink)
{
    uint32_t acc = 0;
    const size_t stride = (size_t)gridDim.x * 256;
    for (int ps = 0; ps < passes; ++ps) {
        // every pass gives a workgroup another part of the buffer (and another L2): a buffer larger than the
        // L2s is read from the level behind them in every pass, not from the workgroup's own lines
        const unsigned vb = (blockIdx.x + (unsigned)ps * 2731u) % gridDim.x;
        size_t i = (size_t)vb * 256 + threadIdx.x;
        for (; i + 3 * stride < n16; i += 4 * stride) {
            const uint4 a = p[i], b = p[i + stride], c = p[i + 2 * stride], d = p[i + 3 * stride];
            acc ^= a.x ^ a.y ^ a.z ^ a.w ^ b.x ^ b.y ^ b.z ^ b.w ^ c.x ^ c.y ^ c.z ^ c.w ^ d.x ^ d.y ^ d.z ^ d.w;
        }
        for (; i < n16; i += stride) {
            const uint4 a = p[i];
            acc ^= a.x ^ a.y ^ a.z ^ a.w;
        }
        asm volatile("" : "+s"(p)::"memory");      // the next pass reads through a pointer the compiler cannot relate to this one
    }
    if (acc == 0x9e3779b9u)
        *sink = acc;
}

// ---------------------------------------------------------------- forward (Section 2, Section 5.1)
//
// One launch for all tables.  A wavefront takes a block of consecutive bags (bag id = t*B + b) and
// reads their offsets with one coalesced load.  The bags are pooled G at a time, one bag per lane
// group (LPR = pow2ceil(D/EPL) lanes x EPL-element vector loads cover a row): every group streams
// its own bag's rows with kFwdUnroll row loads in flight, accumulates in fp32 registers and writes
// its D_t pooled values with one coalesced store -- no cross-group reduction is needed.  Bags of one
// batch always belong to one table, so the lane mapping is uniform inside a batch.
//
// The inner loop is branch-free so that all loads of a step are issued back to back: slots past the
// end of a bag load from kNoRow, in a table too tall for 32-bit offsets a row of zeros kept in the workspace;
// column offsets past D are clamped (those lanes never store), and the indices of the next step are requested
// before the rows of the current step are consumed.
//
// Bound by L2 trips in flight.  A probe that gathers 256-byte rows, 62 % of them from 2 MiB (what the L2s find of a
// Zipf batch) and the rest from 1 GiB, reaches 13.7 TB/s whatever the rows in flight; 196 M lookups of 64 and 128
// fp16 columns take 2.83 ms, 12.9 TB/s.  Offsets formed once a lookup by one lane and mixed FMAs left 9 vector
// instructions a row of 27, which is 1 % there, 6 % where bags are short (64 tables, 3 lookups: 109 -> 103 us) and
// 11 % in calls of few bags (24,000 of 20 lookups, 128 fp16 columns: 16.1 -> 14.3 us).
// 4 pooled values in the output type OT (float, or __half rounded to nearest even)
__device__ __forceinline__ void store_out4(float* p, float a, float b, float c, float d)
{
    *reinterpret_cast<float4*>(p) = make_float4(a, b, c, d);
}
__device__ __forceinline__ void store_out4(__half* p, float a, float b, float c, float d)
{
    uint2 v;
    *reinterpret_cast<__half2*>(&v.x) = __floats2half2_rn(a, b);
    *reinterpret_cast<__half2*>(&v.y) = __floats2half2_rn(c, d);
    *reinterpret_cast<uint2*>(p) = v;
}

template <typename WT, int EPL, int KMAX, typename OT>
__global__ __launch_bounds__(kFwdThreads) void forward_kernel(
    const TableMeta* __restrict__ meta, const WT* __restrict__ weights,
    const int32_t* __restrict__ indices, const int64_t* __restrict__ offsets,
    OT* __restrict__ out, const void* __restrict__ zero_row, int32_t B, int32_t num_bags,
    int32_t sumD, int32_t n_total, int32_t bags_per_wave, int32_t table_major)
{
    using IO = RowIO<WT, EPL>;
    using Vec = typename IO::Vec;
    constexpr int kWaves = kFwdThreads / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = threadIdx.x >> 6;
    const int j0 = uniform((blockIdx.x * kWaves + wv) * bags_per_wave);
    if (j0 >= num_bags)
        return;
    const int nbags = min(bags_per_wave, num_bags - j0);  // <= 63

    const int my_o = (int)offsets[j0 + min(lane, nbags)];
    const uint32_t last = (uint32_t)(n_total - 1);
    const WT* __restrict__ zrow = static_cast<const WT*>(zero_row);

    int r = 0;
    while (r < nbags) {
        const int j = j0 + r;
        const int t = j / B;
        const TableMeta m = meta[t];
        const int D = m.dim;
        const int lprl = m.lpr_fwd();
        const int LPR = 1 << lprl;
        const int G = kWave >> lprl;
        const int sub = lane & (LPR - 1);
        const int grp = lane >> lprl;
        const int same_table = (t + 1) * B - j;  // bags from j on that still belong to table t
        const int nb = min(G, min(nbags - r, same_table));
        const bool active = grp < nb;
        const int rr = active ? r + grp : r;
        // both shuffles run with every lane enabled: a bpermute cannot read a disabled lane
        const int start = __shfl(my_o, rr);
        const int next = __shfl(my_o, rr + 1);
        const int len = active ? next - start : 0;
        const WT* __restrict__ wbase = weights + m.woff;

        int eoff[KMAX];
        bool evalid[KMAX];
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            const int e0 = (sub + k * LPR) * EPL;
            evalid[k] = e0 < D;
            eoff[k] = min(e0, D - EPL);
        }
        // fp32 tables: one accumulator per load slot, added pairwise at the end -- the rounding error of a
        // long bag grows with the number of terms each accumulator sees.  (Sums of fp16 values in fp32 are
        // exact for thousands of terms: one accumulator.)
        static_assert(kFwdUnroll == 4, "the four accumulators of an fp32 table are added pairwise below");
        constexpr int NACC = sizeof(WT) == 4 ? kFwdUnroll : 1;
        float accs[NACC][KMAX][EPL];
#pragma unroll
        for (int q = 0; q < NACC; ++q)
#pragma unroll
            for (int k = 0; k < KMAX; ++k)
#pragma unroll
                for (int e = 0; e < EPL; ++e)
                    accs[q][k][e] = 0.f;

        if (__ballot(len > 0) != 0ull && LPR >= kFwdUnroll) {
            // The address unit spends as long on a 4-byte load as on a 16-byte one, so the indices are not
            // loaded once per row: the LPR lanes of a group load the bag's next LPR indices with ONE
            // instruction (lane `sub` the sub-th of them) a block ahead of their use, and every row load
            // takes its index, or its row's offset, from the group's lanes by a shuffle.
            const int gbase = lane & ~(LPR - 1);
            int nxt = indices[min((uint32_t)(start + sub), last)];
            const uint64_t table_bytes = (uint64_t)m.rows * (uint32_t)D * sizeof(WT);
            Vec raw[kFwdUnroll][KMAX];
            auto add_rows = [&]() {
                __builtin_amdgcn_sched_barrier(0);       // all rows of a step are requested before the first is added
#pragma unroll
                for (int u = 0; u < kFwdUnroll; ++u)
#pragma unroll
                    for (int k = 0; k < KMAX; ++k)
                        IO::add(accs[u % NACC][k], raw[u][k]);
            };
            if (table_bytes <= kBufferBytes) {
                const __amdgpu_buffer_rsrc_t table = row_buffer(wbase, table_bytes);
                const uint32_t row_bytes = (uint32_t)D * (uint32_t)sizeof(WT);
                for (int block = 0; __ballot(block < len) != 0ull; block += LPR) {
                    const uint32_t cur = block + sub < len ? (uint32_t)nxt * row_bytes : kNoRow;
                    nxt = indices[min((uint32_t)(start + block + LPR + sub), last)];
                    for (int i = 0; i < LPR && __ballot(block + i < len) != 0ull; i += kFwdUnroll) {
#pragma unroll
                        for (int u = 0; u < kFwdUnroll; ++u) {
                            const uint32_t row = (uint32_t)__builtin_amdgcn_ds_bpermute((gbase + i + u) * 4, (int)cur);
#pragma unroll
                            for (int k = 0; k < KMAX; ++k)
                                raw[u][k] = load_buffer<Vec>(table, row + (uint32_t)eoff[k] * (uint32_t)sizeof(WT));
                        }
                        add_rows();
                    }
                }
            } else {
                for (int block = 0; __ballot(block < len) != 0ull; block += LPR) {
                    const int cur = nxt;
                    nxt = indices[min((uint32_t)(start + block + LPR + sub), last)];
                    for (int i = 0; i < LPR && __ballot(block + i < len) != 0ull; i += kFwdUnroll) {
#pragma unroll
                        for (int u = 0; u < kFwdUnroll; ++u) {
                            const int idx = __builtin_amdgcn_ds_bpermute((gbase + i + u) * 4, cur);
                            const WT* rp = block + i + u < len ? wbase + (int64_t)idx * D : zrow;
#pragma unroll
                            for (int k = 0; k < KMAX; ++k)
                                raw[u][k] = IO::ldv(rp + eoff[k]);
                        }
                        add_rows();
                    }
                }
            }
        } else if (__ballot(len > 0) != 0ull) {
            // rows of one or two lanes: every lane loads its own indices
            int idx[kFwdUnroll];
#pragma unroll
            for (int u = 0; u < kFwdUnroll; ++u)
                idx[u] = indices[min((uint32_t)(start + u), last)];
            for (int it = 0; __ballot(it < len) != 0ull; it += kFwdUnroll) {
                Vec raw[kFwdUnroll][KMAX];
#pragma unroll
                for (int u = 0; u < kFwdUnroll; ++u) {
                    const WT* rp = (it + u < len) ? wbase + (int64_t)idx[u] * D : zrow;
#pragma unroll
                    for (int k = 0; k < KMAX; ++k)
                        raw[u][k] = IO::ldv(rp + eoff[k]);
                }
#pragma unroll
                for (int u = 0; u < kFwdUnroll; ++u)
                    idx[u] = indices[min((uint32_t)(start + it + kFwdUnroll + u), last)];
#pragma unroll
                for (int u = 0; u < kFwdUnroll; ++u)
#pragma unroll
                    for (int k = 0; k < KMAX; ++k)
                        IO::add(accs[u % NACC][k], raw[u][k]);
            }
        }
        float acc[KMAX][EPL];
#pragma unroll
        for (int k = 0; k < KMAX; ++k)
#pragma unroll
            for (int e = 0; e < EPL; ++e) {
                if (NACC == 4)
                    acc[k][e] = (accs[0][k][e] + accs[1 % NACC][k][e]) + (accs[2 % NACC][k][e] + accs[3 % NACC][k][e]);
                else
                    acc[k][e] = accs[0][k][e];
            }

        if (active) {
            const int b = j - t * B + grp;
            // batch-major: row b of [B, sumD] at column col; table-major: row b of the table's own [B, D] block
            OT* op = table_major ? out + (int64_t)B * m.col + (int64_t)b * D : out + (int64_t)b * sumD + m.col;
#pragma unroll
            for (int k = 0; k < KMAX; ++k) {
                if (evalid[k]) {
#pragma unroll
                    for (int q = 0; q < EPL; q += 4)
                        store_out4(op + eoff[k] + q, acc[k][q], acc[k][q + 1], acc[k][q + 2], acc[k][q + 3]);
                }
            }
        }
        r += nb;
    }
}

// Calls of few bags: one bag per wavefront, its lookups spread over all lane groups (group g takes lookups g, g + G,
// ...), whose sums a butterfly adds at the end.  Such a call cannot fill the chip with bags, so what counts is the
// length of a bag's chain of dependent loads and that no lane group is idle: forward_kernel would use one of its G
// groups and four rows a step.  A step takes as many rows per group as the bag still needs, 1, 2, 4 or 8: a short bag
// issues no loads of the zero row beyond its last step.
//
// Per call, forward_kernel -> this kernel (dim 128, 20 lookups a bag): fp32 256 bags 5.6 -> 3.9 us, 2048 8.1 -> 5.8,
// 24,000 26.8 -> 22.3; fp16 256 bags 5.9 -> 3.7, 24,000 28.2 -> 16.2; fp32 dim 512, 30 lookups, 65,536 bags 321 -> 287.
constexpr int kBagUnroll = 8;                     // 76 registers for fp32 rows of up to 256 elements, 6 wavefronts a SIMD

template <typename WT, int EPL, int KMAX, typename OT>
__global__ __launch_bounds__(kFwdThreads) void forward_bag_kernel(
    const TableMeta* __restrict__ meta, const WT* __restrict__ weights,
    const int32_t* __restrict__ indices, const int64_t* __restrict__ offsets,
    OT* __restrict__ out, const void* __restrict__ zero_row, int32_t B, int32_t num_bags,
    int32_t sumD, int32_t n_total, int32_t table_major)
{
    using IO = RowIO<WT, EPL>;
    using Vec = typename IO::Vec;
    const int lane = threadIdx.x & (kWave - 1);
    const int j = uniform(blockIdx.x * (kFwdThreads / kWave) + (threadIdx.x >> 6));
    if (j >= num_bags)
        return;
    const int start = (int)offsets[j];
    const int len = (int)offsets[j + 1] - start;
    const uint32_t last = (uint32_t)(n_total - 1);
    const WT* __restrict__ zrow = static_cast<const WT*>(zero_row);
    const int t = j / B;
    const TableMeta m = meta[t];
    const int D = m.dim;
    const int lprl = m.lpr_fwd();
    const int LPR = 1 << lprl;
    const int G = kWave >> lprl;
    const int sub = lane & (LPR - 1);
    const int grp = lane >> lprl;
    const WT* __restrict__ wbase = weights + m.woff;

    int eoff[KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k)
        eoff[k] = min((sub + k * LPR) * EPL, D - EPL);
    // as in forward_kernel: four accumulators for fp32 tables, one for fp16
    constexpr int NACC = sizeof(WT) == 4 ? 4 : 1;
    float accs[NACC][KMAX][EPL];
#pragma unroll
    for (int q = 0; q < NACC; ++q)
#pragma unroll
        for (int k = 0; k < KMAX; ++k)
#pragma unroll
            for (int e = 0; e < EPL; ++e)
                accs[q][k][e] = 0.f;

    if (len > 0) {
        // Up to 8 groups: a step of 8 G lookups lies inside a block of 64, loaded with one instruction a block ahead
        // and handed out by shuffles.  More groups (rows of up to four lanes): every lane loads its own indices.
        const bool blocks = G * kBagUnroll <= kWave;
        const uint64_t table_bytes = (uint64_t)m.rows * (uint32_t)D * sizeof(WT);
        const bool buffer = blocks && table_bytes <= kBufferBytes;   // a lane forms the byte offset of its lookup's row
        const __amdgpu_buffer_rsrc_t table = row_buffer(wbase, buffer ? table_bytes : 0);
        const uint32_t row_bytes = (uint32_t)D * (uint32_t)sizeof(WT);
        int cur = 0, nxt = 0;
        if (blocks)
            nxt = indices[min((uint32_t)(start + lane), last)];
        auto step = [&](auto rows, int it) {
            constexpr int U = decltype(rows)::value;
            Vec raw[U][KMAX];
            if (buffer) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t row = (uint32_t)__builtin_amdgcn_ds_bpermute(((it & (kWave - 1)) + u * G + grp) * 4, cur);
#pragma unroll
                    for (int k = 0; k < KMAX; ++k)
                        raw[u][k] = load_buffer<Vec>(table, row + (uint32_t)eoff[k] * (uint32_t)sizeof(WT));
                }
            } else {
                int idx[U];
                if (blocks) {
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        idx[u] = __shfl(cur, (it + u * G + grp) & (kWave - 1));
                } else {
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        idx[u] = indices[min((uint32_t)(start + it + u * G + grp), last)];
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const WT* rp = it + u * G + grp < len ? wbase + (int64_t)idx[u] * D : zrow;
#pragma unroll
                    for (int k = 0; k < KMAX; ++k)
                        raw[u][k] = IO::ldv(rp + eoff[k]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int k = 0; k < KMAX; ++k)
                    IO::add(accs[u % NACC][k], raw[u][k]);
        };
        for (int it = 0; it < len; it += kBagUnroll * G) {
            if (blocks && (it & (kWave - 1)) == 0) {
                cur = !buffer ? nxt : it + lane < len ? (int)((uint32_t)nxt * row_bytes) : (int)kNoRow;
                if (len - it > kWave)
                    nxt = indices[min((uint32_t)(start + it + kWave + lane), last)];
            }
            const int left = len - it;
            if (left > 4 * G)
                step(std::integral_constant<int, 8>(), it);
            else if (left > 2 * G)
                step(std::integral_constant<int, 4>(), it);
            else if (left > G)
                step(std::integral_constant<int, 2>(), it);
            else
                step(std::integral_constant<int, 1>(), it);
        }
    }
    float acc[KMAX][EPL];
#pragma unroll
    for (int k = 0; k < KMAX; ++k)
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
            if (NACC == 4)
                acc[k][e] = (accs[0][k][e] + accs[1 % NACC][k][e]) + (accs[2 % NACC][k][e] + accs[3 % NACC][k][e]);
            else
                acc[k][e] = accs[0][k][e];
        }
    for (int o = LPR; o < kWave; o <<= 1)
#pragma unroll
        for (int k = 0; k < KMAX; ++k)
#pragma unroll
            for (int e = 0; e < EPL; ++e)
                acc[k][e] += __shfl_xor(acc[k][e], o);
    if (grp == 0) {
        const int b = j - t * B;
        OT* op = table_major ? out + (int64_t)B * m.col + (int64_t)b * D : out + (int64_t)b * sumD + m.col;
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            if ((sub + k * LPR) * EPL < D) {
#pragma unroll
                for (int q = 0; q < EPL; q += 4)
                    store_out4(op + eoff[k] + q, acc[k][q], acc[k][q + 1], acc[k][q + 2], acc[k][q + 3]);
            }
        }
    }
}

// ---------------------------------------------------------------- workgroup scan helper (256 threads)

__device__ __forceinline__ uint32_t block_exclusive_scan_256(uint32_t v, uint32_t* s_wave /*[4]*/,
                                                             uint32_t& block_total)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x >> 6;
    uint32_t incl = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t up = __shfl_up(incl, o);
        if (lane >= o)
            incl += up;
    }
    if (lane == kWave - 1)
        s_wave[wave] = incl;
    __syncthreads();
    uint32_t woff = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const uint32_t c = s_wave[w];
        if (w < wave)
            woff += c;
        tot += c;
    }
    block_total = tot;
    __syncthreads();
    return woff + incl - v;
}

// ---------------------------------------------------------------- fused aggregation + row-wise AdaGrad
//
// Section 5.1: all gradients of one row are aggregated on chip and the optimizer runs once per row.
// Section 5.2: m += mean_d(G_d^2); w -= lr * G / (sqrt(m) + eps)  (updated moment, eps outside the root).
//
// Each wavefront owns a span of SPAN consecutive sorted positions and every run that STARTS inside it.
// The span's run descriptors and payloads are staged in LDS once.  Lane mapping: a row of D floats
// is covered by LPR = pow2ceil(D/8) lanes, two float4 blocks per lane, so G = 64/LPR rows are
// fetched per load instruction.  The runs of the span are sorted by length class (a counting sort with
// ballots into a byte list in LDS) and handled class by class, so that every step is full:
//   * runs of one or two lookups: several per lane group and step (as many as the registers hold);
//   * runs of up to kShortRun lookups: one per lane group; all gradient rows, weight rows and moments
//     of a step are requested before anything is consumed, and all groups apply their update together;
//   * runs of up to 4 x 2^j lookups, 2^j <= G: teams of 2^j lane groups, G / 2^j runs per step, the
//     members' sums combined with an xor butterfly;
//   * longer runs use the whole wavefront in several steps (groups take alternate lookups); up to the
//     call's long_run lookups the owner follows the run past its span and finishes it;
//   * a longer run is not summed here.  Past the call's dense threshold it is queued, per table, for
//     dense_rows_kernel (counts x gradient block).  Below it, while a table's gradient block fits an L2
//     (by_position), its pieces of kPosPiece lookups are listed for window_runs_kernel right away; beyond that
//     the run is queued, per table, for window_runs_kernel (pieces by bag window).  Those write fp32 partial
//     rows to the workspace, and the fix-up kernel adds a run's partial rows in a fixed order and applies the update.  In
//     small and middle calls workgroups of this launch do all of that (kLongSmall, kLongPieces).
// The single-lookup rows of the tail of the index distribution move a row, its moment and one gradient row
// each and run at the rate of the memory system; the steps of the longer runs are bound by how fast gradient
// rows come out of the caches, so nothing here is arranged around instruction counts.
// Either way each touched row is read, updated and written exactly once, nothing is accumulated
// with atomics, and the summation order is fixed: results are bit-identical run to run.
//
// All gathers are branch-free (slots past the end of a run read a row of zeros kept in the
// workspace, column offsets past D are clamped) so that the loads of a step are issued back to
// back and waited for once.

// Table of a linear row id, for a whole wavefront (key uniform): 64 borders per step instead of one per step of a
// bisection, whose dependent loads the start of every span would wait for one after the other.
__device__ __forceinline__ int find_table(const uint32_t* __restrict__ row_base, int T, uint32_t key)
{
    const int lane = threadIdx.x & (kWave - 1);
    int lo = 0, n = T;  // row_base[lo] <= key < row_base[lo + n]
    while (n > 1) {
        const int step = (n + kWave - 1) / kWave;
        const int i = lane * step;
        const uint64_t le = __ballot(i < n && row_base[lo + min(i, n - 1)] <= key);
        const int k = (__popcll(le) - 1) * step;
        lo += k;
        n = min(step, n - k);
    }
    return lo;
}

// Optimizer of the fused epilogue (Section 5.1 names AdaGrad and Adam next to the row-wise AdaGrad of
// Section 5.2).  state0: row-wise AdaGrad -> one moment per row (indexed by linear row id);
// AdaGrad -> sum of squares per element; Adam -> first moment per element, state1 -> second moment.
// Per-element states are indexed like the flat weight array.
constexpr int kOptRowwiseAdagrad = 0;
constexpr int kOptAdagrad = 1;
constexpr int kOptAdam = 2;

struct OptParams {
    float* state0;
    float* state1;
    float lr;
    float eps;
    float beta1;
    float beta2;
    float inv_bc1;   // 1 / (1 - beta1^step)
    float inv_bc2;   // 1 / (1 - beta2^step)
};

struct BwdArgs {
    const TableMeta* meta;
    const uint32_t* row_base;
    const uint32_t* sorted_keys;
    const int32_t* sorted_vals;
    const uint32_t* unique_keys;
    const int32_t* seg_offsets;
    const int32_t* unit_first_run;   // runs that start before position i * kSpanUnit
    Counters* counters;
    const void* grad_out;   // [B, sumD] in the gradient type (float, __half or __hip_bfloat16)
    void* weights;
    float* partials;      // [num_chunks][2][dpad]
    struct LongRun* long_list;   // long runs for the fix-up kernel
    struct WinPiece* pieces;
    const float* zero_row;  // >= 2 KiB of zeros
    int32_t n;
    int32_t long_run;      // runs longer than this are long: kLongRun, or kPosPiece in a small call that cuts them by position
    int32_t small;         // long runs are those that sort_small_kernel listed, each summed by a workgroup of this kernel
    int32_t span_blocks;   // small: workgroups of spans; those of long runs follow
    int32_t piece_blocks;  // > 0: long runs are found by position, not listed; this many workgroups of the update kernel, in front of
                           // those of the spans, sum their pieces, a wavefront per partial row there could be
    int32_t grad_bytes;    // bytes per gradient element (sizes the bag windows)
    uint32_t* piece_done;  // [n / kPosSlot] (piece_blocks) pieces summed so far of the long run that starts there (zero between updates)
    const uint32_t* small_long;   // small: indices of the long runs, their number in front
    int32_t by_position;   // long runs are cut by position (their pieces are listed by the update kernel), not by bag window
    int32_t T;
    int32_t sumD;
    int32_t dpad;
    int32_t batch;
    int32_t table_major;   // gradient layout: 0 = [B, sumD] rows, 1 = one [B, D_t] block per table
    // dense hot rows (runs longer than dense_thr): queued per table by the update kernel, summed by dense_rows_kernel
    int32_t dense_thr;     // >= kDenseMinRun; INT32_MAX switches the dense path off
    int32_t dense_slices;  // ceil(batch / kDenseSlice): partial rows per dense run
    const int32_t* tstart; // [T+1] first sorted position of every table
    uint32_t* dense_cnt;   // [T] dense runs queued per table (zero between updates)
    uint32_t* dense_list;  // table t's queue starts at entry tstart[t] / dense_thr + t
    uint32_t* dense_dirty; // [T] set by dense_rows_kernel when a table's gradient block holds Inf / NaN
    // long runs (kLongRun < length <= dense_thr): queued per table, summed window by window by window_runs_kernel
    uint32_t* win_cnt;     // [T] (zero between updates)
    uint32_t* win_list;    // table t's queue starts at entry tstart[t] / kLongRun + t
    OptParams opt;
};
// (as for the sort's arguments: what the update reads of them lies in the first 256 bytes)
static_assert(offsetof(BwdArgs, opt) + offsetof(OptParams, beta1) <= 256, "row-wise AdaGrad");

struct WinPiece {        // 16 bytes: what a wavefront needs to sum one piece, in one load
    int32_t p0, p1;      // sorted positions of the piece
    int32_t slot;        // partial row it writes; < 0: merged into the piece that starts at an earlier window
    int32_t t;           // table
};

struct LongRun {         // 32 bytes: what a wavefront of the fix-up kernel needs to finish a run
    uint32_t key;        // linear row id
    int32_t t;           // table
    int32_t s, e;        // sorted positions of the run
    uint32_t pad[4];
};

// Lists the long runs of the lanes in `todo` (one run per lane: length, first position, row id, table) for the
// fix-up kernel and their pieces for window_runs_kernel.  The order of the lists depends on the order of the atomics,
// what a piece's partial row holds, where it lies and the order a run's are added in do not.
__device__ __forceinline__ void list_position_pieces(const BwdArgs& a, uint64_t todo, int len, int first, uint32_t key, int t)
{
    const int lane = threadIdx.x & (kWave - 1);
    while (todo != 0ull) {
        const int src = __ffsll((unsigned long long)todo) - 1;
        todo &= todo - 1;
        const int L = __shfl(len, src), s = __shfl(first, src), k = __shfl((int)key, src);
        const int np = position_pieces(L);
        uint32_t base = 0;
        if (lane == 0) {
            // one atomic for both lists: all runs of a call add to this word, at 6 ns each
            static_assert(offsetof(Counters, long_count) % 8 == 0 && offsetof(Counters, win_pieces) == offsetof(Counters, long_count) + 4, "");
            const unsigned long long was = atomicAdd(reinterpret_cast<unsigned long long*>(&a.counters->long_count),
                                                     (unsigned long long)np << 32 | 1ull);
            base = (uint32_t)(was >> 32);
            a.long_list[(uint32_t)was] = LongRun{(uint32_t)k, t, s, s + L, {0, 0, 0, 0}};
        }
        base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
        for (int i = lane; i < np; i += kWave) {
            WinPiece p;
            p.p0 = position_of_piece(s, L, np, i);
            p.p1 = position_of_piece(s, L, np, i + 1);
            p.slot = p.p0 / kPosSlot;
            p.t = t;
            a.pieces[base + i] = p;
        }
    }
}

__device__ __forceinline__ float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ void acc4(float (&a)[4], const float4 v)
{
    a[0] += v.x; a[1] += v.y; a[2] += v.z; a[3] += v.w;
}

// Gradient rows in their storage type: Vec is what one lane loads for a block of 4 elements.  `requested` stands between
// the loads of a step and its first addition.
template <typename GT>
struct GradIO;

template <>
struct GradIO<float> {
    using Vec = float4;
    __device__ static __forceinline__ Vec ldv(const float* p) { return *reinterpret_cast<const float4*>(p); }
    __device__ static __forceinline__ void requested() {}
    __device__ static __forceinline__ void add(float (&a)[4], const Vec v) { acc4(a, v); }
};

template <>
struct GradIO<__half> {
    using Vec = uint2;
    __device__ static __forceinline__ Vec ldv(const __half* p) { return *reinterpret_cast<const uint2*>(p); }
    // The additions are asm, which the scheduler otherwise moves between the loads, and a row's trip to memory then follows the
    // other's.  Update after one sort, Zipf, without / with: 64 columns, fp32 rows, 6 M lookups 296 / 282 us; 128, 0.2 M 33 / 30,
    // 6 M 502 / 489; 512, 0.2 M in fp16 69 / 56, element-wise AdaGrad 6 M 1635 / 1542; pieces of 7 M lookups 247 / 117.
    __device__ static __forceinline__ void requested() { __builtin_amdgcn_sched_barrier(0); }
    __device__ static __forceinline__ void add(float (&a)[4], const Vec v) { RowIO<__half, 4>::add(a, v); }
};

template <>
struct GradIO<__hip_bfloat16> {
    using Vec = uint2;
    __device__ static __forceinline__ Vec ldv(const __hip_bfloat16* p) { return *reinterpret_cast<const uint2*>(p); }
    __device__ static __forceinline__ void requested() {}
    // bfloat16 is the upper half of a float: widening is a 16-bit shift
    __device__ static __forceinline__ void add(float (&a)[4], const Vec v)
    {
        a[0] += __uint_as_float(v.x << 16); a[1] += __uint_as_float(v.x & 0xffff0000u);
        a[2] += __uint_as_float(v.y << 16); a[3] += __uint_as_float(v.y & 0xffff0000u);
    }
};

// An element of a partial row that a wavefront of another L2 adds up in the same launch: goes around the L2s both ways.
struct SharedFloat {
    float x;
};

template <>
struct GradIO<SharedFloat> {
    using Vec = float4;
    __device__ static __forceinline__ Vec ldv(const SharedFloat* p)
    {
        const uint64_t* q = reinterpret_cast<const uint64_t*>(p);
        const uint64_t a = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t b = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return make_float4(__uint_as_float((uint32_t)a), __uint_as_float((uint32_t)(a >> 32)), __uint_as_float((uint32_t)b),
                           __uint_as_float((uint32_t)(b >> 32)));
    }
    __device__ static __forceinline__ void requested() {}
    __device__ static __forceinline__ void add(float (&a)[4], const Vec v) { acc4(a, v); }
};

// Per-lane column geometry of a D-element row covered by LPR lanes with two 4-element blocks each.
struct Cols {
    int e0, e1;      // clamped element offsets of the two blocks (always loadable)
    bool c0, c1;     // whether the block really belongs to the row
    int sub, grp, lprl;
    __device__ __forceinline__ Cols(int D, int lprl_, int lane) : lprl(lprl_)
    {
        const int LPR = 1 << lprl;
        sub = lane & (LPR - 1);
        grp = lane >> lprl;
        const int a = sub * 4, b = (sub + LPR) * 4;
        c0 = a < D;
        c1 = b < D;
        e0 = min(a, D - 4);
        e1 = min(b, D - 4);
    }
};

// Whole-wavefront fp32 sum of the rows rowptr(i) (element type GT), i in [p0, p1), p1 > p0; rowptr must
// be valid for every i in the range.  Afterwards every lane group holds the complete sums.
template <typename GT, typename RowPtr>
__device__ __forceinline__ void wave_gather_sum(RowPtr rowptr, int p0, int p1, const float* __restrict__ zero_row_f,
                                                const Cols& c, float (&acc)[2][4])
{
    using GIO = GradIO<GT>;
    const GT* zero_row = reinterpret_cast<const GT*>(zero_row_f);
    const int G = kWave >> c.lprl;
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            acc[k][e] = 0.f;
    for (int i0 = p0; i0 < p1; i0 += G * kBwdUnroll) {
        typename GIO::Vec v[kBwdUnroll][2];
        const GT* rp[kBwdUnroll];
#pragma unroll
        for (int u = 0; u < kBwdUnroll; ++u) {
            const int i = i0 + u * G + c.grp;
            const GT* p = rowptr(min(i, p1 - 1));
            rp[u] = i < p1 ? p : zero_row;
        }
#pragma unroll
        for (int u = 0; u < kBwdUnroll; ++u) {
            v[u][0] = GIO::ldv(rp[u] + c.e0);
            v[u][1] = GIO::ldv(rp[u] + c.e1);
        }
        GIO::requested();
#pragma unroll
        for (int u = 0; u < kBwdUnroll; ++u) {
            GIO::add(acc[0], v[u][0]);
            GIO::add(acc[1], v[u][1]);
        }
    }
    for (int s = 1 << c.lprl; s < kWave; s <<= 1) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc[k][e] += __shfl_xor(acc[k][e], s);
    }
}

// The same, of the rows base + payload(i) * stride, where a row takes the whole wavefront (1 << c.lprl == kWave, rows of more than
// 256 columns).  A run or piece of 128 such rows is a chain of trips: 32 with four rows in flight, 16 with the eight that go on
// at once here (six of fp32).  A row is the same for all lanes, so its address is a scalar, and the rows take the registers that
// four rows and their addresses take: the kernel keeps its wavefronts (five or six a SIMD), and the narrower tables of a call
// lose nothing.  Update, us, four rows / these / eight with vector addresses in an instance of their own for every call with a
// wide table, which had four wavefronts a SIMD: 4 tables of 512 fp32 columns, 70,000 Zipf lookups 39.5 / 38.7 / 35.6, uniform
// 59.8 / 59.8 / 62.5, bf16 gradients 39.9 / 30.3 / 31.2; 4..512 columns, 0.15 M 37.1 / 34.9 / 35.6, bf16 39.2 / 31.4 / 35.3;
// 12 tables of 64 columns, 0.48 M, beside 4 of 512 with 800, fp16 29.3 / 28.8 / 37.5 (eight fp32 rows with scalar addresses take
// 114 registers: 35.3 for the first of these, 61.8 for the second, 54.4 for 51.6 of 4..512 columns, 0.4 M).
template <typename GT, typename Payload>
__device__ __forceinline__ void sum_wide_rows(Payload payload, const GT* base, int64_t stride, int p0, int p1, const GT* zero_row, const Cols& c,
                                              float (&acc)[2][4])
{
    using GIO = GradIO<GT>;
    constexpr int kRows = sizeof(GT) == 4 ? 6 : 8;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t o0 = (uint32_t)c.e0 * (uint32_t)sizeof(GT), o1 = (uint32_t)c.e1 * (uint32_t)sizeof(GT);
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            acc[k][e] = 0.f;
    for (int first = p0; first < p1; first += kWave) {
        const int cnt = min(kWave, p1 - first);
        const int mine = payload(min(first + lane, p1 - 1));
        for (int i0 = 0; i0 < cnt; i0 += kRows) {
            typename GIO::Vec v[kRows][2];
            uint32_t l0 = o0, l1 = o1;
            asm volatile("" : "+v"(l0), "+v"(l1));   // (widened here, a scalar address and a 32-bit offset are one load)
#pragma unroll
            for (int x = 0; x < kRows; ++x) {
                int64_t at = (int64_t)__builtin_amdgcn_readlane(mine, min(i0 + x, cnt - 1)) * stride;
                asm volatile("" : "+s"(at));         // (no branch around the product)
                const char* row = reinterpret_cast<const char*>(i0 + x < cnt ? base + at : zero_row);
                v[x][0] = GIO::ldv(reinterpret_cast<const GT*>(row + l0));
                v[x][1] = GIO::ldv(reinterpret_cast<const GT*>(row + l1));
            }
            GIO::requested();
#pragma unroll
            for (int x = 0; x < kRows; ++x) {
                GIO::add(acc[0], v[x][0]);
                GIO::add(acc[1], v[x][1]);
            }
        }
    }
}

// The optimizer state of the row held by this lane's group, requested together with the row itself.
template <int OPT>
struct OptRow {
    float m_old;         // row-wise AdaGrad
    float4 s0[2];        // AdaGrad sum of squares / Adam first moment, this lane's two blocks
    float4 s1[2];        // Adam second moment
    // key: linear row id; wel: index of the row's first element in the flat weight array
    __device__ __forceinline__ void load(const OptParams& p, uint32_t key, int64_t wel, const Cols& c)
    {
        if (OPT == kOptRowwiseAdagrad)
            m_old = p.state0[key];
        if (OPT == kOptAdagrad || OPT == kOptAdam) {
            s0[0] = ld4(p.state0 + wel + c.e0);
            s0[1] = ld4(p.state0 + wel + c.e1);
        }
        if (OPT == kOptAdam) {
            s1[0] = ld4(p.state1 + wel + c.e0);
            s1[1] = ld4(p.state1 + wel + c.e1);
        }
    }
};

__device__ __forceinline__ void st4(float* p, const float (&f)[4])
{
    *reinterpret_cast<float4*>(p) = make_float4(f[0], f[1], f[2], f[3]);
}
__device__ __forceinline__ void un4(const float4 v, float (&f)[4]) { f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w; }

// One block (4 elements) of the element-wise rules; g: aggregated gradient, w: weights (updated in place).
// Hardware reciprocal / square root (1 ulp each): far inside the 1e-5 tolerance of the result.
template <int OPT>
__device__ __forceinline__ void elementwise_block(const OptParams& p, const float (&g)[4], float (&w)[4],
                                                  const float4 s0v, const float4 s1v, float* s0p, float* s1p)
{
    float a[4], b[4];
    un4(s0v, a);
    if (OPT == kOptAdagrad) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            a[e] += g[e] * g[e];
            w[e] -= p.lr * g[e] * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(a[e]) + p.eps);
        }
        st4(s0p, a);
    } else {
        un4(s1v, b);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            a[e] = p.beta1 * a[e] + (1.0f - p.beta1) * g[e];
            b[e] = p.beta2 * b[e] + (1.0f - p.beta2) * g[e] * g[e];
            w[e] -= p.lr * (a[e] * p.inv_bc1) *
                    __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(b[e] * p.inv_bc2) + p.eps);
        }
        st4(s0p, a);
        st4(s1p, b);
    }
}

// The optimizer epilogue for the row held by this lane's group (wv: the row's old values, raw).
//   row-wise AdaGrad (Section 5.2): m += mean_d(G_d^2); w -= lr * G / (sqrt(m) + eps)
//   AdaGrad: S_d += G_d^2; w_d -= lr * G_d / (sqrt(S_d) + eps)
//   Adam (lazy, bias-corrected): m = b1 m + (1-b1) G; v = b2 v + (1-b2) G^2;
//                                w -= lr * (m / (1-b1^t)) / (sqrt(v / (1-b2^t)) + eps)
template <typename WT, int OPT>
__device__ __forceinline__ void optimizer_epilogue(WT* __restrict__ wrow, const typename RowIO<WT, 4>::Vec (&wv)[2],
                                                   const float (&acc)[2][4], int D, const Cols& c, bool writer,
                                                   const OptParams& p, uint32_t key, int64_t wel,
                                                   const OptRow<OPT>& st)
{
    if (OPT == kOptRowwiseAdagrad) {
        float ss0 = acc[0][0] * acc[0][0] + acc[0][1] * acc[0][1] + acc[0][2] * acc[0][2] + acc[0][3] * acc[0][3];
        float ss1 = acc[1][0] * acc[1][0] + acc[1][1] * acc[1][1] + acc[1][2] * acc[1][2] + acc[1][3] * acc[1][3];
        float ss = (c.c0 ? ss0 : 0.f) + (c.c1 ? ss1 : 0.f);
        for (int s = 1; s < (1 << c.lprl); s <<= 1)
            ss += __shfl_xor(ss, s);
        // hardware reciprocal / square root (1 ulp each): far inside the 1e-5 tolerance of the result
        const float m_new = st.m_old + ss * __builtin_amdgcn_rcpf((float)D);
        const float scale = p.lr * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(m_new) + p.eps);
        if (writer) {
            float w[4];
            if (c.c0) {
                RowIO<WT, 4>::unpack(wv[0], w);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    w[e] -= scale * acc[0][e];
                RowIO<WT, 4>::store(wrow + c.e0, w);
            }
            if (c.c1) {
                RowIO<WT, 4>::unpack(wv[1], w);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    w[e] -= scale * acc[1][e];
                RowIO<WT, 4>::store(wrow + c.e1, w);
            }
            if (c.sub == 0)
                p.state0[key] = m_new;
        }
    } else if (writer) {
        float w[4];
        if (c.c0) {
            RowIO<WT, 4>::unpack(wv[0], w);
            elementwise_block<OPT>(p, acc[0], w, st.s0[0], st.s1[0], p.state0 + wel + c.e0, p.state1 + wel + c.e0);
            RowIO<WT, 4>::store(wrow + c.e0, w);
        }
        if (c.c1) {
            RowIO<WT, 4>::unpack(wv[1], w);
            elementwise_block<OPT>(p, acc[1], w, st.s0[1], st.s1[1], p.state0 + wel + c.e1, p.state1 + wel + c.e1);
            RowIO<WT, 4>::store(wrow + c.e1, w);
        }
    }
}

__device__ __forceinline__ void store_partial(float* __restrict__ dst, const float (&acc)[2][4], const Cols& c)
{
    if (c.grp == 0) {
        if (c.c0)
            *reinterpret_cast<float4*>(dst + c.e0) = make_float4(acc[0][0], acc[0][1], acc[0][2], acc[0][3]);
        if (c.c1)
            *reinterpret_cast<float4*>(dst + c.e1) = make_float4(acc[1][0], acc[1][1], acc[1][2], acc[1][3]);
    }
}

__device__ __forceinline__ void store_shared(float* __restrict__ dst, const float (&acc)[2][4], const Cols& c)
{
    auto st = [](float* p, const float (&v)[4]) {
        uint64_t* q = reinterpret_cast<uint64_t*>(p);
        __hip_atomic_store(q, (uint64_t)__float_as_uint(v[1]) << 32 | __float_as_uint(v[0]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(q + 1, (uint64_t)__float_as_uint(v[3]) << 32 | __float_as_uint(v[2]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    if (c.grp == 0) {
        if (c.c0)
            st(dst + c.e0, acc[0]);
        if (c.c1)
            st(dst + c.e1, acc[1]);
    }
}

// Sum of the gradient rows of the sorted positions [p0, p1) of one table, by one wavefront; every lane group has it.
template <typename GT, bool WIDE = false>
__device__ __forceinline__ void sum_lookups(const BwdArgs& a, const TableMeta& m, const Cols& c, int p0, int p1, float (&acc)[2][4])
{
    using GIO = GradIO<GT>;
    const int lane = threadIdx.x & (kWave - 1);
    const GT* __restrict__ grad_out = static_cast<const GT*>(a.grad_out);
    const GT* zero_row = reinterpret_cast<const GT*>(a.zero_row);
    const int32_t* __restrict__ vals = a.sorted_vals;
    const int64_t stride = a.table_major ? m.dim : a.sumD;
    const GT* gb = a.table_major ? grad_out + (int64_t)a.batch * m.col : grad_out + m.col;
    if (WIDE && 1 << c.lprl == kWave) {
        sum_wide_rows([&](int i) { return vals[i]; }, gb, stride, p0, p1, zero_row, c, acc);
        return;
    }
    const int G = kWave >> c.lprl;
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int x = 0; x < 4; ++x)
            acc[k][x] = 0.f;
    for (int base = p0; base < p1; base += kWave) {
        const int cnt = min(kWave, p1 - base);
        const int myv = vals[min(base + lane, p1 - 1)];     // 64 payloads with one coalesced load
        for (int i0 = 0; i0 < cnt; i0 += G * kBwdUnroll) {
            typename GIO::Vec v[kBwdUnroll][2];
            const GT* rp[kBwdUnroll];
#pragma unroll
            for (int x = 0; x < kBwdUnroll; ++x) {
                const int i = i0 + x * G + c.grp;
                const int b = __shfl(myv, min(i, cnt - 1));
                rp[x] = i < cnt ? gb + (int64_t)b * stride : zero_row;
            }
#pragma unroll
            for (int x = 0; x < kBwdUnroll; ++x) {
                v[x][0] = GIO::ldv(rp[x] + c.e0);
                v[x][1] = GIO::ldv(rp[x] + c.e1);
            }
            GIO::requested();
#pragma unroll
            for (int x = 0; x < kBwdUnroll; ++x) {
                GIO::add(acc[0], v[x][0]);
                GIO::add(acc[1], v[x][1]);
            }
        }
    }
    for (int sft = 1 << c.lprl; sft < kWave; sft <<= 1) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int x = 0; x < 4; ++x)
                acc[k][x] += __shfl_xor(acc[k][x], sft);
    }
}

// One wavefront sums the gradient rows of one piece and writes its partial row.
template <typename GT>
__device__ __forceinline__ void sum_piece(const BwdArgs& a, const int4 rec /* p0, p1, slot, t */)
{
    const TableMeta m = a.meta[rec.w];
    const Cols c(m.dim, m.lpr_bwd(), threadIdx.x & (kWave - 1));
    float acc[2][4];
    sum_lookups<GT>(a, m, c, rec.x, rec.y, acc);
    store_partial(a.partials + (int64_t)rec.z * a.dpad, acc, c);
}

// Long runs by position need no list: partial rows are numbered by position, kPosSlot positions each, and at most one piece
// starts in those of a number (at most one long run does), always of the last run that starts before their end.
struct FoundPiece {
    int run, s, e;           // index and positions of the run
    int p0, p1;              // positions of the piece
    bool found;              // a piece of a long run starts there
};

__device__ __forceinline__ FoundPiece find_piece(const BwdArgs& a, int slot)
{
    static_assert(kPosSlot % kSpanUnit == 0, "");
    FoundPiece f;
    const bool valid = slot < (a.n + kPosSlot - 1) / kPosSlot;
    const int end = min(a.n, (valid ? slot + 1 : 1) * kPosSlot);
    f.run = a.unit_first_run[(end + kSpanUnit - 1) / kSpanUnit] - 1;
    f.s = a.seg_offsets[f.run];
    f.e = a.seg_offsets[f.run + 1];
    const int len = f.e - f.s, np = position_pieces(len);
    const int i = first_piece_from(len, np, slot * kPosSlot - f.s);
    f.p0 = position_of_piece(f.s, len, np, i);
    f.p1 = position_of_piece(f.s, len, np, i + 1);
    f.found = valid && len > a.long_run && i < np && f.p0 < (slot + 1) * kPosSlot;
    return f;
}

// One wavefront sums the gradient rows of a piece and writes its partial row.  The one that is the last of its run's to do so
// adds the partial rows up in their order and applies the update: whichever wavefront that is, the sum is the same.  (A launch
// of its own for the last part took 5 to 11 us, most of it its latency.)
//
// What orders a row's stores, in one wavefront, before its loads, in another, is gfx950 and not the language's memory model, by
// which relaxed atomics order nothing else.  Stores of agent scope go through the wavefront's L2 to memory, and the counter that
// s_waitcnt waits for counts a store as done when memory has it (the only dirty lines that a release would write back are others);
// the count is an atomic where memory is; loads of agent scope are served from there, and none is issued before the branch on
// the count.  The two asm statements keep the compiler from moving any of it.  Fences of agent scope, in place of them, write
// the whole L2 back and invalidate it for every piece: update of 8 tables of 128 columns, 0.5 M Zipf 1.2 lookups 46 -> 118 us.
template <typename WT, typename GT, int OPT>
__device__ __forceinline__ void piece_of_found_run(const BwdArgs& a, int slot, int run, int s, int e, int p0, int p1)
{
    using IO = RowIO<WT, 4>;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t key = (uint32_t)uniform((int)a.unique_keys[run]);
    const TableMeta m = a.meta[uniform(find_table(a.row_base, a.T, key))];
    const Cols c(m.dim, m.lpr_bwd(), lane);
    const int np = position_pieces(e - s);
    float acc[2][4];
    constexpr bool kWide = OPT == kOptRowwiseAdagrad;
    sum_lookups<GT, kWide>(a, m, c, p0, p1, acc);
    store_shared(a.partials + (int64_t)slot * a.dpad, acc, c);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    uint32_t* done = a.piece_done + s / kPosSlot;
    uint32_t before = 0;
    if (lane == 0)
        before = __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (uniform((int)before) != np - 1)
        return;
    asm volatile("" ::: "memory");
    if (lane == 0)
        __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int64_t wel = m.woff + (int64_t)(key - m.rbase) * m.dim;
    const SharedFloat* rows = reinterpret_cast<const SharedFloat*>(a.partials);
    auto slot_of = [&](int i) { return position_of_piece(s, e - s, np, i) / kPosSlot; };
    WT* wrow = static_cast<WT*>(a.weights) + wel;
    typename IO::Vec wvv[2];
    OptRow<OPT> st;
    wvv[0] = IO::ldv(wrow + c.e0);
    wvv[1] = IO::ldv(wrow + c.e1);
    st.load(a.opt, key, wel, c);
    if (kWide && 1 << c.lprl == kWave)
        sum_wide_rows(slot_of, rows, a.dpad, 0, np, reinterpret_cast<const SharedFloat*>(a.zero_row), c, acc);
    else
        wave_gather_sum<SharedFloat>([&](int i) { return rows + (int64_t)slot_of(i) * a.dpad; }, 0, np, a.zero_row, c, acc);
    optimizer_epilogue<WT, OPT>(wrow, wvv, acc, m.dim, c, c.grp == 0, a.opt, key, wel, st);
}

// A long run of a small call, by one workgroup: its wavefronts sum a share each, the first adds the shares in their order
// and applies the update.  One launch less for the pieces and one for the fix-up, which are empty as a rule and cost 4 us
// each all the same (2048 lookups, 64 columns: step of 20.6 -> 17.3 us).
template <typename WT, typename GT, int OPT>
__device__ __forceinline__ void small_long_run(const BwdArgs& a, int i, float (*s_part)[kMaxDim])
{
    using IO = RowIO<WT, 4>;
    constexpr int kWaves = kBwdThreads / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = uniform(threadIdx.x >> 6);
    const uint32_t listed = a.small_long[0];
    const int run = (int)a.small_long[1 + i];            // (there is room for every workgroup's)
    if (i >= (int)listed)
        return;
    const uint32_t key = (uint32_t)uniform((int)a.unique_keys[run]);
    const int s = uniform(a.seg_offsets[run]), e = uniform(a.seg_offsets[run + 1]);
    const int t = uniform(find_table(a.row_base, a.T, key));
    const TableMeta m = a.meta[t];
    const Cols c(m.dim, m.lpr_bwd(), lane);
    const int64_t wel = m.woff + (int64_t)(key - m.rbase) * m.dim;
    WT* wrow = static_cast<WT*>(a.weights) + wel;
    typename IO::Vec wvv[2];
    OptRow<OPT> st;
    if (wave == 0) {
        wvv[0] = IO::ldv(wrow + c.e0);
        wvv[1] = IO::ldv(wrow + c.e1);
        st.load(a.opt, key, wel, c);
    }
    float acc[2][4];
    sum_lookups<GT>(a, m, c, position_of_piece(s, e - s, kWaves, wave), position_of_piece(s, e - s, kWaves, wave + 1), acc);
    store_partial(s_part[wave], acc, c);
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int w = 1; w < kWaves; ++w) {
            acc4(acc[0], ld4(&s_part[w][c.e0]));
            acc4(acc[1], ld4(&s_part[w][c.e1]));
        }
        optimizer_epilogue<WT, OPT>(wrow, wvv, acc, m.dim, c, c.grp == 0, a.opt, key, wel, st);
    }
}

// One step of the update kernel: up to NB * (G >> tsl) runs of one table at once.  The G lane groups of the
// wavefront form teams of 1 << tsl groups; a team takes NB runs from the class list (entries i0 .. i0 + cnt - 1,
// run indices of the wavefront's span), every member group fetches up to ML gradient rows of each (member m takes
// the lookups m, m + team size, ...), the members' sums are combined with an xor butterfly, and member 0 applies
// the update.  All weight rows, moments and gradient rows of the step are requested before anything is consumed:
// the number of rows in flight per wavefront, not the instruction count, bounds this kernel.
template <typename WT, typename GT, int OPT, int ML, int NB>
__device__ __forceinline__ void run_batch(const BwdArgs& a, WT* __restrict__ wtab, int64_t woff,
                                          const GT* __restrict__ gb, int sumD,
                                          const int32_t* __restrict__ s_seg, const uint32_t* __restrict__ s_key,
                                          const int32_t* __restrict__ s_val, const uint8_t* __restrict__ s_list,
                                          int q0, int i0, int cnt, int tsl, uint32_t rbase, int D, const Cols& c)
{
    using IO = RowIO<WT, 4>;
    using GIO = GradIO<GT>;
    const int teams = (kWave >> c.lprl) >> tsl;
    const int team = c.grp >> tsl;
    const int member = c.grp & ((1 << tsl) - 1);
    typename IO::Vec wv[NB][2];
    OptRow<OPT> st[NB];
    uint32_t key[NB];
    int vbase[NB], len[NB], run[NB];
    bool act[NB];
    // all LDS reads of a level are issued together: the row requests below start one LDS round trip
    // after the other, not one per run
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int li = j * teams + team;
        act[j] = li < cnt;
        run[j] = s_list[i0 + (act[j] ? li : 0)];     // idle teams shadow the first run: loads stay valid
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        key[j] = s_key[run[j]];
        vbase[j] = s_seg[run[j]];
        len[j] = s_seg[run[j] + 1];
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        len[j] = act[j] ? len[j] - vbase[j] : 0;
        vbase[j] -= q0;
        const uint64_t rel = (uint64_t)(key[j] - rbase) * (uint32_t)D;
        wv[j][0] = IO::ldv(wtab + rel + c.e0);
        wv[j][1] = IO::ldv(wtab + rel + c.e1);
        st[j].load(a.opt, key[j], woff + (int64_t)rel, c);
    }
    typename GIO::Vec v[NB][ML][2];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const GT* rp[ML];
#pragma unroll
        for (int u = 0; u < ML; ++u) {
            const int pos = member + (u << tsl);
            const bool ok = pos < len[j];
            const int b = s_val[vbase[j] + (ok ? pos : 0)];
            rp[u] = ok ? gb + (uint64_t)(uint32_t)b * (uint32_t)sumD : reinterpret_cast<const GT*>(a.zero_row);
        }
#pragma unroll
        for (int u = 0; u < ML; ++u) {
            v[j][u][0] = GIO::ldv(rp[u] + c.e0);
            v[j][u][1] = GIO::ldv(rp[u] + c.e1);
        }
    }
    GIO::requested();
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        float acc[2][4];
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc[k][e] = 0.f;
#pragma unroll
        for (int u = 0; u < ML; ++u) {
            GIO::add(acc[0], v[j][u][0]);
            GIO::add(acc[1], v[j][u][1]);
        }
        for (int sh = 1 << c.lprl; sh < (1 << (c.lprl + tsl)); sh <<= 1) {
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc[k][e] += __shfl_xor(acc[k][e], sh);
        }
        uint32_t kj = key[j];
        asm volatile("" : "+v"(kj));    // the store addresses are formed again here, not kept in registers meanwhile
        const uint64_t rel = (uint64_t)(kj - rbase) * (uint32_t)D;
        optimizer_epilogue<WT, OPT>(wtab + rel, wv[j], acc, D, c, act[j] && member == 0, a.opt, kj,
                                    woff + (int64_t)rel, st[j]);
    }
}

// SPAN: sorted positions owned by one wavefront.  LONG: who sums the long runs.  (In one kernel the scalar registers did not do:
// 0.3 % of 0.65 M lookups; with kLongSmall and kLongPieces in one 2048 lookups took 0.2 us more.)
enum LongRuns {
    kLongListed,       // the spans list them for other kernels
    kLongSmall,        // workgroups of this launch (a.small)
    kLongPieces,       // workgroups of this launch sum their pieces (a.piece_blocks)
};

template <typename WT, typename GT, int OPT, int SPAN, int LONG>
// (sum_wide_rows fits the wavefronts that the kernel has without it)
__global__ __launch_bounds__(kBwdThreads, LONG == kLongPieces && OPT == kOptRowwiseAdagrad ? (sizeof(GT) == 4 ? 5 : 6) : 1)
void reduce_update_kernel(BwdArgs a)
{
    using IO = RowIO<WT, 4>;
    const GT* __restrict__ grad_out = static_cast<const GT*>(a.grad_out);
    constexpr int kWaves = kBwdThreads / kWave;
    constexpr int kRounds = SPAN < kWave ? 1 : SPAN / kWave;   // staging rounds of one entry per lane
    constexpr int kStaged = kRounds * kWave;      // positions whose payloads are staged: the span's, and those after a short one
    constexpr int kSegCap = (kRounds + 1) * kWave; // >= SPAN + 1
    constexpr int kValCap = kStaged + kLongRun;   // a run owned by the span ends within this window
    // row-wise AdaGrad keeps one moment per row, so several runs per lane group fit in registers; the
    // element-wise optimizers carry whole state rows and take one run per group
    constexpr int kNB1 = OPT != kOptRowwiseAdagrad ? 1 : sizeof(WT) == 2 ? 4 : 2;   // runs of one lookup per group
    constexpr int kNB2 = OPT != kOptRowwiseAdagrad ? 1 : 2;                          // runs of two lookups per group
    constexpr bool kWide = LONG == kLongPieces && OPT == kOptRowwiseAdagrad;
    static_assert(SPAN <= 256, "run indices of a span are kept in bytes");
    static_assert(kShortRun == 4, "run_batch is instantiated for 1..4 lookups");
    __shared__ int32_t s_seg_all[kWaves][kSegCap];
    __shared__ uint32_t s_key_all[kWaves][kStaged];
    __shared__ __align__(16) int32_t s_val_all[kWaves][kValCap];
    __shared__ uint8_t s_list_all[kWaves][kStaged];

    const int lane = threadIdx.x & (kWave - 1);
    const int wv = threadIdx.x >> 6;
    int block = (int)blockIdx.x;
    if constexpr (LONG == kLongSmall) {
        if (block >= a.span_blocks) {
            static_assert(sizeof(s_val_all) >= sizeof(float) * kWaves * kMaxDim && kValCap % 4 == 0, "");
            small_long_run<WT, GT, OPT>(a, block - a.span_blocks, reinterpret_cast<float(*)[kMaxDim]>(&s_val_all[0][0]));
            return;
        }
    }
    if constexpr (LONG == kLongPieces) {
        if (block < a.piece_blocks) {
            // beside the spans: in a launch of its own after them a piece added a chain of up to 128 rows to calls that are little
            // more than such chains, and 5 us to those without long runs (40 tables of 4..512 columns, 0.17 M lookups: step of
            // 105 -> 86 us; Adam, 0.44 M 190 -> 184; 512 columns, 0.2 M 171 -> 154; pieces of 64 lookups: 87 and 165)
            const int slot = uniform(block * kWaves + wv);
            const FoundPiece f = find_piece(a, slot);
            if (uniform(f.found))
                piece_of_found_run<WT, GT, OPT>(a, slot, uniform(f.run), uniform(f.s), uniform(f.e), uniform(f.p0), uniform(f.p1));
            return;
        }
        block -= a.piece_blocks;
    }
    const int k = uniform(block * kWaves + wv);
    const int q0 = k * SPAN;
    if (q0 >= a.n)
        return;
    int32_t* s_seg = s_seg_all[wv];
    uint32_t* s_key = s_key_all[wv];
    int32_t* s_val = s_val_all[wv];
    uint8_t* s_list = s_list_all[wv];

    const int q1 = min(a.n, q0 + SPAN);
    const int ub = a.unit_first_run[q0 / kSpanUnit];
    const int ue = a.unit_first_run[(q1 + kSpanUnit - 1) / kSpanUnit];
    const int nruns = ue - ub;  // runs that start in [q0, q1): at most SPAN
    if (nruns == 0)
        return;     // the span lies inside one run: its owner, or (long runs) another kernel, sums all of it
    WT* __restrict__ weights = static_cast<WT*>(a.weights);
    const int32_t* __restrict__ vals = a.sorted_vals;

    // ---- stage run descriptors and payloads (wavefront-private LDS); straight-line clamped loads
    {
        int sg[kRounds + 1];
        uint32_t ky[kRounds];
        int vl[kRounds];
#pragma unroll
        for (int i = 0; i < kRounds + 1; ++i)
            sg[i] = a.seg_offsets[ub + min(i * kWave + lane, nruns)];
#pragma unroll
        for (int i = 0; i < kRounds; ++i)
            ky[i] = a.unique_keys[ub + min(i * kWave + lane, nruns - 1)];
#pragma unroll
        for (int i = 0; i < kRounds; ++i)
            vl[i] = vals[min(q0 + i * kWave + lane, a.n - 1)];
#pragma unroll
        for (int i = 0; i < kRounds + 1; ++i)
            s_seg[i * kWave + lane] = sg[i];
#pragma unroll
        for (int i = 0; i < kRounds; ++i) {
            s_key[i * kWave + lane] = ky[i];
            s_val[i * kWave + lane] = vl[i];
        }
    }
    __threadfence_block();
    __builtin_amdgcn_wave_barrier();
    // the last run that starts here may continue past the span: stage its payloads too, unless it is
    // a long run (those are not summed here)
    {
        const int e_last = uniform(s_seg[nruns]);
        const int s_last = uniform(s_seg[nruns - 1]);
        if (e_last > q0 + kStaged && e_last - s_last <= a.long_run) {
            for (int p = q0 + kStaged + lane; p < e_last; p += kWave)
                s_val[p - q0] = vals[p];
            __threadfence_block();
            __builtin_amdgcn_wave_barrier();
        }
    }

    const uint64_t lt = (1ull << lane) - 1ull;
    // entries [0, count) of s_list <- the span's runs of class cl, in run order
    auto build_list = [&](const int (&cls)[kRounds], int cl, int first) {
        int n = first;
#pragma unroll
        for (int i = 0; i < kRounds; ++i) {
            const uint64_t mk = __ballot(cls[i] == cl);
            if (cls[i] == cl)
                s_list[n + __popcll(mk & lt)] = (uint8_t)(i * kWave + lane);
            n += __popcll(mk);
        }
        return n;
    };
    auto run_len = [&](int li) {
        const int run = s_list[li];
        return uniform(s_seg[run + 1] - s_seg[run]);
    };

    int ra = 0;
    while (ra < nruns) {
        // ---- the runs [ra, rb) of the table of run ra (a span rarely touches more than one table)
        const uint32_t key0 = (uint32_t)uniform((int)s_key[ra]);
        const int t = uniform(find_table(a.row_base, a.T, key0));
        TableMeta m = a.meta[t];            // wavefront-uniform: kept in scalar registers
        m.woff = ((int64_t)uniform((int)(m.woff >> 32)) << 32) | (uint32_t)uniform((int)m.woff);
        m.rbase = (uint32_t)uniform((int)m.rbase);
        m.dim = uniform(m.dim);
        m.col = uniform(m.col);
        m.lanes = (uint32_t)uniform((int)m.lanes);
        const uint32_t t_hi = (uint32_t)uniform((int)a.row_base[t + 1]);
        int rb = 0;
#pragma unroll
        for (int i = 0; i < kRounds; ++i) {
            const int run = i * kWave + lane;
            rb += __popcll(__ballot(run < nruns && s_key[min(run, nruns - 1)] < t_hi));
        }
        const int D = m.dim;
        const int lprl = m.lpr_bwd();
        const int lgG = 6 - lprl;
        const int G = 1 << lgG;
        const GT* gb = a.table_major ? grad_out + (int64_t)a.batch * m.col : grad_out + m.col;
        const int sumD = a.table_major ? m.dim : (int)a.sumD;   // distance between the gradient rows of consecutive bags
        WT* wtab = weights + m.woff;
        const Cols c(D, lprl, lane);

        // ---- classes by length: 0 .. 3: one .. four lookups; 3 + j: up to 4 << j lookups, summed by a team of
        // 1 << j lane groups (while that is at most a wavefront); 14: whole wavefront, several steps;
        // 15: long, queued for the fix-up kernel and, per table, for the kernel that sums it
        int cls[kRounds];
#pragma unroll
        for (int i = 0; i < kRounds; ++i) {
            const int run = i * kWave + lane;
            const bool valid = run >= ra && run < rb;
            const int rc = valid ? run : ra;
            const int len = s_seg[rc + 1] - s_seg[rc];
            int cl;
            if (len <= kShortRun) {
                cl = len - 1;
            } else if (len > a.long_run) {
                cl = 15;
            } else {
                const int tl = 32 - __clz((len - 1) >> 2);     // smallest tl with (4 << tl) >= len
                cl = tl <= lgG ? 3 + tl : 14;
            }
            cls[i] = valid ? cl : -1;
            if constexpr (LONG != kLongListed)
                continue;
            const bool cut = a.by_position && len <= a.dense_thr;
            if (a.by_position)
                list_position_pieces(a, __ballot(valid && cl == 15 && cut), len, s_seg[rc], s_key[rc], t);
            if (valid && cl == 15 && !cut) {
                if (len > a.dense_thr) {
                    const uint32_t dslot = atomicAdd(&a.dense_cnt[t], 1u);
                    a.dense_list[a.tstart[t] / a.dense_thr + t + (int)dslot] = (uint32_t)(ub + run);
                } else {
                    const uint32_t wslot = atomicAdd(&a.win_cnt[t], 1u);
                    a.win_list[a.tstart[t] / kLongRun + t + (int)wslot] = (uint32_t)(ub + run);
                }
                const uint32_t slot = atomicAdd(&a.counters->long_count, 1u);
                a.long_list[slot] = LongRun{s_key[rc], t, s_seg[rc], s_seg[rc + 1], {0, 0, 0, 0}};
            }
        }

        // ---- runs of up to four lookups, shortest first: as many per step as the registers hold
        {
            int nshort = build_list(cls, 0, 0);
            nshort = build_list(cls, 1, nshort);
            nshort = build_list(cls, 2, nshort);
            nshort = build_list(cls, 3, nshort);
            __threadfence_block();
            __builtin_amdgcn_wave_barrier();
            int i = 0;
            while (i < nshort) {
                const int rem = nshort - i;
                if (kNB1 > 1 && rem > G) {
                    const int cand = min(kNB1 * G, rem);
                    if (run_len(i + cand - 1) == 1) {
                        if (kNB1 > 2 && cand > 2 * G)
                            run_batch<WT, GT, OPT, 1, kNB1>(a, wtab, m.woff, gb, sumD, s_seg, s_key, s_val, s_list, q0, i, cand, 0, m.rbase, D, c);
                        else
                            run_batch<WT, GT, OPT, 1, 2>(a, wtab, m.woff, gb, sumD, s_seg, s_key, s_val, s_list, q0, i, cand, 0, m.rbase, D, c);
                        i += cand;
                        continue;
                    }
                }
                if (kNB2 > 1 && rem > G) {
                    const int cand = min(2 * G, rem);
                    const int ml = run_len(i + cand - 1);
                    if (ml <= 2) {
                        if (ml == 1)
                            run_batch<WT, GT, OPT, 1, 2>(a, wtab, m.woff, gb, sumD, s_seg, s_key, s_val, s_list, q0, i, cand, 0, m.rbase, D, c);
                        else
                            run_batch<WT, GT, OPT, 2, 2>(a, wtab, m.woff, gb, sumD, s_seg, s_key, s_val, s_list, q0, i, cand, 0, m.rbase, D, c);
                        i += cand;
                        continue;
                    }
                }
                const int cand = min(G, rem);
                switch (run_len(i + cand - 1)) {
                    case 1: run_batch<WT, GT, OPT, 1, 1>(a, wtab, m.woff, gb, sumD, s_seg, s_key, s_val, s_list, q0, i, cand, 0, m.rbase, D, c); break;
                    case 2: run_batch<WT, GT, OPT, 2, 1>(a, wtab, m.woff, gb, sumD, s_seg, s_key, s_val, s_list, q0, i, cand, 0, m.rbase, D, c); break;
                    case 3: run_batch<WT, GT, OPT, 3, 1>(a, wtab, m.woff, gb, sumD, s_seg, s_key, s_val, s_list, q0, i, cand, 0, m.rbase, D, c); break;
                    default: run_batch<WT, GT, OPT, 4, 1>(a, wtab, m.woff, gb, sumD, s_seg, s_key, s_val, s_list, q0, i, cand, 0, m.rbase, D, c); break;
                }
                i += cand;
            }
            __threadfence_block();
            __builtin_amdgcn_wave_barrier();
        }

        // ---- teams of 2, 4, ... lane groups: runs of up to 4 lookups per member group, one step each
        for (int tl = 1; tl <= lgG; ++tl) {
            const int cnt = build_list(cls, 3 + tl, 0);
            __threadfence_block();
            __builtin_amdgcn_wave_barrier();
            const int teams = G >> tl;
            for (int i = 0; i < cnt; i += teams)
                run_batch<WT, GT, OPT, 4, 1>(a, wtab, m.woff, gb, sumD, s_seg, s_key, s_val, s_list, q0, i, min(teams, cnt - i), tl, m.rbase, D, c);
            __threadfence_block();
            __builtin_amdgcn_wave_barrier();
        }

        // ---- longer runs: the whole wavefront, several steps
        {
            const int cnt = build_list(cls, 14, 0);
            __threadfence_block();
            __builtin_amdgcn_wave_barrier();
            for (int i = 0; i < cnt; ++i) {
                const int run = uniform((int)s_list[i]);
                const uint32_t key = (uint32_t)uniform((int)s_key[run]);
                const int s0 = uniform(s_seg[run]);
                const int len0 = uniform(s_seg[run + 1]) - s0;
                const int64_t rel = (int64_t)(key - m.rbase) * D;
                WT* wrow = wtab + rel;
                typename IO::Vec wvv[2];
                OptRow<OPT> st;
                float acc[2][4];
                const bool wide = kWide && 1 << c.lprl == kWave;
                wvv[0] = IO::ldv(wrow + c.e0);
                wvv[1] = IO::ldv(wrow + c.e1);
                st.load(a.opt, key, m.woff + rel, c);
                if (wide)
                    sum_wide_rows([&](int p) { return s_val[p - q0]; }, gb, sumD, s0, s0 + len0, reinterpret_cast<const GT*>(a.zero_row), c, acc);
                else
                    wave_gather_sum<GT>([&](int p) { return gb + (int64_t)s_val[p - q0] * sumD; }, s0, s0 + len0, a.zero_row,
                                        c, acc);
                optimizer_epilogue<WT, OPT>(wrow, wvv, acc, D, c, c.grp == 0, a.opt, key, m.woff + rel, st);
            }
            __threadfence_block();
            __builtin_amdgcn_wave_barrier();
        }
        ra = rb;
    }
}

// ---------------------------------------------------------------- dense hot rows
//
// Under a skewed index distribution a few rows per table are looked up by a large share of the bags
// (Section 5.1 aggregates all of their gradients before the one optimizer step).  Gathering one gradient
// row per lookup re-reads the table's [B, D_t] gradient block once per such row.  For a run longer than
// the call's dense threshold (about one lookup per 8 bags) the sum is formed the other way round:
//     G[r, :] = sum_b count[r, b] * grad[b, :]
// with count[r, b] = how often bag b looks row r up.  kDenseRows runs of one table form a group and share
// ONE pass over the gradient block; a work unit is (group, slice of kDenseSlice bags) and writes one fp32
// partial row per run into the slots of the chunks that run covers completely (the update kernel leaves
// them unused); the fix-up kernel adds a run's partial rows in slice order and applies the single step.
// Counts are exact integers built with LDS integer atomics from the run's sorted payloads; the float sum of
// a (run, slice) has a fixed order that does not depend on which other runs share the group, so results
// are bit-identical run to run.  A bag with a non-finite gradient must only reach the rows it looks up:
// such a bag takes a select-based path instead of multiplying by a zero count.

struct DenseGroup {      // 32 bytes
    int32_t t;           // table
    int32_t first;       // index of the group's first run in the compact run list
    int32_t nrows;       // runs in the group (1..kDenseRows)
    int32_t gbase;       // first group of the table
    int32_t ng;          // groups of the table
    int32_t pad[3];
};

struct DenseArgs {              // also used for the windowed runs (groups of one run, slices = windows)
    BwdArgs b;
    const uint32_t* drun;       // compact list of runs (run index u), grouped by table
    const DenseGroup* dgroup;
    int32_t* dbounds;           // [run][nsub + 1] first sorted position of the run whose bag is >= c * slice_bags
    const uint32_t* nruns;      // number of runs in drun (device counter)
    int32_t nsub;               // number of slices = ceil(batch / slice_bags)
    int32_t slice_bags;
};

// one workgroup: per-table queues -> compact run list + groups of at most rpg runs; clears the per-table
// counters.  cnt / list: the queues (table t's starts at entry tstart[t] / base_div + t).
__global__ __launch_bounds__(256) void run_plan_kernel(BwdArgs a, uint32_t* __restrict__ cnt,
                                                       const uint32_t* __restrict__ list, int base_div, int rpg,
                                                       uint32_t* __restrict__ drun, DenseGroup* __restrict__ dgroup,
                                                       uint32_t* __restrict__ out_runs, uint32_t* __restrict__ out_groups,
                                                       uint32_t* __restrict__ clear_flags)
{
    __shared__ uint32_t s_wave[4];
    __shared__ uint32_t s_c[256], s_rfirst[256], s_gfirst[256];
    uint32_t carry_r = 0, carry_g = 0;
    for (int base = 0; base < a.T; base += 256) {
        const int t = base + threadIdx.x;
        const uint32_t c = t < a.T ? cnt[t] : 0u;
        const uint32_t g = (c + rpg - 1) / rpg;
        if (t < a.T && clear_flags)
            clear_flags[t] = 0;
        uint32_t tot_r, tot_g;
        const uint32_t ex_r = block_exclusive_scan_256(c, s_wave, tot_r);
        const uint32_t ex_g = block_exclusive_scan_256(g, s_wave, tot_g);
        s_c[threadIdx.x] = c;
        s_rfirst[threadIdx.x] = carry_r + ex_r;
        s_gfirst[threadIdx.x] = carry_g + ex_g;
        if (c > 0)
            cnt[t] = 0;
        __syncthreads();
        // short queues (the usual case) are copied by their own thread, all tables at once ...
        if (c > 0 && c <= 64) {
            const uint32_t rfirst = carry_r + ex_r, gfirst = carry_g + ex_g;
            const uint32_t* q = list + (a.tstart[t] / base_div + t);
            for (uint32_t i = 0; i < c; ++i)
                drun[rfirst + i] = q[i];
            for (uint32_t gi = 0; gi < g; ++gi) {
                DenseGroup d;
                d.t = t;
                d.first = (int32_t)(rfirst + gi * rpg);
                d.nrows = (int32_t)min((uint32_t)rpg, c - gi * rpg);
                d.gbase = (int32_t)gfirst;
                d.ng = (int32_t)g;
                d.pad[0] = d.pad[1] = d.pad[2] = 0;
                dgroup[gfirst + gi] = d;
            }
        }
        // ... long ones (a queue can be long when the batch is small) by the whole workgroup, one table after the other
        const int nt = min(256, a.T - base);
        for (int tt = 0; tt < nt; ++tt) {
            const uint32_t ct = s_c[tt];
            if (ct <= 64)
                continue;
            const uint32_t rfirst = s_rfirst[tt], gfirst = s_gfirst[tt];
            const uint32_t gt = (ct + rpg - 1) / rpg;
            const uint32_t* q = list + (a.tstart[base + tt] / base_div + base + tt);
            for (uint32_t i = threadIdx.x; i < ct; i += 256)
                drun[rfirst + i] = q[i];
            for (uint32_t gi = threadIdx.x; gi < gt; gi += 256) {
                DenseGroup d;
                d.t = base + tt;
                d.first = (int32_t)(rfirst + gi * rpg);
                d.nrows = (int32_t)min((uint32_t)rpg, ct - gi * rpg);
                d.gbase = (int32_t)gfirst;
                d.ng = (int32_t)gt;
                d.pad[0] = d.pad[1] = d.pad[2] = 0;
                dgroup[gfirst + gi] = d;
            }
        }
        __syncthreads();
        carry_r += tot_r;
        carry_g += tot_g;
    }
    if (threadIdx.x == 0) {
        *out_runs = carry_r;
        if (out_groups)
            *out_groups = carry_g;
    }
}

// one wavefront per listed run: where the run's payloads (ascending bags) cross every multiple of slice_bags
__global__ __launch_bounds__(256) void run_bounds_kernel(DenseArgs d)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int wave_global = uniform(blockIdx.x * 4 + (threadIdx.x >> 6));
    const int wave_total = gridDim.x * 4;
    const int nruns = (int)*d.nruns;
    const int nb = d.nsub + 1;
    const int32_t* __restrict__ vals = d.b.sorted_vals;
    for (int i = wave_global; i < nruns; i += wave_total) {
        const int u = (int)d.drun[i];
        const int s = d.b.seg_offsets[u];
        const int e = d.b.seg_offsets[u + 1];
        for (int c = lane; c < nb; c += kWave) {
            const int target = c * d.slice_bags;
            int lo = s, hi = e;              // first p in [s, e) with vals[p] >= target
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (vals[mid] < target)
                    lo = mid + 1;
                else
                    hi = mid;
            }
            d.dbounds[(int64_t)i * nb + c] = c == d.nsub ? e : lo;
        }
    }
}

typedef float mfma_f4 __attribute__((ext_vector_type(4)));

// the four gradient values of one 16-byte (fp32) / 8-byte (16-bit) load as floats
__device__ __forceinline__ void grad_floats(const float4 v, float (&g)[4]) { g[0] = v.x; g[1] = v.y; g[2] = v.z; g[3] = v.w; }
__device__ __forceinline__ void grad_floats_half(const uint2 v, float (&g)[4])
{
    const float2 x = __half22float2(*reinterpret_cast<const __half2*>(&v.x));
    const float2 y = __half22float2(*reinterpret_cast<const __half2*>(&v.y));
    g[0] = x.x; g[1] = x.y; g[2] = y.x; g[3] = y.y;
}
__device__ __forceinline__ void grad_floats_bf16(const uint2 v, float (&g)[4])
{
    g[0] = __uint_as_float(v.x << 16); g[1] = __uint_as_float(v.x & 0xffff0000u);
    g[2] = __uint_as_float(v.y << 16); g[3] = __uint_as_float(v.y & 0xffff0000u);
}
template <typename GT> struct GradFloats;
template <> struct GradFloats<float> { __device__ static __forceinline__ void get(const float4 v, float (&g)[4]) { grad_floats(v, g); } };
template <> struct GradFloats<__half> { __device__ static __forceinline__ void get(const uint2 v, float (&g)[4]) { grad_floats_half(v, g); } };
template <> struct GradFloats<__hip_bfloat16> { __device__ static __forceinline__ void get(const uint2 v, float (&g)[4]) { grad_floats_bf16(v, g); } };

// One (group, slice) unit for a table of D columns: RT tiles of 16 runs, CL loads of 64 columns per bag.
// The contraction runs on the matrix cores in fp32 (v_mfma_f32_16x16x4_f32: 16 runs x 16 columns x 4 bags;
// operand A = counts, lane l holds run l%16 of bag l/16; operand B = gradient, lane l holds one column of
// bag l/16; a lane's gradient load covers columns 4*(l%16)..+3, so tile q of a load takes component q and
// holds columns 4*(l%16)+q; result tile: lane l holds runs 4*(l/16)+i, i = 0..3).  Counts are exact small
// integers, products and sums are fp32: the same arithmetic as adding the gradient row count times.
//
// The count table of the whole slice is one byte per (bag, run), built with LDS integer atomics on the
// containing words.  A bag that holds one row 256 times or more would overflow its byte, and 0 x Inf / NaN of
// a bag's gradient would reach runs the bag does not look up: both cases only set the table's dirty flag;
// the fix-up kernel then ignores the partial rows of that table's dense runs and sums those runs by gathering.
template <typename GT, int RT, int CL>
__device__ __forceinline__ void dense_unit(const DenseArgs& d, const DenseGroup& grp, const TableMeta& m, int j,
                                           uint32_t* __restrict__ s_cnt, int32_t* __restrict__ s_p0,
                                           int32_t* __restrict__ s_pre, int32_t* __restrict__ s_slot,
                                           uint32_t& dirty_bits)
{
    using GIO = GradIO<GT>;
    constexpr int kWaves = kDenseThreads / kWave;
    constexpr int kBagsPerWave = kDenseSlice / kWaves;        // 256 bags = 64 steps of 4
    constexpr int kSteps = kBagsPerWave / 4;
    constexpr int kUnroll = CL == 2 ? 2 : 4;                  // steps whose gradient loads are issued together
    constexpr int kLoads = 8;                                 // payload loads in flight per thread while counting
    const BwdArgs& a = d.b;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = threadIdx.x >> 6;
    const int l16 = lane & 15, kq = lane >> 4;
    const int D = m.dim;
    const int nb = a.dense_slices + 1;
    const int64_t stride = a.table_major ? D : a.sumD;
    const GT* __restrict__ grad_out = static_cast<const GT*>(a.grad_out);
    const GT* gb = a.table_major ? grad_out + (int64_t)a.batch * m.col : grad_out + m.col;
    const int32_t* __restrict__ vals = a.sorted_vals;
    const uint8_t* s_cnt8 = reinterpret_cast<const uint8_t*>(s_cnt);
    const int sl_lo = j * kDenseSlice;
    const int sl_n = min(kDenseSlice, a.batch - sl_lo);       // >= 1

    // ---- count table of the slice
    __syncthreads();
    for (int i = threadIdx.x; i < kDenseSlice * kDenseRows / 16; i += kDenseThreads)
        reinterpret_cast<uint4*>(s_cnt)[i] = make_uint4(0u, 0u, 0u, 0u);
    if (threadIdx.x < kDenseRows) {
        int p0 = 0, cntr = 0, slot = 0;
        if ((int)threadIdx.x < grp.nrows) {
            const int64_t bi = (int64_t)(grp.first + threadIdx.x) * nb + j;
            p0 = d.dbounds[bi];
            cntr = d.dbounds[bi + 1] - p0;
            const int u = (int)d.drun[grp.first + threadIdx.x];
            slot = (a.seg_offsets[u] / kChunk + 1) * 2 + j;
        }
        s_p0[threadIdx.x] = p0;
        s_slot[threadIdx.x] = slot;
        int incl = cntr;   // inclusive prefix over the group's runs inside the first wavefront
#pragma unroll
        for (int o = 1; o < kDenseRows; o <<= 1) {
            const int up = __shfl_up(incl, o);
            if ((int)threadIdx.x >= o)
                incl += up;
        }
        s_pre[threadIdx.x + 1] = incl;
        if (threadIdx.x == 0)
            s_pre[0] = 0;
    }
    __syncthreads();
    const int tot = s_pre[kDenseRows];
    for (int f0 = 0; f0 < tot; f0 += kDenseThreads * kLoads) {
        int rr[kLoads], bb[kLoads];
#pragma unroll
        for (int x = 0; x < kLoads; ++x) {       // all loads are issued before the first atomic
            const int f = f0 + x * kDenseThreads + threadIdx.x;
            int lo = 0, hi = kDenseRows;         // last r with s_pre[r] <= f
#pragma unroll
            for (int st = 0; st < 5; ++st) {
                const int mid = (lo + hi) >> 1;
                if (s_pre[mid] <= f)
                    lo = mid;
                else
                    hi = mid;
            }
            rr[x] = f < tot ? lo : -1;
            bb[x] = f < tot ? vals[s_p0[lo] + (f - s_pre[lo])] : 0;
        }
#pragma unroll
        for (int x = 0; x < kLoads; ++x) {
            if (rr[x] >= 0) {
                const int sh = 8 * (rr[x] & 3);
                const uint32_t old = atomicAdd(&s_cnt[(bb[x] - sl_lo) * (kDenseRows / 4) + (rr[x] >> 2)], 1u << sh);
                if (((old >> sh) & 0xffu) == 0xffu)
                    dirty_bits = 0x7f800000u;    // the byte wrapped around
            }
        }
    }
    __syncthreads();

    for (int cbase = 0; cbase < D; cbase += CL * 64) {
        int coff[CL];
#pragma unroll
        for (int cl = 0; cl < CL; ++cl)
            coff[cl] = min(cbase + cl * 64 + 4 * l16, D - 4);   // columns past D are computed and dropped
        mfma_f4 acc[RT][CL][4];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int cl = 0; cl < CL; ++cl)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    acc[rt][cl][q] = mfma_f4{0.f, 0.f, 0.f, 0.f};

        // ---- counts x gradient rows on the matrix cores; a wavefront takes kBagsPerWave consecutive bags.
        // Bags past the end of the batch have all-zero counts; their gradient operand is the batch's last row.
        const int wbase = wv * kBagsPerWave;
        const uint8_t* ap = s_cnt8 + (wbase + kq) * kDenseRows + l16;
        if (wbase < sl_n) {
            for (int s0 = 0; s0 < kSteps; s0 += kUnroll) {
                typename GIO::Vec raw[kUnroll][CL];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    const int x = min(wbase + (s0 + u) * 4 + kq, sl_n - 1);
                    const GT* rp = gb + (int64_t)(sl_lo + x) * stride;
#pragma unroll
                    for (int cl = 0; cl < CL; ++cl)
                        raw[u][cl] = GIO::ldv(rp + coff[cl]);
                }
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    float av[RT];
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
                        av[rt] = (float)ap[((s0 + u) * 4) * kDenseRows + rt * 16];
#pragma unroll
                    for (int cl = 0; cl < CL; ++cl) {
                        float g[4];
                        GradFloats<GT>::get(raw[u][cl], g);
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            dirty_bits = max(dirty_bits, __float_as_uint(g[q]) & 0x7f800000u);   // Inf / NaN: all ones
#pragma unroll
                            for (int rt = 0; rt < RT; ++rt)
                                acc[rt][cl][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[rt], g[q], acc[rt][cl][q], 0, 0, 0);
                        }
                    }
                }
            }
        }
        // ---- wavefronts of the workgroup, in wavefront order, one tile of 16 runs at a time through LDS.
        // The count table is overwritten: a further column pass (rows wider than CL * 64) builds it again.
        constexpr int kCH = CL < 2 ? CL : 2;                // 64-column loads per pass through LDS
        constexpr int kW = kCH * 64;                        // columns per pass
        float* s_red = reinterpret_cast<float*>(s_cnt);     // [kWaves][16][kW] floats <= 32 KiB
        for (int rt = 0; rt < RT; ++rt) {
            for (int ch = 0; ch < CL; ch += kCH) {
                __syncthreads();
#pragma unroll
                for (int cl = 0; cl < CL; ++cl) {
                    if (cl >= ch && cl < ch + kCH) {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            *reinterpret_cast<float4*>(&s_red[(wv * 16 + 4 * kq + i) * kW + (cl - ch) * 64 + 4 * l16]) =
                                make_float4(acc[rt][cl][0][i], acc[rt][cl][1][i], acc[rt][cl][2][i], acc[rt][cl][3][i]);
                    }
                }
                __syncthreads();
                for (int idx = threadIdx.x; idx < 16 * (kW / 4); idx += kDenseThreads) {
                    const int r = idx / (kW / 4);
                    const int c4 = (idx - r * (kW / 4)) * 4;
                    const int row = rt * 16 + r;
                    const int col = cbase + ch * 64 + c4;
                    if (row < grp.nrows && col < D) {
                        float4 sum = *reinterpret_cast<const float4*>(&s_red[r * kW + c4]);
#pragma unroll
                        for (int w2 = 1; w2 < kWaves; ++w2) {
                            const float4 v = *reinterpret_cast<const float4*>(&s_red[(w2 * 16 + r) * kW + c4]);
                            sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
                        }
                        *reinterpret_cast<float4*>(a.partials + (int64_t)s_slot[row] * a.dpad + col) = sum;
                    }
                }
            }
        }
        if (cbase + CL * 64 < D) {
            // rebuild the count table for the next column pass (only rows wider than 128 columns get here)
            __syncthreads();
            for (int i = threadIdx.x; i < kDenseSlice * kDenseRows / 16; i += kDenseThreads)
                reinterpret_cast<uint4*>(s_cnt)[i] = make_uint4(0u, 0u, 0u, 0u);
            __syncthreads();
            for (int f = threadIdx.x; f < tot; f += kDenseThreads) {
                int lo = 0, hi = kDenseRows;
#pragma unroll
                for (int st = 0; st < 5; ++st) {
                    const int mid = (lo + hi) >> 1;
                    if (s_pre[mid] <= f)
                        lo = mid;
                    else
                        hi = mid;
                }
                const int b = vals[s_p0[lo] + (f - s_pre[lo])];
                atomicAdd(&s_cnt[(b - sl_lo) * (kDenseRows / 4) + (lo >> 2)], 1u << (8 * (lo & 3)));
            }
            __syncthreads();
        }
    }
}

template <typename GT>
__global__ __launch_bounds__(kDenseThreads, 4) void dense_rows_kernel(DenseArgs d)
{
    __shared__ __align__(16) uint32_t s_cnt[kDenseSlice * kDenseRows / 4];   // 32 KiB; reused for the cross-wave sums
    __shared__ int32_t s_p0[kDenseRows], s_pre[kDenseRows + 1], s_slot[kDenseRows];
    const BwdArgs& a = d.b;
    const int ngroups = (int)a.counters->dense_groups;
    const int nslices = a.dense_slices;
    const int total = ngroups * nslices;
    // Work units in an order that keeps the groups of one (table, slice) next to each other, and the
    // workgroups that share an L2 (every 8th one) on neighbouring units: they then read the same piece of
    // the gradient block at about the same time.
    const int xcd = blockIdx.x & 7, nper = gridDim.x >> 3, within = blockIdx.x >> 3;
    const int per_xcd = (total + 7) / 8;
    for (int w = within; w < per_xcd; w += nper) {
        const int unit = xcd * per_xcd + w;
        if (unit >= total)
            break;
        // unit -> (group, slice): the units of table t are [gbase * nslices, (gbase + ng) * nslices), slice-major
        const DenseGroup any = d.dgroup[unit / nslices];
        const int local = unit - any.gbase * nslices;
        const int j = local / any.ng;
        const DenseGroup grp = d.dgroup[any.gbase + (local - j * any.ng)];
        const TableMeta m = a.meta[grp.t];
        uint32_t dirty_bits = 0;
        // 128 columns per pass (64 for narrow tables); wider rows take further passes over the same bags
        if (grp.nrows > 16) {
            if (m.dim > 64)
                dense_unit<GT, 2, 2>(d, grp, m, j, s_cnt, s_p0, s_pre, s_slot, dirty_bits);
            else
                dense_unit<GT, 2, 1>(d, grp, m, j, s_cnt, s_p0, s_pre, s_slot, dirty_bits);
        } else {
            if (m.dim > 64)
                dense_unit<GT, 1, 2>(d, grp, m, j, s_cnt, s_p0, s_pre, s_slot, dirty_bits);
            else
                dense_unit<GT, 1, 1>(d, grp, m, j, s_cnt, s_p0, s_pre, s_slot, dirty_bits);
        }
        if (__ballot(dirty_bits == 0x7f800000u) != 0ull && (threadIdx.x & (kWave - 1)) == 0)
            atomicOr(&a.dense_dirty[grp.t], 1u);
    }
}

// ---------------------------------------------------------------- long runs in pieces
//
// By position (the gradient block fits an L2): pieces of kPosPiece lookups, one wavefront each.  In a small call
// what counts is the length of the chain a wavefront follows -- four rows in flight per lane group, so 128
// lookups of a 512-column row are 32 trips to the L2, about 20 us -- and that there are pieces for every CU.
//
// By bag window, beyond that:
// A run of kLongRun < L <= dense threshold lookups is cut into pieces by bag window (the batch is divided
// into at most kWinMax windows of win_bags bags); the payloads of a run ascend by bag, so a piece is a
// contiguous part of the run.  One wavefront sums one piece (one gathered gradient row per lookup) and
// writes one fp32 partial row; the fix-up kernel adds a run's partial rows in window order.  Pieces are
// processed table by table, window by window, run by run, and the wavefronts that share an L2 work on
// neighbouring pieces: the gradient rows they gather then come from one window of one table's gradient
// block (2 MiB for 128 fp32 columns) instead of from all of it, and are mostly found in L2.
// The partial rows of a run live in the slots of the chunks it covers completely (two per chunk).  A run
// too short to own kWinMax slots merges neighbouring windows in pairs or fours (8 or 4 pieces).

// Bag windows of a table with D columns: about 2 MiB of its gradient block each (a power of two of at least
// 1024 bags), at most kWinMax windows per batch.
struct WinGeom {
    int bags, nwin;
};

__device__ __forceinline__ WinGeom window_geom(int batch, int D, int grad_bytes)
{
    WinGeom g;
    g.bags = 1024;
    while (g.bags * 2 * D * grad_bytes <= (2 << 20))
        g.bags <<= 1;
    g.nwin = (batch + g.bags - 1) / g.bags;
    if (g.nwin > kWinMax) {
        g.bags = ((batch + kWinMax - 1) / kWinMax + 1023) / 1024 * 1024;
        g.nwin = (batch + g.bags - 1) / g.bags;
    }
    g.nwin = max(g.nwin, 1);
    return g;
}

// pieces a run of sorted positions [s, e) is cut into: as many windows as it has slots for, as a power of two
__device__ __forceinline__ int window_step(int s, int e, int nwin)
{
    const int slots = 2 * ((e - 1) / kChunk - s / kChunk - 1);     // >= 6 for a run longer than kLongRun
    int step = 1;                                                  // windows per piece
    while ((nwin + step - 1) / step > slots)
        step <<= 1;
    return step;
}

// one workgroup: exclusive prefixes of the per-table queue lengths (wpre[T] = number of windowed runs) and of
// the per-table piece counts, runs x windows (ppre[T] = number of pieces); clears the queue lengths and the
// piece-claim counters for this update
__global__ __launch_bounds__(256) void window_plan_kernel(BwdArgs a, uint32_t* __restrict__ wpre,
                                                          uint32_t* __restrict__ ppre)
{
    __shared__ uint32_t s_wave[4];
    uint32_t carry = 0, carry_p = 0;
    for (int base = 0; base < a.T; base += 256) {
        const int t = base + threadIdx.x;
        const uint32_t c = t < a.T ? a.win_cnt[t] : 0u;
        const uint32_t np = t < a.T ? c * (uint32_t)window_geom(a.batch, a.meta[t].dim, a.grad_bytes).nwin : 0u;
        uint32_t tot, tot_p;
        const uint32_t ex = block_exclusive_scan_256(c, s_wave, tot);
        const uint32_t ex_p = block_exclusive_scan_256(np, s_wave, tot_p);
        if (t < a.T) {
            wpre[t] = carry + ex;
            ppre[t] = carry_p + ex_p;
            if (c > 0)
                a.win_cnt[t] = 0;
        }
        carry += tot;
        carry_p += tot_p;
    }
    if (threadIdx.x == 0) {
        wpre[a.T] = carry;
        ppre[a.T] = carry_p;
        a.counters->win_runs = carry;
        a.counters->win_pieces = carry_p;
    }
    if (threadIdx.x < 8)
        a.counters->win_next[threadIdx.x][0] = 0;
}

// Sixteen lanes per windowed run (four runs per wavefront): where the run's payloads (ascending bags) cross the
// window borders, written as the run's piece records.  Run ri belongs to the table t with wpre[t] <= ri <
// wpre[t + 1] and is entry ri - wpre[t] of that table's queue; the pieces of table t are
// [ppre[t], ppre[t + 1]), window-major, run-minor.
__global__ __launch_bounds__(256) void window_pieces_kernel(BwdArgs a, const uint32_t* __restrict__ wpre,
                                                            const uint32_t* __restrict__ ppre)
{
    static_assert(kWinMax == 16, "one 16-lane group per run");
    const int lane = threadIdx.x & (kWave - 1);
    const int sub = lane & 15;
    const int nruns = (int)wpre[a.T];
    const int32_t* __restrict__ vals = a.sorted_vals;
    const int groups_total = gridDim.x * (256 / 16);
    for (int ri0 = (blockIdx.x * 256 + (int)threadIdx.x) >> 4; ri0 - (ri0 & 3) < nruns; ri0 += groups_total) {
        const bool live = ri0 < nruns;               // the four groups of a wavefront stay together for the shuffle
        const int ri = live ? ri0 : nruns - 1;
        int t0 = 0, t1 = a.T;                        // wpre[t0] <= ri < wpre[t1]
        while (t1 - t0 > 1) {
            const int mid = (t0 + t1) >> 1;
            if ((int)wpre[mid] <= ri)
                t0 = mid;
            else
                t1 = mid;
        }
        const int gbase = (int)wpre[t0], ng = (int)wpre[t0 + 1] - gbase;
        const WinGeom wg = window_geom(a.batch, a.meta[t0].dim, a.grad_bytes);
        const int nwin = wg.nwin;
        const int u = (int)a.win_list[a.tstart[t0] / kLongRun + t0 + (ri - gbase)];
        const int s = a.seg_offsets[u];
        const int e = a.seg_offsets[u + 1];
        const int step = window_step(s, e, nwin);
        int bound = e;                               // first p in [s, e) with vals[p] >= sub * win_bags
        if (sub < nwin) {
            const int target = sub * wg.bags;
            int lo = s, hi = e;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (vals[mid] < target)
                    lo = mid + 1;
                else
                    hi = mid;
            }
            bound = lo;
        }
        const int up = __shfl(bound, (lane & ~15) | min(sub + step, 15));
        if (live && sub < nwin) {
            WinPiece p;
            p.p0 = bound;
            p.p1 = sub + step >= nwin ? e : up;
            p.slot = sub % step == 0 ? (s / kChunk + 1) * 2 + sub / step : -1;
            p.t = t0;
            a.pieces[(int64_t)ppre[t0] + (int64_t)sub * ng + (ri - gbase)] = p;
        }
    }
}

template <typename GT>
__global__ __launch_bounds__(kBwdThreads) void window_runs_kernel(BwdArgs a)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int total = (int)a.counters->win_pieces;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.counters->long_todo = a.counters->long_count;
        a.counters->long_count = 0;
    }
    // The workgroups that share an L2 (every 8th block) take the pieces of one eighth of the list.
    const int xcd = blockIdx.x & 7;
    const int per_xcd = (total + 7) / 8;
    if (a.by_position) {
        // pieces of equal length over a gradient block that fits an L2: a fixed assignment, wavefront by wavefront
        const int step = (int)(gridDim.x >> 3) * (kBwdThreads / kWave);
        for (int w = uniform((int)(blockIdx.x >> 3) * (kBwdThreads / kWave) + (int)(threadIdx.x >> 6)); w < per_xcd; w += step) {
            const int piece = xcd * per_xcd + w;
            if (piece >= total)
                break;
            sum_piece<GT>(a, *reinterpret_cast<const int4*>(&a.pieces[piece]));
        }
        return;
    }
    // By bag window: kWinBatch consecutive unclaimed pieces at a time (one integer atomic per batch; the wavefronts
    // of the workgroup then share the batch out through LDS): whatever the pieces' lengths, the wavefronts of an L2
    // domain are always at work on neighbouring pieces.  Which wavefront sums a piece has no influence on the result.
    __shared__ int s_batch, s_taken;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) {
            s_batch = (int)atomicAdd(&a.counters->win_next[xcd][0], (uint32_t)kWinBatch);
            s_taken = 0;
        }
        __syncthreads();
        const int batch0 = s_batch;
        if (batch0 >= per_xcd)
            break;
        for (;;) {
            int w = 0;
            if (lane == 0)
                w = atomicAdd(&s_taken, 1);
            w = uniform(w);
            if (w >= kWinBatch || batch0 + w >= per_xcd)
                break;
            const int piece = xcd * per_xcd + batch0 + w;
            if (piece >= total)
                break;
            const int4 rec = *reinterpret_cast<const int4*>(&a.pieces[piece]);
            if (rec.z >= 0)          // < 0: merged into the piece that starts at an earlier window
                sum_piece<GT>(a, rec);
        }
    }
}

// One wavefront per queued long run: adds the run's partial rows in order (one per bag slice of a dense
// run, one per window piece otherwise) and applies the run's single optimizer step.
template <typename WT, typename GT, int OPT>
__global__ __launch_bounds__(kBwdThreads) void long_run_fixup_kernel(BwdArgs a)
{
    using IO = RowIO<WT, 4>;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave_global = uniform(blockIdx.x * (kBwdThreads / kWave) + (threadIdx.x >> 6));
    const int wave_total = gridDim.x * (kBwdThreads / kWave);
    WT* __restrict__ weights = static_cast<WT*>(a.weights);
    float acc[2][4];
    auto fix = [&](uint32_t key, int t, int s, int e) {
        const bool dense = e - s > a.dense_thr;
        const TableMeta m = a.meta[t];
        const Cols c(m.dim, m.lpr_bwd(), lane);
        const int k0 = s / kChunk;
        const float* pbase = a.partials;
        const int64_t dpad = a.dpad;
        const int64_t wel = m.woff + (int64_t)(key - m.rbase) * m.dim;
        WT* wrow = weights + wel;
        typename IO::Vec wvv[2];
        wvv[0] = IO::ldv(wrow + c.e0);
        wvv[1] = IO::ldv(wrow + c.e1);
        OptRow<OPT> st;
        st.load(a.opt, key, wel, c);
        if (a.by_position && !dense) {
            const int np = position_pieces(e - s);
            wave_gather_sum<float>([&](int cc) { return pbase + (int64_t)(position_of_piece(s, e - s, np, cc) / kPosSlot) * dpad; },
                                   0, np, a.zero_row, c, acc);
        } else if (dense && a.dense_dirty[t] != 0u) {
            // the table's gradient block holds Inf / NaN, which the dense sums leave out: this run is
            // summed the plain way, one gathered gradient row per lookup (a rare, slow path)
            const GT* gb = a.table_major ? static_cast<const GT*>(a.grad_out) + (int64_t)a.batch * m.col
                                         : static_cast<const GT*>(a.grad_out) + m.col;
            const int64_t gstride = a.table_major ? m.dim : a.sumD;
            const int32_t* __restrict__ vals = a.sorted_vals;
            wave_gather_sum<GT>([&](int i) { return gb + (int64_t)vals[i] * gstride; }, s, e, a.zero_row, c, acc);
        } else if (dense) {
            // one partial row per slice of bags, kept in the slots of the chunks the run covers completely
            wave_gather_sum<float>([&](int cc) { return pbase + ((int64_t)(k0 + 1) * 2 + cc) * dpad; }, 0,
                                   a.dense_slices, a.zero_row, c, acc);
        } else {
            const int nwin = window_geom(a.batch, m.dim, a.grad_bytes).nwin;
            const int step = window_step(s, e, nwin);
            wave_gather_sum<float>([&](int cc) { return pbase + ((int64_t)(k0 + 1) * 2 + cc) * dpad; }, 0,
                                   (nwin + step - 1) / step, a.zero_row, c, acc);
        }
        optimizer_epilogue<WT, OPT>(wrow, wvv, acc, m.dim, c, c.grp == 0, a.opt, key, wel, st);
    };
    const int cnt = (int)a.counters->long_todo;
    if (blockIdx.x == 0 && threadIdx.x == 0)
        a.counters->win_pieces = 0;
    for (int i = wave_global; i < cnt; i += wave_total) {
        const LongRun rec = a.long_list[i];
        fix(rec.key, rec.t, rec.s, rec.e);
    }
}

// ---------------------------------------------------------------- input validation (slow path)

__global__ __launch_bounds__(256) void check_inputs_kernel(
    const TableMeta* __restrict__ meta, const uint32_t* __restrict__ row_base,
    const int32_t* __restrict__ indices, const int64_t* __restrict__ offsets, int64_t num_indices,
    int32_t B, int32_t num_bags, Counters* __restrict__ counters)
{
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= num_bags)
        return;
    uint32_t flags = 0;
    const int64_t lo = offsets[j], hi = offsets[j + 1];
    if ((j == 0 && lo != 0) || (j == num_bags - 1 && hi != num_indices) || lo > hi || lo < 0 ||
        hi > num_indices) {
        flags |= 1u;
    } else {
        const int t = j / B;
        const int64_t H = (int64_t)row_base[t + 1] - (int64_t)row_base[t];
        for (int64_t p = lo; p < hi; ++p) {
            const int64_t r = indices[p];
            if (r < 0 || r >= H)
                flags |= 2u;
        }
    }
    (void)meta;
    if (flags)
        atomicOr(&counters->check_flags, flags);
}

__global__ void clear_num_unique_kernel(Counters* counters) { counters->num_unique = 0; }

__global__ void clear_check_flags_kernel(Counters* counters) { counters->check_flags = 0; }

}  // namespace tbe
