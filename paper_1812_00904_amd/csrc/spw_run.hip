// Multi-RHS column dots for gfx950, the run kernel: one chunk per wave, column
// lanes x positions of one run.  The columns without nonzeros and the zone sums are
// done by the caller (spw_tile.hip).  Shared helpers: spw_device.h.
#include <type_traits>

#include "spw_device.h"

namespace spw {
namespace {

// ------------------------------------------------------------------------
// Multi-RHS column dots: U = C^T V for up to 64 right-hand sides.
//
// One wave takes a chunk of 64*ITEMS positions for all k <= L*CW columns.  Lane
// s*L + cl holds columns cl*CW .. of position S*t + s of step t (S = 64 / L): S
// nonzeros a step, each against L*CW adjacent entries of its row of V.  All of them
// belong to the same run of a column but for the steps that a column start falls
// into, so the walk is the same for the whole wave: column starts are scalar bit
// tests, a step without one is one gather and CW fused multiply-adds a lane, and
// only a start costs more (its step is split by lane masks and the finished sums
// join a queue).  Finished columns are added across the S position rows of the wave
// four at a time (two for S = 2) and go out in one store.
//
// What bounds it: over the matrix's own storage, whose V mostly comes from the L2 (63 to 82 % hits),
// the L1.  A gather of 64 x 16 bytes takes 16 cycles to read out and, where
// its lines miss (nearly all: V is far larger), as many to fill, whatever its lanes read, so
// a lane reads 16 bytes where the block is wide enough; after that the column starts, about
// 15 vector and 25 scalar instructions each.  A fill and a read of every gathered byte at 64
// bytes a cycle and CU are 1.3 ms for k = 64 on 20,000 x 5e6 with 5e7 nonzeros, where this
// takes 1.75 (cdot_tile, whose lanes test every position: 2.18); k = 16 0.56 (0.77), k = 32
// 0.94 (1.21).  Over the blocked transpose of 20,000 x 2e6 with 2e7: binary64 k = 16 0.35
// (0.57), k = 64 1.37 (1.53), binary32 k = 16 0.32 (0.40), k = 32 0.33 (0.51).  There nearly every
// gathered row comes from beyond the L2 (8 to 18 % hits), and the rate of that is the bound: 20,000 x
// 5e6, 5e7 nonzeros, k = 64 25.3 GB in 3.42 ms, binary32 k = 16 5.9 GB in 0.80 ms, 7.4 TB/s.
//
// The indices and values go through LDS, 256 positions at a time: a batch of 16 (8
// for S = 2) consecutive positions is stored as [s][t], so that a lane reads its
// positions of a batch with wide reads, and the next 256 are fetched into a dozen
// registers while these are walked (a whole chunk in registers cost a wave per SIMD).
// ------------------------------------------------------------------------
constexpr int RUN_BLOCK = 256;
constexpr int RUN_POS = 256;                    // positions staged at a time
// positions per batch, and the LDS bytes of a batch's rows and values (padded against bank conflicts)
template <int L> constexpr int run_batch() { return WAVE / L == 2 ? 8 : 16; }
template <int L> constexpr int run_off() { return run_batch<L>() * 4 + 16; }
template <int L> constexpr int run_val() { return run_batch<L>() * 8 + 16; }
template <int L> constexpr int run_stage_bytes() { return RUN_POS / run_batch<L>() * (run_off<L>() + run_val<L>()); }

// CW consecutive entries of a row of V, aligned to one entry.
template <typename VecT, int CW> struct VecRow {
    VecT v[CW];
    __device__ __forceinline__ void load(const VecT *p)
    {
        if constexpr (CW == 1) {
            v[0] = *p;
        } else {
            typedef VecT vec_u __attribute__((ext_vector_type(CW), aligned(sizeof(VecT))));
            const vec_u w = *reinterpret_cast<const vec_u *>(p);
#pragma unroll
            for (int i = 0; i < CW; ++i) v[i] = w[i];
        }
    }
};

// Adds the two 32-lane halves of a wave: lane l gets x(l) + x(l xor 32).
__device__ __forceinline__ double add_halves(double x)
{
    const uint64_t a = __builtin_bit_cast(uint64_t, x);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)a, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(a >> 32), false, false);
    return __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) +
           __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
}

// A wave's LDS of cdot_run: the staged positions, then the queue of four finished columns.
template <int L, int CW> constexpr int run_wave_lds() { return run_stage_bytes<L>() + 4 * WAVE * CW * 8; }
// Resident workgroups per CU to leave registers for.
template <int L, int CW> constexpr int run_wgs() { return CW == 4 ? 3 : L == 8 ? 5 : 4; }

// Elements e of a 16-byte group of stored values or indices.
template <typename ValT> struct RunVal;
template <> struct RunVal<double> {
    f64x2_t w;
    __device__ __forceinline__ void load(const double *p) { w = __builtin_nontemporal_load(reinterpret_cast<const f64x2_t *>(p)); }
    __device__ __forceinline__ double get(int e) const { return w[e]; }
};
template <> struct RunVal<float> {
    f32x4_t w;
    __device__ __forceinline__ void load(const float *p) { w = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t *>(p)); }
    __device__ __forceinline__ double get(int e) const { return (double)w[e]; }
};
template <> struct RunVal<Bf16> {
    u32x4_t w;
    __device__ __forceinline__ void load(const Bf16 *p) { w = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p)); }
    __device__ __forceinline__ double get(int e) const { return bf16_bits_to_f64((w[e >> 1] >> ((e & 1) * 16)) & 0xFFFFu); }
};
template <typename IdxT> struct RunIdx {
    u32x4_t w;
    __device__ __forceinline__ void load(const IdxT *p) { w = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p)); }
    __device__ __forceinline__ uint32_t get(int e) const
    {
        if constexpr (sizeof(IdxT) == 2) return (w[e >> 1] >> ((e & 1) * 16)) & 0xFFFFu;
        else return w[e];
    }
};

// OutT: the type of U (binary64 partial sums for binary32 inputs, or VecT).
// V: rows of ldv entries.  k <= L*CW.
template <typename IdxT, typename ValT, typename VecT, int ITEMS, int L, int CW, typename OutT>
__global__ __launch_bounds__(RUN_BLOCK, (run_wgs<L, CW>())) void cdot_run(
    const IdxT *__restrict__ idx, const ValT *__restrict__ val, const uint16_t *__restrict__ heads,
    const int4 *__restrict__ cinfo, const int32_t *__restrict__ segcol, int64_t nnz, int nchunks, int k,
    const VecT *__restrict__ V, int64_t ldv, OutT *__restrict__ U, int64_t ldu,
    double *__restrict__ carry)
{
    constexpr int S = WAVE / L;                   // positions per step
    constexpr int BP = run_batch<L>(), T = BP / S;            // positions and steps per batch
    constexpr int WCH = WAVE * ITEMS;             // positions per chunk
    constexpr int LPS = RUN_POS / ITEMS;          // layout lanes per stage
    constexpr int NW = RUN_BLOCK / WAVE;
    constexpr int QUEUE = 4;
    static_assert(S == 2 || S == 4 || S == 8, "32, 16 or 8 column lanes");
    __shared__ __attribute__((aligned(16))) char lds_all[NW * run_wave_lds<L, CW>()];

    const int lane = threadIdx.x & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int s = lane / L, cl = lane % L;
    typedef __attribute__((address_space(3))) char lds_char;
    typedef __attribute__((address_space(3))) uint32_t lds_u1;
    typedef __attribute__((address_space(3))) double lds_d1;
    lds_char *off_lds = (lds_char *)(lds_all + wave * run_wave_lds<L, CW>());
    lds_char *val_lds = off_lds + RUN_POS / BP * run_off<L>();
    lds_d1 *queue = (lds_d1 *)(off_lds + run_stage_bytes<L>());

    const int stride = gridDim.x * NW;
    int c = blockIdx.x * NW + wave;
    if (c >= nchunks) return;

    // A stage's 16-byte groups: group u holds elements gi*G .. of layout lane ll = u mod LPS,
    // gi = u / LPS, which are consecutive positions; they go to the lanes in turn.
    constexpr int GV = ValGroup<ValT>::G, GI = 16 / (int)sizeof(IdxT);
    constexpr int UV = RUN_POS / GV, UI = RUN_POS / GI;       // groups of values and of indices
    constexpr int NV = (UV + WAVE - 1) / WAVE, NI = (UI + WAVE - 1) / WAVE;
    RunVal<ValT> A[NV];
    RunIdx<IdxT> R[NI];
    auto fetch = [&](int c, int h) __attribute__((always_inline)) {
        const int64_t at = (int64_t)c * WCH;
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int u = j * WAVE + lane;
            if (UV % WAVE == 0 || u < UV) A[j].load(val + at + ((u / LPS) * WAVE + h * LPS + u % LPS) * GV);
        }
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int u = j * WAVE + lane;
            if (UI % WAVE == 0 || u < UI) R[j].load(idx + at + ((u / LPS) * WAVE + h * LPS + u % LPS) * GI);
        }
    };
    // rows as byte offsets (2-byte rows: below 2^32) or row numbers
    constexpr bool SMALL = sizeof(IdxT) == 2;
    const uint32_t ld_bytes = (uint32_t)(ldv * (int64_t)sizeof(VecT));
    // place of position p of the stage, which is the first of a group of consecutive ones
    auto slot = [](int p, int e) { return (((p + e) % BP) % S) * T + ((p + e) % BP) / S; };
    auto stage = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int u = j * WAVE + lane, p = (u % LPS) * ITEMS + (u / LPS) * GV;
            if (UV % WAVE == 0 || u < UV) {
                lds_d1 *d = (lds_d1 *)(val_lds + (p / BP) * run_val<L>());
#pragma unroll
                for (int e = 0; e < GV; ++e) d[slot(p, e)] = A[j].get(e);
            }
        }
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int u = j * WAVE + lane, p = (u % LPS) * ITEMS + (u / LPS) * GI;
            if (UI % WAVE == 0 || u < UI) {
                lds_u1 *d = (lds_u1 *)(off_lds + (p / BP) * run_off<L>());
#pragma unroll
                for (int e = 0; e < GI; ++e) d[slot(p, e)] = SMALL ? R[j].get(e) * ld_bytes : R[j].get(e);
            }
        }
    };

    fetch(c, 0);
    uint32_t heads_next = heads[(int64_t)c * WAVE + lane];
    for (;;) {
        const int cn = c + stride < nchunks ? c + stride : c;
        const int4 cv = cinfo[c];
        const int jlo = __builtin_amdgcn_readfirstlane(cv.x), seg0 = __builtin_amdgcn_readfirstlane(cv.y);
        const int nseg = __builtin_amdgcn_readfirstlane(cv.z), flags = __builtin_amdgcn_readfirstlane(cv.w);
        const int n = (int)min((int64_t)WCH, nnz - (int64_t)c * WCH);
        const int c0 = cl * CW;                   // first column of this lane
        const bool colok = c0 < k;
        // lanes past the last column read the last group of CW columns; their sums go nowhere
        const int vc = colok ? c0 : (k - 1) / CW * CW;
        const uint32_t lane_off = (uint32_t)(vc * (int)sizeof(VecT));

        const int64_t lane_u = (S == 2 ? s : s & 3) * ldu + c0;   // this lane's place in a group of output rows
        double acc[CW];
#pragma unroll
        for (int w = 0; w < CW; ++w) acc[w] = 0.0;
        int queued = 0, qseg = 0;                 // finished columns in the queue, segment of the first
        const uint32_t head_word = lane == 0 ? heads_next & ~1u : heads_next;
        heads_next = heads[(int64_t)cn * WAVE + lane];

        auto put = [&](OutT *p, const double *v) __attribute__((always_inline)) {
            if (c0 + CW <= k) {
                typedef OutT out_u __attribute__((ext_vector_type(CW), aligned(sizeof(OutT))));
                if constexpr (CW == 1) {
                    *p = (OutT)v[0];
                } else {
                    out_u o;
#pragma unroll
                    for (int w = 0; w < CW; ++w) o[w] = (OutT)v[w];
                    *reinterpret_cast<out_u *>(p) = o;
                }
            } else {
#pragma unroll
                for (int w = 0; w < CW; ++w)
                    if (c0 + w < k) p[w] = (OutT)v[w];
            }
        };
        // one queued column's CW sums, over the position rows r0 .. r0+ROWS-1
        constexpr int ROWS = S < 4 ? S : 4;
        const int r0 = S == 8 ? (s >> 2) * 4 : 0;
        auto queue_sum = [&](int i, double *t) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < ROWS; ++r)
#pragma unroll
                for (int w = 0; w < CW; ++w) {
                    const double x = queue[(i * WAVE + (r0 + r) * L + cl) * CW + w];
                    t[w] = r == 0 ? x : t[w] + x;
                }
            if constexpr (S == 8) {
#pragma unroll
                for (int w = 0; w < CW; ++w) t[w] = add_halves(t[w]);
            }
        };
        // the queued segments out: segment qseg + i by the lanes with s = i mod 4
        const bool dense = (flags & CHUNK_DENSE) != 0;
        auto flush = [&]() __attribute__((always_inline)) {
            qseg = __builtin_amdgcn_readfirstlane(qseg);
            const bool first_cut = qseg == 0 && !(flags & CHUNK_START_HEAD);
            const bool last_cut = qseg + queued == nseg && (flags & CHUNK_END_CONT);
            const bool plain = dense && !first_cut && !last_cut;
            OutT *urow = U + (int64_t)(jlo + qseg) * ldu;      // the same for the whole wave
#pragma unroll
            for (int h = 0; h < (S == 2 ? 2 : 1); ++h) {
                const int i = S == 2 ? 2 * h + s : s & 3;
                double t[CW];
                queue_sum(i, t);
                if (plain) {
                    if (i < queued && colok && s < 4) put(urow + lane_u + (S == 2 ? 2 * h * ldu : 0), t);
                } else if (i < queued && colok && s < 4) {
                    // a segment cut on both sides (the chunk lies inside one column) is the left carry
                    const int q = qseg + i;
                    double *cr = nullptr;
                    if (first_cut && q == 0) cr = carry + (2 * (int64_t)c) * k;
                    else if (last_cut && q == nseg - 1) cr = carry + (2 * (int64_t)c + 1) * k;
                    if (cr) {
#pragma unroll
                        for (int w = 0; w < CW; ++w)
                            if (c0 + w < k) cr[c0 + w] = t[w];
                    } else {
                        const int64_t col = dense ? (int64_t)jlo + q : (int64_t)segcol[seg0 + q];
                        put(U + col * ldu + c0, t);
                    }
                }
            }
            qseg += queued;
            queued = 0;
        };
        auto push = [&](const double *v) __attribute__((always_inline)) {
#pragma unroll
            for (int w = 0; w < CW; ++w) queue[(queued * WAVE + lane) * CW + w] = v[w];
            if (++queued == QUEUE) flush();
        };

        struct Batch {
            double a[T];
            VecRow<VecT, CW> g[T];
        };
        Batch B0, B1;
        uint32_t o[T];                            // rows of the batch that is gathered next
        auto read_rows = [&](int b) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < T; ++t) o[t] = *((const lds_u1 *)(off_lds + b * run_off<L>()) + s * T + t);
        };
        auto gather = [&](Batch &B, int b) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                if constexpr (SMALL)
                    B.g[t].load(reinterpret_cast<const VecT *>(reinterpret_cast<const char *>(V) +
                                                               (o[t] + lane_off)));
                else
                    B.g[t].load(V + (int64_t)(int32_t)o[t] * ldv + vc);
            }
#pragma unroll
            for (int t = 0; t < T; ++t) B.a[t] = *((const lds_d1 *)(val_lds + b * run_val<L>()) + s * T + t);
        };
        // lanes of the position rows lo .. hi-1 take step t of the batch; a branch, not a
        // select (the empty statement keeps it one), so that the others run nothing
        auto take = [&](const Batch &B, int t, int lo, int hi) __attribute__((always_inline)) {
            if ((unsigned)(lane - lo * L) < (unsigned)((hi - lo) * L)) {
#pragma unroll
                for (int w = 0; w < CW; ++w) {
                    acc[w] = __fma_rn(B.a[t], (double)B.g[t].v[w], acc[w]);
                    asm volatile("" : "+v"(acc[w]));
                }
            }
        };
        auto compute = [&](const Batch &B, uint32_t m) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                uint32_t hb = (m >> (S * t)) & ((1u << S) - 1u);
                if (hb == 0) {
#pragma unroll
                    for (int w = 0; w < CW; ++w) acc[w] = __fma_rn(B.a[t], (double)B.g[t].v[w], acc[w]);
                } else {
                    // every start closes the open column after the positions before it
                    int lo = 0;
                    do {
                        const int hi = __builtin_ctz(hb);
                        take(B, t, lo, hi);
                        push(acc);
#pragma unroll
                        for (int w = 0; w < CW; ++w) acc[w] = 0.0;
                        lo = hi;
                        hb &= hb - 1;
                    } while (hb);
                    take(B, t, lo, S);
                }
            }
        };
        // column starts of the batch at position p0; the first position after the last
        // nonzero of a short chunk counts as one, so that the padding after it stays out of
        // every column
        auto starts = [&](int p0) __attribute__((always_inline)) -> uint32_t {
            uint32_t m = (uint32_t)__builtin_amdgcn_readlane((int)head_word, p0 / ITEMS);
            if constexpr (BP < ITEMS) m = (m >> (p0 % ITEMS)) & ((1u << BP) - 1u);
            if constexpr (BP > ITEMS) m |= (uint32_t)__builtin_amdgcn_readlane((int)head_word, p0 / ITEMS + 1) << ITEMS;
            if ((unsigned)(n - p0) < (unsigned)BP) m |= 1u << (n - p0);
            return m;
        };
        for (int h = 0; h * RUN_POS < n; ++h) {
            wave_sync();                          // the reads of the previous stage are done
            stage();
            wave_sync();
            const bool more = (h + 1) * RUN_POS < n;
            fetch(more ? c : cn, more ? h + 1 : 0);
            const int p0 = h * RUN_POS, last = (min(n - p0, RUN_POS) - 1) / BP;
            read_rows(0);
            gather(B0, 0);
            read_rows(min(1, last));
            gather(B1, min(1, last));
            read_rows(min(2, last));
            for (int b = 0;; b += 2) {
                compute(B0, starts(p0 + b * BP));
                gather(B0, min(b + 2, last));
                read_rows(min(b + 3, last));
                if (b + 1 > last) break;
                compute(B1, starts(p0 + (b + 1) * BP));
                gather(B1, min(b + 3, last));
                read_rows(min(b + 4, last));
                if (b + 2 > last) break;
            }
        }
        if (n % BP == 0) push(acc);               // the last column; a short batch pushed it at its end
        if (queued > 0) flush();
        if (c + stride >= nchunks) break;
        c += stride;
    }
}

// The rows of a k-wide block, renumbered (inv NULL: as they are) and padded to ldo entries.
__global__ void gather_padded(const int32_t *__restrict__ inv, int64_t rows, int k, const double *__restrict__ in,
                              int64_t ldv, double *__restrict__ out, int ldo)
{
    const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (g >= rows * k) return;
    const int64_t r = g / k;
    const int cc = (int)(g - r * k);
    out[r * ldo + cc] = in[(int64_t)(inv ? inv[r] : r) * ldv + cc];
}

template <int ITEMS, int L, int CW, typename IdxT, typename ValT, typename VecT, typename OutT>
int launch_run_shape(const spw_matrix_s &A, const ColDot &C, int k, const VecT *V, int64_t ldv, OutT *U,
                     int64_t ldu, hipStream_t stream)
{
    auto kern = cdot_run<IdxT, ValT, VecT, ITEMS, L, CW, OutT>;
    // persistent: as many workgroups as the chip keeps resident
    static const int per_cu = [&] {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void *)kern, RUN_BLOCK, 0) != hipSuccess || nb < 1) {
            (void)hipGetLastError();
            nb = 1;
        }
        return nb;
    }();
    const int64_t want = (C.zp.n_chunks + RUN_BLOCK / WAVE - 1) / (RUN_BLOCK / WAVE);
    const unsigned grid =
        (unsigned)std::max<int64_t>(1, std::min<int64_t>((int64_t)device_cu_count(A.device) * per_cu, want));
    hipLaunchKernelGGL(kern, dim3(grid), dim3(RUN_BLOCK), 0, stream, (const IdxT *)C.d_idx, (const ValT *)C.d_val,
                       C.d_heads, (const int4 *)C.d_cinfo, C.d_segcol, C.nnz, (int)C.zp.n_chunks, k, V, ldv, U, ldu,
                       A.scratch.carry);
    return (int)hipGetLastError();
}

// The narrowest group of 16, 32 or 64 columns that holds k, in lanes of 16 bytes (8 for
// binary32 up to 16 columns: eight positions a step instead of sixteen).
template <int ITEMS, typename IdxT, typename ValT, typename VecT, typename OutT>
int launch_run(const spw_matrix_s &A, const ColDot &C, int k, const VecT *V, int64_t ldv, OutT *U,
               int64_t ldu, hipStream_t stream)
{
    if (k <= 16) return launch_run_shape<ITEMS, 8, 2, IdxT, ValT, VecT, OutT>(A, C, k, V, ldv, U, ldu, stream);
    if constexpr (sizeof(VecT) == 8) {
        if (k <= 32)
            return launch_run_shape<ITEMS, 16, 2, IdxT, ValT, VecT, OutT>(A, C, k, V, ldv, U, ldu, stream);
        return launch_run_shape<ITEMS, 32, 2, IdxT, ValT, VecT, OutT>(A, C, k, V, ldv, U, ldu, stream);
    } else {
        if (k <= 32)
            return launch_run_shape<ITEMS, 8, 4, IdxT, ValT, VecT, OutT>(A, C, k, V, ldv, U, ldu, stream);
        return launch_run_shape<ITEMS, 16, 4, IdxT, ValT, VecT, OutT>(A, C, k, V, ldv, U, ldu, stream);
    }
}

// The matrix's own column dots, binary64 vectors: over a copy of the short block whose rows
// are renumbered and padded to the power of two.
template <typename IdxT, typename ValT>
int run_own(const spw_matrix_s &A, const ColDot &C, const int32_t *inv, int k, const double *V, int64_t ldv, double *U,
            int64_t ldu, hipStream_t stream)
{
    const int32_t width = coldot_tile_width(k);
    if (A.scratch.kcap < width) return (int)hipErrorInvalidValue;
    double *vp = A.scratch.vperm;
    hipLaunchKernelGGL(gather_padded, dim3(blocks_for(C.rows * k, 256)), dim3(256), 0, stream, inv, C.rows, k, V,
                       ldv, vp, (int)width);
    int e = (int)hipGetLastError();
    if (e) return e;
    if (C.zp.chunk == 1024) return launch_run<16, IdxT, ValT, double, double>(A, C, k, vp, width, U, ldu, stream);
    if (C.zp.chunk == 512) return launch_run<8, IdxT, ValT, double, double>(A, C, k, vp, width, U, ldu, stream);
    return (int)hipErrorNotSupported;
}

// The kept transpose, over the caller's own block.
template <typename ValT, typename VecT, typename OutT>
int run_transpose(const spw_matrix_s &A, const ColDot &C, int k, const VecT *V, int64_t ldv, OutT *U, int64_t ldu,
                  hipStream_t stream)
{
    if (C.zp.chunk != 1024) return (int)hipErrorNotSupported;
    if (C.idx_kind == IdxKind::I32)
        return launch_run<16, int32_t, ValT, VecT, OutT>(A, C, k, V, ldv, U, ldu, stream);
    if constexpr (std::is_same<OutT, VecT>::value)
        return launch_run<16, uint16_t, ValT, VecT, OutT>(A, C, k, V, ldv, U, ldu, stream);
    return (int)hipErrorNotSupported;             // binary64 partial sums: several blocks, 4-byte indices
}

}  // namespace

bool coldot_run_takes(const spw_matrix_s &A, const ColDot &C, spw_dtype vdt, int32_t k, int64_t ldv)
{
    if (k <= 8) return false;
    // A wave takes about 0.16 us a column start.  Where a few chunks have most of the starts (columns
    // by descending length: up to the whole chunk's, 160 us) their waves are the last to end, however
    // even the others are: not worth it past about a third of the call, 6.5e-7 us a nonzero and column
    // (binary64, 5,000 rows, 35 a column on average, ordered / not, us, tile and run: 4e6 k = 16 65 and
    // 162 / 62 and 50, 1.25e7 k = 32 231 and 281 / 220 and 192, k = 64 454 and 407 / 423 and 310; 2.5e7 k = 16 293 and
    // 316 / 302 and 221, k = 32 478 and 442).  Chunks of up to 48 starts are no longer than their gathers.
    if (C.most_segs > 48 && (int64_t)C.most_segs * 700000 > C.nnz * k) return false;
    if (&C == &A.cd) {
        if (vdt != SPW_F64) return false;
        // A wave walks its chunk's column starts one after the other, where the tile's lanes take
        // a few positions each: short columns need a wide block to pay for their starts, and a
        // matrix of few chunks a wave has nothing to hide them behind.  Tile and run (us, 5,000
        // rows, binary64), k = 16: 1e6 nonzeros 10 a column 29 and 33, 30 a column 26 and 27; 4e6 10
        // a column 61 and 67, 30 a column 54 and 52; 1.6e7 3, 6 and 10 a column 357 and 383, 274 and
        // 260, 233 and 210.  k = 32: 1e6 3 and 10 a column 46 and 55, 39 and 38; 8e6 1.5 a column
        // 455 and 445.  k = 64: 5e5 3 and 6 a column 58 and 62, 51 and 50; 2e6 1.5 a column 243 and 194.
        const int64_t filled = C.cols - C.n_empty;
        const int64_t least = k <= 16 ? (C.nnz < (int64_t)1 << 23 ? 30 : 8)
                              : k <= 32 ? (C.nnz < (int64_t)1 << 22 ? 8 : 0)
                                        : (C.nnz < (int64_t)1 << 21 ? 6 : 0);
        return C.nnz >= least * filled;
    }
    // the transpose gathers the caller's rows: whole 16-byte groups of columns; 2-byte rows
    // are kept as 32-bit byte offsets.  Its columns are long, only the size counts (k = 16,
    // binary32, tile and run: 5e5 nonzeros 19 and 23 to 26, 1e6 20 to 26 and 23 to 27, 2e6 58 and 42).
    const int64_t es = vdt == SPW_F64 ? 8 : 4;
    if (k <= 16 && C.nnz < (int64_t)5 << 18) return false;
    return (k * es) % 16 == 0 && (C.idx_kind == IdxKind::I32 || ldv * es < 65536);
}

int launch_coldot_run(const spw_matrix_s &A, const ColDot &C, const int32_t *inv, spw_dtype vdt, int32_t k, const void *V,
                      int64_t ldv, void *U, int64_t ldu, void *stream_, bool out_f64)
{
    hipStream_t stream = (hipStream_t)stream_;
    if (!coldot_run_takes(A, C, vdt, k, ldv)) return (int)hipErrorNotSupported;
    return with_types(A.value_storage, vdt, [&](auto vt, auto xt) -> int {
        using ValT = decltype(vt);
        using VecT = decltype(xt);
        const VecT *v = (const VecT *)V;
        if (&C == &A.cd) {
            if constexpr (std::is_same<VecT, double>::value)
                return C.idx_kind == IdxKind::U16
                           ? run_own<uint16_t, ValT>(A, C, inv, k, v, ldv, (double *)U, ldu, stream)
                           : run_own<int32_t, ValT>(A, C, inv, k, v, ldv, (double *)U, ldu, stream);
            return (int)hipErrorNotSupported;
        }
        if (out_f64 && !std::is_same<VecT, double>::value)
            return run_transpose<ValT, VecT, double>(A, C, k, v, ldv, (double *)U, ldu, stream);
        return run_transpose<ValT, VecT, VecT>(A, C, k, v, ldv, (VecT *)U, ldu, stream);
    });
}

}  // namespace spw
