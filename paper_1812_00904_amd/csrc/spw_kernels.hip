// HIP kernels for gfx950 (CDNA4, wave64) and their launch glue.
//
// Both products are bound by HBM bandwidth (about 0.17 flop per byte for
// binary64 values with 2-byte row indices): no MFMA.  What decides their speed
// on this chip is (a) keeping enough bytes in flight per CU and (b) keeping
// the gathers of the dense vectors off the texture path when their addresses
// diverge across a wave (each distinct cache line costs the L1 a cycle).  So
// both kernels run persistent workgroups whose waves work independently (no
// workgroup barrier inside the main loops), and the gathers go to LDS or are
// arranged so that the lanes of one instruction touch few cache lines.
//
// Column dots (u_j = sum_i v_i b_ij over a CSC matrix B; the paper's v^T A,
// Section IV-A): each wave takes equal-nonzero chunks of 64*ITEMS positions
// (the paper's nonzero split, Section II, with a wave as the processor).  The
// most used entries of v (rows renumbered by count) are staged in LDS.  A lane
// walks ITEMS consecutive positions, closing a run at every column end; runs
// inside a lane are final, the first/last run of each lane are joined across
// the wave by a segmented scan, and a column cut by a chunk boundary leaves a
// carry that the zone kernel adds in ascending chunk order.
//
// Scatter product (y = B x; the paper's A x, Section III): a row panel of y
// lives in LDS per workgroup.  The panel's rows are dealt to the 4 waves of
// the workgroup (balanced by count), and each wave streams, in column order,
// only the nonzeros of its own rows, adding them into LDS.  No two waves touch
// the same LDS entry, and a wave adds in program order, so every sum is formed
// in a fixed order; the per-workgroup partial vectors are then added in
// ascending workgroup order (the paper's y = sum_i y_(i)).  Consecutive lanes
// hold consecutive nonzeros of one column range, so an x gather instruction
// touches only a few cache lines.  No floating-point atomics touch global
// memory: results are bit-identical from run to run.
#include "spw_device.h"

namespace spw {
namespace {

template <typename IdxT, typename ValT, int ITEMS> struct VtmChunk {
    ValRaw<ValT, ITEMS> a;
    IdxRaw<IdxT, ITEMS> r;
    uint32_t mask;              // column-start bits of the lane's positions
};

// MULTI = false: one vector (k = 1, v and out.u[0] unit-stride).
// MULTI = true: k <= MULTI_MAX columns; v is a row-major rows x k block and
// column col goes to out.u[col] with stride out.ld[col].  Each chunk is loaded
// once and reduced once per column with exactly the single-vector arithmetic,
// so every column equals the single-vector result bit for bit.  The hot rows
// are staged in LDS as vh[r*k + col].
// wchunks: NULL, or per worker the first chunk of its run, P+1 entries
// (column and merge-path partitioning: worker w reduces chunks wchunks[w] .. wchunks[w+1]-1
// instead of every P-th chunk).  A worker is a wave, or the two waves of a 1,024-thread
// workgroup that take its chunks in turn (chunks of 512: vtm_block_for).
// CAP: segments of a chunk that a wave stages (vtm_stage); gap_max: see vtm_reduce_staged.
template <int BLOCK, int ITEMS, int CAP, typename IdxT, typename ValT, typename VecT, bool MULTI>
__global__ __launch_bounds__(BLOCK) void vtm_wave(
    const IdxT *__restrict__ idx, const ValT *__restrict__ val, const uint16_t *__restrict__ heads,
    const int4 *__restrict__ cinfo, const int32_t *__restrict__ segcol, int64_t nnz, int64_t nchunks,
    const int32_t *__restrict__ wchunks, const VecT *__restrict__ v, int k, int vhot, ColOut<VecT> out,
    double *__restrict__ carry, int gap_max)
{
    if (!MULTI) k = 1;
    const int64_t ldv = k;
    constexpr int NW = BLOCK / WAVE;
    constexpr int WCH = WAVE * ITEMS;
    extern __shared__ double lds[];
    // LDS: each wave's segment stage, then the hot rows of v
    constexpr int STAGED = stage_stride(CAP);
    VecT *vh = reinterpret_cast<VecT *>(lds + NW * STAGED);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    __attribute__((address_space(3))) double *stage =
        (__attribute__((address_space(3))) double *)(lds + wave * STAGED);
    const int lane = threadIdx.x & (WAVE - 1);

    if (MULTI) {
        stage_rows<BLOCK, 8, VecT>(vh, vhot * k, [&](int i) {
            const int r = i / k;
            return v[(int64_t)r * ldv + (i - r * k)];
        });
    } else {
        stage_rows<BLOCK, 16, VecT>(vh, vhot, [&](int i) { return v[i]; });
    }
    __syncthreads();
    const __attribute__((address_space(3))) VecT *vh3 = (const __attribute__((address_space(3))) VecT *)vh;
    const __attribute__((address_space(1))) VecT *vg1 = (const __attribute__((address_space(1))) VecT *)v;

    int64_t stride = (int64_t)gridDim.x * NW;
    int64_t c = (int64_t)blockIdx.x * NW + wave;
    int64_t cend = nchunks;
    if (wchunks) {
        constexpr int WAVES = BLOCK > VTM_BLOCK ? BLOCK / VTM_BLOCK : 1;     // of one worker
        const int64_t w = c / WAVES;
        cend = wchunks[w + 1];
        c = wchunks[w] + c % WAVES;
        stride = WAVES;
    }
    if (c >= cend) return;

    // Two chunk buffers used alternately (no register copies, so no wait for
    // data still in flight): while one chunk is reduced, the next one's
    // values, indices and column-start bits are being fetched.
    typedef VtmChunk<IdxT, ValT, ITEMS> Chunk;
    Chunk A, B;
    auto load_chunk = [&](Chunk &C, int64_t cc) {
        const int64_t cb = cc * WCH;
        C.a.load(val + cb, lane);
        C.r.load(idx + cb, lane);
        C.mask = heads[cc * WAVE + lane];
    };
    // Reduces chunk cc held in C (description ci), after issuing the loads of
    // chunk cn into N (when cn < cend).
    auto step = [&](Chunk &C, Chunk &N, int64_t cc, int4 ci, int64_t cn) {
        const int s = (int)(cc * WCH);
        const int e = (int)min((int64_t)s + WCH, nnz);
        for (int col = 0; col < k; ++col) {
            double prod[ITEMS];
            // The LDS reads and the global reads are typed with their address
            // spaces, so they stay ds_reads and global loads (a select between
            // two generic pointers would become one flat load, which every
            // later wait on either counter has to cover), and all LDS reads are
            // issued before the first global read, so none waits for another.
            VecT lv[ITEMS], gv[ITEMS];
            // The wave issues its reads at raised priority and drops back for
            // the product and the reduction: a wave with reads to issue then
            // wins the issue slot over one that is reducing, which keeps more
            // reads in flight per CU.
            __builtin_amdgcn_s_setprio(3);
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) lv[i] = vh3[min(C.r.get(i), vhot - 1) * k + col];
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                const int ri = C.r.get(i);
                gv[i] = 0;
                if (ri >= vhot) gv[i] = vg1[(int64_t)ri * ldv + col];
            }
            if (col == 0) {
                // The next chunk's loads go out after the gathers (the
                // scheduling barriers keep that order): the load counter
                // retires in order, so the wait for the gathers then leaves
                // the prefetch in flight.  The loads are issued on every path
                // (after the wave's last chunk they fetch the current one
                // again, unused) so that the wait can count them.
                __builtin_amdgcn_sched_barrier(0);
                load_chunk(N, cn < cend ? cn : cc);
                __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_s_setprio(0);
            // a select of the two loaded values, not of two addresses: the
            // gathers stay ahead of the prefetch
#pragma unroll
            for (int i = 0; i < ITEMS; ++i)
                prod[i] = C.a.get(i) * (double)(C.r.get(i) < vhot ? lv[i] : gv[i]);
            VecT *uc = MULTI ? out.u[col] : out.u[0];
            const int64_t ldu = MULTI ? out.ld[col] : 1;
            // full chunk, output view within 2^31 bytes, and its segments fit the stage (none
            // empty inside, without one)
            if constexpr (STAGED > 0) {
                const bool staged = e - s == WCH && ci.z <= CAP &&
                                    ldu <= (int64_t)(1 << 28) / (WCH * (int64_t)sizeof(VecT));
                if (staged)
                    vtm_reduce_staged<ITEMS, CAP, VecT>(prod, C.mask, ci, segcol, cc, lane, uc, ldu, carry, k, col, stage,
                                                   gap_max);
                else
                    vtm_reduce_chunk<ITEMS, VecT>(prod, C.mask, s, e, ci, segcol, cc, lane, uc, ldu, carry, k, col);
            } else {
                const bool dense_full = e - s == WCH && (ci.w & CHUNK_DENSE) &&
                                        ldu <= (int64_t)(1 << 28) / (WCH * (int64_t)sizeof(VecT));
                if (dense_full)
                    vtm_reduce_dense_direct<ITEMS, VecT>(prod, C.mask, ci, segcol, cc, lane, uc, ldu, carry, k, col);
                else
                    vtm_reduce_chunk<ITEMS, VecT>(prod, C.mask, s, e, ci, segcol, cc, lane, uc, ldu, carry, k, col);
            }
        }
    };

    // chunk sequence c, c + stride, ...; chunk descriptions are loaded one step ahead
    auto ci_at = [&](int64_t cc) { return cc < cend ? cinfo[cc] : make_int4(0, 0, 0, 0); };
    int4 ci0 = cinfo[c];
    load_chunk(A, c);
    for (;;) {
        const int64_t c1 = c + stride;
        const int4 ci1 = ci_at(c1);
        step(A, B, c, ci0, c1);
        if (c1 >= cend) break;
        const int64_t c2 = c1 + stride;
        ci0 = ci_at(c2);
        step(B, A, c1, ci1, c2);
        if (c2 >= cend) break;
        c = c2;
    }
}

// Columns without nonzeros: u_j = 0.
template <typename VecT>
__global__ void zero_cols(const int32_t *__restrict__ cols, int64_t count, VecT *__restrict__ u)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < count) u[cols[i]] = (VecT)0;
}

// Zone reduction: u[j_k] = right carry of the first chunk + left carries of the
// following chunks of S_k, in ascending chunk order.
template <typename VecT>
__global__ void zone_fixup(const int32_t *__restrict__ zcol, const int32_t *__restrict__ zfirst,
                           const int32_t *__restrict__ zlast, int64_t nz, const double *__restrict__ carry,
                           VecT *__restrict__ u)
{
    const int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (k >= nz) return;
    u[zcol[k]] = (VecT)zone_sum(carry, zfirst[k], zlast[k], 1, 0);
}

// Renumber a short vector: out[r] = in[inv[r]].
template <typename VecT>
__global__ void gather_vec(const int32_t *__restrict__ inv, int64_t len, const VecT *__restrict__ in,
                           VecT *__restrict__ out)
{
    const int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (r < len) out[r] = in[inv[r]];
}

// ------------------------------------------------------------------------
// Scatter product over one row panel.  Panel q holds the internal rows
// r = q (mod P) for P panels, so every panel sees about the same share of each
// column, and the workgroups of different panels that cover the same column
// range gather the same x entries at about the same time (the second and
// later reads hit in cache instead of HBM).
// Storage: blocks of 64*MV_ITEMS nonzeros.  A block holds nonzeros of one
// wave's rows, in column order, from one workgroup's column range.  Logical
// nonzero j*64 + lane sits at word slot ((j/4)*64 + lane)*4 + j%4 and at value
// slot ((j/2)*64 + lane)*2 + j%2, so every load instruction reads one
// contiguous span while each add instruction covers 64 consecutive nonzeros
// (whose x entries share a few cache lines).  A word is
// (panel slot << 16 | column - block column base).  The streams are read
// with non-temporal loads so they do not push x out of the caches.
//   blocks : (column base, count) per block
//   wg_blk : per workgroup, NW+1 offsets into blocks: wave w owns [wg_blk[w], wg_blk[w+1])
//   x      : input, entry j at x[j*ldx]
//   partial: per-workgroup partial sums, one per row
// The loop keeps two blocks of words/values and one block of x gathers in
// flight.  Dynamic LDS: one double per slot.
// ------------------------------------------------------------------------
constexpr int MV_ITEMS = 16;
constexpr int MV_BLK = WAVE * MV_ITEMS;

template <typename ValT> struct MvBlk {
    uint32_t w[MV_ITEMS];
    ValRaw<ValT, MV_ITEMS> a;
    int2 bd;
};

template <typename ValT>
__device__ __forceinline__ void mv_load(MvBlk<ValT> &B, const uint32_t *__restrict__ packed,
                                        const ValT *__restrict__ val, const int2 *__restrict__ blocks, int b, int lane)
{
    B.bd = blocks[b];
    const int64_t base = (int64_t)b * MV_BLK;
#pragma unroll
    for (int g = 0; g < MV_ITEMS / 4; ++g) {
        const u32x4_t q = ld_stream<true>(reinterpret_cast<const u32x4_t *>(packed + base + (int64_t)(g * 64 + lane) * 4));
        B.w[4 * g] = q.x;
        B.w[4 * g + 1] = q.y;
        B.w[4 * g + 2] = q.z;
        B.w[4 * g + 3] = q.w;
    }
    B.a.template load<true>(val + base, lane);
}

// The LDS panel's shape: slots of all, rows, and 2^cs copies of each row in front; hot, nhot: the
// rows with more slots (of this range's panel).
struct MvPanel {
    int slots, rows, cs, nhot;
    const HotRow *hot;
};
__device__ __forceinline__ MvPanel mv_panel(int slots, int rows, int cs, const HotRow *__restrict__ hot,
                                            const int2 *__restrict__ wg_hot, int range)
{
    const int2 h = wg_hot ? wg_hot[range] : make_int2(0, 0);
    return MvPanel{slots, rows, cs, h.y, hot + h.x};
}

// A thread's first row of mv_write_panel's: read when the range begins, not when it ends.
constexpr int HOT_LANES = 8;
template <int KC> __device__ __forceinline__ HotRow mv_hot(const MvPanel &pn)
{
    return (int)threadIdx.x < pn.nhot * KC * HOT_LANES ? pn.hot[threadIdx.x / (HOT_LANES * KC)] : HotRow{};
}

// KC panels to their partial sums, one a row: the slots that a row has more (63 at most) are added to
// its first by eight threads a row, then the row's copies pairwise.  All of the workgroup's waves come
// here with their adds to the panel made or under way.  The end of a range counts, in small products
// most of all, so its loads don't wait for one another: 29,966 x 2.5e6 with 257,000 nonzeros, twelve
// columns, 78 us of mv_bucket with a test for the copies at every element, 71 like this.  The slots
// cost, against one sum a row, 0.7 us of a pair of 74 (9e6 nonzeros, 19,996 rows) and 2.2 us of 242 for
// four columns over 5e7 with a thread a row and its descriptor read at the end, 0.6 and 1.7 like this.
template <int BLOCK, int KC>
__device__ __forceinline__ void mv_write_panel(double *ypan, const MvPanel &pn, HotRow h, double *__restrict__ out,
                                               int64_t col_stride)
{
    const int rows = pn.rows, cs = pn.cs, tid = threadIdx.x;
    __syncthreads();
    if (pn.nhot > 0) {
        const int n = pn.nhot * KC * HOT_LANES, lane = tid % HOT_LANES;
        for (int i = tid; i < n; i += BLOCK) {
            const int g = i / HOT_LANES;
            if (i != tid) h = pn.hot[g / KC];
            double *y = ypan + (g % KC) * pn.slots, a[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) a[t] = lane + HOT_LANES * t < h.more ? y[h.first + lane + HOT_LANES * t] : 0.0;
            double s = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
            s += __shfl_xor(s, 1);
            s += __shfl_xor(s, 2);
            s += __shfl_xor(s, 4);
            if (lane == 0) y[h.local] += s;
        }
        __syncthreads();
    }
    if (cs == 0) {
#pragma unroll
        for (int c = 0; c < KC; ++c)
            for (int i = tid; i < rows; i += BLOCK) out[c * col_stride + i] = ypan[c * pn.slots + i];
        return;
    }
    for (int i = tid; i < rows; i += BLOCK) {
        double s[KC];
        auto each = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < KC; ++c) f(s[c], ypan + c * pn.slots + i);
        };
        each([&](double &t, const double *p) { t = p[0] + p[rows]; });
        if (cs >= 2) each([&](double &t, const double *p) { t += p[2 * rows] + p[3 * rows]; });
        if (cs >= 3)
            each([&](double &t, const double *p) {
                t += (p[4 * rows] + p[5 * rows]) + (p[6 * rows] + p[7 * rows]);
            });
        if (cs >= 4)
            each([&](double &t, const double *p) {
                t += ((p[8 * rows] + p[9 * rows]) + (p[10 * rows] + p[11 * rows])) +
                     ((p[12 * rows] + p[13 * rows]) + (p[14 * rows] + p[15 * rows]));
            });
#pragma unroll
        for (int c = 0; c < KC; ++c) out[c * col_stride + i] = s[c];
    }
}

// One workgroup range of the scatter product into the LDS panel ypan, written
// to out (mv_write_panel).
template <int BLOCK, typename ValT, typename VecT>
__device__ __forceinline__ void mv_range(const uint32_t *__restrict__ packed, const ValT *__restrict__ val,
                                         const int2 *__restrict__ blocks, const int32_t *__restrict__ wg_blk,
                                         int range, const VecT *__restrict__ x, int64_t ldx,
                                         double *__restrict__ out, const MvPanel &pn, double *ypan)
{
    constexpr int NW = BLOCK / WAVE;
    const int tid = threadIdx.x, wave = tid / WAVE, lane = tid & (WAVE - 1);
    const HotRow hot = mv_hot<1>(pn);
    for (int i = tid; i < pn.slots; i += BLOCK) ypan[i] = 0.0;
    __syncthreads();

    const int32_t *wb = wg_blk + (int64_t)range * (NW + 1);
    const int b0 = wb[wave], b1 = wb[wave + 1];
    // Two block buffers used alternately: while block b is added, the x
    // entries of block b+1 and the words/values of block b+2 are being
    // fetched.  (The compiler issues block b+1's gathers ahead of block b's
    // products, so each step first waits for the words those gathers index;
    // a form of this loop without that wait, tried, was no faster.)
    MvBlk<ValT> B0, B1;
    VecT x0[MV_ITEMS], x1[MV_ITEMS];
    // padding slots hold word 0, so their gather reads x[column base]: no branch.
    // A unit-stride x (every single-vector call) takes 32-bit column offsets.
    auto gather = [&](const MvBlk<ValT> &B, VecT *xv) {
        if (ldx == 1) {
#pragma unroll
            for (int j = 0; j < MV_ITEMS; ++j) xv[j] = x[B.bd.x + (int)(B.w[j] & 0xFFFFu)];
        } else {
#pragma unroll
            for (int j = 0; j < MV_ITEMS; ++j) xv[j] = x[(int64_t)(B.bd.x + (int)(B.w[j] & 0xFFFFu)) * ldx];
        }
    };
    auto add_block = [&](const MvBlk<ValT> &B, const VecT *xv, double *p, uint32_t *row) {
#pragma unroll
        for (int j = 0; j < MV_ITEMS; ++j) {
            p[j] = B.a.get(j) * (double)xv[j];
            row[j] = B.w[j] >> 16;
        }
    };
    auto commit = [&](int count, const double *p, const uint32_t *row) {
        if (count == MV_BLK) {                    // a full block: every item is a nonzero
#pragma unroll
            for (int j = 0; j < MV_ITEMS; ++j)
                __hip_atomic_fetch_add(&ypan[row[j]], p[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            return;
        }
        const int lim = count - lane;             // item j is a nonzero when j*64 < lim
#pragma unroll
        for (int j = 0; j < MV_ITEMS; ++j)
            if (j * WAVE < lim) __hip_atomic_fetch_add(&ypan[row[j]], p[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    // The loads and gathers are issued on every path, of the last block again
    // past the end of the range (so each buffer is written on every path and
    // the compiler keeps the two in place instead of copying between them).
    // Ranges of one or two blocks (small matrices) skip those repeats.
    if (b0 < b1 && b1 - b0 <= 2) {
        mv_load(B0, packed, val, blocks, b0, lane);
        gather(B0, x0);
        if (b1 - b0 == 2) mv_load(B1, packed, val, blocks, b0 + 1, lane);
        double p[MV_ITEMS];
        uint32_t row[MV_ITEMS];
        add_block(B0, x0, p, row);
        if (b1 - b0 == 2) gather(B1, x1);
        commit(B0.bd.y, p, row);
        if (b1 - b0 == 2) {
            add_block(B1, x1, p, row);
            commit(B1.bd.y, p, row);
        }
    } else if (b0 < b1) {
        const int last = b1 - 1;
        mv_load(B0, packed, val, blocks, b0, lane);
        gather(B0, x0);
        mv_load(B1, packed, val, blocks, min(b0 + 1, last), lane);
        for (int b = b0;; b += 2) {
            double p[MV_ITEMS];
            uint32_t row[MV_ITEMS];
            add_block(B0, x0, p, row);
            int cnt = B0.bd.y;
            gather(B1, x1);
            mv_load(B0, packed, val, blocks, min(b + 2, last), lane);
            commit(cnt, p, row);
            if (b + 1 >= b1) break;
            add_block(B1, x1, p, row);
            cnt = B1.bd.y;
            gather(B0, x0);
            mv_load(B1, packed, val, blocks, min(b + 3, last), lane);
            commit(cnt, p, row);
            if (b + 2 >= b1) break;
        }
    }
    mv_write_panel<BLOCK, 1>(ypan, pn, hot, out, 0);
}

template <int BLOCK, typename ValT, typename VecT>
__global__ __launch_bounds__(BLOCK) void mv_bucket(
    const uint32_t *__restrict__ packed, const ValT *__restrict__ val, const int2 *__restrict__ blocks,
    const int32_t *__restrict__ wg_blk, const int32_t *__restrict__ wg_order, const VecT *__restrict__ x, int64_t ldx,
    double *__restrict__ partial, int slots, int rows, int cs, const HotRow *__restrict__ hot,
    const int2 *__restrict__ wg_hot)
{
    extern __shared__ double ypan[];
    const int range = wg_order[blockIdx.x];
    mv_range<BLOCK, ValT, VecT>(packed, val, blocks, wg_blk, range, x, ldx,
                                      partial + (int64_t)range * rows, mv_panel(slots, rows, cs, hot, wg_hot, range),
                                      ypan);
}

// ------------------------------------------------------------------------
// Scatter product for several columns of x at once (k >= 2).
//
// A workgroup runs one range for a group of KC <= 4 columns: its LDS holds KC
// copies of the row panel, and a lane adds its nonzero into each of them.  What
// bounds one column after another is the instruction stream and the address
// unit, not memory: every column decoded the same words, re-read the same
// values and touched the same lines of a row-major X.  With KC columns a lane
// decodes a word once, reads the KC adjacent entries of its row of X with
// 16-byte loads, and only the products and the LDS additions grow with KC.
// Every row of a column is summed by the same wave in the same order as in the
// single-column product, so the results are the same bit for bit.
//
// The x entries live in a ring of one block (four sub-blocks of four items a
// lane): after sub-block s of block b has been multiplied, its place takes the
// entries of sub-block s of block b+1, whose words are in registers, and the
// words and values of block b+2 replace those of sub-block s just used.  So
// the loads run four sub-blocks ahead without a copy between registers.  The
// LDS panels allow one workgroup per CU (one wave per SIMD), so the registers
// this takes (about 230 for four binary64 columns) cost no occupancy.
// ------------------------------------------------------------------------
constexpr int MV_SUB = 4;                       // items of a lane per sub-block
constexpr int MV_NSUB = MV_ITEMS / MV_SUB;
constexpr int MV_COLS = 4;                      // columns a workgroup takes at once, at most

// Values of items 4*s .. 4*s+3 of one lane of a block.
template <typename ValT> struct MvVal;
template <> struct MvVal<double> {
    double a[MV_SUB];
    __device__ __forceinline__ void load(const double *base, int s, int lane)
    {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f64x2_t w = *reinterpret_cast<const f64x2_t *>(base + ((2 * s + h) * 64 + lane) * 2);
            a[2 * h] = w.x;
            a[2 * h + 1] = w.y;
        }
    }
    __device__ __forceinline__ double get(int i) const { return a[i]; }
};
template <> struct MvVal<float> {
    float a[MV_SUB];
    __device__ __forceinline__ void load(const float *base, int s, int lane)
    {
        const f32x4_t w = *reinterpret_cast<const f32x4_t *>(base + (s * 64 + lane) * 4);
        a[0] = w.x;
        a[1] = w.y;
        a[2] = w.z;
        a[3] = w.w;
    }
    __device__ __forceinline__ double get(int i) const { return (double)a[i]; }
};
template <> struct MvVal<Bf16> {
    uint32_t w[2];
    __device__ __forceinline__ void load(const Bf16 *base, int s, int lane)
    {
        typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
        const u32x2_t q = *reinterpret_cast<const u32x2_t *>(base + ((s >> 1) * 64 + lane) * 8 + (s & 1) * 4);
        w[0] = q.x;
        w[1] = q.y;
    }
    __device__ __forceinline__ double get(int i) const
    {
        return bf16_bits_to_f64((w[i >> 1] >> ((i & 1) * 16)) & 0xFFFFu);
    }
};

// KC adjacent entries of a row of X.  A row starts on a multiple of the entry
// size only, so the wide loads are typed with that alignment.
template <typename VecT, int KC> struct MvRow;
template <int KC> struct MvRow<double, KC> {
    double v[KC];
    __device__ __forceinline__ void load(const double *p)
    {
        typedef double f64x2_u __attribute__((ext_vector_type(2), aligned(8)));
#pragma unroll
        for (int h = 0; h < KC / 2; ++h) {
            const f64x2_u w = *reinterpret_cast<const f64x2_u *>(p + 2 * h);
            v[2 * h] = w.x;
            v[2 * h + 1] = w.y;
        }
        if (KC & 1) v[KC - 1] = p[KC - 1];
    }
};
template <int KC> struct MvRow<float, KC> {
    float v[KC];
    __device__ __forceinline__ void load(const float *p)
    {
        if constexpr (KC == 4) {
            typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));
            const f32x4_u w = *reinterpret_cast<const f32x4_u *>(p);
            v[0] = w.x;
            v[1] = w.y;
            v[2] = w.z;
            v[3] = w.w;
        } else {
            if constexpr (KC >= 2) {
                typedef float f32x2_u __attribute__((ext_vector_type(2), aligned(4)));
                const f32x2_u w = *reinterpret_cast<const f32x2_u *>(p);
                v[0] = w.x;
                v[1] = w.y;
            }
            if constexpr (KC & 1) v[KC - 1] = p[KC - 1];
        }
    }
};

// A group of adjacent columns of one row-major block: kc columns from x on,
// rows ld entries apart; slot is the partial-sum slot of its first column.
template <typename VecT> struct MvGroups {
    const VecT *x[MULTI_MAX];
    int64_t ld[MULTI_MAX];
    int32_t kc[MULTI_MAX], slot[MULTI_MAX];
};

template <typename ValT> struct MvStage {
    uint32_t w[MV_ITEMS];
    MvVal<ValT> a[MV_NSUB];
};

// One range for KC columns.  WIDE: the row stride of X is too large for 32-bit
// byte offsets inside a block's 65,536 columns.
template <int BLOCK, typename ValT, typename VecT, int KC, bool WIDE>
__device__ __forceinline__ void mv_range_cols(const uint32_t *__restrict__ packed, const ValT *__restrict__ val,
                                              const int2 *__restrict__ blocks, const int32_t *__restrict__ wb,
                                              const VecT *__restrict__ x, int64_t ldx, double *__restrict__ out,
                                              int64_t col_stride, const MvPanel &pn, double *ypan)
{
    const int slots = pn.slots;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const HotRow hot = mv_hot<KC>(pn);
    for (int i = tid; i < KC * slots; i += BLOCK) ypan[i] = 0.0;
    __syncthreads();
    const int b0 = __builtin_amdgcn_readfirstlane(wb[wave]), b1 = __builtin_amdgcn_readfirstlane(wb[wave + 1]);
    const uint32_t ld_bytes = (uint32_t)(ldx * (int64_t)sizeof(VecT));
    typedef MvRow<VecT, KC> Row;
    MvStage<ValT> S0, S1;
    Row xr[MV_NSUB][MV_SUB];
    int base0 = 0, base1 = 0, cnt0 = 0, cnt1 = 0;
    auto load = [&](MvStage<ValT> &S, int s, int b) {
        const int64_t at = (int64_t)b * MV_BLK;
        const u32x4_t q = *reinterpret_cast<const u32x4_t *>(packed + at + (s * 64 + lane) * 4);
        S.w[4 * s] = q.x;
        S.w[4 * s + 1] = q.y;
        S.w[4 * s + 2] = q.z;
        S.w[4 * s + 3] = q.w;
        S.a[s].load(val + at, s, lane);
    };
    auto describe = [&](int b, int &base, int &cnt) {
        const int2 d = blocks[b];
        base = __builtin_amdgcn_readfirstlane(d.x);
        cnt = __builtin_amdgcn_readfirstlane(d.y);
    };
    // padding slots hold word 0, so their gather reads the block's first column: no branch
    auto gather = [&](const MvStage<ValT> &S, int s, int base) {
        const VecT *xb = x + (int64_t)base * ldx;
#pragma unroll
        for (int j = 0; j < MV_SUB; ++j) {
            const uint32_t c = S.w[4 * s + j] & 0xFFFFu;
            if constexpr (WIDE) xr[s][j].load(xb + (int64_t)c * ldx);
            else xr[s][j].load(reinterpret_cast<const VecT *>(reinterpret_cast<const char *>(xb) + c * ld_bytes));
        }
    };
    double p[MV_SUB][KC];
    uint32_t row[MV_SUB];
    auto multiply = [&](const MvStage<ValT> &S, int s) {
#pragma unroll
        for (int j = 0; j < MV_SUB; ++j) {
            row[j] = S.w[4 * s + j] >> 16;
#pragma unroll
            for (int c = 0; c < KC; ++c) p[j][c] = S.a[s].get(j) * (double)xr[s][j].v[c];
        }
    };
    auto commit = [&](int s, int cnt) {
        const int lim = cnt - lane;              // item i is a nonzero when i*64 < lim
#pragma unroll
        for (int j = 0; j < MV_SUB; ++j) {
            if (cnt == MV_BLK || (4 * s + j) * WAVE < lim) {
#pragma unroll
                for (int c = 0; c < KC; ++c)
                    __hip_atomic_fetch_add(&ypan[c * slots + row[j]], p[j][c], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
    };
    if (b0 < b1 && b1 - b0 <= 2) {
        // one or two blocks (small matrices): no repeats of the last block, and no
        // loads past a block's last nonzero
        for (int b = b0; b < b1; ++b) {
            describe(b, base0, cnt0);
#pragma unroll
            for (int s = 0; s < MV_NSUB; ++s)
                if (s * MV_SUB * WAVE < cnt0) load(S0, s, b);
#pragma unroll
            for (int s = 0; s < MV_NSUB; ++s)
                if (s * MV_SUB * WAVE < cnt0) gather(S0, s, base0);
#pragma unroll
            for (int s = 0; s < MV_NSUB; ++s)
                if (s * MV_SUB * WAVE < cnt0) {
                    multiply(S0, s);
                    commit(s, cnt0);
                }
        }
    } else if (b0 < b1) {
        const int last = b1 - 1;
        describe(b0, base0, cnt0);
        describe(b0 + 1, base1, cnt1);
#pragma unroll
        for (int s = 0; s < MV_NSUB; ++s) load(S0, s, b0);
#pragma unroll
        for (int s = 0; s < MV_NSUB; ++s) load(S1, s, b0 + 1);
#pragma unroll
        for (int s = 0; s < MV_NSUB; ++s) gather(S0, s, base0);
        // block b in C, block b+1 in N; past the end of the range the last block
        // is loaded again, unused
        auto block = [&](MvStage<ValT> &C, const MvStage<ValT> &N, int b, int &cnt_c, int &base_c, int base_n) {
            const int b2 = min(b + 2, last);
            int base2, cnt2;
            describe(b2, base2, cnt2);
#pragma unroll
            for (int s = 0; s < MV_NSUB; ++s) {
                multiply(C, s);
                gather(N, s, base_n);
                load(C, s, b2);
                commit(s, cnt_c);
            }
            base_c = base2;
            cnt_c = cnt2;
        };
        for (int b = b0;; b += 2) {
            block(S0, S1, b, cnt0, base0, base1);
            if (b + 1 >= b1) break;
            block(S1, S0, b + 1, cnt1, base1, base0);
            if (b + 2 >= b1) break;
        }
    }
    mv_write_panel<BLOCK, KC>(ypan, pn, hot, out, col_stride);
}

// Groups of columns in one launch: workgroup (group, range).  The groups of one
// range, and the ranges of neighbouring columns, are dispatched to one XCD
// (workgroup ids are dealt to the 8 XCDs round-robin, so id b runs on XCD b mod 8),
// so they share the blocks and the lines of X through its L2 (ordinary loads: the lines
// stay for the others).  The tables are picked by a chain of selects on the group,
// so they stay in kernel arguments.  Column c of the launch keeps its partial
// sums in slot c (W ranges of one double per row each).
template <int BLOCK, typename ValT, typename VecT>
__global__ __launch_bounds__(BLOCK) void mv_bucket_cols(
    const uint32_t *__restrict__ packed, const ValT *__restrict__ val, const int2 *__restrict__ blocks,
    const int32_t *__restrict__ wg_blk, const int32_t *__restrict__ wg_order, MvGroups<VecT> groups, int ngroups,
    double *__restrict__ partial, int slots, int rows, int cs, const HotRow *__restrict__ hot,
    const int2 *__restrict__ wg_hot, int W)
{
    constexpr int NW = BLOCK / WAVE;
    extern __shared__ double ypan[];
    const int xcd = blockIdx.x % 8, i = blockIdx.x / 8;
    const int g = i % ngroups, at = (i / ngroups) * 8 + xcd;
    if (at >= W) return;
    const int range = wg_order[at];
    const VecT *x = groups.x[0];
    int64_t ld = groups.ld[0];
    int kc = groups.kc[0], slot = groups.slot[0];
#pragma unroll
    for (int t = 1; t < MULTI_MAX; ++t) {
        x = g == t ? groups.x[t] : x;
        ld = g == t ? groups.ld[t] : ld;
        kc = g == t ? groups.kc[t] : kc;
        slot = g == t ? groups.slot[t] : slot;
    }
    const int64_t col_stride = (int64_t)W * rows;
    double *out = partial + slot * col_stride + (int64_t)range * rows;
    const MvPanel pn = mv_panel(slots, rows, cs, hot, wg_hot, range);
    const int32_t *wb = wg_blk + (int64_t)range * (NW + 1);
    auto run = [&](auto cols, auto wide) {
        mv_range_cols<BLOCK, ValT, VecT, decltype(cols)::value, decltype(wide)::value>(
            packed, val, blocks, wb, x, ld, out, col_stride, pn, ypan);
    };
    // a block spans fewer than 65,536 columns: 32-bit byte offsets below this stride
    if (ld * (int64_t)sizeof(VecT) < 65536) {
        if (kc == 1) run(IntC<1>(), IntC<0>());
        else if (kc == 2) run(IntC<2>(), IntC<0>());
        else if (kc == 3) run(IntC<3>(), IntC<0>());
        else run(IntC<4>(), IntC<0>());
    } else {
        if (kc == 1) run(IntC<1>(), IntC<1>());
        else if (kc == 2) run(IntC<2>(), IntC<1>());
        else if (kc == 3) run(IntC<3>(), IntC<1>());
        else run(IntC<4>(), IntC<1>());
    }
}

// y[caller row] = sum over the panel's workgroups of their partials.  Internal row r
// belongs to panel r mod npanels, at panel-local row r / npanels; a
// workgroup takes 32 consecutive rows of one panel, eight threads a row: thread t
// adds partials t, t+8, t+16, ... in ascending order with up to sixteen loads in
// flight (a chain of dependent trips to memory bounds this kernel, not its
// bytes), then the eight sums are combined pairwise, so the order of every
// addition is fixed.  FEW: panels of at most eight workgroups, where one thread takes a
// whole row, in the same order, and the panels are one sequence of rows, so that small
// ones fill a workgroup too (2e6 x 2e6 in 98 panels of two or three workgroups: 83 us with
// eight threads a row, five of them idle, now 43; 500,000 rows in 49 panels 32 and 17).
// Column blockIdx.y: its partials start col_stride doubles further, its output is out.u[column].
constexpr int MV_FEW = 8;
template <typename VecT, bool FEW>
__global__ __launch_bounds__(256) void mv_reduce(const double *__restrict__ partial, int panel_rows, int panel_blocks,
                                                 const PanelDesc *__restrict__ panels, int npanels,
                                                 const int32_t *__restrict__ inv, ColOut<VecT> out, int64_t col_stride)
{
    __shared__ double sums[8][32];
    VecT *y = out.u[0];
    int64_t ldy = out.ld[0];
#pragma unroll
    for (int c = 1; c < MULTI_MAX; ++c) {
        y = blockIdx.y == c ? out.u[c] : y;
        ldy = blockIdx.y == c ? out.ld[c] : ldy;
    }
    int p, local, t = 0;
    if constexpr (FEW) {
        const uint32_t g = blockIdx.x * 256u + threadIdx.x;
        p = (int)min(g / (uint32_t)panel_rows, (uint32_t)npanels - 1u);
        local = (int)(g - (uint32_t)p * (uint32_t)panel_rows);
    } else {
        p = blockIdx.x / panel_blocks;
        local = (blockIdx.x - p * panel_blocks) * 32 + (threadIdx.x & 31);
        t = threadIdx.x >> 5;
    }
    const PanelDesc pd = panels[p];
    const bool live = local < pd.rows;
    const double *src = partial + blockIdx.y * col_stride + (int64_t)pd.wg0 * panel_rows + local;
    const int64_t r = (int64_t)local * npanels + p;
    int64_t to = r;
    if (inv && t == 0 && live) to = inv[r];       // beside the partial sums, not after them
    if constexpr (FEW) {
        if (!live) return;
        double a[MV_FEW];
#pragma unroll
        for (int i = 0; i < MV_FEW; ++i) a[i] = i < pd.nwg ? src[(int64_t)i * panel_rows] : 0.0;
        y[to * ldy] = (VecT)(((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7])));
        return;
    }
    double s = 0.0;
    if (live) {
        auto add = [&](auto loads) __attribute__((always_inline)) {
            constexpr int U = decltype(loads)::value;
            for (int w = t; w < pd.nwg; w += 8 * U) {
                double a[U];
#pragma unroll
                for (int i = 0; i < U; ++i) a[i] = w + 8 * i < pd.nwg ? src[(int64_t)(w + 8 * i) * panel_rows] : 0.0;
#pragma unroll
                for (int i = 0; i < U; ++i)
                    if (w + 8 * i < pd.nwg) s += a[i];
            }
        };
        if (pd.nwg <= 8 * 4) add(IntC<4>());
        else add(IntC<16>());
    }
    sums[t][threadIdx.x & 31] = s;
    __syncthreads();
    if (t == 0 && live) {
        const int l = threadIdx.x;
        const double y0 = (sums[0][l] + sums[1][l]) + (sums[2][l] + sums[3][l]);
        const double y1 = (sums[4][l] + sums[5][l]) + (sums[6][l] + sums[7][l]);
        y[to * ldy] = (VecT)(y0 + y1);
    }
}

// Multi-vector helpers over column tables (k <= MULTI_MAX columns).
template <typename VecT>
__global__ void zero_cols_tab(const int32_t *__restrict__ cols, int64_t count, int k, ColOut<VecT> out)
{
    const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (g >= count * k) return;
    const int64_t i = g / k;
    const int c = (int)(g - i * k);
    out.u[c][(int64_t)cols[i] * out.ld[c]] = (VecT)0;
}

template <typename VecT>
__global__ void zone_fixup_tab(const int32_t *__restrict__ zcol, const int32_t *__restrict__ zfirst,
                               const int32_t *__restrict__ zlast, int64_t nz, int k,
                               const double *__restrict__ carry, ColOut<VecT> out)
{
    const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (g >= nz * k) return;
    const int64_t z = g / k;
    const int cc = (int)(g - z * k);
    out.u[cc][(int64_t)zcol[z] * out.ld[cc]] = (VecT)zone_sum(carry, zfirst[z], zlast[z], k, cc);
}

// out[r*k + c] = column c of the table at caller row inv[r] (or r).
template <typename VecT>
__global__ void gather_tab(const int32_t *__restrict__ inv, int64_t rows, int k, ColIn<VecT> in,
                           VecT *__restrict__ out)
{
    const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (g >= rows * k) return;
    const int64_t r = g / k;
    const int c = (int)(g - r * k);
    const int64_t src = inv ? inv[r] : r;
    out[g] = in.v[c][src * in.ld[c]];
}

// Resident column-dot workgroups per CU for a workgroup of `block` threads:
// smaller workgroups run two to a CU (8 waves, as one 512-thread workgroup),
// each with half the LDS.
int vtm_wgs_per_cu(int block) { return block >= VTM_BLOCK ? VTM_WG_PER_CU : VTM_BLOCK / block; }
// LDS of one column-dot workgroup outside the hot rows: the waves' segment stages.
int64_t vtm_stage_bytes(int block, int cap)
{
    return (int64_t)(block / WAVE) * stage_stride(cap) * (int64_t)sizeof(double);
}
// Hot rows of v that fit beside the stages, for k columns.
template <typename VecT>
int64_t hot_rows_limit(int64_t k, int block, int cap)
{
    return (LDS_BYTES / vtm_wgs_per_cu(block) - 256 - vtm_stage_bytes(block, cap)) / ((int64_t)sizeof(VecT) * k);
}

// Whether the single-vector column dots fit 16 waves per CU (128 registers
// per lane): binary32 vectors with 4- or 2-byte values, or chunks of 512
// (8 positions per lane) of any type.
template <int ITEMS, typename ValT, typename VecT>
constexpr bool vtm_fits_1024()
{
    return (sizeof(VecT) == 4 && sizeof(ValT) <= 4) || ITEMS <= 8;
}

// The column-dot workgroup size for a single-vector call: the matrix's choice
// for the vector type (spw_create_opts.wg_size or the tuner's), else 1,024
// threads for binary32 vectors with 4- or 2-byte values (16 waves hide more
// latency) and 512 otherwise.  1,024 needs few enough registers (above).  The worker
// tables of the column and merge-path partitions assume eight workers a workgroup: 512 threads,
// and under column partitioning 1,024 with chunks of 512 where one worker has more than twice the average
// nonzeros, two waves a worker.  There it alone decides, and its chunks of 512 take one wave
// 0.97 us each, of 1,024 1.42 (19,996 x 1.36e6, 9e6 nonzeros, one vector, us: chunks of 1,024 86, of 512 105
// and by two waves 71; columns by descending length 4,600, 6,300, 3,880).  The chunks, and so the
// results, are those of the other modes.
template <int ITEMS, typename ValT, typename VecT>
int vtm_block_for(const spw_matrix_s &A, bool colpart)
{
    const bool pairs = ITEMS == 8 && A.partition == SPW_PART_COLUMN &&
                       A.cd.worker_max_nnz * A.cd.n_workers > 2 * A.cd.nnz;
    if (colpart) return pairs ? 2 * VTM_BLOCK : VTM_BLOCK;
    int b = A.vtm_block[sizeof(VecT) == 8 ? 0 : 1];
    if (b == 0) b = (sizeof(VecT) == 4 && sizeof(ValT) <= 4) ? VTM_BLOCK_F32 : VTM_BLOCK;
    if (b == 1024 && !vtm_fits_1024<ITEMS, ValT, VecT>()) b = VTM_BLOCK;
    return b;
}

// The segments of a chunk that the column dots stage for these vectors.  A stage takes LDS from
// the hot rows of v, so it is as large as the columns need:
// - binary64 vectors 256, or 512 where more than one chunk in eight has more than 256 (columns
//   of one or two nonzeros; chunks of 512 only);
// - binary32 vectors none with chunks of 1,024, and with chunks of 512 only where columns are
//   short (fewer than two nonzeros, two and a half for several vectors: 8e6, one a column, binary32
//   values, us without and with, one vector 39 / 30, three 132 / 76)
//   or have empty ones among them all over (3 a column 36 / 32, 97 / 87) and, for one
//   vector, all of v still fits: sixteen waves' stages take 19,000 of 40,000 hot rows (50,000 rows, uniform,
//   2.9e7 nonzeros, binary32 values: 66 us without, 100 with them; no empty columns, 20,000 rows,
//   eight vectors at 5e7 595 and 665).
template <typename ValT, typename VecT>
int vtm_stage(const spw_matrix_s &A, int k)
{
    const ColDot &C = A.cd;
    if (sizeof(VecT) == 8) return C.stage64;
    if (C.zp.chunk != 512) return 0;
    if (2 * C.nnz < (k > 1 ? 5 : 4) * (C.cols - C.n_empty)) return 512;
    const bool fits = k > 1 || A.rows <= hot_rows_limit<VecT>(1, vtm_block_for<8, ValT, VecT>(A, C.d_wchunks), 512);
    return C.gaps && fits ? 512 : 0;
}

template <int ITEMS, int CAP, typename IdxT, typename ValT, typename VecT, bool MULTI>
int launch_vtm_wave_items(const spw_matrix_s &A, const VecT *vin, int k, const ColOut<VecT> &out,
                          hipStream_t stream, void *stop)
{
    const ColDot &C = A.cd;
    const int cus = device_cu_count(A.device);
    // column partitioning: one wave per worker of the plan (single-vector calls)
    const int32_t *wch = (!MULTI && C.d_wchunks) ? C.d_wchunks : nullptr;
    const int block = MULTI ? VTM_BLOCK : vtm_block_for<ITEMS, ValT, VecT>(A, wch != nullptr);
    const int vhot = (int)std::min<int64_t>(A.rows, hot_rows_limit<VecT>(k, block, CAP));
    const size_t lds = (size_t)vtm_stage_bytes(block, CAP) + (size_t)vhot * k * sizeof(VecT);
    auto run = [&](auto kernel) -> int {
        const int nw = block / WAVE;
        const int64_t wgs_needed = (C.zp.n_chunks + nw - 1) / nw;
        const unsigned grid =
            wch ? (unsigned)(C.n_workers / (VTM_BLOCK / WAVE))
                : (unsigned)std::max<int64_t>(1, std::min<int64_t>((int64_t)cus * vtm_wgs_per_cu(block), wgs_needed));
        return launch_kernel(kernel, dim3(grid), dim3(block), lds, stream, stop, (const IdxT *)C.d_idx,
                             (const ValT *)C.d_val, C.d_heads, (const int4 *)C.d_cinfo, C.d_segcol, C.nnz,
                             C.zp.n_chunks, wch, vin, k, vhot, out, A.scratch.carry, C.gap_max);
    };
    if constexpr (!MULTI && vtm_fits_1024<ITEMS, ValT, VecT>()) {
        if (block == 1024) {
            static const bool attr_w = allow_full_lds(vtm_wave<1024, ITEMS, CAP, IdxT, ValT, VecT, MULTI>);
            (void)attr_w;
            return run(vtm_wave<1024, ITEMS, CAP, IdxT, ValT, VecT, MULTI>);
        }
    }
    if constexpr (!MULTI) {
        if (block == 256) {
            static const bool attr_q = allow_full_lds(vtm_wave<256, ITEMS, CAP, IdxT, ValT, VecT, MULTI>);
            (void)attr_q;
            return run(vtm_wave<256, ITEMS, CAP, IdxT, ValT, VecT, MULTI>);
        }
    }
    static const bool attr = allow_full_lds(vtm_wave<VTM_BLOCK, ITEMS, CAP, IdxT, ValT, VecT, MULTI>);
    (void)attr;
    return run(vtm_wave<VTM_BLOCK, ITEMS, CAP, IdxT, ValT, VecT, MULTI>);
}

// Chunks of 1,024 (16 positions per lane) or 512 (8 per lane) nonzeros; stage: vtm_stage.
template <typename IdxT, typename ValT, typename VecT, bool MULTI>
int launch_vtm_wave(const spw_matrix_s &A, int stage, const VecT *vin, int k, const ColOut<VecT> &out,
                    hipStream_t stream, void *stop)
{
    constexpr int SMALL = sizeof(VecT) == 8 ? 256 : 0;
    if (A.cd.zp.chunk == 1024)
        return launch_vtm_wave_items<16, SMALL, IdxT, ValT, VecT, MULTI>(A, vin, k, out, stream, stop);
    if (A.cd.zp.chunk == 512 && stage == 512)
        return launch_vtm_wave_items<8, 512, IdxT, ValT, VecT, MULTI>(A, vin, k, out, stream, stop);
    if (A.cd.zp.chunk == 512)
        return launch_vtm_wave_items<8, SMALL, IdxT, ValT, VecT, MULTI>(A, vin, k, out, stream, stop);
    return (int)hipErrorNotSupported;
}

// Which list of empty columns the column-dot kernel leaves to zero_cols: 0 all of them, 1 those
// not written with the segments of chunks staged for binary64 vectors, 2 for binary32 ones.
template <typename VecT>
int empty_set(int stage)
{
    return stage == 0 ? 0 : sizeof(VecT) == 8 ? 1 : 2;
}
// The largest output stride of the staged copy (the kernel's own condition).
template <typename VecT>
int64_t staged_ld_limit(const ColDot &C)
{
    return (int64_t)(1 << 28) / (C.zp.chunk * (int64_t)sizeof(VecT));
}

template <typename ValT, typename VecT>
int vtm_typed(const spw_matrix_s &A, const VecT *v, VecT *u, bool renumbered, hipStream_t stream)
{
    const ColDot &C = A.cd;
    int e;
    if (C.cols == 0) return 0;
    // the kernel writes the empty columns between a staged chunk's segments itself, unless
    // there is nothing else to do
    const int stage = vtm_stage<ValT, VecT>(A, 1);
    const int set = C.nnz == 0 ? 0 : empty_set<VecT>(stage);
    const int64_t n_empty = C.n_empty_of[set];
    if (n_empty > 0) {
        ProfScope ps(stream, "zero_cols");
        hipLaunchKernelGGL(zero_cols<VecT>, dim3(blocks_for(n_empty, 256)), dim3(256), 0, stream, C.d_empty_of[set],
                           n_empty, u);
        if ((e = (int)hipGetLastError())) return e;
    }
    if (C.nnz == 0) return 0;
    const VecT *vin = v;
    if (A.relabeled && !renumbered) {
        ProfScope ps(stream, "gather_vec");
        VecT *vp = reinterpret_cast<VecT *>(A.scratch.vperm);
        hipLaunchKernelGGL(gather_vec<VecT>, dim3(blocks_for(A.rows, 256)), dim3(256), 0, stream, A.d_inv, A.rows, v,
                           vp);
        if ((e = (int)hipGetLastError())) return e;
        vin = vp;
    }
    {
        ProfScope ps(stream, "vtm_wave");
        ColOut<VecT> out{};
        out.u[0] = u;
        out.ld[0] = 1;
        void *stop = C.n_zones > 0 ? nullptr : take_stop();
        e = C.idx_kind == IdxKind::U16 ? launch_vtm_wave<uint16_t, ValT, VecT, false>(A, stage, vin, 1, out, stream, stop)
                                       : launch_vtm_wave<int32_t, ValT, VecT, false>(A, stage, vin, 1, out, stream, stop);
        if (e) return e;
    }
    if (C.n_zones > 0) {
        ProfScope ps(stream, "zone_fixup");
        e = launch_kernel(zone_fixup<VecT>, dim3(blocks_for(C.n_zones, 256)), dim3(256), 0, stream, take_stop(),
                          C.d_zone_col, C.d_zone_first, C.d_zone_last, C.n_zones, A.scratch.carry, u);
        if (e) return e;
    }
    return 0;
}

// Up to MULTI_MAX columns in one pass, each with its own input and output
// base and stride; every column is bit-identical to the single-vector product.
template <typename ValT, typename VecT>
int vtm_cols_typed(const spw_matrix_s &A, int k, const ColIn<VecT> &in, const ColOut<VecT> &out, bool last,
                   hipStream_t stream)
{
    const ColDot &C = A.cd;
    int e;
    if (C.cols == 0) return 0;
    bool wide = false;                            // an output stride the staged copy does not take
    for (int c = 0; c < k; ++c) wide = wide || out.ld[c] > staged_ld_limit<VecT>(C);
    const int stage = vtm_stage<ValT, VecT>(A, k);
    const int set = C.nnz == 0 || wide ? 0 : empty_set<VecT>(stage);
    const int64_t n_empty = C.n_empty_of[set];
    if (n_empty > 0) {
        ProfScope ps(stream, "zero_cols");
        hipLaunchKernelGGL(zero_cols_tab<VecT>, dim3(blocks_for(n_empty * k, 256)), dim3(256), 0, stream,
                           C.d_empty_of[set], n_empty, k, out);
        if ((e = (int)hipGetLastError())) return e;
    }
    if (C.nnz == 0) return 0;
    VecT *vp = reinterpret_cast<VecT *>(A.scratch.vperm);
    {
        // the k inputs, renumbered when the rows are, as one rows x k block
        ProfScope ps(stream, "gather_vec");
        hipLaunchKernelGGL(gather_tab<VecT>, dim3(blocks_for(A.rows * k, 256)), dim3(256), 0, stream,
                           A.relabeled ? A.d_inv : nullptr, A.rows, k, in, vp);
        if ((e = (int)hipGetLastError())) return e;
    }
    {
        ProfScope ps(stream, "vtm_wave_multi");
        void *stop = C.n_zones > 0 || !last ? nullptr : take_stop();
        e = C.idx_kind == IdxKind::U16 ? launch_vtm_wave<uint16_t, ValT, VecT, true>(A, stage, vp, k, out, stream, stop)
                                       : launch_vtm_wave<int32_t, ValT, VecT, true>(A, stage, vp, k, out, stream, stop);
        if (e) return e;
    }
    if (C.n_zones > 0) {
        ProfScope ps(stream, "zone_fixup");
        e = launch_kernel(zone_fixup_tab<VecT>, dim3(blocks_for(C.n_zones * k, 256)), dim3(256), 0, stream,
                          last ? take_stop() : nullptr, C.d_zone_col, C.d_zone_first, C.d_zone_last, C.n_zones, k,
                          A.scratch.carry, out);
        if (e) return e;
    }
    return 0;
}

template <typename VecT>
void fill_tables(int k, const void *const *in, const int64_t *ldi, void *const *out, const int64_t *ldo,
                 ColIn<VecT> &ti, ColOut<VecT> &to)
{
    ti = ColIn<VecT>{};
    to = ColOut<VecT>{};
    for (int c = 0; c < k; ++c) {
        ti.v[c] = (const VecT *)in[c];
        ti.ld[c] = ldi[c];
        to.u[c] = (VecT *)out[c];
        to.ld[c] = ldo[c];
    }
}

// Sums the partials of `k` columns into their outputs.
template <typename VecT>
int launch_mv_reduce(const spw_matrix_s &A, const double *partial, int k, const ColOut<VecT> &out, bool last,
                     hipStream_t stream)
{
    ProfScope ps(stream, "mv_reduce");
    auto run = [&](auto kernel, unsigned blocks, unsigned panel_blocks) {
        return launch_kernel(kernel, dim3(blocks, (unsigned)k), dim3(256), 0, stream, last ? take_stop() : nullptr, partial,
                             (int)A.panel_rows, (int)panel_blocks, A.d_panels, (int)A.n_panels,
                             A.relabeled ? A.d_inv : nullptr, out, A.mv_wgs * A.panel_rows);
    };
    if (A.panel_wgs <= MV_FEW) return run(mv_reduce<VecT, true>, blocks_for(A.n_panels * A.panel_rows, 256), 0u);
    const unsigned panel_blocks = blocks_for(A.panel_rows, 32);
    return run(mv_reduce<VecT, false>, (unsigned)A.n_panels * panel_blocks, panel_blocks);
}

// Columns of one launch that share an LDS panel: as many as fit, at most MV_COLS.
int mv_cols_together(const spw_matrix_s &A)
{
    return (int)std::max<int64_t>(1, std::min<int64_t>(MV_COLS, mv_lds_rows_limit(SPW_F64, 1) / A.panel_slots));
}

// One launch of the scatter kernel for k <= MULTI_MAX columns with their own
// inputs and outputs (the partial sums hold k columns), then their reductions in
// one launch.  Columns that are adjacent entries of the same rows are taken
// in groups of up to mv_cols_together, of sizes that differ by one at most.
template <typename ValT, typename VecT>
int mv_cols_typed(const spw_matrix_s &A, int k, const ColIn<VecT> &in, const ColOut<VecT> &out, bool last,
                  hipStream_t stream)
{
    int e;
    const int W = (int)A.mv_wgs;
    if (W > 0) {
        static const bool attr = allow_full_lds(mv_bucket_cols<MV_BLOCK, ValT, VecT>);
        (void)attr;
        const int most = mv_cols_together(A);
        MvGroups<VecT> gr{};
        int ng = 0, widest = 1;
        for (int c = 0; c < k;) {
            int run = 1;                          // adjacent columns from c on
            while (c + run < k && in.v[c + run] == in.v[c] + run && in.ld[c + run] == in.ld[c]) ++run;
            const int parts = (run + most - 1) / most;
            for (int q = 0; q < parts; ++q, ++ng) {
                const int a = run * q / parts, n = run * (q + 1) / parts - a;
                gr.x[ng] = in.v[c + a];
                gr.ld[ng] = in.ld[c + a];
                gr.kc[ng] = n;
                gr.slot[ng] = c + a;
                widest = std::max(widest, n);
            }
            c += run;
        }
        ProfScope ps(stream, "mv_bucket");
        hipLaunchKernelGGL((mv_bucket_cols<MV_BLOCK, ValT, VecT>), dim3((unsigned)(8 * ng * ((W + 7) / 8))),
                           dim3(MV_BLOCK), (size_t)A.panel_slots * 8 * (size_t)widest, stream,
                           (const uint32_t *)A.d_mpacked, (const ValT *)A.d_mval, (const int2 *)A.d_mblocks,
                           A.d_wg_blk, A.d_wg_order, gr, ng, A.scratch.partial_cols, (int)A.panel_slots,
                           (int)A.panel_rows, A.row_copies_log, A.d_hot, (const int2 *)A.d_wg_hot, W);
        if ((e = (int)hipGetLastError())) return e;
    }
    return launch_mv_reduce<VecT>(A, A.scratch.partial_cols, k, out, last, stream);
}

// k right-hand sides, up to pcols columns a launch when the multi-column partial
// sums are there, else one column after another.
template <typename ValT, typename VecT>
int mv_typed(const spw_matrix_s &A, int32_t k, const VecT *x, int64_t ldx, VecT *y, int64_t ldy, hipStream_t stream)
{
    if (A.rows == 0) return 0;
    int e;
    if (k > 1 && A.mv_wgs > 0 && A.scratch.partial_cols && A.scratch.pcols > 0) {
        const int most = std::min<int>(A.scratch.pcols, MULTI_MAX);
        for (int32_t c0 = 0; c0 < k; c0 += most) {
            const int kb = std::min<int>(most, k - c0);
            ColIn<VecT> in{};
            ColOut<VecT> out{};
            for (int c = 0; c < kb; ++c) {
                in.v[c] = x + c0 + c;
                in.ld[c] = ldx;
                out.u[c] = y + c0 + c;
                out.ld[c] = ldy;
            }
            if ((e = mv_cols_typed<ValT, VecT>(A, kb, in, out, c0 + kb == k, stream))) return e;
        }
        return 0;
    }
    static const bool attr = allow_full_lds(mv_bucket<MV_BLOCK, ValT, VecT>);
    (void)attr;
    for (int32_t c = 0; c < k; ++c) {
        if (A.mv_wgs > 0) {
            ProfScope ps(stream, "mv_bucket");
            const size_t lds = (size_t)A.panel_slots * 8;
            hipLaunchKernelGGL((mv_bucket<MV_BLOCK, ValT, VecT>), dim3((unsigned)A.mv_wgs), dim3(MV_BLOCK), lds,
                               stream, (const uint32_t *)A.d_mpacked, (const ValT *)A.d_mval,
                               (const int2 *)A.d_mblocks, A.d_wg_blk, A.d_wg_order, x + c, ldx, A.scratch.partial,
                               (int)A.panel_slots, (int)A.panel_rows, A.row_copies_log, A.d_hot, (const int2 *)A.d_wg_hot);
            if ((e = (int)hipGetLastError())) return e;
        }
        ColOut<VecT> out{};
        out.u[0] = y + c;
        out.ld[0] = ldy;
        if ((e = launch_mv_reduce<VecT>(A, A.scratch.partial, 1, out, c + 1 == k, stream))) return e;
    }
    return 0;
}

}  // namespace

int64_t mv_lds_rows_limit(spw_dtype vdt, int32_t k)
{
    (void)vdt;
    return std::min<int64_t>((LDS_BYTES - 256) / (8 * std::max<int32_t>(k, 1)), 65536);
}
int64_t mv_block_nnz() { return MV_BLK; }
int64_t mv_waves() { return MV_BLOCK / WAVE; }
int64_t vtm_chunk_default() { return (int64_t)WAVE * VTM_ITEMS; }
bool vtm_chunk_supported(int64_t chunk) { return chunk == 512 || chunk == 1024; }
int64_t vtm_workers(int device, int64_t nchunks)
{
    const int64_t nw = VTM_BLOCK / WAVE;
    const int64_t wgs = std::max<int64_t>(1, std::min<int64_t>((int64_t)device_cu_count(device) * VTM_WG_PER_CU,
                                                               (nchunks + nw - 1) / nw));
    return wgs * nw;
}

int device_cu_count(int device)
{
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) return 256;
    return cus > 0 ? cus : 256;
}

int launch_vtm(const spw_matrix_s &A, spw_dtype vdt, const void *v, void *u, void *stream, bool renumbered)
{
    return with_types(A.value_storage, vdt, [&](auto vt, auto xt) {
        using ValT = decltype(vt);
        using VecT = decltype(xt);
        return vtm_typed<ValT, VecT>(A, (const VecT *)v, (VecT *)u, renumbered, (hipStream_t)stream);
    });
}

int launch_vtm_cols(const spw_matrix_s &A, spw_dtype vdt, int32_t k, const void *const *in, const int64_t *ldi,
                    void *const *out, const int64_t *ldo, void *stream, bool last)
{
    if (k < 1 || k > MULTI_MAX) return (int)hipErrorInvalidValue;
    return with_types(A.value_storage, vdt, [&](auto vt, auto xt) {
        using ValT = decltype(vt);
        using VecT = decltype(xt);
        ColIn<VecT> ti;
        ColOut<VecT> to;
        fill_tables<VecT>(k, in, ldi, out, ldo, ti, to);
        return vtm_cols_typed<ValT, VecT>(A, k, ti, to, last, (hipStream_t)stream);
    });
}

int launch_vtm_multi(const spw_matrix_s &A, spw_dtype vdt, int32_t k, const void *v, int64_t ldv, void *u,
                     int64_t ldu, void *stream)
{
    const size_t es = vdt == SPW_F64 ? 8 : 4;
    for (int c0 = 0; c0 < k; c0 += MULTI_MAX) {
        const int kk = std::min(MULTI_MAX, k - c0);
        const void *in[MULTI_MAX];
        void *out[MULTI_MAX];
        int64_t li[MULTI_MAX], lo[MULTI_MAX];
        for (int c = 0; c < kk; ++c) {
            in[c] = (const char *)v + (size_t)(c0 + c) * es;
            out[c] = (char *)u + (size_t)(c0 + c) * es;
            li[c] = ldv;
            lo[c] = ldu;
        }
        const int e = launch_vtm_cols(A, vdt, kk, in, li, out, lo, stream, c0 + kk == k);
        if (e) return e;
    }
    return 0;
}

int launch_mv(const spw_matrix_s &A, spw_dtype vdt, int32_t k, const void *x, int64_t ldx, void *y, int64_t ldy,
              void *stream)
{
    return with_types(A.value_storage, vdt, [&](auto vt, auto xt) {
        using ValT = decltype(vt);
        using VecT = decltype(xt);
        return mv_typed<ValT, VecT>(A, k, (const VecT *)x, ldx, (VecT *)y, ldy, (hipStream_t)stream);
    });
}

int launch_mv_cols(const spw_matrix_s &A, spw_dtype vdt, int32_t k, const void *const *in, const int64_t *ldi,
                   void *const *out, const int64_t *ldo, void *stream)
{
    if (k < 1 || k > MULTI_MAX) return (int)hipErrorInvalidValue;
    if (k == 1 || A.scratch.pcols < k || !A.scratch.partial_cols) {
        // one column, or no multi-column partial sums: one pass per column
        for (int c = 0; c < k; ++c) {
            const int e = launch_mv(A, vdt, 1, in[c], ldi[c], out[c], ldo[c], stream);
            if (e) return e;
        }
        return 0;
    }
    return with_types(A.value_storage, vdt, [&](auto vt, auto xt) {
        using ValT = decltype(vt);
        using VecT = decltype(xt);
        ColIn<VecT> ti;
        ColOut<VecT> to;
        fill_tables<VecT>(k, in, ldi, out, ldo, ti, to);
        if (A.rows == 0) return 0;
        return mv_cols_typed<ValT, VecT>(A, k, ti, to, true, (hipStream_t)stream);
    });
}

}  // namespace spw
