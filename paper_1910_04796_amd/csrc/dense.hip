// dense.hip -- densification path: merge blocks into panels, one MFMA GEMM
// (FP64, or FP32 for single-precision matrices), split the result back into
// the blocks of C.
//
// Paper, Sec. III: when the inputs are dense, all blocks handled by a worker
// are coalesced into one large block by copying them into new buffers, the
// product becomes a single GEMM, and C is undensified at the end.  With one
// rank and one panel (Eqs. (1)-(2) with P~ = 1, t = 1) the panels are the
// whole matrices: A -> Ap (M x K), B -> Bp (K x N), both column-major and
// zero-padded to the GEMM tile.  The undensify step is fused into the GEMM
// epilogue, which writes C = beta*C + alpha*(Ap Bp) straight into C's
// blocks through per-row and per-column (block, offset) maps.
//
// GEMM: 128 x 128 output tile per 512-thread workgroup, k step 16, LDS double
// buffered and filled straight from memory; each wave owns 64 rows x 32
// columns as 4 x 2 MFMA tiles of v_mfma_f64_16x16x4 (FP64 in, FP64
// accumulate); with k step 32, 256 threads and 64 x 64 outputs per wave.
// Workgroup ids are remapped
// so that the tiles dispatched to one XCD form a contiguous band of
// 8 tile-rows (shared A panels stay in that XCD's L2).  When the output
// has too few tiles to fill the GPU (M = N = 1408 with K in the millions:
// 121 tiles for 256 CUs), k is split across workgroups; the partial tiles
// are summed in a fixed order by a second kernel that applies the epilogue.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "dev_util.h"
#include "internal.h"
#include "launch_rules.h"
#include "mfma_util.h"

namespace bsmm {

namespace {

// One operand of a densified product and its panel.
template <class T> struct MergeArgs {
    int32_t nbr, full_nbc;  // block rows; block columns when every block is stored, else 0
    int64_t nnzb;
    const int32_t *rbs, *cbs;
    const int64_t *row_off, *col_off, *rp;
    const int32_t *ci;
    const int64_t *blk_off;
    const T *data;
    T *panel;
    int64_t ld, ncols, rows, cols;  // of the panel; of the matrix
    int64_t pad_first;              // padding: first column that has any (ncols: none)
};

// Zeros in the padding of two column-major panels of ld x ncols whose merges
// fill rows x cols: the rows below in the first columns, then whole columns
// (one workgroup per column; the first wgs_a workgroups serve a).
template <class T>
__global__ __launch_bounds__(256) void k_zero_padding(MergeArgs<T> a, MergeArgs<T> b, int wgs_a) {
    const bool first = (int)blockIdx.x < wgs_a;
    const MergeArgs<T> &g = first ? a : b;
    const int64_t wg = first ? blockIdx.x : blockIdx.x - wgs_a, wgs = first ? wgs_a : gridDim.x - wgs_a;
    for (int64_t c = g.pad_first + wg; c < g.ncols; c += wgs)
        for (int64_t r = (c < g.cols ? g.rows : 0) + threadIdx.x; r < g.ld; r += blockDim.x) g.panel[c * g.ld + r] = T(0);
}

constexpr int BM = 128, BN = 128;
constexpr int kGroupM = 8;

// Merge of blocks of 64 elements or more: one wave per block (block row
// found by binary search in the row pointer, or by division when every
// block is stored), copying the column-major block into the column-major panel;
// consecutive lanes write consecutive rows of a column.  Both operands in
// one launch (the first wgs_a workgroups serve a), which fills the GPU where
// one alone does not: 1,900 x 2,300 and 2,300 x 1,700 in {5,13,22}-blocks 2 x 38
// us, together 41; 8192 x 8192 in 32-blocks 2 x 209 us, together 406 (5.3 TB/s).
template <class T>
__global__ __launch_bounds__(256) void k_merge_block(MergeArgs<T> a, MergeArgs<T> b, int wgs_a) {
    const bool first = (int)blockIdx.x < wgs_a;
    const MergeArgs<T> &g = first ? a : b;
    const int64_t wg = first ? blockIdx.x : blockIdx.x - wgs_a, wgs = first ? wgs_a : gridDim.x - wgs_a;
    const int64_t waves = wgs * (blockDim.x / kWave);
    for (int64_t p = wg * (blockDim.x / kWave) + wave_id(); p < g.nnzb; p += waves) {
        int32_t lo = g.full_nbc ? (int32_t)((uint32_t)p / (uint32_t)g.full_nbc) : 0;
        int32_t hi = g.full_nbc ? lo : g.nbr;  // row = last lo with rp[lo] <= p
        while (hi - lo > 1) {
            const int32_t mid = (lo + hi) >> 1;
            if (g.rp[mid] <= p) lo = mid;
            else hi = mid;
        }
        const int32_t row = lo;
        const int m = g.rbs[row];
        const int64_t r0 = g.row_off[row];
        const int32_t j = g.ci[p];
        const int n = g.cbs[j];
        const int64_t c0 = g.col_off[j];
        const T *src = g.data + g.blk_off[p];
        T *panel = g.panel;
        const int64_t len = (int64_t)m * n, ld = g.ld;
        if (len < (1 << 20) && m < 4096) {
            const float rcp = 1.0f / (float)m;
            for (int e = lane_id(); e < len; e += kWave) {
                int ii;
                const int jj = divmod_small(e, m, rcp, &ii);
                panel[(c0 + jj) * ld + r0 + ii] = src[e];
            }
        } else {
            for (int64_t e = lane_id(); e < len; e += kWave)
                panel[(c0 + e / m) * ld + r0 + e % m] = src[e];
        }
    }
}

// Merge of blocks of fewer than 64 elements, where one wave per block would
// leave most lanes idle: one wave per chunk of 64 consecutive blocks.  Lane
// l takes block p0 + l (its block row by binary search in the row pointer,
// all lanes at once), and a running sum of the block lengths over the wave
// lays the chunk's elements out in one flat range; the wave walks that
// range 64 elements at a time, each lane stepping forward through the 64
// running sums in LDS to its block, and copies from the column-major block
// into the column-major panel (ld = panel rows).
constexpr int kMergeWaves = 4;
template <class T>
__global__ __launch_bounds__(kMergeWaves * kWave) void k_merge_chunk(
    int32_t nbr, int64_t nnzb, const int32_t *rbs, const int32_t *cbs, const int64_t *row_off,
    const int64_t *col_off, const int64_t *rp, const int32_t *ci, const int64_t *blk_off, const T *data,
    T *panel, int64_t ld) {
    __shared__ int64_t s_end[kMergeWaves][kWave], s_src[kMergeWaves][kWave], s_dst[kMergeWaves][kWave];
    __shared__ int32_t s_m[kMergeWaves][kWave];
    const int w = wave_id(), l = lane_id();
    const int64_t step = (int64_t)gridDim.x * kMergeWaves * kWave;
    for (int64_t p0 = ((int64_t)blockIdx.x * kMergeWaves + w) * kWave; p0 < nnzb; p0 += step) {
        const int64_t p = p0 + l;
        int64_t len = 0, src = 0, dst = 0;
        int m = 1;
        if (p < nnzb) {
            int32_t lo = 0, hi = nbr;  // row = last lo with rp[lo] <= p
            while (hi - lo > 1) {
                const int32_t mid = (lo + hi) >> 1;
                if (rp[mid] <= p) lo = mid;
                else hi = mid;
            }
            m = rbs[lo];
            const int32_t j = ci[p];
            len = (int64_t)m * cbs[j];
            src = blk_off[p];
            dst = col_off[j] * ld + row_off[lo];
        }
        int64_t end = len;  // inclusive running sum over the wave
        for (int d = 1; d < kWave; d <<= 1) {
            const int64_t v = __shfl_up(end, d, kWave);
            if (l >= d) end += v;
        }
        s_end[w][l] = end;
        s_src[w][l] = src;
        s_dst[w][l] = dst;
        s_m[w][l] = m;
        wave_lds_sync();
        const int64_t total = __shfl(end, kWave - 1, kWave);
        int b = 0;  // first block whose running sum exceeds e (e only grows)
        for (int64_t e = l; e < total; e += kWave) {
            while (s_end[w][b] <= e) ++b;
            const int64_t off = e - (b ? s_end[w][b - 1] : 0);
            const int mb = s_m[w][b];
            int64_t jj, ii;
            if (off < (1 << 20) && mb < 4096) {
                int r;
                jj = divmod_small((int)off, mb, 1.0f / (float)mb, &r);
                ii = r;
            } else {
                jj = off / mb;
                ii = off - jj * mb;
            }
            panel[s_dst[w][b] + jj * ld + ii] = data[s_src[w][b] + off];
        }
        wave_lds_sync();  // every lane has read the chunk before it is replaced
    }
}

struct GemmArgs {
    const void *Ap;     // M_pad x K_pad, column-major, ld = lda (element type of the matrices)
    const void *Bp;     // K_pad x N_pad, column-major, ld = ldb
    int64_t lda, ldb;
    int tiles_m, tiles_n, ktiles;
    int64_t M, N;       // true sizes (rows/cols of C)
    double alpha, beta;
    void *C;            // C block data
    const int64_t *c_blk_off;
    const int32_t *c_map;   // nbr*nbc block index map, or null when C is full
    int32_t c_nbc;
    const int32_t *c_rbs;
    const int2 *rmap, *cmap;
    int tile0, ntiles;  // tiles of this launch
    // Split k: workgroup (tile, split) sums k tiles
    // [split * kt_per, (split + 1) * kt_per) into part[split] (unscaled, per
    // tile in the waves' accumulator order); k_splitk_reduce applies the
    // epilogue.
    int splits, kt_per;
    void *part;
};

// The place in LDS of the g-th 16 bytes of a column of the B tile is
// g ^ b_swizzle(col): the columns whose first bytes share a bank take
// different places, so the 16 columns that are read together at one k lie on
// distinct banks.
template <class T, int KB>
__device__ __forceinline__ int b_swizzle(int col) {
    constexpr int kGran = KB * (int)sizeof(T) / 16, kShare = 16 / kGran;  // columns per 256 bytes of banks
    return (kShare > 1 ? col / kShare : col) & (kGran - 1);
}

// Copy of one k step of KB from the panels straight into LDS, 16 bytes per
// lane and 1 KB per wave and instruction: A as [k][row], B as [col][place].
// A wave's KBs start at scalar addresses and its lanes add a fixed offset to
// them, so a step costs the vector unit next to nothing: FP64 MFMAs and
// vector instructions of a SIMD exclude each other here, and the 60 vector
// instructions that each 32 MFMAs carried for addresses, bank swizzles and
// LDS stores were most of what the matrix cores lost (86 % busy; 93 % now).
// FP64 offsets have 32 bits (the widest is that of B's last column in a KB:
// dense_multiply_t picks the k step by it), FP32 ones 64.
template <class T, int KB, int NTH>
struct StepCopy {
    static constexpr int kGran = KB * (int)sizeof(T) / 16;                // 16-byte places of a column
    static constexpr int kVec = 16 / (int)sizeof(T);                      // elements per lane
    static constexpr int kPer = KB * (int)sizeof(T) / 8 / (NTH / kWave);  // KBs of each tile per wave
    typedef typename std::conditional<sizeof(T) == 8, uint32_t, int64_t>::type Off;
    typedef __attribute__((address_space(1))) const void *Src;
    typedef __attribute__((address_space(3))) void *Dst;
    const char *a, *b[kPer];  // of the wave, at k = 0
    Off a_off, b_off[kPer];   // of the lane, bytes
    int64_t lda;
    int lds;  // the wave's first element in a tile

    __device__ __forceinline__ StepCopy(const T *Ablk, const T *Bblk, int64_t lda_, int64_t ldb, int w, int lane)
        : lda(lda_ * (int64_t)sizeof(T)) {
        lds = w * kPer * 64 * kVec;
        a = reinterpret_cast<const char *>(Ablk + (int64_t)(lds / BM) * lda_);
        a_off = (Off)(lane * kVec / BM) * (Off)lda + (lane * kVec % BM) * (int)sizeof(T);
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int p0 = w * kPer * 64 + i * 64, c0 = p0 / kGran, col = (p0 + lane) / kGran;
            b[i] = reinterpret_cast<const char *>(Bblk + (int64_t)c0 * ldb);
            b_off[i] = (Off)(col - c0) * (Off)(ldb * (int64_t)sizeof(T)) +
                       (((p0 + lane) % kGran) ^ b_swizzle<T, KB>(col)) * 16;
        }
    }
    __device__ __forceinline__ void operator()(int kt, T *As, T *Bs) const {
        const int64_t k0 = (int64_t)kt * KB;
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            __builtin_amdgcn_global_load_lds((Src)(a + (k0 + i * (64 * kVec / BM)) * lda + a_off),
                                             (Dst)(As + lds + i * 64 * kVec), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            __builtin_amdgcn_global_load_lds((Src)(b[i] + k0 * (int)sizeof(T) + b_off[i]),
                                             (Dst)(Bs + lds + i * 64 * kVec), 16, 0, 0);
    }
};

// This wave's copies to LDS have landed, then every wave of the workgroup is here.
__device__ __forceinline__ void step_sync() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

// One k step: wave (wm, wn) multiplies rows (2 t + wm) * 16 .. + 15 (t < 4)
// with columns wn * 16 NT ...  The rows of a wave alternate with the other's
// so that the four reads of a k lie 512 bytes apart in pairs: one address
// register serves all k of the step through the instructions' offsets.
template <class T, int KB, int NT>
__device__ __forceinline__ void gemm_step(const T *As, const T *Bs, int w, int lane,
                                          typename Mfma<T>::acc_t (&acc)[4][NT]) {
    constexpr int kVec = 16 / (int)sizeof(T);
    const int wm = w & 1, wn = w >> 1, l16 = lane & 15, lk = lane >> 4;
#pragma unroll
    for (int ks = 0; ks < KB / 4; ++ks) {
        const int k = ks * 4 + lk;
        T a[4], b[NT];
#pragma unroll
        for (int t = 0; t < 4; ++t) a[t] = As[k * BM + (t * 2 + wm) * 16 + l16];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int col = wn * 16 * NT + t * 16 + l16;
            b[t] = Bs[col * KB + ((k / kVec) ^ b_swizzle<T, KB>(col)) * kVec + k % kVec];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] = Mfma<T>::step(a[i], b[j], acc[i][j]);
    }
}

// Tiles in groups of kGroupM tile rows, the row index fastest: the tiles of an
// XCD share panels of A and B in its L2.
__device__ __forceinline__ void tile_at(const GemmArgs &g, int tile, int &tm, int &tn) {
    const int per_group = kGroupM * g.tiles_n;
    const int group = tile / per_group;
    const int first_m = group * kGroupM;
    const int gsz = min(g.tiles_m - first_m, kGroupM);
    const int in_group = tile - group * per_group;
    tm = first_m + in_group % gsz;
    tn = in_group / gsz;
}

// KB = 16: 64 KB of LDS, two workgroups per CU; KB = 32: 128 KB, one
// workgroup per CU with twice the prefetch distance and half the barriers.
// NT: 16-column tiles per wave.  Bound by the matrix cores.  N = 8192 in
// FP64: 16.82 ms with two waves per SIMD (NT = 4), 16.40 with four (NT = 2,
// which cover each other's barriers), 15.15 with copies straight to LDS and
// no address arithmetic in the loop (72.6 of 77.8 TFLOP/s); the same copies
// with 59 vector instructions per step for addresses: 16.37.
template <class T, int KB, int NT, int MINW, bool SPLIT>
__global__ __launch_bounds__(1024 / NT, MINW) void k_dgemm_mfma(GemmArgs g) {
    constexpr int NTH = 1024 / NT;
    // Two buffers of one k step, as objects of their own: the compiler sees
    // then that the copies into one do not touch what is read from the other
    // and does not end them before every LDS read.
    __shared__ __attribute__((aligned(16))) T As0[KB * BM], As1[KB * BM], Bs0[BN * KB], Bs1[BN * KB];

    // XCD-aware remap: each XCD takes a band of consecutive tiles (split k:
    // consecutive logical ids walk the tiles of one split).
    const int nwg = gridDim.x;
    int logical = blockIdx.x;
    {
        const int xcd = blockIdx.x & 7, rest = nwg & 7;
        logical = xcd * (nwg >> 3) + min(xcd, rest) + (blockIdx.x >> 3);
    }
    int split = 0, kt0 = 0, kt1 = g.ktiles;
    if (SPLIT) {
        split = logical / g.ntiles;
        logical -= split * g.ntiles;
        kt0 = split * g.kt_per;
        kt1 = min(g.ktiles, kt0 + g.kt_per);
    }
    int tm, tn;
    tile_at(g, g.tile0 + logical, tm, tn);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = tid >> 6;
    const int wm = w & 1, wn = w >> 1;
    const int l16 = lane & 15, lk = lane >> 4;

    const T *Ablk = static_cast<const T *>(g.Ap) + (int64_t)tm * BM;
    const T *Bblk = static_cast<const T *>(g.Bp) + (int64_t)tn * BN * g.ldb;

    typename Mfma<T>::acc_t acc[4][NT];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = Mfma<T>::zero();

    const StepCopy<T, KB, NTH> copy(Ablk, Bblk, g.lda, g.ldb, __builtin_amdgcn_readfirstlane(w), lane);
    copy(kt0, As0, Bs0);
    step_sync();
    for (int kt = kt0;;) {
        if (kt + 1 < kt1) copy(kt + 1, As1, Bs1);
        gemm_step<T, KB, NT>(As0, Bs0, w, lane, acc);
        step_sync();
        if (++kt >= kt1) break;
        if (kt + 1 < kt1) copy(kt + 1, As0, Bs0);
        gemm_step<T, KB, NT>(As1, Bs1, w, lane, acc);
        step_sync();
        if (++kt >= kt1) break;
    }

    // Epilogue: element e of lane l holds row Mfma<T>::row(e, l / 16),
    // column l % 16 of its 16 x 16 tile.
    const T alpha = (T)g.alpha, beta = (T)g.beta;
    if (SPLIT) {
        // Partial sums in the accumulators' own order: per 16 columns and
        // 64 rows, four consecutive 64-lane vectors.
        typename Mfma<T>::acc_t *P = static_cast<typename Mfma<T>::acc_t *>(g.part) +
                                     ((int64_t)split * g.ntiles + logical) * 4096 + lane;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) P[((wn * NT + j) * 8 + i * 2 + wm) * 64] = acc[i][j];
        return;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int64_t col = (int64_t)tn * BN + wn * 16 * NT + j * 16 + l16;
            if (col >= g.N) continue;
            const int2 cm = g.cmap[col];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t row = (int64_t)tm * BM + (i * 2 + wm) * 16 + Mfma<T>::row(e, lk);
                if (row >= g.M) continue;
                const int2 rm = g.rmap[row];
                const int64_t bidx = (int64_t)rm.x * g.c_nbc + cm.x;
                const int32_t blk = g.c_map ? g.c_map[bidx] : (int32_t)bidx;
                if (blk < 0) continue;
                T *dst = static_cast<T *>(g.C) + g.c_blk_off[blk] + rm.y + (int64_t)g.c_rbs[rm.x] * cm.y;
                const T prod = alpha * acc[i][j][e];
                *dst = (beta == T(0)) ? prod : fma(beta, *dst, prod);
            }
        }
    }
}

// Split-k epilogue: C(row, col) = beta C + alpha * (sum of the partials in
// split order), written into C's blocks.  One wave per 64 x 16 strip of a
// tile: it adds the strip's partials as the GEMM's lanes
// held them (32 bytes per lane, contiguous), turns the sums through LDS and
// writes C with consecutive lanes on consecutive rows of a column, the order
// of C's blocks.  Bound by HBM (the partials are read once).
template <class T>
__global__ __launch_bounds__(64) void k_splitk_reduce(GemmArgs g) {
    typedef typename Mfma<T>::acc_t V;
    __shared__ T s_out[16][65];
    const T alpha = (T)g.alpha, beta = (T)g.beta;
    const int lane = threadIdx.x, l16 = lane & 15, lk = lane >> 4;
    const int64_t strips = (int64_t)g.ntiles * 16, plane = (int64_t)g.ntiles * 4096;
    for (int64_t st = blockIdx.x; st < strips; st += gridDim.x) {
        const int64_t tile = st >> 4;
        const int part = (int)st & 15;  // 16 columns (part / 2) of one half of the rows (part % 2)
        int tm, tn;
        tile_at(g, g.tile0 + (int)tile, tm, tn);
        const int64_t row0 = (int64_t)tm * BM + (part & 1) * 64;
        const int64_t col0 = (int64_t)tn * BN + (part >> 1) * 16;
        if (row0 >= g.M || col0 >= g.N) continue;
        const V *p = static_cast<const V *>(g.part) + tile * 4096 + part * 256 + lane;
        V v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = p[i * 64];
        for (int sp = 1; sp < g.splits; ++sp) {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] += p[sp * plane + i * 64];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) s_out[l16][16 * i + Mfma<T>::row(e, lk)] = v[i][e];
        __syncthreads();
        const int64_t row = row0 + lane;
        const bool in = row < g.M;
        const int2 rm = in ? g.rmap[row] : make_int2(0, 0);
        const int ld = in ? g.c_rbs[rm.x] : 0;
        const int ncol = (int)min((int64_t)16, g.N - col0);
        // All lookups, then all old values, then the stores: one column after
        // the other made 16 chains of dependent loads (210 tiles of 2 parts
        // with beta = 1: 28 us, 23 so).
        T *dst[16];
        T old[16];
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            const int2 cm = g.cmap[col0 + min(c, ncol - 1)];
            const int64_t bidx = (int64_t)rm.x * g.c_nbc + cm.x;
            const int32_t blk = !in || c >= ncol ? -1 : g.c_map ? g.c_map[bidx] : (int32_t)bidx;
            dst[c] = blk < 0 ? nullptr : static_cast<T *>(g.C) + g.c_blk_off[blk] + rm.y + (int64_t)ld * cm.y;
        }
        if (beta != T(0)) {
#pragma unroll
            for (int c = 0; c < 16; ++c)
                if (dst[c]) old[c] = *dst[c];
        }
#pragma unroll
        for (int c = 0; c < 16; ++c)
            if (dst[c]) {
                const T prod = alpha * s_out[c][lane];
                *dst[c] = (beta == T(0)) ? prod : fma(beta, old[c], prod);
            }
        __syncthreads();  // the strip has been written before s_out is reused
    }
}

// c_map[I*nbc + J] = CSR position of block (I,J) in C, or -1.
__global__ __launch_bounds__(256) void k_block_map(int32_t nbr, int32_t nbc, const int64_t *rp,
                                                   const int32_t *ci, int32_t *map) {
    for (int32_t row = blockIdx.x; row < nbr; row += gridDim.x) {
        for (int j = threadIdx.x; j < nbc; j += blockDim.x) map[(int64_t)row * nbc + j] = -1;
        __syncthreads();
        for (int64_t p = rp[row] + threadIdx.x; p < rp[row + 1]; p += blockDim.x)
            map[(int64_t)row * nbc + ci[p]] = (int32_t)p;
        __syncthreads();
    }
}

}  // namespace

// Compute units of the current device (cached per device).
int cu_count() {
    static std::atomic<int> cache[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
        (void)hipGetLastError();
        return 256;
    }
    int n = cache[dev].load(std::memory_order_relaxed);
    if (n > 0) return n;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
        (void)hipGetLastError();
        return 256;
    }
    cache[dev].store(n, std::memory_order_relaxed);
    return n;
}


namespace {

template <class T>
MergeArgs<T> merge_args(const bsmm_matrix_s *M, T *panel, int64_t ld, int64_t ncols) {
    MergeArgs<T> g{M->nbr, M->full() ? M->nbc : 0, M->nnzb, M->d_rbs(), M->d_cbs(), M->d_row_off(), M->d_col_off(),
                   M->d_row_ptr(), M->d_col_ind(), M->d_blk_off(), (const T *)M->d_raw(), panel, ld, ncols, M->rows(),
                   M->cols(), 0};
    if (ld == M->rows()) g.pad_first = M->cols();  // no rows to pad: only the last columns
    return g;
}

// The panels of both operands: zeros in the padding of an operand that stores
// every block, everywhere else, then the blocks (those of fewer than 64
// elements in chunks of 64 blocks per wave).
template <class T>
int merge_panels(const bsmm_matrix_s *A, const bsmm_matrix_s *B, MergeArgs<T> a, MergeArgs<T> b, hipStream_t s) {
    for (MergeArgs<T> *g : {&a, &b})
        if (!g->full_nbc) {
            BSMM_TRY(fill_zero_bytes(g->panel, sizeof(T) * g->ld * g->ncols, s));
            g->pad_first = g->ncols;
        }
    const int64_t pa = a.ncols - a.pad_first, pb = b.ncols - b.pad_first;
    if (pa + pb > 0) {
        const unsigned ga = pa ? grid_of(pa, 1, kMaxGridBlocks / 2) : 0, gb = pb ? grid_of(pb, 1, kMaxGridBlocks / 2) : 0;
        hipLaunchKernelGGL(k_zero_padding<T>, dim3(ga + gb), dim3(256), 0, s, a, b, (int)ga);
        BSMM_TRY(launch_check("zero_padding"));
    }
    unsigned g[2] = {0, 0};
    const bsmm_matrix_s *M[2] = {A, B};
    for (int i = 0; i < 2; ++i) {
        const MergeArgs<T> &x = i ? b : a;
        if (x.nnzb == 0) continue;
        if ((int64_t)M[i]->max_rbs * M[i]->max_cbs >= kWave) {
            g[i] = grid_of(x.nnzb, 4, kMaxGridBlocks / 2);
            continue;
        }
        hipLaunchKernelGGL(k_merge_chunk<T>, dim3(grid_of(x.nnzb, kMergeWaves * kWave)), dim3(kMergeWaves * kWave), 0, s,
                           x.nbr, x.nnzb, x.rbs, x.cbs, x.row_off, x.col_off, x.rp, x.ci, x.blk_off, x.data, x.panel, x.ld);
        BSMM_TRY(launch_check("merge_chunk"));
    }
    if (g[0] + g[1] == 0) return BSMM_OK;
    hipLaunchKernelGGL(k_merge_block<T>, dim3(g[0] + g[1]), dim3(256), 0, s, a, b, (int)g[0]);
    return launch_check("merge_block");
}

template <class T>
int dense_multiply_t(const bsmm_matrix_s *A, const bsmm_matrix_s *B, bsmm_matrix_s *C,
                     double alpha, double beta, hipStream_t s) {
    const int64_t M = A->rows(), K = A->cols(), N = B->cols();
    if (M == 0 || N == 0 || C->nnzb == 0) return BSMM_OK;
    if (alpha == 0.0 || K == 0) return scale_blocks(C, nullptr, beta, s);
    // The FP64 copies add 32-bit offsets of up to seven columns of B with k
    // step 16 and three with 32 (past the latter's limit, K = 1.7e8, the two
    // panels would not fit into memory).
    const bool far = sizeof(T) == 8 && K > (int64_t(1) << 26) - 64;
    const int KB = options().dense_kb == 32 || far ? 32 : 16;
    const int64_t Mp = ceil_div(M, BM) * BM, Np = ceil_div(N, BN) * BN, Kp = ceil_div(K, KB) * KB;
    const int64_t tiles = (Mp / BM) * (Np / BN);
    if (tiles > kMaxGridBlocks || Mp * Kp > (int64_t(1) << 47) || Kp * Np > (int64_t(1) << 47)) {
        set_error(BSMM_ERANGE, "dense panels too large");
        return BSMM_ERANGE;
    }
    DevBuf ap, bp, cmap;
    BSMM_TRY(ap.reserve(sizeof(T) * Mp * Kp, s));
    BSMM_TRY(bp.reserve(sizeof(T) * Kp * Np, s));
    BSMM_TRY(merge_panels<T>(A, B, merge_args<T>(A, ap.as<T>(), Mp, Kp), merge_args<T>(B, bp.as<T>(), Kp, Np), s));
    const int32_t *d_cmap = nullptr;
    if (!C->full()) {
        const int64_t cells = (int64_t)C->nbr * C->nbc;
        if (cells > (int64_t(1) << 30)) {
            set_error(BSMM_ENOTSUP, "dense path on a sparse C with more than 2^30 block cells");
            return BSMM_ENOTSUP;
        }
        BSMM_TRY(cmap.reserve(sizeof(int32_t) * cells, s));
        hipLaunchKernelGGL(k_block_map, dim3(grid_rows(C->nbr)), dim3(256), 0, s, C->nbr, C->nbc,
                           C->d_row_ptr(), C->d_col_ind(), cmap.as<int32_t>());
        BSMM_TRY(launch_check("block_map"));
        d_cmap = cmap.as<int32_t>();
    }
    GemmArgs g{};
    g.Ap = ap.p;
    g.Bp = bp.p;
    g.lda = Mp;
    g.ldb = Kp;
    g.tiles_m = (int)(Mp / BM);
    g.tiles_n = (int)(Np / BN);
    g.ktiles = (int)(Kp / KB);
    g.M = M;
    g.N = N;
    g.alpha = alpha;
    g.beta = beta;
    g.C = C->d_raw();
    g.c_blk_off = C->d_blk_off();
    g.c_map = d_cmap;
    g.c_nbc = C->nbc;
    g.c_rbs = C->d_rbs();
    g.rmap = C->d_row_map();
    g.cmap = C->d_col_map();
    const int64_t slots = (int64_t)cu_count() * (KB == 32 ? 1 : 2);
    int64_t part_cap = int64_t(1) << 31;
    if (const ScratchArena *ar = scratch_arena()) {
        // Allocation-free: the partials take what the panels have left.
        part_cap = std::min<int64_t>(part_cap, (int64_t)(ar->cap - ar->used) - 512);
        part_cap = std::max<int64_t>(part_cap, 0);
    }
    const int64_t tile_bytes = (int64_t)sizeof(T) * BM * BN;
    const DenseParts d = dense_parts(tiles, g.ktiles, slots, tile_bytes, part_cap, sizeof(T) == 8 ? 4.0 : 2.0);
    const int64_t splits = d.splits, whole = d.whole;
    DevBuf part;
    if (splits > 1) {
        g.kt_per = (int)d.kt_per;
        g.splits = (int)splits;
        BSMM_TRY(part.reserve(tile_bytes * splits * (tiles - whole), s));
        g.part = part.p;
    }
    {
        KernelTimer kt(0, s);
        if (whole) {
            const dim3 grid((unsigned)whole);
            if (KB == 32) hipLaunchKernelGGL((k_dgemm_mfma<T, 32, 4, 1, false>), grid, dim3(256), 0, s, g);
            else hipLaunchKernelGGL((k_dgemm_mfma<T, 16, 2, 4, false>), grid, dim3(512), 0, s, g);
        }
        g.tile0 = (int)whole;
        g.ntiles = (int)(tiles - whole);
        if (splits > 1) {
            const dim3 grid((unsigned)(g.ntiles * splits));
            if (KB == 32) hipLaunchKernelGGL((k_dgemm_mfma<T, 32, 4, 1, true>), grid, dim3(256), 0, s, g);
            else hipLaunchKernelGGL((k_dgemm_mfma<T, 16, 2, 4, true>), grid, dim3(512), 0, s, g);
        }
    }
    BSMM_TRY(launch_check("dgemm_mfma"));
    if (splits == 1) return BSMM_OK;
    hipLaunchKernelGGL(k_splitk_reduce<T>, dim3(grid_of((int64_t)g.ntiles * 16, 1)), dim3(64), 0, s, g);
    return launch_check("splitk_reduce");
}

}  // namespace

int dense_multiply(const bsmm_matrix_s *A, const bsmm_matrix_s *B, bsmm_matrix_s *C,
                   double alpha, double beta, hipStream_t s) {
    if (C->dtype == BSMM_F32) return dense_multiply_t<float>(A, B, C, alpha, beta, s);
    return dense_multiply_t<double>(A, B, C, alpha, beta, s);
}

}  // namespace bsmm
