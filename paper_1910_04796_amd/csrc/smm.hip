// smm.hip -- batched small-block GEMM over the product stacks.
//
// Paper, Sec. II: the stacks of small block products are processed by
// dedicated small-matrix kernels (LIBCUSMM on NVIDIA GPUs, parametrised by
// the amount of work per thread block, the elements computed per thread and
// the tiling).  This is the gfx950 counterpart, written for wave64:
//
//  * a wavefront is split into G groups of L lanes; a group owns one run
//    (all products of one C block) at a time, so C stays in registers for
//    the whole run and is read-modified-written exactly once;
//  * every lane holds a TM x TN register tile of C (FP64 VALU FMAs: on
//    MI355X the FP64 vector rate equals the FP64 matrix rate, so small
//    blocks need no padding to MFMA shapes);
//  * each product's A block (m x k) and B block (k x n), contiguous in
//    memory, are staged into the group's LDS region with coalesced loads
//    and read back per k step, A as TM consecutive values, B as TN values
//    of one row;
//  * long k is split into chunks that fit the region; tile sets larger than
//    one wavefront are covered in passes;
//  * a variant runs each C block on matrix cores (register tile "16 x 16" in
//    the parameter space; the plain rule takes it for blocks of 25 elements
//    up to 64 x 64).
//
// The epilogue applies C = beta*C + alpha*acc (beta == 0 overwrites).
#include <algorithm>
#include <cmath>
#include <mutex>

#include "dev_util.h"
#include "internal.h"
#include "launch_rules.h"
#include "mfma_util.h"

namespace bsmm {

namespace {

template <class T, int TM, int TN>
__global__ __launch_bounds__(256) void k_smm_valu(SmmArgs p) {
    extern __shared__ double lds_raw[];
    T *lds = reinterpret_cast<T *>(lds_raw);
    const T *A = static_cast<const T *>(p.A);
    const T *B = static_cast<const T *>(p.B);
    T *C = static_cast<T *>(p.C);
    const T alpha = (T)p.alpha, beta = (T)p.beta;
    const int lane = lane_id();
    const int g = lane / p.L;
    const int gl = lane - g * p.L;
    const bool in_group = g < p.G;
    T *reg = lds + (size_t)(wave_id() * p.G + (in_group ? g : 0)) * p.region;
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / kWave);
    const int64_t wid = (int64_t)blockIdx.x * (blockDim.x / kWave) + wave_id();
    const int m = p.m, n = p.n;
    const int tiles = p.tiles_m * p.tiles_n;

    for (int64_t rb = p.run_begin + wid * p.G; rb < p.run_end; rb += waves * p.G) {
        const int64_t r = rb + g;
        const bool has = in_group && r < p.run_end;
        const int64_t q0 = has ? p.run_ptr[r] : 0;
        const int64_t q1 = has ? p.run_ptr[r + 1] : 0;
        const int64_t nq = wave_max(q1 - q0);
        for (int pass = 0; pass < p.passes; ++pass) {
            const int t = pass * p.L + gl;
            const bool tile_ok = has && t < tiles;
            const int it = tile_ok ? t % p.tiles_m : 0;
            const int jt = tile_ok ? t / p.tiles_m : 0;
            const int i0 = it * TM, j0 = jt * TN;
            T acc[TM][TN];
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int b = 0; b < TN; ++b) acc[a][b] = T(0);

            for (int64_t qi = 0; qi < nq; ++qi) {
                const bool act = has && qi < q1 - q0;
                ulonglong2 pr = make_ulonglong2(0ull, 0ull);
                if (act) pr = p.prods[q0 + qi];
                const int64_t a_off = (int64_t)(pr.x & ((1ull << 48) - 1));
                const int k = act ? (int)(pr.x >> 48) : 0;
                const int64_t b_off = (int64_t)pr.y;
                const int kmax = wave_max(k);
                for (int kc0 = 0; kc0 < kmax; kc0 += p.kc_max) {
                    const int kc = act ? std::min(p.kc_max, k - kc0) : 0;
                    // stage A(:, kc0:kc0+kc) (contiguous) and B(kc0:kc0+kc, :)
                    if (kc > 0) {
                        const T *ga = A + a_off + (int64_t)m * kc0;
                        const int na = m * kc;
                        for (int e = gl; e < na; e += p.L) reg[e] = ga[e];
                        T *rbuf = reg + na;
                        const T *gb = B + b_off + kc0;
                        if (kc == k) {
                            const int nb = k * n;
                            for (int e = gl; e < nb; e += p.L) rbuf[e] = gb[e];
                        } else {
                            const int nb = kc * n;
                            const float rcp = 1.0f / (float)kc;
                            for (int e = gl; e < nb; e += p.L) {
                                int kk;
                                const int j = divmod_small(e, kc, rcp, &kk);
                                rbuf[e] = gb[(int64_t)j * k + kk];
                            }
                        }
                    }
                    wave_lds_sync();
                    if (tile_ok && kc > 0) {
                        const T *As = reg + i0;
                        const T *Bs = reg + m * kc + (int64_t)j0 * kc;
                        for (int kk = 0; kk < kc; ++kk) {
                            T av[TM], bv[TN];
#pragma unroll
                            for (int a = 0; a < TM; ++a) av[a] = As[kk * m + a];
#pragma unroll
                            for (int b = 0; b < TN; ++b) bv[b] = Bs[b * kc + kk];
#pragma unroll
                            for (int a = 0; a < TM; ++a)
#pragma unroll
                                for (int b = 0; b < TN; ++b) acc[a][b] = fma(av[a], bv[b], acc[a][b]);
                        }
                    }
                    wave_lds_sync();
                }
            }
            if (tile_ok) {
                T *c = C + p.run_coff[r];
#pragma unroll
                for (int b = 0; b < TN; ++b) {
                    const int j = j0 + b;
                    if (j >= n) break;
#pragma unroll
                    for (int a = 0; a < TM; ++a) {
                        const int i = i0 + a;
                        if (i < m) {
                            T *dst = c + (int64_t)j * m + i;
                            const T prod = alpha * acc[a][b];
                            *dst = (beta == T(0)) ? prod : fma(beta, *dst, prod);
                        }
                    }
                }
            }
        }
    }
}

// MFMA variant (parameter set tm = tn = 16): one wave owns one run at a time
// and keeps the C block as MT x NT tiles of 16 x 16 x 4 MFMA accumulators
// (m <= 16 MT, n <= 16 NT): v_mfma_f64_16x16x4 for FP64, v_mfma_f32_16x16x4 for
// FP32.  Operands come straight from the contiguous A and B blocks; lanes past a
// block's rows or columns read what follows in the block, or zero past its end
// (they only reach results that are not stored), and k past the block is zero
// on both sides.
// Both instructions take lane l's operands at row (or column) l % 16 and
// k = l / 16 of the step.

// Where an operand's values lie.
enum OperandLayout {
    kAlongTile,  // consecutive values run along the tile's rows (columns):
                 // A in place (column-major), B from row-major copies
    kAlongK      // consecutive values run along k: B in place, A from
                 // row-major copies
};

// Row (column) of a block that lane index r = 0..15 of tile t stands for.
// Two neighbouring tiles interleave their 32 rows, so that one load of two
// consecutive values serves both.
template <int NTILE> __device__ __forceinline__ int tile_row(int t, int r) {
    return (t | 1) < NTILE ? 32 * (t >> 1) + 2 * r + (t & 1) : 16 * t + r;
}

// One operand's loads, a chunk of 8 values of k at a time: lane group lk
// supplies k = 2 lk + s of the chunk to MFMA step s.  The chunk is a buffer
// from its first value to the end of its block, so what lies past the block
// reads as zero (rows and columns past the block reach results that are not
// stored) and the lanes' offsets stay the same for all products of a run.
template <class T, int NTILE, OperandLayout LAY> struct Operand {
    static constexpr uint32_t kSize = sizeof(T);
    const char *data;
    const char *at;   // the chunk
    uint32_t bytes;   // from there to the end of the block; 0: past the run
    uint32_t step;    // bytes of a chunk
    int ext;          // rows (columns) of the block
    // Byte offsets of the lane: kAlongTile: column s of the first two tiles
    // (of the only one); kAlongK: row of tile t.
    uint32_t off[LAY == kAlongTile ? 2 : NTILE];

    __device__ __forceinline__ void init(const void *d, int ext_, int lr, int lk) {
        data = static_cast<const char *>(d);
        ext = ext_;
        step = (LAY == kAlongTile ? 8 * (uint32_t)ext : 8u) * kSize;
        if (LAY == kAlongTile) {
            off[0] = (2 * lk * (uint32_t)ext + (NTILE > 1 ? 2 * lr : lr)) * kSize;
            off[1] = off[0] + (uint32_t)ext * kSize;
        }
    }
    __device__ __forceinline__ void block(uint64_t elem, int k, int lr, int lk) {
        at = data + elem * kSize;
        bytes = (uint32_t)ext * (uint32_t)k * kSize;
        if (LAY == kAlongK) {
#pragma unroll
            for (int t = 0; t < NTILE; ++t)
                off[t] = ((uint32_t)tile_row<NTILE>(t, lr) * (uint32_t)k + 2 * lk) * kSize;
        }
    }
    __device__ __forceinline__ void next_chunk() {
        at += step;
        bytes -= step;
    }
    // left: values of k from the chunk's first one.
    __device__ __forceinline__ void load(int left, int lr, int lk, T (&f)[2][NTILE]) const {
        const BufferRsrc r = buffer_at(at, bytes);
        if (LAY == kAlongTile) {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
#pragma unroll
                for (int t = 0; t + 1 < NTILE; t += 2) Mfma<T>::load2(r, off[s] + 16 * t * kSize, f[s][t], f[s][t + 1]);
                if (NTILE == 1) f[s][0] = Mfma<T>::load(r, off[s]);
                else if (NTILE & 1) f[s][NTILE - 1] = Mfma<T>::load(r, off[s] + (16 * (NTILE - 1) - lr) * kSize);
            }
        } else {
            // Past the row's last k lies the next row: such lanes read past
            // the buffer, and half a pair is cleared by mfma_chunk.
#pragma unroll
            for (int t = 0; t < NTILE; ++t) Mfma<T>::load2(r, 2 * lk < left ? off[t] : kPastBuffer, f[0][t], f[1][t]);
        }
    }
};

// One chunk of 8 values of k of a product: its operands, and how many values
// from the chunk's first one lie inside the block (0: past the run).
template <class T, int MT, int NT> struct Chunk {
    T a[2][MT], b[2][NT];
    int left;
};

template <class T, int MT, int NT, OperandLayout LA, OperandLayout LB>
__device__ __forceinline__ void mfma_chunk(Chunk<T, MT, NT> &c, int lk, typename Mfma<T>::acc_t (&acc)[MT][NT]) {
    if (LA == kAlongK) {
#pragma unroll
        for (int i = 0; i < MT; ++i) c.a[1][i] = 2 * lk + 1 < c.left ? c.a[1][i] : T(0);
    }
    if (LB == kAlongK) {
#pragma unroll
        for (int j = 0; j < NT; ++j) c.b[1][j] = 2 * lk + 1 < c.left ? c.b[1][j] : T(0);
    }
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] = Mfma<T>::step(c.a[s][i], c.b[s][j], acc[i][j]);
}

// Products [q0, q1) of one run into the MT x NT accumulator tiles of an
// m x n C block (q0, q1, m and n the same on every lane: descriptors, depths
// and block addresses stay on the scalar unit).  The products' chunks follow
// one another without a break: the operands of the next chunk (of the next
// product where one ends) are on their way while a chunk is multiplied, the
// descriptor of the product after it one product earlier.
//
// Two chunk variables in turn and no vector instruction besides loads and
// MFMAs: on FP64, whose MFMAs and vector instructions exclude each other, the
// copies between chunk variables, offsets and tail masks took a quarter of the
// MFMAs' time.  23-blocks at 20 % 1.75 -> 1.50 ms, {5,13,23} at 25 % 296 -> 241
// us, uniform 64-blocks at 20 % 1.68 -> 1.30 ms (FP32: 0.69 -> 0.57).  More
// chunks ahead gain nothing (2, 3, 5: the same within 2 %).
template <class T, int MT, int NT, OperandLayout LA, OperandLayout LB>
__device__ __forceinline__ void mfma_products(const SmmArgs &p, int m, int n, int64_t q0, int64_t q1,
                                              typename Mfma<T>::acc_t (&acc)[MT][NT]) {
    typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
    const u64x2 *prods = reinterpret_cast<const u64x2 *>(p.prods);
    const int lane = lane_id();
    const int lr = lane & 15, lk = lane >> 4;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = Mfma<T>::zero();
    if (q0 >= q1) return;
    Operand<T, MT, LA> oa;
    Operand<T, NT, LB> ob;
    oa.init(LA == kAlongK ? p.A_t : p.A, m, lr, lk);
    ob.init(LB == kAlongTile ? p.B_t : p.B, n, lr, lk);
    u64x2 nxt = scalar_at(prods, q0);
    int64_t q = q0;
    int left = 0;
    auto advance = [&] {  // to product q
        left = (int)(nxt.x >> 48);
        oa.block(nxt.x & ((1ull << 48) - 1), left, lr, lk);
        ob.block(nxt.y, left, lr, lk);
        if (q >= q1) {
            left = 0;
            oa.bytes = ob.bytes = 0;
        }
        ++q;
        nxt = scalar_at(prods, min(q, q1 - 1));
    };
    auto load = [&](Chunk<T, MT, NT> &c) {
        oa.load(left, lr, lk, c.a);
        ob.load(left, lr, lk, c.b);
        c.left = left;
        left -= 8;
        oa.next_chunk();
        ob.next_chunk();
        if (left <= 0) advance();
    };
    Chunk<T, MT, NT> c0, c1;
    advance();
    load(c0);
    asm volatile("" : "+s"(c0.left));  // (a known first chunk would get a copy of the loop)
    do {
        load(c1);
        mfma_chunk<T, MT, NT, LA, LB>(c0, lk, acc);
        load(c0);
        // (A branch around so many accumulators would copy them; zeros add nothing.)
        if (MT * NT > 8 || c1.left > 0) mfma_chunk<T, MT, NT, LA, LB>(c1, lk, acc);
    } while (c0.left > 0);
}

// C block (column-major, ld = m) <- beta C + alpha acc, or the unscaled
// accumulators into a partial block when alpha is not applied here.  With
// SUMSQ, returns on every lane the squared Frobenius norm of the stored
// block (summed in FP64: each lane's elements in order, then across the
// wave in a fixed order).  The block is a buffer: columns past it lie past
// the buffer's end, and so do the offsets of rows past it, so all elements
// are loaded (a tile column's together; one after another, each behind the
// store before it, they made up a third of a short accumulating launch: 72
// runs 10.5 -> 9 us) and stored without branches.
template <class T, int MT, int NT, bool SUMSQ>
__device__ __forceinline__ double mfma_store(T *c, int m, int n,
                                             const typename Mfma<T>::acc_t (&acc)[MT][NT],
                                             bool partial, T alpha, T beta) {
    constexpr uint32_t kSize = sizeof(T);
    const int lane = lane_id();
    const int lr = lane & 15, lk = lane >> 4;
    const BufferRsrc r = buffer_at(c, (uint32_t)m * (uint32_t)n * kSize);
    uint32_t ro[MT][4];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = tile_row<MT>(i, Mfma<T>::row(e, lk));
            ro[i][e] = row < m ? (uint32_t)row * kSize : kPastBuffer;
        }
    double ss = 0.0;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int col = tile_row<NT>(j, lr);
        const uint32_t co = (uint32_t)col * (uint32_t)m * kSize;
        T v[MT][4];
        if (partial) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[i][e] = acc[i][j][e];
        } else if (beta == T(0)) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[i][e] = alpha * acc[i][j][e];
        } else {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[i][e] = Mfma<T>::load(r, co + ro[i][e]);
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const T prod = alpha * acc[i][j][e];
                    v[i][e] = fma(beta, v[i][e], prod);
                }
        }
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                Mfma<T>::store(r, co + ro[i][e], v[i][e]);
                if (SUMSQ) {
                    const double x = ro[i][e] != kPastBuffer && col < n ? (double)v[i][e] : 0.0;
                    ss = fma(x, x, ss);
                }
            }
    }
    return SUMSQ ? wave_sum(ss) : 0.0;
}

template <class T, int MT, int NT>
__global__ __launch_bounds__(256) void k_smm_mfma(SmmArgs p) {
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x / kWave);
    const int64_t wid = (int64_t)blockIdx.x * (blockDim.x / kWave) + uniform(wave_id());
    const int m = p.m, n = p.n;
    const int S = p.split > 1 ? p.split : 1;
    const int64_t items = (p.run_end - p.run_begin) * S;
    for (int64_t it = wid; it < items; it += waves) {
        // Item = (run, segment): segment sg of S takes products
        // [len sg / S, len (sg + 1) / S) of the run.
        const int64_t r = p.run_begin + it / S;
        const int sg = (int)(it % S);
        const int64_t rq0 = scalar_at(p.run_ptr, r), len = scalar_at(p.run_ptr, r + 1) - rq0;
        const int64_t q0 = rq0 + len * sg / S, q1 = rq0 + len * (sg + 1) / S;
        T *c = S > 1 ? static_cast<T *>(p.part) + it * (int64_t)m * n : static_cast<T *>(p.C) + scalar_at(p.run_coff, r);
        typename Mfma<T>::acc_t acc[MT][NT];
        mfma_products<T, MT, NT, kAlongTile, kAlongK>(p, m, n, q0, q1, acc);
        mfma_store<T, MT, NT, false>(c, m, n, acc, S > 1, (T)p.alpha, (T)p.beta);
    }
}

// Runs of every class with C blocks up to 32 x 32 in one launch, in the
// order of a schedule that groups the runs by 2-D tiles of C blocks: the
// waves in flight then work on nearby block rows and block columns and
// share their A and B blocks in the caches.  Schedule entry: run << 16 |
// m << 8 | n.  Static mode: a wave takes every so many-th entry of its XCD;
// dynamic mode: waves take the next one from the XCD's counter.
template <class T, int MT, int NT, OperandLayout LA, OperandLayout LB>
__device__ __forceinline__ void sched_run(const SmmArgs &p, int64_t r, int m, int n) {
    typename Mfma<T>::acc_t acc[MT][NT];
    T *c = static_cast<T *>(p.C) + scalar_at(p.run_coff, r);
    mfma_products<T, MT, NT, LA, LB>(p, m, n, scalar_at(p.run_ptr, r), scalar_at(p.run_ptr, r + 1), acc);
    // One store path: the norm is summed whether or not the filter wants it.
    const double ss = mfma_store<T, MT, NT, true>(c, m, n, acc, false, (T)p.alpha, (T)p.beta);
    if (p.norm2 && lane_id() == 0) p.norm2[p.run_cblk[r]] = ss;
}

// Segments of 2^sched_seg_bits schedule entries go to the XCDs in turn
// (workgroup g runs on XCD g % 8) and each XCD's waves take theirs in order, so
// that the runs of a tile meet in one L2: banded 30 % 639 -> 611 ms, banded 10 %
// 67.8 -> 64.9 against one order for all XCDs, with tiles of 32 x 32; segments
// of 32 to 1,024 entries differ by 2 %.  The next entry is taken when the last
// one is done, not ahead of it: runs taken one after the other also start one
// after the other, and share operands while they are at the same k (taken
// ahead: 30 % 563 -> 608 ms).
//
// One counter per XCD.  Updates of one address follow one another about 15 ns
// apart, so a single counter bounded launches of many short runs
// ({5,13,23}-blocks at 25 %, 48,000 runs: 505 us; four or eight counters 300 us).
// An XCD that is done does not help the others: reading eight counters in
// every wave costs 70 us at the end, more than the XCDs differ.  So a short
// schedule has shorter segments, eight or more for each XCD (schedule_segment_bits).
// Fewest runs for which the MFMA classes go through the scheduled launch, and
// the most classes that keep a launch each below that in a plan: a launch takes
// 6 us, a graph of 9 or 16 of them 95 to 125 us to start, a scheduled replay
// 31 us (9 classes, plan, as a graph and so: 12 x 12 blocks, 8 products a run 96
// and 31 us, 4 x 4 blocks 95 and 30; 16 classes of 400 x 400 x 400 as a graph 115).
constexpr int64_t kSchedMinRuns = 4096;
constexpr int kSchedFewClasses = 6;

template <class T, OperandLayout LA, OperandLayout LB>
__device__ __forceinline__ void sched_loop(const SmmArgs &p) {
    const int wpw = blockDim.x / kWave;
    // A wave takes `chunk` consecutive entries at a time (short runs: fewer
    // counter updates), the first ones by its number in its XCD.
    const int chunk = max(p.sched_chunk, 1), seg = p.sched_seg_bits;
    const int x = blockIdx.x % kXcds;
    const int64_t waves = (int64_t)((gridDim.x - x + kXcds - 1) / kXcds) * wpw;
    int64_t pos = ((int64_t)(blockIdx.x / kXcds) * wpw + uniform(wave_id())) * chunk;
    while (true) {
        const int64_t it = (((pos >> seg) * kXcds + x) << seg) + (pos & ((1 << seg) - 1));
        if (it >= p.n_sched) break;  // pos only grows, and `it` with it
        const int64_t end = min(it + chunk, p.n_sched);
        for (int64_t i = it; i < end; ++i) {
            const unsigned long long e = scalar_at(p.sched, i);
            const int64_t r = (int64_t)(e >> 16);
            const int m = (int)((e >> 8) & 255), n = (int)(e & 255);
            if (m > 16) {
                if (n > 16) sched_run<T, 2, 2, LA, LB>(p, r, m, n);
                else sched_run<T, 2, 1, LA, LB>(p, r, m, n);
            } else {
                if (n > 16) sched_run<T, 1, 2, LA, LB>(p, r, m, n);
                else sched_run<T, 1, 1, LA, LB>(p, r, m, n);
            }
        }
        if (p.sched_mode == 0) {
            pos += waves * chunk;
        } else {
            unsigned long long t = 0;
            if (lane_id() == 0) t = atomicAdd(&p.next[x * kSchedCounterStride], 1ull);
            pos = (waves + uniform((int64_t)t)) * chunk;
        }
    }
}

template <class T, OperandLayout LA, OperandLayout LB>
__global__ __launch_bounds__(256, 4) void k_smm_mfma_sched(SmmArgs p) {
    sched_loop<T, LA, LB>(p);
}

// Row-major copies of a matrix's blocks at the blocks' own offsets: a wave
// takes kTurnBlocks consecutive blocks of a block row (their lookups side by
// side, one per lane) and turns each through LDS (blocks of up to kTurnElems
// elements, what a wave's registers read ahead, whose columns fit with an odd
// stride), so that reads and writes are both contiguous; the next block's
// elements are read while this one is written.  Bound by HBM
// (16 bytes per FP64 element); 1.44 GB of 5-to-32-sided blocks 1,146 us with
// one lookup per block and no read ahead, 642 us so (4.5 TB/s).
constexpr int kTurnElems = 1024;
constexpr int kTurnBlocks = 8;
template <class T>
__global__ __launch_bounds__(256) void k_transpose_blocks(int32_t nbr, const int64_t *rp, const int32_t *ci,
                                                          const int32_t *rbs, const int32_t *cbs,
                                                          const int64_t *blk_off, const T *src, T *dst) {
    constexpr int kRegs = kTurnElems / kWave;
    __shared__ T lds[4][kTurnElems + 64];
    T *buf = lds[wave_id()];
    const int lane = lane_id();
    const int64_t step = 4 * (int64_t)gridDim.y * kTurnBlocks;
    for (int32_t r = blockIdx.x; r < nbr; r += gridDim.x) {
        const int m = rbs[r];
        const int ld = m | 1;  // odd: the column reads spread over the banks
        const float rm = 1.0f / (float)m;
        const int64_t p1 = rp[r + 1];
        for (int64_t p0 = rp[r] + ((int64_t)blockIdx.y * 4 + wave_id()) * kTurnBlocks; p0 < p1; p0 += step) {
            const int nb = (int)min((int64_t)kTurnBlocks, p1 - p0);
            int64_t my_off = 0;
            int my_k = 0;
            if (lane < nb) {
                my_off = blk_off[p0 + lane];
                my_k = cbs[ci[p0 + lane]];
            }
            T v[kRegs];
            auto turned = [&](int k) { return (int64_t)m * k <= kTurnElems && (int64_t)ld * k <= kTurnElems + 64; };
            auto fetch = [&](int b) {
                const T *sb = src + __shfl(my_off, b, kWave);
                const int k = __shfl(my_k, b, kWave);
                if (!turned(k)) return;
                const int len = m * k;
#pragma unroll
                for (int u = 0; u < kRegs; ++u)
                    if (u * kWave < len && u * kWave + lane < len) v[u] = sb[u * kWave + lane];
            };
            fetch(0);
            for (int b = 0; b < nb; ++b) {
                const int k = __shfl(my_k, b, kWave);
                const T *sb = src + __shfl(my_off, b, kWave);
                T *db = dst + __shfl(my_off, b, kWave);
                const int64_t len = (int64_t)m * k;
                if (turned(k)) {
#pragma unroll
                    for (int u = 0; u < kRegs; ++u) {
                        const int e = u * kWave + lane;
                        if (u * kWave < len && e < len) {
                            int i;
                            const int j = divmod_small(e, m, rm, &i);
                            buf[j * ld + i] = v[u];
                        }
                    }
                    wave_lds_sync();
                    if (b + 1 < nb) fetch(b + 1);
                    const float rk = 1.0f / (float)k;
                    for (int e = lane; e < (int)len; e += kWave) {
                        int j;
                        const int i = divmod_small(e, k, rk, &j);
                        db[e] = buf[j * ld + i];
                    }
                    wave_lds_sync();
                } else {
                    if (b + 1 < nb) fetch(b + 1);
                    for (int64_t e = lane; e < len; e += kWave) {
                        const int64_t i = e / k, j = e - i * k;
                        db[e] = sb[j * m + i];
                    }
                }
            }
        }
    }
}

__global__ void k_zero_counters(unsigned long long *p) { p[threadIdx.x * kSchedCounterStride] = 0ull; }

// Epilogue of split runs: C block of run r = beta C + alpha * (sum of its
// segments' partial blocks in segment order); one thread per element.
template <class T>
__global__ __launch_bounds__(256) void k_smm_split_reduce(SmmArgs p) {
    const int64_t mn = (int64_t)p.m * p.n;
    const int64_t total = (p.run_end - p.run_begin) * mn;
    const T *part = static_cast<const T *>(p.part);
    T *C = static_cast<T *>(p.C);
    const T alpha = (T)p.alpha, beta = (T)p.beta;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t rl = t / mn, e = t - rl * mn;
        const T *w = part + rl * p.split * mn + e;
        T v = w[0];
        for (int sg = 1; sg < p.split; ++sg) v += w[sg * mn];
        T *dst = C + p.run_coff[p.run_begin + rl] + e;
        const T prod = alpha * v;
        *dst = (beta == T(0)) ? prod : fma(beta, *dst, prod);
    }
}

using SmmKernel = void (*)(SmmArgs);

template <class T, int MT> SmmKernel pick_mfma_nt(int nt) {
    switch (nt) {
    case 1: return k_smm_mfma<T, MT, 1>;
    case 2: return k_smm_mfma<T, MT, 2>;
    case 3: return k_smm_mfma<T, MT, 3>;
    case 4: return k_smm_mfma<T, MT, 4>;
    default: return nullptr;
    }
}

// MFMA kernels for C blocks up to 64 x 64 (MT, NT in 1..4).
template <class T> SmmKernel mfma_kernel_for(int mt, int nt) {
    switch (mt) {
    case 1: return pick_mfma_nt<T, 1>(nt);
    case 2: return pick_mfma_nt<T, 2>(nt);
    case 3: return pick_mfma_nt<T, 3>(nt);
    case 4: return pick_mfma_nt<T, 4>(nt);
    default: return nullptr;
    }
}

// Register-tile shapes with a compiled kernel: TM, TN in {1,2,3,4,5,6,8}.
template <class T, int TM> SmmKernel pick_tn(int tn) {
    switch (tn) {
    case 1: return k_smm_valu<T, TM, 1>;
    case 2: return k_smm_valu<T, TM, 2>;
    case 3: return k_smm_valu<T, TM, 3>;
    case 4: return k_smm_valu<T, TM, 4>;
    case 5: return k_smm_valu<T, TM, 5>;
    case 6: return k_smm_valu<T, TM, 6>;
    case 8: return k_smm_valu<T, TM, 8>;
    default: return nullptr;
    }
}

template <class T> SmmKernel kernel_for(int tm, int tn) {
    switch (tm) {
    case 1: return pick_tn<T, 1>(tn);
    case 2: return pick_tn<T, 2>(tn);
    case 3: return pick_tn<T, 3>(tn);
    case 4: return pick_tn<T, 4>(tn);
    case 5: return pick_tn<T, 5>(tn);
    case 6: return pick_tn<T, 6>(tn);
    case 8: return pick_tn<T, 8>(tn);
    default: return nullptr;
    }
}

thread_local double *t_norm_sink = nullptr;

// The scheduled kernel reading A (or B) from row-major copies.
template <class T> SmmKernel sched_kernel_t(bool a_rows, bool b_rows) {
    if (a_rows) return k_smm_mfma_sched<T, kAlongK, kAlongK>;
    return b_rows ? k_smm_mfma_sched<T, kAlongTile, kAlongTile> : k_smm_mfma_sched<T, kAlongTile, kAlongK>;
}
SmmKernel sched_kernel(int dtype, bool a_rows, bool b_rows) {
    return dtype == BSMM_F32 ? sched_kernel_t<float>(a_rows, b_rows) : sched_kernel_t<double>(a_rows, b_rows);
}

bool is_sched_kernel(const void *fn) {
    for (int dtype : {BSMM_F64, BSMM_F32})
        for (int rows = 0; rows < 3; ++rows)
            if (fn == (const void *)sched_kernel(dtype, rows == 1, rows == 2)) return true;
    return false;
}

// Fewest products per block of B for which the scheduled launch reads B
// from row-major copies.  A fragment of B in place touches one 64-byte
// piece of 16 columns, from a copy one 128-byte piece of 4 rows of k: a
// third fewer cache lines, which the launch feels once each B block is read
// many times, while the copy costs one read and one write of B (and a launch).
// Measured (whole multiply, in place -> from copies): FP64 banded 30 % 664 ->
// 563 ms, 10 % 82.6 -> 70.1 ms, 5 % 30.4 -> 27.7 ms; 23-blocks at 20 % (70
// products per B block) 1.95 -> 1.90 ms, at 10 % (35) 0.90 -> 0.85 ms;
// {5,13,23}-blocks, N = 3000, at 25 % (55) 398 -> 413 us, at 10 % (22) 218 -> 237
// us; banded 2 % and 1 % the same.  FP32, which the masks of B in place cost
// more: banded 10 % 50.7 -> 40.5 ms, N = 24,000 9.89 -> 8.87 ms, 23-blocks at 20
// % 1.29 -> 1.16 ms, N = 3000 at 25 % 311 -> 314 us.
constexpr int64_t kCopyBMinUses = 48;

constexpr int kLdsBudget = 64 * 1024;  // bytes of LDS per workgroup

}  // namespace

void set_norm_sink(double *norm2) { t_norm_sink = norm2; }
double *norm_sink() { return t_norm_sink; }


// Plain parameter rule: the smallest square register tile T (1..8) for
// which ceil(m/T) * ceil(n/T) <= 64 lanes (blocks above 64 use T = 8 and
// passes), the largest k chunk that fits, and as many waves per workgroup
// (up to 4) as 64 KB of LDS allow.
SmmParams plain_params(int m, int n) {
    int t = 8;
    for (int c = 1; c < 8; ++c)
        if (c != 7 && ceil_div(m, c) * ceil_div(n, c) <= kWave) {
            t = c;
            break;
        }
    return SmmParams{t, t, 0, 0};
}

// The plain path's launch: the MFMA kernel for blocks of up to 64 x 64 whose
// tiles are worth a wave (at least 25 elements and 200 multiply-adds per
// product), the register-tile rule else.  MFMA over register tiles, 15,000
// and more runs of 1 / 8 / 32 products: 13 x 13 x 5 0.68 / 0.55 / 0.50,
// 6 x 6 x 6 0.80 / 0.84 / 0.79, 5 x 5 x 23 1.03 / 0.73 / 0.70, but 5 x 5 x 5
// 1.52 / 1.22 / 1.24, 4 x 4 x 32 1.38 / 1.07 / 1.09, 4 x 4 x 4 2.9 / 2.0 / 2.3.
static SmmParams plain_launch(int m, int n, int k) {
    if (m <= 64 && n <= 64 && m * n >= 25 && (int64_t)m * n * k >= 200)
        return SmmParams{kMfmaTile, kMfmaTile, 0, 4};
    return plain_params(m, n);
}

int plan_smm(const SmmParams &prm, int m, int n, int kmax, int dtype, SmmLaunch *out) {
    const bool f32 = dtype == BSMM_F32;
    const size_t esize = f32 ? sizeof(float) : sizeof(double);
    out->dtype = dtype;
    if (prm.tm == kMfmaTile && prm.tn == kMfmaTile) {
        const int mt = (int)ceil_div(m, 16), nt = (int)ceil_div(n, 16);
        SmmKernel fn = f32 ? mfma_kernel_for<float>(mt, nt) : mfma_kernel_for<double>(mt, nt);
        if (!fn) {
            set_error(BSMM_ENOTSUP, "MFMA small-block kernel covers blocks up to 64 x 64, not %dx%d", m, n);
            return BSMM_ENOTSUP;
        }
        SmmArgs a{};
        a.m = m;
        a.n = n;
        a.tiles_m = mt;
        a.tiles_n = nt;
        a.L = kWave;
        a.G = 1;
        a.passes = 1;
        out->fn = (void *)fn;
        out->args = a;
        out->waves = prm.waves > 0 ? std::min(prm.waves, 4) : 4;
        out->lds = 0;
        return BSMM_OK;
    }
    const int TM = prm.tm, TN = prm.tn;
    SmmKernel fn = f32 ? kernel_for<float>(TM, TN) : kernel_for<double>(TM, TN);
    if (!fn) {
        set_error(BSMM_EINVAL, "no small-block kernel for register tile %dx%d", TM, TN);
        return BSMM_EINVAL;
    }
    SmmArgs a{};
    a.m = m;
    a.n = n;
    a.tiles_m = (int)ceil_div(m, TM);
    a.tiles_n = (int)ceil_div(n, TN);
    const int tiles = a.tiles_m * a.tiles_n;
    a.L = std::min(tiles, kWave);
    a.G = kWave / a.L;
    a.passes = (int)ceil_div(tiles, a.L);
    // LDS region per group: A chunk (m x kc) + B chunk (n_pad x kc) + slack
    // for the tail reads of the last register tile.
    const int n_pad = a.tiles_n * TN;
    const int waves_req = prm.waves > 0 ? std::min(prm.waves, 4) : 1;
    const int max_group_elems = (int)(kLdsBudget / esize / a.G / waves_req);
    int kc = (max_group_elems - TM - 3) / (m + n_pad);
    kc = std::min(kc, std::max(1, kmax));
    if (prm.kc > 0) kc = std::min(kc, prm.kc);
    if (kc < 1) {
        set_error(BSMM_ENOTSUP, "block shape %dx%d with tile %dx%d does not fit in LDS", m, n, TM, TN);
        return BSMM_ENOTSUP;
    }
    a.kc_max = kc;
    a.region = (m + n_pad) * kc + TM + 2;
    a.region = (a.region + 1) & ~1;
    const size_t wave_bytes = esize * (size_t)a.G * a.region;
    int waves = prm.waves > 0 ? waves_req
                              : (int)std::max<int64_t>(1, std::min<int64_t>(4, kLdsBudget / wave_bytes));
    if (wave_bytes * waves > (size_t)kLdsBudget) {
        set_error(BSMM_ENOTSUP, "small-block launch needs more than 64 KB of LDS");
        return BSMM_ENOTSUP;
    }
    out->fn = (void *)fn;
    out->args = a;
    out->waves = waves;
    out->lds = wave_bytes * waves;
    return BSMM_OK;
}

static unsigned split_reduce_grid(const SmmArgs &a) {
    return grid_of((a.run_end - a.run_begin) * (int64_t)a.m * a.n, 256, 8192);
}

unsigned smm_grid(const SmmLaunch &L, int64_t nruns) {
    const int64_t waves_needed = ceil_div(nruns * std::max(L.args.split, 1), L.args.G);
    // At most 32 waves per CU (256 CUs) in the grid, whatever the waves per
    // workgroup; the kernels stride over the remaining runs.
    int64_t wg_cap = 256 * 32 / std::max(L.waves, 1);
    if (is_sched_kernel(L.fn)) {
        // Only resident workgroups: later ones would begin with the runs
        // that their numbers stand for when the others are far ahead.
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, L.fn, 64 * L.waves, 0) != hipSuccess || per_cu < 1) {
            (void)hipGetLastError();
            per_cu = 5;
        }
        if (L.args.sched_per_cu > 0) per_cu = std::min(per_cu, L.args.sched_per_cu);
        wg_cap = (int64_t)cu_count() * per_cu;
        return std::max<unsigned>(grid_of(waves_needed, L.waves, wg_cap), kXcds);  // every part has its waves
    }
    return grid_of(waves_needed, L.waves, wg_cap);
}

int launch_smm(SmmLaunch L, const void *A, const void *B, void *C, const int64_t *run_coff,
               const int64_t *run_ptr, const ulonglong2 *prods, int64_t rb, int64_t re,
               double alpha, double beta, hipStream_t s) {
    SmmArgs a = L.args;
    a.A = A;
    a.B = B;
    a.C = C;
    a.run_coff = run_coff;
    a.run_ptr = run_ptr;
    a.prods = prods;
    a.run_begin = rb;
    a.run_end = re;
    a.alpha = alpha;
    a.beta = beta;
    if (L.jit_fn)
        return launch_jit_smm(L.jit_fn, smm_grid(L, re - rb), L.waves, A, B, C, run_coff, run_ptr, prods,
                              rb, re, alpha, beta, s);
    if (is_sched_kernel(L.fn) && a.sched_mode == 1) {
        hipLaunchKernelGGL(k_zero_counters, dim3(1), dim3(kXcds), 0, s, a.next);
        BSMM_TRY(launch_check("zero_counters"));
    }
    {
        KernelTimer kt(1, s);
        hipLaunchKernelGGL((SmmKernel)L.fn, dim3(smm_grid(L, re - rb)), dim3(64 * L.waves), L.lds, s,
                           a);
    }
    BSMM_TRY(launch_check("smm_valu"));
    if (a.split <= 1) return BSMM_OK;
    if (L.dtype == BSMM_F32)
        hipLaunchKernelGGL(k_smm_split_reduce<float>, dim3(split_reduce_grid(a)), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL(k_smm_split_reduce<double>, dim3(split_reduce_grid(a)), dim3(256), 0, s, a);
    return launch_check("smm_split_reduce");
}

// Average products per run of every class (tuned path: the run length is
// part of the parameter lookup), from the per-class run and product counts
// the stack builder read back.
static void class_run_lengths(const Stacks &st, std::vector<int> *out) {
    out->assign(st.n_classes, 1);
    if ((int)st.class_prod_begin.size() != st.n_classes + 1) return;
    for (int cl = 0; cl < st.n_classes; ++cl) {
        const int64_t runs = st.class_begin[cl + 1] - st.class_begin[cl];
        const int64_t prods = st.class_prod_begin[cl + 1] - st.class_prod_begin[cl];
        if (runs > 0) (*out)[cl] = (int)std::max<int64_t>(1, (prods + runs / 2) / runs);
    }
}

// The k under which tuned parameters are looked up: a run mixes the k of
// A's block columns, and a product's work grows with k, so the key is the
// block-column size k carrying the most work (count of columns of size k,
// times k; ties: the smaller k).
static int representative_k(const bsmm_matrix_s *A) {
    std::vector<int32_t> v = A->cbs;
    if (v.empty()) return 1;
    std::sort(v.begin(), v.end());
    int best = v[0];
    int64_t bestw = 0;
    for (size_t i = 0; i < v.size();) {
        size_t j = i;
        while (j < v.size() && v[j] == v[i]) ++j;
        const int64_t w = (int64_t)(j - i) * v[i];
        if (w > bestw) {
            bestw = w;
            best = v[i];
        }
        i = j;
    }
    return best;
}

// Segments per run for a class of `runs` runs holding `prods` products on
// the one-wave-per-run MFMA kernel: enough (run, segment) items for about
// 16 waves per CU when the runs alone are fewer, each segment at least 16
// products long, at most 64 segments and 1 GiB of partial blocks.
static int split_for(int64_t runs, int64_t prods, int m, int n, size_t esize) {
    const int64_t target = (int64_t)cu_count() * 16;
    if (runs <= 0 || runs >= target) return 1;
    int64_t S = ceil_div(target, runs);
    S = std::min<int64_t>(S, prods / runs / 16);
    S = std::min<int64_t>(S, 64);
    S = std::min<int64_t>(S, (int64_t(1) << 30) / (runs * (int64_t)m * n * (int64_t)esize));
    return (int)std::max<int64_t>(S, 1);
}

// Row-major copies of M's blocks into buf (the data of this call: a
// replayed plan copies again, since the values may have changed).
static int copy_rows(const bsmm_matrix_s *M, DevBuf &buf, hipStream_t s) {
    BSMM_TRY(buf.reserve(M->esize() * (size_t)(M->storage + 1), s));
    if (M->nnzb == 0) return BSMM_OK;
    // About 4,096 workgroups, also where there are few block rows.
    const unsigned gy = (unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(4096, M->nbr), 1024));
    const dim3 grid(grid_rows(M->nbr), gy);
    if (M->dtype == BSMM_F32)
        hipLaunchKernelGGL(k_transpose_blocks<float>, grid, dim3(256), 0, s, M->nbr, M->d_row_ptr(),
                           M->d_col_ind(), M->d_rbs(), M->d_cbs(), M->d_blk_off(),
                           (const float *)M->d_raw(), buf.as<float>());
    else
        hipLaunchKernelGGL(k_transpose_blocks<double>, grid, dim3(256), 0, s, M->nbr, M->d_row_ptr(),
                           M->d_col_ind(), M->d_rbs(), M->d_cbs(), M->d_blk_off(),
                           (const double *)M->d_raw(), buf.as<double>());
    return launch_check("transpose_blocks");
}

// What the launch of class cl would gain (us, estimated) from others beside it
// when its runs are few: the time of one run's products one after the other,
// less the 1 us that the host's 5 us for a launch hide beside the kernel's start.  A wave takes 7.5 GFLOP/s on
// the register-tile kernel, 36 (FP32 twice that) on the MFMA kernel and there at
// least 0.25 us for a product and 0.14 for each 8 values of k; a wave of that
// kernel on every SIMD leaves nothing to gain.
static double launch_gain_us(const Stacks &st, int cl, const SmmLaunch &L, double k) {
    if ((int)st.class_prod_begin.size() != st.n_classes + 1) return 0.0;
    const double runs = (double)(st.class_begin[cl + 1] - st.class_begin[cl]);
    const double prods = (double)(st.class_prod_begin[cl + 1] - st.class_prod_begin[cl]);
    const double flops = 2.0 * st.row_sizes[cl / st.ncs] * st.col_sizes[cl % st.ncs] * k;
    const int split = std::max(L.args.split, 1);
    const double chain = prods / std::max(runs, 1.0) / split;
    if (L.args.kc_max > 0) return std::max(chain * flops / 7.5e3 - 1.0, 0.0);  // k chunks in LDS: register tiles
    const double us = std::max(0.25 + 0.14 * std::ceil(k / 8.0), flops / (L.dtype == BSMM_F32 ? 72e3 : 36e3));
    return std::max(chain * us - 1.0, 0.0) * std::max(1.0 - runs * split / (4.0 * cu_count()), 0.0);
}

int run_stacks(const bsmm_matrix_s *A, const bsmm_matrix_s *B, bsmm_matrix_s *C, Stacks &st,
               double alpha, double beta, hipStream_t s, StackExec *ex) {
    ex->launches.clear();
    ex->parts.clear();
    st.n_sched = 0;
    st.n_jit = 0;
    if (st.n_runs == 0) return BSMM_OK;
    const int kmax = std::max(1, A->max_cbs);
    const int64_t chunk = options().stack_chunk;
    const bool tuned = options().stack_kernel == 1;
    const int krep = representative_k(A);
    // Every product has the same depth when A's block columns share one size.
    const int uniform_k = !A->cbs.empty() &&
                                  *std::min_element(A->cbs.begin(), A->cbs.end()) == A->max_cbs
                              ? A->max_cbs
                              : 0;
    std::vector<int64_t> run_ptr_h;
    if (chunk > 0) {
        run_ptr_h.resize(st.n_runs + 1);
        BSMM_HIP(hipMemcpyAsync(run_ptr_h.data(), st.run_ptr.p, sizeof(int64_t) * (st.n_runs + 1),
                                hipMemcpyDeviceToHost, s));
        BSMM_HIP(hipStreamSynchronize(s));
    }
    std::vector<int> rlen;
    if (tuned) {
        // Row panels share the whole multiply's run lengths, so every panel
        // picks the same parameters as one whole stack would.
        if ((int)st.run_len_hint.size() == st.n_classes) rlen = st.run_len_hint;
        else class_run_lengths(st, &rlen);
    }
    LaunchList &launches = ex->launches;
    // Tuned path with a tile size: the MFMA classes of blocks up to 32 x 32
    // whose runs need no splitting go to one scheduled launch.
    // (the plain path too, except in the scratch region, which the schedule
    // would share with the products: its classes keep their own launches).
    const bool sched_on = (tuned || !scratch_arena()) && chunk <= 0 && options().stack_tile > 0 &&
                          (int)st.class_prod_begin.size() == st.n_classes + 1;
    std::vector<char> eligible(st.n_classes, 0);
    const double mean_k = (double)A->cols() / std::max(A->nbc, 1);
    double sum_us = 0.0, longest_us = 0.0;  // of launch_gain_us over the classes' own launches
    auto own_launch = [&](int cl, const SmmLaunch &L) {
        launches.push_back({L, {st.class_begin[cl], st.class_begin[cl + 1]}});
        if (!tuned || options().plan_cache) return;  // never or always a graph
        const double us = launch_gain_us(st, cl, L, mean_k);
        sum_us += us;
        longest_us = std::max(longest_us, us);
    };
    for (int cl = 0; cl < st.n_classes; ++cl) {
        const int64_t rb = st.class_begin[cl], re = st.class_begin[cl + 1];
        if (re <= rb) continue;
        const int m = st.row_sizes[cl / st.ncs], n = st.col_sizes[cl % st.ncs];
        SmmParams prm = tuned ? select_params(m, n, krep, rlen[cl]) : plain_launch(m, n, krep);
        SmmLaunch L;
        BSMM_TRY(plan_smm(prm, m, n, kmax, C->dtype, &L));
        if (chunk <= 0 && prm.tm == kMfmaTile && (int)st.class_prod_begin.size() == st.n_classes + 1) {
            // The plain path never splits a run: its sums keep one order.
            const int S = !tuned ? 1
                                 : split_for(re - rb, st.class_prod_begin[cl + 1] - st.class_prod_begin[cl],
                                             m, n, C->esize());
            if (tuned && options().jit && S == 1 && uniform_k > 0) {
                // One product depth: a kernel compiled for this (m, n, k).
                if (hipFunction_t f = jit_smm_kernel(C->dtype, m, n, uniform_k)) {
                    L.jit_fn = f;
                    launches.push_back({L, {rb, re}});
                    ++st.n_jit;
                    continue;
                }
            }
            if (sched_on && S == 1 && m <= 32 && n <= 32) {
                eligible[cl] = 1;
                continue;
            }
            if (S > 1) {
                DevBuf part;
                BSMM_TRY(part.reserve(C->esize() * (size_t)(re - rb) * S * m * n, s));
                L.args.split = S;
                L.args.part = part.as<double>();
                ex->parts.push_back(std::move(part));
            }
        }
        if (chunk <= 0) {
            own_launch(cl, L);
            continue;
        }
        // Batches of at most `chunk` products; a run is never split.
        int64_t b0 = rb;
        while (b0 < re) {
            int64_t b1 = b0 + 1;
            while (b1 < re && run_ptr_h[b1 + 1] - run_ptr_h[b0] <= chunk) ++b1;
            launches.push_back({L, {b0, b1}});
            b0 = b1;
        }
    }
    int64_t sched_runs = 0, sched_prods = 0;
    int sched_classes = 0;
    for (int cl = 0; cl < st.n_classes; ++cl)
        if (eligible[cl]) {
            ++sched_classes;
            sched_runs += st.class_begin[cl + 1] - st.class_begin[cl];
            sched_prods += st.class_prod_begin[cl + 1] - st.class_prod_begin[cl];
        }
    if (sched_on && sched_runs > 0 && sched_runs < kSchedMinRuns &&
        (sched_classes <= kSchedFewClasses || !options().plan_cache || scratch_arena())) {
        // Too few runs for the scheduling passes to pay off: those classes
        // take their own launches after all (with a scratch arena always, as
        // the schedule would need room there).
        for (int cl = 0; cl < st.n_classes; ++cl) {
            if (!eligible[cl]) continue;
            const int m = st.row_sizes[cl / st.ncs], n = st.col_sizes[cl % st.ncs];
            SmmLaunch L;
            BSMM_TRY(plan_smm(tuned ? select_params(m, n, krep, rlen[cl]) : plain_launch(m, n, krep), m, n, kmax,
                              C->dtype, &L));
            own_launch(cl, L);
            eligible[cl] = 0;
        }
        sched_runs = 0;
    }
    if (sched_on && sched_runs > 0) {
        BSMM_TRY(build_schedule(C, st, eligible, options().stack_tile, s));
        SmmLaunch L;
        // No copies with a scratch arena (they are as large as the operands).
        const bool at = options().stack_at == 1 && !scratch_arena();
        bool bt = !at && !scratch_arena() && B->nnzb > 0 &&
                  st.n_prod / B->nnzb >= kCopyBMinUses;
        if (at) BSMM_TRY(st.a_t.reserve(A->esize() * (size_t)(A->storage + 1), s));
        // Without room for the copy B is read in place (the same bits): C may
        // be grown already and earlier row panels written.
        if (bt && st.b_t.reserve(B->esize() * (size_t)(B->storage + 1), s) != BSMM_OK) {
            clear_error();
            bt = false;
        }
        ex->reads_a_t = at;
        ex->reads_b_t = bt;
        L.fn = (void *)sched_kernel(C->dtype, at, bt);
        L.args.A_t = at ? st.a_t.p : nullptr;
        L.args.B_t = bt ? st.b_t.p : nullptr;
        L.dtype = C->dtype;
        L.args.L = kWave;
        L.args.G = 1;
        L.args.passes = 1;
        L.args.sched = st.sched.as<unsigned long long>();
        L.args.n_sched = st.n_sched;
        L.args.next = st.sched_next.as<unsigned long long>();
        L.args.sched_mode = options().stack_sched;
        L.args.norm2 = norm_sink();
        L.args.run_cblk = st.run_cblk.as<int64_t>();
        // About four products per counter update: runs of one product go
        // four at a time, runs of four or more one at a time (banded 1 %,
        // two products per run: 1.26 / 1.25 / 1.26 / 1.29 / 1.33 ms for 1 / 2
        // / 4 / 8 / 16 runs per update).
        const int64_t mean_len = std::max<int64_t>(1, sched_prods / sched_runs);
        L.args.sched_chunk = mean_len >= 4 ? 1 : mean_len >= 2 ? 2 : 4;
        L.args.sched_seg_bits = schedule_segment_bits(st.n_sched, kXcds);
        // Waves in flight share what an L2 holds, so fewer of them find more
        // there: FP64 three waves per SIMD (2 / 3 / 4 / 5: banded 10 % 61.6 / 58.6
        // / 60.3 / 60.9 ms, 30 % 540 / 537 / 564 / 565, 1 % - / 1.23 / 1.24 / 1.22),
        // FP32, half the bytes each, four (banded 10 % 7.25 / 6.75 / 6.75 with 3
        // / 4 / 5); launches of few runs also four, to end together (48,000
        // runs 251 / 236 / 233 us with 3 / 4 / 5).
        L.args.sched_per_cu = C->dtype == BSMM_F64 && st.n_sched >= 65536 ? 3 : 4;
        L.waves = 4;
        L.lds = 0;
        launches.push_back({L, {0, st.n_sched}});
    }
    // Instantiating a graph may allocate device memory: a multiply running
    // on a scratch arena launches its classes one by one instead, and so
    // does one with run-time compiled kernels (module functions, which a
    // graph kernel node does not take).  Without a plan a graph is built for one
    // use, 150 to 190 us, which its launches have to save by running side by
    // side: it is worth it when all but the longest gain 160 us so.  Tuned, graph
    // and one by one, us: 8 x 8 blocks of 65 and 70, 6 products a run 478 and 997;
    // of 33 to 64, 40 products 669 and 1345, 5 products 363 and 424, 2 products
    // 329 and 209; 12 x 12 blocks of 5 to 32, 40 products 458 and 500, 13 products
    // 344 and 340, 5 products 360 and 206; 40 x 40 blocks of 40 and 64, 40 products
    // 632 and 564; 398 classes of 3.3 short products a run 2.08 and 2.69 ms, 630 of
    // one product 3.97 and 3.20.  More than three launches of many runs gain by it
    // whatever their length.
    const bool worth_graph =
        launches.size() > 1 && (options().plan_cache || sum_us - longest_us > 160.0 ||
                                (launches.size() > 3 && st.n_runs >= kSchedMinRuns));
    if (tuned && chunk <= 0 && worth_graph && !scratch_arena() && st.n_jit == 0) {
        BSMM_TRY(build_graph(launches, A, B, C, st, alpha, beta, &ex->exec));
        BSMM_HIP(hipEventCreateWithFlags(&ex->done, hipEventDisableTiming));
    }
    return replay_stacks(*ex, A, B, C, st, alpha, beta, s);
}

namespace {
std::mutex g_retire_mu;
std::vector<std::pair<hipGraphExec_t, hipEvent_t>> g_retired;

// Destroys the retired graphs whose last launch has completed.
void reap_retired_locked() {
    std::vector<std::pair<hipGraphExec_t, hipEvent_t>> keep;
    for (auto &r : g_retired) {
        const hipError_t q = r.second ? hipEventQuery(r.second) : hipSuccess;
        if (q == hipErrorNotReady) {
            if (hipPeekAtLastError() == hipErrorNotReady) (void)hipGetLastError();
            keep.push_back(r);
            continue;
        }
        (void)hipGraphExecDestroy(r.first);
        if (r.second) (void)hipEventDestroy(r.second);
    }
    g_retired.swap(keep);
}
}  // namespace

void retire_graph(hipGraphExec_t exec, hipEvent_t done) {
    std::lock_guard<std::mutex> lk(g_retire_mu);
    g_retired.push_back({exec, done});
    reap_retired_locked();
    // Bounded backlog: wait for the oldest retired graph when many are pending.
    while (g_retired.size() > 64) {
        if (g_retired.front().second) (void)hipEventSynchronize(g_retired.front().second);
        reap_retired_locked();
    }
}

int replay_stacks(const StackExec &ex, const bsmm_matrix_s *A, const bsmm_matrix_s *B,
                  bsmm_matrix_s *C, Stacks &st, double alpha, double beta, hipStream_t s) {
    // Same buffers (the launches hold their addresses), this call's values;
    // later row panels of one multiply find them there.
    if (ex.reads_a_t && !st.a_t_fresh) BSMM_TRY(copy_rows(A, st.a_t, s));
    if (ex.reads_b_t && !st.b_t_fresh) BSMM_TRY(copy_rows(B, st.b_t, s));
    if (ex.reads_a_t) st.a_t_fresh = true;
    if (ex.reads_b_t) st.b_t_fresh = true;
    if (ex.exec) {
        {
            KernelTimer kt(1, s);
            BSMM_HIP(hipGraphLaunch(ex.exec, s));
        }
        if (ex.done) BSMM_HIP(hipEventRecord(ex.done, s));
        return BSMM_OK;
    }
    for (auto &l : ex.launches)
        BSMM_TRY(launch_smm(l.first, A->d_raw(), B->d_raw(), C->d_raw(),
                            st.run_coff.as<int64_t>(), st.run_ptr.as<int64_t>(),
                            st.prods.as<ulonglong2>(), l.second.first, l.second.second, alpha, beta,
                            s));
    return BSMM_OK;
}

// Tuned path: all shape classes as independent kernel nodes of one hipGraph
// (launched once, classes run concurrently).  The kernel arguments are
// copied into the graph when the nodes are added.
int build_graph(const LaunchList &launches, const bsmm_matrix_s *A, const bsmm_matrix_s *B,
                bsmm_matrix_s *C, const Stacks &st, double alpha, double beta,
                hipGraphExec_t *out) {
    hipGraph_t graph = nullptr;
    BSMM_HIP(hipGraphCreate(&graph, 0));
    int status = BSMM_OK;
    for (size_t i = 0; i < launches.size() && status == BSMM_OK; ++i) {
        const SmmLaunch &L = launches[i].first;
        SmmArgs a = L.args;
        a.A = A->d_raw();
        a.B = B->d_raw();
        a.C = C->d_raw();
        a.run_coff = st.run_coff.as<int64_t>();
        a.run_ptr = st.run_ptr.as<int64_t>();
        a.prods = st.prods.as<ulonglong2>();
        a.run_begin = launches[i].second.first;
        a.run_end = launches[i].second.second;
        a.alpha = alpha;
        a.beta = beta;
        void *argp = &a;
        hipKernelNodeParams kp{};
        kp.func = L.fn;
        kp.gridDim = dim3(smm_grid(L, a.run_end - a.run_begin));
        kp.blockDim = dim3(64 * L.waves);
        kp.sharedMemBytes = (unsigned)L.lds;
        kp.kernelParams = &argp;
        kp.extra = nullptr;
        hipGraphNode_t node, zero;
        const bool counter = is_sched_kernel(L.fn) && a.sched_mode == 1;
        void *zargp = &a.next;
        if (counter) {
            // The dynamic schedule's run counter starts at zero every replay
            // (a kernel node: memset nodes are not used in the graph).
            hipKernelNodeParams zp{};
            zp.func = (void *)k_zero_counters;
            zp.gridDim = dim3(1);
            zp.blockDim = dim3(kXcds);
            zp.sharedMemBytes = 0;
            zp.kernelParams = &zargp;
            zp.extra = nullptr;
            if (hipGraphAddKernelNode(&zero, graph, nullptr, 0, &zp) != hipSuccess) {
                set_error(BSMM_EDEVICE, "hipGraphAddKernelNode failed");
                status = BSMM_EDEVICE;
                break;
            }
        }
        if (hipGraphAddKernelNode(&node, graph, counter ? &zero : nullptr, counter ? 1 : 0, &kp) !=
            hipSuccess) {
            set_error(BSMM_EDEVICE, "hipGraphAddKernelNode failed");
            status = BSMM_EDEVICE;
        } else if (a.split > 1) {
            // The class's split-run epilogue runs after its kernel.
            hipKernelNodeParams rp{};
            rp.func = L.dtype == BSMM_F32 ? (void *)k_smm_split_reduce<float>
                                          : (void *)k_smm_split_reduce<double>;
            rp.gridDim = dim3(split_reduce_grid(a));
            rp.blockDim = dim3(256);
            rp.sharedMemBytes = 0;
            rp.kernelParams = &argp;
            rp.extra = nullptr;
            hipGraphNode_t rnode;
            if (hipGraphAddKernelNode(&rnode, graph, &node, 1, &rp) != hipSuccess) {
                set_error(BSMM_EDEVICE, "hipGraphAddKernelNode failed");
                status = BSMM_EDEVICE;
            }
        }
    }
    if (status == BSMM_OK && hipGraphInstantiate(out, graph, nullptr, nullptr, 0) != hipSuccess) {
        set_error(BSMM_EDEVICE, "hipGraphInstantiate failed");
        *out = nullptr;
        status = BSMM_EDEVICE;
    }
    (void)hipGraphDestroy(graph);
    (void)hipGetLastError();
    return status;
}

}  // namespace bsmm
