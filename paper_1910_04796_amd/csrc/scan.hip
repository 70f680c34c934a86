// scan.hip -- device exclusive prefix sums (three-phase, recursive).
#include "dev_util.h"
#include "internal.h"

namespace bsmm {

namespace {
constexpr int kScanThreads = 256;
constexpr int kScanItems = 4;
constexpr int kScanPass = kScanThreads * kScanItems;  // values a workgroup scans at a time
// Values per workgroup, taken in passes: two levels reach 16.7 M values, so
// a scan is three launches (one below a tile); with tiles of one pass, the
// index scans of C blocks took five, and a multiply of short kernels waits
// for its launches.
constexpr int kScanTile = 4 * kScanPass;

// Up to two arrays of n values each, scanned by the same launches (the grid's
// second dimension).
struct ScanPair {
    const int64_t *in[2];
    int64_t *out[2];
    int64_t *sums[2];
};

// Each workgroup scans one tile; tile totals go to sums (one tile: to out[n]).
__global__ __launch_bounds__(kScanThreads) void k_scan_tile(ScanPair a, int64_t n) {
    __shared__ int64_t lds[16];
    const int64_t *in = a.in[blockIdx.y];
    int64_t *out = a.out[blockIdx.y], *sums = a.sums[blockIdx.y];
    const int64_t tile = (int64_t)blockIdx.x * kScanTile;
    int64_t carry = 0;
    for (int64_t pass = tile; pass < min(tile + kScanTile, n); pass += kScanPass) {
        const int64_t base = pass + (int64_t)threadIdx.x * kScanItems;
        int64_t v[kScanItems];
        int64_t local = 0;
#pragma unroll
        for (int i = 0; i < kScanItems; ++i) {
            v[i] = (base + i < n) ? in[base + i] : 0;
            local += v[i];
        }
        int64_t total;
        int64_t run = carry + block_exclusive_scan(local, lds, &total);
#pragma unroll
        for (int i = 0; i < kScanItems; ++i) {
            if (base + i < n) out[base + i] = run;
            run += v[i];
        }
        carry += total;
    }
    if (threadIdx.x == 0) {
        if (sums) sums[blockIdx.x] = carry;
        else out[n] = carry;
    }
}

__global__ __launch_bounds__(kScanThreads) void k_scan_add(ScanPair a, int64_t n) {
    int64_t *out = a.out[blockIdx.y];
    const int64_t *offs = a.sums[blockIdx.y];
    const int64_t add = offs[blockIdx.x];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    for (int64_t i = base + threadIdx.x; i < min(base + kScanTile, n); i += kScanThreads) out[i] += add;
    if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = offs[gridDim.x];
}

__global__ void k_set_zero_i64(ScanPair a) { *a.out[blockIdx.x] = 0; }

int scan(ScanPair a, int arrays, int64_t n, hipStream_t s) {
    if (n <= 0) {
        hipLaunchKernelGGL(k_set_zero_i64, dim3(arrays), dim3(1), 0, s, a);
        return launch_check("scan_zero");
    }
    const int64_t tiles = ceil_div(n, kScanTile);
    DevBuf sums[2];
    if (tiles > 1)
        for (int i = 0; i < arrays; ++i) {
            BSMM_TRY(sums[i].reserve(sizeof(int64_t) * (tiles + 1), s));
            a.sums[i] = sums[i].as<int64_t>();
        }
    hipLaunchKernelGGL(k_scan_tile, dim3((unsigned)tiles, arrays), dim3(kScanThreads), 0, s, a, n);
    BSMM_TRY(launch_check("scan_tile"));
    if (tiles == 1) return BSMM_OK;
    ScanPair up{};
    for (int i = 0; i < arrays; ++i) up.in[i] = up.out[i] = a.sums[i];
    BSMM_TRY(scan(up, arrays, tiles, s));
    hipLaunchKernelGGL(k_scan_add, dim3((unsigned)tiles, arrays), dim3(kScanThreads), 0, s, a, n);
    return launch_check("scan_add");
}
}  // namespace

int scan_exclusive_i64(const int64_t *in, int64_t *out, int64_t n, hipStream_t s) {
    ScanPair a{};
    a.in[0] = in;
    a.out[0] = out;
    return scan(a, 1, n, s);
}

int scan_exclusive_pair(const int64_t *in0, int64_t *out0, const int64_t *in1, int64_t *out1, int64_t n,
                        hipStream_t s) {
    ScanPair a{};
    a.in[0] = in0;
    a.out[0] = out0;
    a.in[1] = in1;
    a.out[1] = out1;
    return scan(a, 2, n, s);
}

}  // namespace bsmm
