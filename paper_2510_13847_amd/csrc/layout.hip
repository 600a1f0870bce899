// One-time cluster-contiguous layout of the LM head.
//
// The paper partitions the vocabulary into M disjoint clusters of free sizes
// (Sec. 4.2, "Vocabulary partition").  Storing every cluster as one run of
// consecutive rows turns the shortlist gather of the head into whole-slab
// streams.  The layout is a stable counting sort of the tokens by cluster id
// (ties keep ascending vocabulary id), followed by a row-permuting copy.
#include <algorithm>
#include <atomic>

#include "dyna_device.h"

namespace dyna {
namespace {

constexpr int kChunk = 4096;  // tokens per counting workgroup
constexpr int kCountThreads = 1024;
constexpr size_t kCountLds = 128 * 1024;  // budget of the per-wave counters

// Waves of a counting workgroup: as many as have 16-bit counters for every
// cluster within the LDS budget (16 up to 4096 clusters, 8 up to 8192).
int count_waves(int32_t M) {
    int w = kCountThreads / kWave;
    while (w > 1 && (size_t)w * (size_t)M * 2 > kCountLds) w >>= 1;
    return w;
}

// Per chunk of kChunk tokens: the rank of every token among the earlier
// tokens of its cluster inside the chunk, and the chunk's per-cluster counts
// (ids outside [0, M) are skipped).  Every wave takes a run of consecutive
// tokens, 64 at a time: the lanes with the same id find each other by one
// ballot per id bit, so a token's rank inside its wave is the wave's counter
// plus the earlier lanes of its group.  The waves' counters are then
// prefixed in wave order.  (A loop that compared each token with the 255
// before it took 69 us at 128256 tokens; this takes 7.)
__global__ __launch_bounds__(kCountThreads) void layout_count_kernel(const int32_t* __restrict__ cluster_of, int32_t V,
                                                                     int32_t M, int id_bits,
                                                                     int32_t* __restrict__ rank,
                                                                     int32_t* __restrict__ cnt) {
    extern __shared__ uint16_t counters[];  // [waves][M]
    __shared__ uint16_t in_wave[kChunk];    // rank of each token among its wave's
    const int nw = blockDim.x / kWave;
    const int w = threadIdx.x / kWave, lane = lane_id();
    const int64_t base = (int64_t)blockIdx.x * kChunk;
    const int span = kChunk / nw;  // tokens per wave (a multiple of 64)
    for (int i = threadIdx.x; i < nw * M; i += blockDim.x) counters[i] = 0;
    __syncthreads();
    volatile uint16_t* own = counters + (size_t)w * M;
    for (int i = w * span + lane; i < (w + 1) * span; i += kWave) {
        const int64_t v = base + i;
        int c = v < V ? cluster_of[v] : -1;
        if (c < 0 || c >= M) c = -1;
        uint64_t same = __ballot(c >= 0);
        for (int bit = 0; bit < id_bits; ++bit) {
            const bool one = (c >> bit) & 1;
            const uint64_t ones = __ballot(one);
            same &= one ? ones : ~ones;
        }
        if (c >= 0) {
            const int before = own[c];
            in_wave[i] = (uint16_t)(before + __popcll(same & ((1ull << lane) - 1)));
            // the group's last lane counts the group
            if ((same >> lane) == 1) own[c] = (uint16_t)(before + __popcll(same));
        }
        wave_lds_order();
    }
    __syncthreads();
    for (int m = threadIdx.x; m < M; m += blockDim.x) {
        int run = 0;
        for (int q = 0; q < nw; ++q) {
            const int n = counters[(size_t)q * M + m];
            counters[(size_t)q * M + m] = (uint16_t)run;  // (at most kChunk)
            run += n;
        }
        cnt[(int64_t)blockIdx.x * M + m] = run;
    }
    __syncthreads();
    for (int i = w * span + lane; i < (w + 1) * span; i += kWave) {
        const int64_t v = base + i;
        if (v >= V) break;
        const int c = cluster_of[v];
        if (c >= 0 && c < M) rank[v] = in_wave[i] + counters[(size_t)w * M + c];
    }
}

// Single workgroup: cluster totals, their exclusive scan (the CSR offsets),
// and per (chunk, cluster) the first layout row of that chunk's tokens.  The
// clusters go 1024 at a time (one per thread, so that the counts are read
// coalesced), a thread's counts of kScanFlight chunks at once.
constexpr int kScanThreads = 1024;
constexpr int kScanFlight = 32;
__global__ __launch_bounds__(kScanThreads) void layout_scan_kernel(int32_t M, int32_t nchunks,
                                                                   int32_t* __restrict__ cnt,
                                                                   int32_t* __restrict__ offsets) {
    __shared__ int tmp[kScanThreads / kWave + 1];
    int carry = 0;
    for (int m0 = 0; m0 < M; m0 += kScanThreads) {
        const int m = m0 + (int)threadIdx.x;
        const bool in = m < M;
        int x[kScanFlight];
        int local = 0;
        for (int c0 = 0; c0 < nchunks; c0 += kScanFlight) {
#pragma unroll
            for (int q = 0; q < kScanFlight; ++q)
                x[q] = in && c0 + q < nchunks ? cnt[(int64_t)(c0 + q) * M + m] : 0;
#pragma unroll
            for (int q = 0; q < kScanFlight; ++q) local += x[q];
        }
        int total;
        int run = carry + block_exclusive_scan<kScanThreads>(local, tmp, &total);
        carry += total;
        if (in) offsets[m] = run;
        for (int c0 = 0; c0 < nchunks; c0 += kScanFlight) {
            if (nchunks > kScanFlight) {  // (else still in registers)
#pragma unroll
                for (int q = 0; q < kScanFlight; ++q)
                    x[q] = in && c0 + q < nchunks ? cnt[(int64_t)(c0 + q) * M + m] : 0;
            }
#pragma unroll
            for (int q = 0; q < kScanFlight; ++q) {
                if (in && c0 + q < nchunks) cnt[(int64_t)(c0 + q) * M + m] = run;
                run += x[q];
            }
        }
    }
    if (threadIdx.x == 0) offsets[M] = carry;
}

// perm[row] = token.  Tokens with an id outside [0, M) have no row; the rows
// past the last cluster, which they leave over, hold -1.
__global__ void layout_scatter_kernel(const int32_t* __restrict__ cluster_of, int32_t V, int32_t M,
                                      const int32_t* __restrict__ rank,
                                      const int32_t* __restrict__ base,
                                      const int32_t* __restrict__ offsets,
                                      int32_t* __restrict__ perm) {
    const int32_t covered = offsets[M];
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < V;
         v += (int64_t)gridDim.x * blockDim.x) {
        if (v >= covered) perm[v] = -1;
        const int c = cluster_of[v];
        if (c < 0 || c >= M) continue;
        const int64_t chunk = v / kChunk;
        perm[base[chunk * M + c] + rank[v]] = (int32_t)v;
    }
}

// W_perm[j] = W[perm[j]]: one wave per row, 16-byte vectors, kCopyFlight of
// them in flight per lane, streamed past the caches on both sides.  Where a
// bad cluster id leaves rows over, nothing is copied (the host reports the id
// afterwards): W_perm stays as it was.  One row per wave up to kCopyBlocks
// workgroups (16.8 million rows); a launch holds less than 2^32 threads, so
// longer tables go round.
constexpr int kCopyFlight = 8;
constexpr int64_t kCopyBlocks = 1 << 22;
__global__ __launch_bounds__(256) void layout_copy_rows_kernel(const u32x4* __restrict__ W,
                                                               u32x4* __restrict__ Wp,
                                                               const int32_t* __restrict__ perm,
                                                               const int32_t* __restrict__ covered, int32_t V,
                                                               int32_t vec_per_row) {
    const int lane = lane_id();
    if (*covered != V) return;
    const int64_t stride = (int64_t)gridDim.x * (blockDim.x / kWave);
    for (int64_t j = blockIdx.x * (int64_t)(blockDim.x / kWave) + threadIdx.x / kWave; j < V; j += stride) {
        const int64_t src = perm[j];
        const u32x4* s = W + src * vec_per_row;
        u32x4* d = Wp + j * vec_per_row;
        for (int i0 = lane; i0 < vec_per_row; i0 += kCopyFlight * kWave) {
            u32x4 x[kCopyFlight];
#pragma unroll
            for (int q = 0; q < kCopyFlight; ++q)
                if (i0 + q * kWave < vec_per_row) x[q] = __builtin_nontemporal_load(s + i0 + q * kWave);
#pragma unroll
            for (int q = 0; q < kCopyFlight; ++q)
                if (i0 + q * kWave < vec_per_row) __builtin_nontemporal_store(x[q], d + i0 + q * kWave);
        }
    }
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

}  // namespace

size_t layout_ws_bytes(int32_t V, int32_t M) {
    const int64_t nchunks = (V + kChunk - 1) / kChunk;
    return align256(sizeof(int32_t) * (size_t)V) + align256(sizeof(int32_t) * (size_t)nchunks * M) +
           256;
}

dyna_status launch_cluster_csr(const int32_t* cluster_of, int32_t V, int32_t M, int32_t* perm,
                               int32_t* offsets, void* ws, hipStream_t stream) {
    const int32_t nchunks = (V + kChunk - 1) / kChunk;
    char* p = static_cast<char*>(ws);
    int32_t* rank = reinterpret_cast<int32_t*>(p);
    p += align256(sizeof(int32_t) * (size_t)V);
    int32_t* cnt = reinterpret_cast<int32_t*>(p);
    const int nw = count_waves(M);
    const size_t lds = (size_t)nw * (size_t)M * sizeof(uint16_t);
    static std::atomic<uint64_t> allowed{0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
        return set_error(DYNA_ERR_HIP, "layout: device");
    if (!(allowed.load() & (1ull << dev))) {
        if (hipFuncSetAttribute((const void*)layout_count_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)kCountLds) != hipSuccess)
            return set_error(DYNA_ERR_HIP, "layout: LDS attribute");
        allowed.fetch_or(1ull << dev);
    }
    int id_bits = 1;
    while ((1 << id_bits) < M) ++id_bits;
    layout_count_kernel<<<nchunks, nw * kWave, lds, stream>>>(cluster_of, V, M, id_bits, rank, cnt);
    if (dyna_status s = check_launch("layout_count_kernel"); s != DYNA_OK) return s;
    layout_scan_kernel<<<1, kScanThreads, 0, stream>>>(M, nchunks, cnt, offsets);
    if (dyna_status s = check_launch("layout_scan_kernel"); s != DYNA_OK) return s;
    layout_scatter_kernel<<<(V + 255) / 256, 256, 0, stream>>>(cluster_of, V, M, rank, cnt, offsets, perm);
    return check_launch("layout_scatter_kernel");
}

dyna_status launch_build_layout(const int32_t* cluster_of, int32_t V, int32_t M, const void* W_lm,
                                int32_t wdtype, int32_t d, void* W_perm, int32_t* perm,
                                int32_t* offsets, void* ws, size_t ws_bytes,
                                int32_t* host_offsets_out, hipStream_t stream) {
    (void)ws_bytes;
    if (dyna_status s = launch_cluster_csr(cluster_of, V, M, perm, offsets, ws, stream); s != DYNA_OK) return s;
    const int elt = wdtype == DYNA_BF16 ? 2 : 4;
    const int32_t vec_per_row = (int32_t)((int64_t)d * elt / 16);
    const int64_t blocks = std::min<int64_t>(((int64_t)V + 3) / 4, kCopyBlocks);
    layout_copy_rows_kernel<<<(unsigned)blocks, 256, 0, stream>>>(
        static_cast<const u32x4*>(W_lm), static_cast<u32x4*>(W_perm), perm, offsets + M, V, vec_per_row);
    if (dyna_status s = check_launch("layout_copy_rows_kernel"); s != DYNA_OK) return s;
    // the offsets come back behind the copy, so that the GPU never waits for the host
    if (hipMemcpyAsync(host_offsets_out, offsets, sizeof(int32_t) * (size_t)(M + 1), hipMemcpyDeviceToHost,
                       stream) != hipSuccess ||
        hipStreamSynchronize(stream) != hipSuccess)
        return set_error(DYNA_ERR_HIP, "build_layout: device copy/synchronise failed");
    // an id outside [0, M) is in no cluster, so the clusters do not cover V
    if (host_offsets_out[M] != V) return set_error(DYNA_ERR_DEVICE_DATA, "build_layout: cluster id outside [0, M)");
    return DYNA_OK;
}

}  // namespace dyna
