// Building the partition: spherical k-means over the LM-head rows (Sec. 4.2,
// "Vocabulary partition": the clusters come from spherical k-means on the
// column-normalised head, one point per vocabulary entry).
//
// One round is an assignment and an update.
//  * Assignment: every row goes to the centroid of largest cosine
//    similarity.  Dividing a row by its norm does not change which centroid
//    wins, so the raw bf16 rows are scored against the bf16 unit centroids:
//    a dense V x M x d product on the matrix cores with an argmax epilogue
//    (assign.hip; the fixed DYNA_OPT_KMEANS_CFG shapes on the union-row
//    kernel), so no V x M score matrix is ever written.  Ties go to the lower
//    centroid id.
//  * Update: a stable counting sort of the assignment (the layout's CSR
//    kernels) lists each cluster's rows in ascending id; one workgroup per
//    cluster sums its unit rows in that order in fp32 and divides by the
//    norm of the sum.  An empty cluster (or a zero sum) keeps its centroid.
// Every sum runs in a fixed order, so a run is bit-identical to the next.
#include "dyna_device.h"

namespace dyna {
namespace {

constexpr int kKmThreads = 256;

// bf16 bits of x, rounded to nearest with ties to even (NaN stays a quiet NaN).
__device__ __forceinline__ uint16_t to_bf16_rne(float x) {
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Centroid m starts at the unit row init_ids[m]; an id outside [0, V) gives a
// zero centroid and sets *bad.  Also clears the assignment's per-row maxima.
__global__ __launch_bounds__(kKmThreads) void centroid_init_kernel(const uint16_t* __restrict__ W,
                                                                   const int32_t* __restrict__ init_ids,
                                                                   int32_t V, int32_t d, float* __restrict__ mu32,
                                                                   uint16_t* __restrict__ mu16,
                                                                   unsigned long long* __restrict__ keys,
                                                                   int32_t* __restrict__ bad) {
    const int64_t m = blockIdx.x;
    for (int64_t i = m * kKmThreads + threadIdx.x; i < V; i += (int64_t)gridDim.x * kKmThreads) keys[i] = 0;
    const int32_t v = init_ids[m];
    const bool ok = v >= 0 && v < V;
    if (!ok && threadIdx.x == 0) atomicOr(bad, 1);
    __shared__ float red[kKmThreads / kWave];
    float ss = 0.0f;
    for (int c = threadIdx.x; ok && c < d; c += kKmThreads) {
        const float x = __uint_as_float((uint32_t)W[(int64_t)v * d + c] << 16);
        ss = fmaf(x, x, ss);
    }
    ss = wave_sum(ss);
    if (lane_id() == 0) red[threadIdx.x / kWave] = ss;
    __syncthreads();
    float tot = 0.0f;
#pragma unroll
    for (int w = 0; w < kKmThreads / kWave; ++w) tot += red[w];
    const float sc = tot > 0.0f ? 1.0f / sqrtf(tot) : 0.0f;  // an all-zero row has no direction
    for (int c = threadIdx.x; c < d; c += kKmThreads) {
        const float x = ok ? __uint_as_float((uint32_t)W[(int64_t)v * d + c] << 16) * sc : 0.0f;
        mu32[m * d + c] = x;
        mu16[m * d + c] = to_bf16_rne(x);
    }
}

__global__ void clear_word_kernel(int32_t* p) { *p = 0; }

// Also clears n_keys words of the assignment's per-row maxima.
__global__ void f32_to_bf16_kernel(const float* __restrict__ src, uint16_t* __restrict__ dst, int64_t n,
                                   unsigned long long* __restrict__ keys, int64_t n_keys) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = to_bf16_rne(src[i]);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n_keys; i += (int64_t)gridDim.x * blockDim.x)
        keys[i] = 0;
}

// Plan over every row: chunk c is rows [16c, 16c + 16), output slot = row,
// and stands for all B centroids.
__global__ void full_plan_kernel(int32_t V, int32_t B, Plan plan) {
    const int64_t n = ((int64_t)V + kChunkRows - 1) / kChunkRows;
    for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < n; c += (int64_t)gridDim.x * blockDim.x)
        plan.chunks[c] = Chunk{(int32_t)(c * kChunkRows), (int32_t)min<int64_t>(kChunkRows, V - c * kChunkRows),
                               (int32_t)(c * kChunkRows), B};
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        plan.hdr->n_chunks = (int32_t)n;
        plan.hdr->n_entries = 0;
    }
}

// mu[m] = (sum of the unit rows of cluster m, in ascending row id) / its norm;
// an empty cluster or a zero sum keeps mu[m].  One workgroup of NT threads per
// cluster; thread t owns columns 8 t + 8 NT j, j < J.  The rows stream in
// batches of U, the next batch in flight while the current one's norms are
// summed across the workgroup (a pass of its own for the norms read every row
// once more: 152 us over 128256 x 4096 rows).  With many clusters it is bound
// by HBM: 1024 clusters of 128256 x 4096 rows 190-197 us, 5.3-5.5 TB/s, with
// EU waves per SIMD so that four workgroups share a compute unit and all
// clusters run at once.  With few clusters a workgroup's time is its batches'
// latency, so the batches are longer.
template <int NT, int J, int U, int EU>
__global__ __launch_bounds__(NT, EU) void centroid_update_kernel(const uint16_t* __restrict__ W,
                                                                 const int32_t* __restrict__ perm,
                                                                 const int32_t* __restrict__ offsets, int32_t d,
                                                                 float* __restrict__ mu32,
                                                                 uint16_t* __restrict__ mu16) {
    constexpr int NW = NT / kWave;
    constexpr int COLS = 8 * NT;  // columns one pass of the workgroup covers
    __shared__ float red[2][NW][U];
    const int64_t m = blockIdx.x;
    const int32_t i0 = offsets[m], i1 = offsets[m + 1];
    if (i0 >= i1) return;  // empty: unchanged (whole workgroup)
    float s[J][8];
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int e = 0; e < 8; ++e) s[j][e] = 0.0f;
    u32x4 x[U][J], y[U][J];
    int32_t v[U];
    // rows i .. i + U - 1 (past the cluster: zeros, which add nothing)
    auto ids = [&](int32_t i) {
#pragma unroll
        for (int q = 0; q < U; ++q) v[q] = i + q < i1 ? perm[i + q] : -1;
    };
    auto load = [&]() {
#pragma unroll
        for (int q = 0; q < U; ++q)
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int c0 = 8 * (int)threadIdx.x + COLS * j;
                y[q][j] = u32x4{0u, 0u, 0u, 0u};
                if (v[q] >= 0 && c0 < d)
                    y[q][j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(W + (int64_t)v[q] * d + c0));
            }
    };
    ids(i0);
    load();
    ids(i0 + U);
    int at = 0;
    for (int32_t i = i0; i < i1; i += U, at ^= 1) {
#pragma unroll
        for (int q = 0; q < U; ++q)
#pragma unroll
            for (int j = 0; j < J; ++j) x[q][j] = y[q][j];
        if (i + U < i1) {
            load();
            ids(i + 2 * U);
        }
        // the batch's squared norms (two places in turn: one barrier a batch)
        float norm[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            float n = 0.0f;
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float lo = bf16_lo(x[q][j][e]), hi = bf16_hi(x[q][j][e]);
                    n = fmaf(lo, lo, n);
                    n = fmaf(hi, hi, n);
                }
            norm[q] = wave_sum(n);
            if (NW > 1 && lane_id() == 0) red[at][threadIdx.x / kWave][q] = norm[q];
        }
        if constexpr (NW > 1) lds_barrier();  // the next batch's loads stay in flight
#pragma unroll
        for (int q = 0; q < U; ++q) {
            float n = norm[q];
            if constexpr (NW > 1) {
                n = 0.0f;
#pragma unroll
                for (int w = 0; w < NW; ++w) n += red[at][w][q];
            }
            const float sc = n > 0.0f ? 1.0f / sqrtf(n) : 0.0f;  // an all-zero row adds nothing
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    s[j][2 * e] = fmaf(bf16_lo(x[q][j][e]), sc, s[j][2 * e]);
                    s[j][2 * e + 1] = fmaf(bf16_hi(x[q][j][e]), sc, s[j][2 * e + 1]);
                }
        }
    }
    __syncthreads();
    float ss = 0.0f;
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int e = 0; e < 8; ++e) ss = fmaf(s[j][e], s[j][e], ss);
    ss = wave_sum(ss);
    if (lane_id() == 0) red[0][threadIdx.x / kWave][0] = ss;
    __syncthreads();
    float tot = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) tot += red[0][w][0];
    if (!(tot > 0.0f)) return;  // zero sum: unchanged
    const float rn = 1.0f / sqrtf(tot);
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int c0 = 8 * (int)threadIdx.x + COLS * j;
        if (c0 < d) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float y = s[j][e] * rn;
                mu32[m * d + c0 + e] = y;
                mu16[m * d + c0 + e] = to_bf16_rne(y);
            }
        }
    }
}

size_t al256(size_t x) { return (x + 255) & ~size_t(255); }

// Workspace views.
struct KmWs {
    uint16_t* mu16;    // [M, d]
    float* mu32;       // [M, d] (used when the caller keeps no centroids)
    int32_t* assign;   // [V] (used when the caller keeps no assignment)
    int32_t* perm;     // [V]
    int32_t* offsets;  // [M + 1]
    int32_t* bad;      // [1]
    unsigned long long* keys;  // [V] the assignment's per-row maxima
    Plan plan;
    void* csr;         // layout_ws_bytes(V, M)
    size_t bytes;
};

KmWs km_carve(int32_t V, int32_t d, int32_t M, void* base) {
    KmWs w{};
    char* p = static_cast<char*>(base);
    size_t off = 0;
    auto take = [&](size_t n) -> void* {
        void* q = p ? p + off : nullptr;
        off += al256(n);
        return q;
    };
    const int64_t n_chunks = ((int64_t)V + kChunkRows - 1) / kChunkRows;
    w.mu16 = static_cast<uint16_t*>(take(sizeof(uint16_t) * (size_t)M * d));
    w.mu32 = static_cast<float*>(take(sizeof(float) * (size_t)M * d));
    w.assign = static_cast<int32_t*>(take(sizeof(int32_t) * (size_t)V));
    w.perm = static_cast<int32_t*>(take(sizeof(int32_t) * (size_t)V));
    w.offsets = static_cast<int32_t*>(take(sizeof(int32_t) * ((size_t)M + 1)));
    w.bad = static_cast<int32_t*>(take(sizeof(int32_t)));
    w.keys = static_cast<unsigned long long*>(take(sizeof(unsigned long long) * (size_t)V));
    w.plan.hdr = static_cast<PlanHeader*>(take(sizeof(PlanHeader)));
    w.plan.chunks = static_cast<Chunk*>(take(sizeof(Chunk) * (size_t)n_chunks));
    w.plan.list = static_cast<ListEntry*>(take(sizeof(ListEntry)));
    w.plan.max_chunks = (int32_t)n_chunks;
    w.plan.max_entries = 1;
    w.csr = take(layout_ws_bytes(V, M));
    w.bytes = off;
    return w;
}

// w.keys is zero on entry and on return.
dyna_status launch_assign(const uint16_t* W, int32_t V, int32_t d, const uint16_t* mu16, int32_t M, int32_t* assign,
                          float* score, const KmWs& w, hipStream_t stream) {
    if (option_kmeans_cfg() == 0) return launch_nearest_centroid(W, V, d, mu16, M, w.keys, assign, score, stream);
    if (dyna_status s = launch_full_plan(V, M, w.plan, stream); s != DYNA_OK) return s;
    RowdotArgs a{};
    a.W = W;
    a.wdtype = DYNA_BF16;
    a.K = d;
    a.v = mu16;
    a.vdtype = DYNA_BF16;
    a.B = M;
    a.out = score;
    a.ld = 0;
    a.act = DYNA_ACT_NONE;
    a.plan = w.plan;
    a.max_chunks_bound = w.plan.max_chunks;
    a.vid_out = assign;
    return launch_union_argmax(a, option_kmeans_cfg(), stream);
}

dyna_status launch_update(const uint16_t* W, int32_t V, int32_t d, const int32_t* assign, int32_t M,
                          const KmWs& w, float* mu32, hipStream_t stream) {
    if (dyna_status s = launch_cluster_csr(assign, V, M, w.perm, w.offsets, w.csr, stream); s != DYNA_OK) return s;
    auto launch = [&](int threads, auto kernel) -> dyna_status {
        kernel<<<M, threads, 0, stream>>>(W, w.perm, w.offsets, d, mu32, w.mu16);
        return check_launch("centroid_update_kernel");
    };
    // Long batches (16 rows; 8 beyond 2048 columns, whose registers hold no
    // more) while the clusters are few, shorter ones and more workgroups per
    // compute unit beyond; up to 512 columns a wave holds the whole row, and its
    // sum needs no barrier.  Whole update of 128256 rows, with the norms'
    // separate pass before, with batches of 4 everywhere, and now: 256 columns,
    // 64 clusters 735, 1053 and 625 us, 1024: 231, 232, 142; 1024 columns, 64: 761,
    // 970, 717, 768: 217, 161, 146; 4096 columns, 128: 692, 593, 576.
    if (d <= 512) return launch(64, centroid_update_kernel<64, 1, 16, 2>);
    if (d <= 2048)
        return M <= 512 ? launch(256, centroid_update_kernel<256, 1, 16, 2>)
                        : launch(256, centroid_update_kernel<256, 1, 8, 4>);
    if (d <= 4096)
        return M <= 256 ? launch(256, centroid_update_kernel<256, 2, 8, 2>)
                        : launch(256, centroid_update_kernel<256, 2, 4, 4>);
    if (d <= 8192) return launch(256, centroid_update_kernel<256, 4, 4, 2>);
    return set_error(DYNA_ERR_UNSUPPORTED, "k-means: d=%d > 8192", d);
}

}  // namespace

dyna_status launch_full_plan(int32_t V, int32_t M, const Plan& plan, hipStream_t stream) {
    const int64_t n = ((int64_t)V + kChunkRows - 1) / kChunkRows;
    const unsigned blocks = (unsigned)std::min<int64_t>(1024, (n + 255) / 256);
    full_plan_kernel<<<std::max(1u, blocks), 256, 0, stream>>>(V, M, plan);
    return check_launch("full_plan_kernel");
}

size_t kmeans_ws_bytes(int32_t V, int32_t d, int32_t M) { return km_carve(V, d, M, nullptr).bytes; }

dyna_status kmeans_assign(const void* W, int32_t V, int32_t d, const float* centroids, int32_t M,
                          int32_t* out_assign, float* out_score, void* ws, hipStream_t stream) {
    const KmWs w = km_carve(V, d, M, ws);
    const int64_t n = (int64_t)M * d;
    f32_to_bf16_kernel<<<(unsigned)std::min<int64_t>(4096, (n + 255) / 256), 256, 0, stream>>>(centroids, w.mu16, n,
                                                                                         w.keys, V);
    if (dyna_status s = check_launch("f32_to_bf16_kernel"); s != DYNA_OK) return s;
    return launch_assign(static_cast<const uint16_t*>(W), V, d, w.mu16, M, out_assign, out_score, w, stream);
}

dyna_status kmeans_update(const void* W, int32_t V, int32_t d, const int32_t* assign, int32_t M, float* centroids,
                          void* ws, hipStream_t stream) {
    const KmWs w = km_carve(V, d, M, ws);
    const uint16_t* Wb = static_cast<const uint16_t*>(W);
    const int64_t n = (int64_t)M * d;
    // the bf16 copy of kept (empty-cluster) centroids stays consistent
    f32_to_bf16_kernel<<<(unsigned)std::min<int64_t>(4096, (n + 255) / 256), 256, 0, stream>>>(centroids, w.mu16, n,
                                                                                         nullptr, 0);
    if (dyna_status s = check_launch("f32_to_bf16_kernel"); s != DYNA_OK) return s;
    return launch_update(Wb, V, d, assign, M, w, centroids, stream);
}

dyna_status kmeans_run(const void* W, int32_t V, int32_t d, int32_t M, const int32_t* init_ids, int32_t iters,
                       int32_t* out_cluster_of, float* out_centroids, void* ws, hipStream_t stream) {
    const KmWs w = km_carve(V, d, M, ws);
    const uint16_t* Wb = static_cast<const uint16_t*>(W);
    float* mu32 = out_centroids ? out_centroids : w.mu32;
    int32_t* assign = out_cluster_of ? out_cluster_of : w.assign;
    clear_word_kernel<<<1, 1, 0, stream>>>(w.bad);
    centroid_init_kernel<<<M, kKmThreads, 0, stream>>>(Wb, init_ids, V, d, mu32, w.mu16, w.keys, w.bad);
    if (dyna_status s = check_launch("centroid_init_kernel"); s != DYNA_OK) return s;
    for (int32_t it = 0; it < iters; ++it) {
        if (dyna_status s = launch_assign(Wb, V, d, w.mu16, M, assign, nullptr, w, stream); s != DYNA_OK)
            return s;
        if (dyna_status s = launch_update(Wb, V, d, assign, M, w, mu32, stream); s != DYNA_OK) return s;
    }
    int32_t bad = 0;
    if (hipMemcpyAsync(&bad, w.bad, sizeof(int32_t), hipMemcpyDeviceToHost, stream) != hipSuccess ||
        hipStreamSynchronize(stream) != hipSuccess)
        return set_error(DYNA_ERR_HIP, "k-means: device copy/synchronise failed");
    if (bad) return set_error(DYNA_ERR_DEVICE_DATA, "k-means: an initial id lies outside [0, V)");
    return DYNA_OK;
}

}  // namespace dyna
