// Nearest centroid of every row (the k-means assignment, Sec. 4.2 "Vocabulary
// partition"): a dense V x M x d bf16 product on the matrix cores whose
// results are reduced to one argmax per row and never stored.
//
// The product is bound by the matrix cores, and next by LDS: an operand piece
// read from LDS has to feed many products.  Four waves of a workgroup, one
// per SIMD, each hold a 128 x 128 block of fp32 products in registers (the
// workgroup's tile is 256 rows by 256 centroids), so a k step of 16 reads 8
// operand pieces for 16 v_mfma_f32_32x32x16_bf16: 75% of the LDS rate at the
// matrix cores' full rate, where the eight-wave 32 x 256 blocks used before
// asked for 112%.
//
//  * A stage is 64 columns of the tile's rows and centroids (32 KiB each,
//    loaded straight to LDS).  The 160 KiB hold three stages of rows, which
//    come from HBM and are loaded two stages ahead, and two of centroids,
//    which L2 serves and which are loaded one stage ahead.
//  * The operand pieces of the next k step are read while the current one's
//    products run; the last step of a stage runs after the barrier that
//    starts the next stage, so its products cover that stage's first reads.
//  * The centroids are the left operand: a lane then holds 64 centroids of
//    one row per 32-row block, and the argmax is almost entirely inside the
//    lane.  Tiles of one row block (one per 256 centroids) run side by side
//    on one XCD, so the rows come from HBM once; the tiles' winners meet in
//    one 64-bit maximum per row, (value, lower id), whose result does not
//    depend on the order.
//
// Measured, 128256 x 4096 rows against 1024 centroids (1.08 TFLOP), by card:
// 1292 -> 835-863 us on rows with cluster structure (1.25-1.29 PFLOP/s) and
// 1349-1419 -> 864-968 us on random ones; a library GEMM of this shape, which
// also writes its 263 MB result, 936 us.  Steps on the
// way (random rows): both operands two stages deep 1118 us, three stages of
// rows 1047, loads between the products 1017, reads between them too 1002.
// Without the loads the products alone take 790 us.
#include <atomic>

#include "dyna_device.h"

namespace dyna {
namespace {

typedef __attribute__((address_space(3))) void* lds_ptr;
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kAsThreads = 256;
constexpr int kAsWaves = kAsThreads / kWave;
constexpr int kAsKB = 64;               // columns of a stage
constexpr int kAsRowB = kAsKB * 2;      // bytes of a row's stage
constexpr int kAsSteps = kAsKB / 16;    // MFMA k steps of a stage
constexpr int kAsRing = 3;              // stages of rows in LDS (and two of centroids)
constexpr int kAsXcds = 8;              // workgroups go to the XCDs in turn

// 16 bytes per lane straight to LDS at dst + 16 * lane.
__device__ __forceinline__ void load_lds16(__amdgpu_buffer_rsrc_t rsrc, char* dst, uint32_t voff, int soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr)dst, 16, (int)voff, soff, 0, 0);
}

struct AssignArgs {
    const uint16_t* W;   // [V, K] rows
    const uint16_t* mu;  // [M, K] centroids
    int32_t V, K, M;
    unsigned long long* keys;  // [V] running maxima of (value, ~id)
};

// A tile: rows [r0, r0 + nr), centroids [c0, c0 + nc).
struct AsTile {
    int r0, nr, c0, nc;
};

// F: 32-wide blocks of rows and of centroids per wave (tile side 64 F).
template <int F>
__global__ __launch_bounds__(kAsThreads, 1) void nearest_centroid_kernel(AssignArgs a) {
    constexpr int SIDE = 64 * F;
    constexpr int HALF = SIDE * kAsRowB;     // bytes of the rows (or centroids) of a stage
    constexpr int NI = SIDE / 8 / kAsWaves;  // loads per wave, stage and operand (8 rows each)
    static_assert(NI % 2 == 0, "the slot rule takes a load's parity");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = lane_id();
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wc = wv & 1, wr = wv >> 1;     // this wave's half of the centroids and of the rows
    const int K = a.K;
    const int nkb = (K + kAsKB - 1) / kAsKB;

    // tiles of this workgroup: row blocks go round the XCDs, and an XCD's
    // workgroups take the centroid groups of a row block side by side
    const int nrb = (a.V + SIDE - 1) / SIDE, ng = (a.M + SIDE - 1) / SIDE;
    const int xcd = blockIdx.x % kAsXcds, per = gridDim.x / kAsXcds;
    const int64_t n_tiles = (int64_t)((nrb - xcd + kAsXcds - 1) / kAsXcds) * ng;
    auto tile_of = [&](int64_t t) {
        AsTile s;
        s.r0 = ((int)(t / ng) * kAsXcds + xcd) * SIDE;
        s.c0 = (int)(t % ng) * SIDE;
        s.nr = min(SIDE, a.V - s.r0);
        s.nc = min(SIDE, a.M - s.c0);
        return s;
    };
    const int64_t t0 = blockIdx.x / kAsXcds;
    if (t0 >= n_tiles) return;  // whole workgroup

    // issue side: a wave instruction loads 8 rows of 128 bytes; lane l takes
    // row l / 8, and LDS slot l % 8 of a row holds its piece
    // slot ^ (row / 2 % 8): the 16 rows that an operand read touches at once
    // then lie in 16 different 16-byte slots of the 256 bytes of LDS banks
    const int sub = lane >> 3;
    auto piece = [&](int i) { return (lane & 7) ^ (sub >> 1) ^ (4 * (i & 1)); };
    // One operand's stages in the order they are consumed.  Rows past the end
    // repeat the last one (their products are not used).
    struct Feed {
        int64_t t;  // tile and k block of the next stage
        int kb;
        uint32_t off[NI];
        const uint16_t* base;
        int n;  // valid rows
    };
    auto aim = [&](Feed& f, const uint16_t* base, int n) {
        f.base = base;
        f.n = n;
#pragma unroll
        for (int i = 0; i < NI; ++i)
            f.off[i] = (uint32_t)(min((wv * NI + i) * 8 + sub, n - 1) * K + piece(i) * 8) * 2u;
    };
    auto aim_rows = [&](Feed& f) {
        const AsTile s = tile_of(f.t);
        aim(f, a.W + (int64_t)s.r0 * K, s.nr);
    };
    auto aim_centroids = [&](Feed& f) {
        const AsTile s = tile_of(f.t);
        aim(f, a.mu + (int64_t)s.c0 * K, s.nc);
    };
    // load i of the next stage of f; past the last tile nothing is read
    auto issue = [&](const Feed& f, char* stage, int i) {
        const bool out = f.kb * kAsKB + piece(i) * 8 >= K || f.t >= n_tiles;
        // pieces past K are beyond the buffer: zero in both operands
        load_lds16(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(f.base), (short)0, f.n * K * 2, 0x00027000),
                   stage + (wv * NI + i) * 1024, f.off[i] | (out ? 0x80000000u : 0u), f.kb * kAsRowB);
    };
    // moves f to its next stage; true at another tile
    auto advance = [&](Feed& f) -> bool {
        if (++f.kb < nkb) return false;
        f.kb = 0;
        f.t += per;
        return f.t < n_tiles;
    };

    // consume side: operand pieces of k step s; a lane holds row (lane % 32)
    // of a block, columns 16 s + 8 (lane / 32) ..
    const int r32 = lane & 31, kh = lane >> 5;
    int xb = 0, cb = 0;  // ring places of the current stage
    u32x4 xf[2][F], cf[2][F];
    // piece p < 2F of k step s of the current stage into operand set `set`
    auto fetch = [&](int s, int set, int p) {
        const int at = ((2 * s + kh) ^ ((r32 >> 1) & 7)) * 16;
        if (p < F)
            cf[set][p] = *reinterpret_cast<const u32x4*>(smem + (kAsRing + cb) * HALF +
                                                         (wc * 32 * F + p * 32 + r32) * kAsRowB + at);
        else
            xf[set][p - F] = *reinterpret_cast<const u32x4*>(smem + xb * HALF +
                                                             (wr * 32 * F + (p - F) * 32 + r32) * kAsRowB + at);
    };
    f32x16 acc[F][F];  // [centroid block][row block]
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
            for (int j = 0; j < F; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    };
    auto product = [&](int set, int i, int j) {
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, cf[set][i]),
                                                            __builtin_bit_cast(bf16x8, xf[set][j]), acc[i][j], 0, 0, 0);
    };
    // The products of operand set `set`, and between them the reads of k step
    // `s` into the other set (s < 0: none) and, at the start of a stage, the
    // next stages' loads, so that the matrix cores do not wait for the issue
    // of either.  (The order is pinned; left alone, the compiler sinks the
    // reads to their uses.)
    auto step = [&](int set, int s, auto&& between) {
#pragma unroll
        for (int m = 0; m < F * F; ++m) {
            if (s >= 0 && m % (F / 2) == 0) fetch(s, set ^ 1, m / (F / 2));
            between(m);
            product(set, m / F, m % F);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto nothing = [](int) {};
    // best (value, lower id) of every row of the tile over its centroids
    auto settle = [&](const AsTile& t) {
        const int cbase = wc * 32 * F + 4 * kh;
#pragma unroll
        for (int j = 0; j < F; ++j) {
            float best = -__builtin_inff();
            int id = cbase;
#pragma unroll
            for (int i = 0; i < F; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    // ascending ids, strictly larger values: ties (and NaN,
                    // which is never larger) leave the lower id
                    const int c = cbase + 32 * i + 8 * (r >> 2) + (r & 3);
                    const bool gt = acc[i][j][r] > best && c < t.nc;
                    best = gt ? acc[i][j][r] : best;
                    id = gt ? c : id;
                }
            // a lane whose centroids all lie past the end reports none
            uint64_t key = cbase < t.nc ? sel_key(best, (uint32_t)(t.c0 + id)) : 0;
            const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute((lane ^ 32) << 2, (int)(uint32_t)key);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute((lane ^ 32) << 2, (int)(uint32_t)(key >> 32));
            const uint64_t other = ((uint64_t)hi << 32) | lo;
            key = other > key ? other : key;
            const int row = wr * 32 * F + 32 * j + r32;
            if (kh == 0 && row < t.nr && key != 0) atomicMax(a.keys + t.r0 + row, (unsigned long long)key);
        }
    };

    Feed fx, fc;
    fx.t = fc.t = t0;
    fx.kb = fc.kb = 0;
    aim_rows(fx);
    aim_centroids(fc);
    int xi = 0, ci = 0;  // ring places of the next stages to load
    auto next_rows = [&]() {
        if (advance(fx)) aim_rows(fx);
        xi = xi + 1 == kAsRing ? 0 : xi + 1;
    };
    auto next_centroids = [&]() {
        if (advance(fc)) aim_centroids(fc);
        ci ^= 1;
    };
    auto xdst = [&]() { return smem + xi * HALF; };
    auto cdst = [&]() { return smem + (kAsRing + ci) * HALF; };
#pragma unroll
    for (int i = 0; i < NI; ++i) issue(fx, xdst(), i);
    next_rows();
#pragma unroll
    for (int i = 0; i < NI; ++i) issue(fc, cdst(), i);
    next_centroids();
#pragma unroll
    for (int i = 0; i < NI; ++i) issue(fx, xdst(), i);  // the next stage's rows, behind this one's
    next_rows();
    clear();
    for (int64_t t = t0; t < n_tiles; t += per) {
        for (int kb = 0; kb < nkb; ++kb) {
            // this stage has arrived (every wave's loads; only the next one's
            // rows may be missing), and every wave has read the last piece of
            // the stage before it
            stage_barrier<NI>();
            if (kb > 0) {
                // the last k step of the stage before
                step(1, 0, [&](int m) {
                    constexpr int PER = (2 * NI + F * F - 1) / (F * F);
#pragma unroll
                    for (int i = m * PER; i < (m + 1) * PER && i < 2 * NI; ++i) {
                        if (i < NI) issue(fc, cdst(), i);
                        else issue(fx, xdst(), i - NI);
                    }
                });
            } else {
#pragma unroll
                for (int p = 0; p < 2 * F; ++p) fetch(0, 0, p);
#pragma unroll
                for (int i = 0; i < NI; ++i) issue(fc, cdst(), i);
#pragma unroll
                for (int i = 0; i < NI; ++i) issue(fx, xdst(), i);
            }
            next_centroids();
            next_rows();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 1; s < kAsSteps; ++s) step((s & 1) ^ 1, s, nothing);
            xb = xb + 1 == kAsRing ? 0 : xb + 1;
            cb ^= 1;
        }
        step(1, -1, nothing);
        settle(tile_of(t));
        clear();
    }
}

// assign[v], score[v] (optional) from the rows' maxima, which are left at 0
// for the next assignment.
__global__ __launch_bounds__(256) void assign_finish_kernel(unsigned long long* __restrict__ keys, int32_t V,
                                                            int32_t* __restrict__ assign, float* __restrict__ score) {
    const int64_t v = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (v >= V) return;
    const uint64_t key = keys[v];
    keys[v] = 0;
    assign[v] = (int32_t)key_id(key);
    if (score != nullptr) score[v] = key_val(key);
}

template <int F>
dyna_status launch_nearest_f(const AssignArgs& a, hipStream_t stream) {
    constexpr int LDS = (kAsRing + 2) * 64 * F * kAsRowB;
    static_assert(LDS <= 160 * 1024, "LDS per block");
    static std::atomic<uint64_t> allowed{0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return set_error(DYNA_ERR_HIP, "assign: device");
    if (!(allowed.load() & (1ull << dev))) {
        if (hipFuncSetAttribute((const void*)nearest_centroid_kernel<F>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                LDS) != hipSuccess)
            return set_error(DYNA_ERR_HIP, "assign: LDS attribute");
        allowed.fetch_or(1ull << dev);
    }
    launch_timed_kernel(nearest_centroid_kernel<F>, dim3(F == 4 ? 256 : 512), dim3(kAsThreads), LDS, stream, a);
    return check_launch("nearest_centroid_kernel");
}

}  // namespace

dyna_status launch_nearest_centroid(const void* W, int32_t V, int32_t d, const uint16_t* mu, int32_t M,
                                    unsigned long long* keys, int32_t* assign, float* score, hipStream_t stream) {
    const AssignArgs a{static_cast<const uint16_t*>(W), mu, V, d, M, keys};
    // 128 x 128 tiles (two workgroups per compute unit) where 256 x 256 ones
    // would leave compute units idle: 20000 x 1024 rows and 300 centroids 85
    // us before, 22 with them; 8192 x 256 and 64: 21 and 8
    const int64_t tiles = (((int64_t)V + 255) / 256) * (((int64_t)M + 255) / 256);
    const dyna_status st = tiles >= 256 ? launch_nearest_f<4>(a, stream) : launch_nearest_f<2>(a, stream);
    if (st != DYNA_OK) return st;
    assign_finish_kernel<<<(unsigned)(((int64_t)V + 255) / 256), 256, 0, stream>>>(keys, V, assign, score);
    return check_launch("assign_finish_kernel");
}

}  // namespace dyna
