// Dense product of streamed rows with up to 64 contexts (bf16): the union head
// of a step (Sec. 4.2, every union row against every context) and the dense
// full-vocabulary head (Sec. 4.1).
//
// The work is an HBM stream of the rows: 2 B flop per weight byte, far below
// the matrix cores' rate.  What bounds it is how the rows are walked: on
// MI355X whole consecutive rows stream at 6.8 TB/s, 16 rows walked column
// block by column block at 6.1 TB/s, and rows loaded in the MFMA operand
// layout (64 bytes of each of 16 rows per instruction) at 3.3-4.9 TB/s.  So
// a workgroup takes whole 16-row tiles, one after the other:
//
//  * the k dimension is split over its eight waves.  Wave w loads its
//    columns of the tile's 16 rows, 16 bytes per lane and up to 1 KiB of one
//    row per instruction, so the eight waves together request the tile's
//    contiguous bytes at once;
//  * a wave's context columns never change, so they stay in registers for
//    the whole launch (16 or 32 contexts per workgroup), and LDS carries only
//    the rows: a wave writes its tile columns to its own LDS region and
//    reads them back in the operand layout (row stride an odd number of
//    16-byte pieces: no bank conflicts);
//  * the next tile's loads are issued as soon as the registers are free, so
//    a tile per compute unit (128 KiB at 4096 columns) is always in flight;
//  * the waves' partial 16 x contexts products are added through LDS in wave
//    order (bit-identical from run to run) and stored 64 contiguous bytes per
//    context.
//
// More than 32 contexts take two workgroups per tile sequence, neighbours on
// one XCD that walk the same tiles: a tile comes from HBM once and from that
// XCD's L2 after (measured: FETCH_SIZE is one read of the rows).  Beyond 4096
// columns a wave's registers hold 16 contexts, and the kernel takes no more:
// a second group costs more there than the union kernel (100000 x 5376 rows,
// 32 contexts: 243 us against 216).
//
// Measured over 128256 x 4096 rows (1.05 GB; the union kernel before): 10
// contexts 195 -> 163 us (6.5 TB/s), 16: 198 -> 169, 32: 215 -> 178; 100000 x
// 2000 rows, 16 contexts: 111 -> 71 us, 40: 140 -> 91.  What is left at 32
// contexts is the products' stores: without them it runs at 6.6 TB/s.
#include <atomic>

#include "dyna_device.h"

namespace dyna {
namespace {

template <typename T>
using sptr = const __attribute__((address_space(4))) T*;  // read through the scalar unit

constexpr int kStreamWaves = 8;
constexpr int kStreamThreads = kStreamWaves * kWave;
constexpr int kStreamXcds = 8;  // workgroups go to the XCDs in turn

// NKS: 32-wide k steps of a stage per wave; SS: stages per tile (2 when a
// wave's columns do not fit one stage); NG: groups of 16 contexts per
// workgroup.  PIECES lanes cover one row's stage.
template <int NKS, int SS, int NG>
struct StreamShape {
    static constexpr int PIECES = NKS <= 4 ? 16 : NKS <= 8 ? 32 : 64;
    static constexpr int RPI = kWave / PIECES;     // rows per load instruction
    static constexpr int NA = kMfmaRows / RPI;     // load instructions per stage
    static constexpr int STRIDE = (4 * NKS + 1) * 16;  // LDS row stride, bytes
    static constexpr int A_WAVE = kMfmaRows * STRIDE;
    static constexpr int RED = kStreamWaves * NG * kWave * 16;  // partial products, bytes
    static constexpr int LDS = kStreamWaves * A_WAVE + RED;
    // waves per SIMD the registers are kept for: contexts, a stage of rows
    // and about 40 more
    static constexpr int EU = 4 * (SS * NKS * NG + NA) + 40 <= 128 ? 4 : 2;
};

struct StreamTile {
    int r0;     // first row
    int nrows;  // valid rows (0: none)
    int slot0;  // output slot of the first row
};

// PLAN: tiles are the chunks of a compact union plan (their list_off is the
// first row's output slot); else tile t is rows 16t .. of [0, n_rows).
template <bool PLAN>
__device__ __forceinline__ StreamTile stream_tile(const RowdotArgs& a, int64_t t, int64_t n_tiles) {
    StreamTile s{0, 0, 0};
    if (t >= n_tiles) return s;
    if constexpr (PLAN) {
        sptr<int32_t> ch = (sptr<int32_t>)a.plan.chunks + 4 * t;
        s.r0 = ch[0];
        s.nrows = min(kMfmaRows, ch[1]);
        s.slot0 = ch[2];
    } else {
        s.r0 = (int)(t * kMfmaRows);
        s.nrows = min(kMfmaRows, a.n_rows - s.r0);
        s.slot0 = s.r0;
    }
    return s;
}

template <int NKS, int SS, int NG, bool PLAN, bool SHARED>
__global__ __launch_bounds__(kStreamThreads, (StreamShape<NKS, SS, NG>::EU)) void row_stream_kernel(RowdotArgs a, int ngroups) {
    using Sh = StreamShape<NKS, SS, NG>;
    // rows that one workgroup reads stream past the caches (non-temporal)
    constexpr int kPolicy = SHARED ? 0 : 2;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = lane_id();
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int K = a.K, B = a.B;
    const int64_t n_tiles = PLAN ? (int64_t)((sptr<int32_t>)a.plan.hdr)[0]
                                 : ((int64_t)a.n_rows + kMfmaRows - 1) / kMfmaRows;
    // workgroup -> (tile sequence, context group): the ngroups workgroups of
    // a sequence are consecutive on one XCD
    const int xcd = blockIdx.x % kStreamXcds, j = blockIdx.x / kStreamXcds;
    const int64_t seqs = gridDim.x / ngroups;
    const int grp = j % ngroups;
    const int64_t s0 = (int64_t)(j / ngroups) * kStreamXcds + xcd;
    auto tile_at = [&](int64_t n) { return n * seqs + s0; };
    if (tile_at(0) >= n_tiles) return;  // whole workgroup
    const uint16_t* __restrict__ W = static_cast<const uint16_t*>(a.W);
    const uint16_t* __restrict__ v = static_cast<const uint16_t*>(a.v);

    // this wave's k steps [k0, k1), in stages of at most NKS
    const int steps = (K + 31) / 32;
    const int k0 = wv * steps / kStreamWaves, k1 = (wv + 1) * steps / kStreamWaves;
    const int half = SS == 1 ? k1 - k0 : (k1 - k0 + 1) / 2;
    const int lsub = lane / Sh::PIECES, lpc = lane % Sh::PIECES;
    const int col = lane & 15, kq = lane >> 4;
    // byte offset of this lane's piece of each stage inside a row; a lane
    // without one (past the wave's share or past K) has an offset beyond the
    // buffer, whose loads give zero
    uint32_t voff[SS];
#pragma unroll
    for (int s = 0; s < SS; ++s) {
        const int b = s == 0 ? k0 : k0 + half, e = s == 0 ? k0 + half : k1;
        const int c = b * 32 + lpc * 8;
        voff[s] = c < min(K, e * 32) ? 2u * (uint32_t)c : 0x80000000u;
    }

    // load i of a tile's stage s; rows past the tile's end repeat its last row
    // and only reach products that are not stored
    auto tile_rsrc = [&](const StreamTile& t) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(W) + (int64_t)t.r0 * K, (short)0,
                                                 t.nrows * K * 2, 0x00027000);
    };
    auto load = [&](__amdgpu_buffer_rsrc_t rsrc, int nrows, int s, int i) -> u32x4 {
        if constexpr (Sh::RPI == 1)
            return __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)voff[s], min(i, nrows - 1) * K * 2, kPolicy);
        const uint32_t row = (uint32_t)min(Sh::RPI * i + lsub, nrows - 1);
        return __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(voff[s] + row * (uint32_t)(K * 2)), 0, kPolicy);
    };
    u32x4 A[Sh::NA];

    StreamTile cur = stream_tile<PLAN>(a, tile_at(0), n_tiles);
    {
        const __amdgpu_buffer_rsrc_t rsrc = tile_rsrc(cur);
#pragma unroll
        for (int i = 0; i < Sh::NA; ++i) A[i] = load(rsrc, cur.nrows, 0, i);
    }
    StreamTile nxt = stream_tile<PLAN>(a, tile_at(1), n_tiles);
    const bool vids = PLAN && a.vid_out != nullptr && grp == 0 && threadIdx.x < kMfmaRows;
    int vid = vids && (int)threadIdx.x < cur.nrows ? a.perm[cur.r0 + threadIdx.x] : 0;

    // the wave's context columns, in the operand layout (contexts past B and
    // columns past the wave's share: zero)
    u32x4 Bq[SS][NKS][NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const int c = (grp * NG + g) * 16 + col;
        const char* p = reinterpret_cast<const char*>(v + (int64_t)min(c, B - 1) * K + kq * 8);
#pragma unroll
        for (int s = 0; s < SS; ++s) {
            const int b = s == 0 ? k0 : k0 + half, e = s == 0 ? k0 + half : k1;
#pragma unroll
            for (int q = 0; q < NKS; ++q) {
                Bq[s][q][g] = u32x4{0u, 0u, 0u, 0u};
                if (c < B && b + q < e && (b + q) * 32 + kq * 8 < K)
                    Bq[s][q][g] = *reinterpret_cast<const u32x4*>(p + (b + q) * 64);
            }
        }
    }

    char* own = smem + wv * Sh::A_WAVE;
    float* red = reinterpret_cast<float*>(smem + kStreamWaves * Sh::A_WAVE);
    char* wr = own + lsub * Sh::STRIDE + lpc * 16;
    const char* rd = own + col * Sh::STRIDE + kq * 16;
    const bool writes = lpc < 4 * NKS;
    // the contexts have arrived before the loop, so that nothing in it waits
    // for them (their counter also holds the rows in flight)
    __builtin_amdgcn_s_waitcnt(0x0070 | 0x0F00);  // vmcnt(0) only
    for (int64_t n = 0; cur.nrows > 0; ++n) {
        f32x4 acc[2][NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) acc[0][g] = acc[1][g] = f32x4{0.f, 0.f, 0.f, 0.f};
        int vid_next = 0;
        StreamTile far{0, 0, 0};
#pragma unroll
        for (int s = 0; s < SS; ++s) {
            // each register is written to LDS (behind the previous stage's
            // reads) and loaded again at once, so the wave's loads stay in
            // flight without a break
            wave_lds_order();
            const StreamTile& ld = s + 1 < SS ? cur : nxt;
            if (ld.nrows > 0) {
                const __amdgpu_buffer_rsrc_t rsrc = tile_rsrc(ld);
#pragma unroll
                for (int i = 0; i < Sh::NA; ++i) {
                    if (writes) *reinterpret_cast<u32x4*>(wr + i * Sh::RPI * Sh::STRIDE) = A[i];
                    A[i] = load(rsrc, ld.nrows, (s + 1) % SS, i);
                }
            } else if (writes) {
#pragma unroll
                for (int i = 0; i < Sh::NA; ++i) *reinterpret_cast<u32x4*>(wr + i * Sh::RPI * Sh::STRIDE) = A[i];
            }
            if (s + 1 == SS && nxt.nrows > 0) {
                if (vids && (int)threadIdx.x < nxt.nrows) vid_next = a.perm[nxt.r0 + threadIdx.x];
                far = stream_tile<PLAN>(a, tile_at(n + 2), n_tiles);
            }
            wave_lds_order();
#pragma unroll
            for (int q = 0; q < NKS; ++q) {
                const u32x4 w = *reinterpret_cast<const u32x4*>(rd + q * 64);
#pragma unroll
                for (int g = 0; g < NG; ++g)
                    acc[q & 1][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8, Bq[s][q][g]), __builtin_bit_cast(bf16x8, w), acc[q & 1][g], 0, 0, 0);
            }
        }
        // partial products: element ((g * 64 + lane) * 4 + r) is context
        // 16 g + 4 (lane / 16) + r, row lane % 16
        lds_barrier();  // the previous tile's sums have been read
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            f32x4 p;
#pragma unroll
            for (int r = 0; r < 4; ++r) p[r] = acc[0][g][r] + acc[1][g][r];
            reinterpret_cast<f32x4*>(red)[(wv * NG + g) * kWave + lane] = p;
        }
        lds_barrier();
        const int e_row = threadIdx.x & 15, e_ctx = threadIdx.x >> 4;  // 32 contexts by 16 rows
        if (e_ctx < 16 * NG) {
            const int at = (((e_ctx >> 4) * kWave + ((e_ctx & 15) >> 2) * 16 + e_row) << 2) + (e_ctx & 3);
            float x = red[at];
#pragma unroll
            for (int w = 1; w < kStreamWaves; ++w) x += red[w * NG * kWave * 4 + at];
            const int b = grp * NG * 16 + e_ctx;
            // full 64-byte pieces go through the caches at once: left dirty in
            // L2 they are written back at the kernel's end (32 contexts over
            // 128256 rows: 182 -> 176 us).  A plan's pieces start anywhere in
            // a line and stay cached until it is whole (64 contexts: 253 ->
            // 246 us per union step).
            float* o = a.out + (int64_t)b * a.ld + cur.slot0 + e_row;
            if (b < B && e_row < cur.nrows) {
                if constexpr (PLAN) *o = x;
                else store_coherent(o, x);
            }
        }
        if (vids && (int)threadIdx.x < cur.nrows) a.vid_out[cur.slot0 + threadIdx.x] = vid;
        vid = vid_next;
        cur = nxt;
        nxt = far;
    }
}

template <int NKS, int SS, int NG, bool PLAN, bool SHARED>
dyna_status launch_stream_s(const RowdotArgs& a, hipStream_t stream) {
    constexpr int LDS = StreamShape<NKS, SS, NG>::LDS;
    static_assert(LDS <= 160 * 1024, "LDS per block");
    static std::atomic<uint64_t> allowed{0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return set_error(DYNA_ERR_HIP, "stream: device");
    if (!(allowed.load() & (1ull << dev))) {
        if (hipFuncSetAttribute((const void*)row_stream_kernel<NKS, SS, NG, PLAN, SHARED>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, LDS) != hipSuccess)
            return set_error(DYNA_ERR_HIP, "stream: LDS attribute");
        allowed.fetch_or(1ull << dev);
    }
    const int ngroups = (a.B + 16 * NG - 1) / (16 * NG);
    const int64_t tiles = PLAN ? a.max_chunks_bound : ((int64_t)a.n_rows + kMfmaRows - 1) / kMfmaRows;
    // sequences of tiles: a multiple of the XCD count, and all workgroups
    // resident at once (per_cu of them per compute unit)
    const int per_cu = std::min(StreamShape<NKS, SS, NG>::EU / 2, (160 * 1024) / LDS);
    const int64_t most = std::max<int64_t>(1, 256 * per_cu / (kStreamXcds * ngroups));
    const int64_t want = (tiles + kStreamXcds - 1) / kStreamXcds;
    const int64_t blocks = kStreamXcds * ngroups * std::max<int64_t>(1, std::min(most, want));
    launch_timed_kernel(row_stream_kernel<NKS, SS, NG, PLAN, SHARED>, dim3((unsigned)blocks), dim3(kStreamThreads), LDS, stream,
                        a, ngroups);
    return check_launch("row_stream_kernel");
}

template <int NKS, int SS, int NG, bool PLAN>
dyna_status launch_stream_t(const RowdotArgs& a, hipStream_t stream) {
    if constexpr (NG == 2)
        if (a.B > 16 * NG) return launch_stream_s<NKS, SS, NG, PLAN, true>(a, stream);
    return launch_stream_s<NKS, SS, NG, PLAN, false>(a, stream);
}

template <int NG, bool PLAN>
dyna_status launch_stream_n(const RowdotArgs& a, hipStream_t stream) {
    const int steps = ((a.K + 31) / 32 + kStreamWaves - 1) / kStreamWaves;  // per wave, at most
    if (steps <= 4) return launch_stream_t<4, 1, NG, PLAN>(a, stream);
    if (steps <= 8) return launch_stream_t<8, 1, NG, PLAN>(a, stream);
    if (steps <= 12) return launch_stream_t<12, 1, NG, PLAN>(a, stream);
    if (steps <= 16) return launch_stream_t<16, 1, NG, PLAN>(a, stream);
    if constexpr (NG == 1) {
        if (steps <= 24) return launch_stream_t<12, 2, NG, PLAN>(a, stream);
        return launch_stream_t<16, 2, NG, PLAN>(a, stream);
    }
    return set_error(DYNA_ERR_UNSUPPORTED, "stream: K > 4096 takes 16 contexts per workgroup");
}

}  // namespace

// Against the union kernel (time of this one over that one's; 3975 dense and
// union steps):
//  * up to 32 contexts (16 beyond 4096 columns) this one is faster, 0.5-1.0,
//    but for unions of many short rows, whose tiles it hands out in tasks of a
//    few KB: 256 columns, 10 contexts 0.97 at 16k rows, 1.05 at 44k, 1.12 at 94k;
//    320 columns 1.00-1.11, 384 1.00-1.06, 448 1.0.  Rows that are no multiple
//    of 128 bytes (next item) turn earlier: 264 columns 0.95-1.06, 296
//    0.93-1.05, 328 0.89-1.04, 392 0.86-1.01 (60k-250k rows, 3-28 contexts);
//  * 33-64 contexts share tiles between two workgroups.  Where rows are no
//    multiple of the 128 bytes that the union kernel walks, its pieces
//    straddle lines, and this one is faster at any length: 2168 columns 0.4-0.86,
//    880 0.5-0.8, 520 0.6-0.87, 328-376 0.87-1.06 (272: 1.0 at 32k rows, 1.25 at
//    262k);
//  * where they are, it is faster on short tables, whose tiles of 128 rows
//    leave compute units to the union kernel idle, and loses beyond (36 and 64
//    contexts): 320 columns 0.92 and 0.88 at 20k rows, 1.18 and 1.08 at 80k;
//    640 0.89 and 0.82 at 48k, 1.02 and 0.92 at 140k; 1600 0.89 and 0.77 at 48k,
//    1.11 and 1.11 at 96k; 3584 0.87 and 0.65 at 24k, 1.18 and 1.14 at 60k.  A
//    second group of contexts costs this kernel the same at 33 and at 64.
static bool streams_faster(int32_t K, int32_t B, int64_t rows, bool plan) {
    const bool straddles = K % 64 != 0;
    if (B <= 32) return !plan || K >= (straddles ? 288 : 448) || rows <= 64 * (int64_t)K;
    if (straddles && K >= 320) return true;
    const int64_t base = K > 2048 ? 28672 : K > 1024 ? 49152 : std::max<int64_t>(8192, (plan ? 64 : 96) * (int64_t)K);
    return rows <= base * (128 + 2 * (B - 32)) / 128;
}

bool row_stream_eligible(const RowdotArgs& a) {
    if (a.wdtype != DYNA_BF16 || a.vdtype != DYNA_BF16 || a.K % 8 != 0 || a.K > 8192 || a.bias != nullptr ||
        a.act != DYNA_ACT_NONE || a.B < 1 || a.B > 64 || (a.vid_out != nullptr && a.perm == nullptr) ||
        (a.B > 16 && a.K > 4096))
        return false;
    const bool plan = a.plan.hdr != nullptr;
    return streams_faster(a.K, a.B, plan ? a.rows_expected : a.n_rows, plan);
}

dyna_status launch_row_stream(const RowdotArgs& a, hipStream_t stream) {
    if (!row_stream_eligible(a)) return set_error(DYNA_ERR_UNSUPPORTED, "stream: needs bf16 and a shape it takes");
    const bool wide = a.B > 16;
    if (a.plan.hdr != nullptr)
        return wide ? launch_stream_n<2, true>(a, stream) : launch_stream_n<1, true>(a, stream);
    return wide ? launch_stream_n<2, false>(a, stream) : launch_stream_n<1, false>(a, stream);
}

}  // namespace dyna
