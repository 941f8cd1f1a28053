// Integer GEMM for few output tiles: small output tiles, the reduction split
// over the waves of a workgroup.
//
// The 256 x 256 and 128 x 256 tiles of the large-batch GEMM leave most of
// the chip idle when n or d_out is small (a decode step through a
// 4096 -> 4096 projection is 16 such tiles), and every one of them walks all
// of d_in alone.  Here a workgroup owns a tile of 16 A tokens by 16 B
// outputs and its 8 waves take every eighth 64-byte chunk of the rows, so a
// tile is read by 8 waves at once and the chip holds many tiles.  The waves'
// int32 partial sums meet in LDS; integer sums do not depend on the order,
// so the results equal the large-tile kernel's bit for bit.
//
// Each wave streams its chunks through an LDS ring of its own (D stages of
// A + B copies of 1 KiB, global_load_lds_dwordx4), so the main loop has no
// barriers: a wave waits for its own copies (vmcnt), reads a chunk's
// fragments, refills the stage and multiplies.  Copies go through LDS
// because the MFMA layout wants consecutive lanes on different rows: loading
// fragments straight into registers that way ran at 14 bytes per clock and
// CU, with four consecutive lanes on 64 contiguous bytes it is 25 or more
// (257 x 14336 -> 4096: 33 us against 22 us).  A lane's 16 bytes are 32
// packed INT4 codes (two v_mfma_i32_16x16x64_i8, widened in registers to
// 16 * code as in the large-tile kernel) or 16 int8 codes (one).  Both
// operands are read the same way, so the index pairs match (a permutation of
// the reduction index).
//
// Bound by the operand stream of a CU (A + B KiB per chunk for A B MFMA
// tiles), at the smallest sizes by HBM.  Kernel times against the large
// tiles, back-to-back calls, weights in the last-level cache:
//   n x d_in -> d_out          large tiles    split    tile
//   1 x 4096 -> 4096           32.0 us         4.1 us  16 x 16
//   48 x 4096 -> 14336         33.8 us         7.3 us  48 x 64
//   257 x 14336 -> 4096        90.2 us        22.4 us  80 x 64
//   1000 x 14336 -> 4096       94.1 us        62.2 us  128 x 64
//   100 x 4096 -> 14336, int8  48.6 us        18.1 us  128 x 64
#include "device_common.h"
#include "kernels.h"

namespace catk {

constexpr int kSpWaves = 8;
constexpr int kSpThreads = kSpWaves * kWave;
constexpr int kSpChunk = 64;               // bytes of a row per chunk
constexpr int kSpXcd = 8;

// Position swizzle of a row's four 16-byte units: 16 rows at one unit, and 8
// rows at units q and q ^ 2, fall on distinct 16-byte bank groups.
__device__ __forceinline__ int sp_swz(int row) { return (row >> 2) & 3; }

// Waits until at most N of this wave's copies are in flight; LDS reads stay
// behind it.
template <int N>
__device__ __forceinline__ void sp_wait_copies() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0)" ::"i"(N) : "memory");
}
// Waits for this wave's LDS reads.
__device__ __forceinline__ void sp_wait_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

__device__ __forceinline__ i32x4 sp_widen(u32x4 v, int half) {
    const uint32_t w0 = v[2 * half], w1 = v[2 * half + 1];
    return i32x4{static_cast<int>(unpack_lo16(w0)), static_cast<int>(unpack_hi16(w0)),
                 static_cast<int>(unpack_lo16(w1)), static_cast<int>(unpack_hi16(w1))};
}

template <bool I8, bool ASYM, int A, int B, int D>
__global__ __launch_bounds__(kSpThreads) void split_gemm_kernel(
    const uint8_t* __restrict__ qx, const float* __restrict__ s_x,
    const uint8_t* __restrict__ qw, const float* __restrict__ s_w, int64_t n, int64_t d_in,
    int64_t d_out, float* __restrict__ y, int32_t* __restrict__ acc_out,
    const float* __restrict__ zmin_x, const int32_t* __restrict__ rsum_w) {
    static_assert(!(I8 && ASYM), "asymmetric codes are INT4");
    constexpr int BM = 16 * A, BN = 16 * B;
    static_assert(BM + BN <= kSpThreads, "one thread per row and output scale");
    constexpr int L = A + B;               // 1 KiB copies per chunk
    static_assert(L * D < 64, "copies in flight must fit the vmcnt range");
    // accumulator tiles reduced per round: 8 waves x RT KiB of LDS
    constexpr int RT = A * B < 8 ? A * B : 8;
    constexpr int ROUNDS = (A * B + RT - 1) / RT;
    constexpr int UNITS = (D * L > RT ? D * L : RT) * kWave;
    __shared__ __attribute__((aligned(16))) u32x4 lds[kSpWaves][UNITS];
    __shared__ float scale[BM + BN];
    __shared__ uint32_t extra[ASYM ? BM + BN : 1];

    // XCD x walks one contiguous range of tiles, the row tiles of a column
    // panel next to each other: its weights then enter that XCD's L2 once
    const int64_t tiles_m = (n + BM - 1) / BM;
    const int64_t tiles_n = (d_out + BN - 1) / BN;
    const int64_t T = tiles_m * tiles_n;
    const int64_t per_xcd = (T + kSpXcd - 1) / kSpXcd;
    const int64_t tau = (blockIdx.x % kSpXcd) * per_xcd + blockIdx.x / kSpXcd;
    if (tau >= T) return;
    const int64_t m0 = (tau % tiles_m) * BM;
    const int64_t n0 = (tau / tiles_m) * BN;

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int l16 = lane & 15, q4 = lane >> 4;
    const uint32_t rb = static_cast<uint32_t>(I8 ? d_in : d_in / 2);
    const int nk = static_cast<int>((rb + kSpChunk - 1) / kSpChunk);
    const int rows_a = static_cast<int>(n - m0 < BM ? n - m0 : BM);
    const int rows_b = static_cast<int>(d_out - n0 < BN ? d_out - n0 : BN);
    // this thread's scale (rows first, then outputs), read now and put in
    // LDS after the main loop
    float sc = 0.0f;
    uint32_t ex = 0;
    if (tid < BM) {
        const int64_t t = m0 + tid < n ? m0 + tid : n - 1;
        sc = s_x[t];
        if constexpr (ASYM) ex = __float_as_uint(zmin_x[t]);
    } else if (tid < BM + BN) {
        const int64_t o = n0 + tid - BM < d_out ? n0 + tid - BM : d_out - 1;
        sc = s_w[o];
        if constexpr (ASYM) ex = static_cast<uint32_t>(rsum_w[o]);
    }

    // Copy g of a chunk (g < A: 16 token rows, else 16 output rows) fills 64
    // slots: slot s holds row s / 4, unit (s % 4) ^ swz(row).  Four
    // consecutive lanes read 64 contiguous bytes.  Rows past the end of a
    // matrix read its last row (their outputs are never stored).
    const int cr = lane >> 2;
    const uint32_t cu = 16u * static_cast<uint32_t>((lane & 3) ^ sp_swz(cr));
    uint32_t src[L];
#pragma unroll
    for (int g = 0; g < L; ++g) {
        const int r = 16 * (g < A ? g : g - A) + cr;
        const int last = (g < A ? rows_a : rows_b) - 1;
        src[g] = static_cast<uint32_t>(r < last ? r : last) * rb;
    }
    const uint8_t* const base_a = qx + m0 * rb;
    const uint8_t* const base_b = qw + n0 * rb;
    const uint32_t ring = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(lds_addr(&lds[wave][0])));
    auto issue = [&](int chunk, int st) {
        uint32_t col = static_cast<uint32_t>(chunk) * kSpChunk + cu;
        col = col < rb ? col : 0;          // past the row's end: any unit of it
#pragma unroll
        for (int g = 0; g < L; ++g)
            dma16(g < A ? base_a : base_b, src[g] + col, ring + static_cast<uint32_t>((st * L + g) * 1024));
    };
    u32x4 fa[A], fb[B];
    const int slot = l16 * 4 + (q4 ^ sp_swz(l16));
    auto read = [&](int st) {
#pragma unroll
        for (int b = 0; b < B; ++b) fb[b] = lds[wave][(st * L + A + b) * kWave + slot];
#pragma unroll
        for (int a = 0; a < A; ++a) fa[a] = lds[wave][(st * L + a) * kWave + slot];
    };
    i32x4 acc[A][B];
#pragma unroll
    for (int a = 0; a < A; ++a)
#pragma unroll
        for (int b = 0; b < B; ++b) acc[a][b] = i32x4{0, 0, 0, 0};
    auto compute = [&](int chunk) {
        if (static_cast<uint32_t>(chunk + 1) * kSpChunk > rb) {
            // ragged last chunk: units past the row's end are zeros in A
            const bool past = static_cast<uint32_t>(chunk) * kSpChunk + 16u * static_cast<uint32_t>(q4) >= rb;
#pragma unroll
            for (int a = 0; a < A; ++a) fa[a] = past ? u32x4{0u, 0u, 0u, 0u} : fa[a];
        }
#pragma unroll
        for (int half = 0; half < (I8 ? 1 : 2); ++half) {
            i32x4 wb[B];
#pragma unroll
            for (int b = 0; b < B; ++b)
                wb[b] = I8 ? __builtin_bit_cast(i32x4, fb[b]) : sp_widen(fb[b], half);
#pragma unroll
            for (int a = 0; a < A; ++a) {
                const i32x4 wa = I8 ? __builtin_bit_cast(i32x4, fa[a]) : sp_widen(fa[a], half);
#pragma unroll
                for (int b = 0; b < B; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wa, wb[b], acc[a][b], 0, 0, 0);
            }
        }
    };
    // wave w takes chunks w, w + 8, ...: cnt of them through a ring of D
    // stages of its own; no other wave touches it, so no barriers.  A stage
    // is refilled once its fragments are in registers.
    const int cnt = nk > wave ? (nk - wave + kSpWaves - 1) / kSpWaves : 0;
#pragma unroll
    for (int s = 0; s < D; ++s)
        if (s < cnt) issue(wave + s * kSpWaves, s);
    int i = 0, st = 0;
    for (; i + D < cnt; ++i) {
        sp_wait_copies<(D - 1) * L>();
        read(st);
        sp_wait_reads();
        issue(wave + (i + D) * kSpWaves, st);
        compute(wave + i * kSpWaves);
        st = st + 1 == D ? 0 : st + 1;
    }
    sp_wait_copies<0>();
    for (; i < cnt; ++i) {
        read(st);
        compute(wave + i * kSpWaves);
        st = st + 1 == D ? 0 : st + 1;
    }

    if (tid < BM + BN) {
        scale[tid] = sc;
        if constexpr (ASYM) extra[tid] = ex;
    }
    // partial sums, RT accumulator tiles per round: slot (tile, lane) holds
    // the lane's 4 rows of one output column
    constexpr int kShift = I8 ? 0 : 8;
#pragma unroll
    for (int rd = 0; rd < ROUNDS; ++rd) {
        __syncthreads();     // the ring (or the last round) is read
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            const int tl = rd * RT + i;
            if (tl < A * B) lds[wave][i * kWave + lane] = __builtin_bit_cast(u32x4, acc[tl / B][tl % B]);
        }
        __syncthreads();
        // RT <= 8 tiles, 8 waves: wave i sums tile rd * RT + i
        const int tl = rd * RT + wave;
        if (wave < RT && tl < A * B) {
            i32x4 v = __builtin_bit_cast(i32x4, lds[0][wave * kWave + lane]);
#pragma unroll
            for (int w = 1; w < kSpWaves; ++w) {
                const i32x4 p = __builtin_bit_cast(i32x4, lds[w][wave * kWave + lane]);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] += p[e];
            }
            const int row = (tl / B) * 16 + 4 * q4;
            const int col = (tl % B) * 16 + l16;
            if (col < rows_b) {
                const float sw = scale[BM + col];
                const int rs = ASYM ? static_cast<int>(extra[BM + col]) : 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (row + e >= rows_a) continue;
                    const int64_t off = (m0 + row + e) * d_out + n0 + col;
                    int a = v[e] >> kShift;
                    float yv;
                    if constexpr (ASYM) {
                        a += 8 * rs;
                        const float t1 = static_cast<float>(a) * scale[row + e];
                        const float t2 = __uint_as_float(extra[row + e]) * static_cast<float>(rs);
                        yv = (t1 + t2) * sw;
                    } else {
                        yv = (static_cast<float>(a) * scale[row + e]) * sw;
                    }
                    y[off] = yv;
                    if (acc_out) acc_out[off] = a;
                }
            }
        }
    }
}

// ---------------------------------------------------------------- dispatch
// Tile shapes (tokens / 16, outputs / 16, ring stages).  Stages: as many as
// keep 24-64 KiB of copies in flight per CU; more measured the same.
struct SpTile {
    int a, b;
};
#define CAT_SPLIT_TILES(V) \
    V(0, 1, 1, 4) V(1, 1, 2, 4) V(2, 2, 2, 2) V(3, 4, 2, 3) V(4, 2, 4, 3) V(5, 3, 4, 1) V(6, 4, 4, 1) \
    V(7, 5, 4, 1) V(8, 6, 4, 1) V(9, 8, 4, 1)
#define CAT_SPLIT_AB(id, A, B, D) {A, B},
static constexpr SpTile kSpTiles[] = {CAT_SPLIT_TILES(CAT_SPLIT_AB)};
#undef CAT_SPLIT_AB
constexpr int kSpTileCount = sizeof(kSpTiles) / sizeof(kSpTiles[0]);

static int64_t sp_tiles(int64_t n, int64_t d_out, const SpTile& t) {
    return ((n + 16 * t.a - 1) / (16 * t.a)) * ((d_out + 16 * t.b - 1) / (16 * t.b));
}

// A launch covers fewer than 2^32 threads.
constexpr int64_t kSpMaxTiles = int64_t{1} << 22;
// Beyond four tiles per CU the large tiles' lower operand traffic wins: 1228
// x 13856 -> 8120 (5 rounds of 128 x 64) took 184 us against 166, 3132 x
// 13312 -> 5320 (9 rounds) 311 against 282.
constexpr int64_t kSpMaxRounds = 4;

// Estimated clocks of the best tile shape (the largest value if none fits).
// A CU takes ceil(tiles / CUs) tiles.  Per 64-byte chunk a tile costs 36
// clocks per KiB copied (28 bytes per clock and CU) and the part of its MFMAs
// that does not hide behind the copies (6 clocks per 16 x 16 pair of packed
// chunks, 3 for int8); per tile it costs a fixed part and the reduction and
// stores, 340 clocks per 16 x 16 outputs.  Fitted to measured times over n =
// 1 .. 2700, d_in = 32 .. 14336 and d_out = 512 .. 16384.
int64_t split_gemm_cost(bool i8, int64_t n, int64_t d_in, int64_t d_out, int64_t cus, int& tile) {
    const int64_t nk = ((i8 ? d_in : d_in / 2) + kSpChunk - 1) / kSpChunk;
    int64_t best = INT64_MAX;
    for (int v = 0; v < kSpTileCount; ++v) {
        const SpTile t = kSpTiles[v];
        const int64_t tiles = sp_tiles(n, d_out, t);
        if (tiles > kSpMaxTiles) continue;
        const int64_t rounds = (tiles + cus - 1) / cus;
        if (rounds > kSpMaxRounds) continue;
        const int64_t ab = t.a * t.b;
        const int64_t cost = rounds * (nk * (36 * (t.a + t.b) + (i8 ? 3 : 6) * ab) + 600 + 340 * ab);
        if (cost < best) {
            best = cost;
            tile = v;
        }
    }
    return best;
}

template <bool I8, bool ASYM>
static hipError_t split_launch(int tile, const uint8_t* codes_x, const float* s_x,
                               const uint8_t* codes_w, const float* s_w, int64_t n, int64_t d_in,
                               int64_t d_out, float* y, int32_t* acc_out, const float* zmin_x,
                               const int32_t* rsum_w, hipStream_t stream) {
    const int64_t T = sp_tiles(n, d_out, kSpTiles[tile]);
    const dim3 grid(static_cast<uint32_t>((T + kSpXcd - 1) / kSpXcd * kSpXcd)), block(kSpThreads);
    switch (tile) {
#define CAT_SPLIT_CASE(id, A, B, D)                                                                \
    case id:                                                                                       \
        hipLaunchKernelGGL((split_gemm_kernel<I8, ASYM, A, B, D>), grid, block, 0, stream,         \
                           codes_x, s_x, codes_w, s_w, n, d_in, d_out, y, acc_out, zmin_x, rsum_w); \
        break;
        CAT_SPLIT_TILES(CAT_SPLIT_CASE)
#undef CAT_SPLIT_CASE
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_split_gemm(int tile, bool i8, const uint8_t* codes_x, const float* s_x,
                             const uint8_t* codes_w, const float* s_w, int64_t n, int64_t d_in,
                             int64_t d_out, float* y, int32_t* acc_out, const float* zmin_x,
                             const int32_t* rsum_w, hipStream_t stream) {
    if (zmin_x)
        return split_launch<false, true>(tile, codes_x, s_x, codes_w, s_w, n, d_in, d_out, y,
                                         acc_out, zmin_x, rsum_w, stream);
    if (i8)
        return split_launch<true, false>(tile, codes_x, s_x, codes_w, s_w, n, d_in, d_out, y,
                                         acc_out, nullptr, nullptr, stream);
    return split_launch<false, false>(tile, codes_x, s_x, codes_w, s_w, n, d_in, d_out, y, acc_out,
                                      nullptr, nullptr, stream);
}

}  // namespace catk
