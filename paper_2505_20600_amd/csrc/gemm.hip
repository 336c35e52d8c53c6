// Row GEMMs of the block over the packed masked rows only (Table 1: the
// projections and the feed-forward scale with the masked-row count):
//
//     out[m][n] = epilogue( sum_k A[m][k] * W[n][k] + bias[n] )
//
// Both operands are K-contiguous (activations [M][K], Linear weights
// [N][K]), the native operand layout of the CDNA4 matrix cores. The weight
// tile is the MFMA "A" operand and the activation tile the "B" operand, so
// each lane ends up with four consecutive output columns of one row; the
// tile is restaged through LDS so that consecutive lanes write consecutive
// columns.
//
// Epilogues: bias; bias + residual (out-projection and MLP-down); bias +
// GELU (MLP-up, to 3.3e-7); QKV, which writes Q to its own buffer
// and the fresh K/V of each masked token straight into that token's row of
// the working K/V (the K/V cache of Fig. 7 with the masked rows replaced).
//
// bf16 tiles: BM x BN from 64 x 64 to 256 x 256, operands copied global ->
// LDS without staging registers into 2-4 stages of 64-deep K steps, the 256 x
// 256 and 256 x 192 ones refilled region by region (gemm_pp_kernel); fp32:
// 64 x 64 or 32 x 32 tiles through registers, double-buffered. The host picks tile,
// stage count and K split from a step-time table measured on MI355X; split
// workgroups write float32 partials, summed in a fixed order by a second
// kernel that applies the epilogue (or, before a LayerNorm, by the fused
// sum + LayerNorm kernel in rows.hip). Launches with more tiles than the
// CUs hold at once run persistent workgroups.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace ms {
namespace {

constexpr int kThreads = 256;
constexpr int kCUs = 256;

// GELU(x) = x (1 + erf(x / sqrt 2)) / 2 = max(x, 0) - |x| erfc(|x| / sqrt 2) / 2, with
// erfc(y) by Abramowitz & Stegun, Handbook of Mathematical Functions, formula
// 7.1.26: t (a1 + t (a2 + t (a3 + t (a4 + t a5)))) exp(-y^2), t = 1 / (1 + p y),
// |error| <= 1.5e-7. An absolute bound: the result is within 3.3e-7 of GELU over
// [-12, 12], far below the bf16 rounding of most outputs, but the tail of negative x
// is relatively off by 0.2% at -5 and 3% at -12 (as 0.5 x (1 + erf) loses it to the
// subtraction). One reciprocal, one exponential and twelve other instructions (the
// epilogue of a 256 x 256 tile evaluates 128 per lane, ~60 cycles each as
// 0.5 x (1 + erf)).
// |x| is taken of min(x, FLT_MAX), so that +inf gives +inf and not inf - inf * 0;
// -inf gives NaN, as x (1 + erf) does.
__device__ __forceinline__ float gelu(float x) {
    const float ax = fabsf(fminf(x, 3.402823466e+38f));
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f * 0.70710678118654752f, ax, 1.0f));
    float q = fmaf(0.5f * 1.061405429f, t, 0.5f * -1.453152027f);
    q = fmaf(q, t, 0.5f * 1.421413741f);
    q = fmaf(q, t, 0.5f * -0.284496736f);
    q = fmaf(q, t, 0.5f * 0.254829592f);
    q *= t * __builtin_amdgcn_exp2f(x * (x * (-0.5f * 1.4426950408889634f)));
    return fmaf(-ax, q, fmaxf(x, 0.f));
}

// v + bias, and GELU where the epilogue has it.
template <int EPI>
__device__ __forceinline__ void epilogue_math(float v[4], const float bv[4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] += bv[r];
    if constexpr (EPI == kEpiBiasGelu) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = gelu(v[r]);
    }
}

// Where output columns n.. of packed row m go (kEpiQKV: a group of columns that
// starts below g.d ends there, d and n being multiples of the group).
template <int EPI, typename T = bf16_t>
__device__ __forceinline__ T* epilogue_dst(const GemmDesc& g, int m, int n) {
    if (EPI == kEpiQKV && n >= g.d) return static_cast<T*>(g.kv) + (long)g.rows[m] * g.kvld + (n - g.d);
    return static_cast<T*>(g.C) + (long)m * g.ldc + n;
}

template <typename T, int EPI>
__device__ __forceinline__ void epilogue_store(const GemmDesc& g, int m, int n, float v[4]) {
    float bv[4];
    load4<T>(static_cast<const T*>(g.bias) + n, bv);
    epilogue_math<EPI>(v, bv);
    if constexpr (epi_resid(EPI)) {
        float rv[4];
        load4<T>(static_cast<const T*>(g.R) + (long)m * g.ldr + n, rv);
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] += rv[r];
    }
    store4<T>(epilogue_dst<EPI, T>(g, m, n), v);
}

// Epilogue of an unsplit, residual-free tile of the eight- or four-wave kernels
// (two waves along m, WN along n; SM x SN 16 x 16 blocks each): run on the
// registers, staged in LDS as bf16 (16-byte chunks XOR-swizzled by the row) and
// stored row by row, 16 bytes per lane: an MFMA block leaves a lane 4 columns of
// one row, so direct stores write 32-byte pieces of 16 rows. Against staging the
// float32 tile, in two passes where it does not fit: 8547x3456x1152 (256x256
// tiles, bias) 77.4 -> 67.8 us, 8547x4608x1152 (GELU) 127.3 -> 118.2 us.
// Starts and ends with the workgroup past its last LDS read.
template <int EPI, int BM, int BN, int WN, int SM, int SN>
__device__ __forceinline__ void store_tile_bf16(const GemmDesc& g, void* smem, const f32x4_t (&acc)[SN][SM], int m0, int n0,
                                                int tid, int wm, int wn) {
    constexpr int CPR = BN / 8, THREADS = 2 * WN * kWave;
    const int l16 = tid % 16, grp = tid % kWave / 16;
    bf16_t* const sb = static_cast<bf16_t*>(smem);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < SN; ++i) {
        const int nl = wn * (BN / WN) + i * 16 + grp * 4;
        float bv[4];
        load4<bf16_t>(static_cast<const bf16_t*>(g.bias) + min(n0 + nl, g.N - 4), bv);
#pragma unroll
        for (int j = 0; j < SM; ++j) {
            const int ml = wm * (BM / 2) + j * 16 + l16;
            float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
            epilogue_math<EPI>(v, bv);
            store4<bf16_t>(sb + ml * BN + (((nl / 8) ^ (ml & 7)) * 8) + nl % 8, v);
        }
    }
    __syncthreads();
    const bool wide = g.ldc % 8 == 0 && (EPI != kEpiQKV || g.kvld % 8 == 0);   // 16-byte aligned rows
    for (int idx = tid; idx < BM * CPR; idx += THREADS) {
        const int ml = idx / CPR, c = idx % CPR;
        const int m = m0 + ml, n = n0 + c * 8;
        if (m >= g.M || n >= g.N) continue;
        const vec16 t = ld16(sb + ml * BN + ((c ^ (ml & 7)) * 8));
        bf16_t* const o = epilogue_dst<EPI>(g, m, n);
        if (wide && n + 8 <= g.N) {
            st16(o, t);
        } else {   // N is a multiple of 4
            *reinterpret_cast<uint2*>(o) = make_uint2(t.w[0], t.w[1]);
            if (n + 4 < g.N) *reinterpret_cast<uint2*>(o + 4) = make_uint2(t.w[2], t.w[3]);
        }
    }
    __syncthreads();
}

// Residual outputs and split-K partials: the float32 tile is staged in PASSES
// passes (16-byte chunks XOR-swizzled by the row), each wave row's blocks spread
// evenly over them; a lane then takes 8 columns of a row (16-byte residual loads
// and stores; 8547x1152x1152 34.6 -> 34.1 us against 4 columns), of a partial 4
// (32 bytes per lane: 1434x768x3072 in four ranges 18.2 -> 19.2 us). Starts and ends with the workgroup past its last LDS read.
template <int EPI, int BM, int BN, int WN, int SM, int SN, int PASSES>
__device__ __forceinline__ void store_tile_f32(const GemmDesc& g, void* smem, const f32x4_t (&acc)[SN][SM], int m0, int n0,
                                               int kz, int tid, int wm, int wn) {
    static_assert(SM % PASSES == 0, "passes");
    constexpr int CPR = BN / 8, THREADS = 2 * WN * kWave, JP = SM / PASSES, RW = JP * 16;   // rows of a wave row per pass
    const int l16 = tid % 16, grp = tid % kWave / 16;
    float* const sc = static_cast<float*>(smem);
    const bool wide = g.ldc % 8 == 0 && (!epi_resid(EPI) || g.ldr % 8 == 0) && (EPI != kEpiQKV || g.kvld % 8 == 0);
    __syncthreads();
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
#pragma unroll
        for (int i = 0; i < SN; ++i) {
            const int nl = wn * (BN / WN) + i * 16 + grp * 4;
#pragma unroll
            for (int j = 0; j < JP; ++j) {
                const int ml = wm * RW + j * 16 + l16;
                const f32x4_t& a = acc[i][pass * JP + j];
                *reinterpret_cast<float4*>(sc + ml * BN + (((nl / 4) ^ (ml & 15)) * 4)) = make_float4(a[0], a[1], a[2], a[3]);
            }
        }
        __syncthreads();
        if (g.ksplit > 1) {
            constexpr int CPF = BN / 4;
            for (int idx = tid; idx < 2 * RW * CPF; idx += THREADS) {
                const int ml = idx / CPF, c = idx % CPF;
                const int m = m0 + (ml / RW) * (BM / 2) + pass * RW + ml % RW, n = n0 + c * 4;
                if (m < g.M && n < g.N)
                    st16(g.part + ((long)kz * g.M + m) * g.N + n, ld16(sc + ml * BN + ((c ^ (ml & 15)) * 4)));
            }
            __syncthreads();
            continue;
        }
        // Kernels without a residual never come here (store_tile_bf16 takes their unsplit
        // tiles). Compiled without it they need 8 to 19 registers less but their main
        // loops are scheduled worse: block of 1434 rows at d 768 100.3 -> 100.9 us, of 1024
        // at d 1152 129.5 -> 130.7.
        for (int idx = tid; idx < 2 * RW * CPR; idx += THREADS) {
            const int ml = idx / CPR, c = idx % CPR;
            const int m = m0 + (ml / RW) * (BM / 2) + pass * RW + ml % RW, n = n0 + c * 8;
            if (m >= g.M || n >= g.N) continue;
            float v[8];
            load4<float>(sc + ml * BN + (((2 * c) ^ (ml & 15)) * 4), v);
            load4<float>(sc + ml * BN + (((2 * c + 1) ^ (ml & 15)) * 4), v + 4);
            if (wide && n + 8 <= g.N) {
                const vec16 bw = ld16(static_cast<const bf16_t*>(g.bias) + n);
                vec16 rw = {{0u, 0u, 0u, 0u}}, ow;
                if constexpr (epi_resid(EPI)) rw = ld16(static_cast<const bf16_t*>(g.R) + (long)m * g.ldr + n);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float bv[4], rv[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const uint32_t wb = bw.w[2 * h + r / 2], wr = rw.w[2 * h + r / 2];
                        bv[r] = __uint_as_float(r & 1 ? wb & 0xffff0000u : wb << 16);
                        rv[r] = __uint_as_float(r & 1 ? wr & 0xffff0000u : wr << 16);
                    }
                    epilogue_math<EPI>(v + 4 * h, bv);
                    if constexpr (epi_resid(EPI)) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) v[4 * h + r] += rv[r];
                    }
                    ow.w[2 * h] = pack_bf16x2(v[4 * h], v[4 * h + 1]);
                    ow.w[2 * h + 1] = pack_bf16x2(v[4 * h + 2], v[4 * h + 3]);
                }
                st16(epilogue_dst<EPI>(g, m, n), ow);
            } else {
                epilogue_store<bf16_t, EPI>(g, m, n, v);
                if (n + 4 < g.N) epilogue_store<bf16_t, EPI>(g, m, n + 4, v + 4);
            }
        }
        __syncthreads();
    }
}

// Tile of logical block id `lb` in groups of up to `gm` m-tiles: ids run over
// the m-tiles of a group first, then over n, then to the next group, so that
// the 32 consecutive ids one XCD runs at once cover a 4 x 8 block of tiles
// (12 operand slices per K step in its L2) instead of a 16 x 2 strip (18).
// Measured on MI355X against m-fastest order: -15% time on 6144x3072x3072,
// -11% on 8192x1152x4608, -2..-4% on the other large shapes, equal on small M.
// From 4096 rows on, groups of 8 m-tiles: at c4 (8 x ~860 masked rows) the
// step is 2.6% shorter, mostly in the attention that follows the QKV
// projection; below that, 4 (8 is 0.25% slower at c2).
constexpr int kGroupM = 4;
constexpr int kGroupMLarge = 8;
constexpr int kGroupLargeRows = 4096;

struct TileIdx {
    int kz, m0, n0;
};

__device__ __forceinline__ TileIdx tile_of(int lb, int tiles_m, int tiles_n, int bm, int bn, int gm) {
    const int per_k = tiles_m * tiles_n;
    const int kz = lb / per_k;
    const int r = lb - kz * per_k;
    const int group = r / (gm * tiles_n);
    const int gm0 = group * gm;
    const int gsize = min(gm, tiles_m - gm0);
    const int within = r - group * gm * tiles_n;
    return TileIdx{kz, (gm0 + within % gsize) * bm, (within / gsize) * bn};
}

template <typename T, int BM, int BN, int EPI>
__global__ __launch_bounds__(kThreads) void gemm_kernel(GemmDesc g) {
    using E = Elt<T>;
    using frag_t = typename E::frag_t;
    constexpr int BK = 128 / sizeof(T);     // one 128-byte row chunk per K step
    constexpr int V = 16 / sizeof(T);       // elements per 16-byte vector
    constexpr int LDS = BK + V;             // padded LDS row (elements): 144 bytes
    constexpr int CHUNKS = BK / V;          // 16-byte chunks per tile row (8)
    constexpr int ROWS_PER_PASS = kThreads / CHUNKS;   // 32
    constexpr int PA = BM / ROWS_PER_PASS;
    constexpr int PW = BN / ROWS_PER_PASS;
    constexpr int SM = BM / 32;             // 16-row MFMA blocks per wave (rows m)
    constexpr int SN = BN / 32;             // 16-col MFMA blocks per wave (cols n)
    __shared__ __attribute__((aligned(16))) T sA[2][BM * LDS];
    __shared__ __attribute__((aligned(16))) T sW[2][BN * LDS];

    const int tid = threadIdx.x;
    const int lane = tid % kWave;
    const int wave = tid / kWave;
    const int wm = wave & 1, wn = wave >> 1;
    const int M = g.M, N = g.N, K = g.K;
    // 1-D launch: each XCD takes a contiguous range of logical ids (k split
    // slowest), mapped to tiles in grouped order
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    const int lb = xcd_logical_block(blockIdx.x, tiles_m * tiles_n * g.ksplit);
    const TileIdx ti = tile_of(lb, tiles_m, tiles_n, BM, BN, g.group_m);
    const int kz = ti.kz, m0 = ti.m0, n0 = ti.n0;
    const int kbeg = kz * g.kchunk;
    const int kend = min(K, kbeg + g.kchunk);
    const T* __restrict__ A = static_cast<const T*>(g.A);
    const T* __restrict__ W = static_cast<const T*>(g.W);

    const int lr = tid / CHUNKS;
    const int lc = tid % CHUNKS;
    vec16 ra[PA], rw[PW];
    auto gload = [&](int k0) {
#pragma unroll
        for (int i = 0; i < PA; ++i) {
            const int m = min(m0 + lr + ROWS_PER_PASS * i, M - 1);
            ra[i] = ld16(A + (long)m * g.lda + k0 + lc * V);
        }
#pragma unroll
        for (int i = 0; i < PW; ++i) {
            const int n = min(n0 + lr + ROWS_PER_PASS * i, N - 1);
            rw[i] = ld16(W + (long)n * K + k0 + lc * V);
        }
    };
    auto sstore = [&](int buf) {
#pragma unroll
        for (int i = 0; i < PA; ++i) st16(&sA[buf][(lr + ROWS_PER_PASS * i) * LDS + lc * V], ra[i]);
#pragma unroll
        for (int i = 0; i < PW; ++i) st16(&sW[buf][(lr + ROWS_PER_PASS * i) * LDS + lc * V], rw[i]);
    };

    f32x4_t acc[SN][SM];
#pragma unroll
    for (int i = 0; i < SN; ++i)
#pragma unroll
        for (int j = 0; j < SM; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    const int nk = (kend - kbeg) / BK;
    if (nk > 0) {
        gload(kbeg);
        sstore(0);
    }
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int buf = kt & 1;
        if (kt + 1 < nk) gload(kbeg + (kt + 1) * BK);
#pragma unroll
        for (int ks = 0; ks < BK / E::kKStep; ++ks) {
            const int kk = ks * E::kKStep + (lane / 16) * E::kKPerLane;
            // all activation fragments, then one weight fragment at a time
            frag_t fa[SM];
#pragma unroll
            for (int j = 0; j < SM; ++j)
                fa[j] = *reinterpret_cast<const frag_t*>(&sA[buf][(wm * (BM / 2) + j * 16 + lane % 16) * LDS + kk]);
#pragma unroll
            for (int i = 0; i < SN; ++i) {
                const frag_t fw = *reinterpret_cast<const frag_t*>(&sW[buf][(wn * (BN / 2) + i * 16 + lane % 16) * LDS + kk]);
#pragma unroll
                for (int j = 0; j < SM; ++j) acc[i][j] = E::mma(fw, fa[j], acc[i][j]);
            }
        }
        if (kt + 1 < nk) sstore(buf ^ 1);
        __syncthreads();
    }

#pragma unroll
    for (int i = 0; i < SN; ++i) {
        const int n = n0 + wn * (BN / 2) + i * 16 + (lane / 16) * 4;
        if (n >= N) continue;
#pragma unroll
        for (int j = 0; j < SM; ++j) {
            const int m = m0 + wm * (BM / 2) + j * 16 + lane % 16;
            if (m >= M) continue;
            float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
            if (g.ksplit == 1) {
                epilogue_store<T, EPI>(g, m, n, v);
            } else {
                *reinterpret_cast<float4*>(g.part + ((long)kz * M + m) * N + n) =
                    make_float4(v[0], v[1], v[2], v[3]);
            }
        }
    }
}

// bf16 main loop with direct global->LDS loads (gfx950 buffer_load_dwordx4
// ... lds, one buffer resource per tile and operand, so rows past M or N read
// as zeros) into S LDS stages, so S-1 K steps are in flight without staging
// registers.
// LDS rows are 128 bytes (one K step of 64 bf16) with their eight 16-byte
// chunks XOR-swizzled by (row >> 1) & 7: each load instruction fills 1 KB
// (8 rows) contiguously, and the 16-row MFMA fragment reads of one K chunk
// still touch 16 distinct bank groups. The copies are issued as opaque
// instructions (dma_buf16) and ordered by explicit counter waits: a compiler
// that sees them must assume each may write the stage being read and drains
// every load in flight before the first fragment read of each step.

// Waves per workgroup of this kernel: 192x192 tiles run eight (2 x 4, 96 x 48
// outputs each), the other tiles four (2 x 2). 192-wide tiles fill the 256 CUs
// in whole waves where the projection widths are multiples of 192 and not of
// 256 (1152, 3072, 4608, 12288 columns); 192x192 holds three stages in LDS and
// quantises rows more finely than 256-row tiles.
constexpr int dl_waves(int bm, int bn) { return bm * bn >= 192 * 192 ? 8 : 4; }

// Waits until all but the last `left` issued stages have landed (never more than R
// are in flight behind the one waited for; towards the end of K fewer).
template <int R, int IPW>
__device__ __forceinline__ void wait_stages(int left) {
    if (left >= R) wait_vmcnt<R * IPW>();
    else if constexpr (R > 0) wait_stages<R - 1, IPW>(left);
}

template <int BM, int BN, int S, int EPI>
__global__ __launch_bounds__(kWave * dl_waves(BM, BN)) void gemm_dl_kernel(GemmDesc g) {
    static_assert(S >= 2 && S <= 4, "stages");
    constexpr int NW = dl_waves(BM, BN);
    constexpr int WM = 2, WN = NW / 2;          // wave grid: WM along m, WN along n
    using E = Elt<bf16_t>;
    using frag_t = typename E::frag_t;
    constexpr int BK = 64;
    constexpr int ROWE = 64;                    // elements per LDS row
    constexpr int IPW = (BM + BN) / (8 * NW);   // 1 KB load instructions per wave per stage
    constexpr int IA = BM / (8 * NW);           // of which for the activation tile
    constexpr int SM = BM / WM / 16;            // 16-row MFMA blocks per wave (rows m)
    constexpr int SN = BN / WN / 16;            // 16-col MFMA blocks per wave (cols n)
    static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "load split");
    // S activation stages, then S weight stages; after the main loop the
    // same LDS stages the output tile
    __shared__ __attribute__((aligned(1024))) bf16_t smem[S * (BM + BN) * ROWE];
    bf16_t* const sAb = smem;
    bf16_t* const sWb = smem + S * BM * ROWE;
    // passes that stage the float32 tile: one, or two when only half fits
    constexpr int kLdsBytes = S * (BM + BN) * ROWE * 2;
    constexpr int kOutPasses = kLdsBytes >= BM * BN * 4 ? 1 : 2;
    static_assert(kLdsBytes * 2 >= BM * BN * 4 && WM == 2, "output staging");

    const int tid = threadIdx.x;
    const int lane = tid % kWave;
    const int wave = tid / kWave;
    const int wm = wave % WM, wn = wave / WM;
    const int M = g.M, N = g.N, K = g.K;
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    const int total = tiles_m * tiles_n * g.ksplit;
    const bf16_t* __restrict__ A = static_cast<const bf16_t*>(g.A);
    const bf16_t* __restrict__ W = static_cast<const bf16_t*>(g.W);

    // Persistent when the grid is smaller than the tile count: workgroup b
    // takes physical ids b, b + grid, ... (the grid is a multiple of the XCD
    // count, so every id maps to a tile of the workgroup's own XCD).
    // Tile state: split index, tile origin, K range, and the tile's operand
    // rows as buffer resources (rows past M or N read as zeros).
    int kz, m0, n0, kbeg, nk;
    u32x4_t rA, rW;
    auto setup = [&](int hw) {
        const TileIdx ti = tile_of(xcd_logical_block(hw, total), tiles_m, tiles_n, BM, BN, g.group_m);
        kz = ti.kz; m0 = ti.m0; n0 = ti.n0;
        kbeg = kz * g.kchunk;
        nk = (min(K, kbeg + g.kchunk) - kbeg) / BK;
        rA = raw_rsrc(A + (size_t)m0 * g.lda, (uint32_t)((size_t)min(BM, M - m0) * g.lda * 2));
        rW = raw_rsrc(W + (size_t)n0 * K, (uint32_t)((size_t)min(BN, N - n0) * K * 2));
    };
    // per load instruction this lane's byte offset inside the tile's rows
    // (row * ld + swizzled chunk)
    uint32_t voff[IPW];
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
        const int blk = i * NW + wave;                      // 8-row block
        const bool isA = i < IA;
        const int rloc = (isA ? blk : blk - BM / 8) * 8 + lane / 8;
        const int c = (lane % 8) ^ ((rloc >> 1) & 7);
        voff[i] = (uint32_t)((isA ? rloc * g.lda : rloc * K) + c * 8) * 2u;
    }
    // the wave's 1 KB destination of each load instruction inside a stage (bytes)
    uint32_t ldst[IPW];
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
        const int blk = i * NW + wave;
        ldst[i] = i < IA ? lds_addr(sAb + blk * 512) : lds_addr(sWb + (blk - BM / 8) * 512);
    }
    constexpr uint32_t kStageA = BM * ROWE * 2, kStageW = BN * ROWE * 2;   // bytes
    auto issue = [&](int kt, int st) {
        const uint32_t k0 = (uint32_t)(kbeg + kt * BK) * 2u;
#pragma unroll
        for (int i = 0; i < IPW; ++i) {
            if (i < IA) dma_buf16(rA, voff[i], k0, ldst[i] + st * kStageA);
            else dma_buf16(rW, voff[i], k0, ldst[i] + st * kStageW);
        }
    };
    auto prologue = [&]() {
#pragma unroll
        for (int st = 0; st < S - 1; ++st)
            if (st < nk) issue(st, st);
    };

    // fragment offsets inside a stage: row r, logical chunk ks*4 + grp, swizzled by (r >> 1) & 7
    const int sw = (lane % 16) >> 1;
    const int grp = lane / 16;

    int hw = blockIdx.x;
    setup(hw);
    prologue();
    for (;;) {
    f32x4_t acc[SN][SM];
#pragma unroll
    for (int i = 0; i < SN; ++i)
#pragma unroll
        for (int j = 0; j < SM; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int kt = 0; kt < nk; ++kt) {
        const int st = kt % S;
        // stage kt complete (the loads of the later stages may stay in
        // flight); the barrier also ends every wave's reads of the stage
        // refilled next, read in step kt - 1
        wait_stages<S - 2, IPW>(nk - kt - 1);
        barrier_only();
        // The 8-wave tiles spread this step's copies over the MFMA groups of
        // the first half step, so the matrix cores start right after the
        // barrier (measured +3..12% on their shapes); the 4-wave tiles issue
        // them at once, which keeps their shorter prefetch distance whole.
        const bool more_k = kt + S - 1 < nk;
        const int k_next = kbeg + (kt + S - 1) * BK, st_next = (kt + S - 1) % S;
        if (NW != 8 && more_k) issue(kt + S - 1, st_next);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int ch = ((ks * 4 + grp) ^ sw) * 8;
            frag_t fa[SM];
#pragma unroll
            for (int j = 0; j < SM; ++j)
                fa[j] = *reinterpret_cast<const frag_t*>(sAb + st * BM * ROWE + (wm * (BM / WM) + j * 16 + lane % 16) * ROWE + ch);
#pragma unroll
            for (int i = 0; i < SN; ++i) {
                const frag_t fw = *reinterpret_cast<const frag_t*>(sWb + st * BN * ROWE + (wn * (BN / WN) + i * 16 + lane % 16) * ROWE + ch);
#pragma unroll
                for (int j = 0; j < SM; ++j) acc[i][j] = E::mma(fw, fa[j], acc[i][j]);
                if (NW == 8 && ks == 0 && more_k) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int q = i * IPW / SN; q < (i + 1) * IPW / SN; ++q) {
                        if (q < IA) dma_buf16(rA, voff[q], (uint32_t)k_next * 2u, ldst[q] + st_next * kStageA);
                        else dma_buf16(rW, voff[q], (uint32_t)k_next * 2u, ldst[q] + st_next * kStageW);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    }

    const int hw_next = hw + (int)gridDim.x;
    if (!epi_resid(EPI) && g.ksplit == 1) store_tile_bf16<EPI, BM, BN, WN, SM, SN>(g, smem, acc, m0, n0, tid, wm, wn);
    else store_tile_f32<EPI, BM, BN, WN, SM, SN, kOutPasses>(g, smem, acc, m0, n0, kz, tid, wm, wn);
    if (hw_next >= total) return;
    hw = hw_next;
    setup(hw);
    prologue();
    }
}

// The 256-row, eight-wave tiles (256 x 256 and 256 x 192; waves 2 x 4, 128 x 64
// or 128 x 48 outputs each): the K step of 64 runs in four phases, each the
// products of one quarter of a wave's rows (32) with all of its columns. Phase
// q's MFMAs read registers only; meanwhile the next quarter's rows are read
// from LDS, and in phase 3 each 16-column block of the weights is replaced by
// the next step's as soon as its last product is issued.
//
// An LDS stage is refilled region by region (a quarter of the rows, or one
// 16-column block of every wave: 8 KB, one copy per wave): a region's reads
// are complete at the barrier after the phase that used them, so step k + 2's
// weights are copied in phases 1 and 2 of step k, its rows in phases 3 and 0.
// Every copy has four to six phases to land, and at each phase start the copies
// issued after the one it needs may stay in flight (a fixed count per phase).
// Copies past the last K step go through an empty buffer resource (zeros, no
// traffic), so the counts hold to the end.
//
// Why: with a whole stage per K step, copied under the step before and waited
// for at its end, the matrix cores were busy 41-43% of the time (MLP projections of
// a 19-block d 3072 stack), here 55-58%: the
// operands of more than one step are in flight, and no MFMA waits for an LDS
// read issued in its own phase. A step of 256 x 256 x 64 on every CU takes 1.5
// us, against 1.1 without the copies, 1.3 without the LDS reads and 0.9 with the
// MFMAs alone: what is left is the operand
// stream from L2 (64 KB per CU and step) under the LDS reads. Against the
// stage-per-step loop (bf16 outputs staged in both): 16384x3072x12288 1006 ->
// 930 us, 3732x3072x12288 276 -> 235, 3732x12288x3072 273 -> 240, 12288x6144x3072
// 407 -> 355, 4096^3 112 -> 105. One barrier per two phases, wave priorities
// and four waves of 128 x 128 were even or slower (the last by 35%).
template <int BN>
struct PpCfg {
    static constexpr int SN = BN / 64;                  // 16-column blocks per wave
    static constexpr int kStage = (256 + BN) * 128;     // bytes
    static constexpr int W0 = 256 * 128;                // regions of 8 KB: A0..A3, then the W blocks
    // copies in flight at the start of phase 0..3: issued (order W, A0..A3 of a
    // step) after the region the phase reads
    static constexpr int V0 = 2 + SN + 2, V1 = 1 + SN + 4, V2 = SN + 4 + 2, V3 = 3 + SN;
};

template <int BN, int EPI>
__global__ __launch_bounds__(512) void gemm_pp_kernel(GemmDesc g) {
    using C = PpCfg<BN>;
    using E = Elt<bf16_t>;
    using frag_t = typename E::frag_t;
    constexpr int BM = 256, SM = 8, SN = C::SN, NW = 8;
    __shared__ __attribute__((aligned(1024))) uint8_t smem[2 * C::kStage];
    const uint32_t lds0 = lds_addr(smem);

    const int tid = threadIdx.x;
    const int lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wm = wave % 2, wn = wave / 2;
    const int M = g.M, N = g.N, K = g.K;
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    const int total = tiles_m * tiles_n * g.ksplit;
    const bf16_t* __restrict__ A = static_cast<const bf16_t*>(g.A);
    const bf16_t* __restrict__ W = static_cast<const bf16_t*>(g.W);

    // A region's 64 rows: A quarter q has rows wm' 128 + q 32 + 0..31 of both
    // wave rows, W block i columns wn' 16 SN + i 16 + 0..15 of the four wave
    // columns. This wave copies rows 8 wave .. 8 wave + 7: this lane's byte
    // offset inside the tile's operand (quarter and block are scalar offsets).
    const int rr = wave * 8 + lane / 8;
    const int chunk = (lane % 8) ^ ((rr >> 1) & 7);
    const uint32_t va = (uint32_t)(((rr / 32) * 128 + rr % 32) * g.lda + chunk * 8) * 2u;
    const uint32_t vw = (uint32_t)(((rr / 16) * 16 * SN + rr % 16) * K + chunk * 8) * 2u;
    const uint32_t astep = (uint32_t)g.lda * 64u, wstep = (uint32_t)K * 32u;   // 32 rows, 16 columns

    // LDS fragment addresses: row l16 of the wave's rows in a region, logical
    // chunk ks * 4 + lane group
    const int l16 = lane % 16, grp = lane / 16;
    const uint32_t f0 = l16 * 128 + ((grp ^ (l16 >> 1)) * 16), f1 = l16 * 128 + (((4 + grp) ^ (l16 >> 1)) * 16);
    const uint32_t pa[2] = {lds0 + wm * 4096 + f0, lds0 + wm * 4096 + f1};
    const uint32_t pw[2] = {lds0 + C::W0 + wn * 2048 + f0, lds0 + C::W0 + wn * 2048 + f1};
    typedef const __attribute__((address_space(3))) frag_t* lfrag;

    int hw = blockIdx.x;
    for (;;) {
    const TileIdx ti = tile_of(xcd_logical_block(hw, total), tiles_m, tiles_n, BM, BN, g.group_m);
    const int kz = ti.kz, m0 = ti.m0, n0 = ti.n0;
    const int kbeg = kz * g.kchunk;
    const int nk = (min(K, kbeg + g.kchunk) - kbeg) / 64;
    u32x4_t rA = raw_rsrc(A + (size_t)m0 * g.lda, (uint32_t)((size_t)min(BM, M - m0) * g.lda * 2));
    u32x4_t rW = raw_rsrc(W + (size_t)n0 * K, (uint32_t)((size_t)min(BN, N - n0) * K * 2));
    const uint32_t bytesA = rA[2], bytesW = rW[2];
    // region copies of K step kt into stage st = kt % 2; past the end through an empty resource
    auto copy_a = [&](int st, int kt, int q) {
        rA[2] = kt < nk ? bytesA : 0u;
        dma_buf16(rA, va, (uint32_t)(kbeg + kt * 64) * 2u + q * astep, lds0 + st * C::kStage + q * 8192 + wave * 1024);
    };
    auto copy_w = [&](int st, int kt, int i) {
        if (i >= SN) return;
        rW[2] = kt < nk ? bytesW : 0u;
        dma_buf16(rW, vw, (uint32_t)(kbeg + kt * 64) * 2u + i * wstep, lds0 + st * C::kStage + C::W0 + i * 8192 + wave * 1024);
    };
    auto read_a = [&](int st, int q, frag_t (&f)[2][2]) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            uint32_t b = pa[ks] + st * C::kStage;
            asm volatile("" : "+v"(b));   // one address: region and block offsets fold into the reads
#pragma unroll
            for (int j = 0; j < 2; ++j) f[j][ks] = *(lfrag)(uintptr_t)(b + q * 8192 + j * 2048);
        }
    };
    auto read_w = [&](int st, int i, frag_t (&f)[2]) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            uint32_t b = pw[ks] + st * C::kStage;
            asm volatile("" : "+v"(b));
            f[ks] = *(lfrag)(uintptr_t)(b + i * 8192);
        }
    };

    f32x4_t acc[SN][SM];
#pragma unroll
    for (int i = 0; i < SN; ++i)
#pragma unroll
        for (int j = 0; j < SM; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    frag_t fa[2][2][2], fw[SN][2];   // two sets of a quarter's rows; the wave's columns

    // phase q of K step kt (stage st)
    auto phase = [&](auto stage, auto quarter, int kt) {
        constexpr int st = decltype(stage)::value, q = decltype(quarter)::value;
        constexpr int V = q == 0 ? C::V0 : q == 1 ? C::V1 : q == 2 ? C::V2 : C::V3;
        __builtin_amdgcn_sched_barrier(0);
        wait_vmcnt<V>();
        barrier_only();
#pragma unroll
        for (int i = 0; i < SN; ++i) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][2 * q + j] = E::mma(fw[i][ks], fa[q & 1][j][ks], acc[i][2 * q + j]);
            __builtin_amdgcn_sched_barrier(0);
            if (i == 0) read_a(q == 3 ? st ^ 1 : st, (q + 1) & 3, fa[(q + 1) & 1]);
            if (q == 3) read_w(st ^ 1, i, fw[i]);
            if (i == 1) {
                if (q == 0) { copy_a(st ^ 1, kt + 1, 2); copy_a(st ^ 1, kt + 1, 3); }
                if (q == 1) { copy_w(st, kt + 2, 0); copy_w(st, kt + 2, 1); }
                if (q == 2) { copy_w(st, kt + 2, 2); copy_w(st, kt + 2, 3); }
                if (q == 3) { copy_a(st, kt + 2, 0); copy_a(st, kt + 2, 1); }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto kstep = [&](auto stage, int kt) {
        phase(stage, std::integral_constant<int, 0>{}, kt);
        phase(stage, std::integral_constant<int, 1>{}, kt);
        phase(stage, std::integral_constant<int, 2>{}, kt);
        phase(stage, std::integral_constant<int, 3>{}, kt);
    };
#pragma unroll
    for (int i = 0; i < SN; ++i) copy_w(0, 0, i);
#pragma unroll
    for (int q = 0; q < 4; ++q) copy_a(0, 0, q);
#pragma unroll
    for (int i = 0; i < SN; ++i) copy_w(1, 1, i);
    copy_a(1, 1, 0);
    copy_a(1, 1, 1);
    wait_vmcnt<3 + SN + 2>();   // W and A0 of step 0
    barrier_only();
    read_a(0, 0, fa[0]);
#pragma unroll
    for (int i = 0; i < SN; ++i) read_w(0, i, fw[i]);
    // in pairs of steps (the stages are compile-time constants); an odd last one
    // multiplies the zeros of the empty copies
    // (one loop exit: a second one made the compiler keep two copies of acc)
    for (int kt = 0; kt < nk; kt += 2) {
        kstep(std::integral_constant<int, 0>{}, kt);
        kstep(std::integral_constant<int, 1>{}, kt + 1);
    }
    wait_all();   // the zero copies too: the stages take the output next

    const int hw_next = hw + (int)gridDim.x;
    if (!epi_resid(EPI) && g.ksplit == 1) store_tile_bf16<EPI, BM, BN, 4, SM, SN>(g, smem, acc, m0, n0, tid, wm, wn);
    else store_tile_f32<EPI, BM, BN, 4, SM, SN, 2>(g, smem, acc, m0, n0, kz, tid, wm, wn);
    if (hw_next >= total) return;
    hw = hw_next;
    }
}

// Split-K: sum the partials in split order, then the epilogue.
template <typename T, int EPI>
__global__ __launch_bounds__(256) void gemm_reduce_kernel(GemmDesc g) {
    const long n4 = (long)g.M * g.N / 4;
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n4) return;
    const int m = (int)(i / (g.N / 4));
    const int n = (int)(i - (long)m * (g.N / 4)) * 4;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < g.ksplit; ++s) {
        const float4 p = *reinterpret_cast<const float4*>(g.part + ((long)s * g.M + m) * g.N + n);
        v[0] += p.x; v[1] += p.y; v[2] += p.z; v[3] += p.w;
    }
    epilogue_store<T, EPI>(g, m, n, v);
}

template <typename T, int BM, int BN>
hipError_t launch_tile(const GemmDesc& g, hipStream_t s) {
    dim3 grid(((g.N + BN - 1) / BN) * ((g.M + BM - 1) / BM) * g.ksplit), block(kThreads);
    switch (g.epilogue) {
        case kEpiBias: hipLaunchKernelGGL((gemm_kernel<T, BM, BN, kEpiBias>), grid, block, 0, s, g); break;
        case kEpiBiasResid: hipLaunchKernelGGL((gemm_kernel<T, BM, BN, kEpiBiasResid>), grid, block, 0, s, g); break;
        case kEpiBiasGelu: hipLaunchKernelGGL((gemm_kernel<T, BM, BN, kEpiBiasGelu>), grid, block, 0, s, g); break;
        case kEpiQKV: hipLaunchKernelGGL((gemm_kernel<T, BM, BN, kEpiQKV>), grid, block, 0, s, g); break;
        case kEpiBiasResidMlp: hipLaunchKernelGGL((gemm_kernel<T, BM, BN, kEpiBiasResidMlp>), grid, block, 0, s, g); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Grid of a direct-to-LDS launch: one workgroup per tile, or, past what the
// CUs hold at once, that many persistent workgroups (a multiple of the XCD
// count) looping over the tiles.
unsigned dl_grid(int resident, long tiles) {
    static const bool off = [] {   // tuning knob MS_GEMM_PERSISTENT=0: one workgroup per tile
        const char* v = std::getenv("MS_GEMM_PERSISTENT");
        return v && std::strcmp(v, "0") == 0;
    }();
    if (off || tiles <= resident) return (unsigned)tiles;
    return (unsigned)(resident - resident % kXcds);
}

template <int BM, int BN, int S, int EPI>
hipError_t launch_dl_epi(const GemmDesc& g, hipStream_t s) {
    const long tiles = (long)((g.N + BN - 1) / BN) * ((g.M + BM - 1) / BM) * g.ksplit;
    const int threads = kWave * dl_waves(BM, BN);
    static const int resident = [threads] {   // workgroups of this kernel the CUs hold at once
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, gemm_dl_kernel<BM, BN, S, EPI>, threads, 0) !=
                hipSuccess || per_cu < 1)
            per_cu = 1;
        return per_cu * kCUs;
    }();
    const unsigned grid = dl_grid(resident, tiles);
    hipLaunchKernelGGL((gemm_dl_kernel<BM, BN, S, EPI>), dim3(grid), dim3(threads), 0, s, g);
    return hipGetLastError();
}

template <int BN, int EPI>
hipError_t launch_pp_epi(const GemmDesc& g, hipStream_t s) {
    const long tiles = (long)((g.N + BN - 1) / BN) * ((g.M + 255) / 256) * g.ksplit;
    hipLaunchKernelGGL((gemm_pp_kernel<BN, EPI>), dim3(dl_grid(kCUs, tiles)), dim3(512), 0, s, g);
    return hipGetLastError();
}

template <int BN>
hipError_t launch_pp(const GemmDesc& g, hipStream_t s) {
    switch (g.epilogue) {
        case kEpiBias: return launch_pp_epi<BN, kEpiBias>(g, s);
        case kEpiBiasResid: return launch_pp_epi<BN, kEpiBiasResid>(g, s);
        case kEpiBiasGelu: return launch_pp_epi<BN, kEpiBiasGelu>(g, s);
        case kEpiQKV: return launch_pp_epi<BN, kEpiQKV>(g, s);
        case kEpiBiasResidMlp: return launch_pp_epi<BN, kEpiBiasResidMlp>(g, s);
        default: return hipErrorInvalidValue;
    }
}

template <int BM, int BN, int S>
hipError_t launch_dl(const GemmDesc& g, hipStream_t s) {
    switch (g.epilogue) {
        case kEpiBias: return launch_dl_epi<BM, BN, S, kEpiBias>(g, s);
        case kEpiBiasResid: return launch_dl_epi<BM, BN, S, kEpiBiasResid>(g, s);
        case kEpiBiasGelu: return launch_dl_epi<BM, BN, S, kEpiBiasGelu>(g, s);
        case kEpiQKV: return launch_dl_epi<BM, BN, S, kEpiQKV>(g, s);
        case kEpiBiasResidMlp: return launch_dl_epi<BM, BN, S, kEpiBiasResidMlp>(g, s);
        default: return hipErrorInvalidValue;
    }
}

template <typename T>
hipError_t launch_reduce(const GemmDesc& g, hipStream_t s) {
    const long n4 = (long)g.M * g.N / 4;
    dim3 grid((unsigned)((n4 + 255) / 256)), block(256);
    switch (g.epilogue) {
        case kEpiBias: hipLaunchKernelGGL((gemm_reduce_kernel<T, kEpiBias>), grid, block, 0, s, g); break;
        case kEpiBiasResid: hipLaunchKernelGGL((gemm_reduce_kernel<T, kEpiBiasResid>), grid, block, 0, s, g); break;
        case kEpiBiasGelu: hipLaunchKernelGGL((gemm_reduce_kernel<T, kEpiBiasGelu>), grid, block, 0, s, g); break;
        case kEpiQKV: hipLaunchKernelGGL((gemm_reduce_kernel<T, kEpiQKV>), grid, block, 0, s, g); break;
        case kEpiBiasResidMlp: hipLaunchKernelGGL((gemm_reduce_kernel<T, kEpiBiasResidMlp>), grid, block, 0, s, g); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

// Tile and stage choice from a measured cost model. A launch of g workgroups of a tile
// and stage count costs about steps x a(g) + b(g) us: a(g) per 64-deep K step of the
// whole grid, b(g) the work outside the K loop (prologue, epilogue, stores). Split-K
// multiplies the groups, divides the steps and adds the partial-sum pass. a, b and the
// pass's price are a least-squares fit (relative errors, non-negative) to 50000
// measured launches on MI355X: 1220 shapes of 16 to 16384 rows, the four projections of
// models 64 to 4096 wide, each over the tiles, stages and splits within twice the best
// one's estimate, in graphs of launches whose operands rotate over 300 MB. Times of one
// operand set, from L2, had misled the choice: 4096x1024x4096 128x128 tiles at 65 us
// instead of 128x64 at 44, 512x1024x1024 a split in four at 12.7 instead of none at 8.1.
// Over those shapes the choice is 1.3% slower than the best measured one (geometric
// mean, worst 31%), against 7.5% (72%) with that table.
namespace {
constexpr int kCostN = 15;
// g / 256 up to one workgroup per CU, the busiest CU's workgroups beyond (linear
// between these, in proportion past the last)
constexpr double kCostAt[kCostN] = {0.25, 0.5, 1, 2, 3, 4, 5, 6, 7, 8, 12, 16, 24, 32, 48};
struct TileCost {
    int bm, bn, stages;
    double step[kCostN];   // a, us per K step
    double tile[kCostN];   // b, us per launch
};
constexpr TileCost kCost[] = {
    {256, 256, 2, {1.153, 1.113, 1.467, 2.768, 4.323, 5.256, 6.176, 8.451, 9.427, 11.142, 17.706, 22.925, 35.281, 46.687, 70.807},
     {9.3, 9.8, 10.3, 17.0, 27.9, 53.9, 81.8, 69.3, 102.1, 96.0, 149.2, 198.3, 263.2, 351.8, 519.9}},
    {256, 192, 2, {0.962, 0.917, 1.064, 2.128, 3.353, 4.762, 5.279, 6.194, 7.153, 8.568, 13.287, 18.546, 27.009, 36.713, 56.483},
     {7.6, 8.9, 9.1, 15.9, 24.4, 25.9, 47.4, 65.5, 79.5, 81.1, 121.6, 150.9, 224.4, 296.9, 386.9}},
    {192, 192, 2, {1.024, 1.023, 1.037, 2.018, 3.010, 4.215, 4.740, 6.233, 7.313, 8.058, 12.272, 16.655, 24.696, 32.866, 49.132},
     {5.2, 6.4, 7.2, 11.1, 15.9, 18.0, 30.4, 26.5, 30.3, 49.4, 68.2, 90.5, 165.5, 214.6, 317.3}},
    {192, 192, 3, {0.791, 0.793, 0.874, 1.756, 2.731, 3.868, 4.521, 5.751, 6.421, 6.938, 11.042, 15.018, 22.788, 30.906, 47.176},
     {7.3, 7.7, 7.2, 11.6, 17.1, 21.0, 31.0, 31.8, 43.0, 63.3, 75.0, 110.5, 164.9, 202.4, 298.3}},
    {256, 128, 2, {1.008, 0.993, 1.013, 1.969, 3.136, 4.120, 5.272, 6.122, 6.325, 6.936, 12.015, 16.492, 24.488, 31.480, 47.089},
     {7.6, 7.0, 7.9, 13.0, 16.6, 27.0, 27.3, 37.4, 49.8, 76.0, 84.4, 94.1, 171.7, 216.5, 304.8}},
    {256, 128, 3, {1.378, 1.185, 1.079, 2.449, 3.395, 4.570, 5.681, 6.230, 6.361, 7.366, 11.383, 16.072, 24.341, 32.520, 48.521},
     {5.7, 6.2, 8.2, 10.0, 14.4, 21.5, 21.2, 35.0, 48.0, 67.3, 95.7, 107.1, 160.8, 204.5, 296.8}},
    {128, 128, 2, {0.706, 0.709, 0.762, 0.876, 1.582, 1.828, 2.446, 2.862, 3.390, 3.724, 6.013, 7.377, 11.409, 15.064, 24.211},
     {3.8, 4.6, 5.4, 6.4, 8.2, 10.1, 10.7, 11.9, 10.8, 15.6, 11.8, 34.1, 65.3, 98.9, 139.8}},
    {128, 128, 3, {0.834, 0.730, 0.671, 1.514, 2.280, 2.948, 3.645, 4.361, 4.965, 5.616, 8.400, 9.217, 14.150, 18.688, 28.924},
     {4.4, 4.6, 5.5, 6.3, 8.3, 12.4, 10.3, 11.2, 14.0, 16.1, 16.4, 54.3, 86.2, 120.2, 188.0}},
    {128, 128, 4, {0.856, 0.732, 0.657, 1.512, 2.264, 2.935, 3.616, 4.306, 4.924, 5.574, 8.309, 9.093, 13.996, 18.517, 28.601},
     {3.7, 4.6, 5.8, 6.6, 8.6, 12.6, 10.5, 11.7, 13.7, 15.9, 15.6, 56.6, 91.7, 128.1, 206.9}},
    {128, 64, 2, {0.465, 0.558, 0.577, 0.672, 0.870, 1.418, 1.469, 1.772, 2.096, 2.303, 3.488, 4.598, 7.454, 10.587, 15.275},
     {3.2, 3.6, 4.0, 4.2, 5.3, 5.7, 6.5, 7.7, 7.9, 9.9, 10.4, 12.1, 7.9, 8.3, 45.6}},
    {128, 64, 3, {0.500, 0.522, 0.488, 0.699, 1.056, 1.380, 1.817, 2.057, 2.172, 2.700, 3.693, 5.293, 8.321, 11.032, 16.383},
     {3.1, 3.6, 4.1, 4.3, 5.9, 5.7, 5.7, 8.0, 9.2, 8.9, 13.3, 13.6, 9.6, 15.3, 50.4}},
    {128, 64, 4, {0.488, 0.511, 0.460, 0.997, 1.665, 2.318, 2.809, 3.158, 3.484, 4.170, 5.805, 7.373, 9.927, 12.763, 18.744},
     {3.1, 3.6, 4.3, 5.6, 5.1, 5.1, 6.4, 9.1, 10.9, 9.8, 14.0, 20.8, 37.9, 60.3, 123.2}},
    {64, 128, 2, {0.508, 0.567, 0.586, 0.677, 0.888, 1.385, 1.485, 1.758, 2.134, 2.298, 3.387, 4.695, 7.017, 10.186, 15.405},
     {3.3, 3.7, 4.4, 4.6, 5.8, 6.3, 7.4, 9.9, 8.3, 11.0, 13.5, 13.2, 23.4, 25.8, 37.7}},
    {64, 128, 3, {0.469, 0.445, 0.449, 0.619, 1.036, 1.319, 1.651, 1.895, 2.233, 2.532, 3.711, 4.980, 7.996, 10.714, 16.323},
     {3.3, 4.0, 4.6, 5.1, 6.2, 7.0, 7.9, 10.7, 9.9, 12.6, 15.6, 19.5, 22.3, 26.2, 39.0}},
    {64, 128, 4, {0.456, 0.438, 0.439, 0.832, 1.277, 1.711, 2.136, 2.529, 2.981, 3.349, 5.198, 6.765, 10.058, 13.569, 20.259},
     {3.4, 4.1, 4.8, 6.5, 7.5, 9.0, 11.2, 13.7, 14.9, 19.1, 24.5, 34.9, 51.0, 70.6, 116.1}},
    {64, 64, 2, {0.405, 0.514, 0.495, 0.505, 0.603, 0.748, 1.167, 1.189, 1.452, 1.531, 2.632, 3.470, 5.288, 7.679, 11.794},
     {2.7, 2.9, 3.2, 3.7, 4.4, 5.0, 5.3, 6.6, 4.9, 7.5, 9.6, 13.6, 11.4, 1.0, 1.0}},
    {64, 64, 3, {0.309, 0.318, 0.332, 0.401, 0.606, 0.798, 0.999, 1.170, 1.450, 1.513, 2.371, 3.103, 4.769, 7.022, 10.417},
     {2.9, 3.2, 3.5, 3.9, 4.6, 5.1, 4.9, 6.3, 4.5, 7.2, 9.1, 12.2, 10.7, 1.5, 1.0}},
    {64, 64, 4, {0.297, 0.299, 0.297, 0.408, 0.655, 0.814, 1.032, 1.174, 1.499, 1.588, 2.386, 3.198, 4.897, 6.722, 10.247},
     {3.0, 3.2, 3.6, 4.1, 5.1, 5.4, 5.8, 7.2, 5.5, 8.4, 11.2, 13.3, 15.4, 12.7, 14.6}},
};

double interp(const double* v, double x) {
    if (x <= kCostAt[0]) return v[0];
    for (int i = 1; i < kCostN; ++i)
        if (x <= kCostAt[i])
            return v[i - 1] + (v[i] - v[i - 1]) * (x - kCostAt[i - 1]) / (kCostAt[i] - kCostAt[i - 1]);
    return v[kCostN - 1] * x / kCostAt[kCostN - 1];
}

// Modelled time of `steps` K steps of an M x N product in `ks` K ranges, without the
// partial-sum pass.
double tile_us(const TileCost& c, int M, int N, int steps, int ks) {
    const long groups = (long)((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn) * ks;
    const double x = groups <= kCUs ? (double)groups / kCUs : (double)((groups + kCUs - 1) / kCUs);
    return ((steps + ks - 1) / ks) * interp(c.step, x) + interp(c.tile, x);
}

// The same for float32, per 32-deep step (bias epilogue, K = 256 and 1024). 32 x 32
// tiles are the quicker ones while the launch is short of workgroups (a step waits
// for its loads: 0.36 us against 0.76 at n = 1), 64 x 64 read half as much per
// product. Before, 64 x 64 and no K split: 205x256x1024 26 -> 8 us, 205x768x256
// 9.3 -> 5.1, 800x512x2048 50 -> 30, 3000x512x2048 82 -> 67.
constexpr TileCost kCostF32[] = {
    {64, 64, 2, {0.76, 0.76, 0.76, 1.34, 1.85, 2.43, 2.95, 3.45, 4.05, 4.62, 6.63, 8.90, 13.0, 17.1, 25.6},
     {4.0, 4.0, 4.0, 5.1, 6.8, 7.0, 10.0, 12.0, 10.5, 9.5, 13.8, 14.6, 23.0, 32.0, 48.0}},
    {32, 32, 2, {0.356, 0.356, 0.356, 0.483, 0.693, 0.882, 1.07, 1.26, 1.44, 1.63, 2.31, 3.15, 4.50, 5.74, 8.60},
     {2.35, 2.35, 2.35, 2.45, 2.78, 2.92, 3.2, 3.5, 3.9, 4.3, 6.3, 6.5, 8.0, 10.2, 15.0}},
};

GemmPlan plan_f32(int M, int N, int K, size_t part_capacity_floats) {
    GemmPlan p{64, 64, 1, 2};
    const int steps = K / 32;
    double best = 1e30;
    for (const TileCost& c : kCostF32) {
        for (int ks = 1; ks <= 8 && ks <= steps; ++ks) {
            if (ks > 1 && (size_t)ks * M * N > part_capacity_floats) break;
            double us = tile_us(c, M, N, steps, ks);
            // partial sums: 2.1 us at two planes of 205 x 256, 4.0 at eight
            if (ks > 1) us += 2.0 + 0.25 * ks + ((double)ks * 4 + 4) * M * N / 4.0e6;
            if (us < best * 0.97) {
                best = us;
                p = GemmPlan{c.bm, c.bn, ks, c.stages};
            }
        }
    }
    return p;
}
}  // namespace

GemmPlan plan_gemm(int dtype, int M, int N, int K, size_t part_capacity_floats, bool ln_sum) {
    GemmPlan p{64, 64, 1, 2};
    if (dtype != kBF16) return plan_f32(M, N, K, part_capacity_floats);
    const int steps = K / 64;
    double best = 1e30;
    static const double split_scale = [] {   // tuning knob MS_GEMM_SPLIT_COST: scales the split-K pass cost
        const char* v = std::getenv("MS_GEMM_SPLIT_COST");
        return v ? std::max(0.0, std::atof(v)) : 1.0;
    }();
    for (const TileCost& c : kCost) {
        for (int ks = 1; ks <= 8 && ks <= steps; ++ks) {
            if (ks > 1 && (size_t)ks * M * N > part_capacity_floats) break;
            double us = tile_us(c, M, N, steps, ks);
            // partial sums: ks float planes read, one bf16 plane written, ~4 TB/s, + a launch;
            // as part of the LayerNorm that would follow anyway 2 us less (block of 205 rows
            // at d 768 54.3 -> 53.0 us; 4 us less: 12 blocks of 1229 rows 1092 -> 1103)
            if (ks > 1) us += split_scale * ((ln_sum ? -0.5 : 1.54) + 0.27 * ks + ((double)ks * 4 + 2) * M * N / 4.0e6);
            if (us < best) {
                best = us;
                p = GemmPlan{c.bm, c.bn, ks, c.stages};
            }
        }
    }
    if (const char* f = std::getenv("MS_GEMM_TILE")) {   // tuning override "BMxBN"
        int bm = 0, bn = 0;
        if (std::sscanf(f, "%dx%d", &bm, &bn) == 2) {
            for (const TileCost& c : kCost)
                if (c.bm == bm && c.bn == bn && c.stages == 2) p = GemmPlan{bm, bn, 1, 2};
        }
    }
    return p;
}

// Largest stage count whose LDS fits next to nothing else (160 KB per CU).
int max_stages(int bm, int bn) {
    const int per = (bm + bn) * 64 * 2;
    return std::min(4, (160 * 1024) / per);
}

hipError_t launch_gemm(int dtype, GemmDesc& g, hipStream_t s) {
    if (g.M == 0) return hipSuccess;
    const int bk = dtype == kBF16 ? 64 : 32;
    if (g.ksplit < 1) g.ksplit = 1;
    // K range per split, a multiple of the K step
    const int steps = g.K / bk;
    const int per = (steps + g.ksplit - 1) / g.ksplit;
    g.kchunk = per * bk;
    g.ksplit = (steps + per - 1) / per;
    static const int group_m = [] {   // tuning knob MS_GEMM_GROUP (tiles_m or more: m fastest)
        const char* v = std::getenv("MS_GEMM_GROUP");
        return v ? std::max(1, std::atoi(v)) : 0;
    }();
    g.group_m = group_m > 0 ? group_m : (g.M >= kGroupLargeRows ? kGroupMLarge : kGroupM);
    if (dtype != kBF16) return g.bm == 32 ? launch_tile<float, 32, 32>(g, s) : launch_tile<float, 64, 64>(g, s);
    // main loop: direct-to-LDS (default) or the register-staged double buffer
    // (tuning knob MS_GEMM_PIPE=staged); MS_GEMM_STAGES overrides the stage count
    static const bool staged = [] {
        const char* v = std::getenv("MS_GEMM_PIPE");
        return v && std::strcmp(v, "staged") == 0;
    }();
    // tuning knob MS_GEMM_STAGES: the stage count of every direct-to-LDS
    // launch (read per launch, so a test can take each stage variant in turn)
    const char* fs = std::getenv("MS_GEMM_STAGES");
    const int force_stages = fs ? std::atoi(fs) : 0;
    if (staged) {
        if (g.bm == 256 && g.bn == 256) return launch_tile<bf16_t, 256, 256>(g, s);
        if (g.bm == 256 && g.bn == 128) return launch_tile<bf16_t, 256, 128>(g, s);
        if (g.bm == 128 && g.bn == 128) return launch_tile<bf16_t, 128, 128>(g, s);
        if (g.bm == 128 && g.bn == 64) return launch_tile<bf16_t, 128, 64>(g, s);
        if (g.bm == 64 && g.bn == 128) return launch_tile<bf16_t, 64, 128>(g, s);
        return launch_tile<bf16_t, 64, 64>(g, s);
    }
    int st = force_stages > 0 ? force_stages : (g.stages > 0 ? g.stages : 2);
    st = std::max(2, std::min(st, max_stages(g.bm, g.bn)));
    if (g.bm == 256 && g.bn == 256) return launch_pp<256>(g, s);
    if (g.bm == 256 && g.bn == 192) return launch_pp<192>(g, s);
    if (g.bm == 192 && g.bn == 192) return st >= 3 ? launch_dl<192, 192, 3>(g, s) : launch_dl<192, 192, 2>(g, s);
    if (g.bm == 256 && g.bn == 128) return st >= 3 ? launch_dl<256, 128, 3>(g, s) : launch_dl<256, 128, 2>(g, s);
    if (g.bm == 128 && g.bn == 128)
        return st >= 4 ? launch_dl<128, 128, 4>(g, s) : st == 3 ? launch_dl<128, 128, 3>(g, s) : launch_dl<128, 128, 2>(g, s);
    if (g.bm == 128 && g.bn == 64)
        return st >= 4 ? launch_dl<128, 64, 4>(g, s) : st == 3 ? launch_dl<128, 64, 3>(g, s) : launch_dl<128, 64, 2>(g, s);
    if (g.bm == 64 && g.bn == 128)
        return st >= 4 ? launch_dl<64, 128, 4>(g, s) : st == 3 ? launch_dl<64, 128, 3>(g, s) : launch_dl<64, 128, 2>(g, s);
    return st >= 4 ? launch_dl<64, 64, 4>(g, s) : st == 3 ? launch_dl<64, 64, 3>(g, s) : launch_dl<64, 64, 2>(g, s);
}

hipError_t launch_gemm_reduce(int dtype, const GemmDesc& g, hipStream_t s) {
    if (g.M == 0 || g.ksplit <= 1) return hipSuccess;
    return dtype == kBF16 ? launch_reduce<bf16_t>(g, s) : launch_reduce<float>(g, s);
}

}  // namespace ms
