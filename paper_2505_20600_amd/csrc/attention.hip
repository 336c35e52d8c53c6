// Mask-aware attention (Sec. 3.1, Fig. 5): only the masked tokens are
// queried, and each query attends over the keys/values of every token of its
// request, fresh rows for masked tokens and cached rows for the others (the
// LLM-decoding analogy of that subsection). Softmax is the full, unmasked one.
//
// Two kernels, one for bf16 (further down) and one for float32: workgroup =
// (query tile of 64 packed rows of one segment, head); four waves, sixteen
// queries each. Key/value tiles of 64 tokens are staged in LDS and shared by
// the four waves. Online softmax in float32 with exp2 and a log2(e)-prescaled
// score.
//
// MFMA orientation: the scores are computed transposed, S^T = K Q^T, so each
// lane holds one query column and four keys per 16-key subtile. That is
// exactly the per-lane data the B operand of O^T = V^T P^T needs, so the
// probabilities never leave registers; V is stored transposed in LDS so the
// A operand (V^T rows) reads contiguous keys. The pairing of MFMA K-slots to
// keys only has to agree between the two operands of one instruction, which
// it does by construction.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace ms {
namespace {

constexpr int kThreads = 256;
constexpr int kKeyTile = 64;

// float32 kernel, head_dim padded to HDP columns: 64 queries x one head x one key
// range per workgroup. The float32 matrix instructions bound it (HDP / 16 x 32 of
// them per 64-key tile and wave, 32 cycles each: 2.0 of 2.3 us per tile and
// workgroup at head_dim 64) once four workgroups share a CU; before the key range
// was split a small request ran on a few CUs, each tile in the 4.2 us of its own
// loads, MFMAs and softmax one after the other.
template <int HDP>
__global__ __launch_bounds__(kThreads) void attention_f32_kernel(AttnDesc a) {
    using T = float;
    using E = Elt<T>;
    using frag_t = typename E::frag_t;
    static_assert(E::kKPerLane == 1, "one key slot per lane");
    constexpr int V = 16 / sizeof(T);            // elements per 16-byte vector
    constexpr int KLDS = HDP + V;                // padded K row (elements)
    constexpr int VLDS = kKeyTile + V;           // padded V^T row (elements)
    constexpr int NKC = HDP / E::kKStep;         // MFMA steps over head_dim for S
    constexpr int NHS = HDP / 16;                // 16-row subtiles of O^T
    __shared__ __attribute__((aligned(16))) T sK[kKeyTile * KLDS];
    __shared__ __attribute__((aligned(16))) T sVt[HDP * VLDS];

    const int tid = threadIdx.x;
    const int lane = tid % kWave;
    const int wave = tid / kWave;
    const int grp = lane / 16;
    const int head = blockIdx.y;
    const int tile = blockIdx.x;
    const int split = blockIdx.z;
    const int hd = a.hd, d = a.d, T_ = a.T;

    // segment of this query tile
    int s = 0;
    while (s + 1 < a.nseg && a.cu_tiles[s + 1] <= tile) ++s;
    const int b = a.seg_req[s];
    const int row0 = a.seg_start[s] + (tile - a.cu_tiles[s]) * kQTile;
    const int row_end = a.seg_start[s + 1];
    const int qrow = row0 + wave * 16 + lane % 16;
    const bool qvalid = qrow < row_end;

    // zero the head_dim padding of the LDS tiles once; tile loads never touch it
    if (hd < HDP) {
        for (int i = tid; i < kKeyTile * (HDP - hd); i += kThreads) {
            const int r = i / (HDP - hd), c = hd + i % (HDP - hd);
            sK[r * KLDS + c] = T(0);
        }
        for (int i = tid; i < (HDP - hd) * kKeyTile; i += kThreads) {
            const int r = hd + i / kKeyTile, c = i % kKeyTile;
            sVt[r * VLDS + c] = T(0);
        }
    }

    // Q^T fragments (B operand): query = lane % 16, head_dim slots by lane group
    frag_t qf[NKC];
    const T* __restrict__ q = static_cast<const T*>(a.q);
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) {
        const int k = kc * E::kKStep + grp * E::kKPerLane;
        qf[kc] = (qvalid && k < hd) ? q[(long)qrow * d + head * hd + k] : 0.f;
    }

    f32x4_t oacc[NHS];
#pragma unroll
    for (int h = 0; h < NHS; ++h) oacc[h] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;

    const T* __restrict__ kv = static_cast<const T*>(a.kv);
    const long req_base = (long)b * T_;
    const int chunks = hd / V;                     // 16-byte chunks per key row
    const int ntiles = (T_ + kKeyTile - 1) / kKeyTile;
    const int kt_end = min(ntiles, (split + 1) * a.tiles_per_split);

    for (int kt = split * a.tiles_per_split; kt < kt_end; ++kt) {
        const int k0 = kt * kKeyTile;
        __syncthreads();
        for (int i = tid; i < kKeyTile * chunks; i += kThreads) {
            const int kk = i / chunks, c = i % chunks;
            const int t = k0 + kk;
            vec16 kvec = {{0u, 0u, 0u, 0u}}, vvec = {{0u, 0u, 0u, 0u}};
            if (t < T_) {
                const T* src = kv + (req_base + t) * 2 * d + head * hd + c * V;
                kvec = ld16(src);
                vvec = ld16(src + d);
            }
            st16(&sK[kk * KLDS + c * V], kvec);
            const T* ve = reinterpret_cast<const T*>(&vvec);
#pragma unroll
            for (int e = 0; e < V; ++e) sVt[(c * V + e) * VLDS + kk] = ve[e];
        }
        __syncthreads();

        // S^T subtiles: keys ks*16 + 4*grp + r, query lane % 16
        float sc[4][4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            f32x4_t acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kc = 0; kc < NKC; ++kc) {
                const int k = kc * E::kKStep + grp * E::kKPerLane;
                const frag_t kf = *reinterpret_cast<const frag_t*>(&sK[(ks * 16 + lane % 16) * KLDS + k]);
                acc = E::mma(kf, qf[kc], acc);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int t = k0 + ks * 16 + grp * 4 + r;
                sc[ks][r] = t < T_ ? acc[r] * a.scale_log2 : -INFINITY;
            }
        }

        float mx = -INFINITY;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int r = 0; r < 4; ++r) mx = fmaxf(mx, sc[ks][r]);
        mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
        mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
        const float m_new = fmaxf(m_run, mx);
        const float corr = (m_run == -INFINITY) ? 0.f : fast_exp2(m_run - m_new);
        const float m_ref = m_new == -INFINITY ? 0.f : m_new;   // scores of -inf only so far: weights 0
        float psum = 0.f;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                sc[ks][r] = fast_exp2(sc[ks][r] - m_ref);
                psum += sc[ks][r];
            }
        l_run = l_run * corr + psum;
        m_run = m_new;
#pragma unroll
        for (int h = 0; h < NHS; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r) oacc[h][r] *= corr;

        // O^T += V^T P^T
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int key = ks * 16 + grp * 4 + r;
#pragma unroll
                for (int h = 0; h < NHS; ++h) {
                    const frag_t vf = sVt[(h * 16 + lane % 16) * VLDS + key];
                    oacc[h] = E::mma(vf, sc[ks][r], oacc[h]);
                }
            }
    }

    float l = l_run;
    l += __shfl_xor(l, 16, kWave);
    l += __shfl_xor(l, 32, kWave);
    // a key range of weight 0 leaves zeros for the combine; the whole row's result stays 0 / 0
    const float inv_l = a.nsplit > 1 && l == 0.f ? 0.f : 1.0f / l;
    if (qvalid) {
        const long orow = (long)split * a.M + qrow;   // nsplit 1: the output row itself
        T* __restrict__ o = a.nsplit > 1 ? a.part_o : static_cast<T*>(a.o);
#pragma unroll
        for (int h = 0; h < NHS; ++h) {
            const int c = h * 16 + grp * 4;
            if (c < hd) {
                float v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = oacc[h][r] * inv_l;
                store4<T>(o + orow * d + head * hd + c, v);
            }
        }
        if (a.nsplit > 1 && grp == 0)
            *reinterpret_cast<float2*>(a.part_ml + 2 * (orow * a.n_heads + head)) = make_float2(m_run, l);
    }
}

__device__ __forceinline__ f32x4_t mfma32(bf16x8_t a, bf16x8_t b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// ---------------------------------------------------------------------------
// bf16 kernel, head_dim any multiple of 8 up to 128.
//
// Workgroup = 128 packed query rows of one segment x one head x one key range;
// each wave owns 32 queries (two 16-query MFMA column blocks), so every K and
// V fragment read from LDS feeds two MFMAs. Transposed scores S^T = K Q^T
// leave the probabilities in the B-operand layout of O^T = V^T P^T. K and V
// tiles of 64 keys go global -> LDS with buffer_load_dwordx4 ... lds (no
// staging registers, no VALU work to store them) into S stages, in natural
// [key][head_dim] layout;
// the PV operand V^T is read with the gfx950 transpose read
// ds_read_b64_tr_b16: within each 16-lane group, lane i receives element
// (i & 3) of the 8 bytes addressed by lane 4e + (i >> 2), e = 0..3. Each
// lane therefore addresses V[key0 + (l16 >> 2)][hd0 + 4 (l16 & 3)] and
// receives V[key0 + e][hd0 + l16], e = 0..3: four keys of one head_dim row,
// in the k-slot order of P^T. Keys past the end read as zeros (buffer bound).
// The softmax denominator comes from V^T rows of ones: a constant operand
// where head_dim is a multiple of 16, else the padding rows of the last
// 16-row block, whose lanes address a small LDS block of ones.
//
// LDS banks: a ds_read_b128 is served in groups of 16 lanes (0-3, 12-15 and
// 20-27; 4-11, 16-19 and 28-31; the same of the upper half), so a K fragment
// read (16 rows, chunk g of lane group g) mixes two chunk columns. k_swz XORs
// the 16-byte chunks of a row so that each group falls into 16 different bank
// groups at every even chunk count (head_dim 64: 4.6 cycles per read, 8.4 with
// a swizzle that only separates the 16 rows of one column); odd counts (72,
// 104, ...) stay two-way. The transpose reads take 4 rows x 32 bytes per
// 16-lane group, which v_swz keeps apart for rows of 128 and 256 bytes.
//
// What bounds it: at two or three workgroups per CU the matrix cores are busy 37%
// (head_dim 72, 4096 rows) to 46% (128, a 19-block stack) of the time, the rest is the softmax (per 64-key tile and wave 32
// exponentials at 8.6 cycles and ~110 other VALU instructions at 3-5, against
// 576 MFMA cycles at head_dim 64 and 1088 at 128), of which only a part runs
// under another wave's MFMAs, and the start and end of each workgroup. The
// running maximum is subtracted by starting the score accumulators at -m (in the
// exponent's FMA instead of there: 329 -> 333 us for a block of 4096 rows at d 1152),
// and its row reduction runs only when some lane's maximum calls for a rescale.
// Measured at 4 x ~1450 rows of 24 heads of 128 over 4608 keys 364 -> 339 us,
// 4096 rows of 16 heads of 72 over 4096 keys 103 (with combine) -> 95 us; the
// head_dims that had a register-staged kernel before: 96 with 2.6k rows of 12
// heads over 2745 keys 182 -> 62 us. 32 x 32 x 16 MFMAs with the denominator on
// v_dot2 (a software pipeline over 32-key blocks, scheduled by hand or by the
// compiler) were 10-20% slower.
// ---------------------------------------------------------------------------

constexpr float kRescaleLog2 = 8.0f;   // softmax weights may reach 2^8 before a rescale
// Score accumulators start at minus the running maximum, but not beyond this: a score
// far above the maximum so far would be rounded to the digits of the latter (a first
// key tile near the type's lowest value left the others' scores none). 2^14 leaves them
// 2^-10, below the rounding of the weights, and a tile's ordinary path as it was.
constexpr float kStartMax = 16384.0f;

template <int HD>
struct DmaCfg {
    // 32-deep QK steps; the last one's padding slots multiply zeros by zeros.
    // (A 16-deep MFMA for a short remainder takes the same 16 cycles, and one
    // that continued the accumulators of a 32-deep one right before it gave a
    // query block wrong scores now and then, 390 of 1500 runs at head_dim 48; the
    // cause was not found, so that form is not used.)
    static constexpr int NK32 = (HD + 31) / 32;
    static constexpr int ROWB = HD * 2;                 // bytes per K / V row
    static constexpr bool SWZ = ROWB == 128 || ROWB == 256;   // V rows swizzled
    static constexpr int TILEB = kKeyTile * ROWB;       // bytes per K (or V) tile
    static constexpr bool KTAIL = HD % 32 != 0;         // the last QK step has padding slots
    static constexpr int KPAD = 16;                     // zeros past the K tile, read by the padding slots
    static constexpr int STAGEB = 2 * TILEB + KPAD;     // K tile, pad, V tile
    static constexpr int INSTR = TILEB / 1024;          // 1 KB copies per tile
    static constexpr int NQ = 2 * INSTR;                // copies per stage (K then V)
    static constexpr int IPW_MAX = (NQ + 3) / 4;       // copies per wave per stage (most)
    static constexpr bool SUM_IN_PAD = (HD % 16) != 0;
    static constexpr int NHS = (HD + 15) / 16 + (SUM_IN_PAD ? 0 : 1);
    static constexpr int NREAL = (HD + 15) / 16;        // O^T subtiles with V rows
    static_assert(TILEB % 1024 == 0, "tile copies");
};

// 16-byte chunk swizzles of a V and of a K row (XOR of the chunk index; see
// the kernel comment).
template <int ROWB>
__device__ __forceinline__ int v_swz(int r) {
    if constexpr (ROWB == 128) return 2 * ((r >> 1) & 3) + ((r >> 3) & 1);
    else if constexpr (ROWB == 256) return 2 * (r & 7) + ((r >> 3) & 1);
    else return 0;
}
template <int ROWB>
__device__ __forceinline__ int k_swz(int r) {
    if constexpr (ROWB == 256) return r & 15;
    else if constexpr (ROWB == 128) return (r >> 1) & 7;
    else if constexpr (ROWB % 128 == 64) return (r >> 1) & 3;
    else return 0;
}

typedef const __attribute__((address_space(3))) uint8_t* lds_cptr;

__device__ __forceinline__ bf16x4_t ld_tr16(lds_cptr p) {
    typedef short s4 __attribute__((ext_vector_type(4)));
    const s4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s4*)(p));
    return __builtin_bit_cast(bf16x4_t, v);
}

// Workgroups per CU the register budget is set for: four up to head_dim 48
// (128 VGPRs, no spills), three for 56 and 64, two above (whose registers then
// allow two or three).
constexpr int dma_occupancy(int hd) { return hd <= 48 ? 4 : hd <= 64 ? 3 : 2; }

template <int HD>
__global__ __launch_bounds__(kThreads, dma_occupancy(HD)) void attention_dma_kernel(AttnDesc a) {
    using C = DmaCfg<HD>;
    constexpr int S = 2;   // LDS stages
    __shared__ __attribute__((aligned(1024))) uint8_t smem[S * C::STAGEB + 16];
    const uint32_t lds0 = lds_addr(smem);
    const uint32_t ones_rel = S * C::STAGEB;            // 8 bytes of bf16 ones (SUM_IN_PAD)

    const int tid = threadIdx.x;
    const int lane = tid % kWave;
    const int wave = tid / kWave;
    const int grp = lane / 16;
    const int l16 = lane % 16;
    const int total = a.n_qtiles_fast * a.nsplit * a.n_heads;
    const int lb = xcd_logical_block(blockIdx.x, total);
    const int head = lb / (a.nsplit * a.n_qtiles_fast);
    const int split = (lb / a.n_qtiles_fast) % a.nsplit;
    const int T_ = a.T, d = a.d;

    int tile = lb % a.n_qtiles_fast, seg = 0, row0 = 0, row_end = 0;
    for (; seg < a.nseg; ++seg) {
        const int r0 = a.seg_start[seg], r1 = a.seg_start[seg + 1];
        const int nt = (r1 - r0 + kFastQTile - 1) / kFastQTile;
        if (tile < nt) { row0 = r0 + tile * kFastQTile; row_end = r1; break; }
        tile -= nt;
    }
    if (seg >= a.nseg) return;
    const int b = a.seg_req[seg];
    const int ntiles_all = (T_ + kKeyTile - 1) / kKeyTile;
    const int kt0 = split * a.tiles_per_split;
    const int kt1 = min(ntiles_all, kt0 + a.tiles_per_split);
    const int nt = max(0, kt1 - kt0);

    // constant LDS: the K pads' zeros and the ones block
    if (tid < S) *reinterpret_cast<uint4*>(smem + tid * C::STAGEB + C::TILEB) = make_uint4(0u, 0u, 0u, 0u);
    if (tid == S) *reinterpret_cast<uint2*>(smem + S * C::STAGEB) = make_uint2(0x3f803f80u, 0x3f803f80u);

    // buffer resource over request b's K/V block [T][2][d]
    const u32x4_t rsrc = raw_rsrc(static_cast<const bf16_t*>(a.kv) + (long)b * T_ * 2 * d, (uint32_t)T_ * 4u * (uint32_t)d);
    // per copy of this wave: fixed per-lane global byte offset and LDS destination in a stage
    uint32_t voff[C::IPW_MAX], ldst[C::IPW_MAX];
#pragma unroll
    for (int i = 0; i < C::IPW_MAX; ++i) {
        const int q = min(i * 4 + wave, C::NQ - 1);
        const bool isV = q >= C::INSTR;
        const int pos = (q % C::INSTR) * 1024 + lane * 16;
        const int r = pos / C::ROWB;
        const int c = ((pos % C::ROWB) / 16) ^ (isV ? v_swz<C::ROWB>(r) : k_swz<C::ROWB>(r));
        voff[i] = (uint32_t)(r * 4 * d + (isV ? 2 * d : 0) + head * C::ROWB + c * 16);
        ldst[i] = __builtin_amdgcn_readfirstlane((uint32_t)((isV ? C::TILEB + C::KPAD : 0) + (q % C::INSTR) * 1024));
    }
    auto issue = [&](int kt, int st) {
        const uint32_t soff = (uint32_t)kt * kKeyTile * 4u * (uint32_t)d;
        const uint32_t sbase = lds0 + st * C::STAGEB;
#pragma unroll
        for (int i = 0; i < C::IPW_MAX; ++i)
            if (i * 4 + wave < C::NQ) dma_buf16(rsrc, voff[i], soff, sbase + ldst[i]);
    };

    // Q^T fragments (B operand)
    bf16x8_t qf[2][C::NK32];
    const bf16_t* __restrict__ q = static_cast<const bf16_t*>(a.q);
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        const int qrow = row0 + wave * 32 + qb * 16 + l16;
        const bool valid = qrow < row_end;
        const bf16_t* qp = q + (long)qrow * d + head * HD;
#pragma unroll
        for (int kc = 0; kc < C::NK32; ++kc) {
            vec16 v = {{0u, 0u, 0u, 0u}};
            if (valid && kc * 32 + grp * 8 < HD) v = ld16(qp + kc * 32 + grp * 8);
            qf[qb][kc] = __builtin_bit_cast(bf16x8_t, v);
        }
    }

    // fragment read offsets inside a stage (bytes)
    const int fK = k_swz<C::ROWB>(l16);
    uint32_t koff[C::NK32];
#pragma unroll
    for (int kc = 0; kc < C::NK32; ++kc) koff[kc] = l16 * C::ROWB + (((4 * kc + grp) ^ fK) * 16);
    // last QK step of a head_dim that is not a multiple of 32, per 16-key
    // block: lanes whose slots lie past the row read the stage's block of zeros
    uint32_t kofft[C::KTAIL ? 4 : 1];
    if constexpr (C::KTAIL) {
        const int col = (C::NK32 - 1) * 64 + grp * 16;   // bytes
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) kofft[ks] = col < C::ROWB ? (ks * 16 + l16) * C::ROWB + col : C::TILEB;
    }
    const int rowA = 4 * grp + (l16 >> 2);
    const int fV = v_swz<C::ROWB>(rowA);
    uint32_t voffh[C::NREAL];
#pragma unroll
    for (int h = 0; h < C::NREAL; ++h) {
        const int hd = 16 * h + 4 * (l16 & 3);
        voffh[h] = C::TILEB + C::KPAD + rowA * C::ROWB + (((hd / 8) ^ fV) * 16) + (hd % 8) * 2;
    }
    const bool ones_lane = C::SUM_IN_PAD && (16 * (C::NREAL - 1) + 4 * (l16 & 3)) >= HD;

    f32x4_t oacc[2][C::NHS];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb)
#pragma unroll
        for (int h = 0; h < C::NHS; ++h) oacc[qb][h] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const float cs = a.scale_log2, rescale_at = kRescaleLog2 / cs;
    // running maximum per query (-inf: no score above -inf yet); the scores' accumulators
    // start at negm, minus the maximum within +-kStartMax
    float m_run[2] = {-INFINITY, -INFINITY};
    f32x4_t negm[2] = {f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}};
    bool beyond = true;   // some query's maximum lies beyond it: every tile is shifted
    const bf16x8_t onesf = __builtin_bit_cast(bf16x8_t, make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u));

    // S^T + negm of one tile (QK^T) into sacc, keys past T masked
    auto qk = [&](uint32_t sbase, int k0, bool tail, f32x4_t (&sacc)[2][4]) {
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) sacc[qb][ks] = negm[qb];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
            for (int kc = 0; kc < C::NK32; ++kc) {
                const bool pad = C::KTAIL && kc == C::NK32 - 1;
                const bf16x8_t kf = *reinterpret_cast<const bf16x8_t*>(
                    smem + sbase + (pad ? kofft[C::KTAIL ? ks : 0] : koff[kc] + ks * 16 * C::ROWB));
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) sacc[qb][ks] = mfma32(kf, qf[qb][kc], sacc[qb][ks]);
            }
        }
        if (tail) {
#pragma unroll
            for (int qb = 0; qb < 2; ++qb)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (k0 + ks * 16 + grp * 4 + r >= T_) sacc[qb][ks][r] = -INFINITY;
        }
    };
    // online softmax in place: sacc becomes the weights; running maxima and accumulators updated
    auto softmax = [&](f32x4_t (&sacc)[2][4], bool first) {
        // Rescale only when some score exceeds its query's running maximum by
        // more than 8 in the exp2 domain: below that the stale maximum
        // keeps the weights <= 256, exact in bf16 and fp32 alike, and numerator
        // and denominator share it. This keeps the row reductions and the
        // accumulators out of VALU work on almost every tile.
        float mx[2];
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
            mx[qb] = fmaxf(fmaxf(sacc[qb][0][0], sacc[qb][0][1]), sacc[qb][0][2]);
#pragma unroll
            for (int i = 3; i < 15; i += 2)
                mx[qb] = fmaxf(fmaxf(mx[qb], sacc[qb][i / 4][i % 4]), sacc[qb][(i + 1) / 4][(i + 1) % 4]);
            mx[qb] = fmaxf(mx[qb], sacc[qb][3][3]);
        }
        if (beyond || __any(fmaxf(mx[0], mx[1]) > rescale_at)) {
            bool far = false;
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
                const float rm = rows_max(mx[qb]);
                const bool none = m_run[qb] == -INFINITY;
                // the scores' new maximum and the old one, both less the accumulators' start
                const float was = none ? -INFINITY : m_run[qb] + negm[qb][0];
                const float up = fmaxf(rm, was);
                const bool still = up == -INFINITY;   // weights exp2(-inf) = 0
                if (!first) {   // nothing summed yet
                    const float corr = none ? 0.f : fast_exp2((was - up) * cs);
#pragma unroll
                    for (int h = 0; h < C::NHS; ++h) oacc[qb][h] *= corr;
                }
                m_run[qb] = fmaxf(m_run[qb], rm - negm[qb][0]);
                const float n = m_run[qb] == -INFINITY ? 0.f : -fminf(fmaxf(m_run[qb], -kStartMax), kStartMax);
                negm[qb] = f32x4_t{n, n, n, n};
                far |= fabsf(m_run[qb]) > kStartMax;
                const float off = still ? 0.f : up;
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int r = 0; r < 4; ++r) sacc[qb][ks][r] -= off;
            }
            beyond = __any(far);
        }
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int r = 0; r < 4; ++r) sacc[qb][ks][r] = fast_exp2(sacc[qb][ks][r] * cs);
    };
    // O^T += V^T P^T for one tile
    auto pv = [&](uint32_t sbase, f32x4_t (&sacc)[2][4]) {
        // O^T += V^T P^T; k-slots 0..3 = keys 32c + 4*grp + e, 4..7 = keys 32c + 16 + 4*grp + e
        uint32_t vbase[C::NREAL];
#pragma unroll
        for (int h = 0; h < C::NREAL; ++h) {
            vbase[h] = lds0 + sbase + voffh[h];
            asm volatile("" : "+v"(vbase[h]));   // keep the sum: offsets are added per read
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            // all V^T operands of this 32-key block first, so their reads overlap
            bf16x8_t vf[C::NHS];
#pragma unroll
            for (int h = 0; h < C::NHS; ++h) {
                if (h >= C::NREAL) {
                    vf[h] = onesf;
                } else {
                    // one base address per head_dim block and tile; the key-block and
                    // second-half offsets fold into the read instructions
                    lds_cptr p0 = (lds_cptr)(uintptr_t)vbase[h] + (32 * c) * C::ROWB;
                    lds_cptr p1 = (lds_cptr)(uintptr_t)vbase[h] + (32 * c + 16) * C::ROWB;
                    if (h == C::NREAL - 1 && ones_lane) { p0 = (lds_cptr)(uintptr_t)(lds0 + ones_rel); p1 = p0; }
                    const bf16x4_t lo = ld_tr16(p0), hi = ld_tr16(p1);
                    vf[h] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                }
            }
            bf16x8_t pf[2];
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
                uint4 w;
                w.x = pack_bf16x2(sacc[qb][2 * c][0], sacc[qb][2 * c][1]);
                w.y = pack_bf16x2(sacc[qb][2 * c][2], sacc[qb][2 * c][3]);
                w.z = pack_bf16x2(sacc[qb][2 * c + 1][0], sacc[qb][2 * c + 1][1]);
                w.w = pack_bf16x2(sacc[qb][2 * c + 1][2], sacc[qb][2 * c + 1][3]);
                pf[qb] = __builtin_bit_cast(bf16x8_t, w);
            }
#pragma unroll
            for (int h = 0; h < C::NHS; ++h)
#pragma unroll
                for (int qb = 0; qb < 2; ++qb) oacc[qb][h] = mfma32(vf[h], pf[qb], oacc[qb][h]);
        }
    };

    const int kfull = min(kt1, max(kt0, T_ / kKeyTile));
    auto fence_q = [&]() {
        // The Q fragments are complete here. Re-defining them through an empty asm
        // statement tells the compiler so; otherwise it makes the first MFMA of
        // every tile wait for all loads in flight, including the next prefetch.
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
#pragma unroll
            for (int kc = 0; kc < C::NK32; ++kc) asm volatile("" : "+v"(qf[qb][kc]));
        }
    };
    f32x4_t sa[2][4];
    const bool active = row0 + wave * 32 < row_end;
    // two stages: step t reads stage t % 2 while tile t + 1 loads into the other
    if (nt > 0) issue(kt0, 0);
    fence_q();
    for (int t = 0; t < nt; ++t) {
        wait_all();   // tile t has landed, and this wave's reads of the stage refilled below are done
        barrier_only();
        if (t + 1 < nt) issue(kt0 + t + 1, (t + 1) % S);
        const int kt = kt0 + t;
        if (!active) continue;   // every row of this wave lies past the segment: it only copies
        qk((t % S) * C::STAGEB, kt * kKeyTile, kt >= kfull, sa);
        softmax(sa, t == 0);
        pv((t % S) * C::STAGEB, sa);
    }

    // Output (or this key range's partial, in float32) through LDS: a lane
    // holds 4 consecutive head_dim values of one query row per 16 x 16 block, so
    // direct stores write 8- or 16-byte pieces of 16 rows; staged in the (now
    // free) stage memory, each wave writes its 32 rows as row-contiguous 16-byte
    // vectors. Rows of 128 / 256 bytes (float32: of a power of two) XOR-swizzle
    // their 16-byte chunks by the row.
    constexpr int CH = HD / 8;                     // 16-byte chunks per row
    constexpr int CF = HD / 4;                     // the same of a float32 row
    constexpr int SWM = C::SWZ ? (CH >= 16 ? 15 : CH - 1) : 0;
    constexpr int SWF = (CF & (CF - 1)) == 0 ? (CF >= 16 ? 15 : CF - 1) : 0;
    __syncthreads();   // every wave is past its last read of the stages
    uint8_t* const so = smem + wave * 32 * C::ROWB * (a.nsplit == 1 ? 1 : 2);
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        float l;
        if constexpr (C::SUM_IN_PAD) {
            // the last 8 rows of the last subtile are the ones rows: lane groups 2-3 hold them
            const float t0 = grp >= 2 ? oacc[qb][C::NHS - 1][0] : 0.f;
            auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(t0), __float_as_uint(t0), false, false);
            l = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
        } else {
            l = oacc[qb][C::NHS - 1][0];
        }
        // normalised by this key range's own sum; bf16 rows of the output, or
        // float32 rows of the partial (zeros for a range of weight 0)
        const float inv_l = a.nsplit > 1 && l == 0.f ? 0.f : 1.0f / l;
        const int rl = qb * 16 + l16;
#pragma unroll
        for (int h = 0; h < C::NHS; ++h) {
            const int cidx = h * 16 + grp * 4;
            if (cidx < HD) {
                float v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = oacc[qb][h][r] * inv_l;
                if (a.nsplit == 1)
                    store4<bf16_t>(reinterpret_cast<bf16_t*>(so + rl * C::ROWB + (((cidx / 8) ^ (rl & SWM)) * 16) + (cidx % 8) * 2), v);
                else
                    store4<float>(reinterpret_cast<float*>(so + rl * 2 * C::ROWB) + ((cidx / 4) ^ (rl & SWF)) * 4, v);
            }
        }
        const int qrow = row0 + wave * 32 + rl;
        if (a.nsplit > 1 && grp == 0 && qrow < row_end)
            *reinterpret_cast<float2*>(a.part_ml + 2 * (((long)split * a.M + qrow) * a.n_heads + head)) =
                make_float2(m_run[qb], l);
    }
    __syncthreads();
    if (a.nsplit == 1) {
        bf16_t* const dst = static_cast<bf16_t*>(a.o);
        for (int k = lane; k < 32 * CH; k += kWave) {
            const int rl = k / CH, c = k % CH;
            const int qrow = row0 + wave * 32 + rl;
            if (qrow < row_end)
                st16(dst + (long)qrow * d + head * HD + c * 8, ld16(so + rl * C::ROWB + ((c ^ (rl & SWM)) * 16)));
        }
    } else {
        float* const dst = a.part_o + (long)split * a.M * d;
        for (int k = lane; k < 32 * CF; k += kWave) {
            const int rl = k / CF, c = k % CF;
            const int qrow = row0 + wave * 32 + rl;
            if (qrow < row_end)
                st16(dst + (long)qrow * d + head * HD + c * 4, ld16(so + rl * 2 * C::ROWB + ((c ^ (rl & SWF)) * 16)));
        }
    }
}

// Combine of the key-range partials, fixed split order: range s, with running
// max m_s (exp2 domain), sum l_s and normalised output O_s, has weight
// l_s 2^((m_s - m) c) (m the largest m_s, c the log2-domain scale), and the output is the weighted mean of
// the O_s. One thread per 4 columns of a row (16-byte vectors); with the
// split count NS known at compile time every partial of the thread is loaded
// before the first is used (NS = 0: any count, in chunks of 8). The arithmetic
// and its order do not depend on NS.
template <typename T, int NS>
__global__ __launch_bounds__(256) void attention_combine_kernel(AttnDesc a) {
    // running maxima: raw scores from the bf16 kernel, scaled to the log2 domain from the float32 one
    const float mscale = sizeof(T) == 2 ? a.scale_log2 : 1.0f;
    const long n4 = (long)a.M * a.d / 4;
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n4) return;
    const long m = i / (a.d / 4);
    const int col = (int)(i - m * (a.d / 4)) * 4;
    const int head = col / a.hd;
    const int ns = NS > 0 ? NS : a.nsplit;
    auto ml_of = [&](int s) { return a.part_ml + 2 * (((long)s * a.M + m) * a.n_heads + head); };
    auto po_of = [&](int s) { return a.part_o + ((long)s * a.M + m) * a.d + col; };
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    float L = 0.f;
    auto add = [&](float2 ml, float gmax, float4 po) {
        const float w = fast_exp2((ml.x - gmax) * mscale) * ml.y;
        L += w;
        acc[0] += w * po.x; acc[1] += w * po.y; acc[2] += w * po.z; acc[3] += w * po.w;
    };
    constexpr int CH = NS > 0 ? NS : 8;
    float gmax = -INFINITY;
    float2 ml[CH];
    float4 po[CH];
    auto load = [&](int s0) {
#pragma unroll
        for (int j = 0; j < CH; ++j)
            if (NS > 0 || s0 + j < ns) {
                ml[j] = *reinterpret_cast<const float2*>(ml_of(s0 + j));
                po[j] = *reinterpret_cast<const float4*>(po_of(s0 + j));
            }
    };
    if constexpr (NS > 0) {
        load(0);
#pragma unroll
        for (int j = 0; j < CH; ++j) gmax = fmaxf(gmax, ml[j].x);
#pragma unroll
        for (int j = 0; j < CH; ++j) add(ml[j], gmax, po[j]);
    } else {
        for (int s0 = 0; s0 < ns; s0 += CH) {
            float mv[CH];
#pragma unroll
            for (int j = 0; j < CH; ++j) mv[j] = s0 + j < ns ? ml_of(s0 + j)[0] : -INFINITY;
#pragma unroll
            for (int j = 0; j < CH; ++j) gmax = fmaxf(gmax, mv[j]);
        }
        for (int s0 = 0; s0 < ns; s0 += CH) {
            load(s0);
#pragma unroll
            for (int j = 0; j < CH; ++j)
                if (s0 + j < ns) add(ml[j], gmax, po[j]);
        }
    }
    const float inv = 1.0f / L;
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] *= inv;
    store4<T>(static_cast<T*>(a.o) + m * a.d + col, acc);
}

// Columns the float32 kernel pads a head to.
int f32_head_cols(int hd) { return hd <= 32 ? 32 : hd <= 48 ? 48 : 64; }

}  // namespace

// Split of the key range. Workgroups run in rounds of as many as the CUs hold
// (set by the registers of each head_dim). Fitted to forced splits of 176 blocks on
// MI355X (1 to 32 ranges, head_dim 16 to 128, 52 to 2867 rows over 256 to 4096 keys): a
// round with k workgroups per CU takes about 6 + 1.5 (k - 1) us to start and end plus,
// per 64-key tile, the tile's MFMA count times 0.0115 + 0.0067 k us (12% more where an
// odd row length leaves bank conflicts); the combine a launch, the partials' bytes at
// ~6 TB/s and, past eight ranges, 3 us more (partials in chunks of eight, one after
// the other). The planned split is 0.4% behind the best of these blocks (geometric mean,
// worst 4.8%); with 2.5 (k - 1) and no price on more than eight ranges it was 1.5%
// (18%): 230 rows of 3 heads of 128 over 2304 keys 47.1 -> 39.8 us.
// Against a fixed target of 640 workgroups: no split at 16 requests of 10 to 60% of
// 1024 keys (attention and combine 26.2 -> 22.7 us), 512 groups instead of 640 at 1024
// rows of 16 heads of 72 (38.7 -> 36.0).
double attention_cost_us(int dtype, int base, int nsplit, int tps, int hd, int M, int d) {
    // float32, the same terms from splits of 48 blocks at head_dim 32, 40 and 64: a 64-key
    // tile takes (0.020 + 0.042 k) us per padded column with k workgroups on a CU (the
    // second term is the float32 matrix rate), a round 2.0 us + 0.8 per further
    // workgroup. The registers hold four workgroups per CU at 48 and 64 columns and five
    // at 32, where rounds of eight come nearer the measured times (the next workgroups
    // start as the first end). The planned split is 0.8% behind the best of these blocks
    // (geometric mean, worst 4.7%; with rounds of eight, six and four 1.2%, 6.3%).
    // 205 rows of 4 heads of 64 over 1024 keys (16 workgroups unsplit) 67 -> 9 us
    // with the combine, 410 rows of 4 heads over 4096 keys 290 -> 36 us.
    if (dtype != kBF16) {
        const int hdp = f32_head_cols(hd), per_cu = hdp == 32 ? 8 : 4;
        const long groups = (long)base * nsplit, slots = 256L * per_cu, rest = groups % slots;
        auto round_us = [&](long k) { return 2.0 + 0.8 * (k - 1) + tps * hdp * (0.020 + 0.042 * k); };
        double us = (double)(groups / slots) * round_us(per_cu);
        if (rest) us += round_us((rest + 255) / 256);
        if (nsplit > 1) us += 2.5 + 0.1 * nsplit + (4.0 * nsplit + 4) * M * d / 6.0e6;
        return us;
    }
    const int per_cu = hd <= 16 ? 5 : hd <= 48 ? 4 : hd <= 88 ? 3 : 2;
    const int mfmas = 8 * ((hd + 31) / 32) + 4 * ((hd + 15) / 16 + (hd % 16 == 0));
    const double unit = mfmas * (hd % 16 ? 1.12 : 1.0);
    auto round_us = [&](long k) { return tps * unit * (0.0115 + 0.0067 * k) + 6.0 + 1.5 * (k - 1); };
    const long groups = (long)base * nsplit, slots = 256L * per_cu, rest = groups % slots;
    double us = (double)(groups / slots) * round_us(per_cu);
    if (rest) us += round_us((rest + 255) / 256);
    if (nsplit > 1) us += 1.5 + 0.05 * nsplit + (nsplit > 8 ? 3.0 : 0.0) + (4.0 * nsplit + 2) * M * d / 6.0e6;
    return us;
}

// bf16, head_dim a multiple of 8 up to 128: the direct-to-LDS kernel (its
// partials combined below when the key range is split). fp32, head_dim up to
// 64: the register-staged kernel, its key range split and combined the same way.
hipError_t launch_attention(int dtype, const AttnDesc& a, hipStream_t s) {
    if (a.M == 0) return hipSuccess;
    dim3 block(kThreads);
    if (dtype == kBF16) {
        dim3 grid(a.n_qtiles_fast * a.n_heads * a.nsplit);
        switch (a.hd) {
#define MS_HD(n) case n: hipLaunchKernelGGL((attention_dma_kernel<n>), grid, block, 0, s, a); break;
            MS_HD(8) MS_HD(16) MS_HD(24) MS_HD(32) MS_HD(40) MS_HD(48) MS_HD(56) MS_HD(64)
            MS_HD(72) MS_HD(80) MS_HD(88) MS_HD(96) MS_HD(104) MS_HD(112) MS_HD(120) MS_HD(128)
#undef MS_HD
            default: return hipErrorInvalidValue;
        }
    } else {
        if (a.hd > 64) return hipErrorInvalidValue;
        const dim3 grid(a.n_qtiles, a.n_heads, a.nsplit);
        const int cols = f32_head_cols(a.hd);
        if (cols == 32) hipLaunchKernelGGL((attention_f32_kernel<32>), grid, block, 0, s, a);
        else if (cols == 48) hipLaunchKernelGGL((attention_f32_kernel<48>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((attention_f32_kernel<64>), grid, block, 0, s, a);
    }
    return hipGetLastError();
}

template <typename T>
void launch_combine(const AttnDesc& a, hipStream_t s) {
    const long n4 = (long)a.M * a.d / 4;
    const dim3 grid((unsigned)((n4 + 255) / 256)), block(256);
    switch (a.nsplit) {
#define MS_NS(n) case n: hipLaunchKernelGGL((attention_combine_kernel<T, n>), grid, block, 0, s, a); break;
        MS_NS(2) MS_NS(3) MS_NS(4) MS_NS(5) MS_NS(6) MS_NS(7) MS_NS(8)
#undef MS_NS
        default: hipLaunchKernelGGL((attention_combine_kernel<T, 0>), grid, block, 0, s, a); break;
    }
}

hipError_t launch_attention_combine(int dtype, const AttnDesc& a, hipStream_t s) {
    if (a.M == 0 || a.nsplit <= 1) return hipSuccess;
    if (dtype == kBF16) launch_combine<bf16_t>(a, s);
    else launch_combine<float>(a, s);
    return hipGetLastError();
}

}  // namespace ms
