// Dense part of a GraphSAGE-mean layer (Eq. 1 of the paper in its GraphSAGE form):
//   Z = H_self W_self + Agg W_neigh + b  (ReLU on hidden layers), its backward, a fused SGD step,
// and the softmax cross-entropy on the root rows.  The contractions run on the bf16 matrix cores
// (v_mfma_f32_32x32x16_bf16) with float accumulation; operands are staged through LDS.
#include <type_traits>

#include "cr_common.h"
#include "linear_bwd.h"

namespace cr {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4v __attribute__((ext_vector_type(4)));
typedef short v4s16 __attribute__((ext_vector_type(4)));

constexpr int TN_BM = 32;     // rows of the operands staged per step of the TN product (a multiple of 16; 96-row splits hold two)
constexpr int TN_ROW = 160;   // staged row of the TN product: 128 columns + 32 of padding (320 bytes: the four rows that half a wave
                              // reads with one transpose read lie 16 banks apart)

// the larger of the two, NaN if x is one (fmaxf would give the bound instead: 0 under a ReLU, -inf without one)
__device__ __forceinline__ float at_least(float x, float bound) { return __builtin_elementwise_maximum(x, bound); }

constexpr int LDS_ROW = 40;   // 32 bf16 of payload + 8 of padding per staged row (80 bytes)

__device__ __forceinline__ bf16x8 lds_read8(const uint16_t *p)
{
    return *reinterpret_cast<const bf16x8 *>(p);
}

// ------------------------------------------------------------------------------------------------
// C[m][n] = sum_k A[m][k] * B[n][k]     (both operands contiguous along k)
//   A = [A0 | A1]: columns < K0 come from A0, the rest from A1 (same row stride)
//   C = [C0 | C1]: columns < N0 go to C0, the rest to C1 (same row stride)
// Workgroup tile 128 (m) x 64 (n), four waves of 32 x 64; the weights are the first MFMA operand so
// that a lane ends up with four consecutive n of one row m (vector stores along the row).
// ------------------------------------------------------------------------------------------------
struct NtArgs {
    const int32_t *hdr;
    int32_t max_rows;
    const uint16_t *A0, *A1;
    int64_t lda;
    int32_t K0, K;
    const uint16_t *B;       // [N][K]
    int32_t N;
    const float *bias;       // [N] or NULL
    int32_t relu;
    float *C0, *C1;
    int64_t ldc;
    int32_t N0;
    uint16_t *Cb;            // bf16 copy of C (single destination) or NULL
    int64_t ldcb;
};

struct NtState {
    const uint16_t *A0, *A1;
    int K0, K;
    int64_t ga0, ga1;
    const uint16_t *gb;       // B row (n0 + tid/4), chunk column kc*8
    int kc, a_row0, a_row1, b_row, act_row, lr, half;
};

// the pieces one thread fetches for one 32-wide K step: two of A, NB of B (rows b_row + 64*i)
template <int NB>
struct NtFetch {
    u32x4v a0, a1, b0, b1, b2, b3;
};

template <int NB>
__device__ __forceinline__ NtFetch<NB> nt_fetch(const NtState &st, int step)
{
    NtFetch<NB> f;
    const int k0 = step * 32;
    const uint16_t *src = k0 < st.K0 ? st.A0 + k0 : st.A1 + (k0 - st.K0);
    f.a0 = *reinterpret_cast<const u32x4v *>(src + st.ga0 + st.kc * 8);
    f.a1 = *reinterpret_cast<const u32x4v *>(src + st.ga1 + st.kc * 8);
    const uint16_t *b = st.gb + k0;
    f.b0 = *reinterpret_cast<const u32x4v *>(b);
    f.b1 = f.b2 = f.b3 = f.b0;
    if constexpr (NB > 1) f.b1 = *reinterpret_cast<const u32x4v *>(b + (int64_t)64 * st.K);
    if constexpr (NB > 2) {
        f.b2 = *reinterpret_cast<const u32x4v *>(b + (int64_t)128 * st.K);
        f.b3 = *reinterpret_cast<const u32x4v *>(b + (int64_t)192 * st.K);
    }
    return f;
}

// one K step: stage the fetched pieces, barrier, MFMA (wave tile 32 m x NTILES*32 n)
template <int NTILES>
__device__ __forceinline__ void nt_step(const NtState &st, const NtFetch<NTILES / 2> &f, int &buf,
                                        uint16_t (&As)[2][128][LDS_ROW], uint16_t (&Bs)[2][NTILES * 32][LDS_ROW],
                                        f32x16 (&acc)[NTILES])
{
    constexpr int NB = NTILES / 2;
    *reinterpret_cast<u32x4v *>(&As[buf][st.a_row0][st.kc * 8]) = f.a0;
    *reinterpret_cast<u32x4v *>(&As[buf][st.a_row1][st.kc * 8]) = f.a1;
    *reinterpret_cast<u32x4v *>(&Bs[buf][st.b_row][st.kc * 8]) = f.b0;
    if constexpr (NB > 1) *reinterpret_cast<u32x4v *>(&Bs[buf][st.b_row + 64][st.kc * 8]) = f.b1;
    if constexpr (NB > 2) {
        *reinterpret_cast<u32x4v *>(&Bs[buf][st.b_row + 128][st.kc * 8]) = f.b2;
        *reinterpret_cast<u32x4v *>(&Bs[buf][st.b_row + 192][st.kc * 8]) = f.b3;
    }
    __syncthreads();               // tile `buf` is complete; everyone is also done reading tile `buf ^ 1`
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        const int ko = kk * 16 + 8 * st.half;
        const bf16x8 act = lds_read8(&As[buf][st.act_row][ko]);
#pragma unroll
        for (int t = 0; t < NTILES; ++t) {
            const bf16x8 wgt = lds_read8(&Bs[buf][t * 32 + st.lr][ko]);
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wgt, act, acc[t], 0, 0, 0);
        }
    }
    buf ^= 1;
}

// ------------------------------------------------------------------------------------------------
// Workgroup tile 128 (m) x NTILES*32 (n), four waves of 32 x NTILES*32; the weights are the first MFMA
// operand so that a lane ends up with four consecutive n of one row m (vector stores along the row).
// K is consumed in chunks of CH 32-wide steps (single steps for the remainder): every global load of a
// chunk is issued before the first one is used, so a chunk costs one memory round trip; its steps then
// go through double-buffered LDS tiles with one barrier each.  NTILES = 8 covers a whole 256-wide
// layer, so the activations are read once (see launch_nt for why it is not the default).
// ------------------------------------------------------------------------------------------------
template <int NTILES, int CH>
__device__ __forceinline__ void gemm_nt_body(const NtArgs &a, uint32_t bid, uint32_t ncol, uint16_t (&As)[2][128][LDS_ROW],
                                             uint16_t (&Bs)[2][NTILES * 32][LDS_ROW])
{
    constexpr int BN = NTILES * 32, NB = NTILES / 2;
    const int M = min(a.hdr[CR_HDR_N_DST], a.max_rows);
    // the column tiles of one row tile run next to each other on one XCD: the activations come from HBM once
    uint32_t tile;
    if (!xcd_compact(bid, (uint32_t)((M + 127) / 128) * ncol, tile)) return;
    const int m0 = (int)(tile / ncol) * 128, n0 = (int)(tile % ncol) * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, lr = lane & 31;

    // staging assignment: A 128 rows x 4 chunks of 8, two per thread; B BN rows x 4 chunks, NB per thread
    const int a_row0 = tid >> 2, a_row1 = (tid + 256) >> 2, kc = tid & 3;
    const int64_t ga0 = (int64_t)min(m0 + a_row0, M - 1) * a.lda;
    const int64_t ga1 = (int64_t)min(m0 + a_row1, M - 1) * a.lda;
    const uint16_t *gb = a.B + (int64_t)(n0 + (tid >> 2)) * a.K + kc * 8;

    // (the accumulators start from the bias, which travels with the first chunk; added behind the loop it was a round trip of its own)
    f32x16 acc[NTILES];
#pragma unroll
    for (int t = 0; t < NTILES; ++t)
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) {
            const float4 bq = a.bias ? *reinterpret_cast<const float4 *>(a.bias + n0 + t * 32 + 8 * grp + 4 * half) : make_float4(0.f, 0.f, 0.f, 0.f);
            acc[t][grp * 4 + 0] = bq.x; acc[t][grp * 4 + 1] = bq.y; acc[t][grp * 4 + 2] = bq.z; acc[t][grp * 4 + 3] = bq.w;
        }

    const int nsteps = a.K / 32;
    int buf = 0;
    NtState st{a.A0, a.A1, a.K0, a.K, ga0, ga1, gb, kc, a_row0, a_row1, tid >> 2, wave * 32 + lr, lr, half};
    int s0 = 0;
    for (; s0 + CH <= nsteps; s0 += CH) {
        NtFetch<NB> f[CH];
#pragma unroll
        for (int i = 0; i < CH; ++i) f[i] = nt_fetch<NB>(st, s0 + i);
#pragma unroll
        for (int i = 0; i < CH; ++i) nt_step<NTILES>(st, f[i], buf, As, Bs, acc);
    }
    while (s0 < nsteps) {         // the remaining steps (K not a multiple of 32 * CH), again fetched together: up to three at a time
        const int rem = nsteps - s0;
        const NtFetch<NB> f0 = nt_fetch<NB>(st, s0), f1 = nt_fetch<NB>(st, min(s0 + 1, nsteps - 1)),
                          f2 = nt_fetch<NB>(st, min(s0 + 2, nsteps - 1));
        nt_step<NTILES>(st, f0, buf, As, Bs, acc);
        if (rem > 1) nt_step<NTILES>(st, f1, buf, As, Bs, acc);
        if (rem > 2) nt_step<NTILES>(st, f2, buf, As, Bs, acc);
        s0 += 3;
    }

    // Epilogue through LDS (the staging tiles are free after one more barrier): a lane holds 4-column pieces of one
    // row, which would go out as 8/16-byte stores scattered over 32 rows; staged, a wave writes whole 128-byte row
    // segments.  Each wave uses its own quarter of As.
    static_assert(NTILES == 2, "the staged epilogue is laid out for a 32 x 64 wave tile");
    __syncthreads();
    char *region = reinterpret_cast<char *>(&As[0][0][0]) + wave * (2 * 128 * LDS_ROW * 2 / 4);     // 5120 bytes
    const int mw = m0 + wave * 32;
    float v[2][4][4];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[t][grp][i] = acc[t][grp * 4 + i];
            if (a.relu) {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[t][grp][i] = v[t][grp][i] < 0.f ? 0.f : v[t][grp][i];
            }
        }
    if (a.Cb) {      // both 32-column halves at once: rows of 64 bf16 (+8 of padding)
        uint16_t (*ob)[72] = reinterpret_cast<uint16_t (*)[72]>(region);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) {
                const uint32_t lo = pack_bf16x2(v[t][grp][0], v[t][grp][1]);
                const uint32_t hi = pack_bf16x2(v[t][grp][2], v[t][grp][3]);
                *reinterpret_cast<uint2 *>(&ob[lr][t * 32 + 8 * grp + 4 * half]) = make_uint2(lo, hi);
            }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int c = it * 64 + lane, row = c >> 3, c8 = (c & 7) * 8;
            const u32x4v x = *reinterpret_cast<const u32x4v *>(&ob[row][c8]);
            if (mw + row < M) *reinterpret_cast<u32x4v *>(a.Cb + (int64_t)(mw + row) * a.ldcb + n0 + c8) = x;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    if (a.C0) {      // one 32-column half at a time: rows of 32 floats (+4 of padding)
        float (*of)[36] = reinterpret_cast<float (*)[36]>(region);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int grp = 0; grp < 4; ++grp)
                *reinterpret_cast<float4 *>(&of[lr][8 * grp + 4 * half]) = make_float4(v[t][grp][0], v[t][grp][1], v[t][grp][2], v[t][grp][3]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int c = it * 64 + lane, row = c >> 3, c4 = (c & 7) * 4;
                const float4 x = *reinterpret_cast<const float4 *>(&of[row][c4]);
                const int n = n0 + t * 32 + c4;
                if (mw + row < M) {
                    float *dst = n < a.N0 ? a.C0 + (int64_t)(mw + row) * a.ldc + n : a.C1 + (int64_t)(mw + row) * a.ldc + (n - a.N0);
                    *reinterpret_cast<float4 *>(dst) = x;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    }
}

// Register budget: up to four waves per SIMD.  Four K steps of prefetch at this occupancy measured faster
// than eight steps at two waves per SIMD on the products that fill the chip; a product with few workgroups and a
// long K loop (the reddit-like input layer: 88 row tiles, K = 1216) gains nothing from occupancy and takes the
// eight-step instantiation, which halves the round trips of its K loop.
template <int NTILES, int CH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(CH == 4 ? 3 : 1, CH == 4 ? 4 : 2))) void gemm_nt_kernel(NtArgs a)
{
    __shared__ __attribute__((aligned(16))) uint16_t As[2][128][LDS_ROW];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[2][NTILES * 32][LDS_ROW];
    gemm_nt_body<NTILES, CH>(a, blockIdx.y * gridDim.x + blockIdx.x, gridDim.x, As, Bs);
}

// ------------------------------------------------------------------------------------------------
// The same product for blocks of few rows (the layers next to the roots: about a thousand rows), where the tiled
// kernel above leaves most of the chip idle and spends its time in K steps taken one after another.  Workgroup tile
// 32 (m) x 64 (n); K is taken in chunks of 256 columns, two of them on their way at once, which are K = 512's single round trip
// to memory.  They travel as whole rows (half a wave reads 512 contiguous bytes) and through LDS: with the MFMA fragments straight
// from memory, 16 bytes of 32 rows per load, the kernel was bound by the address unit (4.5 of 7.5 us for 1024 x 512 -> 192; the
// kernel now takes 5.0; 64 rows x 128 -> 64 with the loss 8.1 -> 5.8).  The loads do not wait for the row count.  The four waves split a chunk between them (wave w takes the
// 16-wide steps w, w + 4, ...); their partial tiles meet in LDS and are added in a fixed order.
// ------------------------------------------------------------------------------------------------
constexpr int SMALL_KC = 256;
constexpr int SMALL_LROW = SMALL_KC + 8;        // staged row: 256 bf16 + 8 of padding
constexpr int SMALL_ROW = 68;     // floats per staged row: 64 + 4 of padding (272 bytes, keeps 16-byte alignment)

// loss part of the fused top-layer launch (XENT == true): the product's rows are the roots, its columns the classes
struct XentArgs {
    int32_t n_classes;
    const int32_t *labels, *root_ids;
    float *loss, *row_loss;
    uint16_t *d_logits_bf16;      // [max_rows][64]
    unsigned long long *acc;      // tickets and the fixed-point sum of the workgroups' loss shares; zero between calls
};

// XENT == true (one column tile: at most 64 classes; no ReLU, no bf16 copy): a workgroup holds whole rows of
// logits after the reduction, so the softmax cross-entropy of its rows, their gradient and its share of the mean
// loss are taken right there; the shares meet in one device-side accumulator.
template <bool XENT>
__global__ __launch_bounds__(256) void gemm_nt_small_kernel(NtArgs a, XentArgs x)
{
    __shared__ __attribute__((aligned(16))) uint16_t tile[(32 + 64) * SMALL_LROW];      // A's rows, then B's
    __shared__ float wg_loss[32];
    float (*red)[32][SMALL_ROW] = reinterpret_cast<float (*)[32][SMALL_ROW]>(tile);      // [4], once the staged rows are done with
    static_assert(4 * 32 * SMALL_ROW * sizeof(float) <= sizeof(tile), "the partial tiles fit the staged rows' room");
    const int m0 = (int)blockIdx.y * 32, n0 = (int)blockIdx.x * 64;
    const int K = a.K, nchunk = (K + SMALL_KC - 1) / SMALL_KC;
    // staging: piece p = i * 256 + thread = (row p / 32, 16-byte piece p % 32): four of A and eight of B per thread; pieces past
    // the end of K repeat the first one and are not used
    const int srow = (int)threadIdx.x >> 5, spiece = ((int)threadIdx.x & 31) * 8;
    auto fetch = [&](u32x4v (&f)[12], int c) {
        const int k = c * SMALL_KC + spiece < K ? c * SMALL_KC + spiece : 0;
        const uint16_t *src = k < a.K0 ? a.A0 + k : a.A1 + (k - a.K0);
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = *reinterpret_cast<const u32x4v *>(src + (int64_t)min(m0 + i * 8 + srow, a.max_rows - 1) * a.lda);
#pragma unroll
        for (int i = 0; i < 8; ++i) f[4 + i] = *reinterpret_cast<const u32x4v *>(a.B + (int64_t)(n0 + i * 8 + srow) * K + k);
    };
    auto stage = [&](const u32x4v (&f)[12]) {
#pragma unroll
        for (int i = 0; i < 12; ++i) *reinterpret_cast<u32x4v *>(&tile[(i * 8 + srow) * SMALL_LROW + spiece]) = f[i];
    };
    u32x4v f0[12], f1[12];
    fetch(f0, 0);
    if (nchunk > 1) fetch(f1, 1);
    const int M = min(a.hdr[CR_HDR_N_DST], a.max_rows);
    if (XENT && M <= 0) {
        if (blockIdx.y == 0 && threadIdx.x == 0) x.loss[0] = 0.f;
        return;
    }
    if (m0 >= M) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, lr = lane & 31;
    const int nk = a.K / 16;
    // the label of the row this thread will finish: requested now (two dependent loads), used after the product
    int label = 0;
    if constexpr (XENT) label = x.labels[x.root_ids[min(m0 + (tid >> 3), M - 1)]];
    const int c8 = (tid & 7) * 8, n = n0 + c8;
    float4 q0 = make_float4(0.f, 0.f, 0.f, 0.f), q1 = q0;
    if (a.bias) {
        q0 = *reinterpret_cast<const float4 *>(a.bias + n);
        q1 = *reinterpret_cast<const float4 *>(a.bias + n + 4);
    }

    f32x16 acc[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;

    auto multiply = [&](int c) {
        const int steps = min(SMALL_KC / 16, nk - c * (SMALL_KC / 16));
#pragma unroll
        for (int i = 0; i < SMALL_KC / 64; ++i) {
            const int s = wave + 4 * i;
            if (s >= steps) break;                              // (uniform over the wave)
            const uint16_t *p = tile + s * 16 + 8 * half;
            const bf16x8 act = lds_read8(p + lr * SMALL_LROW);
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_read8(p + (32 + lr) * SMALL_LROW), act, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_read8(p + (64 + lr) * SMALL_LROW), act, acc[1], 0, 0, 0);
        }
        __syncthreads();                                        // the staged rows are done with
    };
    for (int c = 0; c < nchunk; c += 2) {
        stage(f0);
        __syncthreads();
        if (c + 2 < nchunk) fetch(f0, c + 2);
        multiply(c);
        if (c + 1 >= nchunk) break;
        stage(f1);
        __syncthreads();
        if (c + 3 < nchunk) fetch(f1, c + 3);
        multiply(c + 1);
    }
    // a lane holds, for row lr, the columns t*32 + 8*grp + 4*half .. + 4
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int grp = 0; grp < 4; ++grp)
            *reinterpret_cast<float4 *>(&red[wave][lr][t * 32 + 8 * grp + 4 * half]) =
                make_float4(acc[t][grp * 4 + 0], acc[t][grp * 4 + 1], acc[t][grp * 4 + 2], acc[t][grp * 4 + 3]);
    __syncthreads();
    const int row = tid >> 3;
    if (!XENT && m0 + row >= M) return;
    const bool row_ok = m0 + row < M;
    float v[8];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const float4 p0 = *reinterpret_cast<const float4 *>(&red[0][row][c8 + 4 * h]), p1 = *reinterpret_cast<const float4 *>(&red[1][row][c8 + 4 * h]);
        const float4 p2 = *reinterpret_cast<const float4 *>(&red[2][row][c8 + 4 * h]), p3 = *reinterpret_cast<const float4 *>(&red[3][row][c8 + 4 * h]);
        v[4 * h + 0] = (p0.x + p1.x) + (p2.x + p3.x); v[4 * h + 1] = (p0.y + p1.y) + (p2.y + p3.y);
        v[4 * h + 2] = (p0.z + p1.z) + (p2.z + p3.z); v[4 * h + 3] = (p0.w + p1.w) + (p2.w + p3.w);
    }
    if (a.bias) {
        v[0] += q0.x; v[1] += q0.y; v[2] += q0.z; v[3] += q0.w; v[4] += q1.x; v[5] += q1.y; v[6] += q1.z; v[7] += q1.w;
    }
    if (a.relu) {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = v[i] < 0.f ? 0.f : v[i];
    }
    const int64_t m = min(m0 + row, M - 1);
    if (a.C0 && row_ok) {
        float *dst = n < a.N0 ? a.C0 + m * a.ldc + n : a.C1 + m * a.ldc + (n - a.N0);    // (N0 is a multiple of 32: no piece straddles)
        *reinterpret_cast<float4 *>(dst) = make_float4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<float4 *>(dst + 4) = make_float4(v[4], v[5], v[6], v[7]);
    }
    if (a.Cb && row_ok) {
        u32x4v xb;
#pragma unroll
        for (int i = 0; i < 4; ++i) xb[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
        *reinterpret_cast<u32x4v *>(a.Cb + m * a.ldcb + n) = xb;
    }
    if constexpr (XENT) {
        // the eight threads of a row sit in eight neighbouring lanes; rows past the last one compute on row M - 1 and store nothing
        const int C = x.n_classes;
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 8; ++i) mx = fmaxf(mx, n + i < C ? v[i] : -INFINITY);
#pragma unroll
        for (int off = 1; off < 8; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
        float e[8], den = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            e[i] = n + i < C ? expf(v[i] - mx) : 0.f;
            den += e[i];
        }
#pragma unroll
        for (int off = 1; off < 8; off <<= 1) den += __shfl_xor(den, off);
        const float inv_n = 1.0f / (float)M;
        u32x4v dq;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float d0 = 0.f, d1 = 0.f;
            if (n + 2 * i < C) d0 = (e[2 * i] / den - (n + 2 * i == label ? 1.f : 0.f)) * inv_n;
            if (n + 2 * i + 1 < C) d1 = (e[2 * i + 1] / den - (n + 2 * i + 1 == label ? 1.f : 0.f)) * inv_n;
            dq[i] = pack_bf16x2(d0, d1);
        }
        if (row_ok) *reinterpret_cast<u32x4v *>(x.d_logits_bf16 + m * 64 + n) = dq;
        if ((tid & 7) == 0) wg_loss[row] = 0.f;
        __syncthreads();
        if (label >= n && label < n + 8) {          // the thread that holds the label's logit
            float zl = v[0];
#pragma unroll
            for (int i = 1; i < 8; ++i) zl = label == n + i ? v[i] : zl;
            const float rl = -(zl - mx - logf(den));
            if (row_ok) { x.row_loss[m] = rl; wg_loss[row] = rl; }
        }
        __syncthreads();
        if (tid < 64) {
            float t = tid < 32 ? wg_loss[tid] : 0.f;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off);
            if (tid == 0) {
                // One 64-bit atomic per workgroup carries its share of the loss (fixed point, 2^-20, bits 0..39: integer
                // sums do not depend on the order of arrival, so the mean is reproducible), a ticket (bits 40..55) and a
                // mark for a share that is not finite (bits 56..62).  The workgroup whose ticket is the last one has the
                // whole sum in hand.  No fence, no access to another workgroup's data: the atomic is performed at the
                // memory side.
                const bool finite = t == t && fabsf(t) <= 8192.0f;       // 32 rows of at most ~100 each
                const unsigned long long share = finite ? (unsigned long long)(fmaxf(t, 0.f) * 1048576.0f + 0.5f) : 0ull;
                const unsigned long long add = share | (1ull << 40) | (finite ? 0ull : 1ull << 56);
                const unsigned long long after = __hip_atomic_fetch_add(x.acc, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + add;
                if ((int)((after >> 40) & 0xFFFFull) == (M + 31) / 32) {
                    const float mean = (float)((double)(after & ((1ull << 40) - 1ull)) * (1.0 / 1048576.0) / (double)M);
                    x.loss[0] = (after >> 56) ? __builtin_nanf("") : mean;
                    __hip_atomic_store(x.acc, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// The same product for the input layer of the large workloads: tens of thousands of rows, N = 256, any K (K <= 256 takes
// the streaming kernel further down; this one serves wider inputs, e.g. 602 features.  GraphSAGE: self | aggregate;
// one-operand layers: all of K from one array).  The tiled kernel above reads every activation row four times (once per 64-column
// tile) and spends most of its time moving operands; here a workgroup takes 128 rows and ALL columns, so activations pass
// through a compute unit once:
//   - K is taken in chunks of 64 columns, each operand array's columns in chunks of their own (an array's last chunk may
//     hold 32).  A chunk is fetched with coalesced 16-byte loads, four pieces of activations and eight of weights per thread,
//     while the chunk before it is multiplied, and laid out in LDS with rows padded by 16 bytes, so that the MFMA fragments are
//     conflict-free 16-byte LDS reads;
//   - a wave owns 64 rows x 128 columns: per 16-wide K step six fragment reads feed eight MFMAs (LDS and matrix cores are about
//     equally busy);
//   - 55 KB of LDS and at most 256 registers: two workgroups per compute unit, two waves per SIMD.  One workgroup's MFMAs run
//     while the other stages, waits at a barrier or stores.  That is what the kernel is built around: 256-row tiles of four waves
//     alone on their compute unit (chunks of 128 columns, 256 accumulators per lane) took 73 us for 131 K rows x 608 -> 256
//     where this takes 67, and a last round of few tiles costs half as much with tiles of half the height;
//   - the accumulators start from the bias; ReLU and the bf16 conversion happen on the way through LDS again, from
//     where 256-byte row pieces leave.
// ------------------------------------------------------------------------------------------------
constexpr int WIDE_ROWS = 128;          // rows per workgroup
constexpr int WIDE_KC = 64;             // K of one chunk
constexpr int WIDE_N = 256;
constexpr int WIDE_LROW = WIDE_KC + 8;  // staged row: 64 bf16 + 8 of padding (144 bytes)
constexpr int WIDE_OROW = 128 + 8;      // staged output row of one wave

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_nt_wide_kernel(NtArgs a)
{
    constexpr int KSTEPS = WIDE_KC / 16, AP = WIDE_ROWS * 8 / 256, WP = WIDE_N * 8 / 256;     // pieces of 16 bytes per thread
    __shared__ __attribute__((aligned(16))) uint16_t lds[(WIDE_ROWS + WIDE_N) * WIDE_LROW];
    __shared__ __attribute__((aligned(16))) float bias_s[WIDE_N];
    uint16_t *As = lds;                                        // [128 m][WIDE_LROW]
    uint16_t *Ws = lds + WIDE_ROWS * WIDE_LROW;                // [256 n][WIDE_LROW]
    static_assert(4 * 32 * WIDE_OROW <= (WIDE_ROWS + WIDE_N) * WIDE_LROW, "output staging must fit");
    const int M = min(a.hdr[CR_HDR_N_DST], a.max_rows);
    if ((int)blockIdx.x * WIDE_ROWS >= M) return;
    // the last tile is moved back so that it ends at the last row: it recomputes a few rows of its neighbour (same
    // values, written twice) and no load has to be clamped to the row count.  With fewer than 128 rows the one tile
    // reads rows past the last one: they exist (the arrays hold max_rows >= 16384 rows), rows are independent, and
    // results past the last row are not stored.
    const int m0 = max(0, min((int)blockIdx.x * WIDE_ROWS, M - WIDE_ROWS));
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, lr = lane & 31;
    const int wr = (wave & 1) * 64, wc = (wave >> 1) * 128;    // this wave's rows and columns of the tile
    const int K = a.K, K0 = a.K0;
    // Column k of the product sits in the first operand array for k < K0 and in the second from there on.  Each array's
    // columns are taken in chunks of their own (the first array's chunks, then the second's), so a chunk lies in one array
    // whatever K0 is.  Widths are multiples of 32: an array's last chunk holds 64 columns or 32.
    const int nchunk0 = (K0 + WIDE_KC - 1) / WIDE_KC;
    const int nchunk = nchunk0 + (K - K0 + WIDE_KC - 1) / WIDE_KC;
    auto chunk_off = [&](int c) { return (c < nchunk0 ? c : c - nchunk0) * WIDE_KC; };
    auto chunk_cols = [&](int c) { return min(WIDE_KC, (c < nchunk0 ? K0 : K - K0) - chunk_off(c)); };

    // staging assignment: piece p = i * 256 + tid of a chunk = (row p / 8, 16-byte piece p % 8).  An address is a base that is
    // the same for the whole workgroup (chunk, 32-row group i) plus one per-thread offset that serves all pieces of an
    // operand.  Pieces past a chunk of 32 columns are loaded from the chunk's first piece and not staged.
    const int srow = tid >> 3, spiece = tid & 7;
    // (past the last chunk its own pieces are fetched again: a load under a condition would be waited for at once)
    u32x4v wreg[WP], areg0[AP], areg1[AP];
    auto fetch_a = [&](u32x4v (&r)[AP], int c0) {
        const int c = min(c0, nchunk - 1);
        const int sp = spiece * 8 < chunk_cols(c) ? spiece * 8 : 0;
        const uint16_t *A = (c < nchunk0 ? a.A0 : a.A1) + chunk_off(c) + (int64_t)m0 * a.lda;
#pragma unroll
        for (int i = 0; i < AP; ++i) r[i] = *reinterpret_cast<const u32x4v *>(A + (int64_t)(i * 32) * a.lda + (uint32_t)(srow * (int)a.lda + sp));
    };
    auto fetch_w = [&](int c0) {
        const int c = min(c0, nchunk - 1);
        const int sp = spiece * 8 < chunk_cols(c) ? spiece * 8 : 0;
        const uint16_t *W = a.B + (c < nchunk0 ? 0 : K0) + chunk_off(c);
#pragma unroll
        for (int i = 0; i < WP; ++i) wreg[i] = *reinterpret_cast<const u32x4v *>(W + (int64_t)(i * 32) * K + (uint32_t)(srow * K + sp));
    };
    auto stage = [&](const u32x4v (&r)[AP], int c) {
        if (spiece * 8 >= chunk_cols(c)) return;
#pragma unroll
        for (int i = 0; i < AP; ++i) *reinterpret_cast<u32x4v *>(&As[(i * 32 + srow) * WIDE_LROW + spiece * 8]) = r[i];
#pragma unroll
        for (int i = 0; i < WP; ++i) *reinterpret_cast<u32x4v *>(&Ws[(i * 32 + srow) * WIDE_LROW + spiece * 8]) = wreg[i];
    };
    fetch_a(areg0, 0);
    fetch_w(0);
    fetch_a(areg1, 1);
    if (tid < WIDE_N / 4)
        *reinterpret_cast<float4 *>(&bias_s[tid * 4]) = a.bias ? *reinterpret_cast<const float4 *>(a.bias + tid * 4) : make_float4(0.f, 0.f, 0.f, 0.f);
    stage(areg0, 0);
    __syncthreads();

    // the accumulators start from the bias (a lane's 4-column pieces: columns wc + t*32 + 8*grp + 4*half .. + 4)
    f32x16 acc[2][4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) {
            const float4 bq = *reinterpret_cast<const float4 *>(&bias_s[wc + t * 32 + 8 * grp + 4 * half]);
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) {
                acc[rb][t][grp * 4 + 0] = bq.x; acc[rb][t][grp * 4 + 1] = bq.y; acc[rb][t][grp * 4 + 2] = bq.z; acc[rb][t][grp * 4 + 3] = bq.w;
            }
        }
    const uint16_t *arow0 = As + (wr + lr) * WIDE_LROW + 8 * half, *arow1 = arow0 + 32 * WIDE_LROW;
    const uint16_t *wrow = Ws + (wc + lr) * WIDE_LROW + 8 * half;
    auto step = [&](int ks) {
        const bf16x8 a0 = lds_read8(arow0 + ks * 16), a1 = lds_read8(arow1 + ks * 16);
        bf16x8 w[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) w[t] = lds_read8(wrow + t * 32 * WIDE_LROW + ks * 16);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            acc[0][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[t], a0, acc[0][t], 0, 0, 0);
            acc[1][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[t], a1, acc[1][t], 0, 0, 0);
        }
    };
    // chunk c is in LDS, the activations of chunk c + 1 are on their way in `next`, those of c + 2 go to `after`
    auto chunk = [&](int c, const u32x4v (&next)[AP], u32x4v (&after)[AP]) {
        fetch_w(c + 1);
        fetch_a(after, c + 2);
        step(0);
        step(1);
        if (chunk_cols(c) > 32) {                              // (uniform)
#pragma unroll
            for (int ks = 2; ks < KSTEPS; ++ks) step(ks);
        }
        __syncthreads();                                       // every wave is done reading this chunk
        stage(next, min(c + 1, nchunk - 1));
        __syncthreads();
    };
    for (int c = 0; c < nchunk; c += 2) {
        chunk(c, areg1, areg0);
        if (c + 1 >= nchunk) break;
        chunk(c + 1, areg0, areg1);
    }

    // epilogue: ReLU, bf16, 32 rows at a time; a lane holds, for row lr of each block, the columns t*32 + 8*grp + 4*half .. + 4
    const float floor_v = a.relu ? 0.f : -INFINITY;
    uint16_t *ob = lds + wave * 32 * WIDE_OROW;
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) {
                const float v0 = at_least(acc[rb][t][grp * 4 + 0], floor_v), v1 = at_least(acc[rb][t][grp * 4 + 1], floor_v);
                const float v2 = at_least(acc[rb][t][grp * 4 + 2], floor_v), v3 = at_least(acc[rb][t][grp * 4 + 3], floor_v);
                *reinterpret_cast<uint2 *>(&ob[lr * WIDE_OROW + t * 32 + 8 * grp + 4 * half]) = make_uint2(pack_bf16x2(v0, v1), pack_bf16x2(v2, v3));
            }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const int mw = m0 + wr + rb * 32;
#pragma unroll
        for (int it = 0; it < 8; ++it) {
            const int c = it * 64 + lane, row = c >> 4, c8 = (c & 15) * 8;
            const u32x4v x = *reinterpret_cast<const u32x4v *>(&ob[row * WIDE_OROW + c8]);
            if (mw + row < M) *reinterpret_cast<u32x4v *>(a.Cb + (int64_t)(mw + row) * a.ldcb + wc + c8) = x;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

// ------------------------------------------------------------------------------------------------
// The same product again for K <= 256 (the input layer of the papers-like workload: 2 x 128 features): the weights
// of a wave's 64 output columns fit its registers (64 x 256 bf16 = 128 registers per lane), so they are fetched once
// per workgroup and only activations pass through LDS.  One persistent workgroup per compute unit walks over tiles
// of 64 rows (tile t, t + gridDim.x, ..):
//   - a tile's activations (64 rows x K) travel global -> registers -> LDS; the loads of tiles t+1 and t+2 are in
//     flight while tile t is multiplied (two register sets, two LDS buffers, one barrier per tile), so a compute unit
//     keeps two tiles (64 KB) on the way and the chip about 16 MB: enough to cover the memory latency at full rate;
//   - a wave multiplies all 64 rows by its own 64 columns: per 16-wide K step two fragment reads feed four MFMAs
//     (the activation fragments are the only LDS reads of the K loop);
//   - bias, ReLU and the bf16 conversion happen in the wave's own LDS patch, from where 128-byte row pieces leave;
//     the stores of tile t overlap the loads of the tiles behind it.
// With K = N = 256 the product moves 1 KB per row against 131 K multiply-adds: even at the full memory rate the matrix
// cores can be busy for about 30 % of the time at most.
// ------------------------------------------------------------------------------------------------
constexpr int STREAM_ROWS = 64;
constexpr int STREAM_KMAX = 256;
constexpr int STREAM_LROW = STREAM_KMAX + 8;    // staged activation row: 256 bf16 + 8 of padding (528 bytes)
constexpr int STREAM_OROW = 64 + 8;             // staged output row of one wave
constexpr size_t STREAM_LDS_BYTES = ((size_t)2 * STREAM_ROWS * STREAM_LROW + (size_t)4 * STREAM_ROWS * STREAM_OROW) * sizeof(uint16_t) +
                                    WIDE_N * sizeof(float);

// KS: 16-wide K steps held in registers (8: K <= 128, 16: K <= 256; columns from K on count as zeros).  FULL: at least
// 64 rows, so that every tile is a whole one and nothing in the tile loop is conditional: every wait on the counter of
// outstanding memory operations then leaves exactly the newer loads and stores in flight.
// UNIFORM: each wave's sixteen pieces of a row lie in one operand array (K0 = K or a multiple of 128): a load address is
// then a base that is the same for the whole wave (array, tile, row group) plus one 32-bit offset per thread that never
// changes, so no address registers are computed per tile (the compiler puts such temporaries into the registers the
// previous tile's loads went to, and then waits for loads that have long been consumed).
template <int KS, bool FULL, bool UNIFORM>
__device__ __forceinline__ void nt_stream_body(const NtArgs &a, const int M, uint16_t *stream_lds, u32x4v (&wraw)[KS])
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, lr = lane & 31;
    uint16_t *As0 = stream_lds, *As1 = stream_lds + STREAM_ROWS * STREAM_LROW;
    uint16_t *ob = stream_lds + 2 * STREAM_ROWS * STREAM_LROW + wave * STREAM_ROWS * STREAM_OROW;
    float *bias_s = reinterpret_cast<float *>(stream_lds + 2 * STREAM_ROWS * STREAM_LROW + 4 * STREAM_ROWS * STREAM_OROW);
    const int ntiles = (M + STREAM_ROWS - 1) / STREAM_ROWS;
    const int K = a.K, K0 = a.K0;

    // staging: a thread moves the same 16-byte piece (columns 8 kp ..) of eight rows (srow, srow + 8, ..) of every tile;
    // a wave covers 16 pieces (256 bytes) of four rows per load.
    // The last tile is moved back so that it ends at the last row (it recomputes rows of its neighbour: same values,
    // written twice); with fewer than 64 rows the one tile reads rows past the last one: they exist (the arrays hold
    // max_rows >= 16384 rows), rows are independent, and results past the last row are not stored.  A fetch for a tile
    // past the last one, or of a piece past K, still issues its eight loads (all of the first operand's first bytes).
    const int uwave = __builtin_amdgcn_readfirstlane(wave);
    const int kp = (lane & 15) + 16 * (uwave & 1), srow = (lane >> 4) + 4 * (uwave >> 1);
    const bool mine = kp * 8 < K;
    const uint16_t *col_src = !mine ? a.A0 : (kp * 8 < K0 ? a.A0 + kp * 8 : a.A1 + (kp * 8 - K0));
    // (UNIFORM: the wave's array, the second one addressed from K0 columns in front of it; the host has checked that
    // the arrays are shorter than 2^31 bytes)
    const bool second = 128 * (uwave & 1) >= K0;
    const uint64_t base_v = reinterpret_cast<uint64_t>(second ? a.A1 - K0 : a.A0);
    const uint16_t *wave_src = reinterpret_cast<const uint16_t *>(
        ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(base_v >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((int)base_v));
    const uint32_t ld_bytes = (uint32_t)__builtin_amdgcn_readfirstlane((int)(a.lda * 2));
    const uint32_t records = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)a.max_rows * ld_bytes + (second ? 2u * (uint32_t)K0 : 0u)));
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(wave_src), 0, (int)records, 0x00020000);
    // (a thread without a piece of its own -- columns from K on -- reads its array's first bytes: with the second array
    // that is K0 columns past the shifted base, not the base itself, which lies in front of the array)
    const uint32_t lane_off = mine ? (uint32_t)srow * ld_bytes + 16u * (uint32_t)kp : (second ? 2u * (uint32_t)K0 : 0u);
    auto tile_m0 = [&](int t) { return max(0, min(t * STREAM_ROWS, M - STREAM_ROWS)); };
    auto fetch = [&](u32x4v (&r)[8], int t) {
        if constexpr (UNIFORM) {
            // buffer loads: descriptor and row offset in scalar registers, the thread's offset in one register that
            // never changes (a tile past the last one: the first tile's rows again, they exist)
            const uint32_t row0 = t < ntiles ? (uint32_t)tile_m0(t) : 0u;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                r[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)lane_off, (int)((row0 + 8u * i) * ld_bytes), 0);
        } else {
            const bool real = mine && t < ntiles;
            const int64_t ld = real ? a.lda : 0;
            const uint16_t *src = real ? col_src + (int64_t)(tile_m0(t) + srow) * ld : a.A0;
#pragma unroll
            for (int i = 0; i < 8; ++i) r[i] = *reinterpret_cast<const u32x4v *>(src + (int64_t)(8 * i) * ld);
        }
    };
    auto stage = [&](uint16_t *As, const u32x4v (&r)[8]) {
        if (!mine) return;
#pragma unroll
        for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x4v *>(&As[(8 * i + srow) * STREAM_LROW + kp * 8]) = r[i];
    };
    const int step = (int)gridDim.x;
    int t = (int)blockIdx.x;
    u32x4v ra[8], rb[8];
    fetch(ra, t);
    fetch(rb, t + step);
    // The wave's weights, which came as whole rows, through its quarter of the activations' buffers into registers: columns
    // 64 wave + 32 cb + lr, eight k from 16 ks + 8 half on.
    bf16x8 wf[2][KS];
    {
        uint16_t *w = stream_lds + wave * 32 * STREAM_LROW;
        static_assert(4 * 32 == 2 * STREAM_ROWS, "32 weight rows per wave fill the two buffers");
        const int wrow = lane / (2 * KS), wcol = lane % (2 * KS) * 8;
        const u32x4v zero = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
#pragma unroll
            for (int i = 0; i < KS; ++i)
                *reinterpret_cast<u32x4v *>(&w[(i * (32 / KS) + wrow) * STREAM_LROW + wcol]) = wcol < K ? wraw[i] : zero;
            if (cb == 0) {
#pragma unroll
                for (int i = 0; i < KS; ++i)
                    wraw[i] = *reinterpret_cast<const u32x4v *>(a.B + (int64_t)(64 * wave + (KS + i) * (32 / KS) + wrow) * a.K + (wcol < a.K ? wcol : 0));
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) wf[cb][ks] = lds_read8(&w[lr * STREAM_LROW + ks * 16 + 8 * half]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        __syncthreads();
    }
    const float floor_v = a.relu ? 0.f : -INFINITY;
    // Two sets of accumulators: while the MFMAs of a tile fill one, the other -- the tile before -- is converted and
    // written to the wave's LDS patch, a sixteenth (K <= 128: an eighth) per K step, in the shadow of that step's MFMAs;
    // this wave is alone on its SIMD, so nothing else would fill the vector pipe while the matrix pipe runs, nor the
    // matrix pipe during a separate epilogue.
    // piece 0..15 of a tile's results: a lane holds, for row lr of each 32-row block rb, the columns
    // 32 cb + 8 grp + 4 half .. + 4 of the wave's 64
    auto convert_piece = [&](const f32x16 (&acc)[2][2], int piece) {
        const int cb = piece >> 3, grp = (piece >> 1) & 3, rb = piece & 1;
        const int n = 32 * cb + 8 * grp + 4 * half;
        const float v0 = at_least(acc[rb][cb][grp * 4 + 0], floor_v), v1 = at_least(acc[rb][cb][grp * 4 + 1], floor_v);
        const float v2 = at_least(acc[rb][cb][grp * 4 + 2], floor_v), v3 = at_least(acc[rb][cb][grp * 4 + 3], floor_v);
        *reinterpret_cast<uint2 *>(&ob[(rb * 32 + lr) * STREAM_OROW + n]) = make_uint2(pack_bf16x2(v0, v1), pack_bf16x2(v2, v3));
    };
    // the patch leaves as 128-byte row pieces (store_out: 61 K rows forward, their weight gradient and step 44.4 -> 42.9 us)
    auto flush = [&](int t) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const int m0 = tile_m0(t);
#pragma unroll
        for (int it = 0; it < 8; ++it) {
            const int c = it * 64 + lane, row = c >> 3, c8 = (c & 7) * 8;
            const u32x4v x = *reinterpret_cast<const u32x4v *>(&ob[row * STREAM_OROW + c8]);
            if (FULL || m0 + row < M) store_out(reinterpret_cast<u32x4v *>(a.Cb + (int64_t)(m0 + row) * a.ldcb + 64 * wave + c8), x);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // the patch is rewritten for the next tile
    };
    auto multiply = [&](const uint16_t *As, f32x16 (&acc)[2][2], const f32x16 (&prev)[2][2], auto with_prev) {
        constexpr bool PREV = decltype(with_prev)::value;
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) {
                const float4 bq = *reinterpret_cast<const float4 *>(&bias_s[64 * wave + 32 * cb + 8 * grp + 4 * half]);
#pragma unroll
                for (int rb = 0; rb < 2; ++rb) {
                    acc[rb][cb][grp * 4 + 0] = bq.x; acc[rb][cb][grp * 4 + 1] = bq.y; acc[rb][cb][grp * 4 + 2] = bq.z; acc[rb][cb][grp * 4 + 3] = bq.w;
                }
            }
        const uint16_t *ar0 = As + lr * STREAM_LROW + 8 * half, *ar1 = ar0 + 32 * STREAM_LROW;
        // (fragments are requested two K steps ahead: four MFMAs do not cover an LDS round trip)
        bf16x8 f0[3], f1[3];
        f0[0] = lds_read8(ar0); f1[0] = lds_read8(ar1);
        f0[1] = lds_read8(ar0 + 16); f1[1] = lds_read8(ar1 + 16);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks + 2 < KS) {
                f0[(ks + 2) % 3] = lds_read8(ar0 + (ks + 2) * 16);
                f1[(ks + 2) % 3] = lds_read8(ar1 + (ks + 2) * 16);
            }
            const bf16x8 a0 = f0[ks % 3], a1 = f1[ks % 3];
            acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[0][ks], a0, acc[0][0], 0, 0, 0);
            acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[0][ks], a1, acc[1][0], 0, 0, 0);
            acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[1][ks], a0, acc[0][1], 0, 0, 0);
            acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[1][ks], a1, acc[1][1], 0, 0, 0);
            if constexpr (PREV) {
#pragma unroll
                for (int q = 0; q < 16 / KS; ++q) convert_piece(prev, ks * (16 / KS) + q);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto convert_all = [&](const f32x16 (&acc)[2][2]) {
#pragma unroll
        for (int piece = 0; piece < 16; ++piece) convert_piece(acc, piece);
    };

    if (tid < WIDE_N / 4)
        *reinterpret_cast<float4 *>(&bias_s[tid * 4]) = a.bias ? *reinterpret_cast<const float4 *>(a.bias + tid * 4) : make_float4(0.f, 0.f, 0.f, 0.f);
    if (!mine) {                 // columns from K on stay zero in both buffers
        const u32x4v zero = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            *reinterpret_cast<u32x4v *>(&As0[(8 * i + srow) * STREAM_LROW + kp * 8]) = zero;
            *reinterpret_cast<u32x4v *>(&As1[(8 * i + srow) * STREAM_LROW + kp * 8]) = zero;
        }
    }
    stage(As0, ra);
    __syncthreads();
    f32x16 acc_a[2][2], acc_b[2][2];
    // tile t sits in the first buffer, tile t + step is on its way into rb
    fetch(ra, t + 2 * step);
    multiply(As0, acc_a, acc_b, std::false_type{});
    for (;;) {
        // acc_a holds tile t; tile t + step (if there is one) is on its way into rb
        if (t + step >= ntiles) {
            convert_all(acc_a);
            flush(t);
            break;
        }
        stage(As1, rb);
        __syncthreads();
        fetch(rb, t + 3 * step);
        multiply(As1, acc_b, acc_a, std::true_type{});
        flush(t);
        t += step;
        // acc_b holds tile t; tile t + step is on its way into ra
        if (t + step >= ntiles) {
            convert_all(acc_b);
            flush(t);
            break;
        }
        stage(As0, ra);
        __syncthreads();
        fetch(ra, t + 3 * step);
        multiply(As0, acc_a, acc_b, std::true_type{});
        flush(t);
        t += step;
    }
}

// The wave's weights are requested before the row count is read (they do not depend on it): the two round trips to
// memory overlap.  They are requested as whole rows of the transposed weights (a load covers two to four of them) and take their
// places in the body: as MFMA fragments, 16 bytes of 32 rows per load, they kept the address unit busy for 4.2 us of 18, and the
// first activations were requested behind them.
template <int KS>
__device__ __forceinline__ void nt_stream_run(const NtArgs &a, uint16_t *stream_lds)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wrow = lane / (2 * KS), wcol = lane % (2 * KS) * 8;      // 2 KS pieces of 16 bytes per row, 32 / KS rows per load
    u32x4v wraw[KS];
#pragma unroll
    for (int i = 0; i < KS; ++i)
        wraw[i] = *reinterpret_cast<const u32x4v *>(a.B + (int64_t)(64 * wave + i * (32 / KS) + wrow) * a.K + (wcol < a.K ? wcol : 0));
    asm volatile("" ::: "memory");      // (keeps the loads above from being moved below the branch on the row count)
    const int M = min(a.hdr[CR_HDR_N_DST], a.max_rows);
    if ((int)blockIdx.x * STREAM_ROWS >= M) return;
    const bool uniform = a.K0 == a.K || a.K0 % 128 == 0;
    if (M < STREAM_ROWS) nt_stream_body<KS, false, false>(a, M, stream_lds, wraw);
    else if (uniform) nt_stream_body<KS, true, true>(a, M, stream_lds, wraw);
    else nt_stream_body<KS, true, false>(a, M, stream_lds, wraw);
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_nt_stream_kernel(NtArgs a)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t stream_lds[];
    if (a.K <= 128) nt_stream_run<8>(a, stream_lds);
    else nt_stream_run<16>(a, stream_lds);
}

// The streaming and the wide kernel: below this their 64- and 128-row tiles leave compute units idle that the tiled kernel's
// 128 x 64 tiles fill.  K = 256 (streaming): 6.7 against 8.7 us at 8192 rows, 7.8 against 9.5 at 12288; K = 512 (wide) 9.0
// against 13.3 and 11.3 against 13.6, 14.4 at 16384; K = 1216 16.4 against 26.1 and 23.3 against 28.1, 29.5 at 16384.
constexpr int NT_WIDE_MIN_ROWS = 16384;

constexpr int NT_SMALL_ROWS = 2048;    // blocks of at most this many rows (by capacity) take the kernel above

// Wider tiles (NTILES = 4, 8) read the activations fewer times but measured slower on MI355X for the
// layer widths of this path (K = 256..512, N = 256): these products are bound by memory round trips
// and occupancy, not by the matrix cores, so the smallest tile at the highest occupancy wins.
constexpr int64_t NT_DEEP_MAX_BLOCKS = 512;   // at most two workgroups per compute unit and ...
constexpr int NT_DEEP_MIN_K = 768;            // ... a K loop of at least 24 steps: eight steps of prefetch

static void launch_nt(const NtArgs &a, hipStream_t s)
{
    // many rows, bf16 output only, K small enough for the weights to stay in registers: the streaming kernel
    if (a.max_rows >= NT_WIDE_MIN_ROWS && a.N == WIDE_N && a.K <= STREAM_KMAX && a.K % 8 == 0 && a.K0 % 8 == 0 && a.A1 != nullptr &&
        a.Cb != nullptr && a.C0 == nullptr && a.ldcb == a.N && (int64_t)a.max_rows * a.lda < (1ll << 29)) {
        static PerDevice asked;
        if (lds_opt_in(asked, reinterpret_cast<const void *>(&gemm_nt_stream_kernel), STREAM_LDS_BYTES)) {
            const int64_t tiles = ceil_div(a.max_rows, STREAM_ROWS);
            hipLaunchKernelGGL(gemm_nt_stream_kernel, dim3((unsigned)(tiles < 256 ? tiles : 256)), dim3(256), STREAM_LDS_BYTES, s, a);
            return;
        }
    }
    // many rows, wider inputs, bf16 output only
    if (a.max_rows >= NT_WIDE_MIN_ROWS && a.N == WIDE_N && a.K0 % 32 == 0 && a.K % 32 == 0 && a.A1 != nullptr && a.Cb != nullptr &&
        a.C0 == nullptr && a.ldcb == a.N && a.lda < (1 << 20)) {
        hipLaunchKernelGGL(gemm_nt_wide_kernel, dim3((unsigned)ceil_div(a.max_rows, WIDE_ROWS)), dim3(256), 0, s, a);
        return;
    }
    // xcd_compact needs the grid rounded up to a multiple of eight blocks
    const unsigned ncol = (unsigned)(a.N / 64);
    if (a.max_rows <= NT_SMALL_ROWS) {
        hipLaunchKernelGGL(gemm_nt_small_kernel<false>, dim3(ncol, (unsigned)ceil_div(a.max_rows, 32)), dim3(256), 0, s, a, XentArgs{});
        return;
    }
    const dim3 grid(ncol, (unsigned)ceil_div(a.max_rows, 128) + (7 + ncol - 1) / ncol);
    if ((int64_t)grid.x * grid.y <= NT_DEEP_MAX_BLOCKS && a.K >= NT_DEEP_MIN_K) hipLaunchKernelGGL((gemm_nt_kernel<2, 8>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((gemm_nt_kernel<2, 4>), grid, dim3(256), 0, s, a);
}

// ------------------------------------------------------------------------------------------------
// P[s][k][n] = sum_{m in split s} A[m][k] * Z[m][n]      (both operands strided along m).  Also the
// column sums of Z per split (bias gradient).
// Workgroup tile 128 (k) x 128 (n), four waves of 64 x 64; TN_BM rows of m per step (one barrier per step: taller
// steps spread its cost and the LDS round trip over more MFMAs).  Half of the
// threads stage A, half stage Z: a thread fetches one 8-column chunk of TN_BM / 8 consecutive rows and
// writes it transposed as eight 64-bit LDS stores (four m of one column each), so the MFMA operands
// are again 16-byte reads along m.  Global loads run three steps ahead in a register ring.
// ------------------------------------------------------------------------------------------------
struct TnArgs {
    const int32_t *hdr;
    int32_t max_rows;
    const uint16_t *A0, *A1;
    int64_t lda;
    int32_t K0, K2;
    const uint16_t *Z;       // [M][N]
    int32_t N;
    int32_t slots;           // partial slots available
    float *partial;          // [S][K2 + 1][N]: row K2 holds the column sums of Z (bias gradient)
};

// T = [buffer][operand: 0 = A, 1 = Z][m][column]: the tiles are staged as they come from memory (row-major);
// the transposition the MFMA operands need (eight consecutive m of one column per lane) is done by the LDS
// transpose read of gfx950.  Row stride 320 bytes: the four 64-byte row pieces that 32 lanes read fall into disjoint
// banks.  `bid` is the workgroup's number among the `ntile` x (splits) workgroups of the product.
// SUBS == 2: eight waves, the second four take the later half of the split's steps with tiles and accumulators of their own; the
// halves are added through LDS at the end (the earlier half first, so in a fixed order).
template <int SUBS>
__device__ __forceinline__ void gemm_tn_body(const TnArgs &a, uint32_t bid, uint32_t ntile, uint16_t (&Tall)[SUBS][2][2][TN_BM][TN_ROW])
{
    const int M = min(a.hdr[CR_HDR_N_DST], a.max_rows);
    // the tiles of one split run next to each other on one XCD (they share the split's rows of A and Z);
    // splits past the last row stay inactive, and the reduction skips them too
    uint32_t work;
    const int rows_per_split = rows_per_split_for(M, a.slots);
    if (!xcd_compact(bid, (uint32_t)((M + rows_per_split - 1) / rows_per_split) * ntile, work)) return;
    const int split = (int)(work / ntile), tile_id = (int)(work % ntile);
    const int sub = SUBS > 1 ? (int)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 8)) : 0;
    const int split_begin = split * rows_per_split, split_end = min(M, split_begin + rows_per_split);
    const int nsteps = ((split_end - split_begin + TN_BM - 1) / TN_BM + SUBS - 1) / SUBS;       // steps of either half
    const int m_begin = min(split_end, split_begin + sub * nsteps * TN_BM);
    const int m_end = min(split_end, m_begin + nsteps * TN_BM);
    uint16_t (&T)[2][2][TN_BM][TN_ROW] = Tall[sub];
    const int n_tiles = (a.N + 127) / 128;
    const int k_tiles_part = (a.K0 + 127) / 128;   // k-tiles per operand part (self | agg): a tile never straddles the two
    const int kt = tile_id / n_tiles;
    const int part = kt / k_tiles_part;
    const int kp0 = (kt % k_tiles_part) * 128;     // first column of the tile inside its part
    const int k0 = part * a.K0 + kp0;              // first row of the output tile
    const int k_valid = min(128, a.K0 - kp0);
    const int n0 = (tile_id % n_tiles) * 128;
    const int tid = threadIdx.x & 255, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, lr = lane & 31;
    const int wk = wave >> 1, wn = wave & 1;

    // staging role: waves 0,1 stage A, waves 2,3 stage Z.  Buffer loads return zero past the end of the
    // split's rows (and for columns outside the tile), so no load sits under a branch and the loads of
    // three steps stay in flight together.
    const int op = tid >> 7;                       // 0: A, 1: Z (uniform per wave)
    const int st = tid & 127, mg = st >> 4, sc = (st & 15) * 8;
    // (op is the same for a whole wave; the descriptor is built from values the compiler can see are wave-uniform --
    // with a descriptor it takes for lane-dependent it wraps every load in a loop over the distinct descriptors and then
    // waits for nearly all earlier loads before each new one, which undoes the ring)
    const uint64_t base_v = reinterpret_cast<uint64_t>(op == 0 ? (part == 0 ? a.A0 : a.A1) : a.Z);
    const uint16_t *base = reinterpret_cast<const uint16_t *>(
        ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(base_v >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((int)base_v));
    const uint32_t ld_bytes = (uint32_t)__builtin_amdgcn_readfirstlane((int)((op == 0 ? a.lda : (int64_t)a.N) * 2));
    const bool col_ok = op == 0 ? sc < k_valid : n0 + sc < a.N;
    const uint32_t col_bytes = (uint32_t)((op == 0 ? kp0 + sc : n0 + sc) * 2);
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(base), 0, (int)((uint32_t)m_end * ld_bytes), 0x00020000);

    constexpr int RPT = TN_BM / 8;                 // rows per thread and step: row group mg takes rows mg * RPT .. + RPT
    uint4 ring[3][RPT];
    auto fetch = [&](uint4 (&r)[RPT], int step) {
        const uint32_t mrow = (uint32_t)(m_begin + step * TN_BM + mg * RPT);
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const uint32_t off = col_ok ? (mrow + i) * ld_bytes + col_bytes : 0xFFFFFFF0u;
            const u32x4v v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 0, 0);
            r[i] = make_uint4(v[0], v[1], v[2], v[3]);
        }
    };
    // a thread holds an 8-column chunk of RPT consecutive rows: plain 16-byte stores
    float cacc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};      // column sums of Z over this thread's rows (kt == 0 only)
    const bool do_colsum = kt == 0 && op == 1;
    auto stage = [&](const uint4 (&r)[RPT], int buf) {
#pragma unroll
        for (int i = 0; i < RPT; ++i) *reinterpret_cast<uint4 *>(&T[buf][op][mg * RPT + i][sc]) = r[i];
        if (do_colsum) {
#pragma unroll
            for (int i = 0; i < RPT; ++i) {
                cacc[0] += __uint_as_float(r[i].x << 16); cacc[1] += __uint_as_float(r[i].x & 0xFFFF0000u);
                cacc[2] += __uint_as_float(r[i].y << 16); cacc[3] += __uint_as_float(r[i].y & 0xFFFF0000u);
                cacc[4] += __uint_as_float(r[i].z << 16); cacc[5] += __uint_as_float(r[i].z & 0xFFFF0000u);
                cacc[6] += __uint_as_float(r[i].w << 16); cacc[7] += __uint_as_float(r[i].w & 0xFFFF0000u);
            }
        }
    };
    // MFMA operand of lane (lr, half) for the 32-column sub-tile at col0: rows m0 + 8 half .. + 8 of column
    // col0 + lr.  A 16-lane group reads a 4 (m) x 16 (columns) piece: lane i of the group supplies the address of
    // row i / 4, columns 4 (i % 4) .. + 4 and receives column i's four rows.
    const int tl = lane & 15, tcol = ((lane >> 4) & 1) * 16;
    auto operand = [&](int buf, int which, int col0, int m0) -> bf16x8 {
        const uint16_t *p = &T[buf][which][m0 + 8 * half + (tl >> 2)][col0 + tcol + 4 * (tl & 3)];
        const v4s16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((v4s16 __attribute__((address_space(3))) *)p);
        const v4s16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((v4s16 __attribute__((address_space(3))) *)(p + 4 * TN_ROW));
        typedef short v8s16 __attribute__((ext_vector_type(8)));
        const v8s16 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(bf16x8, both);
    };

    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    fetch(ring[0], 0);
    fetch(ring[1], 1);
    fetch(ring[2], 2);
    stage(ring[0], 0);
    __syncthreads();

    auto body = [&](int t, uint4 (&slot_next_fetch)[RPT], const uint4 (&slot_next_stage)[RPT]) {
        const int buf = t & 1;
        fetch(slot_next_fetch, t + 3);             // the slot that held step t (already staged)
#pragma unroll
        for (int kk = 0; kk < TN_BM / 16; ++kk) {
            bf16x8 x[2], z[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                x[i] = operand(buf, 0, wk * 64 + i * 32, kk * 16);
                z[i] = operand(buf, 1, wn * 64 + i * 32, kk * 16);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[i], z[j], acc[i][j], 0, 0, 0);
        }
        // (unconditional, also after the last step, where it stores the zeros that loads past the end return: with a
        // branch here the compiler sees a path on which a ring slot's loads are never waited for, and drains every
        // outstanding load at the head of the loop)
        stage(slot_next_stage, buf ^ 1);
        __syncthreads();
    };
    int t = 0;
    // (Written out: with the same steps in unrolled loops over the slots the compiler takes 44 registers more, which leaves two
    // waves per SIMD instead of three where the product shares its launch with the input gradient's.  Two operands of 256 -> 256,
    // both products: 12288 rows 26.4 -> 23.7 us, 65536 76 -> 69; one of 256 -> 512: 25.8 -> 23.1 and 66 -> 61.)
    for (; t + 3 <= nsteps; t += 3) {
        body(t, ring[0], ring[1]);
        body(t + 1, ring[1], ring[2]);
        body(t + 2, ring[2], ring[0]);
    }
    if (t < nsteps) body(t, ring[0], ring[1]);
    if (t + 1 < nsteps) body(t + 1, ring[1], ring[2]);

    // the halves meet: each wave hands 32 of its 64 rows of the tile to its counterpart and finishes the other 32
    float *meet = reinterpret_cast<float *>(&Tall[0][0][0][0][0]);
    constexpr int MEET = 4 * 2 * 16 * 64;          // floats that one half hands over
    if constexpr (SUBS > 1) {
        static_assert(2 * MEET * sizeof(float) + 16 * 128 * sizeof(float) <= sizeof(Tall), "the halves meet in the staging tiles' room");
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) meet[sub * MEET + ((wave * 2 + j) * 16 + r) * 64 + lane] = sub == 0 ? acc[1][j][r] : acc[0][j][r];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float other = meet[(1 - sub) * MEET + ((wave * 2 + j) * 16 + r) * 64 + lane];
                if (sub == 0) acc[0][j][r] += other;
                else acc[1][j][r] += other;
            }
    }

    float *P = a.partial + (int64_t)split * (a.K2 + 1) * a.N;
    // (store_out: the reduction reads a split's sums on every XCD.  The same pass 44.4 -> 42.8 us.  A row's address is scalar and
    // the lane's place in it one 32-bit offset: with an address and two comparisons per value this was 2 of 18 us.  Widths are
    // multiples of 32 and 64: a 32-row piece of a wave's tile is inside or outside as a whole.)
    {
        const int row0 = __builtin_amdgcn_readfirstlane(wk) * 64, col0 = n0 + __builtin_amdgcn_readfirstlane(wn) * 64;
        const uint32_t lane_off = (uint32_t)(4 * half * a.N + lr) * 4u;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if ((SUBS > 1 && i != sub) || row0 + i * 32 >= k_valid || col0 >= a.N) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                char *row = reinterpret_cast<char *>(P + (int64_t)(k0 + row0 + i * 32 + 8 * (r >> 2) + (r & 3)) * a.N + col0);
#pragma unroll
                for (int j = 0; j < 2; ++j) store_out(reinterpret_cast<float *>(row + 128 * j + lane_off), acc[i][j][r]);
            }
        }
    }
    // bias gradient: the row groups' column sums meet in LDS and are added in a fixed order
    if (kt == 0) {
        // (one half: the staging tiles are free now; two: behind what the halves hand over)
        float (*csum)[128] = reinterpret_cast<float (*)[128]>(meet + (SUBS > 1 ? 2 * MEET : 0));
        if (op == 1) {
#pragma unroll
            for (int c = 0; c < 8; ++c) csum[sub * 8 + mg][sc + c] = cacc[c];
        }
        __syncthreads();
        if (sub == 0 && tid < 128 && n0 + tid < a.N) {
            float tot = 0.f;
#pragma unroll
            for (int g8 = 0; g8 < 8 * SUBS; ++g8) tot += csum[g8][tid];
            P[(int64_t)a.K2 * a.N + n0 + tid] = tot;
        }
    }
}

__global__ __launch_bounds__(256) void gemm_tn_kernel(TnArgs a)
{
    __shared__ __attribute__((aligned(16))) uint16_t T[1][2][2][TN_BM][TN_ROW];
    gemm_tn_body<1>(a, blockIdx.y * gridDim.x + blockIdx.x, gridDim.x, T);
}

// Blocks of many rows.  One workgroup of four waves per compute unit (the split plan) leaves every SIMD a single wave, which
// waits out its own chain of transpose reads, MFMAs, staging and barrier in each step (1250 cycles, of which the MFMAs are 256);
// more loads in flight change nothing (three to eight steps ahead: the same), a second workgroup does but doubles the
// partial sums.  Eight waves in two halves give every SIMD two waves with the partial sums of one workgroup:
// 131 K rows x 608 x 256 (graph attention on the reddit-like graph) 87 -> 69 us, 61 K rows x 256 x 256 (papers) 21.6 -> 20.0;
// with the reduction of the partial sums 81 -> 67 us (131 K rows x 608 x 256), 27.6 -> 26.6 (66 K x 256 x 256), 21.5 -> 20.7 (33 K);
// at 16 K rows 19.4 -> 19.8 (256 x 256), 23.0 -> 22.5 (608 x 256), 33.6 -> 30.4 (1216 x 256): about where it begins to pay.  Where the input gradient is wanted too, the next kernel serves.
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_tn_tall_kernel(TnArgs a)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t tn_lds[];
    gemm_tn_body<2>(a, blockIdx.y * gridDim.x + blockIdx.x, gridDim.x, *reinterpret_cast<uint16_t (*)[2][2][2][TN_BM][TN_ROW]>(tn_lds));
}
constexpr size_t TN_TALL_LDS_BYTES = sizeof(uint16_t) * 2 * 2 * 2 * TN_BM * TN_ROW;
constexpr int TN_TALL_MIN_ROWS = 16384;

static bool tn_tall_ready()
{
    static PerDevice asked;
    return lds_opt_in(asked, reinterpret_cast<const void *>(&gemm_tn_tall_kernel), TN_TALL_LDS_BYTES);
}

// The two products of a layer's backward pass that need nothing from each other (weight gradient, input
// gradient) in one launch: both are short and bound by memory round trips, so side by side they take about as
// long as the longer one.  The first `tn_blocks` workgroups (a multiple of eight, so that both parts keep their
// XCD mapping) run the weight-gradient product, the rest the input-gradient product.
__global__ __launch_bounds__(256) void gemm_tn_nt_kernel(TnArgs t, NtArgs n, uint32_t tn_blocks, uint32_t tn_tiles, uint32_t nt_cols)
{
    __shared__ __attribute__((aligned(16))) uint16_t lds[2 * 2 * TN_BM * TN_ROW];
    static_assert(sizeof(lds) >= sizeof(uint16_t) * (2 * 128 * LDS_ROW + 2 * 64 * LDS_ROW), "the staging tiles of either product fit");
    if (blockIdx.x < tn_blocks) {
        gemm_tn_body<1>(t, blockIdx.x, tn_tiles, *reinterpret_cast<uint16_t (*)[1][2][2][TN_BM][TN_ROW]>(lds));
    } else {
        gemm_nt_body<2, 4>(n, blockIdx.x - tn_blocks, nt_cols, *reinterpret_cast<uint16_t (*)[2][128][LDS_ROW]>(lds),
                           *reinterpret_cast<uint16_t (*)[2][64][LDS_ROW]>(lds + 2 * 128 * LDS_ROW));
    }
}

__global__ __launch_bounds__(256) void sgd_reduce_kernel(SgdArgs a)
{
    __shared__ float4 red[4][64];
    sgd_reduce_body(a, blockIdx.x, red);
}

__global__ __launch_bounds__(256) void refresh_shadows_kernel(const float *W, int F_in, int F_out, int F_pad, int N_pad, int n_op,
                                                              uint16_t *W_bf16, uint16_t *Wt_bf16)
{
    const int K2 = n_op * F_pad;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)K2 * N_pad) return;
    const int k2 = (int)(idx / N_pad), n = (int)(idx % N_pad);
    const int kin = k2 % F_pad, part = k2 / F_pad;
    uint16_t wb = 0;
    if (kin < F_in && n < F_out) wb = f32_to_bf16(W[(int64_t)(part * F_in + kin) * F_out + n]);
    W_bf16[(int64_t)k2 * N_pad + n] = wb;
    Wt_bf16[(int64_t)n * K2 + k2] = wb;
}

// ------------------------------------------------------------------------------------------------
// softmax cross-entropy on the root rows: one wave per row, lane i takes the columns i, i + 64, ..
// NV > 0: at most 64 NV columns, read once and kept in registers; 0: any number, read three times.  A row is a chain of round
// trips (row count, root id, label); the logits travel meanwhile.
// MEAN: the mean loss too.  The workgroups' shares meet in acc[0], as in the fused top layer: one 64-bit atomic carries the share in
// fixed point (2^-20, bits 0..43), a ticket (44..53) and a mark (54..63) for a share that does not fit (not finite, or beyond 2^14);
// such a share is added to the double in acc[1] first.  1024 rows of 172 classes, the layer with its loss and
// both directions: 31.2 us with a launch of its own for the mean and the row read three times, 30.0 now.
// ------------------------------------------------------------------------------------------------
constexpr int XENT_WAVES = 8;
constexpr int XENT_MEAN_ROWS = 2048;       // most rows (by capacity) of the one-launch form: at most 256 shares of 2^14 each

template <int NV, bool MEAN>
__global__ __launch_bounds__(XENT_WAVES * WAVE) void xent_rows_kernel(const int32_t *hdr, int max_rows, const float *logits, int64_t ld, int C,
                                                                      const int32_t *labels, const int32_t *root_ids, float *row_loss,
                                                                      float *d_logits, uint16_t *d_logits_bf16, float *loss, unsigned long long *acc)
{
    __shared__ float part[XENT_WAVES];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE)), lane = lane_id();
    const int row = (int)blockIdx.x * XENT_WAVES + wave, rc = min(row, max_rows - 1);
    const float *z = logits + (int64_t)rc * ld;
    float x[NV > 0 ? NV : 1];
    if constexpr (NV > 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) x[k] = lane + k * WAVE < ld ? z[lane + k * WAVE] : 0.f;
    }
    const int n = min(hdr[CR_HDR_N_DST], max_rows);
    if ((int)blockIdx.x * XENT_WAVES >= n) {
        if (MEAN && blockIdx.x == 0 && threadIdx.x == 0) loss[0] = 0.f;
        return;
    }
    const bool row_ok = row < n;
    if (row_ok) {
        const int label = labels[root_ids[row]];
        float mx = -INFINITY;
        if constexpr (NV > 0) {
#pragma unroll
            for (int k = 0; k < NV; ++k) mx = fmaxf(mx, lane + k * WAVE < C ? x[k] : -INFINITY);
        } else {
            for (int c = lane; c < C; c += WAVE) mx = fmaxf(mx, z[c]);
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
        float den = 0.f, e[NV > 0 ? NV : 1];
        if constexpr (NV > 0) {
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                e[k] = lane + k * WAVE < C ? expf(x[k] - mx) : 0.f;
                den += e[k];
            }
        } else {
            for (int c = lane; c < C; c += WAVE) den += expf(z[c] - mx);
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) den += __shfl_xor(den, off);
        const float inv_n = 1.0f / (float)n;
        auto put = [&](int c, float ec) {
            float d = 0.f;
            if (c < C) d = (ec / den - (c == label ? 1.f : 0.f)) * inv_n;
            if (d_logits) d_logits[(int64_t)row * ld + c] = d;
            if (d_logits_bf16) d_logits_bf16[(int64_t)row * ld + c] = f32_to_bf16(d);
        };
        float zl = 0.f;                                        // the label's logit
        if constexpr (NV > 0) {
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                const float v = __shfl(x[k], label & (WAVE - 1));
                zl = (label >> 6) == k ? v : zl;
                if (lane + k * WAVE < ld) put(lane + k * WAVE, e[k]);
            }
        } else {
            zl = z[label];
            for (int c = lane; c < ld; c += WAVE) put(c, c < C ? expf(z[c] - mx) : 0.f);
        }
        const float rl = -(zl - mx - logf(den));
        if (lane == 0) {
            row_loss[row] = rl;
            part[wave] = rl;
        }
    } else if (lane == 0) {
        part[wave] = 0.f;
    }
    if constexpr (MEAN) {
        __syncthreads();
        if (threadIdx.x != 0) return;
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < XENT_WAVES; ++w) t += part[w];
        const bool fits = t >= 0.f && t <= 16384.0f;           // (a row's loss is not negative but for rounding)
        const float small = t < 0.f && t > -1.0f ? 0.f : t;
        double *rest = reinterpret_cast<double *>(acc + 1);
        unsigned long long add = (1ull << 44) | (fits ? (unsigned long long)(t * 1048576.0f + 0.5f) : 0ull);
        if (!fits && small != 0.f) {
            const double before = __hip_atomic_fetch_add(rest, (double)t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("" ::"v"(before) : "memory");          // (the addition has returned before the ticket is drawn)
            add |= 1ull << 54;
        }
        const unsigned long long after = __hip_atomic_fetch_add(acc, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + add;
        if ((int)((after >> 44) & 0x3FFull) == (n + XENT_WAVES - 1) / XENT_WAVES) {
            double sum = (double)(after & ((1ull << 44) - 1ull)) * (1.0 / 1048576.0);
            if (after >> 54) sum += __builtin_bit_cast(double, __hip_atomic_exchange(acc + 1, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            loss[0] = (float)(sum / (double)n);
            __hip_atomic_store(acc, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

__global__ __launch_bounds__(1024) void xent_mean_kernel(const int32_t *hdr, int max_rows, const float *row_loss, float *loss)
{
    __shared__ float part[16];
    const int n = min(hdr[CR_HDR_N_DST], max_rows);
    float s = 0.f;
    for (int i = threadIdx.x; i < n; i += 1024) s += row_loss[i];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    if (lane_id() == 0) part[threadIdx.x / WAVE] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.f;
        for (int w = 0; w < 16; ++w) t += part[w];
        loss[0] = n > 0 ? t / (float)n : 0.f;
    }
}

// rows' losses and gradients, and the mean loss: with `scratch` and few enough rows in one launch, else in two
static void launch_xent(const int32_t *hdr, int max_rows, const float *logits, int64_t ld, int C, const int32_t *labels, const int32_t *root_ids,
                        float *loss, float *row_loss, float *d_logits, uint16_t *d_logits_bf16, void *scratch, hipStream_t s)
{
    const bool one = scratch != nullptr && max_rows <= XENT_MEAN_ROWS;
    unsigned long long *acc = one ? static_cast<unsigned long long *>(scratch) + 2 : nullptr;      // (the fused top layer's word is the first)
    const dim3 grid((unsigned)ceil_div(max_rows, XENT_WAVES)), block(XENT_WAVES * WAVE);
#define CR_XENT(NV)                                                                                                                        \
    do {                                                                                                                                   \
        if (one) hipLaunchKernelGGL((xent_rows_kernel<NV, true>), grid, block, 0, s, hdr, max_rows, logits, ld, C, labels, root_ids,       \
                                    row_loss, d_logits, d_logits_bf16, loss, acc);                                                         \
        else hipLaunchKernelGGL((xent_rows_kernel<NV, false>), grid, block, 0, s, hdr, max_rows, logits, ld, C, labels, root_ids,          \
                                row_loss, d_logits, d_logits_bf16, loss, acc);                                                             \
    } while (0)
    if (ld <= 64) CR_XENT(1);
    else if (ld <= 128) CR_XENT(2);
    else if (ld <= 256) CR_XENT(4);
    else CR_XENT(0);
#undef CR_XENT
    if (!one) hipLaunchKernelGGL(xent_mean_kernel, dim3(1), dim3(1024), 0, s, hdr, max_rows, row_loss, loss);
}

// arg-max of every root row against its label; the workgroup's count is added to a device counter
__global__ __launch_bounds__(256) void count_correct_kernel(const int32_t *hdr, int max_rows, const float *logits, int64_t ld,
                                                            int C, const int32_t *labels, const int32_t *root_ids, int32_t *count)
{
    __shared__ int hits[4];
    const int n = min(hdr[CR_HDR_N_DST], max_rows);
    const int row = blockIdx.x * 4 + threadIdx.x / WAVE;
    const int lane = lane_id();
    int hit = 0;
    if (row < n) {
        const float *z = logits + (int64_t)row * ld;
        float best = -INFINITY;
        int arg = 0x7FFFFFFF;
        for (int c = lane; c < C; c += WAVE) {
            const float x = z[c];
            if (x > best) { best = x; arg = c; }          // ascending c per lane: the first maximum stays
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const float ob = __shfl_xor(best, off);
            const int oa = __shfl_xor(arg, off);
            if (ob > best || (ob == best && oa < arg)) { best = ob; arg = oa; }
        }
        hit = arg == labels[root_ids[row]] ? 1 : 0;
    }
    if (lane == 0) hits[threadIdx.x / WAVE] = hit;
    __syncthreads();
    if (threadIdx.x == 0) {
        const int s = hits[0] + hits[1] + hits[2] + hits[3];
        if (s) atomicAdd(count, s);
    }
}

static void split_plan(int F_pad, int N_pad, int n_op, int max_rows, int &rows_per_split, int &n_splits)
{
    const int tiles = (int)(n_op * ceil_div(F_pad, 128) * ceil_div(N_pad, 128));
    // one workgroup per compute unit: with two (the kernel's residency) the product itself is no faster, and the partial
    // sums -- written once and read once by the reduction -- double
    int target = 256 / tiles;
    if (target < 1) target = 1;
    if (target > 128) target = 128;
    int rows = (int)round_up(ceil_div(max_rows, target), 96);
    if (rows < 96) rows = 96;
    rows_per_split = rows;
    n_splits = (int)ceil_div(max_rows, rows);
}

}  // namespace cr

using namespace cr;

static cr_status check_layer(const cr_sage_layer *L, int &F_pad, int &N_pad)
{
    CR_REQUIRE(L != nullptr, CR_ERR_INVALID_ARG, "layer is NULL");
    CR_REQUIRE(L->F_in >= 1 && L->F_in <= 8192 && L->F_out >= 1 && L->F_out <= 8192, CR_ERR_INVALID_ARG,
               "layer dims (%d, %d) outside 1..8192", L->F_in, L->F_out);
    CR_REQUIRE(L->n_operands == 1 || L->n_operands == 2, CR_ERR_INVALID_ARG, "layer n_operands = %d must be 1 or 2", L->n_operands);
    CR_REQUIRE(L->W && L->W_bf16 && L->Wt_bf16, CR_ERR_INVALID_ARG, "layer has a NULL array");
    CR_REQUIRE(aligned16(L->W) && aligned16(L->bias) && aligned16(L->W_bf16) && aligned16(L->Wt_bf16), CR_ERR_INVALID_ARG,
               "layer arrays must be 16-byte aligned");
    F_pad = (int)round_up(L->F_in, 32);
    N_pad = (int)round_up(L->F_out, 64);
    return CR_OK;
}

extern "C" cr_status cr_sage_padded_dims(int32_t F_in, int32_t F_out, int32_t *F_pad, int32_t *N_pad)
{
    CR_REQUIRE(F_in >= 1 && F_in <= 8192 && F_out >= 1 && F_out <= 8192, CR_ERR_INVALID_ARG, "layer dims (%d, %d) outside 1..8192", F_in, F_out);
    CR_REQUIRE(F_pad && N_pad, CR_ERR_INVALID_ARG, "outputs must not be NULL");
    *F_pad = (int32_t)round_up(F_in, 32);
    *N_pad = (int32_t)round_up(F_out, 64);
    return CR_OK;
}

extern "C" cr_status cr_sage_refresh_shadows(const cr_sage_layer *layer, void *stream)
{
    int F_pad, N_pad;
    cr_status st = check_layer(layer, F_pad, N_pad);
    if (st != CR_OK) return st;
    if (dry_run()) return CR_OK;
    const int64_t n = (int64_t)layer->n_operands * F_pad * N_pad;
    hipLaunchKernelGGL(refresh_shadows_kernel, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, static_cast<hipStream_t>(stream),
                       layer->W, layer->F_in, layer->F_out, F_pad, N_pad, layer->n_operands, layer->W_bf16, layer->Wt_bf16);
    CR_LAUNCH_CHECK();
    return CR_OK;
}

extern "C" cr_status cr_sage_linear_fwd(const cr_sage_layer *layer, const int32_t *hdr, int32_t max_rows,
                                        const uint16_t *h_self, const uint16_t *agg, int64_t ld_in, int relu,
                                        float *out, uint16_t *out_bf16, void *stream)
{
    int F_pad, N_pad;
    cr_status st = check_layer(layer, F_pad, N_pad);
    if (st != CR_OK) return st;
    CR_REQUIRE(hdr != nullptr && max_rows >= 1, CR_ERR_INVALID_ARG, "hdr must not be NULL and max_rows must be positive");
    const int n_op = layer->n_operands;
    CR_REQUIRE(agg && aligned16(h_self) && aligned16(agg), CR_ERR_INVALID_ARG, "h_self / agg must be 16-byte aligned device pointers");
    CR_REQUIRE((h_self != nullptr) == (n_op == 2), CR_ERR_INVALID_ARG, "h_self must be given for a two-operand layer and NULL for a one-operand layer");
    CR_REQUIRE(ld_in >= F_pad && ld_in % 8 == 0, CR_ERR_INVALID_ARG, "ld_in = %lld must be a multiple of 8 and >= %d", (long long)ld_in, F_pad);
    CR_REQUIRE(out || out_bf16, CR_ERR_INVALID_ARG, "no output requested");
    CR_REQUIRE(aligned16(out) && aligned16(out_bf16), CR_ERR_INVALID_ARG, "outputs must be 16-byte aligned");
    if (dry_run()) return CR_OK;
    NtArgs a;
    a.hdr = hdr; a.max_rows = max_rows; a.A0 = n_op == 2 ? h_self : agg; a.A1 = agg; a.lda = ld_in; a.K0 = F_pad; a.K = n_op * F_pad;
    a.B = layer->Wt_bf16; a.N = N_pad; a.bias = layer->bias; a.relu = relu ? 1 : 0;
    a.C0 = out; a.C1 = nullptr; a.ldc = N_pad; a.N0 = N_pad; a.Cb = out_bf16; a.ldcb = N_pad;
    launch_nt(a, static_cast<hipStream_t>(stream));
    CR_LAUNCH_CHECK();
    return CR_OK;
}

extern "C" cr_status cr_sage_linear_fwd_xent(const cr_sage_layer *layer, const int32_t *hdr, int32_t max_rows,
                                             const uint16_t *h_self, const uint16_t *agg, int64_t ld_in, float *logits,
                                             int32_t n_classes, const int32_t *labels, const int32_t *root_ids, float *loss,
                                             float *row_loss, uint16_t *d_logits_bf16, void *scratch, void *stream)
{
    int F_pad, N_pad;
    cr_status st = check_layer(layer, F_pad, N_pad);
    if (st != CR_OK) return st;
    CR_REQUIRE(hdr != nullptr && max_rows >= 1, CR_ERR_INVALID_ARG, "hdr must not be NULL and max_rows must be positive");
    const int n_op = layer->n_operands;
    CR_REQUIRE(agg && aligned16(h_self) && aligned16(agg), CR_ERR_INVALID_ARG, "h_self / agg must be 16-byte aligned device pointers");
    CR_REQUIRE((h_self != nullptr) == (n_op == 2), CR_ERR_INVALID_ARG, "h_self must be given for a two-operand layer and NULL for a one-operand layer");
    CR_REQUIRE(ld_in >= F_pad && ld_in % 8 == 0, CR_ERR_INVALID_ARG, "ld_in = %lld must be a multiple of 8 and >= %d", (long long)ld_in, F_pad);
    CR_REQUIRE(logits && d_logits_bf16 && aligned16(logits) && aligned16(d_logits_bf16), CR_ERR_INVALID_ARG,
               "logits / d_logits_bf16 must be 16-byte aligned device pointers");
    CR_REQUIRE(labels && root_ids && loss && row_loss, CR_ERR_INVALID_ARG, "labels / root_ids / loss / row_loss must not be NULL");
    CR_REQUIRE(n_classes >= 1 && n_classes <= layer->F_out, CR_ERR_INVALID_ARG, "need 1 <= n_classes <= F_out");
    CR_REQUIRE(scratch != nullptr && aligned16(scratch), CR_ERR_INVALID_ARG, "scratch must be a 16-byte aligned device pointer");
    if (dry_run()) return CR_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    NtArgs a;
    a.hdr = hdr; a.max_rows = max_rows; a.A0 = n_op == 2 ? h_self : agg; a.A1 = agg; a.lda = ld_in; a.K0 = F_pad; a.K = n_op * F_pad;
    a.B = layer->Wt_bf16; a.N = N_pad; a.bias = layer->bias; a.relu = 0;
    a.C0 = logits; a.C1 = nullptr; a.ldc = N_pad; a.N0 = N_pad; a.Cb = nullptr; a.ldcb = N_pad;
    if (N_pad == 64 && max_rows <= NT_SMALL_ROWS) {
        XentArgs x;
        x.n_classes = n_classes; x.labels = labels; x.root_ids = root_ids; x.loss = loss; x.row_loss = row_loss;
        x.d_logits_bf16 = d_logits_bf16; x.acc = static_cast<unsigned long long *>(scratch);
        hipLaunchKernelGGL(gemm_nt_small_kernel<true>, dim3(1, (unsigned)ceil_div(max_rows, 32)), dim3(256), 0, s, a, x);
    } else {
        launch_nt(a, s);
        launch_xent(hdr, max_rows, logits, N_pad, n_classes, labels, root_ids, loss, row_loss, nullptr, d_logits_bf16, scratch, s);
    }
    CR_LAUNCH_CHECK();
    return CR_OK;
}

extern "C" cr_status cr_sage_linear_bwd_workspace_bytes(int32_t F_in, int32_t F_out, int32_t max_rows, size_t *bytes)
{
    CR_REQUIRE(F_in >= 1 && F_in <= 8192 && F_out >= 1 && F_out <= 8192, CR_ERR_INVALID_ARG, "layer dims (%d, %d) outside 1..8192", F_in, F_out);
    CR_REQUIRE(max_rows >= 1 && bytes != nullptr, CR_ERR_INVALID_ARG, "max_rows must be positive and bytes not NULL");
    const int F_pad = (int)round_up(F_in, 32), N_pad = (int)round_up(F_out, 64);
    int rows, splits, splits1;
    split_plan(F_pad, N_pad, 2, max_rows, rows, splits);
    split_plan(F_pad, N_pad, 1, max_rows, rows, splits1);       // enough for either kind of layer
    const size_t need2 = (size_t)splits * (2 * F_pad + 1) * N_pad, need1 = (size_t)splits1 * (F_pad + 1) * N_pad;
    Carver c(nullptr);
    c.take<float>(need2 > need1 ? need2 : need1);
    *bytes = c.bytes();
    return CR_OK;
}

cr_status cr::linear_bwd_products(const cr_sage_layer *layer, const int32_t *hdr, int32_t max_rows, const uint16_t *h_self,
                                  const uint16_t *agg, int64_t ld_in, const uint16_t *dz_bf16, float lr, float weight_decay,
                                  float *d_self, float *d_agg, uint16_t *d_in_bf16, float *dW_out, float *db_out, void *ws,
                                  size_t ws_bytes, void *stream, SgdArgs *deferred)
{
    int F_pad, N_pad;
    cr_status st = check_layer(layer, F_pad, N_pad);
    if (st != CR_OK) return st;
    CR_REQUIRE(hdr != nullptr && max_rows >= 1, CR_ERR_INVALID_ARG, "hdr must not be NULL and max_rows must be positive");
    const int n_op = layer->n_operands;
    CR_REQUIRE(agg && dz_bf16 && aligned16(h_self) && aligned16(agg) && aligned16(dz_bf16), CR_ERR_INVALID_ARG,
               "h_self / agg / dz_bf16 must be 16-byte aligned device pointers");
    CR_REQUIRE((h_self != nullptr) == (n_op == 2), CR_ERR_INVALID_ARG, "h_self must be given for a two-operand layer and NULL for a one-operand layer");
    CR_REQUIRE(n_op == 2 || d_self == nullptr, CR_ERR_INVALID_ARG, "a one-operand layer has no d_self");
    CR_REQUIRE(ld_in >= F_pad && ld_in % 8 == 0, CR_ERR_INVALID_ARG, "ld_in = %lld must be a multiple of 8 and >= %d", (long long)ld_in, F_pad);
    CR_REQUIRE(n_op == 1 || (d_self == nullptr) == (d_agg == nullptr), CR_ERR_INVALID_ARG, "d_self and d_agg must be given together");
    CR_REQUIRE(aligned16(d_self) && aligned16(d_agg) && aligned16(d_in_bf16), CR_ERR_INVALID_ARG, "d_self / d_agg / d_in_bf16 must be 16-byte aligned");
    CR_REQUIRE(lr == lr && weight_decay == weight_decay, CR_ERR_INVALID_ARG, "lr / weight_decay is NaN");
    CR_REQUIRE(!(d_agg || d_in_bf16) || (n_op * F_pad) % 64 == 0, CR_ERR_UNSUPPORTED,
               "input gradients of a one-operand layer need F_in rounded up to 32 to be a multiple of 64");
    CR_REQUIRE((int64_t)max_rows * ld_in * 2 < 0x7FFFFFFFll && (int64_t)max_rows * N_pad * 2 < 0x7FFFFFFFll, CR_ERR_UNSUPPORTED,
               "operand of %d rows exceeds the 2 GiB reach of 32-bit buffer offsets", max_rows);
    int rows, splits;
    split_plan(F_pad, N_pad, n_op, max_rows, rows, splits);
    Carver c(ws);
    float *partial = c.take<float>((size_t)splits * (n_op * F_pad + 1) * N_pad);
    CR_REQUIRE(ws != nullptr && aligned16(ws), CR_ERR_INVALID_ARG, "workspace must be a 16-byte aligned device pointer");
    CR_REQUIRE(ws_bytes >= c.bytes(), CR_ERR_CAPACITY, "workspace of %zu bytes, %zu needed", ws_bytes, c.bytes());
    if (dry_run()) return CR_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);

    const unsigned tn_tiles = (unsigned)(n_op * ceil_div(F_pad, 128) * ceil_div(N_pad, 128));
    const bool want_input = d_agg || d_in_bf16;
    if (want_input) {
        // the input-gradient product shares the launch and the 512 resident workgroup slots: fewer, longer splits so
        // that both parts fit one round (its tiles counted at ~0.7 of the capacity, the usual fill of a sampled block)
        const int64_t nt_share = (int64_t)(n_op * F_pad / 64) * ceil_div(max_rows, 128) * 7 / 10;
        const int64_t room = (512 - nt_share) / tn_tiles;
        if (room >= 8 && room < splits) splits = (int)room;
    }
    TnArgs t;
    t.hdr = hdr; t.max_rows = max_rows; t.A0 = n_op == 2 ? h_self : agg; t.A1 = agg; t.lda = ld_in; t.K0 = F_pad; t.K2 = n_op * F_pad;
    t.Z = dz_bf16; t.N = N_pad; t.slots = splits; t.partial = partial;
    const dim3 tn_grid(tn_tiles, (unsigned)splits + (7 + tn_tiles - 1) / tn_tiles);
    if (want_input) {   // also the gradient w.r.t. the layer's inputs (weights from before the step), in the same launch
        // (At any number of rows.  The whole call with the products in launches of their own, the tall kernel and what launch_nt
        // picks, at 16384 / 32768 / 65536 / 131072 rows: two operands of 256 -> 256, float gradients, 34 / 48 / 76 / 156 us against
        // 26 / 40 / 69 / 155 here; one operand of 256 -> 256, bf16 gradients, which the streaming product serves, 30 / 36 / 47 / 66
        // against 22 / 25 / 39 / 65; one of 256 -> 512, 35 / 43 / 64 / 113 against 27 / 36 / 61 / 115.)
        NtArgs a;
        a.hdr = hdr; a.max_rows = max_rows; a.A0 = dz_bf16; a.A1 = nullptr; a.lda = N_pad; a.K0 = N_pad; a.K = N_pad;
        a.B = layer->W_bf16; a.N = n_op * F_pad; a.bias = nullptr; a.relu = 0;
        a.C0 = n_op == 2 ? d_self : d_agg; a.C1 = d_agg; a.ldc = F_pad; a.N0 = F_pad; a.Cb = d_in_bf16; a.ldcb = n_op * F_pad;
        const unsigned nt_cols = (unsigned)(a.N / 64);
        const unsigned tn_blocks = (unsigned)round_up((int64_t)tn_tiles * splits + 7, 8);
        const unsigned nt_blocks = (unsigned)round_up((int64_t)nt_cols * ceil_div(max_rows, 128) + 7, 8);
        hipLaunchKernelGGL(gemm_tn_nt_kernel, dim3(tn_blocks + nt_blocks), dim3(256), 0, s, t, a, tn_blocks, tn_tiles, nt_cols);
    } else if (max_rows >= TN_TALL_MIN_ROWS && tn_tall_ready()) {
        hipLaunchKernelGGL(gemm_tn_tall_kernel, tn_grid, dim3(512), TN_TALL_LDS_BYTES, s, t);
    } else {
        hipLaunchKernelGGL(gemm_tn_kernel, tn_grid, dim3(256), 0, s, t);
    }
    SgdArgs g;
    g.hdr = hdr; g.max_rows = max_rows; g.n_splits = splits; g.partial = partial;
    g.F_in = layer->F_in; g.F_out = layer->F_out; g.F_pad = F_pad; g.N_pad = N_pad; g.n_op = n_op; g.W = layer->W; g.bias = layer->bias;
    g.W_bf16 = layer->W_bf16; g.Wt_bf16 = layer->Wt_bf16; g.lr = lr; g.wd = weight_decay; g.dW_out = dW_out; g.db_out = db_out;
    if (deferred) *deferred = g;
    else hipLaunchKernelGGL(sgd_reduce_kernel, dim3(sgd_reduce_blocks(F_pad, N_pad, n_op)), dim3(256), 0, s, g);
    CR_LAUNCH_CHECK();
    return CR_OK;
}

extern "C" cr_status cr_sage_linear_bwd(const cr_sage_layer *layer, const int32_t *hdr, int32_t max_rows,
                                        const uint16_t *h_self, const uint16_t *agg, int64_t ld_in,
                                        const uint16_t *dz_bf16, float lr, float weight_decay, float *d_self,
                                        float *d_agg, uint16_t *d_in_bf16, float *dW_out, float *db_out, void *ws,
                                        size_t ws_bytes, void *stream)
{
    return linear_bwd_products(layer, hdr, max_rows, h_self, agg, ld_in, dz_bf16, lr, weight_decay, d_self, d_agg, d_in_bf16,
                               dW_out, db_out, ws, ws_bytes, stream, nullptr);
}

extern "C" cr_status cr_sage_linear_bwd_input(const cr_sage_layer *layer, const int32_t *hdr, int32_t max_rows,
                                              const uint16_t *dz_bf16, float *d_self, float *d_agg, uint16_t *d_in_bf16,
                                              void *stream)
{
    int F_pad, N_pad;
    cr_status st = check_layer(layer, F_pad, N_pad);
    if (st != CR_OK) return st;
    CR_REQUIRE(hdr != nullptr && max_rows >= 1, CR_ERR_INVALID_ARG, "hdr must not be NULL and max_rows must be positive");
    CR_REQUIRE(dz_bf16 && aligned16(dz_bf16), CR_ERR_INVALID_ARG, "dz_bf16 must be a 16-byte aligned device pointer");
    const int n_op = layer->n_operands;
    CR_REQUIRE(n_op == 2 || d_self == nullptr, CR_ERR_INVALID_ARG, "a one-operand layer has no d_self");
    CR_REQUIRE(n_op == 1 || (d_self == nullptr) == (d_agg == nullptr), CR_ERR_INVALID_ARG, "d_self and d_agg must be given together");
    CR_REQUIRE(d_agg || d_in_bf16, CR_ERR_INVALID_ARG, "no output requested");
    CR_REQUIRE(aligned16(d_self) && aligned16(d_agg) && aligned16(d_in_bf16), CR_ERR_INVALID_ARG, "d_self / d_agg / d_in_bf16 must be 16-byte aligned");
    CR_REQUIRE((n_op * F_pad) % 64 == 0, CR_ERR_UNSUPPORTED, "input gradients of a one-operand layer need F_in rounded up to 32 to be a multiple of 64");
    if (dry_run()) return CR_OK;
    NtArgs a;
    a.hdr = hdr; a.max_rows = max_rows; a.A0 = dz_bf16; a.A1 = nullptr; a.lda = N_pad; a.K0 = N_pad; a.K = N_pad;
    a.B = layer->W_bf16; a.N = n_op * F_pad; a.bias = nullptr; a.relu = 0;
    a.C0 = n_op == 2 ? d_self : d_agg; a.C1 = d_agg; a.ldc = F_pad; a.N0 = F_pad; a.Cb = d_in_bf16; a.ldcb = n_op * F_pad;
    launch_nt(a, static_cast<hipStream_t>(stream));
    CR_LAUNCH_CHECK();
    return CR_OK;
}

extern "C" cr_status cr_softmax_xent(const int32_t *hdr, int32_t max_rows, const float *logits, int64_t ld,
                                     int32_t n_classes, const int32_t *labels, const int32_t *root_ids, float *loss,
                                     float *row_loss, float *d_logits, uint16_t *d_logits_bf16, void *stream)
{
    CR_REQUIRE(hdr != nullptr && max_rows >= 1, CR_ERR_INVALID_ARG, "hdr must not be NULL and max_rows must be positive");
    CR_REQUIRE(logits && labels && root_ids && loss && row_loss, CR_ERR_INVALID_ARG, "logits / labels / root_ids / loss / row_loss must not be NULL");
    CR_REQUIRE(n_classes >= 1 && ld >= n_classes, CR_ERR_INVALID_ARG, "need 1 <= n_classes <= ld");
    if (dry_run()) return CR_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    launch_xent(hdr, max_rows, logits, ld, n_classes, labels, root_ids, loss, row_loss, d_logits, d_logits_bf16, nullptr, s);
    CR_LAUNCH_CHECK();
    return CR_OK;
}

namespace cr {
// acc[0] += value * rows, acc[1] += rows, acc[2] = their ratio (one thread: the calls of a pass are ordered on their stream)
__global__ void mean_accumulate_kernel(const int32_t *hdr, int max_rows, const float *value, double *acc)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const int n = min(hdr[CR_HDR_N_DST], max_rows);
    if (n <= 0) return;
    const double sum = acc[0] + (double)value[0] * (double)n, rows = acc[1] + (double)n;
    acc[0] = sum;
    acc[1] = rows;
    acc[2] = sum / rows;
}
}  // namespace cr

extern "C" cr_status cr_mean_accumulate(const int32_t *hdr, int32_t max_rows, const float *value, double *acc, void *stream)
{
    CR_REQUIRE(hdr != nullptr && max_rows >= 1, CR_ERR_INVALID_ARG, "hdr must not be NULL and max_rows must be positive");
    CR_REQUIRE(value != nullptr && acc != nullptr, CR_ERR_INVALID_ARG, "value / acc must not be NULL");
    CR_REQUIRE((reinterpret_cast<uintptr_t>(acc) & 7u) == 0, CR_ERR_INVALID_ARG, "acc must be 8-byte aligned");
    if (dry_run()) return CR_OK;
    hipLaunchKernelGGL(mean_accumulate_kernel, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream), hdr, max_rows, value, acc);
    CR_LAUNCH_CHECK();
    return CR_OK;
}

extern "C" cr_status cr_count_correct(const int32_t *hdr, int32_t max_rows, const float *logits, int64_t ld,
                                      int32_t n_classes, const int32_t *labels, const int32_t *root_ids,
                                      int32_t *count, void *stream)
{
    CR_REQUIRE(hdr != nullptr && max_rows >= 1, CR_ERR_INVALID_ARG, "hdr must not be NULL and max_rows must be positive");
    CR_REQUIRE(logits && labels && root_ids && count, CR_ERR_INVALID_ARG, "logits / labels / root_ids / count must not be NULL");
    CR_REQUIRE(n_classes >= 1 && ld >= n_classes, CR_ERR_INVALID_ARG, "need 1 <= n_classes <= ld");
    if (dry_run()) return CR_OK;
    hipLaunchKernelGGL(count_correct_kernel, dim3((unsigned)ceil_div(max_rows, 4)), dim3(256), 0, static_cast<hipStream_t>(stream), hdr,
                       max_rows, logits, ld, n_classes, labels, root_ids, count);
    CR_LAUNCH_CHECK();
    return CR_OK;
}
