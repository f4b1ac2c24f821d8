// sma_f32.hip -- state-memory attention, forward and backward, on the fp32
// matrix instructions: fp32 storage at every shape, and either storage at the
// shapes outside the bf16 kernels' set (any chunk size S >= 1, N in {16, 32,
// 64, 128}, P = 64).  The paper trains at S = 16, N in {16, 64} (MQAR,
// App. D.1) and evaluates one checkpoint at S = 64 and 32 (Sec. 5.2).
//
// Every product but k_bsma's runs on v_mfma_f32_16x16x4_f32 (32 cycles of a SIMD each), so
// operands, sums and probabilities are fp32 throughout, as the definitions
// have them.  What bounds these kernels is that instruction's rate (154 TFLOP/s
// measured on a large matrix product): a wave's vector work per memory is about
// an eighth of its MFMA time, and one 16-byte LDS read feeds four to eight
// MFMAs.  Hence the layout: a memory dH_j is staged once per block as float
// rows of 64 columns in 16-byte chunks (chunk c of row n at c ^ (n & 15)), and
// both operand forms read it without bank conflicts, four values at a time:
//   rows p (contraction over n): lane (m, g) reads dH[16k + 4g + s][4m .. 4m+3]
//     at step s: element i belongs to row 4m + i, i.e. to the tile of rows
//     p = i (mod 4); four tiles per read;
//   rows n (contraction over p): lane (m, g) reads dH[16nt + m][16k + 4g .. +3]:
//     element s is the operand of step s, whose k index g means p = 16k + 4g + s.
// Lane (m, g) = (lane % 16, lane / 16); a wave's columns are 16 tokens.  With
// these orders a lane's accumulators of one token are 16 consecutive p (rows
// p) or 4 consecutive n (rows n), and its own operands are float4 pieces of
// q, C, e and dy rows.  The row scale r_j joins the token operand (or the row
// read), so no second copy of the memories is made.
//
// Measured, with the kernels these replaced (VALU dot products per token, and
// for fp32 storage at the tuned shapes bf16-style kernels of eight fp32 MFMAs a
// step): B 64, L 512, 4 heads, N 64, S 16, fp32: forward 3523 -> 354 us (94
// TFLOP/s), token side 6276 -> 908 (92), memory side 2257 -> 369 (90); B 2,
// L 2048, 8 heads, N 128, S 32, bf16: forward 5414 -> 96; B 2, L 2048, 24
// heads, N 128, S 256, fp32: 378 -> 125, 328 -> 294 and 577 -> 155.
//
//   k_fsma      per (64 tokens, b, h), 16 tokens a wave: U = dH^T (r . Qbar) and
//               V = dH^T C from the same reads, l = U . Ebar, the online
//               softmax of Alg. 1, the gated residual.  Tokens of a wave may
//               belong to different chunks (each is masked by its own).
//   k_fsma_split  the same where those blocks are few: 16 tokens a block, the
//               memories over its four waves.
//   k_bsma      the forward for bf16 storage and N >= 32, on the bf16
//               instructions with exact or split operands (comment there).
//   k_fbwd_prep Qbar and Ebar of every token (float).
//   k_fbwd_tok  per (64 tokens, b, h): pass 1 over the memories for the logits,
//               dy . V_j, the exact log-sum-exp of these logits and
//               Dy = R . dy; pass 2 for dl_j = g p_j (dy . V_j - Dy) and
//               dEbar += dH^T (r . Qbar dl), dQbar += r . dH (Ebar dl),
//               dC += dH (dy g p), accumulated in MFMA registers over the
//               memories; per head, the finishing kernel sums a group's heads.
//   k_fbwd_mem  per (b, h, up to 16 memories): M1 = sum_t (g p_j C_t)^T dy_t and
//               M2 = sum_t (dl_j Qbar_t)^T Ebar_t over the later tokens, staged
//               16 at a time for all the block's memories; then the gradient
//               through r_j.
#include <type_traits>

#include "f32_tiles.hpp"

namespace dart {
namespace {

constexpr int kP = 64;
constexpr int kFT = 256;   // threads: 4 waves
constexpr int kFTok = 64;  // tokens per block, 16 a wave

// One memory on its way from HBM to LDS: thread (row tid / 16 + 16 k, chunk
// tid % 16), loaded a memory ahead of its use and stored with its row scales
// when the other buffer is free.
template <typename T, int N>
struct MemStage {
    static constexpr int K = N / 16;
    float v[K][4];
    __device__ __forceinline__ void load(const T* __restrict__ src, int tid) {
#pragma unroll
        for (int k = 0; k < K; ++k) load4(src + tid * 4 + k * 1024, v[k]);
    }
    __device__ __forceinline__ void store(char* tile, float* r, float eps, int normalize, int tid) const {
        const int row = tid >> 4, c = tid & 15;
        char* dst = tile + row * 256 + ((c ^ row) << 4);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            *reinterpret_cast<f32x4*>(dst + k * 4096) = f32x4{v[k][0], v[k][1], v[k][2], v[k][3]};
            const float ss = dpp_group_sum<16>(v[k][0] * v[k][0] + v[k][1] * v[k][1] + v[k][2] * v[k][2] + v[k][3] * v[k][3]);
            if (c == 0) r[row + 16 * k] = normalize ? 1.0f / sqrtf(ss * (1.0f / kP) + eps) : 1.0f;
        }
    }
};

// Byte offsets of a lane's reads of a staged memory.
struct TileOff {
    int p[4];  // rows p: step s of a 16-row block (+ 4096 per block)
    int n[4];  // rows n: 16-column block k (+ 4096 per row tile)
    __device__ __forceinline__ void init(int m, int g) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            p[s] = (4 * g + s) * 256 + ((m ^ (4 * g + s)) << 4);
            n[s] = m * 256 + (((4 * s + g) ^ m) << 4);
        }
    }
};

// Row pieces of one token in operand order: v[k][s] = row[16 k + 4 g + s].
template <typename T, int K>
__device__ __forceinline__ void load_row(const T* __restrict__ row, int g, float (&v)[K][4]) {
#pragma unroll
    for (int k = 0; k < K; ++k) load4(row + 16 * k + 4 * g, v[k]);
}
// ... and in accumulator order: v[4 r + i] = row[16 g + 4 r + i].
template <typename T>
__device__ __forceinline__ void load_acc(const T* __restrict__ row, int g, float (&v)[4][4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) load4(row + 16 * g + 4 * r, v[r]);
}
// RMSNorm in place of a row whose pieces the four lanes (m, 0..3) hold.
template <int K>
__device__ __forceinline__ void norm_pieces(float (&v)[K][4], const float* __restrict__ w, int first, int step, float eps) {
    float ss = 0.f;
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int s = 0; s < 4; ++s) ss += v[k][s] * v[k][s];
    const float inv = 1.0f / sqrtf(row4_sum(ss) * (1.0f / (16 * K)) + eps);
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int s = 0; s < 4; ++s) v[k][s] *= inv * (w ? w[first + step * k + s] : 1.0f);
}

// U += dH^T (r . q) and V += dH^T c for the wave's 16 tokens.
template <int N>
__device__ __forceinline__ void read_memory(const char* tile, const float* r, const TileOff& off, int g,
                                            const float (&q)[N / 16][4], const float (&c)[N / 16][4],
                                            f32x4 (&U)[4], f32x4 (&V)[4]) {
#pragma unroll
    for (int k = 0; k < N / 16; ++k) {
        const f32x4 rk = *reinterpret_cast<const f32x4*>(r + 16 * k + 4 * g);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const f32x4 a = lds4(tile + off.p[s] + 4096 * k);
            const float bq = q[k][s] * rk[s];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                U[i] = mfma4(a[i], bq, U[i]);
                V[i] = mfma4(a[i], c[k][s], V[i]);
            }
        }
    }
}
// Dot of a column's accumulators with a row in accumulator order, in all four
// lanes of the column.
__device__ __forceinline__ float col_dot(const f32x4 (&U)[4], const float (&e)[4][4]) {
    float s[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        s[i] = U[i][0] * e[0][i] + U[i][1] * e[1][i] + U[i][2] * e[2][i] + U[i][3] * e[3][i];
    return row4_sum((s[0] + s[1]) + (s[2] + s[3]));
}

// e^(a - b) of two logits.  They stay in natural units, and their difference is
// scaled for the base-2 exponential: scaled each, both would be rounded at their own
// size (the attention's dC 5.9e-7 to 7.9e-7 from 64 bits at N 16 and 64, where
// 1/sqrt(N) is exact; 3.2e-7 to 4.6e-7 this way, no slower).
__device__ __forceinline__ float exp_diff(float a, float b) { return fast_exp2((a - b) * kLog2e); }

// ---- forward -----------------------------------------------------------------------
// Block order: heaviest (latest) tokens first, and blockIdx % (B H) = (b, h), so
// that for a multiple of eight (b, h) the blocks that read the same memories
// share an XCD's L2.
template <typename T, int N>
__global__ __launch_bounds__(kFT, 2) void k_fsma(
    const T* __restrict__ q, const T* __restrict__ e, const T* __restrict__ Cm,
    const T* __restrict__ mem, const T* __restrict__ z, const T* y_ssd, T* y, float* __restrict__ lse,
    const float* __restrict__ qw, const float* __restrict__ ew, float eps, int normalize,
    int z_per_head, int64_t L, int H, int G, int S, int64_t Mcap, int BH, int nblk) {
    constexpr int K = N / 16;
    __shared__ __attribute__((aligned(16))) char s_h[2][N * 256];
    __shared__ __attribute__((aligned(16))) float s_r[2][N];
    const int tid = threadIdx.x, lane = tid & 63, m = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned blk = (unsigned)flat_block(), bq = blk / (unsigned)BH;
    if (bq >= (unsigned)nblk) return;
    const int bh = (int)(blk % (unsigned)BH);
    const int64_t tb = (int64_t)(nblk - 1 - (int)bq) * kFTok;
    const int64_t b = bh / H;
    const int h = bh % H;
    const int grp = (int)((int64_t)h * G / H);
    const int64_t tw = tb + wave * 16, t = tw + m;
    const int64_t tc = t < L ? t : L - 1;  // tokens past the end repeat the last one, masked
    const int64_t last = tb + kFTok - 1 < L ? tb + kFTok - 1 : L - 1;
    const int64_t jb = last / S;  // memories this block stages
    const int64_t jw = tw < L ? (tw + 15 < last ? tw + 15 : last) / S : 0;  // and this wave reads
    const int64_t jt = t < L ? t / S : 0;                                    // and this token attends
    const int64_t row = (b * L + tc) * G + grp;
    const T* mh = mem + (b * Mcap * H + h) * (int64_t)(N * kP);
    const int64_t mstep = (int64_t)H * N * kP;
    MemStage<T, N> st;
    if (jb > 0) st.load(mh, tid);
    float qv[K][4], cv[K][4], ev[4][4];
    load_row<T, K>(q + row * N, g, qv);
    load_row<T, K>(Cm + row * N, g, cv);
    load_acc<T>(e + row * kP, g, ev);
    if (normalize) {
        norm_pieces<K>(qv, qw, 4 * g, 16, eps);
        norm_pieces<4>(ev, ew, 16 * g, 4, eps);
    }
    if (jb > 0) st.store(s_h[0], s_r[0], eps, normalize, tid);
    TileOff off;
    off.init(m, g);
    const float isn = 1.0f / sqrtf((float)N);
    float mx = -INFINITY, d = 0.f;
    f32x4 O[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) O[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int64_t j = 0; j < jb; ++j) {
        const int buf = (int)(j & 1);
        __syncthreads();
        if (j + 1 < jb) st.load(mh + (j + 1) * mstep, tid);
        if (j < jw) {
            f32x4 U[4], V[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) U[i] = V[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            read_memory<N>(s_h[buf], s_r[buf], off, g, qv, cv, U, V);
            const float l = col_dot(U, ev) * isn;
            if (j < jt) {  // the four lanes of a column agree
                const float mn = fmaxf(mx, l);
                const float al = exp_diff(mx, mn), pw = exp_diff(l, mn);
                mx = mn;
                d = d * al + pw;
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) O[i][r] = O[i][r] * al + pw * V[i][r];
            }
        }
        if (j + 1 < jb) st.store(s_h[buf ^ 1], s_r[buf ^ 1], eps, normalize, tid);
    }
    if (t >= L) return;
    const int64_t bt = b * L + t;
    const int64_t yi = (bt * H + h) * kP + 16 * g;
    const float f = jt > 0 ? silu(to_f(z[z_per_head ? bt * H + h : bt])) / d : 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float v[4];
        load4(y_ssd + yi + 4 * r, v);
        if (jt > 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] += f * O[i][r];
        }
        store4(y + yi + 4 * r, v);
    }
    if (lse && g == 0) lse[bt * H + h] = jt > 0 ? mx + log2f(d) * kLn2 : -INFINITY;
}

// ... where those blocks leave the chip idle: 16 tokens per block, wave w on the
// memories w, w + 4, ..., merged at the end.  A block of 64 tokens is a serial
// chain of memories at one SIMD's MFMA rate per wave (N 32: 2048 cycles a
// memory), which nothing shortens inside its CU; this takes four times as many
// CUs and a quarter of the chain.  A wave reads its operands from global memory
// in MFMA order (four rows of 256 bytes per load, 32 rows ahead of their use),
// without LDS or barriers before the merge.
template <typename T, int N>
__global__ __launch_bounds__(kFT, 2) void k_fsma_split(
    const T* __restrict__ q, const T* __restrict__ e, const T* __restrict__ Cm,
    const T* __restrict__ mem, const T* __restrict__ z, const T* y_ssd, T* y, float* __restrict__ lse,
    const float* __restrict__ qw, const float* __restrict__ ew, float eps, int normalize,
    int z_per_head, int64_t L, int H, int G, int S, int64_t Mcap, int BH, int nblk) {
    constexpr int K = N / 16, KC = K < 2 ? K : 2, NC = K / KC;  // 16-row blocks: all, per chunk of loads
    __shared__ float s_o[4][18][64];
    const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned blk = (unsigned)flat_block(), bq = blk / (unsigned)BH;
    if (bq >= (unsigned)nblk) return;
    const int bh = (int)(blk % (unsigned)BH);
    const int64_t tw = (int64_t)(nblk - 1 - (int)bq) * 16;
    const int64_t b = bh / H;
    const int h = bh % H;
    const int grp = (int)((int64_t)h * G / H);
    const int64_t t = tw + m, tc = t < L ? t : L - 1;
    const int64_t jw = (tw + 15 < L ? tw + 15 : L - 1) / S;
    const int64_t jt = t < L ? t / S : 0;
    const int64_t row = (b * L + tc) * G + grp;
    const int64_t mstep = (int64_t)H * N * kP;
    const T* mh = mem + (b * Mcap * H + h) * (int64_t)(N * kP) + g * 4 * kP + 4 * m;
    float nx[KC][4][4];
    auto load = [&](const T* src) {
#pragma unroll
        for (int k = 0; k < KC; ++k)
#pragma unroll
            for (int s = 0; s < 4; ++s) load4(src + (16 * k + s) * kP, nx[k][s]);
    };
    if (wave < jw) load(mh + wave * mstep);
    const int64_t bt = b * L + tc;
    const int64_t yi = (bt * H + h) * kP + 16 * g + 4 * wave;
    float yv[4];
    load4(y_ssd + yi, yv);
    const float zv = jw > 0 ? to_f(z[z_per_head ? bt * H + h : bt]) : 0.f;
    float qv[K][4], cv[K][4], ev[4][4];
    load_row<T, K>(q + row * N, g, qv);
    load_row<T, K>(Cm + row * N, g, cv);
    load_acc<T>(e + row * kP, g, ev);
    if (normalize) {
        norm_pieces<K>(qv, qw, 4 * g, 16, eps);
        norm_pieces<4>(ev, ew, 16 * g, 4, eps);
    }
    const float isn = 1.0f / sqrtf((float)N);
    // finite, so that a wave without memories (or with logits of -inf) merges as 0
    float mx = -__FLT_MAX__, d = 0.f;
    f32x4 O[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) O[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int64_t j = wave; j < jw; j += 4) {
        f32x4 U[4], V[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) U[i] = V[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            float a[KC][4][4];
#pragma unroll
            for (int k = 0; k < KC; ++k)
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int i = 0; i < 4; ++i) a[k][s][i] = nx[k][s][i];
            if (c + 1 < NC) load(mh + j * mstep + (c + 1) * KC * 16 * kP);
            else if (j + 4 < jw) load(mh + (j + 4) * mstep);
#pragma unroll
            for (int k = 0; k < KC; ++k)
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const float* v = a[k][s];
                    const float ss = dpp_group_sum<16>(v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3]);
                    const float r = normalize ? 1.0f / sqrtf(ss * (1.0f / kP) + eps) : 1.0f;
                    const float bq4 = qv[KC * c + k][s] * r;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        U[i] = mfma4(v[i], bq4, U[i]);
                        V[i] = mfma4(v[i], cv[KC * c + k][s], V[i]);
                    }
                }
        }
        const float l = col_dot(U, ev) * isn;
        if (j < jt) {
            const float mn = fmaxf(mx, l);
            const float al = exp_diff(mx, mn), pw = exp_diff(l, mn);
            mx = mn;
            d = d * al + pw;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) O[i][r] = O[i][r] * al + pw * V[i][r];
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) s_o[wave][4 * r + i][lane] = O[i][r];
    s_o[wave][16][lane] = mx;
    s_o[wave][17][lane] = d;
    __syncthreads();
    if (t >= L) return;
    if (jt > 0) {  // wave r adds up the channels 16 g + 4 r + i
        float v[4] = {0.f, 0.f, 0.f, 0.f};
        mx = fmaxf(fmaxf(s_o[0][16][lane], s_o[1][16][lane]), fmaxf(s_o[2][16][lane], s_o[3][16][lane]));
        d = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float al = exp_diff(s_o[w][16][lane], mx);
            d += al * s_o[w][17][lane];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] += al * s_o[w][4 * wave + i][lane];
        }
        const float f = silu(zv) / d;
#pragma unroll
        for (int i = 0; i < 4; ++i) yv[i] += f * v[i];
    }
    store4(y + yi, yv);
    if (lse && g == 0 && wave == 0) lse[bt * H + h] = jt > 0 ? mx + log2f(d) * kLn2 : -INFINITY;
}

// ---- forward, bf16 storage ------------------------------------------------------------
// The same with the products on the bf16 matrix instructions, eight times the
// fp32 ones' rate, and nothing rounded on the way: a stored memory and C are
// bf16 as they stand, so V = dH^T C^T is exact in its operands, and the logit
// contracts over p first, W = dH Ebar^T with Ebar as three bf16 (8 bits each,
// all 24 of the float), then l = sum_n Qbar_n r_n W_n in float.  (The other order
// would need that split of r . dH or Qbar.)  Rows of 128 bytes in LDS, 16-byte
// chunks swizzled by row.  Eight waves: four take the even memories of the
// block's 64 tokens, four the odd ones, and their softmax states merge at the
// end, so that the heaviest blocks of a small problem are half as long.
// Bound by the 64 MFMAs per 16 tokens and memory and the vector work beside them
// (two operations per W element, and the staging), two waves a SIMD at N = 128.
// B 2, L 2048, 8 heads, N 128, S 32: 96 us (the VALU kernel before the matrix
// ones 5414, the fp32 instructions 466); 79 with Ebar cut to two bf16 and the
// hardware's approximate 1/sqrt, which put the logits 1.9e-5 from 64 bits instead
// of 1.0e-6 (the VALU kernel 1.4e-6).
template <int N>
struct MemStage16 {
    static constexpr int K = N / 32;  // 16-byte pieces per thread
    uint4 v[K];
    __device__ __forceinline__ void load(const bf16* __restrict__ src, int tid) {
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = reinterpret_cast<const uint4*>(src)[tid + k * kFT];
    }
    __device__ __forceinline__ void store(char* tile, float* r, float eps, int normalize, int tid) const {
        const int row = tid >> 3, c = tid & 7;
        float mine = 0.f;  // lane c of a row's eight finishes the row of piece c
#pragma unroll
        for (int k = 0; k < K; ++k) {
            *reinterpret_cast<uint4*>(tile + SwzTile<128>::off(row, c * 16) + k * 4096) = v[k];
            const uint32_t w[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
            float ss = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bf16x2 h = __builtin_bit_cast(bf16x2, w[i]);
                ss = __builtin_amdgcn_fdot2_f32_bf16(h, h, ss, false);
            }
            ss = dpp_group_sum<8>(ss);
            mine = c == k ? ss : mine;
        }
        if (c < K) r[row + 32 * c] = normalize ? 1.0f / sqrtf(mine * (1.0f / kP) + eps) : 1.0f;
    }
};

template <int N>
__global__ __launch_bounds__(2 * kFT, N < 128 ? 4 : 2) void k_bsma(
    const bf16* __restrict__ q, const bf16* __restrict__ e, const bf16* __restrict__ Cm,
    const bf16* __restrict__ mem, const bf16* __restrict__ z, const bf16* y_ssd, bf16* y,
    float* __restrict__ lse, const float* __restrict__ qw, const float* __restrict__ ew, float eps,
    int normalize, int z_per_head, int64_t L, int H, int G, int S, int64_t Mcap, int BH, int nblk) {
    constexpr int NT = N / 16, KS = N / 32;
    __shared__ __attribute__((aligned(16))) char s_h[2][2][N < 64 ? 64 * 128 : N * 128];  // [buffer][memory of the step]
    __shared__ __attribute__((aligned(16))) float s_r[2][2][N];
    const int tid = threadIdx.x & (kFT - 1), lane = tid & 63, m = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int odd = __builtin_amdgcn_readfirstlane(threadIdx.x / kFT);
    const unsigned blk = (unsigned)flat_block(), bq = blk / (unsigned)BH;
    if (bq >= (unsigned)nblk) return;
    const int bh = (int)(blk % (unsigned)BH);
    const int64_t tb = (int64_t)(nblk - 1 - (int)bq) * kFTok;
    const int64_t b = bh / H;
    const int h = bh % H;
    const int grp = (int)((int64_t)h * G / H);
    const int64_t tw = tb + wave * 16, t = tw + m;
    const int64_t tc = t < L ? t : L - 1;
    const int64_t last = tb + kFTok - 1 < L ? tb + kFTok - 1 : L - 1;
    const int64_t jb = last / S;
    const int64_t jw = tw < L ? (tw + 15 < last ? tw + 15 : last) / S : 0;
    const int64_t jt = t < L ? t / S : 0;
    const int64_t row = (b * L + tc) * G + grp;
    const bf16* mh = mem + (b * Mcap * H + h) * (int64_t)(N * kP);
    const int64_t mstep = (int64_t)H * N * kP;
    MemStage16<N> st;  // memory 2 s + odd of step s
    if (odd < jb) st.load(mh + odd * mstep, tid);
    float qv[NT][4];
    load_row<bf16, NT>(q + row * N, g, qv);
    if (normalize) norm_pieces<NT>(qv, qw, 4 * g, 16, eps);
    bf16x8 eh[2], em[2], el[2], cf[KS];
    {
        // Ebar in operand order: elements 32 ks + 8 g + 0 .. 7
        float ev[4][4];
#pragma unroll
        for (int k = 0; k < 4; ++k) load4(e + row * kP + 32 * (k >> 1) + 8 * g + 4 * (k & 1), ev[k]);
        float ss = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i) ss += ev[k][i] * ev[k][i];
        const float inv = normalize ? 1.0f / sqrtf(row4_sum(ss) * (1.0f / kP) + eps) : 1.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int p = 32 * (k >> 1) + 8 * g + 4 * (k & 1) + i;
                const float v = ev[k][i] * (inv * (normalize && ew ? ew[p] : 1.0f));
                const bf16 hi = (bf16)v, mid = (bf16)(v - (float)hi);
                eh[k >> 1][4 * (k & 1) + i] = hi;
                em[k >> 1][4 * (k & 1) + i] = mid;
                el[k >> 1][4 * (k & 1) + i] = (bf16)((v - (float)hi) - (float)mid);
            }
    }
#pragma unroll
    for (int k = 0; k < KS; ++k) {
        const bf16x4 c0 = *reinterpret_cast<const bf16x4*>(Cm + row * N + 32 * k + 4 * g);
        const bf16x4 c1 = *reinterpret_cast<const bf16x4*>(Cm + row * N + 32 * k + 16 + 4 * g);
        cf[k] = bf16x8{c0[0], c0[1], c0[2], c0[3], c1[0], c1[1], c1[2], c1[3]};
    }
    if (odd < jb) st.store(s_h[0][odd], s_r[0][odd], eps, normalize, tid);
    // lane offsets of the two readings: rows n (k steps of 32 p), and the
    // transposing reads of column tile pt (k steps of 32 n: 32 rows further)
    uint32_t on[2];
    KmOffBf16<128> ot[4];
#pragma unroll
    for (int k = 0; k < 2; ++k) on[k] = (uint32_t)SwzTile<128>::off(m, (32 * k + 8 * g) * 2);
#pragma unroll
    for (int pt = 0; pt < 4; ++pt) ot[pt].init(4 * g, 16 + 4 * g, 16 * pt, lane);
    const float isn = 1.0f / sqrtf((float)N);
    float mx = -INFINITY, d = 0.f;
    f32x4 O[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) O[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int64_t j = odd; j - odd < jb; j += 2) {
        const int buf = (int)((j >> 1) & 1);
        __syncthreads();
        if (j + 2 < jb) st.load(mh + (j + 2) * mstep, tid);
        if (j < jw) {
            const char* tile = s_h[buf][odd];
            float l4[2] = {0.f, 0.f};
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                bf16x8 a[2];
#pragma unroll
                for (int k = 0; k < 2; ++k) a[k] = *reinterpret_cast<const bf16x8*>(tile + on[k] + 2048 * n);
                // the small parts first
                f32x4 w = mma16(mma16(f32x4{0.f, 0.f, 0.f, 0.f}, a[0], el[0]), a[1], el[1]);
                w = mma16(mma16(w, a[0], em[0]), a[1], em[1]);
                w = mma16(mma16(w, a[0], eh[0]), a[1], eh[1]);
                const f32x4 rn = *reinterpret_cast<const f32x4*>(&s_r[buf][odd][16 * n + 4 * g]);
#pragma unroll
                for (int i = 0; i < 4; ++i) l4[n & 1] += qv[n][i] * rn[i] * w[i];
            }
            const float l = row4_sum(l4[0] + l4[1]) * isn;
            const bool at = j < jt, grow = at && l > mx;
            if (__builtin_amdgcn_ballot_w64(grow)) {  // (rare after the first memories)
                const float mn = grow ? l : mx, al = grow ? exp_diff(mx, mn) : 1.f;
                mx = mn;
                d *= al;
#pragma unroll
                for (int i = 0; i < 4; ++i) O[i] *= al;
            }
            const float pw = at ? exp_diff(l, mx) : 0.f;
            d += pw;
#pragma unroll
            for (int pt = 0; pt < 4; ++pt) {
                f32x4 V = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < KS; ++k) V = mma16(V, ot[pt].read(tile, 4096 * k), cf[k]);
                if (at) O[pt] += V * pw;  // (0 times an infinity or NaN of a memory past the token's is not 0)
            }
        }
        if (j + 2 < jb) st.store(s_h[buf ^ 1][odd], s_r[buf ^ 1][odd], eps, normalize, tid);
    }
    // the two halves of a token's memories meet in the waves of the even ones
    // (O, maximum and sum where the memories were)
    static_assert(sizeof(s_h) >= 18 * 256 * 4, "room for 256 lanes");
    float* so = reinterpret_cast<float*>(&s_h[0][0][0]) + (wave * 64 + lane) * 18;
    __syncthreads();
    if (odd) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) so[4 * i + r] = O[i][r];
        so[16] = mx;
        so[17] = d;
    }
    __syncthreads();
    if (odd || t >= L) return;
    if (jt > 1) {
        const float m1 = so[16], mn = fmaxf(mx, m1);
        const float a0 = exp_diff(mx, mn), a1 = exp_diff(m1, mn);
        mx = mn;
        d = d * a0 + so[17] * a1;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) O[i][r] = O[i][r] * a0 + so[4 * i + r] * a1;
    }
    const int64_t bt = b * L + t;
    const int64_t yi = (bt * H + h) * kP + 4 * g;
    const float f = jt > 0 ? silu(to_f(z[z_per_head ? bt * H + h : bt])) / d : 0.f;
#pragma unroll
    for (int pt = 0; pt < 4; ++pt) {
        float v[4];
        load4(y_ssd + yi + 16 * pt, v);
        if (jt > 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] += f * O[pt][i];
        }
        store4(y + yi + 16 * pt, v);
    }
    if (lse && g == 0) lse[bt * H + h] = jt > 0 ? mx + log2f(d) * kLn2 : -INFINITY;
}

// ---- backward ----------------------------------------------------------------------
// One wave per 16 (b, t, group) rows: Qbar (without the 1/sqrt(N)) and Ebar.
template <typename T, int N>
__global__ __launch_bounds__(kFT) void k_fbwd_prep(const T* __restrict__ q, const T* __restrict__ e,
                                                   const float* __restrict__ qw, const float* __restrict__ ew,
                                                   float eps, int normalize, float* __restrict__ qb,
                                                   float* __restrict__ eb, int64_t rows) {
    constexpr int K = N / 16;
    const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    const int64_t r0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16 + m;
    const int64_t row = r0 < rows ? r0 : rows - 1;
    float qv[K][4], ev[4][4];
    load_row<T, K>(q + row * N, g, qv);
    load_row<T, 4>(e + row * kP, g, ev);
    if (normalize) {
        norm_pieces<K>(qv, qw, 4 * g, 16, eps);
        norm_pieces<4>(ev, ew, 4 * g, 16, eps);
    }
    if (r0 >= rows) return;
#pragma unroll
    for (int k = 0; k < K; ++k) store4(qb + row * N + 16 * k + 4 * g, qv[k]);
#pragma unroll
    for (int k = 0; k < 4; ++k) store4(eb + row * kP + 16 * k + 4 * g, ev[k]);
}

// gp and dl, [b][h][memory][Ls]: pass 1 leaves the logit and
// dy . V_j there, pass 2 turns them into g p_j and dl_j / sqrt(N) for the
// memory kernel.  Blocks as in the forward, without those of chunk 0 alone.
template <typename T, int N>
__global__ __launch_bounds__(kFT, 2) void k_fbwd_tok(
    const float* __restrict__ qb, const float* __restrict__ eb, const T* __restrict__ Cm,
    const T* __restrict__ mem, const T* __restrict__ z, const T* __restrict__ dy, float eps,
    int normalize, int z_per_head, float* gp, float* dl, float* __restrict__ rdy,
    float* __restrict__ part, int64_t L, int64_t Ls, int H, int G, int S, int64_t Mcap, int64_t Mp,
    int BH, int nblk, int used) {
    constexpr int K = N / 16;
    __shared__ __attribute__((aligned(16))) char s_h[2][N * 256];
    __shared__ __attribute__((aligned(16))) float s_r[2][N];
    const int tid = threadIdx.x, lane = tid & 63, m = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned blk = (unsigned)flat_block(), bq = blk / (unsigned)BH;
    if (bq >= (unsigned)used) return;
    const int bh = (int)(blk % (unsigned)BH);
    const int64_t tb = (int64_t)(nblk - 1 - (int)bq) * kFTok;
    const int64_t b = bh / H;
    const int h = bh % H;
    const int grp = (int)((int64_t)h * G / H);
    const int64_t tw = tb + wave * 16, t = tw + m;
    const int64_t tc = t < L ? t : L - 1;
    const int64_t last = tb + kFTok - 1 < L ? tb + kFTok - 1 : L - 1;
    const int64_t jb = last / S;
    const int64_t jw = tw < L ? (tw + 15 < last ? tw + 15 : last) / S : 0;
    const int64_t jt = t < L ? t / S : 0;
    const int64_t bt = b * L + tc, row = bt * G + grp;
    const T* mh = mem + (b * Mcap * H + h) * (int64_t)(N * kP);
    const int64_t mstep = (int64_t)H * N * kP;
    // this token's column of the (memory, token) arrays
    const int64_t col = (int64_t)bh * Mp * Ls + tc;
    MemStage<T, N> st;
    if (jb > 0) {
        st.load(mh, tid);
        st.store(s_h[0], s_r[0], eps, normalize, tid);
    }
    TileOff off;
    off.init(m, g);
    float qv[K][4];
    load_row<float, K>(qb + row * N, g, qv);
    const float isn = 1.0f / sqrtf((float)N);
    float mx = -INFINITY, d = 0.f, sd = 0.f;
    {
        float cv[K][4], ev[4][4], dv[4][4];
        load_row<T, K>(Cm + row * N, g, cv);
        load_acc<float>(eb + row * kP, g, ev);
        load_acc<T>(dy + (bt * H + h) * kP, g, dv);
        for (int64_t j = 0; j < jb; ++j) {
            const int buf = (int)(j & 1);
            __syncthreads();
            // the last step brings memory 0 back for pass 2
            st.load(mh + (j + 1 < jb ? j + 1 : 0) * mstep, tid);
            if (j < jw) {
                f32x4 U[4], V[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) U[i] = V[i] = f32x4{0.f, 0.f, 0.f, 0.f};
                read_memory<N>(s_h[buf], s_r[buf], off, g, qv, cv, U, V);
                const float l = col_dot(U, ev) * isn, dw = col_dot(V, dv);
                if (j < jt) {
                    const float mn = fmaxf(mx, l);
                    const float al = exp_diff(mx, mn), pw = exp_diff(l, mn);
                    mx = mn;
                    d = d * al + pw;
                    sd = sd * al + pw * dw;
                    if (g == 0) {
                        gp[col + j * Ls] = l;
                        dl[col + j * Ls] = dw;
                    }
                }
            }
            st.store(s_h[buf ^ 1], s_r[buf ^ 1], eps, normalize, tid);
        }
    }
    const float Dy = sd / d, gd = silu(to_f(z[z_per_head ? bt * H + h : bt])) / d;
    if (jt > 0 && g == 0) rdy[bt * H + h] = Dy;
    float ev[4][4], dv[4][4];
    load_row<float, 4>(eb + row * kP, g, ev);
    load_row<T, 4>(dy + (bt * H + h) * kP, g, dv);
    f32x4 aE[4], aC[K], aQ[K];
#pragma unroll
    for (int i = 0; i < 4; ++i) aE[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < K; ++k) aC[k] = aQ[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int64_t j = 0; j < jb; ++j) {
        const int buf = (int)((jb + j) & 1);
        // the barrier also orders pass 1's stores of the logits before the loads here
        __syncthreads();
        if (j + 1 < jb) st.load(mh + (j + 1) * mstep, tid);
        if (j < jw) {
            float gpv = 0.f, dlv = 0.f;
            if (j < jt) {
                gpv = gd * exp_diff(gp[col + j * Ls], mx);
                dlv = gpv * (dl[col + j * Ls] - Dy) * isn;
            }
            // every lane of the column has read them before they are replaced
            __builtin_amdgcn_wave_barrier();
            if (j < jt && g == 0) {
                gp[col + j * Ls] = gpv;
                dl[col + j * Ls] = dlv;
            }
            const char* tile = s_h[buf];
            const float* r = s_r[buf];
            // A memory's sums are formed apart and added to the earlier ones' as a
            // whole: one chain over all memories rounds at every 4 products (B 2,
            // L 1000, 4 heads, N 16, S 16: dq 1.24e-6 and dC 8.6e-7 from 64 bits,
            // 1.11e-6 and 7.6e-7 so; a layer's training step takes 0.5 % longer).
            f32x4 e1[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) e1[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const f32x4 rk = *reinterpret_cast<const f32x4*>(r + 16 * k + 4 * g);
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const f32x4 a = lds4(tile + off.p[s] + 4096 * k);
                    const float bq = qv[k][s] * rk[s] * dlv;
#pragma unroll
                    for (int i = 0; i < 4; ++i) e1[i] = mfma4(a[i], bq, e1[i]);
                }
            }
            // (a branch: 0 times an infinity or NaN of a memory past the token's is not 0)
            if (j < jt) {
#pragma unroll
                for (int i = 0; i < 4; ++i) aE[i] += e1[i];
            }
            float eg[4][4], dg[4][4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    eg[k][s] = ev[k][s] * dlv;
                    dg[k][s] = dv[k][s] * gpv;
                }
#pragma unroll
            for (int nt = 0; nt < K; ++nt) {
                const float rn = r[16 * nt + m];
                f32x4 c1 = f32x4{0.f, 0.f, 0.f, 0.f}, q1 = c1;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const f32x4 a = lds4(tile + off.n[k] + 4096 * nt);
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        c1 = mfma4(a[s], dg[k][s], c1);
                        q1 = mfma4(a[s] * rn, eg[k][s], q1);
                    }
                }
                if (j < jt) {
                    aC[nt] += c1;
                    aQ[nt] += q1;
                }
            }
        }
        if (j + 1 < jb) st.store(s_h[buf ^ 1], s_r[buf ^ 1], eps, normalize, tid);
    }
    if (jt == 0) return;  // the finishing kernel reads no partial of chunk 0
    float* pr = part + (bt * H + h) * (int64_t)(2 * N + kP);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const float vq[4] = {aQ[k][0], aQ[k][1], aQ[k][2], aQ[k][3]};
        const float vc[4] = {aC[k][0], aC[k][1], aC[k][2], aC[k][3]};
        store4(pr + 16 * k + 4 * g, vq);
        store4(pr + N + kP + 16 * k + 4 * g, vc);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float ve[4] = {aE[0][r], aE[1][r], aE[2][r], aE[3][r]};
        store4(pr + N + 16 * g + 4 * r, ve);
    }
}

// Memory side.  A block takes NR of the N rows (rows are independent, the
// gradient through r_j included) of JJ memories; its waves split the rows (WN of
// them, NTW row tiles each) and, for NR < 64, the memories, JW each: at most 128
// accumulator registers.  Token rows in LDS with 16 floats of padding (the four
// k groups of a read then fall on different banks).
template <int NR>
struct MemSplit {
    static constexpr int WN = NR / 16 < 4 ? NR / 16 : 4;
    static constexpr int NTW = NR / 16 / WN;
    static constexpr int WJ = 4 / WN;
    static constexpr int JWMAX = 4 / NTW;
};
template <typename T, int N, int NR, int JW>
__global__ __launch_bounds__(kFT, 2) void k_fbwd_mem(
    const float* __restrict__ qb, const float* __restrict__ eb, const T* __restrict__ Cm,
    const T* __restrict__ dy, const T* __restrict__ mem, const float* __restrict__ gp,
    const float* __restrict__ dl, float* __restrict__ dmem, float eps, int normalize, int64_t L,
    int64_t Ls, int H, int G, int S, int64_t Mcap, int64_t Mp, int BH) {
    using Sp = MemSplit<NR>;
    constexpr int NTW = Sp::NTW, WN = Sp::WN, JJ = JW * Sp::WJ;
    constexpr int TT = 16;
    constexpr int RN = NR + 16, RP = kP + 16;       // row pitches in floats
    constexpr int CN = (TT * NR / 4 + kFT - 1) / kFT;  // float4 pieces per thread of C or Qbar
    constexpr int CF = (2 * JJ * TT + kFT - 1) / kFT;  // factors per thread
    __shared__ __attribute__((aligned(16))) float s_c[2][TT][RN], s_q[2][TT][RN], s_y[2][TT][RP], s_e[2][TT][RP];
    __shared__ float s_f[2][2][JJ][TT];
    const int tid = threadIdx.x, lane = tid & 63, m = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % WN, wj = wave / WN;
    // heaviest memories first
    const unsigned blk = (unsigned)flat_block(), per = (unsigned)BH * (N / NR);
    const int64_t j0 = (int64_t)(blk / per) * JJ;
    const int bh = (int)(blk % per % (unsigned)BH);
    const int n0 = (int)(blk % per / (unsigned)BH) * NR;
    if (j0 >= Mcap) return;
    const int64_t b = bh / H;
    const int h = bh % H;
    const int grp = (int)((int64_t)h * G / H);
    f32x4 m1[JW][NTW][4], m2[JW][NTW][4];
#pragma unroll
    for (int a = 0; a < JW; ++a)
#pragma unroll
        for (int n = 0; n < NTW; ++n)
#pragma unroll
            for (int p = 0; p < 4; ++p) m1[a][n][p] = m2[a][n][p] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int64_t tbeg = (j0 + 1) * S;  // memories past Mp - 1 start at or past L
    float rc[CN][4], rq[CN][4], ry[4], re[4], rf[CF];
    auto load = [&](int64_t t0) {
#pragma unroll
        for (int k = 0; k < CN; ++k) {
            const int i = tid + k * kFT;
            if (i < TT * NR / 4) {
                const int64_t t = t0 + i / (NR / 4);
                const int64_t row = (b * L + (t < L ? t : L - 1)) * G + grp;
                load4(Cm + row * N + n0 + 4 * (i % (NR / 4)), rc[k]);
                load4(qb + row * N + n0 + 4 * (i % (NR / 4)), rq[k]);
            }
        }
        const int64_t t = t0 + (tid >> 4);
        const int64_t bt = b * L + (t < L ? t : L - 1);
        load4(dy + (bt * H + h) * kP + 4 * (tid & 15), ry);
        load4(eb + (bt * G + grp) * kP + 4 * (tid & 15), re);
#pragma unroll
        for (int k = 0; k < CF; ++k) {
            const int i = tid + k * kFT;
            const int64_t j = j0 + (i / TT) % JJ, tf = t0 + i % TT;
            rf[k] = 0.f;
            // written for the tokens after the memory's chunk only
            if (i < 2 * JJ * TT && j < Mp && tf < L && tf >= (j + 1) * S)
                rf[k] = (i < JJ * TT ? gp : dl)[((int64_t)bh * Mp + j) * Ls + tf];
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int k = 0; k < CN; ++k) {
            const int i = tid + k * kFT;
            if (i < TT * NR / 4) {
                store4(&s_c[buf][i / (NR / 4)][4 * (i % (NR / 4))], rc[k]);
                store4(&s_q[buf][i / (NR / 4)][4 * (i % (NR / 4))], rq[k]);
            }
        }
        store4(&s_y[buf][tid >> 4][4 * (tid & 15)], ry);
        store4(&s_e[buf][tid >> 4][4 * (tid & 15)], re);
#pragma unroll
        for (int k = 0; k < CF; ++k) {
            const int i = tid + k * kFT;
            if (i < 2 * JJ * TT) (&s_f[buf][0][0][0])[i] = rf[k];
        }
    };
    int buf = 0;
    if (j0 < Mp && tbeg < L) {
        load(tbeg);
        store(0);
    }
    int64_t t0 = tbeg;
    // Until the last of the block's memories is attended (RAMP), a token's operands
    // are taken for the memories before its chunk only: a factor of 0 would let
    // its infinities and NaN through to the others.
    auto sweep = [&](int64_t end, auto ramp) __attribute__((always_inline)) {
        for (; t0 < end; t0 += TT, buf ^= 1) {
            __syncthreads();
            const bool more = t0 + TT < L;
            if (more) load(t0 + TT);
#pragma unroll
            for (int ks = 0; ks < TT / 4; ++ks) {
                const int t = 4 * ks + g;
                float ac[NTW], aq[NTW];
#pragma unroll
                for (int n = 0; n < NTW; ++n) {
                    ac[n] = s_c[buf][t][wn * 16 * NTW + NTW * m + n];
                    aq[n] = s_q[buf][t][wn * 16 * NTW + NTW * m + n];
                }
                const f32x4 vy = *reinterpret_cast<const f32x4*>(&s_y[buf][t][4 * m]);
                const f32x4 ve = *reinterpret_cast<const f32x4*>(&s_e[buf][t][4 * m]);
#pragma unroll
                for (int a = 0; a < JW; ++a) {
                    const float fg = s_f[buf][0][wj * JW + a][t], fd = s_f[buf][1][wj * JW + a][t];
                    const bool in = !decltype(ramp)::value || t0 + t >= (j0 + wj * JW + a + 1) * S;
#pragma unroll
                    for (int n = 0; n < NTW; ++n) {
                        const float c1 = in ? ac[n] * fg : 0.f, q1 = in ? aq[n] * fd : 0.f;
#pragma unroll
                        for (int p = 0; p < 4; ++p) {
                            m1[a][n][p] = mfma4(c1, in ? vy[p] : 0.f, m1[a][n][p]);
                            m2[a][n][p] = mfma4(q1, in ? ve[p] : 0.f, m2[a][n][p]);
                        }
                    }
                }
            }
            if (more) store(buf ^ 1);
        }
    };
    if (j0 < Mp) {
        if constexpr (JJ > 1) sweep((j0 + JJ) * S < L ? (j0 + JJ) * S : L, std::true_type());
        sweep(L, std::false_type());
    }
    // through r_j: ddH = M1 + r M2 - (r^3 / P) rowsum(dH M2) dH; lane: row
    // NTW (4 g + r) + n of the wave's rows, columns 4 m .. 4 m + 3
#pragma unroll
    for (int a = 0; a < JW; ++a) {
        const int64_t j = j0 + wj * JW + a;
        if (j >= Mcap) continue;
        const T* hs = mem + ((b * Mcap + j) * H + h) * (int64_t)(N * kP);
        float* out = dmem + ((b * Mcap + j) * H + h) * (int64_t)(N * kP);
#pragma unroll
        for (int n = 0; n < NTW; ++n)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int o = (n0 + wn * 16 * NTW + NTW * (4 * g + r) + n) * kP + 4 * m;
                float o4[4] = {0.f, 0.f, 0.f, 0.f};
                if (j < Mp) {
                    float hv[4];
                    load4(hs + o, hv);
                    float s1 = 0.f, s2 = 0.f;
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        s1 += hv[p] * hv[p];
                        s2 += hv[p] * m2[a][n][p][r];
                    }
                    s1 = dpp_group_sum<16>(s1);
                    s2 = dpp_group_sum<16>(s2);
                    const float rr = normalize ? 1.0f / sqrtf(s1 * (1.0f / kP) + eps) : 1.0f;
                    const float cr = normalize ? rr * rr * rr * (1.0f / kP) * s2 : 0.f;
#pragma unroll
                    for (int p = 0; p < 4; ++p) o4[p] = m1[a][n][p][r] + rr * m2[a][n][p][r] - cr * hv[p];
                }
                store4(out + o, o4);
            }
    }
}

// ---- launchers -----------------------------------------------------------------------
template <typename T, int N>
hipError_t run_fsma(const Shape& s, const SmaArgs& a, const void* q, const void* e, const void* Cm,
                    const void* mem, const void* z, const void* ys, void* y, float* lse, hipStream_t st) {
    const int BH = (int)(s.B * s.H);
    const int nblk = (int)((s.L + kFTok - 1) / kFTok);
    prof_begin("k_sma", st);
    // (at N = 16 a bf16 k step of 32 would be half empty)
    if constexpr (sizeof(T) == 2 && N >= 32) {
        k_bsma<N><<<flat_grid((int64_t)BH * nblk, 2 * kFT), 2 * kFT, 0, st>>>(
            (const T*)q, (const T*)e, (const T*)Cm, (const T*)mem, (const T*)z, (const T*)ys, (T*)y, lse,
            a.qw, a.ew, a.eps, a.normalize, a.z_per_head, s.L, s.H, s.G, s.S, s.Mcap, BH, nblk);
    } else if ((int64_t)BH * nblk <= device_cu_count()) {
        // (fp32, blocks of 64 tokens at most one per CU: L 512, 2 heads, N 32, S 64
        // 19.0 -> 12.5 us; L 1024, 8 heads, N 64, S 16 184 -> 91; L 2048, 8 heads,
        // N 128, S 64, 256 blocks, 177 -> 132.  At two per CU the waves of k_fsma
        // fill the SIMDs and its shared staging wins: L 4096, 8 heads, N 128,
        // S 256 118 against 131; at eight 608 against 896)
        const int n16 = (int)((s.L + 15) / 16);
        k_fsma_split<T, N><<<flat_grid((int64_t)BH * n16, kFT), kFT, 0, st>>>(
            (const T*)q, (const T*)e, (const T*)Cm, (const T*)mem, (const T*)z, (const T*)ys, (T*)y, lse,
            a.qw, a.ew, a.eps, a.normalize, a.z_per_head, s.L, s.H, s.G, s.S, s.Mcap, BH, n16);
    } else {
        k_fsma<T, N><<<flat_grid((int64_t)BH * nblk, kFT), kFT, 0, st>>>(
            (const T*)q, (const T*)e, (const T*)Cm, (const T*)mem, (const T*)z, (const T*)ys, (T*)y, lse,
            a.qw, a.ew, a.eps, a.normalize, a.z_per_head, s.L, s.H, s.G, s.S, s.Mcap, BH, nblk);
    }
    prof_end(st);
    return hipGetLastError();
}

template <typename T, int N>
hipError_t run_fsma_bwd(const Shape& s, const SmaArgs& a, const void* q, const void* e,
                        const void* Cm, const void* mem, const void* z, const void* dy,
                        const GenBwdWs& w, float* dmem, hipStream_t st) {
    const int64_t Mp = s.M > 1 ? s.M - 1 : 0;
    const int BH = (int)(s.B * s.H);
    if (Mp > 0) {
        const int64_t rows = s.B * s.L * s.G;
        prof_begin("k_bwd_prep", st);
        k_fbwd_prep<T, N><<<(unsigned)((rows + 63) / 64), kFT, 0, st>>>(
            (const T*)q, (const T*)e, a.qw, a.ew, a.eps, a.normalize, w.qb, w.eb, rows);
        prof_end(st);
        const int64_t nblk = (s.L + kFTok - 1) / kFTok, used = nblk - s.S / kFTok;
        prof_begin("k_bwd_tokens", st);
        k_fbwd_tok<T, N><<<flat_grid(BH * used, kFT), kFT, 0, st>>>(
            w.qb, w.eb, (const T*)Cm, (const T*)mem, (const T*)z, (const T*)dy, a.eps, a.normalize,
            a.z_per_head, w.gp, w.dl, w.rdy, w.part, s.L, w.Ls, s.H, s.G, s.S, s.Mcap, Mp, BH, (int)nblk, (int)used);
        prof_end(st);
    }
    // As many memories per block as the registers hold (the token stream is then
    // staged least often), unless that leaves fewer blocks than two per CU: then
    // one memory and at most 64 rows a block, which also evens out the blocks'
    // unequal token ranges (B 2, L 2048, 24 heads, N 128, S 256: 166 us; one
    // memory of 128 rows a block 232 us).
    constexpr int JJ = MemSplit<N>::JWMAX * MemSplit<N>::WJ;
    const int64_t full = BH * ((s.Mcap + JJ - 1) / JJ);
    auto mem_side = [&](auto nr, auto jw, int64_t blocks) {
        k_fbwd_mem<T, N, decltype(nr)::value, decltype(jw)::value><<<flat_grid(blocks, kFT), kFT, 0, st>>>(
            w.qb, w.eb, (const T*)Cm, (const T*)dy, (const T*)mem, w.gp, w.dl, dmem, a.eps, a.normalize,
            s.L, w.Ls, s.H, s.G, s.S, s.Mcap, Mp, BH);
    };
    prof_begin("k_bwd_mem", st);
    if (full >= 2 * device_cu_count()) {
        mem_side(std::integral_constant<int, N>(), std::integral_constant<int, MemSplit<N>::JWMAX>(), full);
    } else {
        constexpr int NR = N < 64 ? N : 64, WJ = MemSplit<NR>::WJ;
        mem_side(std::integral_constant<int, NR>(), std::integral_constant<int, 1>(),
                 BH * (N / NR) * ((s.Mcap + WJ - 1) / WJ));
    }
    prof_end(st);
    return hipGetLastError();
}

}  // namespace

#define DART_BY_N(FN, T, ...)               \
    switch (s.N) {                          \
        case 16: return FN<T, 16>(__VA_ARGS__);  \
        case 32: return FN<T, 32>(__VA_ARGS__);  \
        case 64: return FN<T, 64>(__VA_ARGS__);  \
        case 128: return FN<T, 128>(__VA_ARGS__); \
    }                                       \
    return hipErrorInvalidValue

hipError_t launch_fsma(const Shape& s, const SmaArgs& a, const void* q, const void* e,
                       const void* Cm, const void* mem, const void* z, const void* y_ssd, void* y,
                       float* lse, hipStream_t st) {
    if (s.dtype == 1) {
        DART_BY_N(run_fsma, bf16, s, a, q, e, Cm, mem, z, y_ssd, y, lse, st);
    }
    DART_BY_N(run_fsma, float, s, a, q, e, Cm, mem, z, y_ssd, y, lse, st);
}

hipError_t launch_fsma_bwd(const Shape& s, const SmaArgs& a, const void* q, const void* e,
                           const void* Cm, const void* mem, const void* z, const void* dy,
                           const GenBwdWs& w, float* dmem, hipStream_t st) {
    if (s.dtype == 1) {
        DART_BY_N(run_fsma_bwd, bf16, s, a, q, e, Cm, mem, z, dy, w, dmem, st);
    }
    DART_BY_N(run_fsma_bwd, float, s, a, q, e, Cm, mem, z, dy, w, dmem, st);
}

}  // namespace dart
