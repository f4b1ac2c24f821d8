// scan_bwd.hip -- backward of the chunked SSD scan and of its chunk memories on
// the fp32 matrix instructions: fp32 storage at every shape, and either storage
// at the shapes outside the bf16 kernels' set (scan_bwd_mfma.hip).
//
// Paper: Sec. 2 (the recurrence H_t = a_t H_{t-1} + dt_t B_t^T x_t,
// y_t = C_t H_t, a_t = exp(dt_t A_h)) and Sec. 3 / App. A (the chunk memory
// dH_[c], the chunk's own contribution).  Gradients of
//   loss = sum_t dy_t . y_t + sum_c <dmem_c, dH_[c]> + <dh_last, H_{L-1}>
// with respect to x, dt, A, B, C and h0.
//
// The sequence is cut into pieces of at most 64 tokens that nest with the
// memory chunks: a chunk of S >= 64 tokens is ceil(S / 64) pieces, and for
// S < 64 a piece is floor(64 / S) whole chunks.  With cs the inclusive
// cumulative log decay inside a piece (e its last token), H the state entering
// it and R the adjoint of the state leaving it, M1[s,t] = e^{cs_s - cs_t} C_s.B_t
// and M2[s,t] = e^{cs_s - cs_t} dy_s.x_t for t <= s:
//   dx_t = dt_t [sum_s M1[s,t] dy_s + e^{cs_e - cs_t} B_t W + B_t D_t],
//   dB_t = dt_t [sum_s M2[s,t] C_s + e^{cs_e - cs_t} W x_t + D_t x_t],
//   dC_s = sum_t M2[s,t] dt_t B_t + e^{cs_s} H dy_s,
// where a chunk's dmem reaches its own tokens only: for S >= 64 decayed from
// the chunk's end to the piece's end and added to R (W = R + D, D_t = 0), for
// S < 64 inside the piece (W = R, D_t = e^{cs_ce - cs_t} dmem_c(t), ce the
// chunk's last token).  The decay gradient dL/dl_t (l_t = dt_t A_h) is the sum
// over the (input s', output s) pairs with s' < t <= s, from piece-local parts
// only, so no sum runs (and cancels) over the whole sequence:
//   inside the piece: sum_{s >= t} (r_s - c_s), r and c the row and column sums
//     of P[s,t] = M1[s,t] (dy_s . x_t) dt_t;
//   input inside, leaving: sum_{s' < t} dt_s' x_s' . (e^{cs_e - cs_s'} B_s' W),
//     and the same with D_s' over the tokens s' of t's own chunk;
//   entering, output inside: sum_{s >= t} e^{cs_s} C_s . (H dy_s);
//   entering and leaving: e^{cs_e} (<R, H> + <D, H_own>), H_own the part of H
//     from the piece's own chunk.
// ddt_t = x_t . (dx_t / dt_t) + A_h dL/dl_t, dA_h = sum_{b,t} dt_t dL/dl_t.
//
// Kernels, in launch order:
//   k_fs_contract  per (b, piece, h): dH = sum_s (B_s dt_s e^{cs_e - cs_s})^T x_s,
//                  dR = sum_s (C_s e^{cs_s})^T dy_s and the piece's log decay;
//   k_fs_pass      per (b, h, 1024 elements): forward over the pieces, dH becomes
//                  the entering state H; then backward, dR becomes W (and dh0),
//                  with the sums of the entering-and-leaving terms;
//   k_fs_tokens    per (b, piece, block of heads of one group): everything else.
//                  C_s . B_t depends on the group only: its tiles are formed once
//                  per block, and the heads' dt_t M2 are summed before the two
//                  contractions over C and B, also once per block;
//   k_fs_finish    dB, dC summed over a group's head blocks, dA over pieces.
//
// All products are v_mfma_f32_16x16x4_f32, whose rate (32 cycles each) bounds
// k_fs_tokens; operand layouts as in sma_f32.hip: lane (m, g) = (lane % 16,
// lane / 16), tiles of 64-float rows in LDS in 16-byte chunks.  An accumulator
// tile (rows s = 4 g + r, column t = m) is the next product's operand as it
// stands: at step r its k index g means s = 4 g + r.
#include <type_traits>

#include "f32_tiles.hpp"

namespace dart {
namespace {

constexpr int kP = 64;
constexpr int kBT = 256;  // threads: 4 waves

// ---- per (b, piece, h): the piece's contributions ---------------------------------
// The four waves split the N rows (WN of them, NTW row tiles each) and, for
// N < 64, the column tiles.  Rows arrive 16 tokens at a time.  HBM-bound: 2 N P
// floats are written per 64 tokens of a head.
template <typename T, int N>
__global__ __launch_bounds__(kBT, 2) void k_fs_contract(
    const T* __restrict__ x, const float* __restrict__ dt, const float* __restrict__ A,
    const T* __restrict__ Bm, const T* __restrict__ Cm, const T* __restrict__ dy,
    float* __restrict__ dH, float* __restrict__ dR, float* __restrict__ lda, Pieces pc, int H, int G,
    int64_t blocks) {
    constexpr int WN = N / 16 < 4 ? N / 16 : 4, NTW = N / 16 / WN, PT = WN;  // column tiles per wave
    constexpr int TT = 16, RN = N + 16, RP = kP + 16;
    constexpr int CN = (TT * N / 4 + kBT - 1) / kBT;
    __shared__ __attribute__((aligned(16))) float s_b[2][TT][RN], s_c[2][TT][RN], s_x[2][TT][RP], s_y[2][TT][RP];
    __shared__ float s_f[2][kQ];
    const int64_t blk = flat_block();
    if (blk >= blocks) return;
    const int tid = threadIdx.x, lane = tid & 63, m = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % WN, p0 = wave / WN * PT;
    const int h = (int)(blk % H);
    const int64_t bk = blk / H, b = bk / pc.nk, k = bk - b * pc.nk;
    const int grp = (int)((int64_t)h * G / H);
    int64_t t0, t1;
    piece_range(pc, k, t0, t1);
    if (wave == 0) {
        PieceDecay pd;
        pd.load(dt, A[h], b, pc.L, H, h, t0, t1, lane);
        const bool in = t0 + lane < t1;
        s_f[0][lane] = in ? fast_exp2(log_to_end(pd.T, lane >> 4, pd.te)) * pd.d : 0.f;
        s_f[1][lane] = in ? fast_exp2(log_from_start(pd.T, lane >> 4, pd.cl)) : 0.f;
        if (lane == 0) lda[(b * H + h) * pc.nk + k] = tiles_between(pd.T, -1, 4);
    }
    float rb[CN][4], rc[CN][4], rx[4], ry[4];
    auto load = [&](int64_t tt) {
#pragma unroll
        for (int q = 0; q < CN; ++q) {
            const int i = tid + q * kBT;
            if (i < TT * N / 4) {
                const int64_t t = tt + i / (N / 4) < t1 ? tt + i / (N / 4) : t1 - 1;
                const int64_t o = ((b * pc.L + t) * G + grp) * N + 4 * (i % (N / 4));
                load4(Bm + o, rb[q]);
                load4(Cm + o, rc[q]);
            }
        }
        const int64_t t = tt + (tid >> 4) < t1 ? tt + (tid >> 4) : t1 - 1;
        const int64_t o = ((b * pc.L + t) * H + h) * kP + 4 * (tid & 15);
        load4(x + o, rx);
        load4(dy + o, ry);
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int q = 0; q < CN; ++q) {
            const int i = tid + q * kBT;
            if (i < TT * N / 4) {
                store4(&s_b[buf][i / (N / 4)][4 * (i % (N / 4))], rb[q]);
                store4(&s_c[buf][i / (N / 4)][4 * (i % (N / 4))], rc[q]);
            }
        }
        store4(&s_x[buf][tid >> 4][4 * (tid & 15)], rx);
        store4(&s_y[buf][tid >> 4][4 * (tid & 15)], ry);
    };
    f32x4 mh[NTW][PT], mr[NTW][PT];
#pragma unroll
    for (int n = 0; n < NTW; ++n)
#pragma unroll
        for (int p = 0; p < PT; ++p) mh[n][p] = mr[n][p] = f32x4{0.f, 0.f, 0.f, 0.f};
    load(t0);
    store(0);
    int buf = 0;
    for (int64_t tt = t0; tt < t1; tt += TT, buf ^= 1) {
        __syncthreads();
        const bool more = tt + TT < t1;
        if (more) load(tt + TT);
#pragma unroll
        for (int ks = 0; ks < TT / 4; ++ks) {
            const int t = 4 * ks + g;
            const float fx = s_f[0][(int)(tt - t0) + t], fy = s_f[1][(int)(tt - t0) + t];
            float ab[NTW], ac[NTW];
#pragma unroll
            for (int n = 0; n < NTW; ++n) {
                ab[n] = s_b[buf][t][wn * 16 * NTW + NTW * m + n] * fx;
                ac[n] = s_c[buf][t][wn * 16 * NTW + NTW * m + n] * fy;
            }
            const f32x4 vx = *reinterpret_cast<const f32x4*>(&s_x[buf][t][4 * m]);
            const f32x4 vy = *reinterpret_cast<const f32x4*>(&s_y[buf][t][4 * m]);
#pragma unroll
            for (int n = 0; n < NTW; ++n)
#pragma unroll
                for (int p = 0; p < PT; ++p) {
                    // the wave's column tiles (all four for N >= 64)
                    const float px = PT == 4 ? vx[p] : vx[p0 + p], py = PT == 4 ? vy[p] : vy[p0 + p];
                    mh[n][p] = mfma4(ab[n], px, mh[n][p]);
                    mr[n][p] = mfma4(ac[n], py, mr[n][p]);
                }
        }
        if (more) store(buf ^ 1);
    }
    const int64_t base = blk * (int64_t)(N * kP);
#pragma unroll
    for (int n = 0; n < NTW; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t o = base + (wn * 16 * NTW + NTW * (4 * g + r) + n) * kP + 4 * m + p0;
            if constexpr (PT == 4) {
                const float vh[4] = {mh[n][0][r], mh[n][1][r], mh[n][2][r], mh[n][3][r]};
                const float vr[4] = {mr[n][0][r], mr[n][1][r], mr[n][2][r], mr[n][3][r]};
                store4(dH + o, vh);
                store4(dR + o, vr);
            } else {
#pragma unroll
                for (int p = 0; p < PT; ++p) {
                    dH[o + p] = mh[n][p][r];
                    dR[o + p] = mr[n][p][r];
                }
            }
        }
}

// ---- per (b, h, 1024 elements): the passes over the pieces --------------------------
// In place: dH -> H (the state entering each piece), dR -> W.  kpart [b][h][k]
// [nkp]: each wave's parts of e^{cs_e} <R, H> and, OWN, of e^{cs_e} <D, H_own>.  suf [b][h][k]:
// the decay from a piece's end to its chunk's end (every block of a (b, h)
// writes the same values and reads its own).
template <bool OWN>
__global__ __launch_bounds__(256) void k_fs_pass(float* dH, float* dR,
                                                 const float* __restrict__ lda, const float* __restrict__ h0,
                                                 const float* __restrict__ dhl, const float* __restrict__ dmem,
                                                 float* __restrict__ dh0, float* __restrict__ kpart,
                                                 float* suf, Pieces pc, int H, int NP, int64_t Mcap) {
    const int h = blockIdx.y;
    const int64_t b = blockIdx.z, bh = b * H + h;
    const int tid = threadIdx.x, lane = tid & 63;
    const int e0 = (blockIdx.x * 256 + tid) * 4;  // NP is a multiple of 1024
    const int nw = gridDim.x * 4, wv = blockIdx.x * 4 + (tid >> 6), nkp = OWN ? 2 * nw : nw;
    const float* ld = lda + bh * pc.nk;
    float* kp = kpart + bh * pc.nk * nkp + wv;
    const int64_t step = (int64_t)H * NP;
    float* ph = dH + (b * pc.nk * H + h) * (int64_t)NP + e0;
    float* pr = dR + (b * pc.nk * H + h) * (int64_t)NP + e0;
    const float* pm = dmem ? dmem + (b * Mcap * H + h) * (int64_t)NP + e0 : nullptr;
    if (OWN) {
        // one thread per chunk
        for (int64_t k = (int64_t)tid * pc.nq; k < pc.nk; k += 256 * pc.nq) {
            const int64_t last = (k + pc.nq < pc.nk ? k + pc.nq : pc.nk) - 1;
            float a = 1.f;
            for (int64_t q = last; q >= k; --q) {
                suf[bh * pc.nk + q] = a;
                a *= fast_exp2(ld[q]);
            }
        }
        __syncthreads();
    }
    // U pieces' values are loaded while the U before them are used, ahead of
    // those pieces' stores: the chains over the pieces are short, the loads'
    // latency is what bounds them (memory operations complete in order)
    constexpr int U = 4;
    float hc[4] = {0.f, 0.f, 0.f, 0.f}, ho[4] = {0.f, 0.f, 0.f, 0.f}, dm[4] = {0.f, 0.f, 0.f, 0.f};
    if (h0) load4(h0 + bh * (int64_t)NP + e0, hc);
    int i = 0;  // piece of its chunk
    struct Fwd {
        float d[U][4], a[U], sf[U];
    };
    auto fload = [&](int64_t k0, Fwd& f) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = k0 + u < pc.nk ? k0 + u : pc.nk - 1;
            load4(ph + k * step, f.d[u]);
            f.a[u] = fast_exp2(ld[k]);
            f.sf[u] = OWN ? suf[bh * pc.nk + k] : 0.f;
        }
    };
    auto fstep = [&](int64_t k0, const Fwd& f) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = k0 + u;
            if (k >= pc.nk) continue;
            store4(ph + k * step, hc);
            if (OWN) {
                if (i == 0) {
                    if (pm) load4(pm + k / pc.nq * step, dm);
                    ho[0] = ho[1] = ho[2] = ho[3] = 0.f;
                }
                float s = (ho[0] * dm[0] + ho[1] * dm[1]) + (ho[2] * dm[2] + ho[3] * dm[3]);
                s = row4_sum(dpp_group_sum<16>(s));
                if (lane == 0) kp[k * nkp + nw] = f.a[u] * f.sf[u] * s;
#pragma unroll
                for (int q = 0; q < 4; ++q) ho[q] = f.a[u] * ho[q] + f.d[u][q];
                if (++i == pc.nq) i = 0;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) hc[q] = f.a[u] * hc[q] + f.d[u][q];
        }
    };
    {
        Fwd f0, f1;
        fload(0, f0);
        for (int64_t k0 = 0; k0 < pc.nk; k0 += 2 * U) {
            fload(k0 + U, f1);
            fstep(k0, f0);
            fload(k0 + 2 * U, f0);
            fstep(k0 + U, f1);
        }
    }
    float r[4] = {0.f, 0.f, 0.f, 0.f}, dd[4] = {0.f, 0.f, 0.f, 0.f};
    if (dhl) load4(dhl + bh * (int64_t)NP + e0, r);
    const bool nest = pc.S >= kQ;  // a chunk's dmem leaves with its pieces
    struct Bwd {
        float d[U][4], h[U][4], a[U];
    };
    auto bload = [&](int64_t k0, Bwd& f) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = k0 - u > 0 ? k0 - u : 0;
            load4(pr + k * step, f.d[u]);
            load4(ph + k * step, f.h[u]);
            f.a[u] = fast_exp2(ld[k]);
        }
    };
    auto bstep = [&](int64_t k0, const Bwd& f) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = k0 - u;
            if (k < 0) continue;
            if (nest && pm) {
                const int64_t c = k / pc.nq;
                if (k == pc.nk - 1 || (k + 1) / pc.nq != c) load4(pm + c * step, dd);
            }
            float s = 0.f, w4[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                w4[q] = r[q] + dd[q];
                s += r[q] * f.h[u][q];
                r[q] = f.a[u] * r[q] + f.d[u][q];
                dd[q] *= f.a[u];
            }
            store4(pr + k * step, w4);
            s = row4_sum(dpp_group_sum<16>(s)) * f.a[u];
            if (lane == 0) kp[k * nkp] = s;
        }
    };
    {
        Bwd f0, f1;
        bload(pc.nk - 1, f0);
        for (int64_t k0 = pc.nk - 1; k0 >= 0; k0 -= 2 * U) {
            bload(k0 - U, f1);
            bstep(k0, f0);
            bload(k0 - 2 * U, f0);
            bstep(k0 - U, f1);
        }
    }
    if (dh0) store4(dh0 + bh * (int64_t)NP + e0, r);
}

// ---- per (b, piece, block of heads): the token gradients ----------------------------
// A wave owns 16 tokens, as columns t of the tiles with s >= t and as rows of
// dB, dC and dx.
// 256 registers and at most 68 KB of LDS: two blocks per CU.  W and H stand in
// LDS together up to N = 64, so that one wait covers both (the whole backward at
// B 64, L 512, H 4, N 64, S 16 is 3 % faster so, 281 us, than with H staged over W);
// at N = 128 the second tile would leave one block per CU.  SMALL: S < 64.  The
// registers don't hold it all: 33 to 67 spill at N 64, 112 to 157 at N 128.
template <typename T, int N, bool SMALL>
__global__ __launch_bounds__(kBT, 2) void k_fs_tokens(
    const T* __restrict__ x, const float* __restrict__ dt, const float* __restrict__ A,
    const T* __restrict__ Bm, const T* __restrict__ Cm, const T* __restrict__ dy,
    const float* __restrict__ Hs, const float* __restrict__ Ws, const float* __restrict__ dmem,
    const float* __restrict__ kpart, float* __restrict__ dx, float* __restrict__ ddt,
    float* __restrict__ dBp, float* __restrict__ dCp, float* __restrict__ dAp, Pieces pc, int H, int G,
    int64_t Mcap, int hpb, int nkp, int64_t blocks) {
    constexpr int K = N / 16, NV = K < 4 ? K : 4, NQ = K / NV;
    constexpr int MP = kQ + 4;  // row pitch of the summed M2, in floats
    constexpr bool BOTH = N <= 64;  // W and H at once
    __shared__ __attribute__((aligned(16))) char s_xy[2 * kQ * 256], s_w[(BOTH ? 2 : 1) * N * 256];
    char* const s_h = s_w + (BOTH ? N * 256 : 0);
    __shared__ __attribute__((aligned(16))) float s_cl[kQ], s_lo[kQ], s_te[kQ], s_dt[kQ];
    __shared__ f32x4 s_T;
    __shared__ float s_r[4][kQ], s_c[kQ], s_v[kQ], s_d[kQ], s_u[kQ], s_bx[kQ];
    static_assert(kQ * MP * 4 <= 2 * kQ * 256, "the summed M2 takes the place of x and dy");
    const int64_t blk = flat_block();
    if (blk >= blocks) return;
    char* s_x = s_xy;
    char* s_y = s_xy + kQ * 256;
    const int tid = threadIdx.x, lane = tid & 63, m = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nhb = H / hpb;
    const int64_t bk = blk / nhb, b = bk / pc.nk, k = bk - b * pc.nk;
    const int hb = (int)(blk - bk * nhb), h0 = hb * hpb;
    const int grp = (int)((int64_t)h0 * G / H);
    int64_t t0, t1;
    piece_range(pc, k, t0, t1);
    const int nt = (int)(t1 - t0);
    const int tl = 16 * w + m;  // this lane's token
    const bool valid = tl < nt;
    const bool used = 16 * w < nt;  // any token in the wave
    // a row of the piece, clamped to its last token (whose x, dy and dt are
    // taken as zero, so that it adds nothing)
    auto row = [&](int s) { return b * pc.L + t0 + (s < nt ? s : nt - 1); };
    const int64_t bt = row(tl);
    float bv[K][4];
#pragma unroll
    for (int q = 0; q < K; ++q) load4(Bm + (bt * G + grp) * N + 16 * q + 4 * g, bv[q]);
    // C_s . B_t of the tiles s >= t
    f32x4 g1[4], mb[4], aB[K], aC[K];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        g1[j] = mb[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (j >= w && 16 * j < nt) {
            const T* cr = Cm + (row(16 * j + m) * G + grp) * N + 4 * g;
#pragma unroll
            for (int q = 0; q < K; ++q) {
                float c4[4];
                load4(cr + 16 * q, c4);
                f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < 4; ++s) a = mfma4(c4[s], bv[q][s], a);
                g1[j] += a;
            }
        }
    }
#pragma unroll
    for (int q = 0; q < K; ++q) aB[q] = aC[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    // NV consecutive elements
    auto vec = [&](const T* p, float (&v)[NV]) {
        if constexpr (NV == 4) {
            load4(p, v);
        } else {
#pragma unroll
            for (int i = 0; i < NV; ++i) v[i] = to_f(p[i]);
        }
    };
    PieceOff<N> off;
    off.init(m, g);
    char* const xr = s_x + w * 4096;  // the wave's rows of x and dy
    char* const yr = s_y + w * 4096;
    for (int hh = 0; hh < hpb; ++hh) {
        const int h = h0 + hh;
        const float Ah = A[h];
        const int64_t st = ((b * pc.nk + k) * H + h) * (int64_t)(N * kP);
        __syncthreads();  // the last head's reads are done
        PieceOff<N>::stage(Ws + st, s_w, tid);
        if constexpr (BOTH) PieceOff<N>::stage(Hs + st, s_h, tid);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int s = (tid >> 4) + 16 * q, c = tid & 15;
            float x4[4] = {0.f, 0.f, 0.f, 0.f}, y4[4] = {0.f, 0.f, 0.f, 0.f};
            if (s < nt) {
                load4(x + (row(s) * H + h) * kP + 4 * c, x4);
                load4(dy + (row(s) * H + h) * kP + 4 * c, y4);
            }
            const int o = s * 256 + ((c ^ (s & 15)) << 4);
            *reinterpret_cast<f32x4*>(s_x + o) = f32x4{x4[0], x4[1], x4[2], x4[3]};
            *reinterpret_cast<f32x4*>(s_y + o) = f32x4{y4[0], y4[1], y4[2], y4[3]};
        }
        if (w == 0) {
            PieceDecay pd;
            pd.load(dt, Ah, b, pc.L, H, h, t0, t1, lane);
            s_cl[lane] = pd.cl;
            s_lo[lane] = pd.lo;
            s_te[lane] = pd.te;
            s_dt[lane] = pd.d;
            if (lane == 0) s_T = pd.T;
        }
        __syncthreads();
        const f32x4 tt = s_T;
        const float ct = s_cl[tl], tlo = s_lo[tl], te = s_te[tl], dtt = s_dt[tl];
        if (used) {
            f32x4 xt[4], di[4], bw[4], bd[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                xt[q] = lds4(xr + off.oc[q]);
                di[q] = bw[q] = bd[q] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (j >= w && 16 * j < nt) {
                    f32x4 g2 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int q = 0; q < 4; q += 2)
                        g2 += mfma16(lds4(s_y + j * 4096 + off.oc[q]), xt[q]) +
                              mfma16(lds4(s_y + j * 4096 + off.oc[q + 1]), xt[q + 1]);
                    const f32x4 cs = *reinterpret_cast<const f32x4*>(s_cl + 16 * j + 4 * g);
                    const f32x4 slo = *reinterpret_cast<const f32x4*>(s_lo + 16 * j + 4 * g);
                    f32x4 m1, ps;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float l = j == w ? log_decay_in(cs[r], slo[r], ct, tlo) : log_decay_over(tt, j, cs[r], w, te);
                        const float e = fast_exp2(fminf(l, 0.f));
                        const bool on = j != w || 4 * g + r >= m;  // (selected: 0 times an infinity is not 0)
                        m1[r] = on ? e * g1[j][r] : 0.f;
                        mb[j][r] += on ? dtt * (e * g2[r]) : 0.f;
                        ps[r] = dpp_group_sum<16>(on ? m1[r] * (g2[r] * dtt) : 0.f);
                    }
                    if (m == 0) *reinterpret_cast<f32x4*>(&s_r[w][16 * j + 4 * g]) = ps;
                    if (j == w && any_nonfinite(g2)) {
                        // dy_s of the tokens s >= t alone
#pragma unroll 1
                        for (int q = 0; q < 4; ++q)
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                const int s = 4 * q + r;
                                const float f = __shfl(m1[r], 16 * q + m, 64);
#pragma unroll
                                for (int r2 = 0; r2 < 4; ++r2) {
                                    const f32x4 yv = lds4(yr + s * 256 + (((4 * g + r2) ^ s) << 4));
#pragma unroll
                                    for (int i = 0; i < 4; ++i)
                                        if (s >= m) di[i][r2] += f * yv[i];
                                }
                            }
                    } else {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const f32x4 a = lds4(s_y + j * 4096 + off.op[r]);
#pragma unroll
                            for (int i = 0; i < 4; ++i) di[i] = mfma4(a[i], m1[r], di[i]);
                        }
                    }
                }
            }
            // B_t W
#pragma unroll
            for (int q = 0; q < K; ++q)
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const f32x4 a = off.state_p(s_w, q, s);
#pragma unroll
                    for (int i = 0; i < 4; ++i) bw[i] = mfma4(a[i], bv[q][s], bw[i]);
                }
            const float fw = fast_exp2(log_to_end(tt, w, te));
            // the chunks of the wave's tokens, each dmem_c for its own tokens only
            const int64_t c0 = (t0 + 16 * w) / pc.S;
            const int nc = SMALL && dmem ? (int)((t0 + (16 * w + 15 < nt ? 16 * w + 15 : nt - 1)) / pc.S - c0) + 1 : 0;
            // whether a token is the chunk's, and then f = e^{cs_ce - cs_t}
            auto own = [&](int c, float& f) {
                const int lo = (int)((c0 + c) * pc.S - t0), hi = lo + pc.S < nt ? lo + pc.S : nt;
                const bool in = tl >= lo && tl < hi;
                const float ce = s_cl[hi - 1];
                f = in ? fast_exp2((hi - 1) >> 4 == w ? log_decay_in(ce, s_lo[hi - 1], ct, tlo)
                                                      : log_decay_over(tt, (hi - 1) >> 4, ce, w, te)) : 0.f;
                return in;
            };
            auto dmem_of = [&](int c) { return dmem + ((b * Mcap + c0 + c) * H + h) * (int64_t)(N * kP); };
            if constexpr (SMALL) {
                for (int c = 0; c < nc; ++c) {
                    float fd;
                    const bool in = own(c, fd);
                    const float* dm = dmem_of(c) + 4 * g * kP + 4 * m;
                    f32x4 b1[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) b1[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int q = 0; q < K; ++q)
#pragma unroll
                        for (int s = 0; s < 4; ++s) {
                            const f32x4 a = *reinterpret_cast<const f32x4*>(dm + (16 * q + s) * kP);
                            const float bq = bv[q][s] * fd;
#pragma unroll
                            for (int i = 0; i < 4; ++i) b1[i] = mfma4(a[i], bq, b1[i]);
                        }
#pragma unroll
                    for (int i = 0; i < 4; ++i) bd[i] = in ? b1[i] : bd[i];
                }
            }
            // dx, and x_t . of its three parts
            float si = 0.f, sw = 0.f, sd = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const f32x4 xv = lds4(xr + m * 256 + (((4 * g + r) ^ m) << 4));
                float o[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float wv = fw * bw[i][r];
                    si += xv[i] * di[i][r];
                    sw += xv[i] * wv;
                    if constexpr (SMALL) sd += xv[i] * bd[i][r];
                    o[i] = dtt * (SMALL ? di[i][r] + wv + bd[i][r] : di[i][r] + wv);
                }
                if (valid) store4(dx + (bt * H + h) * kP + 16 * g + 4 * r, o);
            }
            si = row4_sum(si);
            sw = row4_sum(sw);
            if constexpr (SMALL) sd = row4_sum(sd);
            if (g == 0) {
                s_c[tl] = dtt * si;
                s_v[tl] = dtt * sw;
                s_d[tl] = dtt * sd;
                s_bx[tl] = si + sw + sd;
            }
            // dB += dt (e^{cs_e - cs_t} W + D_t) x_t
            f32x4 xs[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) xs[q] = xt[q] * (dtt * fw);
#pragma unroll
            for (int tile = 0; tile < K; ++tile)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 a = off.state_n(s_w, tile, q);
#pragma unroll
                    for (int s = 0; s < 4; ++s) aB[tile] = mfma4(a[s], xs[q][s], aB[tile]);
                }
            if constexpr (SMALL) {
                for (int c = 0; c < nc; ++c) {
                    float fx;
                    const bool in = own(c, fx);
                    const float* dm = dmem_of(c) + NV * m * kP + 4 * g;
#pragma unroll
                    for (int q = 0; q < 4; ++q) xs[q] = xt[q] * (dtt * fx);
#pragma unroll
                    for (int tile = 0; tile < K; ++tile) {
                        f32x4 b1 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const f32x4 a = *reinterpret_cast<const f32x4*>(
                                dm + (16 * NV * (tile / NV) + tile % NV) * kP + 16 * q);
#pragma unroll
                            for (int s = 0; s < 4; ++s) b1 = mfma4(a[s], xs[q][s], b1);
                        }
                        if (in) aB[tile] += b1;
                    }
                }
            }
        }
        if constexpr (!BOTH) {
            __syncthreads();  // W is read
            PieceOff<N>::stage(Hs + st, s_h, tid);
            __syncthreads();
        }
        if (used) {
            // dC += e^{cs_s} H dy_s, and its dot with C_s
            f32x4 ys[4];
            const float ec = valid ? fast_exp2(log_from_start(tt, w, ct)) : 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) ys[q] = lds4(yr + off.oc[q]) * ec;
            float u = 0.f;
#pragma unroll
            for (int qn = 0; qn < NQ; ++qn) {
                f32x4 acc[NV];
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int q = 0; q < 4; q += 2)
                        acc[i] += mfma16(off.state_n(s_h, qn * NV + i, q), ys[q]) +
                                  mfma16(off.state_n(s_h, qn * NV + i, q + 1), ys[q + 1]);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float c4[NV];
                    vec(Cm + (bt * G + grp) * N + 16 * NV * qn + NV * (4 * g + r), c4);
#pragma unroll
                    for (int i = 0; i < NV; ++i) u += acc[i][r] * c4[i];
                }
#pragma unroll
                for (int i = 0; i < NV; ++i) aC[qn * NV + i] += acc[i];
            }
            u = row4_sum(u);
            if (g == 0) s_u[tl] = u;
        }
        __syncthreads();
        if (w == 0) {
            // the decay gradient: lane = token
            const bool ok = lane < nt;
            float F = 0.f, v = 0.f, vd = 0.f;
            if (ok) {
                for (int ww = 0; ww <= lane >> 4; ++ww) F += s_r[ww][lane];
                F += s_u[lane] - s_c[lane];
                v = s_v[lane];
                vd = s_d[lane];
            }
            // first token of this token's chunk inside the piece
            const int seg = pc.S < kQ ? lane - (int)((t0 + lane) % pc.S) : 0;
            float sv = v, svd = vd;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const float dn = __shfl_down(F, o, 64), up = __shfl_up(sv, o, 64), ud = __shfl_up(svd, o, 64);
                if (lane + o < 64) F += dn;
                if (lane >= o) sv += up;
                if (lane - o >= seg) svd += ud;
            }
            const float pv = __shfl_up(sv, 1, 64), pd = __shfl_up(svd, 1, 64);
            float Kt = 0.f;
            const float* kp = kpart + ((b * H + h) * pc.nk + k) * nkp;
            for (int q = lane; q < nkp; q += 64) Kt += kp[q];
            Kt = row4_sum(dpp_group_sum<16>(Kt));
            const float dl = F + Kt + (lane > 0 ? pv : 0.f) + (lane > seg ? pd : 0.f);
            float da = 0.f;
            if (ok) {
                ddt[(b * pc.L + t0 + lane) * H + h] = s_bx[lane] + Ah * dl;
                da = s_dt[lane] * dl;
            }
            da = row4_sum(dpp_group_sum<16>(da));
            if (lane == 0) dAp[(b * pc.nk + k) * H + h] = da;
        }
    }
    // the heads' sum of dt_t M2: rows t in LDS for the products over t
    __syncthreads();
    float* s_m = reinterpret_cast<float*>(s_xy);
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (j >= w) *reinterpret_cast<f32x4*>(s_m + tl * MP + 16 * j + 4 * g) = mb[j];
    __syncthreads();
    if (!used) return;
    // C and B rows of the wave's own tile with an infinity or NaN: each token
    // takes the rows s >= t (of C) and t <= s (of B) alone
    bool bad = false;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (j == w) bad = any_nonfinite(g1[j]);
    if (bad) {
#pragma unroll 1
        for (int s = 0; s < 16 && 16 * w + s < nt; ++s) {
            const float mc = s_m[tl * MP + 16 * w + s], mt = s_m[(16 * w + s) * MP + tl];
#pragma unroll
            for (int qn = 0; qn < NQ; ++qn)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float c4[NV], b4[NV];
                    const int64_t o = (row(16 * w + s) * G + grp) * N + 16 * NV * qn + NV * (4 * g + r);
                    vec(Cm + o, c4);
                    vec(Bm + o, b4);
#pragma unroll
                    for (int i = 0; i < NV; ++i) {
                        if (s >= m) aB[qn * NV + i][r] += mc * c4[i];
                        if (s <= m) aC[qn * NV + i][r] += mt * b4[i];
                    }
                }
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (bad && j == w) continue;
        if (j >= w && 16 * j < nt) {
#pragma unroll
            for (int qn = 0; qn < NQ; ++qn) {
                f32x4 t[NV];
#pragma unroll
                for (int i = 0; i < NV; ++i) t[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float a[NV];
                    vec(Cm + (row(16 * j + 4 * g + r) * G + grp) * N + 16 * NV * qn + NV * m, a);
#pragma unroll
                    for (int i = 0; i < NV; ++i) t[i] = mfma4(a[i], mb[j][r], t[i]);
                }
#pragma unroll
                for (int i = 0; i < NV; ++i) aB[qn * NV + i] += t[i];
            }
        }
        if (j <= w) {
            float mt[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) mt[r] = s_m[(16 * j + 4 * g + r) * MP + tl];
#pragma unroll
            for (int qn = 0; qn < NQ; ++qn) {
                f32x4 t[2][NV];
#pragma unroll
                for (int i = 0; i < NV; ++i) t[0][i] = t[1][i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float a[NV];
                    vec(Bm + (row(16 * j + 4 * g + r) * G + grp) * N + 16 * NV * qn + NV * m, a);
#pragma unroll
                    for (int i = 0; i < NV; ++i) t[r >> 1][i] = mfma4(a[i], mt[r], t[r >> 1][i]);
                }
#pragma unroll
                for (int i = 0; i < NV; ++i) aC[qn * NV + i] += t[0][i] + t[1][i];
            }
        }
    }
    if (!valid) return;
    float* outB = dBp + (bt * nhb + hb) * (int64_t)N;
    float* outC = dCp + (bt * nhb + hb) * (int64_t)N;
#pragma unroll
    for (int qn = 0; qn < NQ; ++qn)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int n = 16 * NV * qn + NV * (4 * g + r);
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                outB[n + i] = aB[qn * NV + i][r];
                outC[n + i] = aC[qn * NV + i][r];
            }
        }
}

// ---- group sums of dB, dC; dA over batch and pieces ----------------------------------
// The first H blocks sum dA of one head each, the others dB and dC.
template <int N>
__global__ __launch_bounds__(256) void k_fs_finish(const float* __restrict__ dBp,
                                                   const float* __restrict__ dCp,
                                                   const float* __restrict__ dAp,
                                                   float* __restrict__ dB, float* __restrict__ dC,
                                                   float* __restrict__ dA, int64_t rows, int H,
                                                   int G, int hpb, int64_t arows) {
    if ((int)blockIdx.x < H) {
        __shared__ float red[4];
        float s = 0.f;
        for (int64_t r = threadIdx.x; r < arows; r += 256) s += dAp[r * H + blockIdx.x];
        s = row4_sum(dpp_group_sum<16>(s));
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
        __syncthreads();
        if (threadIdx.x == 0) dA[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
        return;
    }
    const int64_t i = ((int64_t)(blockIdx.x - H) * 256 + threadIdx.x) * 4;
    if (i >= rows * N) return;
    const int nhb = H / hpb, per = (H / G) / hpb;
    const int64_t row = i / N;  // (b, t, g)
    const int n = (int)(i - row * N);
    const int64_t bt = row / G;
    const int g = (int)(row - bt * G);
    float sb[4] = {0.f, 0.f, 0.f, 0.f}, sc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int q = 0; q < per; ++q) {
        const int64_t o = (bt * nhb + g * per + q) * (int64_t)N + n;
        float vb[4], vc[4];
        load4(dBp + o, vb);
        load4(dCp + o, vc);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            sb[j] += vb[j];
            sc[j] += vc[j];
        }
    }
    store4(dB + i, sb);
    store4(dC + i, sc);
}

struct SbwdWs {
    float* lda;
    float* dH;
    float* dR;
    float* kpart;
    float* suf;
    float* dBp;
    float* dCp;
    float* dAp;
    size_t total;
};

// Workspace: the pieces' log decays [B][H][nk]; their contributions, then
// entering states, and adjoint contributions, then leaving adjoints
// [B][nk][H][N][P]; per-wave entering-and-leaving sums [B][H][nk][nkp];
// decays to the chunk's end [B][H][nk]; per-head-block dB, dC partials
// [B][L][H / hpb][N]; dA partials [B][nk][H].  All float.
SbwdWs sbwd_layout(const Shape& s, void* base) {
    const Pieces pc = pieces_of(s);
    const size_t NP = (size_t)s.N * s.P;
    const size_t BHK = (size_t)s.B * s.H * pc.nk;
    const int nhb = s.H / piece_heads_per_block(s, pc.nk);
    SbwdWs w;
    size_t o = 0;
    char* p = reinterpret_cast<char*>(base);
    auto take = [&](size_t bytes) {
        float* r = p ? reinterpret_cast<float*>(p + o) : nullptr;
        o += align256(bytes);
        return r;
    };
    w.lda = take(4 * BHK);
    w.dH = take(4 * BHK * NP);
    w.dR = take(4 * BHK * NP);
    w.kpart = take(4 * BHK * ((NP + 1023) / 1024 * 4) * (pc.nq > 1 ? 2 : 1));
    w.suf = take(4 * BHK);
    w.dBp = take(4 * (size_t)s.B * s.L * nhb * s.N);
    w.dCp = take(4 * (size_t)s.B * s.L * nhb * s.N);
    w.dAp = take(4 * BHK);
    w.total = o;
    return w;
}

template <typename T, int N>
hipError_t run_sbwd(const Shape& s, const void* x, const float* dt, const float* A,
                    const void* Bm, const void* Cm, const float* h0, const void* dy,
                    const float* dmem, const float* dhl, float* dx, float* ddt, float* dA,
                    float* dB, float* dC, float* dh0, void* ws, hipStream_t st) {
    const SbwdWs w = sbwd_layout(s, ws);
    const Pieces pc = pieces_of(s);
    constexpr int NP = N * kP;
    const int64_t units = s.B * pc.nk * s.H;
    prof_begin("k_sbwd_contract", st);
    k_fs_contract<T, N><<<flat_grid(units, kBT), kBT, 0, st>>>((const T*)x, dt, A, (const T*)Bm, (const T*)Cm,
                                                          (const T*)dy, w.dH, w.dR, w.lda, pc, s.H, s.G, units);
    prof_end(st);
    const dim3 pg((unsigned)((NP + 1023) / 1024), (unsigned)s.H, (unsigned)s.B);
    prof_begin("k_sbwd_pass", st);
    if (pc.nq > 1) {
        k_fs_pass<true><<<pg, 256, 0, st>>>(w.dH, w.dR, w.lda, h0, dhl, dmem, dh0, w.kpart, w.suf, pc, s.H, NP, s.Mcap);
    } else {
        k_fs_pass<false><<<pg, 256, 0, st>>>(w.dH, w.dR, w.lda, h0, dhl, dmem, dh0, w.kpart, w.suf, pc, s.H, NP, s.Mcap);
    }
    prof_end(st);
    const int hpb = piece_heads_per_block(s, pc.nk);
    const int64_t blocks = s.B * pc.nk * (s.H / hpb);
    prof_begin("k_sbwd_tokens", st);
    auto tokens = [&](auto small) {
        k_fs_tokens<T, N, decltype(small)::value><<<flat_grid(blocks, kBT), kBT, 0, st>>>(
            (const T*)x, dt, A, (const T*)Bm, (const T*)Cm, (const T*)dy, w.dH, w.dR, dmem, w.kpart, dx, ddt,
            w.dBp, w.dCp, w.dAp, pc, s.H, s.G, s.Mcap, hpb, (int)pg.x * (pc.nq > 1 ? 8 : 4), blocks);
    };
    if (s.S < kQ) tokens(std::true_type()); else tokens(std::false_type());
    prof_end(st);
    const int64_t rows = s.B * s.L * s.G;
    prof_begin("k_sbwd_finish", st);
    k_fs_finish<N><<<(unsigned)(s.H + (rows * N / 4 + 255) / 256), 256, 0, st>>>(
        w.dBp, w.dCp, w.dAp, dB, dC, dA, rows, s.H, s.G, hpb, s.B * pc.nk);
    prof_end(st);
    return hipGetLastError();
}

template <typename T>
hipError_t run_sbwd_n(const Shape& s, const void* x, const float* dt, const float* A,
                      const void* Bm, const void* Cm, const float* h0, const void* dy,
                      const float* dmem, const float* dhl, float* dx, float* ddt, float* dA,
                      float* dB, float* dC, float* dh0, void* ws, hipStream_t st) {
    switch (s.N) {
        case 16: return run_sbwd<T, 16>(s, x, dt, A, Bm, Cm, h0, dy, dmem, dhl, dx, ddt, dA, dB, dC, dh0, ws, st);
        case 32: return run_sbwd<T, 32>(s, x, dt, A, Bm, Cm, h0, dy, dmem, dhl, dx, ddt, dA, dB, dC, dh0, ws, st);
        case 64: return run_sbwd<T, 64>(s, x, dt, A, Bm, Cm, h0, dy, dmem, dhl, dx, ddt, dA, dB, dC, dh0, ws, st);
        case 128: return run_sbwd<T, 128>(s, x, dt, A, Bm, Cm, h0, dy, dmem, dhl, dx, ddt, dA, dB, dC, dh0, ws, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace

size_t ssd_bwd_workspace_bytes(const Shape& s) {
    return bf16_shape(s) ? sbwd_mfma_workspace_bytes(s) : sbwd_layout(s, nullptr).total;
}

hipError_t launch_ssd_bwd(const Shape& s, const void* x, const float* dt, const float* A,
                          const void* Bm, const void* Cm, const float* h0, const void* dy,
                          const float* dmem, const float* dh_last, float* dx, float* ddt, float* dA,
                          float* dB, float* dC, float* dh0, void* ws, hipStream_t st) {
    if (bf16_shape(s))
        return launch_ssd_bwd_mfma(s, x, dt, A, Bm, Cm, h0, dy, dmem, dh_last, dx, ddt, dA, dB, dC, dh0, ws, st);
    if (s.dtype == 1)
        return run_sbwd_n<bf16>(s, x, dt, A, Bm, Cm, h0, dy, dmem, dh_last, dx, ddt, dA, dB, dC, dh0, ws, st);
    return run_sbwd_n<float>(s, x, dt, A, Bm, Cm, h0, dy, dmem, dh_last, dx, ddt, dA, dB, dC, dh0, ws, st);
}

}  // namespace dart
