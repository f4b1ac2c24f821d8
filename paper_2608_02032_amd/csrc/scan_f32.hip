// scan_f32.hip -- the chunked SSD scan with its memories on the fp32 matrix
// instructions: fp32 storage at every shape, and either storage at the shapes
// outside the bf16 kernels' set (any chunk size S >= 1, N in {16, 32, 64, 128},
// P = 64).
//
// Paper: Sec. 2 (recurrence H_t = a_t H_{t-1} + dt_t B_t^T x_t, y_t = C_t H_t),
// Sec. 3 / App. A (the memory dH_[c] of every chunk).  The sequence is cut into
// pieces of at most 64 tokens that nest with the memory chunks (f32_tiles.hpp):
// a state product costs the same per token at any piece length, the products
// inside a piece grow with it, and short pieces keep the decays' exponents (and
// their rounding) small.
//   k_fs_state  per (b, piece, h): for S <= 64 each chunk's memory, and the
//               piece's contribution to the state, on MFMA;
//   k_fs_states per (b, h, 256 elements): the pass over the pieces; a
//               contribution becomes the state entering its piece, and for
//               S > 64 the contributions of a chunk's pieces its memory;
//   k_fs_out    per (b, piece, block of heads of one group): y = (decay o
//               C B^T)(dt x) + e^{cs} C H, the tiles of C B^T formed once per
//               block for all its heads.
// Operand layouts as in scan_bwd.hip.
//
// Measured, with the kernels these replaced: B 2, L 2048, 24 heads, N 128,
// S 256, fp32 (three MFMA kernels with the Gram tiles through memory, and the
// state pass) 132 -> 102 us; B 64, L 512, 4 heads, N 64, S 16, fp32 (token by
// token) 234 -> 107; B 2, L 2048, 8 heads, N 128, S 32, bf16 99 -> 47.
#include <type_traits>

#include "f32_tiles.hpp"

namespace dart {
namespace {

constexpr int kP = 64;
constexpr int kFT = 256;
constexpr int kPassT = 64;

// The waves split the N rows (WN of them, NTW row tiles each) and, for N < 64,
// the column tiles (PT each).  HBM-bound: N P floats are written per piece.
template <typename T, int N>
__global__ __launch_bounds__(kFT) void k_fs_state(const T* __restrict__ x, const float* __restrict__ dt,
                                                  const float* __restrict__ A, const T* __restrict__ Bm,
                                                  T* __restrict__ mem, float* __restrict__ dH,
                                                  float* __restrict__ lda, Pieces pc, int H, int G,
                                                  int64_t Mcap, int64_t blocks) {
    constexpr int WN = N / 16 < 4 ? N / 16 : 4, NTW = N / 16 / WN, PT = WN;
    __shared__ __attribute__((aligned(16))) float s_b[kQ][N + 16], s_x[kQ][kP + 16];
    __shared__ float s_f[kQ], s_a[kQ];
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
    const int nt = (int)(t1 - t0);
    float rb[N / 16][4], rx[4][4];
#pragma unroll
    for (int q = 0; q < N / 16; ++q) {
        const int i = tid + q * kFT, s = i / (N / 4);
        const int64_t t = t0 + (s < nt ? s : nt - 1);
        load4(Bm + ((b * pc.L + t) * G + grp) * N + 4 * (i % (N / 4)), rb[q]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int s = (tid >> 4) + 16 * q;
        const int64_t t = t0 + (s < nt ? s : nt - 1);
        load4(x + ((b * pc.L + t) * H + h) * kP + 4 * (tid & 15), rx[q]);
    }
    if (wave == 0) {
        PieceDecay pd;
        pd.load(dt, A[h], b, pc.L, H, h, t0, t1, lane);
        // to the last token of this token's chunk inside the piece
        float to = log_to_end(pd.T, lane >> 4, pd.te);
        if (pc.S < kQ) {
            int e = lane - lane % (int)pc.S + (int)pc.S - 1;  // (a piece starts with a chunk)
            e = e < nt ? e : nt - 1;
            const float ce = __shfl(pd.cl, e, 64), le = __shfl(pd.lo, e, 64);
            to = e >> 4 == lane >> 4 ? log_decay_in(ce, le, pd.cl, pd.lo)
                                     : log_decay_over(pd.T, e >> 4, ce, lane >> 4, pd.te);
            // a chunk's decay, at its first token: from the token before it to its last
            const int q = lane > 0 ? lane - 1 : 0;
            const float cq = __shfl(pd.cl, q, 64), lq = __shfl(pd.lo, q, 64), tq = __shfl(pd.te, q, 64);
            s_a[lane] = fast_exp2(e >> 4 == q >> 4 ? log_decay_in(ce, le, cq, lq)
                                                   : log_decay_over(pd.T, e >> 4, ce, q >> 4, tq));
        }
        s_f[lane] = lane < nt ? fast_exp2(to) * pd.d : 0.f;
        if (lane == 0) lda[(b * H + h) * pc.nk + k] = tiles_between(pd.T, -1, 4);
    }
#pragma unroll
    for (int q = 0; q < N / 16; ++q) {
        const int i = tid + q * kFT;
        store4(&s_b[i / (N / 4)][4 * (i % (N / 4))], rb[q]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) store4(&s_x[(tid >> 4) + 16 * q][4 * (tid & 15)], rx[q]);
    __syncthreads();
    f32x4 sum[NTW][PT];
#pragma unroll
    for (int n = 0; n < NTW; ++n)
#pragma unroll
        for (int p = 0; p < PT; ++p) sum[n][p] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int per = pc.S < kQ ? pc.S : kQ;  // tokens of one memory in the piece
    T* mo = pc.S <= kQ ? mem + ((b * Mcap + k * (pc.Q / per)) * H + h) * (int64_t)(N * kP) : nullptr;
    for (int lo = 0; lo < nt; lo += per) {
        const int hi = lo + per < nt ? lo + per : nt;
        f32x4 acc[NTW][PT];
#pragma unroll
        for (int n = 0; n < NTW; ++n)
#pragma unroll
            for (int p = 0; p < PT; ++p) acc[n][p] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int k8 = lo & ~3; k8 < hi; k8 += 8) {
            // the operands of two products are read before the first: short
            // memories are a chain of such reads
            float ab[2][NTW];
            f32x4 vx[2];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                // tokens of another memory leave no operand, whatever they hold
                const int t = k8 + 4 * ks + g, tc = t < kQ ? t : kQ - 1;
                const bool in = t >= lo && t < hi;
                const float f = s_f[tc];
#pragma unroll
                for (int n = 0; n < NTW; ++n) ab[ks][n] = in ? s_b[tc][wn * 16 * NTW + NTW * m + n] * f : 0.f;
                vx[ks] = in ? *reinterpret_cast<const f32x4*>(&s_x[tc][4 * m]) : f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int n = 0; n < NTW; ++n)
#pragma unroll
                    for (int p = 0; p < PT; ++p)
                        acc[n][p] = mfma4(ab[ks][n], PT == 4 ? vx[ks][p] : vx[ks][p0 + p], acc[n][p]);
        }
        const float a = lo > 0 ? s_a[lo] : 0.f;
#pragma unroll
        for (int n = 0; n < NTW; ++n) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (!mo) break;
                T* o = mo + (wn * 16 * NTW + NTW * (4 * g + r) + n) * kP + 4 * m + p0;
                if constexpr (PT == 4) {
                    const float v[4] = {acc[n][0][r], acc[n][1][r], acc[n][2][r], acc[n][3][r]};
                    store4(o, v);
                } else {
#pragma unroll
                    for (int p = 0; p < PT; ++p) o[p] = from_f<T>(acc[n][p][r]);
                }
            }
#pragma unroll
            for (int p = 0; p < PT; ++p) sum[n][p] = sum[n][p] * a + acc[n][p];
        }
        if (mo) mo += H * (int64_t)(N * kP);
    }
    const int64_t base = blk * (int64_t)(N * kP);
#pragma unroll
    for (int n = 0; n < NTW; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float* o = dH + base + (wn * 16 * NTW + NTW * (4 * g + r) + n) * kP + 4 * m + p0;
            if constexpr (PT == 4) {
                const float v[4] = {sum[n][0][r], sum[n][1][r], sum[n][2][r], sum[n][3][r]};
                store4(o, v);
            } else {
#pragma unroll
                for (int p = 0; p < PT; ++p) o[p] = sum[n][p][r];
            }
        }
}

// In place: a piece's contribution becomes the state entering it.  Four pieces'
// contributions are loaded while the four before them are used, ahead of their
// stores (memory operations complete in order).  Where few waves run, the
// instructions of one bound it: no index arithmetic or test per piece, the
// chunks' sums only where they are wanted, and blocks of one wave, which spread
// over four times as many CUs (64 pieces of 8 heads, N 32: 8.8 us, 14.0 with
// 256 threads and an index product and three branches per piece).
template <typename T>
__global__ __launch_bounds__(kPassT) void k_fs_states(float* dH, const float* __restrict__ lda,
                                                   const float* __restrict__ h0, float* __restrict__ h_last,
                                                   T* __restrict__ mem, Pieces pc, int H, int NP, int64_t Mcap) {
    const int h = blockIdx.y;
    const int64_t b = blockIdx.z, bh = b * H + h;
    const int e0 = (blockIdx.x * kPassT + threadIdx.x) * 4;
    if (e0 >= NP) return;
    const float* ld = lda + bh * pc.nk;
    const int64_t step = (int64_t)H * NP;
    float* ph = dH + (b * pc.nk * H + h) * (int64_t)NP + e0;
    T* pm = pc.S > kQ ? mem + (b * Mcap * H + h) * (int64_t)NP + e0 : nullptr;
    float hc[4] = {0.f, 0.f, 0.f, 0.f}, own[4] = {0.f, 0.f, 0.f, 0.f};
    if (h0) load4(h0 + bh * (int64_t)NP + e0, hc);
    constexpr int U = 4;
    struct Part {
        float d[U][4], a[U];
    };
    const float *pl = ph, *al = ld;  // the next piece to load: the last one again past the end, not used
    const float* const ae = ld + pc.nk - 1;
    auto load = [&](Part& f) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            load4(pl, f.d[u]);
            f.a[u] = fast_exp2(*al);
            const bool more = al < ae;
            pl += more ? step : 0;
            al += more;
        }
    };
    int64_t left = pc.nk;
    int i = 0;  // piece of its chunk
    // OWN: with the sums of a chunk's pieces; TAIL: pieces may have run out
    auto pass = [&](auto OWN) __attribute__((always_inline)) {
        auto run = [&](const Part& f, auto TAIL) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (decltype(TAIL)::value && u >= left) break;
                store4(ph, hc);
                ph += step;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    hc[q] = f.a[u] * hc[q] + f.d[u][q];
                    if constexpr (decltype(OWN)::value) own[q] = (i == 0 ? 0.f : f.a[u] * own[q]) + f.d[u][q];
                }
                if (decltype(OWN)::value && (++i == pc.nq || u + 1 == left)) {
                    store4(pm, own);
                    pm += step;
                    i = 0;
                }
            }
            left -= U;
        };
        Part f0, f1;
        load(f0);
        while (left >= 2 * U) {
            load(f1);
            run(f0, std::false_type{});
            load(f0);
            run(f1, std::false_type{});
        }
        load(f1);
        if (left > 0) run(f0, std::true_type{});
        if (left > 0) run(f1, std::true_type{});
    };
    if (pm)
        pass(std::true_type{});
    else
        pass(std::false_type{});
    if (h_last) store4(h_last + bh * (int64_t)NP + e0, hc);
}

// A wave owns 16 tokens s, as columns of the tiles with t <= s and of y.  In its
// own tile a zero factor does not keep the infinity or NaN of a token t > s out
// of y_s; such a tile is summed token by token instead.  C . B is formed
// of sums of 16 products, and a tile's products are added to the earlier ones' as
// a whole (one chain over N and the tokens, rounded at each, put y of strong
// decays at N 128 2.1e-7 from 64 bits, 1.1e-7 so).
template <typename T, int N>
__global__ __launch_bounds__(kFT, 2) void k_fs_out(const T* __restrict__ x, const float* __restrict__ dt,
                                                   const float* __restrict__ A, const T* __restrict__ Bm,
                                                   const T* __restrict__ Cm, const float* __restrict__ Hs,
                                                   T* __restrict__ y, Pieces pc, int H, int G, int hpb,
                                                   int64_t blocks) {
    constexpr int K = N / 16;
    __shared__ __attribute__((aligned(16))) char s_x[kQ * 256], s_w[N * 256];
    __shared__ __attribute__((aligned(16))) float s_cl[kQ], s_lo[kQ], s_te[kQ], s_dt[kQ];
    __shared__ f32x4 s_T;
    const int64_t blk = flat_block();
    if (blk >= blocks) return;
    const int tid = threadIdx.x, lane = tid & 63, m = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nhb = H / hpb;
    const int64_t bk = blk / nhb, b = bk / pc.nk, k = bk - b * pc.nk;
    const int h0 = (int)(blk - bk * nhb) * hpb;
    const int grp = (int)((int64_t)h0 * G / H);
    int64_t t0, t1;
    piece_range(pc, k, t0, t1);
    const int nt = (int)(t1 - t0), tl = 16 * w + m;
    const bool used = 16 * w < nt;
    // a row of the piece, clamped to its last token (tokens past the end have
    // x and dt zero and are not stored)
    auto row = [&](int s) { return b * pc.L + t0 + (s < nt ? s : nt - 1); };
    const int64_t bt = row(tl);
    float cv[K][4];
#pragma unroll
    for (int q = 0; q < K; ++q) load4(Cm + (bt * G + grp) * N + 16 * q + 4 * g, cv[q]);
    f32x4 g1[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        g1[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (j <= w && 16 * j < nt) {
            const T* br = Bm + (row(16 * j + m) * G + grp) * N + 4 * g;
#pragma unroll
            for (int q = 0; q < K; ++q) {
                float b4[4];
                load4(br + 16 * q, b4);
                f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < 4; ++s) a = mfma4(b4[s], cv[q][s], a);
                g1[j] += a;
            }
        }
    }
    PieceOff<N> off;
    off.init(m, g);
    for (int hh = 0; hh < hpb; ++hh) {
        const int h = h0 + hh;
        if (hh > 0) __syncthreads();
        PieceOff<N>::stage(Hs + ((b * pc.nk + k) * H + h) * (int64_t)(N * kP), s_w, tid);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int s = (tid >> 4) + 16 * q, c = tid & 15;
            float x4[4] = {0.f, 0.f, 0.f, 0.f};
            if (s < nt) load4(x + (row(s) * H + h) * kP + 4 * c, x4);
            *reinterpret_cast<f32x4*>(s_x + s * 256 + ((c ^ (s & 15)) << 4)) = f32x4{x4[0], x4[1], x4[2], x4[3]};
        }
        if (w == 0) {
            PieceDecay pd;
            pd.load(dt, A[h], b, pc.L, H, h, t0, t1, lane);
            s_cl[lane] = pd.cl;
            s_lo[lane] = pd.lo;
            s_te[lane] = pd.te;
            s_dt[lane] = pd.d;
            if (lane == 0) s_T = pd.T;
        }
        __syncthreads();
        if (!used) continue;
        const f32x4 tt = s_T;
        const float cs = s_cl[tl], cl = s_lo[tl];
        f32x4 yi[4], yw[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) yi[i] = yw[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < K; ++q)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const f32x4 a = off.state_p(s_w, q, s);
#pragma unroll
                for (int i = 0; i < 4; ++i) yw[i] = mfma4(a[i], cv[q][s], yw[i]);
            }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j <= w && 16 * j < nt) {
                const f32x4 ct = *reinterpret_cast<const f32x4*>((j == w ? s_cl : s_te) + 16 * j + 4 * g);
                const f32x4 tlo = *reinterpret_cast<const f32x4*>(s_lo + 16 * j + 4 * g);
                const f32x4 dtt = *reinterpret_cast<const f32x4*>(s_dt + 16 * j + 4 * g);
                float bq[4];
                f32x4 yj[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) yj[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float l = j == w ? log_decay_in(cs, cl, ct[r], tlo[r]) : log_decay_over(tt, w, cs, j, ct[r]);
                    const float e = fast_exp2(fminf(l, 0.f)) * dtt[r];
                    bq[r] = j == w && 4 * g + r > m ? 0.f : e * g1[j][r];
                    const f32x4 a = lds4(s_x + j * 4096 + off.op[r]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) yj[i] = mfma4(a[i], bq[r], yj[i]);
                }
                if (j == w && any_nonfinite(yj)) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) yj[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int t = 4 * q + r;
                            const float f = __shfl(bq[r], 16 * q + m, 64);
#pragma unroll
                            for (int r2 = 0; r2 < 4; ++r2) {
                                const f32x4 xv = lds4(s_x + j * 4096 + t * 256 + (((4 * g + r2) ^ t) << 4));
#pragma unroll
                                for (int i = 0; i < 4; ++i)
                                    if (t <= m) yj[i][r2] += f * xv[i];
                            }
                        }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) yi[i] += yj[i];
            }
        }
        if (tl < nt) {
            const float ec = fast_exp2(log_from_start(tt, w, cs));
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float o[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = yi[i][r] + ec * yw[i][r];
                store4(y + (bt * H + h) * kP + 16 * g + 4 * r, o);
            }
        }
    }
}

struct FScanWs {
    float* lda;  // [B][H][nk]
    float* dH;   // [B][nk][H][N][P]: contributions, then entering states
    size_t total;
};
FScanWs fscan_ws(const Shape& s, void* base) {
    const size_t BHK = (size_t)s.B * s.H * pieces_of(s).nk;
    char* p = reinterpret_cast<char*>(base);
    FScanWs w;
    w.lda = reinterpret_cast<float*>(p);
    w.dH = p ? reinterpret_cast<float*>(p + align256(4 * BHK)) : nullptr;
    w.total = align256(4 * BHK) + align256(4 * BHK * s.N * (size_t)s.P);
    return w;
}

template <typename T, int N>
hipError_t run_fscan(const Shape& s, const void* x, const float* dt, const float* A, const void* Bm,
                     const void* Cm, const float* h0, void* y, void* mem, float* hl, void* ws, hipStream_t st) {
    const Pieces pc = pieces_of(s);
    const FScanWs w = fscan_ws(s, ws);
    constexpr int NP = N * kP;
    const int64_t units = s.B * pc.nk * s.H;
    prof_begin("k_chunk_state", st);
    k_fs_state<T, N><<<flat_grid(units, kFT), kFT, 0, st>>>((const T*)x, dt, A, (const T*)Bm, (T*)mem, w.dH,
                                                       w.lda, pc, s.H, s.G, s.Mcap, units);
    prof_end(st);
    prof_begin("k_state_pass", st);
    k_fs_states<T><<<dim3((NP + 4 * kPassT - 1) / (4 * kPassT), (unsigned)s.H, (unsigned)s.B), kPassT, 0, st>>>(
        w.dH, w.lda, h0, hl, (T*)mem, pc, s.H, NP, s.Mcap);
    prof_end(st);
    const int hpb = piece_heads_per_block(s, pc.nk);
    const int64_t blocks = s.B * pc.nk * (s.H / hpb);
    prof_begin("k_chunk_out", st);
    k_fs_out<T, N><<<flat_grid(blocks, kFT), kFT, 0, st>>>((const T*)x, dt, A, (const T*)Bm, (const T*)Cm, w.dH,
                                                      (T*)y, pc, s.H, s.G, hpb, blocks);
    prof_end(st);
    return hipGetLastError();
}

}  // namespace

// At least the parts that callers know the workspace by, per chunk and (b, h): a
// log decay and an entry state in the storage dtype, and at N >= 32 with S in
// {64, 128, 256} three floats per token and a group's causal Gram tiles, elsewhere
// two states in float.  The pieces need less at small S, and more where a chunk
// is several pieces.
size_t fscan_workspace_bytes(const Shape& s) {
    const size_t chunks = (size_t)s.B * s.M * s.H, state = (size_t)s.N * s.P, need = fscan_ws(s, nullptr).total;
    size_t known = align256(4 * chunks) + align256(elem_bytes(s.dtype) * chunks * state);
    if (s.N >= 32 && (s.S == 64 || s.S == 128 || s.S == 256))
        known += align256(4 * chunks * 3 * s.S) + align256(4 * (size_t)s.B * s.G * s.M * (s.S / 32) * (s.S / 32 + 1) * 512);
    else
        known += 2 * align256(4 * chunks * state);
    return need > known ? need : known;
}

hipError_t launch_fscan(const Shape& s, const void* x, const float* dt, const float* A, const void* Bm,
                        const void* Cm, const float* h0, void* y_ssd, void* mem, float* h_last, void* ws,
                        hipStream_t st) {
#define DART_FS(T, NN) run_fscan<T, NN>(s, x, dt, A, Bm, Cm, h0, y_ssd, mem, h_last, ws, st)
    if (s.dtype == 1) {
        switch (s.N) {
            case 16: return DART_FS(bf16, 16);
            case 32: return DART_FS(bf16, 32);
            case 64: return DART_FS(bf16, 64);
            case 128: return DART_FS(bf16, 128);
        }
    } else {
        switch (s.N) {
            case 16: return DART_FS(float, 16);
            case 32: return DART_FS(float, 32);
            case 64: return DART_FS(float, 64);
            case 128: return DART_FS(float, 128);
        }
    }
#undef DART_FS
    return hipErrorInvalidValue;
}

}  // namespace dart
