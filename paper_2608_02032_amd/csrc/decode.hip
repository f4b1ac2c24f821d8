// decode.hip -- single-token decode step over the cached chunk memories.
//
// Paper: Sec. 4 "Inference Cache" (the decode cache is one N x P memory per
// completed chunk plus the recurrent state), Sec. 3 (SMA over strictly earlier
// chunks, gated residual) and App. B.1 (normalised score branch).  Keys depend
// on the current token (K = r (.) (dH E_t)), so every step re-reads every
// cached memory: the step is a stream over B*H*m*N*P storage elements and is
// bound by HBM bandwidth.
//
//   k_decode_partial      a block per (split, head, batch) streams up to
//                         decode_mps() memories, one wave per memory at a time;
//                         lanes own 8 consecutive p of N/8 rows.  Each wave
//                         keeps the next memory's rows in flight while it
//                         reduces the current one (r, the logit and C dH on
//                         the fly; online softmax (m, d, O[P])).  Waves merge
//                         in LDS; one partial per split goes to the workspace.
//                         After these (or in k_decode_state_merge, state_apart()),
//                         a block per (head, batch) makes the recurrent update of
//                         h_state and of the running chunk contribution,
//                         y_ssd = C h_state, and the append of the running
//                         contribution when the token closes its chunk (slot m,
//                         never read by this step).
//   k_decode_merge        a wave per (head, batch): the deterministic LSE merge
//                         of the split partials and y = y_ssd + SiLU(z) R.
//   k_decode_one          both in one launch, a block of eight waves per (head,
//                         batch), where decode_in_one() says so.
// A block requests q, e and C, then its first memory rows, and forms the row
// norms while those are on their way (loads return in order: with the rows
// first, or after the norms, 384 (b, h) of bf16, N 128, one memory take 8.0 us in
// the streaming kernel, 7.9 so; 2048 (b, h) of fp32, N 16, 64 memories 109 and 107
// us a step).
// Measured, N 128, S 256, bf16, ragged contexts, against the state update in the
// merging kernel, the first loads after the set-up and the split index fastest:
// B 16, 24 heads, up to 16384: 74 -> 51 us; B 64, 32 heads, up to 32768: 436 ->
// 374.  B 1, context 4095: 12.1 -> 10.5 (and one launch instead of two).
#include "dart_common.hpp"
#include "dart_internal.hpp"

#include <cstdlib>
#include <mutex>
#include <type_traits>

#include "dart.h"

namespace dart {
namespace {

constexpr int kP = 64;
constexpr int kThreads = 256;
// Memories per split.  Long splits amortise each block's set-up (measured:
// at 64 x 32 heads and 256 memories, 128-memory splits beat 32-memory ones by
// 4 % on a uniform batch and 18 % on a ragged one); the split size is halved
// (down to 8) while that leaves fewer than 4096 blocks (16 per CU).
// DART_DECODE_MPS in {8, 16, 32, 64, 128} forces a size, and with it the step in
// splits (tuning); the workspace is sized for the smallest.
int forced_mps() {
    static const int forced = [] {
        const char* e = getenv("DART_DECODE_MPS");
        const int x = e ? atoi(e) : 0;
        return (x == 8 || x == 16 || x == 32 || x == 64 || x == 128) ? x : 0;
    }();
    return forced;
}
int decode_mps(int64_t bh, int64_t m) {
    if (forced_mps()) return forced_mps();
    int mps = 128;
    while (mps > 8 && bh * ((m + mps - 1) / mps) < 4096) mps >>= 1;
    return mps;
}
constexpr int kMinMPS = kDecodeMinMemPerSplit;

__device__ __forceinline__ bf16x2 as_bf2(uint32_t u) { return __builtin_bit_cast(bf16x2, u); }
__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(as_bf2(a), as_bf2(b), c, false);
}
__device__ __forceinline__ uint32_t pack_bf2(float lo, float hi) {
    const bf16x2 v{(bf16)lo, (bf16)hi};
    return __builtin_bit_cast(uint32_t, v);
}

// One memory row chunk held by a lane: 8 consecutive p of one row n.
template <typename T> struct RowChunk;
template <> struct RowChunk<bf16> { uint4 v; };
template <> struct RowChunk<float> { f32x4 a, b; };

// The cache is read once per step: nontemporal loads keep it from displacing
// anything in the caches (and stream faster than ordinary loads).
__device__ __forceinline__ void load_row(const bf16* p, RowChunk<bf16>& r) {
    const u32x4_nt w = __builtin_nontemporal_load(reinterpret_cast<const u32x4_nt*>(p));
    r.v = make_uint4(w.x, w.y, w.z, w.w);
}
__device__ __forceinline__ void load_row(const float* p, RowChunk<float>& r) {
    r.a = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
    r.b = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p + 4));
}

// Workspace layout: partials [B][H][nsplit][P+2] (O[P], m, d), then y_ssd
// [B][H][P] (float).
inline size_t decode_part_floats(int64_t B, int H, int nsplit) {
    return (size_t)B * H * nsplit * (kP + 2);
}

// By a block of 64 WAVES threads; s_y holds a row per wave.  At N = 128 the rows of B
// and C come through LDS (s_bc): as elements of each thread's own rows they are
// 16 loads more in flight per thread, 0.2 us of a 5.5 us step without memories.
// (With fewer rows the barrier costs as much: 2048 (b, h), N 64, one memory 33.2 us
// without and 34.5 with it.)
template <int N> constexpr bool stage_bc() { return N == 128; }
template <typename T, int N, int WAVES>
__device__ __forceinline__ void state_update(const T* __restrict__ x, const float* __restrict__ dt,
                                             const float* __restrict__ A, const T* __restrict__ Bm,
                                             const T* __restrict__ Cm, float* __restrict__ h_state,
                                             float* __restrict__ chunk_acc, T* __restrict__ mem,
                                             int H, int G, int S, int64_t Mcap, int64_t pos,
                                             int64_t m, int64_t b, int h, int g, float (*s_y)[kP],
                                             float (*s_bc)[stage_bc<N>() ? N : 1]) {
    constexpr int RG = 4 * WAVES, K = (N + RG - 1) / RG;  // row groups, rows per thread
    const int tid = threadIdx.x;
    const int pq = tid & 15, rg = tid >> 4;  // p quad, row group
    const bool reset = (pos % S) == 0;
    const bool append = (pos % S) == S - 1;
    const int64_t sbase = (b * H + h) * (int64_t)N * kP;
    float hs[K][4], ca[K][4], xv[4], yp[4] = {0.f, 0.f, 0.f, 0.f}, bt = 0.f, ct = 0.f;
    if (stage_bc<N>() && tid < N) {
        bt = to_f(Bm[(b * G + g) * N + tid]);
        ct = to_f(Cm[(b * G + g) * N + tid]);
    }
    if constexpr (stage_bc<N>()) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int n = rg + RG * k;
#pragma unroll
        for (int i = 0; i < 4; ++i) ca[k][i] = 0.f;
        if (n >= N) continue;
        load4(h_state + sbase + n * kP + 4 * pq, hs[k]);
        if (!reset) load4(chunk_acc + sbase + n * kP + 4 * pq, ca[k]);
    }
    load4(x + (b * H + h) * kP + 4 * pq, xv);
    const float dtv = dt[b * H + h];
    const float a = __expf(dtv * A[h]);
    T* mdst = mem + ((b * Mcap + m) * H + h) * (int64_t)N * kP;
    if constexpr (stage_bc<N>()) {
        __builtin_amdgcn_sched_barrier(0);
        if (tid < N) {
            s_bc[0][tid] = bt;
            s_bc[1][tid] = ct;
        }
        lds_barrier();  // (the state stays in flight)
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int n = rg + RG * k;
        if (n >= N) continue;
        const float bn = dtv * (stage_bc<N>() ? s_bc[0][n] : to_f(Bm[(b * G + g) * N + n]));
        const float cn = stage_bc<N>() ? s_bc[1][n] : to_f(Cm[(b * G + g) * N + n]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float u = bn * xv[i];
            hs[k][i] = a * hs[k][i] + u;
            ca[k][i] = a * ca[k][i] + u;
            yp[i] += cn * hs[k][i];
        }
        store4(h_state + sbase + n * kP + 4 * pq, hs[k]);
        store4(chunk_acc + sbase + n * kP + 4 * pq, ca[k]);
        if (append) store4(mdst + n * kP + 4 * pq, ca[k]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) yp[i] = row4_sum(yp[i]);
    if ((tid & 63) < 16) store4(&s_y[tid >> 6][4 * pq], yp);
}

// One token's attention over memories, a wave at a time: lanes own 8
// consecutive p (po) of rows n = rg + 8 k.
template <typename T, int N>
struct Attend {
    static constexpr int R = N / 8;
    using Rows = RowChunk<T>[R];
    float eb[8], qb[R], cb[R];
    uint32_t ebp[4], cbp[R / 2];  // packed bf16 copies for the dot2 path
    float mx, den, o[8];
    float eps;
    int normalize, po, rg;

    __device__ __forceinline__ void load(const T* src, Rows& xr) const {
#pragma unroll
        for (int k = 0; k < R; ++k) load_row(src + (rg + 8 * k) * kP + po * 8, xr[k]);
    }
    // s_q, s_e: Qbar log2(e)/sqrt(N) and Ebar in LDS
    __device__ __forceinline__ void init(const float* s_q, const float* s_e) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            eb[i] = s_e[po * 8 + i];
            o[i] = 0.f;
        }
#pragma unroll
        for (int k = 0; k < R; ++k) qb[k] = s_q[rg + 8 * k];
#pragma unroll
        for (int i = 0; i < 4; ++i) ebp[i] = pack_bf2(eb[2 * i], eb[2 * i + 1]);
#pragma unroll
        for (int k = 0; k < R / 2; ++k) cbp[k] = pack_bf2(cb[2 * k], cb[2 * k + 1]);
        mx = -INFINITY;
        den = 0.f;
    }
    __device__ __forceinline__ void load_c(const T* crow) {
#pragma unroll
        for (int k = 0; k < R; ++k) cb[k] = to_f(crow[rg + 8 * k]);
    }
    __device__ __forceinline__ void reduce(const Rows& xr) {
        float lsum = 0.f, v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = 0.f;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            float ss, kv;
            if constexpr (sizeof(T) == 2) {
                const uint32_t w[4] = {xr[k].v.x, xr[k].v.y, xr[k].v.z, xr[k].v.w};
                ss = dot2(w[0], w[0], 0.f);
                kv = dot2(w[0], ebp[0], 0.f);
#pragma unroll
                for (int i = 1; i < 4; ++i) {
                    ss = dot2(w[i], w[i], ss);
                    kv = dot2(w[i], ebp[i], kv);
                }
                if (k & 1) {
                    // value side: pair rows k-1 and k so one dot2 covers both
                    // (v_perm: the low halves of rows k-1, k, then the high halves)
                    const uint32_t u[4] = {xr[k - 1].v.x, xr[k - 1].v.y, xr[k - 1].v.z,
                                           xr[k - 1].v.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t lo = __builtin_amdgcn_perm(w[i], u[i], 0x05040100u);
                        const uint32_t hi = __builtin_amdgcn_perm(w[i], u[i], 0x07060302u);
                        v[2 * i] = dot2(lo, cbp[k >> 1], v[2 * i]);
                        v[2 * i + 1] = dot2(hi, cbp[k >> 1], v[2 * i + 1]);
                    }
                }
            } else {
                const float xv[8] = {xr[k].a[0], xr[k].a[1], xr[k].a[2], xr[k].a[3],
                                     xr[k].b[0], xr[k].b[1], xr[k].b[2], xr[k].b[3]};
                ss = 0.f;
                kv = 0.f;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    ss += xv[i] * xv[i];
                    kv += xv[i] * eb[i];
                    v[i] += cb[k] * xv[i];
                }
            }
            // the row's sum of squares over its 8 lanes (DPP), then its inverse
            // RMS; the logit partial kv is summed over the lanes once per memory
            ss = dpp_group_sum<8>(ss);
            const float r = normalize ? __builtin_amdgcn_rsqf(ss * (1.0f / kP) + eps) : 1.0f;
            lsum += qb[k] * r * kv;
        }
        lsum = dpp_group_sum<16>(lsum);
        lsum = row4_sum(lsum);
        const float mn = fmaxf(mx, lsum);
        const float al = fast_exp2(mx - mn), pw = fast_exp2(lsum - mn);
        den = den * al + pw;
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = o[i] * al + pw * v[i];
        mx = mn;
    }
    // the wave's (O, m, d) into its row of s_part
    __device__ __forceinline__ void publish(float* row) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            o[i] += shfl_xor(o[i], 8);
            o[i] += shfl_xor(o[i], 16);
            o[i] += shfl_xor(o[i], 32);
        }
        if (rg == 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) row[po * 8 + i] = o[i];
        }
        if (po == 0 && rg == 0) {
            row[kP] = mx;
            row[kP + 1] = den;
        }
    }
};

// n / d and n % d, in 32 bits where n fits (a division in 64 is some hundred
// instructions ahead of the block's first load).
__device__ __forceinline__ void div_mod(int64_t n, int d, int64_t& quot, int& rem) {
    if (n <= 0xFFFFFFFFll) {
        const unsigned u = (unsigned)n, k = u / (unsigned)d;
        quot = k;
        rem = (int)(u - k * (unsigned)d);
    } else {
        quot = n / d;
        rem = (int)(n - quot * d);
    }
}
// Block id's (b, h) and split, with (b, h) fastest of BH = d, or the split of
// ns = d.
__device__ __forceinline__ void split_block(int64_t id, int64_t d, bool bh_fastest, int64_t& bh, int& s) {
    int64_t k, r;
    if (id <= 0xFFFFFFFFll) {
        const unsigned u = (unsigned)id, v = u / (unsigned)d;
        k = v;
        r = u - v * (unsigned)d;
    } else {
        k = id / d;
        r = id - k * d;
    }
    bh = bh_fastest ? r : k;
    s = (int)(bh_fastest ? k : r);
}

// Qbar log2(e)/sqrt(N) by wave 0, Ebar by wave 1, into LDS.  Requested ahead of the
// memories (loads return in order), so that the norms are formed while those
// are on their way.
template <typename T, int N>
struct NormQE {
    float v0, v1;
    __device__ __forceinline__ void request(const T* __restrict__ qrow, const T* __restrict__ erow) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        v0 = v1 = 0.f;
        if (wave == 0) {
            if (lane < N) v0 = to_f(qrow[lane]);
            if (lane + 64 < N) v1 = to_f(qrow[lane + 64]);
        } else if (wave == 1) {
            v0 = to_f(erow[lane]);
        }
    }
    __device__ __forceinline__ void finish(const float* __restrict__ qw, const float* __restrict__ ew, float eps,
                                           int normalize, float* s_q, float* s_e) const {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        if (wave > 1) return;
        float ss = v0 * v0 + v1 * v1;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) ss += shfl_xor(ss, o);
        if (wave == 0) {
            const float inv = (normalize ? 1.0f / sqrtf(ss * (1.0f / N) + eps) : 1.0f) *
                              (kLog2e / sqrtf((float)N));
            if (lane < N) s_q[lane] = v0 * inv * (qw ? qw[lane] : 1.0f);
            if (lane + 64 < N) s_q[lane + 64] = v1 * inv * (qw ? qw[lane + 64] : 1.0f);
        } else {
            const float inv = normalize ? 1.0f / sqrtf(ss * (1.0f / kP) + eps) : 1.0f;
            s_e[lane] = v0 * inv * (ew ? ew[lane] : 1.0f);
        }
    }
};

// STATE: the blocks past the stream's make the state updates.
// (bf16, N = 64: held to the 128 registers of four waves a SIMD.)
template <typename T, int N, bool STATE>
__global__ __launch_bounds__(kThreads, (sizeof(T) == 2 && N == 64 ? 4 : 1)) void k_decode_partial(
    const T* __restrict__ x, const float* __restrict__ dt, const float* __restrict__ A,
    const T* __restrict__ Bm, float* __restrict__ h_state, float* __restrict__ chunk_acc,
    T* mem, float* __restrict__ yssd, const T* __restrict__ q, const T* __restrict__ e,
    const T* __restrict__ Cm, const float* __restrict__ qw, const float* __restrict__ ew,
    float* __restrict__ part, float eps, int normalize, int H, int G, int S, int64_t Mcap,
    int64_t pos, const int64_t* __restrict__ pos_rows, int64_t pos_lim, int nsplit, int mps, int ns,
    int64_t BH, bool bh_fastest) {
    const int64_t id = flat_block(), nstream = BH * ns;
    if (id >= (STATE ? nstream + BH : nstream)) return;  // (past the last block of the grid's last row)
    // A (b, h)'s splits one after the other, or with (b, h) fastest where the host says
    // so.  The state blocks come last and overlap the stream's end.
    const bool state = STATE && id >= nstream;
    int64_t bh = id - nstream, b;
    int s = 0, h;
    if (!state) split_block(id, bh_fastest ? BH : ns, bh_fastest, bh, s);
    div_mod(bh, H, b, h);
    const int g = (int)((int64_t)h * G / H);
    if (pos_rows) {
        // ragged batch: this row's own position; rows outside [0, pos_lim]
        // take no part in the step
        pos = pos_rows[b];
        if (pos < 0 || pos > pos_lim) return;
    }
    const int64_t m = pos / S;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    __shared__ float s_q[N];
    __shared__ float s_e[kP];
    __shared__ __attribute__((aligned(16))) float s_part[4][kP + 4];
    if constexpr (STATE) if (state) {
        float(*s_y)[kP] = reinterpret_cast<float(*)[kP]>(&s_part[0][0]);
        __shared__ float s_bc[2][stage_bc<N>() ? N : 1];
        state_update<T, N, 4>(x, dt, A, Bm, Cm, h_state, chunk_acc, mem, H, G, S, Mcap, pos, m, b, h, g, s_y, s_bc);
        __syncthreads();
        if (tid < kP) yssd[(b * H + h) * kP + tid] = (s_y[0][tid] + s_y[1][tid]) + (s_y[2][tid] + s_y[3][tid]);
        return;
    }
    const int64_t j0 = (int64_t)s * mps;
    const int64_t j1 = (j0 + mps < m) ? j0 + mps : m;
    if (j0 >= j1) return;  // block-uniform: no cached memory in this split

    // wave w takes memories j0 + w, j0 + w + 4, ...; the next one's rows are
    // loaded before the current one is reduced (two register buffers)
    const T* src = mem + (b * Mcap * H + h) * (int64_t)N * kP;
    const int64_t step = (int64_t)H * N * kP;
    Attend<T, N> at;
    at.po = lane & 7;
    at.rg = lane >> 3;
    at.eps = eps;
    at.normalize = normalize;
    typename Attend<T, N>::Rows xa, xb;
    NormQE<T, N> nq;
    nq.request(q + (b * G + g) * N, e + (b * G + g) * kP);
    at.load_c(Cm + (b * G + g) * N);
    __builtin_amdgcn_sched_barrier(0);
    int64_t j = j0 + wave;
    if (j < j1) at.load(src + j * step, xa);
    __builtin_amdgcn_sched_barrier(0);
    nq.finish(qw, ew, eps, normalize, s_q, s_e);
    lds_barrier();  // (the first rows stay in flight)
    at.init(s_q, s_e);
    while (j < j1) {
        if (j + 4 < j1) at.load(src + (j + 4) * step, xb);
        at.reduce(xa);
        j += 4;
        if (j >= j1) break;
        if (j + 4 < j1) at.load(src + (j + 4) * step, xa);
        at.reduce(xb);
        j += 4;
    }
    at.publish(s_part[wave]);
    __syncthreads();
    if (tid < kP) {
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < 4; ++w) M = fmaxf(M, s_part[w][kP]);
        float D = 0.f, O = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float mw = s_part[w][kP];
            if (mw == -INFINITY) continue;
            const float sc = fast_exp2(mw - M);
            D += s_part[w][kP + 1] * sc;
            O += s_part[w][tid] * sc;
        }
        float* out = part + (((b * H + h) * nsplit) + s) * (kP + 2);
        out[tid] = O;
        if (tid == 0) {
            out[kP] = M;
            out[kP + 1] = D;
        }
    }
}

// The LSE merge of a (b, h)'s split partials and the gate, by one wave (lane = p),
// in two steps: `request` loads what the merge begins with (the gate, and the
// statistics of the split of the lane's number), so that the latency passes
// behind other work, `finish` merges and writes y (ys: y_ssd of the lane's column).
template <typename T>
struct Merge {
    const float* pb;
    float zz, m0, d0;
    int ns;
    __device__ __forceinline__ void request(const T* __restrict__ z, const float* __restrict__ part, int64_t bh,
                                            int64_t b, int64_t m, int nsplit, int z_per_head, int mps) {
        const int p = threadIdx.x & 63;
        zz = to_f(z_per_head ? z[bh] : z[b]);
        ns = (int)((m + mps - 1) / mps);
        pb = part + bh * nsplit * (int64_t)(kP + 2);
        m0 = -INFINITY;
        d0 = 0.f;
        if (p < ns) {
            m0 = pb[p * (kP + 2) + kP];
            d0 = pb[p * (kP + 2) + kP + 1];
        }
    }
    __device__ __forceinline__ void finish(T* __restrict__ y, float ys, int64_t bh) const {
        const int p = threadIdx.x & 63;
        float R = 0.f;
        if (ns > 0) {
            // maximum and sum with a split per lane, O with a column per lane
            float M = m0, D, O = 0.f;
            for (int s = p + 64; s < ns; s += 64) M = fmaxf(M, pb[s * (kP + 2) + kP]);
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) M = fmaxf(M, shfl_xor(M, o));
            D = p < ns ? d0 * fast_exp2(m0 - M) : 0.f;
            for (int s = p + 64; s < ns; s += 64) D += pb[s * (kP + 2) + kP + 1] * fast_exp2(pb[s * (kP + 2) + kP] - M);
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) D += shfl_xor(D, o);
#pragma unroll 8
            for (int s = 0; s < ns; ++s) O += pb[s * (kP + 2) + p] * fast_exp2(pb[s * (kP + 2) + kP] - M);
            R = O / D;
        }
        y[bh * kP + p] = from_f<T>(ys + silu(zz) * R);
    }
};

// After a stream that made the state updates: one wave per (b, h).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_decode_merge(
    const T* __restrict__ z, T* __restrict__ y, const float* __restrict__ part,
    const float* __restrict__ yssd, int H, int S, int64_t pos, const int64_t* __restrict__ pos_rows,
    int64_t pos_lim, int nsplit, int z_per_head, int mps, int64_t BH) {
    const int64_t bh = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (bh >= BH) return;
    int64_t b;
    int h;
    div_mod(bh, H, b, h);
    if (pos_rows) {
        pos = pos_rows[b];
        if (pos < 0 || pos > pos_lim) return;  // the row takes no part in the step
    }
    Merge<T> mg;
    mg.request(z, part, bh, b, pos / S, nsplit, z_per_head, mps);
    mg.finish(y, yssd[bh * kP + (threadIdx.x & 63)], bh);
}

// After a stream that did not, or without one: a block per (b, h) makes the state
// update, then its first wave merges.
template <typename T, int N>
__global__ __launch_bounds__(kThreads) void k_decode_state_merge(
    const T* __restrict__ x, const float* __restrict__ dt, const float* __restrict__ A,
    const T* __restrict__ Bm, const T* __restrict__ Cm, const T* __restrict__ z,
    float* __restrict__ h_state, float* __restrict__ chunk_acc, T* __restrict__ mem,
    T* __restrict__ y, const float* __restrict__ part, int H, int G, int S, int64_t Mcap, int64_t pos,
    const int64_t* __restrict__ pos_rows, int64_t pos_lim, int nsplit, int z_per_head, int mps) {
    const int h = blockIdx.x;
    const int64_t b = blockIdx.y;
    if (pos_rows) {
        pos = pos_rows[b];
        if (pos < 0 || pos > pos_lim) return;
    }
    __shared__ __attribute__((aligned(16))) float s_y[4][kP];
    __shared__ float s_bc[2][stage_bc<N>() ? N : 1];
    const int tid = threadIdx.x;
    Merge<T> mg;
    if (tid < kP) mg.request(z, part, b * H + h, b, pos / S, nsplit, z_per_head, mps);
    state_update<T, N, 4>(x, dt, A, Bm, Cm, h_state, chunk_acc, mem, H, G, S, Mcap, pos, pos / S, b, h,
                          (int)((int64_t)h * G / H), s_y, s_bc);
    lds_barrier();
    if (tid >= kP) return;
    mg.finish(y, (s_y[0][tid] + s_y[1][tid]) + (s_y[2][tid] + s_y[3][tid]), b * H + h);
}

// The whole step of one (b, h) in one block of eight waves: wave w takes
// memories w, w + 8, ..., after its part of the state update.
constexpr int kOneWaves = 8;
template <typename T, int N>
__global__ __launch_bounds__(64 * kOneWaves, 2) void k_decode_one(
    const T* __restrict__ x, const float* __restrict__ dt, const float* __restrict__ A,
    const T* __restrict__ Bm, float* __restrict__ h_state, float* __restrict__ chunk_acc, T* mem,
    const T* __restrict__ q, const T* __restrict__ e, const T* __restrict__ Cm,
    const T* __restrict__ z, T* __restrict__ y, const float* __restrict__ qw,
    const float* __restrict__ ew, float eps, int normalize, int H, int G, int S, int64_t Mcap,
    int64_t pos, const int64_t* __restrict__ pos_rows, int64_t pos_lim, int z_per_head) {
    const int h = blockIdx.x;
    const int64_t b = blockIdx.y;
    const int g = (int)((int64_t)h * G / H);
    if (pos_rows) {
        pos = pos_rows[b];
        if (pos < 0 || pos > pos_lim) return;
    }
    const int64_t m = pos / S;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    __shared__ float s_q[N];
    __shared__ float s_e[kP];
    __shared__ float s_part[kOneWaves][kP + 2];
    __shared__ __attribute__((aligned(16))) float s_y[kOneWaves][kP];
    __shared__ float s_bc[2][stage_bc<N>() ? N : 1];
    const T* src = mem + (b * Mcap * H + h) * (int64_t)N * kP;
    const int64_t step = (int64_t)H * N * kP;
    Attend<T, N> at;
    at.po = lane & 7;
    at.rg = lane >> 3;
    at.eps = eps;
    at.normalize = normalize;
    typename Attend<T, N>::Rows xa;
    NormQE<T, N> nq;
    nq.request(q + (b * G + g) * N, e + (b * G + g) * kP);
    at.load_c(Cm + (b * G + g) * N);
    __builtin_amdgcn_sched_barrier(0);
    if (wave < m) at.load(src + wave * step, xa);
    __builtin_amdgcn_sched_barrier(0);
    nq.finish(qw, ew, eps, normalize, s_q, s_e);
    state_update<T, N, kOneWaves>(x, dt, A, Bm, Cm, h_state, chunk_acc, mem, H, G, S, Mcap, pos, m, b, h, g, s_y, s_bc);
    lds_barrier();
    at.init(s_q, s_e);
    for (int64_t j = wave; j < m; j += kOneWaves) {
        if (j >= kOneWaves) at.load(src + j * step, xa);
        at.reduce(xa);
    }
    at.publish(s_part[wave]);
    __syncthreads();
    if (tid >= kP) return;
    float ys = 0.f, M = -INFINITY, D = 0.f, O = 0.f;
#pragma unroll
    for (int w = 0; w < kOneWaves; ++w) {
        ys += s_y[w][tid];
        M = fmaxf(M, s_part[w][kP]);
    }
#pragma unroll
    for (int w = 0; w < kOneWaves; ++w) {
        const float mw = s_part[w][kP];
        if (mw == -INFINITY) continue;
        const float sc = fast_exp2(mw - M);
        D += s_part[w][kP + 1] * sc;
        O += s_part[w][tid] * sc;
    }
    const float R = m > 0 ? O / D : 0.f;
    const float zz = to_f(z_per_head ? z[b * H + h] : z[b]);
    y[(b * H + h) * kP + tid] = from_f<T>(ys + silu(zz) * R);
}

// One launch where it is the shorter way: at most two memories per wave and the
// blocks resident at once, one per CU at N = 128, two at 64, four at 32, or soon
// (eight at 16).  bf16, N 128, 16 memories: 256 (b, h) 20.8 us against 23.3 in two
// launches, 384 33.3 against 31.5.  In fp32 twelve memories and more are better
// spread over the chip where two splits of each (b, h) fit on it (N = 128: 32 (b, h)
// of 12 memories 19.3 us against 16.1, of 10 15.8 and 15.1; 128 of 9 19.3 and 22.0;
// 240 of 16 33.0 and 39.0), or they are a quarter to half of its CUs (N = 64: 128
// (b, h) of 16 memories 15.7 against 13.8, of 12 13.3 and 13.4; 160 of 16 17.2 and 19.8).  At fp32, N = 128,
// the streaming kernel has one wave a SIMD and the one launch is the shorter way
// for any number of blocks (2048 (b, h): 1 memory 76 us against 84, 16 272 against
// 297).
template <typename T, int N>
inline bool decode_in_one(int64_t bh, int64_t m) {
    const int64_t cus = device_cu_count();
    const bool wide = sizeof(T) == 4 && N == 128;
    const bool spread = wide ? 2 * bh <= cus : sizeof(T) == 4 && N == 64 && 4 * bh >= cus && 2 * bh <= cus;
    if (forced_mps() || m < 1 || m > 2 * kOneWaves || (spread && m >= 12)) return false;
    return wide || bh <= cus * (N == 128 ? 1 : 128 / N);
}
// Otherwise, or without memories: whether the state updates have their own
// kernel.  In the stream they save a pass over the chip (context 20000, B 8, 24
// heads: 51.2 us against 52.7), but there they run in blocks of many registers:
// after a stream of gigabytes (context 65536, B 64, 32 heads, 8.6 GB: 1274 us in
// the stream, 1260 apart; 3.6 GB the same), where the stream is no longer than
// the states' own traffic (2048 (b, h), N 128, 1 memory: 63.4 and 60.6; 3: 68.2 and
// 70.2), and for fp32 at N = 128 with a block per CU or more (768 (b, h), 3
// memories: 49.7 and 43.5) the kernel of few registers is faster.
template <typename T, int N>
inline bool state_apart(int64_t bh, int64_t m) {
    const int64_t cus = device_cu_count();
    return m == 0 || bh * m * N * kP * (int64_t)sizeof(T) >= (int64_t)4 << 30 ||
           (bh > cus && m * (int64_t)sizeof(T) <= 4) || (sizeof(T) == 4 && N == 128 && bh >= cus);
}

// Whether the stream's blocks go with (b, h) fastest, not a (b, h)'s splits one after
// the other (1253 us against 1265 at B 64, context 65536).  In a ragged batch of an
// even number of splits: its short rows leave the later splits empty, and with the
// split index fastest (8 XCDs, workgroups dealt in turn) a split falls to 8 / k of
// the XCDs only, k the common factor of 8 and the number, some of which then get the
// empty ones (2048 (b, h), N 128, 2 splits of 255 memories at most: 808 us, 706 so;
// 240, 8 of 64: 73 and 53).  Odd numbers deal every split over all of them (13
// splits, 384 (b, h) of fp32, N 64: 127 us, 137 with (b, h) fastest), and with few
// blocks the last splits, together and mostly empty, would leave the full ones in
// front to one round of the chip (32 (b, h) of fp32, N 128, 10 splits: 19.9 and
// 31.0).  Over 526 shapes, bf16 and fp32, N 64 and 128, 8 to 960 (b, h), the
// line lies at CUs / k (b, h): 0.90 to 1.00 of the time below it, up
// to 1.75 times past it.
inline bool stream_bh_fastest(int64_t bh, int ns) {
    const int k = ns % 8 == 0 ? 8 : ns % 4 == 0 ? 4 : ns % 2 == 0 ? 2 : 1;
    return k > 1 && bh * k > device_cu_count();
}

// Number of splits of a step that attends m memories.
inline int decode_splits(const Shape& s, int64_t m) {
    if (m <= 0) return 0;
    const int mps = decode_mps(s.B * s.H, m);
    return (int)((m + mps - 1) / mps);
}

// nsplit_stride: the partials' split stride in the workspace (0: the
// workspace's worst case over positions that fit the cache).
template <typename T, int N>
hipError_t run_decode(const Shape& s, const SmaArgs& a, int64_t pos, const int64_t* pos_rows,
                      const void* x, const float* dt, const float* A, const void* Bm,
                      const void* Cm, const void* q, const void* e, const void* z, float* h_state,
                      float* chunk_acc, void* mem, void* y, void* ws, int nsplit_stride,
                      hipStream_t st) {
    // ragged batches size the grid for the largest position (pos = pos_lim)
    const int64_t m = pos / s.S;
    if (decode_in_one<T, N>(s.B * s.H, m)) {
        prof_begin("k_decode_one", st);
        k_decode_one<T, N><<<dim3((unsigned)s.H, (unsigned)s.B), 64 * kOneWaves, 0, st>>>(
            (const T*)x, dt, A, (const T*)Bm, h_state, chunk_acc, (T*)mem, (const T*)q, (const T*)e,
            (const T*)Cm, (const T*)z, (T*)y, a.qw, a.ew, a.eps, a.normalize, s.H, s.G, s.S, s.Mcap, pos,
            pos_rows, pos, a.z_per_head);
        prof_end(st);
        return hipGetLastError();
    }
    const int mps = decode_mps(s.B * s.H, m);
    const int nsplit_cap =
        nsplit_stride > 0 ? nsplit_stride : (int)((s.Mcap + kMinMPS - 1) / kMinMPS);
    float* part = reinterpret_cast<float*>(ws);
    float* yssd = part + decode_part_floats(s.B, s.H, nsplit_cap);
    const int ns = m > 0 ? (int)((m + mps - 1) / mps) : 0;
    const int64_t BH = s.B * s.H;
    const bool apart = state_apart<T, N>(BH, m);
    auto stream = [&](auto state) {
        constexpr bool STATE = decltype(state)::value;
        prof_begin("k_decode_partial", st);
        k_decode_partial<T, N, STATE><<<flat_grid(BH * (STATE ? ns + 1 : ns), kThreads), kThreads, 0, st>>>(
            (const T*)x, dt, A, (const T*)Bm, h_state, chunk_acc, (T*)mem, yssd, (const T*)q, (const T*)e,
            (const T*)Cm, a.qw, a.ew, part, a.eps, a.normalize, s.H, s.G, s.S, s.Mcap, pos, pos_rows, pos,
            nsplit_cap, mps, ns, BH, pos_rows && stream_bh_fastest(BH, ns));
        prof_end(st);
    };
    if (!apart) stream(std::true_type()); else if (m > 0) stream(std::false_type());
    if (apart) {
        prof_begin("k_decode_state_merge", st);
        k_decode_state_merge<T, N><<<dim3((unsigned)s.H, (unsigned)s.B), kThreads, 0, st>>>(
            (const T*)x, dt, A, (const T*)Bm, (const T*)Cm, (const T*)z, h_state, chunk_acc, (T*)mem, (T*)y,
            part, s.H, s.G, s.S, s.Mcap, pos, pos_rows, pos, nsplit_cap, a.z_per_head, mps);
    } else {
        prof_begin("k_decode_merge", st);
        k_decode_merge<T><<<(unsigned)((BH + 3) / 4), kThreads, 0, st>>>(
            (const T*)z, (T*)y, part, yssd, s.H, s.S, pos, pos_rows, pos, nsplit_cap, a.z_per_head, mps, BH);
    }
    prof_end(st);
    return hipGetLastError();
}

template <typename T>
hipError_t run_decode_n(const Shape& s, const SmaArgs& a, int64_t pos, const int64_t* pr,
                        const void* x, const float* dt, const float* A, const void* Bm,
                        const void* Cm, const void* q, const void* e, const void* z, float* hs,
                        float* ca, void* mem, void* y, void* ws, int nss, hipStream_t st) {
    switch (s.N) {
        case 16: return run_decode<T, 16>(s, a, pos, pr, x, dt, A, Bm, Cm, q, e, z, hs, ca, mem, y, ws, nss, st);
        case 32: return run_decode<T, 32>(s, a, pos, pr, x, dt, A, Bm, Cm, q, e, z, hs, ca, mem, y, ws, nss, st);
        case 64: return run_decode<T, 64>(s, a, pos, pr, x, dt, A, Bm, Cm, q, e, z, hs, ca, mem, y, ws, nss, st);
        case 128: return run_decode<T, 128>(s, a, pos, pr, x, dt, A, Bm, Cm, q, e, z, hs, ca, mem, y, ws, nss, st);
    }
    return hipErrorInvalidValue;
}

// Fixed device scratch of the allocation-free decode step: the partials
// [B][H][nsplit][P+2] of that step's own split count and y_ssd [B][H][P]
// (float).  Each device holds its own copy; host code reaches it only through
// the address hipGetSymbolAddress returns on that device.
static __device__ __align__(256) char scratch[DART_DECODE_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// The current device's scratch address, looked up once per device (with that
// device current) and kept.
hipError_t scratch_address(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

// Prefill -> decode handoff for row b of length L_b (lengths[b]; rows with
// L_b < 0 are left untouched): h_state = h_last and chunk_acc = the running
// contribution of the partial chunk floor(L_b/S), which the forward scan left
// in mem slot floor(L_b/S) (0 when L_b is a multiple of S: the next token
// opens a chunk).
template <typename T, int N>
__global__ __launch_bounds__(kThreads) void k_decode_handoff(const T* __restrict__ mem,
                                                             const float* __restrict__ h_last,
                                                             const int64_t* __restrict__ lengths,
                                                             float* __restrict__ h_state,
                                                             float* __restrict__ chunk_acc, int H,
                                                             int S, int64_t Mcap) {
    const int h = blockIdx.x;
    const int64_t b = blockIdx.y;
    const int64_t len = lengths[b];
    if (len < 0) return;
    const int64_t mi = len / S;
    const bool partial = (len % S) != 0 && mi < Mcap;
    const int64_t base = (b * H + h) * (int64_t)N * kP;
    const T* src = mem + ((b * Mcap + (partial ? mi : 0)) * H + h) * (int64_t)N * kP;
    for (int e0 = threadIdx.x * 4; e0 < N * kP; e0 += kThreads * 4) {
        float v[4];
        load4(h_last + base + e0, v);
        store4(h_state + base + e0, v);
        if (partial) {
            load4(src + e0, v);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = 0.f;
        }
        store4(chunk_acc + base + e0, v);
    }
}

template <typename T>
hipError_t run_handoff_n(const Shape& s, const void* mem, const float* h_last,
                         const int64_t* lengths, float* h_state, float* chunk_acc, hipStream_t st) {
    const dim3 grid((unsigned)s.H, (unsigned)s.B);
    prof_begin("k_decode_handoff", st);
    switch (s.N) {
        case 16: k_decode_handoff<T, 16><<<grid, kThreads, 0, st>>>((const T*)mem, h_last, lengths, h_state, chunk_acc, s.H, s.S, s.Mcap); break;
        case 32: k_decode_handoff<T, 32><<<grid, kThreads, 0, st>>>((const T*)mem, h_last, lengths, h_state, chunk_acc, s.H, s.S, s.Mcap); break;
        case 64: k_decode_handoff<T, 64><<<grid, kThreads, 0, st>>>((const T*)mem, h_last, lengths, h_state, chunk_acc, s.H, s.S, s.Mcap); break;
        case 128: k_decode_handoff<T, 128><<<grid, kThreads, 0, st>>>((const T*)mem, h_last, lengths, h_state, chunk_acc, s.H, s.S, s.Mcap); break;
        default: prof_end(st); return hipErrorInvalidValue;
    }
    prof_end(st);
    return hipGetLastError();
}

}  // namespace

size_t decode_workspace_bytes(const Shape& s) {
    const int64_t nsplit = (s.Mcap + kMinMPS - 1) / kMinMPS;
    return align256(sizeof(float) * (decode_part_floats(s.B, s.H, (int)(nsplit > 0 ? nsplit : 1)) +
                                     (size_t)s.B * s.H * s.P));
}

hipError_t launch_decode(const Shape& s, const SmaArgs& a, int64_t pos, const int64_t* pos_rows,
                         const void* x, const float* dt, const float* A, const void* Bm,
                         const void* Cm, const void* q, const void* e, const void* z,
                         float* h_state, float* chunk_acc, void* mem, void* y, void* ws,
                         hipStream_t st) {
    if (s.dtype == 1)
        return run_decode_n<bf16>(s, a, pos, pos_rows, x, dt, A, Bm, Cm, q, e, z, h_state, chunk_acc,
                                  mem, y, ws, 0, st);
    return run_decode_n<float>(s, a, pos, pos_rows, x, dt, A, Bm, Cm, q, e, z, h_state, chunk_acc, mem,
                               y, ws, 0, st);
}

size_t decode_noalloc_scratch_bytes(const Shape& s, int64_t pos) {
    const int ns = decode_splits(s, pos / s.S);
    return sizeof(float) * (decode_part_floats(s.B, s.H, ns > 0 ? ns : 1) + (size_t)s.B * s.H * s.P);
}

hipError_t launch_decode_noalloc(const Shape& s, const SmaArgs& a, int64_t pos, const void* x,
                                 const float* dt, const float* A, const void* Bm, const void* Cm,
                                 const void* q, const void* e, const void* z, float* h_state,
                                 float* chunk_acc, void* mem, void* y, hipStream_t st) {
    void* ws = nullptr;
    const hipError_t err = scratch_address(&ws);
    if (err != hipSuccess) return err;
    const int ns = decode_splits(s, pos / s.S);
    const int nss = ns > 0 ? ns : 1;
    if (s.dtype == 1)
        return run_decode_n<bf16>(s, a, pos, nullptr, x, dt, A, Bm, Cm, q, e, z, h_state, chunk_acc,
                                  mem, y, ws, nss, st);
    return run_decode_n<float>(s, a, pos, nullptr, x, dt, A, Bm, Cm, q, e, z, h_state, chunk_acc, mem,
                               y, ws, nss, st);
}

hipError_t launch_decode_handoff(const Shape& s, const void* mem, const float* h_last,
                                 const int64_t* lengths, float* h_state, float* chunk_acc,
                                 hipStream_t st) {
    if (s.dtype == 1) return run_handoff_n<bf16>(s, mem, h_last, lengths, h_state, chunk_acc, st);
    return run_handoff_n<float>(s, mem, h_last, lengths, h_state, chunk_acc, st);
}

}  // namespace dart
