// block.hip -- the steps either side of the path in a DART (Mamba-2) block:
// the causal width-4 convolution with SiLU over the x, B, C channels of the
// input projection (and its carried state, the decode cache of the
// convolution), the step sizes dt = softplus(raw + bias), and the gated
// RMSNorm ahead of the output projection.  The paper fixes the convolution
// width (4) and RMSNorm (App. D.2, the text after Table 8); the rest follows
// the Mamba-2 block it builds on.  All three are elementwise or row-local and
// bound by HBM: every input element is read once, every output written once.
#include "dart_common.hpp"
#include "dart_internal.hpp"

namespace dart {
namespace {

constexpr int kConvTok = 64;  // tokens per thread of the scalar convolution
constexpr int kConvTok4 = 32; // tokens per thread of the 4-channel convolution
constexpr int kConvU = 4;     // rows of a batch of its loads and of its backward's

template <typename T> using Vec4 = T __attribute__((ext_vector_type(4)));

// SiLU through the hardware reciprocal (about 1 ulp) instead of an IEEE
// division: these kernels evaluate it once per element they stream.
__device__ __forceinline__ float silu_rcp(float v) {
    return v * __builtin_amdgcn_rcpf(1.0f + __expf(-v));
}

// One thread per (channel, run of kConvTok tokens): the last three inputs
// live in registers, so each input element is loaded once; consecutive
// threads take consecutive channels (coalesced rows).
template <typename T>
__global__ __launch_bounds__(256) void k_conv1d_silu(const T* __restrict__ in, int64_t stride,
                                                     const float* __restrict__ w,
                                                     const float* __restrict__ bias,
                                                     const float* __restrict__ st_in,
                                                     float* __restrict__ st_out,
                                                     T* __restrict__ out, int64_t L, int C) {
    const int c = blockIdx.x * 256 + threadIdx.x;
    const int64_t t0 = (int64_t)blockIdx.y * kConvTok;
    const int64_t b = blockIdx.z;
    if (c >= C) return;
    const float w0 = w[c * 4 + 0], w1 = w[c * 4 + 1], w2 = w[c * 4 + 2], w3 = w[c * 4 + 3];
    const float bc = bias ? bias[c] : 0.f;
    const T* src = in + (b * L) * stride + c;
    // inputs t0 - 3 .. t0 - 1 (carried state before token 0)
    float win[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int64_t s = t0 - 3 + i;
        win[i] = s >= 0 ? to_f(src[s * stride]) : (st_in ? st_in[(b * C + c) * 3 + (3 + s)] : 0.f);
    }
    const int64_t t1 = t0 + kConvTok < L ? t0 + kConvTok : L;
    T* dst = out + (b * L) * C + c;
    for (int64_t t = t0; t < t1; ++t) {
        const float v = to_f(src[t * stride]);
        const float a = bc + w0 * win[0] + w1 * win[1] + w2 * win[2] + w3 * v;
        dst[t * C] = from_f<T>(silu_rcp(a));
        win[0] = win[1];
        win[1] = win[2];
        win[2] = v;
    }
    if (st_out && t1 == L) {
        // the last three inputs, oldest first
#pragma unroll
        for (int i = 0; i < 3; ++i) st_out[(b * C + c) * 3 + i] = win[i];
    }
}

// The same convolution with 4 consecutive channels per thread (8-byte rows
// of bf16, 16 of fp32): used when C, the row stride and the pointers are
// multiples of 4 elements.  HBM-bound.  A wave's memory operations complete in
// order, so a load issued behind a store waits for it: the next kConvU rows are
// requested ahead of the current ones' stores, the rows before the run and the
// first batch together (32768 tokens of 1792 bf16 channels, 235 MB, before the
// backward: 57 us with 8 channels per thread, its loads behind the stores and up to three
// exposed latencies before the first token; 48 us, 4.9 TB/s.  8 channels per
// thread in this form spill).
template <typename T>
__global__ __launch_bounds__(64) void k_conv1d_silu_v4(const T* __restrict__ in, int64_t stride,
                                                        const float* __restrict__ w,
                                                        const float* __restrict__ bias,
                                                        const float* __restrict__ st_in,
                                                        float* __restrict__ st_out,
                                                        T* __restrict__ out, int64_t L, int C) {
    const unsigned c0 = (blockIdx.x * 64 + threadIdx.x) * 4;
    const int64_t t0 = (int64_t)blockIdx.y * kConvTok4;
    const int64_t b = blockIdx.z;
    if (c0 >= (unsigned)C) return;
    const T* src = in + (b * L) * stride;  // (uniform; c0 is the lane's offset)
    const int64_t t1 = t0 + kConvTok4 < L ? t0 + kConvTok4 : L;
    T* dst = out + (b * L) * C;
    // kConvU rows ahead of the stores of the rows before them; past the end the
    // last row is read and not used
    auto load = [&](int64_t t, Vec4<T>(&f)[kConvU]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kConvU; ++u)
            f[u] = *reinterpret_cast<const Vec4<T>*>(src + (t + u < t1 ? t + u : t1 - 1) * stride + c0);
        __builtin_amdgcn_sched_barrier(0);
    };
    Vec4<T> hr[3], f0[kConvU], f1[kConvU];
#pragma unroll
    for (int k = 0; k < 3; ++k)
        hr[k] = *reinterpret_cast<const Vec4<T>*>(src + (t0 > 0 ? t0 - 3 + k : 0) * stride + c0);
    int64_t t = t0;
    load(t, f0);
    float wk[4][4], bc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) load4(w + (c0 + i) * 4, wk[i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) bc[i] = 0.f;
    if (bias) {
#pragma unroll
        for (int i = 0; i < 4; ++i) bc[i] = bias[c0 + i];
    }
    // the three tokens before the run (the carried state before token 0)
    float win[3][4];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) win[k][i] = t0 > 0 ? (float)hr[k][i] : 0.f;
    if (t0 == 0 && st_in) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k) win[k][i] = st_in[(b * C + c0 + i) * 3 + k];
    }
    auto run = [&](int64_t t, const Vec4<T>(&f)[kConvU], bool all) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kConvU; ++u) {
            if (!all && t + u >= t1) break;
            float o[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float v = (float)f[u][i];
                const float a = bc[i] + wk[i][0] * win[0][i] + wk[i][1] * win[1][i] +
                                wk[i][2] * win[2][i] + wk[i][3] * v;
                o[i] = silu_rcp(a);
                win[0][i] = win[1][i];
                win[1][i] = win[2][i];
                win[2][i] = v;
            }
            store4(dst + (t + u) * C + c0, o);
        }
    };
    for (; t + 2 * kConvU <= t1; t += 2 * kConvU) {
        load(t + kConvU, f1);
        run(t, f0, true);
        load(t + 2 * kConvU, f0);
        run(t + kConvU, f1, true);
    }
    if (t < t1) {
        if (t + kConvU < t1) load(t + kConvU, f1);
        run(t, f0, false);
        if (t + kConvU < t1) run(t + kConvU, f1, false);
    }
    if (st_out && t1 == L) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k) st_out[(b * C + c0 + i) * 3 + k] = win[k][i];
    }
}

template <typename T>
__global__ __launch_bounds__(256) void k_dt_softplus(const T* __restrict__ raw, int64_t stride,
                                                     const float* __restrict__ bias,
                                                     float* __restrict__ dt, int64_t rows, int H) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= rows * H) return;
    const int64_t r = i / H;
    const int h = (int)(i - r * H);
    const float v = to_f(raw[r * stride + h]) + (bias ? bias[h] : 0.f);
    // softplus, log1p(exp(v)) without overflow
    dt[i] = v > 20.f ? v + log1pf(__expf(-v)) : log1pf(__expf(v));
}

// One wave per (row, group): u = y SiLU(z), out = u rsqrt(mean(u^2) + eps) w.
// Lanes take 8 consecutive channels at a time (group and the row strides are
// multiples of 8); the group sum is a wave reduction in a fixed order.
template <typename T>
__global__ __launch_bounds__(256) void k_gated_rmsnorm(const T* __restrict__ y,
                                                       const T* __restrict__ z, int64_t zstride,
                                                       const float* __restrict__ w, float eps,
                                                       T* __restrict__ out, int64_t rows, int D,
                                                       int group) {
    const int lane = threadIdx.x & 63;
    const int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int ngr = D / group;
    if (item >= rows * ngr) return;
    const int64_t r = item / ngr;
    const int g0 = (int)(item - r * ngr) * group;
    const T* yr = y + r * D + g0;
    const T* zr = z + r * zstride + g0;
    T* orow = out + r * D + g0;
    // groups of up to 2048 channels stay in registers between the two
    // passes (four pieces of 8 per lane); longer groups read y and z again
    constexpr int KEEP = 4;
    float u[KEEP][8], wv[KEEP][8];
    float ss = 0.f;
#pragma unroll
    for (int q = 0; q < KEEP; ++q) {
        const int k = lane * 8 + q * 512;
        if (k < group) {
            float yv[8], zv[8];
            load8_nt(yr + k, yv);
            load8_nt(zr + k, zv);
            // the weights of these channels, loaded with the data (vector
            // loads; 8 consecutive floats at a multiple of 8)
            if (w) {
                load8(w + g0 + k, wv[q]);
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) wv[q][i] = 1.f;
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                u[q][i] = yv[i] * silu_rcp(zv[i]);
                ss += u[q][i] * u[q][i];
            }
        }
    }
    for (int k = lane * 8 + KEEP * 512; k < group; k += 512) {
        float yv[8], zv[8];
        load8(yr + k, yv);
        load8(zr + k, zv);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float uu = yv[i] * silu_rcp(zv[i]);
            ss += uu * uu;
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) ss += __shfl_xor(ss, o, 64);
    const float inv = 1.0f / sqrtf(ss / group + eps);
#pragma unroll
    for (int q = 0; q < KEEP; ++q) {
        const int k = lane * 8 + q * 512;
        if (k < group) {
            float o[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) o[i] = u[q][i] * inv * wv[q][i];
            store8_nt(orow + k, o);
        }
    }
    for (int k = lane * 8 + KEEP * 512; k < group; k += 512) {
        float yv[8], zv[8], o[8];
        load8(yr + k, yv);
        load8(zr + k, zv);
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = yv[i] * silu_rcp(zv[i]) * inv * (w ? w[g0 + k + i] : 1.f);
        store8(orow + k, o);
    }
}

// ---- backward of the block kernels ------------------------------------------------
// Gradients for a loss whose gradient with respect to each kernel's output is
// `dout` (float).  Sums over tokens or rows (weights, biases) go to per-block
// partials in the workspace and a second kernel adds them in a fixed order.

__device__ __forceinline__ float silu_grad_f(float u) {
    const float sg = 1.0f / (1.0f + __expf(-u));
    return sg * (1.0f + u * (1.0f - sg));
}

constexpr int kConvBwdTok = 32;  // tokens per thread of the convolution backward

// One thread per (channel, run of kConvBwdTok tokens, batch row).  With
// u_t = bias + sum_k w_k in[t-3+k] and du_t = dout_t SiLU'(u_t):
//   din[s] = w3 du_s + w2 du_{s+1} + w1 du_{s+2} + w0 du_{s+3},
//   dw_k = sum_t du_t in[t-3+k],  dbias = sum_t du_t,
//   dstate[j] (input -3+j) = sum_{t <= j} du_t w_{j-t}.
// A run computes du for its own tokens and the three after it, so din of its
// tokens is complete; the weight sums cover its own tokens only.
template <typename T>
__global__ __launch_bounds__(256) void k_conv1d_silu_bwd(
    const T* __restrict__ in, int64_t stride, const float* __restrict__ w,
    const float* __restrict__ bias, const float* __restrict__ st_in,
    const float* __restrict__ dout, float* __restrict__ din, int64_t dstride,
    float* __restrict__ dst_in, float* __restrict__ part, int64_t L, int C, int nruns) {
    const int c = blockIdx.x * 256 + threadIdx.x;
    const int run = blockIdx.y;
    const int64_t b = blockIdx.z;
    if (c >= C) return;
    const int64_t t0 = (int64_t)run * kConvBwdTok;
    const int64_t t1 = t0 + kConvBwdTok < L ? t0 + kConvBwdTok : L;
    const int64_t tend = t1 + 3 < L ? t1 + 3 : L;
    const float w0 = w[c * 4 + 0], w1 = w[c * 4 + 1], w2 = w[c * 4 + 2], w3 = w[c * 4 + 3];
    const float bc = bias ? bias[c] : 0.f;
    const T* src = in + (b * L) * stride + c;
    const float* dsrc = dout + (b * L) * C + c;
    float* dd = din + (b * L) * dstride + c;
    float win[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int64_t s = t0 - 3 + i;
        win[i] = s >= 0 ? to_f(src[s * stride]) : (st_in ? st_in[(b * C + c) * 3 + (3 + s)] : 0.f);
    }
    float q0 = 0.f, q1 = 0.f, q2 = 0.f, q3 = 0.f;  // du at t-3 .. t
    float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f, ab = 0.f;
    float d0 = 0.f, d1 = 0.f, d2 = 0.f;  // du at t0, t0+1, t0+2
    for (int64_t t = t0; t < tend; ++t) {
        const float v = to_f(src[t * stride]);
        const float u = bc + w0 * win[0] + w1 * win[1] + w2 * win[2] + w3 * v;
        const float du = dsrc[t * C] * silu_grad_f(u);
        if (t < t1) {
            a0 += du * win[0];
            a1 += du * win[1];
            a2 += du * win[2];
            a3 += du * v;
            ab += du;
        }
        if (t == t0) d0 = du;
        if (t == t0 + 1) d1 = du;
        if (t == t0 + 2) d2 = du;
        q0 = q1;
        q1 = q2;
        q2 = q3;
        q3 = du;
        if (t - 3 >= t0) dd[(t - 3) * dstride] = w3 * q0 + w2 * q1 + w1 * q2 + w0 * q3;
        win[0] = win[1];
        win[1] = win[2];
        win[2] = v;
    }
    // tokens whose later inputs end at L (du beyond L is zero); q3 = du at
    // tend - 1 and so on
    for (int64_t s = (tend - 3 > t0 ? tend - 3 : t0); s < t1; ++s) {
        const int64_t k = tend - s;  // 3, 2 or 1 tokens from s to the end
        float v = 0.f;
        if (k == 3) v = w3 * q1 + w2 * q2 + w1 * q3;
        if (k == 2) v = w3 * q2 + w2 * q3;
        if (k == 1) v = w3 * q3;
        dd[s * dstride] = v;
    }
    if (dst_in && t0 == 0) {
        dst_in[(b * C + c) * 3 + 0] = d0 * w0;
        dst_in[(b * C + c) * 3 + 1] = d0 * w1 + d1 * w0;
        dst_in[(b * C + c) * 3 + 2] = d0 * w2 + d1 * w1 + d2 * w0;
    }
    float* pr = part + ((b * nruns + run) * (int64_t)C + c) * 5;
    pr[0] = a0;
    pr[1] = a1;
    pr[2] = a2;
    pr[3] = a3;
    pr[4] = ab;
}

// The same for four consecutive channels per thread (8-byte rows of bf16, 16
// of fp32, 16-byte gradients): used when the channel count, the row strides
// and the pointers are multiples of 4 elements.  HBM-bound, every input read
// once plus three tokens of overlap per run; loads ahead of the stores as in the
// forward.  587 MB at 32768 tokens of 1792 bf16 channels: 167 us with the loads
// behind the stores, 152 so (kernel trace of a layer's calls; one channel per
// thread and 2-byte loads took a tenth longer than the former, runs of 16 tokens
// 5 % longer, of 64 the same).  The block of a 130M-parameter model's layer, with
// the forward above: 465 -> 442 us; 453 with this kernel held to 168
// registers, 445 with batches of two tokens.
template <typename T>
__global__ __launch_bounds__(64) void k_conv1d_silu_bwd_v4(
    const T* __restrict__ in, int64_t stride, const float* __restrict__ w,
    const float* __restrict__ bias, const float* __restrict__ st_in,
    const float* __restrict__ dout, float* __restrict__ din, int64_t dstride,
    float* __restrict__ dst_in, float* __restrict__ part, int64_t L, int C, int nruns) {
    const unsigned c0 = (blockIdx.x * 64 + threadIdx.x) * 4;
    const int run = blockIdx.y;
    const int64_t b = blockIdx.z;
    if (c0 >= (unsigned)C) return;
    const int64_t t0 = (int64_t)run * kConvBwdTok;
    const int64_t t1 = t0 + kConvBwdTok < L ? t0 + kConvBwdTok : L;
    const T* src = in + (b * L) * stride;  // (uniform; c0 is the lane's offset)
    const float* dsrc = dout + (b * L) * C;
    float* dd = din + (b * L) * dstride;
    float q[3][4];  // du at t-3, t-2, t-1 (zero before t0)
    float acc[4][5];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        q[0][i] = q[1][i] = q[2][i] = 0.f;
#pragma unroll
        for (int k = 0; k < 5; ++k) acc[i][k] = 0.f;
    }
    const int64_t n = t1 - t0;
    struct Rows {
        Vec4<T> v[kConvU];
        f32x4 d[kConvU];
    };
    // tokens t0 + k .. of `in` and `dout`, ahead of the stores of the tokens
    // before them; past the sequence's end the last row is read and not used
    auto load = [&](int64_t k, Rows& f) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kConvU; ++u) {
            const int64_t t = t0 + k + u < L ? t0 + k + u : L - 1;
            f.v[u] = *reinterpret_cast<const Vec4<T>*>(src + t * stride + c0);
            f.d[u] = *reinterpret_cast<const f32x4*>(dsrc + t * C + c0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    Vec4<T> hr[3];
    Rows f0, f1;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        hr[k] = *reinterpret_cast<const Vec4<T>*>(src + (t0 > 0 ? t0 - 3 + k : 0) * stride + c0);
    load(0, f0);
    load(kConvU, f1);
    float wk[4][4], bc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        load4(w + (c0 + i) * 4, wk[i]);
        bc[i] = 0.f;
    }
    if (bias) {
#pragma unroll
        for (int i = 0; i < 4; ++i) bc[i] = bias[c0 + i];
    }
    // the three tokens before the run (the carried state before token 0)
    float win[3][4];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) win[k][i] = t0 > 0 ? (float)hr[k][i] : 0.f;
    if (t0 == 0 && st_in) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k) win[k][i] = st_in[(b * C + c0 + i) * 3 + k];
    }
    // token t (own: t < t1; the three after it complete din of the last own
    // tokens; beyond L du is zero): du, the weight sums and din of token t - 3.
    // `all`: tokens of the run that follow its first three.
    auto step = [&](int64_t k, const Rows& f, bool all) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kConvU; ++u) {
            const int64_t t = t0 + k + u;
            const bool own = all || k + u < n, inside = all || t < L;
            float v[4], dv[4], o[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[i] = inside ? (float)f.v[u][i] : 0.f;
                dv[i] = inside ? f.d[u][i] : 0.f;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float uu = bc[i] + wk[i][0] * win[0][i] + wk[i][1] * win[1][i] + wk[i][2] * win[2][i] + wk[i][3] * v[i];
                // (past the end uu may overflow where no token's did, and 0 times the
                // NaN that makes of it is not 0)
                const float du = inside ? dv[i] * silu_grad_f(uu) : 0.f;
                if (own) {
                    acc[i][0] += du * win[0][i];
                    acc[i][1] += du * win[1][i];
                    acc[i][2] += du * win[2][i];
                    acc[i][3] += du * v[i];
                    acc[i][4] += du;
                }
                o[i] = wk[i][3] * q[0][i] + wk[i][2] * q[1][i] + wk[i][1] * q[2][i] + wk[i][0] * du;
                q[0][i] = q[1][i];
                q[1][i] = q[2][i];
                q[2][i] = du;
                win[0][i] = win[1][i];
                win[1][i] = win[2][i];
                win[2][i] = v[i];
            }
            if (all || (k + u >= 3 && k + u < n + 3)) store4(dd + (t - 3) * dstride + c0, o);
            if (!all && dst_in && t == 2) {
                // du of tokens 0, 1 and 2 stand in q
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float* ds = dst_in + (b * C + c0 + i) * 3;
                    ds[0] = q[0][i] * wk[i][0];
                    ds[1] = q[0][i] * wk[i][1] + q[1][i] * wk[i][0];
                    ds[2] = q[0][i] * wk[i][2] + q[1][i] * wk[i][1] + q[2][i] * wk[i][0];
                }
            }
        }
    };
    step(0, f0, false);
    int64_t k = kConvU;
    for (; k + 2 * kConvU <= n; k += 2 * kConvU) {
        load(k + kConvU, f0);
        step(k, f1, true);
        load(k + 2 * kConvU, f1);
        step(k + kConvU, f0, true);
    }
    for (; k < n + 3; k += 2 * kConvU) {
        load(k + kConvU, f0);
        step(k, f1, false);
        if (k + kConvU >= n + 3) break;
        load(k + 2 * kConvU, f1);
        step(k + kConvU, f0, false);
    }
    float* pr = part + ((b * nruns + run) * (int64_t)C + c0) * 5;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        float o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = acc[(4 * k + i) / 5][(4 * k + i) % 5];
        store4(pr + 4 * k, o);
    }
}

// Sum of nparts partial rows of K floats per item: out[i][k] = sum_p part[p][i][k].
// A block serves COLS columns with LANES waves' worth of threads each, which add
// every LANES-th row, and adds their sums in a fixed order.  The kernel is bound
// by the latency of its loads: one thread per column walking all rows serially
// took 274 us per call at 1024 rows of 8960 columns (35 blocks), 16 lanes 9 us.  One
// or two rows are added as they are, without the exchange (a norm backward of 8
// rows of 256 channels 6.4 -> 5.9 us; of four rows, 16 lanes are faster again).
constexpr int kSumLanes = 16, kSumFew = 2;  // lanes; rows that one lane takes
template <int LANES, int COLS>
__global__ __launch_bounds__(LANES * COLS) void k_sum_parts(const float* __restrict__ part,
                                                            int64_t nparts, int64_t width,
                                                            float* __restrict__ out, int K, int keep,
                                                            float* __restrict__ out2) {
    const int col = threadIdx.x % COLS, pl = threadIdx.x / COLS;
    const int64_t i = flat_block() * COLS + col;
    float s = 0.f;
    if (i < width) {
#pragma unroll 8
        for (int64_t p = pl; p < nparts; p += LANES) s += part[p * width + i];
    }
    if constexpr (LANES > 1) {
        __shared__ float s_sum[LANES][COLS];
        s_sum[pl][col] = s;
        __syncthreads();
        if (pl != 0) return;
#pragma unroll
        for (int k = 1; k < LANES; ++k) s += s_sum[k][col];
    }
    if (i >= width) return;
    // items of K values: the first `keep` go to out ([item][keep]), the rest
    // (at most one) to out2 ([item])
    const int64_t item = i / K;
    const int k = (int)(i - item * K);
    if (k < keep) {
        if (out) out[item * keep + k] = s;
    } else if (out2) {
        out2[item] = s;
    }
}
void sum_parts(const float* part, int64_t nparts, int64_t width, float* out, int K, int keep, float* out2,
               hipStream_t st) {
    prof_begin("k_sum_parts", st);
    if (nparts <= kSumFew)
        k_sum_parts<1, 256><<<flat_grid((width + 255) / 256, 256), 256, 0, st>>>(part, nparts, width, out, K, keep, out2);
    else
        k_sum_parts<kSumLanes, 64><<<flat_grid((width + 63) / 64, 64 * kSumLanes), 64 * kSumLanes, 0, st>>>(
            part, nparts, width, out, K, keep, out2);
    prof_end(st);
}

// dt = softplus(raw + bias): draw = ddt sigmoid(raw + bias), dbias = sum over
// rows.  A block serves kDtRows rows of up to 256 heads: its threads tile
// (rows at a time) x heads, so that few heads still fill the block, and each
// head's row sums meet in LDS in a fixed order, by halves.  Latency-bound: with one
// thread per head walking the 256 rows serially, 24 heads and 32768 rows took 118 us
// (24 of 256 threads active), this tiling 7 us; 4 heads and 4096 rows 46 and
// 5.2 (7.7 with the sums of the up to 256 row lanes added one by one).
constexpr int kDtRows = 256;
constexpr int kDtThreads = 1024;
template <typename T>
__global__ __launch_bounds__(kDtThreads) void k_dt_softplus_bwd(const T* __restrict__ raw, int64_t stride,
                                                         const float* __restrict__ bias,
                                                         const float* __restrict__ ddt,
                                                         float* __restrict__ draw,
                                                         int64_t dstride, float* __restrict__ part,
                                                         int64_t rows, int H) {
    __shared__ float s_acc[kDtThreads];
    const int64_t first = ((int64_t)blockIdx.z * gridDim.x + blockIdx.x) * 256;
    if (first >= H) return;
    const int h0 = (int)first;
    const int hc = H - h0 < 256 ? H - h0 : 256;  // heads of this block
    const int nrl = (int)blockDim.x / hc;        // rows at a time
    const int rl = threadIdx.x / hc, h = h0 + threadIdx.x % hc;
    const int64_t rb = blockIdx.y;
    const int64_t r0 = rb * kDtRows;
    const int64_t r1 = r0 + kDtRows < rows ? r0 + kDtRows : rows;
    float acc = 0.f;
    if (rl < nrl) {
        const float bh = bias ? bias[h] : 0.f;
#pragma unroll 4
        for (int64_t r = r0 + rl; r < r1; r += nrl) {
            const float v = to_f(raw[r * stride + h]) + bh;
            const float g = ddt[r * H + h] / (1.0f + __expf(-v));
            draw[r * dstride + h] = g;
            acc += g;
        }
    }
    s_acc[threadIdx.x] = acc;
    for (int n = r1 - r0 < nrl ? (int)(r1 - r0) : nrl; n > 1;) {
        const int half = (n + 1) / 2;
        __syncthreads();
        if (rl < n - half) s_acc[threadIdx.x] = acc += s_acc[threadIdx.x + half * hc];
        n = half;
    }
    if ((int)threadIdx.x < hc) part[rb * H + h] = acc;
}

// Gated RMSNorm backward, one block per (kNormRows rows, group), its four
// waves taking every fourth row; a row's channels of the group (at most 2048:
// KEEP pieces of 256, 4 channels per lane) stay in registers between the sums
// and the gradients, so every input is read once.
// With u = y SiLU(z), inv = (mean u^2 + eps)^-1/2, g = dout (.) w:
//   du = inv g - u inv^3 (g . u) / group,  dy = du SiLU(z),
//   dz = du y SiLU'(z),  dw += dout u inv (summed over the block's rows).
// HBM-bound: 805 MB at 32768 rows of 1536 bf16 channels take 160 us (5.0
// TB/s).  KEEP fits the group, so short groups keep more waves resident; 16 rows
// go to four waves, and a lane's stores are 16 bytes so that a wave's cover
// whole lines.  (One wave per 16 rows, reading the inputs twice: 229 us;
// 8 channels per lane, whose stores leave every other 16 bytes to the next
// instruction: 265 us; ordinary loads 172 us, nontemporal stores 187 us.)
constexpr int kNormRows = 16;
template <typename T, int KEEP>
__global__ __launch_bounds__(256) void k_gated_rmsnorm_bwd(
    const T* __restrict__ y, const T* __restrict__ z, int64_t zstride, const float* __restrict__ w,
    float eps, const float* __restrict__ dout, float* __restrict__ dy, float* __restrict__ dz,
    int64_t dzstride, float* __restrict__ part, int64_t rows, int D, int group) {
    __shared__ float s_w[3][KEEP * 256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int ngr = D / group;
    const int64_t blk = flat_block(), rb = blk / ngr;
    const int g0 = (int)(blk - rb * ngr) * group;
    if (rb * kNormRows >= rows) return;
    float wacc[KEEP][4], wv[KEEP][4];
#pragma unroll
    for (int q = 0; q < KEEP; ++q) {
        const int k = lane * 4 + q * 256;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            wacc[q][i] = 0.f;
            wv[q][i] = w && k < group ? w[g0 + k + i] : 1.f;
        }
    }
    const int64_t r1 = (rb + 1) * kNormRows < rows ? (rb + 1) * kNormRows : rows;
    for (int64_t r = rb * kNormRows + wave; r < r1; r += 4) {
        float yv[KEEP][4], zv[KEEP][4], dv[KEEP][4], ss = 0.f, gu = 0.f;
#pragma unroll
        for (int q = 0; q < KEEP; ++q) {
            const int k = lane * 4 + q * 256;
            if (k < group) {
                load4_nt(y + r * D + g0 + k, yv[q]);
                load4_nt(z + r * zstride + g0 + k, zv[q]);
                load4_nt(dout + r * D + g0 + k, dv[q]);
            }
        }
#pragma unroll
        for (int q = 0; q < KEEP; ++q) {
            if (lane * 4 + q * 256 < group) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float u = yv[q][i] * silu_rcp(zv[q][i]);
                    ss += u * u;
                    gu += dv[q][i] * wv[q][i] * u;
                }
            }
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            ss += __shfl_xor(ss, o, 64);
            gu += __shfl_xor(gu, o, 64);
        }
        const float inv = 1.0f / sqrtf(ss / group + eps);
        const float c3 = inv * inv * inv * gu / group;
#pragma unroll
        for (int q = 0; q < KEEP; ++q) {
            const int k = lane * 4 + q * 256;
            if (k < group) {
                float oy[4], oz[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float sz = silu_rcp(zv[q][i]);
                    const float u = yv[q][i] * sz;
                    const float du = inv * (dv[q][i] * wv[q][i]) - u * c3;
                    oy[i] = du * sz;
                    oz[i] = du * yv[q][i] * silu_grad_f(zv[q][i]);
                    wacc[q][i] += dv[q][i] * u * inv;
                }
                store4(dy + r * D + g0 + k, oy);
                store4(dz + r * dzstride + g0 + k, oz);
            }
        }
    }
    // the waves' weight sums, added in wave order (the first wave's alone of one row)
    const bool alone = r1 - rb * kNormRows == 1;
    if (!alone) {
#pragma unroll
        for (int q = 0; q < KEEP; ++q) {
            if (wave > 0) store4(&s_w[wave - 1][lane * 4 + q * 256], wacc[q]);
        }
        __syncthreads();
    }
    if (wave > 0) return;
#pragma unroll
    for (int q = 0; q < KEEP; ++q) {
        const int k = lane * 4 + q * 256;
        if (k < group) {
#pragma unroll
            for (int v = 0; v < 3; ++v) {
                if (alone) break;
                float o[4];
                load4(&s_w[v][k], o);
#pragma unroll
                for (int i = 0; i < 4; ++i) wacc[q][i] += o[i];
            }
            store4(part + rb * D + g0 + k, wacc[q]);
        }
    }
}

template <typename T>
void run_gated_rmsnorm_bwd(int64_t blocks, const T* y, const T* z, int64_t zstride, const float* w,
                           float eps, const float* dout, float* dy, float* dz, int64_t dzstride,
                           float* part, int64_t rows, int D, int group, hipStream_t st) {
#define DART_NB(K) \
    k_gated_rmsnorm_bwd<T, K><<<flat_grid(blocks, 256), 256, 0, st>>>(y, z, zstride, w, eps, dout, dy, dz, dzstride, part, rows, D, group)
    if (group <= 512) DART_NB(2);
    else if (group <= 1024) DART_NB(4);
    else if (group <= 1536) DART_NB(6);
    else DART_NB(8);
#undef DART_NB
}

}  // namespace

hipError_t launch_conv1d_silu(int dtype, int64_t B, int64_t L, int C, int64_t stride,
                              const void* in, const float* w, const float* bias,
                              const float* st_in, float* st_out, void* out, hipStream_t st) {
    const dim3 grid((unsigned)((C + 255) / 256), (unsigned)((L + kConvTok - 1) / kConvTok),
                    (unsigned)B);
    const size_t es = dtype == 1 ? 2 : 4;
    if (C % 4 == 0 && stride % 4 == 0 && (uintptr_t)in % (4 * es) == 0 &&
        (uintptr_t)out % (4 * es) == 0 && (uintptr_t)w % 16 == 0) {
        const dim3 g4((unsigned)((C / 4 + 63) / 64), (unsigned)((L + kConvTok4 - 1) / kConvTok4),
                      (unsigned)B);
        prof_begin("k_conv1d_silu", st);
        if (dtype == 1) {
            k_conv1d_silu_v4<bf16><<<g4, 64, 0, st>>>((const bf16*)in, stride, w, bias, st_in,
                                                      st_out, (bf16*)out, L, C);
        } else {
            k_conv1d_silu_v4<float><<<g4, 64, 0, st>>>((const float*)in, stride, w, bias, st_in,
                                                       st_out, (float*)out, L, C);
        }
        prof_end(st);
        return hipGetLastError();
    }
    prof_begin("k_conv1d_silu", st);
    if (dtype == 1) {
        k_conv1d_silu<bf16><<<grid, 256, 0, st>>>((const bf16*)in, stride, w, bias, st_in, st_out,
                                                  (bf16*)out, L, C);
    } else {
        k_conv1d_silu<float><<<grid, 256, 0, st>>>((const float*)in, stride, w, bias, st_in,
                                                   st_out, (float*)out, L, C);
    }
    prof_end(st);
    return hipGetLastError();
}

hipError_t launch_dt_softplus(int dtype, int64_t rows, int H, const void* raw, int64_t stride,
                              const float* bias, float* dt, hipStream_t st) {
    const unsigned blocks = (unsigned)((rows * H + 255) / 256);
    prof_begin("k_dt_softplus", st);
    if (dtype == 1) {
        k_dt_softplus<bf16><<<blocks, 256, 0, st>>>((const bf16*)raw, stride, bias, dt, rows, H);
    } else {
        k_dt_softplus<float><<<blocks, 256, 0, st>>>((const float*)raw, stride, bias, dt, rows, H);
    }
    prof_end(st);
    return hipGetLastError();
}

hipError_t launch_gated_rmsnorm(int dtype, int64_t rows, int D, int group, const void* y,
                                const void* z, int64_t zstride, const float* w, float eps,
                                void* out, hipStream_t st) {
    const int64_t items = rows * (D / group);
    const unsigned blocks = (unsigned)((items + 3) / 4);
    prof_begin("k_gated_rmsnorm", st);
    if (dtype == 1) {
        k_gated_rmsnorm<bf16><<<blocks, 256, 0, st>>>((const bf16*)y, (const bf16*)z, zstride, w,
                                                      eps, (bf16*)out, rows, D, group);
    } else {
        k_gated_rmsnorm<float><<<blocks, 256, 0, st>>>((const float*)y, (const float*)z, zstride,
                                                       w, eps, (float*)out, rows, D, group);
    }
    prof_end(st);
    return hipGetLastError();
}

size_t conv1d_silu_bwd_workspace_bytes(int64_t B, int64_t L, int C) {
    const int64_t nruns = (L + kConvBwdTok - 1) / kConvBwdTok;
    return align256(sizeof(float) * (size_t)B * nruns * C * 5);
}

hipError_t launch_conv1d_silu_bwd(int dtype, int64_t B, int64_t L, int C, int64_t stride,
                                  const void* in, const float* w, const float* bias,
                                  const float* st_in, const float* dout, float* din,
                                  int64_t dstride, float* dw, float* db, float* dst_in, void* ws,
                                  hipStream_t st) {
    const int nruns = (int)((L + kConvBwdTok - 1) / kConvBwdTok);
    float* part = reinterpret_cast<float*>(ws);
    const size_t es = dtype == 1 ? 2 : 4;
    const bool aligned4 = C % 4 == 0 && stride % 4 == 0 && dstride % 4 == 0 && (uintptr_t)in % (4 * es) == 0 &&
                    ((uintptr_t)w | (uintptr_t)dout | (uintptr_t)din | (uintptr_t)ws) % 16 == 0;
    const dim3 grid((unsigned)((C + 255) / 256), (unsigned)nruns, (unsigned)B);
    // below a wave of the four-channel form per CU, its fourfold work per thread is the
    // longer chain (1792 bf16 channels: 256 tokens, 56 waves, 16.6 us against 14.5 with
    // a channel per thread; 1024 tokens 18.3 and 16.4; 2048, 448 waves, 20.5 and 23.0)
    const bool v4 = aligned4 && (int64_t)grid.x * nruns * B > device_cu_count();
    prof_begin("k_conv1d_silu_bwd", st);
    if (dtype == 1 && v4) {
        k_conv1d_silu_bwd_v4<bf16><<<grid, 64, 0, st>>>((const bf16*)in, stride, w, bias, st_in, dout,
                                                        din, dstride, dst_in, part, L, C, nruns);
    } else if (v4) {
        k_conv1d_silu_bwd_v4<float><<<grid, 64, 0, st>>>((const float*)in, stride, w, bias, st_in, dout,
                                                         din, dstride, dst_in, part, L, C, nruns);
    } else if (dtype == 1) {
        k_conv1d_silu_bwd<bf16><<<grid, 256, 0, st>>>((const bf16*)in, stride, w, bias, st_in, dout,
                                                      din, dstride, dst_in, part, L, C, nruns);
    } else {
        k_conv1d_silu_bwd<float><<<grid, 256, 0, st>>>((const float*)in, stride, w, bias, st_in,
                                                       dout, din, dstride, dst_in, part, L, C, nruns);
    }
    prof_end(st);
    const int64_t width = (int64_t)C * 5;
    sum_parts(part, B * nruns, width, dw, 5, 4, db, st);
    return hipGetLastError();
}

size_t dt_softplus_bwd_workspace_bytes(int64_t rows, int H) {
    return align256(sizeof(float) * (size_t)((rows + kDtRows - 1) / kDtRows) * H);
}

hipError_t launch_dt_softplus_bwd(int dtype, int64_t rows, int H, const void* raw, int64_t stride,
                                  const float* bias, const float* ddt, float* draw,
                                  int64_t dstride, float* dbias, void* ws, hipStream_t st) {
    const int64_t nrb = (rows + kDtRows - 1) / kDtRows;
    float* part = reinterpret_cast<float*>(ws);
    const dim3 hg = flat_grid(((int64_t)H + 255) / 256, kDtThreads), grid(hg.x, (unsigned)nrb, hg.y);
    // no more threads than a block has (row, head) pairs, and at least a row of them
    const int64_t pairs = (rows < kDtRows ? rows : kDtRows) * (H < 256 ? H : 256);
    const unsigned threads = pairs < kDtThreads ? (unsigned)(pairs + 63) / 64 * 64 : kDtThreads;
    prof_begin("k_dt_softplus_bwd", st);
    if (dtype == 1) {
        k_dt_softplus_bwd<bf16><<<grid, threads, 0, st>>>((const bf16*)raw, stride, bias, ddt, draw,
                                                      dstride, part, rows, H);
    } else {
        k_dt_softplus_bwd<float><<<grid, threads, 0, st>>>((const float*)raw, stride, bias, ddt, draw,
                                                       dstride, part, rows, H);
    }
    prof_end(st);
    if (dbias) sum_parts(part, nrb, H, dbias, 1, 1, nullptr, st);
    return hipGetLastError();
}

size_t gated_rmsnorm_bwd_workspace_bytes(int64_t rows, int D) {
    return align256(sizeof(float) * (size_t)((rows + kNormRows - 1) / kNormRows) * D);
}

hipError_t launch_gated_rmsnorm_bwd(int dtype, int64_t rows, int D, int group, const void* y,
                                    const void* z, int64_t zstride, const float* w, float eps,
                                    const float* dout, float* dy, float* dz, int64_t dzstride,
                                    float* dw, void* ws, hipStream_t st) {
    const int64_t nrb = (rows + kNormRows - 1) / kNormRows;
    float* part = reinterpret_cast<float*>(ws);
    const int64_t blocks = nrb * (D / group);
    prof_begin("k_gated_rmsnorm_bwd", st);
    if (dtype == 1) {
        run_gated_rmsnorm_bwd((int64_t)blocks, (const bf16*)y, (const bf16*)z, zstride, w, eps, dout, dy,
                              dz, dzstride, part, rows, D, group, st);
    } else {
        run_gated_rmsnorm_bwd((int64_t)blocks, (const float*)y, (const float*)z, zstride, w, eps, dout,
                              dy, dz, dzstride, part, rows, D, group, st);
    }
    prof_end(st);
    if (dw) sum_parts(part, nrb, D, dw, 1, 1, nullptr, st);
    return hipGetLastError();
}

}  // namespace dart
