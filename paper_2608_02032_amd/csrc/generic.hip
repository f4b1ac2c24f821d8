// generic.hip -- the untuned path: every shape outside the tuned set
// (N in {32, 64, 128} with S in {64, 128, 256}), i.e. any chunk size S >= 1
// and N in {16, 32, 64, 128}, P = 64, both storage dtypes.  Plain fp32 VALU
// kernels, correct before fast; the tuned MFMA kernels serve the benchmark
// shapes.  The paper trains at S = 16, N in {16, 64} (MQAR, App. D.1) and
// evaluates one checkpoint at S = 64 and 32 (Sec. 5.2).
//
// Scan (Sec. 2 recurrence, Sec. 3 / App. A chunk memories), chunk-parallel
// with the recurrence itself inside each chunk:
//   k_gscan_chunk  per (b, c, h): run the chunk's tokens from a zero state;
//                  the state at the chunk's end is dH_[c] (App. A), kept in
//                  float and written to the memories in the storage dtype;
//                  the chunk's log decay sum_t dt_t A_h;
//   k_gscan_pass   per (b, h, 1024 state elements): H_[c] = e^{lda_c} H_[c-1]
//                  + dH_[c] over the chunks, in float; every chunk's entry
//                  state (float, and in the storage dtype for the backward)
//                  and h_last;
//   k_gscan_out    per (b, c, h): run the chunk's tokens again from its entry
//                  state, y_t = C_t H_t.
// (SMA at these shapes: sma_f32.hip.)
#include "dart_common.hpp"
#include "dart_internal.hpp"

namespace dart {
namespace {

constexpr int kP = 64;
constexpr int kGT = 256;  // threads per block

// Thread layout over an N x P state: row group rg = tid / 16 holds rows
// rg + 16 k (k < N / 16, so N >= 16), column quad pq = tid % 16 holds
// columns 4 pq .. 4 pq + 3.
template <int N>
struct StateLayout {
    static constexpr int RK = N / 16;
    static_assert(N % 16 == 0, "N must be a multiple of 16");
};

// ---- scan --------------------------------------------------------------------------
constexpr int kScanTok = 32;  // tokens staged per barrier in k_gscan_chunk

template <typename T, int N>
__global__ __launch_bounds__(kGT) void k_gscan_chunk(const T* __restrict__ x,
                                                     const float* __restrict__ dt,
                                                     const float* __restrict__ A,
                                                     const T* __restrict__ Bm, T* __restrict__ mem,
                                                     float* __restrict__ dh32,
                                                     float* __restrict__ lda, int64_t L, int H,
                                                     int G, int S, int64_t M, int64_t Mcap) {
    constexpr int RK = StateLayout<N>::RK;
    const int64_t c = blockIdx.x;
    const int h = blockIdx.y;
    const int64_t b = blockIdx.z;
    const int g = (int)((int64_t)h * G / H);
    const int tid = threadIdx.x, rg = tid >> 4, pq = tid & 15;
    const int64_t t0 = c * S;
    const int64_t t1 = t0 + S < L ? t0 + S : L;
    const float Ah = A[h];
    __shared__ float s_x[kScanTok][kP], s_B[kScanTok][N], s_d[kScanTok];
    float st[RK][4];
#pragma unroll
    for (int k = 0; k < RK; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) st[k][i] = 0.f;
    float la = 0.f;
    for (int64_t tb = t0; tb < t1; tb += kScanTok) {
        const int nt = (int)(t1 - tb < kScanTok ? t1 - tb : kScanTok);
        __syncthreads();
        for (int e = tid; e < nt * kP; e += kGT) {
            const int k = e / kP, p = e % kP;
            s_x[k][p] = to_f(x[((b * L + tb + k) * H + h) * kP + p]);
        }
        for (int e = tid; e < nt * N; e += kGT) {
            const int k = e / N, n = e % N;
            s_B[k][n] = to_f(Bm[((b * L + tb + k) * G + g) * N + n]);
        }
        if (tid < nt) s_d[tid] = dt[(b * L + tb + tid) * H + h];
        __syncthreads();
        for (int k = 0; k < nt; ++k) {
            const float d = s_d[k];
            const float a = __expf(d * Ah);
            la += d * Ah;
#pragma unroll
            for (int kk = 0; kk < RK; ++kk) {
                const float bn = d * s_B[k][rg + 16 * kk];
#pragma unroll
                for (int i = 0; i < 4; ++i) st[kk][i] = a * st[kk][i] + bn * s_x[k][4 * pq + i];
            }
        }
    }
    const int64_t ch = (b * M + c) * H + h;
#pragma unroll
    for (int k = 0; k < RK; ++k) {
        const int o = (rg + 16 * k) * kP + 4 * pq;
        store4(dh32 + ch * (int64_t)N * kP + o, st[k]);
        if (mem) store4(mem + ((b * Mcap + c) * H + h) * (int64_t)N * kP + o, st[k]);
    }
    if (tid == 0) lda[(b * H + h) * M + c] = la;
}

template <typename T>
__global__ __launch_bounds__(kGT) void k_gscan_pass(const float* __restrict__ dh32,
                                                    const float* __restrict__ lda,
                                                    const float* __restrict__ h0,
                                                    float* __restrict__ st32, T* __restrict__ states,
                                                    float* __restrict__ h_last, int H, int NP,
                                                    int64_t M) {
    const int h = blockIdx.y;
    const int64_t b = blockIdx.z;
    const int e0 = (blockIdx.x * kGT + threadIdx.x) * 4;
    if (e0 >= NP) return;
    float hc[4] = {0.f, 0.f, 0.f, 0.f};
    if (h0) load4(h0 + (b * H + h) * (int64_t)NP + e0, hc);
    for (int64_t c = 0; c < M; ++c) {
        const int64_t o = ((b * M + c) * H + h) * (int64_t)NP + e0;
        store4(st32 + o, hc);
        if (states) store4(states + o, hc);
        float d4[4];
        load4(dh32 + o, d4);
        const float a = __expf(lda[(b * H + h) * M + c]);
#pragma unroll
        for (int i = 0; i < 4; ++i) hc[i] = a * hc[i] + d4[i];
    }
    if (h_last) store4(h_last + (b * H + h) * (int64_t)NP + e0, hc);
}

template <typename T, int N>
__global__ __launch_bounds__(kGT) void k_gscan_out(const T* __restrict__ x,
                                                   const float* __restrict__ dt,
                                                   const float* __restrict__ A,
                                                   const T* __restrict__ Bm, const T* __restrict__ Cm,
                                                   const float* __restrict__ st32,
                                                   T* __restrict__ y, int64_t L, int H, int G, int S,
                                                   int64_t M) {
    constexpr int RK = StateLayout<N>::RK;
    const int64_t c = blockIdx.x;
    const int h = blockIdx.y;
    const int64_t b = blockIdx.z;
    const int g = (int)((int64_t)h * G / H);
    const int tid = threadIdx.x, rg = tid >> 4, pq = tid & 15;
    const int64_t t0 = c * S;
    const int64_t t1 = t0 + S < L ? t0 + S : L;
    const float Ah = A[h];
    __shared__ float s_x[2][kP], s_B[2][N], s_C[2][N];
    __shared__ float s_d[2];
    __shared__ float s_y[2][16][kP];
    float st[RK][4];
    const float* src = st32 + ((b * M + c) * H + h) * (int64_t)N * kP;
#pragma unroll
    for (int k = 0; k < RK; ++k) load4(src + (rg + 16 * k) * kP + 4 * pq, st[k]);
    // token t uses buffer (t - t0) & 1; one barrier per token orders both the
    // staged inputs and the partial sums of the previous token
    for (int64_t t = t0; t < t1; ++t) {
        const int bf = (int)((t - t0) & 1);
        if (tid < kP) s_x[bf][tid] = to_f(x[((b * L + t) * H + h) * kP + tid]);
        if (tid < N) {
            s_B[bf][tid] = to_f(Bm[((b * L + t) * G + g) * N + tid]);
            s_C[bf][tid] = to_f(Cm[((b * L + t) * G + g) * N + tid]);
        }
        if (tid == 0) s_d[bf] = dt[(b * L + t) * H + h];
        __syncthreads();
        if (t > t0 && tid < kP) {
            float ys = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) ys += s_y[bf ^ 1][r][tid];
            y[((b * L + (t - 1)) * H + h) * kP + tid] = from_f<T>(ys);
        }
        const float d = s_d[bf];
        const float a = __expf(d * Ah);
        float yp[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < RK; ++k) {
            const int n = rg + 16 * k;
            const float bn = d * s_B[bf][n], cn = s_C[bf][n];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                st[k][i] = a * st[k][i] + bn * s_x[bf][4 * pq + i];
                yp[i] += cn * st[k][i];
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) s_y[bf][rg][4 * pq + i] = yp[i];
        // the next token's barrier (or the one below) orders these writes
        // before their sum; the buffer is rewritten two tokens later, after
        // the reads of the next token's barrier interval
    }
    __syncthreads();
    if (t1 > t0 && tid < kP) {
        const int bf = (int)((t1 - 1 - t0) & 1);
        float ys = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) ys += s_y[bf][r][tid];
        y[((b * L + (t1 - 1)) * H + h) * kP + tid] = from_f<T>(ys);
    }
}

// ---- launchers -----------------------------------------------------------------------
template <typename T, int N>
hipError_t run_gscan(const Shape& s, const void* x, const float* dt, const float* A,
                     const void* Bm, const void* Cm, const float* h0, void* y, void* mem,
                     float* hl, const GenScanWs& w, hipStream_t st) {
    const dim3 grid((unsigned)s.M, (unsigned)s.H, (unsigned)s.B);
    prof_begin("k_gscan_chunk", st);
    k_gscan_chunk<T, N><<<grid, kGT, 0, st>>>((const T*)x, dt, A, (const T*)Bm, (T*)mem, w.dh32,
                                              w.lda, s.L, s.H, s.G, s.S, s.M, s.Mcap);
    prof_end(st);
    const int NP = N * kP;
    prof_begin("k_gscan_pass", st);
    k_gscan_pass<T><<<dim3((unsigned)((NP / 4 + kGT - 1) / kGT), (unsigned)s.H, (unsigned)s.B), kGT,
                      0, st>>>(w.dh32, w.lda, h0, w.st32, (T*)w.states, hl, s.H, NP, s.M);
    prof_end(st);
    prof_begin("k_gscan_out", st);
    k_gscan_out<T, N><<<grid, kGT, 0, st>>>((const T*)x, dt, A, (const T*)Bm, (const T*)Cm, w.st32,
                                            (T*)y, s.L, s.H, s.G, s.S, s.M);
    prof_end(st);
    return hipGetLastError();
}

template <typename T, int N>
hipError_t run_scan_states(const Shape& s, const void* x, const float* dt, const float* A,
                           const void* Bm, const float* h0, float* lda, float* dh32, float* st32,
                           hipStream_t st) {
    prof_begin("k_gscan_chunk", st);
    k_gscan_chunk<T, N><<<dim3((unsigned)s.M, (unsigned)s.H, (unsigned)s.B), kGT, 0, st>>>(
        (const T*)x, dt, A, (const T*)Bm, nullptr, dh32, lda, s.L, s.H, s.G, s.S, s.M, s.M);
    prof_end(st);
    const int NP = N * kP;
    prof_begin("k_gscan_pass", st);
    k_gscan_pass<T><<<dim3((unsigned)((NP / 4 + kGT - 1) / kGT), (unsigned)s.H, (unsigned)s.B), kGT,
                      0, st>>>(dh32, lda, h0, st32, nullptr, nullptr, s.H, NP, s.M);
    prof_end(st);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_scan_states_f32(const Shape& s, const void* x, const float* dt, const float* A,
                                  const void* Bm, const float* h0, float* lda, float* dh32,
                                  float* st32, hipStream_t st) {
#define DART_SS(T, NN) run_scan_states<T, NN>(s, x, dt, A, Bm, h0, lda, dh32, st32, st)
    if (s.dtype == 1) {
        switch (s.N) {
            case 16: return DART_SS(bf16, 16);
            case 32: return DART_SS(bf16, 32);
            case 64: return DART_SS(bf16, 64);
            case 128: return DART_SS(bf16, 128);
        }
    } else {
        switch (s.N) {
            case 16: return DART_SS(float, 16);
            case 32: return DART_SS(float, 32);
            case 64: return DART_SS(float, 64);
            case 128: return DART_SS(float, 128);
        }
    }
#undef DART_SS
    return hipErrorInvalidValue;
}

bool tuned_shape(const Shape& s) {
    return (s.N == 32 || s.N == 64 || s.N == 128) && (s.S == 64 || s.S == 128 || s.S == 256);
}

hipError_t launch_gscan(const Shape& s, const void* x, const float* dt, const float* A,
                        const void* Bm, const void* Cm, const float* h0, void* y_ssd, void* mem,
                        float* h_last, const GenScanWs& w, hipStream_t st) {
#define DART_GS(T, NN) run_gscan<T, NN>(s, x, dt, A, Bm, Cm, h0, y_ssd, mem, h_last, w, st)
    if (s.dtype == 1) {
        switch (s.N) {
            case 16: return DART_GS(bf16, 16);
            case 32: return DART_GS(bf16, 32);
            case 64: return DART_GS(bf16, 64);
            case 128: return DART_GS(bf16, 128);
        }
    } else {
        switch (s.N) {
            case 16: return DART_GS(float, 16);
            case 32: return DART_GS(float, 32);
            case 64: return DART_GS(float, 64);
            case 128: return DART_GS(float, 128);
        }
    }
#undef DART_GS
    return hipErrorInvalidValue;
}

}  // namespace dart
