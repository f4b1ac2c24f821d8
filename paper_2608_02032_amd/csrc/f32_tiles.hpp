// f32_tiles.hpp -- shared pieces of the kernels on the fp32 matrix instructions
// (sma_f32.hip, scan_f32.hip, scan_bwd.hip).
#pragma once

#include "dart_common.hpp"
#include "dart_internal.hpp"

namespace dart {

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 lds4(const char* p) { return *reinterpret_cast<const f32x4*>(p); }
// A tile's sum of 16 products (four steps), formed of two sums of 8: rounded at
// fewer of them than one chain, and the two overlap.
__device__ __forceinline__ f32x4 mfma16(const f32x4& a, const f32x4& b) {
    const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
    return mfma4(a[1], b[1], mfma4(a[0], b[0], zero)) + mfma4(a[3], b[3], mfma4(a[2], b[2], zero));
}

// The scan's pieces of a sequence: at most kQ tokens, nested with the memory
// chunks (a chunk of S >= kQ tokens is nq pieces, the last one shorter; for
// S < kQ a piece is Q / S whole chunks).
constexpr int kQ = 64;
struct Pieces {
    int64_t L, nk;
    int S, nq, Q;
};
inline Pieces pieces_of(const Shape& s) {
    Pieces p;
    p.L = s.L;
    p.S = s.S;
    if (s.S >= kQ) {
        p.nq = (s.S + kQ - 1) / kQ;
        p.Q = kQ;
        p.nk = (s.M - 1) * p.nq + (s.L - (s.M - 1) * s.S + kQ - 1) / kQ;
    } else {
        p.nq = 1;
        p.Q = kQ / s.S * s.S;
        p.nk = (s.L + p.Q - 1) / p.Q;
    }
    return p;
}
__device__ __forceinline__ void piece_range(const Pieces& p, int64_t k, int64_t& t0, int64_t& t1) {
    if (p.S >= kQ) {
        const int64_t c = k / p.nq, end = (c + 1) * p.S < p.L ? (c + 1) * p.S : p.L;
        t0 = c * p.S + (k - c * p.nq) * kQ;
        t1 = t0 + kQ < end ? t0 + kQ : end;
    } else {
        t0 = k * p.Q;
        t1 = t0 + p.Q < p.L ? t0 + p.Q : p.L;
    }
}

// v of the lane N to the left in the row of 16 lanes, zero in its first N lanes.
template <int N>
__device__ __forceinline__ double row_shr(double v) {
    const int2 u = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_update_dpp(0, u.x, 0x110 + N, 0xF, 0xF, true),
                                                __builtin_amdgcn_update_dpp(0, u.y, 0x110 + N, 0xF, 0xF, true)));
}
__device__ __forceinline__ double read_lane(double v, int lane) {
    const int2 u = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_readlane(u.x, lane), __builtin_amdgcn_readlane(u.y, lane)));
}

// The decays of one piece, lane = token: dt (0 past the piece's end), the
// inclusive cumulative log decay cl + lo inside its 16-token tile (log2 units), te
// the log decay from the token to its tile's end, and the four tiles' totals T.
// Formed in 64 bits: the decay between two tokens of a tile is the difference of
// two sums that may be far larger, and in 32 bits it keeps the rounding of those
// (dt A = -1.6 a token: 1e-6 of a decay that its own rounding puts at 1e-7);
// across tiles it is a sum of non-positive terms.
struct PieceDecay {
    float d, cl, lo, te;
    f32x4 T;
    __device__ __forceinline__ void load(const float* __restrict__ dt, float Ah, int64_t b, int64_t L, int H,
                                         int h, int64_t t0, int64_t t1, int lane) {
        d = t0 + lane < t1 ? dt[(b * L + t0 + lane) * H + h] : 0.f;
        // a decay below the float range is zero however far below, and without the
        // bound an infinite one would make a NaN of every difference over it
        double c = t0 + lane < t1 ? (double)d * (double)Ah * 1.4426950408889634 : 0.0;
        c = c < -160.0 ? -160.0 : c;
        c += row_shr<1>(c);
        c += row_shr<2>(c);
        c += row_shr<4>(c);
        c += row_shr<8>(c);
        cl = (float)c;
        lo = (float)(c - (double)cl);
        double own = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double t = read_lane(c, 16 * i + 15);
            T[i] = (float)t;
            own = lane >> 4 == i ? t : own;
        }
        te = (float)(own - c);
    }
};
// Sum of the tile totals between tiles a and b (exclusive).
__device__ __forceinline__ float tiles_between(const f32x4& T, int a, int b) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) s += i > a && i < b ? T[i] : 0.f;
    return s;
}
// Log decay from token t to token s >= t of its tile, and of a later tile js.
__device__ __forceinline__ float log_decay_in(float cs, float slo, float ct, float tlo) { return (cs - ct) + (slo - tlo); }
__device__ __forceinline__ float log_decay_over(const f32x4& T, int js, float cs, int jt, float te) {
    return te + tiles_between(T, jt, js) + cs;
}
// ... from token t to the piece's end, and from its start to token s.
__device__ __forceinline__ float log_to_end(const f32x4& T, int jt, float te) { return te + tiles_between(T, jt, 4); }
__device__ __forceinline__ float log_from_start(const f32x4& T, int js, float cs) {
    return tiles_between(T, -1, js) + cs;
}

// Whether any lane of the wave holds a non-finite value in its accumulators.
template <int NT>
__device__ __forceinline__ bool any_nonfinite(const f32x4 (&v)[NT]) {
    f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) s[r] = __builtin_fmaf(v[i][r], 0.f, s[r]);
    const bool bad = (s[0] + s[1]) + (s[2] + s[3]) != 0.f;  // (NaN)
    return __builtin_expect(__builtin_amdgcn_ballot_w64(bad) != 0, 0);
}
__device__ __forceinline__ bool any_nonfinite(const f32x4& v) {
    const f32x4 a[1] = {v};
    return any_nonfinite(a);
}

// Heads per block of the per-piece output kernels: the more, the fewer repeats
// of the per-group products (and partials), while two blocks per CU remain.
inline int piece_heads_per_block(const Shape& s, int64_t nk) {
    const int per = s.H / s.G;
    int best = 1;
    for (int c = 2; c <= 8; ++c)
        if (per % c == 0 && s.B * nk * (s.H / c) >= 2 * device_cu_count()) best = c;
    return best;
}

// Byte offsets of a lane's LDS reads of tiles of 64-float rows in 16-byte
// chunks, (m, g) = (lane % 16, lane / 16): rows of x or dy hold chunk c of row
// s at c ^ (s & 15); a state's row n holds chunk c at c ^ ((n / NV) & 15) with
// NV = min(4, N / 16), and its N-row products take the rows in the order
// n = 16 NV q + NV m + i (tile q NV + i), so that NV consecutive n of a B or C
// row are one load for NV tiles.  Both readings of either are free of bank
// conflicts.
template <int N>
struct PieceOff {
    static constexpr int K = N / 16, NV = K < 4 ? K : 4, NQ = K / NV;
    int oc[4];  // row m, chunk 4 q + g
    int op[4];  // row 4 g + q, chunk m
    int on[4];  // a state tile's row m, chunk 4 q + g
    int ow[4];  // a state's rows 16 q + 4 g + s, chunk m
    __device__ __forceinline__ void init(int m, int g) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            oc[q] = m * 256 + (((4 * q + g) ^ m) << 4);
            op[q] = (4 * g + q) * 256 + ((m ^ (4 * g + q)) << 4);
            on[q] = NV * m * 256 + (((4 * q + g) ^ m) << 4);
            // key 4 q + g for NV = 4 (by q mod 4), 8 q + 2 g + s / 2 for NV = 2,
            // 4 g + s for NV = 1
            ow[q] = NV == 4 ? g * 1024 + (((4 * q + g) ^ m) << 4)
                  : NV == 2 ? g * 1024 + ((((8 * (q >> 1) + 2 * g + (q & 1)) & 15) ^ m) << 4)
                            : g * 1024 + (((4 * g + q) ^ m) << 4);
        }
    }
    // row 16 q + 4 g + s, columns 4 m ..
    __device__ __forceinline__ f32x4 state_p(const char* tile, int q, int s) const {
        return lds4(tile + ow[NV == 4 ? q & 3 : NV == 2 ? 2 * q + (s >> 1) : s] + (16 * q + s) * 256);
    }
    // the tile's row m, columns 16 q + 4 g ..
    __device__ __forceinline__ f32x4 state_n(const char* state, int tile, int q) const {
        return lds4(state + on[q] + (16 * NV * (tile / NV) + tile % NV) * 256);
    }
    // DMA of one state [N][64] into its tile by the block's 256 threads
    __device__ __forceinline__ static void stage(const float* src, char* tile, int tid) {
        const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const int i = tid + q * 256, n = i >> 4, c = (i & 15) ^ ((n / NV) & 15);
            lds_dma16(src + n * 64 + 4 * c, tile + (w * 64 + q * 256) * 16);
        }
    }
};

}  // namespace dart
