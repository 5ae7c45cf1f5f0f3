// Control-variate network on the gfx950 matrix cores: packing of the FP32
// master weights into split-BF16 MFMA fragments, evaluation with value /
// gradient / Laplacian channels, the squared-loss gradient and Adam.
//
// Fragment layout (v_mfma_f32_16x16x32_bf16, 64 lanes, lane = 16 g + i):
//   A (16 x 32, weights):      lane holds row i, K slots (g, e), e = 0..7
//   B (32 x 16, activations):  lane holds column i, K slots (g, e)
//   D (16 x 16, FP32):         lane holds rows 4 g + r, column i, r = 0..3
// The K slot (kc, g, e) of K chunk kc is mapped to the hidden unit
//   16 (2 kc + e / 4) + 4 g + e % 4,
// which is the set of units the lanes of one column hold in D after a layer
// (tile t = 2 kc + e / 4, row 4 g + e % 4): with the weights packed in that
// order, the four units a lane holds go to the next layer's operand as they are.
// Points are the 16 columns of a tile.
#include "mlp.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>

namespace dwos_mlp_k {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__host__ __device__ constexpr int slot_unit(int kc, int g, int e) {
    return 16 * (2 * kc + (e >> 2)) + 4 * g + (e & 3);
}

__device__ inline f32x4 mma3(const bf16x8& ah, const bf16x8& al, const bf16x8& bh, const bf16x8& bl,
                             f32x4 acc) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, acc, 0, 0, 0);
    return acc;
}

// x = hi + lo with hi = bf16(x) (round to nearest even) and lo = bf16(x - hi)
__device__ inline void split(float x, __bf16& hi, __bf16& lo) {
    hi = (__bf16)x;
    lo = (__bf16)(x - (float)hi);
}

// ---------------------------------------------------------------------------
// packing: one thread per (direction, layer, fragment, lane)
//   direction 0: A = W_l      (rows = output units, K = input slots)
//   direction 1: A = W_l^T    (rows = input units,  K = output-unit slots)
// ---------------------------------------------------------------------------
__global__ void pack_kernel(const float* __restrict__ theta, u32x4* __restrict__ packed) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= 2 * kLayers * kFrags * 64) return;
    const int lane = idx & 63, f = (idx >> 6) & 7, l = (idx >> 9) & 3, dir = idx >> 11;
    const int mt = f >> 1, kc = f & 1, i = lane & 15, g = lane >> 4;
    const float* W = theta + (size_t)l * kLayerSize;
    bf16x8 hi, lo;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int k = slot_unit(kc, g, e);
        const float w = dir == 0 ? W[(16 * mt + i) * kWidth + k] : W[k * kWidth + 16 * mt + i];
        __bf16 h, o;
        split(w, h, o);
        hi[e] = h;
        lo[e] = o;
    }
    const size_t at = ((((size_t)dir * kLayers + l) * kFrags + f) * 64 + lane) * 2;
    packed[at] = __builtin_bit_cast(u32x4, hi);
    packed[at + 1] = __builtin_bit_cast(u32x4, lo);
}

// Input features of a lane's units 16 t + 4 g + r (r = 0..3).
template <int D>
struct FeatureRows {
    float b[4][D], bb[4];      // frequency (0 unless a Fourier feature) and its square
    int kind[4];               // 0 sine, 1 cosine, 2 + c coordinate c, -1 zero
    __device__ inline void load(const float* __restrict__ B, int F, int t, int g) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int f = 16 * t + 4 * g + r;
            kind[r] = f < F ? 0 : f < 2 * F ? 1 : f < 2 * F + D ? 2 + f - 2 * F : -1;
            bb[r] = 0.f;
#pragma unroll
            for (int c = 0; c < D; ++c) {
                b[r][c] = f < 2 * F ? B[(f < F ? f : f - F) * D + c] : 0.f;
                bb[r] += b[r][c] * b[r][c];
            }
        }
    }
    // ch 0 = value, ch 1..D = d/dx_c, ch D+1 = Laplacian
    template <int NC>
    __device__ inline void eval(const float x[D], float act[NC][4]) const {
        constexpr float kTwoPi = 6.28318530717958647692f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float th = 0.f, sn, cs;
#pragma unroll
            for (int c = 0; c < D; ++c) th += b[r][c] * x[c];
            sincosf(kTwoPi * th, &sn, &cs);
            const float v = kind[r] == 0 ? sn : kind[r] == 1 ? cs : 0.f;    // value
            const float dv = kind[r] == 0 ? cs : kind[r] == 1 ? -sn : 0.f;  // its derivative in th
            act[0][r] = v;
#pragma unroll
            for (int c = 0; c < D; ++c) act[0][r] = kind[r] == 2 + c ? x[c] : act[0][r];
            if constexpr (NC > 1) {
#pragma unroll
                for (int c = 0; c < D; ++c) act[1 + c][r] = kind[r] == 2 + c ? 1.f : kTwoPi * b[r][c] * dv;
                act[D + 1][r] = -(kTwoPi * kTwoPi) * bb[r] * v;
            }
        }
    }
};

// ---------------------------------------------------------------------------
// A block of four wavefronts takes the same 16 points through the network (a
// column set is one channel of 16 points; S of them are in flight), each
// wavefront computing 16 of the 64 units of every layer.  What a wavefront
// keeps of a point -- pre-activations of all layers, its rows of all weight
// gradients -- then fits its registers, and the layers meet in LDS.
//
// LDS holds activations as the MFMA operands: [set][hi, lo][unit tile], a tile
// being 64 slots of four units of a point in BF16.  A lane writes its four units
// of a point; a layer product reads them back as K slots, and the
// weight-gradient products, which contract over points and channels, read the
// same tile transposed (ds_read_b64_tr_b16: of the 16 slots that the lanes of
// one g name, rows of four in lane order, lane i gets element i of each row).
// Unit group c of point p is in slot 16 c + (p ^ 4 c): the 16 lanes that LDS
// serves at a time then touch every bank once in either access (with the 16
// units of a point next to each other it took four times as long: 64 of the
// 120 us of an evaluation, 121 of the 297 us of a gradient).
// ---------------------------------------------------------------------------
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
constexpr int kTileBytes = 16 * 16 * 2;
constexpr int kSetBytes = 2 * 4 * kTileBytes;
constexpr int kNetWaves = 4;

__device__ inline bf16x8 join(bf16x4 a, bf16x4 b) {
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

__device__ inline int slot_bytes(int c, int p) { return 8 * (16 * c + (p ^ (4 * c))); }

// this lane's four units (of the wavefront's tile w) of set q; at = slot_bytes(g, i)
__device__ inline void put_set(lds_char* buf, int q, int w, int at, const float v[4]) {
    bf16x4 hi, lo;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        __bf16 h, o;
        split(v[r], h, o);
        hi[r] = h;
        lo[r] = o;
    }
    lds_char* to = buf + q * kSetBytes + w * kTileBytes + at;
    *(lds_bf16x4*)to = hi;
    *(lds_bf16x4*)(to + 4 * kTileBytes) = lo;
}

// K slots of chunk kc of set q, as a B operand; at = slot_bytes(g, i)
__device__ inline bf16x8 get_slots(const lds_char* buf, int q, int part, int kc, int at) {
    const lds_char* from = buf + q * kSetBytes + (4 * part + 2 * kc) * kTileBytes + at;
    return join(*(const lds_bf16x4*)from, *(const lds_bf16x4*)(from + kTileBytes));
}

// unit i of points 4 g .. 4 g + 3 of unit tile t of set q; at = slot_bytes(i % 4, 4 g + i / 4)
__device__ inline bf16x4 get_points(lds_char* buf, int q, int part, int t, int at) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
        (lds_bf16x4*)(buf + q * kSetBytes + (4 * part + t) * kTileBytes + at));
}

struct RowWeights { bf16x8 h[2], l[2]; };      // K chunks of 16 rows of a layer
__device__ inline RowWeights load_rows(const u32x4* __restrict__ layer, int w, int lane) {
    RowWeights o;
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) {
        const int fr = (w * 2 + kc) * 64 + lane;
        o.h[kc] = __builtin_bit_cast(bf16x8, layer[2 * fr]);
        o.l[kc] = __builtin_bit_cast(bf16x8, layer[2 * fr + 1]);
    }
    return o;
}

template <int S>
__device__ inline void rows_product(const RowWeights& wt, const lds_char* buf, int at, f32x4 acc[S]) {
#pragma unroll
    for (int q = 0; q < S; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < 2; ++kc)
#pragma unroll
        for (int q = 0; q < S; ++q)
            acc[q] = mma3(wt.h[kc], wt.l[kc], get_slots(buf, q, 0, kc, at), get_slots(buf, q, 1, kc, at), acc[q]);
}

// Layer outputs of NC channels from the pre-activation derivatives z[1..] and
// h = tanh(z[0]) (h' = 1 - h^2, h'' = -2 h (1 - h^2))
template <int D, int NC>
__device__ inline void outputs(const float h, const float* z, float* out) {
    out[0] = h;
    if constexpr (NC > 1) {
        const float s = 1.f - h * h;
        float zz = 0.f;
#pragma unroll
        for (int c = 0; c < D; ++c) {
            zz += z[1 + c] * z[1 + c];
            out[1 + c] = s * z[1 + c];
        }
        out[D + 1] = s * z[D + 1] - 2.f * h * s * zz;
    }
}

template <class TX>
struct EvalArgs {
    const u32x4* packed;
    const float* theta;
    const float* B;
    int F;
    const TX* X;
    int64_t n;
    const int32_t* mask;
    int mask_div, mask_min;
    int chunk;           // MASKED: points a block looks through at a time, a multiple of 256
    float* N;
    float* G;
    float* L;
};

// ---------------------------------------------------------------------------
// evaluation: N, and with LAP the gradient and Laplacian channels, carried
// through each layer by the chain rule.  A wavefront keeps its rows of all
// four layers in registers.  (With 64 KB of weights staged in LDS and a tile
// of points to each wavefront, every block of the 1024 staged them for one
// tile per wavefront: 65,536 points with derivatives 115 us, now 78 us, of which
// issuing the vector arithmetic of tanh, sincos and the BF16 splits is 45.)
//
// MASKED: a block looks through `chunk` points at a time and evaluates those that
// the mask lets through, listed in LDS, in full tiles (a point's result does not
// depend on its column).  Of the walks around an object one in ninety runs nested
// walks: 4.2 M points took 840 us, with derivatives 950, where a block skipped
// tiles of 64 and 16 points without any, and take 115 and 115.
// ---------------------------------------------------------------------------
constexpr int kEvalChunk = 1024;      // most points a block looks through at a time
template <int D, bool LAP, class TX, bool MASKED>
__global__ void __launch_bounds__(64 * kNetWaves, 2) eval_kernel(EvalArgs<TX> a) {
    constexpr int NC = LAP ? D + 2 : 1, NT = LAP ? 1 : 4, S = NC * NT;
    __shared__ __align__(16) char s_act[2][S * kSetBytes];
    __shared__ float s_out[kNetWaves][S * 16];
    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4, w = threadIdx.x >> 6;
    const int at = slot_bytes(g, i);
    lds_char* buf[2] = {(lds_char*)s_act[0], (lds_char*)s_act[1]};
    FeatureRows<D> fr;
    fr.load(a.B, a.F, w, g);
    RowWeights wt[kLayers];
    float bias[kLayers][4], w5[4];
#pragma unroll
    for (int l = 0; l < kLayers; ++l) {
        wt[l] = load_rows(a.packed + (size_t)l * kPackLayerU4, w, lane);
#pragma unroll
        for (int r = 0; r < 4; ++r) bias[l][r] = a.theta[l * kLayerSize + kWidth * kWidth + 16 * w + 4 * g + r];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) w5[r] = a.theta[kLayers * kLayerSize + 16 * w + 4 * g + r];
    const float b5 = a.theta[kLayers * kLayerSize + kWidth];
    // 16 NT points; point(j): the j-th, or -1
    auto tiles = [&](auto point) {
        float x[NT][D], act[S][4];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int64_t p = point(nt * 16 + i);
#pragma unroll
            for (int c = 0; c < D; ++c) x[nt][c] = p >= 0 ? (float)a.X[p * D + c] : 0.f;
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) fr.template eval<NC>(x[nt], act + nt * NC);
#pragma unroll
        for (int q = 0; q < S; ++q) put_set(buf[0], q, w, at, act[q]);
        __syncthreads();
#pragma unroll
        for (int l = 0; l < kLayers; ++l) {
            f32x4 acc[S];
            rows_product<S>(wt[l], buf[l & 1], at, acc);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float z[NC], out[NC];
#pragma unroll
                    for (int ch = 0; ch < NC; ++ch) z[ch] = acc[nt * NC + ch][r];
                    outputs<D, NC>(tanhf(z[0] + bias[l][r]), z, out);
#pragma unroll
                    for (int ch = 0; ch < NC; ++ch) act[nt * NC + ch][r] = out[ch];
                }
            if (l + 1 < kLayers) {
#pragma unroll
                for (int q = 0; q < S; ++q) put_set(buf[(l + 1) & 1], q, w, at, act[q]);
                __syncthreads();
            }
        }
#pragma unroll
        for (int q = 0; q < S; ++q) {
            float o = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) o += w5[r] * act[q][r];
            o += __shfl_xor(o, 16);
            o += __shfl_xor(o, 32);
            if (g == 0) s_out[w][q * 16 + i] = o;
        }
        __syncthreads();
        if (threadIdx.x < S * 16) {
            const int q = threadIdx.x >> 4, nt = q / NC, ch = q - nt * NC;
            const int64_t p = point(nt * 16 + (int)(threadIdx.x & 15));
            if (p >= 0) {
                float o = 0.f;
#pragma unroll
                for (int k = 0; k < kNetWaves; ++k) o += s_out[k][threadIdx.x];
                if (ch == 0) a.N[p] = o + b5;
                else if (ch <= D) { if (a.G) a.G[p * D + ch - 1] = o; }
                else if (a.L) a.L[p] = o;
            }
        }
    };
    if constexpr (MASKED) {
        __shared__ unsigned short s_list[kEvalChunk];
        __shared__ int s_count;
        for (int64_t p0 = (int64_t)blockIdx.x * a.chunk; p0 < a.n; p0 += (int64_t)gridDim.x * a.chunk) {
            __syncthreads();                       // the last chunk's list is read
            if (threadIdx.x == 0) s_count = 0;
            __syncthreads();
            for (int j = threadIdx.x; j < a.chunk; j += 64 * kNetWaves) {
                const int64_t p = p0 + j;
                const bool in = p < a.n && a.mask[p / a.mask_div] >= a.mask_min;
                const unsigned long long m = __ballot(in);
                int base = 0;
                if (lane == 0 && m) base = atomicAdd(&s_count, __popcll(m));
                base = __builtin_amdgcn_readfirstlane(base);
                if (in) s_list[base + __popcll(m & ((1ull << lane) - 1ull))] = (unsigned short)j;
            }
            __syncthreads();
            const int count = s_count;
            for (int t = 0; t < count; t += 16 * NT)
                tiles([&](int j) { return t + j < count ? p0 + (int64_t)s_list[t + j] : (int64_t)-1; });
        }
    } else {
        for (int64_t p0 = (int64_t)blockIdx.x * (16 * NT); p0 < a.n; p0 += (int64_t)gridDim.x * (16 * NT))
            tiles([&](int j) { return p0 + j < a.n ? p0 + j : (int64_t)-1; });
    }
}

// sum over the 16 columns (lanes with the same g)
__device__ inline float col_sum(float v) {
    v += __shfl_xor(v, 1);
    v += __shfl_xor(v, 2);
    v += __shfl_xor(v, 4);
    v += __shfl_xor(v, 8);
    return v;
}

struct TrainArgs {
    const u32x4* packed;
    const float* theta;
    const float* B;
    int F;
    const float* X;
    const float* nbar;   // LOSS: targets; else adjoints of N
    const float* lbar;   // LOSS: weights or null (1); else adjoints of Lap N, or null
    int64_t n;
    float* part;         // kPartial sums per block
};
constexpr int kPartial = kThetaSize + 1;      // the parameters' gradient and the loss

// ---------------------------------------------------------------------------
// Parameter gradients.  LOSS: of sum 1/2 w (N - t)^2 over the points (value
// channel, four tiles of points at a time); else of sum Nbar N + Lbar Lap N
// with the value, gradient and Laplacian channels of one tile.  Backward, with
// h = tanh z, s = 1 - h^2, Q = sum_c z_c^2:
//   zbar_L = s abar_L,  zbar_c = s abar_c - 4 h s z_c abar_L,
//   zbar = s abar - 2 h s sum_c z_c abar_c - (2 h s z_L + 2 s (s - 2 h^2) Q) abar_L
// Every channel goes back through W^T, and dW = sum over points and channels of
// zbar a^T, all on the matrix cores in one pass; the blocks' sums are added by
// sum_kernel in one order.  (As one kernel that left every layer's operands and
// pre-activations in memory, 1 GB for 65,536 points, added each tile's bias
// gradients with atomics, and was followed by a product over that memory:
// 0.78 + 0.29 ms, now 0.22 + 0.01.  One block per CU: two, at 256 registers a
// lane, spill 125 of them and take 0.24 ms.)
// ---------------------------------------------------------------------------
template <int D, bool LOSS>
__global__ void __launch_bounds__(64 * kNetWaves, 1) grad_kernel(TrainArgs a) {
    constexpr int NC = LOSS ? 1 : D + 2, NT = LOSS ? 4 : 1, S = NC * NT;
    __shared__ __align__(16) char s_act[3][S * kSetBytes];
    __shared__ float s_out[kNetWaves][S * 16];
    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4, w = threadIdx.x >> 6;
    const int at = slot_bytes(g, i), att = slot_bytes(i & 3, 4 * g + (i >> 2));
    __shared__ float s_bias[kLayers + 1][kWidth];       // and the output layer's weights
    lds_char *feat = (lds_char*)s_act[0], *abuf = (lds_char*)s_act[1], *dbuf = (lds_char*)s_act[2];
    const int u0 = 16 * w + 4 * g;             // the lane's units u0 + r
    s_bias[w][lane] = a.theta[w * kLayerSize + kWidth * kWidth + lane];
    if (w == 0) s_bias[kLayers][lane] = a.theta[kLayers * kLayerSize + lane];
    const float b5 = a.theta[kLayers * kLayerSize + kWidth];
    FeatureRows<D> fr;
    fr.load(a.B, a.F, w, g);
    __syncthreads();
    f32x4 dW[kLayers][4];
    float gb[kLayers][4], gw5[4], gb5 = 0.f, loss = 0.f;
#pragma unroll
    for (int l = 0; l < kLayers; ++l)
#pragma unroll
        for (int k = 0; k < 4; ++k) { dW[l][k] = f32x4{0.f, 0.f, 0.f, 0.f}; gb[l][k] = 0.f; }
#pragma unroll
    for (int k = 0; k < 4; ++k) gw5[k] = 0.f;
    // the next layer's weights and the next points are loaded while a layer is computed
    RowWeights wn = load_rows(a.packed, w, lane);
    float xn[NT][D], nbn[NT], lbn[NT];
    auto fetch = [&](int64_t it) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int64_t p = (it * NT + nt) * 16 + i;
            const bool valid = p < a.n;
#pragma unroll
            for (int c = 0; c < D; ++c) xn[nt][c] = valid ? a.X[p * D + c] : 0.f;
            nbn[nt] = valid ? a.nbar[p] : 0.f;
            lbn[nt] = valid ? (a.lbar ? a.lbar[p] : (LOSS ? 1.f : 0.f)) : 0.f;
        }
    };
    fetch(blockIdx.x);
    for (int64_t it = blockIdx.x; it * (16 * NT) < a.n; it += gridDim.x) {
        float act[S][4], z[kLayers][S][4];     // z: tanh z of the value channel, z of the others
        float nb[NT], lb[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            nb[nt] = nbn[nt];
            lb[nt] = lbn[nt];
            fr.template eval<NC>(xn[nt], act + nt * NC);
        }
        fetch(it + gridDim.x);
#pragma unroll
        for (int q = 0; q < S; ++q) put_set(feat, q, w, at, act[q]);
        f32x4 acc[S];
#pragma unroll
        for (int l = 0; l < kLayers; ++l) {
            const RowWeights wt = wn;
            wn = load_rows(a.packed + (l + 1 < kLayers ? (size_t)(l + 1) * kPackLayerU4
                                                       : kPackDirU4 + (size_t)l * kPackLayerU4), w, lane);
            __syncthreads();
            rows_product<S>(wt, l == 0 ? feat : (l & 1) ? abuf : dbuf, at, acc);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float zz[NC], out[NC];
#pragma unroll
                    for (int ch = 0; ch < NC; ++ch) zz[ch] = acc[nt * NC + ch][r];
                    zz[0] = tanhf(zz[0] + s_bias[l][u0 + r]);
                    outputs<D, NC>(zz[0], zz, out);
#pragma unroll
                    for (int ch = 0; ch < NC; ++ch) {
                        z[l][nt * NC + ch][r] = zz[ch];
                        act[nt * NC + ch][r] = out[ch];
                    }
                }
            if (l + 1 < kLayers) {
#pragma unroll
                for (int q = 0; q < S; ++q) put_set((l & 1) ? dbuf : abuf, q, w, at, act[q]);
            }
        }
        // output layer: the adjoints of N and Lap N, then of the last layer's outputs
        float w5[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) w5[r] = s_bias[kLayers][u0 + r];
        if constexpr (LOSS) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                float o = 0.f;
#pragma unroll
                for (int r = 0; r < 4; ++r) o += w5[r] * act[nt][r];
                o += __shfl_xor(o, 16);
                o += __shfl_xor(o, 32);
                if (g == 0) s_out[w][nt * 16 + i] = o;
            }
            __syncthreads();
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                float o = 0.f;
#pragma unroll
                for (int k = 0; k < kNetWaves; ++k) o += s_out[k][nt * 16 + i];
                const float e = o + b5 - nb[nt];
                loss += 0.5f * lb[nt] * e * e;
                nb[nt] = lb[nt] * e;
            }
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            gb5 += nb[nt];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                gw5[r] += nb[nt] * act[nt * NC][r];
                if constexpr (!LOSS) gw5[r] += lb[nt] * act[D + 1][r];
#pragma unroll
                for (int ch = 0; ch < NC; ++ch) act[nt * NC + ch][r] = 0.f;   // becomes abar
                act[nt * NC][r] = nb[nt] * w5[r];
                if constexpr (!LOSS) act[D + 1][r] = lb[nt] * w5[r];
            }
        }
#pragma unroll
        for (int l = kLayers - 1; l >= 0; --l) {
            if (l < kLayers - 1) __syncthreads();   // abuf and dbuf are read
            // the layer's inputs (the last layer's are there from the forward pass)
            if (l > 0 && l < kLayers - 1) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    float in[NC][4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float zz[NC], out[NC];
#pragma unroll
                        for (int ch = 0; ch < NC; ++ch) zz[ch] = z[l > 0 ? l - 1 : 0][nt * NC + ch][r];
                        outputs<D, NC>(zz[0], zz, out);
#pragma unroll
                        for (int ch = 0; ch < NC; ++ch) in[ch][r] = out[ch];
                    }
#pragma unroll
                    for (int ch = 0; ch < NC; ++ch) put_set(abuf, nt * NC + ch, w, at, in[ch]);
                }
            }
            // pre-activation adjoints
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float h = z[l][nt * NC][r], s = 1.f - h * h;
                    if constexpr (LOSS) {
                        act[nt][r] *= s;
                    } else {
                        const float aL = act[D + 1][r], zL = z[l][D + 1][r];
                        float Q = 0.f, za = 0.f;
#pragma unroll
                        for (int c = 0; c < D; ++c) {
                            const float zc = z[l][1 + c][r];
                            Q += zc * zc;
                            za += zc * act[1 + c][r];
                            act[1 + c][r] = s * act[1 + c][r] - 4.f * h * s * zc * aL;
                        }
                        act[0][r] = s * act[0][r] - 2.f * h * s * za -
                                    (2.f * h * s * zL + 2.f * s * (s - 2.f * h * h) * Q) * aL;
                        act[D + 1][r] = s * aL;
                    }
                    gb[l][r] += act[nt * NC][r];
                }
#pragma unroll
            for (int q = 0; q < S; ++q) put_set(dbuf, q, w, at, act[q]);
            const RowWeights wt = wn;
            if (l > 0) wn = load_rows(a.packed + (l > 1 ? kPackDirU4 + (size_t)(l - 1) * kPackLayerU4 : 0), w, lane);
            __syncthreads();
            // dW rows of this wavefront: K = points of two sets at a time
            lds_char* in = l == 0 ? feat : abuf;
#pragma unroll
            for (int q = 0; q + 1 < S; q += 2) {
                const bf16x8 dh = join(get_points(dbuf, q, 0, w, att), get_points(dbuf, q + 1, 0, w, att));
                const bf16x8 dl = join(get_points(dbuf, q, 1, w, att), get_points(dbuf, q + 1, 1, w, att));
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    dW[l][t] = mma3(dh, dl, join(get_points(in, q, 0, t, att), get_points(in, q + 1, 0, t, att)),
                                    join(get_points(in, q, 1, t, att), get_points(in, q + 1, 1, t, att)), dW[l][t]);
            }
            if constexpr (S & 1) {
                const s16x4 dh = __builtin_bit_cast(s16x4, get_points(dbuf, S - 1, 0, w, att));
                const s16x4 dl = __builtin_bit_cast(s16x4, get_points(dbuf, S - 1, 1, w, att));
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const s16x4 ih = __builtin_bit_cast(s16x4, get_points(in, S - 1, 0, t, att));
                    const s16x4 il = __builtin_bit_cast(s16x4, get_points(in, S - 1, 1, t, att));
                    dW[l][t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(dh, ih, dW[l][t], 0, 0, 0);
                    dW[l][t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(dh, il, dW[l][t], 0, 0, 0);
                    dW[l][t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(dl, ih, dW[l][t], 0, 0, 0);
                }
            }
            if (l > 0) {
                rows_product<S>(wt, dbuf, at, acc);
#pragma unroll
                for (int q = 0; q < S; ++q)
#pragma unroll
                    for (int r = 0; r < 4; ++r) act[q][r] = acc[q][r];
            }
        }
        __syncthreads();                       // the buffers are free for the next points
    }
    float* out = a.part + (size_t)blockIdx.x * kPartial;
#pragma unroll
    for (int l = 0; l < kLayers; ++l)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
            for (int t = 0; t < 4; ++t) out[l * kLayerSize + (u0 + r) * kWidth + 16 * t + i] = dW[l][t][r];
            const float b = col_sum(gb[l][r]);
            if (i == 0) out[l * kLayerSize + kWidth * kWidth + u0 + r] = b;
        }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float b = col_sum(gw5[r]);
        if (i == 0) out[kLayers * kLayerSize + u0 + r] = b;
    }
    gb5 = col_sum(gb5);
    loss = col_sum(loss);
    if (threadIdx.x == 0) {
        out[kLayers * kLayerSize + kWidth] = gb5;
        out[kThetaSize] = loss;
    }
}

// grad (and the loss, if asked for) = the blocks' sums
__global__ void __launch_bounds__(256) sum_kernel(const float* __restrict__ part, int blocks, float* __restrict__ grad,
                                                  float* __restrict__ loss) {
    __shared__ double s[4][64];
    const int k = blockIdx.x * 64 + (threadIdx.x & 63), slice = threadIdx.x >> 6;
    double v = 0.0;
    if (k < kPartial) {
#pragma unroll 8
        for (int b = slice; b < blocks; b += 4) v += (double)part[(size_t)b * kPartial + k];
    }
    s[slice][threadIdx.x & 63] = v;
    __syncthreads();
    if (slice == 0 && k < kPartial) {
        const float t = (float)((s[0][threadIdx.x] + s[1][threadIdx.x]) + (s[2][threadIdx.x] + s[3][threadIdx.x]));
        if (k < kThetaSize) grad[k] = t;
        else if (loss) *loss = t;
    }
}

__global__ void zero_kernel(float* __restrict__ p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.f;
}

// Adam (Kingma and Ba, Algorithm 1) on the FP32 master parameters
__global__ void adam_kernel(float* __restrict__ theta, float* __restrict__ m, float* __restrict__ v,
                            const float* __restrict__ g, int64_t n, float lr, float b1, float b2,
                            float eps, float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    theta[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

}  // namespace dwos_mlp_k

namespace dwos_host {

using namespace dwos_mlp_k;

hipError_t pack(dwos_mlp* m, hipStream_t s) {
    hipLaunchKernelGGL(pack_kernel, dim3(blocks_for(2 * kLayers * kFrags * 64, 256)), dim3(256), 0, s,
                       m->theta.as<float>(), m->packed.as<u32x4>());
    return hipGetLastError();
}

hipError_t zero(float* p, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(zero_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

// Blocks of a persistent launch over groups of `points` points: at most
// `per_cu` per CU.
unsigned net_grid(const dwos_mlp* m, int64_t n, int points, int per_cu) {
    return (unsigned)std::min<int64_t>((n + points - 1) / points, (int64_t)per_cu * m->cu_count);
}

template <class TX>
hipError_t mlp_eval_launch(const dwos_mlp* m, hipStream_t s, const TX* X, int64_t n,
                           const int32_t* mask, int mask_div, int mask_min, float* N, float* G,
                           float* L) {
    if (n <= 0) return hipSuccess;
    EvalArgs<TX> a{m->packed.as<u32x4>(), m->theta.as<float>(), m->B.as<float>(), m->F, X, n,
                   mask, mask_div < 1 ? 1 : mask_div, mask_min, 0, N, G, L};
    const bool lap = G || L;
    int points = lap ? 16 : 64;
    if (mask) {
        // as many points as give every resident block a share, in whole rounds
        // of its threads
        const int64_t share = n / (2 * m->cu_count) / 256 * 256;
        points = a.chunk = (int)std::min<int64_t>(kEvalChunk, std::max<int64_t>(256, share));
    }
    const dim3 grid(net_grid(m, n, points, 2)), block(64 * kNetWaves);
    auto go = [&](auto dim, auto with_lap, auto masked) {
        constexpr int D = decltype(dim)::value;
        constexpr bool LAP = decltype(with_lap)::value, MASKED = decltype(masked)::value;
        hipLaunchKernelGGL((eval_kernel<D, LAP, TX, MASKED>), grid, block, 0, s, a);
    };
    auto by_mask = [&](auto dim, auto with_lap) {
        if (mask) go(dim, with_lap, std::true_type{});
        else go(dim, with_lap, std::false_type{});
    };
    auto by_lap = [&](auto dim) {
        if (lap) by_mask(dim, std::true_type{});
        else by_mask(dim, std::false_type{});
    };
    if (m->dim == 2) by_lap(std::integral_constant<int, 2>{});
    else by_lap(std::integral_constant<int, 3>{});
    return hipGetLastError();
}

template hipError_t mlp_eval_launch<float>(const dwos_mlp*, hipStream_t, const float*, int64_t,
                                           const int32_t*, int, int, float*, float*, float*);
template hipError_t mlp_eval_launch<double>(const dwos_mlp*, hipStream_t, const double*, int64_t,
                                            const int32_t*, int, int, float*, float*, float*);

// grad (and *loss) from TrainArgs without its workspace
template <bool LOSS>
hipError_t grad_launch(dwos_mlp* m, hipStream_t s, TrainArgs a, float* loss) {
    hipError_t e;
    if (a.n <= 0) {
        if (loss && (e = zero(loss, 1, s)) != hipSuccess) return e;
        return zero(m->grad.as<float>(), kThetaSize, s);
    }
    const unsigned grid = net_grid(m, a.n, LOSS ? 64 : 16, 1);
    if ((e = m->ws.reserve((size_t)m->cu_count * kPartial * sizeof(float))) != hipSuccess) return e;
    a.part = m->ws.as<float>();
    if (m->dim == 2) hipLaunchKernelGGL((grad_kernel<2, LOSS>), dim3(grid), dim3(64 * kNetWaves), 0, s, a);
    else hipLaunchKernelGGL((grad_kernel<3, LOSS>), dim3(grid), dim3(64 * kNetWaves), 0, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(sum_kernel, dim3(blocks_for(kPartial, 64)), dim3(256), 0, s, a.part, (int)grid,
                       m->grad.as<float>(), loss);
    return hipGetLastError();
}

hipError_t mlp_loss_grad_launch(dwos_mlp* m, hipStream_t s, const float* X, const float* T,
                                const float* w, int64_t n, float* loss) {
    return grad_launch<true>(m, s, {m->packed.as<u32x4>(), m->theta.as<float>(), m->B.as<float>(), m->F, X, T, w, n,
                                    nullptr}, loss);
}

hipError_t mlp_vjp_launch(dwos_mlp* m, hipStream_t s, const float* X, const float* Nbar,
                          const float* Lbar, int64_t n) {
    return grad_launch<false>(m, s, {m->packed.as<u32x4>(), m->theta.as<float>(), m->B.as<float>(), m->F, X, Nbar, Lbar,
                                     n, nullptr}, nullptr);
}

hipError_t mlp_adam_launch(dwos_mlp* m, hipStream_t s, float lr, float beta1, float beta2, float eps) {
    m->step += 1;
    const float c1 = (float)(1.0 - std::pow((double)beta1, (double)m->step));
    const float c2 = (float)(1.0 - std::pow((double)beta2, (double)m->step));
    hipLaunchKernelGGL(adam_kernel, dim3(blocks_for(kThetaSize, 256)), dim3(256), 0, s,
                       m->theta.as<float>(), m->m.as<float>(), m->v.as<float>(), m->grad.as<float>(),
                       (int64_t)kThetaSize, lr, beta1, beta2, eps, c1, c2);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return pack(m, s);
}

}  // namespace dwos_host

// ===========================================================================
// C ABI (declared in include/dwos.h)
// ===========================================================================
using dwos_host::fail;

extern "C" {

int32_t dwos_mlp_theta_size(void) { return dwos_mlp_k::kThetaSize; }

dwos_status dwos_mlp_create(int32_t dim, int32_t F, const float* B, void* stream, dwos_mlp** out) {
    if (!out) return fail(DWOS_EINVAL, "mlp_create: NULL out");
    *out = nullptr;
    if (dim != 2 && dim != 3) return fail(DWOS_EINVAL, "mlp_create: dim must be 2 or 3");
    if (F < 0 || 2 * F + dim > dwos_mlp_k::kWidth) return fail(DWOS_EINVAL, "mlp_create: need 0 <= 2F + dim <= 64");
    if (F > 0 && !B) return fail(DWOS_EINVAL, "mlp_create: NULL frequencies");
    for (int i = 0; i < F * dim; ++i)
        if (!std::isfinite(B[i])) return fail(DWOS_EINVAL, "mlp_create: non-finite frequency");
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess || n < 1) return fail(DWOS_EDEVICE, "mlp_create: no GPU");
    auto m = new (std::nothrow) dwos_mlp();
    if (!m) return fail(DWOS_ENOMEM, "mlp_create: out of host memory");
    auto bail = [&](dwos_status st) { delete m; return st; };
    m->dim = dim;
    m->F = F;
    m->stream = static_cast<hipStream_t>(stream);
    if (hipGetDevice(&m->device) != hipSuccess ||
        hipDeviceGetAttribute(&m->cu_count, hipDeviceAttributeMultiprocessorCount, m->device) != hipSuccess)
        return bail(fail(DWOS_EDEVICE, "mlp_create: hipGetDevice"));
    using namespace dwos_mlp_k;
    const size_t tb = (size_t)kThetaSize * sizeof(float);
    if (m->theta.reserve(tb) || m->m.reserve(tb) || m->v.reserve(tb) || m->grad.reserve(tb) ||
        m->B.reserve(std::max<size_t>(1, (size_t)F * dim) * sizeof(float)) ||
        m->packed.reserve((size_t)kPackU4 * 16) || m->loss.reserve(sizeof(float)))
        return bail(fail(DWOS_ENOMEM, "mlp_create: device allocation failed"));
    hipStream_t s = m->stream;
    hipError_t e = hipSuccess;
    if (F > 0) e = hipMemcpyAsync(m->B.ptr, B, (size_t)F * dim * sizeof(float), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = dwos_host::zero(m->theta.as<float>(), kThetaSize, s);
    if (e == hipSuccess) e = dwos_host::zero(m->m.as<float>(), kThetaSize, s);
    if (e == hipSuccess) e = dwos_host::zero(m->v.as<float>(), kThetaSize, s);
    if (e == hipSuccess) e = dwos_host::pack(m, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return bail(fail(DWOS_EDEVICE, std::string("mlp_create: ") + hipGetErrorString(e)));
    *out = m;
    return DWOS_OK;
}

void dwos_mlp_destroy(dwos_mlp* m) {
    if (!m) return;
    (void)hipSetDevice(m->device);
    (void)hipStreamSynchronize(m->stream);
    delete m;
}

dwos_status dwos_mlp_set_params(dwos_mlp* m, const float* theta) {
    if (!m || !theta) return fail(DWOS_EINVAL, "mlp_set_params: NULL argument");
    using namespace dwos_mlp_k;
    HIP_OK(hipSetDevice(m->device));
    hipStream_t s = m->stream;
    HIP_OK(hipMemcpyAsync(m->theta.ptr, theta, (size_t)kThetaSize * sizeof(float), hipMemcpyDeviceToDevice, s));
    HIP_OK(dwos_host::zero(m->m.as<float>(), kThetaSize, s));
    HIP_OK(dwos_host::zero(m->v.as<float>(), kThetaSize, s));
    m->step = 0;
    HIP_OK(dwos_host::pack(m, s));
    return DWOS_OK;
}

dwos_status dwos_mlp_get_params(dwos_mlp* m, float* theta) {
    if (!m || !theta) return fail(DWOS_EINVAL, "mlp_get_params: NULL argument");
    HIP_OK(hipSetDevice(m->device));
    HIP_OK(hipMemcpyAsync(theta, m->theta.ptr, (size_t)dwos_mlp_k::kThetaSize * sizeof(float),
                          hipMemcpyDeviceToDevice, m->stream));
    return DWOS_OK;
}

dwos_status dwos_mlp_eval(dwos_mlp* m, const float* X, int64_t n, float* N, float* grad, float* lap) {
    if (!m) return fail(DWOS_EINVAL, "mlp_eval: NULL network");
    if (n < 0 || (n > 0 && (!X || !N))) return fail(DWOS_EINVAL, "mlp_eval: bad arguments");
    HIP_OK(hipSetDevice(m->device));
    HIP_OK(dwos_host::mlp_eval_launch<float>(m, m->stream, X, n, nullptr, 1, 0, N, grad, lap));
    return DWOS_OK;
}

dwos_status dwos_mlp_loss_grad(dwos_mlp* m, const float* X, const float* T, const float* w, int64_t n,
                               float* loss, float* grad) {
    if (!m) return fail(DWOS_EINVAL, "mlp_loss_grad: NULL network");
    if (n < 0 || (n > 0 && (!X || !T))) return fail(DWOS_EINVAL, "mlp_loss_grad: bad arguments");
    HIP_OK(hipSetDevice(m->device));
    HIP_OK(dwos_host::mlp_loss_grad_launch(m, m->stream, X, T, w, n, loss));
    if (grad)
        HIP_OK(hipMemcpyAsync(grad, m->grad.ptr, (size_t)dwos_mlp_k::kThetaSize * sizeof(float),
                              hipMemcpyDeviceToDevice, m->stream));
    return DWOS_OK;
}

dwos_status dwos_mlp_vjp(dwos_mlp* m, const float* X, const float* Nbar, const float* Lbar, int64_t n,
                         float* grad) {
    if (!m) return fail(DWOS_EINVAL, "mlp_vjp: NULL network");
    if (n < 0 || (n > 0 && (!X || !Nbar))) return fail(DWOS_EINVAL, "mlp_vjp: bad arguments");
    HIP_OK(hipSetDevice(m->device));
    HIP_OK(dwos_host::mlp_vjp_launch(m, m->stream, X, Nbar, Lbar, n));
    if (grad)
        HIP_OK(hipMemcpyAsync(grad, m->grad.ptr, (size_t)dwos_mlp_k::kThetaSize * sizeof(float),
                              hipMemcpyDeviceToDevice, m->stream));
    return DWOS_OK;
}

dwos_status dwos_mlp_adam_step(dwos_mlp* m, float lr, float beta1, float beta2, float eps) {
    if (!m) return fail(DWOS_EINVAL, "mlp_adam_step: NULL network");
    if (!(lr > 0.f) || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps > 0.f))
        return fail(DWOS_EINVAL, "mlp_adam_step: bad hyperparameters");
    HIP_OK(hipSetDevice(m->device));
    HIP_OK(dwos_host::mlp_adam_launch(m, m->stream, lr, beta1, beta2, eps));
    return DWOS_OK;
}

}  // extern "C"
