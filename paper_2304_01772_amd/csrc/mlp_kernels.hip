// Surrogate MLP 4-128-128-3 (SiLU) on gfx950 matrix cores.
//
// The network maps normalised Hamiltonian parameters (beta, Jx, Jy, h) to
// normalised equilibrium observables; it steers the parameter optimisation
// of the paper's optimisation experiments (Results) while Monte Carlo checks
// its answers.  Weights and activations enter the matrix cores as BF16
// (round to nearest even from FP32), products accumulate in FP32
// (gfx950's v_mfma_f32_16x16x32_bf16: a 16x16 tile per wave, K = 32).  Rounding points (the oracle mirrors them):
//   forward : xb = bf16(x); z1 = W1b xb + b1; h1 = bf16(silu z1);
//             z2 = W2b h1 + b2; h2 = bf16(silu z2); y = W3b h2 + b3
//   backward: dY = 2 w (y - t) / B (FP32);  dW3 = sum dY h2, dH2 = W3b^T dY;
//             dz2 = dH2 silu'(z2); dz2b = bf16(dz2);
//             dW2 = sum dz2b h1 (MFMA), dH1 = W2b^T dz2b (MFMA);
//             dz1 = dH1 silu'(z1); dW1 = sum dz1 xb; dx = W1b^T dz1;
//             bias gradients are FP32 sums of the unrounded dz.
// Batch sums are per-workgroup partials reduced in a fixed order, so the
// result does not depend on scheduling.  Each workgroup (4 waves) handles
// 64 samples, 16 per wave.
#include "spinmc_internal.hpp"

namespace spinmc {

namespace {

constexpr int kIn = 4, kH = 128, kOut = 3;
constexpr int oW1 = 0, ob1 = oW1 + kH * kIn, oW2 = ob1 + kH, ob2 = oW2 + kH * kH,
              oW3 = ob2 + kH, ob3 = oW3 + kOut * kH, kNP = ob3 + kOut;
constexpr int kSamplesPerWG = 64;
constexpr int kPadK = 8;             // LDS row padding (bf16 elements) against bank conflicts
constexpr int kST = kSamplesPerWG + kPadK;  // row stride of sample-major transposed tiles

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));

// Operand fragment of a 16 x 32 tile (rows r, k in [k0, k0 + 32)) from a
// row-major bf16 tile: lane l holds row l % 16, k0 + 8 (l / 16) .. + 7, one
// 16-byte load (row strides and k0 keep it 16-byte aligned).
__device__ __forceinline__ bf16x8 frag(const uint16_t* base, int stride, int k0) {
    const int l = threadIdx.x & 63;
    const uint16_t* p = base + (l & 15) * stride + k0 + 8 * (l >> 4);
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p));
}

__device__ __forceinline__ float4v mfma(bf16x8 a, bf16x8 b, float4v c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

}  // namespace

// --------------------------------------------------------------- forward
namespace {

// Four times the sigmoid, 1 / a with a = (1 + e^-z) / 4, as v_rcp_f32 and one Newton
// step: bit for bit the IEEE division's for every a from 1/4 to 2^126 (all 1.08e9
// compared on the card) in three instructions for its ten, and never subnormal, which
// v_rcp_f32 would flush.  At an infinite a, where the sigmoid is 0, the step is 0 * inf:
// GUARD takes the maximum with 0; without, a NaN that reaches the outputs tells.
template <bool GUARD>
__device__ __forceinline__ float sigm_x4(float z) {
    const float a = __builtin_fmaf(__expf(-z), 0.25f, 0.25f);
    const float r = __builtin_amdgcn_rcpf(a);
    const float s = __builtin_fmaf(__builtin_fmaf(-a, r, 1.0f), r, r);
    return GUARD ? fmaxf(s, 0.0f) : s;
}
// z / 4 first: exact, where the sigmoid alone would be subnormal
template <bool GUARD>
__device__ __forceinline__ float silu(float z) {
    return 0.25f * z * sigm_x4<GUARD>(z);
}
__device__ __forceinline__ float dsilu(float z) {
    const float s = sigm_x4<true>(z);
    return 0.25f * (1.0f + z * (1.0f - 0.25f * s)) * s;
}

// two values as BF16 in one word (v_cvt_pk_bf16_f32, nearest even), a low
__device__ __forceinline__ uint32_t pk_bf(float a, float b) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    bf16x2 v;
    v[0] = (__bf16)a;
    v[1] = (__bf16)b;
    return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ bf16x8 as_frag(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// Weights in LDS as whole MFMA A operands: 64 lanes x 16 bytes each, so that
// a wave reads one with a conflict-free ds_read_b128.  Rows of A are output
// neurons, columns of B samples, and row 4 g + i of row tile nt is neuron
// tile_neuron(nt, g) + i, so that a result lane (g = lane / 16) holds, of the
// tiles 2 kt and 2 kt + 1, the neurons 32 kt + 8 g .. + 7 of one sample:
// packed as BF16 they are its B operand of k tile kt in the next layer.
// Activations never leave registers.
struct FwdWeights {
    uint4 w1[8 * 64];       // row tile nt, k = the 4 inputs (lanes g = 0), rest 0
    uint4 w2[8 * 4 * 64];   // row tile nt, k tile kt
    uint4 w3[4 * 64];       // k tile kt, rows 0..2, rest 0
    float4 b1[32], b2[32];  // biases by four neurons
};

// silu(z) as the BF16 words of row tile nt
template <bool GUARD>
__device__ __forceinline__ void put_silu(uint32_t (&h)[16], int nt, const float4v& z) {
    h[2 * nt] = pk_bf(silu<GUARD>(z[0]), silu<GUARD>(z[1]));
    h[2 * nt + 1] = pk_bf(silu<GUARD>(z[2]), silu<GUARD>(z[3]));
}

__device__ __forceinline__ uint4 pk8(const float4& u, const float4& v) {
    return make_uint4(pk_bf(u.x, u.y), pk_bf(u.z, u.w), pk_bf(v.x, v.y), pk_bf(v.z, v.w));
}

__device__ __forceinline__ int tile_neuron(int nt, int g) {
    return 32 * (nt >> 1) + 8 * g + 4 * (nt & 1);
}
// neuron of row r of row tile nt
__device__ __forceinline__ int row_neuron(int nt, int r) { return tile_neuron(nt, r >> 2) + (r & 3); }

__device__ __forceinline__ void stage_fwd(const float* P, FwdWeights& S) {
    const int tid = (int)threadIdx.x, nthr = (int)blockDim.x;
    const float4* W2 = reinterpret_cast<const float4*>(P + oW2);
    // all of a thread's loads of W2 before its conversions
    constexpr int kU = 8;
    for (int d0 = tid; d0 < 2048; d0 += kU * nthr) {
        float4 u[kU], v[kU];
#pragma unroll
        for (int j = 0; j < kU; ++j) {
            const int d = d0 + j * nthr;
            if (d < 2048) {
                const int f = d >> 6, l = d & 63;
                const int n = row_neuron(f >> 2, l & 15), q = 8 * (f & 3) + 2 * (l >> 4);
                u[j] = W2[n * 32 + q];
                v[j] = W2[n * 32 + q + 1];
            }
        }
#pragma unroll
        for (int j = 0; j < kU; ++j) {
            const int d = d0 + j * nthr;
            if (d < 2048) S.w2[d] = pk8(u[j], v[j]);
        }
    }
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int d = tid; d < 512; d += nthr) {
        const int l = d & 63;
        const bool in = l < 16;
        S.w1[d] = pk8(in ? reinterpret_cast<const float4*>(P + oW1)[row_neuron(d >> 6, l)] : zero, zero);
    }
    for (int d = tid; d < 256; d += nthr) {
        const int l = d & 63, n = l & 15, q = 8 * (d >> 6) + 2 * (l >> 4);
        const float4* W3 = reinterpret_cast<const float4*>(P + oW3);
        const bool in = n < kOut;
        S.w3[d] = pk8(in ? W3[n * 32 + q] : zero, in ? W3[n * 32 + q + 1] : zero);
    }
    for (int d = tid; d < 64; d += nthr)
        (d < 32 ? S.b1 : S.b2)[d & 31] =
            reinterpret_cast<const float4*>(P + (d < 32 ? ob1 : ob2))[d & 31];
}

// Input and output scaling of spinmc_mlp_predict (null pointers: none).
struct Affine {
    const float *lo, *hi, *mu, *sd;
};

__device__ __forceinline__ float4 load_x(const float* x, size_t s, bool vec) {
    const float* p = x + 4 * s;
    return vec ? *reinterpret_cast<const float4*>(p) : make_float4(p[0], p[1], p[2], p[3]);
}

__device__ __forceinline__ void store_act(float* p, const float4v& z, bool vec) {
    if (vec) {
        *reinterpret_cast<float4v*>(p) = z;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = z[i];
    }
}

__device__ __forceinline__ float4v plus(const float4v& z, const float4& b) {
    return float4v{z[0] + b.x, z[1] + b.y, z[2] + b.z, z[3] + b.w};
}

// The lane, and the end of a row tile.  GUARD is a repetition behind a branch that is
// hardly ever taken: the lane is opaque and the tiles stay in sequence, since otherwise
// the compiler keeps the first run's operands for it, in twice the registers.
template <bool GUARD>
__device__ __forceinline__ int own_lane() {
    int l = (int)threadIdx.x & 63;
    if (GUARD) asm volatile("" : "+v"(l));
    return l;
}
template <bool GUARD>
__device__ __forceinline__ void tile_end() {
    if (GUARD) __builtin_amdgcn_sched_barrier(0);
}

// Both hidden layers for C tiles of 16 samples (lane l of tile c: sample
// s[c], neurons tile_neuron(nt, l / 16) + i): the pre-activations go to act if it
// is given, h2 receives the B operands of the output layer.
template <int C, bool GUARD>
__device__ __forceinline__ void hidden_layers(const FwdWeights& S, const uint4 (&xb)[C],
                                              const size_t (&s)[C], int B, float* act, bool vec,
                                              uint32_t (&h2)[C][16]) {
    const int l = own_lane<GUARD>(), g = l >> 4;
    uint32_t h1[C][16];
#pragma unroll
    for (int nt = 0; nt < 8; ++nt) {
        const int n0 = tile_neuron(nt, g);
        const float4 b = S.b1[n0 >> 2];
        const bf16x8 w = as_frag(S.w1[nt * 64 + l]);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const float4v z = plus(mfma(w, as_frag(xb[c]), float4v{0.f, 0.f, 0.f, 0.f}), b);
            if (act && s[c] < (size_t)B) store_act(act + s[c] * 2 * kH + n0, z, vec);
            put_silu<GUARD>(h1[c], nt, z);
        }
        tile_end<GUARD>();
    }
#pragma unroll
    for (int nt = 0; nt < 8; ++nt) {
        const int n0 = tile_neuron(nt, g);
        const float4 b = S.b2[n0 >> 2];
        float4v z[C];
#pragma unroll
        for (int c = 0; c < C; ++c) z[c] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) {
            const bf16x8 w = as_frag(S.w2[(nt * 4 + kt) * 64 + l]);
#pragma unroll
            for (int c = 0; c < C; ++c)
                z[c] = mfma(w, as_frag(make_uint4(h1[c][4 * kt], h1[c][4 * kt + 1], h1[c][4 * kt + 2],
                                                  h1[c][4 * kt + 3])), z[c]);
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            z[c] = plus(z[c], b);
            if (act && s[c] < (size_t)B) store_act(act + s[c] * 2 * kH + kH + n0, z[c], vec);
            put_silu<GUARD>(h2[c], nt, z[c]);
        }
        tile_end<GUARD>();
    }
}

// The same for one tile with the pre-activations kept.
__device__ __forceinline__ void hidden_layers_z(const FwdWeights& S, const uint4& xb, float4v (&z1)[8],
                                                float4v (&z2)[8], uint32_t (&h1)[16],
                                                uint32_t (&h2)[16]) {
    const int l = (int)threadIdx.x & 63, g = l >> 4;
#pragma unroll
    for (int nt = 0; nt < 8; ++nt) {
        z1[nt] = plus(mfma(as_frag(S.w1[nt * 64 + l]), as_frag(xb), float4v{0.f, 0.f, 0.f, 0.f}),
                      S.b1[tile_neuron(nt, g) >> 2]);
        put_silu<true>(h1, nt, z1[nt]);
    }
#pragma unroll
    for (int nt = 0; nt < 8; ++nt) {
        float4v z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
            z = mfma(as_frag(S.w2[(nt * 4 + kt) * 64 + l]),
                     as_frag(make_uint4(h1[4 * kt], h1[4 * kt + 1], h1[4 * kt + 2], h1[4 * kt + 3])), z);
        z2[nt] = plus(z, S.b2[tile_neuron(nt, g) >> 2]);
        put_silu<true>(h2, nt, z2[nt]);
    }
}

// Output layer: lanes 0..15 hold the three outputs of their sample.
__device__ __forceinline__ float4v output_layer(const FwdWeights& S, const uint32_t (&h2)[16]) {
    const int l = (int)threadIdx.x & 63;
    float4v y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
        y = mfma(as_frag(S.w3[kt * 64 + l]),
                 as_frag(make_uint4(h2[4 * kt], h2[4 * kt + 1], h2[4 * kt + 2], h2[4 * kt + 3])), y);
    return y;
}

}  // namespace

namespace {

// The tile groups of a wave, from q on in steps of dq.  Returns true in a lane whose
// outputs hold a NaN.
template <int C, bool AFF, bool GUARD>
__device__ __forceinline__ bool forward_tiles(const FwdWeights& S, const float* P, const float* x,
                                              int B, float* y, float* act, const Affine& af, int q,
                                              int dq) {
    const int l = own_lane<GUARD>(), g = l >> 4;
    const bool vec = ((uintptr_t)x & 15u) == 0, avec = ((uintptr_t)act & 15u) == 0;
    const float bo[3] = {P[ob3], P[ob3 + 1], P[ob3 + 2]};
    const int groups = (B - 1) / (16 * C) + 1;  // (no sum that passes 32 bits)
    float sum = 0.f;  // of the outputs before the scaling: NaN if any is
    // the first run of one tile a wave (C = 1) needs no loop: the grid covers the samples
    do {
        uint4 xb[C];
        size_t s[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            s[c] = (size_t)(q * C + c) * 16 + (l & 15);
            xb[c] = make_uint4(0u, 0u, 0u, 0u);
            if (g == 0 && s[c] < (size_t)B) {
                float4 v = load_x(x, s[c], vec);
                if (AFF) {
                    v.x = 2.0f * (v.x - af.lo[0]) / (af.hi[0] - af.lo[0]) - 1.0f;
                    v.y = 2.0f * (v.y - af.lo[1]) / (af.hi[1] - af.lo[1]) - 1.0f;
                    v.z = 2.0f * (v.z - af.lo[2]) / (af.hi[2] - af.lo[2]) - 1.0f;
                    v.w = 2.0f * (v.w - af.lo[3]) / (af.hi[3] - af.lo[3]) - 1.0f;
                }
                xb[c].x = pk_bf(v.x, v.y);
                xb[c].y = pk_bf(v.z, v.w);
            }
        }
        uint32_t h2[C][16];
        hidden_layers<C, GUARD>(S, xb, s, B, act, avec, h2);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const float4v o = output_layer(S, h2[c]);
            if (g == 0 && s[c] < (size_t)B) {
#pragma unroll
                for (int j = 0; j < kOut; ++j) {
                    float v = o[j] + bo[j];
                    sum += 0.0f * v;
                    if (AFF) v = v * af.sd[j] + af.mu[j];
                    y[s[c] * kOut + j] = v;
                }
            }
        }
        q += dq;
    } while ((GUARD || C > 1) && q < groups);
    return sum != sum;
}

}  // namespace

// A wave takes C tiles of 16 samples at a time, tile groups strided over the
// launch's waves, so that the weights are staged once per workgroup.  Bound
// by vector issue, most of it the SiLUs (256 a sample): at 10^5 points 391
// workgroups share 256 units, and a unit with two issues for 12.9 of the 14.1
// us that its waves live; the matrix instructions take 2.3 of them.  82 us
// with a workgroup (and its own staging and conversion of the weights) per 64
// samples and activations through LDS; a call of predict 26.8 with divisions
// in the SiLUs, 21.3 now.
// Registers for four waves a SIMD: the two workgroups a unit that the grid asks for.
template <int C, bool AFF>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4)))
k_mlp_fwd(const float* P, const float* x, int B, float* y, float* act, Affine af) {
    __shared__ FwdWeights S;
    stage_fwd(P, S);
    __syncthreads();
    const int waves = (int)blockDim.x >> 6;
    const int q = (int)blockIdx.x * waves + ((int)threadIdx.x >> 6), dq = (int)gridDim.x * waves;
    if (q > (B - 1) / (16 * C)) return;
    // a wave with a NaN repeats its tiles with the guard
    if (__any(forward_tiles<C, AFF, false>(S, P, x, B, y, act, af, q, dq)))
        for (int t = q * C; t < q * C + C && t <= (B - 1) / 16; ++t)
            forward_tiles<1, AFF, true>(S, P, x, B, y, act, af, t, dq * C);
}

// -------------------------------------------------------------- backward
namespace {

// FP32 buffer of one value per (sample, neuron): row stride 144, so that the
// 16 neurons x 4 samples of an FP32 MFMA operand read 64 different banks.
constexpr int kSF = kH + 16;

struct BwdShared {
    union {
        FwdWeights f;
        float h2[kSamplesPerWG * kSF];  // after the forward: bf16(silu z2) as FP32
    };
    uint4 w2t[8 * 4 * 64];                   // W2^T operands (rows: layer-1 neurons)
    float4 w3[kOut][kH / 4];                 // bf16(W3) as FP32
    float ba[kSamplesPerWG][16];             // [bf16(x) (4) | 1 | dY (3) | 0 ...]
    uint16_t h1t[kH * kST], dz2t[kH * kST];  // [neuron][sample] as BF16
    float dz[kSamplesPerWG * kSF];           // dz2, then dz1
    float loss[4];
};

__device__ __forceinline__ void stage_w2t(const float* P, uint4* w2t) {
    const float4* W2 = reinterpret_cast<const float4*>(P + oW2);
    // task: layer-1 neurons 4 m .. + 3 against layer-2 neurons 8 o8 .. + 7
    for (int q = (int)threadIdx.x; q < 32 * 16; q += (int)blockDim.x) {
        const int m = q & 31, o8 = q >> 5;
        float4 v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = W2[(8 * o8 + j) * 32 + m];
        const int kt = o8 >> 2, g = o8 & 3;
        const int nt = 2 * (m >> 3) + (m & 1), r = 4 * ((m >> 1) & 3);
        uint4* d = w2t + (nt * 4 + kt) * 64 + r + 16 * g;
        d[0] = make_uint4(pk_bf(v[0].x, v[1].x), pk_bf(v[2].x, v[3].x), pk_bf(v[4].x, v[5].x),
                          pk_bf(v[6].x, v[7].x));
        d[1] = make_uint4(pk_bf(v[0].y, v[1].y), pk_bf(v[2].y, v[3].y), pk_bf(v[4].y, v[5].y),
                          pk_bf(v[6].y, v[7].y));
        d[2] = make_uint4(pk_bf(v[0].z, v[1].z), pk_bf(v[2].z, v[3].z), pk_bf(v[4].z, v[5].z),
                          pk_bf(v[6].z, v[7].z));
        d[3] = make_uint4(pk_bf(v[0].w, v[1].w), pk_bf(v[2].w, v[3].w), pk_bf(v[4].w, v[5].w),
                          pk_bf(v[6].w, v[7].w));
    }
}

__device__ __forceinline__ float bf_lo(uint32_t v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float bf_hi(uint32_t v) { return __uint_as_float(v & 0xFFFF0000u); }

// Sums over the workgroup's 64 samples of v[sample][neuron] ba[sample][col]
// for the wave's neuron tile, on FP32 matrix instructions: lane l holds
// neurons 16 tile + 4 (l / 16) + i of column l % 16.
__device__ __forceinline__ float4v sample_sums(const float* v, const float (&ba)[16], int tile) {
    const int l = (int)threadIdx.x & 63;
    const float* p = v + (l >> 4) * kSF + 16 * tile + (l & 15);
    float4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 16; ++k)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(p[4 * k * kSF], ba[k], acc, 0, 0, 0);
    return acc;
}

}  // namespace

// Partial gradients of 64 samples into part[wg][kNP + 1] (last: loss) and
// input gradients dx (optional).  FWD: the forward of the same samples first
// (a training step's one pass: pre-activations stay in registers and go to
// act on the side); otherwise they come from act.  Four waves, 16 samples
// each, in the forward's layout (a lane: one sample, eight groups of four
// neurons): dz2 packed as BF16 is its own operand of dH1 = W2^T dz2; only
// dW2, whose sum runs over samples, needs [neuron][sample] copies in LDS, and
// the sums that stay FP32 (dW1, dW3 and the biases) run on FP32 matrix
// instructions against one [sample][x | 1 | dY] table.  A step of 1024
// samples is 16 workgroups, one chain of latencies each: forward and backward
// as two launches with VALU sums and LDS activations 17.2 + 31.9 us, now 20.0.
template <bool FWD>
__global__ void __launch_bounds__(256) k_mlp_bwd(const float* P, const float* x, float* act,
                                                 const float* t, const float* w, int B,
                                                 float* part, float* dx) {
    __shared__ BwdShared S;
    const int tid = (int)threadIdx.x, wave = tid >> 6, l = tid & 63, g = l >> 4, sl = l & 15;
    const int base = (int)blockIdx.x * kSamplesPerWG;
    const bool vec = ((uintptr_t)x & 15u) == 0, avec = ((uintptr_t)act & 15u) == 0;
    const int row = 16 * wave + sl;  // the lane's sample within the workgroup
    const size_t s[1] = {(size_t)base + row};
    const bool in = s[0] < (size_t)B;
    float4 xv = make_float4(0.f, 0.f, 0.f, 0.f);
    float tv[kOut] = {0.f, 0.f, 0.f}, wv[kOut], bo[kOut];
    if (in) {
        xv = load_x(x, s[0], vec);
#pragma unroll
        for (int j = 0; j < kOut; ++j) tv[j] = t[s[0] * kOut + j];
    }
#pragma unroll
    for (int j = 0; j < kOut; ++j) {
        wv[j] = w[j];
        bo[j] = P[ob3 + j];
    }
    stage_fwd(P, S.f);
    stage_w2t(P, S.w2t);
    for (int d = tid; d < kOut * kH / 4; d += 256) {
        const float4 v = reinterpret_cast<const float4*>(P + oW3)[d];
        const uint32_t a = pk_bf(v.x, v.y), b = pk_bf(v.z, v.w);
        (&S.w3[0][0])[d] = make_float4(bf_lo(a), bf_hi(a), bf_lo(b), bf_hi(b));
    }
    __syncthreads();
    // pre-activations of both layers, neurons tile_neuron(nt, g) + i
    float4v z1[8], z2[8];
    uint32_t h1[16], h2[16];
    const uint32_t xa = pk_bf(xv.x, xv.y), xc = pk_bf(xv.z, xv.w);
    if (FWD) {
        const uint4 xb[1] = {g == 0 ? make_uint4(xa, xc, 0u, 0u) : make_uint4(0u, 0u, 0u, 0u)};
        hidden_layers_z(S.f, xb[0], z1, z2, h1, h2);
#pragma unroll
        for (int nt = 0; nt < 8; ++nt) {
            if (!in) break;
            store_act(act + s[0] * 2 * kH + tile_neuron(nt, g), z1[nt], avec);
            store_act(act + s[0] * 2 * kH + kH + tile_neuron(nt, g), z2[nt], avec);
        }
    } else {
#pragma unroll
        for (int nt = 0; nt < 8; ++nt) {
            z1[nt] = z2[nt] = float4v{0.f, 0.f, 0.f, 0.f};
            if (in) {
                z1[nt] = *reinterpret_cast<const float4v*>(act + s[0] * 2 * kH + tile_neuron(nt, g));
                z2[nt] = *reinterpret_cast<const float4v*>(act + s[0] * 2 * kH + kH + tile_neuron(nt, g));
            }
        }
#pragma unroll
        for (int nt = 0; nt < 8; ++nt) {
            put_silu<true>(h1, nt, z1[nt]);
            put_silu<true>(h2, nt, z2[nt]);
        }
    }
    if (!in) {  // samples past B: nothing to add
#pragma unroll
        for (int k = 0; k < 16; ++k) h1[k] = h2[k] = 0u;
    }
    // outputs (lanes g = 0), dY and the loss
    const float4v o = output_layer(S.f, h2);
    float dY[kOut], lossp = 0.f;
#pragma unroll
    for (int j = 0; j < kOut; ++j) {
        const float e = (o[j] + bo[j]) - tv[j];
        if (g == 0 && in) lossp += wv[j] * e * e;
        const float d = in ? 2.0f * wv[j] * e / (float)B : 0.f;
        dY[j] = __shfl(d, sl, 64);  // the sample's lane of g = 0
    }
    for (int k = 8; k >= 1; k >>= 1) lossp += __shfl_xor(lossp, k, 64);
    if (l == 0) S.loss[wave] = lossp;
    if (g == 0) {
        float4* r = reinterpret_cast<float4*>(S.ba[row]);
        r[0] = make_float4(bf_lo(xa), bf_hi(xa), bf_lo(xc), bf_hi(xc));
        r[1] = make_float4(1.0f, dY[0], dY[1], dY[2]);
        r[2] = r[3] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();  // the forward's operands are free from here
    // dz2 = (W3b^T dY) silu'(z2)
    uint32_t dzb[16];
#pragma unroll
    for (int nt = 0; nt < 8; ++nt) {
        const int n0 = tile_neuron(nt, g);
        float4 v[kOut];
#pragma unroll
        for (int j = 0; j < kOut; ++j) v[j] = S.w3[j][n0 >> 2];
        float4v d;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float dh = 0.f;
#pragma unroll
            for (int j = 0; j < kOut; ++j)
                dh += dY[j] * (i == 0 ? v[j].x : (i == 1 ? v[j].y : (i == 2 ? v[j].z : v[j].w)));
            d[i] = in ? dh * dsilu(z2[nt][i]) : 0.f;
        }
        *reinterpret_cast<float4v*>(S.dz + row * kSF + n0) = d;
        dzb[2 * nt] = pk_bf(d[0], d[1]);
        dzb[2 * nt + 1] = pk_bf(d[2], d[3]);
        *reinterpret_cast<float4*>(S.h2 + row * kSF + n0) =
            make_float4(bf_lo(h2[2 * nt]), bf_hi(h2[2 * nt]), bf_lo(h2[2 * nt + 1]),
                        bf_hi(h2[2 * nt + 1]));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int sh = 16 * (i & 1);
            S.h1t[(n0 + i) * kST + row] = (uint16_t)(h1[2 * nt + (i >> 1)] >> sh);
            S.dz2t[(n0 + i) * kST + row] = (uint16_t)(dzb[2 * nt + (i >> 1)] >> sh);
        }
    }
    __syncthreads();
    float* pg = part + (size_t)blockIdx.x * (kNP + 1);
    float ba[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) ba[k] = S.ba[4 * k + g][sl];
    // dW3 (columns 5..7 against h2), db2 (column 4 against dz2)
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const int tile = 2 * wave + m;
        const float4v a3 = sample_sums(S.h2, ba, tile), a2 = sample_sums(S.dz, ba, tile);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int n = 16 * tile + 4 * g + i;
            if (sl >= 5 && sl < 8) pg[oW3 + (sl - 5) * kH + n] = a3[i];
            if (sl == 4) pg[ob2 + n] = a2[i];
        }
    }
    if (wave == 0) {  // db3: columns 5..7 against ones
        float4v a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 16; ++k)
            a = __builtin_amdgcn_mfma_f32_16x16x4f32(1.0f, ba[k], a, 0, 0, 0);
        if (g == 0 && sl >= 5 && sl < 8) pg[ob3 + sl - 5] = a[0];
    }
    // dW2 = dz2b^T h1 (M = out neuron, N = in neuron, K = 64 samples): wave
    // owns out-tiles 2*wave, 2*wave+1
    for (int mt = 2 * wave; mt < 2 * wave + 2; ++mt) {
#pragma unroll
        for (int nt = 0; nt < kH / 16; ++nt) {
            float4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kt = 0; kt < kSamplesPerWG / 32; ++kt)
                acc = mfma(frag(S.dz2t + mt * 16 * kST, kST, 32 * kt),
                           frag(S.h1t + nt * 16 * kST, kST, 32 * kt), acc);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                pg[oW2 + (mt * 16 + 4 * g + i) * kH + nt * 16 + sl] = acc[i];
        }
    }
    // dH1 = W2b^T dz2b, dz1 = dH1 silu'(z1)
    float4v d1[8];
#pragma unroll
    for (int nt = 0; nt < 8; ++nt) {
        float4v acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
            acc = mfma(as_frag(S.w2t[(nt * 4 + kt) * 64 + l]),
                       as_frag(make_uint4(dzb[4 * kt], dzb[4 * kt + 1], dzb[4 * kt + 2],
                                          dzb[4 * kt + 3])), acc);
#pragma unroll
        for (int i = 0; i < 4; ++i) d1[nt][i] = in ? acc[i] * dsilu(z1[nt][i]) : 0.f;
    }
    if (dx) {
        // each lane its 32 neurons, then the four lanes of the sample
        float v[kIn] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int nt = 0; nt < 8; ++nt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float4 q = reinterpret_cast<const float4*>(P + oW1)[tile_neuron(nt, g) + i];
                const uint32_t a = pk_bf(q.x, q.y), b = pk_bf(q.z, q.w);
                v[0] += d1[nt][i] * bf_lo(a);
                v[1] += d1[nt][i] * bf_hi(a);
                v[2] += d1[nt][i] * bf_lo(b);
                v[3] += d1[nt][i] * bf_hi(b);
            }
#pragma unroll
        for (int k = 0; k < kIn; ++k) {
            v[k] += __shfl_xor(v[k], 16, 64);
            v[k] += __shfl_xor(v[k], 32, 64);
            if (g == 0 && in) dx[s[0] * kIn + k] = v[k];
        }
    }
    __syncthreads();  // every wave has read dz2
#pragma unroll
    for (int nt = 0; nt < 8; ++nt)
        *reinterpret_cast<float4v*>(S.dz + row * kSF + tile_neuron(nt, g)) = d1[nt];
    __syncthreads();
    // dW1 (columns 0..3), db1 (column 4)
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const int tile = 2 * wave + m;
        const float4v a1 = sample_sums(S.dz, ba, tile);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int n = 16 * tile + 4 * g + i;
            if (sl < kIn) pg[oW1 + n * kIn + sl] = a1[i];
            if (sl == 4) pg[ob1 + n] = a1[i];
        }
    }
    if (tid == 0) pg[kNP] = (S.loss[0] + S.loss[1] + S.loss[2] + S.loss[3]) / (float)B;
}

// Sum of the per-workgroup partials of entry i in their order, 16 loads in
// flight at a time.
__device__ __forceinline__ float partial_sum(const float* part, int n_wg, int i) {
    float s = 0.f;
    for (int g0 = 0; g0 < n_wg; g0 += 16) {
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u)
            v[u] = g0 + u < n_wg ? part[(size_t)(g0 + u) * (kNP + 1) + i] : 0.f;
#pragma unroll
        for (int u = 0; u < 16; ++u)
            if (g0 + u < n_wg) s += v[u];
    }
    return s;
}

// Fixed-order sum of the per-workgroup partials.
__global__ void k_mlp_reduce(const float* part, int n_wg, float* grad, float* loss) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i > kNP) return;
    const float s = partial_sum(part, n_wg, i);
    if (i < kNP)
        grad[i] = s;
    else if (loss)
        *loss = s;
}

__global__ void k_mlp_adam(float* p, const float* g, float* m, float* v, int n, float lr, float b1,
                           float b2, float eps, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float mh = mi / c1, vh = vi / c2;
    p[i] -= lr * mh / (sqrtf(vh) + eps);
}

// The fixed-order sum of k_mlp_reduce and the Adam update of k_mlp_adam in
// one pass over the parameters (the same arithmetic in the same order).
__global__ void k_mlp_reduce_adam(const float* part, int n_wg, float* grad, float* loss,
                                  float* p, float* m, float* v, float lr, float b1, float b2,
                                  float eps, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i > kNP) return;
    const float gi = partial_sum(part, n_wg, i);
    if (i == kNP) {
        if (loss) *loss = gi;
        return;
    }
    if (grad) grad[i] = gi;
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float mh = mi / c1, vh = vi / c2;
    p[i] -= lr * mh / (sqrtf(vh) + eps);
}

// Few samples: one tile a wave, four waves a workgroup, as many workgroups as
// the samples need (the chip is not filled and latency counts).  From 32768
// samples (two such workgroups on every CU) two tiles a wave share each
// weight operand read from LDS, and 512 workgroups of eight waves stride over
// the samples.
static hipError_t launch_fwd(const float* params, const float* x, int B, float* y, float* act,
                             const Affine* af, hipStream_t s) {
    const Affine none{nullptr, nullptr, nullptr, nullptr};
    if (B < 32768) {
        const dim3 g((B + 63) / 64), b(256);
        if (af)
            hipLaunchKernelGGL((k_mlp_fwd<1, true>), g, b, 0, s, params, x, B, y, act, *af);
        else
            hipLaunchKernelGGL((k_mlp_fwd<1, false>), g, b, 0, s, params, x, B, y, act, none);
    } else {
        const int64_t need = ((int64_t)B + 255) / 256;
        const dim3 g((unsigned)(need < 512 ? need : 512)), b(512);
        if (af)
            hipLaunchKernelGGL((k_mlp_fwd<2, true>), g, b, 0, s, params, x, B, y, act, *af);
        else
            hipLaunchKernelGGL((k_mlp_fwd<2, false>), g, b, 0, s, params, x, B, y, act, none);
    }
    return hipGetLastError();
}

hipError_t launch_mlp_train_step(float* params, const float* x, const float* t, const float* w,
                                 int B, float* grad, float* m, float* v, int step, float lr,
                                 float b1, float b2, float eps, float* loss, float* act,
                                 float* scratch, hipStream_t s) {
    const int g = (B + kSamplesPerWG - 1) / kSamplesPerWG;
    hipLaunchKernelGGL(k_mlp_bwd<true>, dim3(g), dim3(256), 0, s, params, x, act, t, w, B, scratch,
                       (float*)nullptr);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const float c1 = (float)(1.0 - std::pow((double)b1, (double)step));
    const float c2 = (float)(1.0 - std::pow((double)b2, (double)step));
    hipLaunchKernelGGL(k_mlp_reduce_adam, dim3((kNP + 1 + 255) / 256), dim3(256), 0, s, scratch, g,
                       grad, loss, params, m, v, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t launch_mlp_forward(const float* params, const float* x, int B, float* y, float* act,
                              hipStream_t s) {
    return launch_fwd(params, x, B, y, act, nullptr, s);
}

hipError_t launch_mlp_predict(const float* params, const float* x, int B, const float* xlo,
                              const float* xhi, const float* ymu, const float* ysd, float* y,
                              hipStream_t s) {
    const Affine af{xlo, xhi, ymu, ysd};
    return launch_fwd(params, x, B, y, nullptr, &af, s);
}

hipError_t launch_mlp_backward(const float* params, const float* x, const float* act,
                               const float* t, const float* w, int B, float* grad, float* dx,
                               float* loss, float* scratch, hipStream_t s) {
    const int g = (B + kSamplesPerWG - 1) / kSamplesPerWG;
    hipLaunchKernelGGL(k_mlp_bwd<false>, dim3(g), dim3(256), 0, s, params, x, const_cast<float*>(act),
                       t, w, B, scratch, dx);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_mlp_reduce, dim3((kNP + 1 + 255) / 256), dim3(256), 0, s, scratch, g,
                       grad, loss);
    return hipGetLastError();
}

hipError_t launch_mlp_adam(float* params, const float* grad, float* m, float* v, int n, int step,
                           float lr, float b1, float b2, float eps, hipStream_t s) {
    const float c1 = (float)(1.0 - std::pow((double)b1, (double)step));
    const float c2 = (float)(1.0 - std::pow((double)b2, (double)step));
    hipLaunchKernelGGL(k_mlp_adam, dim3((n + 255) / 256), dim3(256), 0, s, params, grad, m, v, n,
                       lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

int mlp_num_params() { return kNP; }
int mlp_scratch_floats(int B) { return ((B + kSamplesPerWG - 1) / kSamplesPerWG) * (kNP + 1); }

}  // namespace spinmc
