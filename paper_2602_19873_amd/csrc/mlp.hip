// Learned smoothing-length seed: features, an 8 -> 64 -> 64 -> 1 ReLU MLP on
// the bf16 matrix cores (FP32 accumulate), its gradient and Adam. The network
// output is added to the cube-root rule's step, -feature0 / 3, so an untrained
// network reproduces the plain rule.
//
// Matrix-core layout (v_mfma_f32_16x16x16_bf16, wave64): for lane l with
// s = l % 16 and g = l / 16, the A operand holds A[s][4g .. 4g+3], the B
// operand B[4g .. 4g+3][s], and the accumulator D[4g .. 4g+3][s]. Activations
// are kept transposed (units x samples), so a layer's accumulator fragment is
// directly the next layer's B operand: W1 X^T, then W2 H1^T, 16 samples per
// tile. The backward pass forms W2^T delta2 the same way; the two weight
// gradients contract over samples and go through a per-wave LDS transpose.
#include "internal.h"

namespace sfcnl {
namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kIn = SFCNL_HSEED_NFEAT;  // 8 features
constexpr int kHid = 64;
constexpr int kOffW1 = 0, kOffB1 = 512, kOffW2 = 576, kOffB2 = 4672, kOffW3 = 4736, kOffB3 = 4800;
constexpr int kNParam = SFCNL_MLP_NPARAM;  // 4801
constexpr int kWaves = 4;
constexpr int kInferBlocks = 512;  // inference: two blocks per CU share the samples (256: 3 % slower, 1,024: 1 %)
constexpr int kRedWords = 4 * (16 + 16) + 2;  // registers of a wave's partial gradient and loss
// Row stride of the 64-wide weight rows in LDS: 34 words, so that the 16 rows
// of a fragment read lie on different banks (64 shorts: all on one).
constexpr int kRowW = kHid + 4;

// float -> bfloat16, round to nearest even (NaN stays NaN)
__device__ __forceinline__ short f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (short)0x7FC0;
    return (short)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ float bf2f(short b) { return __uint_as_float((uint32_t)(uint16_t)b << 16); }
__device__ __forceinline__ float qbf(float f) { return bf2f(f2bf(f)); }

__device__ __forceinline__ f32x4 mfma(bf16x4 a, bf16x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// Weights of one block, rounded to bf16 once.
struct WeightsLds {
    short W1[kHid * 16];     // [unit][feature], features 8..15 zero
    short W2[kHid * kRowW];   // [out unit][in unit]
    short W2T[kHid * kRowW];  // [in unit][out unit]
    float b1[kHid], b2[kHid], w3q[kHid];
    float b3;
};

// (256 threads; every load is in flight before the first is used)
__device__ __forceinline__ void load_weights(WeightsLds &L, const float *__restrict__ p) {
    constexpr int kT = 256;
    const int t = threadIdx.x;
    float w1[kHid * kIn / kT], w2[kHid * kHid / kT];
#pragma unroll
    for (int k = 0; k < kHid * kHid / kT; k++) w2[k] = p[kOffW2 + k * kT + t];
#pragma unroll
    for (int k = 0; k < kHid * kIn / kT; k++) w1[k] = p[kOffW1 + k * kT + t];
    const float v1 = p[kOffB1 + (t & 63)], v2 = p[kOffB2 + (t & 63)], v3 = p[kOffW3 + (t & 63)], v4 = p[kOffB3];
#pragma unroll
    for (int k = 0; k < kHid * kHid / kT; k++) {
        const int e = k * kT + t, u = e / kHid, f = e % kHid;
        const short w = f2bf(w2[k]);
        L.W2[u * kRowW + f] = w;
        L.W2T[f * kRowW + u] = w;
    }
#pragma unroll
    for (int k = 0; k < kHid * kIn / kT; k++) {
        const int e = k * kT + t, u = e / kIn, f = e % kIn;
        L.W1[u * 16 + f] = f2bf(w1[k]);
        L.W1[u * 16 + kIn + f] = 0;
    }
    if (t < kHid) {
        L.b1[t] = v1;
        L.b2[t] = v2;
        L.w3q[t] = qbf(v3);
    }
    if (t == 0) L.b3 = v4;
    __syncthreads();
}

__device__ __forceinline__ bf16x4 lds4(const short *p) { return *reinterpret_cast<const bf16x4 *>(p); }

// Features of sample s as the B operand (lanes g = 0, 1 carry features
// 4g .. 4g+3; the K padding 8..15 is zero).
__device__ __forceinline__ bf16x4 load_x(const uint16_t *__restrict__ feat, int64_t idx, bool valid, int g) {
    bf16x4 x = {0, 0, 0, 0};
    if (valid && g < 2) {
        const uint2 w = *reinterpret_cast<const uint2 *>(feat + idx * kIn + 4 * g);
        x[0] = (short)(w.x & 0xFFFFu);
        x[1] = (short)(w.x >> 16);
        x[2] = (short)(w.y & 0xFFFFu);
        x[3] = (short)(w.y >> 16);
    }
    return x;
}

struct Fwd {
    f32x4 z1[4], z2[4];  // pre-activations (with bias)
    bf16x4 h1[4];        // relu(z1) in bf16: B operands of layer 2
    f32x4 h2[4];         // relu(z2) rounded to bf16
    float y;             // output of sample s (same in the 4 lanes of s)
};

__device__ __forceinline__ void forward_tile(const WeightsLds &L, bf16x4 x, int s, int g, Fwd &F) {
    // x: this lane's B-operand slice of the sample features (see load_x)
#pragma unroll
    for (int mt = 0; mt < 4; mt++) {
        const f32x4 z = mfma(lds4(&L.W1[(mt * 16 + s) * 16 + 4 * g]), x, f32x4{0, 0, 0, 0});
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const float v = z[i] + L.b1[mt * 16 + 4 * g + i];
            F.z1[mt][i] = v;
            F.h1[mt][i] = f2bf(fmaxf(v, 0.0f));
        }
    }
    float part = 0.0f;
#pragma unroll
    for (int mt = 0; mt < 4; mt++) {
        f32x4 acc = {0, 0, 0, 0};
#pragma unroll
        for (int kt = 0; kt < 4; kt++) acc = mfma(lds4(&L.W2[(mt * 16 + s) * kRowW + kt * 16 + 4 * g]), F.h1[kt], acc);
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int u = mt * 16 + 4 * g + i;
            const float v = acc[i] + L.b2[u];
            F.z2[mt][i] = v;
            F.h2[mt][i] = qbf(fmaxf(v, 0.0f));
            part = __builtin_fmaf(L.w3q[u], F.h2[mt][i], part);
        }
    }
    part += __shfl_xor(part, 16, 64);
    part += __shfl_xor(part, 32, 64);
    // residual on the cube-root rule: -feature0 / 3 = log((target / (n+1))^(1/3));
    // lane s (g = 0) holds feature 0 of sample s
    const float f0 = __shfl(bf2f(x[0]), s, 64);
    F.y = part + L.b3 - f0 * (1.0f / 3.0f);
}

// Inference keeps its weights in registers: a wave loads its fragments once and
// runs groups of four 16-sample tiles through them, the next group's features
// loading behind this one's layers. The products of the hidden layers are those
// of forward_tile, in its order, so that every hidden activation rounds to the
// same bf16 value; relu and rounding take three vector instructions per two
// values, and the output layer is a product too (w3 in rows 0, 4, 8 and 12, so
// that each lane group has every output and lane l keeps sample l's). Before,
// every tile read its weights from LDS (all 16 rows of a fragment on one bank),
// rounded with six integer instructions per value and waited for its features:
// 77 -> 24 us for 1,000,003 samples.
union Frag4 {
    bf16x4 v;
    bf16x2_t p[2];
};

__device__ __forceinline__ bf16x2_t round2(float a, float b) {
    return __builtin_convertvector(f32x2{a, b}, bf16x2_t);
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_mlp_infer(
    const float *__restrict__ params, int64_t n, const uint16_t *__restrict__ feat, float *__restrict__ out) {
    const int lane = sfc_lane(), s = lane & 15, g = lane >> 4;
    const int64_t ngroups = (n + kWave - 1) / kWave;
    const int64_t wave = (int64_t)blockIdx.x * kWaves + threadIdx.x / kWave;
    const int64_t nw = (int64_t)gridDim.x * kWaves;
    if (wave >= ngroups) return;
    // features 4g .. 4g + 3 of sample s of each tile (groups 2 and 3: the padding)
    struct Group {
        uint2 f[4];
    };
    auto load = [&](int64_t t) {
        Group r;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int64_t idx = t * kWave + 16 * k + s;
            r.f[k] = *reinterpret_cast<const uint2 *>(feat + (idx < n ? idx : n - 1) * kIn + 4 * (g & 1));
        }
        return r;
    };
    Group next = load(wave);
    Frag4 w1[4], w2[4][4], w3[4];
    f32x4 b1[4], b2[4];
#pragma unroll
    for (int mt = 0; mt < 4; mt++) {
#pragma unroll
        for (int q = 0; q < 2; q++) {
            const float *r = params + kOffW1 + (mt * 16 + s) * kIn + 4 * (g & 1) + 2 * q;
            const bf16x2_t w = round2(r[0], r[1]);
            w1[mt].p[q] = g < 2 ? w : bf16x2_t{0, 0};
#pragma unroll
            for (int kt = 0; kt < 4; kt++) {
                const float *c = params + kOffW2 + (mt * 16 + s) * kHid + kt * 16 + 4 * g + 2 * q;
                w2[mt][kt].p[q] = round2(c[0], c[1]);
            }
            const float *o = params + kOffW3 + mt * 16 + 4 * g + 2 * q;
            const bf16x2_t v = round2(o[0], o[1]);
            w3[mt].p[q] = (s & 3) == 0 ? v : bf16x2_t{0, 0};
        }
#pragma unroll
        for (int i = 0; i < 4; i++) {
            b1[mt][i] = params[kOffB1 + mt * 16 + 4 * g + i];
            b2[mt][i] = params[kOffB2 + mt * 16 + 4 * g + i];
        }
    }
    const float b3 = params[kOffB3];
    // relu is the median of v, 0 and a register holding +inf: one instruction, 0
    // for NaN (a maximum, or a median of constants, would quiet v first)
    float inf = INFINITY;
    asm("" : "+v"(inf));
    auto activate = [&](f32x4 z, f32x4 b) {
        Frag4 f;
        f.p[0] = round2(__builtin_amdgcn_fmed3f(z[0] + b[0], 0.0f, inf), __builtin_amdgcn_fmed3f(z[1] + b[1], 0.0f, inf));
        f.p[1] = round2(__builtin_amdgcn_fmed3f(z[2] + b[2], 0.0f, inf), __builtin_amdgcn_fmed3f(z[3] + b[3], 0.0f, inf));
        return f;
    };
    for (int64_t t = wave; t < ngroups; t += nw) {
        const Group f = next;
        if (t + nw < ngroups) next = load(t + nw);
        float out_l = 0.0f;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const uint2 fk = f.f[k];
            const bf16x4 x = __builtin_bit_cast(bf16x4, make_uint2(g < 2 ? fk.x : 0u, g < 2 ? fk.y : 0u));
            Frag4 h[4];
#pragma unroll
            for (int mt = 0; mt < 4; mt++) h[mt] = activate(mfma(w1[mt].v, x, f32x4{0, 0, 0, 0}), b1[mt]);
            f32x4 y = {0, 0, 0, 0};
#pragma unroll
            for (int mt = 0; mt < 4; mt++) {
                f32x4 acc = {0, 0, 0, 0};
#pragma unroll
                for (int kt = 0; kt < 4; kt++) acc = mfma(w2[mt][kt].v, h[kt].v, acc);
                y = mfma(w3[mt].v, activate(acc, b2[mt]).v, y);
            }
            // residual on the cube-root rule: -feature0 / 3 = log((target / (n+1))^(1/3));
            // lane s of the tile (g = 0) holds feature 0 of sample s
            const float f0 = __shfl(__uint_as_float(fk.x << 16), s, kWave);
            const float r = y[0] + b3 - f0 * (1.0f / 3.0f);
            out_l = g == k ? r : out_l;
        }
        const int64_t idx = t * kWave + lane;
        if (idx < n) out[idx] = out_l;
    }
}

// Sum over the 16 lanes that share lane / 16 (DPP: quad swaps, then the
// mirrored half row and row).
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float row_sum(float v) {
    return dpp_add<0x140>(dpp_add<0x141>(dpp_add<0x4E>(dpp_add<0xB1>(v))));
}

// Gradient of the mean squared error over a batch: each wave accumulates its
// tiles, the block's four waves join theirs in LDS, and the block writes one
// partial gradient (kNParam floats) and partial loss. One tile per wave up to
// the block limit: at batch 8,192 128 blocks of one tile per wave and 128 rows
// for the reduction, against 64 blocks of two tiles per wave and 256 rows,
// whose lane sums went through LDS exchanges (192 per wave): 32 -> 18 us.
__global__ __launch_bounds__(256) void k_mlp_grad(const float *__restrict__ params, int64_t nsamp,
                                                  const uint16_t *__restrict__ feat, const float *__restrict__ target,
                                                  int64_t batch, int64_t start, int64_t mul, int64_t add,
                                                  float *__restrict__ partial) {
    __shared__ WeightsLds L;
    __shared__ short T1[kWaves][kHid * 16], T2[kWaves][kHid * 16], T3[kWaves][kHid * 16], TX[kWaves][16 * 16];
    load_weights(L, params);
    const int lane = sfc_lane(), s = lane & 15, g = lane >> 4;
    const int w = threadIdx.x / kWave;
    const int64_t ntiles = (batch + 15) / 16;
    const int64_t wave = (int64_t)blockIdx.x * kWaves + w;
    const int64_t nw = (int64_t)gridDim.x * kWaves;
    const float inv_b = 2.0f / (float)batch;

    f32x4 dW2[4][4], dW1[4];
    float dw3[4][4], db2[4][4], db1[4][4];
    float db3 = 0.0f, loss = 0.0f;
#pragma unroll
    for (int a = 0; a < 4; a++) {
        dW1[a] = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int b = 0; b < 4; b++) {
            dW2[a][b] = f32x4{0, 0, 0, 0};
            dw3[a][b] = db2[a][b] = db1[a][b] = 0.0f;
        }
    }
    for (int64_t t = wave; t < ntiles; t += nw) {
        const int64_t k = t * 16 + s;
        const bool v = k < batch;
        const int64_t idx = v ? (int64_t)(((unsigned __int128)(uint64_t)(start + k) * (uint64_t)mul + (uint64_t)add) %
                                          (uint64_t)nsamp)
                              : 0;
        const bf16x4 x = load_x(feat, idx, v, g);
        Fwd F;
        forward_tile(L, x, s, g, F);
        const float r = v ? F.y - target[idx] : 0.0f;
        if (g == 0) loss = __builtin_fmaf(r, r, loss);
        const float dy = r * inv_b;
        if (g == 0) db3 += dy;
        // layer 3 and the error entering layer 2
        bf16x4 d2b[4];
#pragma unroll
        for (int mt = 0; mt < 4; mt++) {
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int u = mt * 16 + 4 * g + i;
                dw3[mt][i] = __builtin_fmaf(dy, F.h2[mt][i], dw3[mt][i]);
                const float d2 = F.z2[mt][i] > 0.0f ? L.w3q[u] * dy : 0.0f;
                db2[mt][i] += d2;
                d2b[mt][i] = f2bf(d2);
            }
        }
        // error entering layer 1: W2^T delta2
        bf16x4 d1b[4];
#pragma unroll
        for (int mt = 0; mt < 4; mt++) {
            f32x4 acc = {0, 0, 0, 0};
#pragma unroll
            for (int kt = 0; kt < 4; kt++) acc = mfma(lds4(&L.W2T[(mt * 16 + s) * kRowW + kt * 16 + 4 * g]), d2b[kt], acc);
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const float d1 = F.z1[mt][i] > 0.0f ? acc[i] : 0.0f;
                db1[mt][i] += d1;
                d1b[mt][i] = f2bf(d1);
            }
        }
        // transposes for the contractions over samples
        short *t1 = T1[w], *t2 = T2[w], *t3 = T3[w], *tx = TX[w];
#pragma unroll
        for (int mt = 0; mt < 4; mt++) {
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int u = mt * 16 + 4 * g + i;
                t1[u * 16 + s] = F.h1[mt][i];
                t2[u * 16 + s] = d2b[mt][i];
                t3[u * 16 + s] = d1b[mt][i];
            }
        }
#pragma unroll
        for (int i = 0; i < 4; i++) tx[(4 * g + i) * 16 + s] = x[i];  // feature 4g+i of sample s (zero for g >= 2)
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // dW2[u2][u1] += sum_s delta2[u2][s] h1[u1][s]
#pragma unroll
        for (int mt = 0; mt < 4; mt++) {
            const bf16x4 a = lds4(&t2[(mt * 16 + s) * 16 + 4 * g]);
#pragma unroll
            for (int nt = 0; nt < 4; nt++) dW2[mt][nt] = mfma(a, lds4(&t1[(nt * 16 + s) * 16 + 4 * g]), dW2[mt][nt]);
        }
        // dW1[u1][f] += sum_s delta1[u1][s] x[f][s]
        const bf16x4 bx = lds4(&tx[s * 16 + 4 * g]);
#pragma unroll
        for (int mt = 0; mt < 4; mt++) dW1[mt] = mfma(lds4(&t3[(mt * 16 + s) * 16 + 4 * g]), bx, dW1[mt]);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    // sum the per-sample partials over the 16 lanes of each g
#pragma unroll
    for (int mt = 0; mt < 4; mt++) {
#pragma unroll
        for (int i = 0; i < 4; i++) {
            dw3[mt][i] = row_sum(dw3[mt][i]);
            db2[mt][i] = row_sum(db2[mt][i]);
            db1[mt][i] = row_sum(db1[mt][i]);
        }
    }
    for (int d = 1; d < 64; d <<= 1) {
        db3 += __shfl_xor(db3, d, 64);
        loss += __shfl_xor(loss, d, 64);
    }
    // join the waves' registers in LDS, register by register (the lane sums
    // once per row: lane 16 g holds registers i of group g)
    __shared__ float s_red[kWaves / 2][kRedWords][kWave];
    auto registers = [&](auto &&f) __attribute__((always_inline)) {
        int k = 0;
#pragma unroll
        for (int mt = 0; mt < 4; mt++) {
#pragma unroll
            for (int nt = 0; nt < 4; nt++)
#pragma unroll
                for (int i = 0; i < 4; i++) dW2[mt][nt][i] = f(k++, dW2[mt][nt][i]);
#pragma unroll
            for (int i = 0; i < 4; i++) {
                dW1[mt][i] = f(k++, dW1[mt][i]);
                dw3[mt][i] = f(k++, dw3[mt][i]);
                db2[mt][i] = f(k++, db2[mt][i]);
                db1[mt][i] = f(k++, db1[mt][i]);
            }
        }
        db3 = f(k++, db3);
        loss = f(k++, loss);
    };
    for (int half = kWaves / 2; half > 0; half >>= 1) {
        if (w >= half && w < 2 * half) registers([&](int k, float v) { return s_red[w - half][k][lane] = v; });
        __syncthreads();
        if (w < half) registers([&](int k, float v) { return v + s_red[w][k][lane]; });
        __syncthreads();
    }
    if (w != 0) return;
    float *out = partial + (int64_t)blockIdx.x * (kNParam + 1);
#pragma unroll
    for (int mt = 0; mt < 4; mt++) {
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int u = mt * 16 + 4 * g + i;
#pragma unroll
            for (int nt = 0; nt < 4; nt++) out[kOffW2 + u * kHid + nt * 16 + s] = dW2[mt][nt][i];
            if (s < kIn) out[kOffW1 + u * kIn + s] = dW1[mt][i];
            if (s == 0) {
                out[kOffW3 + u] = dw3[mt][i];
                out[kOffB2 + u] = db2[mt][i];
                out[kOffB1 + u] = db1[mt][i];
            }
        }
    }
    if (lane == 0) {
        out[kOffB3] = db3;
        out[kNParam] = loss;
    }
}

// Sum of the block partials; index kNParam is the loss (mean over the batch).
// A block takes 64 parameters, its four waves every fourth row each (eight rows
// in flight at a time), and joins the four sums in LDS: 76 blocks of four
// chains instead of 19 blocks whose threads each walked 256 rows one load after
// another (57 -> 4 us at batch 8,192).
__global__ __launch_bounds__(256) void k_mlp_reduce(const float *__restrict__ partial, int nrows, int64_t batch,
                                                    float *__restrict__ grad, float *__restrict__ loss) {
    __shared__ float s_sum[kWaves][kWave];
    const int lane = sfc_lane(), w = threadIdx.x / kWave;
    const int p = blockIdx.x * kWave + lane;
    const int pc = p <= kNParam ? p : kNParam;
    float acc = 0.0f;
    for (int r0 = w; r0 < nrows; r0 += 8 * kWaves) {
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int r = r0 + k * kWaves;
            v[k] = partial[(size_t)(r < nrows ? r : w) * (kNParam + 1) + pc];
        }
#pragma unroll
        for (int k = 0; k < 8; k++) acc += r0 + k * kWaves < nrows ? v[k] : 0.0f;
    }
    s_sum[w][lane] = acc;
    __syncthreads();
    if (w != 0 || p > kNParam) return;
    acc = (s_sum[0][lane] + s_sum[1][lane]) + (s_sum[2][lane] + s_sum[3][lane]);
    if (p < kNParam)
        grad[p] = acc;
    else if (loss)
        *loss = acc / (float)batch;
}

__global__ __launch_bounds__(256) void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                                              float *__restrict__ v, float lr, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kNParam) return;
    const float gi = g[i];
    const float mi = 0.9f * m[i] + 0.1f * gi;
    const float vi = 0.999f * v[i] + 0.001f * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + 1e-8f);
}

// splitmix64 (Steele, Lea & Flood 2014): one 64-bit output per counter value.
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
    uint64_t z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// He-uniform weights for the ReLU layers, small output weights, zero biases.
__global__ __launch_bounds__(256) void k_mlp_init(uint64_t seed, float *__restrict__ p) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kNParam) return;
    const double u = (double)(splitmix64(seed * 0x100000001B3ull + (uint64_t)i) >> 11) * 0x1.0p-53;  // [0, 1)
    float bound = 0.0f;
    if (i < kOffB1)
        bound = sqrtf(6.0f / kIn);
    else if (i >= kOffW2 && i < kOffB2)
        bound = sqrtf(6.0f / kHid);
    else if (i >= kOffW3 && i < kOffB3)
        bound = 0.1f * sqrtf(6.0f / kHid);
    p[i] = (float)((2.0 * u - 1.0) * bound);
}

// Features of particle i (SFC order), all dimensionless:
//   0 log((n_prev + 1) / target)
//   1 log(cluster box diagonal / h)        2 log(super-cluster box diagonal / h)
//   3..5 log((1 + occupancy) / target) of the particle's key-prefix cell at
//        levels L0 - 1, L0, L0 + 1, with L0 the level whose cell edge is
//        closest to h
//   6 log2(edge_0 / h) - L0 (where h falls between levels)
//   7 log(target / 100)
//
// The cells' ends are found by binary searches in the sorted keys. A cell around
// the particle lies in a narrow run of keys around it (mostly a few hundred at
// the coarsest level asked for), so each block stages the keys of its particles
// and kKeyPad to either side in LDS and searches there, the finer cells inside
// the coarser ones; ends beyond the window are searched in memory. (Searching the
// whole array, each step waited on a load: 67 -> 28 us for 1,000,000 uniform
// particles.) kFew: both ends of a cell in memory side by side, which pays while
// the GPU is not full: the core's cells of a condensed system mostly end beyond the
// window, and one search after the other took longer than searching everything in
// memory (Plummer spheres of 30,000 / 100,000 particles 13.9 / 16.6 us then, 15.4 /
// 16.6 one after the other, 13.7 / 14.5 side by side; with the network, uniform
// systems of 1,000,003 64.3 us one after the other, 66.7 side by side).
constexpr int kFeatThreads = 256;
constexpr int kKeyPad = 896;  // 2,048 keys in LDS: 16 KB

// first index in [lo, hi) whose key is not below v
template <typename F>
__device__ __forceinline__ uint32_t lower_bound_key(F &&key, uint32_t lo, uint32_t hi, uint64_t v) {
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (key(mid) < v)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// Two searches side by side, so that each step's two loads are in flight
// together: a.lo becomes the first index in [a.lo, a.hi) whose key is not below
// a.v (a.hi if none is), and b.lo likewise. `own`: an index that may be read.
struct KeySearch {
    uint32_t lo, hi;
    uint64_t v;
};
template <typename F>
__device__ __forceinline__ void lower_bounds(F &&key, KeySearch &a, KeySearch &b, uint32_t own) {
    while (a.lo < a.hi || b.lo < b.hi) {
        const bool ga = a.lo < a.hi, gb = b.lo < b.hi;
        const uint32_t ma = ga ? a.lo + (a.hi - a.lo) / 2 : own, mb = gb ? b.lo + (b.hi - b.lo) / 2 : own;
        const uint64_t ka = key(ma), kb = key(mb);
        if (ga && ka < a.v) a.lo = ma + 1;
        if (ga && !(ka < a.v)) a.hi = ma;
        if (gb && kb < b.v) b.lo = mb + 1;
        if (gb && !(kb < b.v)) b.hi = mb;
    }
}

__device__ __forceinline__ float wave_min(float v, int from, int to) {
    for (int d = from; d < to; d <<= 1) v = fminf(v, __shfl_xor(v, d, 64));
    return v;
}
__device__ __forceinline__ float wave_max(float v, int from, int to) {
    for (int d = from; d < to; d <<= 1) v = fmaxf(v, __shfl_xor(v, d, 64));
    return v;
}

__device__ __forceinline__ float diag(float lx, float ly, float lz, float hx, float hy, float hz) {
    return sqrtf((hx - lx) * (hx - lx) + (hy - ly) * (hy - ly) + (hz - lz) * (hz - lz));
}

// One wavefront = one 64-particle super-cluster (blocks of 256 start at
// multiples of 64): the 8-particle cluster box and the super-cluster box come
// from min / max over lane groups; absent particles are NaN, which fminf and
// fmaxf ignore.
constexpr int64_t kFeatFew = 262144;

template <bool kFew>
__global__ __launch_bounds__(kFeatThreads) void k_features(int64_t n, const uint64_t *__restrict__ keys,
                                                  const float *__restrict__ x, const float *__restrict__ y,
                                                  const float *__restrict__ z, const float *__restrict__ h,
                                                  const int32_t *__restrict__ nnb, float edge0, int target,
                                                  uint16_t *__restrict__ feat, SegTable seg) {
    constexpr int kWin = kFeatThreads + 2 * kKeyPad;
    __shared__ uint64_t s_key[kWin];
    const int64_t b0 = (int64_t)blockIdx.x * kFeatThreads - kKeyPad;  // index of s_key[0] (may be negative)
#pragma unroll
    for (int k = 0; k < kWin / kFeatThreads; k++) {
        const int64_t a = b0 + k * kFeatThreads + threadIdx.x;
        s_key[k * kFeatThreads + threadIdx.x] = keys[a < 0 ? 0 : (a < n ? a : n - 1)];
    }
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool in = i < n;
    const float px = in ? x[i] : NAN, py = in ? y[i] : NAN, pz = in ? z[i] : NAN;
    float clx = wave_min(px, 1, 8), cly = wave_min(py, 1, 8), clz = wave_min(pz, 1, 8);
    float chx = wave_max(px, 1, 8), chy = wave_max(py, 1, 8), chz = wave_max(pz, 1, 8);
    const float slx = wave_min(clx, 8, 64), sly = wave_min(cly, 8, 64), slz = wave_min(clz, 8, 64);
    const float shx = wave_max(chx, 8, 64), shy = wave_max(chy, 8, 64), shz = wave_max(chz, 8, 64);
    if (!in) return;
    // key searches stay inside the particle's own system
    uint32_t klo = 0, khi = (uint32_t)n;
    if (seg.on()) {
        const int sy = seg.sc_sys[i / kScSize];
        klo = seg.pbase[sy];
        khi = klo + seg.count[sy];
        edge0 = seg.edge[sy];
        if ((uint32_t)i >= khi) {  // padding
            *reinterpret_cast<uint4 *>(feat + i * kIn) = make_uint4(0u, 0u, 0u, 0u);
            return;
        }
    }
    const float hi = h[i];
    const float lt = logf((float)target);
    float f[kIn];
    f[0] = nnb ? logf((float)nnb[i] + 1.0f) - lt : 0.0f;  // no count yet: 0
    f[1] = logf(fmaxf(diag(clx, cly, clz, chx, chy, chz) / hi, 1e-3f));
    f[2] = logf(fmaxf(diag(slx, sly, slz, shx, shy, shz) / hi, 1e-3f));
    const float lev = log2f(edge0 / hi);
    int L0 = (int)rintf(lev);
    L0 = L0 < 2 ? 2 : (L0 > 20 ? 20 : L0);
    const uint64_t key = s_key[kKeyPad + threadIdx.x];
    // the cell's run of keys at the three levels, each inside the coarser one's:
    // [ca, cb) holds it; the part of [ca, cb) in the window is [wa, wb)
    uint32_t ca = klo, cb = khi;
    const uint32_t w0 = b0 < 0 ? 0u : (uint32_t)b0;
    const uint32_t w1 = b0 + kWin < n ? (uint32_t)(b0 + kWin) : (uint32_t)n;
    const uint32_t base = (uint32_t)b0;  // (window indices wrap to below kWin)
    auto in_lds = [&](uint32_t k) { return s_key[k - base]; };
    auto in_mem = [&](uint32_t k) { return keys[k]; };
#pragma unroll
    for (int d = -1; d <= 1; d++) {
        const int shift = 3 * (21 - (L0 + d));
        const uint64_t pre = key >> shift;
        const uint64_t va = pre << shift, vb = (pre + 1) << shift;
        const uint32_t wa = ca > w0 ? ca : w0, wb = cb < w1 ? cb : w1;
        // (particle i is inside: the start is at most i, the end above it)
        const bool fa = wa > ca && in_lds(wa) >= va, fb = wb < cb && in_lds(wb - 1u) < vb;  // beyond the window
        if (kFew) {
            KeySearch a{ca, wa, va}, b{wb, cb, vb};
            if (!fa) a.lo = a.hi = lower_bound_key(in_lds, wa, (uint32_t)i, va);
            if (!fb) b.lo = b.hi = lower_bound_key(in_lds, (uint32_t)i + 1u, wb, vb);
            if (fa || fb) lower_bounds(in_mem, a, b, (uint32_t)i);
            ca = a.lo;
            cb = b.lo;
        } else {
            ca = fa ? lower_bound_key(in_mem, ca, wa, va) : lower_bound_key(in_lds, wa, (uint32_t)i, va);
            cb = fb ? lower_bound_key(in_mem, wb, cb, vb) : lower_bound_key(in_lds, (uint32_t)i + 1u, wb, vb);
        }
        f[4 + d] = logf(1.0f + (float)(cb - ca)) - lt;
    }
    f[6] = lev - (float)L0;
    f[7] = lt - logf(100.0f);
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; k++)
        w[k] = (uint32_t)(uint16_t)f2bf(f[2 * k]) | ((uint32_t)(uint16_t)f2bf(f[2 * k + 1]) << 16);
    *reinterpret_cast<uint4 *>(feat + i * kIn) = make_uint4(w[0], w[1], w[2], w[3]);
}

constexpr int kGradMaxRows = 256;  // blocks of the gradient kernel, one partial gradient each

}  // namespace
}  // namespace sfcnl

using namespace sfcnl;

extern "C" int sfcnl_mlp_init(sfcnl_ctx ctx, uint64_t seed, float *d_params) {
    if (!ctx) return SFCNL_E_ARG;
    if (!d_params) return set_err(ctx, SFCNL_E_ARG, "sfcnl_mlp_init: null params");
    k_mlp_init<<<blocks_for(kNParam, 256), 256, 0, ctx->stream>>>(seed, d_params);
    SFCNL_LAUNCHED(ctx);
    return SFCNL_OK;
}

extern "C" int sfcnl_mlp_infer(sfcnl_ctx ctx, const float *d_params, int64_t n, const uint16_t *d_feat, float *d_out) {
    if (!ctx) return SFCNL_E_ARG;
    if (n < 0) return set_err(ctx, SFCNL_E_ARG, "sfcnl_mlp_infer: n < 0");
    if (n == 0) return SFCNL_OK;
    if (!d_params || !d_feat || !d_out) return set_err(ctx, SFCNL_E_ARG, "sfcnl_mlp_infer: null pointer");
    int64_t blocks = (n + kWave * kWaves - 1) / (kWave * kWaves);
    if (blocks > kInferBlocks) blocks = kInferBlocks;
    k_mlp_infer<<<(unsigned)blocks, 256, 0, ctx->stream>>>(d_params, n, d_feat, d_out);
    SFCNL_LAUNCHED(ctx);
    return SFCNL_OK;
}

extern "C" int sfcnl_mlp_grad_workspace(int64_t batch, size_t *ws_bytes) {
    if (batch < 1 || !ws_bytes) return SFCNL_E_ARG;
    *ws_bytes = (size_t)kGradMaxRows * (kNParam + 1) * sizeof(float);
    return SFCNL_OK;
}

extern "C" int sfcnl_mlp_grad(sfcnl_ctx ctx, const float *d_params, int64_t nsamp, const uint16_t *d_feat,
                              const float *d_target, int64_t batch, int64_t start, int64_t mul, int64_t add,
                              void *d_ws, size_t ws_bytes, float *d_grad, float *d_loss) {
    if (!ctx) return SFCNL_E_ARG;
    if (nsamp < 1 || batch < 1 || mul < 1 || add < 0)
        return set_err(ctx, SFCNL_E_ARG, "sfcnl_mlp_grad: need nsamp, batch, mul >= 1 and add >= 0");
    if (!d_params || !d_feat || !d_target || !d_ws || !d_grad)
        return set_err(ctx, SFCNL_E_ARG, "sfcnl_mlp_grad: null pointer");
    size_t need;
    sfcnl_mlp_grad_workspace(batch, &need);
    if (ws_bytes < need) return set_err(ctx, SFCNL_E_ARG, "sfcnl_mlp_grad: workspace %zu < %zu", ws_bytes, need);
    const int64_t ntiles = (batch + 15) / 16;
    int64_t blocks = (ntiles + kWaves - 1) / kWaves;
    if (blocks > kGradMaxRows) blocks = kGradMaxRows;
    float *partial = reinterpret_cast<float *>(d_ws);
    k_mlp_grad<<<(unsigned)blocks, 256, 0, ctx->stream>>>(d_params, nsamp, d_feat, d_target, batch, start, mul, add,
                                                          partial);
    SFCNL_LAUNCHED(ctx);
    k_mlp_reduce<<<blocks_for(kNParam + 1, kWave), 256, 0, ctx->stream>>>(partial, (int)blocks, batch, d_grad, d_loss);
    SFCNL_LAUNCHED(ctx);
    return SFCNL_OK;
}

extern "C" int sfcnl_mlp_adam(sfcnl_ctx ctx, float *d_params, const float *d_grad, float *d_m, float *d_v, int64_t t,
                              float lr) {
    if (!ctx) return SFCNL_E_ARG;
    if (t < 1 || !(lr > 0.0f)) return set_err(ctx, SFCNL_E_ARG, "sfcnl_mlp_adam: need step >= 1 and lr > 0");
    if (!d_params || !d_grad || !d_m || !d_v) return set_err(ctx, SFCNL_E_ARG, "sfcnl_mlp_adam: null pointer");
    const float c1 = (float)(1.0 / (1.0 - pow(0.9, (double)t)));
    const float c2 = (float)(1.0 / (1.0 - pow(0.999, (double)t)));
    k_adam<<<blocks_for(kNParam, 256), 256, 0, ctx->stream>>>(d_params, d_grad, d_m, d_v, lr, c1, c2);
    SFCNL_LAUNCHED(ctx);
    return SFCNL_OK;
}

int sfcnl::features_impl(sfcnl_ctx ctx, int64_t n, const uint64_t *d_keys, const float *d_x, const float *d_y,
                         const float *d_z, const float *d_h, const int32_t *d_nnb, float box_edge, int target,
                         uint16_t *d_feat, const SegTable &seg) {
    const unsigned g = blocks_for(n, kFeatThreads);
    if (n <= kFeatFew)
        k_features<true><<<g, kFeatThreads, 0, ctx->stream>>>(n, d_keys, d_x, d_y, d_z, d_h, d_nnb, box_edge, target, d_feat, seg);
    else
        k_features<false><<<g, kFeatThreads, 0, ctx->stream>>>(n, d_keys, d_x, d_y, d_z, d_h, d_nnb, box_edge, target, d_feat, seg);
    SFCNL_LAUNCHED(ctx);
    return SFCNL_OK;
}

extern "C" int sfcnl_hseed_features(sfcnl_ctx ctx, int64_t n, const uint64_t *d_keys, const float *d_x,
                                    const float *d_y, const float *d_z, const float *d_h, const int32_t *d_nnb,
                                    float box_edge, int target, uint16_t *d_feat) {
    if (!ctx) return SFCNL_E_ARG;
    if (n < 0 || n >= (int64_t(1) << 31)) return set_err(ctx, SFCNL_E_ARG, "sfcnl_hseed_features: n out of range");
    if (n == 0) return SFCNL_OK;
    if (!d_keys || !d_x || !d_y || !d_z || !d_h || !d_feat || !(box_edge > 0.0f) || target < 1)
        return set_err(ctx, SFCNL_E_ARG, "sfcnl_hseed_features: bad argument");
    return features_impl(ctx, n, d_keys, d_x, d_y, d_z, d_h, d_nnb, box_edge, target, d_feat, SegTable{});
}
