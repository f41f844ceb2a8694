// SDF network with reflectiveness head (Sec. "Opaque density representation",
// "Signal representation"; App. C) on the MI355X matrix cores.
//
// Points are the GEMM's long dimension.  Every dense layer runs as an MFMA
// GEMM (FP32: the FP32 instruction for values, operands split in BF16 parts for
// derivatives; or one of the 16-bit forms below) with
// the elementwise work of its neighbours fused into the operand loads
// (softplus, its derivative times a tangent or an adjoint, relu) and the bias /
// relu-mask / accumulate into its epilogue.
//
// Forward call: primal layers, then grad_x f by one reverse sweep
//   G^(8) = w_out, G^(l) = (softplus'(Z^(l)) . G^(l+1)) W_l, grad = J_PE^T G^(0).
// Backward call: J = sum g_f f + g_grad . grad_x f + g_a a.  Since
// g_grad . grad_x f is the directional derivative of f along g_grad, the
// parameter gradient is reverse mode over a primal + tangent forward pass
// (Z, H, Hdot = sp'(Z) Zdot per layer), giving per layer
//   Zdot_bar = sp'(Z) Hdot_bar,  Z_bar = sp'(Z) H_bar + sp''(Z) Zdot Hdot_bar,
//   W_bar = Z_bar^T H + Zdot_bar^T Hdot,  H_bar = Z_bar W,  Hdot_bar = Zdot_bar W,
// where sp''(Z) Zdot = beta sigma(-beta Z) Hdot, so Zdot itself is never stored.
// The training pair of calls keeps the forward's (Z, H) of every layer and the
// sweep's adjoint S = sp'(Z) G^(l+1) to every pre-activation in a caller-owned
// reserve; the backward then runs only the tangent GEMM per layer, and takes
// the tangent pass's adjoints from S (Zdot_bar = half_size S), so one adjoint
// GEMM per layer remains.
// Weight gradients reduce over points in fixed splits (no atomics).
#include <algorithm>
#include <mutex>

#include "rfvr_impl.hpp"

namespace rfvr {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// Eight FP32 operand values (two float4 along k) rounded to BF16 (RNE) for one
// v_mfma_f32_16x16x32_bf16.  A and B fragments use the same slot <-> k
// assignment, so the instruction's sum over its 32 slots is the sum over k.
__device__ __forceinline__ bf16x8 to_bf16x8(floatx4 lo, floatx4 hi) {
    bf16x8 r;
    r[0] = (__bf16)lo[0]; r[1] = (__bf16)lo[1]; r[2] = (__bf16)lo[2]; r[3] = (__bf16)lo[3];
    r[4] = (__bf16)hi[0]; r[5] = (__bf16)hi[1]; r[6] = (__bf16)hi[2]; r[7] = (__bf16)hi[3];
    return r;
}

// the same for one v_mfma_f32_16x16x32_f16 (FP16, RNE)
__device__ __forceinline__ f16x8 to_f16x8(floatx4 lo, floatx4 hi) {
    f16x8 r;
    r[0] = (_Float16)lo[0]; r[1] = (_Float16)lo[1]; r[2] = (_Float16)lo[2]; r[3] = (_Float16)lo[3];
    r[4] = (_Float16)hi[0]; r[5] = (_Float16)hi[1]; r[6] = (_Float16)hi[2]; r[7] = (_Float16)hi[3];
    return r;
}

// x = big + small with big = f16(x), small = f16(x - big): 22 significant bits
__device__ __forceinline__ void split_f16x8(floatx4 lo, floatx4 hi, f16x8& big, f16x8& small) {
    big = to_f16x8(lo, hi);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        small[e] = (_Float16)(lo[e] - (float)big[e]);
        small[4 + e] = (_Float16)(hi[e] - (float)big[4 + e]);
    }
}

// x = p[0] + p[1] + p[2], each BF16 (RNE): the first two remainders are exact in
// FP32 and the third has at most 8 significant bits, so the three parts hold all
// 24 bits of x (down to where the parts leave BF16's normal range, |x| ~ 1e-33);
// the first two alone hold 16
// (two values per conversion instruction: 11 VALU instructions a pair)
__device__ __forceinline__ uint32_t pk_bf16(float x, float y) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{x, y}, b2));
}
template <int N>
__device__ __forceinline__ void split_bf16x8(floatx4 lo, floatx4 hi, bf16x8 (&p)[N]) {
    uintx4 w[N];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float x = e < 2 ? lo[2 * e] : hi[2 * e - 4], y = e < 2 ? lo[2 * e + 1] : hi[2 * e - 3];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const uint32_t b = pk_bf16(x, y);
            w[q][e] = b;
            x -= __uint_as_float(b << 16);
            y -= __uint_as_float(b & 0xffff0000u);
        }
    }
#pragma unroll
    for (int q = 0; q < N; ++q) p[q] = __builtin_bit_cast(bf16x8, w[q]);
}

// A product of one 16 x 16 tile over 32 k from operands split in N parts, smallest
// terms first: in three (FP32), the six part products down to 2^-16 of the leading
// one (the three left out are below 2^-25 of it); in two (BF16X3), three.  TM tiles
// share a point fragment, so that consecutive MFMAs are independent.
// In three parts the five corrections are summed by themselves and added by a vector
// instruction: the matrix core cuts what lies some bits below the largest term of an
// instruction towards minus infinity, so corrections that share an accumulator with
// the leading products lose half a bit there on average, always downwards.  The error
// of one product was small (7e-8), but its mean of -1.5e-8 times the value added up over
// layers and points: parameter gradient 8e-7 against 3.7e-7 of the FP32 instruction, 3.0e-7
// in this form (2^20 points, ReLU masks held; training pair 47.7 -> 48.7 ms).
template <int N, int TM>
__device__ __forceinline__ void mfma_split(const bf16x8 (&w)[TM][N], const bf16x8 (&a)[N], floatx4* acc,
                                           bool points_first) {
    constexpr int NP = N == 3 ? 6 : 3;
    constexpr int PA[6] = {N - 1, 0, N == 3 ? 1 : 0, 1, 0, 0}, PB[6] = {0, N - 1, N == 3 ? 1 : 0, 0, 1, 0};
    const auto mul = [&](int b, int q, floatx4 c) {
        return points_first ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[PA[q]], w[b][PB[q]], c, 0, 0, 0)
                            : __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[b][PB[q]], a[PA[q]], c, 0, 0, 0);
    };
    if constexpr (N == 3) {
        floatx4 t[TM];
#pragma unroll
        for (int b = 0; b < TM; ++b) t[b] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int q = 0; q < NP - 1; ++q)
#pragma unroll
            for (int b = 0; b < TM; ++b) t[b] = mul(b, q, t[b]);
#pragma unroll
        for (int b = 0; b < TM; ++b) acc[b] = mul(b, NP - 1, acc[b]);
#pragma unroll
        for (int b = 0; b < TM; ++b) acc[b] += t[b];
    } else {
#pragma unroll
        for (int q = 0; q < NP; ++q)
#pragma unroll
            for (int b = 0; b < TM; ++b) acc[b] = mul(b, q, acc[b]);
    }
}

// The k of a 32-wide chunk that lane group kg multiplies: kg split_k0 .. + 3 and those
// split_k1 further on.  In three parts eight in a row (a row's chunk is read 128
// bytes at a time).  In two, four of either half, as the single-rounded kernels
// have it: the matrix core adds its k in groups, BF16X3's split rounds the
// activations to 16 bits, and another order moved some across a rounding
// (1e-5 in the gradients).
__host__ __device__ constexpr int split_k0(int parts) { return parts == 3 ? 8 : 4; }
__host__ __device__ constexpr int split_k1(int parts) { return parts == 3 ? 4 : 16; }

// BF16 storage of the single-rounded BF16 backward's arrays (tangents Hdot and
// adjoints Zbar): the BF16 products that read them round them to BF16 (RNE)
// anyway, so they are stored rounded, as raw 16-bit words in buffers sized for
// FP32 (the few FP32 readers, the adjoint epilogue's Hdot and the encoding
// layer's FP32 weight-gradient product, see the rounded values), and widened
// where they are used (a main loop keeps the raw words of its prefetch and
// widens them at the LDS store, so the prefetch stays in flight)
__device__ __forceinline__ uint2 ld_raw_bf16x4(const float* base, long i) {
    return *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(base) + i);
}
__device__ __forceinline__ float4 widen_bf16x4(uint2 r) {
    return make_float4(__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xffff0000u),
                       __uint_as_float(r.y << 16), __uint_as_float(r.y & 0xffff0000u));
}
__device__ __forceinline__ float4 ld_bf16x4(const float* base, long i) { return widen_bf16x4(ld_raw_bf16x4(base, i)); }
__device__ __forceinline__ float ld_bf16(const float* base, long i) {
    return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(base)[i] << 16);
}
__device__ __forceinline__ uint32_t bf16_bits(float x) {
    return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)x);
}
__device__ __forceinline__ void st_bf16x4(float* base, long i, floatx4 v) {
    uint2 r;
    r.x = bf16_bits(v[0]) | (bf16_bits(v[1]) << 16);
    r.y = bf16_bits(v[2]) | (bf16_bits(v[3]) << 16);
    *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(base) + i) = r;
}
__device__ __forceinline__ void st_bf16(float* base, long i, float v) {
    reinterpret_cast<uint16_t*>(base)[i] = (uint16_t)bf16_bits(v);
}
// which operands of a GEMM are held in BF16 storage
enum { ST_A = 1, ST_B = 2, ST_C2 = 4, ST_Y = 8 };

// operand precision of a network GEMM: FP32 (MM_FP32: operands split in three;
// MM_MFMA32: the FP32 instruction, see gemm and gemm_first), BF16 MFMA, BF16 MFMA on split
// operands (a b ~ a_big b_big + a_big b_small + a_small b_big), or FP16 MFMA
// with the weights rounded once and the per-point operand split in two
// (a b ~ a_big b + a_small b, two products).  The per-point operand's rounding
// differs from point to point, and the opacity of neighbouring samples takes
// differences of their SDF values, which magnify it; the weights' rounding is
// a fixed, smooth change of the network.  FP16 serves the forward products only
// (its 5-bit exponent cannot hold the backward's adjoints, which scale with the
// upstream gradients); in the dual forward GEMM, MM_F16 means this form for
// the primal and BF16 for the tangent.
enum { MM_FP32 = 0, MM_BF16 = 1, MM_F16 = 2, MM_BF16X3 = 3, MM_MFMA32 = 4 };

// operand prologues: identity, relu, or SEED: A[p][k] = H -> sp'(Z) colv[k] (the
// normal sweep's seed from the top layer's activation, formed while the tile is
// staged); the softplus activations themselves are written by the producing
// GEMM's epilogue, so no operand is transformed twice
enum { PRO_ID = 0, PRO_SEED = 1, PRO_RELU = 3 };
// epilogues (C = H = sp(Z) of a layer: sp'(Z) = 1 - e^(-beta H), e^(-beta Z) =
// 1 / (e^(beta H) - 1), so Z itself is never stored):
//            BIAS      Y = acc + bias
//            RELUMASK  Y = acc where C > 0, else 0
//            BIAS_SP   Y = softplus(acc + bias)                        (layer activation)
//            DSPMUL    Y = acc * sp'(Z)                                (normal sweep, tangent)
//            TOPADJ    Hbar = acc + scale rowv[p] colv[m], Hdotbar = scale colv[m] with
//                      C = H, C2 = Hdot of the top layer: Y = Zbar, Y2 = Zdotbar
//                      (the top trunk layer's adjoints)
//            ADJ1      Hbar = acc, Hdotbar = scale C3 / sp'(Z) with C = H, C2 = Hdot and
//                      C3 = the normal sweep's adjoint to Z of the layer below:
//                      Y = Zbar = sp'(Z) Hbar + beta sigma(-beta Z) Hdot Hdotbar
//                        = sp'(Z) Hbar + beta exp(-beta Z) Hdot scale C3
//                      (exp(-beta Z) capped at 1e30, where Hdot C3 is below 1e-60)
enum { EPI_BIAS = 0, EPI_RELUMASK = 2, EPI_BIAS_SP = 3, EPI_DSPMUL = 4, EPI_TOPADJ = 6, EPI_ADJ1 = 8 };

// Activation math of the network on the hardware exp2 / log2 / rcp units
// (v_exp_f32, v_log_f32, v_rcp_f32; ~1 ulp each): these run once per element
// in the GEMM epilogues and elementwise kernels, where the correctly rounded
// library forms would add several times their VALU work.
__device__ __forceinline__ float fexp(float x) { return __builtin_amdgcn_exp2f(x * 1.4426950408889634f); }
__device__ __forceinline__ float flog1p_pos(float e) {           // log(1 + e), e in [0, 1]
    return __builtin_amdgcn_logf(1.0f + e) * 0.6931471805599453f;
}
__device__ __forceinline__ float fsig(float x) { return __builtin_amdgcn_rcpf(1.0f + fexp(-x)); }
__device__ __forceinline__ float sp_f(float z, float beta) {
    const float bz = beta * z;
    return fmaxf(z, 0.0f) + flog1p_pos(fexp(-fabsf(bz))) * __builtin_amdgcn_rcpf(beta);
}
__device__ __forceinline__ float sp_d1(float z, float beta) { return fsig(beta * z); }
// sp'(Z) from H = sp(Z): e^(beta H) = 1 + e^(beta Z), so sp'(Z) = 1 - e^(-beta H)
// (absolute error ~1e-7, the rounding of the exponential near 1)
__device__ __forceinline__ float sp_d1_h(float h, float beta) { return 1.0f - fexp(-beta * h); }
__device__ __forceinline__ float sp_d2(float z, float beta) {
    const float s = fsig(beta * z);
    return beta * s * (1.0f - s);
}


// ----------------------------------------------------------------------------
// Y[P x M] = pro(A)[P x K] * B[M x K]^T  (+ epilogue).  K multiple of 32; A and
// B rows hold K valid or zero-padded columns; lda/ldb multiples of 4.
// Block BP (128, or 64: see gemm_launch) points x BM outputs, 4 waves, 16x16x4 MFMA tiles, K chunks of 32
// staged through LDS with the next chunk's global loads in flight during the
// current chunk's MFMAs.  The k index of a lane's MFMA operand is permuted so
// each lane reads 4 consecutive k (one float4) per 16-wide k group.
// ----------------------------------------------------------------------------
// rows per block of a product's weight operand and of its split image
__host__ __device__ constexpr int block_rows(int M) { return M <= 64 ? 64 : 128; }

struct GemmArgs {
    const float* A; long lda;
    const float* B; long ldb;
    const uint16_t* Bx;           // split products: the image of B (k_prep_weights)
    const float* bias;            // EPI_BIAS*: [M] or null
    const float* C;               // EPI_RELUMASK / DSPMUL / TOPADJ: [P][ldc]
    const float* C2;              // EPI_TOPADJ, ADJ1: [P][ldc]
    const float* C3;              // EPI_ADJ1: [P][ldc]
    long ldc;
    float* Y; long ldy;
    float* Y2;                    // EPI_TOPADJ: second output, row stride ldy
    const float* rowv;            // EPI_TOPADJ: [P] or null
    const float* colv;            // EPI_TOPADJ: [M]; PRO_SEED: [K]
    float scale;                  // EPI_TOPADJ, ADJ1
    float* cpart;                 // EPI_TOPADJ: [point tiles][M] column partials of
                                  // rowv[p] scale C + scale C2 (one row per tile), or null
    long P; int M; int K;
    float beta;
};

// Epilogue of a block of BP x BM products, WP x (4 / WP) waves of TP x TM tiles
// of 16 x 16; scr: (TP * 4) * (BM / WM) floats of LDS free for the column partials.
template <int EPI, int BP, int BM, int WP, int ST, int TP, int TM>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& g, floatx4 (&acc)[TP][TM], float* scr, long p0, int m0) {
    constexpr int WM = 4 / WP;
    const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
    const int wp = wv % WP, wm = wv / WP;
    const int li = lane & 15, lg = lane >> 4;
    // The weights are the MFMA's first operand, so a lane's four
    // accumulator values acc[a][b][0..3] are four consecutive outputs
    // m = m0 + wm (BM/WM) + 16 b + 4 lg + v of one point p = p0 + wp (BP/WP)
    // + 16 a + li: one float4 of a row-major [P][ld] array.  Tiles wholly inside
    // the output (with 16-byte aligned rows) load and store float4s without
    // guards; the others clamp their loads into the arrays and guard each
    // store.  A 16-point group's loads are all issued before the first is used.
    constexpr int NC = (EPI == EPI_ADJ1) ? 3 : (EPI == EPI_TOPADJ) ? 2 : (EPI == EPI_DSPMUL || EPI == EPI_RELUMASK) ? 1 : 0;
    auto epilogue = [&](auto guarded) {
        constexpr bool GUARD = decltype(guarded)::value;
        // per-output vector (bias, or the top adjoint's column vector): the same
        // 16 values for every point group of the lane, loaded once
        constexpr bool VEC = (EPI == EPI_BIAS || EPI == EPI_BIAS_SP || EPI == EPI_TOPADJ);
        const float* vsrc = (EPI == EPI_TOPADJ) ? g.colv : g.bias;
        floatx4 vv[VEC ? TM : 1];
        if constexpr (VEC) {
#pragma unroll
            for (int b = 0; b < TM; ++b) {
                const int mb = m0 + wm * (BM / WM) + b * 16 + lg * 4;
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    vv[b][v] = vsrc ? vsrc[GUARD ? min(mb + v, g.M - 1) : mb + v] : 0.0f;
            }
        }
#pragma unroll
        for (int a = 0; a < TP; ++a) {
            const long p = p0 + wp * (BP / WP) + a * 16 + li;
            const bool pin = !GUARD || p < g.P;
            const long pr = pin ? p : g.P - 1;
            floatx4 cl[NC ? NC : 1][TM];
            const float* src[3] = {g.C, g.C2, g.C3};
            if constexpr (NC > 0 && !GUARD) {
#pragma unroll
                for (int b = 0; b < TM; ++b) {
                    const int mb = m0 + wm * (BM / WM) + b * 16 + lg * 4;
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        if ((ST & ST_C2) != 0 && c == 1) {
                            const float4 t = ld_bf16x4(src[c], pr * g.ldc + mb);
                            cl[c][b] = floatx4{t.x, t.y, t.z, t.w};
                        } else {
                            cl[c][b] = *reinterpret_cast<const floatx4*>(src[c] + pr * g.ldc + mb);
                        }
                    }
                }
            }
            float rv = 0.0f;
            if constexpr (EPI == EPI_TOPADJ) rv = g.rowv ? g.scale * g.rowv[pr] : 0.0f;
#pragma unroll
            for (int b = 0; b < TM; ++b) {
                const int mb = m0 + wm * (BM / WM) + b * 16 + lg * 4;
                if constexpr (NC > 0 && GUARD) {
#pragma unroll
                    for (int c = 0; c < NC; ++c)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const long ci = pr * g.ldc + min(mb + v, g.M - 1);
                            cl[c][b][v] = ((ST & ST_C2) != 0 && c == 1) ? ld_bf16(src[c], ci) : src[c][ci];
                        }
                }
                floatx4 y = acc[a][b], y2 = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_SP) y[v] += vv[b][v];
                    if constexpr (EPI == EPI_BIAS_SP) y[v] = sp_f(y[v], g.beta);
                    if constexpr (EPI == EPI_RELUMASK) y[v] = cl[0][b][v] > 0.0f ? y[v] : 0.0f;
                    if constexpr (EPI == EPI_DSPMUL) y[v] *= sp_d1_h(cl[0][b][v], g.beta);
                    if constexpr (EPI == EPI_TOPADJ) {
                        const float cv = vv[b][v];
                        const float hb = __builtin_fmaf(rv, cv, y[v]);
                        const float hdb = g.scale * cv;
                        const float em = fexp(-g.beta * cl[0][b][v]);   // 1 - sp'(Z)
                        const float sg = 1.0f - em;
                        y[v] = sg * hb + g.beta * em * cl[1][b][v] * hdb;
                        y2[v] = sg * hdb;
                    }
                    if constexpr (EPI == EPI_ADJ1) {
                        // the sweep kept S = sp'(Z) G, so sigma(-beta Z) G = exp(-beta Z) S,
                        // with exp(-beta Z) = 1 / (e^(beta H) - 1)
                        const float bh = g.beta * cl[0][b][v];
                        const float ex = __builtin_amdgcn_rcpf(fexp(bh) - 1.0f);
                        const float sg = 1.0f - fexp(-bh);
                        y[v] = sg * y[v] + g.beta * fminf(ex, 1e30f) * cl[1][b][v] * (g.scale * cl[2][b][v]);
                    }
                }
                constexpr bool TWO = (EPI == EPI_TOPADJ);
                constexpr bool YB = (ST & ST_Y) != 0;
                if constexpr (!GUARD) {
                    if constexpr (YB) st_bf16x4(g.Y, p * g.ldy + mb, y);
                    else *reinterpret_cast<floatx4*>(g.Y + p * g.ldy + mb) = y;
                    if constexpr (TWO) *reinterpret_cast<floatx4*>(g.Y2 + p * g.ldy + mb) = y2;
                } else if (pin) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        if (mb + v >= g.M) continue;
                        if constexpr (YB) st_bf16(g.Y, p * g.ldy + mb + v, y[v]);
                        else g.Y[p * g.ldy + mb + v] = y[v];
                        if constexpr (TWO) g.Y2[p * g.ldy + mb + v] = y2[v];
                    }
                }
                if constexpr (GUARD && NC >= 2) __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (EPI == EPI_TOPADJ) {
                if (g.cpart) {
                    // the group's share of the output layer's weight gradient,
                    // sum_p (rowv[p] scale H + scale Hdot) per column: a fixed-order
                    // sum over the 16 lanes of the same columns (lane bits 0-3:
                    // the points), one row per (group, wave) into LDS
#pragma unroll
                    for (int b = 0; b < TM; ++b) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            float c = pin ? __builtin_fmaf(rv, cl[0][b][v], g.scale * cl[1][b][v]) : 0.0f;
#pragma unroll
                            for (int o = 1; o < 16; o <<= 1) c += __shfl_xor(c, o);
                            if (li == 0) scr[(a * 4 + wv) * (BM / WM) + b * 16 + lg * 4 + v] = c;
                        }
                    }
                }
            }
            // the next group's loads stay behind this group's stores
            if constexpr (NC >= 2) __builtin_amdgcn_sched_barrier(0);
        }
    };
    const bool aligned = (((g.ldy | g.ldc) & 3) == 0) &&
                         (((uintptr_t)g.Y | (uintptr_t)g.Y2 | (uintptr_t)g.C | (uintptr_t)g.C2 | (uintptr_t)g.C3) & 15) == 0;
    if (aligned && p0 + BP <= g.P && m0 + BM <= g.M) epilogue(std::false_type{});
    else epilogue(std::true_type{});
    if constexpr (EPI == EPI_TOPADJ) {
        if (g.cpart) {
            // the tile's column sums: one thread per column adds the rows of
            // its waves along points and their groups in a fixed order (the LDS
            // tiles were last read before the main loop's final barrier; the
            // rows above were written after it); one partial row per tile
            __syncthreads();
            if (tid < BM) {
                const int wmc = tid / (BM / WM), col = tid % (BM / WM);
                float t = 0.0f;
                for (int q = 0; q < WP; ++q)
                    for (int a = 0; a < TP; ++a) t += scr[(a * 4 + (wmc * WP + q)) * (BM / WM) + col];
                if (m0 + tid < g.M) g.cpart[(p0 / BP) * (long)g.M + m0 + tid] = t;
            }
        }
    }
}

template <int PRO, int EPI, int BM, int MM, int ST = 0, int BP = 128>
__global__ __launch_bounds__(256) void k_gemm_nt(GemmArgs g) {
    // padded LDS rows (BK + 4 floats): the MFMA fragment reads (16 rows, one
    // float4 column) are free of bank conflicts.  Variants measured slower on
    // this shape: an XOR-swizzled unpadded layout, two LDS buffers with one
    // barrier per chunk, 64-deep chunks (all at two waves per SIMD, against
    // three here).
    constexpr int BK = 32, LW = BK + 4, RPF = BK / 4;
    constexpr int WP = (BM == 128 || BP == 64) ? 2 : 4;
    constexpr int WM = 4 / WP;
    constexpr int TP = BP / WP / 16;
    constexpr int TM = BM / WM / 16;
    constexpr int NA = BP * BK / 4 / 256;       // float4 per thread, A
    constexpr int NB = BM * BK / 4 / 256;       // float4 per thread, B
    __shared__ float sA[BP * LW];
    __shared__ float sB[BM * LW];
    const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
    const int wp = wv % WP, wm = wv / WP;
    const int li = lane & 15, lg = lane >> 4;
    // Work-groups are dispatched round-robin over the 8 XCDs (id % 8).  The
    // column blocks of one point tile read the same A rows, so they are given
    // ids b, b+8, ... : same XCD (same L2), consecutive in dispatch order.
    const int nmb = (g.M + BM - 1) / BM;
    const long bid = blockIdx.x;
    const long grp = bid / (8L * nmb);
    const int within = (int)(bid % (8L * nmb));
    const int mb = within / 8;
    const long pt = grp * 8 + (within % 8);
    const long p0 = pt * BP;
    const int m0 = mb * BM;
    if (p0 >= g.P) return;                       // padding work-groups of the last group
    floatx4 acc[TP][TM];
#pragma unroll
    for (int a = 0; a < TP; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b) acc[a][b] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};

    float4 ra[(ST & ST_A) ? 1 : NA], rb[NB];
    uint2 ra16[(ST & ST_A) ? NA : 1];
    auto load = [&](int k0) {
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int e = tid + i * 256;
            const int row = e / RPF, c4 = (e % RPF) * 4;
            const long p = p0 + row;
            if constexpr ((ST & ST_A) != 0) {
                ra16[i] = make_uint2(0u, 0u);
                if (p < g.P) ra16[i] = ld_raw_bf16x4(g.A, p * g.lda + k0 + c4);
            } else {
                ra[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (p < g.P) ra[i] = *reinterpret_cast<const float4*>(g.A + p * g.lda + k0 + c4);
            }
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int e = tid + i * 256;
            const int row = e / RPF, c4 = (e % RPF) * 4;
            const int m = m0 + row;
            rb[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (m < g.M) rb[i] = *reinterpret_cast<const float4*>(g.B + (long)m * g.ldb + k0 + c4);
        }
    };
    auto off = [](int row, int q) { return row * LW + 4 * q; };
    auto store = [&](int k0) {
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int e = tid + i * 256;
            float4 v;
            if constexpr ((ST & ST_A) != 0) v = widen_bf16x4(ra16[i]);
            else v = ra[i];
            if constexpr (PRO == PRO_RELU) {
                v.x = fmaxf(v.x, 0.0f); v.y = fmaxf(v.y, 0.0f); v.z = fmaxf(v.z, 0.0f); v.w = fmaxf(v.w, 0.0f);
            }
            if constexpr (PRO == PRO_SEED) {
                const float* w = g.colv + k0 + (e % RPF) * 4;
                v.x = sp_d1_h(v.x, g.beta) * w[0]; v.y = sp_d1_h(v.y, g.beta) * w[1];
                v.z = sp_d1_h(v.z, g.beta) * w[2]; v.w = sp_d1_h(v.w, g.beta) * w[3];
            }
            *reinterpret_cast<float4*>(&sA[off(e / RPF, e % RPF)]) = v;
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int e = tid + i * 256;
            *reinterpret_cast<float4*>(&sB[off(e / RPF, e % RPF)]) = rb[i];
        }
    };
    auto compute = [&]() {
        const float* A_ = sA;
        const float* B_ = sB;
        if constexpr (MM == MM_BF16) {
            // the chunk's two 16-wide k groups feed one 16x16x32 BF16 MFMA
            bf16x8 af[TP], bf[TM];
#pragma unroll
            for (int a = 0; a < TP; ++a) {
                const int row = wp * (BP / WP) + a * 16 + li;
                af[a] = to_bf16x8(*reinterpret_cast<const floatx4*>(&A_[off(row, lg)]),
                                  *reinterpret_cast<const floatx4*>(&A_[off(row, lg + 4)]));
            }
#pragma unroll
            for (int b = 0; b < TM; ++b) {
                const int row = wm * (BM / WM) + b * 16 + li;
                bf[b] = to_bf16x8(*reinterpret_cast<const floatx4*>(&B_[off(row, lg)]),
                                  *reinterpret_cast<const floatx4*>(&B_[off(row, lg + 4)]));
            }
#pragma unroll
            for (int a = 0; a < TP; ++a)
#pragma unroll
                for (int b = 0; b < TM; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[b], af[a], acc[a][b], 0, 0, 0);
        } else if constexpr (MM == MM_F16) {
            // one point row's split at a time (fewer live registers)
            f16x8 bf[TM];
#pragma unroll
            for (int b = 0; b < TM; ++b) {
                const int row = wm * (BM / WM) + b * 16 + li;
                bf[b] = to_f16x8(*reinterpret_cast<const floatx4*>(&B_[off(row, lg)]),
                                 *reinterpret_cast<const floatx4*>(&B_[off(row, lg + 4)]));
            }
#pragma unroll
            for (int a = 0; a < TP; ++a) {
                const int row = wp * (BP / WP) + a * 16 + li;
                f16x8 ab, as;
                split_f16x8(*reinterpret_cast<const floatx4*>(&A_[off(row, lg)]),
                            *reinterpret_cast<const floatx4*>(&A_[off(row, lg + 4)]), ab, as);
#pragma unroll
                for (int b = 0; b < TM; ++b) {
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bf[b], as, acc[a][b], 0, 0, 0);
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bf[b], ab, acc[a][b], 0, 0, 0);
                }
            }
        } else {
#pragma unroll
            for (int kk = 0; kk < BK; kk += 16) {
                floatx4 af[TP], bf[TM];
#pragma unroll
                for (int a = 0; a < TP; ++a)
                    af[a] = *reinterpret_cast<const floatx4*>(&A_[off(wp * (BP / WP) + a * 16 + li, kk / 4 + lg)]);
#pragma unroll
                for (int b = 0; b < TM; ++b)
                    bf[b] = *reinterpret_cast<const floatx4*>(&B_[off(wm * (BM / WM) + b * 16 + li, kk / 4 + lg)]);
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int a = 0; a < TP; ++a)
#pragma unroll
                        for (int b = 0; b < TM; ++b)
                            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(bf[b][s], af[a][s], acc[a][b], 0, 0, 0);
            }
        }
    };
    // one LDS buffer: store, barrier, next chunk's global loads in flight
    // during this chunk's MFMAs, barrier
    load(0);
    for (int k0 = 0; k0 < g.K; k0 += BK) {
        store(k0);
        __syncthreads();
        if (k0 + BK < g.K) load(k0 + BK);
        compute();
        __syncthreads();
    }
    gemm_epilogue<EPI, BP, BM, WP, ST>(g, acc, sA, p0, m0);
}

// ----------------------------------------------------------------------------
// The same product in FP32: every operand split in three BF16 parts
// (mfma_split), because six BF16 MFMAs over 32 k take 96 cycles of a SIMD's
// matrix core where the FP32 instruction takes 256.  The per-point operand is split once, on
// its way into LDS; the weights come split from k_prep_weights.  Both lie in LDS in
// fragment order: [part][16-row tile][slot][8 k], a lane's 16 bytes of a
// fragment in one ds_read_b128 and a wave's in one linear kilobyte.  The store
// side has four lanes on a row (32 bytes of k each, for coalesced global loads);
// slot kg * 16 + (row ^ 2 kg) of (row, kg) keeps both sides free of bank conflicts.
// It serves the derivatives; the values stay on the FP32 instruction (gemm).
// 2^20 x 256 x 256, against the FP32 instruction in the same kernel shape:
// sp'(Z) product 1.21 -> 0.95 ms, weight gradient 1.45 -> 1.0 ms.  The main loop runs at 1.26 PFLOP/s of BF16 products, what a
// large BF16 product reaches on this card (1.31); the epilogue's HBM traffic
// (4.7 TB/s) is not hidden behind it.  Tried and slower: persistent work-groups
// that fetch the next tile's first chunk and their epilogue's operands early
// (training pair 45.4 -> 49.3 ms).
// N = 2 is BF16X3 on the same kernel: two parts of the same image, three products.
// Its former kernels split both operands in registers once per wave that read them
// (150001 x 256 x 256: softplus layer 130 -> 104 us, sp'(Z) product 151 -> 131, dual
// forward 288 -> 240, dual adjoint 323 -> 275, a layer's weight gradients 226 -> 203);
// now bound by HBM and the epilogue, as above.
// ----------------------------------------------------------------------------
__device__ __forceinline__ int frag_slot(int row, int kg) { return kg * 16 + (row ^ (kg * 2)); }

// An infinite operand has no parts (its remainders are NaN), nor has a number that
// rounds to infinity in BF16 (beyond 3.39e38).  Either makes every sum that it enters
// NaN, so a wave that finds one among its sums forms its tiles again on the FP32
// instruction and takes its sums in place of those: infinities propagate as in plain
// FP32, and other points and outputs keep theirs.  Sums with a NaN among their operands
// are NaN either way: one look at the operands leaves them out (without it the backward
// with a NaN point in a thousand took 41 ms at 262144 points, with it 10.5; 8.2 without
// NaN).
template <int TP, int TM>
__device__ __forceinline__ bool any_nan(const floatx4 (&acc)[TP][TM]) {
    float t[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};          // eight chains side by side
#pragma unroll
    for (int a = 0; a < TP; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) t[(b & 1) * 4 + v] = __builtin_fmaf(acc[a][b][v], 0.0f, t[(b & 1) * 4 + v]);
    const float s = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
    return __ballot(s != s) != 0;
}

// four weights of one row from a three-part image (k a multiple of 4)
__device__ __forceinline__ floatx4 image_row4(const uint16_t* img, int bm, int nk, int m, int k) {
    const uint16_t* t = img + ((long)(m / bm) * nk + k / 32) * 3 * bm * 32 + (m % bm / 16) * 512 +
                        ((k % 32 / 8) * 16 + m % 16) * 8 + k % 8;
    floatx4 w = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int q = 2; q >= 0; --q) {               // exact from the smallest part on
        const uint2 r = *reinterpret_cast<const uint2*>(t + (long)q * bm * 32);
        const float4 p = widen_bf16x4(r);
        const float pv[4] = {p.x, p.y, p.z, p.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = (q == 0 && fabsf(pv[e]) == INFINITY) ? pv[e] : w[e] + pv[e];
    }
    return w;
}

// t where acc is no number
__device__ __forceinline__ bool no_number(float x) { return __builtin_fmaf(x, 0.0f, 0.0f) != 0.0f; }
__device__ __forceinline__ void take_where_nan(floatx4& acc, const floatx4& t) {
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] = no_number(acc[v]) ? t[v] : acc[v];
}

// of 16 rows, one per lane modulo 16, those for which a lane has f
__device__ __forceinline__ uint32_t rows_with(bool f) {
    const unsigned long long m = __ballot(f);
    return (uint32_t)((m | m >> 16 | m >> 32 | m >> 48) & 0xffff);
}
// whether a tile has a sum that is no number although its row (4 lg + v, of `rows`) and
// its column (li, of `cols`) are without NaN
__device__ __forceinline__ bool wants_fp32(const floatx4& acc, uint32_t rows, uint32_t cols) {
    const int li = threadIdx.x & 15, lg = (threadIdx.x & 63) >> 4;
    bool w = false;
#pragma unroll
    for (int v = 0; v < 4; ++v) w |= no_number(acc[v]) && !(rows >> (4 * lg + v) & 1) && !(cols >> li & 1);
    return __ballot(w) != 0;
}

// the sums that are no numbers of pro(A) W^T, for the wave's TP x TM tiles from point
// row p and weight row m on (a tile at a time: no second set of accumulators)
template <int PRO, int TP, int TM, bool POINTS_FIRST>
__device__ __forceinline__ void fp32_tiles(floatx4 (&acc)[TP][TM], const float* A, long lda, long P, long p, const uint16_t* img,
                                           int bm, int nk, int m, float beta, const float* colv) {
    const int li = threadIdx.x & 15, lg = (threadIdx.x & 63) >> 4;
    const auto point4 = [&](int a, int k) {
        floatx4 x = *reinterpret_cast<const floatx4*>(A + min(p + a * 16 + li, P - 1) * lda + k);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (PRO == PRO_RELU) x[e] = fmaxf(x[e], 0.0f);
            if constexpr (PRO == PRO_SEED) x[e] = sp_d1_h(x[e], beta) * colv[k + e];
        }
        return x;
    };
    const auto nan4 = [](const floatx4& x) { return x[0] != x[0] || x[1] != x[1] || x[2] != x[2] || x[3] != x[3]; };
    uint32_t np[TP], nw[TM];                     // points and weight rows with a NaN
#pragma unroll
    for (int a = 0; a < TP; ++a) {
        bool f = false;
#pragma unroll 4
        for (int k = 4 * lg; k < nk * 32; k += 16) f |= nan4(point4(a, k));
        np[a] = rows_with(f);
    }
#pragma unroll
    for (int b = 0; b < TM; ++b) {
        bool f = false;
#pragma unroll 4
        for (int k = 4 * lg; k < nk * 32; k += 16) f |= nan4(image_row4(img, bm, nk, m + b * 16 + li, k));
        nw[b] = rows_with(f);
    }
#pragma unroll
    for (int a = 0; a < TP; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b) {
            if (!wants_fp32(acc[a][b], POINTS_FIRST ? np[a] : nw[b], POINTS_FIRST ? nw[b] : np[a])) continue;
            floatx4 t = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
            for (int k = 4 * lg; k < nk * 32; k += 16) {
                const floatx4 x = point4(a, k), w = image_row4(img, bm, nk, m + b * 16 + li, k);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    t = POINTS_FIRST ? __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], w[e], t, 0, 0, 0)
                                     : __builtin_amdgcn_mfma_f32_16x16x4f32(w[e], x[e], t, 0, 0, 0);
            }
            take_where_nan(acc[a][b], t);
        }
}

// T x T tiles; HB output tiles of a wave are multiplied at a time: with two,
// three waves fit on a SIMD (all four, at two waves, read less LDS: better
// where no third work-group would come to the CU anyway).
template <int PRO, int EPI, int T, int HB, int N = 3>
__global__ __launch_bounds__(256, T != 128 ? 4 : (HB == 4 || EPI == EPI_TOPADJ) ? 2 : 3) void k_gemm_nt32(GemmArgs g) {
    constexpr int BP = T, BM = T, BK = 32, WP = 2, WM = 2;
    constexpr int TP = BP / WP / 16, TM = BM / WM / 16;
    constexpr int FT = 64 * 8;                   // 16-bit words of one tile of one part
    constexpr int NA = BP / 64;                  // 8-k pieces of the point chunk per thread
    constexpr int K0 = split_k0(N), K1 = split_k1(N);
    constexpr int NBV = N * BM * BK / 8 / 256;   // 16-byte vectors of the weight chunk per thread
    __shared__ __align__(16) uint16_t sA[N * (BP / 16) * FT];
    __shared__ __align__(16) uint16_t sB[N * (BM / 16) * FT];
    const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
    const int wp = wv % WP, wm = wv / WP;
    const int li = lane & 15, lg = lane >> 4;
    // XCD mapping as in k_gemm_nt
    const int nmb = (g.M + BM - 1) / BM;
    const long bid = blockIdx.x;
    const long grp = bid / (8L * nmb);
    const int within = (int)(bid % (8L * nmb));
    const int mb = within / 8;
    const long pt = grp * 8 + (within % 8);
    const long p0 = pt * BP;
    const int m0 = mb * BM;
    if (p0 >= g.P) return;                       // padding work-groups of the last group
    floatx4 acc[TP][TM];
#pragma unroll
    for (int a = 0; a < TP; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b) acc[a][b] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    const int nk = g.K / BK;
    // the block's part of the image: BM of the bm rows of image block m0 / bm
    const int bm = block_rows(g.M), pv = bm * 4;             // 16-byte vectors of one part of a chunk
    const uintx4* img = reinterpret_cast<const uintx4*>(g.Bx) + (long)(m0 / bm) * nk * (3 * pv) + (m0 % bm) * 4;
    floatx4 ra[NA][2];
    uintx4 rb[NBV];
    auto load = [&](int kc) {
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int u = tid + i * 256;
            // rows beyond the last point repeat it: their products are not stored
            const long p = min(p0 + (u >> 2), g.P - 1);
            const floatx4* q = reinterpret_cast<const floatx4*>(g.A + p * g.lda + kc * BK + (u & 3) * K0);
            ra[i][0] = q[0];
            ra[i][1] = q[K1 / 4];
        }
#pragma unroll
        for (int i = 0; i < NBV; ++i) {
            const int v = i * 256 + tid;
            rb[i] = img[(kc * 3 + v / (BM * 4)) * pv + v % (BM * 4)];
        }
    };
    auto store = [&](int kc) {
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int u = tid + i * 256;
            const int row = u >> 2, kg = u & 3;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if constexpr (PRO == PRO_RELU) ra[i][h][e] = fmaxf(ra[i][h][e], 0.0f);
                    if constexpr (PRO == PRO_SEED)
                        ra[i][h][e] = sp_d1_h(ra[i][h][e], g.beta) * g.colv[kc * BK + kg * K0 + h * K1 + e];
                }
            bf16x8 part[N];
            split_bf16x8(ra[i][0], ra[i][1], part);
#pragma unroll
            for (int q = 0; q < N; ++q)
                *reinterpret_cast<bf16x8*>(&sA[(q * (BP / 16) + (row >> 4)) * FT + frag_slot(row & 15, kg) * 8]) = part[q];
        }
#pragma unroll
        for (int i = 0; i < NBV; ++i) *reinterpret_cast<uintx4*>(&sB[(i * 256 + tid) * 8]) = rb[i];
    };
    load(0);
    for (int kc = 0; kc < nk; ++kc) {
        store(kc);
        __syncthreads();
        if (kc + 1 < nk) load(kc + 1);
#pragma unroll
        for (int h = 0; h < TM; h += HB) {
            bf16x8 wf[HB][N];
#pragma unroll
            for (int b = 0; b < HB; ++b)
#pragma unroll
                for (int q = 0; q < N; ++q)
                    wf[b][q] = *reinterpret_cast<const bf16x8*>(&sB[(q * (BM / 16) + wm * TM + h + b) * FT + lane * 8]);
#pragma unroll
            for (int a = 0; a < TP; ++a) {
                bf16x8 af[N];
#pragma unroll
                for (int q = 0; q < N; ++q)
                    af[q] = *reinterpret_cast<const bf16x8*>(&sA[(q * (BP / 16) + wp * TP + a) * FT + frag_slot(li, lg) * 8]);
                mfma_split<N, HB>(wf, af, &acc[a][h], false);
                if constexpr (HB < TM) __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();
    }
    if constexpr (N == 3) {
        if (any_nan(acc))
            fp32_tiles<PRO, TP, TM, false>(acc, g.A, g.lda, g.P, p0 + wp * (BP / WP), g.Bx, bm, nk, m0 + wm * (BM / WM), g.beta,
                                           g.colv);
    }
    gemm_epilogue<EPI, BP, BM, WP, 0>(g, acc, reinterpret_cast<float*>(sA), p0, m0);
}

// ----------------------------------------------------------------------------
// Two products with one B operand, Y = A B^T and Yd = A2 B^T (a layer's primal
// and tangent, or the two adjoints of its input), the layer's elementwise work
// in the epilogue:
//   EPI2_FWD: Z = acc + bias, H = sp(Z), Hdot = sp'(Z) acc2     -> Y, Y2, Y3
//   EPI2_ADJ: Hbar = acc, Hdotbar = acc2 with C = Z, C2 = Hdot of the layer below:
//             Zbar = sp'(Z) Hbar + beta sigma(-beta Z) Hdot Hdotbar,
//             Zdotbar = sp'(Z) Hdotbar                         -> Y, Y2
// Tiling as k_gemm_nt with BM = 128; the B tile is staged once for both.
// ----------------------------------------------------------------------------
enum { EPI2_FWD = 0, EPI2_ADJ = 1 };

struct DualArgs {
    const float* A; const float* A2; long lda;
    const float* B; long ldb;
    const uint16_t* Bx;                     // split products: the image of B (k_prep_weights)
    const float* bias;
    const float* C; const float* C2;        // EPI2_ADJ: [P][ldy]
    float* Y; float* Y2; float* Y3; long ldy;
    long P; int M; int K;
    float beta;
};

// Epilogue of a dual product: WP waves along points x 2 along outputs, TP x TM
// tiles per wave.
template <int EPI2, int BP, int BM, int WP>
struct DualEpilogue {
    static constexpr int TP = BP / WP / 16, TM = BM / 2 / 16;
    float cz[EPI2 == EPI2_ADJ ? TP : 1][TM][4], chd[EPI2 == EPI2_ADJ ? TP : 1][TM][4];

    __device__ __forceinline__ void prefetch(const DualArgs& g, long p0, int m0) {
        const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, wp = wv % WP, wm = wv / WP, li = lane & 15, lg = lane >> 4;
        // the adjoint epilogue's operands (Z and Hdot of the layer below) do not
        // depend on the products: fetch them before the main loop
        if constexpr (EPI2 == EPI2_ADJ) {
#pragma unroll
            for (int a = 0; a < TP; ++a)
#pragma unroll
                for (int b = 0; b < TM; ++b) {
                    const int m = m0 + wm * (BM / 2) + b * 16 + li;
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const long p = p0 + wp * (BP / WP) + a * 16 + lg * 4 + v;
                        const bool in = m < g.M && p < g.P;
                        cz[a][b][v] = in ? g.C[p * g.ldy + m] : 0.0f;
                        chd[a][b][v] = in ? g.C2[p * g.ldy + m] : 0.0f;
                    }
                }
        }
    }

    __device__ __forceinline__ void finish(const DualArgs& g, floatx4 (&acc)[TP][TM], floatx4 (&acd)[TP][TM], long p0, int m0) {
        const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, wp = wv % WP, wm = wv / WP, li = lane & 15, lg = lane >> 4;
#pragma unroll
        for (int a = 0; a < TP; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b) {
                const int m = m0 + wm * (BM / 2) + b * 16 + li;
                if (m >= g.M) continue;
                const float bias = (EPI2 == EPI2_FWD && g.bias) ? g.bias[m] : 0.0f;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const long p = p0 + wp * (BP / WP) + a * 16 + lg * 4 + v;
                    if (p >= g.P) continue;
                    const long o = p * g.ldy + m;
                    if constexpr (EPI2 == EPI2_FWD) {
                        const float z = acc[a][b][v] + bias;
                        g.Y[o] = z;
                        g.Y2[o] = sp_f(z, g.beta);
                        g.Y3[o] = sp_d1(z, g.beta) * acd[a][b][v];
                    } else {
                        const float z = cz[a][b][v], hd = chd[a][b][v];
                        const float sg = fsig(g.beta * z);
                        const float hb = acc[a][b][v], hdb = acd[a][b][v];
                        g.Y[o] = sg * hb + g.beta * (1.0f - sg) * hd * hdb;
                        g.Y2[o] = sg * hdb;
                    }
                }
            }
    }
};

template <int EPI2, int MM, int NW>
__global__ __launch_bounds__(NW * 64, NW == 4 ? 2 : 1) void k_gemm_dual(DualArgs g) {
    // NW = 8: 4 waves along points x 2 along outputs, 128 x 128 block; NW = 4:
    // 2 x 2 waves, 64 x 128 block.  2 x 4 tiles of 16 x 16 per wave and two
    // accumulator sets (64 registers) either way.
    constexpr int NT = NW * 64;
    constexpr int BP = NW == 8 ? 128 : 64, BM = 128, BK = 32, LW = BK + 4;
    constexpr int WP = NW / 2, TP = BP / WP / 16, TM = BM / 2 / 16;
    constexpr int NA = BP * BK / 4 / NT, NB = BM * BK / 4 / NT;
    __shared__ float sA[BP * LW];
    __shared__ float sA2[BP * LW];
    __shared__ float sB[BM * LW];
    const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
    const int wp = wv % WP, wm = wv / WP;
    const int li = lane & 15, lg = lane >> 4;
    const int nmb = (g.M + BM - 1) / BM;
    const long bid = blockIdx.x;
    const long grp = bid / (8L * nmb);
    const int within = (int)(bid % (8L * nmb));
    const int mb = within / 8;
    const long pt = grp * 8 + (within % 8);
    const long p0 = pt * BP;
    const int m0 = mb * BM;
    if (p0 >= g.P) return;                       // padding work-groups of the last group
    floatx4 acc[TP][TM], acd[TP][TM];
#pragma unroll
    for (int a = 0; a < TP; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b) {
            acc[a][b] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
            acd[a][b] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        }
    DualEpilogue<EPI2, BP, BM, WP> epi;
    epi.prefetch(g, p0, m0);
    float4 ra[NA], ra2[NA], rb[NB];
    auto load = [&](int k0) {
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int e = tid + i * NT;
            const int row = e >> 3, c4 = (e & 7) * 4;
            const long p = p0 + row;
            ra[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            ra2[i] = ra[i];
            if (p < g.P) {
                const long off = p * g.lda + k0 + c4;
                ra[i] = *reinterpret_cast<const float4*>(g.A + off);
                ra2[i] = *reinterpret_cast<const float4*>(g.A2 + off);
            }
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int e = tid + i * NT;
            const int row = e >> 3, c4 = (e & 7) * 4;
            const int m = m0 + row;
            rb[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (m < g.M) rb[i] = *reinterpret_cast<const float4*>(g.B + (long)m * g.ldb + k0 + c4);
        }
    };
    load(0);
    for (int k0 = 0; k0 < g.K; k0 += BK) {
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int e = tid + i * NT;
            const int row = e >> 3, c4 = (e & 7) * 4;
            *reinterpret_cast<float4*>(&sA[row * LW + c4]) = ra[i];
            *reinterpret_cast<float4*>(&sA2[row * LW + c4]) = ra2[i];
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int e = tid + i * NT;
            const int row = e >> 3, c4 = (e & 7) * 4;
            *reinterpret_cast<float4*>(&sB[row * LW + c4]) = rb[i];
        }
        __syncthreads();
        if (k0 + BK < g.K) load(k0 + BK);
        if constexpr (MM == MM_MFMA32) {
#pragma unroll
            for (int kk = 0; kk < BK; kk += 16) {
                floatx4 af[TP], af2[TP], bf[TM];
#pragma unroll
                for (int a = 0; a < TP; ++a) {
                    const int r = (wp * (BP / WP) + a * 16 + li) * LW + kk + lg * 4;
                    af[a] = *reinterpret_cast<const floatx4*>(&sA[r]);
                    af2[a] = *reinterpret_cast<const floatx4*>(&sA2[r]);
                }
#pragma unroll
                for (int b = 0; b < TM; ++b)
                    bf[b] = *reinterpret_cast<const floatx4*>(&sB[(wm * (BM / 2) + b * 16 + li) * LW + kk + lg * 4]);
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int a = 0; a < TP; ++a)
#pragma unroll
                        for (int b = 0; b < TM; ++b) {
                            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[a][s], bf[b][s], acc[a][b], 0, 0, 0);
                            acd[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(af2[a][s], bf[b][s], acd[a][b], 0, 0, 0);
                        }
            }
        } else if constexpr (MM == MM_F16) {
            // primal on FP16 operands (split per-point operand), tangent on BF16
            // (the tangent scales with the upstream gradient): the staged
            // weights are rounded both ways
            f16x8 bh[TM];
            bf16x8 bb[TM];
#pragma unroll
            for (int b = 0; b < TM; ++b) {
                const float* r = &sB[(wm * (BM / 2) + b * 16 + li) * LW + lg * 4];
                const floatx4 lo = *reinterpret_cast<const floatx4*>(r), hi = *reinterpret_cast<const floatx4*>(r + 16);
                bh[b] = to_f16x8(lo, hi);
                bb[b] = to_bf16x8(lo, hi);
            }
#pragma unroll
            for (int a = 0; a < TP; ++a) {
                const int off = (wp * (BP / WP) + a * 16 + li) * LW + lg * 4;
                f16x8 ah, al;
                split_f16x8(*reinterpret_cast<const floatx4*>(&sA[off]),
                            *reinterpret_cast<const floatx4*>(&sA[off + 16]), ah, al);
                const bf16x8 ad = to_bf16x8(*reinterpret_cast<const floatx4*>(&sA2[off]),
                                            *reinterpret_cast<const floatx4*>(&sA2[off + 16]));
#pragma unroll
                for (int b = 0; b < TM; ++b) {
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, bh[b], acc[a][b], 0, 0, 0);
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, bh[b], acc[a][b], 0, 0, 0);
                    acd[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ad, bb[b], acd[a][b], 0, 0, 0);
                }
            }
        } else {
            bf16x8 bb[TM];
#pragma unroll
            for (int b = 0; b < TM; ++b) {
                const float* r = &sB[(wm * (BM / 2) + b * 16 + li) * LW + lg * 4];
                bb[b] = to_bf16x8(*reinterpret_cast<const floatx4*>(r), *reinterpret_cast<const floatx4*>(r + 16));
            }
#pragma unroll
            for (int a = 0; a < TP; ++a) {
                const int off = (wp * (BP / WP) + a * 16 + li) * LW + lg * 4;
#pragma unroll
                for (int which = 0; which < 2; ++which) {
                    const float* r = which ? &sA2[off] : &sA[off];
                    floatx4* dst = which ? acd[a] : acc[a];
                    const bf16x8 ab = to_bf16x8(*reinterpret_cast<const floatx4*>(r), *reinterpret_cast<const floatx4*>(r + 16));
#pragma unroll
                    for (int b = 0; b < TM; ++b)
                        dst[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ab, bb[b], dst[b], 0, 0, 0);
                }
            }
        }
        __syncthreads();
    }
    epi.finish(g, acc, acd, p0, m0);
}

// the dual product on split operands (k_gemm_nt32): 64 points x BM
// outputs, 2 x 2 waves
template <int EPI2, int BM, int N>
__global__ __launch_bounds__(256, 2) void k_gemm_dual32(DualArgs g) {
    constexpr int BP = 64, BK = 32, WP = 2, TP = BP / WP / 16, TM = BM / 2 / 16;
    constexpr int FT = 64 * 8, NBV = N * BM * BK / 8 / 256;
    __shared__ __align__(16) uint16_t sA[2][N * (BP / 16) * FT];
    __shared__ __align__(16) uint16_t sB[N * (BM / 16) * FT];
    const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
    const int wp = wv % WP, wm = wv / WP;
    const int li = lane & 15, lg = lane >> 4;
    const int nmb = (g.M + BM - 1) / BM;
    const long bid = blockIdx.x;
    const long grp = bid / (8L * nmb);
    const int within = (int)(bid % (8L * nmb));
    const int mb = within / 8;
    const long pt = grp * 8 + (within % 8);
    const long p0 = pt * BP;
    const int m0 = mb * BM;
    if (p0 >= g.P) return;                       // padding work-groups of the last group
    floatx4 acc[TP][TM], acd[TP][TM];
#pragma unroll
    for (int a = 0; a < TP; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b) {
            acc[a][b] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
            acd[a][b] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        }
    DualEpilogue<EPI2, BP, BM, WP> epi;
    epi.prefetch(g, p0, m0);
    const int nk = g.K / BK;
    const uintx4* img = reinterpret_cast<const uintx4*>(g.Bx) + (long)mb * nk * (3 * BM * 4);
    const int row = tid >> 2, kg = tid & 3;
    const long pr = min(p0 + row, g.P - 1);      // rows beyond the last point repeat it
    floatx4 ra[2][2];
    uintx4 rb[NBV];
    auto load = [&](int kc) {
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            const floatx4* q = reinterpret_cast<const floatx4*>((w ? g.A2 : g.A) + pr * g.lda + kc * BK + kg * split_k0(N));
            ra[w][0] = q[0];
            ra[w][1] = q[split_k1(N) / 4];
        }
#pragma unroll
        for (int i = 0; i < NBV; ++i) rb[i] = img[(long)kc * (3 * BM * 4) + i * 256 + tid];
    };
    load(0);
    for (int kc = 0; kc < nk; ++kc) {
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            bf16x8 part[N];
            split_bf16x8(ra[w][0], ra[w][1], part);
#pragma unroll
            for (int q = 0; q < N; ++q)
                *reinterpret_cast<bf16x8*>(&sA[w][(q * (BP / 16) + (row >> 4)) * FT + frag_slot(row & 15, kg) * 8]) = part[q];
        }
#pragma unroll
        for (int i = 0; i < NBV; ++i) *reinterpret_cast<uintx4*>(&sB[(i * 256 + tid) * 8]) = rb[i];
        __syncthreads();
        if (kc + 1 < nk) load(kc + 1);
        constexpr int HB = N == 3 && TM == 4 ? 2 : TM;       // output tiles at a time: four would spill
#pragma unroll
        for (int h = 0; h < TM; h += HB) {
            bf16x8 wf[HB][N];
#pragma unroll
            for (int b = 0; b < HB; ++b)
#pragma unroll
                for (int q = 0; q < N; ++q)
                    wf[b][q] = *reinterpret_cast<const bf16x8*>(&sB[(q * (BM / 16) + wm * TM + h + b) * FT + lane * 8]);
#pragma unroll
            for (int a = 0; a < TP; ++a)
#pragma unroll
                for (int w = 0; w < 2; ++w) {
                    bf16x8 af[N];
#pragma unroll
                    for (int q = 0; q < N; ++q)
                        af[q] = *reinterpret_cast<const bf16x8*>(&sA[w][(q * (BP / 16) + wp * TP + a) * FT + frag_slot(li, lg) * 8]);
                    mfma_split<N, HB>(wf, af, (w ? acd[a] : acc[a]) + h, true);
                    if constexpr (HB < TM) __builtin_amdgcn_sched_barrier(0);
                }
        }
        __syncthreads();
    }
    if constexpr (N == 3) {
        const long pw = p0 + wp * (BP / WP);
        const int mw = m0 + wm * (BM / 2);
        if (any_nan(acc)) fp32_tiles<PRO_ID, TP, TM, true>(acc, g.A, g.lda, g.P, pw, g.Bx, BM, nk, mw, g.beta, nullptr);
        if (any_nan(acd)) fp32_tiles<PRO_ID, TP, TM, true>(acd, g.A2, g.lda, g.P, pw, g.Bx, BM, nk, mw, g.beta, nullptr);
    }
    epi.finish(g, acc, acd, p0, m0);
}

// ----------------------------------------------------------------------------
// Weight gradient partials: part[split][M][Kout] = sum over the split's points
// of A[p][m] * pro(B)[p][k], and bpart[split][m] = sum_p A[p][m].  With ST2 >= 0
// a second pair of operands (A2, B2) of the same shape, stored as ST2 says, is summed
// first and scaled by scale2: a trunk layer's two products in one launch, with one set
// of partials (100 MB per layer of 256 columns and 384 splits) where two launches
// wrote and read two.  Training pair of 8 layers: 2.29 -> 2.11 ms at 32768 points
// (FP32), backward with 150001 points in BF16X3 9.13 -> 8.77 ms; no difference at
// 2^20 points in FP32.
// Block 128 (m) x 128 (k), chunks of 32 points kept point-major in LDS (float4
// stores, scalar MFMA operand reads along the point index), next chunk's loads
// in flight during the current chunk's MFMAs.
// ----------------------------------------------------------------------------
struct WgArgs {
    const float* A; long lda;                  // [P][lda], columns 0..M-1
    const float* B; long ldb;                  // [P][ldb], columns 0..Kout-1
    const float *A2, *B2;                      // the second pair (same strides)
    float scale2;
    float* part;                               // [n_split][M][Kout]
    float* bpart;                              // [n_split][M]
    long P; int M; int Kout; long per_split;
    int n_split;
};

// Three waves per SIMD in BF16 storage; in FP32 storage (the plain backward, the head)
// three spill inside the loop (plain backward of 2^20 points, 8 layers of 256: 36.2 ms in
// BF16 and 38.4 in FP16 with three, 31.0 and 33.4 with two; the head alone makes no
// difference of 1 %).  The pair in BF16 storage stays at three (training backward 18.0 |
// 18.2 ms).
template <int PRO, int ST = 0, int ST2 = -1>
__global__ __launch_bounds__(256, ST == 0 ? 2 : 3) void k_gemm_wg(WgArgs g) {
    constexpr int BM = 128, BN = 128, BK = 32, LW = 128 + 4;
    __shared__ float sA[BK * LW];
    __shared__ float sB[BK * LW];
    const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
    const int wp = wv % 2, wn = wv / 2;
    const int li = lane & 15, lg = lane >> 4;
    // the (m, n) blocks of one point split share operand rows: ids 8 apart,
    // same XCD, consecutive in dispatch order
    const int nmb = (g.M + BM - 1) / BM, nnb = (g.Kout + BN - 1) / BN;
    const long bid = blockIdx.x;
    const long grp = bid / (8L * nmb * nnb);
    const int within = (int)(bid % (8L * nmb * nnb));
    const int tile = within / 8;
    const long split = grp * 8 + (within % 8);
    if (split >= g.n_split) return;              // padding work-groups of the last group
    const int m0 = (tile % nmb) * BM, n0 = (tile / nmb) * BN;
    const bool first_n = (tile / nmb) == 0;
    const long pb = split * g.per_split;
    long pe = pb + g.per_split;
    if (pe > g.P) pe = g.P;
    floatx4 acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    float bsum = 0.0f;                         // column sum of A (thread tid < 128 -> column tid)

    // one pair of operands added to acc (and with bias_c the column sums of A)
    const auto pass = [&](auto st_c, auto bias_c, const float* A, const float* B) __attribute__((always_inline)) {
        constexpr int S = decltype(st_c)::value;
        // raw 16-bit words of a BF16-stored operand's prefetch, widened at the LDS store
        float4 ra[(S & ST_A) ? 1 : 4], rb[(S & ST_B) ? 1 : 4];
        uint2 ra16[(S & ST_A) ? 4 : 1], rb16[(S & ST_B) ? 4 : 1];
        auto load = [&](long q0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = tid + i * 256;
                const int row = e >> 5, c4 = (e & 31) * 4;
                const long p = q0 + row;
                if constexpr (S == 0) {
                    ra[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    rb[i] = ra[i];
                    if (p < pe) {
                        if (m0 + c4 < g.M) ra[i] = *reinterpret_cast<const float4*>(A + p * g.lda + m0 + c4);
                        if (n0 + c4 < g.Kout) {
                            const long off = p * g.ldb + n0 + c4;
                            rb[i] = *reinterpret_cast<const float4*>(B + off);
                        }
                    }
                } else {
                    const bool la = p < pe && m0 + c4 < g.M, lb = p < pe && n0 + c4 < g.Kout;
                    if constexpr ((S & ST_A) != 0) ra16[i] = la ? ld_raw_bf16x4(A, p * g.lda + m0 + c4) : make_uint2(0u, 0u);
                    else ra[i] = la ? *reinterpret_cast<const float4*>(A + p * g.lda + m0 + c4) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    if constexpr ((S & ST_B) != 0) rb16[i] = lb ? ld_raw_bf16x4(B, p * g.ldb + n0 + c4) : make_uint2(0u, 0u);
                    else rb[i] = lb ? *reinterpret_cast<const float4*>(B + p * g.ldb + n0 + c4) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                }
            }
        };
        if (pb < pe) load(pb);
        for (long q0 = pb; q0 < pe; q0 += BK) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = tid + i * 256;
                const int row = e >> 5, c4 = (e & 31) * 4;
                const bool live = q0 + row < pe;
                float4 v, u;
                if constexpr ((S & ST_B) != 0) v = widen_bf16x4(rb16[i]);
                else v = rb[i];
                if constexpr ((S & ST_A) != 0) u = widen_bf16x4(ra16[i]);
                else u = ra[i];
                if constexpr (PRO == PRO_RELU) {
                    v.x = fmaxf(v.x, 0.0f); v.y = fmaxf(v.y, 0.0f); v.z = fmaxf(v.z, 0.0f); v.w = fmaxf(v.w, 0.0f);
                }
                if (!live) v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                *reinterpret_cast<float4*>(&sA[row * LW + c4]) = u;
                *reinterpret_cast<float4*>(&sB[row * LW + c4]) = v;
            }
            __syncthreads();
            if (q0 + BK < pe) load(q0 + BK);
            if constexpr (decltype(bias_c)::value) {
                if (first_n && tid < BM) {
#pragma unroll 8
                    for (int r = 0; r < BK; ++r) bsum += sA[r * LW + tid];
                }
            }
            // points lg*4 + s and 16 + lg*4 + s (s < 4) fill the 8 k slots of a
            // lane; the B fragments are converted first and each A fragment
            // just before its products (scheduling barriers keep the order), so
            // that three waves fit on a SIMD
            bf16x8 bf[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                floatx4 b0, b1;
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const int r = lg * 4 + s;
                    b0[s] = sB[r * LW + wn * 64 + b * 16 + li];
                    b1[s] = sB[(r + 16) * LW + wn * 64 + b * 16 + li];
                }
                bf[b] = to_bf16x8(b0, b1);
            }
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                __builtin_amdgcn_sched_barrier(0);
                floatx4 a0, a1;
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const int r = lg * 4 + s;
                    a0[s] = sA[r * LW + wp * 64 + a * 16 + li];
                    a1[s] = sA[(r + 16) * LW + wp * 64 + a * 16 + li];
                }
                const bf16x8 af = to_bf16x8(a0, a1);
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bf[b], acc[a][b], 0, 0, 0);
            }
            __syncthreads();
        }
    };
    if constexpr (ST2 >= 0) {
        pass(std::integral_constant<int, ST2 < 0 ? 0 : ST2>{}, std::false_type{}, g.A2, g.B2);
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[a][b] *= g.scale2;
    }
    pass(std::integral_constant<int, ST>{}, std::true_type{}, g.A, g.B);
    float* out = g.part + split * (long)g.M * g.Kout;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int k = n0 + wn * 64 + b * 16 + li;
            if (k >= g.Kout) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = m0 + wp * 64 + a * 16 + lg * 4 + v;
                if (m < g.M) out[(long)m * g.Kout + k] = acc[a][b][v];
            }
        }
    if (first_n && tid < BM && m0 + tid < g.M) g.bpart[split * (long)g.M + m0 + tid] = bsum;
}

// The weight gradient on split operands (k_gemm_nt32).  The
// contraction runs over points, so a fragment holds 8 points of one column: wave
// w loads points 8 w .. 8 w + 7 of two neighbouring columns per lane (512
// contiguous bytes per row; in 64 x 64 tiles a wave's halves take 8 points each), splits them where they are, and stores each
// column's 8 points as one 16-byte vector per part.  Column c of a 16-column
// tile t lies in slot ((c >> 1) | (c & 1) << 3) ^ (t & 1) << 3: the even and the
// odd columns that 16 lanes store together, and the 16 columns that they load
// together, then fall on different banks.
__device__ __forceinline__ int wg_slot(int c, int t) { return ((c >> 1) | ((c & 1) << 3)) ^ ((t & 1) << 3); }

template <int PRO, int ST = 0, int ST2 = -1, int T = 128, int N = 3>
__global__ __launch_bounds__(256, T == 128 ? 2 : 3) void k_gemm_wg32(WgArgs g) {
    constexpr int BM = T, BN = T, FT = 64 * 8;
    constexpr int LPR = T / 2, KS = 64 / LPR, BK = 32 * KS;   // lanes of a row, 32-point steps per chunk
    constexpr int TW = T / 32;                                // 16 x 16 tiles of a wave, each way
    __shared__ __align__(16) uint16_t sA[KS * N * (BM / 16) * FT];
    __shared__ __align__(16) uint16_t sB[KS * N * (BN / 16) * FT];
    const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
    const int wp = wv % 2, wn = wv / 2;
    const int li = lane & 15, lg = lane >> 4;
    // XCD mapping as in k_gemm_wg
    const int nmb = (g.M + BM - 1) / BM, nnb = (g.Kout + BN - 1) / BN;
    const long bid = blockIdx.x;
    const long grp = bid / (8L * nmb * nnb);
    const int within = (int)(bid % (8L * nmb * nnb));
    const int tile = within / 8;
    const long split = grp * 8 + (within % 8);
    if (split >= g.n_split) return;              // padding work-groups of the last group
    const int m0 = (tile % nmb) * BM, n0 = (tile / nmb) * BN;
    const bool first_n = (tile / nmb) == 0;
    const long pb = split * g.per_split;
    long pe = pb + g.per_split;
    if (pe > g.P) pe = g.P;
    const int lr = lane % LPR, oct = wv * KS + lane / LPR;    // the lane's columns 2 lr, 2 lr + 1 and 8 points
    floatx4 acc[TW][TW];
#pragma unroll
    for (int a = 0; a < TW; ++a)
#pragma unroll
        for (int b = 0; b < TW; ++b) acc[a][b] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    float2 bsum = make_float2(0.0f, 0.0f);       // sums of A's two columns over the lane's points
    const int ca = m0 + 2 * lr, cb = n0 + 2 * lr;
    const bool in_a = ca < g.M, in_b = cb < g.Kout;   // column counts are even
    // one pair of operands added to acc (and with bias_c the column sums of A)
    const auto pass = [&](auto st_c, auto bias_c, const float* A, const float* B) __attribute__((always_inline)) {
        constexpr int S = decltype(st_c)::value;
        float2 ra[8], rb[8];
        uint32_t ra16[8];                            // ST_A: the raw words, widened once they are used
        auto load = [&](long q0) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const long p = q0 + oct * 8 + j;
                if constexpr ((S & ST_A) != 0) ra16[j] = 0u;
                else ra[j] = make_float2(0.0f, 0.0f);
                rb[j] = make_float2(0.0f, 0.0f);
                if (p < pe) {
                    if (in_a) {
                        if constexpr ((S & ST_A) != 0)
                            ra16[j] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint16_t*>(A) + p * g.lda + ca);
                        else
                            ra[j] = *reinterpret_cast<const float2*>(A + p * g.lda + ca);
                    }
                    if (in_b) rb[j] = *reinterpret_cast<const float2*>(B + p * g.ldb + cb);
                }
            }
        };
        // both columns' 8 points, split, into the fragment image of s
        auto put = [&](uint16_t* s, const float2 (&r)[8]) {
            const int t = lr >> 3, c = (2 * lr) & 15;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                floatx4 lo, hi;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    lo[j] = h ? r[j].y : r[j].x;
                    hi[j] = h ? r[4 + j].y : r[4 + j].x;
                }
                bf16x8 part[N];
                split_bf16x8(lo, hi, part);
#pragma unroll
                for (int q = 0; q < N; ++q)
                    *reinterpret_cast<bf16x8*>(&s[(((oct >> 2) * N + q) * (T / 16) + t) * FT + ((oct & 3) * 16 + wg_slot(c + h, t)) * 8]) = part[q];
            }
        };
        if (pb < pe) load(pb);
        for (long q0 = pb; q0 < pe; q0 += BK) {
            if constexpr ((S & ST_A) != 0) {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    ra[j] = make_float2(__uint_as_float(ra16[j] << 16), __uint_as_float(ra16[j] & 0xffff0000u));
            }
            if constexpr (PRO == PRO_RELU) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    rb[j].x = fmaxf(rb[j].x, 0.0f);
                    rb[j].y = fmaxf(rb[j].y, 0.0f);
                }
            }
            if constexpr (decltype(bias_c)::value) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    bsum.x += ra[j].x;
                    bsum.y += ra[j].y;
                }
            }
            put(sA, ra);
            put(sB, rb);
            __syncthreads();
            if (q0 + BK < pe) load(q0 + BK);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                bf16x8 bf[TW][N];
#pragma unroll
                for (int b = 0; b < TW; ++b)
#pragma unroll
                    for (int q = 0; q < N; ++q)
                        bf[b][q] = *reinterpret_cast<const bf16x8*>(
                            &sB[((ks * N + q) * (T / 16) + wn * TW + b) * FT + (lg * 16 + wg_slot(li, wn * TW + b)) * 8]);
#pragma unroll
                for (int a = 0; a < TW; ++a) {
                    bf16x8 af[N];
#pragma unroll
                    for (int q = 0; q < N; ++q)
                        af[q] = *reinterpret_cast<const bf16x8*>(
                            &sA[((ks * N + q) * (T / 16) + wp * TW + a) * FT + (lg * 16 + wg_slot(li, wp * TW + a)) * 8]);
                    mfma_split<N, TW>(bf, af, acc[a], true);
                }
            }
            __syncthreads();
        }
    };
    if constexpr (ST2 >= 0) {
        pass(std::integral_constant<int, ST2 < 0 ? 0 : ST2>{}, std::false_type{}, g.A2, g.B2);
#pragma unroll
        for (int a = 0; a < TW; ++a)
#pragma unroll
            for (int b = 0; b < TW; ++b) acc[a][b] *= g.scale2;
    }
    pass(std::integral_constant<int, ST>{}, std::true_type{}, g.A, g.B);
    if constexpr (N == 3) {
        if (any_nan(acc)) {                      // on the FP32 instruction: see any_nan
            // operands of point q + lg (zero beyond the split): column m of A, k of B
            const auto left = [&](auto st_c, const float* A, int m, long q) {
                if (q + lg >= pe || m >= g.M) return 0.0f;
                return (decltype(st_c)::value & ST_A) ? ld_bf16(A, (q + lg) * g.lda + m) : A[(q + lg) * g.lda + m];
            };
            const auto right = [&](const float* B, int k, long q) {
                const float y = q + lg < pe && k < g.Kout ? B[(q + lg) * g.ldb + k] : 0.0f;
                return PRO == PRO_RELU ? fmaxf(y, 0.0f) : y;
            };
            const auto st1 = std::integral_constant<int, ST>{};
            const auto st2 = std::integral_constant<int, ST2 < 0 ? 0 : ST2>{};
            uint32_t nm[TW], nk[TW];             // columns with a NaN
#pragma unroll
            for (int a = 0; a < TW; ++a) {
                const int m = m0 + (wp * TW + a) * 16 + li, k = n0 + (wn * TW + a) * 16 + li;
                bool fm = false, fk = false;
#pragma unroll 8
                for (long q = pb; q < pe; q += 4) {
                    float x = left(st1, g.A, m, q), y = right(g.B, k, q);
                    if constexpr (ST2 >= 0) {
                        const float x2 = left(st2, g.A2, m, q), y2 = right(g.B2, k, q);
                        fm |= x2 != x2;
                        fk |= y2 != y2;
                    }
                    fm |= x != x;
                    fk |= y != y;
                }
                nm[a] = rows_with(fm);
                nk[a] = rows_with(fk);
            }
            const auto add = [&](auto st_c, const float* A, const float* B, int m, int k, floatx4 t) {
#pragma unroll 1
                for (long q = pb; q < pe; q += 4)
                    t = __builtin_amdgcn_mfma_f32_16x16x4f32(left(st_c, A, m, q), right(B, k, q), t, 0, 0, 0);
                return t;
            };
#pragma unroll
            for (int a = 0; a < TW; ++a)
#pragma unroll
                for (int b = 0; b < TW; ++b) {
                    if (!wants_fp32(acc[a][b], nm[a], nk[b])) continue;
                    const int m = m0 + (wp * TW + a) * 16 + li, k = n0 + (wn * TW + b) * 16 + li;
                    floatx4 t = {0.0f, 0.0f, 0.0f, 0.0f};
                    if constexpr (ST2 >= 0) t = add(st2, g.A2, g.B2, m, k, t) * g.scale2;
                    take_where_nan(acc[a][b], add(st1, g.A, g.B, m, k, t));
                }
        }
    }
    float* out = g.part + split * (long)g.M * g.Kout;
#pragma unroll
    for (int a = 0; a < TW; ++a)
#pragma unroll
        for (int b = 0; b < TW; ++b) {
            const int k = n0 + (wn * TW + b) * 16 + li;
            if (k >= g.Kout) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = m0 + (wp * TW + a) * 16 + lg * 4 + v;
                if (m < g.M) out[(long)m * g.Kout + k] = acc[a][b][v];
            }
        }
    if (first_n) {
        // the column sums of the chunk's octets of points, added in their order
        float2* sb = reinterpret_cast<float2*>(sA);
        sb[tid] = bsum;
        __syncthreads();
        if (tid < LPR && in_a) {
            float2 t = sb[tid];
            for (int w = 1; w < 4 * KS; ++w) {
                t.x += sb[w * LPR + tid].x;
                t.y += sb[w * LPR + tid].y;
            }
            g.bpart[split * (long)g.M + ca] = t.x;
            g.bpart[split * (long)g.M + ca + 1] = t.y;
        }
    }
}

// dst[m][k] (row stride k_real, k < k_real) (+)= sum_{t < n_split} part[t][m][k]
// A work-group takes 64 outputs; its four waves sum every fourth split, with
// eight interleaved chains that keep eight loads in flight, and the four sums are
// added in order.  Bound by HBM (the partials are read once); one thread per
// output instead left 256 of them per CU waiting on 96 loads each (2 x 384 splits
// of 256 x 256: 57 -> 29 us).
__device__ __forceinline__ float wg_chain_sum(const float* __restrict__ q, long stride, int t0, int t1) {
    float c[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    int t = t0;
    for (; t + 32 <= t1 + 3; t += 32) {
#pragma unroll
        for (int u = 0; u < 8; ++u) c[u] += t + 4 * u < t1 ? q[(long)(t + 4 * u) * stride] : 0.0f;
    }
    for (int u = 0; t < t1; t += 4, ++u) c[u & 7] += q[(long)t * stride];
    return ((c[0] + c[1]) + (c[2] + c[3])) + ((c[4] + c[5]) + (c[6] + c[7]));
}

__global__ __launch_bounds__(256) void k_wg_reduce(const float* __restrict__ part, int n_split, int M, int Kout,
                                                   int k_real, float* __restrict__ dst, int accumulate) {
    __shared__ float sh[4][64];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const long o = (long)blockIdx.x * 64 + lane;
    const bool live = o < (long)M * k_real;
    float s = 0.0f;
    if (live) {
        const int m = (int)(o / k_real), k = (int)(o % k_real);
        const long stride = (long)M * Kout;
        const float* q = part + (long)m * Kout + k;
        s = wg_chain_sum(q, stride, wv, n_split);
    }
    sh[wv][lane] = s;
    __syncthreads();
    if (wv != 0 || !live) return;
    s = ((sh[0][lane] + sh[1][lane]) + sh[2][lane]) + sh[3][lane];
    dst[o] = accumulate ? dst[o] + s : s;
}

// ----------------------------------------------------------------------------
// column sums with fused element functions, two fixed-order stages
//   mode 0: X[p][m]      mode 1: s[p] relu(X[p][m])
//   mode 3: s[p] X[p][m] + X2[p][m]   (s may be NULL)
// ----------------------------------------------------------------------------
// 256 / w threads share a column, w the columns rounded up to a power of two
__global__ __launch_bounds__(256) void k_colsum_partial(const float* __restrict__ X,
                                                        const float* __restrict__ X2,
                                                        const float* __restrict__ s, long ldx,
                                                        long P, int M, int w, long rows_per, int mode,
                                                        float beta, float* __restrict__ part) {
    __shared__ float sh[256];
    const int m = threadIdx.x & (w - 1), step = 256 / w;
    const long rb = (long)blockIdx.x * rows_per;
    long re = rb + rows_per;
    if (re > P) re = P;
    float acc = 0.0f;
    if (m < M) {
#pragma unroll 8
        for (long p = rb + threadIdx.x / w; p < re; p += step) {
            const float x = X[p * ldx + m];
            float d;
            if (mode == 0) d = x;
            else if (mode == 1) d = s[p] * fmaxf(x, 0.0f);
            else d = (s ? s[p] * x : 0.0f) + X2[p * ldx + m];
            acc += d;
        }
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    if (threadIdx.x >= M) return;
    acc = sh[m];
    for (int r = 1; r < step; ++r) acc += sh[r * w + m];
    part[(long)blockIdx.x * M + m] = acc;
}

// dst[m] (+)= scale * sum_b part[b][m]: one work-group per column, thread t
// sums rows t, t + 256, ..., then a fixed-order tree over the 256 threads
__global__ __launch_bounds__(256) void k_colsum_final(const float* __restrict__ part, int nb, int M,
                                                      float scale, float* __restrict__ dst, int accumulate) {
    __shared__ float sh[256];
    const int m = blockIdx.x;
    float s = 0.0f;
    for (int b = threadIdx.x; b < nb; b += 256) s += part[(long)b * M + m];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int d = 128; d >= 1; d >>= 1) {
        if (threadIdx.x < d) sh[threadIdx.x] += sh[threadIdx.x + d];
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    s = sh[0] * scale;
    dst[m] = accumulate ? dst[m] + s : s;
}

// ----------------------------------------------------------------------------
// positional encoding (and its tangent along v / half_size), zero padded to ld
// ----------------------------------------------------------------------------
// column e < 3: x_hat_e; e = 3 + 6k + j: sin (j < 3) or cos (j >= 3) of
// 2^k pi x_hat_{j mod 3}; zero padding up to ld (a multiple of 32, at most 96).
// Bound by the store of X.  Eight threads share a point and form each angle's sine
// and cosine once, both into LDS, from where the rows go out in 16-byte stores
// (a thread per column evaluated every pair twice and divided 64-bit indices: 2^20
// rows of 64 columns 159 -> 55 us, with the tangent 239 -> 120).
constexpr int kPePoints = 32;
__global__ __launch_bounds__(256) void k_pe(long n, const float* __restrict__ xyz, float cx, float cy, float cz,
                                            float inv_half, int L, int ld, float* __restrict__ X,
                                            const float* __restrict__ v, float* __restrict__ Xd) {
    extern __shared__ __align__(16) float pe_rows[];      // [Xd ? 2 : 1][kPePoints][ld + 4]
    const int stride = ld + 4, pt = threadIdx.x >> 3, sub = threadIdx.x & 7;
    const long p0 = (long)blockIdx.x * kPePoints, p = p0 + pt;
    float* const r = pe_rows + pt * stride;
    float* const rd = r + kPePoints * stride;
    if (p < n) {
        const float xh[3] = {(xyz[3 * p] - cx) * inv_half, (xyz[3 * p + 1] - cy) * inv_half, (xyz[3 * p + 2] - cz) * inv_half};
        float vd[3] = {0.0f, 0.0f, 0.0f};
        if (v)
            for (int d = 0; d < 3; ++d) vd[d] = v[3 * p + d] * inv_half;
        for (int q = sub; q < 3 * L; q += 8) {
            const int k = q / 3, d = q - 3 * k, e = 3 + 6 * k + d;
            const float scale = (float)(1 << k), x = d == 0 ? xh[0] : (d == 1 ? xh[1] : xh[2]);
            float sn, cs;
            sincospif(scale * x, &sn, &cs);
            r[e] = sn;
            r[e + 3] = cs;
            if (Xd) {
                const float w = 3.14159265358979f * scale * (d == 0 ? vd[0] : (d == 1 ? vd[1] : vd[2]));
                rd[e] = cs * w;
                rd[e + 3] = -sn * w;
            }
        }
        if (sub < 3) {
            r[sub] = sub == 0 ? xh[0] : (sub == 1 ? xh[1] : xh[2]);
            if (Xd) rd[sub] = sub == 0 ? vd[0] : (sub == 1 ? vd[1] : vd[2]);
        }
        for (int e = 3 + 6 * L + sub; e < ld; e += 8) {
            r[e] = 0.0f;
            if (Xd) rd[e] = 0.0f;
        }
    }
    __syncthreads();
    const int rows = (int)min((long)kPePoints, n - p0), row4 = ld / 4;
    for (int i = threadIdx.x; i < rows * row4; i += 256) {
        const int row = i / row4, c = (i - row * row4) * 4;
        const long o = p0 * ld + 4L * i;
        *reinterpret_cast<float4*>(X + o) = *reinterpret_cast<const float4*>(pe_rows + row * stride + c);
        if (Xd) *reinterpret_cast<float4*>(Xd + o) = *reinterpret_cast<const float4*>(pe_rows + (kPePoints + row) * stride + c);
    }
}

// grad_x f = J_PE^T G0 (G0 = dF/dgamma, row stride ld, a multiple of 4): 16
// lanes per point, each taking every 16th float4 of the row (column e < 3:
// x_hat_e, e = 3 + 6k + j: sin (j < 3) or cos (j >= 3) of 2^k pi x_hat_{j mod 3},
// whose derivative is pi 2^k cos or -pi 2^k sin), then a fixed-order sum over
// the 16 lanes per dimension
__global__ void k_pe_grad(long n, const float* __restrict__ xyz, float cx, float cy, float cz,
                          float inv_half, int L, const float* __restrict__ G0, int ld,
                          float* __restrict__ grad) {
    const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const long p = gid / 16;                  // the 16 lanes of a point exit together
    const int l = (int)(gid % 16);
    if (p >= n) return;
    const float xh[3] = {(xyz[3 * p] - cx) * inv_half, (xyz[3 * p + 1] - cy) * inv_half,
                         (xyz[3 * p + 2] - cz) * inv_half};
    const int ne = 3 + 6 * L;
    float acc[3] = {0.0f, 0.0f, 0.0f};
    for (int m = 4 * l; m < ld && m < ne; m += 64) {
        const float4 g4 = *reinterpret_cast<const float4*>(G0 + p * ld + m);
        const float gv[4] = {g4.x, g4.y, g4.z, g4.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = m + q;
            if (e >= ne) break;
            if (e < 3) {
                acc[e] += gv[q];
            } else {
                const int k = (e - 3) / 6, j = (e - 3) % 6, d = j % 3;
                const float scale = (float)(1 << k);
                const float t = scale * xh[d], w = 3.14159265358979f * scale;
                acc[d] += j < 3 ? w * cospif(t) * gv[q] : -w * sinpif(t) * gv[q];
            }
        }
    }
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int o = 8; o >= 1; o >>= 1) acc[d] += __shfl_xor(acc[d], o, 16);
    if (l == 0) {
        grad[3 * p] = acc[0];   // d/dx = (d/dx_hat) / half, times f's half_size
        grad[3 * p + 1] = acc[1];
        grad[3 * p + 2] = acc[2];
    }
}

// Row kernels: 16 lanes per row (four rows per wave), each lane taking every
// 16th float4 of the row (widths are multiples of 64, rows 16-byte aligned),
// then a fixed-order sum over the 16 lanes.
constexpr int kRowLanes = 16;
__device__ __forceinline__ float row_sum16(float acc) {
#pragma unroll
    for (int d = kRowLanes / 2; d >= 1; d >>= 1) acc += __shfl_xor(acc, d, kRowLanes);
    return acc;
}

// out[p] = post(scale * (sum_m w[m] act(Y[p][m]) + b))
//   act: 0 identity, 3 relu ; post: 0 identity, 1 sigmoid
__global__ __launch_bounds__(256) void k_rowdot(long n, const float* __restrict__ Y, long ldy,
                                                int M, int act, int post, const float* __restrict__ w,
                                                const float* __restrict__ b, float scale, float beta,
                                                float* __restrict__ out) {
    const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const long p = gid / kRowLanes;          // the 16 lanes of a row exit together
    const int l = (int)(gid % kRowLanes);
    if (p >= n) return;
    float acc = 0.0f;
    for (int m = 4 * l; m < M; m += 4 * kRowLanes) {
        const float4 y = *reinterpret_cast<const float4*>(Y + p * ldy + m);
        const bool r = act != PRO_ID;
        acc = __builtin_fmaf(w[m], r ? fmaxf(y.x, 0.0f) : y.x, acc);
        acc = __builtin_fmaf(w[m + 1], r ? fmaxf(y.y, 0.0f) : y.y, acc);
        acc = __builtin_fmaf(w[m + 2], r ? fmaxf(y.z, 0.0f) : y.z, acc);
        acc = __builtin_fmaf(w[m + 3], r ? fmaxf(y.w, 0.0f) : y.w, acc);
    }
    acc = row_sum16(acc);
    if (l == 0) {
        const float v = scale * (acc + b[0]);
        out[p] = post ? sigmoidf_(v) : v;
    }
}

// head output adjoint: ybar3 = g_a a (1-a) with a recomputed; Ybar2 = ybar3 w relu'(Y2)
__global__ __launch_bounds__(256) void k_head_out_bwd(long n, const float* __restrict__ Y2, long ld,
                                                      int M, const float* __restrict__ w,
                                                      const float* __restrict__ b,
                                                      const float* __restrict__ g_a,
                                                      float* __restrict__ ybar3,
                                                      float* __restrict__ Ybar2) {
    const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const long p = gid / kRowLanes;          // the 16 lanes of a row exit together
    const int l = (int)(gid % kRowLanes);
    if (p >= n) return;
    float acc = 0.0f;
    for (int m = 4 * l; m < M; m += 4 * kRowLanes) {
        const float4 y = *reinterpret_cast<const float4*>(Y2 + p * ld + m);
        acc = __builtin_fmaf(w[m], fmaxf(y.x, 0.0f), acc);
        acc = __builtin_fmaf(w[m + 1], fmaxf(y.y, 0.0f), acc);
        acc = __builtin_fmaf(w[m + 2], fmaxf(y.z, 0.0f), acc);
        acc = __builtin_fmaf(w[m + 3], fmaxf(y.w, 0.0f), acc);
    }
    acc = row_sum16(acc);
    const float a = sigmoidf_(acc + b[0]);
    const float yb = g_a ? g_a[p] * a * (1.0f - a) : 0.0f;
    if (l == 0) ybar3[p] = yb;
    for (int m = 4 * l; m < M; m += 4 * kRowLanes) {
        const float4 y = *reinterpret_cast<const float4*>(Y2 + p * ld + m);
        float4 o;
        o.x = y.x > 0.0f ? yb * w[m] : 0.0f;
        o.y = y.y > 0.0f ? yb * w[m + 1] : 0.0f;
        o.z = y.z > 0.0f ? yb * w[m + 2] : 0.0f;
        o.w = y.w > 0.0f ? yb * w[m + 3] : 0.0f;
        *reinterpret_cast<float4*>(Ybar2 + p * ld + m) = o;
    }
}

__global__ void k_fill(float* __restrict__ p, long n, float v) {
    const long o = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (o < n) p[o] = v;
}

// All of a call's weight copies in one launch.  Job k makes an operand
// [N][K] of a GEMM from the parameters, element (n, k) = in[n * C + k] or, for
// the transpose, in[k * C + n], zero outside in[R][C]: as FP32 rows (one unit
// per element), or split in three as the image that the FP32 kernels copy to LDS
// (one unit per 8 k of a row): [block of BM rows][32 k][part][16-row tile][k / 8][row][8 k].
constexpr int kPrepJobs = 40;
struct PrepJob {
    const float* in;
    void* out;
    int R, C, K, transpose, bm;    // bm: rows per block of the image, 0 for FP32 rows
    int parts;                     // of the products that read the image (split_k)
};
struct PrepTable {
    PrepJob job[kPrepJobs];
    long begin[kPrepJobs + 1];     // in units
    int n;
};
__global__ void k_prep_weights(PrepTable t) {
    for (long o = (long)blockIdx.x * blockDim.x + threadIdx.x; o < t.begin[t.n];
         o += (long)gridDim.x * blockDim.x) {
        int k = 0;
        while (k + 1 < t.n && o >= t.begin[k + 1]) ++k;
        const PrepJob& j = t.job[k];
        const long u = o - t.begin[k];
        auto at = [&](int n, int kk) {
            const int r = j.transpose ? kk : n, c = j.transpose ? n : kk;
            return (r < j.R && c < j.C) ? j.in[(long)r * j.C + c] : 0.0f;
        };
        if (j.bm == 0) {
            reinterpret_cast<float*>(j.out)[u] = at((int)(u / j.K), (int)(u % j.K));
        } else {
            const int slot = (int)(u % 64), tiles = j.bm / 16, nk = j.K / 32;
            const int tile = (int)(u / 64) % tiles;
            const int blk = (int)(u / 64 / tiles);             // block of rows * nk + 32-wide k chunk
            const int n = (blk / nk) * j.bm + tile * 16 + (slot & 15), k0 = (blk % nk) * 32 + (slot >> 4) * split_k0(j.parts);
            floatx4 lo, hi;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                lo[e] = at(n, k0 + e);
                hi[e] = at(n, k0 + split_k1(j.parts) + e);
            }
            bf16x8 part[3];
            split_bf16x8(lo, hi, part);
#pragma unroll
            for (int e = 0; e < 8; ++e) {        // beyond BF16's range: from its largest number on
                const float x = e < 4 ? lo[e] : hi[e - 4];
                if (fabsf((float)part[0][e]) != INFINITY) continue;
                part[1][e] = part[2][e] = (__bf16)0.0f;
                if (fabsf(x) == INFINITY) continue;
                part[0][e] = (__bf16)copysignf(3.3895313892515355e38f, x);
                part[1][e] = (__bf16)(x - (float)part[0][e]);
                part[2][e] = (__bf16)(x - (float)part[0][e] - (float)part[1][e]);
            }
            uint16_t* out = reinterpret_cast<uint16_t*>(j.out) + (long)blk * 3 * tiles * 512;
#pragma unroll
            for (int q = 0; q < 3; ++q) *reinterpret_cast<bf16x8*>(&out[((long)q * tiles + tile) * 512 + slot * 8]) = part[q];
        }
    }
}

// ============================================================================
// host orchestration
// ============================================================================
namespace {

constexpr long kChunk = 1 << 20;          // points per pass (bounds the workspace)
// Weight-gradient point splits of a pass over P points: at most kWgSplits (three
// rounds of the 512 work-groups that are resident, four tiles of a 256 x 256
// gradient each), of at least 256 points each (a split writes and the reduction reads
// its whole M x K partial: the training pair of 32768 points took 3.12 ms with 342
// splits of 96 points, 2.45 with 128 of 256).  At 2^20 points 256 splits are equal
// and 128 slower (one round of work-groups: 46.5, 46.3 and 47.7 ms).
#ifndef RFVR_WG_SPLITS
#define RFVR_WG_SPLITS 384
#endif
constexpr int kWgSplits = RFVR_WG_SPLITS;
int wg_splits(long P) { return (int)std::min<long>(kWgSplits, std::max<long>((P + 255) / 256, 1)); }
constexpr int kColBlocks = 2048;          // column-sum partial blocks

struct Layout {
    int L, W, in0, in0p, HL, HW;
    long oW[16], ob[16], o_wout, o_bout, oWh[4], obh[4], o_whout, o_bhout, total;
};

int check_net(const rfvr_mlp* n) {
    if (!n) { set_error("mlp descriptor is NULL"); return RFVR_E_INVALID; }
    if (n->n_layers < 1 || n->n_layers > 16 || n->width < 64 || n->width > 256 || n->width % 64 ||
        n->pe_octaves < 0 || n->pe_octaves > 12 || n->head_layers < 1 || n->head_layers > 4 ||
        n->head_width < 64 || n->head_width > 256 || n->head_width % 64) {
        set_error("unsupported network shape (layers 1..16, width 64..256 step 64, octaves 0..12, "
                  "head 1..4 x 64..256 step 64)");
        return RFVR_E_INVALID;
    }
    if ((3 + 6 * n->pe_octaves + 31) / 32 * 32 > n->width) {
        set_error("encoding width (3 + 6 * pe_octaves, padded to 32) must not exceed the layer width");
        return RFVR_E_INVALID;
    }
    if (!(n->softplus_beta > 0.0f) || !(n->half_size > 0.0f) || n->softplus_beta != n->softplus_beta) {
        set_error("softplus_beta and half_size must be > 0");
        return RFVR_E_INVALID;
    }
    if (n->precision != RFVR_PREC_FP32 && n->precision != RFVR_PREC_BF16 && n->precision != RFVR_PREC_BF16X3 &&
        n->precision != RFVR_PREC_F16) {
        set_error("unknown precision %d", n->precision);
        return RFVR_E_INVALID;
    }
    return RFVR_OK;
}

Layout layout(const rfvr_mlp* n) {
    Layout l;
    l.L = n->n_layers; l.W = n->width; l.HL = n->head_layers; l.HW = n->head_width;
    l.in0 = 3 + 6 * n->pe_octaves;
    l.in0p = (l.in0 + 31) / 32 * 32;
    long off = 0;
    for (int i = 0; i < l.L; ++i) {
        const int fin = i == 0 ? l.in0 : l.W;
        l.oW[i] = off; off += (long)l.W * fin;
        l.ob[i] = off; off += l.W;
    }
    l.o_wout = off; off += l.W;
    l.o_bout = off; off += 1;
    for (int h = 0; h < l.HL; ++h) {
        const int fin = h == 0 ? l.W : l.HW;
        l.oWh[h] = off; off += (long)l.HW * fin;
        l.obh[h] = off; off += l.HW;
    }
    l.o_whout = off; off += l.HW;
    l.o_bhout = off; off += 1;
    l.total = off;
    return l;
}

inline unsigned blocks(long n, int t = 256) { return (unsigned)((n + t - 1) / t); }

// device copies of the weights in the layouts the GEMMs read, 256-byte
// aligned: the split image x for the FP32 products, FP32 rows f for the others
// (in the 16-bit forms only the last sweep product, WT[0], reads an image)
struct WMat {
    float* f = nullptr;
    uint16_t* x = nullptr;
    int parts = 3;         // of the products that read x
};
struct Weights {
    WMat Wp[16];           // W_l [W][fin_pad], zero padded
    WMat WT[16];           // W_l^T [fin_pad][W]
    WMat Whp[4];           // Wh_h [HW][fin]
    WMat WhT[4];           // Wh_h^T [fin][HW]
};

size_t image_words(int N, int K) { return (size_t)((N + block_rows(N) - 1) / block_rows(N)) * block_rows(N) * K * 3; }
size_t wmat_bytes(int N, int K, bool split) {
    return align256(split ? sizeof(uint16_t) * image_words(N, K) : sizeof(float) * (size_t)N * K);
}
WMat take_wmat(WsCursor& cur, int N, int K, bool split, int parts = 3) {
    WMat w;
    w.parts = parts;
    if (split) w.x = cur.take<uint16_t>(image_words(N, K));
    else w.f = cur.take<float>((size_t)N * K);
    return w;
}

struct PrepList {
    PrepTable t = {};
    long total = 0;
    // operand [N][K] of in[R][C] (or of its transpose)
    void add(const float* in, const WMat& w, int R, int C, int N, int K, int transpose) {
        PrepJob& j = t.job[t.n];
        j.in = in; j.R = R; j.C = C; j.K = K; j.transpose = transpose;
        j.bm = w.x ? block_rows(N) : 0;
        j.parts = w.parts;
        j.out = w.x ? (void*)w.x : (void*)w.f;
        t.begin[t.n] = total;
        total += w.x ? (long)(image_words(N, K) / 24) : (long)N * K;
        ++t.n;
    }
    hipError_t launch(hipStream_t st) {
        t.begin[t.n] = total;
        long nb = (total + 255) / 256;
        if (nb > 2048) nb = 2048;
        hipLaunchKernelGGL(k_prep_weights, dim3((unsigned)nb), dim3(256), 0, st, t);
        return hipGetLastError();
    }
};

// Which operands are images.  tangent: the pass multiplies tangents by W_l (the
// training backward); the others multiply values, on the FP32 instruction in FP32
// (see gemm).
struct Images {
    bool first, layer, head, transposed;       // W_0, W_l, Wh_h, and the transposes (W_0^T always is one)
};
Images images(int precision, bool tangent) {
    const bool f32 = precision == RFVR_PREC_FP32, x3 = precision == RFVR_PREC_BF16X3;
    return {f32 && tangent, x3 || (f32 && tangent), x3, f32 || x3};
}

size_t weights_bytes(const Layout& l, int precision, bool tangent) {
    const Images im = images(precision, tangent);
    size_t b = 0;
    for (int i = 0; i < l.L; ++i) {
        const int fin = i == 0 ? l.in0p : l.W;
        b += wmat_bytes(l.W, fin, i == 0 ? im.first : im.layer) + wmat_bytes(fin, l.W, im.transposed || i == 0);
    }
    for (int h = 0; h < l.HL; ++h) {
        const int fin = h == 0 ? l.W : l.HW;
        b += wmat_bytes(l.HW, fin, im.head) + wmat_bytes(fin, l.HW, im.transposed);
    }
    return b;
}

Weights take_weights(WsCursor& cur, const Layout& l, int precision, bool tangent) {
    const Images im = images(precision, tangent);
    const int parts = precision == RFVR_PREC_FP32 ? 3 : 2;
    Weights w;
    for (int i = 0; i < l.L; ++i) {
        const int fin = i == 0 ? l.in0p : l.W;
        w.Wp[i] = take_wmat(cur, l.W, fin, i == 0 ? im.first : im.layer, parts);
        w.WT[i] = take_wmat(cur, fin, l.W, im.transposed || i == 0, i == 0 ? 3 : parts);
    }
    for (int h = 0; h < l.HL; ++h) {
        const int fin = h == 0 ? l.W : l.HW;
        w.Whp[h] = take_wmat(cur, l.HW, fin, im.head, parts);
        w.WhT[h] = take_wmat(cur, fin, l.HW, im.transposed, parts);
    }
    return w;
}

hipError_t prep_weights(const Layout& l, const float* P, const Weights& w, hipStream_t st) {
    PrepList q;
    for (int i = 0; i < l.L; ++i) {          // at most 16 layers and 4 head layers: <= 40 jobs
        const int fin = i == 0 ? l.in0 : l.W, finp = i == 0 ? l.in0p : l.W;
        q.add(P + l.oW[i], w.Wp[i], l.W, fin, l.W, finp, 0);
        q.add(P + l.oW[i], w.WT[i], l.W, fin, finp, l.W, 1);
    }
    for (int h = 0; h < l.HL; ++h) {
        const int fin = h == 0 ? l.W : l.HW;
        q.add(P + l.oWh[h], w.Whp[h], l.HW, fin, l.HW, fin, 0);
        q.add(P + l.oWh[h], w.WhT[h], l.HW, fin, fin, l.HW, 1);
    }
    return q.launch(st);
}

// operand form of the forward products (layers, head, the grad_x f sweep) and
// of the backward's products (tangent, adjoints, weight gradients)
int mm_fwd(int precision) {
    switch (precision) {
    case RFVR_PREC_BF16: return MM_BF16;
    case RFVR_PREC_BF16X3: return MM_BF16X3;
    case RFVR_PREC_F16: return MM_F16;
    default: return MM_FP32;
    }
}
int mm_bwd(int precision) { return precision == RFVR_PREC_F16 ? MM_BF16 : mm_fwd(precision); }

// forms that multiply operands split in parts, and how many
constexpr bool is_split(int mm) { return mm == MM_FP32 || mm == MM_BF16X3; }
constexpr int split_parts(int mm) { return mm == MM_FP32 ? 3 : 2; }

// launch context of the network passes: stream and matrix-operand precision
// (16-bit operands, FP32 accumulation; layers reading the encoding stay FP32)
struct Cx {
    hipStream_t st;
    int mm;        // MM_*
};

// point tiles of tp points x output blocks, 8 point tiles per XCD group
dim3 gemm_grid(long P, int tp, int M, int bm) {
    const long groups = ((P + tp - 1) / tp + 7) / 8;
    return dim3((unsigned)(groups * 8 * ((M + bm - 1) / bm)));
}

// Tile of the split products: 128 x 128 where they fill the 256 CUs; below that the
// 64 x 64 ones put four times the work-groups on the chip.  Training backward of the
// 8 x 256 network with 64 | 128, in us: 4096 points (64 large tiles) 637 | 764, 12000
// (192) 838 | 933, 16384 (256) 879 | 858, 20000 (320) 1063 | 1052, 24000 (384) 1127 |
// 1160, 28000 (448) 1231 | 1277, 32768 (512) 1326 | 1274, 131072 4610 | 4365: from
// one tile a CU on either side wins by a few per cent as the last round is full or not.
int split_tile(long P, int M) { return M <= 64 || gemm_grid(P, 128, M, 128).x < 384 ? 64 : 128; }

template <int PRO, int EPI, int MM, int ST = 0>
void gemm_launch(const GemmArgs& a, hipStream_t st) {
    const int bm = block_rows(a.M);
    const dim3 grid = gemm_grid(a.P, 128, a.M, bm);
    if constexpr (MM == MM_FP32 || MM == MM_BF16X3) {
        static_assert(ST == 0, "the split kernel has no BF16 storage");
        constexpr int N = split_parts(MM);
        // Up to two large tiles a CU (512) take all their outputs at a time: two waves per
        // SIMD are all that come then, and LDS is read less; above, three fit in halves.
        // Training backward of the 8 x 256 network, all | halves, in us: 24000 points
        // (384 tiles) 1157 | 1184, 32768 (512) 1266 | 1282, 36000 (576) 1610 | 1577,
        // 65536 2321 | 2379, 2^20 31537 | 31456 (its forward with the sweep 17722 | 17089).
        const dim3 g128 = gemm_grid(a.P, 128, a.M, 128);
        if (split_tile(a.P, a.M) == 64)
            hipLaunchKernelGGL((k_gemm_nt32<PRO, EPI, 64, 2, N>), gemm_grid(a.P, 64, a.M, 64), dim3(256), 0, st, a);
        else if (g128.x <= 512)
            hipLaunchKernelGGL((k_gemm_nt32<PRO, EPI, 128, 4, N>), g128, dim3(256), 0, st, a);
        else
            hipLaunchKernelGGL((k_gemm_nt32<PRO, EPI, 128, 2, N>), g128, dim3(256), 0, st, a);
    } else {
        if constexpr (MM == MM_MFMA32 && ST == 0) {
            // 64 x 64 tiles below two large ones a CU; the sums are the same, a tile's k order
            // does not depend on its size.  Training forward of the 8 x 256 network, 64 |
            // 128, in us: 4096 points 185 | 296, 28000 (448 large tiles) 657 | 748, 32768
            // (512) 668 | 642, 49152 (768) 943 | 936, 65536 1231 | 1311, 98304 1786 | 1740.
            if (grid.x < 512) {
                hipLaunchKernelGGL((k_gemm_nt<PRO, EPI, 64, MM, ST, 64>), gemm_grid(a.P, 64, a.M, 64), dim3(256), 0, st, a);
                return;
            }
        }
        if (bm == 64) hipLaunchKernelGGL((k_gemm_nt<PRO, EPI, 64, MM, ST>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((k_gemm_nt<PRO, EPI, 128, MM, ST>), grid, dim3(256), 0, st, a);
    }
}

template <int PRO, int EPI>
void gemm(const GemmArgs& a, const Cx& cx) {
    // the FP16 form exists for the forward products' epilogues only (a
    // backward context never carries MM_F16: mm_bwd maps it to BF16)
    constexpr bool FWD_EPI = EPI == EPI_BIAS || EPI == EPI_BIAS_SP || EPI == EPI_DSPMUL;
    // The values of layers and head stay on the FP32 instruction in FP32: the signs of
    // the head's pre-activations are its ReLU masks, which the parameter gradient
    // shows.  2^20 points have some ten units per layer whose sign another rounding
    // changes, and those alone move it by 3e-7 to 2.9e-6 (six seeds; all the
    // products of the gradient 3e-7).
    constexpr bool VALUE = EPI == EPI_BIAS || EPI == EPI_BIAS_SP;
    if (cx.mm == MM_BF16) gemm_launch<PRO, EPI, MM_BF16>(a, cx.st);
    else if (cx.mm == MM_BF16X3) gemm_launch<PRO, EPI, MM_BF16X3>(a, cx.st);
    else if (cx.mm == MM_F16) {
        if constexpr (FWD_EPI) gemm_launch<PRO, EPI, MM_F16>(a, cx.st);
        else gemm_launch<PRO, EPI, MM_BF16>(a, cx.st);
    } else if constexpr (VALUE) gemm_launch<PRO, EPI, MM_MFMA32>(a, cx.st);
    else gemm_launch<PRO, EPI, MM_FP32>(a, cx.st);
}

// FP32 GEMM whatever the context (the last sweep product: its result is the
// encoding's adjoint)
template <int PRO, int EPI>
void gemm32(const GemmArgs& a, const Cx& cx) {
    gemm_launch<PRO, EPI, MM_FP32>(a, cx.st);
}

// The first layer's products, FP32 in every form (their operand is the
// encoding).  Only the FP32 training backward's tangent comes with an image.  The
// 16-bit forms keep the FP32 instruction: a last-bit change of this layer would move
// the 16-bit roundings of all that follow (6e-5 of the gradient in the FP16 form),
// and a product over at most 96 k is bound by the activations it writes either way.
template <int EPI, int ST = 0>
void gemm_first(const GemmArgs& a, const Cx& cx) {
    if constexpr (ST == 0) {
        if (!a.B) return gemm_launch<PRO_ID, EPI, MM_FP32>(a, cx.st);
    }
    gemm_launch<PRO_ID, EPI, MM_MFMA32, ST>(a, cx.st);
}

// BF16 GEMM of the single-rounded BF16 backward with the ST_* operands in BF16
// storage
template <int PRO, int EPI, int ST>
void gemm_b16(const GemmArgs& a, const Cx& cx) {
    gemm_launch<PRO, EPI, MM_BF16, ST>(a, cx.st);
}

#ifndef RFVR_DUAL_NW
#define RFVR_DUAL_NW 4
#endif
template <int EPI2>
void gemm_dual(const DualArgs& a, int mm, hipStream_t st) {
    if (EPI2 == EPI2_FWD && mm == MM_FP32) mm = MM_MFMA32;       // values: see gemm
    if (is_split(mm)) {
        const int bm = block_rows(a.M);
        const dim3 grid = gemm_grid(a.P, 64, a.M, bm);
        const auto go = [&](auto n) {
            constexpr int N = decltype(n)::value;
            if (bm == 64) hipLaunchKernelGGL((k_gemm_dual32<EPI2, 64, N>), grid, dim3(256), 0, st, a);
            else hipLaunchKernelGGL((k_gemm_dual32<EPI2, 128, N>), grid, dim3(256), 0, st, a);
        };
        if constexpr (EPI2 == EPI2_ADJ) {
            if (mm == MM_FP32) return go(std::integral_constant<int, 3>{});
        }
        return go(std::integral_constant<int, 2>{});
    }
    constexpr int NW = RFVR_DUAL_NW, BP = NW == 8 ? 128 : 64;
    const dim3 grid = gemm_grid(a.P, BP, a.M, 128);
    if constexpr (EPI2 == EPI2_FWD) {
        if (mm == MM_F16 || mm == MM_MFMA32) {
            if (mm == MM_F16) hipLaunchKernelGGL((k_gemm_dual<EPI2, MM_F16, NW>), grid, dim3(NW * 64), 0, st, a);
            else hipLaunchKernelGGL((k_gemm_dual<EPI2, MM_MFMA32, NW>), grid, dim3(NW * 64), 0, st, a);
            return;
        }
    }
    hipLaunchKernelGGL((k_gemm_dual<EPI2, MM_BF16, NW>), grid, dim3(NW * 64), 0, st, a);
}

DualArgs da(const float* A, const float* A2, long lda, const WMat& B, long ldb, const float* bias,
            const float* C, const float* C2, float* Y, float* Y2, float* Y3, long ldy,
            long P, int M, int K, float beta) {
    DualArgs g;
    g.A = A; g.A2 = A2; g.lda = lda; g.B = B.f; g.ldb = ldb; g.Bx = B.x; g.bias = bias; g.C = C; g.C2 = C2;
    g.Y = Y; g.Y2 = Y2; g.Y3 = Y3; g.ldy = ldy; g.P = P; g.M = M; g.K = K; g.beta = beta;
    return g;
}

GemmArgs ga(const float* A, long lda, const WMat& B, long ldb, const float* bias,
            float* Y, long ldy, long P, int M, int K, float beta, const float* C = nullptr,
            long ldc = 0, float* Y2 = nullptr) {
    GemmArgs g = {};
    g.A = A; g.lda = lda; g.B = B.f; g.ldb = ldb; g.Bx = B.x; g.bias = bias; g.C = C; g.ldc = ldc;
    g.Y = Y; g.ldy = ldy; g.Y2 = Y2; g.P = P; g.M = M; g.K = K; g.beta = beta;
    return g;
}

// 64 x 64 tiles where they cover at most half of what 128 x 128 ones do: the matrix
// cores then bound the padded product (262144 points, 64 x 64 and 64 x 32: 70 and
// 68 -> 33 and 32 us; a trunk's first layer, 256 x 64 at 150001 points: 148 -> 111)
bool wg_narrow(int M, int Kout) {
    const auto area = [&](long t) { return (M + t - 1) / t * t * ((Kout + t - 1) / t * t); };
    return 2 * area(64) <= area(128);
}

// A's and B's product, and with A2 the second pair's times scale2
template <int PRO, int ST = 0, int ST2 = -1>
void wgrad(const float* A, long lda, int M, const float* B, long ldb, int Kout, long P, float* part, float* bpart,
           const Cx& cx, const float* A2 = nullptr, const float* B2 = nullptr, float scale2 = 1.0f) {
    WgArgs g;
    g.A = A; g.lda = lda; g.B = B; g.ldb = ldb; g.part = part; g.bpart = bpart; g.P = P;
    g.A2 = A2; g.B2 = B2; g.scale2 = scale2;
    const int ns = wg_splits(P);
    g.M = M; g.Kout = Kout; g.per_split = ((P + ns - 1) / ns + 31) / 32 * 32;
    g.n_split = ns;
    const bool narrow = is_split(cx.mm) && wg_narrow(M, Kout);
    const int T = narrow ? 64 : 128;
    const long tiles = (long)((M + T - 1) / T) * ((Kout + T - 1) / T);
    const long groups = (ns + 7) / 8;
    const dim3 grid((unsigned)(groups * 8 * tiles));
    // 16-bit storage comes with single BF16 products, or with FP32 ones (the first layer)
    if (cx.mm == MM_BF16) {
        hipLaunchKernelGGL((k_gemm_wg<PRO, ST, ST2>), grid, dim3(256), 0, cx.st, g);
        return;
    }
    if constexpr (ST == 0 && ST2 <= 0) {
        if (cx.mm == MM_BF16X3) {
            if (narrow) hipLaunchKernelGGL((k_gemm_wg32<PRO, ST, ST2, 64, 2>), grid, dim3(256), 0, cx.st, g);
            else hipLaunchKernelGGL((k_gemm_wg32<PRO, ST, ST2, 128, 2>), grid, dim3(256), 0, cx.st, g);
            return;
        }
    }
    if constexpr (ST2 != ST_B) {
        if (narrow) hipLaunchKernelGGL((k_gemm_wg32<PRO, ST, ST2, 64>), grid, dim3(256), 0, cx.st, g);
        else hipLaunchKernelGGL((k_gemm_wg32<PRO, ST, ST2>), grid, dim3(256), 0, cx.st, g);
    }
}

void wg_reduce(const float* part, int n_split, int M, int Kout, int k_real, float* dst, int acc, hipStream_t st) {
    hipLaunchKernelGGL(k_wg_reduce, dim3(blocks((long)M * k_real, 64)), dim3(256), 0, st, part, n_split, M, Kout, k_real,
                       dst, acc);
}

// the positional encoding of n points, and with Xd its tangent along v (or 0)
void encode(long n, const float* xyz, const float* centre, float inv_half, int octaves, int ld, float* X, const float* v,
            float* Xd, hipStream_t st) {
    hipLaunchKernelGGL(k_pe, dim3(blocks(n, kPePoints)), dim3(256), sizeof(float) * (Xd ? 2 : 1) * kPePoints * (ld + 4), st, n,
                       xyz, centre[0], centre[1], centre[2], inv_half, octaves, ld, X, v, Xd);
}

void colsum(const float* X, const float* X2, const float* s, long ldx, long P, int M, int mode,
            float beta, float scale, float* part, float* dst, int acc, hipStream_t st) {
    // at least 64 rows per work-group
    const long nb = std::min<long>(kColBlocks, (P + 63) / 64), per = (P + nb - 1) / nb;
    int w = 1;
    while (w < M) w *= 2;
    hipLaunchKernelGGL(k_colsum_partial, dim3((unsigned)nb), dim3(256), 0, st, X, X2, s, ldx, P, M, w, per, mode, beta, part);
    hipLaunchKernelGGL(k_colsum_final, dim3(M), dim3(256), 0, st, part, (int)nb, M, scale, dst, acc);
}

// --- forward workspace -------------------------------------------------------
// keep: the layers' (Z, H) go to the caller's reserve instead of the workspace
size_t fwd_bytes(const Layout& l, int prec, long n, bool keep) {
    const long c = n < kChunk ? n : kChunk;
    return weights_bytes(l, prec, false) + align256(sizeof(float) * c * l.in0p) +
           (keep ? 0 : (size_t)l.L * align256(sizeof(float) * c * l.W)) + 2 * align256(sizeof(float) * c * l.W) +
           (keep ? 0 : (size_t)l.HL * align256(sizeof(float) * c * l.HW));   // head Y (else in the reserve)
}

// --- backward workspace ------------------------------------------------------
// point rows of the top-adjoint GEMM's column partials: one per point tile
int top_tile(int mm, long P, int M) { return is_split(mm) ? split_tile(P, M) : 128; }
long top_rows(long n, int tile) { return (n + tile - 1) / tile; }

size_t bwd_bytes(const Layout& l, int prec, long n, bool keep) {
    const long c = n < kChunk ? n : kChunk;
    const long wmax = l.W > l.in0p ? l.W : l.in0p;
    return weights_bytes(l, prec, keep) + 2 * align256(sizeof(float) * c * l.in0p) +
           (keep ? 1 : 3) * (size_t)l.L * align256(sizeof(float) * c * l.W) +  // Hdot (and Z, H)
           4 * align256(sizeof(float) * c * l.W) +                  // Hbar, Hdotbar, Zbar, Zdotbar
           (keep ? 1 : 2) * (size_t)l.HL * align256(sizeof(float) * c * l.HW) +  // head Ybar (and Y)
           align256(sizeof(float) * c) +                            // ybar3
           align256(sizeof(float) * kWgSplits * (size_t)l.W * wmax) +
           align256(sizeof(float) * kWgSplits * (size_t)l.W) +
           align256(sizeof(float) * (size_t)kColBlocks * (l.W > l.HW ? l.W : l.HW)) +
           align256(sizeof(float) * (size_t)top_rows(c, 64) * l.W);   // output layer column partials
}

// --- reserve of the training pair, [n][W] per trunk layer: H_i = sp(Z_i) and
// the normal sweep's adjoint S_i = df/dZ_i; then [n][HW] per head layer: its
// output before the relu ----------------------------------------------------------
size_t reserve_layer_bytes(const Layout& l, long n) { return align256(sizeof(float) * (size_t)n * l.W); }
size_t reserve_head_bytes(const Layout& l, long n) { return align256(sizeof(float) * (size_t)n * l.HW); }
size_t reserve_bytes(const Layout& l, long n) {
    return 2 * (size_t)l.L * reserve_layer_bytes(l, n) + (size_t)l.HL * reserve_head_bytes(l, n);
}
float* reserve_h(void* r, const Layout& l, long n, int i) {
    return reinterpret_cast<float*>(static_cast<char*>(r) + (size_t)i * reserve_layer_bytes(l, n));
}
float* reserve_s(void* r, const Layout& l, long n, int i) { return reserve_h(r, l, n, l.L + i); }
float* reserve_y(void* r, const Layout& l, long n, int h) {
    return reinterpret_cast<float*>(static_cast<char*>(r) + 2 * (size_t)l.L * reserve_layer_bytes(l, n) +
                                    (size_t)h * reserve_head_bytes(l, n));
}

int check_buffers(void* ws, size_t ws_bytes, size_t need, void* reserve, size_t reserve_bytes_, size_t rneed) {
    if (!ws || ws_bytes < need || (reinterpret_cast<uintptr_t>(ws) & 255u)) {
        set_error("workspace too small or misaligned: need %zu bytes", need);
        return RFVR_E_WORKSPACE;
    }
    if (rneed && (!reserve || reserve_bytes_ < rneed || (reinterpret_cast<uintptr_t>(reserve) & 255u))) {
        set_error("reserve too small or misaligned: need %zu bytes", rneed);
        return RFVR_E_WORKSPACE;
    }
    return RFVR_OK;
}

int mlp_forward(const rfvr_mlp* net, const float* xyz, long n, float* sdf, float* grad, float* refl,
                void* reserve, size_t reserve_bytes_, void* ws, size_t ws_bytes, hipStream_t st) {
    int rc;
    if ((rc = check_net(net))) return rc;
    if (n < 1 || n > RFVR_MAX_POINTS || !xyz || !net->params) {
        set_error("n in [1, RFVR_MAX_POINTS], xyz and params are required");
        return RFVR_E_INVALID;
    }
    const Layout l = layout(net);
    const bool keep = reserve_bytes_ != 0 || reserve != nullptr;
    if ((rc = check_buffers(ws, ws_bytes, fwd_bytes(l, net->precision, n, keep), reserve, reserve_bytes_,
                            keep ? reserve_bytes(l, n) : 0)))
        return rc;
    const Cx cx{st, mm_fwd(net->precision)};
    const float* P = net->params;
    const float beta = net->softplus_beta, half = net->half_size, inv_half = 1.0f / net->half_size;
    const long chunk = n < kChunk ? n : kChunk;
    WsCursor cur{reinterpret_cast<char*>(ws), 0};
    const Weights w = take_weights(cur, l, net->precision, false);
    float* X0 = cur.take<float>((size_t)chunk * l.in0p);
    float* Hw[16];
    for (int i = 0; i < l.L && !keep; ++i) Hw[i] = cur.take<float>((size_t)chunk * l.W);
    float* G[2] = {cur.take<float>((size_t)chunk * l.W), cur.take<float>((size_t)chunk * l.W)};
    float* Yw[4];
    for (int h = 0; h < l.HL && !keep; ++h) Yw[h] = cur.take<float>((size_t)chunk * l.HW);
    if ((rc = hip_status(prep_weights(l, P, w, st), "mlp weight prep"))) return rc;

    for (long c0 = 0; c0 < n; c0 += chunk) {
        const long m = (n - c0) < chunk ? (n - c0) : chunk;
        const float* x = xyz + 3 * c0;
        encode(m, x, net->centre, inv_half, net->pe_octaves, l.in0p, X0, nullptr, nullptr, st);
        // H_i = sp(H_{i-1} W_i^T + b_i) from the epilogue (the reserve's, or
        // the workspace's until the sweep has used them)
        float* H[16];
        for (int i = 0; i < l.L; ++i) H[i] = keep ? reserve_h(reserve, l, n, i) + c0 * l.W : Hw[i];
        gemm_first<EPI_BIAS_SP>(ga(X0, l.in0p, w.Wp[0], l.in0p, P + l.ob[0], H[0], l.W, m, l.W, l.in0p, beta),
                                    cx);
        for (int i = 1; i < l.L; ++i)
            gemm<PRO_ID, EPI_BIAS_SP>(ga(H[i - 1], l.W, w.Wp[i], l.W, P + l.ob[i], H[i], l.W, m, l.W, l.W, beta),
                                      cx);
        float* Ht = H[l.L - 1];
        if (sdf)
            hipLaunchKernelGGL(k_rowdot, dim3(blocks(m * kRowLanes)), dim3(256), 0, st, m, Ht, (long)l.W, l.W,
                               (int)PRO_ID, 0, P + l.o_wout, P + l.o_bout, half, beta, sdf + c0);
        if (refl || keep) {
            // head layers (the training forward keeps their outputs in the reserve)
            float* Yh[4];
            for (int h = 0; h < l.HL; ++h) Yh[h] = keep ? reserve_y(reserve, l, n, h) + c0 * l.HW : Yw[h];
            gemm<PRO_ID, EPI_BIAS>(ga(Ht, l.W, w.Whp[0], l.W, P + l.obh[0], Yh[0], l.HW, m, l.HW, l.W, beta), cx);
            for (int h = 1; h < l.HL; ++h)
                gemm<PRO_RELU, EPI_BIAS>(ga(Yh[h - 1], l.HW, w.Whp[h], l.HW, P + l.obh[h], Yh[h], l.HW, m, l.HW, l.HW, beta), cx);
            if (refl)
                hipLaunchKernelGGL(k_rowdot, dim3(blocks(m * kRowLanes)), dim3(256), 0, st, m, Yh[l.HL - 1], (long)l.HW,
                                   l.HW, (int)PRO_RELU, 1, P + l.o_whout, P + l.o_bhout, 1.0f, beta, refl + c0);
        }
        if (grad || keep) {
            // adjoint of f w.r.t. Z_{L-1}: S_{L-1} = sp'(Z_{L-1}) w_out, formed from
            // H_{L-1} as the first product's operand (PRO_SEED); then
            // S_{i-1} = (S_i W_i) . sp'(Z_{i-1})
            // (epilogue), and dgamma = S_0 W_0.  The training forward keeps S_i
            // (i < L-1) in the reserve: scaled by half_size, S_i and S_i / sp'(Z_i)
            // are the backward's adjoints of the tangent pass to Zdot_i and Hdot_i,
            // so the backward does not recompute them.
            int cur_g = 0;
            for (int i = l.L - 1; i >= 0; --i) {
                const int mout = i == 0 ? l.in0p : l.W;
                const bool top = i == l.L - 1;
                const float* src = top ? Ht : (keep ? reserve_s(reserve, l, n, i) + c0 * l.W : G[cur_g]);
                float* dst = (keep && i > 0) ? reserve_s(reserve, l, n, i - 1) + c0 * l.W : G[cur_g ^ 1];
                GemmArgs a = ga(src, l.W, w.WT[i], l.W, nullptr, dst, mout, m, mout, l.W, beta,
                                i > 0 ? H[i - 1] : nullptr, l.W);
                a.colv = P + l.o_wout;
                if (i > 0) {
                    if (top) gemm<PRO_SEED, EPI_DSPMUL>(a, cx);
                    else gemm<PRO_ID, EPI_DSPMUL>(a, cx);
                } else {    // the product with W_0 stays FP32
                    if (top) gemm32<PRO_SEED, EPI_BIAS>(a, cx);
                    else gemm32<PRO_ID, EPI_BIAS>(a, cx);
                }
                cur_g ^= 1;
            }
            if (grad)
                hipLaunchKernelGGL(k_pe_grad, dim3(blocks(m * 16)), dim3(256), 0, st, m, x, net->centre[0],
                                   net->centre[1], net->centre[2], inv_half, net->pe_octaves, G[cur_g],
                                   l.in0p, grad + 3 * c0);
        }
        if ((rc = hip_status(hipGetLastError(), "mlp forward"))) return rc;
    }
    return RFVR_OK;
}

// Side stream of the training backward.  A trunk layer's two weight-gradient
// products read its Zbar and arrays that stay fixed during the sweep (the
// reserve's H and S, the tangents, the encoding), and write only their own
// partials and gradient rows; so they run on a second stream beside the chain
// of adjoint products, ordered by events: they start once Zbar is written, and
// the adjoint product that next overwrites that Zbar buffer waits for them.
// One side stream per device, default priority, created on first use and held
// until the process ends; a backward call holds its mutex while it enqueues,
// so calls from several host threads on one device take turns.
struct SideStream {
    hipStream_t ss = nullptr;
    hipEvent_t ready[16] = {}, done[16] = {};
    std::mutex mu;
};
std::mutex g_side_mu;
SideStream* g_side[64] = {};

int side_stream(SideStream** out) {
    int dev = -1;
    int rc;
    if ((rc = hip_status(hipGetDevice(&dev), "hipGetDevice"))) return rc;
    if (dev < 0 || dev >= 64) { set_error("device index %d beyond 64", dev); return RFVR_E_UNSUPPORTED; }
    std::lock_guard<std::mutex> lock(g_side_mu);
    if (!g_side[dev]) {
        SideStream* s = new SideStream();
        if ((rc = hip_status(hipStreamCreateWithFlags(&s->ss, hipStreamNonBlocking), "side stream"))) {
            delete s;
            return rc;
        }
        for (int k = 0; k < 16; ++k) {
            if ((rc = hip_status(hipEventCreateWithFlags(&s->ready[k], hipEventDisableTiming), "side event")) ||
                (rc = hip_status(hipEventCreateWithFlags(&s->done[k], hipEventDisableTiming), "side event")))
                return rc;          // the partly built context is kept out of g_side (leaked, error path)
        }
        g_side[dev] = s;
    }
    *out = g_side[dev];
    return RFVR_OK;
}

int mlp_backward(const rfvr_mlp* net, const float* xyz, long n, const float* g_sdf, const float* g_grad,
                 const float* g_refl, uint32_t flags, float* g_params, void* reserve, size_t reserve_bytes_,
                 void* ws, size_t ws_bytes, hipStream_t st) {
    int rc;
    if ((rc = check_net(net))) return rc;
    if (n < 1 || n > RFVR_MAX_POINTS || !xyz || !net->params || !g_params) {
        set_error("n in [1, RFVR_MAX_POINTS], xyz, params and g_params are required");
        return RFVR_E_INVALID;
    }
    if (flags & ~(uint32_t)RFVR_ACCUMULATE) { set_error("only RFVR_ACCUMULATE is meaningful here"); return RFVR_E_INVALID; }
    const Layout l = layout(net);
    const bool keep = reserve_bytes_ != 0 || reserve != nullptr;
    if ((rc = check_buffers(ws, ws_bytes, bwd_bytes(l, net->precision, n, keep), reserve, reserve_bytes_,
                            keep ? reserve_bytes(l, n) : 0)))
        return rc;
    // cxf: the plain backward's recompute of the forward products, in the
    // forward's operand form; cx: the backward's own products
    const Cx cx{st, mm_bwd(net->precision)}, cxf{st, mm_fwd(net->precision)};
    // the training pair's weight gradients run on the side stream when the
    // products are bound by the matrix cores (FP32); the BF16 forms are bound by
    // HBM and gain nothing measurable from it
    SideStream* side = nullptr;
    std::unique_lock<std::mutex> side_lock;
    if (keep && cx.mm == MM_FP32) {
        if ((rc = side_stream(&side))) return rc;
        side_lock = std::unique_lock<std::mutex>(side->mu);
    }
    const hipStream_t wst = side ? side->ss : st;
    const Cx cxw{wst, cx.mm}, cx32w{wst, MM_FP32};
    // single-rounded BF16 products in the training backward: the tangents Hdot
    // and the adjoints Zbar are stored in BF16 (every product reading them rounds
    // them so), which cuts the HBM bytes of these HBM-bound products by ~30 %
    const bool b16 = keep && cx.mm == MM_BF16;
    const float* P = net->params;
    float* GP = g_params;
    const float beta = net->softplus_beta, half = net->half_size, inv_half = 1.0f / net->half_size;
    const long chunk = n < kChunk ? n : kChunk;
    const long wmax = l.W > l.in0p ? l.W : l.in0p;
    WsCursor cur{reinterpret_cast<char*>(ws), 0};
    const Weights w = take_weights(cur, l, net->precision, keep);
    float* X0 = cur.take<float>((size_t)chunk * l.in0p);
    float* X0d = cur.take<float>((size_t)chunk * l.in0p);
    float *Zw[16], *Hw[16], *Hd[16];
    for (int i = 0; i < l.L && !keep; ++i) Zw[i] = cur.take<float>((size_t)chunk * l.W);
    for (int i = 0; i < l.L && !keep; ++i) Hw[i] = cur.take<float>((size_t)chunk * l.W);
    for (int i = 0; i < l.L; ++i) Hd[i] = cur.take<float>((size_t)chunk * l.W);
    float* Hb = cur.take<float>((size_t)chunk * l.W);
    float* Hdb = cur.take<float>((size_t)chunk * l.W);
    float* Zb = cur.take<float>((size_t)chunk * l.W);
    float* Zdb = cur.take<float>((size_t)chunk * l.W);
    float *Yw[4], *Ybh[4];
    for (int h = 0; h < l.HL && !keep; ++h) Yw[h] = cur.take<float>((size_t)chunk * l.HW);
    for (int h = 0; h < l.HL; ++h) Ybh[h] = cur.take<float>((size_t)chunk * l.HW);
    float* yb3 = cur.take<float>((size_t)chunk);
    float* part = cur.take<float>((size_t)kWgSplits * l.W * wmax);
    float* bpart = cur.take<float>((size_t)kWgSplits * l.W);
    float* cpart = cur.take<float>((size_t)kColBlocks * (l.W > l.HW ? l.W : l.HW));
    float* tpart = cur.take<float>((size_t)top_rows(chunk, 64) * l.W);
    if ((rc = hip_status(prep_weights(l, P, w, st), "mlp weight prep"))) return rc;

    for (long c0 = 0; c0 < n; c0 += chunk) {
        const long m = (n - c0) < chunk ? (n - c0) : chunk;
        const int acc = (c0 > 0 || (flags & RFVR_ACCUMULATE)) ? 1 : 0;
        const int ns = wg_splits(m);
        const float* x = xyz + 3 * c0;
        const float* gf = g_sdf ? g_sdf + c0 : nullptr;
        const float* ga_ = g_refl ? g_refl + c0 : nullptr;
        float *Z[16], *H[16];   // Z: the plain backward's recomputed pre-activations only
        for (int i = 0; i < l.L; ++i) {
            Z[i] = keep ? nullptr : Zw[i];
            H[i] = keep ? reserve_h(reserve, l, n, i) + c0 * l.W : Hw[i];
        }
        // encoding and its tangent along g_grad
        encode(m, x, net->centre, inv_half, net->pe_octaves, l.in0p, X0, g_grad ? g_grad + 3 * c0 : nullptr, X0d, st);
        if (keep) {
            // tangent only: Hdot_i = sp'(Z_i) (Hdot_{i-1} W_i^T), sp'(Z_i) from the
            // reserve's H_i
            const GemmArgs a0 = ga(X0d, l.in0p, w.Wp[0], l.in0p, nullptr, Hd[0], l.W, m, l.W, l.in0p, beta, H[0], l.W);
            if (b16) gemm_first<EPI_DSPMUL, ST_Y>(a0, cx);
            else gemm_first<EPI_DSPMUL>(a0, cx);
            for (int i = 1; i < l.L; ++i) {
                const GemmArgs a = ga(Hd[i - 1], l.W, w.Wp[i], l.W, nullptr, Hd[i], l.W, m, l.W, l.W, beta, H[i], l.W);
                if (b16) gemm_b16<PRO_ID, EPI_DSPMUL, ST_A | ST_Y>(a, cx);
                else gemm<PRO_ID, EPI_DSPMUL>(a, cx);
            }
        } else {
            // one dual GEMM per layer: (Z_i, H_i) and Hdot_i share W_i
            gemm_dual<EPI2_FWD>(da(X0, X0d, l.in0p, w.Wp[0], l.in0p, P + l.ob[0], nullptr, nullptr, Z[0], H[0], Hd[0],
                                   l.W, m, l.W, l.in0p, beta), MM_MFMA32, st);
            for (int i = 1; i < l.L; ++i)
                gemm_dual<EPI2_FWD>(da(H[i - 1], Hd[i - 1], l.W, w.Wp[i], l.W, P + l.ob[i], nullptr, nullptr, Z[i],
                                       H[i], Hd[i], l.W, m, l.W, l.W, beta), cxf.mm, st);
        }
        float* Ht = H[l.L - 1];
        // head forward (the training backward reads it from the reserve)
        float* Yh[4];
        for (int h = 0; h < l.HL; ++h) Yh[h] = keep ? reserve_y(reserve, l, n, h) + c0 * l.HW : Yw[h];
        if (!keep) {
            gemm<PRO_ID, EPI_BIAS>(ga(Ht, l.W, w.Whp[0], l.W, P + l.obh[0], Yh[0], l.HW, m, l.HW, l.W, beta), cxf);
            for (int h = 1; h < l.HL; ++h)
                gemm<PRO_RELU, EPI_BIAS>(ga(Yh[h - 1], l.HW, w.Whp[h], l.HW, P + l.obh[h], Yh[h], l.HW, m, l.HW,
                                           l.HW, beta), cxf);
        }
        // head output: ybar3, Ybar_{HL-1}
        hipLaunchKernelGGL(k_head_out_bwd, dim3(blocks(m * kRowLanes)), dim3(256), 0, st, m, Yh[l.HL - 1], (long)l.HW,
                           l.HW, P + l.o_whout, P + l.o_bhout, ga_, yb3, Ybh[l.HL - 1]);
        colsum(Yh[l.HL - 1], nullptr, yb3, l.HW, m, l.HW, 1, beta, 1.0f, cpart, GP + l.o_whout, acc, st);
        colsum(yb3, nullptr, nullptr, 1, m, 1, 0, beta, 1.0f, cpart, GP + l.o_bhout, acc, st);
        // head hidden layers, top down
        for (int h = l.HL - 1; h >= 0; --h) {
            float* Yb = Ybh[h];
            if (h > 0) {
                wgrad<PRO_RELU>(Yb, l.HW, l.HW, Yh[h - 1], l.HW, l.HW, m, part, bpart, cx);
                wg_reduce(part, ns, l.HW, l.HW, l.HW, GP + l.oWh[h], acc, st);
                hipLaunchKernelGGL(k_colsum_final, dim3(l.HW), dim3(256), 0, st, bpart, ns, l.HW, 1.0f,
                               GP + l.obh[h], acc);
                // Ybar_{h-1} = (Ybar_h Wh_h) . relu'(Y_{h-1})
                gemm<PRO_ID, EPI_RELUMASK>(ga(Yb, l.HW, w.WhT[h], l.HW, nullptr, Ybh[h - 1], l.HW, m, l.HW, l.HW, beta, Yh[h - 1], l.HW), cx);
            } else {
                wgrad<PRO_ID>(Yb, l.HW, l.HW, Ht, l.W, l.W, m, part, bpart, cx);
                wg_reduce(part, ns, l.HW, l.W, l.W, GP + l.oWh[0], acc, st);
                hipLaunchKernelGGL(k_colsum_final, dim3(l.HW), dim3(256), 0, st, bpart, ns, l.HW, 1.0f,
                               GP + l.obh[0], acc);
            }
        }
        // top of the trunk: H_bar = half g_f w_out + Ybar_0 Wh_0 and Hdot_bar =
        // half w_out, turned into the top layer's (Zbar, Zdotbar) in the
        // epilogue, which also forms the column partials of the output layer's
        // weight gradient w_out_bar = half sum_p (g_f H + Hdot) from the same
        // operands
        {
            GemmArgs a = ga(Ybh[0], l.HW, w.WhT[0], l.HW, nullptr, Zb, l.W, m, l.W, l.HW, beta, H[l.L - 1], l.W, Zdb);
            a.C2 = Hd[l.L - 1];
            a.rowv = gf;
            a.colv = P + l.o_wout;
            a.scale = half;
            a.cpart = tpart;
            if (b16) gemm_b16<PRO_ID, EPI_TOPADJ, ST_C2 | ST_Y>(a, cx);      // Zbar (Y) in BF16, Zdotbar (Y2) in FP32
            else gemm<PRO_ID, EPI_TOPADJ>(a, cx);
        }
        // sdf output layer: w_out_bar from the partials, b_out_bar = half sum g_f
        hipLaunchKernelGGL(k_colsum_final, dim3(l.W), dim3(256), 0, st, tpart,
                           (int)top_rows(m, top_tile(cx.mm, m, l.W)), l.W, 1.0f,
                           GP + l.o_wout, acc);
        if (gf) colsum(gf, nullptr, nullptr, 1, m, 1, 0, beta, half, cpart, GP + l.o_bout, acc, st);
        else if (!acc) hipLaunchKernelGGL(k_fill, dim3(1), dim3(64), 0, st, GP + l.o_bout, 1L, 0.0f);
        // trunk layers, top down: the others' (Zbar, Zdotbar) from the dual
        // adjoint GEMM of the layer above
        float *Zb_c = Zb, *Zdb_c = Zdb, *Zb_n = Hb, *Zdb_n = Hdb;
        for (int i = l.L - 1; i >= 0; --i) {
            float* Zb = Zb_c;
            // Zdot_bar_i: from the dual adjoint (plain), or half S_i kept by the
            // training forward (the top layer's from the top-adjoint epilogue)
            const bool kept = keep && i < l.L - 1;
            const float* Zdb = kept ? reserve_s(reserve, l, n, i) + c0 * l.W : Zdb_c;
            const int fin = i == 0 ? l.in0 : l.W, finp = i == 0 ? l.in0p : l.W;
            if (side) {
                // everything up to Zbar_i is enqueued on st
                if ((rc = hip_status(hipEventRecord(side->ready[i], st), "side event record")) ||
                    (rc = hip_status(hipStreamWaitEvent(wst, side->ready[i], 0), "side event wait")))
                    return rc;
            }
            const float s2 = kept ? half : 1.0f;
            if (i == 0) {
                if (b16) wgrad<PRO_ID, ST_A, 0>(Zb, l.W, l.W, X0, l.in0p, finp, m, part, bpart, cx32w, Zdb, X0d, s2);
                else wgrad<PRO_ID, 0, 0>(Zb, l.W, l.W, X0, l.in0p, finp, m, part, bpart, cx32w, Zdb, X0d, s2);
            } else {
                if (b16) wgrad<PRO_ID, ST_A, ST_B>(Zb, l.W, l.W, H[i - 1], l.W, finp, m, part, bpart, cxw, Zdb, Hd[i - 1], s2);
                else wgrad<PRO_ID, 0, 0>(Zb, l.W, l.W, H[i - 1], l.W, finp, m, part, bpart, cxw, Zdb, Hd[i - 1], s2);
                // The chain's next product overwrites Zbar_{i+1}: it waits for the product
                // that reads it (done), not for the reduction, which runs beside it
                // (that left the chip to the reduction alone for 25 of 140 us per layer
                // at 32768 points of 256 columns).
                if (side && (rc = hip_status(hipEventRecord(side->done[i], wst), "side event record"))) return rc;
            }
            wg_reduce(part, ns, l.W, finp, fin, GP + l.oW[i], acc, wst);
            hipLaunchKernelGGL(k_colsum_final, dim3(l.W), dim3(256), 0, wst, bpart, ns, l.W, 1.0f,
                               GP + l.ob[i], acc);
            if (side && i == 0 && (rc = hip_status(hipEventRecord(side->done[0], wst), "side event record"))) return rc;
            if (i > 0 && keep) {
                // the buffer this writes held Zbar_{i+1}, read by that layer's weight gradient
                if (side && i + 1 < l.L && (rc = hip_status(hipStreamWaitEvent(st, side->done[i + 1], 0),
                                                            "side event wait")))
                    return rc;
                // Zbar_{i-1} from Hbar_{i-1} = Zbar_i W_i and Hdotbar_{i-1} = half S_{i-1} / sp'(Z_{i-1})
                GemmArgs a = ga(Zb, l.W, w.WT[i], l.W, nullptr, Zb_n, l.W, m, l.W, l.W, beta, H[i - 1], l.W);
                a.C2 = Hd[i - 1];
                a.C3 = reserve_s(reserve, l, n, i - 1) + c0 * l.W;
                a.scale = half;
                if (b16) gemm_b16<PRO_ID, EPI_ADJ1, ST_A | ST_C2 | ST_Y>(a, cx);
                else gemm<PRO_ID, EPI_ADJ1>(a, cx);
                float* t = Zb_c; Zb_c = Zb_n; Zb_n = t;
            } else if (i > 0) {
                gemm_dual<EPI2_ADJ>(da(Zb, Zdb, l.W, w.WT[i], l.W, nullptr, Z[i - 1], Hd[i - 1], Zb_n, Zdb_n, nullptr,
                                       l.W, m, l.W, l.W, beta), cx.mm, st);
                float* t = Zb_c; Zb_c = Zb_n; Zb_n = t;
                t = Zdb_c; Zdb_c = Zdb_n; Zdb_n = t;
            }
        }
        // join: the next pass reuses the encoding, tangents and partials, and the
        // caller reads the gradient on st
        if (side && (rc = hip_status(hipStreamWaitEvent(st, side->done[0], 0), "side event wait"))) return rc;
        if ((rc = hip_status(hipGetLastError(), "mlp backward"))) return rc;
    }
    return RFVR_OK;
}

}  // namespace
}  // namespace rfvr

using namespace rfvr;

extern "C" {

int64_t rfvr_mlp_param_count(const rfvr_mlp* net) {
    if (check_net(net)) return -1;
    return layout(net).total;
}

size_t rfvr_mlp_forward_ws_bytes(const rfvr_mlp* net, int64_t n) {
    if (check_net(net) || n < 1 || n > RFVR_MAX_POINTS) return 0;
    return fwd_bytes(layout(net), net->precision, (long)n, false);
}

size_t rfvr_mlp_backward_ws_bytes(const rfvr_mlp* net, int64_t n) {
    if (check_net(net) || n < 1 || n > RFVR_MAX_POINTS) return 0;
    return bwd_bytes(layout(net), net->precision, (long)n, false);
}

int rfvr_mlp_forward(const rfvr_mlp* net, const float* xyz, int64_t n, float* sdf, float* grad,
                     float* refl, void* ws, size_t ws_bytes, void* stream) {
    return mlp_forward(net, xyz, (long)n, sdf, grad, refl, nullptr, 0, ws, ws_bytes,
                       reinterpret_cast<hipStream_t>(stream));
}

int rfvr_mlp_backward(const rfvr_mlp* net, const float* xyz, int64_t n, const float* g_sdf,
                      const float* g_grad, const float* g_refl, uint32_t flags, float* g_params,
                      void* ws, size_t ws_bytes, void* stream) {
    return mlp_backward(net, xyz, (long)n, g_sdf, g_grad, g_refl, flags, g_params, nullptr, 0, ws, ws_bytes,
                        reinterpret_cast<hipStream_t>(stream));
}

size_t rfvr_mlp_reserve_bytes(const rfvr_mlp* net, int64_t n) {
    if (check_net(net) || n < 1 || n > RFVR_MAX_POINTS) return 0;
    return reserve_bytes(layout(net), (long)n);
}

size_t rfvr_mlp_forward_train_ws_bytes(const rfvr_mlp* net, int64_t n) {
    if (check_net(net) || n < 1 || n > RFVR_MAX_POINTS) return 0;
    return fwd_bytes(layout(net), net->precision, (long)n, true);
}

size_t rfvr_mlp_backward_train_ws_bytes(const rfvr_mlp* net, int64_t n) {
    if (check_net(net) || n < 1 || n > RFVR_MAX_POINTS) return 0;
    return bwd_bytes(layout(net), net->precision, (long)n, true);
}

int rfvr_mlp_forward_train(const rfvr_mlp* net, const float* xyz, int64_t n, float* sdf, float* grad,
                           float* refl, void* reserve, size_t reserve_bytes_, void* ws, size_t ws_bytes,
                           void* stream) {
    if (!reserve || !reserve_bytes_) { set_error("the training forward needs a reserve"); return RFVR_E_INVALID; }
    return mlp_forward(net, xyz, (long)n, sdf, grad, refl, reserve, reserve_bytes_, ws, ws_bytes,
                       reinterpret_cast<hipStream_t>(stream));
}

int rfvr_mlp_backward_train(const rfvr_mlp* net, const float* xyz, int64_t n, const float* g_sdf,
                            const float* g_grad, const float* g_refl, uint32_t flags, float* g_params,
                            const void* reserve, size_t reserve_bytes_, void* ws, size_t ws_bytes,
                            void* stream) {
    if (!reserve || !reserve_bytes_) { set_error("the training backward needs a reserve"); return RFVR_E_INVALID; }
    return mlp_backward(net, xyz, (long)n, g_sdf, g_grad, g_refl, flags, g_params, const_cast<void*>(reserve),
                        reserve_bytes_, ws, ws_bytes, reinterpret_cast<hipStream_t>(stream));
}

}  // extern "C"

// ============================================================================
// proposal network: gamma_L -> [Linear(width) -> relu] x layers -> Linear(1)
// ============================================================================
namespace rfvr {
namespace {

struct PLayout {
    int L, W, in0, in0p, layers;
    long oW[4], ob[4], o_wout, o_bout, total;
};

int check_prop(const rfvr_proposal* n) {
    if (!n) { set_error("proposal descriptor is NULL"); return RFVR_E_INVALID; }
    if (n->width != 64 || n->layers < 1 || n->layers > 4 || n->pe_octaves < 0 || n->pe_octaves > 5) {
        set_error("unsupported proposal network (width 64, layers 1..4, pe_octaves 0..5)");
        return RFVR_E_INVALID;
    }
    if (!(n->half_size > 0.0f)) { set_error("half_size must be > 0"); return RFVR_E_INVALID; }
    return RFVR_OK;
}

PLayout playout(const rfvr_proposal* n) {
    PLayout l;
    l.L = n->pe_octaves; l.W = n->width; l.layers = n->layers;
    l.in0 = 3 + 6 * l.L;
    l.in0p = (l.in0 + 31) / 32 * 32;
    long off = 0;
    for (int i = 0; i < l.layers; ++i) {
        const int fin = i == 0 ? l.in0 : l.W;
        l.oW[i] = off; off += (long)l.W * fin;
        l.ob[i] = off; off += l.W;
    }
    l.o_wout = off; off += l.W;
    l.o_bout = off; off += 1;
    l.total = off;
    return l;
}

size_t pweights_bytes(const PLayout& l) {
    size_t b = 0;
    for (int i = 0; i < l.layers; ++i) {
        const int finp = i == 0 ? l.in0p : l.W;
        b += wmat_bytes(l.W, finp, false) + wmat_bytes(finp, l.W, true);
    }
    return b;
}

size_t pbytes(const PLayout& l, long n, bool bwd) {
    const long c = n < kChunk ? n : kChunk;
    size_t b = pweights_bytes(l) + align256(sizeof(float) * c * l.in0p) +
               (size_t)l.layers * align256(sizeof(float) * c * l.W);
    if (bwd)
        b += 2 * align256(sizeof(float) * c * l.W) + align256(sizeof(float) * kWgSplits * (size_t)l.W * l.W) +
             align256(sizeof(float) * kWgSplits * (size_t)l.W) + align256(sizeof(float) * (size_t)kColBlocks * l.W);
    return b;
}

// Abar[p][m] = g[p] w[m] relu'(A[p][m]), four columns per thread (M and ld are
// multiples of 4): bound by reading A and writing Abar (one column per thread with
// 64-bit index divisions: 262144 rows of 64 columns 39 -> 20 us)
__global__ __launch_bounds__(256) void k_relu_out_bwd(long n, int M, const float* __restrict__ A, long ld,
                                                      const float* __restrict__ w, const float* __restrict__ g,
                                                      float* __restrict__ Ab) {
    const unsigned m4 = M / 4, per = 256 / m4;            // rows per work-group
    const unsigned row = threadIdx.x / m4, m = (threadIdx.x - row * m4) * 4;
    const long p = (long)blockIdx.x * per + row;
    if (row >= per || p >= n) return;
    const float4 a = *reinterpret_cast<const float4*>(A + p * ld + m);
    const float4 wm = make_float4(w[m], w[m + 1], w[m + 2], w[m + 3]);   // parameters: any 4-byte alignment
    const float gp = g[p];
    float4 o;
    o.x = a.x > 0.0f ? gp * wm.x : 0.0f;
    o.y = a.y > 0.0f ? gp * wm.y : 0.0f;
    o.z = a.z > 0.0f ? gp * wm.z : 0.0f;
    o.w = a.w > 0.0f ? gp * wm.w : 0.0f;
    *reinterpret_cast<float4*>(Ab + p * ld + m) = o;
}

}  // namespace
}  // namespace rfvr

extern "C" {

int64_t rfvr_proposal_param_count(const rfvr_proposal* net) {
    if (check_prop(net)) return -1;
    return playout(net).total;
}

// one pass over all points, two threads per point in its matrix products
constexpr int64_t kPropMaxPoints = (int64_t)1 << 30;

size_t rfvr_proposal_ws_bytes(const rfvr_proposal* net, int64_t n) {
    if (check_prop(net) || n < 1 || n > kPropMaxPoints) return 0;
    return pbytes(playout(net), (long)n, true);
}

static int proposal_pass(const rfvr_proposal* net, const float* xyz, int64_t n, float* logits,
                         const float* g_logits, uint32_t flags, float* g_params, void* ws,
                         size_t ws_bytes, void* stream) {
    int rc;
    if ((rc = check_prop(net))) return rc;
    if (n < 1 || n > kPropMaxPoints || !xyz || !net->params) {
        set_error("n in [1, 2^30], xyz and params are required");
        return RFVR_E_INVALID;
    }
    const bool bwd = g_params != nullptr;
    if (bwd && !g_logits) { set_error("g_logits is required"); return RFVR_E_INVALID; }
    if (flags & ~(uint32_t)RFVR_ACCUMULATE) { set_error("only RFVR_ACCUMULATE is meaningful here"); return RFVR_E_INVALID; }
    const PLayout l = playout(net);
    const size_t need = pbytes(l, (long)n, bwd);
    if (!ws || ws_bytes < need || (reinterpret_cast<uintptr_t>(ws) & 255u)) {
        set_error("workspace too small or misaligned: need %zu bytes", need);
        return RFVR_E_WORKSPACE;
    }
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const Cx cx{st, MM_FP32};
    const float* P = net->params;
    const long chunk = n < kChunk ? (long)n : kChunk;
    WsCursor cur{reinterpret_cast<char*>(ws), 0};
    WMat Wp[4], WT[4];
    for (int i = 0; i < l.layers; ++i) {
        const int finp = i == 0 ? l.in0p : l.W;
        Wp[i] = take_wmat(cur, l.W, finp, false);
        WT[i] = take_wmat(cur, finp, l.W, true);
    }
    float* X0 = cur.take<float>((size_t)chunk * l.in0p);
    float* A[4];
    for (int i = 0; i < l.layers; ++i) A[i] = cur.take<float>((size_t)chunk * l.W);
    float *Ab = nullptr, *Ab2 = nullptr, *part = nullptr, *bpart = nullptr, *cpart = nullptr;
    if (bwd) {
        Ab = cur.take<float>((size_t)chunk * l.W);
        Ab2 = cur.take<float>((size_t)chunk * l.W);
        part = cur.take<float>((size_t)kWgSplits * l.W * l.W);
        bpart = cur.take<float>((size_t)kWgSplits * l.W);
        cpart = cur.take<float>((size_t)kColBlocks * l.W);
    }
    PrepList prep;
    for (int i = 0; i < l.layers; ++i) {
        const int fin = i == 0 ? l.in0 : l.W, finp = i == 0 ? l.in0p : l.W;
        prep.add(P + l.oW[i], Wp[i], l.W, fin, l.W, finp, 0);
        if (bwd && i > 0) prep.add(P + l.oW[i], WT[i], l.W, fin, finp, l.W, 1);
    }
    if ((rc = hip_status(prep.launch(st), "proposal weight prep"))) return rc;
    const float beta = 1.0f, inv_half = 1.0f / net->half_size;
    for (long c0 = 0; c0 < n; c0 += chunk) {
        const long m = (n - c0) < chunk ? (n - c0) : chunk;
        const int acc = (c0 > 0 || (flags & RFVR_ACCUMULATE)) ? 1 : 0, ns = wg_splits(m);
        encode(m, xyz + 3 * c0, net->centre, inv_half, l.L, l.in0p, X0, nullptr, nullptr, st);
        // The FP32 instruction: products over 32 or 64 k are bound by the activations
        // they write either way, and ReLU turns a last-bit change of an input near
        // zero into one of the parameter gradient (1.9e-6 relative against 9e-7).
        gemm_launch<PRO_ID, EPI_BIAS, MM_MFMA32>(ga(X0, l.in0p, Wp[0], l.in0p, P + l.ob[0], A[0], l.W, m, l.W, l.in0p, beta), st);
        for (int i = 1; i < l.layers; ++i)
            gemm_launch<PRO_RELU, EPI_BIAS, MM_MFMA32>(ga(A[i - 1], l.W, Wp[i], l.W, P + l.ob[i], A[i], l.W, m, l.W, l.W, beta), st);
        float* At = A[l.layers - 1];
        if (!bwd) {
            hipLaunchKernelGGL(k_rowdot, dim3(blocks(m * kRowLanes)), dim3(256), 0, st, m, At, (long)l.W, l.W,
                               (int)PRO_RELU, 0, P + l.o_wout, P + l.o_bout, 1.0f, beta, logits + c0);
        } else {
            const float* g = g_logits + c0;
            colsum(At, nullptr, g, l.W, m, l.W, 1, beta, 1.0f, cpart, g_params + l.o_wout, acc, st);
            colsum(g, nullptr, nullptr, 1, m, 1, 0, beta, 1.0f, cpart, g_params + l.o_bout, acc, st);
            hipLaunchKernelGGL(k_relu_out_bwd, dim3(blocks(m, 256 / (l.W / 4))), dim3(256), 0, st, m, l.W, At, (long)l.W,
                               P + l.o_wout, g, Ab);
            for (int i = l.layers - 1; i >= 0; --i) {
                const int fin = i == 0 ? l.in0 : l.W, finp = i == 0 ? l.in0p : l.W;
                if (i == 0)
                    wgrad<PRO_ID>(Ab, l.W, l.W, X0, l.in0p, finp, m, part, bpart, cx);
                else
                    wgrad<PRO_RELU>(Ab, l.W, l.W, A[i - 1], l.W, finp, m, part, bpart, cx);
                wg_reduce(part, ns, l.W, finp, fin, g_params + l.oW[i], acc, st);
                hipLaunchKernelGGL(k_colsum_final, dim3(l.W), dim3(256), 0, st, bpart, ns, l.W, 1.0f,
                               g_params + l.ob[i], acc);
                if (i > 0) {
                    gemm<PRO_ID, EPI_RELUMASK>(ga(Ab, l.W, WT[i], l.W, nullptr, Ab2, l.W, m, l.W, l.W,
                                                  beta, A[i - 1], l.W), cx);
                    float* t = Ab; Ab = Ab2; Ab2 = t;
                }
            }
        }
        if ((rc = hip_status(hipGetLastError(), "proposal network"))) return rc;
    }
    return RFVR_OK;
}

int rfvr_proposal_forward(const rfvr_proposal* net, const float* xyz, int64_t n, float* logits,
                          void* ws, size_t ws_bytes, void* stream) {
    if (!logits) { set_error("logits output is NULL"); return RFVR_E_INVALID; }
    return proposal_pass(net, xyz, n, logits, nullptr, 0, nullptr, ws, ws_bytes, stream);
}

int rfvr_proposal_backward(const rfvr_proposal* net, const float* xyz, int64_t n,
                           const float* g_logits, uint32_t flags, float* g_params,
                           void* ws, size_t ws_bytes, void* stream) {
    if (!g_params) { set_error("g_params output is NULL"); return RFVR_E_INVALID; }
    return proposal_pass(net, xyz, n, nullptr, g_logits, flags, g_params, ws, ws_bytes, stream);
}

}  // extern "C"
