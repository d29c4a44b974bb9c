// predictor.hip - gfx950 kernels and C ABI of the decode-phase reference
// predictor: a one-layer causal Transformer over a sequence's earlier
// boundary states with a bounded key-value cache (the paper's subsection
// "Predicted References for Decode", Eq. decode-predictor).  For t >= 2 it
// turns the previous reconstructed state H-hat^{t-1} of every sequence of a
// decode batch into the reference R_pred^t that the codec then encodes
// against.  The contract of each entry point is documented in include/rac.h.
//
// One step (every launch on the caller's stream; B sequences, width d, model
// width m, h heads of 64 channels, SwiGLU width f, window W):
//   h0 = x W_in^T                                     (x = H-hat^{t-1}, bf16)
//   q, k, v = RMSNorm(h0; g1) W_qkv^T, rotary positions on q and k
//   o  = softmax(q k^T / 8) v over the last min(pos + 1, W) inputs
//   h1 = h0 + o W_o^T
//   h2 = h1 + (silu(n2 W_gate^T) * (n2 W_up^T)) W_down^T,  n2 = RMSNorm(h1; g2)
//   R  = x + RMSNorm(h2; g3) W_out^T                  (bf16)
// The products are bf16 x bf16 with fp32 accumulation on the matrix cores
// (v_mfma_f32_16x16x32_bf16); the residual stream h0..h2 is fp32; the
// normalized activations, o, the SwiGLU output and the cached keys and values
// are bf16.
//
// Mapping onto CDNA4.  Decode batches are skinny (B <= 256 rows against
// weight matrices of up to 8192 x 2048), and a step is a chain of dependent
// launches of a few microseconds each.  So each product is one launch that
// sums its whole K inside a workgroup, folds in the residual, and leaves the
// sums of squares from which the next product forms its own RMSNorm: seven
// launches a step, six products and the attention (and up to three more where
// products are so large that their rows are normalized once, ahead of them).
#include <hip/hip_runtime.h>

#include <stddef.h>
#include <stdint.h>

#include <type_traits>

#include "rac.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kW = 64;           // wavefront
constexpr int kHd = 64;          // channels per head
constexpr float kEps = 1e-6f;    // RMSNorm

__device__ __forceinline__ float bf(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ uint16_t to_bf(float v) {  // round to nearest even (finite)
    const uint32_t u = __float_as_uint(v);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

// ---------------------------------------------------------------------------
// C[b][n] = sum_k A[b][k] W[n][k].  A workgroup owns a tile of 16 TM batch
// rows x 16 TN output columns (COLS TN) over the whole K, and its KW wavefronts split K
// in units of 64, so that every operand byte of the tile is loaded once, by one
// wavefront, with up to Q units in flight.
//
// The matrix core wants row l % 16 in lane l, so operands loaded straight into
// its layout put 16 rows in 16 neighbouring lanes, and the vector memory
// unit then takes a clock per 16 bytes (35 GB/s per compute unit, measured on
// 16 x 16 tiles of K = 8192).  Here neighbouring lanes load whole 128-byte
// lines of a row, and the unit passes through the wavefront's own slice of LDS
// (no barrier) to reach the layout.  A 16-byte piece (row, step of 32, quarter
// q) sits at 64 step + 4 (row ^ 2 step) + (q ^ (row / 4)) of its 2 KB block:
// the writes of 16 lanes and the reads of 16 lanes both touch every bank once.
// With the weights as the first operand lane l receives output columns
// n0 + 4 (l / 16) + r, r < 4, of batch row l % 16: one 16-byte access per lane.
//
// With no K split across workgroups the tile's epilogue sees finished sums, so
// the residual stream and its RMSNorm need no launch of their own: the product
// that forms h (kHidden) adds the residual, stores h and the sum of squares of
// every (row, COLS columns); the product that consumes it (NORM) sums those of
// its rows and forms bf16(h / sqrt(mean(h^2) + eps) * gain) on the way to LDS
// (the largest products read it from a launch of its own, see prod_wide).
enum Epi { kHidden, kQkv, kGate, kOut };

struct Prod {
    const uint16_t* a;      // bf16 [M][K] (without NORM)
    const float* h;         // fp32 [M][K] (NORM)
    const float* ssin;      // [M][nss] sums of squares of h over equal parts of a row (NORM)
    int32_t nss;            // a multiple of 4
    const uint16_t* gain;   // bf16 [K] (NORM)
    const uint16_t* w;      // bf16 [N][K]
    int32_t M, N, K;
    const float* resid;     // kHidden: fp32 [M][N] added to the product, or null
    float* out;             // kHidden, kQkv: fp32 [M][N]
    float* ssout;           // kHidden: [M][N / COLS]
    const uint16_t* resid16;// kOut: bf16 [M][N]
    uint16_t* out16;        // kGate: bf16 [M][N / 2]; kOut: bf16 [M][N]
};

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {  // two bf16, round to nearest even
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

// Orders a wavefront's LDS writes before its later reads by other lanes (LDS
// executes one wavefront's instructions in order; this keeps the compiler
// from reordering them).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// 16-byte slot of (row, step, quarter) in a block of 16 rows x 64 channels.
__device__ __forceinline__ uint32_t slot_of(uint32_t row, uint32_t step, uint32_t q) {
    return 64u * step + 4u * (row ^ (2u * step)) + (q ^ (row >> 2));
}

// One unit (64 channels) of a wavefront's operands as loaded.
template <int TM, int TN, bool NORM>
struct ProdUnit {
    u32x4 w[TN][2];                  // 8 rows x 128 bytes each
    u32x4 a[NORM ? 1 : TM][2];
    f32x4 h[NORM ? TM : 1][4];       // 4 rows x 256 bytes each
    u32x2 g;
};

// Accuracy: the matrix core rounds more than once within an instruction, so the
// error of a sum grows with the chain of instructions on one accumulator.  The
// products onto the model width, whose K reaches 8192, take a new accumulator
// for every unit, add it in fp32 to one of two sums, and add the eight
// wavefronts' sums pairwise.  The error of sums that cancel to 2^-18 of their
// terms' scale, relative to fp32 chains of 128 channels added in order: 1.14 at
// K = 2048, 1.15 at 4096 and 1.18 at 8192; with one accumulator over a
// wavefront's K 1.5, 2.0 and 2.5.  The sums cost 0.2% of a step on average.
template <int TM, int TN, int KW, int Q, int EPI, bool NORM, int COLS = 16>
__global__ __launch_bounds__(kW * KW) void pred_prod(Prod p) {
    constexpr bool kSums = EPI == kHidden;      // a new accumulator every unit, two sums
    constexpr int U = kSums && Q == 1 ? 2 : Q;  // units a round of the loop
    constexpr int WI = COLS / 8;  // eights of weight rows loaded per column tile
    constexpr int F = TM * TN, FPW = (F + KW - 1) / KW;
    constexpr int kBlk = 128;  // 16-byte slots per block of 16 rows x 64 channels
    __shared__ u32x4 stage[KW][(TM + TN) * kBlk];
    static_assert(F * kW <= (TM + TN) * kBlk, "a wavefront's sums fit in its staging slice");
    const uint32_t lane = threadIdx.x & (kW - 1);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kW));
    const int n0 = (int)blockIdx.x * (COLS * TN), m0 = (int)blockIdx.y * (16 * TM);
    const uint32_t lr = lane & 15u, lq = lane >> 4;
    u32x4* const mine = stage[w];
    const int units = p.K >> 6;
    const int u0 = units * w / KW, nu = units * (w + 1) / KW - u0;  // this wavefront's units
    const uint32_t kb = (uint32_t)u0 * 64u;
    // rows past the batch repeat the last one and are not stored; eights (with
    // NORM, fours) of rows wholly past it are not loaded at all
    auto arow = [&](int r) { return (uint32_t)(r < p.M ? r : p.M - 1); };
    uint32_t wo[TN][2], ao[TM][NORM ? 4 : 2];
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int i = 0; i < WI; ++i)
            wo[t][i] = (uint32_t)(n0 + COLS * t + 8 * i + (int)(lane >> 3)) * (uint32_t)p.K + kb + 8u * (lane & 7u);
#pragma unroll
    for (int r = 0; r < TM; ++r) {
        if constexpr (NORM) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                ao[r][i] = arow(m0 + 16 * r + 4 * i + (int)(lane >> 4)) * (uint32_t)p.K + kb + 4u * lr;
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i)
                ao[r][i] = arow(m0 + 16 * r + 8 * i + (int)(lane >> 3)) * (uint32_t)p.K + kb + 8u * (lane & 7u);
        }
    }
    ProdUnit<TM, TN, NORM> st[Q];
    auto load = [&](ProdUnit<TM, TN, NORM>& b, int u) {
        const uint32_t k = (uint32_t)u * 64u;
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int i = 0; i < WI; ++i) b.w[t][i] = *reinterpret_cast<const u32x4*>(p.w + (wo[t][i] + k));
#pragma unroll
        for (int r = 0; r < TM; ++r) {
            if constexpr (NORM) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (m0 + 16 * r + 4 * i < p.M) b.h[r][i] = *reinterpret_cast<const f32x4*>(p.h + (ao[r][i] + k));
            } else {
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (m0 + 16 * r + 8 * i < p.M) b.a[r][i] = *reinterpret_cast<const u32x4*>(p.a + (ao[r][i] + k));
            }
        }
        if constexpr (NORM) b.g = *reinterpret_cast<const u32x2*>(p.gain + (kb + k + 4u * lr));
    };
#pragma unroll
    for (int u = 0; u < Q; ++u)
        if (u < nu) load(st[u], u);
    // what the epilogue adds to this wavefront's parts of the tile
    f32x4 rs[FPW];
    uint2 rs16[FPW];
#pragma unroll
    for (int i = 0; i < FPW; ++i) {
        const int f = w + i * KW, row = m0 + 16 * (f / TN) + (int)lr, col = n0 + COLS * (f % TN) + 4 * (int)lq;
        rs[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        rs16[i] = make_uint2(0u, 0u);
        if (f < F && row < p.M && 4 * (int)lq < COLS) {
            if (EPI == kHidden && p.resid) rs[i] = *reinterpret_cast<const f32x4*>(p.resid + (size_t)row * p.N + col);
            if (EPI == kOut) rs16[i] = *reinterpret_cast<const uint2*>(p.resid16 + (size_t)row * p.N + col);
        }
    }
    float inv[TM][4];  // of the rows this lane loads
    if constexpr (NORM) {
        // lane l sums every fourth group of four of row l / 4's sums of
        // squares, then the row's four lanes add theirs
        const int nq = p.nss >> 2;
#pragma unroll
        for (int r = 0; r < TM; ++r) {
            const f32x4* q = reinterpret_cast<const f32x4*>(p.ssin) + (size_t)arow(m0 + 16 * r + (int)(lane >> 2)) * nq;
            float t = 0.0f;
            // (four loads to a wait, since a wait each is a round trip to L2:
            // a step 25.9 us with one, 25.3 with four at batch 1 (model width
            // 512), 44.0 and 41.9 at batch 16 (1024), 48.4 and 47.4 at 256 (512))
            for (int i = (int)(lane & 3u); i < nq; i += 16) {
                f32x4 v[4];
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    v[x] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                    if (i + 4 * x < nq) v[x] = q[i + 4 * x];
                }
#pragma unroll
                for (int x = 0; x < 4; ++x) t = t + ((v[x][0] + v[x][1]) + (v[x][2] + v[x][3]));
            }
            t = t + __shfl_xor(t, 1);
            t = t + __shfl_xor(t, 2);
            const float iv = 1.0f / __builtin_sqrtf(t / (float)p.K + kEps);
#pragma unroll
            for (int i = 0; i < 4; ++i) inv[r][i] = __shfl(iv, 16 * i + 4 * (int)lq);
        }
    }
    f32x4 acc[kSums ? 2 : 1][F];
#pragma unroll
    for (int f = 0; f < F; ++f) {
        acc[0][f] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (kSums) acc[1][f] = acc[0][f];
    }
    auto put = [&](const ProdUnit<TM, TN, NORM>& b) {
        const uint32_t c = lane & 7u, r8 = lane >> 3;
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int i = 0; i < WI; ++i)
                mine[t * kBlk + slot_of(8u * i + r8, c >> 2, c & 3u)] = b.w[t][i];
#pragma unroll
        for (int r = 0; r < TM; ++r) {
            if constexpr (NORM) {
                const float g0 = __uint_as_float(b.g.x << 16), g1 = __uint_as_float(b.g.x & 0xFFFF0000u);
                const float g2 = __uint_as_float(b.g.y << 16), g3 = __uint_as_float(b.g.y & 0xFFFF0000u);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (m0 + 16 * r + 4 * i >= p.M) continue;
                    const f32x4 h = b.h[r][i];
                    const float iv = inv[r][i];
                    const u32x2 o = {pack2(h[0] * iv * g0, h[1] * iv * g1), pack2(h[2] * iv * g2, h[3] * iv * g3)};
                    const uint32_t sl = slot_of(4u * i + lq, lr >> 3, (lr >> 1) & 3u);
                    reinterpret_cast<u32x2*>(mine + (TN + r) * kBlk)[2u * sl + (lr & 1u)] = o;
                }
            } else {
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (m0 + 16 * r + 8 * i < p.M) mine[(TN + r) * kBlk + slot_of(8u * i + r8, c >> 2, c & 3u)] = b.a[r][i];
            }
        }
    };
    auto product = [&](int i) {  // (unit i of a round)
        f32x4* const into = acc[kSums ? i % 2 : 0];
        f32x4 sum[kSums ? F : 1];
        if constexpr (kSums) {
#pragma unroll
            for (int f = 0; f < F; ++f) sum[f] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        wave_sync();
#pragma unroll
        for (uint32_t step = 0; step < 2u; ++step) {
            const uint32_t sl = slot_of(lr, step, lq);
            bf16x8 wv[TN], av[TM];
#pragma unroll
            for (int t = 0; t < TN; ++t) wv[t] = __builtin_bit_cast(bf16x8, mine[t * kBlk + sl]);
#pragma unroll
            for (int r = 0; r < TM; ++r) av[r] = __builtin_bit_cast(bf16x8, mine[(TN + r) * kBlk + sl]);
#pragma unroll
            for (int r = 0; r < TM; ++r)
#pragma unroll
                for (int t = 0; t < TN; ++t) {
                    f32x4& c = kSums ? sum[r * TN + t] : into[r * TN + t];
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[t], av[r], c, 0, 0, 0);
                }
        }
        wave_sync();
        if constexpr (kSums) {
#pragma unroll
            for (int f = 0; f < F; ++f) into[f] = into[f] + sum[f];
        }
    };
    int u = 0;
    for (; u + U + Q <= nu; u += U) {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            put(st[i % Q]);
            load(st[i % Q], u + Q + i);
            product(i);
        }
    }
    for (; u < nu; u += U) {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            if (u + i < nu) {
                put(st[i % Q]);
                if (u + Q + i < nu) load(st[i % Q], u + Q + i);
                product(i);
            }
        }
    }
    if constexpr (kSums) {
#pragma unroll
        for (int f = 0; f < F; ++f) acc[0][f] = acc[0][f] + acc[1][f];
    }
    // the wavefronts' sums, through each one's own slice
#pragma unroll
    for (int f = 0; f < F; ++f) reinterpret_cast<f32x4*>(mine)[f * kW + lane] = acc[0][f];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < FPW; ++i) {
        const int f = w + i * KW;
        if (f >= F) return;
        auto sum = [&](int x) { return reinterpret_cast<const f32x4*>(stage[x])[f * kW + lane]; };
        f32x4 v;
        if constexpr (KW == 8) {
            v = ((sum(0) + sum(1)) + (sum(2) + sum(3))) + ((sum(4) + sum(5)) + (sum(6) + sum(7)));
        } else {
            static_assert(KW == 4, "four or eight wavefronts");
            v = ((sum(0) + sum(1)) + sum(2)) + sum(3);
        }
        const int row = m0 + 16 * (f / TN) + (int)lr, col = n0 + COLS * (f % TN) + 4 * (int)lq;
        const bool in = row < p.M && 4 * (int)lq < COLS;
        if constexpr (EPI == kHidden) {
            v = rs[i] + v;
            float q = (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]);
            q = q + __shfl_xor(q, 16);
            if constexpr (COLS == 16) q = q + __shfl_xor(q, 32);
            if (in) {
                *reinterpret_cast<f32x4*>(p.out + (size_t)row * p.N + col) = v;
                if (lq == 0) p.ssout[(size_t)row * (p.N / COLS) + col / COLS] = q;
            }
        } else if constexpr (EPI == kQkv) {
            if (in) *reinterpret_cast<f32x4*>(p.out + (size_t)row * p.N + col) = v;
        } else if constexpr (EPI == kOut) {
            const float o0 = __uint_as_float(rs16[i].x << 16) + v[0];
            const float o1 = __uint_as_float(rs16[i].x & 0xFFFF0000u) + v[1];
            const float o2 = __uint_as_float(rs16[i].y << 16) + v[2];
            const float o3 = __uint_as_float(rs16[i].y & 0xFFFF0000u) + v[3];
            if (in)
                *reinterpret_cast<uint2*>(p.out16 + (size_t)row * p.N + col) = make_uint2(pack2(o0, o1), pack2(o2, o3));
        } else {
            // interleaved rows: column 2j is gate j, 2j + 1 is up j
            const float g0 = v[0] / (1.0f + __expf(-v[0])) * v[1];
            const float g1 = v[2] / (1.0f + __expf(-v[2])) * v[3];
            if (in) *reinterpret_cast<uint32_t*>(p.out16 + (size_t)row * (p.N / 2) + col / 2) = pack2(g0, g1);
        }
    }
}

// ---------------------------------------------------------------------------
// The normalized activations of one batch row per workgroup, as the products
// form them while loading (see prod_wide for when this launch pays for itself).
constexpr int kNormThreads = 256;

__global__ __launch_bounds__(kNormThreads) void pred_norm(Prod p, uint16_t* n) {
    const int row = blockIdx.x, t = threadIdx.x;
    const float* const h = p.h + (size_t)row * p.K;
    const float* const ss = p.ssin + (size_t)row * p.nss;
    // (channels 4 t .. 4 t + 3 and, beyond 1024, 1024 + 4 t ..)
    f32x4 hv[2];
    u32x2 gv[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int c = 4 * (t + kNormThreads * i);
        if (c < p.K) {
            hv[i] = *reinterpret_cast<const f32x4*>(h + c);
            gv[i] = *reinterpret_cast<const u32x2*>(p.gain + c);
        }
    }
    // every wavefront sums the row's sums of squares (at most 256)
    const int lane = t & (kW - 1);
    float q = 0.0f;
    for (int i = lane; i < p.nss; i += kW) q = q + ss[i];
    for (int o = 1; o < kW; o <<= 1) q = q + __shfl_xor(q, o);
    const float inv = 1.0f / __builtin_sqrtf(q / (float)p.K + kEps);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int c = 4 * (t + kNormThreads * i);
        if (c < p.K) {
            const float g0 = __uint_as_float(gv[i][0] << 16), g1 = __uint_as_float(gv[i][0] & 0xFFFF0000u);
            const float g2 = __uint_as_float(gv[i][1] << 16), g3 = __uint_as_float(gv[i][1] & 0xFFFF0000u);
            *reinterpret_cast<u32x2*>(n + (size_t)row * p.K + c) =
                u32x2{pack2(hv[i][0] * inv * g0, hv[i][1] * inv * g1), pack2(hv[i][2] * inv * g2, hv[i][3] * inv * g3)};
        }
    }
}

// ---------------------------------------------------------------------------
// Attention of one (sequence, head) per workgroup of NW wavefronts.  Lane d
// holds channel d of the head while q and k get the rotary position (pairs
// (2i, 2i + 1) turned by pos * 10000^(-2i/64): the angle formed and reduced in
// binary64, its sine and cosine in binary32); k and v go to the cache slot
// pos mod W (bf16), and the output is the softmax-weighted sum of the values
// of positions max(0, pos - W + 1) .. pos (the current one is never read back
// from memory in the same launch).
//
// What bounds a launch is its chain of waits, so everything that depends on
// the position alone is requested at once: the keys and values of the first 64
// positions, before q is turned.  Lane (t, c) = (l / 8, l % 8) takes channels
// 8c .. 8c + 7 of positions t, t + 8, ... of a pass: eight neighbouring lanes
// read a key's 128 bytes, and the score, its exponential and its product with
// the value stay in the lane (a key a lane instead, with the scores through
// LDS, measured 6.9 us at batch 256, window 64, 9.3 at batch 16 with 16 heads
// and window 256).  Every lane keeps a running maximum, starting from the
// current position's score; lanes, then wavefronts, are brought to a common
// maximum at the end.  Wavefront w takes cached positions
// 64 (w + NW i) + [0, 64), i = 0, 1, ...
struct AttnArgs {
    const float* qkv;    // [B][3m]: q | k | v
    uint16_t* cache;     // [B][W][2][m] bf16
    const int32_t* pos;  // [B]
    int32_t B, m, heads, window;
    uint16_t* o;         // [B][m] bf16
};

// 10000^(-2i/64), i < 32.  (In constant memory: as a kernel argument indexed by
// lane it was a load from the argument segment.)
__constant__ const double kTheta[kHd / 2] = {
    1.0, 0.7498942093324559, 0.5623413251903491, 0.4216965034285822,
    0.31622776601683794, 0.23713737056616552, 0.1778279410038923, 0.1333521432163324,
    0.1, 0.07498942093324558, 0.05623413251903491, 0.042169650342858224,
    0.03162277660168379, 0.023713737056616554, 0.01778279410038923, 0.01333521432163324,
    0.01, 0.007498942093324558, 0.005623413251903491, 0.004216965034285823,
    0.0031622776601683794, 0.0023713737056616554, 0.0017782794100389228, 0.001333521432163324,
    0.001, 0.0007498942093324559, 0.0005623413251903491, 0.00042169650342858224,
    0.00031622776601683794, 0.00023713737056616554, 0.00017782794100389227, 0.0001333521432163324};

__device__ __forceinline__ void widen8(const u32x4& v, float* f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = __uint_as_float(v[i] << 16);
        f[2 * i + 1] = __uint_as_float(v[i] & 0xFFFF0000u);
    }
}

// Sum over the eight lanes of an aligned block, the same in all of them.
__device__ __forceinline__ float sum8(float v) {
    auto dpp = [](float x, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value,
                                                                     0xF, 0xF, false));
    };
    v = v + dpp(v, std::integral_constant<int, 0xB1>{});   // quad_perm [1,0,3,2]
    v = v + dpp(v, std::integral_constant<int, 0x4E>{});   // quad_perm [2,3,0,1]
    return v + dpp(v, std::integral_constant<int, 0x141>{});  // row_half_mirror
}

template <int NW>
__global__ __launch_bounds__(kW * NW) void pred_attn(AttnArgs a) {
    __shared__ alignas(16) float turned[NW][3][kHd];  // q, and k and v as cached
    __shared__ float wmax[NW], wden[NW];
    __shared__ alignas(16) float wout[NW][kHd];
    const int b = (int)blockIdx.x / a.heads, hh = (int)blockIdx.x % a.heads;
    const int d = threadIdx.x & (kW - 1), w = (int)(threadIdx.x / kW);
    using cptr = const __attribute__((address_space(4))) int32_t*;  // read-only in this launch: a scalar load
    const int32_t pv = ((cptr)a.pos)[b];
    const float* row = a.qkv + (size_t)b * 3 * a.m + hh * kHd;
    float q = row[d], k = row[a.m + d];
    const float v = row[2 * a.m + d];
    const double theta = kTheta[d >> 1];
    const int p = pv < 0 ? 0 : pv;
    const int W = a.window, slot = p % W;
    const int n = p < W ? p : W - 1;  // cached positions attended, besides the current one
    const uint32_t rowk = 2u * (uint32_t)a.m;  // cache elements per (sequence, slot)
    uint16_t* const base = a.cache + (size_t)b * W * rowk + hh * kHd;
    const int t = d >> 3, c = d & 7;
    u32x4 kv[8], vv[8];
    // keys and values of positions j0 + t + 8 u (position j of the n is j + 1
    // .. n slots back: 0 the oldest)
    auto load = [&](int j0) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int j = j0 + t + 8 * u;
            kv[u] = vv[u] = u32x4{0u, 0u, 0u, 0u};
            if (j < n) {
                int s = slot - n + j;
                s = s < 0 ? s + W : s;
                const uint16_t* r = base + (size_t)s * rowk + 8 * c;
                kv[u] = *reinterpret_cast<const u32x4*>(r);
                vv[u] = *reinterpret_cast<const u32x4*>(r + a.m);
            }
        }
    };
    load(kW * w);
    {
        // the angle pos * theta_i in binary64, reduced to [-pi, pi] there (the
        // product k * 2 pi is exact to far below a binary32 ulp for any int32
        // position), then a binary32 sincos
        const double th = (double)p * theta;
        const double kTwoPi = 6.283185307179586476925;
        const float r = (float)(th - kTwoPi * rint(th / kTwoPi));
        float sn, cs;
        sincosf(r, &sn, &cs);
        const float qo = __shfl_xor(q, 1), ko = __shfl_xor(k, 1);
        // (a, b) -> (a cos - b sin, a sin + b cos): the even lane holds a
        q = (d & 1) ? qo * sn + q * cs : q * cs - qo * sn;
        k = (d & 1) ? ko * sn + k * cs : k * cs - ko * sn;
    }
    const uint16_t kb = to_bf(k), vb = to_bf(v);
    if (w == 0) {
        uint16_t* const cur = base + (size_t)slot * rowk;
        cur[d] = kb;
        cur[a.m + d] = vb;
    }
    // (each wavefront through its own copy: no barrier)
    turned[w][0][d] = q;
    turned[w][1][d] = bf(kb);
    turned[w][2][d] = bf(vb);
    wave_sync();
    float qf[8], acc[8];
    float mx = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        qf[i] = turned[w][0][8 * c + i];
        mx = mx + qf[i] * turned[w][1][8 * c + i];
        acc[i] = turned[w][2][8 * c + i];
    }
    // the current position is the first term of lanes (0, c) of wavefront 0
    const bool first = w == 0 && t == 0;
    mx = sum8(mx) * 0.125f;  // 1 / sqrt(64)
    float den = first ? 1.0f : 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = first ? acc[i] : 0.0f;
    for (int j0 = kW * w; j0 < n; j0 += kW * NW) {
        if (j0 != kW * w) load(j0);
        float sc[8];
        float m = mx;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            float f[8];
            widen8(kv[u], f);
            float s = 0.0f;
#pragma unroll
            for (int i = 0; i < 8; ++i) s = s + qf[i] * f[i];
            s = sum8(s) * 0.125f;
            sc[u] = j0 + t + 8 * u < n ? s : -INFINITY;
            m = __builtin_fmaxf(m, sc[u]);
        }
        const float keep = __expf(mx - m);
        mx = m;
        den = den * keep;
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = acc[i] * keep;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float e = __expf(sc[u] - m);
            den = den + e;
            float f[8];
            widen8(vv[u], f);
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] = acc[i] + e * f[i];
        }
    }
    // the eight lanes of every channel block, then the wavefronts
    float m = mx;
    for (int o = 8; o < kW; o <<= 1) m = __builtin_fmaxf(m, __shfl_xor(m, o));
    if constexpr (NW > 1) {
        if (d == 0) wmax[w] = m;
        __syncthreads();
#pragma unroll
        for (int x = 0; x < NW; ++x) m = __builtin_fmaxf(m, wmax[x]);
    }
    const float keep = __expf(mx - m);
    den = den * keep;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = acc[i] * keep;
    for (int o = 8; o < kW; o <<= 1) {
        den = den + __shfl_xor(den, o);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = acc[i] + __shfl_xor(acc[i], o);
    }
    if constexpr (NW > 1) {
        if (d == 0) wden[w] = den;
        if (t == 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) wout[w][8 * c + i] = acc[i];
        }
        __syncthreads();
        if (w != 0) return;
        den = wden[0];
#pragma unroll
        for (int x = 1; x < NW; ++x) den = den + wden[x];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            acc[i] = wout[0][8 * c + i];
#pragma unroll
            for (int x = 1; x < NW; ++x) acc[i] = acc[i] + wout[x][8 * c + i];
        }
    }
    if (t == 0) {
        u32x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = pack2(acc[2 * i] / den, acc[2 * i + 1] / den);
        *reinterpret_cast<u32x4*>(a.o + (size_t)b * a.m + hh * kHd + 8 * c) = o;
    }
}

// ---------------------------------------------------------------------------
// Host side

struct PLayout {
    uint64_t w_in, g1, w_qkv, w_o, g2, w_gu, w_down, g3, w_out, total;  // bytes
};

uint64_t up256(uint64_t v) { return (v + 255u) & ~uint64_t(255); }

bool pcfg_valid(const rac_predictor_config* c) {
    // (every K is a whole number of the products' 64-wide units, every N of
    // their widest tile of 64 columns)
    return c && c->hidden >= 512 && c->hidden <= 8192 && c->hidden % 512 == 0 && c->model >= 128 &&
           c->model <= 2048 && c->model % 128 == 0 && c->heads >= 1 && c->heads * kHd == c->model &&
           c->ffn >= 128 && c->ffn <= 8192 && c->ffn % 128 == 0 && c->window >= 1 && c->window <= 1024 &&
           c->max_batch >= 1 && c->max_batch <= 256;
}

PLayout playout(const rac_predictor_config* c) {
    const uint64_t d = c->hidden, m = c->model, f = c->ffn;
    PLayout L;
    uint64_t o = 0;
    auto take = [&](uint64_t elems) { const uint64_t at = o; o = up256(o + elems * 2u); return at; };
    L.w_in = take(m * d);
    L.g1 = take(m);
    L.w_qkv = take(3 * m * m);
    L.w_o = take(m * m);
    L.g2 = take(m);
    L.w_gu = take(2 * f * m);
    L.w_down = take(m * f);
    L.g3 = take(m);
    L.w_out = take(d * m);
    L.total = o;
    return L;
}

// The total is part of the interface (callers size the scratch by it, and a
// smaller one is refused), so it stays what it was when the products left
// partial sums in memory, where `ss` now is.
struct PWork {
    uint64_t ss, h0, h1, h2, n, qkv, o, gg, total;
};

PWork pwork(const rac_predictor_config* c, int B) {
    const uint64_t m = c->model, f = c->ffn;
    PWork W;
    uint64_t o = 0;
    auto take = [&](uint64_t bytes) { const uint64_t at = o; o = up256(o + bytes); return at; };
    const uint64_t S = c->ffn % 512 == 0 && c->ffn > c->hidden ? f / 512 : (uint64_t)c->hidden / 512;
    W.ss = take(S * B * m * 4);  // [B][m / 8] used at most
    W.h0 = take((uint64_t)B * m * 4);
    W.h1 = take((uint64_t)B * m * 4);
    W.h2 = take((uint64_t)B * m * 4);
    W.n = take((uint64_t)B * m * 2);
    W.qkv = take((uint64_t)B * 3 * m * 4);
    W.o = take((uint64_t)B * m * 2);
    W.gg = take((uint64_t)B * f * 2);
    W.total = o;
    return W;
}

template <int TM, int TN, int KW, int Q, int EPI, bool NORM, int COLS = 16>
rac_status prod_launch(const Prod& p, hipStream_t st) {
    Prod a = p;
    void* args[] = {&a};
    const dim3 grid((unsigned)(p.N / (COLS * TN)), (unsigned)((p.M + 16 * TM - 1) / (16 * TM)), 1u);
    return hipLaunchKernel(reinterpret_cast<const void*>(pred_prod<TM, TN, KW, Q, EPI, NORM, COLS>), grid, dim3(kW * KW),
                           args, 0, st) == hipSuccess
               ? RAC_OK
               : RAC_ERR_HIP;
}

// The tile of a product: the largest of a few whose workgroups still fill the
// chip's 256 compute units (three quarters of them), since a larger tile loads
// fewer bytes per output and a smaller one leaves no unit idle.  Measured one
// product at a time, us, (TM, TN): 16 x 4096 of K = 512: (1, 1) 3.4, (1, 2)
// 3.6; 64 x 4096 of 512: (1, 4) 4.5, (1, 1) 5.2, (2, 4) 5.6; 256 x 4096 of 512:
// (2, 4) 7.9, (4, 4) 9.0, (1, 4) 10.0; 256 x 1024 of 4096: (2, 2) 8.9, (1, 2)
// 11.2, (1, 1) 15; 256 x 512 of 4096: (1, 2) 6.9, (1, 1) 8.4, (2, 2) 8.8.
constexpr int64_t kFill = 192;

int64_t tiles(const Prod& p, int tm, int tn) {
    return (int64_t)((p.M + 16 * tm - 1) / (16 * tm)) * (p.N / (16 * tn));
}

// Products onto the model width (few columns, long K).  Up to 128 of the
// smallest tiles leave half the chip idle: then eight columns a workgroup
// (half of the matrix core's tile unused) on twice the workgroups.  us, 16
// columns and 8: 1 x 512 of K = 4096: 4.6, 4.0; 64 x 512 of 4096 (128 tiles):
// 5.3, 4.9; 128 x 512 of 4096 (256 tiles): 5.5, 7.1.  (2, 4) against (2, 2):
// 143 x 2048 of 8192 (160 tiles) 20.6, 25.4; 256 x 1536 of 3072 9.8, 13.4; 143 x
// 1536 of 3072 (120 tiles) 9.7, 7.8.
rac_status prod_hidden(Prod& p, hipStream_t st) {
    p.nss = p.N / 16;
    if (tiles(p, 1, 1) <= 128) {
        p.nss = p.N / 8;
        return prod_launch<1, 1, 8, 2, kHidden, false, 8>(p, st);
    }
    if (p.M > 16 && tiles(p, 2, 4) >= 160) return prod_launch<2, 4, 8, 1, kHidden, false>(p, st);
    if (p.M > 16 && tiles(p, 2, 2) >= kFill) return prod_launch<2, 2, 8, 2, kHidden, false>(p, st);
    if (tiles(p, 1, 2) >= kFill) return prod_launch<1, 2, 8, 2, kHidden, false>(p, st);
    return prod_launch<1, 1, 8, 2, kHidden, false>(p, st);
}

// Products from the normalized model width (many columns, short K).  A tile
// that normalizes its own rows reads them in fp32 and converts them once per
// column tile; from 9e8 multiply-adds on a launch that writes them as bf16
// first (3 us) saves more than it costs.  us, normalizing and reading bf16:
// 64 x 4096 of K = 512 4.6, 3.5; 256 x 4096 of 512 (5e8) 7.9, 5.6; 64 x 8192 of
// 1024 (5e8) 8.6, 5.6; 256 x 3072 of 1024 (8e8) 10.6, 7.3; 256 x 8192 of 1024
// 21.9, 11.9; 256 x 16384 of 2048 79, 41.
// With bf16 rows the (4, 4) tile is faster where the batch fills its 64 rows
// or K is long: 256 x 8192 of 1024 11.9, (2, 4) 13.4; 96 x 9216 of 1536 12.9,
// 10.3; 143 x 16384 of 2048 30, 39.
template <int EPI>
rac_status prod_wide(const Prod& p, uint16_t* n, hipStream_t st) {
    if ((int64_t)p.M * p.N * p.K >= 900000000) {
        Prod b = p;
        void* args[] = {&b, &n};
        if (hipLaunchKernel(reinterpret_cast<const void*>(pred_norm), dim3((unsigned)p.M), dim3(kNormThreads), args, 0,
                            st) != hipSuccess)
            return RAC_ERR_HIP;
        b.a = n;
        const int pad = (p.M + 63) / 64 * 64;
        if (p.K >= 2048 || 4 * pad <= 5 * p.M) return prod_launch<4, 4, 4, 1, EPI, false>(b, st);
        return prod_launch<2, 4, 4, 1, EPI, false>(b, st);
    }
    if (p.M > 16 && tiles(p, 2, 4) >= kFill) return prod_launch<2, 4, 4, 1, EPI, true>(p, st);
    if (tiles(p, 1, 4) >= kFill) return prod_launch<1, 4, 4, 2, EPI, true>(p, st);
    if (tiles(p, 1, 2) >= kFill) return prod_launch<1, 2, 4, 2, EPI, true>(p, st);
    return prod_launch<1, 1, 4, 2, EPI, true>(p, st);
}

template <int NW>
rac_status attention_launch(const AttnArgs& args, hipStream_t st) {
    AttnArgs a = args;
    void* p[] = {&a};
    return hipLaunchKernel(reinterpret_cast<const void*>(pred_attn<NW>), dim3((unsigned)(a.B * a.heads)),
                           dim3(kW * NW), p, 0, st) == hipSuccess
               ? RAC_OK
               : RAC_ERR_HIP;
}

// As many wavefronts as the window has passes of 64 positions, up to four.
rac_status attention(const rac_predictor_config* cfg, const float* qkv, void* cache, const int32_t* pos, int B,
                     uint16_t* o, hipStream_t st) {
    const AttnArgs a{qkv, static_cast<uint16_t*>(cache), pos, B, cfg->model, cfg->heads, cfg->window, o};
    if (cfg->window <= kW + 1) return attention_launch<1>(a, st);
    if (cfg->window <= 2 * kW + 1) return attention_launch<2>(a, st);
    return attention_launch<4>(a, st);
}

bool al(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

}  // namespace

extern "C" {

rac_status rac_predictor_layout(const rac_predictor_config* cfg, rac_predictor_offsets* out) {
    if (!pcfg_valid(cfg) || !out) return RAC_ERR_INVALID;
    const PLayout L = playout(cfg);
    out->w_in = L.w_in;
    out->g1 = L.g1;
    out->w_qkv = L.w_qkv;
    out->w_o = L.w_o;
    out->g2 = L.g2;
    out->w_gu = L.w_gu;
    out->w_down = L.w_down;
    out->g3 = L.g3;
    out->w_out = L.w_out;
    out->total = L.total;
    return RAC_OK;
}

size_t rac_predictor_cache_bytes(const rac_predictor_config* cfg) {
    if (!pcfg_valid(cfg)) return 0;
    return (size_t)cfg->max_batch * (size_t)cfg->window * 2u * (size_t)cfg->model * 2u;
}

size_t rac_predictor_workspace_bytes(const rac_predictor_config* cfg) {
    if (!pcfg_valid(cfg)) return 0;
    return (size_t)pwork(cfg, cfg->max_batch).total;
}

rac_status rac_predictor_step(const rac_predictor_config* cfg, const void* weights, void* cache, const int32_t* pos,
                              int32_t batch, const void* h_prev, void* ref_out, void* workspace,
                              size_t workspace_bytes, rac_stream_t stream) {
    if (!pcfg_valid(cfg) || batch < 0 || batch > cfg->max_batch) return RAC_ERR_INVALID;
    if (batch == 0) return RAC_OK;
    if (!weights || !cache || !pos || !h_prev || !ref_out || !workspace) return RAC_ERR_INVALID;
    if (!al(weights, 256) || !al(cache, 16) || !al(pos, 4) || !al(h_prev, 16) || !al(ref_out, 16) ||
        !al(workspace, 256))
        return RAC_ERR_ALIGN;
    const PWork W = pwork(cfg, cfg->max_batch);
    if (workspace_bytes < W.total) return RAC_ERR_CAPACITY;
    const PWork Wb = pwork(cfg, batch);  // (layout for this batch; fits in the max-batch one)
    const PLayout L = playout(cfg);
    const int B = batch, d = cfg->hidden, m = cfg->model, f = cfg->ffn;
    const uint8_t* wb = static_cast<const uint8_t*>(weights);
    auto wt = [&](uint64_t off) { return reinterpret_cast<const uint16_t*>(wb + off); };
    uint8_t* ws = static_cast<uint8_t*>(workspace);
    float* ss = reinterpret_cast<float*>(ws + Wb.ss);  // sums of squares of the residual stream, [B][m / 16 or m / 8]
    float* h0 = reinterpret_cast<float*>(ws + Wb.h0);
    float* h1 = reinterpret_cast<float*>(ws + Wb.h1);
    float* h2 = reinterpret_cast<float*>(ws + Wb.h2);
    float* qkv = reinterpret_cast<float*>(ws + Wb.qkv);
    uint16_t* n = reinterpret_cast<uint16_t*>(ws + Wb.n);
    uint16_t* o = reinterpret_cast<uint16_t*>(ws + Wb.o);
    uint16_t* gg = reinterpret_cast<uint16_t*>(ws + Wb.gg);
    const uint16_t* x = static_cast<const uint16_t*>(h_prev);
    hipStream_t st = stream;
    rac_status s;
    Prod p{};
    p.M = B;
    // h0 = x W_in^T
    p.a = x; p.w = wt(L.w_in); p.N = m; p.K = d; p.out = h0; p.ssout = ss;
    if ((s = prod_hidden(p, st)) != RAC_OK) return s;
    // q, k, v; attention over the window
    p.h = h0; p.ssin = ss; p.gain = wt(L.g1); p.w = wt(L.w_qkv); p.N = 3 * m; p.K = m; p.out = qkv;
    if ((s = prod_wide<kQkv>(p, n, st)) != RAC_OK) return s;
    if ((s = attention(cfg, qkv, cache, pos, B, o, st)) != RAC_OK) return s;
    // h1 = h0 + o W_o^T
    p.a = o; p.w = wt(L.w_o); p.N = m; p.K = m; p.resid = h0; p.out = h1;
    if ((s = prod_hidden(p, st)) != RAC_OK) return s;
    // SwiGLU; h2 = h1 + g W_down^T
    p.h = h1; p.gain = wt(L.g2); p.w = wt(L.w_gu); p.N = 2 * f; p.K = m; p.out16 = gg;
    if ((s = prod_wide<kGate>(p, n, st)) != RAC_OK) return s;
    p.a = gg; p.w = wt(L.w_down); p.N = m; p.K = f; p.resid = h1; p.out = h2;
    if ((s = prod_hidden(p, st)) != RAC_OK) return s;
    // R = x + n3 W_out^T (bf16)
    p.h = h2; p.gain = wt(L.g3); p.w = wt(L.w_out); p.N = d; p.K = m; p.resid16 = x;
    p.out16 = static_cast<uint16_t*>(ref_out);
    return prod_wide<kOut>(p, n, st);
}

}  // extern "C"
