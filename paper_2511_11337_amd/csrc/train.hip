// On-device training of the byte-level Mamba predictor: cross-entropy of the
// next byte (paper, Theoretical Framework: the per-step loss whose sum is the
// code length), forward over whole sequences with the activations the
// backward needs, a hand-written reverse pass for every stage and AdamW.
//
// The in-time dependence sits in the causal conv and the selective scan
// (Appendix A: with input-dependent Delta, B, C the recurrence is evaluated by
// a scan during training).  The scan forward keeps h every few steps; the
// backward recomputes h in between and runs the reverse
// recurrence  gh_t = C_t gy_t + exp(Delta_{t+1} A) gh_{t+1}.
//
// Every projection and its input gradient run on k_trow, the weight gradients
// on k_tg_w (k_tg stays for feed-forward widths that k_trow is not built
// for): FP32 operands on v_mfma_f32_16x16x4_f32, or BF16 operands
// (activations, gradients and the weights rounded to bf16 as they are staged)
// on v_mfma_f32_16x16x32_bf16, both accumulating in FP32; the master weights,
// the optimiser and every elementwise step stay FP32.
//
// Training is deterministic: no sum depends on the order in which workgroups
// or waves run.  Sums over rows
// (weight gradients, bias and LayerNorm gradients, the embedding gradient,
// the conv weights) are taken per fixed slice of rows into a partial buffer
// and the slices are then added in increasing order; sums over channel blocks
// or sequences (the scan's dB, dC, dA, dD) are kept per block and added in
// block order; the loss and the gradient norm are summed by fixed trees.
// Two runs from the same weights and data give identical bits.
#include "boa_internal.h"
#include "device_common.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

namespace boa {
namespace {

// ============================================================ GEMM
// C (+)= A . B with A(m, k) = A[m sam + k sak] and B(k, n) = B[k sbk + n sbn]
// (row-major operands used as they are or transposed, by their strides).
// A workgroup of 4 waves owns a 64 x 64 tile of C; each wave a 32 x 32 block
// of 2 x 2 MFMA tiles.  The reduction runs over k in tiles of 32 staged in
// LDS (k-contiguous rows, the MFMA operand order), with the next tile's
// global loads in registers while the current one is multiplied.  AK (BK_)
// selects the thread-to-element map of the global loads: along k when the
// operand is contiguous in k, else along m (n), so that loads coalesce either
// way.  Split reductions (gridDim.z > 1) cover k in [z kspan, (z+1) kspan)
// and write their own partial C + z cstride; the partials are added in z
// order by k_sum_slices.  Within a split the accumulation order over k is
// fixed: increasing, in steps of 4 (FP32) or 32 (BF16).
constexpr int TG_BM = 64, TG_BN = 64, TG_BK = 32;

template <int DT, bool AK, bool BK_>
__global__ __launch_bounds__(256) void k_tg(const float* __restrict__ A, long long sam, long long sak,
                                            const float* __restrict__ B, long long sbk, long long sbn, int M, int N,
                                            long long K, long long kspan, float* __restrict__ C, long long ldc,
                                            long long cstride, int accumulate) {
    using ET = typename std::conditional<DT == 0, float, uint16_t>::type;
    constexpr int RS = DT == 0 ? TG_BK + 4 : TG_BK + 8;      // LDS row stride (elements)
    __shared__ __align__(16) ET As[TG_BM * RS];
    __shared__ __align__(16) ET Bs[TG_BN * RS];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int wm = wv >> 1, wn = wv & 1;
    const int m0 = blockIdx.y * TG_BM, n0 = blockIdx.x * TG_BN;
    const long long kb = (long long)blockIdx.z * kspan;
    const long long ke = K < kb + kspan ? K : kb + kspan;
    // element map of one thread: 8 elements of a 64 x 32 tile
    const int ar = AK ? tid >> 2 : (tid & 7) * 8, ak = AK ? (tid & 3) * 8 : tid >> 3;
    const int br = BK_ ? tid >> 2 : (tid & 7) * 8, bk = BK_ ? (tid & 3) * 8 : tid >> 3;
    float ra[8], rb[8];
    auto load = [&](long long k0) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int m = m0 + ar + (AK ? 0 : j);
            const long long k = k0 + ak + (AK ? j : 0);
            ra[j] = (m < M && k < ke) ? A[(long long)m * sam + k * sak] : 0.0f;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int n = n0 + br + (BK_ ? 0 : j);
            const long long k = k0 + bk + (BK_ ? j : 0);
            rb[j] = (n < N && k < ke) ? B[k * sbk + (long long)n * sbn] : 0.0f;
        }
    };
    auto put = [&](ET* S, int r, int k, const float (&v)[8], bool along_k) {
        if (DT == 0) {
            float* F = reinterpret_cast<float*>(S);
            if (along_k) {
                *reinterpret_cast<float4*>(F + r * RS + k) = make_float4(v[0], v[1], v[2], v[3]);
                *reinterpret_cast<float4*>(F + r * RS + k + 4) = make_float4(v[4], v[5], v[6], v[7]);
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) F[(r + j) * RS + k] = v[j];
            }
        } else {
            uint16_t* H = reinterpret_cast<uint16_t*>(S);
            if (along_k) {
                uint4 u;
                u.x = (uint32_t)f2bf_bits(v[0]) | ((uint32_t)f2bf_bits(v[1]) << 16);
                u.y = (uint32_t)f2bf_bits(v[2]) | ((uint32_t)f2bf_bits(v[3]) << 16);
                u.z = (uint32_t)f2bf_bits(v[4]) | ((uint32_t)f2bf_bits(v[5]) << 16);
                u.w = (uint32_t)f2bf_bits(v[6]) | ((uint32_t)f2bf_bits(v[7]) << 16);
                *reinterpret_cast<uint4*>(H + r * RS + k) = u;
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) H[(r + j) * RS + k] = f2bf_bits(v[j]);
            }
        }
    };
    v4f acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    const int li = lane & 15, lk = lane >> 4;
    if (kb < ke) load(kb);
    for (long long k0 = kb; k0 < ke; k0 += TG_BK) {
        put(As, ar, ak, ra, AK);
        put(Bs, br, bk, rb, BK_);
        __syncthreads();
        if (k0 + TG_BK < ke) load(k0 + TG_BK);
        if (DT == 0) {
            const float* Af = reinterpret_cast<const float*>(As);
            const float* Bf = reinterpret_cast<const float*>(Bs);
#pragma unroll
            for (int ks = 0; ks < TG_BK; ks += 4) {
                float af[2], bf[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) af[i] = Af[(wm * 32 + i * 16 + li) * RS + ks + lk];
#pragma unroll
                for (int j = 0; j < 2; ++j) bf[j] = Bf[(wn * 32 + j * 16 + li) * RS + ks + lk];
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[i], bf[j], acc[i][j], 0, 0, 0);
            }
        } else {
            const uint16_t* Ah = reinterpret_cast<const uint16_t*>(As);
            const uint16_t* Bh = reinterpret_cast<const uint16_t*>(Bs);
            v8bf af[2], bf[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) af[i] = *reinterpret_cast<const v8bf*>(Ah + (wm * 32 + i * 16 + li) * RS + 8 * lk);
#pragma unroll
            for (int j = 0; j < 2; ++j) bf[j] = *reinterpret_cast<const v8bf*>(Bh + (wn * 32 + j * 16 + li) * RS + 8 * lk);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bf[j], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
    }
    // lane holds rows 4 lk + r, column li of each 16 x 16 tile
    float* Cz = C + (long long)blockIdx.z * cstride;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + wm * 32 + i * 16 + 4 * lk + r;
                const int n = n0 + wn * 32 + j * 16 + li;
                if (m < M && n < N) {
                    float* d = Cz + (long long)m * ldc + n;
                    const float v = acc[i][j][r];
                    *d = accumulate ? *d + v : v;
                }
            }
}

// ============================================================ row GEMM on prepared weights
// C = epi(A . W^T) for many rows of A [M][lda] and a weight matrix prepared in
// MFMA fragment order by k_tr_frags (rows padded to 64, columns to KP, both
// with zeros): a workgroup of 4 waves stages BM rows of A in LDS once, rounded
// to the operand type, and wave w computes the column fragments of its groups
// of FN, reading them straight into registers with one step of prefetch.  Per
// output the MFMA sequence is k_tg's (k increasing in steps of 4 / 32 from
// zero).  Bound by HBM: A is read once and C written once (k_tg's 64 x 64
// tiles of scalar loads took 1.47 ms per product of 262112 rows on average at
// d_model 256, this one 0.37 ms, from 0.15 for the x_proj to 0.70 with the
// gate's backward).  BM is 64 (32 for KP >= 512, the LDS of two workgroups
// per CU), or 16 when fewer than 256 workgroups would run.
// Epilogues: 0 store; 1 C = Cin + v (Cin may be C); 2 v += bias, C = v,
// C2 = softplus(v); 3 the gate's backward: v = d gate, C = v silu(z),
// C2 = v y silu'(z).
struct TRow {
    const float* A;
    long long lda;
    int M, K, N;
    const void* W;
    float* C;
    long long ldc;
    int epi;
    const float* Cin;                 // 1: [M][ldc]
    int span;                         // > 0: the reduction is taken in spans of `span` MFMA steps, added in order
    const float* bias;                // 2: [N]
    float* C2;                        // 2: [M][ldc]; 3: [M][ldc2]
    const float* y;                   // 3: [M][ldc]
    const float* z;                   // 3: [M][ldc2]
    long long ldc2;
};
DEVI float dsilu_f(float v) {
    float s = 1.0f / (1.0f + expf(-v));
    return s * (1.0f + v * (1.0f - s));
}

template <int DT, int EPI, int KP, int BM, int FN>
__global__ __launch_bounds__(256, 2) void k_trow(TRow p) {
    constexpr int FM = BM / 16;
    constexpr bool SPLIT = DT == 1 && BM == 16;                // spans occur with few rows only
    constexpr int AS = DT == 0 ? KP + 4 : KP + 8;              // LDS row stride (elements)
    using ET = typename std::conditional<DT == 0, float, uint16_t>::type;
    extern __shared__ __align__(16) unsigned char smem[];
    ET* As = reinterpret_cast<ET*>(smem);
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = blockIdx.x * BM;
#pragma unroll 8
    for (int it = tid; it < BM * KP / 4; it += 256) {
        const int r = it / (KP / 4), k = it % (KP / 4) * 4;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (m0 + r < p.M && k < p.K) v = *reinterpret_cast<const float4*>(p.A + (m0 + r) * p.lda + k);
        if constexpr (DT == 0) {
            *reinterpret_cast<float4*>(As + r * AS + k) = v;
        } else {
            uint2 u;
            u.x = (uint32_t)f2bf_bits(v.x) | ((uint32_t)f2bf_bits(v.y) << 16);
            u.y = (uint32_t)f2bf_bits(v.z) | ((uint32_t)f2bf_bits(v.w) << 16);
            *reinterpret_cast<uint2*>(As + r * AS + k) = u;
        }
    }
    __syncthreads();
    const int li = lane & 15, lk = lane >> 4;
    const int NF = (p.N + 63) / 64 * 4;
    for (int nf0 = wv * FN; nf0 < NF; nf0 += 4 * FN) {
        v4f acc[FM][FN];
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
        v4f tot[SPLIT ? FM : 1][SPLIT ? FN : 1];
        int left = p.span;
        constexpr int S = DT == 0 ? KP / 16 : KP / 32;          // 16-byte loads per fragment and lane
        const uint4* W4 = reinterpret_cast<const uint4*>(p.W) + (long long)nf0 * S * 64 + lane;
        uint4 bc[FN], bn[FN];
#pragma unroll
        for (int j = 0; j < FN; ++j) bc[j] = W4[(long long)j * S * 64];
#pragma unroll 1
        for (int s = 0; s < S; ++s) {
            if (s + 1 < S) {
#pragma unroll
                for (int j = 0; j < FN; ++j) bn[j] = W4[((long long)j * S + s + 1) * 64];
            }
            if constexpr (DT == 0) {
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    float af[FM];
#pragma unroll
                    for (int i = 0; i < FM; ++i) af[i] = As[(i * 16 + li) * AS + 16 * s + 4 * jj + lk];
#pragma unroll
                    for (int j = 0; j < FN; ++j) {
                        const float b = __uint_as_float(jj == 0 ? bc[j].x : jj == 1 ? bc[j].y : jj == 2 ? bc[j].z : bc[j].w);
#pragma unroll
                        for (int i = 0; i < FM; ++i)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[i], b, acc[i][j], 0, 0, 0);
                    }
                }
            } else {
                v8bf af[FM];
#pragma unroll
                for (int i = 0; i < FM; ++i) af[i] = *reinterpret_cast<const v8bf*>(As + (i * 16 + li) * AS + 32 * s + 8 * lk);
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int i = 0; i < FM; ++i)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], *reinterpret_cast<const v8bf*>(&bc[j]),
                                                                            acc[i][j], 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < FN; ++j) bc[j] = bn[j];
            if (SPLIT && p.span > 0 && --left == 0 && s + 1 < S) {
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j) {
                        v4f& t = tot[SPLIT ? i : 0][SPLIT ? j : 0];
                        t = s + 1 == p.span ? acc[i][j] : t + acc[i][j];
                        acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
                    }
                left = p.span;
            }
        }
        if (SPLIT && p.span > 0 && p.span < S) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] = tot[SPLIT ? i : 0][SPLIT ? j : 0] + acc[i][j];
        }
        // the epilogue's operands of 16 rows at a time go out together (the stores
        // may alias them as far as the compiler knows, so it would not move the
        // loads of one output above the store of another)
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            float e1[EPI == 1 || EPI == 3 ? FN : 1][4], e2[EPI == 3 ? FN : 1][4];
            if constexpr (EPI == 1 || EPI == 3) {
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {
                        const int n = (nf0 + j) * 16 + li;
                        const long long m = m0 + i * 16 + 4 * lk + rr;
                        const bool in = n < p.N && m < p.M;
                        e1[j][rr] = in ? (EPI == 1 ? p.Cin : p.y)[m * p.ldc + n] : 0.0f;
                        if constexpr (EPI == 3) e2[j][rr] = in ? p.z[m * p.ldc2 + n] : 0.0f;
                    }
            }
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const int n = (nf0 + j) * 16 + li;
                if (n >= p.N) continue;
                const float bias = EPI == 2 ? p.bias[n] : 0.0f;
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    const long long m = m0 + i * 16 + 4 * lk + rr;
                    if (m >= p.M) continue;
                    const float v = acc[i][j][rr];
                    float* dst = p.C + m * p.ldc + n;
                    if constexpr (EPI == 0) {
                        *dst = v;
                    } else if constexpr (EPI == 1) {
                        *dst = e1[j][rr] + v;
                    } else if constexpr (EPI == 2) {
                        const float u = v + bias;
                        *dst = u;
                        p.C2[m * p.ldc + n] = softplus_f(u);
                    } else {
                        *dst = v * silu_f(e2[j][rr]);
                        p.C2[m * p.ldc2 + n] = v * e1[j][rr] * dsilu_f(e2[j][rr]);
                    }
                }
            }
        }
    }
}

// Weight matrices of one layer (or the head) in fragment order for k_trow:
// job j covers the matrix X [N][K], X(n, k) = src[n sn + k sk] (a weight or its
// transpose), padded with zeros to NP x KP; bf16 or f32 like the launch.
struct FragJob {
    const float* src;
    void* dst;
    int sn, sk, N, K, NP, KP;
};
constexpr int FRAG_JOBS = 12;
struct FragJobs {
    FragJob j[FRAG_JOBS];
};
template <int DT>
__global__ __launch_bounds__(256) void k_tr_frags(FragJobs jobs) {
    const FragJob& q = jobs.j[blockIdx.y];
    const long long n_all = (long long)q.NP * q.KP;
    for (long long i = blockIdx.x * 256LL + threadIdx.x; i < n_all; i += gridDim.x * 256LL) {
        constexpr int J = DT == 0 ? 4 : 8;
        const int j = (int)(i % J);
        long long t = i / J;
        const int lane = (int)(t & 63);
        t >>= 6;
        const int S = q.KP / (4 * J), s = (int)(t % S), nf = (int)(t / S);
        const int n = 16 * nf + (lane & 15);
        const int k = DT == 0 ? 16 * s + 4 * j + (lane >> 4) : 32 * s + 8 * (lane >> 4) + j;
        const float v = n < q.N && k < q.K ? q.src[(long long)n * q.sn + (long long)k * q.sk] : 0.0f;
        if (DT == 0) static_cast<float*>(q.dst)[i] = v;
        else static_cast<uint16_t*>(q.dst)[i] = f2bf_bits(v);
    }
}

// ============================================================ weight gradients
// part[z][N][K] = sum over the rows of slice z of dY[r][n] X[r][k]: a workgroup
// of 8 waves owns a TA x TB tile of the gradient and walks its slice 32 rows at
// a time, the next 32 rows in flight in registers while the current ones are
// multiplied.  Half of the threads load dY, half X: 8 rows x 4 columns each, so
// that a thread holds 8 consecutive rows of a column, the operand order of the
// bf16 MFMA, and no transpose is needed.  A 256 x 256 tile reads dY of the
// in_proj gradient once and X four times; grid.x is the slice, so that the
// tiles of a slice share an XCD's L2.  Bound by HBM (k_tg took 1.46 ms per
// gradient over 262112 rows on average, this one 0.16 ms).
template <int DT, int TA, int TB>
__global__ __launch_bounds__(512) void k_tg_w(const float* __restrict__ dY, long long ldy, int N,
                                              const float* __restrict__ X, long long ldx, int K, long long rows,
                                              long long per, float* __restrict__ part) {
    using ET = typename std::conditional<DT == 0, float, uint16_t>::type;
    constexpr int RS = DT == 0 ? 36 : 40;                       // LDS row stride: 32 rows of the reduction + pad
    constexpr int WA = TA == 256 ? (TB == 256 ? 4 : 8) : 1, WB = 8 / WA;
    constexpr int FA = TA / WA / 16, FB = TB / WB / 16;
    __shared__ __align__(16) ET As[TA * RS];
    __shared__ __align__(16) ET Bs[TB * RS];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nt = (K + TB - 1) / TB;
    const int n0 = (blockIdx.y / nt) * TA, k0 = (blockIdx.y % nt) * TB;
    const long long r0 = blockIdx.x * per, r1 = r0 + per < rows ? r0 + per : rows;
    const bool isA = tid < 256;
    const int cg = (tid & 63) * 4, rg = ((tid >> 6) & 3) * 8;   // 4 columns, 8 rows
    const float* src = isA ? dY : X;
    const long long ld = isA ? ldy : ldx;
    const int c0 = (isA ? n0 : k0) + cg;
    const bool cols = cg < (isA ? TA : TB) && c0 < (isA ? N : K);
    float4 v[8];
    auto load = [&](long long r) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (cols && r + rg + i < r1) v[i] = *reinterpret_cast<const float4*>(src + (r + rg + i) * ld + c0);
        }
    };
    v4f acc[FA][FB];
#pragma unroll
    for (int i = 0; i < FA; ++i)
#pragma unroll
        for (int j = 0; j < FB; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    const int li = lane & 15, lk = lane >> 4;
    const int ra = (wv / WB) * FA * 16, rb = (wv % WB) * FB * 16;
    load(r0);
    for (long long r = r0; r < r1; r += 32) {
        if (cg < (isA ? TA : TB)) {
            ET* S = (isA ? As : Bs) + cg * RS + rg;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float w[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) w[i] = c == 0 ? v[i].x : c == 1 ? v[i].y : c == 2 ? v[i].z : v[i].w;
                if constexpr (DT == 0) {
                    *reinterpret_cast<float4*>(S + c * RS) = make_float4(w[0], w[1], w[2], w[3]);
                    *reinterpret_cast<float4*>(S + c * RS + 4) = make_float4(w[4], w[5], w[6], w[7]);
                } else {
                    uint4 u;
                    u.x = (uint32_t)f2bf_bits(w[0]) | ((uint32_t)f2bf_bits(w[1]) << 16);
                    u.y = (uint32_t)f2bf_bits(w[2]) | ((uint32_t)f2bf_bits(w[3]) << 16);
                    u.z = (uint32_t)f2bf_bits(w[4]) | ((uint32_t)f2bf_bits(w[5]) << 16);
                    u.w = (uint32_t)f2bf_bits(w[6]) | ((uint32_t)f2bf_bits(w[7]) << 16);
                    *reinterpret_cast<uint4*>(S + c * RS) = u;
                }
            }
        }
        __syncthreads();
        if (r + 32 < r1) load(r + 32);
        if constexpr (DT == 0) {
#pragma unroll
            for (int ks = 0; ks < 32; ks += 4) {
                float af[FA], bf[FB];
#pragma unroll
                for (int i = 0; i < FA; ++i) af[i] = As[(ra + i * 16 + li) * RS + ks + lk];
#pragma unroll
                for (int j = 0; j < FB; ++j) bf[j] = Bs[(rb + j * 16 + li) * RS + ks + lk];
#pragma unroll
                for (int i = 0; i < FA; ++i)
#pragma unroll
                    for (int j = 0; j < FB; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[i], bf[j], acc[i][j], 0, 0, 0);
            }
        } else {
            v8bf af[FA];
#pragma unroll
            for (int i = 0; i < FA; ++i) af[i] = *reinterpret_cast<const v8bf*>(As + (ra + i * 16 + li) * RS + 8 * lk);
#pragma unroll
            for (int j = 0; j < FB; ++j) {
                const v8bf bf = *reinterpret_cast<const v8bf*>(Bs + (rb + j * 16 + li) * RS + 8 * lk);
#pragma unroll
                for (int i = 0; i < FA; ++i)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bf, acc[i][j], 0, 0, 0);
            }
        }
        __syncthreads();
    }
    float* out = part + (long long)blockIdx.x * N * K;
#pragma unroll
    for (int i = 0; i < FA; ++i)
#pragma unroll
        for (int j = 0; j < FB; ++j)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const int n = n0 + ra + i * 16 + 4 * lk + rr, k = k0 + rb + j * 16 + li;
                if (n < N && k < K) out[(long long)n * K + k] = acc[i][j][rr];
            }
}

// ============================================================ fixed-order sums
// out[i] (+)= part[i] + part[stride + i] + ... over S slices: a workgroup owns
// 64 columns, wave q adds the slices of the q-th quarter in increasing order
// and the quarters are added in order.  Bound by the latency of its loads,
// which the quarters and the unrolled loop keep in flight together.
__global__ __launch_bounds__(256) void k_sum_slices(const float* __restrict__ part, int S, long long n,
                                                    long long stride, float* __restrict__ out, int accumulate) {
    __shared__ float q_s[4][64];
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const long long i = blockIdx.x * 64LL + lane;
    const int per = (S + 3) / 4, s0 = q * per, s1 = s0 + per < S ? s0 + per : S;
    float v = 0.f;
    if (i < n) {
#pragma unroll 8
        for (int s = s0; s < s1; ++s) v += part[(long long)s * stride + i];
    }
    q_s[q][lane] = v;
    __syncthreads();
    if (q == 0 && i < n) {
        v = ((q_s[0][lane] + q_s[1][lane]) + q_s[2][lane]) + q_s[3][lane];
        out[i] = accumulate ? out[i] + v : v;
    }
}

// the same for the split partials [S][M][N] of a GEMM, into C[m ldc + n]
__global__ void k_sum_slices_2d(const float* __restrict__ part, int S, int M, int N, float* __restrict__ C,
                                long long ldc, int accumulate) {
    long long i = blockIdx.x * 256LL + threadIdx.x;
    const long long n_all = (long long)M * N;
    if (i >= n_all) return;
    float v = part[i];
    for (int s = 1; s < S; ++s) v += part[(long long)s * n_all + i];
    float* d = C + (i / N) * ldc + i % N;
    *d = accumulate ? *d + v : v;
}

// part[s * N + n] = sum over the rows of slice s of X[r ld + n]: wave w of the
// workgroup adds rows r0 + w, r0 + w + 4, ... in order, four columns per lane,
// then the waves are added in order.  N and ld are multiples of 4.
__global__ __launch_bounds__(256) void k_colsum_part(const float* __restrict__ X, long long rows, int ld, int N,
                                                     long long per, float* __restrict__ part) {
    __shared__ float4 w_s[4][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, n = blockIdx.x * 256 + 4 * lane;
    const long long r0 = blockIdx.y * per, r1 = r0 + per < rows ? r0 + per : rows;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
    if (n < N) {
#pragma unroll 4
        for (long long r = r0 + wv; r < r1; r += 4) {
            const float4 v = *reinterpret_cast<const float4*>(X + r * ld + n);
            a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w;
        }
    }
    w_s[wv][lane] = a;
    __syncthreads();
    if (wv == 0 && n < N) {
        for (int k = 1; k < 4; ++k) {
            const float4 v = w_s[k][lane];
            a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w;
        }
        *reinterpret_cast<float4*>(part + (long long)blockIdx.y * N + n) = a;
    }
}

// One workgroup: *out = sum of in[0 .. n) in double; thread t sums t, t + 256,
// ... in order, then a fixed halving tree.  scale multiplies the result.
template <typename TI>
__global__ __launch_bounds__(256) void k_sum_all(const TI* __restrict__ in, long long n, double scale,
                                                 double* __restrict__ out_d, float* __restrict__ out_f) {
    __shared__ double buf[256];
    const int t = threadIdx.x;
    double acc = 0.0;
#pragma unroll 8
    for (long long i = t; i < n; i += 256) acc += (double)in[i];
    buf[t] = acc;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (t < h) buf[t] += buf[t + h];
        __syncthreads();
    }
    if (t == 0) {
        if (out_d) *out_d = buf[0] * scale;
        if (out_f) *out_f = (float)(buf[0] * scale);
    }
}

// ============================================================ elementwise and per-row kernels
__global__ void k_tr_embed(const uint8_t* __restrict__ tok, int B, int T, const float* __restrict__ E, int D,
                           float* __restrict__ r) {
    const int Tn = T - 1;
    long long row = blockIdx.x * 4LL + threadIdx.y;
    if (row >= (long long)B * Tn) return;
    int b = (int)(row / Tn), t = (int)(row % Tn);
    int y = tok[(long long)b * T + t];
    for (int k = threadIdx.x; k < D; k += 64) r[row * D + k] = E[(long long)y * D + k];
}

// Embedding gradient of one slice of rows and 64 columns: one wave adds the
// rows of its slice in order into a [256][64] LDS table (lane = column, so
// no two lanes touch one address; the adds are LDS instructions without a
// return value, in the wave's order, so a row does not wait for the sum of the
// one before); the table is the slice's partial
// part[s][256][D].
__global__ __launch_bounds__(64) void k_tr_embed_bwd_part(const uint8_t* __restrict__ tok, int B, int T,
                                                          const float* __restrict__ dr, int D, long long per,
                                                          float* __restrict__ part) {
    __shared__ float acc[VOCAB][64];
    const int lane = threadIdx.x, c = blockIdx.x * 64 + lane;
    const int Tn = T - 1;
    const long long rows = (long long)B * Tn;
    for (int y = 0; y < VOCAB; ++y) acc[y][lane] = 0.f;
    const long long r0 = blockIdx.y * per, r1 = r0 + per < rows ? r0 + per : rows;
    for (long long r = r0; r < r1; r += 8) {
        int ys[8];
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const long long rr = r + j;
            ys[j] = -1;
            v[j] = 0.f;
            if (rr < r1) {
                const int b = (int)(rr / Tn), t = (int)(rr % Tn);
                ys[j] = tok[(long long)b * T + t];
                v[j] = dr[rr * D + c];
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (ys[j] >= 0) __hip_atomic_fetch_add(&acc[ys[j]][lane], v[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    }
    float* dst = part + (long long)blockIdx.y * VOCAB * D + c;
    for (int y = 0; y < VOCAB; ++y) dst[(long long)y * D] = acc[y][lane];
}

// LayerNorm forward, one wave per row (NV = D / 64 values per lane in
// registers, ln_stats' operations); keeps (mean, rstd)
template <int NV>
__global__ __launch_bounds__(256) void k_tr_ln_fwd(const float* __restrict__ x, long long rows,
                                                   const float* __restrict__ w, const float* __restrict__ b,
                                                   float* __restrict__ out, float* __restrict__ st) {
    constexpr int D = 64 * NV;
    const long long row = blockIdx.x * 4LL + (threadIdx.x >> 6);
    if (row >= rows) return;
    const int lane = threadIdx.x & 63;
    float v[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) v[j] = x[row * D + lane + 64 * j];
    float mu, rs;
    ln_stats_v<NV>(v, D, mu, rs);
#pragma unroll
    for (int j = 0; j < NV; ++j) out[row * D + lane + 64 * j] = ln_apply(v[j], mu, rs, w[lane + 64 * j], b[lane + 64 * j]);
    if (lane == 0) { st[2 * row] = mu; st[2 * row + 1] = rs; }
}

// LayerNorm backward of one slice of rows: dx (+)= rstd (dxh - mean(dxh) -
// xh mean(dxh xh)), dxh = dy w, one wave per row; and the slice's partial sums
// of dy xh and dy (the weight and bias gradients), part[s][2][D]: wave w adds
// its rows r0 + w, r0 + w + 4, ... in order in registers, then the waves are
// added in order.  Bound by HBM: dy, x and dx pass once (a separate dy xh tensor
// and two column sums took 1.06 ms per LayerNorm of 262112 x 256, against
// 0.2 ms).
template <int NV>
__global__ __launch_bounds__(256) void k_tr_ln_bwd(const float* __restrict__ dy, const float* __restrict__ x,
                                                   const float* __restrict__ st, long long rows, long long per,
                                                   const float* __restrict__ w, float* __restrict__ dx, int accumulate,
                                                   float* __restrict__ part) {
    constexpr int D = 64 * NV;
    __shared__ float p_s[4][2 * D];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const long long r0 = blockIdx.x * per, r1 = r0 + per < rows ? r0 + per : rows;
    float wk[NV], gw[NV], gb[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) { wk[j] = w[lane + 64 * j]; gw[j] = 0.f; gb[j] = 0.f; }
#pragma unroll 2
    for (long long row = r0 + wv; row < r1; row += 4) {
        const float mu = st[2 * row], rs = st[2 * row + 1];
        float xh[NV], g[NV], old[NV], s1 = 0.f, s2 = 0.f;
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const long long at = row * D + lane + 64 * j;
            xh[j] = x[at];
            g[j] = dy[at];
            old[j] = accumulate ? dx[at] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            xh[j] = (xh[j] - mu) * rs;
            const float dxh = g[j] * wk[j];
            s1 += dxh;
            s2 += dxh * xh[j];
            gw[j] += g[j] * xh[j];
            gb[j] += g[j];
        }
        s1 = wave_sum(s1) / (float)D;
        s2 = wave_sum(s2) / (float)D;
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const float v = rs * (g[j] * wk[j] - s1 - xh[j] * s2);
            dx[row * D + lane + 64 * j] = accumulate ? old[j] + v : v;
        }
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) { p_s[wv][lane + 64 * j] = gw[j]; p_s[wv][D + lane + 64 * j] = gb[j]; }
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * D; i += 256)
        part[(long long)blockIdx.x * 2 * D + i] = ((p_s[0][i] + p_s[1][i]) + p_s[2][i]) + p_s[3][i];
}

// Causal depthwise conv + SiLU over each sequence (zero before t = 0): one
// thread per channel walks CONV_TS rows with the window in registers, so that
// each x is read once.  Bound by HBM (0.94 ms per 262112 x 512 with one thread
// per element, 0.32 ms now).
constexpr int CONV_TS = 64, CONV_RB = 8;      // rows per thread, rows loaded together
DEVI float conv_at(const float (&cw)[KCONV], float cb, const float (&w)[KCONV]) {
    float acc = cb;
#pragma unroll
    for (int k = 0; k < KCONV; ++k) acc = fmaf(cw[k], w[k], acc);
    return acc;
}
__global__ __launch_bounds__(256) void k_tr_conv_fwd(const float* __restrict__ xz, int Tn, int Di,
                                                     const float* __restrict__ cw, const float* __restrict__ cb,
                                                     float* __restrict__ xs) {
    const int d = blockIdx.x * blockDim.x + threadIdx.x, b = blockIdx.z;
    if (d >= Di) return;
    const int t0 = blockIdx.y * CONV_TS, t1 = t0 + CONV_TS < Tn ? t0 + CONV_TS : Tn;
    const float* x = xz + (long long)b * Tn * 2 * Di + d;
    float* o = xs + (long long)b * Tn * Di + d;
    float c[KCONV], w[KCONV];
#pragma unroll
    for (int k = 0; k < KCONV; ++k) c[k] = cw[d * KCONV + k];
    const float bias = cb[d];
    w[0] = 0.f;
#pragma unroll
    for (int k = 1; k < KCONV; ++k) w[k] = t0 - KCONV + k >= 0 ? x[(long long)(t0 - KCONV + k) * 2 * Di] : 0.f;
    for (int t = t0; t < t1; t += CONV_RB) {
        float v[CONV_RB];
#pragma unroll
        for (int j = 0; j < CONV_RB; ++j) v[j] = t + j < t1 ? x[(long long)(t + j) * 2 * Di] : 0.f;
#pragma unroll
        for (int j = 0; j < CONV_RB; ++j) {
            w[0] = w[1]; w[1] = w[2]; w[2] = w[3]; w[3] = v[j];
            if (t + j < t1) o[(long long)(t + j) * Di] = silu_f(conv_at(c, bias, w));
        }
    }
}

// Conv backward of one slice of CONV_TS rows, one thread per channel.  With
// p_t = dxs_t silu'(xc_t) (xc recomputed from the window): dx_t = sum over k of
// p_{t + 3 - k} w_k, into dxz[:, :Di]; and the slice's partial weight and bias
// gradients in row order, part[s][d K + k] = sum p_t x_{t - back_k},
// part[s][Di K + d] = sum p_t.  Each input is read once, but for three rows
// on either side (two kernels that kept xc and p in memory took 2.5 ms per
// 262112 x 512, 0.43 ms now).
__global__ __launch_bounds__(256) void k_tr_conv_bwd(const float* __restrict__ dxs, const float* __restrict__ xz, int Tn,
                                                     int Di, const float* __restrict__ cw,
                                                     const float* __restrict__ cb, float* __restrict__ dxz,
                                                     float* __restrict__ part) {
    const int d = blockIdx.x * blockDim.x + threadIdx.x, b = blockIdx.z;
    if (d >= Di) return;
    const int t0 = blockIdx.y * CONV_TS, t1 = t0 + CONV_TS < Tn ? t0 + CONV_TS : Tn;
    const float* x = xz + (long long)b * Tn * 2 * Di + d;
    const float* g = dxs + (long long)b * Tn * Di + d;
    float* o = dxz + (long long)b * Tn * 2 * Di + d;
    float c[KCONV], w[KCONV], p[KCONV], aw[KCONV], ab = 0.f;
#pragma unroll
    for (int k = 0; k < KCONV; ++k) { c[k] = cw[d * KCONV + k]; aw[k] = 0.f; p[k] = 0.f; }
    const float bias = cb[d];
    w[0] = 0.f;
#pragma unroll
    for (int k = 1; k < KCONV; ++k) w[k] = t0 - KCONV + k >= 0 ? x[(long long)(t0 - KCONV + k) * 2 * Di] : 0.f;
    // row u enters with its p; row u - 3 then has every p it needs
    for (int u = t0; u < t1 + KCONV - 1; u += CONV_RB) {
        float xv[CONV_RB], gv[CONV_RB];
#pragma unroll
        for (int j = 0; j < CONV_RB; ++j) {
            const bool in = u + j < Tn && u + j < t1 + KCONV - 1;
            xv[j] = in ? x[(long long)(u + j) * 2 * Di] : 0.f;
            gv[j] = in ? g[(long long)(u + j) * Di] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < CONV_RB; ++j) {
            w[0] = w[1]; w[1] = w[2]; w[2] = w[3]; w[3] = xv[j];
            p[0] = p[1]; p[1] = p[2]; p[2] = p[3];
            p[3] = gv[j] * dsilu_f(conv_at(c, bias, w));
            if (u + j < t1) {                       // p[3] belongs to row u + j of this slice
                ab += p[3];
#pragma unroll
                for (int k = 0; k < KCONV; ++k) aw[k] += p[3] * w[k];
            }
            const int t = u + j - (KCONV - 1);
            if (t >= t0 && t < t1) {
                float acc = 0.f;
#pragma unroll
                for (int k = 0; k < KCONV; ++k) acc += p[KCONV - 1 - k] * c[k];
                o[(long long)t * 2 * Di] = acc;
            }
        }
    }
    float* dst = part + ((long long)b * gridDim.y + blockIdx.y) * Di * (KCONV + 1);
#pragma unroll
    for (int k = 0; k < KCONV; ++k) dst[d * KCONV + k] = aw[k];
    dst[Di * KCONV + d] = ab;
}

// feed-forward sub-layer: u += b1 (in place), gu = GELU(u) (exact erf form)
DEVI float gelu_tr(float u) { return 0.5f * u * (1.0f + erff(u * 0.7071067811865476f)); }
DEVI float dgelu_tr(float u) {        // Phi(u) + u phi(u)
    return 0.5f * (1.0f + erff(u * 0.7071067811865476f)) + u * expf(-0.5f * u * u) * 0.3989422804014327f;
}
__global__ void k_tr_bias_gelu(float* __restrict__ u, long long rows, int H, const float* __restrict__ b,
                               float* __restrict__ gu) {
    long long i = blockIdx.x * 256LL + threadIdx.x;
    if (i >= rows * H) return;
    const float v = u[i] + b[i % H];
    u[i] = v;
    gu[i] = gelu_tr(v);
}
// x += b per row (bias of the second feed-forward product)
__global__ void k_tr_add_bias(float* __restrict__ x, long long rows, int N, const float* __restrict__ b) {
    long long i = blockIdx.x * 256LL + threadIdx.x;
    if (i < rows * N) x[i] += b[i % N];
}
// du = dgu * GELU'(u), in place in dgu
__global__ void k_tr_gelu_bwd(float* __restrict__ dgu, const float* __restrict__ u, long long n) {
    long long i = blockIdx.x * 256LL + threadIdx.x;
    if (i < n) dgu[i] *= dgelu_tr(u[i]);
}

// Selective scan, split over time.  The recurrence h_t = exp(dt_t A) h_{t-1} +
// (dt_t x_t) B_t is one multiply and one add per state and step, while the
// output, the gate and the gradients are most of the work and need h only at
// their own step.  So both directions run in two kernels:
//   k_tr_states / k_tr_gstates  the recurrence alone, in order over time; a
//     thread owns one channel and NPT of its 16 states, and the state is
//     written every few steps;
//   k_tr_scan_y / k_tr_scan_bwd  blocks of time in parallel, each from the
//     state at its start.
// Every value is the one a single pass over time computes, with the same
// operations in the same order.  One wave per (sequence, 64 channels) walking
// the whole sequence left a training step of 32 x 8192 tokens at d_inner 512
// with 256 waves, one per compute unit: 8.6 ms forward and 18.1 ms backward
// per layer, against 1.5 ms (states 0.8, outputs 0.7) and 3.6 ms (adjoint states
// 0.6, gradients 3.0 with the softplus) now.
// exp(dt A) = exp2(dt (A log2 e)) on the hardware exp2.
constexpr int SCAN_CH = 64;           // channels per wave (one per lane)
constexpr int SCAN_SB = 64;           // rows staged in LDS at a time
constexpr int SCAN_SUB = 8;           // steps between the states the backward pass starts from
constexpr int SCAN_FWD_BLOCK = 32;    // steps of one k_tr_scan_y wave
constexpr float LOG2E_F = 1.4426950408889634f;

// Geometry of a scan over B sequences of Tn steps: each sequence is cut into
// NC chunks of Tc steps (the last may be short); inside a chunk the state is
// kept every `sub` steps, nsub slots per chunk.
DEVI long long scan_slot(int b, int NC, int c, int n_per, int k) { return ((long long)b * NC + c) * n_per + k; }

// States: one workgroup per (64 channels, chunk, sequence) and per 4 * NPT
// states (blockIdx.x = channel block * (16 / (4 NPT)) + state group); wave w of
// it owns NPT states.  NPT 4 puts all 16 states in one workgroup, which reads
// dt and x once; NPT 1 spreads them over four workgroups, for launches of too
// few channel blocks to fill the GPU.  Bound by the chain of one step (two
// dependent operations) and by issue: the rows of a block are staged in LDS
// while the previous block is walked.  The state before step t goes to
// hsub slot t / sub of its chunk (chunk c of a sequence from slot c nsub of its
// nseq on), and with hsave to hsave[b][t / Tsave].  The
// state at the start of chunk c is h0[b][c h0s] of h0n per sequence (null: zero).  AL:
// sub and Tsave are multiples of 8 (the check then runs once per 8 rows).
template <int NPT, bool AL>
__global__ __launch_bounds__(256) void k_tr_states(const float* __restrict__ xs, const float* __restrict__ dt,
                                                   const float* __restrict__ dbc, int NO, int R,
                                                   const float* __restrict__ A_log, int Tn, int Di, int Tc, int NC,
                                                   const float* __restrict__ h0, int h0n, int h0s,
                                                   float* __restrict__ hsub, int sub, int nsub, int nseq,
                                                   float* __restrict__ hsave, int Tsave, int nsave) {
    constexpr int WS = 4 * NPT, NG = NSTATE / WS;             // states and workgroups per channel block
    constexpr int RPW = SCAN_SB / 4;
    __shared__ float dt_s[SCAN_SB][SCAN_CH], x_s[SCAN_SB][SCAN_CH];
    __shared__ __align__(16) float b_s[SCAN_SB][WS];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int d = (blockIdx.x / NG) * SCAN_CH + lane, c = blockIdx.y, b = blockIdx.z;
    const int n0 = (blockIdx.x % NG) * WS + wv * NPT;
    const bool on = d < Di;
    const int t0 = c * Tc, t1 = t0 + Tc < Tn ? t0 + Tc : Tn;
    const long long row0 = (long long)b * Tn;
    float A2[NPT], h[NPT];
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
        A2[i] = on ? -expf(A_log[d * NSTATE + n0 + i]) * LOG2E_F : 0.f;
        h[i] = on && h0 ? h0[(((long long)b * h0n + (long long)c * h0s) * NSTATE + n0 + i) * Di + d] : 0.f;
    }
    float rd[RPW], rx[RPW], rb[(SCAN_SB * WS + 255) / 256];
    auto fetch = [&](int s0) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int t = s0 + wv + 4 * i;
            const bool in = on && t < t1;
            rd[i] = in ? dt[(row0 + t) * Di + d] : 0.f;
            rx[i] = in ? xs[(row0 + t) * Di + d] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < (SCAN_SB * WS + 255) / 256; ++i) {
            const int e = tid + 256 * i, t = s0 + e / WS;
            rb[i] = e < SCAN_SB * WS && t < t1
                        ? dbc[(row0 + t) * NO + R + (blockIdx.x % NG) * WS + e % WS]
                        : 0.f;
        }
    };
    fetch(t0);
    int next = t0, slot = 0, nexts = hsave ? t0 : INT32_MAX, slots = t0 / (hsave ? Tsave : 1);
    for (int s0 = t0; s0 < t1; s0 += SCAN_SB) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < RPW; ++i) { dt_s[wv + 4 * i][lane] = rd[i]; x_s[wv + 4 * i][lane] = rx[i]; }
#pragma unroll
        for (int i = 0; i < (SCAN_SB * WS + 255) / 256; ++i) {
            const int e = tid + 256 * i;
            if (e < SCAN_SB * WS) b_s[e / WS][e % WS] = rb[i];
        }
        __syncthreads();
        fetch(s0 + SCAN_SB);
        // groups of 8 rows: their exponentials and inputs first (no chain), then
        // the recurrence; rows past t1 are zero and leave h unused
#pragma unroll 1
        for (int t8 = s0; t8 < s0 + SCAN_SB; t8 += 8) {
            float a[8][NPT], u[8][NPT];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int r = t8 - s0 + j;
                const float dtv = dt_s[r][lane], x = x_s[r][lane];
#pragma unroll
                for (int i = 0; i < NPT; ++i) {
                    a[j][i] = exp2_hw(dtv * A2[i]);
                    u[j][i] = dtv * x * b_s[r][wv * NPT + i];
                }
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int t = t8 + j;
                if (!AL || j == 0) {                  // aligned: states fall on group starts only
                    if (t == next && t < t1) {
                        if (on && hsub) {
                            float* o = hsub + (((long long)b * nseq + (long long)c * nsub + slot) * NSTATE + n0) * Di + d;
#pragma unroll
                            for (int i = 0; i < NPT; ++i) o[(long long)i * Di] = h[i];
                        }
                        next += sub;
                        ++slot;
                    }
                    if (t == nexts && t < t1) {
                        if (on) {
                            float* o = hsave + (((long long)b * nsave + slots) * NSTATE + n0) * Di + d;
#pragma unroll
                            for (int i = 0; i < NPT; ++i) o[(long long)i * Di] = h[i];
                        }
                        nexts += Tsave;
                        ++slots;
                    }
                }
#pragma unroll
                for (int i = 0; i < NPT; ++i) h[i] = a[j][i] * h[i] + u[j][i];
            }
        }
    }
}

// The adjoint recurrence alone, from the last step to the first:
// gh <- (gh + C_t dy_t) exp(dt_t A).  gh as it enters the last step of every
// block of TB steps goes to ghb slot b * NBS + c * nblk + k (nblk blocks per
// whole chunk, NBS per sequence).  AL: block ends fall on multiples of 8 rows
// (a single chunk, or Tc a multiple of 8).
// Shape and bound as in k_tr_states.
template <int NPT, bool AL>
__global__ __launch_bounds__(256) void k_tr_gstates(const float* __restrict__ dt, const float* __restrict__ dbc, int NO,
                                                    int R, const float* __restrict__ A_log,
                                                    const float* __restrict__ dy, int Tn, int Di, int Tc, int NC,
                                                    int TB, int nblk, int NBS, float* __restrict__ ghb) {
    constexpr int WS = 4 * NPT, NG = NSTATE / WS;
    constexpr int RPW = SCAN_SB / 4;
    __shared__ float dt_s[SCAN_SB][SCAN_CH], g_s[SCAN_SB][SCAN_CH];
    __shared__ __align__(16) float c_s[SCAN_SB][WS];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int d = (blockIdx.x / NG) * SCAN_CH + lane, b = blockIdx.z;
    const int n0 = (blockIdx.x % NG) * WS + wv * NPT;
    const bool on = d < Di;
    const long long row0 = (long long)b * Tn;
    float A2[NPT], gh[NPT];
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
        A2[i] = on ? -expf(A_log[d * NSTATE + n0 + i]) * LOG2E_F : 0.f;
        gh[i] = 0.f;
    }
    float rd[RPW], rg[RPW], rc[(SCAN_SB * WS + 255) / 256];
    auto fetch = [&](int s1) {                    // rows s1 - SCAN_SB .. s1 - 1, row s1 - 1 - i at place i
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int t = s1 - 1 - (wv + 4 * i);
            const bool in = on && t >= 0 && t < Tn;
            rd[i] = in ? dt[(row0 + t) * Di + d] : 0.f;
            rg[i] = in ? dy[(row0 + t) * Di + d] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < (SCAN_SB * WS + 255) / 256; ++i) {
            const int e = tid + 256 * i, t = s1 - 1 - e / WS;
            rc[i] = e < SCAN_SB * WS && t >= 0 && t < Tn
                        ? dbc[(row0 + t) * NO + R + NSTATE + (blockIdx.x % NG) * WS + e % WS]
                        : 0.f;
        }
    };
    // the walk starts on a row multiple of SCAN_SB, rows past Tn being zero
    const int top = (Tn + SCAN_SB - 1) / SCAN_SB * SCAN_SB;
    fetch(top);
    // block (c, k) that the walk is about to enter, and its last step
    int c = NC - 1, k = (Tn - c * Tc - 1) / TB, next = Tn - 1;
    for (int s1 = top; s1 > 0; s1 -= SCAN_SB) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < RPW; ++i) { dt_s[wv + 4 * i][lane] = rd[i]; g_s[wv + 4 * i][lane] = rg[i]; }
#pragma unroll
        for (int i = 0; i < (SCAN_SB * WS + 255) / 256; ++i) {
            const int e = tid + 256 * i;
            if (e < SCAN_SB * WS) c_s[e / WS][e % WS] = rc[i];
        }
        __syncthreads();
        fetch(s1 - SCAN_SB);
#pragma unroll 1
        for (int j8 = 0; j8 < SCAN_SB; j8 += 8) {
            float a[8][NPT], u[8][NPT];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float dtv = dt_s[j8 + j][lane], g = g_s[j8 + j][lane];
#pragma unroll
                for (int i = 0; i < NPT; ++i) {
                    a[j][i] = exp2_hw(dtv * A2[i]);
                    u[j][i] = c_s[j8 + j][wv * NPT + i] * g;
                }
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                // aligned: a block's last step is the first row of a group, or
                // (the last step of all) follows rows past the end, which leave gh 0
                const int t = s1 - 1 - (j8 + j);
                if (AL ? j == 0 && next >= 0 && next > t - 8 : t == next && t >= 0) {
                    if (on) {
                        float* o = ghb + (((long long)b * NBS + c * nblk + k) * NSTATE + n0) * Di + d;
#pragma unroll
                        for (int i = 0; i < NPT; ++i) o[(long long)i * Di] = gh[i];
                    }
                    if (k > 0) {
                        --k;
                    } else {
                        --c;
                        k = (Tc - 1) / TB;
                    }
                    next = c < 0 ? -1 : c * Tc + (k + 1) * TB - 1;
                    if (c >= 0 && next > c * Tc + Tc - 1) next = c * Tc + Tc - 1;
                }
#pragma unroll
                for (int i = 0; i < NPT; ++i) {
                    gh[i] += u[j][i];
                    gh[i] *= a[j][i];
                }
            }
        }
    }
}

// rows [r0, r1) of B and C (columns R .. R + 31 of dbc, row stride NO) into bc_s
DEVI void stage_bc(float* bc_s, const float* __restrict__ dbc, long long row_base, int r0, int r1, int NO, int R,
                   int tid, int nthreads) {
    for (int i = tid; i < (r1 - r0) * 2 * NSTATE; i += nthreads)
        bc_s[i] = dbc[(row_base + r0 + i / (2 * NSTATE)) * NO + R + i % (2 * NSTATE)];
}

// Output of the scan (and the gate when g is given): one thread per channel,
// one block of TB steps per workgroup row, from the state at the block's
// start (slot k * slots_per_block of the chunk).  Bound by VALU issue (16
// states) with enough blocks in flight to hide the row loads.
__global__ __launch_bounds__(256) void k_tr_scan_y(const float* __restrict__ xs, const float* __restrict__ dt,
                                                   const float* __restrict__ dbc, int NO, int R,
                                                   const float* __restrict__ A_log, const float* __restrict__ Dsk,
                                                   const float* __restrict__ xz, int Tn, int Di, int TB, int nslot,
                                                   int slots_per_block, const float* __restrict__ hsub,
                                                   float* __restrict__ y, float* __restrict__ g) {
    __shared__ __align__(16) float bc_s[SCAN_SB * 2 * NSTATE];
    const int b = blockIdx.z, d = blockIdx.x * blockDim.x + threadIdx.x;
    const bool on = d < Di;
    const int t0 = blockIdx.y * TB, t1 = t0 + TB < Tn ? t0 + TB : Tn;
    const long long row0 = (long long)b * Tn;
    float A2[NSTATE], h[NSTATE];
    const float* hs = hsub + (((long long)b * nslot + (long long)blockIdx.y * slots_per_block) * NSTATE) * Di + (on ? d : 0);
#pragma unroll
    for (int n = 0; n < NSTATE; ++n) {
        A2[n] = on ? -expf(A_log[d * NSTATE + n]) * LOG2E_F : 0.f;
        h[n] = on ? hs[(long long)n * Di] : 0.f;
    }
    const float Dv = on ? Dsk[d] : 0.f;
    for (int s0 = t0; s0 < t1; s0 += SCAN_SB) {
        const int s1 = s0 + SCAN_SB < t1 ? s0 + SCAN_SB : t1;
        __syncthreads();
        stage_bc(bc_s, dbc, row0, s0, s1, NO, R, threadIdx.x, blockDim.x);
        __syncthreads();
        float dtn = 0.f, xn = 0.f, zn = 0.f;
        auto fetch = [&](int t) {
            const long long row = row0 + t;
            dtn = dt[row * Di + d];
            xn = xs[row * Di + d];
            if (g) zn = xz[row * 2 * Di + Di + d];
        };
        if (on) fetch(s0);
        for (int t = s0; t < s1; ++t) {
            const float dtv = dtn, x = xn, z = zn;
            if (on && t + 1 < s1) fetch(t + 1);
            const float* bc = bc_s + (t - s0) * 2 * NSTATE;
            float yv = 0.f;
#pragma unroll
            for (int n = 0; n < NSTATE; ++n) {
                h[n] = exp2_hw(dtv * A2[n]) * h[n] + dtv * x * bc[n];
                yv += h[n] * bc[NSTATE + n];
            }
            yv += Dv * x;
            if (on) {
                y[(row0 + t) * Di + d] = yv;
                if (g) g[(row0 + t) * Di + d] = yv * silu_f(z);
            }
        }
    }
}

// Sums of 32 values (16 dB, 16 dC) over the 64 lanes of a wave by a
// transposing tree: at partner distance m = 32, 16, 8, 4, 2 every lane keeps
// the half of its values selected by its own bit m and adds the partner's copy
// of that half; lane l then holds index l >> 1 summed over the 32 lanes with
// its bit 0, and distance 1 completes the sum.  Fixed order: identical bits on
// every call.  Distances 32 and 16 are register-half swaps, the others DPP
// moves: no LDS permutes.
DEVI float pair_swap32(float a, float b) {       // lanes < 32: a + a'(lane + 32); others: b'(lane - 32) + b
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
DEVI float pair_swap16(float a, float b) {       // the same within each 32 lanes at distance 16
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
constexpr int DPP_ROR8 = 0x128, DPP_XOR3 = 0x1B;
// v[n] for n < 16: the values of distance 32 already combined (pair_swap32 of
// dB_n and dC_n)
DEVI float wave_sum32_tail(float (&v)[NSTATE], int lane) {
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = pair_swap16(v[j], v[8 + j]);
    {
        const bool hi = (lane & 8) != 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float keep = hi ? v[4 + j] : v[j], send = hi ? v[j] : v[4 + j];
            v[j] = keep + dpp_f<DPP_ROR8>(send);
        }
    }
    {
        const bool hi = (lane & 4) != 0;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const float keep = hi ? v[2 + j] : v[j], send = hi ? v[j] : v[2 + j];
            v[j] = keep + dpp_f<DPP_XOR3>(dpp_f<DPP_HALF_MIRROR>(send));      // 7 - i, then i ^ 3: i ^ 4
        }
    }
    const bool hi = (lane & 2) != 0;
    const float keep = hi ? v[1] : v[0], send = hi ? v[0] : v[1];
    const float w = keep + dpp_f<DPP_XOR2>(send);
    return w + dpp_f<DPP_XOR1>(w);
}

// Selective scan backward, blocks of TB steps in parallel (one wave per 64
// channels, up to four channel blocks per workgroup sharing B and C in LDS).
// Inside a block, half sub-blocks of SCAN_SUB / 2 steps run from the last to
// the first: their states h_{t-1} and exp(dt A) are recomputed into registers
// from the state kept at the sub-block's start (hsub; 8 steps of both would
// not fit the 256 registers of two waves per SIMD), then the reverse
// recurrence runs, starting from gh at the block's end (ghb).  dB and dC (sums over channels) are reduced within
// the wave and written as the channel block's partial pbc[block][row][32];
// dA_log and dD (sums over time) are written per (sequence, block) slot as
// pA[slot][d][n], pD[slot][d].  With dtr, dt = softplus(dtr): ddt receives the
// gradient of dtr, and pT[slot][d] its sum (the dt_proj bias).  VALU bound: about 26 instructions per state
// and step.  13 of its registers are spilled (52 B a thread) at two waves per SIMD.
__global__ __launch_bounds__(256, 2) void k_tr_scan_bwd(
    const float* __restrict__ xs, const float* __restrict__ dt, const float* __restrict__ dbc, int NO, int R,
    const float* __restrict__ A_log, const float* __restrict__ Dsk, const float* __restrict__ dy, long long rows, int Tn,
    int Di, int Tc, int NC, int TB, int nblk, const float* __restrict__ hsub, int nsub,
    const float* __restrict__ ghb, const float* __restrict__ dtr, float* __restrict__ dxs, float* __restrict__ ddt,
    float* __restrict__ pbc, float* __restrict__ pA, float* __restrict__ pD, float* __restrict__ pT) {
    __shared__ float4 A_s[NSTATE / 4][256];                  // -exp(A_log), read once per step
    extern __shared__ __align__(16) float bc_s[];            // [TB][32]
    const int b = blockIdx.z, tid = threadIdx.x, lane = tid & 63;
    const int cb = blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(tid >> 6);   // channel block
    const int d = cb * SCAN_CH + lane;
    const bool on = d < Di;
    const int c = blockIdx.y / nblk, k = blockIdx.y % nblk;
    const int ce = (c + 1) * Tc < Tn ? (c + 1) * Tc : Tn;
    const int t0 = c * Tc + k * TB, t1 = t0 + TB < ce ? t0 + TB : ce;
    const long long row0 = (long long)b * Tn;
    stage_bc(bc_s, dbc, row0, t0, t1, NO, R, tid, blockDim.x);
    __syncthreads();
    if (cb * SCAN_CH >= Di) return;
    const long long slot = (long long)b * gridDim.y + blockIdx.y;
    float gh[NSTATE], gA[NSTATE];
#pragma unroll
    for (int n = 0; n < NSTATE; ++n) {
        const float A = on ? -expf(A_log[d * NSTATE + n]) : 0.f;
        reinterpret_cast<float*>(&A_s[n / 4][tid])[n % 4] = A;
        gh[n] = on ? ghb[(slot * NSTATE + n) * Di + d] : 0.f;
        gA[n] = 0.f;
    }
    const float Dv = on ? Dsk[d] : 0.f;
    float gD = 0.f, gT = 0.f;
    constexpr int HS = SCAN_SUB / 2;
#pragma unroll 1
    for (int s = (t1 - t0 - 1) / HS; s >= 0; --s) {              // half sub-blocks
        // A is read again from LDS in every round (the compiler would otherwise
        // keep it in registers across the loop and spill)
        asm volatile("" ::: "memory");
        float A2[NSTATE];
#pragma unroll
        for (int n = 0; n < NSTATE; ++n) A2[n] = reinterpret_cast<const float*>(&A_s[n / 4][tid])[n % 4] * LOG2E_F;
        const int u0 = t0 + s * HS, nu = t1 - u0 < HS ? t1 - u0 : HS;
        const int v0 = t0 + (s / 2) * SCAN_SUB;                  // the state kept at v0 <= u0
        float hist[HS][NSTATE], av[HS][NSTATE], dv[HS], xv[HS], gv[HS], rv[HS];
        const float* hs = hsub + (scan_slot(b, NC, c, nsub, (v0 - c * Tc) / SCAN_SUB) * NSTATE) * Di + (on ? d : 0);
#pragma unroll
        for (int n = 0; n < NSTATE; ++n) hist[0][n] = on ? hs[(long long)n * Di] : 0.f;
#pragma unroll
        for (int j = 0; j < HS; ++j) {
            const bool in = on && j < nu;
            const long long at = (row0 + u0 + j) * Di + d;
            dv[j] = in ? dt[at] : 0.f;
            xv[j] = in ? xs[at] : 0.f;
            gv[j] = in ? dy[at] : 0.f;
            rv[j] = in && dtr ? dtr[at] : 0.f;
        }
        if (u0 > v0) {                                           // uniform: walk the first half without keeping it
            float dw[HS], xw[HS];
#pragma unroll
            for (int j = 0; j < HS; ++j) {
                const long long at = (row0 + v0 + j) * Di + d;
                dw[j] = on ? dt[at] : 0.f;
                xw[j] = on ? xs[at] : 0.f;
            }
#pragma unroll
            for (int j = 0; j < HS; ++j) {
                const float* bc = bc_s + (v0 - t0 + j) * 2 * NSTATE;
#pragma unroll
                for (int n = 0; n < NSTATE; ++n)
                    hist[0][n] = exp2_hw(dw[j] * A2[n]) * hist[0][n] + dw[j] * xw[j] * bc[n];
            }
        }
#pragma unroll
        for (int j = 0; j < HS; ++j) {
            const float* bc = bc_s + (u0 - t0 + (j < nu ? j : 0)) * 2 * NSTATE;
#pragma unroll
            for (int n = 0; n < NSTATE; ++n) {
                av[j][n] = exp2_hw(dv[j] * A2[n]);
                if (j + 1 < HS) hist[j + 1 < HS ? j + 1 : 0][n] = av[j][n] * hist[j][n] + dv[j] * xv[j] * bc[n];
            }
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int j = HS - 1; j >= 0; --j) {
            if (j >= nu) continue;                               // uniform
            const long long row = row0 + u0 + j;
            const float dtv = dv[j], x = xv[j], g = gv[j];
            const float* bc = bc_s + (u0 - t0 + j) * 2 * NSTATE;
            float pv[NSTATE];
            float ddt_v = 0.f, dx_v = 0.f;
#pragma unroll
            for (int n = 0; n < NSTATE; ++n) {
                const float Bn = bc[n], Cn = bc[NSTATE + n], hp = hist[j][n];
                const float a = av[j][n], A = reinterpret_cast<const float*>(&A_s[n / 4][tid])[n % 4];
                const float ht = a * hp + dtv * x * Bn;
                gh[n] += Cn * g;
                const float ga = gh[n] * hp;
                ddt_v += ga * a * A + gh[n] * x * Bn;
                gA[n] += ga * a * dtv;
                dx_v += gh[n] * dtv * Bn;
                // lanes past Di hold zeros throughout (dt, x, dy, h)
                pv[n] = pair_swap32(gh[n] * dtv * x, g * ht);
                gh[n] *= a;
            }
            dx_v += Dv * g;
            gD += g * x;
            if (dtr) {                                           // through dt = softplus(dtr)
                ddt_v = rv[j] > 20.0f ? ddt_v : ddt_v / (1.0f + expf(-rv[j]));
                gT += ddt_v;
            }
            if (on) { ddt[row * Di + d] = ddt_v; dxs[row * Di + d] = dx_v; }
            // dB (index n) and dC (index 16 + n) of this row over the wave's 64 channels
            const float v = wave_sum32_tail(pv, lane);
            if ((lane & 1) == 0) pbc[((long long)cb * rows + row) * 2 * NSTATE + (lane >> 1)] = v;
        }
    }
    if (on) {
#pragma unroll
        for (int n = 0; n < NSTATE; ++n)
            pA[(slot * Di + d) * NSTATE + n] = gA[n] * reinterpret_cast<const float*>(&A_s[n / 4][tid])[n % 4];
        pD[slot * Di + d] = gD;
        if (dtr) pT[slot * Di + d] = gT;
    }
}

// dB, dC of every row: the channel blocks' partials added in block order,
// written into columns R .. R + 31 of ddbc (row stride NO)
__global__ void k_tr_dbc_reduce(const float* __restrict__ pbc, int nblk, long long rows, float* __restrict__ ddbc,
                                int NO, int R) {
    long long i = blockIdx.x * 256LL + threadIdx.x;
    if (i >= rows * 2 * NSTATE) return;
    const long long row = i / (2 * NSTATE);
    const int c = (int)(i % (2 * NSTATE));
    float v = pbc[i];
    for (int k = 1; k < nblk; ++k) v += pbc[(long long)k * rows * 2 * NSTATE + i];
    ddbc[row * NO + R + c] = v;
}

// softmax cross-entropy: rowloss[row] = -log p(target); dlogits = (p - onehot) / ntok
__global__ void k_tr_ce(float* __restrict__ logits, const float* __restrict__ bias, const uint8_t* __restrict__ tok,
                        int B, int T, float* __restrict__ rowloss, float inv_ntok) {
    const int Tn = T - 1;
    long long row = blockIdx.x * 4LL + threadIdx.y;
    if (row >= (long long)B * Tn) return;
    int lane = threadIdx.x;
    int b = (int)(row / Tn), t = (int)(row % Tn);
    int tgt = tok[(long long)b * T + t + 1];
    float* lr = logits + row * 256;
    float l[4];
    for (int i = 0; i < 4; ++i) l[i] = lr[4 * lane + i] + bias[4 * lane + i];
    float m = wave_max(fmaxf(fmaxf(l[0], l[1]), fmaxf(l[2], l[3])));
    float e[4], zs = 0.f;
    for (int i = 0; i < 4; ++i) { e[i] = expf(l[i] - m); zs += e[i]; }
    zs = wave_sum(zs);
    float lse = m + logf(zs);
    for (int i = 0; i < 4; ++i) {
        int a = 4 * lane + i;
        float p = e[i] / zs;
        lr[a] = (p - (a == tgt ? 1.0f : 0.0f)) * inv_ntok;
        if (a == tgt) rowloss[row] = lse - l[i];
    }
}

// per-block partial sums of g^2 over a fixed element range (thread-strided,
// then the wave tree, then the 4 waves in order)
__global__ __launch_bounds__(256) void k_sqsum_part(const float* __restrict__ g, long long n, long long per,
                                                    float* __restrict__ part) {
    __shared__ float w4[4];
    const long long i0 = blockIdx.x * per, i1 = i0 + per < n ? i0 + per : n;
    float acc = 0.f;
    for (long long i = i0 + threadIdx.x; i < i1; i += 256) acc += g[i] * g[i];
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) w4[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = ((w4[0] + w4[1]) + w4[2]) + w4[3];
}

// AdamW with decoupled weight decay and global-norm clipping (norm^2 in *sq)
__global__ void k_adamw(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m,
                        float* __restrict__ v, long long n, float lr, float b1, float b2, float eps, float wd,
                        float bc1, float bc2, float clip, const float* __restrict__ sq) {
    long long i = blockIdx.x * 256LL + threadIdx.x;
    if (i >= n) return;
    float nrm = sqrtf(*sq);
    float sc = clip > 0.f && nrm > clip ? clip / (nrm + 1e-6f) : 1.0f;
    float gi = g[i] * sc;
    float wi = w[i] * (1.0f - lr * wd);
    float mi = b1 * m[i] + (1.0f - b1) * gi;
    float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] = wi - lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

// ============================================================ host side
inline unsigned blocks(long long n, int per = 256) { return (unsigned)((n + per - 1) / per); }

struct Buf {
    void* p = nullptr;
    size_t n = 0;
    Buf() = default;
    Buf(const Buf&) = delete;
    Buf& operator=(const Buf&) = delete;
    Buf(Buf&& o) noexcept : p(o.p), n(o.n) { o.p = nullptr; o.n = 0; }
    ~Buf() { if (p) (void)hipFree(p); }
    hipError_t alloc(size_t b) {
        if (p) { (void)hipFree(p); p = nullptr; }
        n = b;
        return hipMalloc(&p, b ? b : 4);
    }
    // grow only: keeps the allocation when it is large enough
    hipError_t ensure(size_t b) { return (p && n >= b) ? hipSuccess : alloc(b); }
    float* f() const { return static_cast<float*>(p); }
};

// Number of row slices of a fixed-order row reduction (a function of the
// row count only, so the summation order never depends on anything else).
long long row_slices(long long rows, long long max_slices = 256, long long min_rows = 64) {
    long long s = (rows + min_rows - 1) / min_rows;
    return std::max(1LL, std::min(s, max_slices));
}

// GEMM splits: the reduction (K) is split when the output has too few tiles
// to fill the GPU; the split count depends on the shape only.
int gemm_splits(int M, int N, long long K) {
    const long long tiles = (long long)((M + TG_BM - 1) / TG_BM) * ((N + TG_BN - 1) / TG_BN);
    if (tiles >= 1024 || K <= 4 * TG_BK) return 1;
    long long s = (2048 + tiles - 1) / tiles;
    s = std::min(s, (K + 255) / 256);
    return (int)std::max(1LL, s);
}

size_t gemm_ws_floats(int M, int N, long long K) {
    const int S = gemm_splits(M, N, K);
    return S > 1 ? (size_t)S * M * N : 0;
}

}  // namespace

// States of the forward scan that a training call keeps for its backward pass:
// every SCAN_SUB steps (2 d_inner floats a row) in the layers from `fine` on, and
// every `every` steps in the others, whose backward pass makes the closer ones
// again in one buffer of a layer.  All layers keep the close ones while these take
// no more than L + 3 d_inner floats a row; else as many as that leaves beside the
// one buffer, so that a deep model's batch stays within what it takes with states
// every chunk_t steps (16 layers: 19 d_inner floats a row instead of 32).  chunk_t up to
// SCAN_SUB asks for all of them.
struct KeptStates {
    int every = SCAN_SUB, fine = 0;
    static KeptStates of(int L, int Tc) {
        KeptStates k;
        k.every = (Tc + SCAN_SUB - 1) / SCAN_SUB * SCAN_SUB;
        if (k.every > SCAN_SUB && 2 * L > L + 3) k.fine = L - (L + 1) / 2;
        return k;
    }
};

// Training context kept on the model: optimizer moments, step count, the
// activation and gradient buffers of the last (B, T) shape, and scratch.
struct TrainCtx {
    Buf m, v, grad, sqpart, sq;
    long long step = 0;
    // activations (per layer) and backward temporaries, sized for rows x widths
    int B = 0, T = 0, Tc = 0;
    KeptStates kept;
    std::vector<Buf> rin, a, st, xz, xs, dbc, dtr, dt, y, g, hs;
    std::vector<Buf> fr, fu, fg, ff, fst;   // feed-forward: input r, W1 r + b1, GELU of it, W2 . + b2, LN stats
    Buf hsub;                               // fine states of one layer (KeptStates)
    Buf fdu;                                // feed-forward backward: gradient of the hidden row
    Buf wf;                                 // prepared weight matrices of the step
    Buf rfin, rf, stf, logits, rowloss;
    Buf dr, tmp, dyb, dxz, ddbc, ddtr, dxs, ghb, pbc, pA, pD, pT, part, gws;
};

void train_ctx_free(void* p) { delete static_cast<TrainCtx*>(p); }

#define TCHK(expr) do { hipError_t e_ = (expr); if (e_ != hipSuccess) { err = std::string(#expr) + ": " + hipGetErrorString(e_); return BOA_E_DEVICE; } } while (0)

namespace {
// C[M, N] (+)= A . B on k_tg (see above); ws holds split partials
hipError_t gemm(int dt, const float* A, long long sam, long long sak, const float* B, long long sbk, long long sbn,
                int M, int N, long long K, float* C, long long ldc, int accumulate, float* ws, hipStream_t s) {
    if (M <= 0 || N <= 0) return hipSuccess;
    const int S = gemm_splits(M, N, K);
    long long kspan = (K + S - 1) / S;
    kspan = (kspan + TG_BK - 1) / TG_BK * TG_BK;
    dim3 grid((N + TG_BN - 1) / TG_BN, (M + TG_BM - 1) / TG_BM, S);
    float* out = S > 1 ? ws : C;
    const long long ld = S > 1 ? N : ldc;
    const int acc = S > 1 ? 0 : accumulate;
    const bool ak = sak == 1, bk = sbk == 1;
#define TG_LAUNCH(DT, AKV, BKV)                                                                                 \
    hipLaunchKernelGGL((k_tg<DT, AKV, BKV>), grid, dim3(256), 0, s, A, sam, sak, B, sbk, sbn, M, N, K, kspan, \
                       out, ld, (long long)M * N, acc)
    if (dt == 0) {
        if (ak && bk) TG_LAUNCH(0, true, true);
        else if (ak) TG_LAUNCH(0, true, false);
        else if (bk) TG_LAUNCH(0, false, true);
        else TG_LAUNCH(0, false, false);
    } else {
        if (ak && bk) TG_LAUNCH(1, true, true);
        else if (ak) TG_LAUNCH(1, true, false);
        else if (bk) TG_LAUNCH(1, false, true);
        else TG_LAUNCH(1, false, false);
    }
#undef TG_LAUNCH
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || S == 1) return e;
    hipLaunchKernelGGL(k_sum_slices_2d, dim3(blocks((long long)M * N)), dim3(256), 0, s, ws, S, M, N, C, ldc,
                       accumulate);
    return hipGetLastError();
}

// Columns of k_trow for a reduction of K: the next size it is built for, or 0.
int trow_kp(int K) {
    if (K <= 32) return 32;
    if (K <= 64) return 64;
    for (int kp : {128, 256, 512, 1024, 2048})
        if (K == kp) return kp;
    return 0;
}
template <int DT, int EPI, int KP, int BM, int FN>
hipError_t trow_launch(const TRow& p, hipStream_t s) {
    const size_t lds = (size_t)BM * (DT == 0 ? (KP + 4) * 4 : (KP + 8) * 2);
    auto kern = k_trow<DT, EPI, KP, BM, FN>;
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3((p.M + BM - 1) / BM), dim3(256), lds, s, p);
    return hipGetLastError();
}
template <int DT, int EPI, int KP>
hipError_t trow_epi_launch(const TRow& p, hipStream_t s) {
    constexpr int BM = KP <= 256 ? 64 : (KP * (DT == 0 ? 2 : 1) <= 1024 ? 32 : 16);
    const bool wide = p.N > 192;
    if constexpr (BM > 16) {
        if (p.span == 0 && p.M >= 256 * BM)
            return wide ? trow_launch<DT, EPI, KP, BM, 4>(p, s) : trow_launch<DT, EPI, KP, BM, 1>(p, s);
    }
    return wide ? trow_launch<DT, EPI, KP, 16, 4>(p, s) : trow_launch<DT, EPI, KP, 16, 1>(p, s);
}
// the epilogues that a reduction of KP occurs with: 2 with K = dt_rank, 3 with
// K = d_model, 1 with K = d_inner or dt_rank + 32
template <int DT, int KP>
hipError_t trow_kp_launch(const TRow& p, hipStream_t s) {
    if constexpr (KP > 32) {
        if (p.epi == 0) return trow_epi_launch<DT, 0, KP>(p, s);
    }
    if constexpr (KP >= 64 && KP <= 1024) {
        if (p.epi == 1) return trow_epi_launch<DT, 1, KP>(p, s);
    }
    if constexpr (KP == 32) {
        if (p.epi == 2) return trow_epi_launch<DT, 2, KP>(p, s);
    }
    if constexpr (KP >= 64 && KP <= 512) {
        if (p.epi == 3) return trow_epi_launch<DT, 3, KP>(p, s);
    }
    return hipErrorInvalidValue;
}
// p.W prepared with trow_kp(p.K) columns
hipError_t trow(int dt, TRow p, hipStream_t s) {
    const int S = gemm_splits(p.M, p.N, p.K);
    // f32 operands are not rounded again, so their sums may be taken in one chain
    p.span = dt == 1 && S > 1 ? ((p.K + S - 1) / S + TG_BK - 1) / TG_BK : 0;
#define TROW_K(KPV) case KPV: return dt == 0 ? trow_kp_launch<0, KPV>(p, s) : trow_kp_launch<1, KPV>(p, s);
    switch (trow_kp(p.K)) {
        TROW_K(32) TROW_K(64) TROW_K(128) TROW_K(256) TROW_K(512) TROW_K(1024) TROW_K(2048)
        default: return hipErrorInvalidValue;
    }
#undef TROW_K
}

// Slices of a weight gradient's rows: one workgroup per tile and slice, 256 in
// all (each of 8 waves with a quarter of a CU's registers per wave), but at
// least 128 rows per slice.
struct WCut {
    int TA, TB, S;
    long long per;
};
WCut wgrad_cut(int N, int K, long long rows) {
    WCut q;
    q.TA = N <= 64 ? 64 : 256;
    q.TB = N > 64 && K <= 64 ? 64 : 256;
    const long long tiles = (long long)((N + q.TA - 1) / q.TA) * ((K + q.TB - 1) / q.TB);
    long long S = std::max(1LL, std::min(256 / tiles, (rows + 127) / 128));
    if (S > 8) S = S / 8 * 8;
    q.per = ((rows + S - 1) / S + 31) / 32 * 32;
    q.S = (int)((rows + q.per - 1) / q.per);
    return q;
}
// dW [N][K] = dY^T X over the rows (N, K and both strides multiples of 4)
hipError_t wgrad(int dt, const float* dY, int ldy, const float* X, int ldx, int N, int K, float* dW, long long rows,
                 float* ws, hipStream_t s) {
    const WCut q = wgrad_cut(N, K, rows);
    const dim3 grid(q.S, ((N + q.TA - 1) / q.TA) * ((K + q.TB - 1) / q.TB));
    float* out = q.S > 1 ? ws : dW;
#define TGW(DT, A, B) \
    hipLaunchKernelGGL((k_tg_w<DT, A, B>), grid, dim3(512), 0, s, dY, (long long)ldy, N, X, (long long)ldx, K, rows, q.per, out)
    if (dt == 0) {
        if (q.TA == 64) TGW(0, 64, 256);
        else if (q.TB == 64) TGW(0, 256, 64);
        else TGW(0, 256, 256);
    } else {
        if (q.TA == 64) TGW(1, 64, 256);
        else if (q.TB == 64) TGW(1, 256, 64);
        else TGW(1, 256, 256);
    }
#undef TGW
    if (q.S > 1)
        hipLaunchKernelGGL(k_sum_slices, dim3(blocks((long long)N * K, 64)), dim3(256), 0, s, ws, q.S, (long long)N * K,
                           (long long)N * K, dW, 0);
    return hipGetLastError();
}

// out[n] = column sums over the rows of X[:, n], n < N (fixed row slices)
hipError_t colsum(const float* X, long long rows, int ld, int N, float* part, float* out, hipStream_t s) {
    const long long S = row_slices(rows);
    const long long per = (rows + S - 1) / S;
    hipLaunchKernelGGL(k_colsum_part, dim3(blocks(N), (unsigned)S), dim3(256), 0, s, X, rows, ld, N, per, part);
    hipLaunchKernelGGL(k_sum_slices, dim3(blocks(N, 64)), dim3(256), 0, s, part, (int)S, (long long)N, (long long)N, out,
                       0);
    return hipGetLastError();
}
void ln_fwd(const float* x, long long rows, int D, const float* w, const float* b, float* out, float* st, hipStream_t s) {
    const dim3 g(blocks(rows, 4)), t(256);
    switch (D) {
        case 64: hipLaunchKernelGGL(k_tr_ln_fwd<1>, g, t, 0, s, x, rows, w, b, out, st); break;
        case 128: hipLaunchKernelGGL(k_tr_ln_fwd<2>, g, t, 0, s, x, rows, w, b, out, st); break;
        case 256: hipLaunchKernelGGL(k_tr_ln_fwd<4>, g, t, 0, s, x, rows, w, b, out, st); break;
        default: hipLaunchKernelGGL(k_tr_ln_fwd<8>, g, t, 0, s, x, rows, w, b, out, st); break;      // 512
    }
}
// dx (+)= the LayerNorm's input gradient; gwb [2][D] = its weight and bias gradients
void ln_bwd(const float* dy, const float* x, const float* st, long long rows, int D, const float* w, float* dx,
            int accumulate, float* part, float* gwb, hipStream_t s) {
    const long long S = row_slices(rows, 1024, 16), per = (rows + S - 1) / S;
    const dim3 g((unsigned)S), t(256);
    switch (D) {
        case 64: hipLaunchKernelGGL(k_tr_ln_bwd<1>, g, t, 0, s, dy, x, st, rows, per, w, dx, accumulate, part); break;
        case 128: hipLaunchKernelGGL(k_tr_ln_bwd<2>, g, t, 0, s, dy, x, st, rows, per, w, dx, accumulate, part); break;
        case 256: hipLaunchKernelGGL(k_tr_ln_bwd<4>, g, t, 0, s, dy, x, st, rows, per, w, dx, accumulate, part); break;
        default: hipLaunchKernelGGL(k_tr_ln_bwd<8>, g, t, 0, s, dy, x, st, rows, per, w, dx, accumulate, part); break;
    }
    hipLaunchKernelGGL(k_sum_slices, dim3(blocks(2 * D, 64)), dim3(256), 0, s, part, (int)S, 2LL * D, 2LL * D, gwb, 0);
}

// scratch floats the fixed-order row reductions need
size_t part_floats(int B, int Tn, int D, int Di, int H) {
    const long long rows = (long long)B * Tn, S = row_slices(rows);
    const size_t conv = (size_t)B * ((Tn + CONV_TS - 1) / CONV_TS) * Di * (KCONV + 1);
    return std::max<size_t>({(size_t)S * VOCAB * D, (size_t)S * std::max(H, 256), conv,
                             (size_t)row_slices(rows, 1024, 16) * 2 * D});
}

// The prepared weight matrices of a training step: per layer in_proj, x_proj,
// dt_proj, out_proj and their transposes (for the input gradients), with the
// feed-forward sub-layer W1, W2 and theirs; then the head and its transpose.
enum { WF_IN, WF_X, WF_DT, WF_OUT, WF_OUT_T, WF_DT_T, WF_X_T, WF_IN_T, WF_W1, WF_W2, WF_W2_T, WF_W1_T };
struct WMat {
    const float* w;                   // X(n, k) = w[n sn + k sk]
    int sn, sk, N, K;
    size_t at;                        // byte offset of the prepared copy
    size_t bytes(int dt) const {
        const int kp = trow_kp(K);
        return kp ? (size_t)((N + 63) / 64 * 64) * kp * (dt == 0 ? 4 : 2) : 0;
    }
};
// matrices of layer l (l == L: the head and its transpose), placed from *at on
std::vector<WMat> layer_mats(const Layout& L, const float* w, int l, int dt, size_t* at) {
    const int D = L.D, Di = L.Di, R = L.R, NO = R + 2 * NSTATE, H = L.H;
    std::vector<WMat> v;
    auto add = [&](uint64_t off, int N, int K, bool t) {     // stored [N][K]; t: the transpose
        WMat m{w + off, t ? 1 : K, t ? K : 1, t ? K : N, t ? N : K, *at};
        *at += (m.bytes(dt) + 255) / 256 * 256;
        v.push_back(m);
    };
    if (l == L.L) {
        add(L.head_w, 256, D, false);
        add(L.head_w, 256, D, true);
        return v;
    }
    const LayerOff& o = L.layer[l];
    add(o.in_w, 2 * Di, D, false);
    add(o.xw, NO, Di, false);
    add(o.dtw, Di, R, false);
    add(o.out_w, D, Di, false);
    add(o.out_w, D, Di, true);
    add(o.dtw, Di, R, true);
    add(o.xw, NO, Di, true);
    add(o.in_w, 2 * Di, D, true);
    if (H) {
        add(o.ffn_w1, H, D, false);
        add(o.ffn_w2, D, H, false);
        add(o.ffn_w2, D, H, true);
        add(o.ffn_w1, H, D, true);
    }
    return v;
}
size_t wfrag_bytes(const Layout& L) {                        // FP32 copies are the larger ones
    size_t at = 0;
    for (int l = 0; l <= L.L; ++l) (void)layer_mats(L, nullptr, l, 0, &at);
    return at;
}
hipError_t prep_mats(const std::vector<WMat>& v, int dt, uint8_t* base, hipStream_t s) {
    FragJobs jobs{};
    int n = 0;
    for (const WMat& m : v)
        if (const int kp = trow_kp(m.K))
            jobs.j[n++] = FragJob{m.w, base + m.at, m.sn, m.sk, m.N, m.K, (m.N + 63) / 64 * 64, kp};
    if (dt == 0) hipLaunchKernelGGL(k_tr_frags<0>, dim3(128, n), dim3(256), 0, s, jobs);
    else hipLaunchKernelGGL(k_tr_frags<1>, dim3(128, n), dim3(256), 0, s, jobs);
    return hipGetLastError();
}
// Y = X . W^T for the prepared matrix (epi and its operands as in TRow; a
// reduction k_trow is not built for, a feed-forward width, goes to k_tg)
hipError_t lin(int dt, const WMat& m, const uint8_t* base, const float* X, int lx, long long rows, float* Y, int ly,
               TRow p, float* ws, hipStream_t s) {
    if (!trow_kp(m.K))
        return p.epi > 1 ? hipErrorInvalidValue
                         : gemm(dt, X, lx, 1, m.w, m.sk, m.sn, (int)rows, m.N, m.K, Y, ly, p.epi, ws, s);
    p.A = X;
    p.lda = lx;
    p.M = (int)rows;
    p.K = m.K;
    p.N = m.N;
    p.W = base + m.at;
    p.C = Y;
    p.ldc = ly;
    return trow(dt, p, s);
}

// ------------------------------------------------------------ selective scan launches
// How a backward scan is cut: blocks of TB steps inside each of the NC chunks.
struct ScanCut {
    int Tc, NC, nsub, TB, nblk, NBS;
};
// Blocks of 256 steps read the boundary states least; shorter ones are taken
// until there are 4096 waves (four per SIMD) or the block is 32 steps, where
// the 16 exponentials of a wave's start begin to show.
int scan_blocks(int Tn, int Tc, int NC, int TB) {                // of one sequence
    return (NC - 1) * ((Tc + TB - 1) / TB) + (Tn - (NC - 1) * Tc + TB - 1) / TB;
}
ScanCut scan_cut(int B, int Tn, int Di, int Tc) {
    ScanCut q;
    q.Tc = std::min(Tc, Tn);
    q.NC = (Tn + q.Tc - 1) / q.Tc;
    q.nsub = (q.Tc + SCAN_SUB - 1) / SCAN_SUB;
    const long long dblk = (Di + SCAN_CH - 1) / SCAN_CH;
    for (q.TB = 256; q.TB > 32 && dblk * B * scan_blocks(Tn, q.Tc, q.NC, q.TB) < 4096; q.TB /= 2) {}
    q.nblk = (q.Tc + q.TB - 1) / q.TB;
    q.NBS = scan_blocks(Tn, q.Tc, q.NC, q.TB);
    return q;
}
size_t scan_hsub_floats(const ScanCut& q, int B, int Di) { return (size_t)B * q.NC * q.nsub * NSTATE * Di; }
size_t scan_block_floats(const ScanCut& q, int B, int Di) { return (size_t)B * q.NBS * NSTATE * Di; }

// States every `sub` steps (and every Tsave steps into hsave): one state per
// thread when one workgroup per channel block would leave compute units idle
// (5 x 776 steps, d_inner 128: 43 us with one state per thread, 73 us with four;
// with 256 workgroups and more the four-state form reads dt and x once instead of
// four times).
hipError_t scan_states(const float* x, const float* dt, const float* dbc, int NO, int R, const float* A_log, int B,
                       int Tn, int Di, int Tc, int NC, const float* h0, int h0n, int h0s, float* hsub, int sub,
                       int nsub, int nseq, float* hsave, int Tsave, hipStream_t s) {
    const int dblk = (Di + SCAN_CH - 1) / SCAN_CH, nsave = hsave ? (Tn + Tsave - 1) / Tsave : 0;
    const bool few = (long long)dblk * NC * B < 256, al = sub % 8 == 0 && (!hsave || Tsave % 8 == 0);
#define STATES(NPT, AL) hipLaunchKernelGGL((k_tr_states<NPT, AL>), dim3(dblk * (4 / NPT), NC, B), dim3(256), 0, s, x, \
                                           dt, dbc, NO, R, A_log, Tn, Di, Tc, NC, h0, h0n, h0s, hsub, sub, nsub, nseq, hsave, Tsave, nsave)
    if (few && al) STATES(1, true);
    else if (few) STATES(1, false);
    else if (al) STATES(4, true);
    else STATES(4, false);
#undef STATES
    return hipGetLastError();
}
// Outputs from states kept every `sub` steps (nslot per sequence): blocks of
// at least SCAN_FWD_BLOCK steps.
hipError_t scan_y(const float* x, const float* dt, const float* dbc, int NO, int R, const float* A_log,
                  const float* Dsk, const float* xz, int B, int Tn, int Di, const float* hsub, int sub, int nslot,
                  float* y, float* g, hipStream_t s) {
    const int per = (SCAN_FWD_BLOCK + sub - 1) / sub, TB = per * sub;
    const int nt = std::min(256, (Di + 63) / 64 * 64);
    hipLaunchKernelGGL(k_tr_scan_y, dim3((Di + nt - 1) / nt, (Tn + TB - 1) / TB, B), dim3(nt), 0, s, x, dt, dbc, NO, R,
                       A_log, Dsk, xz, Tn, Di, TB, nslot, per, hsub, y, g);
    return hipGetLastError();
}
// The adjoint states at the ends of the blocks (scan_block_floats floats).
hipError_t scan_gstates(const float* dt, const float* dbc, int NO, int R, const float* A_log, const float* dy, int B,
                        int Tn, int Di, const ScanCut& q, float* ghb, hipStream_t s) {
    const int dblk = (Di + SCAN_CH - 1) / SCAN_CH;
    const bool few = (long long)dblk * B < 256, al = q.NC == 1 || q.Tc % 8 == 0;
#define GSTATES(NPT, AL) hipLaunchKernelGGL((k_tr_gstates<NPT, AL>), dim3(dblk * (4 / NPT), 1, B), dim3(256), 0, s, dt, \
                                            dbc, NO, R, A_log, dy, Tn, Di, q.Tc, q.NC, q.TB, q.nblk, q.NBS, ghb)
    if (few && al) GSTATES(1, true);
    else if (few) GSTATES(1, false);
    else if (al) GSTATES(4, true);
    else GSTATES(4, false);
#undef GSTATES
    return hipGetLastError();
}
// Gradients from the states of every SCAN_SUB steps and from the adjoint states;
// pbc, pA, pD and pT are the partial sums (scan_block_floats floats for pA, a 16th of
// it for pD and pT).
hipError_t scan_grads(const float* x, const float* dt, const float* dbc, int NO, int R, const float* A_log,
                      const float* Dsk, const float* dy, int B, int Tn, int Di, const ScanCut& q, const float* hsub,
                      const float* ghb, const float* dtr, float* dx, float* ddt, float* pbc, float* pA, float* pD,
                      float* pT, hipStream_t s) {
    const int dblk = (Di + SCAN_CH - 1) / SCAN_CH, w = std::min(4, dblk);
    hipLaunchKernelGGL(k_tr_scan_bwd, dim3((dblk + w - 1) / w, q.NBS, B), dim3(64 * w),
                       (size_t)q.TB * 2 * NSTATE * sizeof(float), s, x, dt, dbc, NO, R, A_log, Dsk, dy, (long long)B * Tn,
                       Tn, Di, q.Tc, q.NC, q.TB, q.nblk, hsub, q.nsub, ghb, dtr, dx, ddt, pbc, pA, pD, pT);
    return hipGetLastError();
}
}  // namespace

// Sizes the context's buffers for B sequences of T bytes and chunk length Tc.
int train_ensure_buffers(boa_model* m, int B, int T, int Tc, std::string& err) {
    TrainCtx* c = static_cast<TrainCtx*>(m->train);
    if (c->B == B && c->T == T && c->Tc == Tc) return BOA_OK;
    const Layout& L = m->lay;
    const int D = L.D, Di = L.Di, NO = L.R + 2 * NSTATE, Tn = T - 1;
    const size_t rows = (size_t)B * Tn, F = sizeof(float);
    const int dblk = (Di + SCAN_CH - 1) / SCAN_CH;
    const ScanCut q = scan_cut(B, Tn, Di, Tn);
    const KeptStates kept = KeptStates::of(L.L, std::min(Tc, Tn));
    c->B = c->T = c->Tc = 0;
    c->rin.resize(L.L); c->a.resize(L.L); c->st.resize(L.L); c->xz.resize(L.L); 
    c->xs.resize(L.L); c->dbc.resize(L.L); c->dtr.resize(L.L); c->dt.resize(L.L); c->y.resize(L.L);
    c->g.resize(L.L); c->hs.resize(L.L);
    if (L.H) {
        c->fr.resize(L.L); c->fu.resize(L.L); c->fg.resize(L.L); c->ff.resize(L.L); c->fst.resize(L.L);
        for (int l = 0; l < L.L; ++l) {
            TCHK(c->fr[l].ensure(rows * D * F)); TCHK(c->fu[l].ensure(rows * L.H * F));
            TCHK(c->fg[l].ensure(rows * L.H * F)); TCHK(c->ff[l].ensure(rows * D * F));
            TCHK(c->fst[l].ensure(rows * 2 * F));
        }
        TCHK(c->fdu.ensure(rows * L.H * F));
    }
    for (int l = 0; l < L.L; ++l) {
        TCHK(c->rin[l].ensure(rows * D * F)); TCHK(c->a[l].ensure(rows * D * F)); TCHK(c->st[l].ensure(rows * 2 * F));
        TCHK(c->xz[l].ensure(rows * 2 * Di * F));
        TCHK(c->xs[l].ensure(rows * Di * F)); TCHK(c->dbc[l].ensure(rows * NO * F));
        TCHK(c->dtr[l].ensure(rows * Di * F)); TCHK(c->dt[l].ensure(rows * Di * F));
        TCHK(c->y[l].ensure(rows * Di * F)); TCHK(c->g[l].ensure(rows * Di * F));
        TCHK(c->hs[l].ensure((l < kept.fine ? (size_t)B * ((Tn + kept.every - 1) / kept.every) * NSTATE * Di
                                            : scan_hsub_floats(q, B, Di)) * F));
    }
    if (kept.fine) TCHK(c->hsub.ensure(scan_hsub_floats(q, B, Di) * F));
    TCHK(c->wf.ensure(wfrag_bytes(L)));
    TCHK(c->rfin.ensure(rows * D * F));
    TCHK(c->rf.ensure(rows * D * F)); TCHK(c->stf.ensure(rows * 2 * F)); TCHK(c->logits.ensure(rows * 256 * F));
    TCHK(c->rowloss.ensure(rows * F));
    TCHK(c->dr.ensure(rows * D * F)); TCHK(c->tmp.ensure(rows * D * F));
    TCHK(c->dyb.ensure(rows * Di * F)); TCHK(c->dxz.ensure(rows * 2 * Di * F));
    TCHK(c->ddbc.ensure(rows * NO * F)); TCHK(c->ddtr.ensure(rows * Di * F));
    TCHK(c->dxs.ensure(rows * Di * F));
    TCHK(c->ghb.ensure(scan_block_floats(q, B, Di) * F));
    TCHK(c->pbc.ensure((size_t)dblk * rows * 2 * NSTATE * F));
    TCHK(c->pA.ensure(scan_block_floats(q, B, Di) * F)); TCHK(c->pD.ensure(scan_block_floats(q, B, Di) / NSTATE * F));
    TCHK(c->pT.ensure(scan_block_floats(q, B, Di) / NSTATE * F));
    TCHK(c->part.ensure(part_floats(B, Tn, D, Di, L.H) * F));
    // split partials of the weight-gradient GEMMs (the largest of the shapes used)
    size_t ws = 0;
    const long long R = (long long)rows;
    const int Hs = L.H ? L.H : D;
    for (int N : {2 * Di, NO, Di, D, 256, Hs})        // weight gradients [N, K] over the rows
        for (int K : {D, Di, L.R, Hs}) ws = std::max(ws, (size_t)wgrad_cut(N, K, R).S * N * K);
    for (int N : {2 * Di, NO, Di, D, 256, L.R, Hs})   // forward and input gradients of few rows
        for (int K : {D, Di, L.R, 2 * Di, NO, 256, Hs}) ws = std::max(ws, gemm_ws_floats((int)R, N, K));
    TCHK(c->gws.ensure(std::max<size_t>(ws, 1) * F));
    c->B = B; c->T = T; c->Tc = Tc;
    c->kept = kept;
    return BOA_OK;
}

// Standalone selective scan (autograd binding): B and C packed as [rows][32].
int scan_fwd(const float* x, const float* dt, const float* A_log, const float* bc, const float* Dsk, int B, int T,
             int Di, int Tc, float* y, float* hsave, hipStream_t s, std::string& err) {
    Tc = std::min(Tc, T);
    // the states the caller keeps also start the blocks of the output pass,
    // unless they lie so far apart that few blocks would run
    Buf fine;
    const int sub = Tc <= 256 ? Tc : 64, nslot = (T + sub - 1) / sub;
    float* hsub = hsave;
    if (sub != Tc) {
        TCHK(fine.alloc((size_t)B * nslot * NSTATE * Di * sizeof(float)));
        hsub = fine.f();
    }
    TCHK(scan_states(x, dt, bc, 2 * NSTATE, 0, A_log, B, T, Di, T, 1, nullptr, 1, 1, hsub, sub, nslot, nslot,
                     sub != Tc ? hsave : nullptr, Tc, s));
    TCHK(scan_y(x, dt, bc, 2 * NSTATE, 0, A_log, Dsk, nullptr, B, T, Di, hsub, sub, nslot, y, nullptr, s));
    TCHK(hipStreamSynchronize(s));
    return BOA_OK;
}
// How the backward scan of a call is cut for its scratch memory: `seqs` sequences
// at a time and, one at a time, `chunks` of their chunks.
struct BwdPart {
    int seqs, chunks;
};
size_t bwd_floats(const ScanCut& q, int seqs, int chunks, int T, int Di) {
    const long long rows = (long long)seqs * (chunks == q.NC ? T : chunks * q.Tc);
    return (size_t)seqs * chunks * q.nsub * NSTATE * Di + (size_t)(Di + SCAN_CH - 1) / SCAN_CH * rows * 2 * NSTATE +
           scan_block_floats(q, seqs, Di) * 2 + scan_block_floats(q, seqs, Di) / NSTATE + 5 * 64;
}
// Within the memory of one chunk's states of every sequence and the partial sums
// of every row (256 MiB are always granted: 2 x 20000 steps at d_inner 512 took 2.2 ms
// whole and 3.1 in parts), the most sequences, else the most chunks.
BwdPart bwd_part(const ScanCut& q, int B, int T, int Di, int Tc) {
    const size_t rows = (size_t)B * T, dblk = (Di + SCAN_CH - 1) / SCAN_CH;
    const size_t budget = std::max<size_t>((size_t)B * Tc * NSTATE * Di + dblk * rows * 2 * NSTATE, (size_t)64 << 20);
    if (q.NBS <= 32768)
        for (int parts = 1; parts <= B; ++parts) {
            const int seqs = (B + parts - 1) / parts;
            if (bwd_floats(q, seqs, q.NC, T, Di) <= budget) return {seqs, q.NC};
        }
    int chunks = std::max(1, std::min(q.NC, 32768 / q.nblk));
    while (chunks > 1 && bwd_floats(q, 1, chunks, T, Di) > budget) chunks = (chunks + 1) / 2;
    return {1, chunks};
}
int scan_bwd(const float* x, const float* dt, const float* A_log, const float* bc, const float* Dsk, const float* dy,
             int B, int T, int Di, int Tc, const float* hsave, float* dx, float* ddt, float* dbc, float* dA_log,
             float* dD, hipStream_t s, std::string& err) {
    Tc = std::min(Tc, T);
    const int dblk = (Di + SCAN_CH - 1) / SCAN_CH;
    // short chunks go together, to a multiple of 8 steps: to 16 at least, and to 32
    // where they are many enough to fill the chip (a chunk costs its states at its start
    // and at its blocks' ends; 4 x 2000 steps at d_inner 512: 740 us in chunks of 16, 400
    // of 32; 64 steps at d_inner 64: 178 and 203, for the longer chains)
    const int nsave = (T + Tc - 1) / Tc, least = (long long)B * T * Di > 1 << 20 ? 32 : 16;
    int m = (least + Tc - 1) / Tc;
    while (m > 1 && m * Tc % 8) ++m;
    const ScanCut q = scan_cut(B, T, Di, (int)std::min<long long>((long long)m * Tc, T));
    const BwdPart part = bwd_part(q, B, T, Di, Tc);
    // one region for the call: an allocation and its release cost 45 + 80 to 170 us
    // each (64 x 128 steps, d_inner 1024: 1.06 ms of 1.33 in five of them)
    Buf region;
    size_t at = 0;
    auto piece = [&](size_t floats) { const size_t o = at; at += (floats + 63) / 64 * 64; return o; };
    const long long prow = (long long)part.seqs * std::min<long long>(T, (long long)part.chunks * q.Tc);
    const size_t o_hsub = piece((size_t)part.seqs * part.chunks * q.nsub * NSTATE * Di),
                 o_ghb = piece(scan_block_floats(q, part.seqs, Di)), o_pbc = piece((size_t)dblk * prow * 2 * NSTATE),
                 o_pA = piece(scan_block_floats(q, part.seqs, Di)), o_pD = piece(scan_block_floats(q, part.seqs, Di) / NSTATE);
    TCHK(region.alloc(at * sizeof(float)));
    float *hsub = region.f() + o_hsub, *ghb = region.f() + o_ghb, *pbc = region.f() + o_pbc, *pA = region.f() + o_pA,
          *pD = region.f() + o_pD;
    for (int b0 = 0; b0 < B; b0 += part.seqs) {
        const int nb = std::min(part.seqs, B - b0);
        const long long r0 = (long long)b0 * T;
        TCHK(scan_gstates(dt + r0 * Di, bc + r0 * 2 * NSTATE, 2 * NSTATE, 0, A_log, dy + r0 * Di, nb, T, Di, q, ghb, s));
        for (int c0 = 0; c0 < q.NC; c0 += part.chunks) {         // all of them unless nb is 1
            ScanCut p = q;
            p.NC = std::min(part.chunks, q.NC - c0);
            const int Tn = std::min(T - c0 * q.Tc, p.NC * q.Tc);
            p.NBS = scan_blocks(Tn, q.Tc, p.NC, q.TB);
            const long long r = r0 + (long long)c0 * q.Tc, rows = (long long)nb * Tn, blk = (long long)c0 * q.nblk;
            TCHK(scan_states(x + r * Di, dt + r * Di, bc + r * 2 * NSTATE, 2 * NSTATE, 0, A_log, nb, Tn, Di, q.Tc, p.NC,
                             hsave + ((long long)b0 * nsave + (long long)c0 * m) * NSTATE * Di, nsave, m, hsub, SCAN_SUB,
                             q.nsub, p.NC * q.nsub, nullptr, 1, s));
            TCHK(scan_grads(x + r * Di, dt + r * Di, bc + r * 2 * NSTATE, 2 * NSTATE, 0, A_log, Dsk, dy + r * Di, nb, Tn,
                            Di, p, hsub, ghb + blk * NSTATE * Di, nullptr, dx + r * Di, ddt + r * Di, pbc,
                            pA + blk * NSTATE * Di, pD + blk * Di, nullptr, s));
            hipLaunchKernelGGL(k_tr_dbc_reduce, dim3(blocks(rows * 2 * NSTATE)), dim3(256), 0, s, pbc, dblk, rows,
                               dbc + r * 2 * NSTATE, 2 * NSTATE, 0);
        }
        hipLaunchKernelGGL(k_sum_slices, dim3(blocks((long long)Di * NSTATE, 64)), dim3(256), 0, s, pA, nb * q.NBS,
                           (long long)Di * NSTATE, (long long)Di * NSTATE, dA_log, 1);
        hipLaunchKernelGGL(k_sum_slices, dim3(blocks(Di, 64)), dim3(256), 0, s, pD, nb * q.NBS, (long long)Di, (long long)Di,
                           dD, 1);
    }
    TCHK(hipGetLastError());
    TCHK(hipStreamSynchronize(s));
    return BOA_OK;
}

// Forward + backward over B sequences of T bytes (device uint8 [B][T]) with
// projections in dtype dt (BOA_DTYPE_F32 or BOA_DTYPE_BF16).  Writes the mean
// loss (nats) to *d_loss and the gradient (flat layout) to grad.
int loss_grad(boa_model* m, const uint8_t* tok, int B, int T, int Tc, int dt_, double* d_loss, float* grad,
              hipStream_t s, std::string& err) {
    const Layout& L = m->lay;
    const int D = L.D, Di = L.Di, R = L.R, NO = R + 2 * NSTATE, Tn = T - 1;
    const long long rows = (long long)B * Tn;
    if (Tc <= 0) Tc = 256;
    const int dt = dt_ == BOA_DTYPE_BF16 ? 1 : 0;
    int rc = train_ensure_buffers(m, B, T, Tc, err);
    if (rc) return rc;
    TrainCtx* c = static_cast<TrainCtx*>(m->train);
    const ScanCut cut = scan_cut(B, Tn, Di, Tn);
    const float* Wt = m->d_w;
    const size_t F = sizeof(float);
    float* ws = c->gws.f();
    float* part = c->part.f();
    uint8_t* wf = static_cast<uint8_t*>(c->wf.p);
    std::vector<std::vector<WMat>> wm;
    size_t wat = 0;
    for (int l = 0; l <= L.L; ++l) {
        wm.push_back(layer_mats(L, Wt, l, dt, &wat));
        TCHK(prep_mats(wm.back(), dt, wf, s));
    }
    const dim3 cblk(std::min(256, Di)), cgrid((Di + 255) / 256, (Tn + CONV_TS - 1) / CONV_TS, B);
    auto store = [] { return TRow{}; };
    auto add_to = [](const float* Cin) { TRow p{}; p.epi = 1; p.Cin = Cin; return p; };
    // ---------------- forward
    hipLaunchKernelGGL(k_tr_embed, dim3(blocks(rows, 4)), dim3(64, 4), 0, s, tok, B, T, Wt + L.embed, D,
                       c->rin[0].f());
    for (int l = 0; l < L.L; ++l) {
        const LayerOff& o = L.layer[l];
        const std::vector<WMat>& w = wm[l];
        float* rnext = l + 1 < L.L ? c->rin[l + 1].f() : c->rfin.f();
        ln_fwd(c->rin[l].f(), rows, D, Wt + o.norm_w, Wt + o.norm_b, c->a[l].f(), c->st[l].f(), s);
        TCHK(lin(dt, w[WF_IN], wf, c->a[l].f(), D, rows, c->xz[l].f(), 2 * Di, store(), ws, s));
        hipLaunchKernelGGL(k_tr_conv_fwd, cgrid, cblk, 0, s, c->xz[l].f(), Tn, Di, Wt + o.conv_w, Wt + o.conv_b,
                           c->xs[l].f());
        TCHK(lin(dt, w[WF_X], wf, c->xs[l].f(), Di, rows, c->dbc[l].f(), NO, store(), ws, s));
        {
            TRow p{};
            p.epi = 2;
            p.bias = Wt + o.dtb;
            p.C2 = c->dt[l].f();
            TCHK(lin(dt, w[WF_DT], wf, c->dbc[l].f(), NO, rows, c->dtr[l].f(), Di, p, ws, s));
        }
        const bool fine = l >= c->kept.fine;
        float* hsub = fine ? c->hs[l].f() : c->hsub.f();
        TCHK(scan_states(c->xs[l].f(), c->dt[l].f(), c->dbc[l].f(), NO, R, Wt + o.A_log, B, Tn, Di, Tn, 1, nullptr, 1, 1, hsub,
                         SCAN_SUB, cut.nsub, cut.nsub, fine ? nullptr : c->hs[l].f(), c->kept.every, s));
        TCHK(scan_y(c->xs[l].f(), c->dt[l].f(), c->dbc[l].f(), NO, R, Wt + o.A_log, Wt + o.Dsk, c->xz[l].f(), B, Tn, Di,
                    hsub, SCAN_SUB, cut.nsub, c->y[l].f(), c->g[l].f(), s));
        TCHK(lin(dt, w[WF_OUT], wf, c->g[l].f(), Di, rows, L.H ? c->fr[l].f() : rnext, D, add_to(c->rin[l].f()), ws, s));
        if (L.H) {            // r <- LayerNorm(W2 GELU(W1 r + b1) + b2)
            const int H = L.H;
            TCHK(lin(dt, w[WF_W1], wf, c->fr[l].f(), D, rows, c->fu[l].f(), H, store(), ws, s));
            hipLaunchKernelGGL(k_tr_bias_gelu, dim3(blocks(rows * H)), dim3(256), 0, s, c->fu[l].f(), rows, H,
                               Wt + o.ffn_b1, c->fg[l].f());
            TCHK(lin(dt, w[WF_W2], wf, c->fg[l].f(), H, rows, c->ff[l].f(), D, store(), ws, s));
            hipLaunchKernelGGL(k_tr_add_bias, dim3(blocks(rows * D)), dim3(256), 0, s, c->ff[l].f(), rows, D,
                               Wt + o.ffn_b2);
            ln_fwd(c->ff[l].f(), rows, D, Wt + o.ffn_nw, Wt + o.ffn_nb, rnext, c->fst[l].f(), s);
        }
    }
    ln_fwd(c->rfin.f(), rows, D, Wt + L.norm_f_w, Wt + L.norm_f_b, c->rf.f(), c->stf.f(), s);
    TCHK(lin(dt, wm[L.L][0], wf, c->rf.f(), D, rows, c->logits.f(), 256, store(), ws, s));
    hipLaunchKernelGGL(k_tr_ce, dim3(blocks(rows, 4)), dim3(64, 4), 0, s, c->logits.f(), Wt + L.head_b, tok, B, T,
                       c->rowloss.f(), 1.0f / (float)rows);
    hipLaunchKernelGGL((k_sum_all<float>), dim3(1), dim3(256), 0, s, (const float*)c->rowloss.f(), rows,
                       1.0 / (double)rows, d_loss, (float*)nullptr);
    // ---------------- backward (every gradient region is written exactly once)
    float* G = grad;
    float* dr = c->dr.f();
    float* tmp = c->tmp.f();
    const int dblk = (Di + SCAN_CH - 1) / SCAN_CH;
    TCHK(wgrad(dt, c->logits.f(), 256, c->rf.f(), D, 256, D, G + L.head_w, rows, ws, s));
    TCHK(colsum(c->logits.f(), rows, 256, 256, part, G + L.head_b, s));
    TCHK(lin(dt, wm[L.L][1], wf, c->logits.f(), 256, rows, tmp, D, store(), ws, s));          // d rf
    ln_bwd(tmp, c->rfin.f(), c->stf.f(), rows, D, Wt + L.norm_f_w, dr, 0, part, G + L.norm_f_w, s);
    for (int l = L.L - 1; l >= 0; --l) {
        const LayerOff& o = L.layer[l];
        const std::vector<WMat>& w = wm[l];
        if (L.H) {            // through LayerNorm(FFN(r)); no residual around it
            const int H = L.H;
            ln_bwd(dr, c->ff[l].f(), c->fst[l].f(), rows, D, Wt + o.ffn_nw, tmp, 0, part, G + o.ffn_nw, s);   // tmp = d f
            TCHK(wgrad(dt, tmp, D, c->fg[l].f(), H, D, H, G + o.ffn_w2, rows, ws, s));
            TCHK(colsum(tmp, rows, D, D, part, G + o.ffn_b2, s));
            TCHK(lin(dt, w[WF_W2_T], wf, tmp, D, rows, c->fdu.f(), H, store(), ws, s));          // d GELU
            hipLaunchKernelGGL(k_tr_gelu_bwd, dim3(blocks(rows * H)), dim3(256), 0, s, c->fdu.f(), c->fu[l].f(),
                               rows * H);
            TCHK(wgrad(dt, c->fdu.f(), H, c->fr[l].f(), D, H, D, G + o.ffn_w1, rows, ws, s));
            TCHK(colsum(c->fdu.f(), rows, H, H, part, G + o.ffn_b1, s));
            TCHK(lin(dt, w[WF_W1_T], wf, c->fdu.f(), H, rows, dr, D, store(), ws, s));           // d r
        }
        TCHK(wgrad(dt, dr, D, c->g[l].f(), Di, D, Di, G + o.out_w, rows, ws, s));
        {                     // d gate, straight into dy and dz
            TRow p{};
            p.epi = 3;
            p.y = c->y[l].f();
            p.z = c->xz[l].f() + Di;
            p.C2 = c->dxz.f() + Di;
            p.ldc2 = 2 * Di;
            TCHK(lin(dt, w[WF_OUT_T], wf, dr, D, rows, c->dyb.f(), Di, p, ws, s));
        }
        float* hsub = c->hs[l].f();
        if (l < c->kept.fine) {                          // the states every SCAN_SUB steps again
            const int every = c->kept.every, n = (Tn + every - 1) / every;
            hsub = c->hsub.f();
            TCHK(scan_states(c->xs[l].f(), c->dt[l].f(), c->dbc[l].f(), NO, R, Wt + o.A_log, B, Tn, Di, every, n,
                             c->hs[l].f(), n, 1, hsub, SCAN_SUB, every / SCAN_SUB, cut.nsub, nullptr, 1, s));
        }
        TCHK(scan_gstates(c->dt[l].f(), c->dbc[l].f(), NO, R, Wt + o.A_log, c->dyb.f(), B, Tn, Di, cut, c->ghb.f(), s));
        TCHK(scan_grads(c->xs[l].f(), c->dt[l].f(), c->dbc[l].f(), NO, R, Wt + o.A_log, Wt + o.Dsk, c->dyb.f(), B, Tn,
                        Di, cut, hsub, c->ghb.f(), c->dtr[l].f(), c->dxs.f(), c->ddtr.f(), c->pbc.f(), c->pA.f(),
                        c->pD.f(), c->pT.f(), s));
        hipLaunchKernelGGL(k_tr_dbc_reduce, dim3(blocks(rows * 2 * NSTATE)), dim3(256), 0, s, c->pbc.f(), dblk, rows,
                           c->ddbc.f(), NO, R);
        hipLaunchKernelGGL(k_sum_slices, dim3(blocks((long long)Di * NSTATE, 64)), dim3(256), 0, s, c->pA.f(), B * cut.NBS,
                           (long long)Di * NSTATE, (long long)Di * NSTATE, G + o.A_log, 0);
        hipLaunchKernelGGL(k_sum_slices, dim3(blocks(Di, 64)), dim3(256), 0, s, c->pD.f(), B * cut.NBS, (long long)Di, (long long)Di,
                           G + o.Dsk, 0);
        hipLaunchKernelGGL(k_sum_slices, dim3(blocks(Di, 64)), dim3(256), 0, s, c->pT.f(), B * cut.NBS, (long long)Di,
                           (long long)Di, G + o.dtb, 0);
        TCHK(wgrad(dt, c->ddtr.f(), Di, c->dbc[l].f(), NO, Di, R, G + o.dtw, rows, ws, s));
        TCHK(lin(dt, w[WF_DT_T], wf, c->ddtr.f(), Di, rows, c->ddbc.f(), NO, store(), ws, s));      // d delta
        TCHK(wgrad(dt, c->ddbc.f(), NO, c->xs[l].f(), Di, NO, Di, G + o.xw, rows, ws, s));
        TCHK(lin(dt, w[WF_X_T], wf, c->ddbc.f(), NO, rows, c->dxs.f(), Di, add_to(c->dxs.f()), ws, s));   // dxs += ddbc W_x
        {
            const int S = (int)(cgrid.y * cgrid.z);
            const long long stride = (long long)Di * (KCONV + 1);
            hipLaunchKernelGGL(k_tr_conv_bwd, cgrid, cblk, 0, s, c->dxs.f(), c->xz[l].f(), Tn, Di, Wt + o.conv_w,
                               Wt + o.conv_b, c->dxz.f(), part);
            hipLaunchKernelGGL(k_sum_slices, dim3(blocks((long long)Di * KCONV, 64)), dim3(256), 0, s, part, S,
                               (long long)Di * KCONV, stride, G + o.conv_w, 0);
            hipLaunchKernelGGL(k_sum_slices, dim3(blocks(Di, 64)), dim3(256), 0, s, part + (long long)Di * KCONV, S,
                               (long long)Di, stride, G + o.conv_b, 0);
        }
        TCHK(wgrad(dt, c->dxz.f(), 2 * Di, c->a[l].f(), D, 2 * Di, D, G + o.in_w, rows, ws, s));
        TCHK(lin(dt, w[WF_IN_T], wf, c->dxz.f(), 2 * Di, rows, tmp, D, store(), ws, s));            // d a
        ln_bwd(tmp, c->rin[l].f(), c->st[l].f(), rows, D, Wt + o.norm_w, dr, 1, part, G + o.norm_w, s);
    }
    {
        const long long S = row_slices(rows);
        const long long per = (rows + S - 1) / S;
        hipLaunchKernelGGL(k_tr_embed_bwd_part, dim3(D / 64, (unsigned)S), dim3(64), 0, s, tok, B, T, dr, D, per,
                           part);
        hipLaunchKernelGGL(k_sum_slices, dim3(blocks((long long)VOCAB * D, 64)), dim3(256), 0, s, part, (int)S,
                           (long long)VOCAB * D, (long long)VOCAB * D, G + L.embed, 0);
    }
    TCHK(hipGetLastError());
    TCHK(hipStreamSynchronize(s));
    return BOA_OK;
}

int train_ctx_ensure(boa_model* m, std::string& err) {
    if (m->train) return BOA_OK;
    TrainCtx* c = new TrainCtx;
    const size_t n = m->lay.total * sizeof(float);
    if (c->m.alloc(n) != hipSuccess || c->v.alloc(n) != hipSuccess || c->grad.alloc(n) != hipSuccess ||
        c->sqpart.alloc(1024 * sizeof(float)) != hipSuccess || c->sq.alloc(sizeof(float)) != hipSuccess) {
        delete c;
        err = "optimizer state";
        return BOA_E_OOM;
    }
    if (hipMemset(c->m.p, 0, n) != hipSuccess || hipMemset(c->v.p, 0, n) != hipSuccess) {
        delete c;
        err = "optimizer state";
        return BOA_E_DEVICE;
    }
    m->train = c;
    return BOA_OK;
}

// One AdamW step from the gradient in g (device, flat layout): global norm by
// a fixed tree, clipping, decoupled weight decay, bias-corrected moments.
int optimizer_step(boa_model* m, const float* g, const boa_train_opts& o, float lr, hipStream_t s, std::string& err) {
    int rc = train_ctx_ensure(m, err);
    if (rc) return rc;
    TrainCtx* c = static_cast<TrainCtx*>(m->train);
    const long long n = (long long)m->lay.total;
    const long long per = (n + 1023) / 1024;
    hipLaunchKernelGGL(k_sqsum_part, dim3(1024), dim3(256), 0, s, g, n, per, c->sqpart.f());
    hipLaunchKernelGGL((k_sum_all<float>), dim3(1), dim3(256), 0, s, (const float*)c->sqpart.f(), 1024LL, 1.0,
                       (double*)nullptr, c->sq.f());
    c->step += 1;
    const float bc1 = 1.0f - std::pow(o.beta1, (float)c->step), bc2 = 1.0f - std::pow(o.beta2, (float)c->step);
    hipLaunchKernelGGL(k_adamw, dim3(blocks(n)), dim3(256), 0, s, m->d_w, g, c->m.f(), c->v.f(), n, lr, o.beta1,
                       o.beta2, o.eps, o.weight_decay, bc1, bc2, o.grad_clip, c->sq.f());
    TCHK(hipGetLastError());
    TCHK(hipStreamSynchronize(s));
    return BOA_OK;
}

// One optimisation step on device tokens; *loss gets the mean loss (nats).
int train_step(boa_model* m, const uint8_t* tok, int B, int T, const boa_train_opts& o, float lr, double* d_loss,
               hipStream_t s, std::string& err) {
    int rc = train_ctx_ensure(m, err);
    if (rc) return rc;
    TrainCtx* c = static_cast<TrainCtx*>(m->train);
    rc = loss_grad(m, tok, B, T, (int)o.chunk_t, (int)o.dtype, d_loss, c->grad.f(), s, err);
    if (rc) return rc;
    return optimizer_step(m, c->grad.f(), o, lr, s, err);
}

// ============================================================ C ABI
namespace {
boa_train_opts with_defaults(const boa_train_opts* in) {
    boa_train_opts o{};
    if (in) o = *in;
    if (o.lr <= 0.f) o.lr = 1e-3f;
    if (o.beta1 <= 0.f) o.beta1 = 0.9f;
    if (o.beta2 <= 0.f) o.beta2 = 0.999f;
    if (o.eps <= 0.f) o.eps = 1e-8f;
    if (o.weight_decay < 0.f) o.weight_decay = 0.f;
    if (in == nullptr || (in->weight_decay == 0.f && in->lr == 0.f)) o.weight_decay = 0.01f;
    if (in == nullptr || in->grad_clip == 0.f) o.grad_clip = 1.0f;
    if (o.warmup == 0 && (in == nullptr || in->lr == 0.f)) o.warmup = 100;
    if (o.batch == 0) o.batch = 32;
    if (o.seq_len == 0) o.seq_len = 8192;
    if (o.chunk_t == 0) o.chunk_t = 256;
    return o;
}
float lr_at(const boa_train_opts& o, long long step) {   // step counts from 1
    if (o.warmup == 0 || step >= (long long)o.warmup) return o.lr;
    return o.lr * (float)step / (float)o.warmup;
}
uint64_t splitmix64(uint64_t& x) {
    uint64_t z = (x += 0x9E3779B97F4A7C15ULL);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    return z ^ (z >> 31);
}
int scan_chunk(uint32_t chunk_t) { return chunk_t ? (int)std::min<uint32_t>(chunk_t, INT32_MAX) : 256; }
bool train_dtype_ok(uint32_t d) { return d == BOA_DTYPE_F32 || d == BOA_DTYPE_BF16; }
uint64_t fnv1a64(const void* data, size_t n, uint64_t h) {
    const uint8_t* p = static_cast<const uint8_t*>(data);
    for (size_t i = 0; i < n; ++i) { h ^= p[i]; h *= 1099511628211ULL; }
    return h;
}
int refresh_after_update(boa_model* m, hipStream_t s) {
    // derived copies (transposed small weights, bf16 and fragment-ordered projections) follow the master weights
    if (launch_prep(m, s) != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
        return set_error(BOA_E_DEVICE, "refreshing derived weights");
    m->fp_stale = true;
    return BOA_OK;
}
}  // namespace
}  // namespace boa

using namespace boa;

extern "C" int boa_loss_grad_dev(boa_model* m, const uint8_t* d_tokens, uint32_t B, uint32_t T, uint32_t chunk_t,
                                 uint32_t dtype, double* d_loss, float* d_grad, void* stream) {
    if (!m || !d_tokens || !d_loss || !d_grad || B == 0 || T < 2) return set_error(BOA_E_ARG, "bad argument");
    if (!train_dtype_ok(dtype)) return set_error(BOA_E_UNSUPPORTED, "training runs in f32 or bf16");
    std::string err;
    (void)hipSetDevice(m->device);
    int rc = train_ctx_ensure(m, err);
    if (!rc) rc = loss_grad(m, d_tokens, (int)B, (int)T, (int)chunk_t, (int)dtype, d_loss, d_grad, (hipStream_t)stream,
                            err);
    return rc ? set_error(rc, err) : BOA_OK;
}

extern "C" int boa_optimizer_step_dev(boa_model* m, const float* d_grad, const boa_train_opts* opts, void* stream) {
    if (!m || !d_grad) return set_error(BOA_E_ARG, "bad argument");
    std::string err;
    (void)hipSetDevice(m->device);
    boa_train_opts o = with_defaults(opts);
    int rc = train_ctx_ensure(m, err);
    if (rc) return set_error(rc, err);
    TrainCtx* c = static_cast<TrainCtx*>(m->train);
    rc = optimizer_step(m, d_grad, o, lr_at(o, c->step + 1), (hipStream_t)stream, err);
    if (rc) return set_error(rc, err);
    return refresh_after_update(m, (hipStream_t)stream);
}

extern "C" int boa_train_step_dev(boa_model* m, const uint8_t* d_tokens, uint32_t B, uint32_t T,
                                  const boa_train_opts* opts, double* d_loss, void* stream) {
    if (!m || !d_tokens || !d_loss || B == 0 || T < 2) return set_error(BOA_E_ARG, "bad argument");
    boa_train_opts o = with_defaults(opts);
    if (!train_dtype_ok(o.dtype)) return set_error(BOA_E_UNSUPPORTED, "training runs in f32 or bf16");
    std::string err;
    (void)hipSetDevice(m->device);
    int rc = train_ctx_ensure(m, err);
    if (rc) return set_error(rc, err);
    TrainCtx* c = static_cast<TrainCtx*>(m->train);
    rc = train_step(m, d_tokens, (int)B, (int)T, o, lr_at(o, c->step + 1), d_loss, (hipStream_t)stream, err);
    if (rc) return set_error(rc, err);
    return refresh_after_update(m, (hipStream_t)stream);
}

extern "C" int boa_train(boa_model* m, const uint8_t* h_bytes, uint64_t n, const boa_train_opts* opts,
                         float* h_losses, uint64_t n_losses) {
    if (!m || (!h_bytes && n)) return set_error(BOA_E_ARG, "bad argument");
    boa_train_opts o = with_defaults(opts);
    if (!train_dtype_ok(o.dtype)) return set_error(BOA_E_UNSUPPORTED, "training runs in f32 or bf16");
    const uint64_t W = o.seq_len, nwin = W ? n / W : 0;
    if (nwin == 0) return set_error(BOA_E_ARG, "input shorter than one training window");
    const uint32_t B = (uint32_t)std::min<uint64_t>(o.batch, nwin);
    (void)hipSetDevice(m->device);
    hipStream_t s;
    if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) return set_error(BOA_E_DEVICE, "stream");
    Buf d_all, d_tok, d_loss;
    if (d_all.alloc(nwin * W) != hipSuccess || d_tok.alloc((size_t)B * W) != hipSuccess ||
        d_loss.alloc(sizeof(double)) != hipSuccess) {
        (void)hipStreamDestroy(s);
        return set_error(BOA_E_OOM, "training buffers");
    }
    if (hipMemcpy(d_all.p, h_bytes, nwin * W, hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipStreamDestroy(s);
        return set_error(BOA_E_DEVICE, "copying the training bytes");
    }
    std::vector<uint64_t> order(nwin);
    uint64_t rng = o.seed ? o.seed : 1;
    uint64_t pos = nwin;   // forces a shuffle at the first step
    auto next_window = [&]() {
        if (pos >= nwin) {          // new epoch: Fisher-Yates with splitmix64
            for (uint64_t i = 0; i < nwin; ++i) order[i] = i;
            for (uint64_t i = nwin - 1; i > 0; --i) std::swap(order[i], order[splitmix64(rng) % (i + 1)]);
            pos = 0;
        }
        return order[pos++];
    };
    // a model that has already taken steps (a resumed checkpoint) continues
    // the window sequence where those steps left it
    const long long done = m->train ? static_cast<TrainCtx*>(m->train)->step : 0;
    for (long long k = 0; k < done * (long long)B; ++k) (void)next_window();
    int rc = BOA_OK;
    for (uint32_t step = 0; step < o.steps && rc == BOA_OK; ++step) {
        for (uint32_t b = 0; b < B; ++b) {
            const uint64_t w = next_window();
            (void)hipMemcpyAsync(static_cast<uint8_t*>(d_tok.p) + (size_t)b * W,
                                 static_cast<uint8_t*>(d_all.p) + w * W, W, hipMemcpyDeviceToDevice, s);
        }
        rc = boa_train_step_dev(m, static_cast<uint8_t*>(d_tok.p), B, (uint32_t)W, &o,
                                static_cast<double*>(d_loss.p), s);
        if (rc == BOA_OK && h_losses && step < n_losses) {
            double l = 0;
            (void)hipMemcpy(&l, d_loss.p, sizeof(double), hipMemcpyDeviceToHost);
            h_losses[step] = (float)l;
        }
    }
    (void)hipStreamDestroy(s);
    return rc;
}

// Training checkpoint: "BOAT", version 1, config, step count, then the
// float32 master weights, first and second AdamW moments (n each), then an
// FNV-1a hash of everything before it.
extern "C" int boa_train_state_save(const boa_model* m, const char* path) {
    if (!m || !path) return set_error(BOA_E_ARG, "null argument");
    const uint64_t n = m->lay.total;
    std::vector<float> w(n), mo(n, 0.f), vo(n, 0.f);
    int64_t step = 0;
    (void)hipSetDevice(m->device);
    if (hipMemcpy(w.data(), m->d_w, n * sizeof(float), hipMemcpyDeviceToHost) != hipSuccess)
        return set_error(BOA_E_DEVICE, "reading the weights");
    if (m->train) {
        const TrainCtx* c = static_cast<const TrainCtx*>(m->train);
        step = c->step;
        if (hipMemcpy(mo.data(), c->m.p, n * sizeof(float), hipMemcpyDeviceToHost) != hipSuccess ||
            hipMemcpy(vo.data(), c->v.p, n * sizeof(float), hipMemcpyDeviceToHost) != hipSuccess)
            return set_error(BOA_E_DEVICE, "reading the optimiser moments");
    }
    const uint32_t ver = 1;
    uint64_t h = 1469598103934665603ULL;
    h = fnv1a64("BOAT", 4, h);
    h = fnv1a64(&ver, 4, h);
    h = fnv1a64(&m->cfg, sizeof(boa_config), h);
    h = fnv1a64(&step, 8, h);
    h = fnv1a64(w.data(), n * 4, h);
    h = fnv1a64(mo.data(), n * 4, h);
    h = fnv1a64(vo.data(), n * 4, h);
    FILE* f = std::fopen(path, "wb");
    if (!f) return set_error(BOA_E_ARG, std::string("cannot open ") + path);
    bool ok = std::fwrite("BOAT", 1, 4, f) == 4 && std::fwrite(&ver, 4, 1, f) == 1 &&
              std::fwrite(&m->cfg, sizeof(boa_config), 1, f) == 1 && std::fwrite(&step, 8, 1, f) == 1 &&
              std::fwrite(w.data(), 4, n, f) == n && std::fwrite(mo.data(), 4, n, f) == n &&
              std::fwrite(vo.data(), 4, n, f) == n && std::fwrite(&h, 8, 1, f) == 1;
    ok = (std::fclose(f) == 0) && ok;
    return ok ? BOA_OK : set_error(BOA_E_ARG, "short write");
}

extern "C" int boa_train_state_load(boa_model* m, const char* path) {
    if (!m || !path) return set_error(BOA_E_ARG, "null argument");
    FILE* f = std::fopen(path, "rb");
    if (!f) return set_error(BOA_E_ARG, std::string("cannot open ") + path);
    const uint64_t n = m->lay.total;
    char mg[4];
    uint32_t ver = 0;
    boa_config cfg{};
    int64_t step = 0;
    std::vector<float> w(n), mo(n), vo(n);
    uint64_t hs = 0;
    bool ok = std::fread(mg, 1, 4, f) == 4 && std::memcmp(mg, "BOAT", 4) == 0 && std::fread(&ver, 4, 1, f) == 1 &&
              ver == 1 && std::fread(&cfg, sizeof(cfg), 1, f) == 1;
    if (!ok) { std::fclose(f); return set_error(BOA_E_FORMAT, "not a BOAT v1 training checkpoint"); }
    if (std::memcmp(&cfg, &m->cfg, sizeof(cfg)) != 0) {
        std::fclose(f);
        return set_error(BOA_E_MODEL, "checkpoint config differs from the model's");
    }
    ok = std::fread(&step, 8, 1, f) == 1 && std::fread(w.data(), 4, n, f) == n && std::fread(mo.data(), 4, n, f) == n &&
         std::fread(vo.data(), 4, n, f) == n && std::fread(&hs, 8, 1, f) == 1;
    std::fclose(f);
    if (!ok || step < 0) return set_error(BOA_E_FORMAT, "truncated training checkpoint");
    uint64_t h = 1469598103934665603ULL;
    h = fnv1a64("BOAT", 4, h);
    h = fnv1a64(&ver, 4, h);
    h = fnv1a64(&cfg, sizeof(cfg), h);
    h = fnv1a64(&step, 8, h);
    h = fnv1a64(w.data(), n * 4, h);
    h = fnv1a64(mo.data(), n * 4, h);
    h = fnv1a64(vo.data(), n * 4, h);
    if (h != hs) return set_error(BOA_E_CORRUPT, "training checkpoint hash mismatch");
    int rc = boa_model_set_weights(m, w.data(), n);
    if (rc) return rc;
    std::string err;
    rc = train_ctx_ensure(m, err);
    if (rc) return set_error(rc, err);
    TrainCtx* c = static_cast<TrainCtx*>(m->train);
    if (hipMemcpy(c->m.p, mo.data(), n * 4, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(c->v.p, vo.data(), n * 4, hipMemcpyHostToDevice) != hipSuccess)
        return set_error(BOA_E_DEVICE, "writing the optimiser moments");
    c->step = step;
    return BOA_OK;
}

extern "C" int boa_train_steps_done(const boa_model* m, uint64_t* steps) {
    if (!m || !steps) return set_error(BOA_E_ARG, "null argument");
    *steps = m->train ? (uint64_t)static_cast<const TrainCtx*>(m->train)->step : 0;
    return BOA_OK;
}

extern "C" int boa_scan_fwd_dev(const float* d_x, const float* d_dt, const float* d_A_log, const float* d_bc,
                                const float* d_Dskip, uint32_t B, uint32_t T, uint32_t Di, uint32_t chunk_t,
                                float* d_y, float* d_hsave, void* stream) {
    if (!d_x || !d_dt || !d_A_log || !d_bc || !d_Dskip || !d_y || !d_hsave || B == 0 || T == 0 || Di == 0)
        return set_error(BOA_E_ARG, "bad argument");
    std::string err;
    int rc = scan_fwd(d_x, d_dt, d_A_log, d_bc, d_Dskip, (int)B, (int)T, (int)Di, scan_chunk(chunk_t), d_y, d_hsave,
                      (hipStream_t)stream, err);
    return rc ? set_error(rc, err) : BOA_OK;
}

extern "C" int boa_scan_bwd_dev(const float* d_x, const float* d_dt, const float* d_A_log, const float* d_bc,
                                const float* d_Dskip, const float* d_dy, uint32_t B, uint32_t T, uint32_t Di,
                                uint32_t chunk_t, const float* d_hsave, float* d_dx, float* d_ddt, float* d_dbc,
                                float* d_dA_log, float* d_dDskip, void* stream) {
    if (!d_x || !d_dt || !d_A_log || !d_bc || !d_Dskip || !d_dy || !d_hsave || !d_dx || !d_ddt || !d_dbc ||
        !d_dA_log || !d_dDskip || B == 0 || T == 0 || Di == 0)
        return set_error(BOA_E_ARG, "bad argument");
    std::string err;
    int rc = scan_bwd(d_x, d_dt, d_A_log, d_bc, d_Dskip, d_dy, (int)B, (int)T, (int)Di, scan_chunk(chunk_t), d_hsave,
                      d_dx, d_ddt, d_dbc, d_dA_log, d_dDskip, (hipStream_t)stream, err);
    return rc ? set_error(rc, err) : BOA_OK;
}
