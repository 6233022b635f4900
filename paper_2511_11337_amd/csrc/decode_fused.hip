// Fused persistent decoder: one workgroup runs every decoding step of G
// lanes (streams) in a single launch -- embedding, all Mamba blocks, final
// LayerNorm, head, histogram / CDF and range decoding -- with the lanes'
// activations in LDS, the range-decoder state in registers, and the conv and
// scan state of each lane in LDS (one lane per workgroup) or in its own slice
// of device memory.  Decoding is
// inherently sequential per stream (each step needs the byte the previous
// step decoded; paper, Coders & Parallelisation); the per-step kernel chain
// of the step-graph decoder pays a launch and a cold start per kernel, this
// kernel pays them once per call.
//
// Every output element is produced by the same per-element operation
// sequence as in the encoder kernels, so the integer frequency tables (and
// hence the decoded bytes) are identical:
//   LayerNorm      the statistics of ln_stats (each wave takes them for its
//                  row) + ln_apply per element;
//   projections    the same MFMA instruction and k order as the encoder
//                  (f32: 16x16x4 in k steps of 4; bf16: 16x16x32 in k steps of
//                  32; fp8: 16x16x32 fp8 with the same per-row and per-tensor
//                  scales; from zero), the lane's row placed in a 16-row tile
//                  (MFMA rows are independent), or for f32 and one or two
//                  lanes the fmaf sequence that this MFMA is;
//   conv, x_proj, dt, scan, gate, histogram, coder: the shared device
//                  functions with the same operands in the same order.
//
// Projection weights are read in a fragment-ordered copy made at model load,
// so each MFMA operand load of a wave is 1 KiB of contiguous memory.
#include "boa_internal.h"

#include <hip/hip_bf16.h>

#include <type_traits>

#include "hotpath_common.h"

namespace boa {

// ============================================================== fragment-ordered weights
// f32 : element (nf, q, lane, j) = W[16 nf + (lane & 15)][16 q + 4 j + (lane >> 4)]
//       (one float4 per lane per q covers the MFMA k steps 4q .. 4q + 3)
// bf16: element (nf, s, lane, j) = bf16(W[16 nf + (lane & 15)][32 s + 8 (lane >> 4) + j])
__global__ void k_frag_f32(const float* __restrict__ W, int N, int K, float* __restrict__ out) {
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (long long)N * K) return;
    const int j = (int)(i & 3);
    long long t = i >> 2;
    const int lane = (int)(t & 63);
    t >>= 6;
    const int q = (int)(t % (K / 16));
    const int nf = (int)(t / (K / 16));
    out[i] = W[(long long)(16 * nf + (lane & 15)) * K + 16 * q + 4 * j + (lane >> 4)];
}
__global__ void k_frag_f32_pad(const float* __restrict__ W, int N, int NP, int K, float* __restrict__ out) {
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (long long)NP * K) return;
    const int j = (int)(i & 3);
    long long t = i >> 2;
    const int lane = (int)(t & 63);
    t >>= 6;
    const int q = (int)(t % (K / 16));
    const int nf = (int)(t / (K / 16));
    const int row = 16 * nf + (lane & 15);
    out[i] = row < N ? W[(long long)row * K + 16 * q + 4 * j + (lane >> 4)] : 0.0f;
}
hipError_t launch_frag_pad(const float* W, int N, int NP, int K, float* out, hipStream_t s) {
    if (NP % 16 || NP < N || K % 16) return hipErrorInvalidValue;
    const long long n = (long long)NP * K;
    hipLaunchKernelGGL(k_frag_f32_pad, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, W, N, NP, K, out);
    return hipGetLastError();
}
__global__ void k_frag_bf16(const float* __restrict__ W, int N, int K, uint16_t* __restrict__ out) {
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (long long)N * K) return;
    const int j = (int)(i & 7);
    long long t = i >> 3;
    const int lane = (int)(t & 63);
    t >>= 6;
    const int s = (int)(t % (K / 32));
    const int nf = (int)(t / (K / 32));
    out[i] = f2bf_bits(W[(long long)(16 * nf + (lane & 15)) * K + 32 * s + 8 * (lane >> 4) + j]);
}
// Largest |w| of a tensor as float bits (non-negative floats order like their
// unsigned bit patterns, so an integer maximum is exact and order-free).
__global__ void k_amax(const float* __restrict__ W, long long n, unsigned* __restrict__ amax_bits) {
    float m = 0.0f;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
        m = fmaxf(m, fabsf(W[i]));
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) atomicMax(amax_bits, __float_as_uint(m));
}
// fp8: element (nf, p, lane, h, j) = e4m3(W[16 nf + lane % 16][32 (2p + h) + 8 (lane / 16) + j] * 2^-e)
// (16 bytes per lane cover MFMA k steps 2p and 2p + 1); e = fp8_exp(amax),
// written to *ew by element 0.
__global__ void k_frag_fp8(const float* __restrict__ W, int N, int K, const unsigned* __restrict__ amax_bits,
                           int* __restrict__ ew, uint8_t* __restrict__ out) {
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (long long)N * K) return;
    const int e = fp8_exp(__uint_as_float(*amax_bits));
    if (i == 0) *ew = e;
    const int j = (int)(i & 7), h = (int)((i >> 3) & 1), lane = (int)((i >> 4) & 63);
    const long long t = i >> 10;
    const int SP = K / 64;
    const int p = (int)(t % SP), nf = (int)(t / SP);
    const float w = W[(long long)(16 * nf + (lane & 15)) * K + 32 * (2 * p + h) + 8 * (lane >> 4) + j];
    out[i] = fp8_byte(ldexpf(w, -e));
}
hipError_t launch_frag(const float* W, int N, int K, float* f32, uint16_t* b16, uint8_t* f8, unsigned* amax,
                       int* ew, hipStream_t s) {
    if (N % 16 || K % 64) return hipErrorInvalidValue;
    const long long n = (long long)N * K;
    const unsigned nb = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(k_frag_f32, dim3(nb), dim3(256), 0, s, W, N, K, f32);
    hipLaunchKernelGGL(k_frag_bf16, dim3(nb), dim3(256), 0, s, W, N, K, b16);
    hipError_t e = hipMemsetAsync(amax, 0, sizeof(unsigned), s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_amax, dim3(256), dim3(256), 0, s, W, n, amax);
    hipLaunchKernelGGL(k_frag_fp8, dim3(nb), dim3(256), 0, s, W, N, K, amax, ew, f8);
    return hipGetLastError();
}

// ============================================================== fused decoder
namespace {
// Weight pointers reach the kernel through a device array, so the compiler
// cannot prove they address global memory and would emit FLAT loads, which
// share the LDS wait counter and serialise every LDS access behind every
// outstanding weight load.  Casting them to the global address space keeps
// the weight stream asynchronous.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
DEVI float gld(const float* p) { return *(const __attribute__((address_space(1))) float*)p; }
DEVI float4 gld(const float4* p) {
    const f32x4 v = *(const __attribute__((address_space(1))) f32x4*)p;
    return make_float4(v.x, v.y, v.z, v.w);
}
DEVI uint2 gld(const uint2* p) {
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 v = *(const __attribute__((address_space(1))) u32x2*)p;
    return make_uint2(v.x, v.y);
}
// The lanes' conv and scan state is read once and written once per step, a
// stream far larger than the L2: non-temporal accesses keep it from evicting
// the weights, which every workgroup reads every step.
DEVI float gld_nt(const float* p) { return __builtin_nontemporal_load((const __attribute__((address_space(1))) float*)p); }
DEVI float4 gld_nt(const float4* p) {
    const f32x4 v = __builtin_nontemporal_load((const __attribute__((address_space(1))) f32x4*)p);
    return make_float4(v.x, v.y, v.z, v.w);
}
DEVI void gst_nt(float* p, float v) { __builtin_nontemporal_store(v, (__attribute__((address_space(1))) float*)p); }
DEVI void gst_nt(float4* p, float4 v) {
    const f32x4 t = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(t, (__attribute__((address_space(1))) f32x4*)p);
}
// four bf16 (element j in bits 16 j .. 16 j + 15) as exact floats
DEVI float4 bf4(uint2 v) {
    return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u), __uint_as_float(v.y << 16),
                       __uint_as_float(v.y & 0xFFFF0000u));
}
// dt_proj weights of channel d: float [R][Di] copy, or in BF16 mode the bf16
// parameter [Di][R] (R / 4 loads of four)
template <int DT, int RR>
struct DtW {
    static constexpr int NQ = DT == 1 ? RR / 4 : 1;
    float f[DT == 1 ? 1 : RR];
    uint2 q[NQ];
    DEVI void load(const FusedLayer& w, int Di, int d) {
        if (DT == 1) {
            const uint2* src = reinterpret_cast<const uint2*>(w.dtw16 + (long long)d * RR);
#pragma unroll
            for (int i = 0; i < NQ; ++i) q[i] = gld(src + i);
        } else {
#pragma unroll
            for (int k = 0; k < RR; ++k) f[k] = gld(w.dtwT + k * Di + d);
        }
    }
    DEVI void get(float (&o)[RR]) const {
        if (DT == 1) {
#pragma unroll
            for (int i = 0; i < NQ; ++i) {
                const float4 v = bf4(q[i]);
                o[4 * i] = v.x; o[4 * i + 1] = v.y; o[4 * i + 2] = v.z; o[4 * i + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int k = 0; k < RR; ++k) o[k] = f[DT == 1 ? 0 : k];
        }
    }
};
static_assert(sizeof(uint16_t) == 2, "bf16 bits");

constexpr int FNT = 512;              // threads per workgroup
constexpr int FNW = FNT / 64;         // waves

template <int D, int Di, int RR, int G>
struct FusedLds {
    static constexpr int NO = RR + 2 * NSTATE;
    static constexpr int DS = D + 4;          // padded row strides (floats)
    static constexpr int GS = Di + 4;
    static constexpr int XSR = Di + 4;        // row stride of xs (rows 4 banks apart)
    static constexpr int ZS = Di > VOCAB ? Di : VOCAB;     // row stride of the z half / logits
    static constexpr int r = 0;                            // [G][D]    residual stream
    static constexpr int a = r + G * D;                    // [G][DS]   LayerNorm output
    static constexpr int xz = a + G * DS;                  // [G][ZS]   z half of in_proj / logits [G][256]
    static constexpr int g = xz + G * ZS;                  // [G][GS]   gated mixer output
    static constexpr int xs = g + G * GS;                  // [G][XSR]  conv + SiLU output
    static constexpr int dbc = xs + G * XSR;               // [G][NO]   (delta, B, C)
    static constexpr int g8 = dbc + G * NO;                // [G][Di] bytes: fp8 gated rows
    static constexpr int total = g8 + G * Di / 4;          // floats
};

// One projection of the G rows of A: C[row][n] = A[row][:] . W[n][:].  The B
// operand is read in load steps (f32: one float4 = 4 MFMA k steps; bf16: one
// uint4 = one k step; fp8: one uint4 = two k steps) through a register ring
// that keeps about 16 loads per wave in flight.
template <int DT> struct BLoad;
template <> struct BLoad<0> { using T = float4; static constexpr int KPL = 16; };
template <> struct BLoad<1> { using T = uint4; static constexpr int KPL = 32; };
template <> struct BLoad<2> { using T = uint4; static constexpr int KPL = 64; };   // fp8: two k steps of 32

// A wave without work issues the same loads as the others (a branch would keep
// its ring's registers alive around it, and spilled up to 1.4 KB a thread), of the
// first fragments, which it does not use.  Every load lies in its matrix: the
// range check drops what a vector offset takes past the range, but whether it
// counts the scalar offset is the hardware's matter, and a vector offset out of
// range costs a register more than a load of what other waves load too (16 lanes of
// d_model 256 in bf16: 193 us a step against 185).  Where that load costs time (RGemm
// at two lanes: 89.0 us a step of d_model 256, 86.8 without; XRows at d_model 128:
// 12.0 and 11.9) such a wave's range is empty besides, and the memory system drops it;
// with 16 lanes the empty range costs up to 7 %.  load_ok: the 16 bytes at (vo, so)
// lie in the matrix; checked for every wave when this is compiled.
constexpr bool load_ok(int vo, int so, int bytes) { return so >= 0 && vo >= 0 && vo + so + 16 <= bytes; }

// The NF fragments of W are dealt to the waves (wave w owns w, w + 8, ...),
// at most 8 per pass.  issue() requests the first ring of B loads of the
// wave's first pass; it can be called a phase early so the loads arrive while
// other work runs.  run() completes the product and calls f(row, n, v) for
// every output (fp8: rescaled by the row and weight scales).
// fp8: the A rows are E4M3 bytes (row stride 4 * as bytes, scaled by 2^-ea of
// their row).
template <int DT, int G, int K, int NF>
struct FGemm {
    using BT = typename BLoad<DT>::T;
    static constexpr int FALL = (NF + FNW - 1) / FNW;      // fragments per wave
    static constexpr int FPW = FALL < 8 ? FALL : 8;        // per pass
    static constexpr int SK = K / BLoad<DT>::KPL;          // load steps per fragment
    static constexpr int PW = 16 / FPW > 0 ? 16 / FPW : 1;
    static constexpr int P = PW < SK ? PW : SK;            // load steps in flight (power of 2, divides SK)
    static_assert(SK % P == 0, "ring period");
    BT ring[P][FPW];

    // Weight loads are raw buffer loads: the fragment offset (wave-uniform,
    // f0 comes from a scalar) goes in a scalar register, the lane offset is
    // the one vector register, so a load costs no address arithmetic.
    static constexpr int ES = DT == 0 ? 4 : (DT == 1 ? 2 : 1);   // bytes per weight
    static constexpr int RANGE = 16 * NF * K * ES;               // the whole fragment-ordered matrix (16 NF x K)
    static_assert(NF % FNW == 0 || NF < FNW, "a wave has work in every fragment of a pass or in none");
    __host__ __device__ static constexpr bool idle(int f0) { return NF < FNW && f0 >= NF; }
    __host__ __device__ static constexpr int soff(int f0, int st, int j) {
        return (((idle(f0) ? 0 : f0) + FNW * j) * SK + st) * 64 * (int)sizeof(BT);
    }
    static constexpr bool loads_ok() {
        for (int p = 0; p < FALL; p += FPW)
            for (int wv = 0; wv < FNW; ++wv)
                for (int j = 0; j < FPW; ++j)
                    for (int wl = 0; wl < 64; wl += 63)
                        if (!load_ok(wl * (int)sizeof(BT), soff(wv + FNW * p, SK - 1, j), RANGE)) return false;
        return true;
    }
    DEVI static __amdgpu_buffer_rsrc_t rsrc(const void* Wf) {
        static_assert(loads_ok(), "loads past the matrix");
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(Wf), (short)0, RANGE, 0x00020000);   // base, stride 0
    }
    DEVI static BT ld(__amdgpu_buffer_rsrc_t r, int f0, int st, int j, int wl) {
        typedef unsigned int u4v __attribute__((ext_vector_type(4)));
        const u4v v = __builtin_amdgcn_raw_buffer_load_b128(r, wl * (int)sizeof(BT), soff(f0, st, j), 0);
        BT o;
        __builtin_memcpy(&o, &v, sizeof(BT));
        return o;
    }
    DEVI void issue(const void* Wf, int f0, int wl) {
        const __amdgpu_buffer_rsrc_t r = rsrc(Wf);
#pragma unroll
        for (int u = 0; u < P; ++u)
#pragma unroll
            for (int j = 0; j < FPW; ++j) ring[u][j] = ld(r, f0, u, j, wl);
    }
    // the pass over fragments f0, f0 + 8, ... whose first ring is in flight
    // (f1 >= 0: the ring goes on with the first loads of the pass at f1)
    template <class F>
    DEVI void pass(const float* __restrict__ A, int as, const void* __restrict__ Wf, const unsigned* amax_rows,
                   int ew, int wl, int f0, int f1, F& f) {
        const int li = wl & 15, lk = wl >> 4;
        const bool arow = li < G;
        const __amdgpu_buffer_rsrc_t rs = rsrc(Wf);
        v4f acc[FPW];
#pragma unroll
        for (int j = 0; j < FPW; ++j) acc[j] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s0 = 0; s0 < SK; s0 += P) {
#pragma unroll
            for (int u = 0; u < P; ++u) {
                const int st = s0 + u;
                BT cur[FPW];
#pragma unroll
                for (int j = 0; j < FPW; ++j) cur[j] = ring[u][j];
                if (st + P < SK) {
#pragma unroll
                    for (int j = 0; j < FPW; ++j) ring[u][j] = ld(rs, f0, st + P, j, wl);
                } else if (f1 >= 0) {
#pragma unroll
                    for (int j = 0; j < FPW; ++j) ring[u][j] = ld(rs, f1, u, j, wl);
                }
                if (DT == 0) {
                    float av[4];
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj) av[jj] = arow ? A[li * as + 16 * st + 4 * jj + lk] : 0.0f;
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj)
#pragma unroll
                        for (int j = 0; j < FPW; ++j) {
                            const float4 c4 = *reinterpret_cast<const float4*>(&cur[j]);
                            const float b = jj == 0 ? c4.x : jj == 1 ? c4.y : jj == 2 ? c4.z : c4.w;
                            acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[jj], b, acc[j], 0, 0, 0);
                        }
                } else if (DT == 2) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        uint64_t a8 = 0;
                        if (arow)
                            a8 = *reinterpret_cast<const uint64_t*>(reinterpret_cast<const uint8_t*>(A) + li * 4 * as +
                                                                    32 * (2 * st + h) + 8 * lk);
#pragma unroll
                        for (int j = 0; j < FPW; ++j) {
                            const uint4 c4 = *reinterpret_cast<const uint4*>(&cur[j]);
                            const uint64_t b8 = h == 0 ? ((uint64_t)c4.x | ((uint64_t)c4.y << 32))
                                                       : ((uint64_t)c4.z | ((uint64_t)c4.w << 32));
                            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8((long)a8, (long)b8, acc[j], 0, 0, 0);
                        }
                    }
                } else {
                    // bf16: the A rows were rounded to bf16 when written (row
                    // stride 2 * as halves in the same buffer)
                    uint4 uu = make_uint4(0, 0, 0, 0);
                    if (arow)
                        uu = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(A) + li * 2 * as +
                                                             32 * st + 8 * lk);
                    const v8bf av = *reinterpret_cast<const v8bf*>(&uu);
#pragma unroll
                    for (int j = 0; j < FPW; ++j)
                        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            av, *reinterpret_cast<const v8bf*>(&cur[j]), acc[j], 0, 0, 0);
                }
            }
        }
        if (DT == 2) {
#pragma unroll
            for (int j = 0; j < FPW; ++j)
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    const int row = 4 * lk + rr;
                    if (row < G) acc[j][rr] = ldexpf(acc[j][rr], fp8_exp(__uint_as_float(amax_rows[row])) + ew);
                }
        }
#pragma unroll
        for (int j = 0; j < FPW; ++j) {
            const int nf = f0 + FNW * j;
            if (nf >= NF) continue;
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
                if (4 * lk + rr < G) f(4 * lk + rr, 16 * nf + li, acc[j][rr]);
        }
    }
    // every pass of wave wv; the first pass's ring must have been issued
    // (fp8: amax_rows are the A rows' largest magnitudes as float bits, ew
    // W's scale exponent)
    template <class F>
    DEVI void run(const float* __restrict__ A, int as, const void* __restrict__ Wf, int wl, int wv,
                  const unsigned* amax_rows, const int* ewp, F&& f) {
        const int ew = DT == 2 ? *ewp : 0;
#pragma unroll 1
        for (int p = 0; p < FALL; p += FPW)
            pass(A, as, Wf, amax_rows, ew, wl, wv + FNW * p, p + FPW < FALL ? wv + FNW * (p + FPW) : -1, f);
    }
};

// The same product in f32 for one or two rows, on the vector ALU: the MFMA adds
// its four products one after another, each with a single rounding, exactly as
// fmaf in increasing k does, and takes the same time for 1 row as for 16 -- 164k
// cycles of a step of d_model 256, where 5 MB of weights arrive in 85k and a
// row's fmaf take 20k.  Each lane owns one column of four fragments' 64 (column
// lane % 16 of fragment lane / 16) and reads the fragment order's k = 4 j + lk
// values as four float4; sets of four fragments are dealt to the waves.  A step
// of one lane took 101 us with the MFMA and takes 60 so (two lanes: 123 and
// 84; four: 135 and 148).
template <int G, int K, int NF>
struct RGemm {
    static constexpr int NS = NF / 4, SPW = NS > FNW ? NS / FNW : 1;   // sets; per wave
    static constexpr int SP = SPW < 2 ? SPW : 2;                       // per pass
    // k groups in flight; with two rows and a product of at most two rings' length
    // one, since the compiler lays both rings and the rows' operands out at once: at
    // d_model 128 that spilled 118 registers, 49.6 us a step of 256 workgroups
    // (31.5 with a ring of two, 28.6 with one, 32.3 on the MFMA; d_model 64: 17.4 and 16.3)
    static constexpr int SK = K / 16, PW = 4 / SP, P = G == 2 && SK <= 8 ? 1 : PW < SK ? PW : SK;
    static_assert(NF % 4 == 0 && (NS <= FNW || NS % FNW == 0) && SPW % SP == 0 && SK % P == 0, "whole sets and rings");
    f32x4 ring[P][SP][4];
    static constexpr int RANGE = 16 * NF * K * 4;
    __host__ __device__ static constexpr bool idle(int wv) { return wv >= NS; }
    __host__ __device__ static constexpr int voff(int wl) { return ((wl >> 4) * SK * 64 + (wl & 15)) * 16; }
    __host__ __device__ static constexpr int soff(int wv, int s, int q, int lk) {   // set wv + 8 s
        return ((4 * ((idle(wv) ? 0 : wv) + FNW * s) * SK + q) * 64 + 16 * lk) * 16;
    }
    static constexpr bool loads_ok() {
        for (int wv = 0; wv < FNW; ++wv)
            for (int s = 0; s < SPW; ++s)
                for (int wl = 0; wl < 64; wl += 63)
                    if (!load_ok(voff(wl), soff(wv, s, SK - 1, 3), RANGE)) return false;
        return true;
    }
    DEVI static __amdgpu_buffer_rsrc_t rsrc(const void* Wf, int wv) {
        static_assert(loads_ok(), "loads past the matrix");
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(Wf), (short)0, G == 2 && idle(wv) ? 0 : RANGE,
                                                 0x00020000);
    }
    DEVI static f32x4 ld(__amdgpu_buffer_rsrc_t r, int wv, int s, int q, int lk, int vo) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, vo, soff(wv, s, q, lk), 0);
        f32x4 o;
        __builtin_memcpy(&o, &v, sizeof o);
        return o;
    }
    DEVI void issue(const void* Wf, int wv, int wl) {
        const __amdgpu_buffer_rsrc_t r = rsrc(Wf, wv);
        const int vo = voff(wl);
#pragma unroll
        for (int u = 0; u < P; ++u)
#pragma unroll
            for (int s = 0; s < SP; ++s)
#pragma unroll
                for (int lk = 0; lk < 4; ++lk) ring[u][s][lk] = ld(r, wv, s, u, lk, vo);
    }
    template <class F>
    DEVI void run(const float* __restrict__ A, int as, const void* __restrict__ Wf, int wl, int wv, const unsigned*,
                  const int*, F&& f) {
        if (idle(wv)) return;
        const __amdgpu_buffer_rsrc_t r = rsrc(Wf, wv);
        const int vo = voff(wl);
#pragma unroll 1
        for (int p = 0; p < SPW; p += SP) {
            float acc[SP][G];
#pragma unroll
            for (int s = 0; s < SP; ++s)
#pragma unroll
                for (int g = 0; g < G; ++g) acc[s][g] = 0.0f;
            // one ring of k groups from q0, refilled with those of pass pn from qn
            auto period = [&](int q0, int pn, int qn, bool refill) {
#pragma unroll
                for (int u = 0; u < P; ++u) {
                    f32x4 w[SP][4];
#pragma unroll
                    for (int s = 0; s < SP; ++s)
#pragma unroll
                        for (int lk = 0; lk < 4; ++lk) w[s][lk] = ring[u][s][lk];
                    if (refill) {
#pragma unroll
                        for (int s = 0; s < SP; ++s)
#pragma unroll
                            for (int lk = 0; lk < 4; ++lk) ring[u][s][lk] = ld(r, wv, pn + s, qn + u, lk, vo);
                    }
#pragma unroll
                    for (int g = 0; g < G; ++g)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const f32x4 x = *reinterpret_cast<const f32x4*>(A + g * as + 16 * (q0 + u) + 4 * j);
#pragma unroll
                            for (int lk = 0; lk < 4; ++lk)
#pragma unroll
                                for (int s = 0; s < SP; ++s) acc[s][g] = fmaf(x[lk], w[s][lk][j], acc[s][g]);
                        }
                }
            };
#pragma unroll 1
            for (int q0 = 0; q0 + P < SK; q0 += P) period(q0, p, q0 + P, true);
            if (p + SP < SPW) period(SK - P, p + SP, 0, true);
            else period(SK - P, 0, 0, false);
#pragma unroll
            for (int s = 0; s < SP; ++s)
#pragma unroll
                for (int g = 0; g < G; ++g) f(g, 16 * (4 * (wv + FNW * (p + s)) + (wl >> 4)) + (wl & 15), acc[s][g]);
        }
    }
};
template <int DT, int G, int K, int NF>
using Gemm = typename std::conditional<DT == 0 && G <= 2, RGemm<(G <= 2 ? G : 1), K, NF>, FGemm<DT, G, K, NF>>::type;

// LayerNorm of the G residual rows into a_s.  With G >= 8 a wave takes whole
// rows (w, w + 8); with fewer rows the waves share them, wave w normalising the
// 64 elements 64 w % D .. of row 64 w / D (512 elements a pass) after taking
// that row's statistics itself: every wave that reads a row gets the same
// values (ln_stats_v), so no barrier separates statistics from normalisation.
// Either way a thread's elements lie in the same columns of every row (D
// divides 512), so it loads their weights and biases once, ahead of the phase.
template <int D, int G, bool F8>
struct LnPre {
    static constexpr int NV = D / 64;
    static constexpr int NE = G >= FNW || F8 ? NV : 1;   // fp8: every wave needs the whole row's maximum
    float w[NE], b[NE];
    DEVI void load(const float* lw, const float* lb, int wl, int wv) {
        if (G < FNW && 64 * wv >= G * D) return;
#pragma unroll
        for (int j = 0; j < NE; ++j) {
            const int k = NE == 1 ? (64 * wv) % D + wl : 64 * j + wl;
            w[j] = gld(lw + k);
            b[j] = gld(lb + k);
        }
    }
};
// B16: the normalised rows are stored rounded to bf16 (the GEMM's A operand
// in bf16 mode), row stride 2 * ds halves.
// F8: the row's largest normalised magnitude goes to amax_s and the elements
// are stored as E4M3 bytes scaled by 2^-ea (row stride 4 * ds bytes), the A
// operand of the fp8 GEMM.
template <int D, int G, bool B16 = false, bool F8 = false>
DEVI void fused_ln(const float* __restrict__ r_s, float* __restrict__ a_s, int ds, const LnPre<D, G, F8>& pre, int wl,
                   int wv, unsigned* amax_s = nullptr) {
    constexpr int NV = D / 64;
    static_assert(D % 64 == 0 && FNT % D == 0, "rows of whole waves, fixed columns per thread");
    auto put = [&](int row, int k, float y, float am) {
        if (F8) reinterpret_cast<uint8_t*>(a_s)[row * 4 * ds + k] = fp8_byte(ldexpf(y, -fp8_exp(am)));
        else if (B16) reinterpret_cast<uint16_t*>(a_s)[row * 2 * ds + k] = f2bf_bits(y);
        else a_s[row * ds + k] = y;
    };
    if constexpr (G >= FNW) {
        float v[G / FNW][NV];
#pragma unroll
        for (int q = 0; q < G / FNW; ++q)
#pragma unroll
            for (int j = 0; j < NV; ++j) v[q][j] = r_s[(wv + FNW * q) * D + wl + 64 * j];
#pragma unroll
        for (int q = 0; q < G / FNW; ++q) {
            const int row = wv + FNW * q;
            float mu, rs, am = 0.0f;
            ln_stats_v<NV>(v[q], D, mu, rs);
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                v[q][j] = ln_apply(v[q][j], mu, rs, pre.w[j], pre.b[j]);
                if (F8) am = fmaxf(am, fabsf(v[q][j]));
            }
            if (F8) {
                am = wave_max(am);
                if (wl == 0) amax_s[row] = __float_as_uint(am);
            }
#pragma unroll
            for (int j = 0; j < NV; ++j) put(row, 64 * j + wl, v[q][j], am);
        }
    } else {
#pragma unroll
        for (int i1 = 0; i1 < G * D; i1 += FNT) {
            const int i0 = i1 + 64 * wv;                     // wave-uniform
            if (i0 >= G * D) break;
            const int row = i0 / D, kw = (64 * wv) % D;
            float v[NV];
#pragma unroll
            for (int j = 0; j < NV; ++j) v[j] = r_s[row * D + wl + 64 * j];
            float mu, rs, am = 0.0f;
            ln_stats_v<NV>(v, D, mu, rs);
            if (F8) {
#pragma unroll
                for (int j = 0; j < NV; ++j) am = fmaxf(am, fabsf(ln_apply(v[j], mu, rs, pre.w[F8 ? j : 0], pre.b[F8 ? j : 0])));
                am = wave_max(am);
                if (kw == 0 && wl == 0) amax_s[row] = __float_as_uint(am);
            }
            float x = 0.0f, g = pre.w[0], bb = pre.b[0];
#pragma unroll
            for (int j = 0; j < NV; ++j)
                if (64 * j == kw) {
                    x = v[j];
                    if (F8) { g = pre.w[F8 ? j : 0]; bb = pre.b[F8 ? j : 0]; }
                }
            put(row, kw + wl, ln_apply(x, mu, rs, g, bb), am);
        }
    }
    __syncthreads();
}

// x_proj of the G rows of xs_s into dbc_s, the four chains per output of
// xproj_fragment.  Left to one wave per column fragment, as the step kernels
// have it, it was half of a step (48k of 97k cycles at one lane of d_model 256:
// 128 dependent MFMAs behind a ring of four loads); both forms below start
// their weight loads before the conv phase and use more of the waves.
//
// One or two rows: on the vector ALU.  The f32 16x16x4 MFMA adds its four
// products one after another, each with a single rounding, exactly as fmaf in
// increasing k does, so lane (c = lane / 16, lane % 16) of wave f + 4 r runs
// chain c of output 16 f + lane % 16 of row r and the chains meet by lane
// exchanges.  A matrix instruction spends the same time on 1 row
// as on 16.  One lane of d_model 256: 6.8k cycles a step.
template <int Di, int NFX, int NO, int G>
struct XRows {
    static constexpr int SQ = Di / 16, NG = SQ / 4, PG = NG < 4 ? NG : NG > 8 ? 8 : 4;
    static_assert(G <= 2 && NFX <= 4 && FNW == 8, "a wave per (fragment, row)");
    f32x4 ring[PG][4];
    static constexpr int RANGE = 16 * NFX * Di * 4;
    __host__ __device__ static constexpr bool mine(int wv) { return (wv & 3) < NFX && (wv >> 2) < G; }
    __host__ __device__ static constexpr int voff(int wl) { return ((wl >> 4) * 64 + (wl & 15)) * 16; }
    __host__ __device__ static constexpr int soff(int wv, int i, int lk) {
        return (((mine(wv) ? wv & 3 : 0) * SQ + 4 * i) * 64 + 16 * lk) * 16;
    }
    static constexpr bool loads_ok() {
        for (int wv = 0; wv < FNW; ++wv)
            for (int wl = 0; wl < 64; wl += 63)
                if (!load_ok(voff(wl), soff(wv, NG - 1, 3), RANGE)) return false;
        return true;
    }
    DEVI static f32x4 ld(const float* Wf, int wv, int wl, int i, int lk) {
        static_assert(loads_ok(), "loads past the matrix");
        const __amdgpu_buffer_rsrc_t r =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(Wf), (short)0, mine(wv) ? RANGE : 0, 0x00020000);
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, voff(wl), soff(wv, i, lk), 0);
        f32x4 o;
        __builtin_memcpy(&o, &v, sizeof o);
        return o;
    }
    DEVI void issue(const float* Wf, int wv, int wl) {
#pragma unroll
        for (int i = 0; i < PG; ++i)
#pragma unroll
            for (int lk = 0; lk < 4; ++lk) ring[i][lk] = ld(Wf, wv, wl, i, lk);
    }
    DEVI void run(const float* xs, int xsr, const float* Wf, int wv, int wl, float* dbc) {
        if (!mine(wv)) return;
        float acc = 0.0f;
        const float* xrow = xs + (wv >> 2) * xsr + 16 * (wl >> 4);
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            f32x4 w[4];
#pragma unroll
            for (int lk = 0; lk < 4; ++lk) w[lk] = ring[i % PG][lk];
            if (i + PG < NG) {
#pragma unroll
                for (int lk = 0; lk < 4; ++lk) ring[i % PG][lk] = ld(Wf, wv, wl, i + PG, lk);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x4 xv = *reinterpret_cast<const f32x4*>(xrow + 64 * i + 4 * j);
#pragma unroll
                for (int lk = 0; lk < 4; ++lk) acc = fmaf(xv[lk], w[lk][j], acc);
            }
        }
        const int n = 16 * (wv & 3) + (wl & 15);
        float v = acc + __shfl_xor(acc, 16);                 // chains 0 + 1, 2 + 3
        v = v + __shfl_xor(v, 32);
        if (wl < 16 && n < NO) dbc[(wv >> 2) * NO + n] = v;
    }
};
// More rows: on the matrix cores, wave f + 4 h chains 2 h and 2 h + 1 of
// column fragment f; the halves are added through part [2][G][16 NFX].  16
// lanes of d_model 256: 45k cycles a step before, 20k so.
template <int Di, int NFX, int NO, int G>
struct XTile {
    static constexpr int SQ = Di / 16, NG = SQ / 4, PG = NG < 4 ? NG : 4, PN = 16 * NFX;
    f32x4 ring[PG][2];
    static constexpr int RANGE = 16 * NFX * Di * 4;
    __host__ __device__ static constexpr bool mine(int wv) { return (wv & 3) < NFX; }
    __host__ __device__ static constexpr int soff(int wv, int i, int c) {
        return ((mine(wv) ? wv & 3 : 0) * SQ + 4 * i + 2 * (wv >> 2) + c) * 1024;
    }
    static constexpr bool loads_ok() {
        for (int wv = 0; wv < FNW; ++wv)
            for (int wl = 0; wl < 64; wl += 63)
                if (!load_ok(wl * 16, soff(wv, NG - 1, 1), RANGE)) return false;
        return true;
    }
    DEVI static f32x4 ld(const float* Wf, int wv, int wl, int i, int c) {
        static_assert(loads_ok(), "loads past the matrix");
        const __amdgpu_buffer_rsrc_t r =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(Wf), (short)0, RANGE, 0x00020000);
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, wl * 16, soff(wv, i, c), 0);
        f32x4 o;
        __builtin_memcpy(&o, &v, sizeof o);
        return o;
    }
    DEVI void issue(const float* Wf, int wv, int wl) {
#pragma unroll
        for (int i = 0; i < PG; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c) ring[i][c] = ld(Wf, wv, wl, i, c);
    }
    DEVI void run(const float* xs, int xsr, const float* Wf, int wv, int wl, int tid, float* part, float* dbc) {
        if (mine(wv)) {
            const int li = wl & 15, lk = wl >> 4;
            const float* x = xs + (li < G ? li : 0) * xsr + 32 * (wv >> 2) + lk;
            v4f acc[2] = {v4f{0.f, 0.f, 0.f, 0.f}, v4f{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int i = 0; i < NG; ++i) {
                f32x4 w[2];
#pragma unroll
                for (int c = 0; c < 2; ++c) w[c] = ring[i % PG][c];
                if (i + PG < NG) {
#pragma unroll
                    for (int c = 0; c < 2; ++c) ring[i % PG][c] = ld(Wf, wv, wl, i + PG, c);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int c = 0; c < 2; ++c)      // rows from G on: a copy of row 0, not stored
                        acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[64 * i + 16 * c + 4 * j], w[c][j], acc[c], 0, 0, 0);
            }
            const int n = 16 * (wv & 3) + li;
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const int row = 4 * lk + rr;
                if (row < G) part[((wv >> 2) * G + row) * PN + n] = acc[0][rr] + acc[1][rr];
            }
        }
        __syncthreads();
        for (int i = tid; i < G * NO; i += FNT) {
            const int row = i / NO, n = i % NO;
            dbc[i] = part[row * PN + n] + part[(G + row) * PN + n];
        }
    }
};
}  // namespace

// SL: the lanes' conv and scan state live in LDS after the activations
// ([n_layers][G][K-1][Di] then [n_layers][G][N][Di]) instead of device memory.
// Without SL the state lives in device memory, one record per (layer, lane):
// conv window [K-1][Di] (tap t in slot t % 3) and h [N/4][Di] float4, so the
// accesses of a wave are contiguous.
//
// Decoding waves: wave w decodes lanes w, w + 8, ... of the workgroup (one
// lane per wave up to G = 8, two at G = 16).
template <int DT, int D, int Di, int RR, int G, bool SL>
__global__ __launch_bounds__(FNT) void k_dec_fused(FusedArgs a) {
    using S = FusedLds<D, Di, RR, G>;
    constexpr int NO = S::NO, ZS = S::ZS;
    constexpr int LPW = (G + FNW - 1) / FNW;      // lanes decoded per wave
    static_assert(G >= 1 && G <= 16, "at most 16 lanes (one MFMA tile of rows) per workgroup");
    static_assert(!SL || G == 1, "state in LDS with one lane per workgroup only");
    extern __shared__ __align__(16) float sm[];
    float* r_s = sm + S::r;
    float* a_s = sm + S::a;
    float* xz_s = sm + S::xz;
    float* g_s = sm + S::g;
    float* xs_s = sm + S::xs;
    float* dbc_s = sm + S::dbc;
    uint8_t* g8_s = reinterpret_cast<uint8_t*>(sm + S::g8);
    float* cst_s = sm + S::total;                                  // SL only
    float* hst_s = cst_s + (size_t)a.n_layers * G * (KCONV - 1) * Di;
    __shared__ int pos_s[G];
    __shared__ float hb_s[VOCAB];                 // head bias, read every step
    __shared__ unsigned am_ln[G], am_g[G];        // fp8: row maxima of the LayerNorm output and of g
    // wave index as a wave-uniform (scalar) value: weight addresses that depend
    // only on it are formed in scalar registers
    int tid = threadIdx.x, wl = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    // The thread index is made opaque once per phase group: addresses formed
    // from it are then recomputed there (a few integer operations) instead of
    // being kept in registers over the whole step, which spilled.
    auto fresh = [&]() {
        asm volatile("" : "+v"(tid));
        wl = tid & 63;
    };
    const int lane0 = blockIdx.x * G;

    for (int i = tid; i < S::total; i += FNT) sm[i] = 0.0f;
    for (int i = tid; i < VOCAB; i += FNT) hb_s[i] = a.head_b[i];
    // Per decoded lane of this wave: its schedule position, range decoder and
    // the current chunk's payload, output offset and step count (read once
    // per chunk instead of every step).  Decoded bytes gather in the decoding
    // wave's lanes, lane i holding the byte at offset i of the current
    // 64-byte output block; they leave in one store when the block or the
    // chunk ends.
    struct LaneDec {
        int c, pos;
        long long lstep;
        Dec dc;
        const uint8_t* pin;
        uint32_t plen;
        long long obase;
        int csteps;
        uint32_t obyte, pbyte;
    };
    LaneDec ld[LPW];
    auto enter_chunk = [&](LaneDec& q, int ch) {
        q.pin = a.payload + a.pay_off[ch];
        q.plen = (uint32_t)a.pay_len[ch];
        q.obase = a.p.chunk_off[ch];
        q.csteps = a.p.chunk_steps[ch];
    };
#pragma unroll
    for (int k = 0; k < LPW; ++k) {
        LaneDec& q = ld[k];
        q.c = -1; q.pos = -1; q.lstep = 0; q.dc = Dec{}; q.pin = nullptr; q.plen = 0; q.obase = 0; q.csteps = 0;
        q.obyte = 0; q.pbyte = 0;
        const int gl = wv + FNW * k;
        if (gl < G && lane0 + gl < a.lanes) locate(a.p, lane0 + gl, 0, q.c, q.pos);
        if (gl < G && q.pos >= 0) enter_chunk(q, q.c);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < LPW; ++k) {
        const LaneDec& q = ld[k];
        const int gl = wv + FNW * k;
        if (gl < G) {
            if (q.pos >= 0) {
                const int y = a.out[q.obase + q.pos];
                const float* er = a.E + (long long)y * D;
                for (int kk = wl; kk < D; kk += 64) r_s[gl * D + kk] = er[kk];
            }
            if (wl == 0) pos_s[gl] = q.pos;
        }
    }
    __syncthreads();

    // The LayerNorm weights of the next LayerNorm (layer l, or the final one
    // for l == n_layers) are requested one phase ahead
    using GIn = Gemm<DT, G, D, 2 * Di / 16>;
    LnPre<D, G, DT == 2> lnp;
    auto pre_layer = [&](int l) {
        if (l == a.n_layers) lnp.load(a.norm_f_w, a.norm_f_b, wl, wv);
        else lnp.load(a.layers[l].norm_w, a.layers[l].norm_b, wl, wv);
    };
    pre_layer(0);
    for (long long it = 0; it < a.max_steps; ++it) {
        // step position of every slot (-1: idle) as scalars, for the whole step
        int spos[G];
        bool any = false;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            spos[g] = __builtin_amdgcn_readfirstlane(pos_s[g]);
            any = any || spos[g] >= 0;
        }
        if (!any) break;                                 // uniform: read after a barrier
        // the decoding wave requests its next 8 payload bytes now, one per
        // lane (lane i: byte cur + i, zero past the payload); nothing waits
        // for them until the decoding after the model pass
#pragma unroll
        for (int k = 0; k < LPW; ++k) {
            LaneDec& q = ld[k];
            q.pbyte = 0;
            if (wv + FNW * k < G && q.pos >= 0) {
                if (q.pos == 0) dec_reset(q.dc, q.pin, q.plen);
                if (wl < 8 && q.dc.cur + (uint32_t)wl < q.plen)
                    q.pbyte = *(const __attribute__((address_space(1))) uint8_t*)(q.pin + q.dc.cur + wl);
            }
        }

        for (int l = 0; l < a.n_layers; ++l) {
            const FusedLayer& w = a.layers[l];
            fresh();
            // Weights and state are requested ahead of their phase where that
            // hides a latency without delaying other loads: the LayerNorm
            // weights during the previous out_proj (pre_layer), the conv
            // window before the LayerNorm, the conv weights, the x_proj ring and
            // the dt / scan weights before the conv, the out_proj ring at the
            // end of the scan (issued before it, the ring's registers pushed
            // the scan's state loads into spills).
            //
            // Conv window of (slot, channel): a ring of K - 1 taps [K-1][Di] in
            // LDS (SL) or in the slot's device record; tap t of a chunk is
            // slot t % 3, so a step reads three taps and writes one.
            constexpr int CPT = (Di + FNT - 1) / FNT;          // channels per thread
            constexpr int CW = SL ? 1 : CPT * G * (KCONV - 1);
            float cwin[CW];
            auto cwin_dev = [&](int g) {
                return a.conv_state + ((long long)l * a.lanes + lane0 + g) * (KCONV - 1) * Di;
            };
#pragma unroll
            for (int j = 0; j < CPT; ++j) {
                const int d = tid + FNT * j;
                if (Di % FNT && d >= Di) break;
                if (!SL) {
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        const int p = spos[g];
#pragma unroll
                        for (int k = 0; k < KCONV - 1; ++k) {
                            float v = 0.0f;
                            if (p >= KCONV - 1 - k) v = gld_nt(cwin_dev(g) + (p + k) % 3 * Di + d);
                            cwin[(j * G + g) * (KCONV - 1) + k] = v;
                        }
                    }
                }
            }
            // the in_proj ring goes out before the LayerNorm (fp8: after it;
            // there the early ring cost more than it hid)
            GIn gin;
            if (DT != 2) gin.issue(w.in_frag, wv, wl);
            fused_ln<D, G, DT == 1, DT == 2>(r_s, a_s, S::DS, lnp, wl, wv, am_ln);
            if (DT == 2) gin.issue(w.in_frag, wv, wl);
            gin.run(a_s, S::DS, w.in_frag, wl, wv, am_ln, w.in_ew, [&](int row, int n, float v) {
                if (n < Di) xs_s[row * S::XSR + n] = v;
                else xz_s[row * ZS + (n - Di)] = v;
            });
            constexpr bool ONE = Di <= FNT;                    // one channel per thread in the scan
            DtW<DT, RR> pdtw;
            float pA2[NSTATE], pdtb = 0.0f, pDk = 0.0f;
            if (ONE && tid < Di) {
                pdtw.load(w, Di, tid);
#pragma unroll
                for (int n = 0; n < NSTATE; ++n) pA2[n] = gld(w.A2T + n * Di + tid);
                pdtb = gld(w.dtb + tid);
                pDk = gld(w.Dsk + tid);
            }
            constexpr int NFX = (NO + 15) / 16;
            typename std::conditional<(G <= 2), XRows<Di, NFX, NO, (G <= 2 ? G : 1)>, XTile<Di, NFX, NO, G>>::type xp;
            __builtin_amdgcn_sched_barrier(0);       // not among the product's loads: registers
            float ccw[CPT][KCONV], ccb[CPT];
#pragma unroll
            for (int j = 0; j < CPT; ++j) {
                const int d = tid + FNT * j;
                if (Di % FNT && d >= Di) break;
#pragma unroll
                for (int k = 0; k < KCONV; ++k) ccw[j][k] = gld(w.convT + k * Di + d);
                ccb[j] = gld(w.conv_b + d);
            }
            xp.issue(w.xw_frag, wv, wl);
            __syncthreads();
            fresh();
            // causal conv + SiLU in place, a thread per channel, advancing the
            // window (in in_proj's epilogue it read the window in 64-byte pieces
            // after the product: 122k cycles a step of 16 lanes of d_model 256
            // there, 45k in the product and 21k here so)
#pragma unroll
            for (int j = 0; j < CPT; ++j) {
                const int d = tid + FNT * j;
                if (Di % FNT && d >= Di) break;
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int p = spos[g];
                    if (p < 0) continue;
                    float t[KCONV - 1];
                    float* cl = cst_s + (l * G + g) * (KCONV - 1) * Di + d;
#pragma unroll
                    for (int k = 0; k < KCONV - 1; ++k) {
                        if (SL) t[k] = p >= KCONV - 1 - k ? cl[(p + k) % 3 * Di] : 0.0f;
                        else t[k] = cwin[(j * G + g) * (KCONV - 1) + k];
                    }
                    const float x = xs_s[g * S::XSR + d];
                    xs_s[g * S::XSR + d] = conv_silu(ccw[j], ccb[j], t[0], t[1], t[2], x);
                    if (SL) cl[p % 3 * Di] = x;
                    else gst_nt(cwin_dev(g) + p % 3 * Di + d, x);
                }
            }
            __syncthreads();
            // The scan state of DP lane slots is in flight at a time, the first
            // ones' during x_proj.  h of slot g: LDS [N][Di] (SL) or the slot's
            // device record [N/4][Di] float4 (a wave's access is 1 KiB
            // contiguous).  A slot's 16 states go together: in parts of 4 or 8
            // states of 8 or 4 slots, with as many loads in flight, a step of 16
            // lanes of d_model 256 took 212 and 202 us, so 187: 4.8 TB/s, what a
            // plain copy reaches.
            constexpr int DP = G < 4 ? G : 4;
            static_assert(G % DP == 0, "the ring closes on the next channel");
            float hp[DP][NSTATE];
            auto hrec = [&](int g, int d) {
                return reinterpret_cast<float4*>(a.h_state) + ((long long)l * a.lanes + lane0 + g) * (NSTATE / 4) * Di + d;
            };
            auto load_slot = [&](int d, int g) {
                float (&h)[NSTATE] = hp[g % DP];
                const bool live = spos[g] > 0;
                if (SL) {
                    const float* hst = hst_s + (l * G + g) * NSTATE * Di;
#pragma unroll
                    for (int n = 0; n < NSTATE; ++n) h[n] = live ? hst[n * Di + d] : 0.0f;
                } else {
#pragma unroll
                    for (int q = 0; q < NSTATE / 4; ++q) {
                        float4 v4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                        if (live) v4 = gld_nt(hrec(g, d) + q * Di);
                        h[4 * q] = v4.x; h[4 * q + 1] = v4.y;
                        h[4 * q + 2] = v4.z; h[4 * q + 3] = v4.w;
                    }
                }
            };
            if (Di % FNT == 0 || tid < Di) {
#pragma unroll
                for (int g = 0; g < DP; ++g) load_slot(tid, g);
            }
            if constexpr (G <= 2) xp.run(xs_s, S::XSR, w.xw_frag, wv, wl, dbc_s);
            else xp.run(xs_s, S::XSR, w.xw_frag, wv, wl, tid, g_s, dbc_s);
            if (DT == 2 && tid < G) am_g[tid] = 0u;
            using GOut = Gemm<DT, G, Di, D / 16>;
            GOut gout;
            __syncthreads();
            fresh();
            // dt_proj + softplus, selective scan, gate
            for (int d = tid; d < Di; d += FNT) {
                float dtw[RR], A2[NSTATE], dtb, Dk;
                if (ONE) {
                    pdtw.get(dtw);
#pragma unroll
                    for (int n = 0; n < NSTATE; ++n) A2[n] = pA2[n];
                    dtb = pdtb;
                    Dk = pDk;
                } else {
                    {
                        DtW<DT, RR> t;
                        t.load(w, Di, d);
                        t.get(dtw);
                    }
#pragma unroll
                    for (int n = 0; n < NSTATE; ++n) A2[n] = gld(w.A2T + n * Di + d);
                    dtb = gld(w.dtb + d);
                    Dk = gld(w.Dsk + d);
                }
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    if (spos[g] >= 0) {
                        float (&h)[NSTATE] = hp[g % DP];
                        const float* dbc = dbc_s + g * NO;
                        const float gv = scan_update(h, dt_of<RR>(dbc, dtw, dtb), xs_s[g * S::XSR + d], dbc + RR,
                                                     dbc + RR + NSTATE, A2, Dk, xz_s[g * ZS + d]);
                        if (SL) {
                            float* hst = hst_s + (l * G + g) * NSTATE * Di;
#pragma unroll
                            for (int n = 0; n < NSTATE; ++n) hst[n * Di + d] = h[n];
                        } else {
#pragma unroll
                            for (int q = 0; q < NSTATE / 4; ++q)
                                gst_nt(hrec(g, d) + q * Di, make_float4(h[4 * q], h[4 * q + 1], h[4 * q + 2], h[4 * q + 3]));
                        }
                        if (DT == 1) reinterpret_cast<uint16_t*>(g_s)[g * 2 * S::GS + d] = f2bf_bits(gv);
                        else g_s[g * S::GS + d] = gv;
                        if (DT == 2) {            // row maximum: per wave first, then one LDS atomic per wave
                            const float wm = wave_max(fabsf(gv));
                            if (wl == 0) atomicMax(&am_g[g], __float_as_uint(wm));
                        }
                    }
                    if (g + DP < G) load_slot(d, g + DP);
                    else if (Di > FNT && d + FNT < Di) load_slot(d + FNT, g + DP - G);
                }
            }
            fresh();
            gout.issue(w.out_frag, wv, wl);
            __syncthreads();
            pre_layer(l + 1);
            if (DT == 2) {
                // the gated rows as E4M3 bytes scaled by 2^-ea of their row (the
                // row maxima are complete)
                for (int d = tid; d < Di; d += FNT) {
#pragma unroll
                    for (int g = 0; g < G; ++g)
                        if (pos_s[g] >= 0)
                            g8_s[g * Di + d] = fp8_byte(ldexpf(g_s[g * S::GS + d], -fp8_exp(__uint_as_float(am_g[g]))));
                }
                __syncthreads();
            }
            // out_proj, added into the residual stream
            gout.run(DT == 2 ? reinterpret_cast<float*>(g8_s) : g_s, DT == 2 ? Di / 4 : S::GS, w.out_frag, wl, wv, am_g, w.out_ew, [&](int row, int n, float v) {
                r_s[row * D + n] = r_s[row * D + n] + v;
            });
            __syncthreads();
        }
        fresh();
        using GH = Gemm<DT, G, D, VOCAB / 16>;
        GH ghead;
        if (DT != 2) ghead.issue(a.head_frag, wv, wl);   // the head ring goes out before the final LayerNorm
        fused_ln<D, G, DT == 1, DT == 2>(r_s, a_s, S::DS, lnp, wl, wv, am_ln);
        float* lg_s = xz_s;
        {
            if (DT == 2) ghead.issue(a.head_frag, wv, wl);
            ghead.run(a_s, S::DS, a.head_frag, wl, wv, am_ln, a.head_ew, [&](int row, int n, float v) {
                lg_s[row * VOCAB + n] = v + hb_s[n];
            });
        }
        pre_layer(0);                                    // the next step's first LayerNorm
        __syncthreads();

        fresh();
        // histogram, range decoding and the lane's next input row
#pragma unroll
        for (int k = 0; k < LPW; ++k) {
            LaneDec& q = ld[k];
            const int gl = wv + FNW * k;
            if (gl >= G || q.pos < 0) continue;
            const int lane = lane0 + gl;
            QRow qr = quant_row(lg_s + gl * VOCAB, wl);
            const int hit = dec_hit(q.dc, qr.cx, qr.f, wl);
            const unsigned long long bal = __ballot(hit >= 0);
            const int src = bal ? (__ffsll((long long)bal) - 1) : 0;
            int sym = __builtin_amdgcn_readlane(hit, src);  // wave-uniform lane indices: lane reads
            if (sym < 0) sym = 0;                          // unreachable for a valid stream
            const int cl = __builtin_amdgcn_readlane(qr.csel(sym & 3), sym >> 2);
            const int fs = __builtin_amdgcn_readlane(qr.fsel(sym & 3), sym >> 2);
            uint64_t pf = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) pf |= (uint64_t)(__builtin_amdgcn_readlane(q.pbyte, i) & 0xFF) << (8 * i);
            dec_update(q.dc, (uint32_t)cl, (uint32_t)fs, q.pin, q.plen, pf, true);   // every lane, same values
            const long long ob = q.obase;
            const long long oa = ob + q.pos + 1;         // this byte's output index
            const int oi = (int)(oa & 63);
            if (wl == oi) q.obyte = (uint32_t)sym;
            if (oi == 63 || q.pos + 1 >= q.csteps) {     // block full or chunk done
                // the block's bytes from the chunk's first decoded byte on
                const long long ob0 = oa - oi;
                const int lo = ob + 1 > ob0 ? (int)(ob + 1 - ob0) : 0;
                if (wl >= lo && wl <= oi) a.out[ob0 + wl] = (uint8_t)q.obyte;
            }
            int nc, npos, ny;
            if (q.pos + 1 < q.csteps) {
                nc = q.c; npos = q.pos + 1; ny = sym;
            } else {
                locate(a.p, lane, q.lstep + 1, nc, npos);
                if (npos >= 0) enter_chunk(q, nc);
                ny = npos >= 0 ? a.out[q.obase + npos] : -1;
            }
            if (ny >= 0) {
                const float* er = a.E + (long long)ny * D;
                for (int kk = wl; kk < D; kk += 64) r_s[gl * D + kk] = er[kk];
            }
            if (wl == 0) pos_s[gl] = npos;
            q.c = nc;
            q.pos = npos;
            ++q.lstep;
        }
        __syncthreads();
    }
}

size_t fused_lds_bytes(int D, int G, int n_layers, bool state_in_lds) {
    const int Di = 2 * D, RR = (D + 15) / 16, NO = RR + 2 * NSTATE;
    const int ZS = Di > VOCAB ? Di : VOCAB;
    size_t f = (size_t)G * ((size_t)D + (D + 4) + ZS + (Di + 4) + (Di + 4) + NO + Di / 4);
    if (state_in_lds) f += (size_t)n_layers * G * (KCONV - 1 + NSTATE) * Di;
    return f * sizeof(float);
}

template <int DT, int D, int G, bool SL>
hipError_t fused_launch(const FusedArgs& a, int blocks, hipStream_t s) {
    if constexpr (G * D > 16 * 256) {
        return hipErrorInvalidValue;           // beyond the LDS of one CU
    } else {
    constexpr int Di = 2 * D, RR = (D + 15) / 16;
    auto kern = k_dec_fused<DT, D, Di, RR, G, SL>;
    const size_t lds = fused_lds_bytes(D, G, a.n_layers, SL);
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    BOA_LAUNCH(kern, dim3(blocks), dim3(FNT), lds, s, a);
    return hipGetLastError();
    }
}

hipError_t launch_dec_fused(int dtype, int D, int G, bool state_in_lds, const FusedArgs& a, hipStream_t s) {
    if (a.lanes <= 0) return hipSuccess;
    const int blocks = (a.lanes + G - 1) / G;
    if (state_in_lds && G != 1) return hipErrorInvalidValue;
#define FD_G(DTV, DV)                                                                      \
    switch (G) {                                                                           \
        case 1: return state_in_lds ? fused_launch<DTV, DV, 1, true>(a, blocks, s)         \
                                    : fused_launch<DTV, DV, 1, false>(a, blocks, s);       \
        case 2: return fused_launch<DTV, DV, 2, false>(a, blocks, s);                      \
        case 4: return fused_launch<DTV, DV, 4, false>(a, blocks, s);                      \
        case 8: return fused_launch<DTV, DV, 8, false>(a, blocks, s);                      \
        case 16: return fused_launch<DTV, DV, 16, false>(a, blocks, s);                    \
        default: return hipErrorInvalidValue;                                              \
    }
#define FD_D(DTV)                          \
    switch (D) {                           \
        case 64: FD_G(DTV, 64)             \
        case 128: FD_G(DTV, 128)           \
        case 256: FD_G(DTV, 256)           \
        case 512: FD_G(DTV, 512)           \
        default: return hipErrorInvalidValue; \
    }
    if (dtype == BOA_DTYPE_FP8) { FD_D(2) } else if (dtype == BOA_DTYPE_BF16) { FD_D(1) } else { FD_D(0) }
#undef FD_D
#undef FD_G
}

}  // namespace boa
