// Integer-only predictor and coder: the deterministic pipeline the paper
// proposes for decoding on another device (Results & Discussion, portability
// and limitations).  Every projection is INT8 x INT8 with an exact INT32
// accumulation, every other quantity is a fixed-point integer with a stated
// rounding and saturation, and LayerNorm, the exponential, SiLU, softplus and
// the softmax-to-histogram step have integer forms.  Integer sums do not
// depend on their order, so the frequency tables -- and with them the coded
// bytes -- are the same on any device that follows these rules.
//
// The rules (Q formats, rounding shifts, the exponential's table and Taylor
// polynomial, the logarithm's series) are written out at the functions below.
// Weight conversion (boa_qmodel_create) runs on the host in float64 with one
// rounding per value; the kernel then sees only integers.
//
// Kernel shape: one workgroup of 256 threads per chunk walks the chunk's steps
// in order (the state is a recurrence); the conv window and scan state of the
// chunk live in a device buffer, every other vector in LDS.
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "hotpath_common.h"

namespace {

using ll = long long;
constexpr int NT = 256;
constexpr ll SAT23 = (1LL << 23) - 1;
constexpr ll SAT31 = (1LL << 31) - 1;
constexpr ll EPS_Q24 = 168;                       // rint(1e-5 * 2^24)
constexpr int QN = 16;                            // d_state

// 2^(k/16) in Q30
__constant__ ll kT16[16] = {1073741824LL, 1121280436LL, 1170923762LL, 1222764986LL, 1276901417LL, 1333434672LL,
                            1392470869LL, 1454120821LL, 1518500250LL, 1585730000LL, 1655936265LL, 1729250827LL,
                            1805811301LL, 1885761398LL, 1969251188LL, 2056437387LL};
// ln(1 + k/16) in Q30
__constant__ ll kLNC[17] = {0LL, 65095192LL, 126468572LL, 184522808LL, 239598564LL, 291986604LL,
                            341937090LL, 389666807LL, 435364845LL, 479197128LL, 521310048LL, 561833416LL,
                            600882877LL, 638561895LL, 674963409LL, 710171213LL, 744261118LL};
const ll hT16[16] = {1073741824LL, 1121280436LL, 1170923762LL, 1222764986LL, 1276901417LL, 1333434672LL,
                     1392470869LL, 1454120821LL, 1518500250LL, 1585730000LL, 1655936265LL, 1729250827LL,
                     1805811301LL, 1885761398LL, 1969251188LL, 2056437387LL};
// (ln 2)^k / k! in Q30, log2(e) in Q30, 1/5 and 1/3 in Q30
constexpr ll C1 = 744261118LL, C2 = 257941248LL, C3 = 59597083LL, C4 = 10327387LL;
constexpr ll LOG2E = 1549082005LL;
constexpr ll H5 = 214748365LL, H3 = 357913941LL;

// round(x / 2^s), half up (arithmetic shifts are floors); x 2^-s for s < 0
__host__ __device__ inline ll rsh(ll x, int s) {
    if (s > 0) return (x + (1LL << (s - 1))) >> s;
    if (s < 0) return (ll)((unsigned long long)x << (-s));
    return x;
}
__host__ __device__ inline ll clampll(ll x, ll lo, ll hi) { return x < lo ? lo : (x > hi ? hi : x); }
// exact products of operands known to fit in 32 bits (one 32 x 32 -> 64 multiply
// instead of the 64 x 64 sequence)
__host__ __device__ inline ll mul32(ll a, ll b) { return (ll)(int)a * (ll)(int)b; }
__host__ __device__ inline ll mulu32(ll a, ll b) { return (ll)((unsigned long long)(unsigned)a * (unsigned)b); }
// floor(a / b) for b > 0, |a| < 2^62, b < 2^53: the double quotient is within
// 2^-4 of a / b for every use here (numerators exact in double, or the one
// sum of squares whose rounding moves the quotient by under 1/4), so its
// floor is the answer or one off, and the integer checks settle it exactly
__device__ inline ll fdiv(ll a, ll b) {
    ll q = (ll)floor((double)a / (double)b);
    while (q * b > a) --q;
    while ((q + 1) * b <= a) ++q;
    return q;
}
// floor(a / b) for numerators exact in double, 0 <= a, 0 < b < 2^32 and a
// quotient below 2^31: the truncated double quotient is the answer or one off,
// which one remainder tells (a - q b lies within (-b, 2 b)); the loops of fdiv,
// a 64-bit product each, were a ninth of a step
__device__ inline unsigned fdiv32(ll a, unsigned b) {
    const unsigned q = (unsigned)((double)a / (double)b);
    const ll r = a - (ll)((unsigned long long)q * b);
    return r < 0 ? q - 1 : (r >= (ll)b ? q + 1 : q);
}
// 2^30 2^(g / 2^30) for 0 <= g < 2^30: 2^(k/16) from the table times a
// degree-4 Taylor polynomial of 2^u on [0, 1/16), Horner in Q30
__host__ __device__ inline ll exp2_frac(ll g, ll tk) {
    const ll u = g & ((1LL << 26) - 1);
    ll q = C4;                                    // 0 < q <= 2^31, 0 <= u < 2^26, tk < 2^31
    q = C3 + rsh(mulu32(q, u), 30);
    q = C2 + rsh(mulu32(q, u), 30);
    q = C1 + rsh(mulu32(q, u), 30);
    q = (1LL << 30) + rsh(mulu32(q, u), 30);
    return rsh(mulu32(tk, q), 30);
}
// exp(x / 2^24) in Q30 for -2^30 <= x <= 0 (0 below 2^-46), in 32-bit words: each
// product is one 32 x 32 + 64 multiply-add whose rounding is its addend and
// whose shift is the choice of its upper word (u is kept times 4, so that
// >> 30 becomes >> 32) or one funnel shift.  The intermediate ranges are those
// of exp2_frac; p < 2^31, so shifts by 32 and more round to 0.  The pipeline is
// bound by the issue of this integer arithmetic (half of a step's cycles here):
// 1024 chunks of 128 to 384 bytes, d_model 256, encoded and decoded took 118 ms
// with 64-bit values throughout, 87 with these forms, q8 and fdiv32.
// (written as the instruction: from the C expression the compiler widens an
// operand and spends two more multiplies)
__host__ __device__ inline ll mad_i(int a, int b, ll c) {
#ifdef __HIP_DEVICE_COMPILE__
    ll r;
    asm("v_mad_i64_i32 %0, vcc, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c) : "vcc");
    return r;
#else
    return (ll)a * b + c;
#endif
}
__host__ __device__ inline unsigned long long mad_u(unsigned a, unsigned b, unsigned long long c) {
#ifdef __HIP_DEVICE_COMPILE__
    unsigned long long r;
    asm("v_mad_u64_u32 %0, vcc, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c) : "vcc");
    return r;
#else
    return (unsigned long long)a * b + c;
#endif
}
__host__ __device__ inline unsigned hi32(unsigned long long v) { return (unsigned)(v >> 32); }
__host__ __device__ inline unsigned funnel(unsigned long long v, int s) { return (unsigned)(v >> s); }
__host__ __device__ inline unsigned exp_neg32(int x, const unsigned* T16) {
    const ll y = mad_i(x, (int)LOG2E, 1LL << 23);                   // y >> 24 = n 2^30 + g
    const unsigned g = funnel((unsigned long long)y, 24) & ((1u << 30) - 1);
    const unsigned sh = (unsigned)-((int)hi32((unsigned long long)y) >> 22);
    const unsigned u4 = g << 2 & ((1u << 28) - 1);
    constexpr unsigned long long HALF = 1ULL << 31;
    unsigned q = (unsigned)C4;
    q = (unsigned)C3 + hi32(mad_u(q, u4, HALF));
    q = (unsigned)C2 + hi32(mad_u(q, u4, HALF));
    q = (unsigned)C1 + hi32(mad_u(q, u4, HALF));
    q = (1u << 30) + hi32(mad_u(q, u4, HALF));
    const unsigned p = funnel(mad_u(T16[g >> 26], q, 1ULL << 29), 30);
    const unsigned r = (p + ((1u << (sh & 31)) >> 1)) >> (sh & 31);
    return sh > 31 ? 0 : r;
}
__device__ inline ll exp_neg(ll x, const unsigned* T16) {
    return exp_neg32(x < -(64LL << 24) ? -(64 << 24) : (int)x, T16);
}
// exp of the rounded product (dl A) / 2^8 for 0 <= dl <= 2^30, -2^24 <= A <= 0
__host__ __device__ inline unsigned exp_prod(int dl, int A, const unsigned* T16) {
    const ll v = mad_i(dl, A, 128);
    const int hi = (int)hi32((unsigned long long)v);
    return exp_neg32(hi < -64 ? -(1 << 30) : (int)funnel((unsigned long long)v, 8), T16);
}
// clamp to +-(2^31 - 1)
__host__ __device__ inline int sat31(ll v) {
    const int lo = (int)v, hi = (int)(v >> 32);
    const int r = hi == lo >> 31 ? lo : (hi < 0 ? -2147483647 : 2147483647);
    return r < -2147483647 ? -2147483647 : r;
}
// h' = clamp(round(dA h / 2^30) + round(dx B / 2^8)) for dA <= 2^30, |h| < 2^31,
// |dx| <= 2^33, |B| < 2^23; dx = 2^8 dh + d8, so the second rounding needs d8 B only
__host__ __device__ inline int state_next(unsigned dA, int h, int dh, int d8, int B) {
    const int a = (int)funnel((unsigned long long)mad_i((int)dA, h, 1LL << 29), 30);
    return sat31(mad_i(dh, B, (ll)((d8 * B + 128) >> 8)) + a);
}
__device__ inline ll sigmoid_q30(ll u, const unsigned* T16) {          // u Q12
    const ll e = exp_neg(-(u < 0 ? -u : u) << 12, T16);
    return fdiv32(u >= 0 ? 1LL << 60 : e << 30, (1u << 30) + (unsigned)e);
}
__device__ inline ll silu_q12(ll u, const unsigned* T16) {
    return clampll(rsh(mul32(u, sigmoid_q30(u, T16)), 30), -SAT23, SAT23);
}
// ln(1 + w / 2^30) in Q30 for 0 <= w <= 2^30: ln(1 + k/16) from the table plus
// the series of ln(1 + r), r = (1 + w) / (1 + k/16) - 1 < 1/17, to r^5
__device__ inline ll log1p_q30(ll w, const ll* LNC) {
    const ll k = w >> 26;
    const ll c = (1LL << 30) + (k << 26);
    const ll r = fdiv32(((1LL << 30) + w - c) << 30, (unsigned)c);
    ll h = H5;                                    // 0 < h <= 2^30, 0 <= r < 2^26
    h = (1LL << 28) - rsh(mulu32(h, r), 30);
    h = H3 - rsh(mulu32(h, r), 30);
    h = (1LL << 29) - rsh(mulu32(h, r), 30);
    h = (1LL << 30) - rsh(mulu32(h, r), 30);
    return LNC[k] + rsh(mulu32(h, r), 30);
}
__device__ inline ll softplus_q20(ll v, const unsigned* T16, const ll* LNC) {         // v Q12 -> Delta Q20
    const ll w = exp_neg(-(v < 0 ? -v : v) << 12, T16);
    return clampll(((v > 0 ? v : 0) << 8) + rsh(log1p_q30(w, LNC), 10), 0, 1LL << 30);
}
__device__ inline ll isqrt64(ll v) {              // floor(sqrt(v)), 0 <= v < 2^53
    ll r = (ll)sqrt((double)v);                   // the root or one above
    if (mulu32(r, r) > v) --r;
    return mulu32(r + 1, r + 1) <= v ? r + 1 : r;
}
__device__ inline int bitlen(unsigned m) { return m ? 32 - __clz(m) : 0; }

// ---------------------------------------------------------------- model
struct QLayer {
    const int* ln_g; const int* ln_b;
    const int* in_w; const int* in_p;           // words [D/4][2Di]: byte b of (k4, o) = w8[o][4 k4 + b]; [2Di]
    const int* cw; const int* cb;               // [4][Di] Q14; [Di] Q12
    const int* x_w; const int* x_p;             // words [NO][Di/4]; [NO]
    const int* dt_w; const int* dt_p; const int* dtb;   // words [R/4][Di]; [Di]; [Di]
    const int* A; const int* Dq;                // [N][Di] Q12; [Di] Q12
    const int* out_w; const int* out_p;         // words [Di/4][D]; [D]
};
constexpr int QMAX_LAYERS = 16;
struct QArgs {
    QLayer L[QMAX_LAYERS];
    int n_layers, D, Di, R;
    const int* embed;                            // [256][D] Q12
    const int* nf_g; const int* nf_b;
    const int* head_w; const int* head_p; const int* head_b;   // words [D/4][256]; [256]; [256]
};

constexpr int MODE_TABLES = 0, MODE_ENCODE = 1, MODE_DECODE = 2;
struct QJob {
    const uint8_t* in;          // tables: seqs [B][T]; encode: the data; decode: the payloads
    const ll* chunk_off;        // byte offset of each chunk in the data (tables, encode) or output (decode)
    const ll* chunk_len;
    const ll* pay_off;          // encode / decode
    const ll* pay_n;            // encode: capacity; decode: payload length
    const uint8_t* first;       // decode: first byte of each chunk
    uint8_t* out;               // encode: payloads; decode: decoded bytes
    uint32_t* pay_len;          // encode: bytes written (0xFFFFFFFF: over capacity)
    uint16_t* tables;           // tables: [B][T-1][256]
    int* logits;                // tables: [B][T-1][256] Q12
    int* state;                 // per chunk: conv window [L][3][Di], then h [L][N][Di]
    ll state_words;
};

// ---------------------------------------------------------------- block helpers
__device__ inline ll blk_sum(ll v, ll* red) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return red[0] + red[1] + red[2] + red[3];
}
__device__ inline ll blk_max(ll v, ll* red) {
    for (int o = 32; o > 0; o >>= 1) { ll w = __shfl_xor(v, o); v = w > v ? w : v; }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    ll m = red[0];
    for (int i = 1; i < 4; ++i) m = red[i] > m ? red[i] : m;
    return m;
}
// the largest value, lowest index among ties
__device__ inline int blk_argmax(ll v, int idx, ll* red, int* redi) {
    for (int o = 32; o > 0; o >>= 1) {
        ll w = __shfl_xor(v, o);
        int wi = __shfl_xor(idx, o);
        if (w > v || (w == v && wi < idx)) { v = w; idx = wi; }
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) { red[threadIdx.x >> 6] = v; redi[threadIdx.x >> 6] = idx; }
    __syncthreads();
    ll bv = red[0];
    int bi = redi[0];
    for (int i = 1; i < 4; ++i)
        if (red[i] > bv || (red[i] == bv && redi[i] < bi)) { bv = red[i]; bi = redi[i]; }
    return bi;
}

// the largest of non-negative values
__device__ inline int blk_max_i(int v, int* red) {
    for (int o = 32; o > 0; o >>= 1) {
        const int w = __shfl_xor(v, o);
        v = w > v ? w : v;
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    int m = red[0];
    for (int i = 1; i < 4; ++i) m = red[i] > m ? red[i] : m;
    return m;
}
// LayerNorm of D Q12 values (src) into dst; D is a power of two, so the means
// are shifts, and |src - mu| <= sqrt(D) sd bounds the normalised value below
// 2^18, so K = 2^20 makes the numerator of its floor non-negative
template <int D>
__device__ void int_ln(const int* src, int* dst, const int* g, const int* b, ll* red) {
    constexpr int LD = D == 64 ? 6 : D == 128 ? 7 : D == 256 ? 8 : 9;
    static_assert(1 << LD == D, "d_model");
    const int t = threadIdx.x;
    ll s = 0;
    for (int d = t; d < D; d += NT) s += src[d];
    s = blk_sum(s, red);
    const ll mu = s >> LD;
    ll v = 0;
    for (int d = t; d < D; d += NT) { ll dd = src[d] - mu; v += mul32(dd, dd); }   // |dd| < 2^24
    v = blk_sum(v, red);
    const ll sd = isqrt64((v >> LD) + EPS_Q24);
    constexpr ll K = 1 << 20;
    for (int d = t; d < D; d += NT) {
        const ll dd = src[d] - mu;
        const ll nn = (ll)fdiv32(2 * (dd << 12) + sd + K * 2 * sd, (unsigned)(2 * sd)) - K;
        dst[d] = (int)clampll(rsh(mul32(nn, g[d]), 12) + b[d], -SAT23, SAT23);
    }
    __syncthreads();
}
// round(v / 2^e) half up, clamped to +-127, |v| < 2^23
__device__ inline unsigned q8(int v, int e) {
    const int q = e > 0 ? (v + (1 << (e - 1))) >> e : v;
    return (unsigned)(q < -127 ? -127 : (q > 127 ? 127 : q)) & 0xFFu;
}
// dynamic INT8 input of a projection: packs n values of src (n % 4 == 0) into
// words and returns the shift e
__device__ int int_q8(const int* src, int n, int* words, int* red) {
    const int t = threadIdx.x;
    int m = 0;
    for (int i = t; i < n; i += NT) { const int a = src[i] < 0 ? -src[i] : src[i]; m = a > m ? a : m; }
    m = blk_max_i(m, red);
    const int bl = bitlen((unsigned)m);
    const int e = bl > 7 ? bl - 7 : 0;
    for (int w = t; w < n / 4; w += NT) {
        const int4 x = reinterpret_cast<const int4*>(src)[w];
        words[w] = (int)(q8(x.x, e) | q8(x.y, e) << 8 | q8(x.z, e) << 16 | q8(x.w, e) << 24);
    }
    __syncthreads();
    return e;
}

__device__ inline int dot16(int4 a, int4 b, int acc) {
    acc = __builtin_amdgcn_sdot4(a.x, b.x, acc, false);
    acc = __builtin_amdgcn_sdot4(a.y, b.y, acc, false);
    acc = __builtin_amdgcn_sdot4(a.z, b.z, acc, false);
    return __builtin_amdgcn_sdot4(a.w, b.w, acc, false);
}
// Sums over k words of inputs a8 with words w [K4][N]: V adjacent outputs from o
// on, input words k0 .. k0 + K4 - 1 (V words a load).
template <int V, int N, int K4>
__device__ inline void dot_cols(const int* a8, const int* w, int o, int k0, int (&acc)[V]) {
    typedef int vec __attribute__((ext_vector_type(V)));
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] = 0;
    constexpr int U = K4 < 32 / V ? K4 : 32 / V;        // loads in flight
#pragma unroll 1
    for (int k = 0; k < K4; k += U) {
        int b[U][V];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int* src = w + (k0 + k + u) * N + o;
            if constexpr (V == 1) {
                b[u][0] = *src;
            } else {
                const vec x = *reinterpret_cast<const vec*>(src);
#pragma unroll
                for (int v = 0; v < V; ++v) b[u][v] = x[v];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int v = 0; v < V; ++v) acc[v] = __builtin_amdgcn_sdot4(a8[k0 + k + u], b[u][v], acc[v], false);
    }
}
// The N sums of K4 words: wave w takes a quarter of the inputs for all outputs
// (64 lanes x V of them a pass) and the quarters meet in part [4][N].
template <int N, int K4>
__device__ inline void dot_split(const int* a8, const int* w, int* part) {
    constexpr int V = N / 64 < 4 ? N / 64 : 4;
    const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
    for (int o = V * ln; o < N; o += 64 * V) {
        int acc[V];
        dot_cols<V, N, K4 / 4>(a8, w, o, wv * (K4 / 4), acc);
#pragma unroll
        for (int v = 0; v < V; ++v) part[wv * N + o + v] = acc[v];
    }
    __syncthreads();
}

struct QShared {
    alignas(16) int r[512];                      // (16-byte aligned: read four at a time)
    alignas(16) int nrm[512];
    alignas(16) int a8[256];
    alignas(16) int xz[2048];
    alignas(16) int xs[1024];
    alignas(16) int gate[1024];
    int dbc[64];
    int f[256], cx[256];
    ll red[4];
    int redi[4];
    int sym;
    uint32_t D;
    uint64_t v;
    unsigned t16[16];
    ll lnc[17];         // the exponential's and logarithm's tables, read with divergent indexes
};

// DM = d_model: every loop bound below is a compile-time constant.  Four waves
// per SIMD (128 registers) cost 36 spilled registers a thread at d_model 256 (44,
// 41 and 81 at 64, 128 and 512): the state loads ahead are held beside the
// exponentials' values.
template <int DM>
__global__ __launch_bounds__(NT, 4) void k_int_chunk(QArgs a, QJob j, int mode) {
    __shared__ QShared sh;
    const int t = threadIdx.x;
    const ll c = blockIdx.x;
    const ll len = j.chunk_len[c];
    constexpr int D = DM, Di = 2 * DM, R = DM / 16, NO = R + 2 * QN;
    if (len <= 0) {
        if (mode == MODE_ENCODE && t == 0) j.pay_len[c] = 0;
        return;
    }
    int* st = j.state + c * j.state_words;
    for (ll i = t; i < j.state_words; i += NT) st[i] = 0;
    if (t < 16) sh.t16[t] = (unsigned)kT16[t];
    if (t < 17) sh.lnc[t] = kLNC[t];
    const ll off = j.chunk_off[c];
    int y = mode == MODE_DECODE ? j.first[c] : j.in[off];
    if (mode == MODE_DECODE && t == 0) j.out[off] = (uint8_t)y;
    boa::Enc enc;
    boa::Dec dec;
    uint8_t* pay_out = nullptr;
    const uint8_t* pay_in = nullptr;
    uint32_t cap = 0, plen = 0;
    if (mode == MODE_ENCODE) {
        boa::enc_reset(enc);
        pay_out = j.out + j.pay_off[c];
        cap = (uint32_t)j.pay_n[c];
    } else if (mode == MODE_DECODE) {
        pay_in = j.in + j.pay_off[c];
        plen = (uint32_t)j.pay_n[c];
        boa::dec_reset(dec, pay_in, plen);
    }
    __syncthreads();

    for (ll s = 0; s + 1 < len; ++s) {
        for (int d = t; d < D; d += NT) sh.r[d] = a.embed[y * D + d];
        __syncthreads();
        for (int l = 0; l < a.n_layers; ++l) {
            const QLayer& L = a.L[l];
            int* win = st + (ll)l * 3 * Di;
            int* hst = st + (ll)a.n_layers * 3 * Di + (ll)l * QN * Di;
            // LayerNorm, in_proj; the conv's window and weights are requested first
            constexpr int CPT = (Di + NT - 1) / NT;      // channels of a thread
            int cwin[CPT][3], ccw[CPT][5];
#pragma unroll
            for (int q = 0; q < CPT; ++q) {
                const int d = t + NT * q;
                if (Di % NT && d >= Di) break;
#pragma unroll
                for (int k = 0; k < 3; ++k) cwin[q][k] = win[k * Di + d];
#pragma unroll
                for (int k = 0; k < 4; ++k) ccw[q][k] = L.cw[k * Di + d];
                ccw[q][4] = L.cb[d];
            }
            int_ln<D>(sh.r, sh.nrm, L.ln_g, L.ln_b, sh.red);
            int e = int_q8(sh.nrm, D, sh.a8, sh.redi);
            constexpr int VI = 2 * Di / NT < 4 ? 2 * Di / NT : 4;   // adjacent outputs of a thread
            for (int o = VI * t; o < 2 * Di; o += VI * NT) {
                int acc[VI];
                dot_cols<VI, 2 * Di, D / 4>(sh.a8, L.in_w, o, 0, acc);
#pragma unroll
                for (int v = 0; v < VI; ++v) sh.xz[o + v] = (int)clampll(rsh(acc[v], L.in_p[o + v] - e), -SAT23, SAT23);
            }
            __syncthreads();
            // causal conv over x_{t-3} .. x_t, SiLU
#pragma unroll
            for (int q = 0; q < CPT; ++q) {
                const int d = t + NT * q;
                if (Di % NT && d >= Di) break;
                const ll x = sh.xz[d];
                const ll u = clampll(rsh(mul32(ccw[q][0], cwin[q][0]) + mul32(ccw[q][1], cwin[q][1]) +
                                             mul32(ccw[q][2], cwin[q][2]) + mul32(ccw[q][3], x), 14) + ccw[q][4], -SAT23, SAT23);
                win[d] = cwin[q][1];
                win[Di + d] = cwin[q][2];
                win[2 * Di + d] = (int)x;
                sh.xs[d] = (int)silu_q12(u, sh.t16);
            }
            // the scan's states and A of the thread's first channel, needed after x_proj
            int hv[QN], Av[QN];
            auto load_state = [&](int n, int d) {
                Av[n] = L.A[n * Di + d];
                hv[n] = hst[n * Di + d];
            };
            if (Di % NT == 0 || t < Di) {
#pragma unroll
                for (int n = 0; n < QN; ++n) load_state(n, t);
            }
            __syncthreads();
            // x_proj: four threads per output, each a quarter of the inputs, 16 at
            // a time (a wave per output and a shuffle tree took 22k cycles a
            // layer of four chunks a CU, 7k so)
            e = int_q8(sh.xs, Di, sh.a8, sh.redi);
            if (t < 4 * NO) {
                const int o = t >> 2, part = t & 3;
                const int4* wp = reinterpret_cast<const int4*>(L.x_w) + o * (Di / 16) + part;
                const int4* ap = reinterpret_cast<const int4*>(sh.a8) + part;
                int acc = 0;
#pragma unroll
                for (int k = 0; k < Di / 64; ++k) acc = dot16(ap[4 * k], wp[4 * k], acc);
                acc += __shfl_xor(acc, 1);
                acc += __shfl_xor(acc, 2);
                if (part == 0) sh.dbc[o] = (int)clampll(rsh(acc, L.x_p[o] - e), -SAT23, SAT23);
            }
            __syncthreads();
            // dt_proj (its R inputs quantised by every thread alike), softplus,
            // the scan and the gate, one channel per thread
            {
                int m = 0;
                for (int k = 0; k < R; ++k) { const int v = sh.dbc[k] < 0 ? -sh.dbc[k] : sh.dbc[k]; m = v > m ? v : m; }
                const int bl = bitlen((unsigned)m);
                const int e3 = bl > 7 ? bl - 7 : 0;
                int dq[8];
                for (int k4 = 0; k4 < R / 4; ++k4) {
                    unsigned pk = 0;
                    for (int b = 0; b < 4; ++b) pk |= q8(sh.dbc[4 * k4 + b], e3) << (8 * b);
                    dq[k4] = (int)pk;
                }
                for (int d = t; d < Di; d += NT) {
                    int acc = 0;
                    for (int k4 = 0; k4 < R / 4; ++k4) acc = __builtin_amdgcn_sdot4(dq[k4], L.dt_w[k4 * Di + d], acc, false);
                    const ll v = clampll(rsh(acc, L.dt_p[d] - e3) + L.dtb[d], -SAT23, SAT23);
                    const ll dl = softplus_q20(v, sh.t16, sh.lnc);
                    const ll xs = sh.xs[d];
                    const ll dx = rsh(mul32(dl, xs), 20);           // dl <= 2^30, |xs| < 2^23
                    const int dh = (int)(dx >> 8), d8 = (int)(dx & 255);
                    ll ys = 0;
                    // (each state's registers take the next channel's as they become free)
#pragma unroll
                    for (int n = 0; n < QN; ++n) {
                        const int hn = state_next(exp_prod((int)dl, Av[n], sh.t16), hv[n], dh, d8, sh.dbc[R + n]);
                        hst[n * Di + d] = hn;
                        ys = mad_i(sh.dbc[R + QN + n], hn, ys);
                        if (Di > NT && d + NT < Di) load_state(n, d + NT);
                    }
                    const ll yv = clampll(rsh(ys, 16) + rsh(mul32(L.Dq[d], xs), 12), -SAT23, SAT23);
                    sh.gate[d] = (int)clampll(rsh(mul32(yv, silu_q12(sh.xz[Di + d], sh.t16)), 12), -SAT23, SAT23);
                }
            }
            __syncthreads();
            // out_proj and the residual
            e = int_q8(sh.gate, Di, sh.a8, sh.redi);
            dot_split<D, Di / 4>(sh.a8, L.out_w, sh.xz);
            for (int o = t; o < D; o += NT) {
                const int acc = (sh.xz[o] + sh.xz[D + o]) + (sh.xz[2 * D + o] + sh.xz[3 * D + o]);
                const ll pr = clampll(rsh(acc, L.out_p[o] - e), -SAT23, SAT23);
                sh.r[o] = (int)clampll(sh.r[o] + pr, -SAT23, SAT23);
            }
            __syncthreads();
        }
        // final LayerNorm, head: thread t owns symbol t
        int_ln<D>(sh.r, sh.nrm, a.nf_g, a.nf_b, sh.red);
        const int e = int_q8(sh.nrm, D, sh.a8, sh.redi);
        dot_split<256, D / 4>(sh.a8, a.head_w, sh.xz);
        const int acc = (sh.xz[t] + sh.xz[256 + t]) + (sh.xz[512 + t] + sh.xz[768 + t]);
        const ll lg = clampll(rsh(acc, a.head_p[t] - e) + a.head_b[t], -SAT23, SAT23);
        // integer softmax and histogram
        const ll mx = blk_max(lg, sh.red);
        const ll ex = exp_neg((lg - mx) << 12, sh.t16);
        const ll S = blk_sum(ex, sh.red);
        ll f = fdiv(ex << 16, S);
        f = f < 1 ? 1 : f;
        const ll tot = blk_sum(f, sh.red);
        const int am = blk_argmax(f, t, sh.red, sh.redi);
        if (t == am) f += 65536 - tot;
        // exclusive prefix sum: wave scan, then the waves' totals
        ll inc = f;
        for (int o = 1; o < 64; o <<= 1) {
            ll v = __shfl_up(inc, o);
            if ((t & 63) >= o) inc += v;
        }
        __syncthreads();
        if ((t & 63) == 63) sh.red[t >> 6] = inc;
        __syncthreads();
        ll base = 0;
        for (int w = 0; w < (t >> 6); ++w) base += sh.red[w];
        const ll cx = base + inc - f;
        sh.f[t] = (int)f;
        sh.cx[t] = (int)cx;
        if (mode == MODE_TABLES) {
            const ll row = c * (len - 1) + s;
            j.tables[row * 256 + t] = (uint16_t)f;
            j.logits[row * 256 + t] = (int)lg;
            y = j.in[off + s + 1];
        } else if (mode == MODE_ENCODE) {
            y = j.in[off + s + 1];
            __syncthreads();
            if (t == 0) boa::enc_put(enc, (uint32_t)sh.cx[y], (uint32_t)sh.f[y], pay_out, cap);
        } else {
            if (t == 0) { sh.v = boa::dec_v(dec); sh.D = dec.D; }
            __syncthreads();
            if (boa::dec_from(sh.v, sh.D, (uint32_t)cx) && boa::dec_upto(sh.v, sh.D, (uint32_t)(cx + f))) sh.sym = t;
            __syncthreads();
            y = sh.sym;
            if (t == 0) {
                boa::dec_update(dec, (uint32_t)sh.cx[y], (uint32_t)sh.f[y], pay_in, plen);
                j.out[off + s + 1] = (uint8_t)y;
            }
        }
        __syncthreads();
    }
    if (mode == MODE_ENCODE && t == 0) {
        boa::enc_flush(enc, pay_out, cap);
        j.pay_len[c] = enc.cur <= cap ? enc.cur : 0xFFFFFFFFu;
    }
}

// ---------------------------------------------------------------- host conversion
ll fixq(double v, int frac, ll lim) { return clampll((ll)std::nearbyint(std::ldexp(v, frac)), -lim, lim); }

// per-row power-of-two INT8: p = largest integer with max|W_j| 2^p <= 127,
// clamped to [0, 40]; w8 = clamp(rint(W 2^p), -127, 127)
void conv_proj(const float* W, int out, int in, std::vector<int8_t>& w8, std::vector<int>& p) {
    w8.assign((size_t)out * in, 0);
    p.assign(out, 0);
    for (int j = 0; j < out; ++j) {
        double m = 0;
        for (int i = 0; i < in; ++i) m = std::fmax(m, std::fabs((double)W[(size_t)j * in + i]));
        int pj = 0;
        if (m != 0.0) {
            int E = 0;
            const double fr = std::frexp(m, &E);
            pj = fr <= 127.0 / 128.0 ? 7 - E : 6 - E;
            pj = pj < 0 ? 0 : (pj > 40 ? 40 : pj);
        }
        p[j] = pj;
        for (int i = 0; i < in; ++i)
            w8[(size_t)j * in + i] = (int8_t)clampll((ll)std::nearbyint(std::ldexp((double)W[(size_t)j * in + i], pj)), -127, 127);
    }
}
inline int pack4(const int8_t* v) {
    unsigned pk = 0;
    for (int b = 0; b < 4; ++b) pk |= ((unsigned)(uint8_t)v[b]) << (8 * b);
    return (int)pk;
}

}  // namespace

struct boa_qmodel {
    boa_config cfg{};
    int device = 0;
    uint64_t fingerprint = 0;
    int* d_blob = nullptr;
    QArgs args{};
};

#define QCHK(expr)                                                                                 \
    do {                                                                                           \
        hipError_t e_ = (expr);                                                                    \
        if (e_ != hipSuccess)                                                                      \
            return boa::set_error(BOA_E_DEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

extern "C" int boa_qmodel_create(const boa_model* m, boa_qmodel** out) {
    if (!m || !out) return boa::set_error(BOA_E_ARG, "null argument");
    *out = nullptr;
    const boa_config& cfg = m->cfg;
    const boa::Layout& lay = m->lay;
    if (cfg.ffn_mult != 0 || cfg.d_state != 16 || cfg.d_conv != 4 || cfg.n_layers > QMAX_LAYERS || cfg.d_model > 512)
        return boa::set_error(BOA_E_UNSUPPORTED, "integer pipeline: d_state 16, d_conv 4, d_model <= 512, no feed-forward sub-layer");
    std::vector<float> w(lay.total);
    int rc = boa_model_get_weights(m, w.data(), w.size());
    if (rc) return rc;
    const int D = lay.D, Di = lay.Di, R = lay.R, N = lay.N, K = lay.K, NL = lay.L, NO = R + 2 * N;
    std::vector<int> blob;
    std::vector<size_t> at;             // offsets of the pieces, in order
    auto put = [&](const std::vector<int>& v) { at.push_back(blob.size()); blob.insert(blob.end(), v.begin(), v.end()); };
    auto fixv = [&](uint64_t o, size_t n, int frac, ll lim) {
        std::vector<int> v(n);
        for (size_t i = 0; i < n; ++i) v[i] = (int)fixq(w[o + i], frac, lim);
        return v;
    };
    std::vector<int8_t> w8;
    std::vector<int> p;
    // rows-as-outputs words [in/4][out]
    auto words_kmajor = [&](int outn, int inn) {
        std::vector<int> v((size_t)(inn / 4) * outn);
        for (int k = 0; k < inn / 4; ++k)
            for (int o = 0; o < outn; ++o) v[(size_t)k * outn + o] = pack4(&w8[(size_t)o * inn + 4 * k]);
        return v;
    };
    put(fixv(lay.embed, (size_t)256 * D, 12, SAT23));
    put(fixv(lay.norm_f_w, D, 12, SAT23));
    put(fixv(lay.norm_f_b, D, 12, SAT23));
    conv_proj(&w[lay.head_w], 256, D, w8, p);
    put(words_kmajor(256, D));
    put(p);
    put(fixv(lay.head_b, 256, 12, SAT23));
    for (int l = 0; l < NL; ++l) {
        const boa::LayerOff& o = lay.layer[l];
        put(fixv(o.norm_w, D, 12, SAT23));
        put(fixv(o.norm_b, D, 12, SAT23));
        conv_proj(&w[o.in_w], 2 * Di, D, w8, p);
        put(words_kmajor(2 * Di, D));
        put(p);
        std::vector<int> cw((size_t)K * Di);
        for (int d = 0; d < Di; ++d)
            for (int k = 0; k < K; ++k) cw[(size_t)k * Di + d] = (int)fixq(w[o.conv_w + (size_t)d * K + k], 14, 1LL << 20);
        put(cw);
        put(fixv(o.conv_b, Di, 12, SAT23));
        conv_proj(&w[o.xw], NO, Di, w8, p);
        {
            std::vector<int> v((size_t)NO * (Di / 4));
            for (int r = 0; r < NO; ++r)
                for (int k = 0; k < Di / 4; ++k) v[(size_t)r * (Di / 4) + k] = pack4(&w8[(size_t)r * Di + 4 * k]);
            put(v);
        }
        put(p);
        conv_proj(&w[o.dtw], Di, R, w8, p);
        put(words_kmajor(Di, R));
        put(p);
        put(fixv(o.dtb, Di, 12, SAT23));
        // A = -exp(A_log): A_log in Q24 clamped to [-16, 9], the integer exp2
        std::vector<int> A((size_t)N * Di);
        for (int d = 0; d < Di; ++d)
            for (int n = 0; n < N; ++n) {
                const ll a24 = clampll(fixq(w[o.A_log + (size_t)d * N + n], 24, 1LL << 40), -(16LL << 24), 9LL << 24);
                const ll y = rsh(a24 * LOG2E, 24);
                const ll nn = y >> 30;
                const ll g = y - (nn << 30);
                const ll mant = exp2_frac(g, hT16[g >> 26]);
                const ll v = rsh(mant, (int)(18 - nn));
                A[(size_t)n * Di + d] = (int)-(v < (1LL << 24) ? v : (1LL << 24));
            }
        put(A);
        put(fixv(o.Dsk, Di, 12, SAT23));
        conv_proj(&w[o.out_w], D, Di, w8, p);
        put(words_kmajor(D, Di));
        put(p);
    }
    boa_qmodel* q = new boa_qmodel();
    q->cfg = cfg;
    q->device = m->device;
    q->fingerprint = boa::model_fingerprint(m);
    hipError_t he = hipSetDevice(m->device);
    if (he == hipSuccess) he = hipMalloc(&q->d_blob, blob.size() * sizeof(int));
    if (he == hipSuccess) he = hipMemcpy(q->d_blob, blob.data(), blob.size() * sizeof(int), hipMemcpyHostToDevice);
    if (he != hipSuccess) {
        if (q->d_blob) (void)hipFree(q->d_blob);
        delete q;
        return boa::set_error(BOA_E_DEVICE, std::string("integer model upload: ") + hipGetErrorString(he));
    }
    const int* b = q->d_blob;
    size_t i = 0;
    QArgs& A = q->args;
    A.n_layers = NL; A.D = D; A.Di = Di; A.R = R;
    A.embed = b + at[i++]; A.nf_g = b + at[i++]; A.nf_b = b + at[i++];
    A.head_w = b + at[i++]; A.head_p = b + at[i++]; A.head_b = b + at[i++];
    for (int l = 0; l < NL; ++l) {
        QLayer& L = A.L[l];
        L.ln_g = b + at[i++]; L.ln_b = b + at[i++];
        L.in_w = b + at[i++]; L.in_p = b + at[i++];
        L.cw = b + at[i++]; L.cb = b + at[i++];
        L.x_w = b + at[i++]; L.x_p = b + at[i++];
        L.dt_w = b + at[i++]; L.dt_p = b + at[i++]; L.dtb = b + at[i++];
        L.A = b + at[i++]; L.Dq = b + at[i++];
        L.out_w = b + at[i++]; L.out_p = b + at[i++];
    }
    *out = q;
    return BOA_OK;
}

extern "C" void boa_qmodel_free(boa_qmodel* q) {
    if (!q) return;
    if (q->d_blob) {
        (void)hipSetDevice(q->device);
        (void)hipFree(q->d_blob);
    }
    delete q;
}

namespace {
// per-chunk arrays and state in one device allocation; runs the kernel and waits
int run_chunks(const boa_qmodel* q, QJob j, int mode, uint64_t n_chunks, const uint64_t* h_off, const uint64_t* h_len,
               const uint64_t* h_poff, const uint64_t* h_pn, const uint8_t* h_first, void* stream) {
    if (n_chunks == 0) return BOA_OK;
    if (n_chunks > (uint64_t)INT32_MAX) return boa::set_error(BOA_E_ARG, "too many chunks");
    QCHK(hipSetDevice(q->device));
    const ll sw = (ll)q->args.n_layers * (3 + QN) * q->args.Di;
    std::vector<ll> hv((size_t)n_chunks * 4);
    for (uint64_t c = 0; c < n_chunks; ++c) {
        if (h_len[c] > (uint64_t)INT64_MAX / 2) return boa::set_error(BOA_E_ARG, "chunk length out of range");
        hv[c] = (ll)h_off[c];
        hv[n_chunks + c] = (ll)h_len[c];
        hv[2 * n_chunks + c] = h_poff ? (ll)h_poff[c] : 0;
        hv[3 * n_chunks + c] = h_pn ? (ll)h_pn[c] : 0;
        if (h_pn && h_pn[c] > 0xFFFFFFFFull) return boa::set_error(BOA_E_ARG, "payload size beyond 32 bits");
    }
    const size_t arr = hv.size() * sizeof(ll);
    const size_t firsts = h_first ? ((n_chunks + 255) / 256) * 256 : 0;
    const size_t state = (size_t)n_chunks * (size_t)sw * sizeof(int);
    char* buf = nullptr;
    QCHK(hipMalloc(&buf, arr + firsts + state));
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = hipMemcpyAsync(buf, hv.data(), arr, hipMemcpyHostToDevice, s);
    if (e == hipSuccess && h_first) e = hipMemcpyAsync(buf + arr, h_first, n_chunks, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) {
        const ll* dv = (const ll*)buf;
        j.chunk_off = dv;
        j.chunk_len = dv + n_chunks;
        j.pay_off = dv + 2 * n_chunks;
        j.pay_n = dv + 3 * n_chunks;
        j.first = h_first ? (const uint8_t*)(buf + arr) : nullptr;
        j.state = (int*)(buf + arr + firsts);
        j.state_words = sw;
        const dim3 grid((unsigned)n_chunks), blk(NT);
        switch (q->args.D) {
            case 64: hipLaunchKernelGGL(k_int_chunk<64>, grid, blk, 0, s, q->args, j, mode); break;
            case 128: hipLaunchKernelGGL(k_int_chunk<128>, grid, blk, 0, s, q->args, j, mode); break;
            case 256: hipLaunchKernelGGL(k_int_chunk<256>, grid, blk, 0, s, q->args, j, mode); break;
            default: hipLaunchKernelGGL(k_int_chunk<512>, grid, blk, 0, s, q->args, j, mode); break;
        }
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    hipError_t ef = hipFree(buf);
    if (e != hipSuccess) return boa::set_error(BOA_E_DEVICE, std::string("integer pipeline: ") + hipGetErrorString(e));
    if (ef != hipSuccess) return boa::set_error(BOA_E_DEVICE, std::string("hipFree: ") + hipGetErrorString(ef));
    return BOA_OK;
}
}  // namespace

extern "C" int boa_int_tables_dev(const boa_qmodel* q, const uint8_t* d_seqs, uint32_t batch, uint32_t seq_len,
                                  uint16_t* d_tables, int32_t* d_logits, void* stream) {
    if (!q || (batch && (!d_seqs || (seq_len > 1 && (!d_tables || !d_logits)))))
        return boa::set_error(BOA_E_ARG, "null argument");
    std::vector<uint64_t> off(batch), len(batch, seq_len);
    for (uint32_t b = 0; b < batch; ++b) off[b] = (uint64_t)b * seq_len;
    QJob j{};
    j.in = d_seqs;
    j.tables = d_tables;
    j.logits = d_logits;
    return run_chunks(q, j, MODE_TABLES, batch, off.data(), len.data(), nullptr, nullptr, nullptr, stream);
}

extern "C" int boa_int_encode_dev(const boa_qmodel* q, const uint8_t* d_data, const uint64_t* h_chunk_off,
                                  const uint64_t* h_chunk_len, uint64_t n_chunks, uint8_t* d_payload,
                                  const uint64_t* h_pay_off, const uint64_t* h_pay_cap, uint32_t* d_pay_len,
                                  void* stream) {
    if (!q || (n_chunks && (!d_data || !h_chunk_off || !h_chunk_len || !d_payload || !h_pay_off || !h_pay_cap ||
                            !d_pay_len)))
        return boa::set_error(BOA_E_ARG, "null argument");
    QJob j{};
    j.in = d_data;
    j.out = d_payload;
    j.pay_len = d_pay_len;
    return run_chunks(q, j, MODE_ENCODE, n_chunks, h_chunk_off, h_chunk_len, h_pay_off, h_pay_cap, nullptr, stream);
}

extern "C" int boa_int_decode_dev(const boa_qmodel* q, const uint8_t* d_payload, const uint64_t* h_pay_off,
                                  const uint64_t* h_pay_len, const uint8_t* h_first, const uint64_t* h_chunk_off,
                                  const uint64_t* h_chunk_len, uint64_t n_chunks, uint8_t* d_out, void* stream) {
    if (!q || (n_chunks && (!d_payload || !h_pay_off || !h_pay_len || !h_first || !h_chunk_off || !h_chunk_len ||
                            !d_out)))
        return boa::set_error(BOA_E_ARG, "null argument");
    QJob j{};
    j.in = d_payload;
    j.out = d_out;
    return run_chunks(q, j, MODE_DECODE, n_chunks, h_chunk_off, h_chunk_len, h_pay_off, h_pay_len, h_first, stream);
}
