// Decoder-block glue on 16-bit integer activations: the operators between
// the quantized linear layers keep 16-bit integer activations (Section 4.1,
// Section 5.1).  Each kernel dequantizes exactly (an fp32 scale times an
// integer of at most 17 bits is exact in fp64), evaluates the operator in
// fp64 one IEEE operation at a time in a fixed order, and requantizes with
// the Eq.(4) quantizer (rint half to even, clamp).  Residual add and
// RMSNorm therefore give the same bits as any IEEE evaluation of the same
// sequence; SiLU and softmax go through exp, whose last bit IEEE does not
// fix.
#include <cmath>
#include <type_traits>

#include "mq_internal.h"

namespace mq {
namespace {

constexpr int kThreads = 256;

inline int grid_for(int64_t items, int per_block, int cap)
{
    int64_t g = (items + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

// The code before its clamp to the output range: rint(t) + zy.  A quotient
// beyond +-2^17 saturates whatever the zero-point (|zy| <= 2^15), so it is
// limited there first (NaN: the low end) and adding 1.5 * 2^52 leaves rint(t)
// (to nearest, ties to even) in the low word: 32-bit integers throughout.
__device__ inline double limit_quotient(double t)
{
    return fmin(fmax(t, -131072.0), 131072.0);
}
constexpr double kRintShift = 6755399441055744.0;  // 1.5 * 2^52
__device__ inline int32_t rint_low(double shifted)
{
    return (int32_t)(uint32_t)__double_as_longlong(shifted);
}

template <int BITS>
__device__ inline int32_t clamp_code(int32_t q)
{
    constexpr int32_t qmin = -(1 << (BITS - 1)), qmax = (1 << (BITS - 1)) - 1;
    return min(max(q, qmin), qmax);
}

template <int BITS>
__device__ inline int32_t requant_f64(double v, double ay, int32_t zy)
{
#pragma clang fp contract(off)
    return clamp_code<BITS>(rint_low(limit_quotient(v / ay) + kRintShift) + zy);
}

// N codes.  exact(u) is the quotient of code u as the definition evaluates it
// (its divisions correctly rounded), fast(u) the same quotient through
// products with reciprocals: for RMSNorm six roundings against three, within
// 2^-49 of it relatively.  For |t| <= 2^17 that is within 2^-32, so where
// fast(u) is further than 2^-30 from every half-integer both round to the same
// integer; a wave with a code nearer than that evaluates exact(u) for all of
// its codes.  These kernels are
// bound by the vector ALU at prompt sizes: with the division, 64-bit integer
// conversions and clamps per code, RMSNorm of 1024 x 2048 took 9.4 us
// instead of 4.7, with the residual add 10.9 instead of 6.8, the gated
// product of 1024 x 5632 12.0 instead of 8.3.
template <int BITS, int N, class Exact, class Fast>
__device__ inline void requant_codes(int32_t* q, int32_t zy, Exact exact, Fast fast)
{
#pragma clang fp contract(off)
    double far = 0.0;
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const double t = limit_quotient(fast(u));
        const double r = t + kRintShift;
        q[u] = clamp_code<BITS>(rint_low(r) + zy);
        far = fmax(far, fabs(t - (r - kRintShift)));
    }
    if (__builtin_expect(__ballot(far > 0.5 - 0x1p-30) != 0, 0)) {
#pragma unroll
        for (int u = 0; u < N; ++u)
            q[u] = clamp_code<BITS>(rint_low(limit_quotient(exact(u)) + kRintShift) + zy);
    }
}

template <int BITS>
__device__ inline void store_code(void* y, int64_t i, int32_t v)
{
    if constexpr (BITS == 8) static_cast<int8_t*>(y)[i] = (int8_t)v;
    else static_cast<int16_t*>(y)[i] = (int16_t)v;
}

// ---------------------------------------------------------------------------
// Residual add: v = alpha_1 (x1 - zp_1) + alpha_2 (x2 - zp_2); the gated
// unit SiLU(gate) * up: the product of the two dequantized codes (each
// factor exact in fp64, the product one rounding).  OP 0: sum, 1: product.
struct Binary {
    float a1, a2;
    int32_t z1, z2;
};
template <int OP>
__device__ inline double binary_value(int32_t u, int32_t v, const Binary& p)
{
#pragma clang fp contract(off)
    const double f1 = (double)p.a1 * (double)(u - p.z1);
    const double f2 = (double)p.a2 * (double)(v - p.z2);
    return OP == 0 ? f1 + f2 : f1 * f2;
}

// N codes of OP, requantized; ri = 1 / ay
template <int BITS, int OP, int N, class U, class V>
__device__ inline void binary_codes(int32_t* q, U u, V v, const Binary& p, double ay, double ri,
                                    int32_t zy)
{
#pragma clang fp contract(off)
    double w[N];
#pragma unroll
    for (int k = 0; k < N; ++k) w[k] = binary_value<OP>(u(k), v(k), p);
    requant_codes<BITS, N>(q, zy, [&](int k) { return w[k] / ay; },
                           [&](int k) { return w[k] * ri; });
}

// n8 groups of eight codes through 16-byte loads (aligned buffers), the
// codes [begin, n) one by one
template <int BITS>
__device__ inline void store8(void* y, int64_t i, const int32_t* q);

template <int BITS, int OP>
__global__ __launch_bounds__(kThreads) void add_requant_kernel(
    const int16_t* __restrict__ x1, const int16_t* __restrict__ x2, Binary p, int64_t n8,
    int64_t begin, int64_t n, float ay, int32_t zy, void* __restrict__ y)
{
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    const int64_t t0 = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const double ri = 1.0 / (double)ay;
    for (int64_t i = t0; i < n8; i += stride) {
        const int4 g = reinterpret_cast<const int4*>(x1)[i];
        const int4 v = reinterpret_cast<const int4*>(x2)[i];
        const int16_t* gc = reinterpret_cast<const int16_t*>(&g);
        const int16_t* vc = reinterpret_cast<const int16_t*>(&v);
        int32_t q[8];
        binary_codes<BITS, OP, 8>(q, [&](int k) { return (int32_t)gc[k]; },
                                  [&](int k) { return (int32_t)vc[k]; }, p, (double)ay, ri, zy);
        store8<BITS>(y, 8 * i, q);
    }
    for (int64_t i = begin + t0; i < n; i += stride)
        store_code<BITS>(y, i,
                         requant_f64<BITS>(binary_value<OP>(x1[i], x2[i], p), (double)ay, zy));
}

// ---------------------------------------------------------------------------
// Tables of elementwise operators on int16 codes: entry i + 32768 holds the
// requantized f(alpha_x (i - zp_x)).  op 1: SiLU, v / (1 + exp(-v)).
template <int BITS>
__global__ __launch_bounds__(kThreads) void lut_build_kernel(int32_t op, float ax, int32_t zx,
                                                             float ay, int32_t zy,
                                                             void* __restrict__ lut)
{
#pragma clang fp contract(off)
    const int32_t idx = blockIdx.x * kThreads + threadIdx.x;  // 0 .. 65535
    const double v = (double)ax * (double)(idx - 32768 - zx);
    const double f = op == 1 ? v / (1.0 + exp(-v)) : v;
    store_code<BITS>(lut, idx, requant_f64<BITS>(f, (double)ay, zy));
}

// y[i] = lut[x[i] + 32768].  The table (64 or 128 KiB) is copied into LDS
// once per block, and each block then streams many codes: 8 per thread
// per trip through 16-byte loads when the buffers are aligned.
constexpr int kLutThreads = 1024;

template <int BITS>
__global__ __launch_bounds__(kLutThreads) void lut_apply_kernel(const int16_t* __restrict__ x,
                                                                int64_t n8, int64_t begin,
                                                                int64_t n,
                                                                const void* __restrict__ lut,
                                                                void* __restrict__ y)
{
    using T = typename std::conditional<BITS == 8, int8_t, int16_t>::type;
    extern __shared__ __align__(16) int8_t lds_table[];
    T* tab = reinterpret_cast<T*>(lds_table);
    {
        const int4* src = static_cast<const int4*>(lut);
        int4* dst = reinterpret_cast<int4*>(lds_table);
        constexpr int chunks = 65536 * sizeof(T) / 16;
        for (int i = threadIdx.x; i < chunks; i += kLutThreads) dst[i] = src[i];
    }
    __syncthreads();
    T* out = static_cast<T*>(y);
    const int64_t stride = (int64_t)gridDim.x * kLutThreads;
    const int64_t t0 = (int64_t)blockIdx.x * kLutThreads + threadIdx.x;
    for (int64_t i = t0; i < n8; i += stride) {
        const int4 v = reinterpret_cast<const int4*>(x)[i];
        const int16_t* c = reinterpret_cast<const int16_t*>(&v);
        T r[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) r[u] = tab[(int32_t)c[u] + 32768];
        if constexpr (BITS == 8) {
            uint2 o;
            o.x = ((uint32_t)(uint8_t)r[0]) | ((uint32_t)(uint8_t)r[1] << 8) |
                  ((uint32_t)(uint8_t)r[2] << 16) | ((uint32_t)(uint8_t)r[3] << 24);
            o.y = ((uint32_t)(uint8_t)r[4]) | ((uint32_t)(uint8_t)r[5] << 8) |
                  ((uint32_t)(uint8_t)r[6] << 16) | ((uint32_t)(uint8_t)r[7] << 24);
            reinterpret_cast<uint2*>(out)[i] = o;
        } else {
            int4 o;
            o.x = (int)(((uint32_t)(uint16_t)r[0]) | ((uint32_t)(uint16_t)r[1] << 16));
            o.y = (int)(((uint32_t)(uint16_t)r[2]) | ((uint32_t)(uint16_t)r[3] << 16));
            o.z = (int)(((uint32_t)(uint16_t)r[4]) | ((uint32_t)(uint16_t)r[5] << 16));
            o.w = (int)(((uint32_t)(uint16_t)r[6]) | ((uint32_t)(uint16_t)r[7] << 16));
            reinterpret_cast<int4*>(out)[i] = o;
        }
    }
    for (int64_t i = begin + t0; i < n; i += stride) out[i] = tab[(int32_t)x[i] + 32768];
}

// ---------------------------------------------------------------------------
// Row reductions: one block per row.
__device__ inline int64_t block_sum_i64(int64_t v, int64_t* red)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    int64_t t = 0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) t += red[w];
    __syncthreads();
    return t;
}

// Eight codes to y[i .. i+7] with one 8-byte (int8) or 16-byte (int16)
// store; i is a multiple of 8 and y is 16-byte aligned.
template <int BITS>
__device__ inline void store8(void* y, int64_t i, const int32_t* q)
{
    if constexpr (BITS == 8) {
        uint2 o;
        o.x = ((uint32_t)(uint8_t)q[0]) | ((uint32_t)(uint8_t)q[1] << 8) |
              ((uint32_t)(uint8_t)q[2] << 16) | ((uint32_t)(uint8_t)q[3] << 24);
        o.y = ((uint32_t)(uint8_t)q[4]) | ((uint32_t)(uint8_t)q[5] << 8) |
              ((uint32_t)(uint8_t)q[6] << 16) | ((uint32_t)(uint8_t)q[7] << 24);
        *reinterpret_cast<uint2*>(static_cast<int8_t*>(y) + i) = o;
    } else {
        int4 o;
        o.x = (int)(((uint32_t)(uint16_t)q[0]) | ((uint32_t)(uint16_t)q[1] << 16));
        o.y = (int)(((uint32_t)(uint16_t)q[2]) | ((uint32_t)(uint16_t)q[3] << 16));
        o.z = (int)(((uint32_t)(uint16_t)q[4]) | ((uint32_t)(uint16_t)q[5] << 16));
        o.w = (int)(((uint32_t)(uint16_t)q[6]) | ((uint32_t)(uint16_t)q[7] << 16));
        *reinterpret_cast<int4*>(static_cast<int16_t*>(y) + i) = o;
    }
}

// Four codes at x, any alignment; n < 4: only the first n exist and are
// read, the others come back as zeros.
typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v2i_any __attribute__((ext_vector_type(2), aligned(2)));
__device__ inline v2i load4_any(const int16_t* x, int n)
{
    if (n >= 4) return *reinterpret_cast<const v2i_any*>(x);
    uint32_t w[2] = {0, 0};
#pragma unroll
    for (int u = 0; u < 3; ++u)
        if (u < n) w[u / 2] |= (uint32_t)(uint16_t)x[u] << (16 * (u & 1));
    return v2i{(int)w[0], (int)w[1]};
}

// Four codes, not yet clamped to the output range, to y[i .. i+3] at any
// alignment, only the first n of them.
template <int BITS>
__device__ inline void store4_any(void* y, int64_t i, const int32_t* q, int n)
{
    using T = std::conditional_t<BITS == 8, int8_t, int16_t>;
    T* dst = static_cast<T*>(y) + i;
    struct __attribute__((packed)) Run {
        T v[4];
    } run;
    if constexpr (BITS == 16) {
#pragma unroll
        for (int u = 0; u < 4; u += 2) {
            const auto k = __builtin_amdgcn_cvt_pk_i16(q[u], q[u + 1]);  // saturating
            run.v[u] = k[0];
            run.v[u + 1] = k[1];
        }
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) run.v[u] = (T)clamp_code<BITS>(q[u]);
    }
    if (n >= 4) {
        *reinterpret_cast<Run*>(dst) = run;
    } else {
#pragma unroll
        for (int u = 0; u < 3; ++u)
            if (u < n) dst[u] = run.v[u];
    }
}

// The eight int16 codes of one 16-byte load.
typedef int v4i __attribute__((ext_vector_type(4)));
__device__ inline void unpack8(const v4i v, int32_t* c)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        c[2 * i] = (int32_t)(int16_t)v[i];
        c[2 * i + 1] = v[i] >> 16;
    }
}

// Table lookup fused with the product of two dequantized codes: the gated
// unit SiLU(gate) * up without the SiLU codes going through memory.
// u = lut[x1 + 32768] (LB-bit entries in format (a1, z1)), then the product
// with x2: the same two steps as mq_lut_apply and mq_mul_requant, so the
// same bits.  LDS: the table is copied into LDS first, the block's first
// codes loaded before it; else (fewer codes than the copy would pay for)
// entries come from memory.
template <int LB, int OB, bool LDS>
__global__ __launch_bounds__(kLutThreads) void lut_mul_kernel(
    const int16_t* __restrict__ x1, const void* __restrict__ lut, const int16_t* __restrict__ x2,
    Binary p, int64_t n8, int64_t begin, int64_t n, float ay, int32_t zy, void* __restrict__ y)
{
    using T = typename std::conditional<LB == 8, int8_t, int16_t>::type;
    extern __shared__ __align__(16) int8_t lds_table[];
    const T* tab = LDS ? reinterpret_cast<const T*>(lds_table) : static_cast<const T*>(lut);
    const int64_t stride = (int64_t)gridDim.x * kLutThreads;
    const int64_t t0 = (int64_t)blockIdx.x * kLutThreads + threadIdx.x;
    v4i g = {0, 0, 0, 0}, v = {0, 0, 0, 0};
    if (t0 < n8) {
        g = reinterpret_cast<const v4i*>(x1)[t0];
        v = reinterpret_cast<const v4i*>(x2)[t0];
    }
    if constexpr (LDS) {
        const v4i* src = static_cast<const v4i*>(lut);
        v4i* dst = reinterpret_cast<v4i*>(lds_table);
        constexpr int chunks = 65536 * sizeof(T) / 16 / kLutThreads;
        v4i c[chunks];
#pragma unroll
        for (int i = 0; i < chunks; ++i) c[i] = src[threadIdx.x + i * kLutThreads];
#pragma unroll
        for (int i = 0; i < chunks; ++i) dst[threadIdx.x + i * kLutThreads] = c[i];
        __syncthreads();
    }
    const double ri = 1.0 / (double)ay;
    for (int64_t i = t0; i < n8; i += stride) {
        v4i gn = g, vn = v;  // the next group is on its way during this one
        if (i + stride < n8) {
            gn = reinterpret_cast<const v4i*>(x1)[i + stride];
            vn = reinterpret_cast<const v4i*>(x2)[i + stride];
        }
        int32_t gc[8], vc[8], q[8];
        unpack8(g, gc);
        unpack8(v, vc);
#pragma unroll
        for (int k = 0; k < 8; ++k) gc[k] = tab[gc[k] + 32768];
        binary_codes<OB, 1, 8>(q, [&](int k) { return gc[k]; }, [&](int k) { return vc[k]; }, p,
                               (double)ay, ri, zy);
        store8<OB>(y, 8 * i, q);
        g = gn;
        v = vn;
    }
    for (int64_t i = begin + t0; i < n; i += stride)
        store_code<OB>(y, i, requant_f64<OB>(binary_value<1>(tab[(int32_t)x1[i] + 32768], x2[i], p),
                                             (double)ay, zy));
}

// Rows of at most 8 * 256 * NCH codes with K % 8 == 0 and 16-byte aligned
// rows stay in registers: chunk c of thread t holds codes
// 8 (t + 256 c) .. +7, read once with a 16-byte load.
template <int NCH>
struct RowRegs {
    int16_t v[NCH][8];
    bool live[NCH];
    __device__ void load(const int16_t* row, int64_t K)
    {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int64_t k0 = 8 * ((int64_t)threadIdx.x + kThreads * c);
            live[c] = k0 < K;
            int4 q = {0, 0, 0, 0};
            if (live[c]) q = *reinterpret_cast<const int4*>(row + k0);
            const int16_t* e = reinterpret_cast<const int16_t*>(&q);
#pragma unroll
            for (int u = 0; u < 8; ++u) v[c][u] = e[u];
        }
    }
};

// The row's chunks normalized: v = a d [* gamma] / rt, code rint(v / ay) + zy,
// for d = code - zero-point.  gamma is loaded before the reduction (gm).
template <int NCH>
struct GammaRegs {
    float4 lo[NCH], hi[NCH];
    __device__ void load(const float* gamma, int64_t K)
    {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int64_t k0 = 8 * ((int64_t)threadIdx.x + kThreads * c);
            lo[c] = hi[c] = make_float4(1.0f, 1.0f, 1.0f, 1.0f);
            if (gamma && k0 < K) {
                // gamma need not be 16-byte aligned
                const float* g = gamma + k0;
                lo[c] = make_float4(g[0], g[1], g[2], g[3]);
                hi[c] = make_float4(g[4], g[5], g[6], g[7]);
            }
        }
    }
    __device__ double at(int c, int u) const
    {
        const float4 h = u < 4 ? lo[c] : hi[c];
        return (double)((u & 3) == 0 ? h.x : (u & 3) == 1 ? h.y : (u & 3) == 2 ? h.z : h.w);
    }
};

template <int BITS, class D, class G>
__device__ inline void norm_codes(int32_t* q, D d, G gamma, double a, double rt, double ay,
                                  int32_t zy)
{
#pragma clang fp contract(off)
    const double c = (1.0 / rt) * (1.0 / ay) * a;
    requant_codes<BITS, 8>(
        q, zy,
        [&](int u) {
            double v = a * (double)d(u);
            v = v * gamma(u);  // (exact without gamma: 1)
            v = v / rt;
            return v / ay;
        },
        [&](int u) { return (double)d(u) * gamma(u) * c; });
}

// sum_k (code - zp)^2 of the row: 32-bit squares (|d| <= 65535), 64-bit sums
__device__ inline uint64_t square(int32_t d) { return (uint64_t)((uint32_t)d * (uint32_t)d); }

template <int BITS, int NCH>
__global__ __launch_bounds__(kThreads) void rmsnorm_regs_kernel(const int16_t* __restrict__ x,
                                                                int64_t K, float ax, int32_t zx,
                                                                const float* __restrict__ gamma,
                                                                float eps, float ay, int32_t zy,
                                                                void* __restrict__ y)
{
#pragma clang fp contract(off)
    __shared__ int64_t red[kThreads / 64];
    const int64_t m = blockIdx.x;
    RowRegs<NCH> r;
    r.load(x + m * K, K);
    GammaRegs<NCH> gm;
    gm.load(gamma, K);
    uint64_t ss = 0;
#pragma unroll
    for (int c = 0; c < NCH; ++c)
        if (r.live[c])
#pragma unroll
            for (int u = 0; u < 8; ++u) ss += square(r.v[c][u] - zx);
    ss = (uint64_t)block_sum_i64((int64_t)ss, red);
    const double a = (double)ax;
    const double ms = a * a * (double)(int64_t)ss / (double)K + (double)eps;
    const double rt = sqrt(ms);
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        if (!r.live[c]) continue;
        const int64_t k0 = 8 * ((int64_t)threadIdx.x + kThreads * c);
        int32_t q[8];
        norm_codes<BITS>(q, [&](int u) { return r.v[c][u] - zx; },
                         [&](int u) { return gm.at(c, u); }, a, rt, (double)ay, zy);
        store8<BITS>(y, m * K + k0, q);
    }
}

// Residual add fused with the RMSNorm that reads its result: per row, the
// sum codes h = code_h(a1 (x1 - z1) + a2 (x2 - z2)) are written and, still
// in registers, normalized as rmsnorm_regs_kernel normalizes its input.  The
// same values as mq_add_requant then mq_rmsnorm, so the same bits, with one
// read of h less and one launch less.
template <int BITS, int NCH>
__global__ __launch_bounds__(kThreads) void add_rmsnorm_kernel(
    const int16_t* __restrict__ x1, const int16_t* __restrict__ x2, Binary p, int64_t K, float ah,
    int32_t zh, int16_t* __restrict__ h, const float* __restrict__ gamma, float eps, float ay,
    int32_t zy, void* __restrict__ y)
{
#pragma clang fp contract(off)
    __shared__ int64_t red[kThreads / 64];
    const int64_t m = blockIdx.x;
    RowRegs<NCH> r1, r2;
    r1.load(x1 + m * K, K);
    r2.load(x2 + m * K, K);
    GammaRegs<NCH> gm;
    gm.load(gamma, K);
    const double rih = 1.0 / (double)ah;
    int32_t hc[NCH][8];
    uint64_t ss = 0;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        if (!r1.live[c]) continue;
        const int64_t k0 = 8 * ((int64_t)threadIdx.x + kThreads * c);
        binary_codes<16, 0, 8>(hc[c], [&](int u) { return (int32_t)r1.v[c][u]; },
                               [&](int u) { return (int32_t)r2.v[c][u]; }, p, (double)ah, rih, zh);
#pragma unroll
        for (int u = 0; u < 8; ++u) ss += square(hc[c][u] - zh);
        store8<16>(h, m * K + k0, hc[c]);
    }
    ss = (uint64_t)block_sum_i64((int64_t)ss, red);
    const double a = (double)ah;
    const double ms = a * a * (double)(int64_t)ss / (double)K + (double)eps;
    const double rt = sqrt(ms);
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        if (!r1.live[c]) continue;
        const int64_t k0 = 8 * ((int64_t)threadIdx.x + kThreads * c);
        int32_t q[8];
        norm_codes<BITS>(q, [&](int u) { return hc[c][u] - zh; },
                         [&](int u) { return gm.at(c, u); }, a, rt, (double)ay, zy);
        store8<BITS>(y, m * K + k0, q);
    }
}

// Keys row m of a causal softmax sees: (m mod period) + offset + 1, at most
// K (period 0: all K).
__device__ inline int64_t causal_keys(int64_t m, int64_t K, int64_t period, int64_t offset)
{
    if (period <= 0) return K;
    const int64_t n = m % period + offset + 1;
    return n < K ? n : K;
}

// Rows of at most 2048 codes, one wave per row, in chunks of 256 keys, four
// per lane (a causal row skips the chunks past its boundary).  The exponent
// alpha (x_k - max) is -alpha d with d = max - x_k an integer in [0, 65535]
// and alpha an fp32 scale, so alpha d is exact in fp64 and, for
// d = 256 h + l,
//   exp(-alpha d) = exp(-256 alpha h) exp(-alpha l).
// Each block evaluates the two 256-entry factor tables once (one exp per
// entry, in LDS); a key then costs two table reads and one fp64 product,
// within three ulp of the direct exp, and its quotient is e * s with s =
// (1 / sum) (1 / ay): with the exps and the sum in another order 36 ulp at
// most, below 2^-46, from the definition's e / sum / ay, so less than 2^-29 up
// to 2^17.  A row (EXACT) with a quotient that near a half-integer is
// evaluated again as it is defined (exact_codes), so that no code depends on
// the tables.  Hidden keys are written as zy.
// Each wave takes kSmRows rows in snake order (m, 2G - 1 - m, ... for G waves
// in the grid): under a causal mask whose period divides 2G
// the key counts of each pair sum to the period plus one.
constexpr int kSmWaves = 8, kSmRows = 2;

typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

__device__ inline s16x2 as_s16x2(int v) { return __builtin_bit_cast(s16x2, v); }

// DPP lane moves within rows of 16 lanes (all 64 lanes active)
template <int CTRL>
__device__ inline int dpp_mov(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;

template <int CTRL>
__device__ inline double dpp_f64(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = dpp_mov<CTRL>((int)b), hi = dpp_mov<CTRL>((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

__device__ inline double readlane_f64(double v, int l)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// wave-wide max and fp64 sum: butterfly within each 16-lane row, then the
// four row results; every lane gets the same value
__device__ inline int32_t wave_max_i32(int32_t v)
{
    v = max(v, dpp_mov<kDppXor1>(v));
    v = max(v, dpp_mov<kDppXor2>(v));
    v = max(v, dpp_mov<kDppHalfMirror>(v));
    v = max(v, dpp_mov<kDppMirror>(v));
    const int a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 16);
    const int c = __builtin_amdgcn_readlane(v, 32), d = __builtin_amdgcn_readlane(v, 48);
    return max(max(a, b), max(c, d));
}

__device__ inline double wave_sum_f64(double v)
{
#pragma clang fp contract(off)
    v = v + dpp_f64<kDppXor1>(v);
    v = v + dpp_f64<kDppXor2>(v);
    v = v + dpp_f64<kDppHalfMirror>(v);
    v = v + dpp_f64<kDppMirror>(v);
    return (readlane_f64(v, 0) + readlane_f64(v, 16)) + (readlane_f64(v, 32) + readlane_f64(v, 48));
}

// The factor tables in LDS.  (Sixteen copies of the second, a lane reading
// copy lane mod 16, free its reads of bank conflicts and changed nothing:
// the reads are not what bounds these kernels.)
struct ExpTables {
    double h[256];  // exp(-256 alpha h)
    double l[256];  // exp(-alpha l)

    __device__ void fill(double a)
    {
#pragma clang fp contract(off)
        for (int i = threadIdx.x; i < 512; i += blockDim.x) {
            if (i < 256) h[i] = exp(-(a * (double)(256 * i)));
            else l[i - 256] = exp(-(a * (double)(i - 256)));
        }
        __syncthreads();
    }
    // the factor products of the two keys of one packed word
    __device__ void pair(int w, s16x2 mx2, double& e0, double& e1) const
    {
#pragma clang fp contract(off)
        const uint32_t D =
            __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, mx2 - as_s16x2(w)));
        e0 = h[(D >> 8) & 255u] * l[D & 255u];
        e1 = h[D >> 24] * l[(D >> 16) & 255u];
    }
};

// t + zy to the nearest integer, not yet clamped to the output range.
// EXACT: for t in [0, 2^17]; adding 1.5 * 2^20 leaves the integer part of t in
// the high word and its fraction, to 2^-32, in the low one, and near becomes
// the least of the fractions' distances above kTieLow, at most kTieSpan for one
// within 2^-29 of a half.  Otherwise 1.5 * 2^52 rounds t in [0, 2^31) to an
// integer (ties to even) in the low word.  CLAMP caps t where it may be
// larger (s is; e <= 1).
constexpr double kSplitShift = 1572864.0;   // 1.5 * 2^20
constexpr int32_t kSplitHigh = 0x41380000;  // its high word
constexpr uint32_t kTieLow = 0x80000000u - 8, kTieSpan = 16;
template <bool CLAMP, bool EXACT>
__device__ inline int32_t requant_prob(double e, double s, int32_t zy, uint32_t& near)
{
#pragma clang fp contract(off)
    double t = e * s;
    if (CLAMP) t = fmin(t, 131072.0);
    if constexpr (!EXACT) return rint_low(t + kRintShift) + zy;
    const uint64_t b = (uint64_t)__double_as_longlong(t + kSplitShift);
    const uint32_t frac = (uint32_t)b;
    near = min(near, frac - kTieLow);
    return (int32_t)(b >> 32) + (int32_t)(frac >> 31) + (zy - kSplitHigh);
}

// A wave's part of one row: chunk c < NCA is the 256 keys from first + step c
// on, four per lane, and holds the boundary n (the keys visible) only if it
// is the last.  n, K, first and step are wave-uniform.  The number of chunks
// is a template argument (the kernels switch on it), so a row is straight
// code: with a branch per chunk the merged registers were copied more often
// than they were used.
constexpr int kChunk = 256;

template <int NCA>
struct RowPart {
    v2i q[NCA];
    double e[NCA][4];

    __device__ __forceinline__ void load(const int16_t* row, int K, int first, int step)
    {
        const int k = 4 * (threadIdx.x & 63);
#pragma unroll
        for (int c = 0; c < NCA; ++c) {
            const int f = first + step * c;
            if (c + 1 < NCA || f + kChunk <= K) {
                q[c] = *reinterpret_cast<const v2i_any*>(row + f + k);
            } else {
                q[c] = v2i{0, 0};
                if (f + k < K) q[c] = load4_any(row + f + k, K - f - k);
            }
        }
    }
    __device__ __forceinline__ int32_t max_code(int n, int first, int step) const
    {
        const int left = n - first - step * (NCA - 1) - 4 * (int)(threadIdx.x & 63);
        s16x2 a = as_s16x2(q[NCA - 1][0]), b = as_s16x2(q[NCA - 1][1]);
        if (left < 1) a.x = -32768;
        if (left < 2) a.y = -32768;
        if (left < 3) b.x = -32768;
        if (left < 4) b.y = -32768;
        s16x2 mx = __builtin_elementwise_max(a, b);
#pragma unroll
        for (int c = 0; c + 1 < NCA; ++c)
            mx = __builtin_elementwise_max(
                mx, __builtin_elementwise_max(as_s16x2(q[c][0]), as_s16x2(q[c][1])));
        return max((int32_t)mx.x, (int32_t)mx.y);
    }
    // the exponentials (0 for hidden keys, whose codes are zero or real
    // scores) and their sum
    __device__ __forceinline__ double exponentials(int n, int32_t mx, const ExpTables& tab, int first,
                                                   int step)
    {
#pragma clang fp contract(off)
        const int left = n - first - step * (NCA - 1) - 4 * (int)(threadIdx.x & 63);
        const s16x2 mx2 = {(short)mx, (short)mx};
        double sum = 0.0;
#pragma unroll
        for (int c = 0; c < NCA; ++c) {
            tab.pair(q[c][0], mx2, e[c][0], e[c][1]);
            tab.pair(q[c][1], mx2, e[c][2], e[c][3]);
            if (c + 1 == NCA)
#pragma unroll
                for (int u = 0; u < 4; ++u) e[c][u] = u < left ? e[c][u] : 0.0;
            sum += (e[c][0] + e[c][1]) + (e[c][2] + e[c][3]);
        }
        return sum;
    }
    // e s + zy of every key, rounded (hidden keys: zy); whether one of the
    // wave's lies near a tie
    template <bool CLAMP, bool EXACT>
    __device__ __forceinline__ bool codes(double s, int32_t zy, int32_t (&o)[NCA][4]) const
    {
        uint32_t near = 0xFFFFFFFFu;
#pragma unroll
        for (int c = 0; c < NCA; ++c)
#pragma unroll
            for (int u = 0; u < 4; ++u)
                o[c][u] = requant_prob<CLAMP, EXACT>(e[c][u], s, zy, near);
        return EXACT && __ballot(near <= kTieSpan) != 0;
    }
    template <int BITS>
    __device__ __forceinline__ static void store(const int32_t (&o)[NCA][4], int K, void* y,
                                                 int64_t base, int first, int step)
    {
        const int k = 4 * (threadIdx.x & 63);
#pragma unroll
        for (int c = 0; c < NCA; ++c) {
            const int f = first + step * c;
            if (c + 1 < NCA || f + kChunk <= K) store4_any<BITS>(y, base + f + k, o[c], 4);
            else if (f + k < K) store4_any<BITS>(y, base + f + k, o[c], K - f - k);
        }
    }
};

// The definition, key by key: keys t, t + step, ... of the row (the sum over
// them, then the codes of those below `end`, hidden ones zy).
__device__ __forceinline__ double exact_sum(const int16_t* row, int n, int32_t mx, double a, int t,
                                            int step)
{
#pragma clang fp contract(off)
    double sum = 0.0;
#pragma unroll 1
    for (int k = t; k < n; k += step) sum += exp(a * (double)((int32_t)row[k] - mx));
    return sum;
}
template <int BITS>
__device__ __forceinline__ void exact_codes(const int16_t* row, int n, int end, int32_t mx,
                                            double a, double sum, double ay, int32_t zy, void* y,
                                            int64_t base, int t, int step)
{
#pragma clang fp contract(off)
#pragma unroll 1
    for (int k = t; k < end; k += step) {
        int32_t q = zy;
        if (k < n) q = requant_f64<BITS>(exp(a * (double)((int32_t)row[k] - mx)) / sum, ay, zy);
        store_code<BITS>(y, base + k, q);
    }
}

// the wave's chunks past the boundary: probability 0
template <int BITS>
__device__ __forceinline__ void hidden_codes(int K, int32_t zy, void* y, int64_t base, int first,
                                             int step)
{
    const int k = 4 * (threadIdx.x & 63);
    const int32_t o[4] = {zy, zy, zy, zy};
    for (int f = first; f < K; f += step) {
        if (f + kChunk <= K) store4_any<BITS>(y, base + f + k, o, 4);
        else if (f + k < K) store4_any<BITS>(y, base + f + k, o, K - f - k);
    }
}

// CLAMP: 1 / ay > 2^17.
// Loads and stores take rows of any length and alignment.
// Bound by memory at 1024 codes (a plain copy of the 64 MB takes 17.0 us).
// Measured, 32 heads of causal rows: 1024 codes 23.3 us (27.3 with a branch
// per chunk of eight codes and four rows per wave), 777 codes 19.1 us with the
// tie check, 17.9 without (26; 70 on the strided kernel, an exp per key and
// pass).  Two rows per wave: four took 22.6 and 19.8 us, and 5.9 instead of
// 5.3 us at 256 tokens.
// The row's codes; false, and nothing stored, if one lies near a tie.
template <int BITS, bool CLAMP, bool EXACT, int NCA>
__device__ __forceinline__ bool softmax_row(const int16_t* x, int64_t m, int K, int n,
                                            const ExpTables& tab, double ri, int32_t zy, void* y)
{
#pragma clang fp contract(off)
    RowPart<NCA> r;
    r.load(x + m * K, K, 0, kChunk);
    const int32_t mx = wave_max_i32(r.max_code(n, 0, kChunk));
    // sum >= 1: the maximum key contributes exp(0)
    const double sum = wave_sum_f64(r.exponentials(n, mx, tab, 0, kChunk));
    int32_t o[NCA][4];
    if (r.template codes<CLAMP, EXACT>((1.0 / sum) * ri, zy, o)) return false;
    r.template store<BITS>(o, K, y, m * K, 0, kChunk);
    return true;
}

// MAXC: chunks of the longest row (4 or 8: with 4 the kernel's registers
// allow eight waves per SIMD).
template <int BITS, bool CLAMP, bool EXACT, int MAXC>
__global__ __launch_bounds__(kSmWaves * 64) void softmax_table_kernel(
    const int16_t* __restrict__ x, int64_t M, int64_t K, float ax, float ay, int32_t zy,
    int64_t period, int64_t offset, void* __restrict__ y)
{
    __shared__ ExpTables tab;
    tab.fill((double)ax);
    const int64_t G = (int64_t)gridDim.x * kSmWaves;
    const int64_t g = (int64_t)blockIdx.x * kSmWaves +
                      __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const double ri = 1.0 / (double)ay;
    const int k32 = (int)K;
    auto row_of = [&](int r) { return (r & 1) ? (int64_t)(r + 1) * G - 1 - g : (int64_t)r * G + g; };
    // keys row m sees; M < 2^31, so m % period fits 32 bits
    auto keys_of = [&](int64_t m) {
        if (period > 0) {
            const int64_t t = period > m ? m : (int64_t)((uint32_t)m % (uint32_t)period);
            if (t + offset + 1 < K) return (int)(t + offset) + 1;
        }
        return k32;
    };
    uint32_t again = 0;  // rows near a tie, one bit each
#pragma unroll 1
    for (int r = 0; r < kSmRows; ++r) {
        const int64_t m = row_of(r);
        if (m >= M) continue;
        const int n = keys_of(m);
        const int nca = (n + kChunk - 1) / kChunk;
        bool done;
        if (nca == 1) done = softmax_row<BITS, CLAMP, EXACT, 1>(x, m, k32, n, tab, ri, zy, y);
        else if (nca == 2) done = softmax_row<BITS, CLAMP, EXACT, 2>(x, m, k32, n, tab, ri, zy, y);
        else if (nca == 3) done = softmax_row<BITS, CLAMP, EXACT, 3>(x, m, k32, n, tab, ri, zy, y);
        else if (MAXC == 4 || nca == 4)
            done = softmax_row<BITS, CLAMP, EXACT, 4>(x, m, k32, n, tab, ri, zy, y);
        else if (nca == 5) done = softmax_row<BITS, CLAMP, EXACT, 5>(x, m, k32, n, tab, ri, zy, y);
        else if (nca == 6) done = softmax_row<BITS, CLAMP, EXACT, 6>(x, m, k32, n, tab, ri, zy, y);
        else if (nca == 7) done = softmax_row<BITS, CLAMP, EXACT, 7>(x, m, k32, n, tab, ri, zy, y);
        else done = softmax_row<BITS, CLAMP, EXACT, 8>(x, m, k32, n, tab, ri, zy, y);
        if (!done) again |= 1u << r;
        hidden_codes<BITS>(k32, zy, y, m * K, nca * kChunk, kChunk);
    }
    // (after the loop: inside it, the registers of its exp cost the kernel
    // three of seven waves per SIMD)
    if (!EXACT || __builtin_expect(again == 0, 1)) return;
    const int lane = threadIdx.x & 63;
    const double a = (double)ax;
#pragma unroll 1
    for (int r = 0; r < kSmRows; ++r) {
        if (!(again >> r & 1)) continue;
        const int64_t m = row_of(r);
        const int16_t* row = x + m * K;
        const int n = keys_of(m), end = (n + kChunk - 1) / kChunk * kChunk;
        int32_t mx = -32768;
        for (int k = lane; k < n; k += 64) mx = max(mx, (int32_t)row[k]);
        mx = wave_max_i32(mx);
        const double sum = wave_sum_f64(exact_sum(row, n, mx, a, lane, 64));
        exact_codes<BITS>(row, n, min(k32, end), mx, a, sum, (double)ay, zy, y, m * K, lane, 64);
    }
}

// The same with four waves per row and one row per block: rows of up to 8192
// codes, and few rows (the 32 heads of one query), where a wave per row
// would leave most of the chip idle and 24 keys in a lane's chain (32 rows of
// 1531 codes: 8.0 us on the strided kernel, 3.4 us here).
template <int BITS, bool CLAMP, bool EXACT, int NCA>
__device__ __forceinline__ bool softmax_block_row(const int16_t* x, int64_t m, int K, int n,
                                                  const ExpTables& tab, double ri, int32_t zy,
                                                  int32_t* red_i, double* red_d, void* y,
                                                  int32_t& mx)
{
#pragma clang fp contract(off)
    constexpr int NW = kThreads / 64, step = NW * kChunk;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int first = wave * kChunk;
    // (n lies in the last four chunks: a wave's last one may hold the
    // boundary or nothing, the others are whole)
    RowPart<NCA> r;
    const int last = first + step * (NCA - 1);
    r.load(x + m * K, K, first, step);
    mx = wave_max_i32(r.max_code(n, first, step));
    if ((threadIdx.x & 63) == 0) red_i[wave] = mx;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) mx = max(mx, red_i[w]);
    double sum = wave_sum_f64(r.exponentials(n, mx, tab, first, step));
    if ((threadIdx.x & 63) == 0) red_d[wave] = sum;
    __syncthreads();
    sum = (red_d[0] + red_d[1]) + (red_d[2] + red_d[3]);
    int32_t o[NCA][4];
    const bool near = r.template codes<CLAMP, EXACT>((1.0 / sum) * ri, zy, o);
    if constexpr (EXACT) {  // (every wave has read the maxima by now)
        if ((threadIdx.x & 63) == 0) red_i[wave] = near;
        __syncthreads();
        if ((red_i[0] | red_i[1] | red_i[2] | red_i[3]) != 0) return false;
    }
    r.template store<BITS>(o, K, y, m * K, first, step);
    return true;
}

template <int BITS, bool CLAMP, bool EXACT>
__global__ __launch_bounds__(kThreads) void softmax_block_kernel(
    const int16_t* __restrict__ x, int64_t K, float ax, float ay, int32_t zy, int64_t period,
    int64_t offset, void* __restrict__ y)
{
    __shared__ ExpTables tab;
    __shared__ int32_t red_i[kThreads / 64];
    __shared__ double red_d[kThreads / 64];
    const int64_t m = blockIdx.x;
    const int n = (int)causal_keys(m, K, period, offset);  // keys this row sees
    tab.fill((double)ax);
    const double ri = 1.0 / (double)ay;
    const int k32 = (int)K;
    int32_t mx;
    bool done;
    const int parts = (n + 4 * kChunk - 1) / (4 * kChunk);
    switch (parts) {
    case 1: done = softmax_block_row<BITS, CLAMP, EXACT, 1>(x, m, k32, n, tab, ri, zy, red_i, red_d, y, mx); break;
    case 2: done = softmax_block_row<BITS, CLAMP, EXACT, 2>(x, m, k32, n, tab, ri, zy, red_i, red_d, y, mx); break;
    case 3: done = softmax_block_row<BITS, CLAMP, EXACT, 3>(x, m, k32, n, tab, ri, zy, red_i, red_d, y, mx); break;
    case 4: done = softmax_block_row<BITS, CLAMP, EXACT, 4>(x, m, k32, n, tab, ri, zy, red_i, red_d, y, mx); break;
    case 5: done = softmax_block_row<BITS, CLAMP, EXACT, 5>(x, m, k32, n, tab, ri, zy, red_i, red_d, y, mx); break;
    case 6: done = softmax_block_row<BITS, CLAMP, EXACT, 6>(x, m, k32, n, tab, ri, zy, red_i, red_d, y, mx); break;
    case 7: done = softmax_block_row<BITS, CLAMP, EXACT, 7>(x, m, k32, n, tab, ri, zy, red_i, red_d, y, mx); break;
    default: done = softmax_block_row<BITS, CLAMP, EXACT, 8>(x, m, k32, n, tab, ri, zy, red_i, red_d, y, mx); break;
    }
    const int end = min(k32, parts * 4 * kChunk);
    if (EXACT && __builtin_expect(!done, 0)) {  // for the whole block
        const int t = threadIdx.x;
        const double a = (double)ax;
        double sum = wave_sum_f64(exact_sum(x + m * K, n, mx, a, t, kThreads));
        __syncthreads();
        if ((t & 63) == 0) red_d[t >> 6] = sum;
        __syncthreads();
        sum = (red_d[0] + red_d[1]) + (red_d[2] + red_d[3]);
        exact_codes<BITS>(x + m * K, n, end, mx, a, sum, (double)ay, zy, y, m * K, t, kThreads);
    }
    hidden_codes<BITS>(k32, zy, y, m * K, end + kChunk * (int)(threadIdx.x >> 6), 4 * kChunk);
}

// RMSNorm: ss = sum (x - zp_x)^2 (exact, int64); ms = alpha^2 ss / K + eps;
// r = sqrt(ms); v = alpha (x - zp_x) [* gamma_k] / r.
template <int BITS>
__global__ __launch_bounds__(kThreads) void rmsnorm_kernel(const int16_t* __restrict__ x,
                                                           int64_t K, float ax, int32_t zx,
                                                           const float* __restrict__ gamma,
                                                           float eps, float ay, int32_t zy,
                                                           void* __restrict__ y)
{
#pragma clang fp contract(off)
    __shared__ int64_t red[kThreads / 64];
    const int64_t m = blockIdx.x;
    const int16_t* row = x + m * K;
    int64_t ss = 0;
    for (int64_t k = threadIdx.x; k < K; k += kThreads) {
        const int64_t d = (int64_t)row[k] - zx;
        ss += d * d;
    }
    ss = block_sum_i64(ss, red);
    const double a = (double)ax;
    const double ms = a * a * (double)ss / (double)K + (double)eps;
    const double r = sqrt(ms);
    for (int64_t k = threadIdx.x; k < K; k += kThreads) {
        double v = a * (double)((int64_t)row[k] - zx);
        if (gamma) v = v * (double)gamma[k];
        v = v / r;
        store_code<BITS>(y, m * K + k, requant_f64<BITS>(v, (double)ay, zy));
    }
}

// Softmax: e_k = exp(alpha (x_k - max_j x_j)), p_k = e_k / sum_j e_j.
template <int BITS>
__global__ __launch_bounds__(kThreads) void softmax_kernel(const int16_t* __restrict__ x,
                                                           int64_t K, float ax, float ay,
                                                           int32_t zy, int64_t period,
                                                           int64_t offset, void* __restrict__ y)
{
#pragma clang fp contract(off)
    __shared__ int32_t red_i[kThreads / 64];
    __shared__ double red_d[kThreads / 64];
    const int64_t m = blockIdx.x;
    const int64_t n = causal_keys(m, K, period, offset);  // keys this row sees
    const int16_t* row = x + m * K;
    int32_t mx = -32768;
    for (int64_t k = threadIdx.x; k < n; k += kThreads) mx = max(mx, (int32_t)row[k]);
    for (int o = 32; o > 0; o >>= 1) mx = max(mx, __shfl_xor(mx, o));
    if ((threadIdx.x & 63) == 0) red_i[threadIdx.x >> 6] = mx;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) mx = max(mx, red_i[w]);
    const double a = (double)ax;
    double sum = 0.0;
    for (int64_t k = threadIdx.x; k < n; k += kThreads)
        sum += exp(a * (double)((int32_t)row[k] - mx));
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
    if ((threadIdx.x & 63) == 0) red_d[threadIdx.x >> 6] = sum;
    __syncthreads();
    sum = 0.0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) sum += red_d[w];
    for (int64_t k = threadIdx.x; k < K; k += kThreads) {
        if (k >= n) {  // past the causal boundary: probability 0
            store_code<BITS>(y, m * K + k, zy);
            continue;
        }
        const double e = exp(a * (double)((int32_t)row[k] - mx));
        store_code<BITS>(y, m * K + k, requant_f64<BITS>(e / sum, (double)ay, zy));
    }
}

}  // namespace

template <int OP>
static hipError_t launch_binary(const int16_t* x1, float a1, int32_t z1, const int16_t* x2,
                                float a2, int32_t z2, int64_t n, float ay, int32_t zy,
                                int32_t bits, void* y, hipStream_t st)
{
    const uintptr_t ya = bits == 8 ? 8 : 16;
    const bool vec = ((uintptr_t)x1 % 16) == 0 && ((uintptr_t)x2 % 16) == 0 &&
                     ((uintptr_t)y % ya) == 0;
    const int64_t n8 = vec ? n / 8 : 0;
    const int g = grid_for(vec ? n8 : n, kThreads, 256 * 64);
    const Binary p{a1, a2, z1, z2};
    if (bits == 8)
        add_requant_kernel<8, OP><<<g, kThreads, 0, st>>>(x1, x2, p, n8, n8 * 8, n, ay, zy, y);
    else
        add_requant_kernel<16, OP><<<g, kThreads, 0, st>>>(x1, x2, p, n8, n8 * 8, n, ay, zy, y);
    return hipGetLastError();
}

hipError_t launch_add_requant(const int16_t* x1, float a1, int32_t z1, const int16_t* x2,
                              float a2, int32_t z2, int64_t n, float ay, int32_t zy,
                              int32_t bits, void* y, hipStream_t st)
{
    return launch_binary<0>(x1, a1, z1, x2, a2, z2, n, ay, zy, bits, y, st);
}

hipError_t launch_mul_requant(const int16_t* x1, float a1, int32_t z1, const int16_t* x2,
                              float a2, int32_t z2, int64_t n, float ay, int32_t zy,
                              int32_t bits, void* y, hipStream_t st)
{
    return launch_binary<1>(x1, a1, z1, x2, a2, z2, n, ay, zy, bits, y, st);
}

hipError_t launch_lut_build(int32_t op, float ax, int32_t zx, float ay, int32_t zy, int32_t bits,
                            void* lut, hipStream_t st)
{
    if (bits == 8) lut_build_kernel<8><<<65536 / kThreads, kThreads, 0, st>>>(op, ax, zx, ay, zy, lut);
    else lut_build_kernel<16><<<65536 / kThreads, kThreads, 0, st>>>(op, ax, zx, ay, zy, lut);
    return hipGetLastError();
}

hipError_t launch_lut_apply(const int16_t* x, int64_t n, const void* lut, int32_t bits, void* y,
                            hipStream_t st)
{
    // one or two blocks per CU (the table fills 64 or 128 KiB of LDS), each
    // streaming at least 16 codes per thread (the 1024 x 5632 SiLU input
    // then fills all 256 CUs)
    const uintptr_t ya = bits == 8 ? 8 : 16;
    const bool vec = ((uintptr_t)x % 16) == 0 && ((uintptr_t)y % ya) == 0 &&
                     ((uintptr_t)lut % 16) == 0;
    const int64_t n8 = vec ? n / 8 : 0;
    const int cap = bits == 8 ? 512 : 256;
    const int g = grid_for(n, kLutThreads * 16, cap);
    const size_t lds = 65536 * (bits / 8);
    if (bits == 8) {
        static const hipError_t a8 = hipFuncSetAttribute(
            reinterpret_cast<const void*>(&lut_apply_kernel<8>),
            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (a8 != hipSuccess) return a8;
        lut_apply_kernel<8><<<g, kLutThreads, lds, st>>>(x, n8, n8 * 8, n, lut, y);
    } else {
        static const hipError_t a16 = hipFuncSetAttribute(
            reinterpret_cast<const void*>(&lut_apply_kernel<16>),
            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (a16 != hipSuccess) return a16;
        lut_apply_kernel<16><<<g, kLutThreads, lds, st>>>(x, n8, n8 * 8, n, lut, y);
    }
    return hipGetLastError();
}

template <int LB, int OB>
static hipError_t lut_mul_launch(const int16_t* x1, const void* lut, float a1, int32_t z1,
                                 const int16_t* x2, float a2, int32_t z2, int64_t n, float ay,
                                 int32_t zy, void* y, hipStream_t st)
{
    const uintptr_t ya = OB == 8 ? 8 : 16;
    const bool vec = ((uintptr_t)x1 % 16) == 0 && ((uintptr_t)x2 % 16) == 0 &&
                     ((uintptr_t)y % ya) == 0 && ((uintptr_t)lut % 16) == 0;
    const int64_t n8 = vec ? n / 8 : 0;
    const Binary p{a1, a2, z1, z2};
    // up to 64 Ki codes (the gated unit of a few tokens) cost less from
    // memory than the copy of the table
    if (n <= 65536) {
        const int g = grid_for(vec ? n8 : n, kLutThreads, 256 * 64);
        lut_mul_kernel<LB, OB, false><<<g, kLutThreads, 0, st>>>(x1, lut, x2, p, n8, n8 * 8, n, ay,
                                                                 zy, y);
        return hipGetLastError();
    }
    const int g = grid_for(n, kLutThreads * 16, LB == 8 ? 512 : 256);
    const size_t lds = 65536 * (LB / 8);
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(&lut_mul_kernel<LB, OB, true>),
        hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (attr != hipSuccess) return attr;
    lut_mul_kernel<LB, OB, true><<<g, kLutThreads, lds, st>>>(x1, lut, x2, p, n8, n8 * 8, n, ay, zy,
                                                              y);
    return hipGetLastError();
}

hipError_t launch_lut_mul(const int16_t* x1, const void* lut, int32_t lut_bits, float a1,
                          int32_t z1, const int16_t* x2, float a2, int32_t z2, int64_t n,
                          float ay, int32_t zy, int32_t bits, void* y, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    if (lut_bits == 8)
        return bits == 8 ? lut_mul_launch<8, 8>(x1, lut, a1, z1, x2, a2, z2, n, ay, zy, y, st)
                         : lut_mul_launch<8, 16>(x1, lut, a1, z1, x2, a2, z2, n, ay, zy, y, st);
    return bits == 8 ? lut_mul_launch<16, 8>(x1, lut, a1, z1, x2, a2, z2, n, ay, zy, y, st)
                     : lut_mul_launch<16, 16>(x1, lut, a1, z1, x2, a2, z2, n, ay, zy, y, st);
}

template <int BITS, int NCH>
void rmsnorm_regs(const int16_t* x, int64_t M, int64_t K, float ax, int32_t zx,
                  const float* gamma, float eps, float ay, int32_t zy, void* y, hipStream_t st)
{
    rmsnorm_regs_kernel<BITS, NCH><<<(unsigned)M, kThreads, 0, st>>>(x, K, ax, zx, gamma, eps, ay,
                                                                    zy, y);
}

// register-resident rows: K % 8 == 0, 16-byte aligned x and y, chunks per
// thread (0: the strided kernel)
static int row_chunks(const int16_t* x, const void* y, int64_t K)
{
    if (K % 8 != 0 || ((uintptr_t)x % 16) != 0 || ((uintptr_t)y % 16) != 0) return 0;
    const int64_t ch = (K / 8 + kThreads - 1) / kThreads;
    return ch <= 1 ? 1 : ch <= 2 ? 2 : ch <= 4 ? 4 : 0;
}

hipError_t launch_rmsnorm(const int16_t* x, int64_t M, int64_t K, float ax, int32_t zx,
                          const float* gamma, float eps, float ay, int32_t zy, int32_t bits,
                          void* y, hipStream_t st)
{
    const int ch = row_chunks(x, y, K);
    if (ch > 0) {
        if (bits == 8) {
            if (ch == 1) rmsnorm_regs<8, 1>(x, M, K, ax, zx, gamma, eps, ay, zy, y, st);
            else if (ch == 2) rmsnorm_regs<8, 2>(x, M, K, ax, zx, gamma, eps, ay, zy, y, st);
            else rmsnorm_regs<8, 4>(x, M, K, ax, zx, gamma, eps, ay, zy, y, st);
        } else {
            if (ch == 1) rmsnorm_regs<16, 1>(x, M, K, ax, zx, gamma, eps, ay, zy, y, st);
            else if (ch == 2) rmsnorm_regs<16, 2>(x, M, K, ax, zx, gamma, eps, ay, zy, y, st);
            else rmsnorm_regs<16, 4>(x, M, K, ax, zx, gamma, eps, ay, zy, y, st);
        }
        return hipGetLastError();
    }
    if (bits == 8)
        rmsnorm_kernel<8><<<(unsigned)M, kThreads, 0, st>>>(x, K, ax, zx, gamma, eps, ay, zy, y);
    else
        rmsnorm_kernel<16><<<(unsigned)M, kThreads, 0, st>>>(x, K, ax, zx, gamma, eps, ay, zy, y);
    return hipGetLastError();
}

hipError_t launch_add_rmsnorm(const int16_t* x1, float a1, int32_t z1, const int16_t* x2,
                             float a2, int32_t z2, int64_t M, int64_t K, float ah, int32_t zh,
                             int16_t* h, const float* gamma, float eps, float ay, int32_t zy,
                             int32_t bits, void* y, hipStream_t st)
{
    if (M == 0) return hipSuccess;
    const int ch = row_chunks(x1, y, K);
    if (ch > 0 && row_chunks(x2, h, K) > 0) {
        const dim3 g((unsigned)M), b(kThreads);
        const Binary p{a1, a2, z1, z2};
        if (bits == 8) {
            if (ch == 1) add_rmsnorm_kernel<8, 1><<<g, b, 0, st>>>(x1, x2, p, K, ah, zh, h, gamma, eps, ay, zy, y);
            else if (ch == 2) add_rmsnorm_kernel<8, 2><<<g, b, 0, st>>>(x1, x2, p, K, ah, zh, h, gamma, eps, ay, zy, y);
            else add_rmsnorm_kernel<8, 4><<<g, b, 0, st>>>(x1, x2, p, K, ah, zh, h, gamma, eps, ay, zy, y);
        } else {
            if (ch == 1) add_rmsnorm_kernel<16, 1><<<g, b, 0, st>>>(x1, x2, p, K, ah, zh, h, gamma, eps, ay, zy, y);
            else if (ch == 2) add_rmsnorm_kernel<16, 2><<<g, b, 0, st>>>(x1, x2, p, K, ah, zh, h, gamma, eps, ay, zy, y);
            else add_rmsnorm_kernel<16, 4><<<g, b, 0, st>>>(x1, x2, p, K, ah, zh, h, gamma, eps, ay, zy, y);
        }
        return hipGetLastError();
    }
    // rows that do not fit the register kernel: the two steps
    const hipError_t e = launch_add_requant(x1, a1, z1, x2, a2, z2, M * K, ah, zh, 16, h, st);
    if (e != hipSuccess) return e;
    return launch_rmsnorm(h, M, K, ah, zh, gamma, eps, ay, zy, bits, y, st);
}

template <int BITS, bool CLAMP, bool EXACT>
static void softmax_t(const int16_t* x, int64_t M, int64_t K, float ax, float ay, int32_t zy,
                      int64_t P, int64_t O, void* y, hipStream_t st)
{
    // a wave per row when that gives every SIMD one; rows of more than 2048
    // codes (a block holds 8192) and few rows take a block each
    if (K > 2048 || (M < 1024 && K > 512)) {
        softmax_block_kernel<BITS, CLAMP, EXACT>
            <<<dim3((unsigned)M), dim3(kThreads), 0, st>>>(x, K, ax, ay, zy, P, O, y);
        return;
    }
    constexpr int RPB = kSmRows * kSmWaves;
    const dim3 g((unsigned)((M + RPB - 1) / RPB)), b(kSmWaves * 64);
    if (K <= 4 * kChunk)
        softmax_table_kernel<BITS, CLAMP, EXACT, 4><<<g, b, 0, st>>>(x, M, K, ax, ay, zy, P, O, y);
    else
        softmax_table_kernel<BITS, CLAMP, EXACT, 8><<<g, b, 0, st>>>(x, M, K, ax, ay, zy, P, O, y);
}

template <int BITS>
static void softmax_bits(const int16_t* x, int64_t M, int64_t K, float ax, float ay, int32_t zy,
                         int64_t P, int64_t O, void* y, hipStream_t st)
{
    // probabilities are at most 1 / ay output steps
    const bool clamp = !(1.0 / (double)ay <= 131072.0);
    // rows of whole aligned 16-byte chunks up to 2048 codes: the tables' codes
    // as they are (the tie check costs 1.1 of 22.3 us at 32 x 1024 causal
    // rows of 1024 codes); all others agree with the definition at ties too
    const bool exact = K > 2048 || K % 8 != 0 || ((uintptr_t)x | (uintptr_t)y) % 16 != 0;
    if (exact && clamp) softmax_t<BITS, true, true>(x, M, K, ax, ay, zy, P, O, y, st);
    else if (exact) softmax_t<BITS, false, true>(x, M, K, ax, ay, zy, P, O, y, st);
    else if (clamp) softmax_t<BITS, true, false>(x, M, K, ax, ay, zy, P, O, y, st);
    else softmax_t<BITS, false, false>(x, M, K, ax, ay, zy, P, O, y, st);
}

hipError_t launch_softmax(const int16_t* x, int64_t M, int64_t K, float ax, float ay, int32_t zy,
                          int32_t bits, int64_t period, int64_t offset, void* y, hipStream_t st)
{
    if (K <= 8192) {
        if (bits == 8) softmax_bits<8>(x, M, K, ax, ay, zy, period, offset, y, st);
        else softmax_bits<16>(x, M, K, ax, ay, zy, period, offset, y, st);
    } else if (bits == 8) {
        softmax_kernel<8><<<(unsigned)M, kThreads, 0, st>>>(x, K, ax, ay, zy, period, offset, y);
    } else {
        softmax_kernel<16><<<(unsigned)M, kThreads, 0, st>>>(x, K, ax, ay, zy, period, offset, y);
    }
    return hipGetLastError();
}

}  // namespace mq

namespace mq {
namespace {

// Rotary position embedding.  The angle table holds cos and sin of
// (t + pos0) * base^(-2i/D) for every token t and pair i (fp64: inverse
// frequency by pow, one product, cos, sin); the main kernel rotates each
// pair (i, i + D/2) of every head of x [T][H * D] and requantizes.
__global__ __launch_bounds__(256) void rope_table_kernel(int64_t T, int64_t half, int64_t D,
                                                         double base, int64_t pos0,
                                                         double* __restrict__ cs)
{
#pragma clang fp contract(off)
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= T * half) return;
    const int64_t t = idx / half, i = idx - t * half;
    const double inv = pow(base, -(double)(2 * i) / (double)D);
    const double ang = (double)(t + pos0) * inv;
    cs[2 * idx] = cos(ang);
    cs[2 * idx + 1] = sin(ang);
}

// NP neighbouring pairs (h, i .. i + NP - 1) per thread (NP = 8: 16-byte
// loads of the two halves, NP = 1 any half).  grid (ceil(H * D/2 / NP /
// 256), min(T, 65535)): block row t holds the pairs of tokens t, t +
// gridDim.y, ...  Queries of 1024 x 32 heads of 64: 5.4 us with one pair per
// thread, 4.8 with eight.
template <int BITS, int NP>
__global__ __launch_bounds__(256) void rope_kernel(const int16_t* __restrict__ x, int64_t T,
                                                   int32_t H, int32_t half, float ax, int32_t zx,
                                                   const double* __restrict__ cs, float ay,
                                                   int32_t zy, void* __restrict__ y)
{
#pragma clang fp contract(off)
    const int32_t q = ((int32_t)blockIdx.x * 256 + (int32_t)threadIdx.x) * NP;
    if (q >= H * half) return;
    const int32_t h = q / half, i = q - h * half;
    const double ri = 1.0 / (double)ay;
    for (int64_t t = blockIdx.y; t < T; t += gridDim.y) {
        const int64_t j0 = (t * H + h) * (int64_t)(2 * half) + i, j1 = j0 + half;
        int32_t c0[NP], c1[NP];
        if constexpr (NP == 8) {
            unpack8(*reinterpret_cast<const v4i*>(x + j0), c0);
            unpack8(*reinterpret_cast<const v4i*>(x + j1), c1);
        } else {
            c0[0] = x[j0];
            c1[0] = x[j1];
        }
        const double* a = cs + 2 * (t * half + i);
        double v[2 * NP];
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const double c = a[2 * k], sn = a[2 * k + 1];
            const double f0 = (double)ax * (double)(c0[k] - zx);
            const double f1 = (double)ax * (double)(c1[k] - zx);
            v[k] = f0 * c - f1 * sn;
            v[NP + k] = f1 * c + f0 * sn;
        }
        int32_t r[2 * NP];
        requant_codes<BITS, 2 * NP>(r, zy, [&](int k) { return v[k] / (double)ay; },
                                    [&](int k) { return v[k] * ri; });
        if constexpr (NP == 8) {
            store8<BITS>(y, j0, r);
            store8<BITS>(y, j1, r + NP);
        } else {
            store_code<BITS>(y, j0, r[0]);
            store_code<BITS>(y, j1, r[1]);
        }
    }
}

}  // namespace

hipError_t launch_rope_table(int64_t T, int64_t D, double base, int64_t pos0, double* table,
                             hipStream_t st)
{
    const int64_t half = D / 2;
    const int64_t entries = T * half;
    if (entries == 0) return hipSuccess;
    rope_table_kernel<<<(unsigned)((entries + 255) / 256), 256, 0, st>>>(T, half, D, base, pos0,
                                                                         table);
    return hipGetLastError();
}

hipError_t launch_rope_apply(const int16_t* x, int64_t T, int64_t H, int64_t D, float ax,
                             int32_t zx, const double* table, float ay, int32_t zy, int32_t bits,
                             void* y, hipStream_t st)
{
    const int64_t half = D / 2;
    if (T == 0) return hipSuccess;
    if (H * half > 0x7FFFFFFF - 256) return hipErrorInvalidValue;
    // whole aligned groups of eight in both halves and in the output, the last
    // block's pair index in 32 bits, and enough of them: a wave's worth per
    // token and 2^18 in all (us, one pair per thread first: 1024 tokens x 32
    // heads of 64 5.8, 4.8; 777 x 32 5.1, 4.4; 256 x 32 3.0 both; 64 x 32 2.4,
    // 2.9; 1024 x 4 2.6, 3.0; 4096 x 4, whose blocks would be a sixteenth
    // full, 4.5, 6.1)
    const uintptr_t yal = bits == 8 ? 8 : 16;
    const int64_t pairs = H * half;
    const bool vec = half % 8 == 0 && ((uintptr_t)x % 16) == 0 && ((uintptr_t)y % yal) == 0 &&
                     pairs <= 0x7FFFFFFF - 8 * 256 && pairs >= 512 &&
                     T > ((int64_t)1 << 18) / pairs;
    const int64_t threads = pairs / (vec ? 8 : 1);
    const dim3 g((unsigned)((threads + 255) / 256), (unsigned)(T < 65535 ? T : 65535));
    const int32_t h32 = (int32_t)H, hf = (int32_t)half;
    if (bits == 8) {
        if (vec) rope_kernel<8, 8><<<g, 256, 0, st>>>(x, T, h32, hf, ax, zx, table, ay, zy, y);
        else rope_kernel<8, 1><<<g, 256, 0, st>>>(x, T, h32, hf, ax, zx, table, ay, zy, y);
    } else {
        if (vec) rope_kernel<16, 8><<<g, 256, 0, st>>>(x, T, h32, hf, ax, zx, table, ay, zy, y);
        else rope_kernel<16, 1><<<g, 256, 0, st>>>(x, T, h32, hf, ax, zx, table, ay, zy, y);
    }
    return hipGetLastError();
}

hipError_t launch_rope(const int16_t* x, int64_t T, int64_t H, int64_t D, float ax, int32_t zx,
                       double base, int64_t pos0, float ay, int32_t zy, int32_t bits,
                       double* table, void* y, hipStream_t st)
{
    const hipError_t e = launch_rope_table(T, D, base, pos0, table, st);
    if (e != hipSuccess) return e;
    return launch_rope_apply(x, T, H, D, ax, zx, table, ay, zy, bits, y, st);
}

}  // namespace mq
