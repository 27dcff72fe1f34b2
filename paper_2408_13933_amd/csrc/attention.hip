// Helpers of the batched attention matmuls (Section 5.6: in the W8A16
// setting the self-attention products multiply 16-bit by 8-bit activation
// codes): the zero-point sums of both operands and the transpose of the
// value codes into the [group][head dim][token] operand layout.
#include <type_traits>

#include "mq_internal.h"
#include "requant.h"

namespace mq {
namespace {

// ---------------------------------------------------------------------------
// The attention products (one launch, no workspace).  With the 16-bit code
// split as a = 256 h + l + 128 (split_a16),
//   sum_k (a - a_zp)(b - b_zp)
//     = 256 (sum h b - b_zp sum h) + (sum l b - b_zp sum l)
//       + (128 - a_zp)(sum b - K b_zp),
// so each zero-point term is a sum over operands the product reads anyway:
// the row terms are one more MFMA per plane against a constant operand
// -b_zp (the result lands in the accumulator layout, the same in every
// column), the column sums four dot products per fragment.  A separate pass
// for these sums read the 64 MB of probabilities of a 1024-token prompt a
// second time (16.4 us of its 28 us P V).
//
// Operands go from memory to the registers of whole rows' lanes (eight or
// four neighbouring lanes per 128 or 64 bytes of a row) and change to the
// MFMA's layout, where neighbouring lanes hold different rows, through a few
// KB of LDS that belong to the wave alone, so without a barrier.  Loading
// the MFMA's layout straight from memory runs at 37 GB/s per CU instead of
// 90 (every group of four lanes spans four rows): P V over 1024 causal
// tokens took 16.3 us that way.  Which key a column of the product stands
// for is free: column c of fragment i is key CF c + i, so a lane ends with
// CF neighbouring keys of each of its token rows and every row is stored in
// whole 16 CF-code runs without a trip through LDS.  Neither side needs any
// alignment: rows of odd length (a 777-token prompt) take the same loads and
// stores, and only the last step of a row that is no multiple of 64 reads
// through a window that ends at the row's end.
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v4i_u __attribute__((ext_vector_type(4), aligned(1)));

struct AttnArgs {
    const int16_t* a;
    const int8_t* b;
    void* y;
    int64_t lda, a_hs, ldb, b_hs, ldy, y_hs;
    int32_t M, N, K;
    int32_t hpg;       // heads per group
    int32_t flat;      // rows of all heads of a group share tiles (fewer rows than a tile)
    int32_t rtiles;    // row tiles per head (per group when flat)
    int32_t heads;     // heads (groups when flat): row tile sets
    int32_t strips;    // work items along N: column tiles (deep), strips of them (wide)
    int32_t strip_tiles;  // column tiles per wave of a strip (wide)
    int32_t a_zp, b_zp;
    int32_t neg_bzp;   // the constant operand, four bytes: -b_zp, or 64 when
    int32_t neg_shift; // -b_zp = 128, its sums then shifted left by one
    EpiInt epi;
    int32_t epi_lo;    // lower pre-shift bound: -epi.bnd, or INT32_MIN without a pre-shift
    int32_t zp_add;    // output zero-point, 0 when it is in epi.rnd
    int64_t out_causal, in_causal;
};

__device__ __forceinline__ v4i load16(const int8_t* p)
{
    return *reinterpret_cast<const v4i_u*>(p);
}

// Bytes [off, off + 16) of a row of `bytes` bytes, zeros past its end; no
// byte outside the row is read.
__device__ __forceinline__ v4i load16_tail(const int8_t* row, int32_t off, int32_t bytes)
{
    uint64_t lo = 0, hi = 0;
    if (off < bytes) {
        int32_t s = 0;  // bits to drop, 0 .. 120
        if (bytes >= 16) {
            const int32_t start = off < bytes - 16 ? off : bytes - 16;
            const v4i v = load16(row + start);
            lo = (uint64_t)(uint32_t)v[0] | (uint64_t)(uint32_t)v[1] << 32;
            hi = (uint64_t)(uint32_t)v[2] | (uint64_t)(uint32_t)v[3] << 32;
            s = 8 * (off - start);
        } else {
#pragma unroll 1
            for (int32_t i = bytes - 1; i >= off; --i) {
                hi = hi << 8 | lo >> 56;
                lo = lo << 8 | (uint8_t)row[i];
            }
        }
        if (s >= 64) {
            lo = hi;
            hi = 0;
            s -= 64;
        }
        if (s > 0) {
            lo = lo >> s | hi << (64 - s);
            hi >>= s;
        }
    }
    return v4i{(int)(uint32_t)lo, (int)(uint32_t)(lo >> 32), (int)(uint32_t)hi,
               (int)(uint32_t)(hi >> 32)};
}

// The constant operand over the k of one 16-code chunk that exist (n >= 16:
// all of them).
__device__ inline v4i const16(int32_t c4, int32_t n)
{
    v4i r;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const int32_t left = n - 4 * d;
        r[d] = left >= 4 ? c4 : left <= 0 ? 0 : c4 & ((1 << (8 * left)) - 1);
    }
    return r;
}

__device__ __forceinline__ int32_t sum16(const v4i& b, int32_t s)
{
#pragma unroll
    for (int d = 0; d < 4; ++d) s = __builtin_amdgcn_sdot4(b[d], 0x01010101, s, false);
    return s;
}

__device__ __forceinline__ v4i mfma(const v4i& a, const v4i& b, const v4i& c)
{
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}

// One row tile: up to TR rows of one head, or (flat) of a group's heads.
template <int TR>
struct RowTile {
    int32_t h, m0;    // head and first token (flat: first head of the group, first flat row)
    int32_t rows;     // rows that exist from m0 on
    int32_t m_last;   // largest token index in the tile
    __device__ RowTile(const AttnArgs& p, int32_t g, int32_t hg, int32_t rt)
    {
        m0 = rt * TR;
        if (p.flat) {
            h = g * p.hpg;
            rows = p.hpg * p.M - m0;
            m_last = p.M - 1;
        } else {
            h = hg;
            rows = p.M - m0;
            m_last = m0 + TR - 1 < p.M ? m0 + TR - 1 : p.M - 1;
        }
    }
    // head and token of row t of the tile
    __device__ void at(const AttnArgs& p, int32_t t, int32_t& hh, int32_t& m) const
    {
        hh = h;
        m = m0 + t;
        if (p.flat) {
            const int32_t q = (int32_t)((uint32_t)m / (uint32_t)p.M);
            hh += q;
            m -= q * p.M;
        }
    }
};

// Requantized code of the saturated sum c, before its clamp.  SIMPLE: no
// pre-shift and the zero-point in the rounding constant (both the same for
// every output of the call).
template <bool SIMPLE>
__device__ __forceinline__ int32_t attn_round(int32_t c, const AttnArgs& p)
{
    if constexpr (!SIMPLE) {
        c = max(min(c, p.epi.bnd), p.epi_lo);
        c = (int32_t)((uint32_t)c << p.epi.pre);
    }
    int32_t v = (__mulhi(c, p.epi.m0) + p.epi.rnd) >> p.epi.shr;
    if constexpr (!SIMPLE) v += p.zp_add;
    return v;
}

// Clamp the CF neighbouring codes v and store them (n >= CF: whole, else
// the first n) at any alignment.
template <int OBITS, int CF>
__device__ __forceinline__ void store_codes(int8_t* dst, const int32_t* v, int32_t n)
{
    constexpr int32_t qmin = -(1 << (OBITS - 1)), qmax = (1 << (OBITS - 1)) - 1;
    using T = std::conditional_t<OBITS == 8, int8_t, int16_t>;
    if (n >= CF) {
        struct __attribute__((packed)) Run {
            T v[CF];
        } run;
#pragma unroll
        for (int f = 0; f < CF; f += 2) {
            if constexpr (OBITS == 16) {
                const auto k = __builtin_amdgcn_cvt_pk_i16(v[f], v[f + 1]);  // saturating
                run.v[f] = k[0];
                run.v[f + 1] = k[1];
            } else {
                run.v[f] = (T)max(min(v[f], qmax), qmin);
                run.v[f + 1] = (T)max(min(v[f + 1], qmax), qmin);
            }
        }
        *reinterpret_cast<Run*>(dst) = run;
    } else {
#pragma unroll
        for (int f = 0; f < CF; ++f)
            if (f < n) reinterpret_cast<T*>(dst)[f] = (T)max(min(v[f], qmax), qmin);
    }
}

// Store register r of row fragment j (token rows 16 j + 4 kg + r of the
// tile): sum(i) is the saturated sum of column fragment i.  n0: the tile's
// first column.
template <int OBITS, int RF, int CF, bool SIMPLE, class Sum>
__device__ __forceinline__ void store_row(const AttnArgs& p, const RowTile<16 * RF>& rt, int j,
                                          int r, int32_t n0, Sum sum)
{
    constexpr int OB = OBITS / 8;
    const int lane = threadIdx.x & 63, c16 = lane & 15, kg = lane >> 4;
    int8_t* const y = static_cast<int8_t*>(p.y);
    int32_t v[CF];
#pragma unroll
    for (int i = 0; i < CF; ++i) v[i] = attn_round<SIMPLE>(sum(i), p);
    if (!p.flat && rt.rows >= 16 * RF && n0 + 16 * CF <= p.N) {
        // a whole tile: uniform row addresses, one lane offset
        int8_t* const row = y + (rt.h * p.y_hs + (rt.m0 + 16 * j + r) * p.ldy + n0) * OB;
        store_codes<OBITS, CF>(row + (uint32_t)(4 * kg * (int32_t)p.ldy + CF * c16) * OB, v, CF);
        return;
    }
    // (the row index is hidden from the compiler: it would keep the addresses
    // of all the rows in registers across a caller's loop)
    int32_t t = 16 * j + 4 * kg + r;
    asm volatile("" : "+v"(t));
    int32_t h, m;
    rt.at(p, t, h, m);
    const int32_t n = n0 + CF * c16;
    if (t < rt.rows && n < p.N)
        store_codes<OBITS, CF>(y + (h * p.y_hs + m * p.ldy + n) * OB, v, p.N - n);
}

// A wave's staging area: byte offset of 16-byte chunk c of row r.  A: rows of
// 128 bytes, two to a 256-byte bank row; B: rows of 64 bytes, four to a bank
// row.  Sixteen consecutive rows of one chunk (a fragment read) and the
// neighbouring rows of a load (B: rows 16 apart) lie on distinct banks.
__device__ __forceinline__ int a_off(int r, int c)
{
    return (r >> 1) * 256 + ((r & 1) * 8 + (c ^ ((r >> 1) & 7))) * 16;
}
__device__ __forceinline__ int b_off(int r, int c)
{
    return (r >> 2) * 256 + (((r + (r >> 4)) & 3) * 4 + (c ^ ((r >> 2) & 3))) * 16;
}

// The A and B operands of 64-deep steps for a 16 RF x 16 CF tile: the lane's
// row pointers and loads, and the change of layout.
template <int RF, int CF>
struct Operands {
    static constexpr int A_BYTES = 16 * RF * 128, B_BYTES = 16 * CF * 64;
    const int8_t* pa[2 * RF];  // token row 8 i + lane / 8
    const int8_t* pb[CF];      // key row 16 i + lane / 4
    v4i ax[2 * RF], bx[CF];

    __device__ __forceinline__ void rows_a(const AttnArgs& p, const RowTile<16 * RF>& rt)
    {
#pragma unroll
        for (int i = 0; i < 2 * RF; ++i) {
            const int32_t t = 8 * i + (threadIdx.x & 63) / 8;
            int32_t h, m;
            rt.at(p, t < rt.rows ? t : rt.rows - 1, h, m);
            pa[i] = reinterpret_cast<const int8_t*>(p.a + h * p.a_hs + m * p.lda);
        }
    }
    __device__ __forceinline__ void rows_b(const AttnArgs& p, int32_t g, int32_t n0)
    {
#pragma unroll
        for (int i = 0; i < CF; ++i) {
            const int32_t n = n0 + 16 * i + (threadIdx.x & 63) / 4;
            pb[i] = p.b + g * p.b_hs + (n < p.N ? n : p.N - 1) * p.ldb;
        }
    }
    // step s of rows of K codes; WHOLE: every chunk lies inside the row
    template <bool WHOLE>
    __device__ __forceinline__ void load_a(int32_t s, int32_t K)
    {
        const int32_t off = 128 * s + 16 * (threadIdx.x & 7);
#pragma unroll
        for (int i = 0; i < 2 * RF; ++i)
            ax[i] = WHOLE ? load16(pa[i] + off) : load16_tail(pa[i], off, 2 * K);
    }
    template <bool WHOLE>
    __device__ __forceinline__ void load_b(int32_t s, int32_t K)
    {
        const int32_t off = 64 * s + 16 * (threadIdx.x & 3);
#pragma unroll
        for (int i = 0; i < CF; ++i)
            bx[i] = WHOLE ? load16(pb[i] + off) : load16_tail(pb[i], off, K);
    }
    __device__ __forceinline__ void stage_a(int8_t* lds) const
    {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int i = 0; i < 2 * RF; ++i)
            *reinterpret_cast<v4i*>(lds + a_off(8 * i + lane / 8, lane & 7)) = ax[i];
    }
    __device__ __forceinline__ void stage_b(int8_t* lds) const
    {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int i = 0; i < CF; ++i) {
            const int n = 16 * i + lane / 4;  // key n is column n / CF of fragment n % CF
            *reinterpret_cast<v4i*>(lds + b_off(n % CF * 16 + n / CF, lane & 3)) = bx[i];
        }
    }
    __device__ __forceinline__ static void frag_a(const int8_t* lds, int j, v4i& h, v4i& l)
    {
        const int lane = threadIdx.x & 63, r = 16 * j + (lane & 15), c = 2 * (lane >> 4);
        split_a16(*reinterpret_cast<const v4i*>(lds + a_off(r, c)),
                  *reinterpret_cast<const v4i*>(lds + a_off(r, c + 1)), h, l);
    }
    __device__ __forceinline__ static v4i frag_b(const int8_t* lds, int i)
    {
        const int lane = threadIdx.x & 63;
        return *reinterpret_cast<const v4i*>(lds + b_off(16 * i + (lane & 15), lane >> 4));
    }
    // between one lane's store and another's load of the wave's own LDS:
    // the wave's LDS operations complete in order, so only the compiler has
    // to keep theirs
    __device__ __forceinline__ static void turn()
    {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();
    }
};

// K <= 64 KSS <= 128 (queries times keys: K is the head dimension).  Bound by
// its outputs: no loop over K, so the cost is one round trip for the
// operands, the requant of the codes and their stores.  A wave keeps its
// 16 RF token rows in registers and walks over 16 CF-key tiles, the next
// tile's keys on their way while it requantizes this one's sums; the four
// waves of a block take neighbouring tiles in turn (a causal row's last
// tiles spread over them), row tiles from the last (longest) one down.  No
// barrier.  |c| <= 128 * 65535 * 255 < 2^31: the saturation is the identity
// and all terms are formed in int32, wrapping to the exact value.
// WHOLE: K = 64 KSS, no window at a row's end.
// Measured, 32 heads over 4 groups, K = 64, int16 out, against the LDS tile
// with its pass for the sums (or, unaligned or with one query, the generic
// kernel): 1024 causal tokens 26.4 -> 15.4 us, 777 tokens 3704 -> 12.2 us,
// one query over 1531 keys 17.0 -> 3.8 us.
template <int OBITS, int RF, int CF, int KSS, bool WHOLE>
__global__ __launch_bounds__(256, KSS == 1 ? 3 : 1) void attn_wide_kernel(AttnArgs p)
{
    const int lane = threadIdx.x & 63, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // work items: strip of column tiles fastest, then head (group), then
    // row tile
    uint32_t it = blockIdx.x / (uint32_t)p.strips;
    const int32_t strip = (int32_t)(blockIdx.x - it * (uint32_t)p.strips);
    const uint32_t rq = it / (uint32_t)p.heads;
    const int32_t hg = (int32_t)(it - rq * (uint32_t)p.heads);
    const int32_t g = p.flat ? hg : hg / p.hpg;
    const RowTile<16 * RF> rt(p, g, hg, p.rtiles - 1 - (int32_t)rq);
    // columns this tile's rows need
    int32_t n_end = p.N;
    if (p.out_causal >= 0 && rt.m_last + p.out_causal + 1 < n_end)
        n_end = (int32_t)(rt.m_last + p.out_causal) + 1;
    constexpr int32_t TN = 16 * CF;
    const int32_t strip0 = strip * p.strip_tiles * 4 * TN;
    int32_t n0 = strip0 + wave * TN;
    if (n0 >= n_end) return;
    const int32_t s_end = strip0 + p.strip_tiles * 4 * TN;
    if (s_end < n_end) n_end = s_end;

    using Op = Operands<RF, CF>;
    constexpr int STAGE = KSS * (Op::A_BYTES > Op::B_BYTES ? Op::A_BYTES : Op::B_BYTES);
    __shared__ __align__(256) int8_t lds[4 * STAGE];
    int8_t* const mine = lds + wave * STAGE;
    Op op[KSS];
    v4i ah[RF][KSS], al[RF][KSS];
    auto load_b = [&](int32_t nt) {
        op[0].rows_b(p, g, nt);
#pragma unroll
        for (int q = 0; q < KSS; ++q) {
            if (q)
#pragma unroll
                for (int i = 0; i < CF; ++i) op[q].pb[i] = op[0].pb[i];
            op[q].template load_b<WHOLE>(q, p.K);
        }
    };
    op[0].rows_a(p, rt);
#pragma unroll
    for (int q = 0; q < KSS; ++q) {
        if (q)
#pragma unroll
            for (int i = 0; i < 2 * RF; ++i) op[q].pa[i] = op[0].pa[i];
        op[q].template load_a<WHOLE>(q, p.K);
    }
    load_b(n0);
#pragma unroll
    for (int q = 0; q < KSS; ++q) op[q].stage_a(mine + q * Op::A_BYTES);
    Op::turn();
#pragma unroll
    for (int q = 0; q < KSS; ++q)
#pragma unroll
        for (int j = 0; j < RF; ++j) Op::frag_a(mine + q * Op::A_BYTES, j, ah[j][q], al[j][q]);
    Op::turn();
    // the row terms, where the low plane's sums start
    v4i row[RF];
#pragma unroll
    for (int j = 0; j < RF; ++j) {
        row[j] = v4i{0, 0, 0, 0};
        v4i rh = {0, 0, 0, 0};
#pragma unroll
        for (int q = 0; q < KSS; ++q) {
            const v4i c = const16(p.neg_bzp, p.K - (64 * q + 16 * kg));
            rh = mfma(ah[j][q], c, rh);
            row[j] = mfma(al[j][q], c, row[j]);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
            row[j][r] = (int32_t)((((uint32_t)rh[r] << 8) + (uint32_t)row[j][r]) << p.neg_shift);
    }
    const bool simple = p.epi.pre == 0 && p.zp_add == 0;
    for (; n0 < n_end; n0 += 4 * TN) {
#pragma unroll
        for (int q = 0; q < KSS; ++q) op[q].stage_b(mine + q * Op::B_BYTES);
        Op::turn();
        if (n0 + 4 * TN < n_end) load_b(n0 + 4 * TN);
        v4i acch[RF][CF], accl[RF][CF];
        uint32_t coff[CF];
#pragma unroll
        for (int i = 0; i < CF; ++i) {
            int32_t cs = 0;
#pragma unroll
            for (int q = 0; q < KSS; ++q) {
                const v4i b = Op::frag_b(mine + q * Op::B_BYTES, i);
#pragma unroll
                for (int j = 0; j < RF; ++j) {
                    acch[j][i] = mfma(ah[j][q], b, q ? acch[j][i] : v4i{0, 0, 0, 0});
                    accl[j][i] = mfma(al[j][q], b, q ? accl[j][i] : row[j]);
                }
                cs = sum16(b, cs);
            }
            cs += __shfl_xor(cs, 16);
            cs += __shfl_xor(cs, 32);
            coff[i] = (uint32_t)(128 - p.a_zp) * (uint32_t)(cs - p.K * p.b_zp);
        }
        Op::turn();
        auto store = [&](auto form) {
#pragma unroll
            for (int j = 0; j < RF; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    store_row<OBITS, RF, CF, decltype(form)::value>(p, rt, j, r, n0, [&](int i) {
                        return (int32_t)(((uint32_t)acch[j][i][r] << 8) +
                                         (uint32_t)accl[j][i][r] + coff[i]);
                    });
        };
        if (simple) store(std::true_type{});
        else store(std::false_type{});
    }
}

// Any K (probabilities times values: K is the number of keys, N the head
// dimension).  Bound by the stream of A: W waves share a 16 RF x 16 CF tile
// and take its 64-deep steps in turn, so that a tile's whole row range is in
// flight, and meet in LDS, wave w finishing register w of every fragment.
// Each plane's partial sums, its row term included, stay in int32 (128 * 255
// * K < 2^31) and meet in int64 before the saturation.  With causal A a tile
// stops at its last row's boundary, the tiles with the longest rows first.
// Measured, 32 heads over 4 groups, N = 64, int8 out, against the same: 1024
// causal tokens 28.1 -> 15.0 us, 777 tokens 1595 -> 12.7 us, one query over
// 1531 keys 153 -> 5.8 us.
template <int OBITS, int RF, int CF, int W>
__global__ __launch_bounds__(W * 64) void attn_deep_kernel(AttnArgs p)
{
    static_assert(W >= 4, "a wave per accumulator register");
    // a wave's own part stays in its registers (W = 4)
    constexpr int SLOTS = W == 4 ? 3 : 4;
    typedef int vc __attribute__((ext_vector_type(CF)));
    extern __shared__ __align__(16) int8_t smem[];
    vc* part = reinterpret_cast<vc*>(smem);                                 // [W][SLOTS][RF][2][64]
    int32_t* csum = reinterpret_cast<int32_t*>(part + W * SLOTS * RF * 2 * 64);  // [W][CF][16]
    const int lane = threadIdx.x & 63, c16 = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // work items: column tile fastest, then head (group), then row tile
    uint32_t it = blockIdx.x / (uint32_t)p.strips;
    const int32_t nt = (int32_t)(blockIdx.x - it * (uint32_t)p.strips);
    const uint32_t rq = it / (uint32_t)p.heads;
    const int32_t hg = (int32_t)(it - rq * (uint32_t)p.heads);
    const int32_t g = p.flat ? hg : hg / p.hpg;
    const RowTile<16 * RF> rt(p, g, hg, p.rtiles - 1 - (int32_t)rq);
    const int32_t n0 = nt * 16 * CF;
    if (p.out_causal >= 0 && n0 > rt.m_last + p.out_causal) return;  // block-uniform
    int32_t K = p.K;
    if (p.in_causal >= 0) {
        // A holds its zero-point past the boundary, which contributes nothing
        const int64_t need = (rt.m_last + p.in_causal) / 64 * 64 + 64;
        if (need < K) K = (int32_t)need;
    }

    using Op = Operands<RF, CF>;
    Op op;
    op.rows_a(p, rt);
    op.rows_b(p, g, n0);
    int8_t* const mine = smem + wave * (Op::A_BYTES + Op::B_BYTES);  // staging, before the sums
    auto load = [&](int32_t s) {
        if (64 * s + 64 <= p.K) {
            op.template load_a<true>(s, p.K);
            op.template load_b<true>(s, p.K);
        } else {
            op.template load_a<false>(s, p.K);
            op.template load_b<false>(s, p.K);
        }
    };
    v4i acch[RF][CF + 1], accl[RF][CF + 1];  // the last: the row terms
#pragma unroll
    for (int j = 0; j < RF; ++j)
#pragma unroll
        for (int i = 0; i <= CF; ++i) acch[j][i] = accl[j][i] = v4i{0, 0, 0, 0};
    int32_t cs[CF] = {};
    const int32_t steps = (K + 63) / 64;
    if (wave < steps) load(wave);
    for (int32_t s = wave; s < steps; s += W) {
        op.stage_a(mine);
        op.stage_b(mine + Op::A_BYTES);
        Op::turn();
        if (s + W < steps) load(s + W);
        v4i b[CF];
#pragma unroll
        for (int i = 0; i < CF; ++i) {
            b[i] = Op::frag_b(mine + Op::A_BYTES, i);
            cs[i] = sum16(b[i], cs[i]);
        }
        const v4i c = const16(p.neg_bzp, p.K - (64 * s + 16 * kg));
#pragma unroll
        for (int j = 0; j < RF; ++j) {
            v4i ah, al;
            Op::frag_a(mine, j, ah, al);
#pragma unroll
            for (int i = 0; i < CF; ++i) {
                acch[j][i] = mfma(ah, b[i], acch[j][i]);
                accl[j][i] = mfma(al, b[i], accl[j][i]);
            }
            acch[j][CF] = mfma(ah, c, acch[j][CF]);
            accl[j][CF] = mfma(al, c, accl[j][CF]);
        }
        Op::turn();
    }
    __syncthreads();  // the sums take the place of the staging areas
#pragma unroll
    for (int i = 0; i < CF; ++i) {
        cs[i] += __shfl_xor(cs[i], 16);
        cs[i] += __shfl_xor(cs[i], 32);
        if (kg == 0) csum[(wave * CF + i) * 16 + c16] = cs[i];
    }
    auto slot = [&](int w, int r, int j, int pl) -> vc& {
        const int sl = W == 4 ? (r - w + 3) & 3 : r;
        return part[((w * SLOTS + sl) * RF + j) * 2 * 64 + pl * 64 + lane];
    };
    // register r of each column fragment of row fragment j, its row term added
    auto regs = [&](const v4i* acc, int r) {
        vc v;
#pragma unroll
        for (int i = 0; i < CF; ++i)
            v[i] = acc[i][r] + (int32_t)((uint32_t)acc[CF][r] << p.neg_shift);
        return v;
    };
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if (W == 4 && r == wave) continue;
#pragma unroll
        for (int j = 0; j < RF; ++j) {
            slot(wave, r, j, 0) = regs(acch[j], r);
            slot(wave, r, j, 1) = regs(accl[j], r);
        }
    }
    __syncthreads();
    auto finish = [&](auto rv) {
        constexpr int r = decltype(rv)::value;
        int64_t coff[CF];
#pragma unroll
        for (int i = 0; i < CF; ++i) {
            int32_t t = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) t += csum[(w * CF + i) * 16 + c16];
            coff[i] = (int64_t)(128 - p.a_zp) * ((int64_t)t - (int64_t)K * p.b_zp);
        }
#pragma unroll
        for (int j = 0; j < RF; ++j) {
            vc vh, vl;
            if constexpr (W == 4) {
                vh = regs(acch[j], r);
                vl = regs(accl[j], r);
            } else {
                vh = slot(0, r, j, 0);
                vl = slot(0, r, j, 1);
            }
#pragma unroll
            for (int w = W == 4 ? 0 : 1; w < W; ++w) {
                if (W == 4 && w == r) continue;
                vh += slot(w, r, j, 0);
                vl += slot(w, r, j, 1);
            }
            store_row<OBITS, RF, CF, false>(p, rt, j, r, n0, [&](int i) {
                return sat32(((int64_t)vh[i] << 8) + vl[i] + coff[i]);
            });
        }
    };
    if (wave == 0) finish(std::integral_constant<int, 0>{});
    else if (wave == 1) finish(std::integral_constant<int, 1>{});
    else if (wave == 2) finish(std::integral_constant<int, 2>{});
    else if (wave == 3) finish(std::integral_constant<int, 3>{});
}

// Partial sum, for lane li of the LPR lanes that share one row, of the K
// codes starting at x: 16-byte loads when `vec` (x 16-byte aligned), else
// element loads; the LPR partial sums are reduced by the caller.
template <class T>
__device__ inline int64_t row_sum_part(const T* x, int64_t K, int li, int lpr, bool vec)
{
    constexpr int PER = 16 / sizeof(T);  // codes per 16-byte load
    int64_t s = 0;
    int64_t k0 = 0;
    if (vec) {
        const int64_t step = (int64_t)lpr * PER;
        const int64_t full = K / step * step;
        for (int64_t k = (int64_t)li * PER; k < full; k += step) {
            const int4 v = *reinterpret_cast<const int4*>(x + k);
            const T* e = reinterpret_cast<const T*>(&v);
            int32_t t = 0;
#pragma unroll
            for (int i = 0; i < PER; ++i) t += e[i];
            s += t;
        }
        k0 = full;
    }
    for (int64_t k = k0 + li; k < K; k += lpr) s += x[k];
    return s;
}

// LPR lanes (a power of two, at most 64) per row: rows [0, rows_a) are rows
// of A (int16; none when B's zero-point is 0), rows [rows_a, rows_a +
// rows_b) rows of B (int8), each B row once per block of tile_m rows of A
// ([group][m block][n]).  A rows give the term of B's zero-point,
// -b_zp * sum_k (A[k] - a_zp) (int64, exact); B rows give sum_k B[k] over
// k < K, or, with causal activations (in_causal >= 0), over the K range the
// tiled kernel reads for that m block: up to the tile_k stage holding the
// block's last row's boundary.
__global__ __launch_bounds__(256) void attn_sums_kernel(const int16_t* a, int64_t lda, int64_t a_bs,
                                                        int64_t rows_a, int64_t M,
                                                        const int8_t* b, int64_t ldb, int64_t b_bs,
                                                        int64_t rows_b, int64_t N, int64_t K,
                                                        int32_t a_zp, int32_t b_zp, float b_scale,
                                                        int64_t* row_off, int32_t* colsum,
                                                        float* scale_out, bool vec_a, bool vec_b,
                                                        int64_t n_mb, int64_t in_causal,
                                                        int64_t tile_m, int64_t tile_k, int lpr)
{
    const int li = threadIdx.x & (lpr - 1);
    if (blockIdx.x == 0 && threadIdx.x == 0) *scale_out = b_scale;
    const int64_t row = (int64_t)blockIdx.x * (256 / lpr) + threadIdx.x / lpr;
    // rows past the end still take part in the reduction (all lanes of a
    // group reach the shuffles) with a zero sum
    const bool live = row < rows_a + rows_b;
    // row indices below 2^32 (the host's check) divide in 32 bits
    int64_t s = 0;
    if (live && row < rows_a) {
        const uint32_t h = (uint32_t)row / (uint32_t)M, m = (uint32_t)row - h * (uint32_t)M;
        s = row_sum_part(a + (int64_t)h * a_bs + (int64_t)m * lda, K, li, lpr, vec_a);
    } else if (live) {
        const uint32_t r = (uint32_t)(row - rows_a);  // (g * n_mb + mb) * N + n
        const uint32_t q = r / (uint32_t)N, n = r - q * (uint32_t)N;
        const uint32_t g = q / (uint32_t)n_mb, mb = q - g * (uint32_t)n_mb;
        int64_t len = K;
        if (in_causal >= 0) {
            const int64_t m_end = (mb + 1) * tile_m < M ? (mb + 1) * tile_m : M;
            const int64_t need = (m_end + in_causal + tile_k - 1) / tile_k * tile_k;
            if (need < len) len = need;
        }
        s = row_sum_part(b + g * b_bs + n * ldb, len, li, lpr, vec_b);
    }
    for (int o = lpr / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (li != 0 || !live) return;
    if (row < rows_a)
        row_off[row] = -(int64_t)b_zp * (s - K * (int64_t)a_zp);
    else
        colsum[row - rows_a] = (int32_t)s;  // |s| <= 128 K <= 2^23
}

// y[c][r] = x[r][c] through a 64 x 64 LDS tile: one 16-byte load and one
// 16-byte store per thread at any alignment (edges of the matrix by
// element).  Bound by latency at the sizes of a value matrix: 1024 x 256
// took 5.0 us with sixteen one-byte loads and stores per thread one after
// the other, 2.4 us this way.
__global__ __launch_bounds__(256) void transpose_i8_kernel(const int8_t* x, int64_t rows,
                                                           int64_t cols, int64_t ldx, int8_t* y)
{
    __shared__ __align__(4) int8_t t[64][68];  // t[c][r], read by dwords
    const int64_t r0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
    const int row = threadIdx.x >> 2, q = (threadIdx.x & 3) * 16;
    {
        const int64_t r = r0 + row, c = c0 + q;
        v4i v = {0, 0, 0, 0};
        if (r < rows && c < cols) {
            // the row from one tile before this one on: 32-bit offsets
            const int64_t w0 = c0 >= 64 ? c0 - 64 : 0;
            const int64_t left = cols - w0 < 192 ? cols - w0 : 192;
            v = load16_tail(x + r * ldx + w0, (int32_t)(c - w0), (int32_t)left);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) t[q + i][row] = (int8_t)(v[i / 4] >> (8 * (i % 4)));
    }
    __syncthreads();
    const int64_t c = c0 + row, r = r0 + q;
    if (c >= cols || r >= rows) return;
    int8_t* dst = y + c * rows + r;
    v4i v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = *reinterpret_cast<const int*>(&t[row][q + 4 * i]);
    if (r + 16 <= rows) {
        *reinterpret_cast<v4i_u*>(dst) = v;
    } else {
        for (int i = 0; i < 16 && r + i < rows; ++i) dst[i] = t[row][q + i];
    }
}

template <int OBITS, int RF, int CF, int W>
hipError_t launch_deep(const AttnArgs& p, uint32_t blocks, hipStream_t s)
{
    using Op = Operands<RF, CF>;
    constexpr int sums = W * ((W == 4 ? 3 : 4) * RF * 2 * 64 * CF * 4 + CF * 16 * 4);
    constexpr int staging = W * (Op::A_BYTES + Op::B_BYTES);
    constexpr int lds = sums > staging ? sums : staging;
    static const hipError_t attr =
        hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_deep_kernel<OBITS, RF, CF, W>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return attr;
    attn_deep_kernel<OBITS, RF, CF, W><<<dim3(blocks), dim3(W * 64), lds, s>>>(p);
    return hipGetLastError();
}

template <int OBITS>
hipError_t launch_attn_t(AttnArgs& p, int32_t H, int32_t G, hipStream_t s)
{
    // 32 x 64 tiles when there are enough of them, else 16 x 32 ones (one
    // query per head: the keys are all there is to spread).  Fewer rows than
    // a tile: the heads of a group, which share the 8-bit operand, fill it
    // together.
    const bool wide = p.K <= kAttnWideK;
    auto row_tiles = [&](int32_t tr) {
        p.flat = p.M < tr;
        p.heads = p.flat ? G : H;
        p.rtiles = ((p.flat ? p.M * p.hpg : p.M) + tr - 1) / tr;
        return (int64_t)p.rtiles * p.heads;
    };
    int64_t tiles = row_tiles(32) * ((p.N + 63) / 64);
    const bool few = tiles < (wide ? 2048 : 256);
    if (few) tiles = row_tiles(16) * ((p.N + 31) / 32);
    const int64_t rblocks = (int64_t)p.rtiles * p.heads, cols = tiles / rblocks;
    p.strip_tiles = wide && !few ? 4 : 1;
    p.strips = (int32_t)(wide ? (cols + 4 * p.strip_tiles - 1) / (4 * p.strip_tiles) : cols);
    const int64_t blocks = rblocks * p.strips;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), wg(256);
    if (!wide) {
        // four waves per tile; with few tiles sixteen, so that a long row is
        // still read at once
        return few ? launch_deep<OBITS, 1, 2, 16>(p, (uint32_t)blocks, s)
                   : launch_deep<OBITS, 2, 4, 4>(p, (uint32_t)blocks, s);
    }
    if (!few) {
        if (p.K == 64) attn_wide_kernel<OBITS, 2, 4, 1, true><<<grid, wg, 0, s>>>(p);
        else if (p.K == 128) attn_wide_kernel<OBITS, 2, 4, 2, true><<<grid, wg, 0, s>>>(p);
        else attn_wide_kernel<OBITS, 2, 4, 2, false><<<grid, wg, 0, s>>>(p);
    } else {
        if (p.K == 64) attn_wide_kernel<OBITS, 1, 2, 1, true><<<grid, wg, 0, s>>>(p);
        else if (p.K == 128) attn_wide_kernel<OBITS, 1, 2, 2, true><<<grid, wg, 0, s>>>(p);
        else attn_wide_kernel<OBITS, 1, 2, 2, false><<<grid, wg, 0, s>>>(p);
    }
    return hipGetLastError();
}

}  // namespace

// The lane's offset inside a whole tile, 12 rows and less than 64 columns in
// units of up to two bytes, fits 32 bits (store_row).
constexpr int64_t kMaxLdy = (0x7FFFFFFF - 64) / 12;

bool attn_direct_supported(int64_t M, int64_t N, int64_t ldy, int32_t H, int32_t G)
{
    // 32-bit row and column indices, the lane's offset inside a tile, the
    // flat rows of a group and the work items in range
    const int64_t rb = ((M + 15) / 16) * H;
    return M <= 0x3FFFFFFF / (H / G) && N <= 0x3FFFFFFF && ldy <= kMaxLdy &&
           rb <= 0x7FFFFFFF / ((N + 31) / 32);
}

// Where the LDS tiles (qlinear_prefill.hip; with b_zp != 0 after a pass for the
// sums) are faster than the kernels here, for shapes and strides both take.
// Measured over 8 heads of one group and 32 of four, head dimensions 32 .. 256,
// 64 .. 4096 queries over 256 .. 4096 keys, causal and not (us, direct kernel
// first).
bool attn_tiles_better(int64_t M, int64_t N, int64_t K, int32_t H, int32_t b_zp,
                       int64_t out_causal, int64_t in_causal)
{
    if (M <= 16) return false;
    const int64_t cols = (N + 63) / 64, tiles = (M + 31) / 32 * cols * H;  // 32 x 64
    if (K <= kAttnWideK) {
        // Queries times keys.  A head dimension of one or two whole steps
        // walks the keys without a window at each load (full 1024^2, 32
        // heads of 64: 21 against 31; of 128: 28, 38), any other one pays
        // for the windows once the 32 x 64 tiles are in use and the rows are
        // long (of 80: 42, 37; 8 heads of 80 over 256 x 2048: 18.7, 12.5; up
        // to 64 queries or 512 keys even or ahead).
        if (K != 64 && K != 128) return M > 64 && N > 512 && tiles >= 2048;
        // two steps: a long causal triangle leaves the strips uneven (8
        // heads, 4096^2: 78 against 71; 32 heads, 2048^2: 70, 76)
        return K == 128 && out_causal >= 0 && out_causal < M && M > 2048;
    }
    // A product long in K and N, of many rows, reuses its operands more.
    if (N > 256) return true;
    // Probabilities times values: the kernel here reads the probabilities
    // once per 64 columns, the LDS tiles once per 128, after the pass for the
    // sums that reads them too.  Up to 64 columns and with that pass the
    // kernel here is ahead (full 1024^2, 32 heads of 64: 21 against 29);
    // without it (b_zp = 0) the tiles are from 1024 tiles on (21, 19), and
    // with three or more column tiles also with it (32 heads of 256, 1024^2:
    // 67, 43; 8 heads of 256, 512 x 2048, 512 tiles: 17.5, 24.5), with two
    // from 2048 (32 heads of 128, 1024^2: 36, 33; 8 heads, 2048^2: 30, 33).
    // A causal triangle halves what the kernel here reads.
    const bool triangle = in_causal >= 0 && in_causal < M;
    if (triangle)
        return b_zp == 0 ? cols >= 2 && tiles >= 1536 : cols >= 4 && tiles >= 2048;
    if (b_zp == 0 || cols >= 3) return tiles >= 1024 || (tiles >= 768 && K >= 2048);
    return cols == 2 && tiles >= 2048;
}

hipError_t launch_attn_direct(const int16_t* a, int64_t lda, int64_t a_hs, int32_t H,
                              const int8_t* b, int64_t ldb, int64_t b_hs, int32_t G, int64_t M,
                              int64_t N, int64_t K, float a_scale, int32_t a_zp, float b_scale,
                              int32_t b_zp, float out_scale, int32_t out_zp, int32_t out_bits,
                              void* y, int64_t ldy, int64_t y_hs, int64_t out_causal,
                              int64_t in_causal, hipStream_t s)
{
    AttnArgs p;
    p.a = a;
    p.b = b;
    p.y = y;
    p.lda = lda;
    p.a_hs = a_hs;
    p.ldb = ldb;
    p.b_hs = b_hs;
    p.ldy = ldy;
    p.y_hs = y_hs;
    p.M = (int32_t)M;
    p.N = (int32_t)N;
    p.K = (int32_t)K;
    p.hpg = H / G;
    p.a_zp = a_zp;
    p.b_zp = b_zp;
    p.neg_shift = b_zp == -128;
    p.neg_bzp = (int32_t)((uint32_t)(uint8_t)(p.neg_shift ? 64 : -b_zp) * 0x01010101u);
    p.epi = epi_int_params(derive_col_params_v(a_scale, b_scale, out_scale, false, 0.0f, 0, 0));
    p.epi_lo = p.epi.pre ? -p.epi.bnd : INT32_MIN;
    // out_zp * 2^shr joins the rounding constant when the sum stays at most
    // 2^30 (mul_hi plus it cannot overflow int32)
    const int64_t zabs = out_zp < 0 ? -(int64_t)out_zp : (int64_t)out_zp;
    p.zp_add = out_zp;
    if ((int64_t)p.epi.rnd + (zabs << p.epi.shr) <= ((int64_t)1 << 30)) {
        p.epi.rnd += out_zp * (1 << p.epi.shr);
        p.zp_add = 0;
    }
    p.out_causal = out_causal;
    p.in_causal = in_causal;
    return out_bits == 8 ? launch_attn_t<8>(p, H, G, s) : launch_attn_t<16>(p, H, G, s);
}

hipError_t launch_attn_sums(const int16_t* a, int64_t lda, int64_t a_bs, int32_t H, int64_t M,
                            const int8_t* b, int64_t ldb, int64_t b_bs, int32_t G, int64_t N,
                            int64_t K, int32_t a_zp, int32_t b_zp, float b_scale,
                            int64_t* row_off, int32_t* colsum, float* scale_out,
                            int64_t in_causal, int64_t tile_m, int64_t tile_k, hipStream_t s)
{
    // B's zero-point 0: the row terms vanish and A is not read
    const int64_t n_mb = in_causal >= 0 ? (M + tile_m - 1) / tile_m : 1;
    const int64_t rows_a = b_zp != 0 ? (int64_t)H * M : 0, rows_b = (int64_t)G * n_mb * N;
    // lanes per row: enough 16-byte loads of int16 codes to cover K once
    int lpr = 1;
    while (lpr < 64 && (int64_t)lpr * 8 < K) lpr *= 2;
    const int64_t rpb = 256 / lpr;
    const int64_t blocks = (rows_a + rows_b + rpb - 1) / rpb;
    if (blocks == 0) return hipSuccess;
    if (rows_a + rows_b >= ((int64_t)1 << 32) || M >= ((int64_t)1 << 32) ||
        N >= ((int64_t)1 << 32))
        return hipErrorInvalidValue;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    const bool vec_a = (uintptr_t)a % 16 == 0 && (lda * 2) % 16 == 0 && (a_bs * 2) % 16 == 0;
    const bool vec_b = (uintptr_t)b % 16 == 0 && ldb % 16 == 0 && b_bs % 16 == 0;
    attn_sums_kernel<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(
        a, lda, a_bs, rows_a, M, b, ldb, b_bs, rows_b, N, K, a_zp, b_zp, b_scale, row_off, colsum,
        scale_out, vec_a, vec_b, n_mb, in_causal, tile_m, tile_k, lpr);
    return hipGetLastError();
}

hipError_t launch_transpose_i8(const int8_t* x, int64_t rows, int64_t cols, int64_t ldx,
                               int8_t* y, hipStream_t s)
{
    if (rows == 0 || cols == 0) return hipSuccess;
    const int64_t gx = (cols + 63) / 64, gy = (rows + 63) / 64;
    if (gx > 0x7FFFFFFF || gy > 65535) return hipErrorInvalidValue;
    transpose_i8_kernel<<<dim3((unsigned)gx, (unsigned)gy), dim3(256), 0, s>>>(x, rows, cols, ldx,
                                                                              y);
    return hipGetLastError();
}

}  // namespace mq
