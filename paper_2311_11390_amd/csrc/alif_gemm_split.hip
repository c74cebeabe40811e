// FP32 GEMM on the bfloat16 matrix cores (gfx950): the float operands of the Eq. 3
// projections are cut into three bfloat16 pieces while they are staged,
//   v = h + m + l,  h = bf16(v), m = bf16(v - h), l = v - h - m (each rounded to nearest),
// which together hold all 24 bits of v (|m| <= 2^-8, |l| <= 2^-17 of v's binade), and the
// products of pieces are accumulated in FP32:
//   spikes x float   (uint8 and bfloat16 spikes are one piece): x h, x m, x l;
//   float x float    all but l l, which is below 2^-33 of a product. (Without m l and l m
//                    a single product was off by up to 2^-24 more than its rounding.)
// Products of bfloat16 are exact in FP32, and h h is accumulated apart from the rest: sums
// of 8-bit (16-bit) numbers are exact or nearly so, and the rest is 2^-7 of them and less.
// So the error against 64 bits is that of FP32 multiply-adds for sums of one or two terms and
// below it for longer ones (relative 2-norm, 32000 x 700 x 512, 2.5% active, a plain FP32 GEMM
// / this one: current 8.2e-8 / 2.5e-8, dW 1.48e-7 / 9.1e-8, dx 4.0e-7 / 1.27e-7).
//
// Why: v_mfma_f32_32x32x16_bf16 multiplies 16 times as fast as v_mfma_f32_16x16x4_f32,
// so three or eight of them still beat it. us, FP32 kernel -> this one (uint8 spikes): 32000 x
// 700 x 512 current 196 -> 91, dW 239 -> 91, dx 228 -> 192; 65536 x 512 x 512 289 -> 141, 310 ->
// 130, 301 -> 270; 64000 x 200 x 256 79 -> 50, 107 -> 51, 91 -> 82; 1200 x 64 x 64 15.3 -> 13.3,
// 37 -> 23, 15.6 -> 15.2. The matrix cores are busy 28% (current), 36% (dW) and 46% (dx) of that
// time; the conversions (5.5 vector instructions an element and plane triple) and the LDS round
// trip of the pieces take the rest. m l and l m cost dx 13-15% (65536 x 512 x 512 235 without).
//
// Range. A tile whose float operands hold an infinity or a magnitude from 2^60 up
// (where a piece could overflow apart from the others, or 0 x inf turn up between pieces)
// is done over by v_mfma_f32_16x16x4_f32 straight from memory at the end (65536 x 512 x 512 with
// one infinity in W: current 1.02 ms, dx 0.86; with it all past 2^60 dW 0.68 ms; scalar
// multiply-adds took 30, 14 and 34 ms); NaNs pass through the pieces.
// Magnitudes below 2^-110 lose the bits of l that fall under bfloat16's smallest
// subnormal.
//
// Tiling. 256 threads own 128 x 128 of C, each wave 64 x 64 as 2 x 2 accumulators of
// v_mfma_f32_32x32x16_bf16. K moves through two LDS buffers in stages of 32 (four
// planes) or 16 (six planes), 64 KiB and two workgroups a CU, 24 or 32 MFMAs a wave
// between barriers.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "../../include/blockalif.h"
#include "alif_common.h"
#include "alif_gemm.h"

namespace alif {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int ST = 128;        // tile rows and columns
constexpr int NT = 256;        // threads
constexpr float BIG = 1.152921504606847e18f;   // 2^60

template <int DT>
constexpr int planes() { return DT == 0 ? 3 : 1; }
template <int ADT, int BDT>
constexpr int stage_k() { return planes<ADT>() + planes<BDT>() > 4 ? 16 : 32; }
// LDS: arrays of 128 rows of 128 bytes, eight 16-byte chunks (8 k each) a row. Plane p
// of a buffer (A's planes, then B's) has BK / 8 neighbouring chunks of array
// p BK / 64; chunk x of row r sits at x ^ f(r). f takes the row's bits 1-3 to the
// position's three, so the 16 rows of a fragment read fall on the 16 chunk positions of a
// 256-byte line; their order (and bit 0, which a read does not need) is such that the 16
// lanes of an 8-byte store, BK / 4 groups of k of neighbouring rows (K-major) or of rows
// RR apart (R-major), fill 128 bytes. Two R-major operands with 32 k take another
// order than the rest (RM).
template <bool RM, int BK>
__device__ __forceinline__ int lds_swizzle(int row) {
    const int b0 = row & 1, b1 = row >> 1 & 1, b2 = row >> 2 & 1, b3 = row >> 3 & 1;
    return RM ? b2 << 2 | b1 << 1 | b3 : (BK == 32 ? (b1 ^ b0) << 2 | b2 << 1 | b3 : b1 << 2 | (b2 ^ b0) << 1 | b3);
}
template <bool RM, int BK>
__device__ __forceinline__ int lds_at(int plane, int row, int chunk) {
    constexpr int PPA = 64 / BK;   // planes an array
    const int x = (plane % PPA) * (BK / 8) + chunk;
    return plane / PPA * (ST * 64) + row * 64 + (x ^ lds_swizzle<RM, BK>(row)) * 8;
}
template <int BK>
constexpr int buf_elems(int planes) { return (planes * BK + 63) / 64 * (ST * 64); }

// two floats as three packed pairs of bfloat16
__device__ __forceinline__ void split2(float v0, float v1, uint32_t &h, uint32_t &m, uint32_t &l) {
    h = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)v0, (__bf16)v1});
    const float r0 = v0 - __uint_as_float(h << 16), r1 = v1 - __uint_as_float(h & 0xffff0000u);
    m = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)r0, (__bf16)r1});
    const float l0 = r0 - __uint_as_float(m << 16), l1 = r1 - __uint_as_float(m & 0xffff0000u);
    l = __builtin_amdgcn_perm(__float_as_uint(l1), __float_as_uint(l0), 0x07060302u);   // exact
}

// One operand's 128 x BK stage: what this thread loads and where it puts the pieces.
//   KM = 0: k contiguous ([row][k] in memory): BK / 4 threads read one row in runs of 4;
//   KM = 1: rows contiguous ([k][row]): a thread reads RR rows of 4 consecutive k and
//           transposes them in registers.
// Each stage has its own buffer descriptor, which ends where the valid data ends
// (every offset that can pass it is in the instruction's vector offset): rows past the
// valid ones read zeros (KM = 0) or data that reaches only parts of C never stored
// (KM = 1), k past the range is zeroed (KM = 0) or reads zeros (KM = 1).
template <int DT, bool KM, bool RM, int BK>
struct Side {
    static constexpr int NP = planes<DT>();
    static constexpr int ES = DT == 0 ? 4 : (DT == 1 ? 1 : 2);
    static constexpr int EPT = ST * BK / NT;         // elements a thread and stage
    static constexpr int RR = EPT / 4;               // KM: rows a thread
    static constexpr int KG = BK / 4;                // KM: groups of 4 k
    static constexpr int CPR = BK / 4;               // !KM: threads a row
    static constexpr int RPP = NT / CPR;             // !KM: rows a pass
    static constexpr int NL = KM ? 4 : ST / RPP;     // loads
    static constexpr int LB = (KM ? RR : 4) * ES;    // bytes a load
    static constexpr int LW = LB < 4 ? 1 : LB / 4;   // dwords a load
    static_assert(!KM || NT / KG * RR == ST, "row-contiguous threads");

    const char *base;
    uint32_t ext, step, voff0, vstep;
    int span, lk, at;   // k range, this thread's first k of a stage and its LDS element
    struct Regs {
        uint32_t w[NL][LW];
    };
    float big;      // largest magnitude this thread has staged (float, bfloat16)

    __device__ __forceinline__ void init(const void *ptr, long long ld, long long rows, long long row0, int kb, int ke,
                                         int tid) {
        const char *p = static_cast<const char *>(ptr);
        const long long vr = rows - row0;
        span = ke - kb;
        big = 0.0f;
        const int lrow = KM ? tid / KG * RR : tid / CPR;
        if constexpr (KM) {
            lk = tid % KG * 4;
            base = p + ((size_t)kb * ld + row0) * ES;
            ext = (uint32_t)(((size_t)(span - 1) * ld + vr) * ES);
            step = (uint32_t)((size_t)BK * ld * ES);
            voff0 = (uint32_t)(((size_t)lk * ld + lrow) * ES);
            vstep = (uint32_t)(ld * ES);
        } else {
            lk = tid % CPR * 4;
            const long long nr = vr < ST ? vr : ST;
            base = p + ((size_t)row0 * ld + kb) * ES;
            ext = (uint32_t)(((size_t)nr * ld - kb) * ES);
            step = (uint32_t)(BK * ES);
            voff0 = (uint32_t)(((size_t)lrow * ld + lk) * ES);
            vstep = (uint32_t)((size_t)RPP * ld * ES);
        }
        at = lds_at<RM, BK>(0, lrow, lk >> 3) + (lk & 7);
    }
    __device__ __forceinline__ void load(int s, Regs &g) const {
        const uint32_t o = (uint32_t)__builtin_amdgcn_readfirstlane(s) * step;
        const uint64_t bp = reinterpret_cast<uint64_t>(base + o);
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)bp);
        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(bp >> 32));
        const uint32_t n = __builtin_amdgcn_readfirstlane(s * BK < span && o < ext ? ext - o : 0u);
        const rsrc_t r = make_rsrc(reinterpret_cast<const void *>(((uint64_t)hi << 32) | lo), n);
#pragma unroll
        for (int i = 0; i < NL; i++) {
            const uint32_t off = voff0 + (uint32_t)i * vstep;
            if constexpr (LB == 16) {
                const auto x = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
#pragma unroll
                for (int e = 0; e < 4; e++) g.w[i][e] = x[e];
            } else if constexpr (LB == 8) {
                const auto x = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
                g.w[i][0] = x[0];
                g.w[i][1] = x[1];
            } else if constexpr (LB == 4) {
                g.w[i][0] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
            } else if constexpr (LB == 2) {
                g.w[i][0] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0);
            } else {
                g.w[i][0] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b8(r, off, 0, 0);
            }
        }
    }
    // element e of load i as float bits (float), or as a bfloat16 in the upper half
    static __device__ __forceinline__ uint32_t elem(const Regs &g, int i, int e) {
        if constexpr (DT == 0) return g.w[i][e];
        else if constexpr (DT == 1) return __float_as_uint((float)((g.w[i][0] >> (8 * e)) & 0xffu));
        else return (e & 1) ? g.w[i][e / 2] & 0xffff0000u : g.w[i][e / 2] << 16;
    }
    // 4 consecutive k of LDS row lrow + dr from lk on (dr a constant)
    __device__ __forceinline__ void put(__bf16 *buf, int p0, int dr, const uint32_t *v) {
        uint32_t q[NP][2];
#pragma unroll
        for (int e = 0; e < 4; e += 2) {
            if constexpr (DT != 1)
                big = fmaxf(fmaxf(big, fabsf(__uint_as_float(v[e]))), fabsf(__uint_as_float(v[e + 1])));
            if constexpr (NP == 3)
                split2(__uint_as_float(v[e]), __uint_as_float(v[e + 1]), q[0][e / 2], q[1][e / 2], q[2][e / 2]);
            else q[0][e / 2] = __builtin_amdgcn_perm(v[e + 1], v[e], 0x07060302u);   // exact
        }
        // lds_at(p0 + p, lrow + dr, lk / 8): lrow is a multiple of RR (KM) and dr below it, or dr
        // a multiple of 16, so dr and the plane only flip bits of the position in `at`
        constexpr int PPA = 64 / BK;
#pragma unroll
        for (int p = 0; p < NP; p++) {
            const int flip = ((p0 + p) % PPA * (BK / 8) ^ (KM ? lds_swizzle<RM, BK>(dr) : 0)) * 8;
            *reinterpret_cast<uint2 *>(buf + ((at ^ flip) + (p0 + p) / PPA * (ST * 64) + dr * 64)) = uint2{q[p][0], q[p][1]};
        }
    }
    __device__ __forceinline__ void store(const Regs &g, int s, __bf16 *buf, int p0) {
        asm volatile("" : "+v"(at));   // (keeps the addresses derived from it out of registers across stages)
        if constexpr (KM) {
#pragma unroll
            for (int rr = 0; rr < RR; rr++) {
                uint32_t v[4];
#pragma unroll
                for (int j = 0; j < 4; j++) v[j] = elem(g, j, rr);
                put(buf, p0, rr, v);
            }
        } else {
            const int left = span - s * BK - lk;   // valid k of this thread
            const bool tail = (s + 1) * BK > span;
#pragma unroll
            for (int i = 0; i < NL; i++) {
                uint32_t v[4];
#pragma unroll
                for (int e = 0; e < 4; e++) v[e] = elem(g, i, e);
                if (tail)
#pragma unroll
                    for (int e = 0; e < 4; e++) v[e] = e < left ? v[e] : 0u;
                put(buf, p0, i * RPP, v);
            }
        }
    }
};

__device__ __forceinline__ float elem_f32(const void *p, int dt, size_t i) {
    if (dt == 0) return static_cast<const float *>(p)[i];
    if (dt == 1) return (float)static_cast<const uint8_t *>(p)[i];
    return __uint_as_float((uint32_t) static_cast<const uint16_t *>(p)[i] << 16);
}

template <int ADT, bool AKM, int BDT, bool BKM>
__global__ __launch_bounds__(NT, 2) void k_gemm_split(GemmArgs g, int m_tiles, int n_tiles, int kps, int total) {
    if (gemm_gated_off(g.skip_cnt, g.skip_le)) return;
    constexpr int BK = stage_k<ADT, BDT>();
    constexpr int NA = planes<ADT>(), NB = planes<BDT>();
    constexpr bool RM = AKM && BKM && BK == 32;
    constexpr int BUF = buf_elems<BK>(NA + NB);
    extern __shared__ __align__(16) unsigned char lds[];
    __bf16 *L = reinterpret_cast<__bf16 *>(lds);   // two buffers of A's planes and B's

    const int work = xcd_remap(blockIdx.x, total);
    const int tiles = m_tiles * n_tiles;
    const int z = work / tiles, t = work % tiles;
    const long long m0 = (long long)(t / n_tiles) * ST;
    const int n0 = (t % n_tiles) * ST;
    const int kb = z * kps, ke = min(g.K, kb + kps);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int fr = lane & 31, fc = lane >> 5;

    Side<ADT, AKM, RM, BK> sa;
    Side<BDT, BKM, RM, BK> sb;
    sa.init(g.A, g.lda, g.M, m0, kb, ke, tid);
    sb.init(g.B, g.ldb, g.N, n0, kb, ke, tid);

    floatx16 hi[2][2], lo[2][2];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int r = 0; r < 16; r++) hi[i][j][r] = lo[i][j][r] = 0.0f;

    bf16x8 fa[NA][2], fb[NB][2];
    auto frags = [&](const __bf16 *l, int ks) __attribute__((always_inline)) {
        const int c = ks * 2 + fc;
#pragma unroll
        for (int i = 0; i < 2; i++) {
#pragma unroll
            for (int p = 0; p < NA; p++)
                fa[p][i] = *reinterpret_cast<const bf16x8 *>(l + lds_at<RM, BK>(p, wm * 64 + i * 32 + fr, c));
#pragma unroll
            for (int p = 0; p < NB; p++)
                fb[p][i] = *reinterpret_cast<const bf16x8 *>(l + lds_at<RM, BK>(NA + p, wn * 64 + i * 32 + fr, c));
        }
    };
    auto mul = [&](int p, int q) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int j = 0; j < 2; j++) {
                floatx16 &c = p + q == 0 ? hi[i][j] : lo[i][j];
                c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[p][i], fb[q][j], c, 0, 0, 0);
            }
    };
    // the products of one k16 step, the smallest first, in two halves (three products: one)
    auto mul_half = [&](int half) __attribute__((always_inline)) {
        int n = 0;
#pragma unroll
        for (int o = 3; o >= 0; o--)
#pragma unroll
            for (int p = 0; p < NA; p++)
#pragma unroll
                for (int q = 0; q < NB; q++) {
                    if (p + q != o) continue;
                    if (n++ < 4 ? half == 0 : half == 1) mul(p, q);
                }
    };

    // Stage s + 1 is converted and stored to the other LDS buffer between the MFMAs of
    // stage s, and its registers reloaded at once with stage s + 3: two stages in flight.
    const int nk = (ke - kb + BK - 1) / BK;
    typename Side<ADT, AKM, RM, BK>::Regs ra[2];
    typename Side<BDT, BKM, RM, BK>::Regs rb[2];
    sa.load(0, ra[0]);
    sb.load(0, rb[0]);
    sa.load(1, ra[1]);
    sb.load(1, rb[1]);
    sa.store(ra[0], 0, L, 0);
    sb.store(rb[0], 0, L, NA);
    sa.load(2, ra[0]);
    sb.load(2, rb[0]);
    __syncthreads();
    auto stage = [&](int s, auto par) __attribute__((always_inline)) {
        constexpr int P = decltype(par)::value;   // s mod 2
        const __bf16 *cur = L + P * BUF;
        __bf16 *nxt = L + (1 - P) * BUF;
        frags(cur, 0);
        __builtin_amdgcn_sched_barrier(0);
        mul_half(0);
        sa.store(ra[1 - P], s + 1, nxt, 0);
        sa.load(s + 3, ra[1 - P]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (BK == 32) frags(cur, 1);
        mul_half(BK == 32 ? 0 : 1);
        sb.store(rb[1 - P], s + 1, nxt, NA);
        sb.load(s + 3, rb[1 - P]);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
    };
    int s = 0;
    for (; s + 2 <= nk; s += 2) {
        stage(s, std::integral_constant<int, 0>{});
        stage(s + 1, std::integral_constant<int, 1>{});
    }
    if (s < nk) stage(s, std::integral_constant<int, 0>{});

    const bool split = total > tiles;
    float *out = split ? g.C_part + (size_t)z * g.M * g.N : g.C;
    const long long ldc = split ? g.N : g.ldc;
    if (__syncthreads_or(fmaxf(sa.big, sb.big) >= BIG)) {   // see "Range" above
        constexpr int U = 4;   // steps of 4 k in flight
        const int r = lane & 15, q = lane >> 4;
        floatx4 acc[4][4];
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
            for (int j = 0; j < 4; j++) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        size_t ra4[4], rb4[4];   // (rows past the end repeat the last one; their results are dropped)
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const long long m = m0 + wm * 64 + 16 * i + r;
            const int n = min(n0 + wn * 64 + 16 * i + r, g.N - 1);
            ra4[i] = (size_t)(m < g.M ? m : g.M - 1) * (AKM ? 1 : g.lda);
            rb4[i] = (size_t)n * (BKM ? 1 : g.ldb);
        }
        for (int k0 = kb + q; k0 - q < ke; k0 += 4 * U) {   // (uniform)
            float xa[U][4], xb[U][4];
#pragma unroll
            for (int u = 0; u < U; u++) {
                const bool in = k0 + 4 * u < ke;
                const size_t k = min(k0 + 4 * u, ke - 1);
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const float a = elem_f32(g.A, ADT, ra4[i] + k * (AKM ? g.lda : 1));
                    const float b = elem_f32(g.B, BDT, rb4[i] + k * (BKM ? g.ldb : 1));
                    xa[u][i] = in ? a : 0.0f;
                    xb[u][i] = in ? b : 0.0f;
                }
            }
#pragma unroll
            for (int u = 0; u < U; u++)
#pragma unroll
                for (int i = 0; i < 4; i++)
#pragma unroll
                    for (int j = 0; j < 4; j++)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[u][i], xb[u][j], acc[i][j], 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const int n = n0 + wn * 64 + 16 * j + r;
            const float bias = (g.bias && !split && n < g.N) ? g.bias[n] : 0.0f;
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const long long m = m0 + wm * 64 + 16 * i + 4 * q + e;
                    if (m < g.M && n < g.N) out[m * ldc + n] = acc[i][j][e] + bias;
                }
        }
        return;
    }
    // lane l holds column l % 32 and rows 8 (r / 4) + 4 (l / 32) + r % 4 of an accumulator
#pragma unroll
    for (int j = 0; j < 2; j++) {
        const int n = n0 + wn * 64 + j * 32 + fr;
        const float bias = (g.bias && !split && n < g.N) ? g.bias[n] : 0.0f;
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const long long m = m0 + wm * 64 + i * 32 + 8 * (r >> 2) + 4 * fc + (r & 3);
                if (m < g.M && n < g.N) out[m * ldc + n] = (hi[i][j][r] + lo[i][j][r]) + bias;
            }
    }
}

template <int ADT, bool AKM, int BDT, bool BKM>
void go(const GemmArgs &g, int mt, int nt, int kps, int total, hipStream_t st) {
    constexpr int BK = stage_k<ADT, BDT>();
    constexpr size_t sm = (size_t)2 * buf_elems<BK>(planes<ADT>() + planes<BDT>()) * 2;
    hipLaunchKernelGGL((k_gemm_split<ADT, AKM, BDT, BKM>), dim3((unsigned)total), dim3(NT), sm, st, g, mt, nt, kps,
                       total);
}

int es_of(int dt) { return dt == 0 ? 4 : (dt == 1 ? 1 : 2); }

}  // namespace

bool gemm_split_ok(const GemmArgs &g) {
    const bool fwd = g.a_kc && g.b_kc && g.b_dt == 0;
    const bool dx = g.a_kc && g.a_dt == 0 && !g.b_kc && g.b_dt == 0;
    const bool dw = !g.a_kc && g.a_dt == 0 && !g.b_kc;
    if (!(fwd || dx || dw) || g.K <= 0 || g.M <= 0 || g.N <= 0) return false;
    // the vector loads: bases and rows on 16 bytes of float, 4 elements otherwise
    if ((reinterpret_cast<uintptr_t>(g.A) & 15) || (reinterpret_cast<uintptr_t>(g.B) & 15)) return false;
    if (g.lda % 4 != 0 || g.ldb % 4 != 0) return false;
    if (!g.a_kc && (g.M % 4 != 0 || g.lda < g.M)) return false;
    if (!g.b_kc && (g.N % 4 != 0 || g.ldb < g.N)) return false;
    if (g.a_kc && g.lda < g.K) return false;
    if (g.b_kc && g.ldb < g.K) return false;
    if (g.splits > 1 && (g.a_kc || g.b_kc)) return false;
    const size_t kps = (size_t)(g.K + (g.splits > 1 ? g.splits : 1) - 1) / (g.splits > 1 ? g.splits : 1) + 64;
    const size_t lim = (size_t)1 << 31;
    const size_t ea = (g.a_kc ? (size_t)ST * g.lda : kps * g.lda) * es_of(g.a_dt);
    const size_t eb = (g.b_kc ? (size_t)ST * g.ldb : kps * g.ldb) * es_of(g.b_dt);
    return ea < lim && eb < lim;
}

hipError_t gemm_split_launch(const GemmArgs &g, hipStream_t st, int *splits_out) {
    const int bk = (g.a_dt == 0 && g.b_dt == 0) ? 16 : 32;
    const long long mt = (g.M + ST - 1) / ST;
    const int nt = (g.N + ST - 1) / ST;
    const int s = g.splits < 1 ? 1 : g.splits;
    const int kps = ((g.K + s - 1) / s + bk - 1) / bk * bk;
    const int splits = (g.K + kps - 1) / kps;
    const long long total = mt * nt * splits;
    if (total > 0x7fffffffLL) return hipErrorInvalidValue;
    const int m = (int)mt, tt = (int)total;
    *splits_out = splits;
    if (g.a_kc && g.b_kc) {
        if (g.a_dt == 0) go<0, false, 0, false>(g, m, nt, kps, tt, st);
        else if (g.a_dt == 1) go<1, false, 0, false>(g, m, nt, kps, tt, st);
        else go<2, false, 0, false>(g, m, nt, kps, tt, st);
    } else if (g.a_kc) {
        go<0, false, 0, true>(g, m, nt, kps, tt, st);
    } else {
        if (g.b_dt == 0) go<0, true, 0, true>(g, m, nt, kps, tt, st);
        else if (g.b_dt == 1) go<0, true, 1, true>(g, m, nt, kps, tt, st);
        else go<0, true, 2, true>(g, m, nt, kps, tt, st);
    }
    return hipGetLastError();
}

}  // namespace alif
