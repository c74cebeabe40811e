// Forward without traces where the card is not full (T_R 2-32): the recurrence on one wave per
// 64 neurons, its loads and stores on others.
//
// What bounds it: the chain. A row's T / T_R blocks follow each other, and one wave issues an
// instruction about every five cycles, so a block costs what its wave issues. The block
// kernel's one wave at T_R 2-4 issues 95 a block, two thirds of them addresses, loads, stores
// and a table read; its two to four waves at T_R 5-32 meet at one or two barriers a block.
// Here
//   wave 1 loads the input FC_P groups of FC_G blocks ahead and leaves the drive
//          (1 - beta)(I + b) in LDS,
//   wave 0 runs the blocks of a group from LDS, all segments of a block, state in registers
//          (FP64 carries), and leaves each block's carry-in and spike step in LDS,
//   wave 2 writes the spikes of the group before, wave 3 its carries (if they are kept),
// with one barrier a group. The arithmetic is the block kernel's (alif_blocks_impl.h),
// operation by operation and segment by segment, so spikes and carries are the same bits.
// us a block, block kernel / this one (1 x 100 x 8000): T_R 2 0.20 / 0.082, 4 0.31 / 0.152,
// 5 0.45 / 0.18, 8 0.49 / 0.23, 10 0.42 / 0.27, 16 0.46 / 0.36, 20 0.51 / 0.41, 28 0.64 / 0.53,
// 32 0.66 / 0.59; above, eight waves on a block are faster than one.
#include <type_traits>

#include "alif_common.h"
#include "alif_kernels.h"

namespace alif {
namespace {

constexpr int FC_P = 3;   // groups of input in registers

template <int TR>
__global__ __launch_bounds__(256) void k_fwd_chain(FwdArgs a) {
    constexpr BlockConfig cfg = block_config(TR);
    constexpr int L = cfg.len, SEG = (TR + L - 1) / L;   // segments with a step in them
    constexpr int FC_G = TR <= 3 ? 16 : TR <= 4 ? 8 : TR <= 8 ? 4 : 2;  // blocks a group (one barrier each)
    constexpr bool TAB = TR > 4;                         // powers of p in LDS
    __shared__ float in[2][FC_G][TR][64];
    __shared__ float2 out[2][FC_G][64];   // carry-in v, a
    __shared__ uint8_t ots[2][FC_G][64];  // spike step (0: none)
    __shared__ double ptab[TAB ? 64 * TR : 1];
    const int lane = threadIdx.x & 63, role = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int work = xcd_remap(blockIdx.x, gridDim.x);
    const int b = work / a.n_groups, g = work - b * a.n_groups;
    const int N = a.N, T = a.T, NB = a.NB;
    const int n = g * 64 + lane, nc = min(n, N - 1);
    const bool valid = n < N;
    const int groups = (NB + FC_G - 1) / FC_G;
    const int iters = (groups + 1 + FC_P - 1) / FC_P * FC_P;   // barriers of every wave

    const size_t TN = (size_t)T * N;
    const size_t bsi = a.bs_i ? a.bs_i : TN, bss = a.bs_s ? a.bs_s : TN;
    // carry-in of every block, then the final carry (a sub-range's place: see FwdArgs)
    const size_t CN = (size_t)((a.ck_nb ? a.ck_nb : NB) + 1) * N, CE = (size_t)(NB + 1) * N;
    const size_t CO = b * CN + (size_t)a.ck_off * N;
    const bool ck = a.ck.v != nullptr;
    const double lb = -a.dt / (double)a.tau_m[nc], lp = -a.dt / (double)a.tau_a[nc];
    if constexpr (TAB)   // (each lane's neuron is its own in every wave)
        for (int k = role; k < TR; k += blockDim.x >> 6) ptab[lane * TR + k] = exp(lp * (double)k);

    // Rows go into the scalar offset, which the buffer's range check leaves out: they are
    // kept in range here, and lanes past N are out of range by their own offset.
    if (role == 1) {
        const rsrc_t rI = make_rsrc(a.I + b * bsi, (uint32_t)(TN * 4));
        const float bias = a.bias_k ? a.bias_k[nc] : 0.0f;
        const float omb = (float)(-expm1(lb)), ob = (float)(-expm1(lb) * (double)bias);
        const uint32_t n4 = (uint32_t)nc * 4u;
        float x[FC_P][FC_G * TR];
        constexpr int ROWS = FC_G * TR;
        const uint32_t step = (uint32_t)N * 4u;
        // (a group past the last whole one: rows clamped, and no input past the end)
        auto load = [&](float (&d)[ROWS], int q) __attribute__((always_inline)) {
            const int t0 = q * ROWS;
            if (t0 + ROWS <= T) {   // uniform
                uint32_t row = (uint32_t)t0 * step;
#pragma unroll
                for (int i = 0; i < ROWS; i++, row += step)
                    d[i] = __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rI, n4, row, 0));
            } else {
#pragma unroll
                for (int i = 0; i < ROWS; i++)
                    d[i] = __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b32(
                        rI, n4, (uint32_t)min(t0 + i, T - 1) * step, 0));
            }
        };
        auto put = [&](const float (&d)[ROWS], int q) __attribute__((always_inline)) {
            float (&o)[FC_G][TR][64] = in[q & 1];
            const int left = T - q * ROWS;
            if (left >= ROWS) {
#pragma unroll
                for (int i = 0; i < ROWS; i++) o[i / TR][i % TR][lane] = fmaf(omb, d[i], ob);
            } else {
#pragma unroll
                for (int i = 0; i < ROWS; i++) o[i / TR][i % TR][lane] = fmaf(omb, i < left ? d[i] : 0.0f, ob);
            }
        };
#pragma unroll
        for (int p = 0; p < FC_P; p++) load(x[p], p);
        put(x[0], 0);
        load(x[0], FC_P);
        __syncthreads();
        for (int it = 0; it < iters; it += FC_P) {
#pragma unroll
            for (int p = 0; p < FC_P; p++) {
                const int q = it + p + 1;   // (past the last group: not used)
                put(x[(p + 1) % FC_P], q);
                load(x[(p + 1) % FC_P], q + FC_P);
                __syncthreads();
            }
        }
    } else if (role == 2) {
        const int sdt = a.spike_dtype;
        const uint32_t SB = sdt == 0 ? 1u : (sdt == 1 ? 2u : 4u), step = (uint32_t)N * SB;
        const rsrc_t rS = make_rsrc((const char *)a.spikes + b * bss * SB, (uint32_t)(TN * SB));
        const uint32_t ns = valid ? (uint32_t)n * SB : ALIF_OOB;
        uint32_t row = 0;   // the group's first
        __syncthreads();
        for (int it = 0; it < iters; it++) {
            if (it > 0 && it <= groups) {
                int ts[FC_G];
#pragma unroll
                for (int i = 0; i < FC_G; i++) ts[i] = ots[(it - 1) & 1][i][lane];
                const int left = T - (it - 1) * FC_G * TR;   // rows
                auto rows = [&](auto put) __attribute__((always_inline)) {
                    if (left >= FC_G * TR) {
#pragma unroll
                        for (int i = 0; i < FC_G * TR; i++) put(row + i * step, ts[i / TR] == i % TR + 1);
                    } else {
#pragma unroll
                        for (int i = 0; i < FC_G * TR; i++)
                            if (i < left) put(row + i * step, ts[i / TR] == i % TR + 1);
                    }
                };
                if (sdt == 0)
                    rows([&](uint32_t r, bool s) { __builtin_amdgcn_raw_buffer_store_b8((uint8_t)s, rS, ns, r, 0); });
                else if (sdt == 1)
                    rows([&](uint32_t r, bool s) {
                        __builtin_amdgcn_raw_buffer_store_b16(s ? (uint16_t)0x3F80 : (uint16_t)0, rS, ns, r, 0);
                    });
                else
                    rows([&](uint32_t r, bool s) {
                        __builtin_amdgcn_raw_buffer_store_b32(s ? 0x3F800000u : 0u, rS, ns, r, 0);
                    });
                row += FC_G * TR * step;
            }
            __syncthreads();
        }
    } else if (role == 3) {
        const rsrc_t rCv = make_rsrc(a.ck.v + CO, (uint32_t)(CE * 4)), rCa = make_rsrc(a.ck.a + CO, (uint32_t)(CE * 4));
        const rsrc_t rCt = make_rsrc(a.ck.ts + CO, (uint32_t)CE);
        const uint32_t n4 = valid ? (uint32_t)n * 4u : ALIF_OOB, n1 = valid ? (uint32_t)n : ALIF_OOB;
        uint32_t e = 0;   // row of the group's first carry
        auto put = [&](uint32_t e, float2 r, uint8_t ts) __attribute__((always_inline)) {
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(r.x), rCv, n4, e * 4u, 0);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(r.y), rCa, n4, e * 4u, 0);
            __builtin_amdgcn_raw_buffer_store_b8(ts, rCt, n1, e + (uint32_t)N, 0);
        };
        __syncthreads();
        for (int it = 0; it < iters; it++) {
            if (it > 0 && it <= groups) {
                float2 r[FC_G];
                uint8_t ts[FC_G];
#pragma unroll
                for (int i = 0; i < FC_G; i++) {
                    r[i] = out[(it - 1) & 1][i][lane];
                    ts[i] = ots[(it - 1) & 1][i][lane];
                }
                const int left = NB - (it - 1) * FC_G;
                if (left >= FC_G) {
#pragma unroll
                    for (int i = 0; i < FC_G; i++) put(e + (uint32_t)(i * N), r[i], ts[i]);
                } else {
#pragma unroll
                    for (int i = 0; i < FC_G; i++)
                        if (i < left) put(e + (uint32_t)(i * N), r[i], ts[i]);
                }
                e += (uint32_t)(FC_G * N);
            }
            __syncthreads();
        }
    } else {
        const float dd = a.d[nc], th0 = a.theta0[nc];
        if (valid && !params_ok(a.tau_m[n], a.tau_a[n], dd, th0)) atomicOr(a.status, 1u);
        const float beta = (float)exp(lb), pf = (float)exp(lp);
        const double betaT = exp(lb * TR), pT = exp(lp * TR), pTm1 = exp(lp * (TR - 1));
        float bk[L], pt[TR], bsL[SEG];   // beta^(k + 1); p^t; beta^(first step of the segment)
        double pd[TAB ? 1 : TR];         // p^k
        const float bL = (float)exp(lb * (double)L);
        const float bPart = (float)exp(lb * (double)(TR - TR / L * L));   // over a partial segment
#pragma unroll
        for (int k = 0; k < L; k++) bk[k] = (float)exp(lb * (double)(k + 1));
#pragma unroll
        for (int k = 0; k < TR; k++) pt[k] = (float)exp(lp * (double)k);
#pragma unroll
        for (int s = 0; s < SEG; s++) bsL[s] = (float)exp(lb * (double)(s * L));
        if constexpr (!TAB)
#pragma unroll
            for (int k = 0; k < TR; k++) pd[k] = exp(lp * (double)k);
        double v0 = 0.0, a0 = 0.0;
        int cts = 0;
        if (a.init_v && valid) {
            const size_t i = (size_t)b * N + n;
            v0 = a.init_v[i];
            a0 = a.init_a[i];
            cts = a.init_ts[i];
            if (cts < 0 || cts > TR) {
                atomicOr(a.status, 1u);
                cts = 0;
            }
        }
        if (ck && valid) a.ck.ts[CO + n] = (uint8_t)cts;
        float cv = (float)v0, da1 = dd * fmaf(pf, (float)a0, cts == TR ? 1.0f : 0.0f);
        auto block = [&](const float (&x)[TR], float2 &o, uint8_t &ot) __attribute__((always_inline)) {
            // each segment's steps from its start (Prop. 1), the first cts - 1 masked
            float uu[TR];
            auto scan = [&](auto masked) __attribute__((always_inline)) {
#pragma unroll
                for (int t = 0; t < TR; t++) {
                    const float d = decltype(masked)::value && t < TR - 1 && cts > t + 1 ? 0.0f : x[t];
                    uu[t] = t % L == 0 ? d : fmaf(beta, uu[t > 0 ? t - 1 : 0], d);
                }
            };
            if constexpr (TAB) {
                if (__any(cts > 1)) scan(std::true_type{});
                else scan(std::false_type{});
            } else {
                scan(std::true_type{});
            }
            // the membrane's input part at each segment's start, V~ there, and at the block end
            float C[SEG], u = uu[L - 1];
            C[0] = cv;
#pragma unroll
            for (int s = 1; s < SEG; s++) {
                C[s] = fmaf(bsL[s], cv, u);
                u = fmaf((s + 1) * L <= TR ? bL : bPart, u, uu[(s + 1) * L <= TR ? s * L + L - 1 : TR - 1]);
            }
            const double e1 = cts == TR ? pTm1 : 0.0;
            double vn;
            o = make_float2(cv, (float)a0);
            int ts = 0;   // the first step above threshold
            bool spk = false;
            auto above = [&](int t) __attribute__((always_inline)) {
                return fmaf(bk[t % L], C[t / L], uu[t]) > fmaf(pt[t], da1, th0);
            };
            if constexpr (!TAB) {
                // The carry for every place the spike can be in, before the comparison that tells:
                // what follows it is a selection, so the chain from one block's comparison to the
                // next's does not run through the FP64 adaptation.
                double an[TR];     // a after: no spike or one in the last step; a spike in step 1, 2, ...
                float dn[TR + 1];  // a[1] of the next block: no spike; a spike in step 1, 2, ..., T_R
                an[0] = fma(pT, a0, e1);
#pragma unroll
                for (int k = 1; k < TR; k++) an[k] = fma(pT, a0, e1 + pd[TR - 1 - k]);
#pragma unroll
                for (int k = 0; k < TR; k++) dn[k] = fmaf(pf, (float)an[k], 0.0f);
                dn[TR] = fmaf(pf, (float)an[0], 1.0f);
                vn = fma(betaT, v0, (double)u);
                double as = an[0];
                float ds = dn[0];
#pragma unroll
                for (int k = TR - 1; k >= 0; k--) {
                    const bool c = above(k);
                    ts = c ? k + 1 : ts;
                    as = c ? an[k == TR - 1 ? 0 : k + 1] : as;
                    ds = c ? dn[k + 1] : ds;
                    spk |= c;
                }
                a0 = as;
                da1 = dd * ds;
            } else {
                vn = fma(betaT, v0, (double)u);
#pragma unroll
                for (int k = TR - 1; k >= 0; k--) ts = above(k) ? k + 1 : ts;
                spk = ts > 0;
                const double an = fma(pT, a0, e1);
                if (__any(spk)) {
                    const double e2 = ptab[lane * TR + (spk ? max(TR - 1 - ts, 0) : 0)];
                    const double as = fma(pT, a0, e1 + (ts < TR ? e2 : 0.0));
                    a0 = spk ? as : an;
                } else {
                    a0 = an;
                }
                da1 = dd * fmaf(pf, (float)a0, ts == TR ? 1.0f : 0.0f);
            }
            ot = (uint8_t)ts;
            v0 = spk ? 0.0 : vn;
            cv = spk ? 0.0f : (float)vn;
            cts = ts;
        };
        __builtin_amdgcn_s_setprio(3);   // (the other waves have time)
        __syncthreads();
        for (int it = 0; it < iters; it++) {
            const int nb0 = it * FC_G;
            if (nb0 < NB) {
                float x[FC_G][TR];
#pragma unroll
                for (int i = 0; i < FC_G; i++)
#pragma unroll
                    for (int k = 0; k < TR; k++) x[i][k] = in[it & 1][i][k][lane];
                if (nb0 + FC_G <= NB) {
#pragma unroll
                    for (int i = 0; i < FC_G; i++) block(x[i], out[it & 1][i][lane], ots[it & 1][i][lane]);
                } else {
#pragma unroll
                    for (int i = 0; i < FC_G; i++)
                        if (nb0 + i < NB) block(x[i], out[it & 1][i][lane], ots[it & 1][i][lane]);
                }
            }
            __syncthreads();
        }
        if (valid) {
            if (ck) {
                a.ck.v[CO + (size_t)NB * N + n] = (float)v0;
                a.ck.a[CO + (size_t)NB * N + n] = (float)a0;
            }
            if (a.fin_v) {
                const size_t i = (size_t)b * N + n;
                a.fin_v[i] = v0;
                a.fin_a[i] = a0;
                a.fin_ts[i] = cts;
            }
        }
    }
}

}  // namespace

// The chain pays while the card is not full: up to two and a half groups of 64 neurons a CU with
// carries kept, four without (less where the LDS of a workgroup or its registers allow fewer at a
// time); above, the block kernel's waves hide each other's latency and 256 neurons a workgroup
// write rows in wider pieces. us, block kernel / this one: T_R 2: 768 groups 118 / 121 with
// carries, 107 / 65 without; 1024 groups 138 / 165 and 112 / 70; T_R 20 without: 640 groups 55 / 42,
// 1024 groups 77 / 74; T_R 28: 512 groups 48 / 37, 640 groups 61 / 69.
// A call of one block (the recurrent layer over 256 neurons makes one a block) has no chain, but
// its loads and stores still run beside each other: 8 x 320, with carries, T_R 2 6.2 / 5.5, 4 8.3 /
// 5.6, 10 6.1 / 5.5, 20 8.2 / 7.9, 32 11.3 / 11.2; T_R 3, whose groups of 16 blocks are the
// longest to load, 6.9 / 7.0 (32 x 1024: 7.3 / 7.7), and from four blocks on 7.6 / 7.1.
bool fwd_chain_ok(int B, int N, int TR, int NB, bool traces, bool carries) {
    const int most = TR > 24 ? 512 : carries ? 640 : TR == 3 ? 768 : 1024;
    return TR <= 32 && !traces && (TR != 3 || NB >= 4) && (long long)B * ((N + 63) / 64) <= most;
}

hipError_t launch_fwd_chain(FwdArgs a, hipStream_t st) {
    a.n_groups = (a.N + 63) / 64;
    const unsigned grid = (unsigned)(a.B * a.n_groups);
    if (grid == 0) return hipSuccess;
    const dim3 blk(a.ck.v ? 256 : 192);
    switch (a.TR) {
#define ALIF_FC(TR) case TR: hipLaunchKernelGGL((k_fwd_chain<TR>), dim3(grid), blk, 0, st, a); break;
        ALIF_FC(2) ALIF_FC(3) ALIF_FC(4) ALIF_FC(5) ALIF_FC(6) ALIF_FC(7) ALIF_FC(8) ALIF_FC(9) ALIF_FC(10)
        ALIF_FC(11) ALIF_FC(12) ALIF_FC(13) ALIF_FC(14) ALIF_FC(15) ALIF_FC(16) ALIF_FC(17) ALIF_FC(18) ALIF_FC(19)
        ALIF_FC(20) ALIF_FC(21) ALIF_FC(22) ALIF_FC(23) ALIF_FC(24) ALIF_FC(25) ALIF_FC(26) ALIF_FC(27) ALIF_FC(28)
        ALIF_FC(29) ALIF_FC(30) ALIF_FC(31) ALIF_FC(32)
#undef ALIF_FC
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace alif
