// Forward of blocks of two to four steps (a block is one segment of one lane), without
// traces: the recurrence on one wave per 64 neurons, its loads and stores on others.
//
// What bounds it: the chain. A row's T / T_R blocks follow each other, and one wave issues
// an instruction about every five cycles, so a block costs what its wave issues. One wave
// that does everything spends 95 of them a block at T_R 2, two thirds on addresses, loads,
// spike and carry stores and a table read. Here
//   wave 1 loads the input FC_P groups of FC_G blocks ahead and leaves the drive
//          (1 - beta)(I + b) in LDS,
//   wave 0 runs the blocks of a group from LDS, state in registers (FP64 carries), and
//          leaves each block's carry-in and spike step in LDS,
//   wave 2 writes the spikes of the group before, wave 3 its carries (if they are kept),
// with one barrier a group: 37 instructions a block in the chain. The arithmetic is the block
// kernel's (alif_blocks_impl.h), operation by operation, so spikes and carries are the same bits.
// Forward call, us, against the one-wave form: 1 x 100 x 1000: T_R 2 99 -> 49, T_R 4 77 -> 44;
// 1 x 600 x 20000: T_R 2 1853 -> 874, T_R 3 1473 -> 816, T_R 4 1376 -> 756; with carries kept
// 4 x 2048 x 3000, T_R 2: 289 -> 144. A block takes 0.087 us at T_R 2, about 190 cycles.
#include "alif_common.h"
#include "alif_kernels.h"

namespace alif {
namespace {

constexpr int FC_G = 8;   // blocks a group (one barrier each)
constexpr int FC_P = 3;   // groups of input in registers

template <int L, int SDT>
__global__ __launch_bounds__(256) void k_fwd_chain(FwdArgs a) {
    constexpr uint32_t SB = SDT == 0 ? 1u : (SDT == 1 ? 2u : 4u);
    __shared__ float in[2][FC_G][L][64];
    __shared__ uint4 out[2][FC_G][64];   // carry-in v, a; spike step (0: none)
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

    // Rows go into the scalar offset, which the buffer's range check leaves out: they are
    // kept in range here, and lanes past N are out of range by their own offset.
    if (role == 1) {
        const rsrc_t rI = make_rsrc(a.I + b * bsi, (uint32_t)(TN * 4));
        const float bias = a.bias_k ? a.bias_k[nc] : 0.0f;
        const float omb = (float)(-expm1(lb)), ob = (float)(-expm1(lb) * (double)bias);
        const uint32_t n4 = (uint32_t)nc * 4u;
        float x[FC_P][FC_G][L];
        auto load = [&](float (&d)[FC_G][L], int q) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < FC_G; i++)
#pragma unroll
                for (int k = 0; k < L; k++)
                    d[i][k] = __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b32(
                        rI, n4, (uint32_t)(min((q * FC_G + i) * L + k, T - 1) * N) * 4u, 0));
        };
        auto put = [&](const float (&d)[FC_G][L], int q) __attribute__((always_inline)) {
            const int t0 = q * FC_G * L;
#pragma unroll
            for (int i = 0; i < FC_G; i++)
#pragma unroll
                for (int k = 0; k < L; k++)   // (no input past the end of a ragged last block)
                    in[q & 1][i][k][lane] = fmaf(omb, t0 + i * L + k < T ? d[i][k] : 0.0f, ob);
        };
#pragma unroll
        for (int p = 0; p < FC_P; p++) load(x[p], p);
        put(x[0], 0);
        load(x[0], FC_P);
        __syncthreads();
        for (int it = 0; it < iters; it += FC_P) {
#pragma unroll
            for (int p = 0; p < FC_P; p++) {
                const int q = it + p + 1;   // (past the last group: not read)
                put(x[(p + 1) % FC_P], q);
                load(x[(p + 1) % FC_P], q + FC_P);
                __syncthreads();
            }
        }
    } else if (role == 2) {
        const rsrc_t rS = make_rsrc((const char *)a.spikes + b * bss * SB, (uint32_t)(TN * SB));
        const uint32_t ns = valid ? (uint32_t)n * SB : ALIF_OOB;
        auto put = [&](uint32_t row, bool s) __attribute__((always_inline)) {
            if constexpr (SDT == 0) __builtin_amdgcn_raw_buffer_store_b8((uint8_t)s, rS, ns, row, 0);
            else if constexpr (SDT == 1) __builtin_amdgcn_raw_buffer_store_b16(s ? (uint16_t)0x3F80 : (uint16_t)0, rS, ns, row, 0);
            else __builtin_amdgcn_raw_buffer_store_b32(s ? 0x3F800000u : 0u, rS, ns, row, 0);
        };
        const uint32_t step = (uint32_t)N * SB;
        uint32_t row = 0;   // the group's first
        __syncthreads();
        for (int it = 0; it < iters; it++) {
            if (it > 0 && it <= groups) {
                int ts[FC_G];
#pragma unroll
                for (int i = 0; i < FC_G; i++) ts[i] = (int)out[(it - 1) & 1][i][lane].z;
                const int left = T - (it - 1) * FC_G * L;   // rows
                if (left >= FC_G * L) {
#pragma unroll
                    for (int i = 0; i < FC_G * L; i++) put(row + i * step, ts[i / L] == i % L + 1);
                } else {
#pragma unroll
                    for (int i = 0; i < FC_G * L; i++)
                        if (i < left) put(row + i * step, ts[i / L] == i % L + 1);
                }
                row += FC_G * L * step;
            }
            __syncthreads();
        }
    } else if (role == 3) {
        const rsrc_t rCv = make_rsrc(a.ck.v + CO, (uint32_t)(CE * 4)), rCa = make_rsrc(a.ck.a + CO, (uint32_t)(CE * 4));
        const rsrc_t rCt = make_rsrc(a.ck.ts + CO, (uint32_t)CE);
        const uint32_t n4 = valid ? (uint32_t)n * 4u : ALIF_OOB, n1 = valid ? (uint32_t)n : ALIF_OOB;
        uint32_t e = 0;   // row of the group's first carry
        auto put = [&](uint32_t e, uint4 r) __attribute__((always_inline)) {
            __builtin_amdgcn_raw_buffer_store_b32(r.x, rCv, n4, e * 4u, 0);
            __builtin_amdgcn_raw_buffer_store_b32(r.y, rCa, n4, e * 4u, 0);
            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)r.z, rCt, n1, e + (uint32_t)N, 0);
        };
        __syncthreads();
        for (int it = 0; it < iters; it++) {
            if (it > 0 && it <= groups) {
                uint4 r[FC_G];
#pragma unroll
                for (int i = 0; i < FC_G; i++) r[i] = out[(it - 1) & 1][i][lane];
                const int left = NB - (it - 1) * FC_G;
                if (left >= FC_G) {
#pragma unroll
                    for (int i = 0; i < FC_G; i++) put(e + (uint32_t)(i * N), r[i]);
                } else {
#pragma unroll
                    for (int i = 0; i < FC_G; i++)
                        if (i < left) put(e + (uint32_t)(i * N), r[i]);
                }
                e += (uint32_t)(FC_G * N);
            }
            __syncthreads();
        }
    } else {
        const float dd = a.d[nc], th0 = a.theta0[nc];
        if (valid && !params_ok(a.tau_m[n], a.tau_a[n], dd, th0)) atomicOr(a.status, 1u);
        const float beta = (float)exp(lb), pf = (float)exp(lp);
        const double betaT = exp(lb * L), pT = exp(lp * L), pTm1 = exp(lp * (L - 1));
        float bk[L], pt[L];
        double pd[L];   // p^k
#pragma unroll
        for (int k = 0; k < L; k++) {
            bk[k] = (float)exp(lb * (double)(k + 1));
            pt[k] = (float)exp(lp * (double)k);
            pd[k] = exp(lp * (double)k);
        }
        double v0 = 0.0, a0 = 0.0;
        int cts = 0;
        if (a.init_v && valid) {
            const size_t i = (size_t)b * N + n;
            v0 = a.init_v[i];
            a0 = a.init_a[i];
            cts = a.init_ts[i];
            if (cts < 0 || cts > L) {
                atomicOr(a.status, 1u);
                cts = 0;
            }
        }
        if (ck && valid) a.ck.ts[CO + n] = (uint8_t)cts;
        float cv = (float)v0, da1 = dd * fmaf(pf, (float)a0, cts == L ? 1.0f : 0.0f);
        // The carry for every place the spike can be in, before the comparison that tells:
        // what follows it is a selection, so the chain from one block's comparison to the
        // next's does not run through the FP64 adaptation.
        auto block = [&](const float (&x)[L], uint4 &o) __attribute__((always_inline)) {
            float uu[L];
#pragma unroll
            for (int k = 0; k < L; k++) {
                const float d = k < L - 1 && cts > k + 1 ? 0.0f : x[k];   // masked refractory steps
                uu[k] = k == 0 ? d : fmaf(beta, uu[k > 0 ? k - 1 : 0], d);
            }
            const double e1 = cts == L ? pTm1 : 0.0;
            double an[L];    // a after: no spike or one in the last step; a spike in step 1, 2, ...
            float dn[L + 1]; // a[1] of the next block: no spike; a spike in step 1, 2, ..., L
            an[0] = fma(pT, a0, e1);
#pragma unroll
            for (int k = 1; k < L; k++) an[k] = fma(pT, a0, e1 + pd[L - 1 - k]);
#pragma unroll
            for (int k = 0; k < L; k++) dn[k] = fmaf(pf, (float)an[k], 0.0f);
            dn[L] = fmaf(pf, (float)an[0], 1.0f);
            const double vn = fma(betaT, v0, (double)uu[L - 1]);
            o = make_uint4(__float_as_uint(cv), __float_as_uint((float)a0), 0u, 0u);
            int ts = 0;   // the first step above threshold
            bool spk = false;
            double as = an[0];
            float ds = dn[0];
#pragma unroll
            for (int k = L - 1; k >= 0; k--) {
                const bool c = fmaf(bk[k], cv, uu[k]) > fmaf(pt[k], da1, th0);
                ts = c ? k + 1 : ts;
                as = c ? an[k == L - 1 ? 0 : k + 1] : as;
                ds = c ? dn[k + 1] : ds;
                spk |= c;
            }
            o.z = (uint32_t)ts;
            v0 = spk ? 0.0 : vn;
            cv = spk ? 0.0f : (float)vn;
            a0 = as;
            da1 = dd * ds;
            cts = ts;
        };
        __syncthreads();
        for (int it = 0; it < iters; it++) {
            const int nb0 = it * FC_G;
            if (nb0 < NB) {
                float x[FC_G][L];
#pragma unroll
                for (int i = 0; i < FC_G; i++)
#pragma unroll
                    for (int k = 0; k < L; k++) x[i][k] = in[it & 1][i][k][lane];
                if (nb0 + FC_G <= NB) {
#pragma unroll
                    for (int i = 0; i < FC_G; i++) block(x[i], out[it & 1][i][lane]);
                } else {
#pragma unroll
                    for (int i = 0; i < FC_G; i++)
                        if (nb0 + i < NB) block(x[i], out[it & 1][i][lane]);
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

// The chain pays while its card is not full: more groups than about two and a half a CU with
// carries kept, four without, and the block kernel's 256 neurons a workgroup write their rows
// in wider pieces. T_R 2, us, block kernel / this one: 768 groups 118 / 121 with carries, 107 / 65
// without; 1024 groups 138 / 165 and 112 / 70; 2048 groups (T 2000) 577 / 694 and 311 / 356.
bool fwd_chain_ok(int B, int N, int TR, bool traces, bool carries) {
    return block_config(TR).seg == 1 && !traces && (long long)B * ((N + 63) / 64) <= (carries ? 640 : 1024);
}

hipError_t launch_fwd_chain(FwdArgs a, hipStream_t st) {
    a.n_groups = (a.N + 63) / 64;
    const unsigned grid = (unsigned)(a.B * a.n_groups);
    if (grid == 0) return hipSuccess;
    const dim3 blk(a.ck.v ? 256 : 192);
#define ALIF_FC(L)                                                                                     \
    do {                                                                                               \
        if (a.spike_dtype == 0) hipLaunchKernelGGL((k_fwd_chain<L, 0>), dim3(grid), blk, 0, st, a);    \
        else if (a.spike_dtype == 1) hipLaunchKernelGGL((k_fwd_chain<L, 1>), dim3(grid), blk, 0, st, a); \
        else hipLaunchKernelGGL((k_fwd_chain<L, 2>), dim3(grid), blk, 0, st, a);                       \
    } while (0)
    if (a.TR == 2) ALIF_FC(2);
    else if (a.TR == 3) ALIF_FC(3);
    else ALIF_FC(4);
#undef ALIF_FC
    return hipGetLastError();
}

}  // namespace alif
