// Leaky non-spiking readout (paper supplementary, "Readout neurons"):
//   I_r = W_r S,  V_r[t] = beta_r V_r[t-1] + (1 - beta_r) I_r[t],  o = sum_t V_r[t],
// beta_r = exp(-DT / tau_r). The projection runs on the MFMA GEMM; the
// integration runs in FP64, each (batch, readout neuron) row on 32 to 64 threads that take
// a chunk of time each and join their carries through LDS.
// Workspace layout (kept by the caller from forward to backward):
//   I_r [B*T][C] f32 | V_r [B*T][C] f32 | gI_r [B*T][C] f32 | part [B][C] f64 | GEMM split scratch
#include <hip/hip_runtime.h>

#include <cmath>

#include "../../include/blockalif.h"
#include "alif_common.h"
#include "alif_gemm.h"
#include "alif_kernels.h"

namespace alif {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

size_t a256(size_t x) { return (x + 255) & ~(size_t)255; }

struct RoWs {
    float *Ir, *Vr, *gIr;
    double *part;
    void *gemm;
};
RoWs ro_ws(void *ws, int B, int T, int C) {
    const size_t mc = (size_t)B * T * C * sizeof(float);
    char *p = (char *)ws;
    RoWs w;
    w.Ir = (float *)p;
    w.Vr = (float *)(p + a256(mc));
    w.gIr = (float *)(p + 2 * a256(mc));
    w.part = (double *)(p + 3 * a256(mc));
    w.gemm = p + 3 * a256(mc) + a256((size_t)B * C * sizeof(double));
    return w;
}

// Each (b, c) row's recurrence over T is cut into RK chunks of Lc = ceil(T / RK)
// steps. A workgroup holds batch element b = blockIdx.x and CG classes (blockIdx.y
// picks which): thread (k, cl) = (tid / CG, tid % CG) takes chunk k of class cl,
// so consecutive threads read consecutive classes of one step. A chunk first runs
// from zero to get its local end value; through LDS every thread then forms its
// true carry-in,
//   V_in(k) = sum over k' < k of beta^(Lc (k - 1 - k')) e(k')   (Horner over k'),
// and reruns its chunk from it, writing V_r and summing it; the chunk sums are added
// in chunk order. Loads go RU steps at a time, and a chunk of at most RU steps stays in
// registers between the runs. The backward is the same with the reverse recurrence (its
// local value is a geometric sum) and the carry from the chunks after. Every chunk before
// the last non-empty one is full, so beta^Lc is the only decay across chunks.
//
// What bounds it: latency, a row's chunks on one CU. As many chunks as 1024 threads allow,
// up to 64, against 16 (with a second local run in the backward): 32 x 20 x 1000 the forward call
// 72 -> 50 us, the backward call 134 -> 101 us; 32 x 20 x 4000 173 -> 87 and 422 -> 261 us.
constexpr int RKM = 64;  // chunks a row at most
constexpr int RU = 24;   // steps whose loads are issued together (128 registers a thread)
constexpr int RUB = 12;  // in the backward, which reads two rows
constexpr int RCG = 32;  // classes a workgroup at most
constexpr int RTH = 1024;

int ro_chunks(int cg) { return RTH / cg < RKM ? RTH / cg : RKM; }

__device__ __forceinline__ void load_fwd(float (&x)[RU], const float *__restrict__ ir, int C, int t0, int t1) {
#pragma unroll
    for (int u = 0; u < RU; u++) x[u] = t0 + u < t1 ? ir[(size_t)(t0 + u) * C] : 0.0f;
}

// Run v <- beta v + omb I[t] over the up to RU steps from t0, I in x; with STORE, write V_r and sum v.
template <bool STORE>
__device__ __forceinline__ double run_fwd(const float (&x)[RU], float *__restrict__ vr, int C, int t0, int t1,
                                          double beta, double omb, double v, double &sum) {
#pragma unroll
    for (int u = 0; u < RU; u++)
        if (t0 + u < t1) {
            v = fma(beta, v, omb * (double)x[u]);
            if constexpr (STORE) {
                vr[(size_t)(t0 + u) * C] = (float)v;
                sum += v;
            }
        }
    return v;
}

__global__ __launch_bounds__(RTH) void k_readout_fwd(int B, int T, int C, int CG, double dt,
                                                     const float *__restrict__ tau_r, const float *__restrict__ Ir,
                                                     float *__restrict__ Vr, float *__restrict__ o) {
    __shared__ double sh[RTH];
    const int RK = blockDim.x / CG;
    const int k = threadIdx.x / CG, cl = threadIdx.x - k * CG;
    const int b = blockIdx.x, c = blockIdx.y * CG + cl;
    const bool ok = c < C;
    const double lb = -dt / (double)tau_r[ok ? c : 0];
    const double beta = exp(lb), omb = -expm1(lb);
    const int Lc = (T + RK - 1) / RK;
    const int t0 = min(T, k * Lc), t1 = ok ? min(T, t0 + Lc) : t0;
    const float *ir = Ir + (size_t)b * T * C + (ok ? c : 0);
    float *vr = Vr + (size_t)b * T * C + (ok ? c : 0);
    float x[RU];
    double unused = 0.0, e = 0.0;
    for (int tb = t0; tb < t1; tb += RU) {
        load_fwd(x, ir, C, tb, t1);
        e = run_fwd<false>(x, vr, C, tb, t1, beta, omb, e, unused);
    }
    sh[threadIdx.x] = e;
    __syncthreads();
    const double dk = exp(lb * (double)Lc);
    double v = 0.0;
    for (int kk = 0; kk < k; kk++) v = fma(dk, v, sh[kk * CG + cl]);
    double sum = 0.0;
    if (Lc <= RU) {   // uniform
        run_fwd<true>(x, vr, C, t0, t1, beta, omb, v, sum);
    } else {
        for (int tb = t0; tb < t1; tb += RU) {
            load_fwd(x, ir, C, tb, t1);
            v = run_fwd<true>(x, vr, C, tb, t1, beta, omb, v, sum);
        }
    }
    __syncthreads();
    sh[threadIdx.x] = sum;
    __syncthreads();
    if (ok && k == 0) {
        double tot = 0.0;
        for (int kk = 0; kk < RK; kk++) tot += sh[kk * CG + cl];
        o[(size_t)b * C + c] = (float)tot;
    }
}

// reverse recurrence lam[t] = go + beta lam[t+1]; gI_r[t] = (1 - beta) lam[t];
// d/dbeta = sum_t (V_r[t-1] - I_r[t]) lam[t]
__global__ __launch_bounds__(RTH) void k_readout_bwd(int B, int T, int C, int CG, double dt,
                                                     const float *__restrict__ tau_r, const float *__restrict__ Ir,
                                                     const float *__restrict__ Vr, const float *__restrict__ go,
                                                     float *__restrict__ gIr, double *__restrict__ part) {
    __shared__ double sh[RTH];
    const int RK = blockDim.x / CG;
    const int k = threadIdx.x / CG, cl = threadIdx.x - k * CG;
    const int b = blockIdx.x, c = blockIdx.y * CG + cl;
    const bool ok = c < C;
    const double lb = -dt / (double)tau_r[ok ? c : 0];
    const double beta = exp(lb), omb = -expm1(lb);
    const double g = ok ? (double)go[(size_t)b * C + c] : 0.0;
    const int Lc = (T + RK - 1) / RK;
    const int t0 = min(T, k * Lc), t1 = ok ? min(T, t0 + Lc) : t0;
    const size_t base = (size_t)b * T * C + (ok ? c : 0);
    const float *ir = Ir + base, *vr = Vr + base;
    float *gi = gIr + base;
    // the carry at this chunk's end: lambda at step t1 from the T - t1 steps of the later
    // chunks, g (1 + beta + ... + beta^(T - t1 - 1)); none without later steps (0 times an infinite
    // g or an infinite rate is not)
    double lam = 0.0;
    if (t1 < T) lam = omb != 0.0 ? g * (-expm1(lb * (double)(T - t1)) / omb) : g * (double)(T - t1);
    double gb = 0.0;
    for (int tb = t1 - 1; tb >= t0; tb -= RUB) {
        float xi[RUB], xv[RUB];
#pragma unroll
        for (int u = 0; u < RUB; u++) {
            const int t = tb - u;
            xi[u] = t >= t0 ? ir[(size_t)t * C] : 0.0f;
            xv[u] = (t >= t0 && t > 0) ? vr[(size_t)(t - 1) * C] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < RUB; u++) {
            const int t = tb - u;
            if (t >= t0) {
                lam = fma(beta, lam, g);
                gi[(size_t)t * C] = (float)(omb * lam);
                gb = fma((double)xv[u] - (double)xi[u], lam, gb);
            }
        }
    }
    sh[threadIdx.x] = gb;
    __syncthreads();
    if (ok && k == 0) {
        double tot = 0.0;
        for (int kk = 0; kk < RK; kk++) tot += sh[kk * CG + cl];
        part[(size_t)b * C + c] = tot;
    }
}

__global__ void k_readout_tau(int B, int C, double dt, const float *tau_r, const double *part, float *g_tau) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= C) return;
    double s = 0.0;
#pragma unroll 16
    for (int b = 0; b < B; b++) s += part[(size_t)b * C + c];   // (loads in flight, added in order)
    const double tau = tau_r[c];
    g_tau[c] = (float)(s * exp(-dt / tau) * dt / (tau * tau));
}

// ---------------------------------------------------------------------------
// The readout's products for few classes (C <= RO_MAXC), rows of a multiple of four
// hidden neurons. What bounds them: the spikes, read once, or their gradients, written
// once. The GEMMs' tiles are 128 classes wide (at 20 classes 6 of 7 products are padding)
// and rows of a class count that is no multiple of 4 fall to the general kernel. M = B T.
// us a call with GEMMs / with these, forward and backward: 32 x 1000 x 512, 20 classes: 50 / 33 and
// 101 / 70; 35 classes 58 / 44 and 327 / 101; 128 x 1000 x 512, 10 classes 107 / 64 and 1224 / 155;
// errors against 64 bits at most the GEMMs' (weight gradient 2.9e-7 -> 3.8e-8).
// ---------------------------------------------------------------------------
constexpr int RO_MAXC = 48;
constexpr int RO_ROWS = 64;    // rows of gI_r staged in LDS
constexpr int RO_PARTS = 256;  // partial sums of the weight gradient at most

// four consecutive spikes
template <int DT>
__device__ __forceinline__ floatx4 ld_spk4(const void *p, size_t i) {
    if constexpr (DT == 0) return *reinterpret_cast<const floatx4 *>(static_cast<const float *>(p) + i);
    else if constexpr (DT == 1) {
        const uint32_t w = *reinterpret_cast<const uint32_t *>(static_cast<const uint8_t *>(p) + i);
        return floatx4{(float)(w & 0xffu), (float)((w >> 8) & 0xffu), (float)((w >> 16) & 0xffu), (float)(w >> 24)};
    } else {
        const uint2 w = *reinterpret_cast<const uint2 *>(static_cast<const uint16_t *>(p) + i);
        return floatx4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                       __uint_as_float(w.y & 0xffff0000u)};
    }
}

// I_r[m][c] = sum_h S[m][h] W_r[c][h]: a wave takes 16 rows and every class. Lane (r, q) holds
// hidden neurons 16 s + 4 q + e of row r (and of class r), so one 16-byte load feeds four
// v_mfma_f32_16x16x4_f32, which sum q = 0..3 of one e; even and odd s have their own sums.
template <int DT, int NT>
__global__ __launch_bounds__(256) void k_ro_current(long long M, int H, int C, const void *__restrict__ S,
                                                    const float *__restrict__ W, float *__restrict__ Ir) {
    constexpr int U = 4;
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const long long m0 = ((long long)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16;
    if (m0 >= M) return;   // no barrier in this kernel
    const size_t srow = (size_t)(m0 + r < M ? m0 + r : M - 1) * H;
    const float *wrow[NT];
#pragma unroll
    for (int j = 0; j < NT; j++) wrow[j] = W + (size_t)min(16 * j + r, C - 1) * H;
    floatx4 acc[2][NT];
#pragma unroll
    for (int j = 0; j < NT; j++) acc[0][j] = acc[1][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int h0 = 4 * q; h0 < H + 4 * q; h0 += 16 * U) {   // (uniform)
        floatx4 a[U], w[U][NT];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int h = h0 + 16 * u;   // H % 4 == 0: four in range or none
            const bool in = h < H;
            const int hc = in ? h : 0;
            a[u] = ld_spk4<DT>(S, srow + hc);
#pragma unroll
            for (int j = 0; j < NT; j++) w[u][j] = *reinterpret_cast<const floatx4 *>(wrow[j] + hc);
#pragma unroll
            for (int e = 0; e < 4; e++) {
                a[u][e] = in ? a[u][e] : 0.0f;
#pragma unroll
                for (int j = 0; j < NT; j++) w[u][j][e] = in ? w[u][j][e] : 0.0f;
            }
        }
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int e = 0; e < 4; e++)
#pragma unroll
                for (int j = 0; j < NT; j++)
                    acc[u & 1][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][e], w[u][j][e], acc[u & 1][j], 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < NT; j++)
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const long long m = m0 + 4 * q + e;
            if (m < M && 16 * j + r < C) Ir[m * C + 16 * j + r] = acc[0][j][e] + acc[1][j][e];
        }
}

// RO_ROWS rows of gI_r from m0 into LDS, classes padded with zeros to CP
template <int CP>
__device__ __forceinline__ void stage_gir(float (&g)[RO_ROWS][CP], const float *__restrict__ gIr, long long m0,
                                          long long m1, int C) {
    for (int i = threadIdx.x; i < RO_ROWS * CP; i += 256) {
        const int row = i / CP, c = i - row * CP;
        g[row][c] = m0 + row < m1 && c < C ? gIr[(m0 + row) * C + c] : 0.0f;
    }
}

// gS[m][h] = sum_c gI_r[m][c] W_r[c][h]: a lane holds four columns of W_r, a wave takes 16 of
// the staged rows (one LDS broadcast feeds 16 multiply-adds).
template <int CP>
__global__ __launch_bounds__(256) void k_ro_dx(long long M, int H, int C, const float *__restrict__ gIr,
                                               const float *__restrict__ W, float *__restrict__ gS) {
    __shared__ __align__(16) float g[RO_ROWS][CP];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long m0 = (long long)blockIdx.x * RO_ROWS;
    const int h = blockIdx.y * 256 + 4 * lane;
    stage_gir<CP>(g, gIr, m0, M, C);
    floatx4 w[CP];
#pragma unroll
    for (int c = 0; c < CP; c++)
        w[c] = c < C && h < H ? *reinterpret_cast<const floatx4 *>(W + (size_t)c * H + h) : floatx4{0.f, 0.f, 0.f, 0.f};
    __syncthreads();
#pragma unroll 2
    for (int i = 0; i < RO_ROWS / 4; i++) {
        const int row = wave * (RO_ROWS / 4) + i;
        if (m0 + row >= M) break;   // uniform
        floatx4 s = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < CP; c += 4) {
            const floatx4 x = *reinterpret_cast<const floatx4 *>(&g[row][c]);
#pragma unroll
            for (int k = 0; k < 4; k++)
#pragma unroll
                for (int e = 0; e < 4; e++) s[e] = fmaf(x[k], w[c + k][e], s[e]);
        }
        if (h < H) *reinterpret_cast<floatx4 *>(gS + (m0 + row) * H + h) = s;
    }
}

// part[p][c][h] = sum over the p-th share of the rows of gI_r[m][c] S[m][h]: a lane holds four
// columns for every class, the four waves a quarter of the staged rows each.
template <int DT, int CP>
__global__ __launch_bounds__(256) void k_ro_dw(long long M, int H, int C, long long per, const float *__restrict__ gIr,
                                               const void *__restrict__ S, float *__restrict__ part) {
    constexpr int Q = RO_ROWS / 4;
    __shared__ __align__(16) float g[RO_ROWS][CP];
    __shared__ __align__(16) floatx4 sum[CP][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long b0 = blockIdx.x * per, b1 = b0 + per < M ? b0 + per : M;
    const int h = blockIdx.y * 256 + 4 * lane;
    floatx4 acc[CP];
#pragma unroll
    for (int c = 0; c < CP; c++) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (long long m0 = b0; m0 < b1; m0 += RO_ROWS) {
        __syncthreads();
        stage_gir<CP>(g, gIr, m0, b1, C);
        __syncthreads();
        for (int i0 = 0; i0 < Q; i0 += 4) {
            floatx4 s[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {   // (rows past the end: any row, times zero below)
                const long long m = m0 + wave * Q + i0 + i;
                const bool in = m < b1 && h < H;
                s[i] = ld_spk4<DT>(S, in ? (size_t)m * H + h : 0);
#pragma unroll
                for (int e = 0; e < 4; e++) s[i][e] = in ? s[i][e] : 0.0f;
            }
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int c = 0; c < CP; c += 4) {
                    const floatx4 x = *reinterpret_cast<const floatx4 *>(&g[wave * Q + i0 + i][c]);
#pragma unroll
                    for (int k = 0; k < 4; k++)
#pragma unroll
                        for (int e = 0; e < 4; e++) acc[c + k][e] = fmaf(x[k], s[i][e], acc[c + k][e]);
                }
        }
    }
    for (int v = 1; v < 4; v++) {
        __syncthreads();
        if (wave == v)
#pragma unroll
            for (int c = 0; c < CP; c++) sum[c][lane] = acc[c];
        __syncthreads();
        if (wave == 0)
#pragma unroll
            for (int c = 0; c < CP; c++) acc[c] += sum[c][lane];
    }
    if (wave == 0 && h < H)
#pragma unroll
        for (int c = 0; c < CP; c++)
            if (c < C) *reinterpret_cast<floatx4 *>(part + ((size_t)blockIdx.x * C + c) * H + h) = acc[c];
}

// gW[i] = sum_p part[p][i], in FP64 and in order within each of four shares of the parts
__global__ __launch_bounds__(256) void k_ro_dw_sum(int CH, int parts, const float *__restrict__ part,
                                                   float *__restrict__ gW) {
    __shared__ double sh[4][64];
    const int l = threadIdx.x & 63, g = threadIdx.x >> 6, i = blockIdx.x * 64 + l;
    const int per = (parts + 3) / 4, p1 = min(parts, (g + 1) * per);
    double s = 0.0;
    if (i < CH)
#pragma unroll 16
        for (int p = g * per; p < p1; p++) s += (double)part[(size_t)p * CH + i];
    sh[g][l] = s;
    __syncthreads();
    if (g == 0 && i < CH) gW[i] = (float)((sh[0][l] + sh[1][l]) + (sh[2][l] + sh[3][l]));
}

int dw_parts(long long M) {
    const long long p = (M + RO_ROWS - 1) / RO_ROWS;
    return (int)(p < RO_PARTS ? (p < 1 ? 1 : p) : RO_PARTS);
}

bool few_classes(int C, int H) { return C <= RO_MAXC && H % 4 == 0; }
bool aligned(const void *p, size_t to) { return (reinterpret_cast<uintptr_t>(p) & (to - 1)) == 0; }

#define ALIF_RO_CP(GO)                                                                  \
    do {                                                                                \
        if (C <= 8) GO(8); else if (C <= 16) GO(16); else if (C <= 24) GO(24);          \
        else if (C <= 32) GO(32); else if (C <= 40) GO(40); else GO(48);                \
    } while (0)

int dt_code(int spike_dtype) { return spike_dtype == ALIF_SPIKES_U8 ? 1 : (spike_dtype == ALIF_SPIKES_BF16 ? 2 : 0); }

int wsplits(long long M, int N, int K) {
    const long long tiles = (long long)((N + 127) / 128) * ((K + 127) / 128);
    long long s = 512 / (tiles > 0 ? tiles : 1);
    s = s < 1 ? 1 : (s > 64 ? 64 : s);
    if (s > M / 256) s = M / 256 < 1 ? 1 : M / 256;
    return (int)s;
}

}  // namespace
}  // namespace alif

using namespace alif;

extern "C" {

int alif_readout_workspace_bytes(int32_t B, int32_t T, int32_t n_hidden, int32_t C, size_t *bytes) {
    if (B < 0 || T < 0 || n_hidden <= 0 || C <= 0 || !bytes) return alif::set_error(ALIF_EINVAL, "bad readout sizes");
    const size_t mc = (size_t)B * T * C * sizeof(float);
    const long long M = (long long)B * T;
    int s = wsplits(M, C, n_hidden);
    s = s > 1 ? s : 0;
    if (few_classes(C, n_hidden) && dw_parts(M) > s) s = dw_parts(M);
    *bytes = 3 * a256(mc) + a256((size_t)B * C * sizeof(double)) + (size_t)s * C * n_hidden * sizeof(float);
    return ALIF_OK;
}

int alif_readout_forward(int32_t B, int32_t T, int32_t n_hidden, int32_t C, double dt_ms,
                         int32_t spike_dtype, const void *spikes, const float *W_r,
                         const float *tau_r, float *o, void *workspace, void *stream) {
    if (B < 0 || T < 0 || n_hidden <= 0 || C <= 0 || !(dt_ms > 0))
        return alif::set_error(ALIF_EINVAL, "bad readout sizes or dt");
    if (spike_dtype < ALIF_SPIKES_U8 || spike_dtype > ALIF_SPIKES_F32)
        return alif::set_error(ALIF_EINVAL, "unknown spike_dtype");
    if (!spikes || !W_r || !tau_r || !o || !workspace)
        return alif::set_error(ALIF_EINVAL, "NULL readout argument");
    if ((C + RCG - 1) / RCG > 65535)
        return alif::set_error(ALIF_EUNSUPPORTED, "too many readout neurons (C / 32 must stay within 65535)");
    hipStream_t st = (hipStream_t)stream;
    RoWs w = ro_ws(workspace, B, T, C);
    GemmArgs g{};
    g.M = (long long)B * T; g.N = C; g.K = n_hidden;
    g.A = spikes; g.a_dt = dt_code(spike_dtype); g.lda = n_hidden; g.a_kc = 1;
    g.B = W_r; g.b_dt = 0; g.ldb = n_hidden; g.b_kc = 1;
    g.C = w.Ir; g.ldc = C; g.splits = 1;
    hipError_t e;
    const size_t es = spike_dtype == ALIF_SPIKES_U8 ? 1 : (spike_dtype == ALIF_SPIKES_BF16 ? 2 : 4);
    if (g.M > 0 && few_classes(C, n_hidden) && aligned(spikes, 4 * es) && aligned(W_r, 16) && g.M < (1LL << 36)) {
        const dim3 grid((unsigned)((g.M + 63) / 64)), blk(256);
#define ALIF_RO_I(DT, NT) \
    hipLaunchKernelGGL((k_ro_current<DT, NT>), grid, blk, 0, st, g.M, n_hidden, C, spikes, W_r, w.Ir)
#define ALIF_RO_N(DT) do { if (C <= 16) ALIF_RO_I(DT, 1); else if (C <= 32) ALIF_RO_I(DT, 2); else ALIF_RO_I(DT, 3); } while (0)
        if (g.a_dt == 0) ALIF_RO_N(0);
        else if (g.a_dt == 1) ALIF_RO_N(1);
        else ALIF_RO_N(2);
#undef ALIF_RO_N
#undef ALIF_RO_I
        e = hipGetLastError();
    } else {
        e = gemm_launch(g, false, st);
    }
    if (e != hipSuccess) return alif::set_error(ALIF_EHIP, hipGetErrorString(e));
    if (B == 0) return ALIF_OK;
    const int cg = C < RCG ? C : RCG;
    hipLaunchKernelGGL(k_readout_fwd, dim3((unsigned)B, (unsigned)((C + cg - 1) / cg)),
                       dim3(ro_chunks(cg) * cg), 0, st, B, T, C, cg, dt_ms, tau_r, w.Ir, w.Vr, o);
    e = hipGetLastError();
    if (e != hipSuccess) return alif::set_error(ALIF_EHIP, hipGetErrorString(e));
    return ALIF_OK;
}

int alif_readout_backward(int32_t B, int32_t T, int32_t n_hidden, int32_t C, double dt_ms,
                          int32_t spike_dtype, const void *spikes, const float *W_r,
                          const float *tau_r, const float *go, float *grad_spikes,
                          float *grad_W_r, float *grad_tau_r, void *workspace, void *stream) {
    if (B < 0 || T < 0 || n_hidden <= 0 || C <= 0 || !(dt_ms > 0))
        return alif::set_error(ALIF_EINVAL, "bad readout sizes or dt");
    if (!spikes || !W_r || !tau_r || !go || !workspace)
        return alif::set_error(ALIF_EINVAL, "NULL readout argument");
    if ((C + RCG - 1) / RCG > 65535)
        return alif::set_error(ALIF_EUNSUPPORTED, "too many readout neurons (C / 32 must stay within 65535)");
    hipStream_t st = (hipStream_t)stream;
    RoWs w = ro_ws(workspace, B, T, C);
    if (B > 0) {
        const int cg = C < RCG ? C : RCG;
        hipLaunchKernelGGL(k_readout_bwd, dim3((unsigned)B, (unsigned)((C + cg - 1) / cg)),
                           dim3(ro_chunks(cg) * cg), 0, st, B, T, C, cg, dt_ms, tau_r, w.Ir, w.Vr, go, w.gIr, w.part);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return alif::set_error(ALIF_EHIP, hipGetErrorString(e));
    }
    if (grad_tau_r) {
        hipLaunchKernelGGL(k_readout_tau, dim3((C + 127) / 128), dim3(128), 0, st, B, C, dt_ms, tau_r,
                           w.part, grad_tau_r);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return alif::set_error(ALIF_EHIP, hipGetErrorString(e));
    }
    const long long M = (long long)B * T;
    const unsigned cols = (unsigned)((n_hidden + 255) / 256);
    const bool few = M > 0 && M < (1LL << 36) && few_classes(C, n_hidden) && cols <= 65535;
    if (grad_spikes && few && aligned(W_r, 16) && aligned(grad_spikes, 16)) {
        const dim3 grid((unsigned)((M + RO_ROWS - 1) / RO_ROWS), cols), blk(256);
#define ALIF_RO_X(CP) hipLaunchKernelGGL((k_ro_dx<CP>), grid, blk, 0, st, M, n_hidden, C, w.gIr, W_r, grad_spikes)
        ALIF_RO_CP(ALIF_RO_X);
#undef ALIF_RO_X
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return alif::set_error(ALIF_EHIP, hipGetErrorString(e));
    } else if (grad_spikes) {  // gS[m][h] = sum_c gI_r[m][c] W_r[c][h]
        GemmArgs g{};
        g.M = M; g.N = n_hidden; g.K = C;
        g.A = w.gIr; g.a_dt = 0; g.lda = C; g.a_kc = 1;
        g.B = W_r; g.b_dt = 0; g.ldb = n_hidden; g.b_kc = 0;
        g.C = grad_spikes; g.ldc = n_hidden; g.splits = 1;
        hipError_t e = gemm_launch(g, false, st);
        if (e != hipSuccess) return alif::set_error(ALIF_EHIP, hipGetErrorString(e));
    }
    if (grad_W_r) {  // gW_r[c][h] = sum_m gI_r[m][c] S[m][h]
        if (M > 0x7fffffff) return alif::set_error(ALIF_EUNSUPPORTED, "B*T too large");
        const size_t es = spike_dtype == ALIF_SPIKES_U8 ? 1 : (spike_dtype == ALIF_SPIKES_BF16 ? 2 : 4);
        if (few && aligned(spikes, 4 * es) && aligned(w.gemm, 16)) {
            const int parts = dw_parts(M), CH = C * n_hidden;
            const long long per = ((M + parts - 1) / parts + RO_ROWS - 1) / RO_ROWS * RO_ROWS;
            const int used = (int)((M + per - 1) / per);
            const dim3 grid((unsigned)used, cols), blk(256);
            float *part = (float *)w.gemm;
            const int dt = dt_code(spike_dtype);
#define ALIF_RO_W(CP)                                                                                              \
    do {                                                                                                           \
        if (dt == 0) hipLaunchKernelGGL((k_ro_dw<0, CP>), grid, blk, 0, st, M, n_hidden, C, per, w.gIr, spikes, part); \
        else if (dt == 1) hipLaunchKernelGGL((k_ro_dw<1, CP>), grid, blk, 0, st, M, n_hidden, C, per, w.gIr, spikes, part); \
        else hipLaunchKernelGGL((k_ro_dw<2, CP>), grid, blk, 0, st, M, n_hidden, C, per, w.gIr, spikes, part);     \
    } while (0)
            ALIF_RO_CP(ALIF_RO_W);
#undef ALIF_RO_W
            hipLaunchKernelGGL(k_ro_dw_sum, dim3((unsigned)((CH + 63) / 64)), dim3(256), 0, st, CH, used, part, grad_W_r);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return alif::set_error(ALIF_EHIP, hipGetErrorString(e));
            return ALIF_OK;
        }
        GemmArgs g{};
        g.M = C; g.N = n_hidden; g.K = (int)M;
        g.A = w.gIr; g.a_dt = 0; g.lda = C; g.a_kc = 0;
        g.B = spikes; g.b_dt = dt_code(spike_dtype); g.ldb = n_hidden; g.b_kc = 0;
        g.C = grad_W_r; g.ldc = n_hidden;
        g.splits = wsplits(M, C, n_hidden);
        g.C_part = (float *)w.gemm;
        hipError_t e = gemm_launch(g, false, st);
        if (e != hipSuccess) return alif::set_error(ALIF_EHIP, hipGetErrorString(e));
    }
    return ALIF_OK;
}

}  // extern "C"
