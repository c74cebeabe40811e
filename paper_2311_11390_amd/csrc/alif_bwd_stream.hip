// Backward as passes over independent time chunks: the gradients of tau_mem, tau_adapt,
// d, theta0 and bias (all a fit asks for) in one pass forward in time, and dL/dI where it
// is wanted (bwd_stream_gi says by which calls) in one more backward in time.
//
// The sums the reverse adjoint collects,
//   dbeta = sum_t src[t] W[t],   dbias = sum_t src[t] U[t],
//   dp = d sum_t lt[t] Q[t],     dd = sum_t lt[t] a[t],   dtheta0 = sum_t lt[t],
// with src = dL/dV + dL/dS s'(V - theta), lt = dL/dtheta - dL/dS s'(V - theta), are
// inner products of the same local terms with the sensitivities W = dV/dbeta,
// U = dV/dbias and Q = da/dp, which run forward beside the membrane (detached
// policy: the reset, the adaptation jump and the gate are constants):
//   V[t] = (beta V[t-1] + (1 - beta) gate I) (1 - S[t-1]),  a[t] = p a[t-1] + S[t-1],
//   W[t] = (beta W[t-1] + V[t-1] - gate I) (1 - S[t-1]),
//   U[t] = (beta U[t-1] + (1 - beta) gate) (1 - S[t-1]),    Q[t] = p Q[t-1] + a[t-1].
// So nothing has to be kept for a reverse pass, any T_R streams through the same
// registers, and a row's T steps can be cut anywhere: each chunk starts from the V
// and a the forward saved at its first block, with W = U = Q = 0, and also sums
//   CB = sum src pv,  CA = sum lt pa,  pv = prod beta (1 - S),  pa = p^steps,
// the weights its sums have on the W, U and Q that reach it; k_join_chunks joins the
// chunks in time order. A chunk keeps ten doubles a neuron: whether it holds a reset
// (pv = 0, else beta^steps) is the sign of U, which is never negative. Spike steps come from the saved carries, as in the block
// backward; the state between them is recomputed here.
//
// Everything but the surrogate is FP64: on this machine an FP64 multiply-add issues at
// the rate of an FP32 one (no packed FP32 here), and per-step FP32 decays over a chunk
// would lose what a block's rounded powers keep.
//
// What bounds it: HBM. A quiet step is 26 vector instructions and no barrier or LDS (the
// block backward issues 51 and stitches segments behind a barrier a block, on one
// wave-group per 64 neurons whatever T is). Against that kernel, us a call with the join
// and the batch sum: 64 x 256 x 20000, T_R 40: 605 -> 520 (5.0 TB/s; 550 right after a
// forward, when the clock is lower); 4 x 2048 x 20000, T_R 20: 888 -> 272 (4.8 TB/s); 8 x 600 x
// 10000, T_R 100: 606 -> 124; 16 x 256 x 2000, T_R 2: 349 -> 44. Short calls are bound by a chunk's
// latency, some 0.17 us a step: over 500 calls of 250 to 8000 steps none measured slower.
#include "../../include/blockalif.h"
#include "alif_common.h"
#include "alif_kernels.h"

namespace alif {
namespace {

constexpr int ST_WAVES = 4;   // waves (work items) a workgroup
constexpr int ST_FAR = 1 << 30;
constexpr int ST_SIMDS = 1024;   // 256 CUs
constexpr int ST_MOST = 4;       // waves a SIMD that the chunks aim at, at most
constexpr int ST_MIN_STEPS = 24;   // a chunk's set-up (five exponentials, a first load) is worth about 16 steps
constexpr int ST_MAX_CHUNKS = 64;  // the join walks an eighth of them in sequence, 1.4 us each
constexpr int ST_RING = 2;         // groups of steps in registers; 3 measured the same

// KS: steps loaded and processed together; TRS: T_R where a group of KS steps holds
// whole blocks of TRS steps, 0: a block of T_R >= KS steps in ceil(T_R / KS) groups,
// the last one partial.
// GI: each step's src goes into the input-current gradient, for k_gi_reverse.
template <int KS, int TRS, bool GVT, bool GI, int SG>
__global__ __launch_bounds__(64 * ST_WAVES) void k_bwd_stream(BwdArgs a) {
    constexpr int M = TRS > 0 ? KS / TRS : 1;   // blocks a group
    constexpr int RING = ST_RING;               // groups in registers
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int item = xcd_remap(blockIdx.x, gridDim.x) * ST_WAVES + wave;
    // neuron groups fastest: a workgroup's waves read neighbouring columns of the same rows
    const int bc = item / a.n_groups, g = item - bc * a.n_groups;
    const int b = bc / a.chunks, ch = bc - b * a.chunks;
    if (b >= a.B) return;   // no barrier in this kernel
    const int N = a.N, TR = TRS > 0 ? TRS : a.TR;
    const int n = g * 64 + lane, nc = min(n, N - 1);
    const int blk0 = ch * a.nbc, blk1 = min(a.NB, blk0 + a.nbc);
    const int tbeg = blk0 * TR, tend = min(a.T, blk1 * TR);

    const double dt = a.dt, tm = a.tau_m[nc], ta = a.tau_a[nc];
    const double beta = exp(-dt / tm), omb = -expm1(-dt / tm), p = exp(-dt / ta);
    const double dd = a.d[nc], th0 = a.theta0[nc], bias = a.bias_k ? a.bias_k[nc] : 0.0;
    const double ob = omb * bias;

    const size_t TN = (size_t)a.T * N, CN = (size_t)(a.NB + 1) * N;
    // an absent gradient reads the input's rows instead and is zeroed at its use (without
    // dL/dV, dL/dtheta and dL/dI, an absent dL/dS leaves nothing to do)
    const float *I = a.I + b * TN;
    const bool hasS = a.gS != nullptr, hasV = GVT && a.gV != nullptr, hasT = GVT && a.gTH != nullptr;
    const float *gS = hasS ? a.gS + b * TN : I, *gV = hasV ? a.gV + b * TN : I, *gT = hasT ? a.gTH + b * TN : I;
    const uint8_t *cts = a.ck.ts + b * CN;

    double V = a.ck.v[b * CN + (size_t)blk0 * N + nc], av = a.ck.a[b * CN + (size_t)blk0 * N + nc];
    const int ts_in = min((int)cts[(size_t)blk0 * N + nc], TR);
    int tl = ts_in > 0 ? (blk0 - 1) * TR + ts_in - 1 : -ST_FAR;   // last spike before the step
    double W = 0.0, U = 0.0, Q = 0.0, pv = 1.0, pa = 1.0;
    double sb = 0.0, sbias = 0.0, sp = 0.0, sd = 0.0, sth = 0.0, CB = 0.0, CA = 0.0;

    struct Slot {
        float x[KS], gs[KS], gv[GVT ? KS : 1], gt[GVT ? KS : 1];
        int ts[M];
    };
    // group q of the chunk: blocks [blk, blk + M), steps from t (all uniform)
    const int gpb = TRS > 0 ? 1 : (TR + KS - 1) / KS;
    const int groups = !GVT && !GI && !hasS ? 0 : TRS > 0 ? (blk1 - blk0 + M - 1) / M : (blk1 - blk0) * gpb;
    struct Pos {
        int blk, j;
    };
    auto step0 = [&](Pos q) { return TRS > 0 ? q.blk * TR : q.blk * TR + q.j * KS; };
    auto next = [&](Pos q) {
        if constexpr (TRS > 0) return Pos{q.blk + M, 0};
        else return q.j + 1 < gpb ? Pos{q.blk, q.j + 1} : Pos{q.blk + 1, 0};
    };
    // rows past the chunk's end are read from its last row (and not used)
    // Every access is in range (rows and lanes are clamped), so the row goes into the
    // scalar offset, which the buffer's range check leaves out.
    const uint32_t n4 = (uint32_t)nc * 4u;
    const rsrc_t rI = make_rsrc(I, (uint32_t)(TN * 4)), rS = make_rsrc(gS, (uint32_t)(TN * 4));
    const rsrc_t rV = make_rsrc(gV, (uint32_t)(TN * 4)), rT = make_rsrc(gT, (uint32_t)(TN * 4));
    const rsrc_t rC = make_rsrc(cts, (uint32_t)CN);
    const rsrc_t rG = make_rsrc(GI ? a.gI + b * TN : nullptr, GI ? (uint32_t)(TN * 4) : 0u);
    const uint32_t g4 = n < N ? n4 : ALIF_OOB;   // (a store out of range is dropped)
    auto ldf = [&](rsrc_t r, uint32_t row) __attribute__((always_inline)) {
        return __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, n4, row, 0));
    };
    auto load = [&](Slot &s, Pos q) __attribute__((always_inline)) {
        const int t = step0(q);
#pragma unroll
        for (int k = 0; k < KS; k++) {
            const uint32_t r = (uint32_t)(min(t + k, tend - 1) * N) * 4u;
            s.x[k] = ldf(rI, r);
            s.gs[k] = ldf(rS, r);
            if constexpr (GVT) {
                s.gv[k] = ldf(rV, r);
                s.gt[k] = ldf(rT, r);
            }
        }
#pragma unroll
        for (int m = 0; m < M; m++) s.ts[m] = __builtin_amdgcn_raw_buffer_load_b8(rC, nc, (min(q.blk + m, blk1 - 1) + 1) * N, 0);
    };

    // the local terms of step t0 + k, once V, a and the sensitivities are its own
    // (a masked step's U is zero; its source may be infinite)
    auto collect = [&](const Slot &s, int k, int t0, bool gate) __attribute__((always_inline)) {
        const double u = V - fma(dd, av, th0);
        const float gs = (!GVT && !GI) || hasS ? s.gs[k] : 0.0f;
        const double q = (double)(gs * surrogate_grad<SG>((float)u, a.slope));
        double src = q, lt = -q;
        if constexpr (GVT) {
            src = hasV ? (double)s.gv[k] + q : q;
            lt = hasT ? (double)s.gt[k] - q : -q;
        }
        sb = fma(src, W, sb);
        sbias = gate ? fma(src, U, sbias) : sbias;
        sp = fma(lt, Q, sp);
        sd = fma(lt, av, sd);
        sth += lt;
        CB = fma(src, pv, CB);
        CA = fma(lt, pa, CA);
        if constexpr (GI)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint((float)src), rG, g4, (uint32_t)((t0 + k) * N) * 4u, 0);
    };
    auto group = [&](Slot &s, Pos q) __attribute__((always_inline)) {
        const int t0 = step0(q);
        int nv = min(KS, tend - t0);
        if constexpr (TRS == 0) nv = min(nv, TR - q.j * KS);
        int tc[M];   // this block's spike step, ST_FAR if none
        bool act = t0 - tl < TR;
#pragma unroll
        for (int m = 0; m < M; m++) {
            tc[m] = s.ts[m] > 0 ? (q.blk + m) * TR + min(s.ts[m], TR) - 1 : ST_FAR;
            act |= tc[m] < t0 + KS - 1;
        }
        if (nv == KS && !__any(act)) {   // no lane has a reset, a mask or a jump in this group
#pragma unroll
            for (int k = 0; k < KS; k++) {
                const double x = s.x[k];
                W = fma(beta, W, V - (x + bias));
                V = fma(beta, V, fma(omb, x, ob));
                U = fma(beta, U, omb);
                Q = fma(p, Q, av);
                av *= p;
                pv *= beta;
                pa *= p;
                collect(s, k, t0, true);
            }
        } else {
#pragma unroll
            for (int k = 0; k < KS; k++)
                if (k < nv) {   // uniform
                    const int t = t0 + k, c = tc[TRS > 0 ? k / (TRS > 0 ? TRS : 1) : 0];
                    // a spike of the block before counts at this block's first step
                    if (TRS > 0 && k % (TRS > 0 ? TRS : 1) == 0 && k > 0) {
                        const int cp = tc[k / (TRS > 0 ? TRS : 1) - 1];
                        tl = cp < ST_FAR ? cp : tl;
                    }
                    tl = t - 1 == c ? c : tl;
                    const bool spv = t - 1 == tl, gate = t - tl >= TR;
                    const double x = gate ? (double)s.x[k] + bias : 0.0;
                    const double Wn = fma(beta, W, V - x), Vn = fma(beta, V, omb * x);
                    W = spv ? 0.0 : Wn;
                    // (the carry has the reset of a spike before the chunk; an initial state may hold any V)
                    V = spv && (k > 0 || t0 != tbeg) ? 0.0 : Vn;
                    U = gate ? fma(beta, U, omb) : 0.0;   // (zero from the reset to the gate's opening)
                    pv = spv ? 0.0 : pv * beta;
                    Q = fma(p, Q, av);
                    av = fma(p, av, spv ? 1.0 : 0.0);
                    pa *= p;
                    collect(s, k, t0, gate);
                }
        }
        const int cl = tc[M - 1];
        if constexpr (M > 1) {   // (blocks past the chunk's end repeat its last one)
#pragma unroll
            for (int m = 0; m < M; m++) tl = tc[m] < t0 + KS ? tc[m] : tl;
        } else {
            tl = cl < t0 + KS ? cl : tl;
        }
    };

    Slot ring[RING];
    Pos ql{blk0, 0}, qc{blk0, 0};
#pragma unroll
    for (int i = 0; i < RING - 1; i++) {
        load(ring[i], ql);
        ql = next(ql);
    }
    int r = 0;
    for (; r + RING <= groups; r += RING) {
#pragma unroll
        for (int i = 0; i < RING; i++) {
            load(ring[(i + RING - 1) % RING], ql);
            ql = next(ql);
            group(ring[i], qc);
            qc = next(qc);
        }
    }
#pragma unroll
    for (int i = 0; i < RING; i++)
        if (r + i < groups) {   // uniform; at most RING - 1 groups, all loaded
            group(ring[i], qc);
            qc = next(qc);
        }

    if (n < N) {
        const size_t BN = (size_t)a.B * N, S = a.chunks * BN;
        double *o = a.part + (size_t)ch * BN + (size_t)b * N + n;
        o[0] = sb;
        o[S] = dd * sp;
        o[2 * S] = sd;
        o[3 * S] = sth;
        o[4 * S] = sbias;
        if (a.chunks > 1) {
            o[5 * S] = CB;
            o[6 * S] = dd * CA;
            o[7 * S] = W;
            o[8 * S] = pv == 0.0 ? -U : U;
            o[9 * S] = Q;
        }
    }
}

// The chunks' sums of one (b, n) joined in time order: the W, U and Q that reach a chunk
// are those of the chunks before it, decayed by its pv and pa. Two neighbouring chunks
// make one of the same form (Part::then), so JG threads compose a share of the chunks each
// and one adds the shares up through LDS: the 64 chunks of a single row take 8 loads in
// sequence instead of 64. The joined sums go over the first chunks' (a column's are read
// and written by one workgroup). k_finalize then sums over the batch.
constexpr int JG = 8;

struct Part {
    double b, p, d, th, bias, CB, CA, pv, pa, W, U, Q;
    // this chunk followed by x
    __device__ __forceinline__ void then(const Part &x) {
        b += fma(x.CB, W, x.b);
        p += fma(x.CA, Q, x.p);
        d += x.d;
        th += x.th;
        bias += U != 0.0 ? fma(x.CB, U, x.bias) : x.bias;   // (x.CB may be infinite)
        CB = fma(x.CB, pv, CB);
        CA = fma(x.CA, pa, CA);
        W = fma(x.pv, W, x.W);
        U = fma(x.pv, U, x.U);
        Q = fma(x.pa, Q, x.Q);
        pv *= x.pv;
        pa *= x.pa;
    }
};

// Composes the chunks [c0, c1) of column i ([10][chunks][B][N] in a.part).
__device__ __forceinline__ Part compose(const BwdArgs &a, size_t i, int c0, int c1) {
    Part t{0, 0, 0, 0, 0, 0, 0, 1, 1, 0, 0, 0};   // no step
    const size_t BN = (size_t)a.B * a.N, S = (size_t)a.chunks * BN;
    const int n = (int)(i % a.N), steps = a.nbc * a.TR;
    const double lb = -a.dt / (double)a.tau_m[n], lp = -a.dt / (double)a.tau_a[n];
    const double pv = exp(lb * steps), pa = exp(lp * steps);   // over a whole chunk without a reset
    const double last = (double)(a.T - (a.chunks - 1) * steps), pvl = exp(lb * last), pal = exp(lp * last);
#pragma unroll 2
    for (int c = c0; c < c1; c++) {
        const double *q = a.part + (size_t)c * BN + i;
        const double u = q[8 * S];
        const bool end = c == a.chunks - 1;
        t.then(Part{q[0], q[S], q[2 * S], q[3 * S], q[4 * S], q[5 * S], q[6 * S],
                    signbit(u) ? 0.0 : end ? pvl : pv, end ? pal : pa, q[7 * S], fabs(u), q[9 * S]});
    }
    return t;
}
template <int W>
__device__ __forceinline__ void put_part(double *o, const Part &t) {
    o[0] = t.b; o[W] = t.p; o[2 * W] = t.d; o[3 * W] = t.th; o[4 * W] = t.bias; o[5 * W] = t.CB;
    o[6 * W] = t.CA; o[7 * W] = t.pv; o[8 * W] = t.pa; o[9 * W] = t.W; o[10 * W] = t.U; o[11 * W] = t.Q;
}
template <int W>
__device__ __forceinline__ Part get_part(const double *q) {
    return Part{q[0], q[W], q[2 * W], q[3 * W], q[4 * W], q[5 * W], q[6 * W], q[7 * W], q[8 * W], q[9 * W], q[10 * W], q[11 * W]};
}

__global__ __launch_bounds__(64 * JG) void k_join_chunks(BwdArgs a) {
    __shared__ double sh[JG][12][64];
    const int l = threadIdx.x & 63, g = threadIdx.x >> 6;
    const size_t BN = (size_t)a.B * a.N, i = (size_t)blockIdx.x * 64 + l;
    const int per = (a.chunks + JG - 1) / JG;
    Part t{0, 0, 0, 0, 0, 0, 0, 1, 1, 0, 0, 0};
    if (i < BN) t = compose(a, i, g * per, min(a.chunks, (g + 1) * per));
    put_part<64>(&sh[g][0][l], t);
    __syncthreads();
    if (g != 0 || i >= BN) return;
    for (int h = 1; h < JG; h++) t.then(get_part<64>(&sh[h][0][l]));
    double *out = a.part + i;
    out[0] = t.b;
    out[BN] = t.p;
    out[2 * BN] = t.d;
    out[3 * BN] = t.th;
    out[4 * BN] = t.bias;
}

// Few sums: the join and k_finalize in one launch, 32 neurons a workgroup on JP threads each,
// which share out the batch elements and, below JP of those, an element's chunks.
constexpr int JP = 16, JC = 32;

__host__ __device__ constexpr int join_shares(int B) {   // threads an element
    int s = 1;
    while (2 * s * B <= JP) s *= 2;
    return s;
}

__global__ __launch_bounds__(JP * JC) void k_join_finalize(BwdArgs a, FinalizeArgs f) {
    __shared__ double sh[JP][12][JC];
    const int l = threadIdx.x % JC, ph = threadIdx.x / JC, n = blockIdx.x * JC + l;
    const int S = join_shares(a.B), share = ph % S, per = (a.chunks + S - 1) / S;
    double s[5] = {0, 0, 0, 0, 0};
    if (n < a.N)
        for (int b = ph / S; b < a.B; b += JP / S) {   // (S > 1: one element at most)
            const Part t = compose(a, (size_t)b * a.N + n, share * per, min(a.chunks, (share + 1) * per));
            if (S > 1) put_part<JC>(&sh[ph][0][l], t);
            s[0] += t.b; s[1] += t.p; s[2] += t.d; s[3] += t.th; s[4] += t.bias;
        }
    if (S > 1) {   // uniform
        __syncthreads();
        if (share == 0 && ph / S < a.B && n < a.N) {
            Part t = get_part<JC>(&sh[ph][0][l]);
            for (int h = 1; h < S; h++) t.then(get_part<JC>(&sh[ph + h][0][l]));
            s[0] = t.b; s[1] = t.p; s[2] = t.d; s[3] = t.th; s[4] = t.bias;
        }
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < 5; q++) sh[ph][q][l] = s[q];
    __syncthreads();
    if (ph != 0 || n >= a.N) return;
#pragma unroll
    for (int q = 0; q < 5; q++) {
        double t = 0.0;
        for (int k = 0; k < JP; k += S) t += sh[k][q][l];
        s[q] = t;
    }
    finalize_neuron(f, n, s);
}

// The input-current gradient from the src a forward pass left in its place: the adjoint
// of the membrane, backward in time over the same chunks,
//   lam[t] = src[t] + nu[t+1],  nu[t] = beta (1 - S[t-1]) lam[t],  gI[t] = (1 - beta) gate[t] lam[t],
// with the nu that reaches a chunk composed from the CB and pv of the chunks behind it
// (those between it and the last are whole).
// Six vector instructions a step, in FP64 but for src (the FP32 value the block backward
// sums) and gI. What bounds it: HBM, a read and a write a step.
template <int KS, int TRS>
__global__ __launch_bounds__(64 * ST_WAVES) void k_gi_reverse(BwdArgs a) {
    constexpr int M = TRS > 0 ? KS / TRS : 1;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int item = xcd_remap(blockIdx.x, gridDim.x) * ST_WAVES + wave;
    const int bc = item / a.n_groups, g = item - bc * a.n_groups;
    const int b = bc / a.chunks, ch = bc - b * a.chunks;
    if (b >= a.B) return;   // no barrier in this kernel
    const int N = a.N, TR = TRS > 0 ? TRS : a.TR;
    const int n = g * 64 + lane, nc = min(n, N - 1);
    const int blk0 = ch * a.nbc, blk1 = min(a.NB, blk0 + a.nbc);
    const int tbeg = blk0 * TR, tend = min(a.T, blk1 * TR);

    const double dt = a.dt, tm = a.tau_m[nc];
    const double beta = exp(-dt / tm), omb = -expm1(-dt / tm);
    const size_t BN = (size_t)a.B * N, S = a.chunks * BN, TN = (size_t)a.T * N, CN = (size_t)(a.NB + 1) * N;
    double nu = 0.0;
    if (ch < a.chunks - 1) {   // uniform
        const double *q = a.part + (size_t)b * N + nc;
        const double pv = exp(-dt / tm * (double)(a.nbc * TR));
        nu = q[5 * S + (a.chunks - 1) * BN];
#pragma unroll 4
        for (int c = a.chunks - 2; c > ch; c--)
            nu = fma(signbit(q[8 * S + c * BN]) ? 0.0 : pv, nu, q[5 * S + c * BN]);
    }

    struct Slot {
        float x[KS];
        int ts[M + 1];   // spike steps of the block before the group's first, then the group's
    };
    const int gpb = TRS > 0 ? 1 : (TR + KS - 1) / KS;
    const int groups = TRS > 0 ? (blk1 - blk0 + M - 1) / M : (blk1 - blk0) * gpb;
    struct Pos {
        int blk, j;
    };
    auto step0 = [&](Pos q) { return TRS > 0 ? q.blk * TR : q.blk * TR + q.j * KS; };
    auto next = [&](Pos q) {   // (before the chunk's first block: loaded from that block, not used)
        if constexpr (TRS > 0) return Pos{q.blk - M, 0};
        else return q.j > 0 ? Pos{q.blk, q.j - 1} : Pos{q.blk - 1, gpb - 1};
    };
    const uint32_t n4 = (uint32_t)nc * 4u, g4 = n < N ? n4 : ALIF_OOB;
    const rsrc_t rG = make_rsrc(a.gI + b * TN, (uint32_t)(TN * 4)), rC = make_rsrc(a.ck.ts + b * CN, (uint32_t)CN);
    auto load = [&](Slot &s, Pos q) __attribute__((always_inline)) {
        const int t = step0(q);
#pragma unroll
        for (int k = 0; k < KS; k++)
            s.x[k] = __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b32(
                rG, n4, (uint32_t)(max(min(t + k, tend - 1), tbeg) * N) * 4u, 0));
#pragma unroll
        for (int m = 0; m <= M; m++)
            s.ts[m] = __builtin_amdgcn_raw_buffer_load_b8(rC, nc, max(min(q.blk + m, blk1), blk0) * N, 0);
    };
    auto group = [&](const Slot &s, Pos q) __attribute__((always_inline)) {
        const int t0 = step0(q);
        int nv = min(KS, tend - t0);
        if constexpr (TRS == 0) nv = min(nv, TR - q.j * KS);
        int tc[M + 1];   // spike step, ST_FAR if none; the first: -ST_FAR if none
#pragma unroll
        for (int m = 0; m <= M; m++)
            tc[m] = s.ts[m] > 0 ? (q.blk + m - 1) * TR + min(s.ts[m], TR) - 1 : (m ? ST_FAR : -ST_FAR);
        bool act = t0 - tc[0] < TR;
#pragma unroll
        for (int m = 1; m <= M; m++) act |= tc[m] < t0 + KS - 1;
        auto put = [&](int k, double v) __attribute__((always_inline)) {
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint((float)v), rG, g4, (uint32_t)((t0 + k) * N) * 4u, 0);
        };
        if (nv == KS && !__any(act)) {   // no lane has a reset or a mask in this group
#pragma unroll
            for (int k = KS - 1; k >= 0; k--) {
                const double lam = (double)s.x[k] + nu;
                nu = beta * lam;
                put(k, omb * lam);
            }
        } else {
#pragma unroll
            for (int k = KS - 1; k >= 0; k--)
                if (k < nv) {   // uniform
                    constexpr int W = TRS > 0 ? TRS : KS;
                    const int t = t0 + k, c = tc[k / W + 1];
                    int cp = tc[k / W];   // the block before's
                    cp = cp == ST_FAR ? -ST_FAR : cp;
                    const bool spv = t - 1 == c || t - 1 == cp, gate = t <= c && t - cp >= TR;
                    const double lam = (double)s.x[k] + nu;
                    nu = (spv ? 0.0 : beta) * lam;
                    put(k, gate ? omb * lam : 0.0);
                }
        }
    };

    Slot ring[ST_RING];
    Pos ql = TRS > 0 ? Pos{blk0 + (groups - 1) * M, 0} : Pos{blk1 - 1, gpb - 1}, qc = ql;
#pragma unroll
    for (int i = 0; i < ST_RING - 1; i++) {
        load(ring[i], ql);
        ql = next(ql);
    }
    int r = 0;
    for (; r + ST_RING <= groups; r += ST_RING) {
#pragma unroll
        for (int i = 0; i < ST_RING; i++) {
            load(ring[(i + ST_RING - 1) % ST_RING], ql);
            ql = next(ql);
            group(ring[i], qc);
            qc = next(qc);
        }
    }
#pragma unroll
    for (int i = 0; i < ST_RING; i++)
        if (r + i < groups) {   // uniform; at most ST_RING - 1 groups, all loaded
            group(ring[i], qc);
            qc = next(qc);
        }
}

template <int KS, int TRS>
void stream_launch(const BwdArgs &a, unsigned grid, hipStream_t st) {
    const dim3 blk(64 * ST_WAVES);
    const bool gvt = a.gV || a.gTH, gi = a.gI != nullptr;
#define ALIF_ST(SG)                                                                                          \
    do {                                                                                                     \
        if (gvt && gi) hipLaunchKernelGGL((k_bwd_stream<KS, TRS, true, true, SG>), dim3(grid), blk, 0, st, a); \
        else if (gvt) hipLaunchKernelGGL((k_bwd_stream<KS, TRS, true, false, SG>), dim3(grid), blk, 0, st, a); \
        else if (gi) hipLaunchKernelGGL((k_bwd_stream<KS, TRS, false, true, SG>), dim3(grid), blk, 0, st, a); \
        else hipLaunchKernelGGL((k_bwd_stream<KS, TRS, false, false, SG>), dim3(grid), blk, 0, st, a);       \
    } while (0)
    if (a.surrogate == 1) ALIF_ST(1);
    else if (a.surrogate == 2) ALIF_ST(2);
    else ALIF_ST(0);
#undef ALIF_ST
    if (gi) hipLaunchKernelGGL((k_gi_reverse<KS, TRS>), dim3(grid), blk, 0, st, a);
}

}  // namespace

size_t bwd_stream_bytes(int B, int N, int chunks) {
    return (size_t)(chunks > 1 ? 10 * chunks : 5) * B * N * sizeof(double);
}

// The SIMDs work through waves of equal length, so a row cut into c chunks takes as long as the
// SIMD with the most of them: ceil(c waves / 1024) times a chunk's steps and set-up, somewhat
// more where one or two waves leave a SIMD's latency open. The least of that over the counts
// that give a SIMD at most four waves, a chunk a block and 24 steps, and whose sums fit
// the static scratch (whichever scratch a call has, so the bits do not depend on it). us, with
// the join: 64 x 256 x 20000 at T_R 40 by chunks 6 / 8 / 9 / 12 / 13 / 16 / 24: 565 / 525 / 591 /
// 518 / 587 / 546 / 541; 19 x 773 x 13195, T_R 64, 8 / 9 / 12 / 13 / 16: 339 / 406 / 356 / 395 / 348;
// 119 x 77 x 2008, T_R 120 (17 blocks), 9 / 17: 78 / 57.
int bwd_stream_chunks(int B, int T, int N, int TR) {
    const long long waves = (long long)B * ((N + 63) / 64);
    if (waves == 0 || T == 0) return 1;
    const int NB = (T + TR - 1) / TR;
    long long most = (T + ST_MIN_STEPS - 1) / ST_MIN_STEPS;
    most = most < NB ? most : NB;
    most = most < ST_MAX_CHUNKS ? most : ST_MAX_CHUNKS;
    const long long fit = (long long)ALIF_NOALLOC_SCRATCH_BYTES / (long long)(bwd_stream_bytes(B, N, 2) / 2);
    most = most < fit ? most : fit;
    int best = 1;
    double least = 0.0;
    for (int c = 1; c <= most; c++) {
        const int nbc = (NB + c - 1) / c;
        if (c > 1 && ((NB + nbc - 1) / nbc != c || c * waves > (long long)ST_MOST * ST_SIMDS)) continue;
        const long long deep = (c * waves + ST_SIMDS - 1) / ST_SIMDS;
        const double cost = (double)deep * ((double)nbc * TR + 16.0) * (deep == 1 ? 1.3 : deep == 2 ? 1.07 : 1.0);
        if (c == 1 || cost < least) {
            best = c;
            least = cost;
        }
    }
    return best;
}

// Whether a backward that wants dL/dI streams. The block backward runs a row's blocks in
// sequence, 64 to 256 neurons a workgroup, so a call that does not fill the card takes its
// blocks times c(T_R) us; else it moves 12 bytes a step. Streaming takes its set-up, launches
// and join, 0.3 us a step of a chunk in both directions, 0.2 us a chunk composed on the way
// back, and moves 20 bytes a step (the source written and read). Over 500 calls (T_R 2 to 128, 1 to
// 128 rows of 250 to 8000 steps, 20 to 1024 neurons) it never took the slower one. us, block /
// streaming: T_R 2: 32 x 1000 x 512 209 / 80, 64 x 1000 x 512 221 / 149, 64 x 1000 x 1024 247 / 293;
// T_R 10: 64 x 4000 x 256 339 / 294, 64 x 1000 x 512 125 / 153; T_R 40: 16 x 20000 x 128 574 / 199,
// 32 x 1000 x 512 56 / 88; T_R 64: 11 x 1149 x 45 50 / 54 with the chunks of 128 steps this took before.
// A segment of more than eight steps that the block ends inside (and 16 with dL/dV or dL/dtheta)
// does not fit the block kernel's registers, where streaming wins from four blocks on: T_R 50:
// 129 / 67 (8 x 1000 x 1024), 706 / 299 (64 x 1000 x 1024); T_R 100: 1334 / 551 (128 x 1000 x 1024), but 43 / 45
// (70 x 287 x 28, three blocks).
bool bwd_stream_gi(int B, int T, int N, int TR, bool gvt) {
    const BlockConfig c = block_config(TR);
    const int NB = (T + TR - 1) / TR;
    if (NB > 3 && c.seg == 8 && ((c.len >= 8 && TR != c.seg * c.len) || (gvt && c.len == 16))) return true;
    const double steps = (double)B * T * N * 1e-6;
    const double serial = 10.0 + NB * (c.seg == 1 ? 0.26 + 0.05 * TR : 0.6 + 0.02 * TR);
    const int chunks = bwd_stream_chunks(B, T, N, TR);
    const double L = (double)((NB + chunks - 1) / chunks) * TR;
    const double moved = 2.9 * steps * (gvt ? 20.0 / 12 : 1.0);
    const double stream = 14.0 + 0.3 * L + 0.2 * chunks + 4.2 * steps * (gvt ? 28.0 / 20 : 1.0);
    return stream < (serial > moved ? serial : moved);
}

hipError_t launch_bwd_stream(BwdArgs a, const FinalizeArgs &f, hipStream_t st) {
    a.nbc = (a.NB + a.chunks - 1) / a.chunks;
    a.n_groups = (a.N + 63) / 64;
    const long long items = (long long)a.B * a.chunks * a.n_groups;
    if (items == 0) return launch_finalize(f, st);
    const unsigned grid = (unsigned)((items + ST_WAVES - 1) / ST_WAVES);
    if (a.TR == 2) stream_launch<8, 2>(a, grid, st);
    else if (a.TR == 3) stream_launch<6, 3>(a, grid, st);
    else if (a.TR == 4) stream_launch<8, 4>(a, grid, st);
    else {   // the fewest steps lost to the last group, then the longer group
        int ks = 8, lost = (a.TR + 7) / 8 * 8 - a.TR;
        for (int k = 7; k >= 5; k--) {
            const int l = (a.TR + k - 1) / k * k - a.TR;
            if (l < lost) { ks = k; lost = l; }
        }
        if (ks == 8) stream_launch<8, 0>(a, grid, st);
        else if (ks == 7) stream_launch<7, 0>(a, grid, st);
        else if (ks == 6) stream_launch<6, 0>(a, grid, st);
        else stream_launch<5, 0>(a, grid, st);
    }
    // us a call, join and k_finalize / one launch: 1 x 100, 8 chunks 20.4 / 19.2, 64 chunks 31.6 / 23.8;
    // 2 x 1024, 8 chunks 21.1 / 20.2; 4 x 100, 16 chunks 23.2 / 23.2; 8 x 100, 16 chunks 23.7 / 26.3
    // (fewer threads an element). A launch less for the host, too.
    if (a.chunks > 1 && a.B <= 4) {
        hipLaunchKernelGGL(k_join_finalize, dim3((unsigned)((a.N + JC - 1) / JC)), dim3(JP * JC), 0, st, a, f);
        return hipGetLastError();
    }
    if (a.chunks > 1)
        hipLaunchKernelGGL(k_join_chunks, dim3((unsigned)(((size_t)a.B * a.N + 63) / 64)), dim3(64 * JG), 0, st, a);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? launch_finalize(f, st) : e;
}

}  // namespace alif
