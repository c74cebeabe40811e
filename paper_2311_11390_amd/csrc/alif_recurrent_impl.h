// Recurrent ALIF layer: Eq. 3 with the recurrent current W_rec S[t - D] (D >= T_R,
// so a block's recurrent input comes from finished blocks only; Prop. 3 keeps one
// spike per neuron per block), for layers whose whole state fits one workgroup.
//
// One workgroup per batch element holds the whole layer: NG groups of 64
// neurons (lane = neuron) x SEG segment-waves, exactly the per-block arithmetic
// of the block forward (seg_scan / seg_horner / seg_membrane, the same FP64
// carry), so only the segmentation of a block can differ from the per-block
// launches. The blocks of the layer run one after another inside the kernel and
// meet at the workgroup barriers the block integrate already has:
//
//   1. x = feed-forward current of block nb (prefetched) + the recurrent sums
//      gathered at the end of block nb - 1;
//   2. scan, Horner stitch (barrier), membrane, first crossings (barrier);
//   3. every wave knows the spike step of every neuron of block nb from LDS; the
//      spikes whose target step t + D falls into block nb + 1 and into this wave's
//      segment are found with a ballot per neuron group, and for each one, in
//      increasing presynaptic index, the lane adds W_rec[i][j] (one 256-byte row of
//      W_rec^T, L2-resident) to the target step. Older source blocks (D > T_R) come
//      from a small ring of spike steps in LDS.
//
// Summation order: per target step the recurrent term is a sum in FP32 from zero
// over the active presynaptic neurons in increasing index, added once to the
// feed-forward current: the order of the per-block recurrent-current kernel.
//
// Two kernels run it. k_recurrent_fused does all of it and writes every output itself:
// for the calls that want V and theta traces, which only this loop has, and for short
// runs. Its stores cost it half of its time (a workgroup issues them for every step of
// every neuron while one block runs), so with CHUNKED (N a multiple of 16 and room in
// LDS) they go out as 16-byte chunks: the block's current through a wave-private LDS tile,
// and the spikes packed from one ballot per step. k_recurrent_slice leaves these two
// streams to other workgroups: see there.
#pragma once
#include "alif_blocks_impl.h"

namespace alif {

// LDS: pd [NWG][T_R] f64 | X [SEG][NWG] f32 | C [2][SEG][NWG] i32 | ring [R][NWG] u8
template <int SEG, int NG>
__host__ __device__ constexpr size_t rec_smem_fixed(int TR) {
    return (size_t)64 * NG * TR * sizeof(double) + (size_t)3 * SEG * 64 * NG * 4;
}

// LDS of the CHUNKED staging tile: [waves][L][64] floats after the 16-byte aligned fixed part
template <int SEG, int L, int NG>
__host__ __device__ constexpr size_t rec_stage_bytes() {
    return (size_t)NG * SEG * L * 64 * 4;
}
__host__ __device__ constexpr size_t rec_stage_offset(size_t fixed_and_ring) { return (fixed_and_ring + 15) & ~(size_t)15; }

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// Non-temporal (streamed) access for the feed-forward current read once and the
// whole current and spikes written once, so that they pass through L2 without
// evicting the W_rec^T rows the gather reads every block (about 1% of the loop).
constexpr int REC_NT = 2;
__device__ __forceinline__ float ld_f32_nt(rsrc_t r, uint32_t byte_off) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, byte_off, 0, REC_NT));
}

template <int SEG, int L, bool EVEN, int NG, bool TRACES, bool CHUNKED>
__global__ __launch_bounds__(64 * NG * SEG) void k_recurrent_fused(RecArgs a) {
    constexpr int NWG = 64 * NG;
    constexpr int DEPTH = 2;
    constexpr int EV = 4;
    extern __shared__ __align__(16) unsigned char smem[];
    const int TR = a.TR, N = a.N, T = a.T, D = a.D, R = a.ring;
    double *pd_tab = reinterpret_cast<double *>(smem);
    float *exX = reinterpret_cast<float *>(smem + (size_t)NWG * TR * sizeof(double));
    int *exC = reinterpret_cast<int *>(exX + SEG * NWG);
    uint8_t *ring = reinterpret_cast<uint8_t *>(exC + 2 * SEG * NWG);
    // this wave's staging tile [L][64] (CHUNKED)
    float *stg = reinterpret_cast<float *>(
                     smem + rec_stage_offset(rec_smem_fixed<SEG, NG>(TR) + (size_t)R * NWG)) +
                 (size_t)(threadIdx.x >> 6) * L * 64;

    const int b = blockIdx.x;
    build_p_tables<SEG, L, NWG>(pd_tab, nullptr, 0, N, TR, a.dt, a.tau_a);
    Lane<SEG, L, EVEN> c;
    lane_setup<SEG, L, EVEN, NG>(c, N, TR, a.dt, 0, a.tau_m, a.tau_a, a.d, a.theta0, a.bias_k);
    if (c.valid && c.w == 0 && !params_ok(a.tau_m[c.n], a.tau_a[c.n], c.dd, c.th0))
        atomicOr(a.status, 1u);
    const int pdrow = c.nl * TR;
    const int lane = threadIdx.x & 63;

    const size_t TN = (size_t)T * N;
    const int SB = spike_bytes(a.spike_dtype);
    const rsrc_t rIn = make_rsrc(a.I_ff + b * TN, (uint32_t)(TN * 4));
    const rsrc_t rI = make_rsrc(a.I + b * TN, (uint32_t)(TN * 4));
    const rsrc_t rS = make_rsrc((char *)a.spikes + b * TN * SB, (uint32_t)(TN * SB));
    const rsrc_t rV = make_rsrc(a.V ? a.V + b * TN : nullptr, a.V ? (uint32_t)(TN * 4) : 0u);
    const rsrc_t rT = make_rsrc(a.TH ? a.TH + b * TN : nullptr, a.TH ? (uint32_t)(TN * 4) : 0u);
    const rsrc_t rW = make_rsrc(a.WrecT, (uint32_t)((size_t)N * N * 4));
    const size_t CN = (size_t)(a.NB + 1) * N;
    const bool ck = a.ck.v != nullptr;
    const rsrc_t rCv = make_rsrc(ck ? a.ck.v + b * CN : nullptr, ck ? (uint32_t)(CN * 4) : 0u);
    const rsrc_t rCa = make_rsrc(ck ? a.ck.a + b * CN : nullptr, ck ? (uint32_t)(CN * 4) : 0u);
    const rsrc_t rCt = make_rsrc(ck ? a.ck.ts + b * CN : nullptr, ck ? (uint32_t)CN : 0u);
    const uint32_t ck4 = (c.valid && c.w == 0) ? (uint32_t)c.n * 4u : ALIF_OOB;
    const uint32_t ck1 = (c.valid && c.w == 0) ? (uint32_t)c.n : ALIF_OOB;
    // this lane's column of W_rec^T (byte offset within a row), or out of range
    const uint32_t wcol = c.valid ? (uint32_t)c.n * 4u : ALIF_OOB;
    const uint32_t wrow = (uint32_t)N * 4u;
    const int spk_shift = SB == 1 ? 2 : (SB == 2 ? 1 : 0);

    double v0d = 0.0, a0d = 0.0;
    int cts = 0;
    const uint32_t blk4 = (uint32_t)(TR * N) * 4u;
    float buf[DEPTH][L];
#pragma unroll
    for (int i = 0; i < DEPTH; i++)
#pragma unroll
        for (int k = 0; k < L; k++) buf[i][k] = ld_f32_nt(rIn, c.off(k, (uint32_t)min((size_t)i * blk4, TN * 4)));

    // recurrent sums of the next block at this lane's steps; hit: steps with a term (wave-uniform)
    float acc[L];
#pragma unroll
    for (int k = 0; k < L; k++) acc[k] = 0.0f;
    uint32_t hit = 0;
    const int qD = (D + TR - 1) / TR;   // source blocks lie qD or qD - 1 blocks back

    // Gather the recurrent input of block nt from the spikes of blocks < nt
    // (block nt - 1 from the candidate array Cp, older ones from the ring).
    auto gather = [&](int nt, const int *Cp) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < L; k++) acc[k] = 0.0f;
        hit = 0;
        for (int q = 0; q < 2; q++) {
            const int m = nt - qD + q;   // uniform
            if (m < 0 || m >= nt || (q == 1 && D % TR == 0)) continue;
            const int base = (m - nt) * TR + D - 1;   // target offset in block nt = base + t_s
#pragma unroll
            for (int g = 0; g < NG; g++) {
                const int j = g * 64 + lane;
                int tsj;
                if (m == nt - 1) {
                    tsj = ALIF_NO_SPIKE;
#pragma unroll
                    for (int s = 0; s < SEG; s++) tsj = min(tsj, Cp[s * NWG + j]);
                    tsj = tsj <= TR ? tsj : 0;
                } else {
                    tsj = ring[(m % R) * NWG + j];
                }
                const int r = base + tsj;
                // steps past T (padding of a ragged last block) get no recurrent term
                const bool mine = tsj > 0 && j < N && r >= c.t0 && r < c.t0 + c.len && nt * TR + r < T;
                uint64_t mk = __ballot(mine);
                while (mk) {   // EV active inputs at a time: their loads are in flight together
                    int kk[EV];
                    float w[EV];
#pragma unroll
                    for (int e = 0; e < EV; e++) {
                        kk[e] = -1;
                        w[e] = 0.0f;
                        if (mk) {
                            const int l = __builtin_ctzll(mk);
                            mk &= mk - 1;
                            kk[e] = __builtin_amdgcn_readlane(r, l) - c.t0;
                            w[e] = ld_f32(rW, (uint32_t)(g * 64 + l) * wrow + wcol);
                        }
                    }
#pragma unroll
                    for (int e = 0; e < EV; e++) {
#pragma unroll
                        for (int k = 0; k < L; k++) acc[k] = k == kk[e] ? acc[k] + w[e] : acc[k];
                        hit |= kk[e] >= 0 ? 1u << kk[e] : 0u;
                    }
                }
            }
        }
    };

    auto do_block = [&](float (&bi)[L], int nb) __attribute__((always_inline)) {
        const uint32_t bo = (uint32_t)nb * blk4;
        float x[L];
#pragma unroll
        for (int k = 0; k < L; k++) {
            x[k] = (hit >> k) & 1u ? bi[k] + acc[k] : bi[k];   // uniform: a row with a recurrent term
            if constexpr (CHUNKED) stg[k * 64 + lane] = x[k];
            else st_f32(rI, c.off(k, bo), x[k]);
        }
        const float cv = (float)v0d, ca = (float)a0d;
        const int mpre = cts > 0 ? cts - 1 : 0;
        const float a1 = fmaf(c.pf, ca, cts == TR ? 1.0f : 0.0f);
        float uu[L];
        seg_scan(c, x, mpre, uu);
        float E = 0.0f, uTR;
        if constexpr (SEG > 1) {
            exX[c.w * NWG + c.nl] = uu[L - 1];
            __syncthreads();
            seg_horner<SEG, L, EVEN, NWG>(c, exX, E, uTR);
        } else {
            uTR = uu[L - 1];
        }
        float vt[L], th[L];
        const int cand = seg_membrane(c, cv, E, a1, uu, vt, th);
        int *Cp = exC + (nb & 1) * SEG * NWG;
        Cp[c.w * NWG + c.nl] = cand;
        __syncthreads();
        int ts = ALIF_NO_SPIKE;
#pragma unroll
        for (int s = 0; s < SEG; s++) ts = min(ts, Cp[s * NWG + c.nl]);
        if (nb + 1 < a.NB) gather(nb + 1, Cp);   // uniform

        // outputs of block nb (reset after t_s, Eqs. 2 and 5) and its carry-in
        {
            const uint32_t e = (uint32_t)(nb * N);
            st_f32(rCv, ck4 + e * 4u, cv);
            st_f32(rCa, ck4 + e * 4u, ca);
            st_u8(rCt, ck1 + e, (uint8_t)cts);
        }
#pragma unroll
        for (int k = 0; k < L; k++) {
            const int t = c.t0 + k + 1;
            const uint32_t o4 = c.off(k, bo);
            if constexpr (!CHUNKED) st_spike(rS, a.spike_dtype, o4 >> spk_shift | (o4 & ALIF_OOB), t == ts);
            if constexpr (TRACES) {
                const bool after = t > ts;
                st_f32(rV, o4, after ? 0.0f : vt[k]);
                // p^(t - 1 - t_s) when after (clamped into the row for the steps that are not)
                const float pa = (float)pd_tab[pdrow + min(TR - 1, max(0, t - 1 - ts))];
                st_f32(rT, o4, after ? fmaf(c.dd, pa, th[k]) : th[k]);
            }
        }
        const bool spk = ts <= TR;
        const double e1 = cts == TR ? c.pTm1 : 0.0;
        const double e2 = pd_tab[pdrow + max(0, TR - 1 - min(ts, TR))];
        const double extra = e1 + ((spk && ts < TR) ? e2 : 0.0);
        v0d = spk ? 0.0 : fma(c.betaT, v0d, (double)uTR);
        a0d = fma(c.pT, a0d, extra);
        cts = spk ? ts : 0;
        if (R > 0 && c.w == 0) ring[(nb % R) * NWG + c.nl] = (uint8_t)(spk ? ts : 0);
        if constexpr (CHUNKED) {
            const int nw0 = c.n - lane;                     // first neuron of this wave's group
            const int row0 = nb * TR + c.t0;                // first step of this wave's segment
            // spikes: a ballot per step; 16-byte chunks of NPC = 16 / SB neurons, 4 SB per step row
            uint64_t m[L];
#pragma unroll
            for (int k = 0; k < L; k++) m[k] = __ballot(c.t0 + k + 1 == ts);
            const int CPR = 4 * SB, NPC = 16 / SB;
            // a fixed number of store instructions (the f32 count; chunks past CPR L are dropped)
#pragma unroll
            for (int ci0 = 0; ci0 < 16 * L; ci0 += 64) {
                const int ci = ci0 + lane, k = ci / CPR, q = ci - k * CPR;
                uint64_t mk = 0;
#pragma unroll
                for (int kk = 0; kk < L; kk++) mk = k == kk ? m[kk] : mk;
                const uint32_t bits = (uint32_t)(mk >> (q * NPC));
                u32x4_t v;
                if (SB == 1) {   // bytes 0 / 1: spread each nibble to four bytes
                    v.x = ((bits & 15u) * 0x204081u) & 0x01010101u;
                    v.y = (((bits >> 4) & 15u) * 0x204081u) & 0x01010101u;
                    v.z = (((bits >> 8) & 15u) * 0x204081u) & 0x01010101u;
                    v.w = (((bits >> 12) & 15u) * 0x204081u) & 0x01010101u;
                } else if (SB == 2) {   // bfloat16 1.0 = 0x3F80
                    v.x = (bits & 1u ? 0x3F80u : 0u) | (bits & 2u ? 0x3F800000u : 0u);
                    v.y = (bits & 4u ? 0x3F80u : 0u) | (bits & 8u ? 0x3F800000u : 0u);
                    v.z = (bits & 16u ? 0x3F80u : 0u) | (bits & 32u ? 0x3F800000u : 0u);
                    v.w = (bits & 64u ? 0x3F80u : 0u) | (bits & 128u ? 0x3F800000u : 0u);
                } else {
                    v.x = bits & 1u ? 0x3F800000u : 0u;
                    v.y = bits & 2u ? 0x3F800000u : 0u;
                    v.z = bits & 4u ? 0x3F800000u : 0u;
                    v.w = bits & 8u ? 0x3F800000u : 0u;
                }
                const bool ok = ci < CPR * L && k < c.len && nw0 + q * NPC < N;
                const uint32_t off = ok ? (uint32_t)(((size_t)(row0 + k) * N + nw0 + q * NPC) * SB) : ALIF_OOB;
                __builtin_amdgcn_raw_buffer_store_b128(v, rS, off, 0, REC_NT);
            }
            // the whole current of the block from the staging tile: 16 chunks of 4 neurons per step row
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int ci0 = 0; ci0 < 16 * L; ci0 += 64) {
                const int ci = ci0 + lane, k = ci >> 4, q = ci & 15;
                const bool ok = ci < 16 * L && k < c.len && nw0 + 4 * q < N;
                const u32x4_t v = *reinterpret_cast<const u32x4_t *>(&stg[(ok ? k : 0) * 64 + 4 * q]);
                const uint32_t off = ok ? (uint32_t)(((size_t)(row0 + k) * N + nw0 + 4 * q) * 4) : ALIF_OOB;
                __builtin_amdgcn_raw_buffer_store_b128(v, rI, off, 0, REC_NT);
            }
            __builtin_amdgcn_wave_barrier();
        }
        const uint32_t nxt = (uint32_t)min((size_t)(nb + DEPTH) * blk4, TN * 4);
#pragma unroll
        for (int k = 0; k < L; k++) bi[k] = ld_f32_nt(rIn, c.off(k, nxt));
    };

    wait_vmem_all();
    int nb0 = 0;
    for (; nb0 + DEPTH <= a.NB; nb0 += DEPTH) {
#pragma unroll
        for (int i = 0; i < DEPTH; i++) do_block(buf[i], nb0 + i);
    }
#pragma unroll
    for (int i = 0; i < DEPTH; i++)
        if (nb0 + i < a.NB) do_block(buf[i], nb0 + i);   // uniform
    {   // the final carry
        const uint32_t e = (uint32_t)(a.NB * N);
        st_f32(rCv, ck4 + e * 4u, (float)v0d);
        st_f32(rCa, ck4 + e * 4u, (float)a0d);
        st_u8(rCt, ck1 + e, (uint8_t)cts);
    }
}

// ---------------------------------------------------------------------------
// The layer without traces, in slices of blocks.
//
// What bounds it: the chain of blocks on one CU per batch element. Of the 4.1 us a
// block took in one launch that wrote everything (64 x 256 neurons, T_R 40), half went
// into the stores of the whole current and the spikes (8 or 5 bytes a neuron-step, 92 KB
// a block from one CU) while the other CUs idled. Both follow from the feed-forward
// current and the blocks' spike steps alone. So a launch runs the chain for one slice of
// blocks (workgroups below B: one byte a neuron and block out, the spike step) and, on
// the remaining CUs, expands the slice before it: whole current = feed-forward current
// plus the gathered rows of W_rec^T, and the spike raster. The launches order the two,
// so nothing spins; V, a and the last spike step cross slices in a state buffer.
//
// The chain's block: the crossings meet in one LDS word a neuron (a minimum by the lanes
// that crossed), of three copies: block nb's is read until barrier 1 of block nb + 1 and
// reset before barrier 1 of block nb + 2. Blocks without a spike anywhere leave the
// gather after one vote, and the recurrent sums sit in LDS rows that only steps with an
// event touch. 64 x 256 x 20000, T_R 40: 2.01 -> 1.30 ms, 2.3 us a block of the chain.
// What is left is one CU's instruction issue and latency: the loop without memory
// operations takes half of a block's time, the loads of its 40 KB (640 cycles of the CU's
// L1 path) and the gather (an L2 round trip when a spike lands) a quarter each. Two and
// four segments a wave (8 and 4 waves a workgroup, a third fewer instructions) were slower,
// 1.65 and 2.2 us a block against 1.35 without memory operations: a wave issues one of
// its dependent instructions in eight cycles or more, so it takes 16 waves to keep the
// CU's four SIMDs busy. And whatever one of the 16 waves does in a block with a spike, all
// wait for: the power of p comes from a table in memory, asked for with the gather's rows
// (an FP64 exponential in its place cost 0.5 us a block). Registers are capped at 128 by
// the 16 waves, and a spill reloaded in the loop would drain the prefetch every block.
// ---------------------------------------------------------------------------
// LDS: X [SEG][NWG] f32 | ts [3][NWG] i32 | acc [SEG L][NWG] f32 | ring [R][NWG] u8 (below that of
// k_recurrent_fused, whose size decides whether a layer runs here)
template <int SEG, int L, int NG>
constexpr size_t rec_slice_smem(int R) {
    constexpr size_t nwg = (size_t)64 * NG;
    return (SEG + 3) * nwg * 4 + (size_t)SEG * L * nwg * 4 + (size_t)R * nwg;
}

// Expansion of the blocks [xb0, xb1). An item is one segment (the chain's, of L steps) of G
// neighbouring blocks, G L >= 16 rows; a wave takes items in turn, VEC neighbouring neurons a
// lane and as many rows side by side as fit 64 lanes. It streams every row through (the
// current only where it does not lie in place already), except the current of the few rows
// that events land in, which the chain has marked (hits); these follow.
template <int VEC, typename V>
__device__ __forceinline__ void rec_put(V w, V *p) {
    if constexpr (VEC == 4) __builtin_nontemporal_store(w, p);
    else *p = w;
}
template <int SEG, int L, int VEC>
__device__ __forceinline__ void rec_expand(const RecArgs &a, int wave, int waves) {
    constexpr int G = L >= 16 ? 1 : (16 + L - 1) / L, U = VEC == 4 ? 4 : 8;
    const int lane = threadIdx.x & 63;
    const int N = a.N, TR = a.TR, T = a.T, D = a.D;
    int tpr = 1;
    while (tpr < (N + VEC - 1) / VEC && tpr < 64) tpr *= 2;
    const int rpw = 64 / tpr, sub = lane / tpr, col = lane % tpr;
    const int ngrp = (a.xb1 - a.xb0 + G - 1) / G, items = a.B * ngrp * SEG;
    const bool in_place = a.I_ff == a.I;
    const size_t TN = (size_t)T * N;
    typedef float vecf __attribute__((ext_vector_type(VEC)));
    typedef uint8_t vec1 __attribute__((ext_vector_type(VEC)));
    typedef uint16_t vec2 __attribute__((ext_vector_type(VEC)));

    for (int it = wave; it < items; it += waves) {
        const int b = it / (ngrp * SEG), i0 = it - b * (ngrp * SEG);
        const int seg = i0 % SEG, blk0 = a.xb0 + i0 / SEG * G, blk1 = min(a.xb1, blk0 + G);
        const int rows = (blk1 - blk0) * L;   // row q: block blk0 + q / L, step seg L + q % L
        const uint8_t *tsb = a.ts + (size_t)b * a.NB * N;
        const uint32_t *hits = a.hits + (size_t)b * a.NB * SEG + seg;
        for (int c0 = 0; c0 < N; c0 += tpr * VEC) {
            const int n = c0 + col * VEC;   // this lane's neurons n .. n + VEC - 1 (N % VEC == 0)
            const bool okn = n < N;
#pragma unroll 1
            for (int q0 = 0; q0 < rows; q0 += rpw * U) {
                vecf x[U];
                vec1 own[U];
                uint32_t hw[U];
                int step[U];
                bool ok[U];
#pragma unroll
                for (int u = 0; u < U; u++) {
                    const int q = min(q0 + u * rpw + sub, rows - 1), nt = blk0 + q / L, k = seg * L + q % L;
                    step[u] = k;
                    ok[u] = okn && q0 + u * rpw + sub < rows && k < TR && nt * TR + k < T;
                    const size_t o = b * TN + (ok[u] ? (size_t)(nt * TR + k) * N + n : 0);
                    if (!in_place)
                        x[u] = __builtin_nontemporal_load(reinterpret_cast<const vecf *>(a.I_ff + o));
                    own[u] = *reinterpret_cast<const vec1 *>(tsb + (ok[u] ? (size_t)nt * N + n : 0));
                    hw[u] = hits[(size_t)nt * SEG];
                }
#pragma unroll
                for (int u = 0; u < U; u++) {
                    if (!ok[u]) continue;
                    const int q = q0 + u * rpw + sub, nt = blk0 + q / L, k = step[u];
                    const size_t o = b * TN + (size_t)(nt * TR + k) * N + n;
                    if (!in_place && !(hw[u] >> (k - seg * L) & 1u))
                        rec_put<VEC>(x[u], reinterpret_cast<vecf *>(a.I + o));
                    if (a.spike_dtype == 0) {
                        vec1 w;
#pragma unroll
                        for (int v = 0; v < VEC; v++) w[v] = own[u][v] == k + 1 ? 1 : 0;
                        rec_put<VEC>(w, reinterpret_cast<vec1 *>(static_cast<uint8_t *>(a.spikes) + o));
                    } else if (a.spike_dtype == 1) {
                        vec2 w;
#pragma unroll
                        for (int v = 0; v < VEC; v++) w[v] = own[u][v] == k + 1 ? 0x3F80 : 0;
                        rec_put<VEC>(w, reinterpret_cast<vec2 *>(static_cast<uint16_t *>(a.spikes) + o));
                    } else {
                        vecf w;
#pragma unroll
                        for (int v = 0; v < VEC; v++) w[v] = own[u][v] == k + 1 ? 1.0f : 0.0f;
                        rec_put<VEC>(w, reinterpret_cast<vecf *>(static_cast<float *>(a.spikes) + o));
                    }
                }
            }
        }
#pragma unroll 1
        for (int nt = blk0; nt < blk1; nt++)
#pragma unroll 1
            for (uint32_t h = __builtin_amdgcn_readfirstlane(hits[(size_t)nt * SEG]); h; h &= h - 1) {
                const int k = seg * L + __builtin_ctz(h), u = nt * TR + k - D;   // u: the source step
                const uint8_t *src = tsb + (size_t)(u / TR) * N;
                const int ts = u % TR + 1;
#pragma unroll 1
                for (int n = lane * VEC; n - lane * VEC < N; n += 64 * VEC) {
                    vecf acc{};
#pragma unroll 1
                    for (int g = 0; g < N; g += 64)
                        for (uint64_t mk = __ballot(g + lane < N && src[min(g + lane, N - 1)] == ts); mk; mk &= mk - 1)
                            if (n < N)
                                acc += *reinterpret_cast<const vecf *>(a.WrecT + (size_t)(g + __builtin_ctzll(mk)) * N + n);
                    if (n < N) {
                        const size_t o = b * TN + (size_t)(nt * TR + k) * N + n;
                        const vecf x = *reinterpret_cast<const vecf *>(a.I_ff + o);
                        *reinterpret_cast<vecf *>(a.I + o) = x + acc;
                    }
                }
            }
    }
}

template <int SEG, int L, bool EVEN, int NG>
__global__ __launch_bounds__(64 * NG * SEG) void k_recurrent_slice(RecArgs a) {
    constexpr int NWG = 64 * NG, WAVES = NG * SEG;
    constexpr int DEPTH = 2;
    if ((int)blockIdx.x >= a.core) {   // expansion of the slice before
        const int wave = ((int)blockIdx.x - a.core) * WAVES + (int)(threadIdx.x >> 6);
        const int waves = ((int)gridDim.x - a.core) * WAVES;
        const int w = __builtin_amdgcn_readfirstlane(wave);
        if (a.vec4) rec_expand<SEG, L, 4>(a, w, waves);
        else rec_expand<SEG, L, 1>(a, w, waves);
        return;
    }
    extern __shared__ __align__(16) unsigned char smem[];
    const int TR = a.TR, N = a.N, T = a.T, D = a.D, R = a.ring;
    float *exX = reinterpret_cast<float *>(smem);
    int *exT = reinterpret_cast<int *>(exX + SEG * NWG);
    float *accs = reinterpret_cast<float *>(exT + 3 * NWG);
    uint8_t *ring = reinterpret_cast<uint8_t *>(accs + (size_t)SEG * L * NWG);
    const int lane = threadIdx.x & 63;
    float *acc = accs + (size_t)(threadIdx.x >> 6) * L * 64 + lane;   // [L] rows of 64

    const int b = blockIdx.x;
    Lane<SEG, L, EVEN> c;
    lane_setup<SEG, L, EVEN, NG>(c, N, TR, a.dt, 0, a.tau_m, a.tau_a, a.d, a.theta0, a.bias_k);
    const bool first = c.w == 0;
    if (a.nb0 == 0 && c.valid && first && !params_ok(a.tau_m[c.n], a.tau_a[c.n], c.dd, c.th0))
        atomicOr(a.status, 1u);

    const size_t TN = (size_t)T * N;
    const rsrc_t rIn = make_rsrc(a.I_ff + b * TN, (uint32_t)(TN * 4));
    const rsrc_t rW = make_rsrc(a.WrecT, (uint32_t)((size_t)N * N * 4));
    uint8_t *tsb = a.ts + (size_t)b * a.NB * N;
    const rsrc_t rTs = make_rsrc(tsb, (uint32_t)((size_t)a.NB * N));
    const rsrc_t rH = make_rsrc(a.hits + (size_t)b * a.NB * SEG, (uint32_t)((size_t)a.NB * SEG * 4));
    const uint32_t h4 = c.nl == 0 ? (uint32_t)c.w * 4u : ALIF_OOB;   // a lane of each segment
    const size_t CN = (size_t)(a.NB + 1) * N;
    const bool ck = a.ck.v != nullptr;
    const rsrc_t rCv = make_rsrc(ck ? a.ck.v + b * CN : nullptr, ck ? (uint32_t)(CN * 4) : 0u);
    const rsrc_t rCa = make_rsrc(ck ? a.ck.a + b * CN : nullptr, ck ? (uint32_t)(CN * 4) : 0u);
    const rsrc_t rCt = make_rsrc(ck ? a.ck.ts + b * CN : nullptr, ck ? (uint32_t)CN : 0u);
    const uint32_t ck4 = (c.valid && first) ? (uint32_t)c.n * 4u : ALIF_OOB;
    const uint32_t ck1 = (c.valid && first) ? (uint32_t)c.n : ALIF_OOB;
    // this lane's column of W_rec^T (byte offset within a row), or out of range
    const uint32_t wcol = c.valid ? (uint32_t)c.n * 4u : ALIF_OOB;
    const uint32_t wrow = (uint32_t)N * 4u;

    double v0d = 0.0, a0d = 0.0;
    int cts = 0;
    if (a.nb0 > 0 && c.valid) {
        const size_t i = (size_t)b * N + c.n;
        v0d = a.st_v[i];
        a0d = a.st_a[i];
        cts = a.st_ts[i];
    }
    const uint32_t blk4 = (uint32_t)(TR * N) * 4u;
    float buf[DEPTH][L];
    auto load = [&](float (&x)[L], int nb) __attribute__((always_inline)) {
        const uint32_t bo = (uint32_t)min((size_t)nb * blk4, TN * 4);
#pragma unroll
        for (int k = 0; k < L; k++) x[k] = ld_f32_nt(rIn, c.off(k, bo));
    };
#pragma unroll
    for (int i = 0; i < DEPTH; i++) load(buf[i], a.nb0 + i);

    // The recurrent sums of the next block: in LDS rows that only steps with an event touch, or, where
    // a neuron's one wave has few steps, in registers with more events in flight (60 Hz, 64 x 128: T_R 2
    // 1.21 -> 0.99, T_R 4 1.10 -> 1.00 of one launch's time; T_R 4 at 256 neurons, 8 and 16 got slower).
    constexpr bool REG = L <= 2 || (SEG == 1 && NG == 2);
    constexpr int EV = 4;
    float accr[REG ? L : 1];
    uint32_t hit = 0;   // steps of this segment with a recurrent term (wave-uniform)
    const int qD = (D + TR - 1) / TR;   // source blocks lie qD or qD - 1 blocks back

    // The recurrent input of block nt from the spikes of blocks < nt (block nt - 1 from
    // its LDS words tsp, older ones from the ring).
    auto gather = [&](int nt, const int *tsp) __attribute__((always_inline)) {
        hit = 0;
        if constexpr (REG)
#pragma unroll
            for (int k = 0; k < L; k++) accr[k] = 0.0f;
#pragma unroll 1
        for (int q = 0; q < 2; q++) {
            const int m = nt - qD + q;   // uniform
            if (m < 0 || m >= nt || (q == 1 && D % TR == 0)) continue;
            const int base = (m - nt) * TR + D - 1;   // target offset in block nt = base + t_s
            int tsj[NG];
            bool some = false;
#pragma unroll
            for (int g = 0; g < NG; g++) {
                if (m == nt - 1) {
                    const int t = tsp[g * 64 + lane];
                    tsj[g] = t <= TR ? t : 0;
                } else {
                    tsj[g] = ring[(m % R) * NWG + g * 64 + lane];
                }
                some |= tsj[g] > 0;
            }
            if (!__any(some)) continue;
            // steps past T (padding of a ragged last block) get no recurrent term
            const int r_end = min(c.t0 + c.len, T - nt * TR);
#pragma unroll
            for (int g = 0; g < NG; g++) {
                const int t = tsj[g], r = base + t;
                uint64_t mk = __ballot(t > 0 && g * 64 + lane < N && r >= c.t0 && r < r_end);
                if constexpr (REG) {
                    while (mk) {   // EV events at a time: their loads are in flight together
                        int kk[EV];
                        float w[EV];
#pragma unroll
                        for (int e = 0; e < EV; e++) {
                            kk[e] = -1;
                            w[e] = 0.0f;
                            if (mk) {
                                const int l = __builtin_ctzll(mk);
                                mk &= mk - 1;
                                kk[e] = __builtin_amdgcn_readlane(r, l) - c.t0;
                                w[e] = ld_f32(rW, (uint32_t)(g * 64 + l) * wrow + wcol);
                            }
                        }
#pragma unroll
                        for (int e = 0; e < EV; e++) {
#pragma unroll
                            for (int k = 0; k < L; k++) accr[k] = k == kk[e] ? accr[k] + w[e] : accr[k];
                            hit |= kk[e] >= 0 ? 1u << kk[e] : 0u;
                        }
                    }
                }
                while (!REG && mk) {   // two events at a time: their loads are in flight together
                    const int l0 = __builtin_ctzll(mk);
                    mk &= mk - 1;
                    const bool two = mk != 0;
                    const int l1 = two ? __builtin_ctzll(mk) : l0;
                    mk &= mk - 1;
                    const float w0 = ld_f32(rW, (uint32_t)(g * 64 + l0) * wrow + wcol);
                    const float w1 = ld_f32(rW, (uint32_t)(g * 64 + l1) * wrow + wcol);
                    const int k0 = __builtin_amdgcn_readlane(r, l0) - c.t0;
                    const int k1 = __builtin_amdgcn_readlane(r, l1) - c.t0;
                    acc[k0 * 64] = ((hit >> k0) & 1u ? acc[k0 * 64] : 0.0f) + w0;
                    hit |= 1u << k0;
                    if (two) {
                        acc[k1 * 64] = ((hit >> k1) & 1u ? acc[k1 * 64] : 0.0f) + w1;
                        hit |= 1u << k1;
                    }
                }
            }
        }
    };

    auto store_hits = [&](int nb) __attribute__((always_inline)) {   // (block NB: dropped)
        __builtin_amdgcn_raw_buffer_store_b32(hit, rH, h4 + (uint32_t)(nb * SEG) * 4u, 0, 0);
    };

    auto do_block = [&](float (&bi)[L], int nb) __attribute__((always_inline)) {
        if (hit) {   // uniform
#pragma unroll
            for (int k = 0; k < L; k++)
                if ((hit >> k) & 1u) bi[k] += REG ? accr[REG ? k : 0] : acc[k * 64];
        }
        const float cv = (float)v0d, ca = (float)a0d;
        const int mpre = cts > 0 ? cts - 1 : 0;
        const float a1 = fmaf(c.pf, ca, cts == TR ? 1.0f : 0.0f);
        float uu[L];
        seg_scan(c, bi, mpre, uu);
        load(bi, nb + DEPTH);   // (after the gather instead: within 2%)
        int *tsp = exT + nb % 3 * NWG;
        float E = 0.0f, uTR = uu[L - 1];
        float vt[L], th[L];
        int ts;
        if constexpr (SEG > 1) {
            if (first) exT[(nb + 1) % 3 * NWG + c.nl] = ALIF_NO_SPIKE;
            exX[c.w * NWG + c.nl] = uu[L - 1];
            __syncthreads();
            seg_horner<SEG, L, EVEN, NWG>(c, exX, E, uTR);
            const int cand = seg_membrane(c, cv, E, a1, uu, vt, th);
            if (cand <= TR) atomicMin(&tsp[c.nl], cand);
            __syncthreads();
            ts = tsp[c.nl];
        } else {   // a neuron's one wave has its crossing (the copy was last read before barrier nb - 2)
            ts = seg_membrane(c, cv, E, a1, uu, vt, th);
            tsp[c.nl] = ts;
            __syncthreads();
        }
        // p^(T_R - 1 - t_s) of the lanes that spiked; asked for here, it arrives with the gather's rows
        const bool spk = ts <= TR, adapt = spk && ts < TR;
        double e2 = 0.0;
        if (__any(adapt)) e2 = adapt ? a.pd[(size_t)c.n * TR + TR - 1 - ts] : 0.0;
        if (nb + 1 < a.nb1) gather(nb + 1, tsp);   // uniform
        {   // carry-in of block nb, its spike step, the next block's steps with recurrent input
            const uint32_t e = (uint32_t)(nb * N);
            store_hits(nb + 1);
            st_f32(rCv, ck4 + e * 4u, cv);
            st_f32(rCa, ck4 + e * 4u, ca);
            st_u8(rCt, ck1 + e, (uint8_t)cts);
            st_u8(rTs, ck1 + e, (uint8_t)(ts <= TR ? ts : 0));
        }
        const double extra = (cts == TR ? c.pTm1 : 0.0) + e2;
        v0d = spk ? 0.0 : fma(c.betaT, v0d, (double)uTR);
        a0d = fma(c.pT, a0d, extra);
        cts = spk ? ts : 0;
        if (R > 0 && first) ring[(nb % R) * NWG + c.nl] = (uint8_t)(spk ? ts : 0);
    };

    // the spike steps the first block's gather needs, from the slices before
    if (first) {
        const int t = a.nb0 > 0 && c.valid ? (int)tsb[(size_t)(a.nb0 - 1) * N + c.n] : 0;
        if (a.nb0 > 0) exT[(a.nb0 - 1) % 3 * NWG + c.nl] = t > 0 ? t : ALIF_NO_SPIKE;
        exT[a.nb0 % 3 * NWG + c.nl] = ALIF_NO_SPIKE;
        for (int m = max(0, a.nb0 - R); m < a.nb0; m++)
            ring[(m % R) * NWG + c.nl] = c.valid ? tsb[(size_t)m * N + c.n] : 0;
    }
    __syncthreads();
    if (a.nb0 > 0) gather(a.nb0, exT + (a.nb0 - 1) % 3 * NWG);
    store_hits(a.nb0);
    wait_vmem_all();
    int nb = a.nb0;
    for (; nb + DEPTH <= a.nb1; nb += DEPTH) {
#pragma unroll
        for (int i = 0; i < DEPTH; i++) do_block(buf[i], nb + i);
    }
#pragma unroll
    for (int i = 0; i < DEPTH; i++)
        if (nb + i < a.nb1) do_block(buf[i], nb + i);   // uniform
    if (a.nb1 == a.NB) {   // the final carry
        const uint32_t e = (uint32_t)(a.NB * N);
        st_f32(rCv, ck4 + e * 4u, (float)v0d);
        st_f32(rCa, ck4 + e * 4u, (float)a0d);
        st_u8(rCt, ck1 + e, (uint8_t)cts);
    } else if (c.valid && first) {
        const size_t i = (size_t)b * N + c.n;
        a.st_v[i] = v0d;
        a.st_a[i] = a0d;
        a.st_ts[i] = cts;
    }
}

// How many slices. A launch and its set-up cost the chain about 8 us, in which the expansion
// moves 40 MB; the last slice's expansion runs alone. So s slices of a run that expands to
// `bytes` cost 8 (s + bytes / 40 MB / s) us: least at the square root.
inline int rec_slices(double bytes, int NB) {
    int s = (int)(sqrt(bytes / 40e6) + 0.5);
    s = s < NB / 32 ? s : NB / 32;
    return s < 1 ? 1 : (s > 8 ? 8 : s);
}

// Which runs go in slices. They save a chain about 0.1 ns a step and neuron and cost the run
// some 50 us (two more launches, the last slice's expansion): forward, us, one launch / slices:
// 64 x 1000 x 256 182 / 200, 64 x 2500 x 128 284 / 293, 64 x 4000 x 128 442 / 440, 32 x 4000 x 256
// 495 / 413, 64 x 15000 x 64 816 / 558.
// Spikes cost them more: the expansion gathers the rows of W_rec^T once again, beside the chain.
// Slices' time over one launch's with no spikes / at 6 / 15 / 60 Hz (ARP 2 ms, T 10000): 64 x 256: T_R 2
// 0.74 / 0.96 / 0.98 / 1.00, 4 0.87 / 0.99 / 1.02 / 1.06, 8 0.83 / 1.00 / 1.00 / 1.05, 10 0.85 / 0.97 / 0.94 /
// 0.93, 40 0.63 / 0.73 / 0.75 / 0.79; 64 x 128: T_R 2 0.81 / 0.94 / 0.96 / 0.99, 10 0.91 / 1.03 / 1.08 / 1.22, 16
// 0.95 / 1.01 / 1.06 / 1.18, 20 0.80 / 0.89 / 0.96 / 1.07, 40 0.68 / 0.86 / 0.94 / 0.96; 16 x 128, where more CUs
// expand: T_R 10 0.84 / 0.93 / 0.96 / 1.06, 16 0.85 / 0.91 / 0.93 / 1.02. So they are taken where 15 Hz do not
// make them slower. Rows that do not align four neurons expand at a quarter of the rate, which many
// of them beside the chain do not hide: 32 x 127, T_R 24: 0.74 / 0.83 / 0.91 / 1.03; 64 x 127: 0.81 / 1.18 / 1.27 / 1.30.
inline bool rec_sliced(int B, int T, int N, int TR, bool vec4) {
    const bool spikes_ok = B <= 16 || (N <= 128 ? TR <= 4 || TR >= 20 : TR <= 2 || TR >= 8);
    return spikes_ok && (long long)T * N >= (vec4 ? 500000 : 800000) && (vec4 || (long long)B * N <= 4096);
}

// W_rec transposed, and pd[n][k] = p^k in FP64, k < T_R: the values of the block forward's table
static __global__ void k_rec_setup(int N, int TR, double dt, const float *tau_a, const float *Wrec, float *WrecT,
                                   double *pd) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N * N) WrecT[i] = Wrec[(size_t)(i % N) * N + i / N];
    if (i < N * TR) pd[i] = exp(-dt / (double)tau_a[i / TR] * (double)(i % TR));
}

template <int SEG, int L, int NG>
hipError_t recurrent_fused_launch(RecArgs a, hipStream_t st) {
    if (a.B == 0) return hipSuccess;
    const bool even = a.TR == SEG * L;
    const dim3 blk(64 * NG * SEG);
    const int setup = a.N * (a.N > a.TR ? a.N : a.TR);
    hipLaunchKernelGGL(k_rec_setup, dim3((setup + 255) / 256), dim3(256), 0, st, a.N, a.TR, a.dt, a.tau_a, a.Wrec, a.WrecT,
                       a.pd);
    const int sb = a.spike_dtype == 0 ? 1 : (a.spike_dtype == 1 ? 2 : 4);
    a.vec4 = a.N % 4 == 0 && ((reinterpret_cast<uintptr_t>(a.I) | reinterpret_cast<uintptr_t>(a.I_ff)) & 15) == 0 &&
             (reinterpret_cast<uintptr_t>(a.spikes) & (4 * sb - 1)) == 0;
    const bool tr = a.V || a.TH;
    if (tr || !rec_sliced(a.B, a.T, a.N, a.TR, a.vec4)) {
        const size_t base = rec_smem_fixed<SEG, NG>(a.TR) + (size_t)a.ring * 64 * NG;
        const size_t smc = rec_stage_offset(base) + rec_stage_bytes<SEG, L, NG>();
        // chunked stores: whole 16-neuron chunks in every row and room for the staging tile
        const bool chunked = !tr && a.N % 16 == 0 && smc <= (size_t)160 * 1024;
        const size_t smf = chunked ? smc : base;
#define ALIF_LR(EV, TRC, CH) hipLaunchKernelGGL((k_recurrent_fused<SEG, L, EV, NG, TRC, CH>), dim3(a.B), blk, smf, st, a)
        if (even) {
            if (tr) ALIF_LR(true, true, false); else if (chunked) ALIF_LR(true, false, true); else ALIF_LR(true, false, false);
        } else {
            if (tr) ALIF_LR(false, true, false); else if (chunked) ALIF_LR(false, false, true); else ALIF_LR(false, false, false);
        }
#undef ALIF_LR
        return hipGetLastError();
    }
    const size_t sm = rec_slice_smem<SEG, L, NG>(a.ring);
    constexpr int WV = NG * SEG;
    const int slices = rec_slices((double)a.B * a.T * a.N * (8 + sb), a.NB), per = (a.NB + slices - 1) / slices;
    for (int s = 0; s <= slices; s++) {
        a.xb0 = a.nb0;
        a.xb1 = s > 0 ? a.nb1 : 0;
        a.nb0 = s * per < a.NB ? s * per : a.NB;
        a.nb1 = a.nb0 + per < a.NB ? a.nb0 + per : a.NB;
        a.core = a.nb1 > a.nb0 ? a.B : 0;
        if (s == 0) a.xb0 = 0;
        // Beside the chain the expansion gets half of what 16 waves a CU leave: it has a whole
        // slice's time, and at full width it slows the chain's own loads (1.38 against 1.30 ms
        // a layer at 64 x 256 x 20000; a quarter is too few, 1.80 ms). The last one runs alone.
        const int left = 4096 - a.core * WV;
        const int ex = a.xb1 > a.xb0 ? (a.core ? (left > 1024 ? left : 1024) / 2 : 4096) / WV : 0;
        if (a.core + ex == 0) continue;
        const size_t smem = a.core ? sm : 0;
        if (even) hipLaunchKernelGGL((k_recurrent_slice<SEG, L, true, NG>), dim3(a.core + ex), dim3(64 * WV), smem, st, a);
        else hipLaunchKernelGGL((k_recurrent_slice<SEG, L, false, NG>), dim3(a.core + ex), dim3(64 * WV), smem, st, a);
    }
    return hipGetLastError();
}

#define ALIF_INSTANTIATE_REC(S, L, NG) \
    template hipError_t recurrent_fused_launch<S, L, NG>(RecArgs, hipStream_t);

}  // namespace alif
