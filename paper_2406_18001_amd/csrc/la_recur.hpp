// The recurrence of one K-RR index block run inside a lookahead launch (see
// LookaheadArgs): workgroup 0 of the dense FP64, the FP32 and the
// low-precision kernel-block products calls it.
#pragma once

#include "common.hpp"

namespace kdcd {

__device__ __forceinline__ int64_t la_clamp(int64_t v, int64_t lo, int64_t hi)
{
    return v < lo ? lo : (v > hi ? hi : v);
}

__device__ __forceinline__ double la_readlane(double v, int l)
{
    const long long bits = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)bits, l);
    const int hi = __builtin_amdgcn_readlane((int)(bits >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The recurrence of one K-RR index block (Algorithm 4's inner loop, Eq. (3)),
// run by workgroup 0 of a lookahead launch while the other workgroups compute
// the next block's product.  With c_e = y_{S_e} - m alpha_{S_e} - r_e / lambda
// and G[t][u] = W[t][u] / lambda + m [S_t = S_u], the blocks are taken in
// order: block j's c (final once every earlier block is folded in) is
// published in LDS, lanes l < b of every wave form Delta_l = (D_j^{-1} c_j)_l
// and hand Delta_l / lambda to all lanes, and every element u of a later block
// subtracts sum_l W'[jb+l][u] Delta_l / lambda -- one barrier per block.  W' is
// the Gram with lambda m already added where a row's coordinate comes again
// later (the finish pass adds it while it copies such rows), so W' / lambda = G
// on every entry the recurrence reads.  Thread tid owns elements 2 tid
// and 2 tid + 1.  Nothing is written to alpha: the updates go to trace, and the
// summed update of each coordinate (in element order) to Dc on the element
// that the row -> position table names for it.  LB >= b rows a block (rows past b
// repeat row b - 1 and count zero times).  LDS (inside the product's A buffers): S
// of the block, the updates, c of the current and next block, a ring of four
// D_j^{-1}, one bit per element.
//
// Bound by the instructions of a step, one wave a SIMD: buffer loads with the rows
// in scalar offsets (64-bit addresses took a third of the step), neighbouring
// elements on a thread (one 16-byte load a row), and a wave leaves the loop when its
// elements are done.  64 blocks of 8 in a launch with little else: 39 us (80 with
// elements NT apart and 64-bit addresses), of 4: 22 (60).
typedef double LaPair __attribute__((ext_vector_type(2)));

template <int NT, int LB>
__device__ void la_recur(const LookaheadArgs &a, char *smem)
{
    static_assert(kLaEPT == 2, "a thread holds a pair");
    constexpr int NS = 3;
    __builtin_amdgcn_s_setprio(3);                  // ahead of the product's waves on this CU
    int32_t *S_l = reinterpret_cast<int32_t *>(smem);                  // [2 NT]
    double *d_l = reinterpret_cast<double *>(smem + 8 * NT);           // [2 NT]
    double *c_l = reinterpret_cast<double *>(smem + 24 * NT);          // [2][kLaMaxB]
    double *D_l = c_l + 2 * kLaMaxB;                                   // [4][64]
    uint32_t *mark = reinterpret_cast<uint32_t *>(D_l + 4 * 64);       // [2 NT / 32]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sb = a.sb, sk = a.sk, b = a.b;
    const int64_t m = a.m;
    const double inv_lambda = 1.0 / a.lambda, mdbl = a.mdbl;
    // this thread's elements e0, e0 + 1 of the block (sb >= 2; the last thread of an
    // odd block holds only the second of them, one past the end neither)
    const int e0 = min(2 * tid, sb - 2);
    // the wave of the last element runs to the end: it stores D_j^{-1} and the updates
    const bool lead = wid == (sb - 1) / 128;
    const int steps = lead ? sk : (wid < (sb - 1) / 128 ? (128 * wid + 127) / b : 0);

    // Every load of the loop is unconditional: with a fixed number of loads per
    // block the compiler waits for exactly the stage it needs, where a load behind
    // a branch made it wait for all of them.  Blocks past the last read past the end
    // of the buffers, which gives zeros.
    // D_j^{-1} (b*b <= 64 values, lane l: value l; lanes past b*b repeat the last)
    const __amdgpu_buffer_rsrc_t Wb = __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(a.W), 0, 8 * sb * sb, 0x00027000);
    const __amdgpu_buffer_rsrc_t Db = __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(a.Dinv), 0, 8 * sb * b, 0x00027000);
    int doff = 8 * min(lane, b * b - 1), woff = 8 * e0;
    int srow[LB];
#pragma unroll
    for (int l = 0; l < LB; ++l) srow[l] = 8 * sb * min(l, b - 1);
    auto dinv_load = [&]() -> double {              // of the next block
        const uint64_t v = __builtin_bit_cast(uint64_t, __builtin_amdgcn_raw_buffer_load_b64(Db, doff, 0, 0));
        doff += 8 * b * b;
        return __builtin_bit_cast(double, v);
    };
    // W' values of the next block for this thread's elements (used for later blocks)
    auto w_load = [&](LaPair (&w)[LB]) {
#pragma unroll
        for (int l = 0; l < LB; ++l)
            w[l] = __builtin_bit_cast(LaPair, __builtin_amdgcn_raw_buffer_load_b128(Wb, woff, srow[l], 0));
        woff += 8 * sb * b;
    };
    // NS register stages of W' values and D_j^{-1}: block j is folded out of one
    // while the loads of the NS - 1 blocks after it are in flight in the others
    // (the loop is unrolled by NS so that no stage is ever copied: a copy would
    // wait for the loads).  D_j^{-1} goes through a ring of four LDS slots, stored
    // two blocks before its use.
    LaPair w[NS][LB];
    double dreg[NS];
    const double dfirst = dinv_load(), dsecond = dinv_load();
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        dreg[u] = dinv_load();
        if (u < NS - 1) w_load(w[u]);
    }
    if (lead) {
        D_l[0 * 64 + lane] = dfirst;
        D_l[1 * 64 + lane] = dsecond;
    }
    if (tid < 2 * kLaMaxB && tid % kLaMaxB >= b) c_l[tid] = 0.0;       // past b: stays 0
    int32_t Se[2];
    int blk[2];
    double c[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int e = e0 + i;
        const bool act = e >= 2 * tid;
        Se[i] = act ? (int32_t)la_clamp(a.S[e], 0, m - 1) : -1;
        blk[i] = act ? e / b : -1;              // -1: never folded, never published
        c[i] = act ? a.y[Se[i]] - mdbl * a.alpha[Se[i]] - a.r[e] / a.lambda : 0.0;
        if (act) S_l[e] = Se[i];
        if (blk[i] == 0) c_l[e] = c[i];
    }
    for (int x = tid; x < (2 * NT) / 32; x += NT) mark[x] = 0u;
    __syncthreads();
    // an index block holds distinct coordinates (Algorithm 4 samples without
    // replacement inside a block)
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if (blk[i] >= 0)
            for (int q = blk[i] * b; q < blk[i] * b + b; ++q)
                if (q != e0 + i && S_l[q] == Se[i]) set_status(a.status, KDCD_ERR_INDEX_DUPLICATE);
    // lane l < b: row l of the running block's D_j^{-1}, read before the barrier
    // that publishes its c
    const double *drow = D_l + (lane < b ? lane * b : 0);
    double dv[LB];
#pragma unroll
    for (int t = 0; t < LB; ++t) dv[t] = drow[t];

    auto step = [&](int j, const LaPair (&wc)[LB], LaPair (&wf)[LB], double &dr) {
        const double *cn = c_l + (j & 1) * kLaMaxB;
        double cv[LB];
#pragma unroll
        for (int t = 0; t < LB; ++t) cv[t] = cn[t];
        if (lead) D_l[((j + 2) & 3) * 64 + lane] = dr;
        dr = dinv_load();
        w_load(wf);
        double dl = 0.0;
#pragma unroll
        for (int t = 0; t < LB; ++t) dl += dv[t] * cv[t];
        dl = lane < b ? dl : 0.0;
        if (lead && lane < b) d_l[j * b + lane] = dl;
        // (block j + 1's slot was stored at step j - 1, before its barrier)
#pragma unroll
        for (int t = 0; t < LB; ++t) dv[t] = drow[((j + 1) & 3) * 64 + t];
        // Delta / lambda of the block on every lane (lane reads: scalar registers)
        const double dls = dl * inv_lambda;
        double dvs[LB], acc[2] = {0.0, 0.0};
#pragma unroll
        for (int l = 0; l < LB; ++l) dvs[l] = la_readlane(dls, l);   // lanes >= b hold 0
#pragma unroll
        for (int l = 0; l < LB; ++l)
#pragma unroll
            for (int i = 0; i < 2; ++i) acc[i] += wc[l][i] * dvs[l];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (blk[i] > j) c[i] -= acc[i];
            if (blk[i] == j + 1)                // the next block's c
                c_l[((j + 1) & 1) * kLaMaxB + (e0 + i - (j + 1) * b)] = c[i];
        }
        lds_barrier();
    };
    for (int j = 0; j < steps; j += NS) {
#pragma unroll
        for (int u = 0; u < NS; ++u)
            if (j + u < steps) step(j + u, w[u], w[(u + NS - 1) % NS], dreg[u]);
    }
    for (int j = steps; j < sk; ++j) lds_barrier();

    // Canonical element of a coordinate: the one the row table names (its
    // last).  Every earlier element of the coordinate marks the canonical one,
    // and only a marked canonical element sums the coordinate's updates, in
    // element order (a wave looks for the earlier elements of one coordinate
    // together: each lane on its own over the block took 9 us).
    int canon[kLaEPT];   // 1 canonical, 0 not, -1 no element
#pragma unroll
    for (int i = 0; i < kLaEPT; ++i) {
        const int e = tid + i * NT;
        canon[i] = -1;
        if (e < sb) {
            Se[i] = S_l[e];
            const int32_t q = a.pos[Se[i]];
            canon[i] = q == e ? 1 : 0;
            if (q != e && q >= 0 && q < sb) atomicOr(&mark[q >> 5], 1u << (q & 31));
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kLaEPT; ++i) {
        const int e = tid + i * NT;
        const double de = e < sb ? d_l[e] : 0.0;
        double v = canon[i] == 1 ? de : 0.0;
        const bool sum = canon[i] == 1 && (mark[e >> 5] & (1u << (e & 31)));
        for (uint64_t todo = __ballot(sum); todo; todo &= todo - 1) {    // uniform
            const int o = __builtin_ctzll(todo);
            const int32_t So = __builtin_amdgcn_readlane(Se[i], o);
            const int eo = e - lane + o;
            double sacc = 0.0;
            for (int t0 = 0; t0 < eo; t0 += 64) {
                uint64_t hit = __ballot(t0 + lane < eo && S_l[t0 + lane] == So);
                for (; hit; hit &= hit - 1) sacc += d_l[t0 + __builtin_ctzll(hit)];
            }
            if (lane == o) v = sacc + de;
        }
        if (e >= sb) continue;
        a.Dc[e] = v;
        a.Sc[e] = canon[i] == 1 ? Se[i] : -1;
        if (a.trace) a.trace[e] = de;
    }
}

}  // namespace kdcd
