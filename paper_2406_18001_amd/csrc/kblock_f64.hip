// Dense FP64 kernel block on gfx950 MFMA (v_mfma_f64_16x16x4f64).
//
// One launch computes, for the index block S (sb sampled rows):
//   U-tiles:  P = A A_S^T (m x sb), the Table 1 map K = map(P) in the
//             epilogue, and the column sums partial[g][j] = sum_{p in group g}
//             K(a_p, a_{S_j}) beta_p -- the right-hand side U^T beta of
//             Algorithms 2 and 4 -- without ever writing U;
//   W-tiles:  W = K(A_S, A_S) (sb x sb), the sampled Gram V^T U; with a row
//             range (w_row0, w_rows) the rows are S[w_row0 .. w_row0 + w_rows)
//             instead (W then w_rows x sb: index blocks stored back to back
//             give the Gram of one block against the next in one launch).
// Both read the sampled rows straight from A through S (no gather pass).
//
// Tiling: a workgroup of WM waves owns a tile of 16 TM WM rows x 16 TN columns,
// every wave TM x TN MFMA blocks over all of the tile's columns.  A row of A
// then feeds one wave only, so its fragments go from global memory straight to
// that wave's registers -- no LDS, no barrier -- two chunks of 16 doubles ahead;
// the sampled rows, which every wave of the workgroup multiplies, are staged
// through a double-buffered LDS panel.  Against staging both operands in LDS
// (2 x 2 waves) a wave reads one LDS fragment of 16 bytes per lane for 2 TM MFMAs
// instead of one of 8 bytes for one, writes none of A to LDS, and meets one
// barrier per 4 TM TN MFMAs.
//
// What bounds it: f64 MFMA.  A 16 x 16 x 4 step takes 64 cycles of a SIMD (72
// TFLOP/s on this chip with random operands, registers only; a large library
// DGEMM reaches the same), and FP64 vector instructions share the unit: a map of
// 17 of them per element costs as much as 17 more columns of A.  Measured per launch (RBF),
// the LDS-staged tiles' best against this kernel's:
//   200000 x 1024, 512 sampled rows   3850 -> 3110 us (floor 2913)
//    20000 x  512, 512                 200 ->  183    (146)
//   500000 x  256,  64                 461 ->  316    (228)
//     7001 x  333,  63                32.7 -> 15.8    (4.1)
//     2000 x   64,   1                10.4 ->  8.2
// At 16384 rows a launch costs 18 us beyond its MFMA time whatever n is: the
// start of a workgroup (indices, sampled rows, first chunks, one after another),
// the map, and the last workgroups.
// Not kept: A four chunks ahead (more registers, no fewer stalls: 3650 us at 200000
// x 1024), and the first fragments of a chunk read before the barrier that
// precedes it from a third LDS buffer (3355 us).
//
// Inside a chunk, MFMA step ks uses k = 4 (lane / 16) + ks for both operands
// (any bijection of k works as long as A and B agree); a lane's four doubles
// of a row are contiguous in memory.  Rows need no alignment beyond their
// doubles' (global loads of 16 bytes take any 4-byte address), and a last chunk of
// less than 16 columns is loaded element by element.
#include "common.hpp"
#include "exp_tab.hpp"
#include "la_recur.hpp"

namespace kdcd {
namespace {

constexpr int BK = 16;
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));

__device__ __forceinline__ int64_t clampi(int64_t v, int64_t lo, int64_t hi)
{
    return v < lo ? lo : (v > hi ? hi : v);
}

// Logical tile id from the hardware block id: consecutive logical ids land
// on the same XCD (workgroups are dealt round-robin over the 8 XCDs), so the
// column tiles that share one row group of A share that XCD's L2.
__device__ __forceinline__ int xcd_remap(int bid, int total)
{
    const int per = total / 8, rem = total % 8;
    const int x = bid % 8, w = bid / 8;
    return x < rem ? x * (per + 1) + w : rem * (per + 1) + (x - rem) * per + w;
}

// Column sums of MFMA outputs over a wave's four 16-lane rows, for TN values at
// once: v_permlane32/16_swap exchange halves (rows) of two registers, so one
// addition finishes a step of two sums.  Lane l gets the total of value
// sum_slot<TN>(l), column l % 16 (TN 2: each in two rows, TN 1: in all).
__device__ __forceinline__ double swap_add32(double x, double y)
{
    const uint64_t a = (uint64_t)__double_as_longlong(x), b = (uint64_t)__double_as_longlong(y);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
    return __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0])) +
           __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
}
__device__ __forceinline__ double swap_add16(double x, double y)
{
    const uint64_t a = (uint64_t)__double_as_longlong(x), b = (uint64_t)__double_as_longlong(y);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)a, (uint32_t)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
    return __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0])) +
           __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
}
template <int TN> __device__ __forceinline__ double col_sums(const double (&v)[TN])
{
    static_assert(TN == 1 || TN == 2 || TN == 4, "");
    if constexpr (TN == 4) return swap_add16(swap_add32(v[0], v[1]), swap_add32(v[2], v[3]));
    const double a = swap_add32(v[0], v[TN - 1]);
    return swap_add16(a, a);
}
template <int TN> __device__ __forceinline__ int sum_slot(int lane)
{
    return TN == 4 ? ((lane >> 5) & 1) | ((lane >> 3) & 2) : (TN == 2 ? lane >> 5 : 0);
}

// BATCH: several problems share the product (descriptor bd in device memory):
// the map runs once per sigma group, every problem reduces its own beta, and
// the Gram tiles are written once per group.  partial is then [p][group][sb]
// and W is [g][sb][sb].  OCC: waves per SIMD the registers are held to.
// LA: a lookahead launch (workgroup 0 runs la_recur for the previous block,
// workgroups 1 .. kLaLead - 1 return, the product's tiles follow; the product
// also stores the rows of la.pos's coordinates into la.QX).
template <int WM, int TM, int TN, int KIND, bool BATCH, int OCC, bool LA>
__global__ __launch_bounds__(64 * WM) __attribute__((amdgpu_waves_per_eu(OCC))) void kblock_f64_kernel(
    const double *__restrict__ A, int64_t lda, int64_t m, int64_t n,
    const int32_t *__restrict__ S, int32_t sb, const double *__restrict__ norms, KParams kp,
    const double *__restrict__ beta, const double *__restrict__ bscale,
    double *__restrict__ partial, double *__restrict__ W, int32_t n_u_tiles,
    int32_t n_row_groups, int32_t n_w_tiles, int32_t n_tiles_n,
    const BatchDesc *__restrict__ bd, double *__restrict__ U, const int32_t *__restrict__ stop,
    const int32_t *__restrict__ pos, int64_t u_gstride, int32_t w_row0, int32_t w_rows,
    const LookaheadArgs la)
{
    if (stop && *stop) return;   // the solve has converged
    constexpr int NT = 64 * WM;
    constexpr int BM = 16 * TM * WM;
    constexpr int BN = 16 * TN;
    constexpr int SEGB = (BN * 4 + NT - 1) / NT;   // 4-double segments of a B chunk per thread
    constexpr int BBUF = BN * BK;
    constexpr int LADB = LA ? (24 * NT + 8 * (2 * kLaMaxB + 256) + NT / 4) / 8 : 1;

    // B chunks: [block of 16 columns][half: k pair][lane] of two doubles
    constexpr int BSZ = BBUF / 2 > LADB / 4 + 1 ? BBUF / 2 : LADB / 4 + 1;
    __shared__ d2 Bs[2][BSZ];
    __shared__ double red[WM][BN];
    // the tile's rows: index (-1 past the end), beta (scaled), norm, row of W, row of QX
    __shared__ int32_t rsh[BM], wsh[BM], xsh[LA ? BM : 1];
    __shared__ double bsh[BM], nsh[BM];
    __shared__ d2 etab[KIND == KDCD_KERNEL_RBF ? kExpTab : 1];
    // the columns past the last whole chunk, if any (a third B buffer); batched: beta
    // of every problem for the tile's rows [p][BM], column sums [p][WM][BN]
    extern __shared__ double dsh[];
    d2 *Bt = reinterpret_cast<d2 *>(dsh);

    if constexpr (LA) {
        static_assert(sizeof(Bs) >= 8 * (size_t)LADB, "the lookahead recurrence's LDS must fit");
        if (blockIdx.x < kLaLead) {
            if (blockIdx.x == 0 && la.sb > 0) {
                char *smem = reinterpret_cast<char *>(&Bs[0][0]);
                if (la.b > 4) la_recur<NT, 8>(la, smem);
                else la_recur<NT, 4>(la, smem);
            }
            return;
        }
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int total = n_tiles_n * (n_row_groups + n_w_tiles);
    if (!BATCH && !LA && gridDim.y > 1) {        // Gram-only launch of several index blocks
        S += (int64_t)blockIdx.y * sb;
        W += (int64_t)blockIdx.y * w_rows * sb;
    }
    // the leading workgroups of a lookahead launch are a multiple of 8, so
    // bid % 8 is still the XCD of the workgroup
    const int bid = LA ? (int)blockIdx.x - kLaLead : (int)blockIdx.x;
    const int L = xcd_remap(bid, total);
    const int cn = L % n_tiles_n;
    const int rg = L / n_tiles_n;
    const bool is_w = rg >= n_row_groups;
    if (is_w && W == nullptr) return;
    if (KIND == KDCD_KERNEL_RBF) exp_tab_load(etab);   // (read after the K loop's barriers)
    const int col0 = cn * BN;

    // sampled rows feeding the B operand: the indices are loaded first, the
    // wave's first rows of A go out while they arrive
    int32_t sj[SEGB];
#pragma unroll
    for (int i = 0; i < SEGB; ++i) {
        const int seg = tid + i * NT;
        sj[i] = S[clampi(col0 + ((seg < BN * 4) ? (seg >> 2) : 0), 0, sb - 1)];
    }
    double colsum[TN];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) colsum[tn] = 0.0;
    const int np = BATCH ? bd->nprob : 0;
    double *bpsh = dsh + (n % BK ? BBUF : 0), *redb = bpsh + np * BM;
    // batched: problems of every sigma group (bits), staged so that the epilogue
    // reads no descriptor
    __shared__ uint32_t gmask[BATCH ? kMaxSigmas : 1];
    constexpr int PPW = BATCH ? (kMaxProblems + WM - 1) / WM : 1;   // problems staged per wave
    constexpr int RPL = BM / 64;                                    // rows of it per lane
    if constexpr (BATCH) {
        for (int x = tid; x < np * WM * BN; x += NT) redb[x] = 0.0;
        if (tid < kMaxSigmas) {
            uint32_t mk = 0;
            for (int p = 0; p < np; ++p) mk |= bd->group[p] == tid ? 1u << p : 0u;
            gmask[tid] = mk;
        }
        __syncthreads();
    }

    // row tiles of this group: ranges whose lengths differ by at most one, spread
    // evenly over the groups (and so over the XCDs)
    const int rt_first = is_w ? rg - n_row_groups : (int)((int64_t)rg * n_u_tiles / n_row_groups);
    const int rt_end = is_w ? rt_first + 1 : (int)((int64_t)(rg + 1) * n_u_tiles / n_row_groups);
    const int64_t nF = n / BK;                     // whole chunks

    // operand pointers of a row tile; the tile after the last one reads the last
    // one's rows again (ignored)
    auto set_rows = [&](int rt, const double *(&ap)[TM]) {
        const int64_t row0 = (int64_t)(rt < rt_end ? rt : rt_end - 1) * BM;
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const int64_t r = row0 + (wid * TM + tm) * 16 + (lane & 15);
            int64_t row;
            if (is_w) row = clampi(S[w_row0 + clampi(r, 0, w_rows - 1)], 0, m - 1);
            else row = clampi(r, 0, m - 1);
            ap[tm] = A + row * lda + 4 * (lane >> 4);
        }
    };
    const double *bptr[SEGB];
    d2 ra0[TM][2], ra1[TM][2], rb0[SEGB][2], rb1[SEGB][2];
    auto load_a = [&](const double *const (&ap)[TM], int64_t kc, d2 (&ra)[TM][2]) {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const d2u *p = reinterpret_cast<const d2u *>(ap[tm] + kc * BK);
            ra[tm][0] = p[0];
            ra[tm][1] = p[1];
        }
    };
    auto load_b = [&](int64_t kc, d2 (&rb)[SEGB][2]) {
#pragma unroll
        for (int i = 0; i < SEGB; ++i) {
            const d2u *p = reinterpret_cast<const d2u *>(bptr[i] + kc * BK);
            rb[i][0] = p[0];
            rb[i][1] = p[1];
        }
    };
    auto store_b = [&](d2 *buf, const d2 (&rb)[SEGB][2]) {
#pragma unroll
        for (int i = 0; i < SEGB; ++i) {
            const int seg = tid + i * NT;
            if (BN * 4 % NT == 0 || seg < BN * 4) {
                const int r = seg >> 2, c = seg & 3;
                d2 *dst = &buf[((r >> 4) * 2) * 64 + c * 16 + (r & 15)];
                dst[0] = rb[i][0];
                dst[64] = rb[i][1];
            }
        }
    };

    // Pipeline: chunk c of the tile under way is multiplied out of LDS buffer
    // c & 1 (sampled rows) and register stage c & 1 (the wave's rows of A) while
    // chunk c + 1 waits in the other stage and chunk c + 2 is in flight; past the
    // tile's last chunk the stages take the next tile's first ones, so a tile's
    // map and reduction run with the next tile's loads in flight.  Loads are
    // unconditional, so that the compiler waits for exactly the stage it uses;
    // whole pairs in the loop and an odd last chunk after it (one loop exit
    // keeps the accumulators in place).
    const double *aptr[TM], *anext[TM];
    set_rows(rt_first, aptr);
    const int64_t c1 = nF > 1 ? 1 : 0;
    if (nF > 0) {
        load_a(aptr, 0, ra0);
        load_a(aptr, c1, ra1);
    }
#pragma unroll
    for (int i = 0; i < SEGB; ++i)   // (clamped so that every load is in bounds)
        bptr[i] = A + clampi(sj[i], 0, m - 1) * lda + 4 * ((tid + i * NT) & 3);
    if (n % BK) {
#pragma unroll
        for (int i = 0; i < SEGB; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                rb0[i][e >> 1][e & 1] = nF * BK + 4 * ((tid + i * NT) & 3) + e < n ? bptr[i][nF * BK + e] : 0.0;
        store_b(Bt, rb0);
    }
    if (nF > 0) {
        load_b(0, rb0);
        load_b(c1, rb1);
    }
    // per-lane output columns of this wave
    int32_t Sc[TN];
    double nb[TN];
    bool colok[TN];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        const int64_t gcol = col0 + tn * 16 + (lane & 15);
        colok[tn] = gcol < sb;
        Sc[tn] = (int32_t)clampi(S[clampi(gcol, 0, sb - 1)], 0, m - 1);
        nb[tn] = (KIND == KDCD_KERNEL_RBF) ? norms[Sc[tn]] : 0.0;
    }

    if (nF > 0) store_b(Bs[0], rb0);
    lds_barrier();

    for (int rt = rt_first; rt < rt_end; ++rt) {
        const int64_t row0 = (int64_t)rt * BM;
        set_rows(rt + 1, anext);
        // this thread's row of the tile (BM <= NT), and the columns past the last
        // whole chunk: in flight during the loop
        static_assert(BM <= NT, "one row per thread");
        int32_t gr = -1, gw = -1, gx = -1;
        double gb = 0.0, gn = 0.0;
        if (tid < BM) {
            const int64_t r = row0 + tid;
            if (is_w) {
                if (r < w_rows) gr = (int32_t)clampi(S[w_row0 + r], 0, m - 1);
            } else if (r < m) {
                gr = (int32_t)r;
                if (!BATCH) {
                    gb = beta[r];
                    if (bscale) gb *= bscale[r];
                    if (pos) gw = pos[r];
                    if (LA) gx = la.pos[r];
                }
            }
            if (KIND == KDCD_KERNEL_RBF && gr >= 0) gn = norms[gr];
        }
        // batched: this wave's problems' scaled beta for row `lane` (the epilogue of the
        // tile before is behind a barrier; read after the barriers of the loop)
        if constexpr (BATCH) {
            if (!is_w) {
#pragma unroll
                for (int q = 0; q < RPL; ++q) {
                    const int64_t r = clampi(row0 + 64 * q + lane, 0, m - 1);
                    const bool rok = row0 + 64 * q + lane < m;
                    double pb[PPW], psc[PPW];
#pragma unroll
                    for (int i = 0; i < PPW; ++i) {
                        const int p = wid + i * WM;
                        pb[i] = 0.0;
                        psc[i] = 1.0;
                        if (p < np) {
                            pb[i] = bd->beta[p][r];
                            if (bd->bscale[p]) psc[i] = bd->bscale[p][r];
                        }
                    }
#pragma unroll
                    for (int i = 0; i < PPW; ++i)
                        if (wid + i * WM < np)
                            bpsh[(wid + i * WM) * BM + 64 * q + lane] = rok ? pb[i] * psc[i] : 0.0;
                }
            }
        }
        d2 rt0[TM][2];
        if (n % BK) {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    rt0[tm][e >> 1][e & 1] = nF * BK + 4 * (lane >> 4) + e < n ? aptr[tm][nF * BK + e] : 0.0;
        }

        d4 acc[TM][TN];
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) acc[tm][tn] = d4{0.0, 0.0, 0.0, 0.0};
        auto compute = [&](const d2 *buf, const d2 (&ra)[TM][2]) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                d2 b[TN];
#pragma unroll
                for (int tn = 0; tn < TN; ++tn) b[tn] = buf[(tn * 2 + h) * 64 + lane];
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                        for (int tn = 0; tn < TN; ++tn)
                            acc[tm][tn] = __builtin_amdgcn_mfma_f64_16x16x4f64(ra[tm][h][e], b[tn][e],
                                                                               acc[tm][tn], 0, 0, 0);
            }
        };

        const bool odd = nF & 1;
        for (int64_t kc = 0; kc + 1 < nF; kc += 2) {
            // chunks kc + 2 and kc + 3, or (past the end) what stages 0 and 1 take next:
            // an odd last chunk goes to stage 0, the next tile's chunk 0 / 1 otherwise
            const bool w2 = kc + 2 >= nF, w3 = kc + 3 >= nF;
            const int64_t k2 = w2 ? 0 : kc + 2, k3 = w3 ? c1 : kc + 3;
            load_b(k2, rb0);
            compute(Bs[0], ra0);
            load_a(w2 ? anext : aptr, k2, ra0);
            store_b(Bs[1], rb1);             // chunk kc + 1
            lds_barrier();
            load_b(k3, rb1);
            compute(Bs[1], ra1);
            load_a(w3 ? anext : aptr, k3, ra1);
            store_b(Bs[0], rb0);             // chunk kc + 2, or the next tile's chunk 0
            lds_barrier();
        }
        if (odd) {                       // chunk nF - 1, in buffer 0
            load_b(0, rb0);
            compute(Bs[0], ra0);
            load_a(anext, 0, ra0);
            if (nF == 1) {
                load_b(0, rb1);
                load_a(anext, 0, ra1);
            }
        }
        if (n % BK) compute(Bt, rt0);
        if (tid < BM) {
            rsh[tid] = gr;
            bsh[tid] = gb;
            nsh[tid] = gn;
            wsh[tid] = gw;
            if (LA) xsh[tid] = gx;
        }
        lds_barrier();                   // also: every wave is done with buffer 0's odd chunk
        if (odd) store_b(Bs[0], rb0);        // the next tile's chunk 0

        // epilogue: item v of MFMA output lane l is row (l/16) + 4v, column l%16 of its block
        const int lr = wid * TM * 16 + (lane >> 4);
        if constexpr (BATCH) {
            const int ng = bd->ngroups;
            for (int g = 0; g < ng; ++g) {
                KParams kg = kp;
                kg.sigma = bd->sigma[g];
                const uint32_t gm = __builtin_amdgcn_readfirstlane(gmask[g]);
#pragma unroll
                for (int tm = 0; tm < TM; ++tm) {
                    double kv[4][TN];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int32_t grow = rsh[lr + tm * 16 + 4 * v];
                        const double na = nsh[lr + tm * 16 + 4 * v];
#pragma unroll
                        for (int tn = 0; tn < TN; ++tn)
                            kv[v][tn] = (grow >= 0 && colok[tn])
                                            ? kernel_map_tab<KIND>(acc[tm][tn][v], na, nb[tn],
                                                                   grow == Sc[tn], kg, etab)
                                            : 0.0;
                    }
                    if (is_w || U) {   // the Gram of group g, or the monitor's stored kernel block
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int64_t r = row0 + lr + tm * 16 + 4 * v;
                            const bool rok = rsh[lr + tm * 16 + 4 * v] >= 0;
#pragma unroll
                            for (int tn = 0; tn < TN; ++tn) {
                                const int64_t gcol = col0 + tn * 16 + (lane & 15);
                                if (!rok || !colok[tn]) continue;
                                if (is_w) W[((int64_t)g * sb + r) * sb + gcol] = kv[v][tn];
                                else U[(int64_t)g * u_gstride + gcol * m + r] = kv[v][tn];
                            }
                        }
                        if (is_w) continue;
                    }
                    for (uint32_t todo = gm; todo; todo &= todo - 1) {
                        const int p = __builtin_ctz(todo);
                        double bv[4], ps[TN];
#pragma unroll
                        for (int v = 0; v < 4; ++v) bv[v] = bpsh[p * BM + lr + tm * 16 + 4 * v];
#pragma unroll
                        for (int tn = 0; tn < TN; ++tn) {
                            ps[tn] = bv[0] * kv[0][tn];
#pragma unroll
                            for (int v = 1; v < 4; ++v) ps[tn] += bv[v] * kv[v][tn];
                        }
                        const double sum = col_sums<TN>(ps);
                        if (TN == 4 || (TN == 2 && !(lane & 16)) || lane < 16)
                            redb[(p * WM + wid) * BN + sum_slot<TN>(lane) * 16 + (lane & 15)] += sum;
                    }
                }
            }
        } else {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int t = lr + tm * 16 + 4 * v;
                    const int32_t grow = rsh[t];
                    if (grow < 0) continue;
                    const double bval = bsh[t], na = nsh[t];
                    const int32_t wrow = is_w ? (int32_t)(row0 + t) : wsh[t];   // row of W, or -1
                    const int32_t xrow = LA ? xsh[t] : -1;                      // row of QX, or -1
                    const bool wok = is_w || (wrow >= 0 && wrow < sb);
#pragma unroll
                    for (int tn = 0; tn < TN; ++tn)
                        if (colok[tn]) {
                            const double kv = kernel_map_tab<KIND>(acc[tm][tn][v], na, nb[tn],
                                                                   grow == Sc[tn], kp, etab);
                            const int64_t gcol = col0 + tn * 16 + (lane & 15);
                            colsum[tn] += bval * kv;
                            if (U && !is_w) U[gcol * m + grow] = kv;
                            if (wok) W[(int64_t)wrow * sb + gcol] = kv;
                            if (LA && xrow >= 0 && xrow < la.sb)
                                la.QX[(int64_t)xrow * sb + gcol] = kv;
                        }
                }
            }
        }
        lds_barrier();               // the rows' data is read before the next tile's is stored
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) aptr[tm] = anext[tm];
    }
    if (is_w) return;

    if constexpr (BATCH) {   // every problem: waves -> one partial row per group
        __syncthreads();
        for (int x = tid; x < np * BN; x += NT) {
            const int p = x / BN, c = x % BN;
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < WM; ++w) t += redb[(p * WM + w) * BN + c];
            if (col0 + c < sb) partial[((int64_t)p * n_row_groups + rg) * sb + col0 + c] = t;
        }
        return;
    }
    // deterministic column reduction: lanes -> waves -> one partial row per group
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        const double v = wave_sum_xor16_32(colsum[tn]);
        if (lane < 16) red[wid][tn * 16 + lane] = v;
    }
    __syncthreads();
    for (int c = tid; c < BN; c += NT) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < WM; ++w) t += red[w][c];
        if (col0 + c < sb) partial[(int64_t)rg * sb + col0 + c] = t;
    }
}

// pos[] upkeep: clear the previous block's entries, then mark the new one
// (one workgroup, so the clears are ordered before the marks; the marks of a
// repeated row keep its largest position, so the table does not depend on the
// order of the stores).
__global__ __launch_bounds__(1024) void pos_set_kernel(int32_t *__restrict__ pos, int64_t m,
                                                       const int32_t *__restrict__ prevS,
                                                       int32_t prev_sb,
                                                       const int32_t *__restrict__ S, int32_t sb,
                                                       const int32_t *__restrict__ stop)
{
    if (stop && *stop) return;
    for (int t = threadIdx.x; t < prev_sb; t += blockDim.x) {
        const int32_t p = prevS[t];
        if (p >= 0 && p < m) pos[p] = -1;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < sb; t += blockDim.x) {   // a repeated row keeps its last t
        const int32_t p = S[t];
        if (p >= 0 && p < m) atomicMax(&pos[p], t);
    }
}

// Rows of W for repeated indices: row t copies the row written for S_t.
__global__ __launch_bounds__(256) void w_dup_kernel(double *__restrict__ W, int64_t m,
                                                    const int32_t *__restrict__ S, int32_t sb,
                                                    const int32_t *__restrict__ pos,
                                                    const int32_t *__restrict__ stop)
{
    if (stop && *stop) return;
    const int t = blockIdx.x;
    const int32_t p = S[t];
    if (p < 0 || p >= m) return;
    const int32_t r = pos[p];
    if (r == t || r < 0) return;
    for (int j = threadIdx.x; j < sb; j += blockDim.x)
        W[(int64_t)t * sb + j] = W[(int64_t)r * sb + j];
}

constexpr int64_t kMaxRowGroups = 1024;
constexpr int kCUs = 256;

int64_t streamed_row_groups(int tm, int tn, int64_t m, int64_t n, int32_t sb)
{
    // Row tiles per workgroup t: the busiest CU's tiles, ceil(workgroups / CUs) * t,
    // times a tile's MFMA time, plus a start-up of about 3 us (7000 cycles: indices,
    // sampled rows, first chunks, one after another) per round of the two
    // workgroups that a CU holds.  At 200000 x 1024 with 512 sampled rows (1563 x 8
    // tiles) t = 7 gives 49 tiles on the busiest CU where groups of one and two
    // tiles, the longer ones on five of the eight XCDs, took 64.
    const int64_t bm = 64 * tm, n_u = (m + bm - 1) / bm, n_n = (sb + 16 * tn - 1) / (16 * tn);
    const double tile = 256.0 * tm * tn * (double)((n + BK - 1) / BK);
    const int64_t tmin = (n_u + kMaxRowGroups - 1) / kMaxRowGroups;
    int64_t best = (n_u + tmin - 1) / tmin;
    double cost = INFINITY;
    for (int64_t t = tmin; t < tmin + 32 && t <= n_u; ++t) {
        const int64_t g = (n_u + t - 1) / t, wgs = g * n_n;
        if (t > tmin && wgs < 2 * kCUs) break;
        const double c = (double)((wgs + kCUs - 1) / kCUs) * (double)t * tile +
                         7000.0 * (double)((wgs + 2 * kCUs - 1) / (2 * kCUs));
        if (c < cost) {
            cost = c;
            best = g;
        }
    }
    return best;
}

template <int WM, int TM, int TN, bool BATCH, int OCC>
hipError_t launch_tiles(const KBlockArgs &a, hipStream_t st, int nprob = 0)
{
    constexpr int BM = 16 * TM * WM, BN = 16 * TN;
    const kdcd_matrix *A = a.A;
    const int64_t n_u = a.w_only ? 0 : (A->m + BM - 1) / BM;
    const int64_t groups = a.w_only ? 0 : streamed_row_groups(TM, TN, A->m, A->n, a.sb);
    const int32_t w_rows = a.w_rows > 0 ? a.w_rows : a.sb;
    const int64_t n_w = (a.W && !a.pos) ? (w_rows + BM - 1) / BM : 0;
    if (groups + n_w == 0) return hipSuccess;
    const int64_t n_n = (a.sb + BN - 1) / BN;
    const bool la = !BATCH && a.la != nullptr;
    if (la && !(a.pos && a.la->b <= kLaMaxB && a.la->sb <= kLaEPT * 64 * WM))
        return hipErrorInvalidValue;   // the caller checks lookahead_supported first
    const int64_t blocks = n_n * (groups + n_w) + (la ? kLaLead : 0);
    const LookaheadArgs lav = la ? *a.la : LookaheadArgs{};
    dim3 grid((unsigned)blocks, a.w_only && !BATCH ? (unsigned)a.w_batch : 1u), block(64 * WM);
    const size_t dyn = sizeof(double) * (size_t)((A->n % BK ? BN * BK : 0) +
                                                 (BATCH ? nprob * (BM + WM * BN) : 0));
#define KDCD_LAUNCH_F(KIND, LA)                                                                  \
    KDCD_TIMED_LAUNCH((kblock_f64_kernel<WM, TM, TN, KIND, BATCH, (LA && OCC > 3 ? 3 : OCC), LA>), grid, block, dyn, st, \
                       A->values, A->ld, A->m, A->n, a.S, a.sb, a.norms, a.kp, a.beta,           \
                       a.beta_scale, a.partial, a.W, (int32_t)n_u, (int32_t)groups,              \
                       (int32_t)n_w, (int32_t)n_n, a.batch, a.U, a.stop,                         \
                       BATCH ? nullptr : a.pos, a.u_gstride, a.w_row0, w_rows, lav)
#define KDCD_LAUNCH(KIND)                                                                        \
    do {                                                                                          \
        if (la) {                                                                                 \
            if constexpr (!BATCH) KDCD_LAUNCH_F(KIND, true);                                      \
        } else KDCD_LAUNCH_F(KIND, false);                                                        \
    } while (0)
    switch (a.kp.kind) {
    case KDCD_KERNEL_LINEAR: KDCD_LAUNCH(KDCD_KERNEL_LINEAR); break;
    case KDCD_KERNEL_POLY: KDCD_LAUNCH(KDCD_KERNEL_POLY); break;
    default: KDCD_LAUNCH(KDCD_KERNEL_RBF); break;
    }
#undef KDCD_LAUNCH
#undef KDCD_LAUNCH_F
    return hipGetLastError();
}

}  // namespace

// Tile configurations (MFMA blocks per wave; four waves, one above the other).  Saved
// tuning tables hold the ids: a new tile takes a new one, none changes its tile.
struct F64Cfg {
    int tm, tn;
};
constexpr F64Cfg kF64Cfgs[] = {
    {2, 1},   // 0: 128 x 16
    {2, 2},   // 1: 128 x 32
    {1, 4},   // 2: 64 x 64
    {1, 8},   // 3: 64 x 128
    {1, 8},   // 4: 64 x 128 (once with eight waves)
    {2, 4},   // 5: 128 x 64
    {1, 4},   // 6: 64 x 64 (once with fewer registers)
    {1, 2},   // 7: 64 x 32
    {1, 1},   // 8: 64 x 16
};
constexpr int kF64NumCfgs = sizeof(kF64Cfgs) / sizeof(kF64Cfgs[0]);
// Those of the batched launch.
constexpr F64Cfg kF64BatchCfgs[] = {
    {2, 1},   // 0: 128 x 16
    {2, 2},   // 1: 128 x 32
    {1, 4},   // 2: 64 x 64
    {2, 4},   // 3: 128 x 64
    {1, 2},   // 4: 64 x 32
    {1, 1},   // 5: 64 x 16
};
constexpr int kF64BatchNumCfgs = sizeof(kF64BatchCfgs) / sizeof(kF64BatchCfgs[0]);

int f64_config_count() { return kF64NumCfgs; }
int f64_batch_config_count() { return kF64BatchNumCfgs; }

static void shape_of(const F64Cfg &c, int *bm, int *bn, int *waves)
{
    *bm = 64 * c.tm;
    *bn = 16 * c.tn;
    *waves = 4;
}
void f64_config_shape(int id, int *bm, int *bn, int *waves) { shape_of(kF64Cfgs[id], bm, bn, waves); }
void f64_batch_config_shape(int id, int *bm, int *bn, int *waves)
{
    shape_of(kF64BatchCfgs[id >= 0 && id < kF64BatchNumCfgs ? id : 2], bm, bn, waves);
}

static int64_t tiles_of(int64_t m, int32_t sb, int tm, int tn)
{
    return ((m + 64 * tm - 1) / (64 * tm)) * ((sb + 16 * tn - 1) / (16 * tn));
}

// Built-in rule, used when the tuning table has no entry for (n, sb): columns
// as many as the block has (up to 64: the A stream is then read once per 64
// sampled rows) on the 128-row tile, and smaller tiles, rows first, until there
// are two workgroups per CU (m < 0: any large m).
int f64_default_id(int64_t m, int32_t sb)
{
    int tm = 2, tn = sb <= 16 ? 1 : (sb <= 32 ? 2 : 4);
    if (m >= 0 && tiles_of(m, sb, tm, tn) < 512) tm = 1;
    while (m >= 0 && tn > 1 && tiles_of(m, sb, tm, tn) < 512) tn /= 2;
    if (tn == 4) return tm == 2 ? 5 : 2;
    if (tn == 2) return tm == 2 ? 1 : 7;
    return tm == 2 ? 0 : 8;
}

int f64_config_id(int64_t m, int64_t n, int32_t sb)
{
    const int id = tune_lookup(KDCD_F64, n, sb);
    return (id >= 0 && id < kF64NumCfgs) ? id : f64_default_id(m, sb);
}

// The same for the batched launch, where the column sums and betas of every
// problem sit in LDS: 128 rows of them leave room for two workgroups per CU up
// to 20 problems (200000 x 1024, 512 sampled rows, four sigmas, 18 problems: 4.13 ms
// with 128 x 64 tiles against 4.49 with 64 x 64, and 4.96 when only one 128 x 64
// workgroup fits a CU; 5.64 for the LDS-staged tiles).
static int f64_batch_default_id(int64_t m, int32_t sb, int32_t nprob)
{
    int tn = sb <= 16 ? 1 : (sb <= 32 ? 2 : 4);
    if (tn == 4 && nprob <= 20 && (m < 0 || tiles_of(m, sb, 2, 4) >= 256)) return 3;
    while (m >= 0 && tn > 1 && tiles_of(m, sb, 1, tn) < 256) tn /= 2;
    return tn == 4 ? 2 : (tn == 2 ? 4 : 5);
}

int f64_batch_config_id(int64_t m, int64_t n, int32_t sb, int32_t nprob)
{
    const int id = tune_lookup(KDCD_F64 + KDCD_TUNE_BATCH, n, sb);
    return (id >= 0 && id < kF64BatchNumCfgs) ? id : f64_batch_default_id(m, sb, nprob);
}

int64_t kblock_f64_row_groups(int cfg, int64_t m, int64_t n, int32_t sb, bool batch)
{
    F64Cfg c;
    if (batch)
        c = kF64BatchCfgs[cfg >= 0 && cfg < kF64BatchNumCfgs ? cfg
                                                            : f64_batch_config_id(m, n, sb, kMaxProblems)];
    else
        c = kF64Cfgs[cfg >= 0 && cfg < kF64NumCfgs ? cfg : f64_config_id(m, n, sb)];
    return streamed_row_groups(c.tm, c.tn, m, n, sb);
}

// The three parts of a single-problem launch: the row-position update of the
// gathered-Gram mode, the product, and the copies of repeated Gram rows.
hipError_t launch_kblock_f64_pre(const KBlockArgs &a, hipStream_t st)
{
    if (a.batch || !(a.W && a.pos && !a.w_only)) return hipSuccess;
    hipLaunchKernelGGL(pos_set_kernel, dim3(1), dim3(1024), 0, st, a.pos, a.A->m, a.prevS,
                       a.prevS ? a.prev_sb : 0, a.S, a.sb, a.stop);
    return hipGetLastError();
}

hipError_t launch_kblock_f64_main(const KBlockArgs &a, hipStream_t st)
{
    const kdcd_matrix *A = a.A;
    if (a.batch) {
        const int np = a.batch_nprob > 0 ? a.batch_nprob : kMaxProblems;
        switch (a.cfg >= 0 && a.cfg < kF64BatchNumCfgs ? a.cfg : f64_batch_config_id(A->m, A->n, a.sb, kMaxProblems)) {
        case 0: return launch_tiles<4, 2, 1, true, 3>(a, st, np);
        case 1: return launch_tiles<4, 2, 2, true, 2>(a, st, np);
        case 3: return launch_tiles<4, 2, 4, true, 2>(a, st, np);
        case 4: return launch_tiles<4, 1, 2, true, 3>(a, st, np);
        case 5: return launch_tiles<4, 1, 1, true, 3>(a, st, np);
        default: return launch_tiles<4, 1, 4, true, 3>(a, st, np);
        }
    }
    KBlockArgs b = a;
    if (!(a.W && a.pos && !a.w_only)) b.pos = nullptr;
    switch (a.cfg >= 0 && a.cfg < kF64NumCfgs ? a.cfg : f64_config_id(A->m, A->n, a.sb)) {
    case 0: return launch_tiles<4, 2, 1, false, 4>(b, st);
    case 1: return launch_tiles<4, 2, 2, false, 3>(b, st);
    case 3:
    case 4: return launch_tiles<4, 1, 8, false, 2>(b, st);
    case 5: return launch_tiles<4, 2, 4, false, 2>(b, st);
    case 7: return launch_tiles<4, 1, 2, false, 4>(b, st);
    case 8: return launch_tiles<4, 1, 1, false, 4>(b, st);
    default: return launch_tiles<4, 1, 4, false, 3>(b, st);
    }
}

hipError_t launch_kblock_f64_post(const KBlockArgs &a, hipStream_t st)
{
    if (a.batch || !(a.W && a.pos && !a.w_only)) return hipSuccess;
    hipLaunchKernelGGL(w_dup_kernel, dim3((unsigned)a.sb), dim3(256), 0, st, a.W, a.A->m, a.S, a.sb,
                       a.pos, a.stop);
    return hipGetLastError();
}

hipError_t launch_kblock_f64(const KBlockArgs &a, hipStream_t st)
{
    hipError_t e = launch_kblock_f64_pre(a, st);
    if (e == hipSuccess) e = launch_kblock_f64_main(a, st);
    if (e == hipSuccess) e = launch_kblock_f64_post(a, st);
    return e;
}

}  // namespace kdcd
