// K-SVM on small dense problems: all outer iterations in one launch.
//
// A small outer iteration (2000 x 64, s = 1: 1 MB of A, 0.3 MFLOP) is two or three
// kernels that wait for each other: 12.9 us, nearly all of it launches, first
// loads and drained pipelines.  Here one cooperative launch keeps G = ceil(m/64)
// workgroups on the chip for the whole solve.  Workgroup g holds rows 64 g ..
// 64 g + 63 of A in registers and their beta = alpha y in LDS; per outer iteration
// it forms its rows' part of r, publishes it, forms the Gram of the sampled rows
// while the other parts arrive, sums all parts, and runs the recurrence --
// every workgroup the same one, so nothing but the parts of r is exchanged.
//
// Exchange: one 8-byte word per (workgroup, sampled row), written with an agent-scope
// atomic store and polled with agent-scope atomic loads: the word is its own
// flag, since an empty slot holds a signalling NaN that no sum can be.  Three slots
// alternate.  When a workgroup has read all of slot k, every workgroup has
// published k and so has read all of k - 1: it empties its own words of k - 1, waits
// for those stores, and only then publishes k + 1; a reader reaches slot k + 2 (the
// same memory as k - 1) only after it has seen every k + 1, so it never meets an old
// word.  alpha itself is kept by workgroup 0, one block late: it writes block k - 1's
// updates, past the caches, when it has read all of slot k (by then every workgroup
// has read what it needed for block k - 1), and before it publishes k + 1.  A
// workgroup that has read slot k therefore finds in memory every update up to
// block k - 2, and takes those of block k - 1 from its own recurrence.  The last block's
// updates are written when every workgroup has acknowledged its last read.
//
// Every wait ends: the launch is cooperative (all workgroups resident, or the
// launch is refused and the solve takes its ordinary launches), and a poll gives
// up after max_polls rounds (kPersistPolls; 0: at once), which makes this workgroup (and so, in the same way, the
// others) return; the host then restores alpha and runs the ordinary launches.
//
// What bounds it: the exchange (store past the caches, poll, about 2 us) and the chain
// behind it -- 16 dependent MFMAs per 64 columns, the map, three workgroup barriers, the
// recurrence.  Measured per outer iteration, ordinary launches against this: 2000 x 64,
// s = 1 / 8 / 16: 12.9 / 13.4 / 14.0 -> 5.0 / 6.6 / 8.3 us; 2000 x 256, s = 1: 15.7 -> 9.6;
// 20000 x 64, s = 8: 15.1 -> 9.6.  The cooperative launch and the exchange memory cost
// 20 us more per solve.  With 64 sampled rows the recurrence of one wave (LDS reads in
// its chain) takes what the launches did, so s <= 32.
//
// All sums are formed in the order of the ordinary launches (the 64-row tiles of
// the FP64 product, the finish pass's 32 partitions, the recurrence's steps), so the
// iterate has the same bits.
#include "common.hpp"
#include "dcd_step.hpp"
#include "exp_tab.hpp"
#include "svm_persist.hpp"

namespace kdcd {
namespace {

typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));

constexpr int NT = 256;
constexpr int BK = 16;
constexpr int FIN_COLS = 8, FIN_PARTS = 32;      // the finish pass's reduction
constexpr int kMaxWords = 4096;                  // G * s
constexpr uint64_t kEmpty = 0x7ff4dead7ff4deadull;
static_assert((uint32_t)kPersistEmptyWord == (uint32_t)kEmpty, "slots are filled by halves");

__device__ __forceinline__ int64_t clampi(int64_t v, int64_t lo, int64_t hi)
{
    return v < lo ? lo : (v > hi ? hi : v);
}

__device__ __forceinline__ void put(uint64_t *p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t get(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Every store of this wave has reached the agent's coherence point.
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// CB blocks of 16 sampled rows, at most NC chunks of 16 columns.
template <int CB, int NC, int KIND>
__global__ __launch_bounds__(NT) void svm_persist_kernel(
    const double *__restrict__ A, int64_t lda, int64_t m, int64_t n, const double *__restrict__ y,
    const double *__restrict__ norms, KParams kp, double nu, double omega, int32_t s, int64_t H,
    const int32_t *__restrict__ idx, double *alpha, double *__restrict__ trace, uint64_t *slots,
    int32_t *status, int32_t max_polls)
{
    constexpr int SBP = CB * 16;
    constexpr int PF = CB * NC / 4;              // 4-double segments of the sampled rows per thread
    __shared__ d2 Bs[NC][CB * 2 * 64];           // sampled rows, fragment-major chunks
    __shared__ double Wl[SBP * SBP];
    __shared__ double pv[kMaxWords];             // the parts of r
    __shared__ double sh[SBP / FIN_COLS * NT];
    __shared__ double red[4][SBP];
    __shared__ double bsh[64], nsh[64], ysh[64];
    __shared__ int32_t Sl[3][SBP];
    __shared__ d2 etab[KIND == KDCD_KERNEL_RBF ? kExpTab : 1];
    __shared__ int32_t dead;

    if (*status != 0) return;                    // the validation has failed (same for all)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = gridDim.x, g = blockIdx.x;
    const int64_t row0 = (int64_t)g * 64;
    const int nC = (int)((n + BK - 1) / BK);
    const int64_t n_outer = (H + s - 1) / s;
    if (KIND == KDCD_KERNEL_RBF) exp_tab_load(etab);
    if (tid == 0) dead = 0;
    if (tid < 64) {
        const int64_t r = clampi(row0 + tid, 0, m - 1);
        ysh[tid] = y[r];
        bsh[tid] = row0 + tid < m ? alpha[r] * ysh[tid] : 0.0;
        nsh[tid] = KIND == KDCD_KERNEL_RBF ? norms[r] : 0.0;
    }
    // this wave's 16 rows
    d2 ra[NC][2];
    {
        const double *ap = A + clampi(row0 + wid * 16 + (lane & 15), 0, m - 1) * lda + 4 * (lane >> 4);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if ((c + 1) * BK <= n) {
                const d2u *p = reinterpret_cast<const d2u *>(ap + c * BK);
                ra[c][0] = p[0];
                ra[c][1] = p[1];
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    ra[c][e >> 1][e & 1] = c * BK + 4 * (lane >> 4) + e < n ? ap[c * BK + e] : 0.0;
            }
        }
    }
    // segments of the sampled rows this thread stages: row, first column
    int pr[PF], pk[PF];
#pragma unroll
    for (int i = 0; i < PF; ++i) {
        const int seg = tid + i * NT, per = 4 * nC;
        pr[i] = seg / per;
        pk[i] = 4 * (seg - pr[i] * per);
    }
    d2 rb[PF][2];
    auto fetch = [&](const int32_t *S) {         // rows of the block whose indices are in S (LDS)
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            if (pr[i] >= SBP) continue;
            const double *p = A + (int64_t)S[pr[i]] * lda + pk[i];
            if (pk[i] + 4 <= n) {
                const d2u *q = reinterpret_cast<const d2u *>(p);
                rb[i][0] = q[0];
                rb[i][1] = q[1];
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) rb[i][e >> 1][e & 1] = pk[i] + e < n ? p[e] : 0.0;
            }
        }
    };
    auto stage = [&] {
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            if (pr[i] >= SBP) continue;
            d2 *dst = &Bs[pk[i] >> 4][((pr[i] >> 4) * 2) * 64 + ((pk[i] >> 2) & 3) * 16 + (pr[i] & 15)];
            dst[0] = rb[i][0];
            dst[64] = rb[i][1];
        }
    };
    // indices of block k for element `lane` (wave 0), clamped like every index read
    auto index = [&](int64_t k) -> int32_t {
        const int64_t e = k * s + lane;
        return lane < SBP ? (int32_t)clampi(idx[clampi(lane < s ? e : k * s, 0, H - 1)], 0, m - 1) : 0;
    };
    if (wid == 0 && lane < SBP) {
        Sl[0][lane] = index(0);
        Sl[1][lane] = index(n_outer > 1 ? 1 : 0);
    }
    __syncthreads();
    fetch(Sl[0]);
    stage();
    __syncthreads();

    // wave 0, lane t: coordinate t of the block before (-1: none, or not its last
    // occurrence) and its new alpha
    int32_t prevS = -1;
    double prevA = 0.0;
    for (int64_t k = 0; k < n_outer; ++k) {
        const int sb = (int)(k + 1 < n_outer ? (int64_t)s : H - k * s);
        const int32_t *S = Sl[k % 3];
        uint64_t *slot = slots + (k % 3) * (int64_t)G * s;

        // product of this wave's rows with the sampled rows
        d4 acc[CB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) acc[cb] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (c < nC) {                        // uniform
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    d2 b[CB];
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) b[cb] = Bs[c][(cb * 2 + h) * 64 + lane];
#pragma unroll
                    for (int e = 0; e < 2; ++e)
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb)
                            acc[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(ra[c][h][e], b[cb][e], acc[cb], 0, 0, 0);
                }
            }
        }
        int32_t Sc[CB];
        double nb[CB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            Sc[cb] = S[cb * 16 + (lane & 15)];
            nb[cb] = KIND == KDCD_KERNEL_RBF ? norms[Sc[cb]] : 0.0;
        }
        double colsum[CB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) colsum[cb] = 0.0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int t = wid * 16 + (lane >> 4) + 4 * v;
            if (row0 + t >= m) continue;
            const double bval = bsh[t], na = nsh[t];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                if (cb * 16 + (lane & 15) < sb) {
                    const double kv = kernel_map_tab<KIND>(acc[cb][v], na, nb[cb],
                                                           (int32_t)(row0 + t) == Sc[cb], kp, etab);
                    colsum[cb] += bval * kv;
                }
        }
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const double v = wave_sum_xor16_32(colsum[cb]);
            if (lane < 16) red[wid][cb * 16 + lane] = v;
        }
        __syncthreads();
        if (tid < sb) {                          // wave 0: publish
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < 4; ++w) t += red[w][tid];
            uint64_t bits = (uint64_t)__double_as_longlong(t);
            if (bits == kEmpty) bits ^= 1;       // (some other NaN)
            stores_done();                       // alpha of block k - 1, emptied words of k - 2
            put(&slot[(int64_t)g * sb + tid], bits);
        }

        // next block's rows, and the indices of the one after, on their way
        const bool more = k + 1 < n_outer;
        if (more) fetch(Sl[(k + 1) % 3]);
        int32_t inext = 0;
        if (wid == 0 && k + 2 < n_outer) inext = index(k + 2);

        // Gram of the sampled rows: row block wid
        if (wid < CB) {
            d4 wacc[CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) wacc[cb] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                if (c < nC) {                    // uniform
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const d2 a = Bs[c][(wid * 2 + h) * 64 + lane];
                        d2 b[CB];
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb) b[cb] = Bs[c][(cb * 2 + h) * 64 + lane];
#pragma unroll
                        for (int e = 0; e < 2; ++e)
#pragma unroll
                            for (int cb = 0; cb < CB; ++cb)
                                wacc[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[e], b[cb][e], wacc[cb], 0, 0, 0);
                    }
                }
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int t = wid * 16 + (lane >> 4) + 4 * v;
                const int32_t St = S[t];
                const double na = KIND == KDCD_KERNEL_RBF ? norms[St] : 0.0;
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
                    Wl[t * SBP + cb * 16 + (lane & 15)] =
                        kernel_map_tab<KIND>(wacc[cb][v], na, nb[cb], St == Sc[cb], kp, etab);
            }
        }

        // all parts of r
        const int words = G * sb;
        for (int x0 = tid; x0 < words; x0 += 8 * NT) {
            uint64_t v[8];
            int polls = 0;
            bool open;
            do {
                open = false;
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = x0 + u * NT < words ? get(&slot[x0 + u * NT]) : 0;
#pragma unroll
                for (int u = 0; u < 8; ++u) open |= v[u] == kEmpty;
            } while (open && ++polls < max_polls);
            if (open || max_polls == 0) dead = 1;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (x0 + u * NT < words) pv[x0 + u * NT] = __longlong_as_double((long long)v[u]);
        }
        __syncthreads();
        if (dead) {                              // a part never came: the host starts over
            if (tid == 0) set_status(status, kPersistGaveUp);
            return;
        }
        double rho = 0.0, yj = 0.0;
        int32_t Sj = -1;
        if (wid == 0) {
            if (k > 0 && lane < s) put(&slots[((k - 1) % 3) * (int64_t)G * s + (int64_t)g * s + lane], kEmpty);
            uint64_t *av = reinterpret_cast<uint64_t *>(alpha);
            if (g == 0 && prevS >= 0) put(av + prevS, (uint64_t)__double_as_longlong(prevA));
            if (lane < sb) {
                Sj = S[lane];
                yj = y[Sj];
                rho = __longlong_as_double((long long)get(av + Sj));
            }
            if (!more) {                         // the last read of alpha is done
                stores_done();
                if (lane == 0) put(&slots[(n_outer % 3) * (int64_t)G * s + g], 0);
            }
            if (k > 0)
                for (int t = 0; t < s; ++t) {
                    const double pa = readlane_d(prevA, t);
                    if (__builtin_amdgcn_readlane(prevS, t) == Sj) rho = pa;
                }
        }
        {
            const int c = tid % FIN_COLS, part = tid / FIN_COLS;
            for (int cg = 0; cg * FIN_COLS < sb; ++cg) {
                const int col = cg * FIN_COLS + c;
                double t = 0.0;
                if (col < sb)
                    for (int q = part; q < G; q += FIN_PARTS) t += pv[q * sb + col];
                sh[cg * NT + part * FIN_COLS + c] = t;
            }
        }
        __syncthreads();

        // recurrence: lane j of wave 0 owns step j
        if (wid == 0) {
            double r = 0.0;
            if (lane < sb)
                for (int q = 0; q < FIN_PARTS; ++q)
                    r += sh[lane / FIN_COLS * NT + q * FIN_COLS + lane % FIN_COLS];
            const bool act = lane < sb;
            const double g0 = act ? yj * r - 1.0 : 0.0;
            const double eta = act ? Wl[lane * SBP + lane] + omega : 1.0;
            const double inv_eta = eta > 0.0 ? 1.0 / eta : 0.0;
            double gacc = 0.0, theta = 0.0;
            bool last = act;
            for (int t = 0; t < sb; ++t) {
                const double coef = (lane > t && lane < sb) ? readlane_d(yj, t) * yj * Wl[t * SBP + lane] : 0.0;
                const bool dup = (lane > t) && __builtin_amdgcn_readlane(Sj, t) == Sj;
                if (__ballot(dup) != 0 && lane == t) last = false;
                const double gr = g0 + gacc + omega * rho;
                const double th = dcd_theta(rho, gr, inv_eta, nu);
                const double tt = readlane_d(th, t);
                if (lane == t) theta = th;
                gacc += coef * tt;
                rho += dup ? tt : 0.0;
            }
            if (act) {
                const double nv = rho + theta;
                if (g == 0) {
                    if (!isfinite(nv)) set_status(status, KDCD_ERR_NONFINITE);
                    if (trace) trace[k * s + lane] = theta;
                }
                prevA = nv;
                const int64_t own = (int64_t)Sj - row0;
                if (last && own >= 0 && own < 64) bsh[own] = nv * ysh[own];
            }
            prevS = last ? Sj : -1;
            if (k + 2 < n_outer && lane < SBP) Sl[(k + 2) % 3][lane] = inext;
        }
        if (more) stage();
        __syncthreads();
    }
    if (g != 0 || wid != 0) return;
    bool late = false;
    for (int q = lane; q < G; q += 64) {
        int polls = 0;
        while (get(&slots[(n_outer % 3) * (int64_t)G * s + q]) == kEmpty && ++polls < max_polls) {}
        late |= polls >= max_polls;
    }
    if (__ballot(late) != 0) {
        if (lane == 0) set_status(status, kPersistGaveUp);
        return;
    }
    if (prevS >= 0) put(reinterpret_cast<uint64_t *>(alpha) + prevS, (uint64_t)__double_as_longlong(prevA));
}

template <int CB, int NC>
const void *kernel_of(int kind)
{
    switch (kind) {
    case KDCD_KERNEL_LINEAR: return reinterpret_cast<const void *>(&svm_persist_kernel<CB, NC, KDCD_KERNEL_LINEAR>);
    case KDCD_KERNEL_POLY: return reinterpret_cast<const void *>(&svm_persist_kernel<CB, NC, KDCD_KERNEL_POLY>);
    default: return reinterpret_cast<const void *>(&svm_persist_kernel<CB, NC, KDCD_KERNEL_RBF>);
    }
}

// The instantiation for s sampled rows and n columns, or null.
const void *pick(int kind, int32_t s, int64_t n)
{
    if (s <= 16) return n <= 64 ? kernel_of<1, 4>(kind) : (n <= 256 ? kernel_of<1, 16>(kind) : nullptr);
    if (s <= 32) return n <= 64 ? kernel_of<2, 4>(kind) : (n <= 256 ? kernel_of<2, 16>(kind) : nullptr);
    return nullptr;
}

}  // namespace

int64_t svm_persist_groups(const kdcd_matrix *A, int kind, int32_t s, int64_t n_outer)
{
    const int64_t G = (A->m + 63) / 64;
    if (A->format != KDCD_DENSE || n_outer < kPersistMinOuter || G * s > kMaxWords) return 0;
    const void *f = pick(kind, s, A->n);
    if (!f) return 0;
    int dev = 0, coop = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, f, NT, 0) != hipSuccess)
        return 0;
    return G <= (int64_t)per * cus ? G : 0;
}

hipError_t launch_svm_persist(const SvmPersistArgs &a, int64_t groups, hipStream_t st)
{
    const kdcd_matrix *A = a.A;
    const void *f = pick(a.kp.kind, a.s, A->n);
    if (!f) return hipErrorInvalidValue;
    const double *Av = A->values;
    int64_t lda = A->ld, m = A->m, n = A->n, H = a.H;
    KParams kp = a.kp;
    double nu = a.nu, omega = a.omega;
    int32_t s = a.s;
    const double *y = a.y, *norms = a.norms;
    const int32_t *idx = a.idx;
    double *alpha = a.alpha, *trace = a.trace;
    uint64_t *slots = a.slots;
    int32_t *status = a.status;
    int32_t polls = a.polls;
    void *args[] = {&Av, &lda, &m, &n, &y, &norms, &kp, &nu, &omega, &s, &H, &idx, &alpha, &trace, &slots, &status, &polls};
    return hipLaunchCooperativeKernel(f, dim3((unsigned)groups), dim3(NT), args, 0, st);
}

}  // namespace kdcd
