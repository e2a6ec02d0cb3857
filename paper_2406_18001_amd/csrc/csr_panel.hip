// CSR kernel block through a dense panel of the sampled rows (gfx950).
//
// For sparse A the product P = A A_S^T has few useful multiply-adds (nnz of A
// times the sampled rows that store an entry's column) and should cost one
// pass over the CSR arrays.  Per chunk of LPR <= 64 sampled rows three
// launches form it:
//
//   claim    every distinct column of the chunk takes a panel row (an id), and
//            its code word -- the build's epoch and the id -- is written to a
//            table with one word per column of A; the panel row is filled with
//            the "absent" value -0.0;
//   scatter  the sampled rows' values go to panel[id][j];
//   product  every stored entry of A looks its column up (4 bytes, mostly L2
//            hits); the entries whose column is in the panel are compacted into
//            an LDS list of (value, panel row) per wave, and the lanes of a
//            wave -- lane = sampled row, 64 / LPR entries at a time -- walk the
//            list with one coalesced panel read and one FMA per entry.
//
// What bounds it: the panel reads, LPR * 8 bytes per hit through L1 / L2 (news20
// recipe, 64 sampled rows: 5.5e6 hits * 512 B = 2.8 GB against 110 MB of CSR
// arrays).  Measured there, per pass over 64 sampled rows: product 267 us (3.9 GB
// of L2 requests at 14.5 TB/s, 0.8 GB past L2), claim 14, scatter 8; the chunked
// LDS hash it replaces took 2310 us (one pass over A per 3072 stored entries of the
// sampled rows, a table build in every workgroup each time), and with 1 / 8 / 32
// sampled rows 124 / 457 / 1124 us per outer iteration against 117 / 144 / 206.
//
// Taken from 112 stored entries a row on average: below, the per-row work (a join
// of the lanes, the map, the next row's hits) outweighs what the list saves.  At
// 50000 x 50000 with rows of 100 entries an outer iteration with 1 / 16 / 32 / 64
// sampled rows takes 58 / 72 / 100 / 156 us against 40 / 102 / 81 / 149 with the
// broadcast and dense-head kernels; with rows of 130, 70 / 87 / 128 / 198 against
// 85 / 132 / 524 / 1024.  From there on csr_takes_panel (kblock_csr.hip) decides.
//
// Ids are handed out by an atomic counter and differ from run to run, but a
// row's sum only depends on its own entries' order: hit i of a row goes to lane
// group i mod (64 / LPR), the groups meet in a fixed xor tree.  Results are
// deterministic.
//
// Rows are dealt to waves in ranges of equal weight (entries + a constant per
// row; bounds found once per solve), so rows of uneven length balance; a row of
// more than kLongRow entries is walked by all waves of its workgroup.
#include <algorithm>

#include "common.hpp"
#include "csr_panel.hpp"

namespace kdcd {
namespace {

constexpr int PP_NT = 512;                   // threads of a product workgroup
constexpr int PP_NW = PP_NT / 64;
constexpr int PP_MAXGROUPS = 1024;           // four workgroups per CU
constexpr int PP_E = 4;                      // entries per lane per batch
constexpr int PP_BATCH = 64 * PP_E;          // entries of a wave's batch
constexpr int PP_ROWCOST = 16;               // weight of a row beside its entries
// panel reads in flight per lane (few where a step takes many entries)
constexpr int pp_un(int G) { return G >= 4 ? 16 / G : 8; }
constexpr int64_t kLongRow = 2048;           // entries from which a workgroup shares a row
constexpr double kLongRowsMinAvg = 112.0;    // average row length from which this path is taken
constexpr int PP_FBGROUPS = 128;             // row groups of the broadcast fallback
// code word: epoch << 20 | id
constexpr int PP_IDBITS = 20;
constexpr uint32_t PP_IDMASK = (1u << PP_IDBITS) - 1u;
constexpr uint32_t PP_EPOCHS = (1u << (32 - PP_IDBITS)) - 1u;   // epochs 1 .. PP_EPOCHS
// Code words of other epochs are not in the panel.  Every build clears the
// stale words of one slice of the table, so no word lives until its epoch
// number comes round again (a slice is cleared at least every 2047 builds).
constexpr uint32_t PP_SLICES = 1024;
static_assert(2 * PP_SLICES < PP_EPOCHS, "a slice is cleared before an epoch recurs");

struct PanelMeta {
    uint32_t epoch;      // epoch of the panel (0: none built since the init)
    int32_t fallback;    // 1: the chunk's columns exceed the panel
    uint32_t count;      // ids handed out by the build under way
    uint32_t ticket;     // scatter workgroups that are done
};

struct PanelPtrs {
    PanelMeta *meta;
    uint32_t *code;      // n
    int32_t *bound;      // PP_MAXGROUPS * PP_NW + 1 row bounds of the product's waves
    double *panel;       // cap rows of LPR values
};

__host__ __device__ inline size_t pp_al(size_t x) { return (x + 255) & ~size_t(255); }

__host__ __device__ inline size_t pp_fixed_bytes(int64_t n)
{
    return 256 + pp_al(sizeof(uint32_t) * (size_t)n) +
           pp_al(sizeof(int32_t) * (PP_MAXGROUPS * PP_NW + 1));
}

__host__ __device__ inline PanelPtrs pp_ptrs(void *base, int64_t n)
{
    char *p = static_cast<char *>(base);
    PanelPtrs q;
    q.meta = reinterpret_cast<PanelMeta *>(p); p += 256;
    q.code = reinterpret_cast<uint32_t *>(p); p += pp_al(sizeof(uint32_t) * (size_t)n);
    q.bound = reinterpret_cast<int32_t *>(p);
    p += pp_al(sizeof(int32_t) * (PP_MAXGROUPS * PP_NW + 1));
    q.panel = reinterpret_cast<double *>(p);
    return q;
}

__device__ __forceinline__ int64_t clampi(int64_t v, int64_t lo, int64_t hi)
{
    return v < lo ? lo : (v > hi ? hi : v);
}

__device__ __forceinline__ uint32_t next_epoch(uint32_t e) { return e >= PP_EPOCHS ? 1u : e + 1u; }

// Once per solve: no column in the panel, and the rows each product wave takes
// (the first row whose weight before it reaches the wave's share).
__global__ __launch_bounds__(256) void pp_init_kernel(void *base, int64_t n,
                                                      const int64_t *__restrict__ row_ptr,
                                                      int64_t m, int64_t nnz, int32_t nwaves)
{
    const PanelPtrs q = pp_ptrs(base, n);
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    for (int64_t c = i; c < n; c += (int64_t)gridDim.x * 256) q.code[c] = 0u;
    if (i == 0) *q.meta = PanelMeta{0u, 0, 0u, 0u};
    for (int64_t w = i; w <= nwaves; w += (int64_t)gridDim.x * 256) {
        int64_t lo = 0, hi = m;
        const double want = ((double)nnz + (double)PP_ROWCOST * (double)m) * (double)w / nwaves;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if ((double)clampi(row_ptr[mid], 0, nnz) + (double)PP_ROWCOST * (double)mid < want)
                lo = mid + 1;
            else
                hi = mid;
        }
        q.bound[w] = (int32_t)(w == 0 ? 0 : (w == nwaves ? m : lo));
    }
}

// Workgroup (j, part): entries part * 256 + tid, ... of sampled row j.
template <int LPR>
__global__ __launch_bounds__(256) void pp_claim_kernel(const int64_t *__restrict__ row_ptr,
                                                       const int32_t *__restrict__ col_idx,
                                                       int64_t m, int64_t nnz, int64_t n,
                                                       const int32_t *__restrict__ S, uint32_t cap,
                                                       void *base)
{
    const PanelPtrs q = pp_ptrs(base, n);
    const int lane = threadIdx.x & 63;
    const uint32_t epoch = next_epoch(q.meta->epoch);
    const int64_t r = clampi(S[blockIdx.x], 0, m - 1);
    const int64_t e0 = clampi(row_ptr[r], 0, nnz), e1 = clampi(row_ptr[r + 1], 0, nnz);
    const int64_t step = (int64_t)gridDim.y * 256;
    for (int64_t w0 = e0 + (int64_t)blockIdx.y * 256 + (threadIdx.x & ~63); w0 < e1; w0 += step) {
        const int64_t e = w0 + lane;
        const int32_t c = e < e1 ? col_idx[e] : -1;
        bool won = false;
        if (c >= 0 && c < n) {
            uint32_t w = __hip_atomic_load(&q.code[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            // a failed exchange means that another entry of the column has claimed it
            if ((w >> PP_IDBITS) != epoch)
                won = atomicCAS(&q.code[c], w, epoch << PP_IDBITS) == w;
        }
        const uint64_t winners = __ballot(won);
        if (winners == 0) continue;
        uint32_t first = 0;
        if (lane == 0) first = atomicAdd(&q.meta->count, (uint32_t)__popcll(winners));
        first = __shfl(first, 0);
        const uint32_t id = first + (uint32_t)__popcll(winners & ((1ull << lane) - 1ull));
        if (won)
            __hip_atomic_store(&q.code[c], epoch << PP_IDBITS | min(id, PP_IDMASK), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t last = min(first + (uint32_t)__popcll(winners), cap);
        for (int64_t x = (int64_t)first * LPR + lane; x < (int64_t)last * LPR; x += 64)
            q.panel[x] = -0.0;
    }
}

// The sampled rows' values into the panel (a stored -0.0 as +0.0: -0.0 marks
// absent entries); the last workgroup closes the build.
template <int LPR>
__global__ __launch_bounds__(256) void pp_scatter_kernel(const int64_t *__restrict__ row_ptr,
                                                         const int32_t *__restrict__ col_idx,
                                                         const double *__restrict__ val, int64_t m,
                                                         int64_t nnz, int64_t n,
                                                         const int32_t *__restrict__ S,
                                                         uint32_t cap, void *base)
{
    const PanelPtrs q = pp_ptrs(base, n);
    const uint32_t epoch = next_epoch(q.meta->epoch);
    const uint32_t count = q.meta->count;
    if (count <= cap) {
        const int64_t r = clampi(S[blockIdx.x], 0, m - 1);
        const int64_t e0 = clampi(row_ptr[r], 0, nnz), e1 = clampi(row_ptr[r + 1], 0, nnz);
        for (int64_t e = e0 + (int64_t)blockIdx.y * 256 + threadIdx.x; e < e1;
             e += (int64_t)gridDim.y * 256) {
            const int32_t c = col_idx[e];
            if (c < 0 || c >= n) continue;
            const uint32_t id = q.code[c] & PP_IDMASK;
            const double v = val[e];
            if (id < cap) q.panel[(int64_t)id * LPR + blockIdx.x] = v == 0.0 ? 0.0 : v;
        }
    }
    const int64_t slice = (n + PP_SLICES - 1) / PP_SLICES;
    const int64_t c0 = (int64_t)((epoch - 1u) % PP_SLICES) * slice;
    const int64_t c1 = min(c0 + slice, n);
    for (int64_t c = c0 + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x; c < c1;
         c += (int64_t)gridDim.x * gridDim.y * 256)
        if ((q.code[c] >> PP_IDBITS) != epoch) q.code[c] = 0u;
    __syncthreads();
    if (threadIdx.x == 0) {
        // every workgroup has read the meta block before it takes its ticket
        const uint32_t t = atomicAdd(&q.meta->ticket, 1u);
        if (t + 1u == gridDim.x * gridDim.y) {
            q.meta->epoch = epoch;
            q.meta->fallback = count > cap ? 1 : 0;
            q.meta->count = 0u;
            q.meta->ticket = 0u;
        }
    }
}

// Workgroups [0, n_row_groups): the waves' row ranges, reduced against beta;
// the others: one sampled row each against the panel (the Gram W).
template <int LPR, int KIND>
__global__ __launch_bounds__(PP_NT) __attribute__((amdgpu_waves_per_eu(KIND == KDCD_KERNEL_RBF ? 5 : 6))) void pp_product_kernel(
    const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ col_idx,
    const double *__restrict__ val, int64_t m, int64_t nnz, int64_t n,
    const int32_t *__restrict__ S, int32_t sb, int32_t j0, int32_t nj,
    const double *__restrict__ norms, KParams kp, const double *__restrict__ beta,
    const double *__restrict__ bscale, double *__restrict__ partial, double *__restrict__ W,
    int32_t n_row_groups, int32_t fb_groups, const void *__restrict__ pbase, double *__restrict__ U)
{
    constexpr int G = 64 / LPR;                   // entries per step
    constexpr int UN = pp_un(G);
    __shared__ double lval[PP_NW][PP_BATCH];
    __shared__ uint32_t loff[PP_NW][PP_BATCH];
    __shared__ double red[PP_NW][64];
    const PanelPtrs q = pp_ptrs(const_cast<void *>(pbase), n);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane / LPR, jl = lane % LPR;
    const bool is_w = (int)blockIdx.x >= n_row_groups;
    if (q.meta->fallback) {
        // the broadcast kernel runs this chunk on its first fb_groups row
        // groups; the other groups' sums for it are zero
        if (!is_w && (int)blockIdx.x >= fb_groups && tid < nj)
            partial[(int64_t)blockIdx.x * sb + j0 + tid] = 0.0;
        return;
    }
    const uint32_t epoch = q.meta->epoch;
    const uint32_t nlast = (uint32_t)(n - 1);
    const bool jok = jl < nj;
    const int64_t Sj = clampi(S[j0 + (jok ? jl : 0)], 0, m - 1);
    const double nb = (KIND == KDCD_KERNEL_RBF) ? norms[Sj] : 0.0;
    auto rp = [&](int64_t r) { return clampi(row_ptr[clampi(r, 0, m)], 0, nnz); };
    const char *prow = reinterpret_cast<const char *>(q.panel) + 8 * jl;
    double *wval = lval[wid];
    uint32_t *woff = loff[wid];

    // The wave's current batch: entries [ebeg, ebeg + PP_BATCH) (those below
    // elim), its hits compacted in entry order, hit masks per 64 entries.
    uint64_t mask[PP_E];
    bool odd = false;                             // a hit of the batch is infinite or NaN
    auto load_batch = [&](int64_t ebeg, int64_t elim) {
        int32_t cu[PP_E];
        double vu[PP_E];
        uint32_t cd[PP_E];
#pragma unroll
        for (int u = 0; u < PP_E; ++u) {
            const int64_t e = min(ebeg + 64 * u + lane, nnz - 1);
            cu[u] = col_idx[e];
            vu[u] = val[e];
        }
#pragma unroll
        for (int u = 0; u < PP_E; ++u) cd[u] = q.code[min((uint32_t)cu[u], nlast)];
        wave_lds_sync();                          // the previous batch's reads are done
        uint32_t at = 0;
        bool inf = false;
#pragma unroll
        for (int u = 0; u < PP_E; ++u) {
            const bool hit = ebeg + 64 * u + lane < elim && (uint32_t)cu[u] <= nlast &&
                             (cd[u] >> PP_IDBITS) == epoch;
            mask[u] = __ballot(hit);
            inf |= hit && !__builtin_isfinite(vu[u]);
            if (hit) {
                const uint32_t p = at + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask[u] >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)mask[u], 0u));
                wval[p] = vu[u];
                woff[p] = (cd[u] & PP_IDMASK) * (uint32_t)(LPR * sizeof(double));
            }
            at += (uint32_t)__popcll(mask[u]);
        }
        odd = __ballot(inf) != 0;
        wave_lds_sync();
    };
    // hits among the batch's first x entries (0 <= x <= PP_BATCH, uniform)
    auto hits_before = [&](int x) -> int {
        int c = 0;
#pragma unroll
        for (int u = 0; u < PP_E; ++u) {
            const int k = x - 64 * u;
            if (k >= 64) c += __popcll(mask[u]);
            else if (k > 0) c += __popcll(mask[u] & ((1ull << k) - 1ull));
        }
        return c;
    };
    // acc += the hits [h, h1) of the list, hit h + i by lane group i mod G
    auto walk = [&](int h, int h1, double acc) -> double {
        if (odd) {                                // uniform
            // an infinite or NaN value meets only the rows that store its column
            for (int i = h; i < h1; i += G) {
                const int k = min(i + g, h1 - 1);
                const double a = wval[k];
                const double b = *reinterpret_cast<const double *>(prow + woff[k]);
                if (i + g < h1 && __double_as_longlong(b) != INT64_MIN) acc = fma(a, b, acc);
            }
            return acc;
        }
        int i = h;
        for (; i + G * UN <= h1; i += G * UN) {
            double a[UN], b[UN];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                a[u] = wval[i + G * u + g];
                b[u] = *reinterpret_cast<const double *>(prow + woff[i + G * u + g]);
            }
#pragma unroll
            for (int u = 0; u < UN; ++u) acc = fma(a[u], b[u], acc);
        }
        if (i < h1) {
            double a[UN], b[UN];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int k = min(i + G * u + g, h1 - 1);
                a[u] = wval[k];
                b[u] = *reinterpret_cast<const double *>(prow + woff[k]);
            }
#pragma unroll
            for (int u = 0; u < UN; ++u) acc = i + G * u + g < h1 ? fma(a[u], b[u], acc) : acc;
        }
        return acc;
    };
    auto join = [&](double acc) -> double {
#pragma unroll
        for (int o = LPR; o < 64; o <<= 1) acc += __shfl_xor(acc, o);
        return acc;
    };
    double colsum = 0.0;
    // one row's entries [e0, e1), shared by the workgroup's waves; the sum is
    // returned to every lane (of wave 0 also used)
    auto shared_row = [&](int64_t e0, int64_t e1) -> double {
        const int64_t per = ((e1 - e0 + PP_NW - 1) / PP_NW + 63) & ~int64_t(63);
        const int64_t b0 = min(e0 + wid * per, e1), b1 = min(b0 + per, e1);
        double acc = 0.0;
        for (int64_t e = b0; e < b1; e += PP_BATCH) {
            load_batch(e, b1);
            acc = walk(0, hits_before(PP_BATCH), acc);
        }
        acc = join(acc);
        __syncthreads();
        red[wid][lane] = acc;
        __syncthreads();
        double t = 0.0;
        for (int w = 0; w < PP_NW; ++w) t += red[w][jl];
        return t;
    };

    if (is_w) {
        if (W == nullptr) return;
        const int t = (int)blockIdx.x - n_row_groups;
        const int64_t row = clampi(S[t], 0, m - 1);
        const double p = shared_row(rp(row), max(rp(row), rp(row + 1)));
        const double na = (KIND == KDCD_KERNEL_RBF) ? norms[row] : 0.0;
        if (tid < nj) W[(int64_t)t * sb + j0 + tid] = kernel_map<KIND>(p, na, nb, row == Sj, kp);
        return;
    }

    const int64_t ra = q.bound[blockIdx.x * PP_NW + wid];
    const int64_t rb = q.bound[blockIdx.x * PP_NW + wid + 1];
    int64_t ebeg = rp(ra), bend = ebeg;           // the batch; entries below bend are in the list
    const int64_t elim = rp(rb);
    int h = 0;                                    // hits used
    int64_t eprev = ebeg;                         // end of the row before
    // sums of finished rows wait in their lane group's register until G rows
    // (consecutive but for long rows) are mapped together
    double pend = 0.0, pb = 0.0, pn = 0.0;
    int64_t prw = -1;
    int slot = 0;
    auto flush = [&]() {
        if (prw >= 0) {
            const double kv = kernel_map<KIND>(pend, pn, nb, prw == Sj, kp);
            colsum += pb * kv;
            if (U && jok) U[(int64_t)(j0 + jl) * m + prw] = kv;
        }
        prw = -1;
        slot = 0;
    };
    for (int64_t w0 = ra; w0 < rb; w0 += 64) {
        // window of 64 rows: lane l holds row w0 + l's end, beta and norm
        const int64_t wr = min(w0 + lane, m - 1);
        const int64_t wend = rp(wr + 1);
        double wb = beta[wr];
        if (bscale) wb *= bscale[wr];
        const double wn = (KIND == KDCD_KERNEL_RBF) ? norms[wr] : 0.0;
        const int cnt = (int)min<int64_t>(64, rb - w0);
        for (int l = 0; l < cnt; ++l) {
            const int64_t e1 = max(eprev, ((int64_t)__builtin_amdgcn_readlane((int)(wend >> 32), l) << 32) |
                                              (uint32_t)__builtin_amdgcn_readlane((int)wend, l));
            if (e1 - eprev > kLongRow) {          // walked by the whole workgroup below
                eprev = e1;
                ebeg = bend = e1;
                h = 0;
                continue;
            }
            double acc = 0.0;
            for (;;) {
                const int x = (int)(min(e1, bend) - ebeg);
                if (x > 0) {
                    const int h1 = hits_before(x);
                    acc = walk(h, h1, acc);
                    h = h1;
                }
                if (e1 <= bend) break;
                ebeg = bend;
                bend = min(ebeg + PP_BATCH, max(elim, e1));
                load_batch(ebeg, bend);
                h = 0;
            }
            eprev = e1;
            acc = join(acc);
            const double bv = __shfl(wb, l), nv = __shfl(wn, l);
            if (g == slot) {
                pend = acc;
                pb = bv;
                pn = nv;
                prw = w0 + l;
            }
            if (++slot == G) flush();
        }
    }
    flush();

    // long rows of the workgroup's range, in row order
    const int64_t ga = q.bound[blockIdx.x * PP_NW], gb = q.bound[(blockIdx.x + 1) * PP_NW];
    for (int64_t w0 = ga; w0 < gb; w0 += 64) {
        const int64_t wr = w0 + lane;
        const bool lng = wr < gb && rp(wr + 1) - rp(wr) > kLongRow;
        for (uint64_t todo = __ballot(lng); todo; todo &= todo - 1) {
            const int64_t row = w0 + __builtin_ctzll(todo);
            const double p = shared_row(rp(row), rp(row + 1));
            if (wid == 0 && g == 0) {
                double bv = beta[row];
                if (bscale) bv *= bscale[row];
                const double na = (KIND == KDCD_KERNEL_RBF) ? norms[row] : 0.0;
                const double kv = kernel_map<KIND>(p, na, nb, row == Sj, kp);
                colsum += bv * kv;
                if (U && jok) U[(int64_t)(j0 + jl) * m + row] = kv;
            }
        }
    }

    colsum = join(colsum);
    __syncthreads();
    red[wid][lane] = colsum;
    __syncthreads();
    if (tid < nj) {
        double s = 0.0;
        for (int w = 0; w < PP_NW; ++w) s += red[w][tid];
        partial[(int64_t)blockIdx.x * sb + j0 + tid] = s;
    }
}

template <int LPR>
hipError_t launch_chunk(const KBlockArgs &a, int32_t j0, int32_t nj, uint32_t cap, int64_t groups,
                        int32_t fb_groups, bool timed, hipStream_t st)
{
    const kdcd_matrix *A = a.A;
    // workgroups per sampled row: a wave takes 64 entries of an average row in
    // about one step (it also fills its columns' panel rows)
    const double avg = A->m > 0 ? (double)A->nnz / (double)A->m : 0.0;
    const unsigned parts = (unsigned)std::min(32.0, std::max(1.0, avg / 64.0));
    dim3 gridb((unsigned)nj, parts);
    hipLaunchKernelGGL((pp_claim_kernel<LPR>), gridb, dim3(256), 0, st, A->row_ptr, A->col_idx, A->m,
                       A->nnz, A->n, a.S + j0, cap, a.csr_panel);
    hipLaunchKernelGGL((pp_scatter_kernel<LPR>), gridb, dim3(256), 0, st, A->row_ptr, A->col_idx,
                       A->values, A->m, A->nnz, A->n, a.S + j0, cap, a.csr_panel);
    dim3 grid((unsigned)(groups + (a.W ? a.sb : 0))), block(PP_NT);
    ArmedEvents armed = armed_events();
    if (!timed) armed_events() = ArmedEvents{nullptr, nullptr};
#define KDCD_PP(KIND)                                                                            \
    KDCD_TIMED_LAUNCH((pp_product_kernel<LPR, KIND>), grid, block, 0, st, A->row_ptr, A->col_idx, \
                      A->values, A->m, A->nnz, A->n, a.S, a.sb, j0, nj, a.norms, a.kp, a.beta,   \
                      a.beta_scale, a.partial, a.W, (int32_t)groups, fb_groups, a.csr_panel, a.U)
    switch (a.kp.kind) {
    case KDCD_KERNEL_LINEAR: KDCD_PP(KDCD_KERNEL_LINEAR); break;
    case KDCD_KERNEL_POLY: KDCD_PP(KDCD_KERNEL_POLY); break;
    default: KDCD_PP(KDCD_KERNEL_RBF); break;
    }
#undef KDCD_PP
    if (!timed) armed_events() = armed;
    return hipGetLastError();
}

}  // namespace

bool csr_long_rows(const kdcd_matrix *A)
{
    return (double)A->nnz >= kLongRowsMinAvg * (double)A->m;
}

int64_t csr_panel_groups(const kdcd_matrix *A)
{
    // at least 16 rows per workgroup, and a batch of entries per wave
    const int64_t byrows = (A->m + 15) / 16;
    const double weight = (double)A->nnz + (double)PP_ROWCOST * (double)A->m;
    const int64_t byload = (int64_t)(weight / (PP_NW * PP_BATCH)) + 1;
    return std::max<int64_t>(1, std::min<int64_t>(std::min(byrows, byload), PP_MAXGROUPS));
}

size_t csr_dense_panel_min_bytes(int64_t n)
{
    return pp_fixed_bytes(n) + pp_al(16 * (size_t)n) + 16128;
}

size_t csr_dense_panel_full_bytes(const kdcd_matrix *A)
{
    const int64_t ids = std::min<int64_t>(std::min<int64_t>(A->n, A->nnz), 1 << 17);
    return pp_fixed_bytes(A->n) + std::max(pp_al(sizeof(double) * 64 * (size_t)ids),
                                           pp_al(16 * (size_t)A->n) + 16128);
}

CsrPanelPlan csr_panel_plan(const KBlockArgs &a)
{
    const kdcd_matrix *A = a.A;
    CsrPanelPlan p{0, 0, false, false};
    const size_t fixed = pp_fixed_bytes(A->n);
    if (!a.csr_panel || a.csr_panel_bytes <= fixed || A->m > INT32_MAX || A->nnz <= 0) return p;
    const int64_t room = (int64_t)((a.csr_panel_bytes - fixed) / sizeof(double));
    const double avg = (double)A->nnz / (double)std::max<int64_t>(A->m, 1);
    int lpr = a.sb <= 8 ? 8 : (a.sb <= 16 ? 16 : (a.sb <= 32 ? 32 : 64));
    for (;; lpr >>= 1) {
        const int64_t cap = std::min<int64_t>(room / lpr, (int64_t)PP_IDMASK);
        const int64_t rows = std::min<int64_t>(lpr, a.sb);
        const int64_t longest = a.csr_max_row >= 0 ? a.csr_max_row : A->n;
        const bool sure = cap >= std::min<int64_t>(A->n, rows * longest);
        // distinct columns are fewer than entries: twice the average rows' share
        const bool likely = (double)cap >= 2.0 * avg * (double)rows;
        if (sure || likely || lpr == 8) {
            p.lpr = lpr;
            p.cap = (uint32_t)cap;
            p.sure = sure;
            p.fits = sure || likely;
            return p;
        }
    }
}

hipError_t launch_csr_dense_panel_init(const kdcd_matrix *A, void *panel, hipStream_t st)
{
    const int32_t nwaves = (int32_t)csr_panel_groups(A) * PP_NW;
    const int64_t blocks = std::min<int64_t>((std::max<int64_t>(A->n, nwaves + 1) + 255) / 256, 2048);
    hipLaunchKernelGGL(pp_init_kernel, dim3((unsigned)std::max<int64_t>(blocks, 1)), dim3(256), 0, st,
                       panel, A->n, A->row_ptr, A->m, A->nnz, nwaves);
    return hipGetLastError();
}

const int32_t *csr_panel_gate(const void *panel)
{
    return &static_cast<const PanelMeta *>(panel)->fallback;
}

int32_t csr_panel_fallback_groups(const kdcd_matrix *A)
{
    return (int32_t)std::min<int64_t>(csr_panel_groups(A), PP_FBGROUPS);
}

hipError_t launch_csr_panel_chunk(const KBlockArgs &a, const CsrPanelPlan &p, int32_t j0, int32_t nj,
                                  bool timed, hipStream_t st)
{
    const int64_t groups = csr_panel_groups(a.A);
    const int32_t fb = csr_panel_fallback_groups(a.A);
    switch (p.lpr) {
    case 8: return launch_chunk<8>(a, j0, nj, p.cap, groups, fb, timed, st);
    case 16: return launch_chunk<16>(a, j0, nj, p.cap, groups, fb, timed, st);
    case 32: return launch_chunk<32>(a, j0, nj, p.cap, groups, fb, timed, st);
    default: return launch_chunk<64>(a, j0, nj, p.cap, groups, fb, timed, st);
    }
}

}  // namespace kdcd
