// The dense-head panel of a chunk of sampled CSR rows: its layout in workspace memory
// and its build, which kblock_csr.hip launches for a chunk on its own and the K-SVM
// recurrence's launch runs for the next index block.
#pragma once

#include "common.hpp"

namespace kdcd {
namespace {

constexpr int HD_NJ = kCsrHeadRows;        // sampled rows per chunk
constexpr int HD_HEAD = 64;                // largest dense head
constexpr int HD_BUILD_NT = 1024;
constexpr int HD_EPT = 4;                  // stored entries per build thread
constexpr int HD_CAP = HD_BUILD_NT * HD_EPT;   // stored entries of one chunk
constexpr int HD_HS = 2 * HD_CAP;          // build hash slots (power of two)
// code word: epoch << HD_EPOCH_SHIFT | HD_HEADBIT (head) | position or offset
constexpr int HD_EPOCH_SHIFT = 13;
constexpr uint32_t HD_HEADBIT = 1u << 12;
constexpr uint32_t HD_VALMASK = HD_HEADBIT - 1u;
constexpr uint32_t HD_EPOCH_END = 1u << (32 - HD_EPOCH_SHIFT);   // epochs 1 .. END-1
static_assert(HD_CAP <= (int)HD_HEADBIT, "tail offsets fit the code word");
static_assert(HD_HEAD <= (int)HD_HEADBIT, "head positions fit the code word");

// A tail column of the current chunk's panel.
struct __align__(16) TailRec {
    uint32_t mask;       // the sampled rows (bits) that store the column
    uint32_t pad;
    double v0;           // value of the first of them (also at tval[offset])
};

struct PanelMeta {
    uint32_t epoch;      // epoch of the last build (0: none since the init)
    int32_t nh;          // head columns
    int32_t fallback;    // 1: the chunk exceeds HD_CAP, the broadcast kernel runs it
    int32_t pad;
};

struct PanelPtrs {
    PanelMeta *meta;
    uint32_t *code;      // n: code word of every column (another epoch: not in the panel)
    TailRec *tail;       // n: set for the tail columns of the current chunk
    double *tval;        // HD_CAP tail values, per column in sampled-row order
    double *Bh;          // HD_HEAD x HD_NJ
};

__host__ __device__ inline size_t hd_al(size_t x) { return (x + 255) & ~size_t(255); }

__host__ __device__ inline PanelPtrs panel_ptrs(void *base, int64_t n)
{
    char *p = static_cast<char *>(base);
    PanelPtrs q;
    q.meta = reinterpret_cast<PanelMeta *>(p); p += 256;
    q.code = reinterpret_cast<uint32_t *>(p); p += hd_al(sizeof(uint32_t) * (size_t)n);
    q.tail = reinterpret_cast<TailRec *>(p); p += hd_al(sizeof(TailRec) * (size_t)n);
    q.tval = reinterpret_cast<double *>(p); p += hd_al(sizeof(double) * HD_CAP);
    q.Bh = reinterpret_cast<double *>(p);
    return q;
}

inline size_t panel_bytes(int64_t n)
{
    return 256 + hd_al(sizeof(uint32_t) * (size_t)n) + hd_al(sizeof(TailRec) * (size_t)n) +
           hd_al(sizeof(double) * HD_CAP) +
           hd_al(sizeof(double) * HD_HEAD * HD_NJ);
}

__device__ __forceinline__ int64_t hd_clamp(int64_t v, int64_t lo, int64_t hi)
{
    return v < lo ? lo : (v > hi ? hi : v);
}

__device__ __forceinline__ uint32_t hd_hash(int32_t c)
{
    return ((uint32_t)c * 2654435761u) & (HD_HS - 1);
}

// The panel of sampled rows S[0 .. nj) (nj <= HD_NJ), one workgroup of HD_BUILD_NT
// threads.  Entry f of the chunk (its rows' stored entries concatenated in
// sampled-row order) is held by thread f % HD_BUILD_NT; the first entry of a column
// numbers it, so head positions and tail offsets follow the chunk's order and do not
// depend on the order of the hash inserts.
struct HeadBuildLds {
    int32_t hkey[HD_HS];
    uint32_t hmask[HD_HS];
    int32_t hcode[HD_HS];       // first entry of the column, then its code
    int64_t rowbeg[HD_NJ];
    int32_t rowoff[HD_NJ + 1];
    __align__(16) int32_t wsum[2][HD_EPT][HD_BUILD_NT / 64];   // (read 16 bytes at a time)
    int32_t hist[HD_NJ + 2];
    int32_t info[1];
};
__device__ __forceinline__ void csr_panel_build(HeadBuildLds &lds, const int64_t *__restrict__ row_ptr,
                                                const int32_t *__restrict__ col_idx,
                                                const double *__restrict__ val, int64_t m, int64_t nnz,
                                                const int32_t *__restrict__ S, int32_t nj, int64_t n, void *base)
{
    constexpr int NWB = HD_BUILD_NT / 64;
    const PanelPtrs q = panel_ptrs(base, n);
    auto &hkey = lds.hkey;
    auto &hmask = lds.hmask;
    auto &hcode = lds.hcode;
    auto &rowoff = lds.rowoff;
    auto &rowbeg = lds.rowbeg;
    auto &wsum = lds.wsum;
    auto &hist = lds.hist;
    auto &info = lds.info;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    auto rp = [&](int64_t r) { return hd_clamp(row_ptr[hd_clamp(r, 0, m)], 0, nnz); };

    // 1. the new epoch (after the last one every record is reset first); empty
    //    hash; entry ranges of the sampled rows
    uint32_t epoch = q.meta->epoch + 1u;
    if (epoch >= HD_EPOCH_END) {
        for (int64_t c = tid; c < n; c += HD_BUILD_NT) q.code[c] = 0u;
        epoch = 1u;
    }
    for (int x = tid; x < HD_HEAD * HD_NJ; x += HD_BUILD_NT) q.Bh[x] = 0.0;
    for (int x = tid; x < HD_HS; x += HD_BUILD_NT) {
        hkey[x] = -1;
        hmask[x] = 0u;
        hcode[x] = INT32_MAX;
    }
    if (tid < HD_NJ + 2) hist[tid] = 0;
    if (wid == 0) {
        int len = 0;
        int64_t b0 = 0;
        if (lane < nj) {
            const int64_t r = hd_clamp(S[lane], 0, m - 1);
            b0 = rp(r);
            len = (int)(rp(r + 1) - b0);
        }
        int incl = len;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(incl, o, 64);
            if (lane >= o) incl += up;
        }
        if (lane < nj) {
            rowoff[lane + 1] = incl;
            rowbeg[lane] = b0;
        }
        if (lane == 0) rowoff[0] = 0;
    }
    __syncthreads();
    const int total = rowoff[nj];
    if (total > HD_CAP) {
        if (tid == 0) *q.meta = PanelMeta{epoch, 0, 1, 0};
        return;
    }

    // 2. this thread's entries and their sampled rows
    int32_t cc[HD_EPT], jv[HD_EPT], hh[HD_EPT];
    double vv[HD_EPT];
#pragma unroll
    for (int u = 0; u < HD_EPT; ++u) {
        const int f = tid + HD_BUILD_NT * u;
        int jj = 0;
#pragma unroll
        for (int step = 16; step >= 1; step >>= 1)
            if (jj + step < nj && rowoff[jj + step] <= f) jj += step;
        const int64_t e = hd_clamp(rowbeg[jj] + (f - rowoff[jj]), 0, nnz - 1);
        jv[u] = jj;
        cc[u] = f < total ? col_idx[e] : -1;
        vv[u] = f < total ? val[e] : 0.0;
    }
    // 3. hash the columns: slot, sampled-row mask, first entry
#pragma unroll
    for (int u = 0; u < HD_EPT; ++u) {
        hh[u] = -1;
        const int32_t c = cc[u];
        if (c < 0 || c >= n) continue;    // also a malformed matrix (its check reports it)
        uint32_t h = hd_hash(c);
        for (;;) {                         // at most HD_CAP keys in HD_HS slots: ends
            const int32_t old = atomicCAS(&hkey[h], -1, c);
            if (old == -1 || old == c) break;
            h = (h + 1) & (HD_HS - 1);
        }
        hh[u] = (int)h;
        atomicMin(&hcode[h], tid + HD_BUILD_NT * u);
        atomicOr(&hmask[h], 1u << jv[u]);
    }
    __syncthreads();
    // 4. owners (first entries) and the histogram of their sampled-row counts
    bool own[HD_EPT];
    uint32_t mk[HD_EPT];
#pragma unroll
    for (int u = 0; u < HD_EPT; ++u) {
        own[u] = hh[u] >= 0 && hcode[hh[u]] == tid + HD_BUILD_NT * u;
        mk[u] = hh[u] >= 0 ? hmask[hh[u]] : 0u;
        if (own[u]) atomicAdd(&hist[__popc(mk[u])], 1);
    }
    __syncthreads();
    if (tid == 0) {
        int t = HD_NJ + 1, acc = 0;
        while (t > 1 && acc + hist[t - 1] <= HD_HEAD) acc += hist[--t];
        info[0] = t;          // columns stored by >= t sampled rows form the head
    }
    __syncthreads();
    const int tstar = info[0];
    // 5. head positions and tail offsets in chunk order: scans over the waves
    int hx[HD_EPT], tx[HD_EPT];
    bool head[HD_EPT];
#pragma unroll
    for (int u = 0; u < HD_EPT; ++u) {
        head[u] = own[u] && __popc(mk[u]) >= tstar;
        const int a0 = head[u] ? 1 : 0, b0 = (own[u] && !head[u]) ? __popc(mk[u]) : 0;
        int a = a0, b = b0;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int ua = __shfl_up(a, o, 64), ub = __shfl_up(b, o, 64);
            if (lane >= o) {
                a += ua;
                b += ub;
            }
        }
        if (lane == 63) {
            wsum[0][u][wid] = a;
            wsum[1][u][wid] = b;
        }
        hx[u] = a - a0;
        tx[u] = b - b0;
    }
    __syncthreads();
    const uint32_t ep = epoch << HD_EPOCH_SHIFT;
    int oa = 0, ob = 0;
#pragma unroll
    for (int u = 0; u < HD_EPT; ++u) {
        int pa = oa, pb = ob;
        for (int w = 0; w < NWB; ++w) {
            if (w < wid) {
                pa += wsum[0][u][w];
                pb += wsum[1][u][w];
            }
            oa += wsum[0][u][w];
            ob += wsum[1][u][w];
        }
        if (own[u]) hcode[hh[u]] = (int32_t)(ep | (head[u] ? (HD_HEADBIT | (uint32_t)(pa + hx[u]))
                                                              : (uint32_t)(pb + tx[u])));
    }
    const int nh = oa;
    __syncthreads();
    // 6. values into the head block or tval; the owners write the records
#pragma unroll
    for (int u = 0; u < HD_EPT; ++u) {
        if (hh[u] < 0) continue;
        const uint32_t code = (uint32_t)hcode[hh[u]];
        const int jj = jv[u];
        if (code & HD_HEADBIT)
            q.Bh[(code & HD_VALMASK) * HD_NJ + jj] = vv[u];
        else
            q.tval[(code & HD_VALMASK) + __popc(mk[u] & ((1u << jj) - 1u))] = vv[u];
        if (own[u]) {
            q.code[cc[u]] = code;
            if (!(code & HD_HEADBIT)) q.tail[cc[u]] = TailRec{mk[u], 0u, vv[u]};
        }
    }
    if (tid == 0) *q.meta = PanelMeta{epoch, nh, 0, 0};
}

}  // namespace
}  // namespace kdcd
