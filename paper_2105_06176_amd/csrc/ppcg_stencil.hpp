// ppcg_stencil.hpp -- the single-launch PIPECG iteration (ppcg_fused.hpp) for
// matrices whose chunks are described by lists alone: constant-coefficient
// stencils.
//
// A chunk (64 rows, one wavefront) on a shared offset list qualifies when,
// for every entry of the list, the rows that have the entry all hold the same
// value.  The chunk is then
//   * a list of (byte offset of the column from the row, value), and
//   * one 64-bit mask per entry: the lanes whose row has it,
// and the matrix needs no storage per row: offsets, values and masks are the
// same for the wavefront's 64 lanes and come through scalar loads.  Equal lists
// and equal mask sets are stored once (k_st_scan hashes them per chunk, the
// host keeps one chunk of each hash, k_st_verify compares every chunk with its
// representative bit for bit).
//
// With the lists no gather waits for a vector load of a column, a value index
// or a table entry.  The gathers are raw buffer loads: the hardware returns 0 for an
// address outside the vector (the columns that masked-off lanes of the first
// and last rows name), so no column is clamped.  A masked-off lane's gathered
// value is replaced by 0, and the row sum adds the same products in the same
// order as the per-entry storage (whose missing entries are explicit zeros).
//
// Bound by the vector streams on short rows and by the gathers on long ones.
// Measured, us per iteration, k_fused on the one-byte value table, then with
// the chunk lists, then also with the ring of residuals (kStDefer): 128^3
// 7-point 49.4, 32.0, 29.5 (164 MB in the last: 5.6 TB/s, of which about
// 5 us are the launch's start and its reduction); 100^3 26.7, 18.6, 17.4;
// 165^3 125-point 471, 278, 278 (no ring at that size), 150 with st_row_runs
// (100^3 27-point 20.3 and 16.9); 301^2 5-point 6.6, 5.8, 5.8.  Streaming hints (nt) on the loads or stores: 36 to 44 us at
// 128^3, because the vectors then miss the memory-side cache.  Forming z from
// s in every launch (z = A M^-1 s, gathered beside w, instead of z carried;
// 16 bytes per row fewer) measured no faster at 7 points and twice slower at
// 125: the second gather costs what the stream saves.
#pragma once

#include "ppcg_fused.hpp"

namespace ppcg {

// ---------------------------------------------------------------- setup
__device__ __forceinline__ unsigned long long st_mix(unsigned long long h, unsigned long long v)
{
    h ^= v + 0x9E3779B97F4A7C15ull + (h << 6) + (h >> 2);
    h *= 0xBF58476D1CE4E5B9ull;
    return h ^ (h >> 29);
}

// One wavefront per chunk: the value and the lane mask of every entry of the
// chunk's list (at cptr[c] / 64 + k), hashes of (offsets, values) and of the
// masks.  flag[0] |= 1 when an entry holds two different values.  Which rows
// have an entry comes from their CSR columns, not from the stored values: a
// zero that the matrix stores is a value like any other (0 * Inf is NaN),
// where the layout's filler is no entry.
__global__ __launch_bounds__(64) void k_st_scan(int n, int nchunks, const int *__restrict__ rp,
                                                const int *__restrict__ ci, const int64_t *__restrict__ cptr,
                                                const int *__restrict__ cpat, const int *__restrict__ pats,
                                                const double *__restrict__ val, double *__restrict__ tval,
                                                unsigned long long *__restrict__ tmask,
                                                unsigned long long *__restrict__ hash, unsigned *__restrict__ flag)
{
    const int c = blockIdx.x, l = threadIdx.x;
    if (c >= nchunks)
        return;
    const int64_t base = cptr[c];
    const int len = (int)((cptr[c + 1] - base) / kSellC);
    const int *list = pats + cpat[c];
    const int p = c * kSellC + l;
    int e = 0, end = 0;  // this row's entries not yet met
    if (p < n) {
        e = rp[p];
        end = rp[p + 1];
    }
    unsigned long long hl = st_mix(0x1234567ull, (unsigned)len), hm = st_mix(0x7654321ull, (unsigned)len);
    for (int k = 0; k < len; ++k) {
        const unsigned long long v =
            (unsigned long long)__double_as_longlong(val[(size_t)base + (size_t)k * kSellC + l]);
        const bool has = e < end && ci[e] == p + list[k];
        if (has)
            ++e;
        const unsigned long long m = __ballot(has);
        const unsigned long long first = m ? __shfl(v, (int)__ffsll((long long)m) - 1, 64) : 0ull;
        if (__any(has && v != first)) {
            if (l == 0)
                atomicOr(flag, 1u);
            return;
        }
        if (l == 0) {
            tval[base / kSellC + k] = __longlong_as_double((long long)first);
            tmask[base / kSellC + k] = m;
        }
        hl = st_mix(st_mix(hl, (unsigned)list[k]), first);
        hm = st_mix(hm, m);
    }
    if (l == 0) {
        hash[2 * (size_t)c] = hl;
        hash[2 * (size_t)c + 1] = hm;
    }
}

// Copy the representative chunks' lists: items[i] = {chunk, destination, 0:
// offsets and values / 1: masks, unused}; one wavefront per item.
__global__ __launch_bounds__(64) void k_st_copy(const int4 *__restrict__ items, const int64_t *__restrict__ cptr,
                                                const int *__restrict__ cpat, const int *__restrict__ pats,
                                                const double *__restrict__ tval,
                                                const unsigned long long *__restrict__ tmask, int *__restrict__ off,
                                                double *__restrict__ val, unsigned long long *__restrict__ mask)
{
    const int4 it = items[blockIdx.x];
    const int64_t base = cptr[it.x];
    const int len = (int)((cptr[it.x + 1] - base) / kSellC);
    const int *list = pats + cpat[it.x];
    for (int k = threadIdx.x; k < len; k += 64) {
        if (it.z == 0) {
            off[it.y + k] = list[k] * 8;  // byte offset of an FP64 element
            val[it.y + k] = tval[base / kSellC + k];
        } else {
            mask[it.y + k] = tmask[base / kSellC + k];
        }
    }
}

// flag[0] |= 1 when a chunk's lists differ from the ones it was given, 2 when
// st_row_runs has a step to do on it.
__global__ __launch_bounds__(64) void k_st_verify(int nchunks, const int64_t *__restrict__ cptr,
                                                  const int *__restrict__ cpat, const int *__restrict__ pats,
                                                  const double *__restrict__ tval,
                                                  const unsigned long long *__restrict__ tmask,
                                                  int4 *__restrict__ chunk, const int *__restrict__ off,
                                                  const double *__restrict__ val,
                                                  const unsigned long long *__restrict__ mask,
                                                  unsigned *__restrict__ flag)
{
    const int c = blockIdx.x;
    if (c >= nchunks)
        return;
    const int64_t base = cptr[c];
    const int len = (int)((cptr[c + 1] - base) / kSellC);
    const int *list = pats + cpat[c];
    const int4 ch = chunk[c];
    bool bad = ch.z != len;
    for (int k = threadIdx.x; k < len && !bad; k += 64)
        bad = off[ch.x + k] != list[k] * 8 ||
              __double_as_longlong(val[ch.x + k]) != __double_as_longlong(tval[base / kSellC + k]) ||
              mask[ch.y + k] != tmask[base / kSellC + k];
    if (bad)
        atomicOr(flag, 1u);
    // the length of the runs that the whole list consists of
    bool run5 = len > 0 && len % 5 == 0, run3 = len > 0 && len % 3 == 0;
    for (int k = threadIdx.x; k < len; k += 64) {
        const bool next = k > 0 && list[k] == list[k - 1] + 1;
        run5 = run5 && (k % 5 == 0 || next);
        run3 = run3 && (k % 3 == 0 || next);
    }
    const int run = __all(run5) ? 5 : __all(run3) ? 3 : 0;
    if (threadIdx.x == 0) {
        chunk[c].w = run;
        if (run && len >= kStRuns * run)
            atomicOr(flag, 2u);
    }
}

// ---------------------------------------------------------------- iteration
struct StScalars {
    double hist[2 * kStDefer];  // alpha, beta of the updates since the last full ring
    SysState rec;
};

// The handle's vectors lie in one allocation at a fixed distance: one buffer
// resource and a scalar offset name any of them, where a pointer each would
// not fit the scalar registers.
__device__ __forceinline__ double st_vec(StBuf v, int byte, int vec)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(v, byte, vec, 0));
}

__device__ __forceinline__ void st_put(StBuf v, int byte, int vec, double x)
{
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uvec2, x), v, byte, vec, 0);
}

template <bool RUNS>
__device__ __forceinline__ double st_row_any(const SysDesc &d, StChunk ch, StBuf w, int rowb, double d0, double *wl)
{
    if constexpr (RUNS) {
        if (ch[3] == 5)
            return st_row_runs<5>(d, ch, w, rowb, d0, wl);
        if (ch[3] == 3)
            return st_row_runs<3>(d, ch, w, rowb, d0, wl);
    }
    return st_row<true>(d, ch, w, rowb, d0);
}

// k_fused (see ppcg_fused.hpp for the steps) with rows read from the lists;
// the diagonal is constant.  The registers stay at 61 (8 wavefronts per
// SIMD): local copies that the compiler cannot split went to LDS, with
// 10 us per launch.
//
// SOLO: the table is one system's tiles in order, and the descriptor comes
// with the kernel's arguments (the options in it do not: they are read from
// descs[0], so that a captured launch stays valid when they change).  It saves
// two dependent loads at the start of every launch.
// RUNS: some system of the launch has lists of runs (a kernel of its own: with
// both in one, 7-point rows at 128^3 lost 2 % to the extra registers).
template <bool SOLO, bool RUNS>
__global__ __launch_bounds__(kFusedThreads, PPCG_FUSED_WAVES) void k_stencil(const WorkItem *__restrict__ table,
                                                                             const int *__restrict__ count,
                                                                             const SysDesc *__restrict__ descs,
                                                                             int remap, int par, const SysDesc own)
{
    __shared__ double lds[kFusedThreads / 64 * kNumPartials];
    __shared__ StScalars sc;
    __shared__ double win[RUNS ? kFusedThreads / 64 * kStRunLds : 1];
    const int live = SOLO ? own.nftiles : *count;
    if ((int)blockIdx.x >= live)
        return;
    const int pos = remap ? xcd_remap(blockIdx.x, live) : (int)blockIdx.x;
    const WorkItem wi = SOLO ? WorkItem{0, pos} : table[pos];
    const SysDesc &opt = descs[wi.slot], &d = SOLO ? own : opt;
    const int R = d.frows / kFusedThreads;  // rows per thread, 1 .. kFusedRowsPerThread
    // The record and the lists are the same for the workgroup or the
    // wavefront and not written by this launch: scalar loads.
    const __attribute__((address_space(4))) SysState *rin = as_constant((const SysState *)d.frec) + par;
    const int n = d.n;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row0 = wi.tile * d.frows;
    const int c0 = row0 / kSellC + wave;  // this wavefront's chunks: c0 + k * kFusedThreads / kSellC
    const __attribute__((address_space(4))) StChunk *CH = as_constant((const StChunk *)d.schunk);
    const bool some = c0 * kSellC < n;
    StChunk ch = {0, 0, 0, 0};
    if (some)
        ch = CH[c0];
    const int nft = d.nftiles;
    const PPCG_AS1 dvec2 *PR = (const PPCG_AS1 dvec2 *)as_global(d.fpart + (size_t)par * nft * 4);
    dvec2 pa0 = {0.0, 0.0}, pb0 = {0.0, 0.0}, pa1 = {0.0, 0.0}, pb1 = {0.0, 0.0};
    const bool has0 = tid < nft, has1 = tid + kFusedThreads < nft;
    if (has0) {
        pa0 = PR[2 * tid];
        pb0 = PR[2 * tid + 1];
    }
    if (has1) {
        pa1 = PR[2 * (tid + kFusedThreads)];
        pb1 = PR[2 * (tid + kFusedThreads) + 1];
    }
    rec_load(&sc.rec, d.frec + par);
    double hist = 0.0;
    if (tid < 2 * kStDefer)
        hist = as_global(d.shist)[par * kStHist + tid];
    const double d0 = as_constant((const double *)d.dinv)[0];
    __asm__ volatile("" ::: "memory");  // the loads above stay above the check
    if (rin->done) {
        // publish the stop in the other slot too (see k_fused)
        if (wi.tile == 0)  // (each thread stores the word it loaded)
            rec_store(d.frec + (par ^ 1), &sc.rec);
        return;
    }
    // Vectors, by their byte distance from x.  w is double buffered by parity
    // (w and u), because other tiles gather it.
    const int vs = d.vstride;
    const StBuf V = __builtin_amdgcn_make_buffer_rsrc(d.x, 0, 10 * vs, 0x00020000);
    const int oW = (par ? 2 : 3) * vs, oWo = (par ? 3 : 2) * vs, oS = 8 * vs, oZ = 6 * vs, oP = 9 * vs;
    const StBuf wb = st_buf((const double *)((const char *)d.x + oW), n);
    // The update number i of a start.  With the ring of residuals r, q, nv, m
    // it reads r_i from buffer i mod kStDefer and writes r_{i+1} to the next.
    const bool ring = d.sring != 0;
    const ScalarIn c = {rin->gamma_prev, rin->alpha_prev, stop_limit(opt, rin->bnorm2),
                        rin->iter, rin->i_start, rin->phase};
    const int at = (rin->i_start + (rin->phase ? 0 : 1)) & (ring ? kStDefer - 1 : 1);
    static_assert(kStDefer == 4, "the ring is r, q, nv, m");
    auto buf = [vs](int k) { return (k == 0 ? 1 : k == 1 ? 7 : k == 2 ? 5 : 4) * vs; };
    const int oR = buf(ring ? at : 0), oRo = buf(ring ? (at + 1) & (kStDefer - 1) : 0);
    // 0. This thread's first row: the update's operands and n = A m.  A lane
    // past the last row reads zeros and its stores are dropped.
    int ib = row0 + tid < n ? (row0 + tid) * 8 : 0x7ffffff0;
    double w = st_load(wb, ib), s = st_vec(V, ib, oS), z = st_vec(V, ib, oZ), r = st_vec(V, ib, oR);
    double nv = 0.0;
    if (some)
        nv = st_row_any<RUNS>(d, ch, wb, (row0 + tid) * 8, d0, win + (RUNS ? wave * kStRunLds : 0));
    // 1. The previous launch's partials and the scalar recurrences.
    {
        double v[kNumPartials] = {0.0, 0.0, 0.0, 0.0};
        if (has0) {
            v[0] = v[0] + pa0[0];
            v[1] = v[1] + pa0[1];
            v[2] = v[2] + pb0[0];
            v[3] = v[3] + pb0[1];
        }
        if (has1) {
            v[0] = v[0] + pa1[0];
            v[1] = v[1] + pa1[1];
            v[2] = v[2] + pb1[0];
            v[3] = v[3] + pb1[1];
        }
        for (int t = tid + 2 * kFusedThreads; t < nft; t += kFusedThreads) {
            const dvec2 a = PR[2 * t], b = PR[2 * t + 1];
            v[0] = v[0] + a[0];
            v[1] = v[1] + a[1];
            v[2] = v[2] + b[0];
            v[3] = v[3] + b[1];
        }
        if (tid < 2 * kStDefer)
            sc.hist[tid] = hist;
        block_sum<kFusedThreads, kNumPartials>(v, lds);
        if (tid == 0)
            pipecg_scalars(opt, c, v, &sc.rec);
        __syncthreads();
        // (behind the barrier, which would wait for these stores)
        if (wi.tile == 0) {
            rec_store(d.frec + (par ^ 1), &sc.rec);
            rec_store(d.st, &sc.rec);
        }
    }
    if (sc.rec.done) {
        // the updates of x (with the ring, of p and x) deferred so far, so
        // that x is complete when the host reads the state
        if (at > 0)
            for (int k = 0; k < R; ++k) {
                const int i = row0 + k * kFusedThreads + tid;
                if (i < n) {
                    double p = st_vec(V, i * 8, oP), x = st_vec(V, i * 8, 0);
#pragma unroll
                    for (int t = 0; t < kStDefer - 1; ++t)
                        if (t < at) {
                            if (ring)
                                p = d0 * st_vec(V, i * 8, buf(t)) + sc.hist[kStDefer + t] * p;
                            x = x + sc.hist[t] * p;
                        }
                    st_put(V, i * 8, 0, x);
                }
            }
        return;
    }
    const double sa = sc.rec.alpha, sb = sc.rec.beta;
    if (wi.tile == 0 && tid < 2 * kStDefer)
        as_global(d.shist)[(par ^ 1) * kStHist + tid] =
            (tid & (kStDefer - 1)) != at ? hist : tid < kStDefer ? sa : sb;
    // 2. Per row of this thread: n = A m into a register, then the update.
    const bool full = at == (ring ? kStDefer - 1 : 1);
    double acc[kNumPartials] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int k = 0; k < R; ++k) {
        const int i = row0 + k * kFusedThreads + tid;
        if (row0 + k * kFusedThreads + wave * kSellC >= n)
            break;  // uniform per wavefront
        if (k > 0) {
            ib = i < n ? i * 8 : 0x7ffffff0;
            w = st_load(wb, ib);
            s = st_vec(V, ib, oS);
            z = st_vec(V, ib, oZ);
            r = st_vec(V, ib, oR);
            ch = CH[c0 + k * (kFusedThreads / kSellC)];
            nv = st_row_any<RUNS>(d, ch, wb, i * 8, d0, win + (RUNS ? wave * kStRunLds : 0));
        }
        if (ring) {
            if (full) {
                double p = st_vec(V, ib, oP), x = st_vec(V, ib, 0), q[kStDefer];
#pragma unroll
                for (int t = 0; t < kStDefer - 1; ++t)
                    q[t] = st_vec(V, ib, buf(t));
#pragma unroll
                for (int t = 0; t < kStDefer - 1; ++t) {
                    p = d0 * q[t] + sc.hist[kStDefer + t] * p;
                    x = x + sc.hist[t] * p;
                }
                p = d0 * r + sb * p;
                x = x + sa * p;
                st_put(V, ib, oP, p);
                st_put(V, ib, 0, x);
            }
        } else {
            const double pold = st_vec(V, ib, oP), p = d0 * r + sb * pold;
            st_put(V, ib, oP, p);
            if (full) {
                const double x = st_vec(V, ib, 0) + sc.hist[0] * pold;
                st_put(V, ib, 0, x + sa * p);
            }
        }
        z = nv + sb * z;
        s = w + sb * s;
        r = r - sa * s;
        w = w - sa * z;
        const double u = d0 * r;
        acc[0] = acc[0] + r * u;
        acc[1] = acc[1] + w * u;
        acc[2] = acc[2] + u * u;
        acc[3] = acc[3] + r * r;
        st_put(V, ib, oS, s);
        st_put(V, ib, oRo, r);
        st_put(V, ib, oWo, w);
        st_put(V, ib, oZ, z);
    }
    const double t = block_sum4<kFusedThreads>(acc, lds);
    if (tid < kNumPartials)
        as_global(d.fpart)[((size_t)(par ^ 1) * d.nftiles + wi.tile) * 4 + tid] = t;
}

}  // namespace ppcg
