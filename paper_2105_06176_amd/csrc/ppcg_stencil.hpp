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
// Bound by the vector streams (96 bytes per row and iteration) on short rows
// and by the gathers on long ones.  Measured against k_fused on the one-byte
// value table, per iteration: 128^3 7-point 51.1 -> 33.5 us, 165^3 125-point
// 480 -> 300 us, 301^2 5-point 7.4 -> 6.7 us.
#pragma once

#include "ppcg_fused.hpp"

namespace ppcg {

// Largest system: byte offsets of rows and columns fit 31 bits.
constexpr int kStMaxRows = (1 << 28) - (1 << 14);

// ---------------------------------------------------------------- setup
__device__ __forceinline__ unsigned long long st_mix(unsigned long long h, unsigned long long v)
{
    h ^= v + 0x9E3779B97F4A7C15ull + (h << 6) + (h >> 2);
    h *= 0xBF58476D1CE4E5B9ull;
    return h ^ (h >> 29);
}

// One wavefront per chunk: the value and the lane mask of every entry of the
// chunk's list (at cptr[c] / 64 + k), hashes of (offsets, values) and of the
// masks.  flag[0] |= 1 when an entry holds two different values.  An entry is
// absent from a row where the stored value is +0.0 (the layout's filler; a
// stored zero contributes the same nothing).
__global__ __launch_bounds__(64) void k_st_scan(int nchunks, const int64_t *__restrict__ cptr,
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
    unsigned long long hl = st_mix(0x1234567ull, (unsigned)len), hm = st_mix(0x7654321ull, (unsigned)len);
    for (int k = 0; k < len; ++k) {
        const unsigned long long v =
            (unsigned long long)__double_as_longlong(val[(size_t)base + (size_t)k * kSellC + l]);
        const unsigned long long m = __ballot(v != 0ull);
        const unsigned long long first = m ? __shfl(v, (int)__ffsll((long long)m) - 1, 64) : 0ull;
        if (__any(v != 0ull && v != first)) {
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

// flag[0] |= 1 when a chunk's lists differ from the ones it was given.
__global__ __launch_bounds__(64) void k_st_verify(int nchunks, const int64_t *__restrict__ cptr,
                                                  const int *__restrict__ cpat, const int *__restrict__ pats,
                                                  const double *__restrict__ tval,
                                                  const unsigned long long *__restrict__ tmask,
                                                  const int4 *__restrict__ chunk, const int *__restrict__ off,
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
}

// ---------------------------------------------------------------- rows
typedef unsigned uvec2 __attribute__((ext_vector_type(2)));
typedef __amdgpu_buffer_rsrc_t StBuf;

// Raw buffer over n doubles: a load whose 8 bytes are not inside returns 0.
__device__ __forceinline__ StBuf st_buf(const double *p, int n)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, n * 8, 0x00020000);
}

__device__ __forceinline__ double st_load(StBuf b, int byte)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(b, byte, 0, 0));
}

// One chunk's lists (uniform over the wavefront).
struct StLists {
    const __attribute__((address_space(4))) int *off;
    const __attribute__((address_space(4))) double *val;
    const __attribute__((address_space(4))) unsigned long long *mask;
};

// Entries k0 .. k0 + L - 1 of a row: the L gathers back to back, then their
// products added in entry order; each is value * (d0 * w[col]), m = M^-1 w
// formed from the gathered w as everywhere in the single-launch form.
template <int L>
__device__ __forceinline__ void st_span(const StLists &p, int k0, StBuf w, int rowb, double d0, double &n)
{
    double x[L];
#pragma unroll
    for (int j = 0; j < L; ++j)
        x[j] = st_load(w, rowb + p.off[k0 + j]);
#pragma unroll
    for (int j = 0; j < L; ++j) {
        const bool has = __builtin_amdgcn_inverse_ballot_w64(p.mask[k0 + j]);
        n = n + p.val[k0 + j] * (d0 * (has ? x[j] : 0.0));
    }
}

template <int M>
__device__ __forceinline__ void st_tail(int rem, const StLists &p, int k0, StBuf w, int rowb, double d0, double &n)
{
    if constexpr (M > 0) {
        if (rem == M)
            st_span<M>(p, k0, w, rowb, d0, n);
        else
            st_tail<M - 1>(rem, p, k0, w, rowb, d0, n);
    }
}

// (A m)[row] of one lane's row: ch = the chunk's list start, mask start and
// length (uniform).
__device__ __forceinline__ double st_row(const SysDesc &d, int lst, int msk, int len, StBuf w, int rowb, double d0)
{
    constexpr int B = 8;
    const StLists p{as_constant(d.soff) + lst, as_constant(d.sval) + lst, as_constant(d.smask) + msk};
    double n = 0.0;
    int k0 = 0;
    for (; k0 + B <= len; k0 += B)
        st_span<B>(p, k0, w, rowb, d0, n);
    st_tail<B - 1>(len - k0, p, k0, w, rowb, d0, n);
    return n;
}

// k_fused (see ppcg_fused.hpp for the steps) with rows read from the lists;
// the diagonal is constant.
__global__ __launch_bounds__(kFusedThreads, PPCG_FUSED_WAVES) void k_stencil(const WorkItem *__restrict__ table,
                                                                             const int *__restrict__ count,
                                                                             const SysDesc *__restrict__ descs,
                                                                             int remap, int par)
{
    __shared__ double lds[kFusedThreads / 64 * kNumPartials];
    __shared__ FusedScalars sc;
    const int live = *count;
    if ((int)blockIdx.x >= live)
        return;
    const int pos = remap ? xcd_remap(blockIdx.x, live) : (int)blockIdx.x;
    const WorkItem wi = table[pos];
    const SysDesc &d = descs[wi.slot];
    const int R = d.frows / kFusedThreads;  // rows per thread, 1 .. kFusedRowsPerThread
    const SysState *rin = d.frec + par;
    const int n = d.n;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row0 = wi.tile * d.frows;
    const int c0 = row0 / kSellC + wave;
    // lane k < R: the lists of this wavefront's chunk k
    int4 ch = {0, 0, 0, 0};
    {
        const int c = c0 + lane * (kFusedThreads / kSellC);
        if (lane < R && c < (n + kSellC - 1) / kSellC)
            ch = d.schunk[c];
    }
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
    const double d0 = as_constant((const double *)d.dinv)[0];
    __asm__ volatile("" ::: "memory");  // the loads above stay above the check
    if (rin->done) {
        // publish the stop in the other slot too (see k_fused)
        if (wi.tile == 0 && threadIdx.x == 0)
            d.frec[par ^ 1] = *rin;
        return;
    }
    double *const v0 = (double *)d.w, *const v1 = (double *)d.w1;
    const double *gin = par ? v1 : v0;
    double *gout = par ? v0 : v1;
    const StBuf wb = st_buf(gin, n);
    const PPCG_AS1 double *__restrict__ W = as_global(gin);
    PPCG_AS1 double *__restrict__ Wo = as_global(gout);
    PPCG_AS1 double *__restrict__ X = as_global((double *)d.x);
    PPCG_AS1 double *__restrict__ Rv = as_global((double *)d.r);
    PPCG_AS1 double *__restrict__ Z = as_global((double *)d.z);
    PPCG_AS1 double *__restrict__ S = as_global((double *)d.s);
    PPCG_AS1 double *__restrict__ P = as_global((double *)d.p);
    // 0. This thread's first row of n = A m.
    double nv0 = 0.0;
    if (c0 * kSellC < n)  // uniform per wavefront
        nv0 = st_row(d, __builtin_amdgcn_readlane(ch.x, 0), __builtin_amdgcn_readlane(ch.y, 0),
                     __builtin_amdgcn_readlane(ch.z, 0), wb, (row0 + tid) * 8, d0);
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
        block_sum<kFusedThreads, kNumPartials>(v, lds);
        if (tid == 0) {
            SysState loc = *rin;
            if (!loc.phase) {
                loc.alpha_x = loc.alpha;
                loc.x_pending ^= 1;
            }
            scalar_update<kNumPartials>(d, &loc, v);
            sc.alpha = loc.alpha;
            sc.beta = loc.beta;
            sc.alpha_x = loc.alpha_x;
            sc.x_pending = loc.x_pending;
            sc.go = !loc.done;
            sc.x_finish = loc.done && loc.x_pending;
            if (sc.x_finish)
                loc.x_pending = 0;
            if (wi.tile == 0) {
                d.frec[par ^ 1] = loc;
                *d.st = loc;
            }
        }
        __syncthreads();
    }
    if (!sc.go) {
        if (sc.x_finish) {
            const double a = sc.alpha_x;
            for (int k = 0; k < R; ++k) {
                const int i = row0 + k * kFusedThreads + tid;
                if (i < n)
                    X[i] = X[i] + a * P[i];
            }
        }
        return;
    }
    // 2. Per row of this thread: n = A m into a register, then the update.
    const double sa = sc.alpha, sb = sc.beta, ax = sc.alpha_x;
    const bool xp = sc.x_pending != 0;
    double acc[kNumPartials] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int k = 0; k < R; ++k) {
        const int i = row0 + k * kFusedThreads + tid;
        if (row0 + k * kFusedThreads + wave * kSellC >= n)
            break;  // uniform per wavefront
        double z = 0.0, w = 0.0, s = 0.0, p = 0.0, r = 0.0, xo = 0.0;
        if (i < n) {
            z = Z[i];
            w = W[i];
            s = S[i];
            p = P[i];
            r = Rv[i];
            if (xp)
                xo = X[i];
        }
        const double nv = k == 0 ? nv0
                                 : st_row(d, __builtin_amdgcn_readlane(ch.x, k), __builtin_amdgcn_readlane(ch.y, k),
                                          __builtin_amdgcn_readlane(ch.z, k), wb, i * 8, d0);
        if (i < n) {
            const double pold = p;
            double u, mo;
            vma_elem<double, kNumPartials>(sa, sb, nv, z, w, s, p, r, d0, u, mo, acc);
            Z[i] = z;
            S[i] = s;
            P[i] = p;
            Rv[i] = r;
            Wo[i] = w;
            if (xp) {
                const double x1 = xo + ax * pold;
                X[i] = x1 + sa * p;
            }
        }
    }
    block_sum<kFusedThreads, kNumPartials>(acc, lds);
    if (tid == 0) {
        PPCG_AS1 dvec2 *out = (PPCG_AS1 dvec2 *)as_global(d.fpart + ((size_t)(par ^ 1) * d.nftiles + wi.tile) * 4);
        out[0] = dvec2{acc[0], acc[1]};
        out[1] = dvec2{acc[2], acc[3]};
    }
}

}  // namespace ppcg
