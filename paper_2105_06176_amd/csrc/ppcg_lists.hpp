// ppcg_lists.hpp -- SpMV rows of chunks described by lists alone (see
// ppcg_stencil.hpp for the storage).
#pragma once

#include "ppcg_internal.hpp"

namespace ppcg {

// Loads through the constant address space: data that no launch writes while
// this one runs and that is the same for the whole wavefront becomes scalar
// loads.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T *as_constant(const T *p)
{
    return (const __attribute__((address_space(4))) T *)p;
}

// Largest system: the byte offsets of ten vectors fit 31 bits.
constexpr int kStMaxRows = 25000000;

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

// A chunk's list start, mask start, length, and the length of the runs of
// consecutive columns that its whole list consists of (5, 3, else 0).
typedef int StChunk __attribute__((ext_vector_type(4)));

// One chunk's lists (uniform over the wavefront).
struct StLists {
    const __attribute__((address_space(4))) int *off;
    const __attribute__((address_space(4))) double *val;
    const __attribute__((address_space(4))) unsigned long long *mask;
};

// Entries k0 .. k0 + L - 1 of a row: the gathers back to back, then their
// products added in entry order.  SC: each is value * (d0 * w[col]), m = M^-1 w
// formed from the gathered w as everywhere in the single-launch form.
template <bool SC, int L>
__device__ __forceinline__ double st_span(const StLists p, int k0, StBuf w, int rowb, double d0, double a)
{
    double x[L];
#pragma unroll
    for (int j = 0; j < L; ++j)
        x[j] = st_load(w, rowb + p.off[k0 + j]);
#pragma unroll
    for (int j = 0; j < L; ++j) {
        const bool has = __builtin_amdgcn_inverse_ballot_w64(p.mask[k0 + j]);
        const double v = has ? x[j] : 0.0;
        a = a + p.val[k0 + j] * (SC ? d0 * v : v);
    }
    return a;
}

template <bool SC, int M>
__device__ __forceinline__ double st_tail(int rem, const StLists p, int k0, StBuf w, int rowb, double d0, double a)
{
    if constexpr (M > 0) {
        if (rem == M)
            return st_span<SC, M>(p, k0, w, rowb, d0, a);
        return st_tail<SC, M - 1>(rem, p, k0, w, rowb, d0, a);
    } else {
        return a;
    }
}

// Lists that consist of runs of L consecutive columns, L = 5 or 3: N runs a
// step go through LDS.  A 64-lane load of doubles occupies the address unit for
// 16 cycles whatever its lanes do, so one load per entry bounds a long row by
// that unit (165^3 125-point: busy 88 % of 277 us).  Here a wavefront loads
// the first column of each run and, in one more load, the L - 1 columns past
// the 64 rows of all N runs; its lanes then read their L neighbours from LDS,
// at constant offsets.  m = d0 * w is formed once per element, before the LDS.
// N at 165^3 125-point: 1 7.2 ms, 2 6.2, 3 6.2, 4 6.2, 5 7.1 per solve (11.0
// with a load per entry); more scalar registers spill from 4 on.
constexpr int kStRuns = 3;
constexpr int kStRunMax = 5;
constexpr int kStRunLds = kStRuns * (kSellC + kStRunMax - 1);  // doubles per wavefront

// Orders a wavefront's own LDS accesses (the hardware keeps them in order).
__device__ __forceinline__ void st_wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// st_row<true> of a list of runs of L; wl: this wavefront's kStRunLds doubles.
// All 64 lanes call it.
template <int L>
__device__ __forceinline__ double st_row_runs(const SysDesc &d, StChunk ch, StBuf w, int rowb, double d0, double *wl)
{
    constexpr int N = kStRuns, W = kSellC + L - 1, T = L - 1;
    static_assert(N * T <= kSellC && N * W <= kStRunLds, "one load fetches the columns past the rows");
    const int len = ch[2], lane = threadIdx.x & 63;
    const StLists p{as_constant(d.soff) + ch[0], as_constant(d.sval) + ch[0], as_constant(d.smask) + ch[1]};
    // this lane's column past the rows: run lane / T, element kSellC + lane % T
    const int tailb = rowb + 8 * (kSellC - lane + lane % T);
    double *tl = wl + (lane / T) * W + kSellC + lane % T;
    double a = 0.0, x[N], e = 0.0;
    int k0 = 0;
    auto fetch = [&](int k) {
        int o = 0x7fffff00;  // outside: 0
#pragma unroll
        for (int r = N - 1; r >= 0; --r) {
            x[r] = st_load(w, rowb + p.off[k + r * L]);
            if (lane < (r + 1) * T)
                o = tailb + p.off[k + r * L];
        }
        e = st_load(w, o);
    };
    if (N * L <= len)
        fetch(0);
    for (; k0 + N * L <= len; k0 += N * L) {
        st_wave_fence();
#pragma unroll
        for (int r = 0; r < N; ++r)
            wl[r * W + lane] = d0 * x[r];
        if (lane < N * T)
            *tl = d0 * e;
        if (k0 + 2 * N * L <= len)  // the next step's columns
            fetch(k0 + N * L);
        st_wave_fence();
#pragma unroll
        for (int r = 0; r < N; ++r)
#pragma unroll
            for (int j = 0; j < L; ++j) {
                const bool has = __builtin_amdgcn_inverse_ballot_w64(p.mask[k0 + r * L + j]);
                const double t = wl[r * W + lane + j], v = has ? t : 0.0;
                a = a + p.val[k0 + r * L + j] * v;
            }
    }
    for (; k0 < len; k0 += L)
        a = st_span<true, L>(p, k0, w, rowb, d0, a);
    return a;
}

// (A m)[row] (SC) or (A w)[row] of one lane's row of chunk ch.
template <bool SC>
__device__ __forceinline__ double st_row(const SysDesc &d, StChunk ch, StBuf w, int rowb, double d0)
{
    constexpr int B = 8;
    const int len = ch[2];
    const StLists p{as_constant(d.soff) + ch[0], as_constant(d.sval) + ch[0], as_constant(d.smask) + ch[1]};
    double a = 0.0;
    int k0 = 0;
    for (; k0 + B <= len; k0 += B)
        a = st_span<SC, B>(p, k0, w, rowb, d0, a);
    return st_tail<SC, B - 1>(len - k0, p, k0, w, rowb, d0, a);
}

}  // namespace ppcg
