// ppcg_small.hpp -- one-workgroup PIPECG iteration kernel for small systems
// (Algorithm 2 of Tiwari & Vadhiyar, Section III-B, the same arithmetic as
// the fused update + SpMV pair of ppcg_kernels.hpp).
#pragma once

#include "ppcg_kernels.hpp"

namespace ppcg {

// ---------------------------------------------------------------------------
// Small systems: one workgroup of kSmallThreads runs up to `iters` whole
// PIPECG iterations of one system per launch (work item = system).  Thread t
// owns the rows t, t + kSmallThreads, ... (at most kSmallRowsPerThread) and
// keeps their z, s, p, r, w, x and n in registers for the whole launch; m,
// the only vector other rows read (the SpMV gathers), and the state record
// live in LDS.  Vectors and the state are loaded at the start and stored at the end of the launch.
// SELL format only; rows of a wavefront form one SELL chunk, so chunk lengths
// are uniform across each wavefront.
//
// An iteration:
//   update of the thread's rows, m into LDS, the four dot products summed per
//   wavefront                                                    -- barrier --
//   the last wavefront sums the wavefronts' sums and runs the scalar
//   recurrences while all (it too, afterwards) compute n = A m from LDS: the
//   overlap that Algorithm 2 is made for                         -- barrier --
//
// Where the matrix comes from, in order of preference:
//   lists   offsets, values and masks of the chunk through scalar loads
//           (ppcg_lists.hpp); an absent entry reads a slot that holds 0;
//   staged  with the one-byte value table and at most kSmallLdsEntries stored
//           entries, copied into LDS at the start of the launch, each entry
//           as a 16-bit column offset from its row and its value index;
//   memory  columns and values from L2.
// Same values and order in all three, so the same sums.
//
// Bound by issue and by the reductions' chain on one compute unit.  64^2
// 5-point, us per iteration: 512 threads with 8 rows each, the matrix staged,
// the dot products summed one by one and the scalars before the SpMV 6.5; this
// form 2.9 (4.7 with the lists read in every iteration and the scalars kept in
// the LDS record).
constexpr int kSmallThreads = 1024;
constexpr int kSmallRowsPerThread = 4;
constexpr int kSmallMaxRows = kSmallThreads * kSmallRowsPerThread;
constexpr int kSmallLdsEntries = 24576;
constexpr int kSmallWaves = kSmallThreads / 64;
static_assert(kSmallMaxRows <= 32768, "column offsets from the row fit 16 bits");
static_assert(PPCG_SMALL_MAX_ROWS <= kSmallMaxRows, "small systems must fit the register-resident kernel");

// Entries k0 .. k0 + L - 1 of a row from the lists: lane's row at byte rowb
// of the LDS vector m, absent entries at byte zero.
template <int L>
__device__ __forceinline__ double small_span(const StLists p, int k0, const char *m, int rowb, int zero, double a)
{
    double x[L];
#pragma unroll
    for (int j = 0; j < L; ++j) {
        const bool has = __builtin_amdgcn_inverse_ballot_w64(p.mask[k0 + j]);
        x[j] = *(const double *)(m + (has ? rowb + p.off[k0 + j] : zero));
    }
#pragma unroll
    for (int j = 0; j < L; ++j)
        a = a + p.val[k0 + j] * x[j];
    return a;
}

template <int M>
__device__ __forceinline__ double small_tail(int rem, const StLists p, int k0, const char *m, int rowb, int zero,
                                             double a)
{
    if constexpr (M > 0) {
        if (rem == M)
            return small_span<M>(p, k0, m, rowb, zero, a);
        return small_tail<M - 1>(rem, p, k0, m, rowb, zero, a);
    } else {
        return a;
    }
}

// The shared memory of the workgroup.
struct SmallLds {
    double m[kSmallMaxRows + 1];  // the last element is 0
    double part[kNumPartials * kSmallWaves];
    double scal[2];  // alpha, beta of the next update
    int stop;
    SysState loc;    // the state record, written back at the end of the launch
    short lco[kSmallLdsEntries];          // staged matrix: column - row
    unsigned char lvi[kSmallLdsEntries];  // and value index
    double ltab[kMaxValueTable];          // the value table
};

// E > 0: chunk lists of at most E entries.  The LDS address of every entry of
// the thread's rows is formed once (two 16-bit addresses per register), so an
// iteration's gathers issue back to back and wait for nothing.  E = 0: any
// other matrix, see above.
template <int E>
__device__ __forceinline__ void small_run(const SysDesc &d, int iters, SmallLds &L)
{
    constexpr int R = kSmallRowsPerThread;
    SysState *st = d.st;
    const int n = d.n;
    PPCG_AS1 double *__restrict__ X = as_global((double *)d.x);
    PPCG_AS1 double *__restrict__ Rv = as_global((double *)d.r);
    PPCG_AS1 double *__restrict__ Wv = as_global((double *)d.w);
    PPCG_AS1 double *__restrict__ NVv = as_global((double *)d.nv);
    PPCG_AS1 double *__restrict__ Z = as_global((double *)d.z);
    PPCG_AS1 double *__restrict__ S = as_global((double *)d.s);
    PPCG_AS1 double *__restrict__ P = as_global((double *)d.p);
    const PPCG_AS1 double *__restrict__ DI = as_global((const double *)d.dinv);
    const PPCG_AS1 double *__restrict__ val = as_global((const double *)d.val);
    const PPCG_AS1 int *__restrict__ col = as_global(d.col);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double *const m = L.m;
    // u and q are scalings of r and s by the inverse diagonal (see vma_elem):
    // u is formed from r, q never
    double z[R], s[R], p[R], r[R], w[R], nv[R], x[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int i = tid + j * kSmallThreads;
        const bool ok = i < n;
        z[j] = ok ? Z[i] : 0.0;
        s[j] = ok ? S[i] : 0.0;
        p[j] = ok ? P[i] : 0.0;
        r[j] = ok ? Rv[i] : 0.0;
        w[j] = ok ? Wv[i] : 0.0;
        nv[j] = ok ? NVv[i] : 0.0;
        x[j] = ok ? X[i] : 0.0;
    }
    if (tid < (int)(sizeof(SysState) / sizeof(int)))
        ((int *)&L.loc)[tid] = as_global((const int *)st)[tid];
    if (tid == 0) {
        L.stop = st->done;
        L.scal[0] = st->alpha;
        L.scal[1] = st->beta;
        m[kSmallMaxRows] = 0.0;
    }
    ScalarIn c{};
    if (wave == kSmallWaves - 1)
        c = {st->gamma_prev, st->alpha_prev, stop_limit(d, st->bnorm2), st->iter, st->i_start, st->phase};
    // chunk j of this wavefront: rows wave * 64 + j * kSmallThreads + lane
    const bool lists = E > 0 || d.schunk != nullptr;
    int base[R], len[R], msk[R], maxlen = 0;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int ci = wave + j * kSmallWaves;
        base[j] = len[j] = msk[j] = 0;
        if (ci * kSellC < n) {
            if (lists) {
                const StChunk ch = as_constant((const StChunk *)d.schunk)[ci];
                base[j] = ch[0];
                msk[j] = ch[1];
                len[j] = ch[2];
            } else {
                base[j] = (int)as_constant(d.cptr)[ci];
                len[j] = (int)((as_constant(d.cptr)[ci + 1] - as_constant(d.cptr)[ci]) / kSellC);
            }
        }
        maxlen = len[j] > maxlen ? len[j] : maxlen;
    }
    unsigned adr[R][(E + 2) / 2] = {};
    if constexpr (E > 0) {
        static_assert(8 * (kSmallMaxRows + 1) <= 65536, "LDS addresses of m fit 16 bits");
#pragma unroll
        for (int j = 0; j < R; ++j)
#pragma unroll
            for (int k = 0; k < E; ++k) {
                const bool in = k < len[j];
                const unsigned long long has = in ? as_constant(d.smask)[msk[j] + k] : 0ull;
                const int o = in ? as_constant(d.soff)[base[j] + k] : 0;
                const unsigned a = __builtin_amdgcn_inverse_ballot_w64(has)
                                       ? (unsigned)((tid + j * kSmallThreads) * 8 + o)
                                       : (unsigned)(kSmallMaxRows * 8);
                adr[j][k / 2] |= (k & 1) ? a << 16 : a;
            }
    }
    const bool dconst = E > 0 || d.dinv_const != 0;
    const double d0 = as_constant((const double *)d.dinv)[0];
    // staged matrix (uniform over the workgroup)
    const bool staged =
        !lists && d.vidx != nullptr && as_constant(d.cptr)[(n + kSellC - 1) / kSellC] <= kSmallLdsEntries;
    if (staged) {
        for (int t = tid; t < d.nvtab; t += kSmallThreads)
            L.ltab[t] = d.vtab[t];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int row = tid + j * kSmallThreads;
            for (int k = 0; k < len[j]; ++k) {
                const int o = base[j] + lane + k * kSellC;
                L.lco[o] = (short)(col[o] - row);
                L.lvi[o] = d.vidx[o];
            }
        }
    }
    __syncthreads();
    for (int it = 0; it < iters && !L.stop; ++it) {
        const double sa = L.scal[0], sb = L.scal[1];
        double acc[kNumPartials] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int i = tid + j * kSmallThreads;
            if (i < n) {
                double di = d0;
                if (!dconst)
                    di = DI[i];
                double u, mo;
                vma_elem<double, kNumPartials>(sa, sb, nv[j], z[j], w[j], s[j], p[j], r[j], di, u, mo, acc);
                x[j] = x[j] + sa * p[j];  // this kernel updates x every iteration
                m[i] = mo;
            }
        }
        const double ws = wave_sum4(acc);
        if ((lane & 15) == 0)
            L.part[(lane >> 4) * kSmallWaves + wave] = ws;
        __syncthreads();  // m and the wavefronts' sums complete
        if (wave == kSmallWaves - 1) {
            const double t = waves_sum4<kSmallWaves>(L.part);
            const double v[kNumPartials] = {readlane_f64(t, 0), readlane_f64(t, 1), readlane_f64(t, 2),
                                            readlane_f64(t, 3)};
            const ScalarOut o = pipecg_scalars(d, c, v, &L.loc);
            L.scal[0] = o.alpha;
            L.scal[1] = o.beta;
            L.stop = !o.go;
            c = {v[0], o.alpha, c.limit, o.iter, o.i_start, 0};
        }
        // n = A m (stored entries of a system with at most kSmallMaxRows rows
        // fit 32 bits)
        if constexpr (E > 0) {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                // (read again in every iteration: 4 E values do not fit the scalar registers)
                int b = base[j];
                __asm__ volatile("" : "+s"(b));
                double g[E], a = 0.0;
#pragma unroll
                for (int k = 0; k < E; ++k)
                    g[k] = *(const double *)((const char *)m + ((k & 1) ? adr[j][k / 2] >> 16
                                                                          : adr[j][k / 2] & 0xffffu));
#pragma unroll
                for (int k = 0; k < E; ++k)
                    a = a + (k < len[j] ? as_constant(d.sval)[b + k] : 0.0) * g[k];
                nv[j] = a;
            }
        } else if (lists) {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if (len[j] > 0) {
                    const StLists q{as_constant(d.soff) + base[j], as_constant(d.sval) + base[j],
                                    as_constant(d.smask) + msk[j]};
                    const int rowb = (tid + j * kSmallThreads) * 8;
                    double a = 0.0;
                    int k0 = 0;
                    for (; k0 + 8 <= len[j]; k0 += 8)
                        a = small_span<8>(q, k0, (const char *)m, rowb, kSmallMaxRows * 8, a);
                    nv[j] = small_tail<7>(len[j] - k0, q, k0, (const char *)m, rowb, kSmallMaxRows * 8, a);
                }
            }
        } else if (staged) {
            // entry k of all the wavefront's chunks together
#pragma unroll
            for (int j = 0; j < R; ++j)
                nv[j] = 0.0;
            for (int k = 0; k < maxlen; ++k) {
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    if (k < len[j]) {
                        const int o = base[j] + lane + k * kSellC;
                        nv[j] = nv[j] + L.ltab[L.lvi[o]] * m[tid + j * kSmallThreads + L.lco[o]];
                    }
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < R; ++j)
                nv[j] = 0.0;
            for (int k = 0; k < maxlen; ++k) {
                // entry k of every row slot: loads first, then the LDS gathers
                int cv[R];
                double vv[R];
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    cv[j] = 0;
                    vv[j] = 0.0;
                    if (k < len[j]) {
                        const int o = base[j] + lane + k * kSellC;
                        cv[j] = col[o];
                        vv[j] = val[o];
                    }
                }
#pragma unroll
                for (int j = 0; j < R; ++j)
                    if (k < len[j])
                        nv[j] = nv[j] + vv[j] * m[cv[j]];
            }
        }
        __syncthreads();  // the new scalars visible; every wavefront past its reads of m and part
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int i = tid + j * kSmallThreads;
        if (i < n) {
            Z[i] = z[j];
            S[i] = s[j];
            P[i] = p[j];
            Rv[i] = r[j];
            Wv[i] = w[j];
            NVv[i] = nv[j];
            X[i] = x[j];
        }
    }
    if (tid < (int)(sizeof(SysState) / sizeof(int)))
        as_global((int *)st)[tid] = ((const int *)&L.loc)[tid];
}

__global__ __launch_bounds__(kSmallThreads) void k_small_iter(const WorkItem *__restrict__ table,
                                                              const int *__restrict__ count,
                                                              const SysDesc *__restrict__ descs, int iters)
{
    __shared__ SmallLds L;
    if ((int)blockIdx.x >= *count)
        return;
    const SysDesc &d = descs[table[blockIdx.x].slot];
    // (with lists of 7 the addresses do not fit the registers beside the vectors)
    if (d.schunk && d.smaxlen > 0 && d.smaxlen <= 5)
        small_run<5>(d, iters, L);
    else
        small_run<0>(d, iters, L);
}

}  // namespace ppcg
