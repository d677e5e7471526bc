// sigma = H v on a space of at most SEL_ONE (16 384) determinants, fast mode:
// H itself is kept, row by row, as a per-problem table (built on first use),
// and y = H v is a product with the dense copy of v.
//
// Why: on such a space the tile kernel's time is a chain of dependent memory
// round trips (item, description, row bounds, records, entries), ~54 us for
// the 8-orbital, 6-electron space whatever v holds, where reading all of H
// (3 136 rows of 316 entries, 12 MB) takes 5.  The table is limited to
// SMALL_H_BYTES, whose read costs what the tile kernel's latency does.
//
// H is symmetric to the bit (the reversed excitation has the same spectators
// in the same order of additions), so row k holds what enumerating k as a
// source gives, in that order, zero elements included (a fixed row length).
// A product with the whole row also meets the determinants that v does not
// hold, which adds +-0 for a finite element only: with an element that is not
// (infinite integrals, an overflow) the table is not used.
#include <algorithm>

#include "sfci_internal.h"

namespace {

constexpr u64 SMALL_H_BYTES = 128ull << 20;

// One row's entries in the order they are enumerated.
struct SinkRow {
    u32* idx;
    double* val;
    u32 pos;   // wave-uniform
    u32 nonzero;
    bool odd;      // this lane met an element that is not finite
    __device__ __forceinline__ void operator()(bool ok, u64 tgt, double e, double, const Term&) {
        const u64 m = __ballot(ok);
        if (ok) {
            const u32 at = pos + (u32)__popcll(m & ((1ull << lane_id()) - 1ull));
            idx[at] = (u32)tgt;
            val[at] = e;
            odd = odd || !(fabs(e) < INFINITY);
        }
        pos += (u32)__popcll(m);
        nonzero += (u32)__popcll(__ballot(ok && e != 0.0));
    }
};

__global__ __launch_bounds__(SFCI_BLOCK) void k_small_build(SpaceDev sp, Ints I, const u64* __restrict__ binom,
                                                            u32 tps, u32* __restrict__ idx,
                                                            double* __restrict__ val, u32* __restrict__ nz) {
    __shared__ BinomLds B;
    __shared__ WaveLds W[SFCI_WAVES_PER_BLOCK];
    load_binom(B, binom);
    __syncthreads();
    const int wave = threadIdx.x >> 6;
    const u64 N = sp.Na * sp.Nb;
    for (u64 k = (u64)blockIdx.x * SFCI_WAVES_PER_BLOCK + wave; k < N; k += (u64)gridDim.x * SFCI_WAVES_PER_BLOCK) {
        SinkRow sink{idx + k * tps, val + k * tps, 0u, 0u, false};
        enumerate_source<false, SinkRow, true>(sp, I, B, W[wave], k, 1.0, AlphaRange{0, 0}, sink);
        if (lane_id() == 0) nz[k] = sink.nonzero;
        if (sink.odd) nz[N] = 1u;  // (zero before)
    }
}

// A call's input, one workgroup: flags[0] a rank >= N, flags[1] not strictly
// ascending (checked when check != 0; a bad vector counts as empty); the dense
// copy of v, its length, and its terms added to *emitted.
__global__ __launch_bounds__(1024) void k_small_load(const u64* __restrict__ r, const double* __restrict__ a,
                                                     const u64* __restrict__ n_dev, u64 n_host, int check, u64 N,
                                                     const u32* __restrict__ nz, double* __restrict__ vd,
                                                     u64* __restrict__ nnz_out, u64* __restrict__ hist,
                                                     u64* __restrict__ emitted, int* __restrict__ flags) {
    __shared__ int bad[2];
    __shared__ unsigned long long terms;
    const u64 n = n_dev ? *n_dev : n_host;
    if (threadIdx.x == 0) {
        bad[0] = bad[1] = 0;
        terms = 0;
    }
    for (u64 i = threadIdx.x; i < N; i += 1024) vd[i] = 0.0;
    __syncthreads();
    if (check)
        for (u64 i = threadIdx.x; i < n; i += 1024) {
            if (r[i] >= N) bad[0] = 1;
            if (i > 0 && r[i] <= r[i - 1]) bad[1] = 1;
        }
    __syncthreads();
    const bool ok = !bad[0] && !bad[1];
    unsigned long long t = 0;
    if (ok)
        for (u64 i = threadIdx.x; i < n; i += 1024) {
            vd[r[i]] = a[i];
            t += nz[r[i]];
        }
    for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off);
    if ((threadIdx.x & 63) == 0 && t) atomicAdd(&terms, t);
    __syncthreads();
    if (threadIdx.x == 0) {
        if (nnz_out) *nnz_out = ok ? n : 0;
        if (hist) *hist = n;
        *emitted += terms;
        if (check) {
            flags[0] = bad[0];
            flags[1] = bad[1];
        }
    }
}

// y_k = sum of row k times v, a wavefront per row; every slot of D is written.
// Bound by the read of H (12 B per entry; v comes from the caches).
__global__ __launch_bounds__(256) void k_small_sigma(u64 N, u32 tps, const u32* __restrict__ idx,
                                                     const double* __restrict__ val, const double* __restrict__ vd,
                                                     double eps, double* __restrict__ D) {
    const u64 k = (u64)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (k >= N) return;
    const int lane = threadIdx.x & 63;
    const u32* ir = idx + k * tps;
    const double* vr = val + k * tps;
    constexpr int U = 4;
    double s = 0.0;
    for (u32 t0 = 0; t0 < tps; t0 += 64 * U) {
        u32 x[U];
        double e[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const u32 t = t0 + (u32)u * 64 + lane;
            x[u] = t < tps ? ir[t] : 0u;
            e[u] = t < tps ? vr[t] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (e[u] != 0.0) s += e[u] * vd[x[u]];
    }
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    if (lane == 0) D[k] = (eps > 0.0 && fabs(s) < eps) ? 0.0 : s;
}

}  // namespace

bool small_h_ready(sfci_problem* P) {
    if (P->sh_state != 0) return P->sh_state > 0;
    P->sh_state = -1;
    const u64 tps = terms_per_source(P->n, P->na, P->nb), N = P->Ndet;
    if (N > (u64)SEL_ONE || N * tps * 12 > SMALL_H_BYTES) return false;
    const auto drop = [&] {
        for (DevBuf* b : {&P->sh_idx, &P->sh_val, &P->sh_nz, &P->sh_vd}) b->release();
        return false;
    };
    u32 *idx, *nz;
    double* val;
    try {
        idx = (u32*)P->sh_idx.get(N * tps * sizeof(u32));
        val = (double*)P->sh_val.get(N * tps * sizeof(double));
        nz = (u32*)P->sh_nz.get((N + 2) * sizeof(u32));  // terms per column, then the flag of an element not finite
        (void)P->sh_vd.get(N * sizeof(double));
    } catch (const sfci_error& e) {
        if (e.code != SFCI_E_NOMEM) throw;
        return drop();  // no room: the tile kernel serves
    }
    launch_fill_u64((u64*)(nz + (N & ~u64(1))), 1, 0, P->stream);
    const u64 want = (N + SFCI_WAVES_PER_BLOCK - 1) / SFCI_WAVES_PER_BLOCK;
    hipLaunchKernelGGL(k_small_build, dim3((unsigned)std::min<u64>(want, (u64)P->num_cu * 16)), dim3(SFCI_BLOCK), 0,
                       P->stream, SpaceDev{P->n, P->na, P->nb, P->Na, P->Nb}, Ints{P->d_h, P->d_g, P->n}, P->d_binom,
                       (u32)tps, idx, val, nz);
    SFCI_CHECK_HIP(hipGetLastError());
    u32 odd = 0;
    SFCI_CHECK_HIP(hipMemcpyAsync(&odd, nz + N, sizeof(u32), hipMemcpyDeviceToHost, P->stream));
    SFCI_CHECK_HIP(hipStreamSynchronize(P->stream));
    if (odd) return drop();
    small_step_setup(P);
    P->sh_state = 1;
    return true;
}

void launch_small_load(sfci_problem* P, const u64* r, const double* a, const u64* n_dev, u64 n_host, bool check,
                       u64* nnz_out, u64* hist, u64* emitted, int* flags) {
    hipLaunchKernelGGL(k_small_load, dim3(1), dim3(1024), 0, P->stream, r, a, n_dev, n_host, check ? 1 : 0, P->Ndet,
                       (const u32*)P->sh_nz.p, (double*)P->sh_vd.p, nnz_out, hist, emitted, flags);
    SFCI_CHECK_HIP(hipGetLastError());
}

void launch_small_sigma(sfci_problem* P, double eps) {
    hipLaunchKernelGGL(k_small_sigma, dim3((unsigned)((P->Ndet + 3) / 4)), dim3(256), 0, P->stream, P->Ndet,
                       (u32)terms_per_source(P->n, P->na, P->nb), (const u32*)P->sh_idx.p,
                       (const double*)P->sh_val.p, (const double*)P->sh_vd.p, eps, P->d_D);
    SFCI_CHECK_HIP(hipGetLastError());
}
