// Second-order Epstein-Nesbet correction of a variational vector Psi: the
// perturbative correction the paper leaves for future work (its comparison
// of the F2 result with ASCI and that method's Epstein-Nesbet correction).
// Standard partitioning with the diagonal of H as the zeroth-order operator:
//   E0 = <Psi|H|Psi> / <Psi|Psi>,
//   E2 = [ sum over k outside supp(Psi) of (H Psi)_k^2 / (E0 - H_kk) ] / <Psi|Psi>.
// Two forms:
//   * deterministic, or no room for the N_det array: the sort path gives H Psi
//     as a rank-sorted list; one pass forms E0's products over supp(Psi) (each
//     Psi rank searched in H Psi), one the external terms (each H Psi rank
//     searched in Psi) with H_kk in the diagonal element's fixed addition
//     order; deterministic sums run strictly in rank order (the bits of a
//     sequential evaluation);
//   * otherwise H Psi stays in the dense accumulator: E0 is a gather at
//     supp(Psi), those slots are cleared, and every slot still nonzero is an
//     external determinant, taken a target row at a time (k_pt2_rows).
#include <algorithm>

#include "sfci_internal.h"

namespace {

constexpr int PB = 256;

__device__ __forceinline__ bool find_rank(const u64* __restrict__ r, u64 n, u64 key, u64* pos) {
    u64 lo = 0, hi = n;
    while (lo < hi) {
        const u64 mid = lo + ((hi - lo) >> 1);
        if (r[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    *pos = lo;
    return lo < n && r[lo] == key;
}

// prod[t] = Psi_t * y(rank of Psi_t) (0 where H Psi has no entry): the
// products of <Psi|H Psi> in ascending rank (skipping the zero products of
// entries outside supp(Psi) leaves the ordered sum's bits unchanged)
__global__ __launch_bounds__(PB) void k_pt2_inner(const u64* __restrict__ yr, const double* __restrict__ ya,
                                                  const u64* __restrict__ ny, const u64* __restrict__ pr,
                                                  const double* __restrict__ pa, u64 np, double* __restrict__ prod) {
    const u64 n = *ny;
    for (u64 t = (u64)blockIdx.x * PB + threadIdx.x; t < np; t += (u64)gridDim.x * PB) {
        u64 pos;
        prod[t] = find_rank(yr, n, pr[t], &pos) ? pa[t] * ya[pos] : 0.0;
    }
}

__global__ void k_pt2_e0(const double* __restrict__ num, const double* __restrict__ den, double* __restrict__ e0) {
    if (threadIdx.x == 0) *e0 = *num / *den;
}

// prod[i] = y_i^2 / (E0 - H_kk) outside supp(Psi), else 0; counts the external entries
__global__ __launch_bounds__(PB) void k_pt2_outer(SpaceDev sp, Ints I, const u64* __restrict__ binom,
                                                  const u64* __restrict__ yr, const double* __restrict__ ya,
                                                  const u64* __restrict__ ny, const u64* __restrict__ pr, u64 np,
                                                  const double* __restrict__ e0p, double* __restrict__ prod,
                                                  unsigned long long* __restrict__ n_ext) {
    __shared__ BinomLds B;
    load_binom(B, binom);
    __syncthreads();
    const u64 n = *ny;
    const double E0 = *e0p;
    unsigned long long cnt = 0;
    for (u64 i = (u64)blockIdx.x * PB + threadIdx.x; i < n; i += (u64)gridDim.x * PB) {
        u64 pos;
        const double y = ya[i];
        double t = 0.0;
        if (y != 0.0 && !find_rank(pr, np, yr[i], &pos)) {
            const u64 ra = yr[i] / sp.Nb;
            const u32 A = str_unrank(ra, sp.na, sp.n, B);
            const u32 Bs = str_unrank(yr[i] - ra * sp.Nb, sp.nb, sp.n, B);
            const double hkk = diag_element(I, A, Bs);
            t = (y * y) / (E0 - hkk);
            ++cnt;
        }
        prod[i] = t;
    }
    for (int off = 32; off >= 1; off >>= 1) cnt += __shfl_xor(cnt, off);
    if ((threadIdx.x & 63) == 0 && cnt) atomicAdd(n_ext, cnt);
}

// The beta strings, by rank.
__global__ __launch_bounds__(PB) void k_pt2_beta(SpaceDev sp, const u64* __restrict__ binom, u32* __restrict__ bits) {
    __shared__ BinomLds B;
    load_binom(B, binom);
    __syncthreads();
    for (u64 r = (u64)blockIdx.x * PB + threadIdx.x; r < sp.Nb; r += (u64)gridDim.x * PB)
        bits[r] = str_unrank(r, sp.nb, sp.n, B);
}

// The external terms straight from the accumulator, a workgroup per target
// alpha row (or one of segs stretches of it, where rows are few), which clears
// the slots it reads.  H_kk is summed in diag_element's order, so its bits (and
// E0 - H_kk where the two nearly meet) are the list form's: the alpha parts are
// formed once per row, the pair terms come from LDS.  Where most slots hold a
// sum, a lane takes its own four; else they queue in LDS, so that a short Psi
// pays for the determinants it reaches (H_kk formed for every slot took 8.7 ms
// of one entry in 6.9e8 slots at 22 orbitals, the list form 3.9, this 2.7).
// Bound by the adds and LDS reads of H_kk, or the read of the accumulator; the
// list form (compaction, a binary search in Psi, two unranks and ~28 gathers of
// integrals per entry) took 1040 us where this takes 248 us (20 orbitals,
// 2.0e7 external determinants).
constexpr int PT_U = 4, PT_Q = 2 * 128;  // slots a lane takes together; queue of a wavefront
__global__ __launch_bounds__(PB) void k_pt2_rows(SpaceDev sp, Ints I, const u64* __restrict__ binom,
                                                 double* __restrict__ D, const u32* __restrict__ bits, u32 segs,
                                                 const double* __restrict__ e0p, double* __restrict__ part,
                                                 unsigned long long* __restrict__ n_ext) {
    __shared__ BinomLds B;
    __shared__ double K2[32 * 32], J[32 * 32], hd[32], ka[32 * 31 / 2], ea, wsum[PB / 64];
    __shared__ double qy[PB / 64][PT_Q];
    __shared__ u32 qb[PB / 64][PT_Q];
    __shared__ uint8_t occ[32];
    load_binom(B, binom);
    const int n = sp.n, na = sp.na;
    for (int t = threadIdx.x; t < n * n; t += PB) {
        const int p = t / n, q = t - p * n;
        J[t] = I.G(p, p, q, q);
        K2[t] = (I.G(p, p, q, q) - I.G(p, q, q, p));
    }
    if (threadIdx.x < (unsigned)n) hd[threadIdx.x] = I.H(threadIdx.x, threadIdx.x);
    __syncthreads();
    const double E0 = *e0p;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, npair = na * (na - 1) / 2;
    double* const wy = qy[wave];
    u32* const wb = qb[wave];
    unsigned long long cnt = 0;
    double sum = 0.0;
    // H_kk of the current row's determinants with beta strings bt
    const auto diagonal = [&](const auto& bt, auto& e) {
        constexpr int U = sizeof(bt) / sizeof(bt[0]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            e[u] = ea;
            for (u32 m = bt[u]; m; m &= m - 1u) e[u] += hd[__builtin_ctz(m)];
        }
        for (int t = 0; t < npair; ++t) {
            const double k = ka[t];
#pragma unroll
            for (int u = 0; u < U; ++u) e[u] += k;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            for (u32 m = bt[u]; m; m &= m - 1u) {
                const double* Kp = K2 + __builtin_ctz(m) * n;
                for (u32 m2 = m & (m - 1u); m2; m2 &= m2 - 1u) e[u] += Kp[__builtin_ctz(m2)];
            }
        for (int t = 0; t < na; ++t) {
            const double* Jp = J + occ[t] * n;
#pragma unroll
            for (int u = 0; u < U; ++u)
                for (u32 m = bt[u]; m; m &= m - 1u) e[u] += Jp[__builtin_ctz(m)];
        }
    };
    // the queue's last up to 128 determinants, two a lane
    const auto take = [&](int& queued) {
        const int first = queued > 128 ? queued - 128 : 0;
        wave_sync();
        double y[2], e[2];
        u32 bt[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int q = first + u * 64 + lane;
            y[u] = q < queued ? wy[q] : 0.0;
            bt[u] = q < queued ? wb[q] : 0u;
        }
        wave_sync();
        diagonal(bt, e);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (y[u] == 0.0) continue;
            sum += (y[u] * y[u]) / (E0 - e[u]);
            ++cnt;
        }
        queued = first;
    };
    const u64 len = (sp.Nb + segs - 1) / segs;
    for (u64 item = blockIdx.x; item < sp.Na * segs; item += gridDim.x) {
        const u64 row = item / segs, x_lo = (item - row * segs) * len, x_hi = min(sp.Nb, x_lo + len);
        const u32 A = str_unrank_wave(row, na, n, B);
        __syncthreads();  // the previous row's tables are no longer read
        if (threadIdx.x < (unsigned)n && ((A >> threadIdx.x) & 1u))
            occ[__popc(A & ((1u << threadIdx.x) - 1u))] = (uint8_t)threadIdx.x;
        if (threadIdx.x == PB - 1) {
            double e = 0.0;
            for (u32 m = A; m; m &= m - 1u) e += hd[__builtin_ctz(m)];
            ea = e;
        }
        __syncthreads();
        for (int t = threadIdx.x; t < npair; t += PB) {
            const uint16_t pr = decode_pair(t, na);  // lexicographic: diag_element's order
            ka[t] = K2[occ[pr & 255] * n + occ[pr >> 8]];
        }
        __syncthreads();
        double* const Dr = D + row * sp.Nb;
        int queued = 0;
        for (u64 x0 = x_lo + threadIdx.x; x0 - threadIdx.x < x_hi; x0 += (u64)PB * PT_U) {
            double y[PT_U];
            u32 bt[PT_U];
#pragma unroll
            for (int u = 0; u < PT_U; ++u) {
                const u64 x = x0 + (u64)u * PB;
                y[u] = x < x_hi ? Dr[x] : 0.0;
                bt[u] = x < x_hi ? bits[x] : 0u;
            }
            u64 m[PT_U];
            int here = 0;
#pragma unroll
            for (int u = 0; u < PT_U; ++u) {
                m[u] = __ballot(y[u] != 0.0);
                here += __popcll(m[u]);
                if (y[u] != 0.0) Dr[x0 + (u64)u * PB] = 0.0;
            }
            if (here == 0) continue;
            if (here > 128) {
                double e[PT_U];
                diagonal(bt, e);
#pragma unroll
                for (int u = 0; u < PT_U; ++u) {
                    if (y[u] == 0.0) continue;
                    sum += (y[u] * y[u]) / (E0 - e[u]);
                    ++cnt;
                }
                continue;
            }
#pragma unroll
            for (int u = 0; u < PT_U; ++u) {
                const int at = queued + __popcll(m[u] & ((1ull << lane) - 1ull));
                if (y[u] != 0.0) {
                    wy[at] = y[u];
                    wb[at] = bt[u];
                }
                queued += __popcll(m[u]);
            }
            if (queued >= 128) take(queued);
        }
        if (queued) take(queued);
    }
    for (int off = 32; off >= 1; off >>= 1) {
        cnt += __shfl_xor(cnt, off);
        sum += __shfl_xor(sum, off);
    }
    if (lane == 0) {
        if (cnt) atomicAdd(n_ext, cnt);
        wsum[wave] = sum;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < PB / 64; ++w) s += wsum[w];
        part[blockIdx.x] = s;
    }
}

unsigned grid_of(u64 n) {
    u64 g = (n + PB - 1) / PB;
    return (unsigned)std::max<u64>(1, std::min<u64>(g, 16384));
}

}  // namespace

// H Psi as a rank-sorted list: the dense accumulator compacted in rank order
// (the in-order kernel in deterministic mode, the tile kernel otherwise), or
// the sort path where those do not apply.
u64 sigma_full_list(sfci_problem* P, const SigmaLaunch& sl, bool det, u64* emitted, u64** yr, double** ya,
                    u64* cnt_dev) {
    RowTileDesc iod;
    const bool inorder = det && inorder_available(P, sl.cap) && ensure_dense(P) && inorder_pays(P, sl, &iod);
    if (!inorder && (det || !ensure_dense(P))) {
        const u64 n = sigma_list_full(P, sl, emitted, yr, ya);
        launch_set_u64(P, cnt_dev, n);
        return n;
    }
    DenseGuard dense(P);
    if (inorder) launch_sigma_inorder(P, sl, iod, P->d_D, (unsigned long long*)emitted, 0.0);
    else dense_sigma(P, sl, SFCI_DEDUP_DENSE, (unsigned long long*)emitted);
    CandSrc src{};
    src.dense = P->d_D;
    select_prepare(P, src, UINT64_MAX, cnt_dev);
    u64 n = 0;
    SFCI_CHECK_HIP(hipMemcpyAsync(&n, cnt_dev, sizeof(u64), hipMemcpyDeviceToHost, P->stream));
    SFCI_CHECK_HIP(hipStreamSynchronize(P->stream));
    *yr = (u64*)P->ws_list_r.get(std::max<u64>(1, n) * sizeof(u64));
    *ya = (double*)P->ws_list_a.get(std::max<u64>(1, n) * sizeof(double));
    select_write(P, src, *yr, *ya, true);  // rank order; zeroes the accumulator
    dense.done();
    return n;
}

// Gradients of E = <Psi|H|Psi>/<Psi|Psi> at fixed Psi (Hellmann-Feynman form):
// the backward of sigma with v = Psi and cotangent Psi/<Psi|Psi>.  sc[0] holds
// nnz(Psi) on the device; sc[5] is scratch for the transposed vector's count.
void energy_gradients_at(sfci_problem* P, const sfci_svec* psi, u64* sc, double* dh, double* deri) {
    const int n = P->n;
    const u64 n2 = (u64)n * n, n4 = n2 * n2;
    double* sbar = (double*)P->ws_cand_a.get(psi->nnz * sizeof(double));
    launch_div_by_sumsq(P, psi->amp, sc, psi->nnz, sbar);
    double* raw = (double*)P->ws_red.get((2048 + n2 + n4) * sizeof(double));
    const SigmaLaunch sl{psi->rank, psi->amp, sc, psi->nnz};
    DenseGuard dense(P);
    if (rowtile_grad_available(P)) {
        GradJob J{};
        J.P = P;
        J.v = sl;
        J.s_rank = psi->rank;
        J.s_amp = sbar;
        J.s_nnz = sc;
        J.s_cap = psi->nnz;
        J.Rh = raw + 2048;
        J.Rg = raw + 2048 + n2;
        J.dh = dh;
        J.dg = deri;
        J.vt_rank = (u64*)P->ws_list_r.get(psi->nnz * sizeof(u64));
        J.vt_amp = (double*)P->ws_list_a.get(psi->nnz * sizeof(double));
        J.vt_nnz = sc + 5;
        J.pair_sym = true;  // sbar = Psi / <Psi|Psi>
        rowtile_gradients(P->stream, 1, &J, P->grad_ws);
    } else {
        launch_scatter_set(P, P->d_D, psi->rank, sbar, sc, psi->nnz);
        launch_backward_dense(P, sl, P->d_D, nullptr, dh, deri, raw + 2048, raw + 2048 + n2);
        launch_scatter_zero(P, P->d_D, psi->rank, sc, psi->nnz);
    }
    dense.done();
}

extern "C" sfci_status sfci_energy_gradients(sfci_problem* P, const sfci_svec* psi, int32_t deterministic,
                                             double* energy, double* dh, double* deri) {
    try {
        if (!P || !psi || !energy) return (sfci_status)sfci_set_error(SFCI_E_ARG, "NULL argument");
        if (psi->nnz == 0 || !psi->rank || !psi->amp)
            return (sfci_status)sfci_set_error(SFCI_E_ARG, "empty vector");
        validate_vec(P, psi->rank, psi->nnz);
        P->excite_eps = 0.0;  // the energy of the full H
        if ((dh || deri) && !ensure_dense(P))
            return (sfci_status)sfci_set_error(SFCI_E_UNSUPPORTED, "gradients need the dense array (N_det doubles)");
        const bool det = deterministic != 0;
        u64* sc = (u64*)P->ws_lz[0].get(16 * sizeof(u64));  // [0] nnz(Psi) [1] emitted [2] |y| [5] scratch
        double* sd = (double*)(sc + 8);                     // [0] num [1] den [2] E
        launch_fill_u64(sc, 16, 0, P->stream);
        launch_set_u64(P, sc, psi->nnz);
        const SigmaLaunch sl{psi->rank, psi->amp, sc, psi->nnz};
        if (!det && ensure_dense(P)) {
            // H Psi in the accumulator, gathered at supp(Psi)
            DenseGuard dense(P);
            dense_sigma(P, sl, SFCI_DEDUP_AUTO, (unsigned long long*)(sc + 1));
            launch_dot_dense(P, psi->rank, psi->amp, sc, psi->nnz, P->d_D, sd + 0, nullptr, false);
            launch_fill_f64(P->d_D, P->Ndet, 0.0, P->stream);
            dense.done();
        } else {
            u64* yr;
            double* ya;
            sigma_full_list(P, sl, det, sc + 1, &yr, &ya, sc + 2);
            double* prod = (double*)P->ws_prod.get(std::max<u64>(1, psi->nnz) * sizeof(double));
            hipLaunchKernelGGL(k_pt2_inner, dim3(grid_of(psi->nnz)), dim3(PB), 0, P->stream, yr, ya, sc + 2,
                               psi->rank, psi->amp, (u64)psi->nnz, prod);
            launch_sum(P, prod, sc, psi->nnz, sd + 0, det);
        }
        launch_sumsq(P, psi->amp, sc, psi->nnz, sd + 1, det);
        hipLaunchKernelGGL(k_pt2_e0, dim3(1), dim3(64), 0, P->stream, sd + 0, sd + 1, sd + 2);
        SFCI_CHECK_HIP(hipGetLastError());
        if (dh || deri) energy_gradients_at(P, psi, sc, dh, deri);
        double hd[3];
        SFCI_CHECK_HIP(hipMemcpyAsync(hd, sd, sizeof(hd), hipMemcpyDeviceToHost, P->stream));
        SFCI_CHECK_HIP(hipStreamSynchronize(P->stream));
        if (!(hd[1] > 0.0)) return (sfci_status)sfci_set_error(SFCI_E_ARG, "Psi has zero norm");
        *energy = hd[2];
        return SFCI_OK;
    } catch (const sfci_error& e) {
        return (sfci_status)sfci_set_error(e.code, e.msg);
    }
}

extern "C" sfci_status sfci_pt2(sfci_problem* P, const sfci_svec* psi, int32_t deterministic, double* e0,
                                double* e2, uint64_t* n_external) {
    try {
        if (!P || !psi || !e0 || !e2) return (sfci_status)sfci_set_error(SFCI_E_ARG, "NULL argument");
        if (psi->nnz == 0 || !psi->rank || !psi->amp)
            return (sfci_status)sfci_set_error(SFCI_E_ARG, "empty vector");
        validate_vec(P, psi->rank, psi->nnz);
        P->excite_eps = 0.0;  // the correction of the full H
        const bool det = deterministic != 0;
        u64* sc = (u64*)P->ws_lz[0].get(16 * sizeof(u64));  // [0] nnz(Psi) [1] emitted [2] |y| [3] n_ext
        double* sd = (double*)(sc + 8);                     // [0] num [1] den [2] E0 [3] sum
        launch_fill_u64(sc, 16, 0, P->stream);
        launch_set_u64(P, sc, psi->nnz);
        const SigmaLaunch sl{psi->rank, psi->amp, sc, psi->nnz};
        const SpaceDev sp{P->n, P->na, P->nb, P->Na, P->Nb};
        const Ints I{P->d_h, P->d_g, P->n};
        if (!det && ensure_dense(P)) {
            DenseGuard dense(P);
            dense_sigma(P, sl, SFCI_DEDUP_AUTO, (unsigned long long*)(sc + 1));
            launch_dot_dense(P, psi->rank, psi->amp, sc, psi->nnz, P->d_D, sd + 0, nullptr, false);
            launch_sumsq(P, psi->amp, sc, psi->nnz, sd + 1, false);
            hipLaunchKernelGGL(k_pt2_e0, dim3(1), dim3(64), 0, P->stream, sd + 0, sd + 1, sd + 2);
            launch_scatter_zero(P, P->d_D, psi->rank, sc, psi->nnz);
            // a partial sum per workgroup, then the N_beta strings; eight workgroups to a compute unit
            const u64 most = (u64)P->num_cu * 8;
            const u32 segs = (u32)std::max<u64>(1, std::min<u64>(most / P->Na, P->Nb / 2048));
            const unsigned g = (unsigned)std::min<u64>(P->Na * segs, most);
            double* part = (double*)P->ws_prod.get(g * sizeof(double) + P->Nb * sizeof(u32));
            u32* bits = (u32*)(part + g);
            hipLaunchKernelGGL(k_pt2_beta, dim3(grid_of(P->Nb)), dim3(PB), 0, P->stream, sp, P->d_binom, bits);
            hipLaunchKernelGGL(k_pt2_rows, dim3(g), dim3(PB), 0, P->stream, sp, I, P->d_binom, P->d_D, bits, segs,
                               sd + 2, part, (unsigned long long*)(sc + 3));
            dense.done();
            launch_set_u64(P, sc + 2, g);
            launch_sum(P, part, sc + 2, g, sd + 3, false);
        } else {
            u64* yr;
            double* ya;
            const u64 ny = sigma_full_list(P, sl, det, sc + 1, &yr, &ya, sc + 2);
            double* prod = (double*)P->ws_prod.get(std::max<u64>(std::max<u64>(1, ny), psi->nnz) * sizeof(double));
            hipLaunchKernelGGL(k_pt2_inner, dim3(grid_of(psi->nnz)), dim3(PB), 0, P->stream, yr, ya, sc + 2,
                               psi->rank, psi->amp, (u64)psi->nnz, prod);
            launch_sum(P, prod, sc, psi->nnz, sd + 0, det);
            launch_sumsq(P, psi->amp, sc, psi->nnz, sd + 1, det);
            hipLaunchKernelGGL(k_pt2_e0, dim3(1), dim3(64), 0, P->stream, sd + 0, sd + 1, sd + 2);
            hipLaunchKernelGGL(k_pt2_outer, dim3(grid_of(ny)), dim3(PB), 0, P->stream, sp, I, P->d_binom, yr, ya,
                               sc + 2, psi->rank, (u64)psi->nnz, sd + 2, prod, (unsigned long long*)(sc + 3));
            launch_sum(P, prod, sc + 2, std::max<u64>(1, ny), sd + 3, det);
        }
        SFCI_CHECK_HIP(hipGetLastError());
        double hd[4];
        u64 hc[4];
        SFCI_CHECK_HIP(hipMemcpyAsync(hd, sd, sizeof(hd), hipMemcpyDeviceToHost, P->stream));
        SFCI_CHECK_HIP(hipMemcpyAsync(hc, sc, sizeof(hc), hipMemcpyDeviceToHost, P->stream));
        SFCI_CHECK_HIP(hipStreamSynchronize(P->stream));
        if (!(hd[1] > 0.0)) return (sfci_status)sfci_set_error(SFCI_E_ARG, "Psi has zero norm");
        *e0 = hd[2];
        *e2 = hd[3] / hd[1];
        if (n_external) *n_external = hc[3];
        return SFCI_OK;
    } catch (const sfci_error& e) {
        return (sfci_status)sfci_set_error(e.code, e.msg);
    }
}
