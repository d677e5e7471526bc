// Backward of sigma = H v with vbar, row by row: the input's entries are taken
// in chunks of up to 64 of one alpha row A, and a wavefront works on one
// (chunk, kind) item:
//   * alpha-beta doubles of one alpha single i -> a of A: lanes over the beta
//     singles (tabulated), entries in turn; the cotangent is read within the
//     one target row, the weights of the chunk's entries collect in an LDS
//     slab over (j, b) and reach dL/d(ia|jb) once (collecting them over many
//     chunks leaves too few, too uneven items: 491 -> 932 us);
//   * alpha singles and alpha-alpha doubles, beta unchanged: lanes over 64 of
//     A's neighbours, whose element and weight sum stay in registers;
//   * beta singles and beta-beta doubles: the same with the spins exchanged,
//     on chunks of entries that share a beta string (a counting sort of the
//     entries); taken on A's chunks they meet other integrals with every
//     entry, an atomic each (410 -> 277 us with this);
//   * the diagonal: a lane per entry.
// Same-spin doubles add their weight to one slot per orbital pair of pairs
// (R4), which k_expand_pairs spreads over (ia|jb) and (ib|ja).  vbar's partial
// sums are wavefront reductions, added per entry.
//
// Why: the general kernel (backward.hip) walks every source on its own --
// ranks, integrals and cotangent gathered per term, one global FP64 atomic or
// more per term that meets the cotangent (2.4e10 of them per second on this
// device) -- at 2.6e10 terms/s.  16 orbitals, 8 electrons, 1e4 entries against
// 2e5: k_backward 1233 us -> 277 us here (the call 1290 -> 414
// us); 20 orbitals, 9e5 against 9e5: 23.6 ms a call.  Without vbar the tile
// passes (rowtile.hip) stay: they read each row once for all its sources
// (7.3 ms there).
#include <algorithm>
#include <cmath>

#include "sfci_internal.h"

namespace {

constexpr int BW_WAVES = 4;
constexpr int BW_BLOCK = 64 * BW_WAVES;
constexpr int BW_U = 4;  // entries whose loads are in flight together

struct BackRows {
    SpaceDev sp;
    Ints I;
    const u64* binom;
    const double* v_amp;
    const u32* v_beta;  // beta string and beta rank per entry
    const u32* v_rb;
    const uint4* chunk;  // (alpha row, first entry, entries, alpha string)
    const u32* n_chunk;
    // the entries by beta string: chunks (beta rank, first, entries, beta string) of the permuted
    // arrays original entry, alpha rank, alpha string
    const uint4* chunk_b;
    const u32* n_chunk_b;
    const u32 *pk, *pra, *pA;
    const u32* T1;  // beta singles per beta rank: rank | (j n + b) << 21 | phase << 31
    const double* K4;
    const double* Sd;       // dense cotangent
    const u32* row_used;    // per alpha row: the cotangent has an entry there
    double* vbar;
    double *Rh, *Rg, *R4;
    int sA, sB, PA, QA, PB, QB;
    u32 k_dir, kinds;  // of a row's chunk: [0, sA) alpha-beta, [sA, k_dir) alpha neighbours, then the diagonal
    u32 kinds_b;       // of a beta string's chunk: its neighbours by 64
};

__device__ __forceinline__ u32 pair_slot(int x, int y) { return (u32)(y * (y - 1) / 2 + x); }  // x < y

// One chunk's alpha-beta doubles i -> a (target row r2): weights into the slab,
// vbar's sums to its entries; false when the cotangent met none of them.
__device__ __forceinline__ bool back_alpha_beta(const BackRows& p, double* slab, int lane, int i, int a, u32 A,
                                                u32 r2, u32 k0, int cnt) {
    const u32 n = (u32)p.sp.n;
    const double sg = between_parity(A, i, a) ? -1.0 : 1.0;
    const double* Sr = p.Sd + (u64)r2 * p.sp.Nb;
    const double* Gia = p.I.g + ((u32)i * n + a) * (n * n);
    u32 rk = 0;
    double ck = 0.0, vacc = 0.0;
    if (lane < cnt) {
        rk = p.v_rb[k0 + lane];
        ck = sg * p.v_amp[k0 + lane];
    }
    bool any = false;
    for (int s0 = 0; s0 < p.sB; s0 += 64) {
        const int sidx = s0 + lane;
        const bool act = sidx < p.sB;
        for (int q0 = 0; q0 < cnt; q0 += BW_U) {
            u32 te[BW_U];
            double sb[BW_U], x[BW_U];
#pragma unroll
            for (int u = 0; u < BW_U; ++u) {
                const u32 r = (u32)__builtin_amdgcn_readlane((int)rk, min(q0 + u, cnt - 1));
                te[u] = act ? p.T1[(u64)r * (u32)p.sB + sidx] : 0u;
            }
#pragma unroll
            for (int u = 0; u < BW_U; ++u) {
                sb[u] = (act && q0 + u < cnt) ? Sr[te[u] & 0x1FFFFFu] : 0.0;
                x[u] = Gia[(te[u] >> 21) & 1023u];
            }
#pragma unroll
            for (int u = 0; u < BW_U; ++u) {
                if (__ballot(sb[u] != 0.0) == 0) continue;
                any = true;
                const u32 jb = (te[u] >> 21) & 1023u;
                const double ss = (te[u] >> 31) ? -sb[u] : sb[u];
                if (sb[u] != 0.0) atomicAdd(&slab[jb], ss * lane_f64(ck, q0 + u));
                const double tot = wave_sum_dpp(sb[u] != 0.0 ? x[u] * ss : 0.0);
                if (lane == q0 + u) vacc += tot;
            }
        }
    }
    if (p.vbar && vacc != 0.0) unsafeAtomicAdd(p.vbar + k0 + lane, sg * vacc);  // (lanes past cnt hold 0)
    return any;
}

// A chunk's terms with the other spin unchanged: 64 neighbours of the chunk's
// string S (its sA singles, then its doubles), entries in turn.  Entry e of
// the chunk has the other spin's rank ro and string so (a lane each); the
// cotangent of neighbour r2 and entry e is at row(r2) + ro step.  Returns this
// lane's entry's share of vbar.
template <class Row, class Used>
__device__ __forceinline__ double back_neighbours(const BackRows& p, double* slab, int lane, u32 S, const uint8_t* occ,
                                                  const uint8_t* vir, int singles, int doubles, int Q,
                                                  const uint16_t* pO, const uint16_t* pV, const BinomLds& B, int group,
                                                  int cnt, double ck, u32 so, const Row& row, u32 ro, u64 step,
                                                  const Used& used) {
    const int n = p.sp.n;
    const u32 np2 = (u32)(n * (n - 1) / 2);
    auto gi = [&](int a, int b, int c, int d) { return (((u32)a * n + b) * n + c) * n + d; };
    const int t = group * 64 + lane;
    const bool single = t < singles;
    const bool dbl = !single && t < singles + doubles;
    int i = 0, a = 0, j = 0, b = 0, par = 0;
    u32 S2 = S;
    double e0 = 0.0;
    if (single) {
        const int nv = n - __popc(S);
        i = occ[t / nv];
        a = vir[t % nv];
        S2 = S ^ (1u << i) ^ (1u << a);
        par = between_parity(S, i, a);
        e0 = p.I.H(i, a);
        for (u32 m = S & ~(1u << i); m; m &= m - 1u) {
            const int k = __builtin_ctz(m);
            e0 += (p.I.G(i, a, k, k) - p.I.G(i, k, k, a));
        }
    } else if (dbl) {
        const int x = t - singles;
        const unsigned po = pO[x / Q], pv = pV[x % Q];
        i = occ[po & 255];
        j = occ[po >> 8];
        a = vir[pv & 255];
        b = vir[pv >> 8];
        const u32 mid = S ^ (1u << i) ^ (1u << a);
        S2 = mid ^ (1u << j) ^ (1u << b);
        par = between_parity(S, i, a) ^ between_parity(mid, j, b);
        e0 = p.K4[pair_slot(i, j) * np2 + pair_slot(a, b)];
    }
    const u32 r2 = (u32)str_rank(S2, B);
    const bool on = (single || dbl) && used(r2);
    if (__ballot(on) == 0) return 0.0;
    const double sg = par ? -1.0 : 1.0;
    const double* Sr = p.Sd + row(r2);
    double* const O = slab + lane * n;  // singles: the weight by occupied orbital of the other spin
    const bool singles_here = __ballot(single) != 0;
    double W = 0.0, vacc = 0.0;
    for (int q0 = 0; q0 < cnt; q0 += BW_U) {
        double sb[BW_U];
#pragma unroll
        for (int u = 0; u < BW_U; ++u) {
            const u64 r = (u32)__builtin_amdgcn_readlane((int)ro, min(q0 + u, cnt - 1));
            sb[u] = (on && q0 + u < cnt) ? sg * Sr[r * step] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < BW_U; ++u) {
            if (__ballot(sb[u] != 0.0) == 0) continue;
            // (no term where the cotangent is zero, whatever the amplitude: an infinite one would leave NaN)
            const double w = sb[u] != 0.0 ? sb[u] * lane_f64(ck, q0 + u) : 0.0;
            W += w;
            double e = e0;
            if (singles_here) {
                for (u32 m = (u32)__builtin_amdgcn_readlane((int)so, q0 + u); m; m &= m - 1u) {
                    const int k = __builtin_ctz(m);
                    if (single) {
                        e += p.I.G(i, a, k, k);
                        O[k] += w;
                    }
                }
            }
            const double tot = wave_sum_dpp(sb[u] != 0.0 ? e * sb[u] : 0.0);
            if (lane == q0 + u) vacc += tot;
        }
    }
    if (single && on) {
        if (W != 0.0) {
            unsafeAtomicAdd(p.Rh + i * n + a, W);
            for (u32 m = S & ~(1u << i); m; m &= m - 1u) {
                const int k = __builtin_ctz(m);
                unsafeAtomicAdd(p.Rg + gi(i, a, k, k), W);
                unsafeAtomicAdd(p.Rg + gi(i, k, k, a), -W);
            }
        }
        for (int k = 0; k < n; ++k) {
            const double x = O[k];
            if (x != 0.0) {
                unsafeAtomicAdd(p.Rg + gi(i, a, k, k), x);
                O[k] = 0.0;
            }
        }
    } else if (dbl && on && W != 0.0) {
        unsafeAtomicAdd(p.R4 + pair_slot(i, j) * np2 + pair_slot(a, b), W);
    }
    return vacc;
}

__global__ __launch_bounds__(BW_BLOCK) void k_back_rows(BackRows p) {
    extern __shared__ double lds[];
    __shared__ BinomLds B;
    __shared__ uint16_t pairOA[SFCI_MAX_PAIRS], pairVA[SFCI_MAX_PAIRS], pairOB[SFCI_MAX_PAIRS], pairVB[SFCI_MAX_PAIRS];
    __shared__ uint8_t s_occ[BW_WAVES][32], s_vir[BW_WAVES][32];
    load_binom(B, p.binom);
    const int n = p.sp.n, na = p.sp.na, nb = p.sp.nb, nva = n - na, nvb = n - nb;
    for (int t = threadIdx.x; t < p.PA; t += BW_BLOCK) pairOA[t] = decode_pair(t, na);
    for (int t = threadIdx.x; t < p.QA; t += BW_BLOCK) pairVA[t] = decode_pair(t, nva);
    for (int t = threadIdx.x; t < p.PB; t += BW_BLOCK) pairOB[t] = decode_pair(t, nb);
    for (int t = threadIdx.x; t < p.QB; t += BW_BLOCK) pairVB[t] = decode_pair(t, nvb);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const u32 n2 = (u32)(n * n), np2 = (u32)(n * (n - 1) / 2);
    const u32 slab_len = max(n2, 64u * (u32)n);
    double* const slab = lds + (u32)wave * slab_len;  // zero between items
    for (u32 t = lane; t < slab_len; t += 64) slab[t] = 0.0;
    __syncthreads();
    uint8_t *occA = s_occ[wave], *virA = s_vir[wave];
    const u64 Nb = p.sp.Nb;
    auto gi = [&](int a, int b, int c, int d) { return (((u32)a * n + b) * n + c) * n + d; };
    const u64 items_a = (u64)*p.n_chunk * p.kinds, items = items_a + (u64)*p.n_chunk_b * p.kinds_b;
    for (u64 it = (u64)blockIdx.x * BW_WAVES + wave; it < items; it += (u64)gridDim.x * BW_WAVES) {
        // kinds of one chunk next to each other: they share its entries and target rows
        const bool bside = it >= items_a;
        const u64 x = bside ? it - items_a : it;
        const u32 kn = bside ? p.kinds_b : p.kinds;
        const u32 ch = (u32)(x / kn), kind = (u32)(x - (u64)ch * kn);
        const uint4 c4 = bside ? p.chunk_b[ch] : p.chunk[ch];
        const u32 rA = __builtin_amdgcn_readfirstlane(c4.x), k0 = __builtin_amdgcn_readfirstlane(c4.y);
        const int cnt = __builtin_amdgcn_readfirstlane((int)c4.z);
        const u32 A = __builtin_amdgcn_readfirstlane(c4.w);
        wave_sync();
        if (lane < n) {
            const u32 below = (1u << lane) - 1u;
            if ((A >> lane) & 1u) occA[__popc(A & below)] = (uint8_t)lane;
            else virA[lane - __popc(A & below)] = (uint8_t)lane;
        }
        wave_sync();
        if (bside) {
            u32 k = 0, ra = 0, sa = 0;
            double ck = 0.0;
            if (lane < cnt) {
                k = p.pk[k0 + lane];
                ra = p.pra[k0 + lane];
                sa = p.pA[k0 + lane];
                ck = p.v_amp[k];
            }
            const double vacc = back_neighbours(
                p, slab, lane, A, occA, virA, p.sB, p.PB * p.QB, p.QB, pairOB, pairVB, B, (int)kind, cnt, ck, sa,
                [](u32 r2) { return (u64)r2; }, ra, Nb, [](u32) { return true; });
            if (p.vbar && vacc != 0.0) unsafeAtomicAdd(p.vbar + k, vacc);
            wave_sync();
            continue;
        }
        if (kind < (u32)p.sA) {
            const int i = occA[kind / nva], a = virA[kind % nva];
            const u32 r2 = (u32)str_rank(A ^ (1u << i) ^ (1u << a), B);
            if (p.row_used[r2] && back_alpha_beta(p, slab, lane, i, a, A, r2, k0, cnt)) {
                wave_sync();
                double* Rrow = p.Rg + ((u32)i * n + a) * n2;
                for (u32 t = lane; t < n2; t += 64) {
                    const double x = slab[t];
                    if (x != 0.0) {
                        unsafeAtomicAdd(Rrow + t, x);
                        slab[t] = 0.0;
                    }
                }
                wave_sync();
            }
            continue;
        }
        u32 rk = 0, bt = 0;
        double ck = 0.0;
        if (lane < cnt) {
            rk = p.v_rb[k0 + lane];
            bt = p.v_beta[k0 + lane];
            ck = p.v_amp[k0 + lane];
        }
        double vacc = 0.0;  // this lane's entry's share of vbar
        if (kind < p.k_dir) {
            vacc = back_neighbours(p, slab, lane, A, occA, virA, p.sA, p.PA * p.QA, p.QA, pairOA, pairVA, B, (int)kind - p.sA,
                                   cnt, ck, bt, [&](u32 r2) { return (u64)r2 * Nb; }, rk, 1ull,
                                   [&](u32 r2) { return p.row_used[r2] != 0; });
        } else {
            // the diagonal, a lane per entry
            if (!p.row_used[rA]) continue;
            const double sb = lane < cnt ? p.Sd[(u64)rA * Nb + rk] : 0.0;
            if (__ballot(sb != 0.0) == 0) continue;
            const double w = sb != 0.0 ? sb * ck : 0.0;
            if (sb != 0.0) {
                vacc = diag_element(p.I, A, bt) * sb;
                for (u32 m = bt; m; m &= m - 1u) {
                    const int k = __builtin_ctz(m);
                    unsafeAtomicAdd(p.Rh + k * n + k, w);
                    for (u32 m2 = m & (m - 1u); m2; m2 &= m2 - 1u) {
                        const int l = __builtin_ctz(m2);
                        unsafeAtomicAdd(p.Rg + gi(k, k, l, l), w);
                        unsafeAtomicAdd(p.Rg + gi(k, l, l, k), -w);
                    }
                    atomicAdd(&slab[k], w);
                }
            }
            const double W = wave_sum_dpp(w);
            wave_sync();
            if (lane < n) {
                const int k = lane;
                const double o = slab[k];  // entries with k occupied in beta
                slab[k] = 0.0;
                if (o != 0.0)
                    for (u32 m = A; m; m &= m - 1u) {
                        const int l = __builtin_ctz(m);
                        unsafeAtomicAdd(p.Rg + gi(l, l, k, k), o);
                    }
                if ((A >> k) & 1u) {
                    unsafeAtomicAdd(p.Rh + k * n + k, W);
                    for (u32 m = A & ~((2u << k) - 1u); m; m &= m - 1u) {
                        const int l = __builtin_ctz(m);
                        unsafeAtomicAdd(p.Rg + gi(k, k, l, l), W);
                        unsafeAtomicAdd(p.Rg + gi(k, l, l, k), -W);
                    }
                }
            }
        }
        if (p.vbar && vacc != 0.0) unsafeAtomicAdd(p.vbar + k0 + lane, vacc);  // (lanes past cnt hold 0)
        wave_sync();
    }
}

// vbar before its partial sums (an empty v writes nothing: see bad).
__global__ void k_back_zero(double* __restrict__ vbar, const u64* __restrict__ nnz) {
    const u64 n = *nnz;
    for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (u64)gridDim.x * blockDim.x) vbar[i] = 0.0;
}

// The entries by beta string: how many each has, ...
__global__ void k_back_count(const u32* __restrict__ vrb, const u64* __restrict__ nnz, u64* __restrict__ cnt) {
    const u64 n = *nnz;
    for (u64 k = (u64)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (u64)gridDim.x * blockDim.x)
        atomicAdd((unsigned long long*)&cnt[vrb[k]], 1ull);
}

// ... their places (off: exclusive prefix, advanced to each string's end), with alpha rank and string, ...
__global__ __launch_bounds__(256) void k_back_place(SpaceDev sp, const u64* __restrict__ binom,
                                                    const u64* __restrict__ rank, const u32* __restrict__ vrb,
                                                    const u64* __restrict__ nnz, u64* __restrict__ off,
                                                    u32* __restrict__ pk, u32* __restrict__ pra,
                                                    u32* __restrict__ pA) {
    __shared__ BinomLds B;
    load_binom(B, binom);
    __syncthreads();
    const u64 n = *nnz;
    for (u64 k = (u64)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (u64)gridDim.x * blockDim.x) {
        const u64 at = atomicAdd((unsigned long long*)&off[vrb[k]], 1ull);
        const u64 ra = rank[k] / sp.Nb;
        pk[at] = (u32)k;
        pra[at] = (u32)ra;
        pA[at] = str_unrank(ra, sp.na, sp.n, B);
    }
}

// ... and their chunks.
__global__ __launch_bounds__(256) void k_back_chunks_b(SpaceDev sp, const u64* __restrict__ binom,
                                                       const u64* __restrict__ off, uint4* __restrict__ chunk,
                                                       u32* __restrict__ n_chunk) {
    __shared__ BinomLds B;
    load_binom(B, binom);
    __syncthreads();
    for (u64 r = (u64)blockIdx.x * blockDim.x + threadIdx.x; r < sp.Nb; r += (u64)gridDim.x * blockDim.x) {
        const u64 b = r ? off[r - 1] : 0, e = off[r];
        if (e <= b) continue;
        const u32 c = (u32)((e - b + 63) / 64);
        const u32 at = atomicAdd(n_chunk, c);
        const u32 S = str_unrank(r, sp.nb, sp.n, B);
        for (u32 x = 0; x < c; ++x)
            chunk[at + x] = make_uint4((u32)r, (u32)b + 64 * x, (u32)min((u64)64, e - b - 64 * x), S);
    }
}

// The input's chunks (any order) and the cotangent's rows.
__global__ __launch_bounds__(256) void k_back_chunks(SpaceDev sp, const u64* __restrict__ binom,
                                                     const u64* __restrict__ rowbeg, const u64* __restrict__ rowend,
                                                     uint4* __restrict__ chunk, u32* __restrict__ n_chunk) {
    __shared__ BinomLds B;
    load_binom(B, binom);
    __syncthreads();
    const u64 Na = sp.Na;
    for (u64 r = (u64)blockIdx.x * blockDim.x + threadIdx.x; r < Na; r += (u64)gridDim.x * blockDim.x) {
        const u64 b = rowbeg[r], e = rowend[r];
        if (e <= b) continue;
        const u32 c = (u32)((e - b + 63) / 64);
        const u32 at = atomicAdd(n_chunk, c);
        const u32 A = str_unrank(r, sp.na, sp.n, B);
        for (u32 x = 0; x < c; ++x)
            chunk[at + x] = make_uint4((u32)r, (u32)b + 64 * x, (u32)min((u64)64, e - b - 64 * x), A);
    }
}

__global__ void k_back_used(const u64* __restrict__ sr, const u64* __restrict__ n, u64 Nb, u32* __restrict__ used) {
    const u64 m = *n;
    for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (u64)gridDim.x * blockDim.x) {
        const u64 r = sr[i] / Nb;
        if (i == 0 || sr[i - 1] / Nb != r) used[r] = 1u;
    }
}

// Rows or walk.  Rows cost their (chunk, kind) items and every entry's share of
// them (less where the cotangent is in few rows); the walk costs its terms and,
// ten times as much, those that meet the cotangent.  From BD_BLOCK entries of
// each vector: how many begin a row, and how many of BD_PAIRS alpha-beta doubles
// each meet the cotangent.
constexpr int BD_BLOCK = 1024, BD_PAIRS = 4;
enum { BD_NNZ = 0, BD_NNZ_S, BD_STARTS, BD_STARTS_S, BD_HITS };
__global__ __launch_bounds__(BD_BLOCK) void k_back_ask(SpaceDev sp, const u64* __restrict__ binom,
                                                       const u64* __restrict__ rank, const u64* __restrict__ nnz,
                                                       const u64* __restrict__ s_rank, const u64* __restrict__ s_nnz,
                                                       const u32* __restrict__ T1, const double* __restrict__ Sd,
                                                       HostLine out) {
    __shared__ BinomLds B;
    __shared__ u32 s_n[3];
    if (threadIdx.x < 3) s_n[threadIdx.x] = 0;
    load_binom(B, binom);
    __syncthreads();
    const u64 nv = *nnz, ns = *s_nnz, Nb = sp.Nb;
    const u32 sA = (u32)(sp.na * (sp.n - sp.na)), sB = (u32)(sp.nb * (sp.n - sp.nb));
    u32 hits = 0;
    bool first = false, first_s = false;
    if (nv) {
        const u64 k = nv * threadIdx.x / BD_BLOCK, r = rank[k], ra = r / Nb;
        first = k == 0 || rank[k - 1] / Nb != ra;
        if (sA && sB) {
            const u32 A = str_unrank(ra, sp.na, sp.n, B), V = ~A & (sp.n == 32 ? ~0u : (1u << sp.n) - 1u);
            const u32* t = T1 + (r - ra * Nb) * sB;
            const u32 nva = (u32)(sp.n - sp.na);
#pragma unroll
            for (int u = 0; u < BD_PAIRS; ++u) {
                const u32 x = (threadIdx.x * BD_PAIRS + (u32)u) * 2654435761u;  // spread over the singles
                const u32 a = (u32)(((u64)x * sA) >> 32), b = (u32)(((u64)(u32)(x << 11 | x >> 21) * sB) >> 32);
                u32 o = A, w = V;
                for (u32 q = a / nva; q; --q) o &= o - 1u;
                for (u32 q = a % nva; q; --q) w &= w - 1u;
                const u64 r2 = str_rank(A ^ (o & (0u - o)) ^ (w & (0u - w)), B);
                if (Sd[r2 * Nb + (t[b] & 0x1FFFFFu)] != 0.0) ++hits;
            }
        }
    }
    if (ns) {
        const u64 k = ns * threadIdx.x / BD_BLOCK;
        first_s = k == 0 || s_rank[k - 1] / Nb != s_rank[k] / Nb;
    }
    const u32 f = (u32)__popcll(__ballot(first)), fs = (u32)__popcll(__ballot(first_s));
    for (int off = 32; off >= 1; off >>= 1) hits += (u32)__shfl_xor((int)hits, off);
    if (lane_id() == 0) {
        atomicAdd(&s_n[0], f);
        atomicAdd(&s_n[1], fs);
        atomicAdd(&s_n[2], hits);
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    out.p[BD_NNZ] = nv;
    out.p[BD_NNZ_S] = ns;
    out.p[BD_STARTS] = s_n[0];
    out.p[BD_STARTS_S] = s_n[1];
    out.p[BD_HITS] = s_n[2];
    out.answer();
}

// Rg += each pair slot's weight on (ia|jb), minus it on (ib|ja), i < j, a < b
// (every slot meets its own two elements).
__global__ void k_expand_pairs(int n, const double* __restrict__ R4, double* __restrict__ Rg) {
    const u32 np2 = (u32)(n * (n - 1) / 2);
    for (u32 t = blockIdx.x * blockDim.x + threadIdx.x; t < np2 * np2; t += gridDim.x * blockDim.x) {
        const double w = R4[t];
        if (w == 0.0) continue;
        const u32 po = t / np2, pv = t - po * np2;
        int j = 1, b = 1;
        while ((u32)(j * (j + 1) / 2) <= po) ++j;
        while ((u32)(b * (b + 1) / 2) <= pv) ++b;
        const int i = (int)(po - (u32)(j * (j - 1) / 2)), a = (int)(pv - (u32)(b * (b - 1) / 2));
        Rg[(((u32)i * n + a) * n + j) * n + b] += w;
        Rg[(((u32)i * n + b) * n + j) * n + a] -= w;
    }
}

}  // namespace

// From a few thousand entries on the entries decide (back_rows_answer); below,
// the walk per source is a few launches less.  us, source walk and rows, v and
// sbar entries: 8 orbitals, 100 and 100 114 and 164, 1 000 and 1 000 143 and 192;
// 16 orbitals, 1 000 and 20 000 240 and 255, 3 000 and 3 000 249 and 257, 3 000 and
// 100 000 485 and 292, 10 000 and 10 000 548 and 386.  SFCI_BACK_ROWS=0|1 forces
// one form.
bool back_rows_available(sfci_problem* P, u64 nnz, u64 nnz_s) {
    bool pays = nnz >= 4096 || (nnz >= 1024 && nnz_s >= 65536);
    if (const char* env = getenv("SFCI_BACK_ROWS")) pays = env[0] != '0';
    return pays && nnz < (1ull << 31) && P->Na < (1ull << 31) && rowtile_available(P);
}

bool ask_back_rows(sfci_problem* P, const SigmaLaunch& v, const double* D, const u64* s_rank, const u64* s_nnz,
                   HostLine* l) {
    if (getenv("SFCI_BACK_ROWS")) return true;  // (=0 does not come here)
    *l = host_line(P);
    hipLaunchKernelGGL(k_back_ask, dim3(1), dim3(BD_BLOCK), 0, P->stream, SpaceDev{P->n, P->na, P->nb, P->Na, P->Nb},
                       P->d_binom, v.v_rank, v.v_nnz, s_rank, s_nnz, rowtile_T1(P), D, *l);
    SFCI_CHECK_HIP(hipGetLastError());
    return false;
}

// Both forms' times, ms, fitted to 512 calls in 19 spaces (within a third nine
// times in ten).  By sizes alone 116 of them took longer by rows than the walk
// did, up to 2.5 times (entries spread out, few to a row): ms, rows and walk, 18
// orbitals, 9 + 1 electrons, 2e4 and 2e4 entries spread out 1.98 and 0.75, near
// the aufbau string 0.90 and 1.53; 16, 6 + 2, 5e3 and 5e3 spread out 0.38 and 0.22.
// Asking costs 15 us.
bool back_rows_answer(sfci_problem* P, const HostLine& l) {
    const u64* h = wait_line(P, l);
    const int n = P->n, na = P->na, nb = P->nb;
    const double sA = na * (n - na), sB = nb * (n - nb);
    const double dA = (na * (na - 1) / 2) * ((n - na) * (n - na - 1) / 2), dB = (nb * (nb - 1) / 2) * ((n - nb) * (n - nb - 1) / 2);
    const double kA = sA + ceil((sA + dA) / 64) + 1, kB = ceil((sB + dB) / 64);
    const double nv = (double)h[BD_NNZ], ns = (double)h[BD_NNZ_S], Na = (double)P->Na, Nb = (double)P->Nb;
    const double terms = nv * (double)terms_per_source(n, na, nb);
    const double met = terms * ((double)h[BD_HITS] / (BD_BLOCK * BD_PAIRS));
    // chunks by alpha row, by beta string (as of a spread-out vector), rows of the cotangent
    const double ca = nv * ((double)h[BD_STARTS] / BD_BLOCK) + nv / 64;
    const double cb = Nb * (1.0 - exp(-nv / Nb)) + nv / 64;
    const double used = std::min(1.0, ns * ((double)h[BD_STARTS_S] / BD_BLOCK) / Na);
    const double walk = 0.129 + nv * (2.5e-9 * sA * sB + 4.05e-9 * (dA + dB) + 9.1e-7 * (na + nb)) + 4.6e-8 * met;
    const double rows = 0.179 + 3.1e-6 * Na + 7.6e-8 * ns + (3.2e-7 + 5.3e-7 * used) * ca * kA + 7.4e-7 * cb * kB +
                        nv * ((4.1e-8 + 1.08e-7 * used) * kA + 2.3e-7 * kB) + 5.8e-9 * met;
    return rows < 0.97 * walk;
}

// sbar must already be scattered into the (otherwise zero) dense array D.
void launch_back_rows(sfci_problem* P, const SigmaLaunch& v, const RowTileDesc& d, const double* D, const u64* s_rank,
                      const u64* s_nnz, u64 s_cap, double* vbar, double* dh, double* dg, double* Rh, double* Rg,
                      const int* bad) {
    const int n = P->n, na = P->na, nb = P->nb;
    const u64 n2 = (u64)n * n, n4 = n2 * n2, np2 = (u64)n * (n - 1) / 2;
    hipStream_t st = P->stream;
    const RowView rv = rowtile_view(d);
    // [chunks by row | by beta string | permuted entries | zeroed: entries per beta string, pair slots,
    //  the chunks' numbers, rows of sbar]
    const u64 max_a = v.cap / 64 + std::min<u64>(P->Na, v.cap) + 1, max_b = v.cap / 64 + std::min<u64>(P->Nb, v.cap) + 1;
    const u64 perm = (3 * v.cap + 1) / 2, zero_words = P->Nb + np2 * np2 + (P->Na + 2) / 2 + 1;
    u64* ws = (u64*)P->ws_prod.get((2 * (max_a + max_b) + perm + zero_words) * sizeof(u64));
    (void)P->ws_scan.get((P->Nb / 2048 + 1) * sizeof(u64));  // the scan's, before anything is written
    uint4* chunk = (uint4*)ws;
    uint4* chunk_b = chunk + max_a;
    u32* pk = (u32*)(chunk_b + max_b);
    u64* cnt = ws + 2 * (max_a + max_b) + perm;
    double* R4 = (double*)(cnt + P->Nb);
    u32* n_chunk = (u32*)(R4 + np2 * np2);
    u32* used = n_chunk + 2;
    launch_fill_u64(cnt, zero_words, 0, st);
    launch_fill_f64(Rh, n2 + n4, 0.0, st);  // Rh and Rg are adjacent
    if (vbar)
        hipLaunchKernelGGL(k_back_zero, dim3((unsigned)std::max<u64>(1, std::min<u64>((v.cap + 255) / 256, 16384))),
                           dim3(256), 0, st, vbar, v.v_nnz);
    const unsigned gr = (unsigned)std::min<u64>((P->Na + 255) / 256, 16384);
    hipLaunchKernelGGL(k_back_chunks, dim3(gr), dim3(256), 0, st, SpaceDev{n, na, nb, P->Na, P->Nb}, P->d_binom,
                       rv.rowbeg, rv.rowend, chunk, n_chunk);
    const SpaceDev sp{n, na, nb, P->Na, P->Nb};
    const unsigned gv = (unsigned)std::max<u64>(1, std::min<u64>((v.cap + 255) / 256, 16384));
    hipLaunchKernelGGL(k_back_count, dim3(gv), dim3(256), 0, st, rv.v_rb, v.v_nnz, cnt);
    exclusive_scan_u64(P, cnt, cnt, P->Nb, nullptr);
    hipLaunchKernelGGL(k_back_place, dim3(gv), dim3(256), 0, st, sp, P->d_binom, v.v_rank, rv.v_rb, v.v_nnz, cnt, pk,
                       pk + v.cap, pk + 2 * v.cap);
    hipLaunchKernelGGL(k_back_chunks_b, dim3((unsigned)std::min<u64>((P->Nb + 255) / 256, 16384)), dim3(256), 0, st, sp,
                       P->d_binom, (const u64*)cnt, chunk_b, n_chunk + 1);
    hipLaunchKernelGGL(k_back_used, dim3((unsigned)std::max<u64>(1, std::min<u64>((s_cap + 255) / 256, 16384))),
                       dim3(256), 0, st, s_rank, s_nnz, P->Nb, used);
    BackRows p{};
    p.sp = SpaceDev{n, na, nb, P->Na, P->Nb};
    p.I = Ints{P->d_h, P->d_g, n};
    p.binom = P->d_binom;
    p.v_amp = v.v_amp;
    p.v_beta = rv.v_beta;
    p.v_rb = rv.v_rb;
    p.chunk = chunk;
    p.n_chunk = n_chunk;
    p.chunk_b = chunk_b;
    p.n_chunk_b = n_chunk + 1;
    p.pk = pk;
    p.pra = pk + v.cap;
    p.pA = pk + 2 * v.cap;
    p.T1 = rv.T1;
    p.K4 = rv.K4;
    p.Sd = D;
    p.row_used = used;
    p.vbar = vbar;
    p.Rh = Rh;
    p.Rg = Rg;
    p.R4 = R4;
    p.sA = na * (n - na);
    p.sB = nb * (n - nb);
    p.PA = na * (na - 1) / 2;
    p.QA = (n - na) * (n - na - 1) / 2;
    p.PB = nb * (nb - 1) / 2;
    p.QB = (n - nb) * (n - nb - 1) / 2;
    p.k_dir = (u32)(p.sA + (p.sA + p.PA * p.QA + 63) / 64);
    p.kinds = p.k_dir + 1;
    p.kinds_b = (u32)((p.sB + p.PB * p.QB + 63) / 64);
    const size_t lds = (size_t)BW_WAVES * std::max<u64>(n2, 64ull * n) * sizeof(double);
    const u64 items = max_a * p.kinds + max_b * p.kinds_b;
    const unsigned grid = (unsigned)std::max<u64>(1, std::min<u64>((items + BW_WAVES - 1) / BW_WAVES, (u64)P->num_cu * 16));
    // the most any problem asks for: the limit is the function's, not the problem's
    SFCI_CHECK_HIP(hipFuncSetAttribute((const void*)k_back_rows, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)(BW_WAVES * 64 * 32 * sizeof(double))));
    hipLaunchKernelGGL(k_back_rows, dim3(grid), dim3(BW_BLOCK), lds, st, p);
    if (np2 > 0)
        hipLaunchKernelGGL(k_expand_pairs, dim3((unsigned)std::min<u64>((np2 * np2 + 255) / 256, 4096)), dim3(256), 0,
                           st, n, (const double*)R4, Rg);
    launch_symmetrise(P, Rh, Rg, dh, dg, bad);
    SFCI_CHECK_HIP(hipGetLastError());
}
