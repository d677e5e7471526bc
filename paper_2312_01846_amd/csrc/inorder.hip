// Deterministic sigma = H v where a target row fits in LDS: every target adds
// its contributions in ascending source rank (Sec. 2.2's merge order), without
// a sort.
//
// A wavefront owns a target alpha row A' (its N_beta accumulators in LDS) and
// takes the source rows that reach it in ascending rank, each row's entries in
// ascending order.  The targets of one entry are distinct, and so are those of
// the entries of an alpha-double row, so one LDS add instruction never holds
// two terms of a target; a wavefront's LDS instructions complete in the order
// they are issued.  Every sum therefore rounds as the sequential loop's.
//
// Per row: the neighbours of A' with entries are marked in a bitmap over the
// alpha ranks (their rows' occupancy is a bitmap too), which lists them in
// order; 64 listed rows at a time have their bounds, orbitals and elements
// formed a lane each; alpha-double rows add up to 64 entries at once,
// alpha-single rows and the identity row walk their entries over the beta
// tables (T1x: 64-aligned groups, one load per group).  Rows with an all-zero
// (ia|..) slab skip their alpha-beta doubles, and without any nonzero pair
// element (Hubbard models) the same-spin doubles are skipped.
//
// Bound by: LDS adds (random slots, 29 clocks of a compute unit per
// instruction) and, with few resident wavefronts, load latency.  The sort path
// (emission, radix sort, run sums) moves ~60 B per tuple through HBM: 100 000
// entries of a 20-orbital, 4 + 4-electron space 3.85 ms against 19.8, 10 000
// 2.0 against 7.3; a Hubbard ring's iteration (12 sites, M = 100 000) 0.25 ms
// per sigma against 4.6.  What remains is the longest row: one wavefront issues
// an instruction in ~8 clocks, 230 clocks per alpha-single entry (20 011
// entries near the aufbau string of 19 orbitals: 1.2 of the call's 1.5 ms).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "sfci_internal.h"

namespace {

constexpr int IO_MAXW = 8;    // wavefronts per workgroup
constexpr int IO_R = 4;       // alpha-double rows per set of registers
constexpr u32 IO_SLAB = 16;   // groups of beta singles from which a row's (ia|..) is copied to LDS
constexpr int IO_S = 2;       // entries of the identity row whose beta singles are formed together
constexpr int IO_B = 6;       // groups of 64 beta-beta doubles per set of registers
constexpr u64 IO_MAX_ROWS = 65536;   // alpha ranks of the bitmaps
constexpr u64 IO_MAX_NB = 17000;     // slots of a row

struct InOrder {
    SpaceDev sp;
    Ints I;
    const u64* binom;
    const double* v_amp;
    const u32* v_beta;
    const u32* v_rb;
    const u64 *rowbeg, *rowend;
    const u32* astr;  // alpha strings by rank
    const u32* T1x;   // beta singles per beta rank in groups of 64: target | (j n + b) << 16 | phase << 31
    const u32* T1;    // beta singles per beta rank (rank | (j n + b) << 21 | phase << 31), TS their beta part
    const double* TS;
    const u32* T2r;   // beta-beta doubles per beta rank: target, signed element
    const double* T2e;
    const double *K2, *K4;
    const unsigned char* gnz;  // per i n + a: bit 0 some (ia|jb), j != b, nonzero, bit 1 some (ia|jj); [n n]: some K4
    double* D;
    unsigned long long* emitted;
    double eps, eps_x;
    unsigned* counter;
    int sA, sB, PA, QA, dB;
    u32 t1_shift, t1_last;  // log2 of T1x's groups per rank, the last with entries ...
    u64 t1_mask;            // ... and its lanes
    u32 words;              // of a bitmap over the alpha ranks
    u32 off_rows, per_wave; // doubles before the wavefronts' areas, and in each
};

struct Wave {
    double* acc;
    u32* bits;
    uint16_t* list;
    double* slab;  // the (ia|..) of an alpha single, n^2, and 64 elements
    uint8_t *occ, *vir;
    int lane;
};

// The term t of element e as it is added: 0 where it is not emitted (a sum
// that starts at +0 and rounds to nearest is never -0, so +-0 leaves it), and
// the emitted ones of the wavefront counted.
template <bool XS>
__device__ __forceinline__ double io_term(double e, double t, bool dbl, double eps_x, u32& terms) {
    bool keep = e != 0.0;
    if (XS && dbl) keep = keep && !xscreened(t, eps_x) && t != 0.0;
    terms += (u32)__popcll(__ballot(keep));
    return keep ? t : 0.0;
}

// A run of alpha-double rows (the lanes set in rows, of the 64 listed): up to
// 64 entries of a row at a time, IO_R rows in flight in each of two sets.
template <bool XS>
__device__ __forceinline__ void io_doubles(const InOrder& p, const Wave& w, u64 rows, u32 beg, u32 len, double e,
                                           u32& terms) {
    const int lane = w.lane;
    u64 ahead = rows;  // not yet loaded
    u32 rA[IO_R], rB[IO_R];
    double cA[IO_R], cB[IO_R];
    const auto fetch = [&](u32(&r)[IO_R], double(&c)[IO_R]) {
#pragma unroll
        for (int u = 0; u < IO_R; ++u) {
            if (!ahead) break;
            const int j = __builtin_ctzll(ahead);
            ahead &= ahead - 1;
            const u32 k = (u32)__builtin_amdgcn_readlane((int)beg, j) +
                          min((u32)lane, (u32)__builtin_amdgcn_readlane((int)len, j) - 1u);
            r[u] = p.v_rb[k];
            c[u] = p.v_amp[k];
        }
    };
    const auto add = [&](const u32(&r)[IO_R], const double(&c)[IO_R]) {
#pragma unroll
        for (int u = 0; u < IO_R; ++u) {
            if (!rows) break;
            const int j = __builtin_ctzll(rows);
            rows &= rows - 1;
            const u32 l = (u32)__builtin_amdgcn_readlane((int)len, j);
            const double x = lane_f64(e, j);
            const double t = io_term<XS>((u32)lane < l ? x : 0.0, x * c[u], true, p.eps_x, terms);
            if ((u32)lane < l) atomicAdd(&w.acc[r[u]], t);
            if (l > 64) {
                const u32 b = (u32)__builtin_amdgcn_readlane((int)beg, j);
                for (u32 q = 64 + lane; q < l; q += 64)
                    atomicAdd(&w.acc[p.v_rb[b + q]], io_term<XS>(x, x * p.v_amp[b + q], true, p.eps_x, terms));
            }
        }
    };
    fetch(rA, cA);
    while (rows) {
        fetch(rB, cB);
        add(rA, cA);
        fetch(rA, cA);
        add(rB, cB);
    }
}

// An alpha-single row i -> a: per entry the alpha-beta doubles and the target
// with beta unchanged (on the lane behind the last beta single where the last
// group of 64 has one, else an add of its own).  The beta singles of U groups
// are loaded while the U before are added (two sets of registers in turn: a
// copy from one to the other would wait for the loads), and the products carry
// no test, +-0 being left out of no sum, unless an amplitude is not finite.
template <bool XS, bool SLAB, bool OWN, int U>
__device__ __forceinline__ void io_single(const InOrder& p, const Wave& w, u32 beg, u32 end, int i, int a, int par,
                                          double cst, bool ab, u32& terms) {
    const int lane = w.lane, n = p.sp.n;
    const u32 sB = (u32)p.sB, n2 = (u32)(n * n);
    const double* Gia = p.I.g + ((u32)i * n + a) * n2;
    wave_sync();
    if (SLAB) {
        for (u32 t = lane; t < n2; t += 64) w.slab[t] = Gia[t];
    } else if (lane < n) {
        w.slab[lane * (n + 1)] = Gia[lane * (n + 1)];
    }
    double* const elq = w.slab + n2;  // the unsigned direct elements of 64 entries
    const bool last = OWN && (u32)lane == sB;  // OWN: fewer than 64 beta singles
    const u32 shift = OWN ? 0u : p.t1_shift, gm = (1u << shift) - 1u;
    const u64 mask = p.t1_mask;
    const u32 xlast = last ? n2 : 0u;
    for (u32 kb = beg; kb < end; kb += 64) {
        const int cnt = (int)min(64u, end - kb);
        const u32 k = kb + (u32)min(lane, cnt - 1);
        const u32 rk = p.v_rb[k];
        const double ck = p.v_amp[k];
        const u32 bt = p.v_beta[k];
        const u32 off = rk << (shift + 8);
        const int items = cnt << shift;
        u32 tA[U], tB[U];
        const auto fetch = [&](int s0, u32(&t1)[U]) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int s = min(s0 + u, items - 1);
                const u32 o = (u32)__builtin_amdgcn_readlane((int)off, s >> shift) + ((u32)s & gm) * 256u;
                t1[u] = *(const u32*)((const char*)p.T1x + (o + (u32)lane * 4u));
            }
        };
        if (ab) fetch(0, tA);
        wave_sync();
        double el = cst;
        for (u32 m = bt; m; m &= m - 1u) el += w.slab[__builtin_ctz(m) * (n + 1)];
        const double el0 = el;
        el = lane < cnt ? (par ? -el : el) : 0.0;
        const double t0 = io_term<XS>(el, el * ck, false, p.eps_x, terms);
        if (!ab) {
            if (el != 0.0) atomicAdd(&w.acc[rk], t0);
            continue;
        }
        const double cs = par ? -ck : ck;
        const bool direct = !OWN && el != 0.0;
        if (__ballot(fabs(ck) < INFINITY) == ~u64(0)) {
            if (SLAB && OWN) {
                wave_sync();
                elq[lane] = el0;
                wave_sync();
            }
            const auto add = [&](int s0, const u32(&t1)[U], bool full) {
                double x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const u32 jb = (t1[u] >> 16) & 1023u;
                    if (SLAB) {
                        x[u] = w.slab[OWN ? (last ? xlast + (u32)(full ? s0 + u : min(s0 + u, items - 1)) : jb) : jb];
                    } else {
                        x[u] = Gia[jb];
                        if (OWN) {
                            const double e1 = lane_f64(el0, full ? s0 + u : min(s0 + u, items - 1));
                            x[u] = last ? e1 : x[u];
                        }
                    }
                }
                double c[U];
#pragma unroll
                for (int u = 0; u < U; ++u) c[u] = lane_f64(cs, (full ? s0 + u : min(s0 + u, items - 1)) >> shift);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int s = s0 + u;
                    if (!full && s >= items) break;
                    const double pr = x[u] * c[u];
                    double y = __hiloint2double(__double2hiint(pr) ^ (int)(t1[u] & 0x80000000u), __double2loint(pr));
                    bool keep = x[u] != 0.0;
                    if (XS) {
                        keep = keep && !xscreened(y, p.eps_x) && y != 0.0;
                        if (!keep && !last) y = 0.0;
                    }
                    const u32 g = (u32)s & gm;
                    const u64 real = OWN ? mask : g < p.t1_last ? ~u64(0) : g == p.t1_last ? mask : 0;
                    terms += (u32)__popcll(__ballot(keep) & real);
                    atomicAdd(&w.acc[t1[u] & 0xFFFFu], y);
                    if (!OWN && g == 0 && lane == (s >> shift) && direct) atomicAdd(&w.acc[rk], t0);
                }
            };
            for (int s0 = 0; s0 < items; s0 += 2 * U) {
                fetch(s0 + U, tB);
                if (s0 + U <= items) add(s0, tA, true);
                else add(s0, tA, false);
                if (s0 + U >= items) break;
                fetch(s0 + 2 * U, tA);
                if (s0 + 2 * U <= items) add(s0 + U, tB, true);
                else add(s0 + U, tB, false);
            }
        } else {
            for (int q = 0; q < cnt; ++q) {
                const u64 tb = (u64)(u32)__builtin_amdgcn_readlane((int)rk, q) * sB;
                const double c = lane_f64(cs, q);
                for (u32 s = lane; s < sB; s += 64) {
                    const u32 t1 = p.T1[tb + s];
                    const double x1 = Gia[(t1 >> 21) & 1023u];
                    const double pr = x1 * c;
                    const double y =
                        __hiloint2double(__double2hiint(pr) ^ (int)(t1 & 0x80000000u), __double2loint(pr));
                    atomicAdd(&w.acc[t1 & 0x1FFFFFu], io_term<XS>(x1, y, true, p.eps_x, terms));
                }
                if (lane == q) atomicAdd(&w.acc[rk], t0);
            }
        }
    }
}

// The identity row: diagonal, beta singles, beta-beta doubles of every entry.
// In flight: the next IO_B groups of doubles, the beta singles of the next IO_S
// entries and, once those are there, their (jb|kk) of four k.
template <bool XS>
__device__ __forceinline__ void io_identity(const InOrder& p, const Wave& w, u32 beg, u32 end, u32 A, u32 dB,
                                            const double* K2, const double* J, const double* hd, u32& terms) {
    const int lane = w.lane, n = p.sp.n;
    const u32 sB = (u32)p.sB;
    const u32 ng = (dB + 63) / 64;  // groups of doubles per entry
    const bool act = (u32)lane < sB;
    const u32 sl = min((u32)lane, sB ? sB - 1 : 0u);
    const u32 n2 = (u32)(n * n);
    u32 goff[4];  // of the row's first four orbitals: (k, k)
    {
        u32 m = A;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            goff[v] = m ? (u32)__builtin_ctz(m) * (u32)(n + 1) : 0u;
            m &= m - 1u;
        }
    }
    const int nk = min(4, __popc(A));
    double ea = 0.0;
    for (u32 m = A; m; m &= m - 1u) ea += hd[__builtin_ctz(m)];
    for (u32 kb = beg; kb < end; kb += 64) {
        const int cnt = (int)min(64u, end - kb);
        const u32 k = kb + (u32)min(lane, cnt - 1);
        const u32 rk = p.v_rb[k];
        const double ck = p.v_amp[k];
        const u32 bt = p.v_beta[k];
        u32 rA[IO_B], rB[IO_B];
        double eA[IO_B], eB[IO_B];
        int fq = 0;     // what is fetched next: entry and first group
        u32 fg = 0;
        const auto fetch2 = [&](u32(&r)[IO_B], double(&e)[IO_B]) {
            const u64 base = (u64)(u32)__builtin_amdgcn_readlane((int)rk, min(fq, cnt - 1)) * dB;
            const u32* R = p.T2r + base;
            const double* E = p.T2e + base;
#pragma unroll
            for (int v = 0; v < IO_B; ++v) {
                const u32 t = min((fg + (u32)v) * 64 + (u32)lane, dB - 1);
                r[v] = R[t];
                e[v] = E[t];
            }
            fg += IO_B;
            if (fg >= ng) fg = 0, ++fq;
        };
        u32 sA[IO_S], sC[IO_S];
        double xA[IO_S], xC[IO_S], gk[4][IO_S];
        const auto fetch1 = [&](int q0, u32(&t1)[IO_S], double(&x)[IO_S]) {
            if (!sB) return;
#pragma unroll
            for (int u = 0; u < IO_S; ++u) {
                const u32 at = (u32)__builtin_amdgcn_readlane((int)rk, min(q0 + u, cnt - 1)) * sB + sl;
                t1[u] = p.T1[at];
                x[u] = p.TS[at];
            }
        };
        const auto fetchk = [&](const u32(&t1)[IO_S]) {
            if (!sB) return;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (v < nk)
#pragma unroll
                    for (int u = 0; u < IO_S; ++u) gk[v][u] = p.I.g[((t1[u] >> 21) & 1023u) * n2 + goff[v]];
        };
        fetch1(0, sA, xA);
        if (ng) fetch2(rA, eA);
        bool even = true;  // the doubles' next set is A
        double el = ea;
        for (u32 m = bt; m; m &= m - 1u) el += hd[__builtin_ctz(m)];
        for (int s = 0; s < 2; ++s)
            for (u32 m = s ? bt : A; m; m &= m - 1u) {
                const double* Kp = K2 + __builtin_ctz(m) * n;
                for (u32 m2 = m & (m - 1u); m2; m2 &= m2 - 1u) el += Kp[__builtin_ctz(m2)];
            }
        for (u32 m = A; m; m &= m - 1u) {
            const double* Jp = J + __builtin_ctz(m) * n;
            for (u32 m2 = bt; m2; m2 &= m2 - 1u) el += Jp[__builtin_ctz(m2)];
        }
        if (lane >= cnt) el = 0.0;
        const double t0 = io_term<XS>(el, el * ck, false, p.eps_x, terms);
        fetchk(sA);
        const auto add2 = [&](double c, u32 g0, const u32(&r)[IO_B], const double(&e)[IO_B]) {
#pragma unroll
            for (int v = 0; v < IO_B; ++v) {
                if (g0 + (u32)v >= ng) break;
                const bool in = (g0 + (u32)v) * 64 + (u32)lane < dB;
                const double ev = in ? e[v] : 0.0;
                const u32 to = in ? r[v] : (u32)p.sp.Nb + (u32)lane;  // else a slot that nothing reads
                atomicAdd(&w.acc[to], io_term<XS>(ev, ev * c, true, p.eps_x, terms));
            }
        };
        const auto entry = [&](int q, u32 t1, double xs) {
            const double c = lane_f64(ck, q);
            if (lane == q) atomicAdd(&w.acc[rk], t0);
            if (act) {
                const double x = (t1 >> 31) ? -xs : xs;
                atomicAdd(&w.acc[t1 & 0x1FFFFFu], io_term<XS>(x, x * c, false, p.eps_x, terms));
            }
            if (sB > 64) {
                const u32 tb = (u32)__builtin_amdgcn_readlane((int)rk, q) * sB;
                for (u32 s = lane + 64; s < sB; s += 64) {
                    const u32 tx = p.T1[tb + s];
                    const u32 jb = (tx >> 21) & 1023u;
                    double x = p.TS[tb + s];
                    for (u32 m = A; m; m &= m - 1u) x += p.I.g[jb * n2 + __builtin_ctz(m) * (u32)(n + 1)];
                    if (tx >> 31) x = -x;
                    atomicAdd(&w.acc[tx & 0x1FFFFFu], io_term<XS>(x, x * c, false, p.eps_x, terms));
                }
            }
            for (u32 g0 = 0; g0 < ng; g0 += IO_B) {
                if (even) {
                    fetch2(rB, eB);
                    add2(c, g0, rA, eA);
                } else {
                    fetch2(rA, eA);
                    add2(c, g0, rB, eB);
                }
                even = !even;
            }
        };
        const auto group = [&](int q0, u32(&t1)[IO_S], double(&x)[IO_S], u32(&tn)[IO_S], double(&xn)[IO_S]) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (v < nk)
#pragma unroll
                    for (int u = 0; u < IO_S; ++u) x[u] += gk[v][u];
            if (__popc(A) > 4) {
                u32 m = A;
                for (int v = 0; v < 4; ++v) m &= m - 1u;
                for (; m; m &= m - 1u)
#pragma unroll
                    for (int u = 0; u < IO_S; ++u)
                        x[u] += p.I.g[((t1[u] >> 21) & 1023u) * n2 + __builtin_ctz(m) * (u32)(n + 1)];
            }
            fetch1(q0 + IO_S, tn, xn);
#pragma unroll
            for (int u = 0; u < IO_S; ++u) {
                if (u == IO_S / 2) fetchk(tn);
                if (q0 + u < cnt) entry(q0 + u, t1[u], x[u]);
            }
        };
        for (int q0 = 0; q0 < cnt; q0 += 2 * IO_S) {
            group(q0, sA, xA, sC, xC);
            group(q0 + IO_S, sC, xC, sA, xA);
        }
    }
}

template <bool XS>
__global__ __launch_bounds__(64 * IO_MAXW) void k_row_inorder(InOrder p) {
    extern __shared__ double lds[];
    __shared__ BinomLds B;
    __shared__ uint16_t pairO[SFCI_MAX_PAIRS], pairV[SFCI_MAX_PAIRS];
    __shared__ uint8_t s_occ[IO_MAXW][32], s_vir[IO_MAXW][32];
    __shared__ double hd[32];
    load_binom(B, p.binom);
    const int n = p.sp.n, na = p.sp.na, nva = n - na, n2 = n * n;
    double* const K2 = lds;
    double* const J = lds + n2;
    u32* const used = (u32*)(lds + 2 * n2);  // alpha rows with entries
    for (int t = threadIdx.x; t < p.PA; t += blockDim.x) pairO[t] = decode_pair(t, na);
    for (int t = threadIdx.x; t < p.QA; t += blockDim.x) pairV[t] = decode_pair(t, nva);
    for (int t = threadIdx.x; t < n2; t += blockDim.x) {
        const int x = t / n, y = t - x * n;
        K2[t] = p.K2[t];
        J[t] = p.I.G(x, x, y, y);
    }
    if (threadIdx.x < (unsigned)n) hd[threadIdx.x] = p.I.H(threadIdx.x, threadIdx.x);
    for (u32 t = threadIdx.x; t < p.words; t += blockDim.x) {
        u32 m = 0;
        for (u32 b = 0; b < 32; ++b) {
            const u64 r = (u64)t * 32 + b;
            if (r < p.sp.Na && p.rowend[r] > p.rowbeg[r]) m |= 1u << b;
        }
        used[t] = m;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    Wave w;
    w.acc = lds + p.off_rows + (u32)wave * p.per_wave;
    w.slab = w.acc + p.sp.Nb + 64;
    w.bits = (u32*)(w.slab + n2 + 64);
    w.list = (uint16_t*)(w.bits + p.words);
    w.occ = s_occ[wave];
    w.vir = s_vir[wave];
    w.lane = lane;
    const u32 np2 = (u32)(n * (n - 1) / 2);
    const bool doubles = p.gnz[n2] != 0;  // else no same-spin double has an element
    const int K = 1 + p.sA + (doubles ? p.PA * p.QA : 0);
    const u32 dB = doubles ? (u32)p.dB : 0u;
    const u32 Nb = (u32)p.sp.Nb;
    u64 emitted = 0;
    // the heaviest rows tend to be the first: one to a workgroup, then whichever is next
    const unsigned nw = blockDim.x >> 6;
    for (unsigned r = (unsigned)wave * gridDim.x + blockIdx.x; (u64)r < p.sp.Na;) {
        const u32 At = __builtin_amdgcn_readfirstlane(p.astr[r]);
        wave_sync();
        if (lane < n) {
            const u32 below = (1u << lane) - 1u;
            if ((At >> lane) & 1u) w.occ[__popc(At & below)] = (uint8_t)lane;
            else w.vir[lane - __popc(At & below)] = (uint8_t)lane;
        }
        for (u32 x = lane; x < Nb; x += 64) w.acc[x] = 0.0;
        for (u32 x = lane; x < p.words; x += 64) w.bits[x] = 0u;
        wave_sync();
        u32 terms = 0;
        // the rows that reach A', as bits
        for (int t0 = 0; t0 < K; t0 += 64) {
            const int t = t0 + lane;
            if (t >= K) continue;
            u32 As = At;
            if (t > p.sA) {
                const int x = t - 1 - p.sA;
                const u32 po = pairO[x / p.QA], pv = pairV[x % p.QA];
                As ^= (1u << w.occ[po & 255]) ^ (1u << w.occ[po >> 8]) ^ (1u << w.vir[pv & 255]) ^ (1u << w.vir[pv >> 8]);
            } else if (t > 0) {
                As ^= (1u << w.occ[(t - 1) / nva]) ^ (1u << w.vir[(t - 1) % nva]);
            }
            const u32 rs = (u32)str_rank(As, B);
            if ((used[rs >> 5] >> (rs & 31)) & 1u) atomicOr(&w.bits[rs >> 5], 1u << (rs & 31));
        }
        wave_sync();
        // ... in ascending order
        u32 cntl = 0;
        for (u32 x0 = 0; x0 < p.words; x0 += 64) {
            u32 m = (x0 + lane < p.words) ? w.bits[x0 + lane] : 0u;
            if (__ballot(m != 0u) == 0) continue;
            const u32 c = (u32)__popc(m);
            u32 inc = c;
            for (int off = 1; off < 64; off <<= 1) {
                const u32 y = (u32)__shfl_up((int)inc, off);
                if (lane >= off) inc += y;
            }
            u32 at = cntl + inc - c;
            for (; m; m &= m - 1u) w.list[at++] = (uint16_t)((x0 + lane) * 32 + (u32)__builtin_ctz(m));
            cntl += (u32)__builtin_amdgcn_readlane((int)inc, 63);
        }
        wave_sync();
        for (u32 l0 = 0; l0 < cntl; l0 += 64) {
            const int cnt = (int)min(64u, cntl - l0);
            u32 beg = 0, end = 0, info = 0;
            int type = 3;
            double e = 0.0;
            bool ab = false;
            if (lane < cnt) {
                const u32 rs = w.list[l0 + lane];
                const u32 As = p.astr[rs];
                beg = (u32)p.rowbeg[rs];
                end = (u32)p.rowend[rs];
                const u32 d1 = As & ~At, d2 = At & ~As;
                const int x = __popc(d1);
                type = x;  // 0 the row itself, 1 an alpha single, 2 an alpha double
                if (x == 1) {
                    const int i = __builtin_ctz(d1), a = __builtin_ctz(d2);
                    e = p.I.H(i, a);
                    for (u32 m = As & ~(1u << i); m; m &= m - 1u) {
                        const int k = __builtin_ctz(m);
                        e += (p.I.G(i, a, k, k) - p.I.G(i, k, k, a));
                    }
                    info = (u32)i | (u32)a << 8 | (u32)between_parity(As, i, a) << 16;
                    const unsigned char f = p.gnz[i * n + a];
                    ab = (f & 1) != 0 && p.sB > 0;
                    if (f == 0 && e == 0.0) end = beg;  // adds nothing
                } else if (x == 2) {
                    const int i = __builtin_ctz(d1), j = __builtin_ctz(d1 & (d1 - 1u));
                    const int a = __builtin_ctz(d2), b = __builtin_ctz(d2 & (d2 - 1u));
                    const u32 mid = As ^ (1u << i) ^ (1u << a);
                    e = p.K4[(u32)(j * (j - 1) / 2 + i) * np2 + (u32)(b * (b - 1) / 2 + a)];
                    if (between_parity(As, i, a) ^ between_parity(mid, j, b)) e = -e;
                    if (e == 0.0) end = beg;  // adds nothing
                }
            }
            const u32 len = end - beg;
            u64 todo = __ballot(lane < cnt && len != 0);
            const u64 others = todo & __ballot(type < 2);
            while (todo) {
                const int pos = __builtin_ctzll(todo);
                if (!((others >> pos) & 1)) {
                    const u64 stop = others & todo;
                    const u64 run = stop ? todo & ((stop & -stop) - 1) : todo;
                    io_doubles<XS>(p, w, run, beg, len, e, terms);
                    todo &= ~run;
                    continue;
                }
                todo &= todo - 1;
                const u32 b0 = (u32)__builtin_amdgcn_readlane((int)beg, pos);
                const u32 b1 = (u32)__builtin_amdgcn_readlane((int)end, pos);
                if (__builtin_amdgcn_readlane(type, pos) == 1) {
                    const u32 f = (u32)__builtin_amdgcn_readlane((int)info, pos);
                    const int i = (int)(f & 255u), a = (int)((f >> 8) & 255u), par = (int)(f >> 16);
                    const bool x = __builtin_amdgcn_readlane((int)ab, pos) != 0;
                    const double c = lane_f64(e, pos);
                    const bool slab = x && (b1 - b0) << p.t1_shift >= IO_SLAB;
                    if (p.sB < 64) {
                        if (slab) io_single<XS, true, true, 8>(p, w, b0, b1, i, a, par, c, x, terms);
                        else io_single<XS, false, true, 4>(p, w, b0, b1, i, a, par, c, x, terms);
                    } else {
                        if (slab) io_single<XS, true, false, 8>(p, w, b0, b1, i, a, par, c, x, terms);
                        else io_single<XS, false, false, 4>(p, w, b0, b1, i, a, par, c, x, terms);
                    }
                } else {
                    io_identity<XS>(p, w, b0, b1, At, dB, K2, J, hd, terms);
                }
            }
        }
        wave_sync();
        double* Dr = p.D + (u64)r * Nb;
        for (u32 x = lane; x < Nb; x += 64) {
            const double s = w.acc[x];
            Dr[x] = (p.eps > 0.0 && fabs(s) < p.eps) ? 0.0 : s;
        }
        wave_sync();
        emitted += terms;
        unsigned next = 0;
        if (lane == 0) next = atomicAdd(p.counter, 1u) + nw * gridDim.x;
        r = (unsigned)__builtin_amdgcn_readfirstlane((int)next);
    }
    if (lane == 0 && emitted && p.emitted) atomicAdd(p.emitted, (unsigned long long)emitted);
}

// T1x from T1: groups of 64 per beta rank, 1 << shift of them; behind the last
// single, where there are fewer than 64, the rank itself (io_single's OWN form
// adds the direct element there; the other form adds it apart, and its lanes
// without a single must not meet a target), then slots that nothing reads.
__global__ __launch_bounds__(256) void k_io_t1x(u32 Nb, u32 sB, u32 shift, const u32* __restrict__ T1,
                                                u32* __restrict__ T1x) {
    const u64 all = (u64)Nb << (shift + 6);
    for (u64 t = (u64)blockIdx.x * blockDim.x + threadIdx.x; t < all; t += (u64)gridDim.x * blockDim.x) {
        const u32 r = (u32)(t >> (shift + 6)), s = (u32)t & ((64u << shift) - 1u);
        u32 v = s == sB && sB < 64u ? r : Nb + (s & 63u);
        if (s < sB) {
            const u32 x = T1[(u64)r * sB + s];
            v = (x & 0x1FFFFFu) | ((x >> 21) & 1023u) << 16 | (x & 0x80000000u);
        }
        T1x[t] = v;
    }
}

__global__ __launch_bounds__(256) void k_io_strings(SpaceDev sp, const u64* __restrict__ binom, u32* __restrict__ astr) {
    __shared__ BinomLds B;
    load_binom(B, binom);
    __syncthreads();
    for (u64 r = (u64)blockIdx.x * blockDim.x + threadIdx.x; r < sp.Na; r += (u64)gridDim.x * blockDim.x)
        astr[r] = str_unrank(r, sp.na, sp.n, B);
}

// The nonzero (ia|..) slabs and, in the last block, whether any pair element
// is nonzero (a NaN counts).
__global__ void k_io_slabs(int n, const double* __restrict__ g, const double* __restrict__ K4,
                           unsigned char* __restrict__ gnz) {
    const int ia = blockIdx.x, lane = threadIdx.x;
    const u32 np2 = (u32)(n * (n - 1) / 2);
    bool off = false, diag = false;
    if (ia == n * n) {
        for (u32 t = lane; t < np2 * np2; t += 64) off = off || !(K4[t] == 0.0);
    } else {
        for (int t = lane; t < n * n; t += 64) {
            const bool nz = !(g[(size_t)ia * n * n + t] == 0.0);
            if (t / n != t % n) off = off || nz;
            else diag = diag || nz;
        }
    }
    const u64 o = __ballot(off), d = __ballot(diag);
    if (lane == 0) gnz[ia] = (unsigned char)((o ? 1 : 0) | (d ? 2 : 0));
}

// us per entry of a target row's own source row, and of an alpha-single source
// row with and without alpha-beta elements: what the wavefront that owns the
// target row spends on them (inorder_pays).
struct IoWeights {
    float id, single, single0;
};

// The heaviest target row's time (bits of a float) and the entries' number,
// answered by the last workgroup.  state: maximum and ticket, zero between
// launches.  Few, large workgroups: each adds to the queue at state's address.
constexpr int IO_LOAD_WAVES = 16, IO_LOAD_BLOCK = 64 * IO_LOAD_WAVES;
__global__ __launch_bounds__(IO_LOAD_BLOCK) void k_io_load(SpaceDev sp, const u64* __restrict__ binom,
                                                           const u32* __restrict__ astr,
                                                           const u64* __restrict__ beg, const u64* __restrict__ end,
                                                           const unsigned char* __restrict__ gnz, IoWeights w,
                                                           const u64* __restrict__ nnz, unsigned* __restrict__ state,
                                                           HostLine out) {
    __shared__ BinomLds B;
    __shared__ float s_worst[IO_LOAD_WAVES];
    __shared__ uint8_t s_occ[IO_LOAD_WAVES][32], s_vir[IO_LOAD_WAVES][32];
    load_binom(B, binom);
    __syncthreads();
    const int n = sp.n, na = sp.na, nva = n - na, sA = na * nva, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint8_t *occ = s_occ[wave], *vir = s_vir[wave];
    float worst = 0.0f;
    for (u64 r = (u64)blockIdx.x * IO_LOAD_WAVES + wave; r < sp.Na; r += (u64)gridDim.x * IO_LOAD_WAVES) {
        const u32 A = __builtin_amdgcn_readfirstlane(astr[r]);
        wave_sync();
        if (lane < n) {
            const u32 below = (1u << lane) - 1u;
            if ((A >> lane) & 1u) occ[__popc(A & below)] = (uint8_t)lane;
            else vir[lane - __popc(A & below)] = (uint8_t)lane;
        }
        wave_sync();
        float c = lane == 0 ? w.id * (float)(end[r] - beg[r]) : 0.0f;
        for (int t = lane; t < sA; t += 64) {
            const int i = vir[t % nva], a = occ[t / nva];  // the source holds i and lacks a
            const u64 s = str_rank(A ^ (1u << i) ^ (1u << a), B);
            c += ((gnz[i * n + a] & 1) ? w.single : w.single0) * (float)(end[s] - beg[s]);
        }
        for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off);
        worst = fmaxf(worst, c);
    }
    if (lane == 0) s_worst[wave] = worst;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int k = 1; k < IO_LOAD_WAVES; ++k) worst = fmaxf(worst, s_worst[k]);
    __hip_atomic_fetch_max(&state[0], __float_as_uint(worst), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
    if (__hip_atomic_fetch_add(&state[1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != gridDim.x - 1) return;
    out.p[0] = __hip_atomic_exchange(&state[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    out.p[1] = *nnz;
    __hip_atomic_store(&state[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    out.answer();
}

using Geometry = InOrderGeom;

// log2 of the groups of 64 that hold a beta rank's singles.
u32 t1x_shift(u32 sB) {
    u32 s = 0;
    while ((64u << s) < sB) ++s;
    return s;
}

// The wavefronts per workgroup that keep most of them resident.
bool geometry(sfci_problem* P, Geometry* g) {
    const u64 K = 1 + (u64)P->na * (P->n - P->na) +
                  (u64)(P->na * (P->na - 1) / 2) * (u64)((P->n - P->na) * (P->n - P->na - 1) / 2);
    if (P->Na > IO_MAX_ROWS || P->Nb > IO_MAX_NB) return false;
    int maxlds = 0;
    SFCI_CHECK_HIP(hipDeviceGetAttribute(&maxlds, hipDeviceAttributeMaxSharedMemoryPerBlock, P->device));
    hipFuncAttributes attr{};
    SFCI_CHECK_HIP(hipFuncGetAttributes(&attr, (const void*)k_row_inorder<false>));
    // the most any problem may ask for: the limit is the function's, not the problem's
    for (const void* f : {(const void*)k_row_inorder<false>, (const void*)k_row_inorder<true>})
        SFCI_CHECK_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           maxlds - (int)attr.sharedSizeBytes));
    g->words = (u32)((P->Na + 31) / 32);
    g->off_rows = (u32)(2 * P->n * P->n + (g->words + 1) / 2);
    g->per_wave = (u32)(P->Nb + 128 + (u64)P->n * P->n + (g->words + (K + 1) / 2 + 1) / 2 + 1);
    g->waves = 0;
    int best = 0;
    for (int w = 1; w <= IO_MAXW; ++w) {
        const size_t dyn = ((size_t)g->off_rows + (size_t)w * g->per_wave) * sizeof(double);
        const size_t all = dyn + attr.sharedSizeBytes + 64;
        if (all > (size_t)maxlds) break;
        const int blocks = (int)std::min<size_t>((size_t)maxlds / all, (size_t)(16 / w));
        if (blocks * w > best) best = blocks * w, g->waves = w, g->per_cu = blocks, g->lds = dyn;
    }
    return g->waves > 0;
}

}  // namespace

// Up to 2^25 determinants always (the accumulator's write and selection cost
// less than the sort's 12 launches: 3 entries of 23.5M determinants 333 us
// against 790); above, from a quarter as many terms as determinants: 3 000
// entries of 4.5e8 determinants (0.07 terms each) 15.0 ms against 10.4, 30 000
// (0.7) 52 against 63; of 2.4e8 (0.1) 7.5 against 7.0, (1.0) 23 against 41.
// Below 256 rows, many entries always make long rows (ms, in order and sort:
// 190 rows of 4 845 slots, 10 000 entries near the aufbau string 2.5 and 1.8; 91
// rows of 1 001 1.24 and 1.12); else the entries decide (inorder_pays).
bool inorder_available(sfci_problem* P, u64 nnz) {
    Geometry g;
    if (nnz == 0 || (P->Na < 256 && nnz > 4096 && nnz > 40 * P->Na)) return false;
    if (P->Ndet > (u64(1) << 25) && nnz * terms_per_source(P->n, P->na, P->nb) < P->Ndet / 4) return false;
    if (P->io_state == 0) {
        P->io_state = -1;
        if (!geometry(P, &g) || !rowtile_available(P) || rowtile_ntiles(P) != 1) return false;
        const RowTables t = rowtile_tables(P);
        if (P->nb * (P->nb - 1) > 0 && (P->n - P->nb) * (P->n - P->nb - 1) > 0 && !t.T2r) return false;
        const u32 sB = (u32)(P->nb * (P->n - P->nb)), shift = t1x_shift(sB);
        // [T1x | alpha strings | slab flags, n^2 + 1 bytes | k_io_load's two words]
        const size_t t1x = (size_t)P->Nb << (shift + 6), io_words = t1x + P->Na + (32 * 32 + 8) / 4;
        u32* tab;
        try {
            tab = (u32*)P->io_tab.get((io_words + 2) * sizeof(u32));
        } catch (const sfci_error& e) {
            if (e.code != SFCI_E_NOMEM) throw;
            return false;  // no room: the sort path serves
        }
        u32* const astr = tab + t1x;
        SFCI_CHECK_HIP(hipMemsetAsync(tab + io_words, 0, 2 * sizeof(u32), P->stream));
        P->io_state_words = tab + io_words;
        if (sB)
            hipLaunchKernelGGL(k_io_t1x, dim3((unsigned)std::min<size_t>((t1x + 255) / 256, 4096)), dim3(256), 0,
                               P->stream, (u32)P->Nb, sB, shift, t.T1, tab);
        hipLaunchKernelGGL(k_io_strings, dim3((unsigned)std::min<u64>((P->Na + 255) / 256, 1024)), dim3(256), 0,
                           P->stream, SpaceDev{P->n, P->na, P->nb, P->Na, P->Nb}, P->d_binom, astr);
        hipLaunchKernelGGL(k_io_slabs, dim3((unsigned)(P->n * P->n + 1)), dim3(64), 0, P->stream, P->n, P->d_g,
                           t.K4, (unsigned char*)(astr + P->Na));
        SFCI_CHECK_HIP(hipGetLastError());
        std::vector<unsigned char> f(P->n * P->n + 1);
        SFCI_CHECK_HIP(hipMemcpyAsync(f.data(), astr + P->Na, f.size(), hipMemcpyDeviceToHost, P->stream));
        SFCI_CHECK_HIP(hipStreamSynchronize(P->stream));
        P->io_ab = false;
        for (size_t k = 0; k + 1 < f.size(); ++k) P->io_ab = P->io_ab || (f[k] & 1);
        P->io_pairs = f.back() != 0;
        P->io_geom = g;
        P->io_state = 1;
    }
    return P->io_state > 0;
}

// A target row is one wavefront's, so a vector whose entries gather in few
// source rows waits for the longest target row, where the sort path's time
// depends on the number of terms alone.  The row's time and the sort path's, in
// us, fitted to 620 calls in 50 spaces (1 to 42 504 alpha rows, 100 to 200 000
// entries, near the aufbau string and spread out; nine in ten calls near the
// aufbau string within 25 and 13 %); in order below 0.9 of the sort path's.
// Without this rule, ms, in order and sort: 18 orbitals, 3 + 5 electrons, 4 000
// entries near the aufbau string 2.8 and 1.4, 30 000 9.8 and 4.8, but 30 000
// spread out 1.6 and 5.5; 24, 2 + 4, 10 000 5.4 and 2.4; 16, 1 + 7, 4 000 2.6 and
// 1.0; 20, 4 + 4, 10 000 2.5 and 3.0.  Over the 620 the choice costs 0.2 % on
// average against the faster of both, at most 30 %.
// The row's estimate is a launch and a wait (29 us), left out where no vector of
// at most v.cap entries can have such a row.
bool inorder_pays(sfci_problem* P, const SigmaLaunch& v, RowTileDesc* d) {
    const u64 tps = terms_per_source(P->n, P->na, P->nb);
    const int sB = P->nb * (P->n - P->nb);
    const u64 dB = !P->io_pairs ? 0
                                : (u64)(P->nb * (P->nb - 1) / 2) * (u64)((P->n - P->nb) * (P->n - P->nb - 1) / 2);
    IoWeights w;
    const float more = (float)std::max(0, P->na - 4);
    w.id = dB ? 0.45f + 0.065f * (float)((dB + 63) / 64) + 0.125f * more
              : 0.42f + 0.08f * more;  // one full row of a Hubbard ring, us: 12 sites, 6 + 6 522, 14, 4 + 4 415, 7 + 7 2 250
    w.single0 = 0.01f;
    w.single = sB == 0 ? w.single0 : sB < 64 ? 0.073f : sB == 64 ? 0.12f : 0.36f;
    // what remains for the row: the rest of the call, and the N_det array that the sort path does not touch
    const double rest = 198.0 + 7e-6 * (double)std::min<u64>(P->Ndet, u64(1) << 25);
    const auto limit = [&](u64 nnz) {
        const double terms = (double)nnz * (double)tps;
        return 0.9 * (740.0 + 2.78e-5 * terms + 0.0488 * sqrt(terms)) - 2.7e-6 * terms - rest;
    };
    const double ws = P->io_ab ? std::max(w.single, w.single0) : w.single0;
    const auto most = [&](u64 nnz) { return (double)std::min<u64>(nnz, P->Nb) * w.id + (double)nnz * ws; };
    *d = rowtile_prepare(P, v, nullptr, nullptr);
    launch_fill_u64((u64*)P->ws_rt_desc.get(64), 1, 0, P->stream);  // the kernel's row counter
    bool sure = true;
    for (u64 k = 1; sure; k = std::min<u64>(2 * k, v.cap)) {
        sure = most(k) <= limit(k);
        if (k >= v.cap) break;
    }
    if (sure) return true;
    const HostLine line = host_line(P);
    const RowView rv = rowtile_view(*d);
    const u32* astr = (const u32*)P->io_tab.p + ((size_t)P->Nb << (t1x_shift((u32)sB) + 6));
    hipLaunchKernelGGL(k_io_load,
                       dim3((unsigned)std::min<u64>((P->Na + IO_LOAD_WAVES - 1) / IO_LOAD_WAVES, (u64)P->num_cu / 2)),
                       dim3(IO_LOAD_BLOCK), 0,
                       P->stream, SpaceDev{P->n, P->na, P->nb, P->Na, P->Nb}, P->d_binom, astr, rv.rowbeg, rv.rowend,
                       (const unsigned char*)(astr + P->Na), w, v.v_nnz, P->io_state_words, line);
    SFCI_CHECK_HIP(hipGetLastError());
    const u64* h = wait_line(P, line);
    const u32 bits = (u32)h[0];
    float row;
    std::memcpy(&row, &bits, sizeof row);
    return (double)row <= limit(h[1]);
}

void launch_sigma_inorder(sfci_problem* P, const SigmaLaunch& v, const RowTileDesc& d, double* D,
                          unsigned long long* emitted, double eps) {
    if (P->io_state <= 0) throw sfci_error(-8, "in-order sigma: not available");
    const Geometry& g = P->io_geom;
    const RowView rv = rowtile_view(d);
    const RowTables t = rowtile_tables(P);
    InOrder p{};
    p.sp = SpaceDev{P->n, P->na, P->nb, P->Na, P->Nb};
    p.I = Ints{P->d_h, P->d_g, P->n};
    p.binom = P->d_binom;
    p.v_amp = v.v_amp;
    p.v_beta = rv.v_beta;
    p.v_rb = rv.v_rb;
    p.rowbeg = rv.rowbeg;
    p.rowend = rv.rowend;
    const u32 sB = (u32)(P->nb * (P->n - P->nb));
    p.t1_shift = t1x_shift(sB);
    p.t1_last = sB ? (sB - 1) / 64 : 0;
    p.t1_mask = sB && sB % 64 == 0 ? ~u64(0) : (u64(1) << (sB % 64)) - 1;
    p.T1x = (const u32*)P->io_tab.p;
    p.astr = p.T1x + ((size_t)P->Nb << (p.t1_shift + 6));
    p.T1 = t.T1;
    p.TS = t.TS;
    p.T2r = t.T2r;
    p.T2e = t.T2e;
    p.K2 = t.K2;
    p.K4 = t.K4;
    p.gnz = (const unsigned char*)(p.astr + P->Na);
    p.D = D;
    p.emitted = emitted;
    p.eps = eps;
    p.eps_x = P->excite_eps;
    p.counter = (unsigned*)P->ws_rt_desc.get(64);  // zeroed by inorder_pays
    p.sA = P->na * (P->n - P->na);
    p.sB = P->nb * (P->n - P->nb);
    p.PA = P->na * (P->na - 1) / 2;
    p.QA = (P->n - P->na) * (P->n - P->na - 1) / 2;
    p.dB = (P->nb * (P->nb - 1) / 2) * ((P->n - P->nb) * (P->n - P->nb - 1) / 2);
    p.words = g.words;
    p.off_rows = g.off_rows;
    p.per_wave = g.per_wave;
    const unsigned grid = (unsigned)std::min<u64>((P->Na + g.waves - 1) / g.waves, (u64)P->num_cu * g.per_cu);
    auto kern = p.eps_x > 0.0 ? k_row_inorder<true> : k_row_inorder<false>;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * g.waves), g.lds, P->stream, p);
    SFCI_CHECK_HIP(hipGetLastError());
}
