// Sigma by target rows with the sums of a row in an LDS hash table (fast mode,
// the list iteration's and a truncated sigma's way where N_det does not fit).
//
// A target alpha row of a large space receives few terms for its N_beta slots
// (28 orbitals, 12 electrons, 50 000 entries: 4 000 of 376 740 on average), so
// neither a dense tile nor a sort of all terms suits it.  Per sigma:
//   1. every nonempty source row adds its terms and itself to the rows it
//      reaches (3 598 of them there), twice: counts, then lists.  Nonempty
//      source rows are few, so this is far less than asking every target row
//      for its neighbours;
//   2. a workgroup takes a target row, walks its source rows and adds every
//      term to a hash table of beta ranks in LDS; a row of more terms than its
//      table surely holds is taken in parts, by a second hash of the target;
//   3. the finished table is consumed in place (FusedOut): the T gathers, the
//      marks, the candidates above the bound.
// Rows of very many terms go to the tile kernel (heavy_row_terms); few terms,
// and such as gather in few long rows, to the sort path (list_sigma_rows,
// row_passes_pay).
//
// Bound by: the walk over a row's terms, once per part, and the table's LDS
// accesses (key, then an add).  28 orbitals, 50 000 entries, 1.2e9 terms: a
// sigma took 95 ms by emission, sort and run sums; now 15 ms here, 15 ms for the
// heavy rows' tiles and 2.5 ms for the lists.  With one table of 4096 slots for
// all rows this kernel took 28 ms (up to 15 parts); the long rows' table has
// the whole LDS, the short rows' two to a compute unit.
#include <algorithm>

#include "sfci_internal.h"

namespace {

constexpr int HR_BLOCK = 256;  // of the kernels before the rows
// Tables: short rows two or more to a compute unit, longer ones with all of its LDS.
constexpr int HR_W1 = 4, HR_W2 = 16;                 // wavefronts
constexpr u32 HR_SLOTS1 = 4096, HR_SLOTS2 = 12288;   // slots
constexpr u32 HR_ONE1 = HR_SLOTS1 / 4 * 3;           // terms of a row that one table surely holds
constexpr u32 HR_EMPTY = ~0u;
constexpr int HR_PAIR_SHIFT = 40;  // of a row's count: source rows above, terms below

struct HashRows {
    SpaceDev sp;
    Ints I;
    const u64* binom;
    const double* v_amp;
    const u32 *v_beta, *v_rb;
    const u64 *rowbeg, *rowend;
    const u32* T1;
    const double *TS, *K4;
    const u64* pre;     // first source row of every target row in list
    const u64* list;    // source rows: string << 32 | rank
    const u64* cnt;     // terms and source rows per target row
    const u32* rows;    // the target rows
    u64 lo, hi;
    const FusedOut* fo;
    unsigned long long* emitted;
    double eps, eps_x;
    unsigned* counter;
    int sB, PB, QB;
    u32 more;           // parts are taken this many times finer (a part that did not fit)
};

// MurmurHash3's 32-bit finaliser (A. Appleby, public domain): a bijection whose bits all depend on all of x's.
__device__ __forceinline__ u32 hr_mix(u32 x) {
    x ^= x >> 16;
    x *= 0x85ebca6bu;
    x ^= x >> 13;
    x *= 0xc2b2ae35u;
    return x ^ (x >> 16);
}

// ---- who reaches whom ----

__global__ __launch_bounds__(256) void k_hr_nonempty(const u64* __restrict__ beg, const u64* __restrict__ end, u64 Na,
                                                     u32* __restrict__ out, unsigned* __restrict__ n) {
    const int lane = threadIdx.x & 63;
    for (u64 r0 = (u64)blockIdx.x * 256; r0 < Na; r0 += (u64)gridDim.x * 256) {
        const u64 r = r0 + threadIdx.x;
        const bool p = r < Na && end[r] > beg[r];
        const u64 m = __ballot(p);
        if (!m) continue;
        unsigned at = 0;
        if (lane == 0) at = atomicAdd(n, (unsigned)__popcll(m));
        at = (unsigned)__shfl((int)at, 0);
        if (p) out[at + (unsigned)__popcll(m & ((1ull << lane) - 1ull))] = (u32)r;
    }
}

// A wavefront per 64 neighbours of a nonempty source row.  FILL: the source
// row joins the lists, else the counts.
template <bool FILL>
__global__ __launch_bounds__(HR_BLOCK) void k_hr_reach(SpaceDev sp, const u64* __restrict__ binom,
                                                       const u64* __restrict__ beg, const u64* __restrict__ end,
                                                       const u32* __restrict__ src, const unsigned* __restrict__ n_src,
                                                       u64 c_id, u64 c_s, u64* __restrict__ cnt,
                                                       const u64* __restrict__ pre, u32* __restrict__ cursor,
                                                       u64* __restrict__ list) {
    __shared__ BinomLds B;
    __shared__ uint16_t pO[SFCI_MAX_PAIRS], pV[SFCI_MAX_PAIRS];
    __shared__ uint8_t occ[HR_BLOCK / 64][32], vir[HR_BLOCK / 64][32];
    load_binom(B, binom);
    const int n = sp.n, na = sp.na, nva = n - na, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int sA = na * nva, PA = na * (na - 1) / 2, QA = nva * (nva - 1) / 2, K = 1 + sA + PA * QA;
    for (int t = threadIdx.x; t < PA; t += HR_BLOCK) pO[t] = decode_pair(t, na);
    for (int t = threadIdx.x; t < QA; t += HR_BLOCK) pV[t] = decode_pair(t, nva);
    __syncthreads();
    const u64 parts = (u64)(K + 511) / 512, all = (u64)*n_src * parts;
    for (u64 w = (u64)blockIdx.x * (HR_BLOCK / 64) + wave; w < all; w += (u64)gridDim.x * (HR_BLOCK / 64)) {
        const u32 s = src[w / parts];
        const int t0 = (int)(w % parts) * 512, t1 = min(K, t0 + 512);
        const u32 A = str_unrank(s, na, n, B);
        const u64 ne = end[s] - beg[s];
        wave_sync();
        if (lane < n) {
            const u32 below = (1u << lane) - 1u;
            if ((A >> lane) & 1u) occ[wave][__popc(A & below)] = (uint8_t)lane;
            else vir[wave][lane - __popc(A & below)] = (uint8_t)lane;
        }
        wave_sync();
        for (int t = t0 + lane; t < t1; t += 64) {
            u32 At = A;
            u64 c = c_id;
            if (t > sA) {
                const int x = t - 1 - sA;
                const u32 po = pO[x / QA], pv = pV[x % QA];
                At ^= (1u << occ[wave][po & 255]) ^ (1u << occ[wave][po >> 8]) ^ (1u << vir[wave][pv & 255]) ^
                      (1u << vir[wave][pv >> 8]);
                c = 1;
            } else if (t > 0) {
                At ^= (1u << occ[wave][(t - 1) / nva]) ^ (1u << vir[wave][(t - 1) % nva]);
                c = c_s;
            }
            const u64 r = str_rank(At, B);
            if (FILL) {
                const u32 at = atomicAdd(&cursor[r], 1u);
                list[pre[r] + at] = (u64)A << 32 | s;
            } else {
                atomicAdd((unsigned long long*)&cnt[r], (unsigned long long)(ne * c + (1ull << HR_PAIR_SHIFT)));
            }
        }
    }
}

__global__ __launch_bounds__(256) void k_hr_pairs(const u64* __restrict__ cnt, u64 Na, u64* __restrict__ pre) {
    for (u64 r = (u64)blockIdx.x * 256 + threadIdx.x; r < Na; r += (u64)gridDim.x * 256)
        pre[r] = cnt[r] >> HR_PAIR_SHIFT;
}

// ---- the rows ----

struct Table {
    u32* key;
    double* val;
    u32 part, parts;
    bool full;
};

__device__ __forceinline__ u32 hr_scale(u32 x, u32 n) { return (u32)(((u64)x * n) >> 32); }

// Whether target rank rb belongs to the table's part.
__device__ __forceinline__ bool hr_mine(const Table& t, u32 rb) {
    return t.parts == 1 || hr_scale(hr_mix(rb + 0x9e3779b9u), t.parts) == t.part;
}

// v joins the sum of target rank rb (of this part).
template <u32 SLOTS>
__device__ __forceinline__ void hr_add(Table& t, u32 rb, double v) {
    u32 h = hr_scale(hr_mix(rb), SLOTS);
    for (u32 tries = 0; tries < SLOTS; ++tries) {
        u32 k = t.key[h];
        if (k == HR_EMPTY) {
            k = atomicCAS(&t.key[h], HR_EMPTY, rb);
            if (k == HR_EMPTY) k = rb;
        }
        if (k == rb) {
            atomicAdd(&t.val[h], v);
            return;
        }
        h = h + 1 == SLOTS ? 0 : h + 1;
    }
    t.full = true;
}

// The slot of target rank rb, or HR_EMPTY.
template <u32 SLOTS>
__device__ __forceinline__ u32 hr_find(const Table& t, u32 rb) {
    u32 h = hr_scale(hr_mix(rb), SLOTS);
    for (u32 tries = 0; tries < SLOTS; ++tries) {
        const u32 k = t.key[h];
        if (k == rb) return h;
        if (k == HR_EMPTY) return HR_EMPTY;
        h = h + 1 == SLOTS ? 0 : h + 1;
    }
    return HR_EMPTY;
}

template <int WAVES, u32 SLOTS>
__global__ __launch_bounds__(64 * WAVES) void k_hash_rows(HashRows p) {
    constexpr u32 BLOCK = 64 * WAVES;
    constexpr u32 PART = SLOTS / 16 * 11;  // mean terms per part of a long row
    static_assert(SLOTS % BLOCK == 0, "every thread goes through as many slots");
    extern __shared__ double val[];
    u32* const key = (u32*)(val + SLOTS);
    __shared__ BinomLds B;
    __shared__ uint16_t pO[SFCI_MAX_PAIRS], pV[SFCI_MAX_PAIRS];
    __shared__ uint8_t occ[WAVES][32], vir[WAVES][32];
    __shared__ u32 s_item, s_cand[WAVES];
    __shared__ unsigned long long s_cand0;
    load_binom(B, p.binom);
    const int n = p.sp.n, na = p.sp.na, nb = p.sp.nb, nvb = n - nb, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const u64 Nb = p.sp.Nb;
    const u32 np2 = (u32)(n * (n - 1) / 2), n2 = (u32)(n * n), sB = (u32)p.sB;
    for (int t = threadIdx.x; t < p.PB; t += BLOCK) pO[t] = decode_pair(t, nb);
    for (int t = threadIdx.x; t < p.QB; t += BLOCK) pV[t] = decode_pair(t, nvb);
    const FusedOut f = *p.fo;
    u64 terms = 0, distinct = 0;
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_item = atomicAdd(p.counter, 1u);
        __syncthreads();
        const u64 item = p.lo + s_item;
        if (item >= p.hi) break;
        const u64 r = p.rows[item];
        const u64 c = p.cnt[r], total = c & ((1ull << HR_PAIR_SHIFT) - 1ull);
        const u32 np = (u32)(c >> HR_PAIR_SHIFT);
        const u64* src = p.list + p.pre[r];
        const u32 At = str_unrank_wave(r, na, n, B);
        Table tab{key, val, 0, total <= SLOTS / 4 * 3 ? 1u : (u32)((total + PART - 1) / PART) * p.more, false};
        for (; tab.part < tab.parts; ++tab.part) {
            __syncthreads();
            for (u32 x = threadIdx.x; x < SLOTS; x += BLOCK) {
                key[x] = HR_EMPTY;
                val[x] = 0.0;
            }
            __syncthreads();
            const bool count = tab.part == 0;  // every part walks every term
            // 64 source rows a wavefront at a time, dealt out in turn
            for (u32 q0 = 0; q0 < np; q0 += BLOCK) {
                const u32 q = q0 + (u32)lane * WAVES + (u32)wave;
                u32 beg = 0, ne = 0, info = 0, As = 0;
                int type = 3;
                double e = 0.0;
                if (q < np) {
                    const u64 s = src[q];
                    As = (u32)(s >> 32);
                    beg = (u32)p.rowbeg[(u32)s];
                    ne = (u32)p.rowend[(u32)s] - beg;
                    const u32 d1 = As & ~At, d2 = At & ~As;
                    type = __popc(d1);
                    if (type == 1) {
                        const int i = __builtin_ctz(d1), a = __builtin_ctz(d2);
                        e = p.I.H(i, a);
                        for (u32 m = As & ~d1; m; m &= m - 1u) {
                            const int k = __builtin_ctz(m);
                            e += (p.I.G(i, a, k, k) - p.I.G(i, k, k, a));
                        }
                        info = (u32)(i * n + a) | (u32)between_parity(As, i, a) << 31;
                    } else if (type == 2) {
                        const int i = __builtin_ctz(d1), j = __builtin_ctz(d1 & (d1 - 1u));
                        const int a = __builtin_ctz(d2), b = __builtin_ctz(d2 & (d2 - 1u));
                        const u32 mid = As ^ (1u << i) ^ (1u << a);
                        e = p.K4[(u32)(j * (j - 1) / 2 + i) * np2 + (u32)(b * (b - 1) / 2 + a)];
                        if (between_parity(As, i, a) ^ between_parity(mid, j, b)) e = -e;
                        if (e == 0.0) ne = 0;  // adds nothing
                    }
                }
                // alpha doubles: lanes over the flattened (row, entry) list
                {
                    const u32 mine = type == 2 ? ne : 0u;
                    u32 inc = mine;
                    for (int off = 1; off < 64; off <<= 1) {
                        const u32 y = (u32)__shfl_up((int)inc, off);
                        if (lane >= off) inc += y;
                    }
                    const u32 excl = inc - mine, tot = (u32)__shfl((int)inc, 63), from = beg - excl;
                    for (u32 g0 = 0; g0 < tot; g0 += 128) {
                        u32 rb[2];
                        double am[2], el[2];
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const u32 g = g0 + (u32)u * 64 + (u32)lane;
                            int x = 0;
                            for (int step = 32; step >= 1; step >>= 1)
                                if ((u32)__shfl((int)excl, x + step) <= g) x += step;
                            const u32 k = (u32)__shfl((int)from, x) + g;
                            el[u] = __shfl(e, x);
                            rb[u] = g < tot ? p.v_rb[k] : 0u;
                            am[u] = g < tot ? p.v_amp[k] : 0.0;
                        }
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            if (g0 + (u32)u * 64 + (u32)lane >= tot) continue;
                            const double t = el[u] * am[u];
                            if (p.eps_x > 0.0 && (xscreened(t, p.eps_x) || t == 0.0)) continue;
                            if (count) ++terms;
                            if (hr_mine(tab, rb[u])) hr_add<SLOTS>(tab, rb[u], t);
                        }
                    }
                }
                // alpha singles, row by row
                for (u64 m = __ballot(type == 1 && ne != 0); m; m &= m - 1) {
                    const int j = __builtin_ctzll(m);
                    const u32 b = (u32)__builtin_amdgcn_readlane((int)beg, j);
                    const u32 l = (u32)__builtin_amdgcn_readlane((int)ne, j);
                    const u32 f0 = (u32)__builtin_amdgcn_readlane((int)info, j);
                    const double cst = lane_f64(e, j);
                    const double* Gia = p.I.g + (f0 & 0x7fffffffu) * n2;
                    const int par = (int)(f0 >> 31);
                    for (u32 k = lane; k < l; k += 64) {
                        const u32 rb = p.v_rb[b + k];
                        const bool mine = hr_mine(tab, rb);
                        if (!mine && !count) continue;
                        double el = cst;
                        for (u32 mm = p.v_beta[b + k]; mm; mm &= mm - 1u) el += Gia[__builtin_ctz(mm) * (n + 1)];
                        if (el == 0.0) continue;
                        if (count) ++terms;
                        if (mine) hr_add<SLOTS>(tab, rb, (par ? -el : el) * p.v_amp[b + k]);
                    }
                    // lanes over (entry, beta single), two groups in flight
                    const u32 nf = l * sB;
                    for (u32 g0 = 0; g0 < nf; g0 += 128) {
                        u32 te[2];
                        double am[2];
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const u32 g = min(g0 + (u32)u * 64 + (u32)lane, nf - 1);
                            const u32 k = g / sB;
                            te[u] = p.T1[(u64)p.v_rb[b + k] * sB + (g - k * sB)];
                            am[u] = p.v_amp[b + k];
                        }
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            if (g0 + (u32)u * 64 + (u32)lane >= nf) continue;
                            const bool mine = hr_mine(tab, te[u] & 0x1FFFFFu);
                            if (!mine && !count) continue;
                            double el = Gia[(te[u] >> 21) & 1023u];
                            if (el == 0.0) continue;
                            if (par ^ (int)(te[u] >> 31)) el = -el;
                            const double t = el * am[u];
                            if (p.eps_x > 0.0 && (xscreened(t, p.eps_x) || t == 0.0)) continue;
                            if (count) ++terms;
                            if (mine) hr_add<SLOTS>(tab, te[u] & 0x1FFFFFu, t);
                        }
                    }
                }
                // the row itself: its entries dealt to the wavefronts
                const u64 id = __ballot(type == 0 && ne != 0);
                u32 ib = 0, il = 0;
                if (id) {
                    const int j = __builtin_ctzll(id);
                    ib = (u32)__builtin_amdgcn_readlane((int)beg, j);
                    il = (u32)__builtin_amdgcn_readlane((int)ne, j);
                }
                for (u32 k = ib; k < ib + il; ++k) {
                    const u32 Bs = p.v_beta[k], rb = p.v_rb[k];
                    const double am = p.v_amp[k];
                    wave_sync();
                    if (lane < n) {
                        const u32 below = (1u << lane) - 1u;
                        if ((Bs >> lane) & 1u) occ[wave][__popc(Bs & below)] = (uint8_t)lane;
                        else vir[wave][lane - __popc(Bs & below)] = (uint8_t)lane;
                    }
                    wave_sync();
                    const u32 nd = (u32)(p.PB * p.QB);
                    for (u32 o = lane; o < 1 + sB + nd; o += 64) {
                        double el;
                        u32 to = rb;
                        if (o == 0) {
                            el = diag_element(p.I, At, Bs);
                        } else if (o <= sB) {
                            const u64 at = (u64)rb * sB + (o - 1);
                            const u32 te = p.T1[at], jb = (te >> 21) & 1023u;
                            el = p.TS[at];
                            for (u32 mm = At; mm; mm &= mm - 1u)
                                el += p.I.g[jb * n2 + __builtin_ctz(mm) * (u32)(n + 1)];
                            if (te >> 31) el = -el;
                            to = te & 0x1FFFFFu;
                        } else {
                            const u32 x = o - 1 - sB;
                            const u32 po = pO[x / (u32)p.QB], pv = pV[x % (u32)p.QB];
                            const int ii = occ[wave][po & 255], jj = occ[wave][po >> 8];
                            const int aa = vir[wave][pv & 255], bb = vir[wave][pv >> 8];
                            const u32 mid = Bs ^ (1u << ii) ^ (1u << aa);
                            el = p.K4[(u32)(jj * (jj - 1) / 2 + ii) * np2 + (u32)(bb * (bb - 1) / 2 + aa)];
                            if (between_parity(Bs, ii, aa) ^ between_parity(mid, jj, bb)) el = -el;
                            to = (u32)str_rank(mid ^ (1u << jj) ^ (1u << bb), B);
                        }
                        if (el == 0.0) continue;
                        const double t = el * am;
                        if (o > sB && p.eps_x > 0.0 && (xscreened(t, p.eps_x) || t == 0.0)) continue;
                        if (count) ++terms;
                        if (hr_mine(tab, to)) hr_add<SLOTS>(tab, to, t);
                    }
                }
            }
            if (tab.full) atomicOr(f.overflow, 2);
            __syncthreads();
            // the finished sums, as the tile kernel hands over its tiles
            const double eps = p.eps;
            const u64 rowbase = r * Nb;
            auto yval = [&](u32 h) { return (eps > 0.0 && fabs(val[h]) < eps) ? 0.0 : val[h]; };
            auto scan_basis = [&](int l, auto&& fn) {
                const u64* rp = f.rowptr + (u64)l * (f.na_rows + 1);
                const u64 s0 = rp[r], s1 = rp[r + 1];
                const u64* wr = f.Wr + (u64)l * f.cap;
                for (u64 i = s0 + lane; i < s1; i += 64) {
                    const u32 h = hr_find<SLOTS>(tab, (u32)(wr[i] - rowbase));
                    if (h != HR_EMPTY) fn(i, h);
                }
            };
            for (int l = wave; l < f.nl; l += WAVES)
                scan_basis(l, [&](u64 i, u32 h) { f.Y[(u64)l * f.cap + i] = yval(h); });
            if (f.distinct)
                for (u32 x = threadIdx.x; x < SLOTS; x += BLOCK) distinct += yval(x) != 0.0 ? 1u : 0u;
            if (!f.collect) continue;
            __syncthreads();
            for (int l = f.mark_from + wave; l < f.nl; l += WAVES) scan_basis(l, [&](u64, u32 h) { val[h] = 0.0; });
            __syncthreads();
            // counted first: one addition to the list's length per part
            const u64 tb = *f.bound;
            auto cand = [&](u32 x) {
                return ((u64)__double_as_longlong(yval(x)) & 0x7fffffffffffffffull) > tb;
            };
            u32 mine = 0;
            for (u32 x = threadIdx.x; x < SLOTS; x += BLOCK) mine += (u32)__popcll(__ballot(cand(x)));
            if (lane == 0) s_cand[wave] = mine;
            __syncthreads();
            if (threadIdx.x == 0) {
                u32 all = 0;
                for (int w = 0; w < WAVES; ++w) all += s_cand[w];
                s_cand0 = all ? atomicAdd((unsigned long long*)f.Rn, (unsigned long long)all) : 0ull;
            }
            __syncthreads();
            u64 at0 = s_cand0;
            for (int w = 0; w < wave; ++w) at0 += s_cand[w];
            for (u32 x = threadIdx.x; mine && x < SLOTS; x += BLOCK) {
                const bool pk = cand(x);
                const u64 m = __ballot(pk);
                if (pk) {
                    const u64 at = at0 + (u64)__popcll(m & ((1ull << lane) - 1ull));
                    if (at < f.Rcap) {
                        f.Rr[at] = rowbase + key[x];
                        f.Ra[at] = yval(x);
                    } else {
                        atomicOr(f.overflow, 1);
                    }
                }
                at0 += (u64)__popcll(m);
            }
        }
    }
    if (f.distinct) {
        for (int off = 32; off >= 1; off >>= 1) distinct += (u64)__shfl_xor((long long)distinct, off);
        if (lane == 0 && distinct) atomicAdd((unsigned long long*)f.distinct, (unsigned long long)distinct);
    }
    for (int off = 32; off >= 1; off >>= 1) terms += (u64)__shfl_xor((long long)terms, off);
    if (lane == 0 && terms && p.emitted) atomicAdd(p.emitted, (unsigned long long)terms);
}

unsigned hr_grid(u64 n) { return (unsigned)std::max<u64>(1, std::min<u64>((n + 255) / 256, 4096)); }

}  // namespace

u64 hash_rows_parts(u64 terms) {
    constexpr u64 part = HR_SLOTS2 / 16 * 11;  // as in k_hash_rows
    return terms <= HR_SLOTS2 / 4 * 3 ? 1 : (terms + part - 1) / part;
}

// Where each target row's list starts.
static void hr_places(sfci_problem* P) {
    u64* pre = (u64*)P->list_ws.hr_pre.p;
    hipLaunchKernelGGL(k_hr_pairs, dim3(hr_grid(P->Na)), dim3(256), 0, P->stream, (const u64*)P->list_ws.hr_cnt.p, P->Na,
                       pre);
    exclusive_scan_u64(P, pre, pre, P->Na, pre + P->Na);
}

static void hr_unpack(HashReach* out) {
    u64 terms = 0, pairs = 0;
    for (u64& c : out->count) {
        pairs += c >> HR_PAIR_SHIFT;
        c &= (1ull << HR_PAIR_SHIFT) - 1ull;
        terms += c;
    }
    out->terms = terms;
    out->pairs = pairs;
}

void hash_rows_count(sfci_problem* P, const RowTileDesc& all, bool lists_follow, HashReach* out) {
    const RowView v = rowtile_view(all);
    const u64 Na = P->Na;
    const SpaceDev sp{P->n, P->na, P->nb, Na, P->Nb};
    const u64 sB = (u64)P->nb * (P->n - P->nb);
    const u64 dB = (u64)(P->nb * (P->nb - 1) / 2) * (u64)((P->n - P->nb) * (P->n - P->nb - 1) / 2);
    ListWs& ws = P->list_ws;
    u64* cnt = (u64*)ws.hr_cnt.get(Na * sizeof(u64));
    ws.hr_pre.get((Na + 1) * sizeof(u64));
    u32* src = (u32*)ws.hr_src.get((2 * Na + 2) * sizeof(u32));  // [nonempty rows | cursors | count]
    u32* cursor = src + Na;
    unsigned* n_src = cursor + Na;
    launch_fill_u64(cnt, Na, 0, P->stream);
    SFCI_CHECK_HIP(hipMemsetAsync(cursor, 0, (Na + 1) * sizeof(u32), P->stream));
    hipLaunchKernelGGL(k_hr_nonempty, dim3(hr_grid(Na)), dim3(256), 0, P->stream, v.rowbeg, v.rowend, Na, src, n_src);
    hipLaunchKernelGGL(k_hr_reach<false>, dim3((unsigned)P->num_cu * 8), dim3(HR_BLOCK), 0, P->stream, sp, P->d_binom,
                       v.rowbeg, v.rowend, src, n_src, 1 + sB + dB, 1 + sB, cnt, (const u64*)nullptr, (u32*)nullptr,
                       (u64*)nullptr);
    if (lists_follow) hr_places(P);
    out->placed = lists_follow;
    SFCI_CHECK_HIP(hipGetLastError());
    out->count.resize(Na);
    SFCI_CHECK_HIP(hipMemcpyAsync(out->count.data(), cnt, Na * sizeof(u64), hipMemcpyDeviceToHost, P->stream));
    if (lists_follow)
        SFCI_CHECK_HIP(hipMemcpyAsync(&out->pairs, (const u64*)ws.hr_pre.p + Na, sizeof(u64), hipMemcpyDeviceToHost,
                                      P->stream));
    SFCI_CHECK_HIP(hipStreamSynchronize(P->stream));
    if (!lists_follow) hr_unpack(out);
}

bool hash_rows_lists(sfci_problem* P, const RowTileDesc& all, HashReach* reach) {
    const RowView v = rowtile_view(all);
    const u64 Na = P->Na;
    const SpaceDev sp{P->n, P->na, P->nb, Na, P->Nb};
    ListWs& ws = P->list_ws;
    size_t freeb = 0, totb = 0;
    SFCI_CHECK_HIP(hipMemGetInfo(&freeb, &totb));
    if (reach->pairs * sizeof(u64) > (freeb + ws.hr_list.bytes) / 4) return false;
    u64* list = (u64*)ws.hr_list.get(std::max<u64>(1, reach->pairs) * sizeof(u64));
    u32* src = (u32*)ws.hr_src.p;
    u32* cursor = src + Na;
    if (!reach->placed) hr_places(P);
    hipLaunchKernelGGL(k_hr_reach<true>, dim3((unsigned)P->num_cu * 8), dim3(HR_BLOCK), 0, P->stream, sp, P->d_binom,
                       v.rowbeg, v.rowend, src, (const unsigned*)(cursor + Na), 0, 0, (u64*)nullptr,
                       (const u64*)ws.hr_pre.p, cursor, list);
    SFCI_CHECK_HIP(hipGetLastError());
    if (reach->placed) hr_unpack(reach);
    return true;
}

void launch_hash_rows(sfci_problem* P, const SigmaLaunch& sl, const RowTileDesc& all, u64 lo, u64 hi, const u32* rows,
                      const FusedOut* d_fo, unsigned long long* emitted, double eps, u32 more, bool small) {
    const RowView v = rowtile_view(all);
    const RowTables t = rowtile_tables(P);
    ListWs& ws = P->list_ws;
    HashRows p{};
    p.sp = SpaceDev{P->n, P->na, P->nb, P->Na, P->Nb};
    p.I = Ints{P->d_h, P->d_g, P->n};
    p.binom = P->d_binom;
    p.v_amp = sl.v_amp;
    p.v_beta = v.v_beta;
    p.v_rb = v.v_rb;
    p.rowbeg = v.rowbeg;
    p.rowend = v.rowend;
    p.T1 = t.T1;
    p.TS = t.TS;
    p.K4 = t.K4;
    p.pre = (const u64*)ws.hr_pre.p;
    p.list = (const u64*)ws.hr_list.p;
    p.cnt = (const u64*)ws.hr_cnt.p;
    p.rows = rows;
    p.lo = lo;
    p.hi = hi;
    p.fo = d_fo;
    p.emitted = emitted;
    p.eps = eps;
    p.eps_x = P->excite_eps;
    p.counter = (unsigned*)ws.hr_ctr.get(64);
    p.sB = P->nb * (P->n - P->nb);
    p.PB = P->nb * (P->nb - 1) / 2;
    p.QB = (P->n - P->nb) * (P->n - P->nb - 1) / 2;
    p.more = more;
    launch_fill_u64((u64*)p.counter, 1, 0, P->stream);
    const u32 slots = small ? HR_SLOTS1 : HR_SLOTS2;
    const int waves = small ? HR_W1 : HR_W2;
    const size_t lds = slots * (sizeof(double) + sizeof(u32));
    auto kern = small ? k_hash_rows<HR_W1, HR_SLOTS1> : k_hash_rows<HR_W2, HR_SLOTS2>;
    SFCI_CHECK_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    const unsigned g = (unsigned)std::min<u64>(hi - lo, (u64)P->num_cu * (small ? 2 : 1));
    hipLaunchKernelGGL(kern, dim3(g), dim3(64 * waves), lds, P->stream, p);
    SFCI_CHECK_HIP(hipGetLastError());
    SFCI_CHECK_HIP(hipStreamSynchronize(P->stream));
}

u64 hash_rows_small() { return HR_ONE1; }
