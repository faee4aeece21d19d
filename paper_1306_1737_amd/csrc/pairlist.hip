// Cluster-pair search (Sec. 2.3 "Pair list construction", the cluster-pair
// search pseudocode, and Sec. 2.4 "Exclusion treatment"), run entirely on the
// GPU as the paper planned.  One wavefront per i-cluster: for each kept image
// shift it walks the candidate grid columns in increasing column order and
// tests that column's j-clusters 64 at a time (one per lane) against the
// bounding-box criterion; the particle pairs of the candidates that lie outside
// the rBB shortcut are checked by the whole wavefront.  A count pass, a
// deterministic scan and a fill pass give a list whose order depends only on
// the input.
//
// Compiled with -ffp-contract=off: the inclusion predicate and the
// exclusion-in-image test are defined by separately rounded FP32 operations.
#include <cstring>

#include "devptr.h"
#include "internal.h"
#include "scan.h"

namespace {

using mxn::gptr;
using mxn::ld;
using mxn::plain;
using mxn::st;

// Search arguments with plain pointers (kernel arguments of the single-system
// launch) or global ones (read from a device table by the batched launch).
template <template <class> class P>
struct SearchArgsT {
    P<const int> nslots;
    P<const float4> xs;
    P<const int> perm, slot_of;
    P<const float4> bbi_lo, bbi_hi, bbj_lo, bbj_hi, colbb;
    P<const int> zfirst;                 // (x, y) per (column, z bin), see z_index in grid.hip
    P<const int> excl_off, excl_idx;
    float Lx, Ly, Lz, inv_x, inv_y, inv_z;
    int nx, ny, nz;
    float rlist, rl2, rb2;
    P<int> part_count;                   // entries found by each (i-cluster, part)
    P<const int> part_start;             // region of each (i-cluster, part)
    P<int> region_overflow;              // set when a region is too small
    P<nb_jentry> entries;   // each region in (shift, j-cluster) order
    P<float> keys;          // bounding-box distance^2 of each entry (or null)
    P<int> jcount;          // entries per j-cluster, kRankSets counters jstride apart (fill pass; zero before it)
    P<int> jrank;           // each written entry's rank among its j-cluster's entries of the workgroup's set
    int nci_cap, parts, jstride, pad;    // no padding: job tables are compared byte by byte
};
using SearchArgs = SearchArgsT<plain>;
using SearchArgsG = SearchArgsT<gptr>;

__device__ inline SearchArgsG to_global(const SearchArgs &a) {
    SearchArgsG g;
    g.nslots = (gptr<const int>)a.nslots;
    g.xs = (gptr<const float4>)a.xs;
    g.perm = (gptr<const int>)a.perm;
    g.slot_of = (gptr<const int>)a.slot_of;
    g.bbi_lo = (gptr<const float4>)a.bbi_lo;
    g.bbi_hi = (gptr<const float4>)a.bbi_hi;
    g.bbj_lo = (gptr<const float4>)a.bbj_lo;
    g.bbj_hi = (gptr<const float4>)a.bbj_hi;
    g.colbb = (gptr<const float4>)a.colbb;
    g.zfirst = (gptr<const int>)a.zfirst;
    g.excl_off = (gptr<const int>)a.excl_off;
    g.excl_idx = (gptr<const int>)a.excl_idx;
    g.Lx = a.Lx; g.Ly = a.Ly; g.Lz = a.Lz; g.inv_x = a.inv_x; g.inv_y = a.inv_y; g.inv_z = a.inv_z;
    g.nx = a.nx; g.ny = a.ny; g.nz = a.nz;
    g.rlist = a.rlist; g.rl2 = a.rl2; g.rb2 = a.rb2;
    g.part_count = (gptr<int>)a.part_count;
    g.part_start = (gptr<const int>)a.part_start;
    g.region_overflow = (gptr<int>)a.region_overflow;
    g.entries = (gptr<nb_jentry>)a.entries;
    g.keys = (gptr<float>)a.keys;
    g.jcount = (gptr<int>)a.jcount;
    g.jrank = (gptr<int>)a.jrank;
    g.nci_cap = a.nci_cap; g.parts = a.parts; g.jstride = a.jstride;
    return g;
}

// Each j-cluster has a rank counter in kRankSets sets; a workgroup counts in the set of its index (workgroups go to
// the XCDs round-robin by index, so the workgroups of one XCD share a set).
__device__ inline int rank_set(int blk) { return blk & (mxn::kRankSets - 1); }

__device__ inline float sq3(float x, float y, float z) { return (x * x + y * y) + z * z; }

__device__ inline float axis_gap(float jlo, float jhi, float ilo, float ihi) {
    float d1 = jlo - ihi, d2 = ilo - jhi;
    float m = d1 > d2 ? d1 : d2;
    return m > 0.0f ? m : 0.0f;
}

// inclusive sum over the lanes at and below this one (DPP row shifts, then row broadcasts)
__device__ inline int lane_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return x;
}
__device__ inline float lane_value(float x, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}
// orders a wavefront's LDS writes before its reads by other lanes
__device__ inline void lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wavefront per (i-cluster, part): a.parts wavefronts share an i-cluster,
// part p takes the p-th contiguous share of every image shift's candidate
// columns.  Bound by VALU issue (4.8 k instructions per wavefront and 110 us on
// the 96 000-atom 8x8 list when every lane checked its own candidate), hence:
//   - Lane s works out image shift s's candidate columns; only shifts that
//     have any are walked (one, for a cluster away from the faces).  For the
//     zero shift columns before the i-cluster's own hold nothing of the half
//     list and are left out, and so are earlier clusters of a window.
//   - Lanes own candidate columns (the z window looked up in the grid's z
//     index, one load in place of two binary searches of about ten in a row),
//     then, after a scan flattens the windows, candidate j-clusters (box test).
//   - The particle check of the candidates outside the rBB shortcut is taken
//     by all lanes together: the candidates are queued in LDS and 64/N of them
//     are checked at a time, lane = (candidate, j-particle), the M i-particles
//     in scalar registers.  Each loads one coalesced 16 N-byte run per
//     candidate instead of N scattered particles per lane.
//   - In the fill pass lane q holds exclusion partner q of the i-particles; it
//     finds its own candidate among the flattened windows and clears its mask
//     bit through LDS, so no candidate loops over the partners.
// More partners than lanes: each accepted candidate reads them from the CSR.
constexpr int kExclStage = 64;   // exclusion partners held, one per lane

template <int M, int N, bool FILL, class A>
__device__ inline void search_body(const A &a, int blk) {
    constexpr unsigned FULL = (1u << M) - 1u;
    constexpr int G = 64 / N;   // candidates per step of the particle check
    __shared__ unsigned queue[4][64];             // candidates to check: cj * 16 + real slots
    __shared__ unsigned long long mexcl[4][64];   // a batch's masks while partners clear bits
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const unsigned long long below = (1ull << lane) - 1ull;
    const int gw = __builtin_amdgcn_readfirstlane(blk * 4 + w);
    const int P = a.parts, ci = gw / P, part = gw % P;
    if (ci >= a.nci_cap) return;
    const int nci = *a.nslots / M;
    if (ci >= nci) {   // beyond the padded slot count of this sort: contributes nothing to the scans
        if (lane == 0) a.part_count[gw] = 0;
        return;
    }
    int wpos = 0, resv = 0;   // fill pass: this part's reserved region
    if (FILL) {
        wpos = a.part_start[gw];
        resv = a.part_start[gw + 1] - wpos;
    }
    const float4 lo = ld(a.bbi_lo + ci), hi = ld(a.bbi_hi + ci);
    // the i-cluster's real slots: the mask the grid sort stores in its box's lo.w
    const unsigned ireal = __builtin_amdgcn_readfirstlane(__float_as_uint(lo.w));
    // keeps the z windows conservative against rounding: the FP32 squared distances
    // carry a relative error below 1e-6, so sqrt of that error is below 1e-3 rlist
    const float zmargin = 1e-3f + 2e-3f * a.rlist;
    auto col_x = [&](float x) { return max(0, min((int)floorf(x * a.inv_x), a.nx - 1)); };   // as the grid sort
    auto col_y = [&](float y) { return max(0, min((int)floorf(y * a.inv_y), a.ny - 1)); };
    // lane k < M: i-particle k (a dummy's NaN fails every distance test)
    float4 pi = ld(a.xs + ci * M + (lane < M ? lane : 0));
    if (!((ireal >> (lane & (M - 1))) & 1u)) pi.x = __builtin_nanf("");
    // lane q < nexcl: exclusion partner q as slot * 8 + i-index, its position and column.  Its chain of loads
    // (offsets, partner, slot, position) starts here and ends with the first columns' own loads, so that the
    // two overlap (55 -> 51 us).
    int nexcl = 0, xv = 0, xcol_x = -1, xcol_y = -1;
    int e0 = 0, e1 = 0, xe = 0, xa = 0;   // lane k < M: CSR range; lane q: partner's CSR entry and i-index
    bool staged = true, fetch = FILL;     // fetch: the partners are still to be loaded
    float4 xp = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (FILL) {
        const int io = max(0, (int)a.perm[ci * M + (lane & (M - 1))]);
        e0 = a.excl_off[io];
        e1 = a.excl_off[io + 1];
    }
    // lane s: image shift s and its candidate columns, a superset with one column of margin against rounding
    const float sx_l = (float)(lane / 9 - 1) * a.Lx, sy_l = (float)((lane / 3) % 3 - 1) * a.Ly,
                sz_l = (float)(lane % 3 - 1) * a.Lz;
    int cx0_l = max(0, (int)floorf((lo.x + sx_l - a.rlist) * a.inv_x) - 1);
    const int cx1_l = min(a.nx - 1, (int)floorf((hi.x + sx_l + a.rlist) * a.inv_x) + 1);
    const int cy0_l = max(0, (int)floorf((lo.y + sy_l - a.rlist) * a.inv_y) - 1);
    const int cy1_l = min(a.ny - 1, (int)floorf((hi.y + sy_l + a.rlist) * a.inv_y) + 1);
    if (lane == 13) cx0_l = max(cx0_l, col_x(lo.x));   // the own column's row: earlier ones precede it in slot order
    // wrapped particles lie in [0, L): no z window can be hit from beyond that range
    const bool any = lane >= 13 && lane < 27 && cx0_l <= cx1_l && cy0_l <= cy1_l &&
                     !(lo.z + sz_l - a.rlist - zmargin > a.Lz + zmargin || hi.z + sz_l + a.rlist + zmargin < -zmargin);
    if (FILL) {
        const int incl = lane_scan(lane < M && ((ireal >> lane) & 1u) ? e1 - e0 : 0);
        nexcl = __builtin_amdgcn_readlane(incl, M - 1);
        staged = nexcl <= kExclStage && (long)a.nci_cap * M < (1L << 28);   // slot * 8 + i-index fits an int
        fetch = staged && nexcl > 0;
        // partner q's i-particle is the first whose inclusive count exceeds q
        int first = 0;
#pragma unroll
        for (int k = 0; k < M - 1; ++k) {
            const int ik = __builtin_amdgcn_readlane(incl, k);
            if (lane >= ik) { xa = k + 1; first = ik; }
        }
        xe = __shfl(e0, xa, 64) + lane - first;
    }
    int cnt = 0;
    // an i-cluster of padding only has no real particles (and an empty box)
    for (unsigned long long shifts = lo.x <= hi.x ? __ballot(any) : 0ull; shifts; shifts &= shifts - 1ull) {
        const int s = __builtin_ctzll(shifts);
        const float sx = lane_value(sx_l, s), sy = lane_value(sy_l, s), sz = lane_value(sz_l, s);
        const int cx0 = __builtin_amdgcn_readlane(cx0_l, s), cx1 = __builtin_amdgcn_readlane(cx1_l, s);
        const int cy0 = __builtin_amdgcn_readlane(cy0_l, s), cy1 = __builtin_amdgcn_readlane(cy1_l, s);
        const float slx = lo.x + sx, shx = hi.x + sx, sly = lo.y + sy, shy = hi.y + sy, slz = lo.z + sz,
                    shz = hi.z + sz;
        const float px = pi.x + sx, py = pi.y + sy, pz = pi.z + sz;   // lane k: shifted i-particle k
        const int kmin = s == 13 ? (ci * M + 1) / N : 0;   // half list: the first cj with cj * N + N - 1 > ci * M
        const int ncy = cy1 - cy0 + 1, ncols = (cx1 - cx0 + 1) * ncy;
        const float rncy = __builtin_amdgcn_rcpf((float)ncy);
        const int c_lo = ncols * part / P, c_hi = ncols * (part + 1) / P;   // this part's columns
        for (int cb = c_lo; cb < c_hi; cb += 64) {
            // one column per lane (ascending column id): its z window of j-clusters
            int k0 = 0, kc = 0;
            const int cidx = cb + lane;
            if (cidx < c_hi) {
                const int row = (int)(((float)cidx + 0.5f) * rncy);   // cidx / ncy (exact: cidx is below 2^20)
                const int c = (cx0 + row) * a.ny + cy0 + cidx - row * ncy;
                const float4 cbb = ld(a.colbb + c);
                const float gx = axis_gap(cbb.x, cbb.z, slx, shx), gy = axis_gap(cbb.y, cbb.w, sly, shy);
                const float g2 = gx * gx + gy * gy;
                if (g2 < a.rl2) {
                    // a j-cluster in this column lies at least (gx, gy) away in x and y, so
                    // only z gaps below sqrt(rlist^2 - g^2) can pass the box test
                    const float zr = sqrtf(a.rl2 - g2) + zmargin;
                    const int z0 = (c * a.nz + mxn::z_bin(slz - zr, a.inv_z, a.nz)) * 2;
                    const int z1 = (c * a.nz + mxn::z_bin(shz + zr, a.inv_z, a.nz)) * 2;
                    k0 = max((int)a.zfirst[z0], kmin);
                    const int k1 = a.zfirst[z1 + 1];
                    kc = max(0, k1 - k0);
                }
            }
            if (FILL && fetch) {
                fetch = false;
                if (lane < nexcl) {
                    const int ps = a.slot_of[a.excl_idx[xe]];
                    xv = ps * 8 + xa;
                    xp = ld(a.xs + ps);
                    xcol_x = col_x(xp.x);
                    xcol_y = col_y(xp.y);
                }
            }
            // flatten the windows of the 64 columns: exclusive offsets by a wave scan
            const int incl = lane_scan(kc);
            const int total = __builtin_amdgcn_readlane(incl, 63);
            const int excl = incl - kc;
            // lane q: the flattened index of its partner's j-cluster, -1 unless the pair is within rlist in this image
            int xt = -1;
            if (FILL && staged && nexcl > 0) {
                const int pc = (xcol_x - cx0) * ncy + xcol_y - cy0 - cb;
                const int from = pc & 63, off = (xv >> 3) / N - __shfl(k0, from, 64), len = __shfl(kc, from, 64);
                const bool here = lane < nexcl && xcol_x >= cx0 && xcol_y >= cy0 && xcol_y <= cy1 && pc >= 0 &&
                                  pc < min(64, c_hi - cb) && off >= 0 && off < len;
                const int at = __shfl(excl, from, 64) + off, ia = xv & 7;
                const float d2 = sq3(__shfl(px, ia, 64) - xp.x, __shfl(py, ia, 64) - xp.y, __shfl(pz, ia, 64) - xp.z);
                if (here && d2 < a.rl2) xt = at;
            }
            for (int t0 = 0; t0 < total; t0 += 64) {
                const int t = t0 + lane;
                // owner column: the last lane whose exclusive offset is <= t (fixed six-step search,
                // executed by every lane so that all shuffles read active lanes)
                const int tt = t < total ? t : total - 1;
                int own = 0;
#pragma unroll
                for (int step = 32; step > 0; step >>= 1) {
                    const int ev = __shfl(excl, own + step, 64);   // own + step <= 63
                    if (ev <= tt) own += step;
                }
                const int cj = __shfl(k0, own, 64) + (tt - __shfl(excl, own, 64));
                bool acc = false, need = false;
                float d2 = 0.0f;
                int nj = 0;   // the candidate's real slots: the first nj (its box's lo.w holds their mask)
                if (t < total) {
                    const float4 jl = ld(a.bbj_lo + cj), jh = ld(a.bbj_hi + cj);
                    d2 = sq3(axis_gap(jl.x, jh.x, slx, shx), axis_gap(jl.y, jh.y, sly, shy),
                             axis_gap(jl.z, jh.z, slz, shz));
                    nj = __popc(__float_as_uint(jl.w));
                    acc = d2 < a.rl2;
                    need = acc && !(d2 < a.rb2);
                }
                const unsigned long long nm = __ballot(need);
                if (nm) {
                    const int r = __popcll(nm & below), nq = __popcll(nm);
                    if (need) queue[w][r] = ((unsigned)cj << 4) | (unsigned)nj;
                    lds_fence();
                    float qx[M], qy[M], qz[M];
#pragma unroll
                    for (int k = 0; k < M; ++k) {
                        qx[k] = lane_value(px, k);
                        qy[k] = lane_value(py, k);
                        qz[k] = lane_value(pz, k);
                    }
                    const int b = lane % N, g = lane / N;
                    auto check = [&](int q, unsigned cq, const float4 &pj) {   // candidates q .. q + G - 1
                        bool near = false;
#pragma unroll
                        for (int k = 0; k < M; ++k) near |= sq3(qx[k] - pj.x, qy[k] - pj.y, qz[k] - pj.z) < a.rl2;
                        const unsigned long long hb = __ballot(near && b < (int)(cq & 15u));
                        if (need && r >= q && r < q + G) acc = (hb >> ((r - q) * N)) & ((1ull << N) - 1ull);
                    };
                    for (int q0 = 0; q0 < nq; q0 += 2 * G) {   // two steps' loads in flight together
                        const unsigned c0 = queue[w][min(q0 + g, nq - 1)], c1 = queue[w][min(q0 + G + g, nq - 1)];
                        const float4 p0 = ld(a.xs + (int)(c0 >> 4) * N + b), p1 = ld(a.xs + (int)(c1 >> 4) * N + b);
                        check(q0, c0, p0);
                        if (q0 + G < nq) check(q0 + G, c1, p1);
                    }
                    lds_fence();   // the next batch's queue
                }
                const unsigned long long accepted = __ballot(acc);
                if (FILL && accepted) {
                    // mask bit b*M + a: both particles real, slot(i) < slot(j) for the unshifted
                    // self/overlapping pair, not an exclusion in this image
                    constexpr unsigned long long kEach = M == 8 ? 0x0101010101010101ull : 0x1111111111111111ull;
                    unsigned long long mask = (nj * M == 64 ? ~0ull : (1ull << (nj * M)) - 1ull) & (ireal * kEach);
                    if (s == 13 && cj * N < ci * M + M) {
#pragma unroll
                        for (int b = 0; b < N; ++b) {
                            const int tr = cj * N + b - ci * M;
                            const unsigned drop = FULL & ~(tr >= M ? FULL : (tr <= 0 ? 0u : (1u << tr) - 1u));
                            mask &= ~((unsigned long long)drop << (b * M));
                        }
                    }
                    if (staged) {
                        const int xl = xt - t0;
                        const bool hits = xt >= 0 && xl >= 0 && xl < 64;
                        if (__ballot(hits)) {
                            mexcl[w][lane] = mask;
                            lds_fence();
                            const int ps = xv >> 3;
                            if (hits) atomicAnd(&mexcl[w][xl], ~(1ull << ((ps & (N - 1)) * M + (xv & 7))));
                            lds_fence();
                            mask = mexcl[w][lane];
                            lds_fence();
                        }
                    } else if (acc) {   // more partners than lanes: read them from the CSR arrays
                        for (int ia = 0; ia < M; ++ia) {
                            if (!((ireal >> ia) & 1u)) continue;
                            const int io = a.perm[ci * M + ia];
                            const float4 p = ld(a.xs + ci * M + ia);
                            for (int e = a.excl_off[io]; e < a.excl_off[io + 1]; ++e) {
                                const int ps = a.slot_of[a.excl_idx[e]];
                                const int b = ps - cj * N;
                                if (b < 0 || b >= N) continue;
                                const float4 pj = ld(a.xs + ps);
                                if (sq3(p.x + sx - pj.x, p.y + sy - pj.y, p.z + sz - pj.z) < a.rl2)
                                    mask &= ~(1ull << (b * M + ia));
                            }
                        }
                    }
                    const int rank = cnt + __popcll(accepted & below);
                    if (acc && rank < resv) {
                        nb_jentry en;
                        en.cj = cj;
                        en.shift = s;
                        en.mlo = (uint32_t)mask;
                        en.mhi = (uint32_t)(mask >> 32);
                        st(a.entries + wpos + rank, en);
                        if (a.keys) a.keys[wpos + rank] = d2;
                        a.jrank[wpos + rank] = atomicAdd((int *)a.jcount + rank_set(blk) * a.jstride + cj, 1);
                    }
                }
                cnt += __popcll(accepted);
            }
        }
    }
    if (lane == 0) {
        a.part_count[gw] = cnt;
        if (FILL && cnt > resv) atomicOr((int *)a.region_overflow, 1);
    }
}

template <int M, int N, bool FILL>
// Six wavefronts per SIMD (at most 80 VGPRs): 45.7 us on the 96 000-atom 8x8 list.  With one set of rank counters it
// took 50.8, against 53.3 at seven wavefronts, which spill (3 million atoms: 1.01 against 1.11 ms); of the 50.8 the
// rank atomics, about 58 G/s over the whole chip, were 17 (without them 34), and taken in one go at the wavefront's
// end it was 49, and 2 % slower at 3 million.
__attribute__((amdgpu_waves_per_eu(6)))
__global__ __launch_bounds__(256) void k_search(SearchArgs a) {
    search_body<M, N, FILL>(a, blockIdx.x);
}

// Work items: each (i-cluster, part) region cut into runs of at most
// item_entries(N) entries, at the offsets of a scan over the regions' counts.
__device__ inline void items_body(int nparts_total, int parts, int per_item, const int *part_count,
                                  const int *part_start, const int *part_istart, long cap_items, int4 *items, int blk) {
    const int g = blk * blockDim.x + threadIdx.x;
    if (g >= nparts_total) return;
    const int resv = part_start[g + 1] - part_start[g];
    const int cnt = min(part_count[g], resv), start = part_start[g], ip = part_istart[g];
    const int nit = (cnt + per_item - 1) / per_item;
    for (int k = 0; k < nit; ++k) {
        if ((long)ip + k >= cap_items) return;   // overflow: latched by finalize_body
        const int js = start + k * per_item;
        const int je = min(js + per_item, start + cnt);
        items[ip + k] = make_int4(g / parts, js, je, 0);
    }
}

// Order the entries of each (i-cluster, part) region by bounding-box distance
// (ties by canonical position), so that the far entries, whose pairs mostly
// lie beyond the cut-off, share force-kernel passes whose pair work can be
// skipped.  One wavefront per region, rank sort with the keys staged in LDS.
__global__ __launch_bounds__(64) void k_sort_entries(const int *part_start, const int *part_count,
                                                     const nb_jentry *in, const float *keys, nb_jentry *out,
                                                     const int *rank_in, int *rank_out) {
    __shared__ float sk[1024];
    const int g = blockIdx.x, lane = threadIdx.x;
    const int b = part_start[g], n = min(part_count[g], part_start[g + 1] - b);
    const bool staged = n <= 1024;
    if (staged)
        for (int i = lane; i < n; i += 64) sk[i] = keys[b + i];
    __syncthreads();
    for (int i = lane; i < n; i += 64) {
        const float ki = staged ? sk[i] : keys[b + i];
        int r = 0;
        for (int j = 0; j < n; ++j) {
            const float kj = staged ? sk[j] : keys[b + j];
            r += (kj < ki) || (kj == ki && j < i);
        }
        out[b + r] = in[b + i];
        rank_out[b + r] = rank_in[b + i];
    }
}

// Region counts of a count pass (one workgroup of 1024 threads).  out[0]: the largest region count; out[2]: the
// entries; out[1], out[4], out[5]: the work items the counts make with full items (per_item entries), halves and
// quarters.  out is pinned host memory.
__global__ __launch_bounds__(1024) void k_max_count(const int *in, int n, int per_item, int *out) {
    __shared__ int red[5][1024];
    const int t = threadIdx.x;
    int v[5] = {0, 0, 0, 0, 0};   // largest, entries, items of three lengths
    for (int i = t; i < n; i += 1024) {
        const int c = in[i];
        v[0] = max(v[0], c);
        v[1] += c;
#pragma unroll
        for (int k = 0; k < 3; ++k) v[2 + k] += (c + (per_item >> k) - 1) / (per_item >> k);
    }
#pragma unroll
    for (int k = 0; k < 5; ++k) red[k][t] = v[k];
    __syncthreads();
    for (int s = 512; s > 0; s >>= 1) {
        if (t < s) {
            red[0][t] = max(red[0][t], red[0][t + s]);
#pragma unroll
            for (int k = 1; k < 5; ++k) red[k][t] += red[k][t + s];
        }
        __syncthreads();
    }
    if (t == 0) {
        out[0] = red[0][0];
        out[1] = red[2][0];
        out[2] = red[1][0];
        out[4] = red[3][0];
        out[5] = red[4][0];
    }
}

// Cleared counters (no memset: these launches may be captured, and memset nodes have given wrong results on replays).
__global__ void k_clear(int n, int *p) {
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) p[k] = 0;
}

// Uniform regions (region g starts at g * size, g = 0 .. n), cleared j-cluster counters and overflow mark.
__global__ void k_reserve(int n, int size, int *start, int njc, int *jcount, int *totals) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g <= n) start[g] = g * size;
    for (int k = g; k < njc; k += gridDim.x * blockDim.x) jcount[k] = 0;
    if (g == 0) totals[3] = 0;
}

// totals: [0] entries, [1] items (from the scan), [3] region overflow; writes
// [2] = usable item count (0 on overflow: a region, the items or the j-force
// rows outgrown), latches the overflow flag and clears [3] for the next build
__device__ inline void finalize_body(int *totals, long cap_items, long cap_rows, int *flags) {
    if (threadIdx.x != 0) return;
    const bool over = totals[3] != 0 || (long)totals[1] > cap_items || (long)totals[0] > cap_rows;
    totals[2] = over ? 0 : totals[1];
    totals[3] = 0;
    if (over) atomicOr(flags, mxn::FLAG_OVERFLOW);
}


// --------------------------------------------------------------------------
// j-cluster view of a list.  The force kernels store each entry's j-forces
// (instead of adding them to memory with atomics) in a row of a buffer whose
// rows are grouped by j-cluster, so that the reduction reads each j-cluster's
// rows contiguously.  The fill pass (and the prune) take each written entry's
// rank among its j-cluster's entries from a counter per j-cluster, in one of
// kRankSets sets by workgroup (the 1.0 M atomics of the 96 000-atom search
// contend for them: 51 us with one set, 45.7 with two, 44.2 with eight, whose
// scan takes longer than that saves); after the
// build the counters are scanned, sets within a j-cluster and j-clusters in
// turn, into each j-cluster's first row and each set's offset in it (and
// cleared for the next build), and a last pass turns every entry's rank into
// its row (the force kernel then reads one row index per entry instead of
// dependent gathers of the starts: measured cheaper).  The row order within a
// j-cluster depends on timing; the reduction sums in fixed point, so the
// forces do not.
constexpr int kJposBlocks = 1024;   // workgroups of the super-cluster view's row pass

struct FinishArgs {
    int nregions, parts, per_item, pad0;   // no padding: job tables are compared byte by byte
    const int *part_count, *part_start;
    int *part_istart;
    long cap_items, cap_rows;
    int *totals, *flags;
    int *jcount, *joff, *jstart;   // counters and offsets [set][jstride], first rows
    int njc, nsets, jstride, pad1;
    int4 *items;
    const nb_jentry *entries;
    int *jrank;
};

// The counters of four consecutive j-clusters from i on, summed over the sets; with CLEAR the counters are zeroed
// and each set's offset within its j-cluster is written.
template <bool CLEAR>
__device__ inline int4 j_counts(const FinishArgs &a, int i) {
    int n[mxn::kRankSets][4], sum[4] = {0, 0, 0, 0};
    const bool whole = i + 4 <= a.njc && (a.nsets == 1 || (a.jstride & 3) == 0);   // the buffers are 16-byte aligned
#pragma unroll
    for (int s = 0; s < mxn::kRankSets; ++s) {   // every load in flight before the first store
        const int *c = a.jcount + (long)s * a.jstride + i;
        if (whole && s < a.nsets) {
            const int4 x = *reinterpret_cast<const int4 *>(c);
            n[s][0] = x.x; n[s][1] = x.y; n[s][2] = x.z; n[s][3] = x.w;
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) n[s][u] = s < a.nsets && i + u < a.njc ? c[u] : 0;
        }
    }
#pragma unroll
    for (int s = 0; s < mxn::kRankSets; ++s) {
        const long at = (long)s * a.jstride + i;
        if (CLEAR && s < a.nsets) {
            if (whole) {
                *reinterpret_cast<int4 *>(a.jcount + at) = make_int4(0, 0, 0, 0);
                if (a.joff) *reinterpret_cast<int4 *>(a.joff + at) = make_int4(sum[0], sum[1], sum[2], sum[3]);
            } else {
                for (int u = 0; u < 4 && i + u < a.njc; ++u) {
                    a.jcount[at + u] = 0;
                    if (a.joff) a.joff[at + u] = sum[u];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) sum[u] += n[s][u];
    }
    return make_int4(sum[0], sum[1], sum[2], sum[3]);
}

// Exclusive scan of the entry counts of one tile's j-clusters into first rows, after the rows of the tiles before
// it (carry; ends as those of the tiles up to it).
constexpr int kTileJ = 4096;   // four per thread
__device__ inline void j_tile(const FinishArgs &a, int base, int *carry) {
    __shared__ int ws[16];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, i = base + t * 4;
    const int4 v = j_counts<true>(a, i);
    const int mine = (v.x + v.y) + (v.z + v.w);
    const int incl = lane_scan(mine);
    if (lane == 63) ws[w] = incl;
    __syncthreads();
    if (t < 64) {
        const int x = lane_scan(t < 16 ? ws[t] : 0);
        if (t < 16) ws[t] = x;
    }
    __syncthreads();
    const int run = *carry + incl - mine + (w > 0 ? ws[w - 1] : 0);
    if (i < a.njc) a.jstart[i] = run;
    if (i + 1 < a.njc) a.jstart[i + 1] = run + v.x;
    if (i + 2 < a.njc) a.jstart[i + 2] = run + v.x + v.y;
    if (i + 3 < a.njc) a.jstart[i + 3] = run + v.x + v.y + v.z;
    *carry += ws[15];
    __syncthreads();   // ws reused by the next tile
    if (t == 0 && base + kTileJ >= a.njc) a.jstart[a.njc] = *carry;
}

__device__ inline void j_scan(const FinishArgs &a) {
    int carry = 0;
    for (int base = 0; base < a.njc; base += kTileJ) j_tile(a, base, &carry);
}

// After a fill (or prune) pass, two independent workgroups of 1024 threads: the first scans the regions'
// entry counts into item offsets and sets the usable item count (finalize_body, by the thread that wrote
// the totals), the second scans the j-cluster counters.
__device__ inline void finish_body(const FinishArgs &a, int which) {
    if (which == 0) {
        mxn::scan_body(a.part_count, a.part_istart, a.nregions, 2, a.per_item, a.totals + 1, a.totals);
        finalize_body(a.totals, a.cap_items, a.cap_rows, a.flags);
    } else {
        j_scan(a);
    }
}
__global__ __launch_bounds__(1024) void k_finish(FinishArgs a) { finish_body(a, blockIdx.x); }

// The same for long lists in two launches of one workgroup per tile: first the tiles' sums, then each tile's
// scan from the sum of the tiles before it (one workgroup takes 123 us for the 3 million atom list's 380 000
// regions and as many j-clusters).
constexpr int kTileRegions = 8192;   // by 1024 threads
__device__ inline int region_tiles(const FinishArgs &a) { return (a.nregions + kTileRegions - 1) / kTileRegions; }

// sums over the workgroup's 1024 threads
__device__ inline int2 block_sum2(int x, int y) {
    __shared__ int2 red[16];
    const int t = threadIdx.x;
    x = __builtin_amdgcn_readlane(lane_scan(x), 63);
    y = __builtin_amdgcn_readlane(lane_scan(y), 63);
    if ((t & 63) == 0) red[t >> 6] = make_int2(x, y);
    __syncthreads();
    int2 s = make_int2(0, 0);
    for (int k = 0; k < 16; ++k) {
        s.x += red[k].x;
        s.y += red[k].y;
    }
    __syncthreads();
    return s;
}

__global__ __launch_bounds__(1024) void k_finish_sums(FinishArgs a, int2 *sums) {
    const int tr = region_tiles(a), b = blockIdx.x, t = threadIdx.x;
    int x = 0, y = 0;
    if (b < tr) {   // (items, entries) of the tile's regions
        for (int i = b * kTileRegions + t; i < min(a.nregions, (b + 1) * kTileRegions); i += 1024) {
            const int c = a.part_count[i];
            x += (c + a.per_item - 1) / a.per_item;
            y += c;
        }
    } else {
        const int4 v = j_counts<false>(a, (b - tr) * kTileJ + t * 4);
        x = (v.x + v.y) + (v.z + v.w);
    }
    const int2 v = block_sum2(x, y);
    if (t == 0) sums[b] = v;
}

__global__ __launch_bounds__(1024) void k_finish_tiles(FinishArgs a, const int2 *sums) {
    const int tr = region_tiles(a), b = blockIdx.x, t = threadIdx.x;
    const int first = b < tr ? 0 : tr;
    int x = 0, y = 0;
    for (int k = first + t; k < b; k += 1024) {
        x += sums[k].x;
        y += sums[k].y;
    }
    const int2 before = block_sum2(x, y);
    if (b >= tr) {
        int carry = before.x;
        j_tile(a, (b - tr) * kTileJ, &carry);
        return;
    }
    const int base = b * kTileRegions, n = min(kTileRegions, a.nregions - base);
    mxn::scan_body(a.part_count + base, a.part_istart + base, n, 2, a.per_item, nullptr, nullptr, before.x,
                   b == tr - 1);
    if (b == tr - 1 && t == 0) {
        a.totals[1] = before.x + sums[b].x;
        a.totals[0] = before.y + sums[b].y;
        finalize_body(a.totals, a.cap_items, a.cap_rows, a.flags);
    }
}

// After the scans (and the distance sort, if any): one wavefront per region writes the region's work items
// and turns each of its entries' rank into the entry's row (its j-cluster's first row, the offset of the set the
// region's workgroup counted in, and the rank), for a usable list.
__device__ inline void items_rows_body(const FinishArgs &a, int blk) {
    const int g = __builtin_amdgcn_readfirstlane(blk * 4 + (threadIdx.x >> 6)), lane = threadIdx.x & 63;
    if (g >= a.nregions) return;
    const int start = a.part_start[g], resv = a.part_start[g + 1] - start;
    const int cnt = min(a.part_count[g], resv), ip = a.part_istart[g];
    const int nit = (cnt + a.per_item - 1) / a.per_item;
    for (int k = lane; k < nit; k += 64) {
        if ((long)ip + k >= a.cap_items) break;   // overflow: latched by finalize_body
        const int js = start + k * a.per_item;
        a.items[ip + k] = make_int4(g / a.parts, js, min(js + a.per_item, start + cnt), 0);
    }
    if (a.totals[2] == 0) return;   // no usable items (or no entries): the rows are never read
    const int *off = a.joff + (long)rank_set(blk) * a.jstride;
    for (int e = start + lane; e < start + cnt; e += 64) {
        const int cj = a.entries[e].cj;
        a.jrank[e] += a.jstart[cj] + off[cj];
    }
}
__global__ __launch_bounds__(256) void k_items_rows(FinishArgs a) { items_rows_body(a, blockIdx.x); }

// Item offsets of full-length items over unchanged regions; an overflowed list (items, none usable) stays unusable.
__global__ __launch_bounds__(1024) void k_full_items(int nregions, int per_item, const int *part_count,
                                                     int *part_istart, int *totals) {
    const bool usable = totals[2] > 0;
    __syncthreads();   // read before the scan's thread 0 writes the totals
    mxn::scan_body(part_count, part_istart, nregions, 2, per_item, totals + 1, totals);
    if (threadIdx.x == 0 && usable) totals[2] = totals[1];
}

__global__ void k_items(int nparts_total, int parts, int per_item, const int *part_count, const int *part_start,
                        const int *part_istart, long cap_items, int4 *items) {
    items_body(nparts_total, parts, per_item, part_count, part_start, part_istart, cap_items, items, blockIdx.x);
}

// --------------------------------------------------------------------------
// Second stage of a two-stage list (Sec. 2.3: the list built from bounding
// boxes, then cluster pairs whose particles are all beyond a radius removed
// by a particle-distance test on the GPU).  One wavefront per region of the
// outer list: an entry is kept iff a real particle of
// the i-cluster, moved by the entry's image shift, and a real particle of
// the j-cluster are closer than r, formed with the search's own separately
// rounded FP32 operations, at the gathered positions of the call.  Kept
// entries keep their order, masks and region; like the fill pass, each takes
// its rank within its j-cluster.
struct PruneArgs {
    const int *nslots;
    const float4 *xs_now;
    const float4 *bbi_lo, *bbj_lo;   // real-slot masks (w) of the i- and j-clusters
    const int *part_start;      // the regions (the outer list's layout)
    const int *part_count_in;   // entries of the outer list per region
    const int *totals_in;       // the outer list's totals: [1] items, [2] usable items
    const nb_jentry *in;
    int *part_count;            // kept entries per region
    nb_jentry *out;
    int *jcount, *jrank;
    int *region_overflow;
    float Lx, Ly, Lz, r2;
    int nregions, parts, jstride;
};

// Lane = (entry, j-particle), 64/N entries a step: an entry's particles are one coalesced 16 N-byte run (one lane per
// entry read N scattered particles and N permutation words).  The i-particles
// moved by an image shift are formed once per run of equal shifts.  54 us for
// 1.6 M entries (66 us with one lane per entry): the issue of 117 vector
// instructions a step, 32 to 40 us, and the rank atomics, 11.
template <int M, int N>
__global__ __launch_bounds__(256) void k_prune(PruneArgs a) {
    constexpr int G = 64 / N;
    const int lane = threadIdx.x & 63, g = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (g >= a.nregions) return;
    // an overflowed outer list (items counted, none usable) is incomplete, and so is its prune
    if (a.totals_in[2] == 0 && a.totals_in[1] > 0) {
        if (lane == 0) {
            a.part_count[g] = 0;
            if (g == 0) atomicOr(a.region_overflow, 1);
        }
        return;
    }
    const int ci = g / a.parts;
    if (ci >= *a.nslots / M) {
        if (lane == 0) a.part_count[g] = 0;
        return;
    }
    const int start = a.part_start[g];
    const int n_in = min(a.part_count_in[g], a.part_start[g + 1] - start);
    float ix[M], iy[M], iz[M];
    const unsigned ireal = __float_as_uint(a.bbi_lo[ci].w);   // real slots, stored by the grid sort
#pragma unroll
    for (int k = 0; k < M; ++k) {   // a dummy's NaN fails every distance test
        const float4 p = a.xs_now[ci * M + k];
        ix[k] = ((ireal >> k) & 1u) ? p.x : __builtin_nanf("");
        iy[k] = p.y; iz[k] = p.z;
    }
    float px[M], py[M], pz[M];   // i-particles moved by shift cur
    int cur = -1;
    const int b = lane % N, q = lane / N;
    int cnt = 0;
    for (int e0 = 0; e0 < n_in; e0 += 64) {
        const int left = min(64, n_in - e0);
        const nb_jentry en = a.in[start + e0 + min(lane, left - 1)];   // lane's own entry of this run of 64
        const unsigned jl = __float_as_uint(a.bbj_lo[en.cj].w);
        unsigned long long keep = 0;   // bit of each kept entry
        for (int u0 = 0; u0 < left; u0 += G) {
            const int u = min(u0 + q, left - 1);
            const int cj = __shfl(en.cj, u, 64), s = __shfl(en.shift, u, 64);
            const bool real = (__shfl((int)jl, u, 64) >> b) & 1;
            const float4 pj = a.xs_now[cj * N + b];
            const int s0 = __builtin_amdgcn_readfirstlane(s);
            if (s0 != cur) {
                cur = s0;
                const float sx = (float)(s0 / 9 - 1) * a.Lx, sy = (float)((s0 / 3) % 3 - 1) * a.Ly,
                            sz = (float)(s0 % 3 - 1) * a.Lz;
#pragma unroll
                for (int k = 0; k < M; ++k) {
                    px[k] = ix[k] + sx;
                    py[k] = iy[k] + sy;
                    pz[k] = iz[k] + sz;
                }
            }
            bool near = false;
            if (__ballot(s != s0) == 0ull) {
#pragma unroll
                for (int k = 0; k < M; ++k) near |= sq3(px[k] - pj.x, py[k] - pj.y, pz[k] - pj.z) < a.r2;
            } else {   // entries of several image shifts in one step
                const float sx = (float)(s / 9 - 1) * a.Lx, sy = (float)((s / 3) % 3 - 1) * a.Ly,
                            sz = (float)(s % 3 - 1) * a.Lz;
#pragma unroll
                for (int k = 0; k < M; ++k)
                    near |= sq3((ix[k] + sx) - pj.x, (iy[k] + sy) - pj.y, (iz[k] + sz) - pj.z) < a.r2;
            }
            const unsigned long long hb = __ballot(near && real);
            // lane's entry is one of this step's: its N bits
            const int w = lane - u0;
            const bool mine = w >= 0 && w < G && lane < left && ((hb >> ((w & (G - 1)) * N)) & ((1ull << N) - 1ull));
            keep |= __ballot(mine);
        }
        if ((keep >> lane) & 1ull) {
            const int pos = start + cnt + __popcll(keep & ((1ull << lane) - 1ull));
            a.out[pos] = en;
            a.jrank[pos] = atomicAdd(a.jcount + rank_set(blockIdx.x) * a.jstride + en.cj, 1);
        }
        cnt += __popcll(keep);
    }
    if (lane == 0) a.part_count[g] = cnt;
}

// --------------------------------------------------------------------------
// Super-cluster view of an 8x8 list (the grouped layout of Sec. 2.3 and 3.2:
// S consecutive i-clusters share one list of j-clusters).  One workgroup per
// super-cluster gathers the entries of its S i-clusters as 64-bit keys
// (shift, j-cluster, i-cluster within the super-cluster, entry position),
// sorts them in LDS (bitonic), and writes one super-cluster entry per
// distinct (shift, j-cluster): (j-cluster, shift | i-cluster bits << 8 |
// (self i-cluster + 1) << 16, 0, rank among the j-cluster's entries) and a
// record of S exclusion masks, slot g for i-cluster g (slots of i-clusters
// the entry does not reach are not written).  The self i-cluster is the
// one the j-cluster is (zero shift), whose pass is a half triangle; 0 if
// none.  Outputs go to the super-cluster's span of the list's regions (its
// keys fit there, so its entries do too).  The order depends only on the
// list, so the forces do as well.
constexpr int kSciKeys = 4096;

struct SciArgs {
    const int *nslots;
    const int *totals;   // the list's: [2] usable items (0 after an overflow)
    const int *part_start, *part_count;
    const nb_jentry *entries;
    int parts, nregions, S, ngroups;
    int4 *ent;
    uint2 *mask;
    int *count, *base;   // per super-cluster: entries; first position (base[ngroups]: end)
    int *jcount;         // per j-cluster counters (zero before the pass)
};

// exclusive prefix of a flag over the 256 threads, and the flag count
__device__ inline int block_flag_scan(bool f, int *sw, int &total) {
    const unsigned long long b = __ballot(f);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int r = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(b >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)b, 0u));
    if (lane == 0) sw[w] = __popcll(b);
    __syncthreads();
    int off = 0;
    for (int k = 0; k < w; ++k) off += sw[k];
    total = sw[0] + sw[1] + sw[2] + sw[3];
    __syncthreads();
    return off + r;
}

__global__ __launch_bounds__(256) void k_sci_view(SciArgs a) {
    __shared__ unsigned long long key[kSciKeys];
    __shared__ int roff[65];
    __shared__ int sw[4];
    const int grp = blockIdx.x, t = threadIdx.x;
    const int span = a.S * a.parts;
    const int r0 = min(grp * span, a.nregions), r1 = min(r0 + span, a.nregions);
    const int base = a.part_start[r0];
    if (t == 0) {
        a.base[grp] = base;
        if (grp == a.ngroups - 1) a.base[grp + 1] = a.part_start[r1];
        const int nci = *a.nslots / 8;
        const bool usable = a.totals[2] > 0;
        int o = 0;
        for (int r = r0; r < r1; ++r) {
            roff[r - r0] = o;
            const int cap = a.part_start[r + 1] - a.part_start[r];
            o += (usable && r / a.parts < nci) ? min(a.part_count[r], cap) : 0;
        }
        roff[r1 - r0] = o;
    }
    __syncthreads();
    const int n = min(roff[r1 - r0], kSciKeys);   // the host sizes S so that every span fits
    for (int r = r0; r < r1; ++r) {
        const int o = roff[r - r0], cnt = roff[r - r0 + 1] - o, s0 = a.part_start[r];
        const unsigned g = (unsigned)((r - r0) / a.parts);
        for (int k = t; k < cnt && o + k < kSciKeys; k += 256) {
            const nb_jentry e = a.entries[s0 + k];
            const unsigned kk = ((unsigned)e.shift << 27) | ((unsigned)e.cj << 3) | g;
            key[o + k] = ((unsigned long long)kk << 32) | (unsigned)(s0 + k);
        }
    }
    int np = 1;
    while (np < n) np <<= 1;
    for (int k = n + t; k < np; k += 256) key[k] = ~0ull;
    __syncthreads();
    for (int size = 2; size <= np; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int i = t; i < np / 2; i += 256) {
                const int lo = 2 * i - (i & (stride - 1)), hi = lo + stride;
                const bool up = (lo & size) == 0;
                const unsigned long long x = key[lo], y = key[hi];
                if ((x > y) == up) {
                    key[lo] = y;
                    key[hi] = x;
                }
            }
            __syncthreads();
        }
    int done = 0;
    for (int p0 = 0; p0 < n; p0 += 256) {
        const int p = p0 + t;
        unsigned long long kp = 0;
        bool head = false;
        if (p < n) {
            kp = key[p];
            head = p == 0 || (key[p - 1] >> 35) != (kp >> 35);
        }
        int tot;
        const int idx = done + block_flag_scan(head, sw, tot);
        if (head) {
            const int cj = (int)((kp >> 35) & 0xFFFFFFu), shift = (int)(kp >> 59);
            int gm = 0;
            for (int q = p; q < n && (key[q] >> 35) == (kp >> 35); ++q) {
                const int g = (int)((key[q] >> 32) & 7u);
                const nb_jentry e = a.entries[(int)(unsigned)key[q]];
                a.mask[(long)(base + idx) * a.S + g] = make_uint2(e.mlo, e.mhi);
                gm |= 1 << g;
            }
            const int own = cj - grp * a.S;
            const int self = (shift == 13 && own >= 0 && own < a.S) ? own + 1 : 0;
            const int rank = atomicAdd(a.jcount + cj, 1);
            a.ent[base + idx] = make_int4(cj, shift | (gm << 8) | (self << 16), 0, rank);
        }
        done += tot;
    }
    if (t == 0) a.count[grp] = done;
}

// rank -> row for every super-cluster entry of a usable work item
__global__ __launch_bounds__(256) void k_sci_rows(const int *totals, const int4 *items, int4 *ent, const int *jstart) {
    const int lane = threadIdx.x & 63;
    const int total = totals[2];
    for (int t = blockIdx.x * 4 + (threadIdx.x >> 6); t < total; t += gridDim.x * 4) {
        const int4 it = items[t];
        const int e = it.y + lane;
        if (e < it.z) ent[e].w += jstart[ent[e].x];
    }
}

// --------------------------------------------------------------------------
// Batched rebuild of many replicas' lists (the fill pass into the regions the
// replicas' last synchronous builds sized), one launch per stage; a
// workgroup finds its replica by binary search in the stage's prefix of
// share sizes.

struct ListJob {
    SearchArgs a;
    FinishArgs f;
};
static_assert(sizeof(SearchArgs) == 19 * sizeof(void *) + 16 * sizeof(int) &&
                  sizeof(FinishArgs) == 11 * sizeof(void *) + 2 * sizeof(long) + 8 * sizeof(int) &&
                  sizeof(ListJob) == sizeof(SearchArgs) + sizeof(FinishArgs),
              "a job table has padding");

enum { LS_SEARCH, LS_NSTAGES };   // one workgroup per four regions: the search and the last pass

__device__ inline int job_of(const int *off, int n, int b) {
    int lo = 0, hi = n - 1;   // last r with off[r] <= b
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

template <int M, int N>
__global__ __launch_bounds__(256) void kb_search(const ListJob *J, const int *off, int n) {
    const int r = job_of(off, n, blockIdx.x);
    search_body<M, N, true>(to_global(J[r].a), blockIdx.x - off[r]);
}

__global__ __launch_bounds__(1024) void kb_finish(const ListJob *J) { finish_body(J[blockIdx.x / 2].f, blockIdx.x & 1); }

__global__ __launch_bounds__(256) void kb_items_rows(const ListJob *J, const int *off, int n) {
    const int r = job_of(off, n, blockIdx.x);
    items_rows_body(J[r].f, blockIdx.x - off[r]);
}

template <int M, int N>
void run(nb_list *l, SearchArgs &a, bool fill, int nblocks, hipStream_t st) {
    if (fill)
        k_search<M, N, true><<<nblocks, 256, 0, st>>>(a);
    else
        k_search<M, N, false><<<nblocks, 256, 0, st>>>(a);
}

}  // namespace

namespace mxn {

static void clear_ints(void *p, long n, hipStream_t st) {
    k_clear<<<(int)std::min(1024L, (n + 255) / 256), 256, 0, st>>>((int)n, (int *)p);
}

static SearchArgs make_search(const nb_list *l, const int *excl_off, const int *excl_idx) {
    const nb_grid *g = l->grid;
    SearchArgs a{};
    a.nslots = (const int *)g->nslots.p;
    a.xs = (const float4 *)g->xs.p;
    a.perm = (const int *)g->perm.p;
    a.slot_of = (const int *)g->slot_of.p;
    a.bbi_lo = (const float4 *)g->bbi_lo.p;
    a.bbi_hi = (const float4 *)g->bbi_hi.p;
    a.bbj_lo = (const float4 *)(g->nn == g->m ? g->bbi_lo.p : g->bbj_lo.p);
    a.bbj_hi = (const float4 *)(g->nn == g->m ? g->bbi_hi.p : g->bbj_hi.p);
    a.colbb = (const float4 *)g->colbb.p;
    a.zfirst = (const int *)g->zfirst.p;
    a.excl_off = excl_off;
    a.excl_idx = excl_idx;
    a.Lx = g->Lf[0]; a.Ly = g->Lf[1]; a.Lz = g->Lf[2];
    a.inv_x = g->inv_x; a.inv_y = g->inv_y; a.inv_z = g->inv_z;
    a.nx = g->nx; a.ny = g->ny; a.nz = g->nz;
    a.rlist = l->rlist;
    volatile float rl2 = l->rlist * l->rlist, rb2 = l->rbb * l->rbb;
    a.rl2 = rl2; a.rb2 = rb2;
    a.part_count = (int *)l->part_count.p;
    a.part_start = (const int *)l->part_start.p;
    a.region_overflow = (int *)l->totals.p + 3;
    a.nci_cap = g->slots_cap / g->m;
    a.jstride = rank_stride(g->slots_cap / g->nn);
    return a;
}


static FinishArgs make_finish(const nb_list *l, int nregions, int parts) {
    const nb_grid *g = l->grid;
    FinishArgs f{};
    f.nregions = nregions;
    f.parts = parts;
    f.per_item = l->per_item;
    f.part_count = (const int *)l->part_count.p;
    f.part_start = (const int *)l->part_start.p;
    f.part_istart = (int *)l->part_istart.p;
    f.cap_items = l->cap_items;
    f.cap_rows = l->cap_rows;
    f.totals = (int *)l->totals.p;
    f.flags = l->ctx->d_flags;
    f.jcount = (int *)l->jcount.p;
    f.joff = (int *)l->joff.p;
    f.jstart = (int *)l->jstart.p;
    f.njc = g->slots_cap / g->nn;
    f.nsets = kRankSets;
    f.jstride = rank_stride(f.njc);
    f.items = (int4 *)l->items.p;
    f.entries = (const nb_jentry *)l->entries.p;
    f.jrank = (int *)l->jrank.p;
    return f;
}

// counters, offsets and tile sums of a list with njc j-clusters; the sums come after the offsets
static size_t joff_bytes(long njc, long nregions) {
    const long tiles = (nregions + kTileRegions - 1) / kTileRegions + (njc + kTileJ - 1) / kTileJ;
    return (size_t)kRankSets * rank_stride(njc) * 4 + (size_t)tiles * sizeof(int2);
}

// item offsets per region (totals[0] = entries, totals[1] = items), usable count and j-cluster first rows of a
// list after its fill or prune pass
static void finish_list(const FinishArgs &f, hipStream_t st) {
    const int tr = (f.nregions + kTileRegions - 1) / kTileRegions, tj = (f.njc + kTileJ - 1) / kTileJ;
    if (tr <= kOneGroupTiles / 2 && tj <= kOneGroupTiles) {
        k_finish<<<2, 1024, 0, st>>>(f);
    } else {
        int2 *sums = (int2 *)(f.joff + (long)kRankSets * f.jstride);
        k_finish_sums<<<tr + tj, 1024, 0, st>>>(f, sums);
        k_finish_tiles<<<tr + tj, 1024, 0, st>>>(f, sums);
    }
}
// work items and each usable entry's row (after finish_list, and after the distance sort)
static void finish_rows(const FinishArgs &f, hipStream_t st) { k_items_rows<<<(f.nregions + 3) / 4, 256, 0, st>>>(f); }

size_t list_job_size() { return sizeof(ListJob); }
int list_job_stages() { return LS_NSTAGES; }

// The list must have been sized by a synchronous build for its grid's capacity.
void fill_list_job(void *out, nb_list *l, const int *excl_off, const int *excl_idx) {
    ListJob j{};
    j.a = make_search(l, excl_off, excl_idx);
    j.a.jcount = (int *)l->jcount.p;
    j.a.jrank = (int *)l->jrank.p;
    j.a.parts = l->resv_parts;
    j.a.entries = (nb_jentry *)l->entries.p;
    j.a.keys = nullptr;
    j.f = make_finish(l, l->resv_nci * l->resv_parts, l->resv_parts);
    std::memcpy(out, &j, sizeof j);
}

void list_job_blocks(const nb_list *l, int *blocks_per_stage) {
    const long nreg = (long)l->resv_nci * l->resv_parts;
    blocks_per_stage[LS_SEARCH] = (int)((nreg + 3) / 4);
}

int launch_pairlist_batch(hipStream_t st, int m, int nn, const void *jobs, const int *off, int n_rep,
                          const int *total) {
    const ListJob *J = (const ListJob *)jobs;
    const int nb = total[LS_SEARCH];
    if (m == 4 && nn == 4) kb_search<4, 4><<<nb, 256, 0, st>>>(J, off, n_rep);
    else if (m == 4 && nn == 8) kb_search<4, 8><<<nb, 256, 0, st>>>(J, off, n_rep);
    else if (m == 8 && nn == 4) kb_search<8, 4><<<nb, 256, 0, st>>>(J, off, n_rep);
    else kb_search<8, 8><<<nb, 256, 0, st>>>(J, off, n_rep);
    kb_finish<<<2 * n_rep, 1024, 0, st>>>(J);
    kb_items_rows<<<nb, 256, 0, st>>>(J, off, n_rep);
    MXN_HIP(hipGetLastError());
    return NB_OK;
}

constexpr int kSmallItems = 8192;

int launch_pairlist(nb_list *l, const int *excl_off, const int *excl_idx, bool sync, bool by_distance) {
    const nb_grid *g = l->grid;
    nb_ctx *ctx = l->ctx;
    hipStream_t st = ctx->stream;
    const int nci_cap = g->slots_cap / g->m;
    SearchArgs a = make_search(l, excl_off, excl_idx);
    // A synchronous build (also the first, and any after the grid's capacity
    // or cluster shape changed) counts the entries and gives every (i-cluster, part) region the
    // largest count plus a quarter plus 8 (uniform, because a re-sort re-forms
    // the clusters, so a region's next occupant may have any count); later
    // builds search once and fill the regions.
    const bool reserve = sync || !reserved_for(l, g);
    int parts = l->resv_parts;
    if (reserve) {
        // parts per i-cluster: the largest power of two up to 8 that keeps about 6000
        // wavefronts or fewer (measured on MI355X: more parts only add per-part overhead
        // once the GPU holds that many latency-bound wavefronts)
        parts = ctx->search_parts;
        if (parts == 0) {
            const long nci = std::max(1, g->n / g->m);
            parts = 1;
            while (parts < kMaxSearchParts && nci * parts * 2 < 6000) parts *= 2;
        }
    }
    a.parts = parts;
    const int nregions = nci_cap * parts;
    const int nblocks = (int)(((long)nregions + 3) / 4);
    if (reserve) {
        if (g->m == 4 && g->nn == 4) run<4, 4>(l, a, false, nblocks, st);
        else if (g->m == 4 && g->nn == 8) run<4, 8>(l, a, false, nblocks, st);
        else if (g->m == 8 && g->nn == 4) run<8, 4>(l, a, false, nblocks, st);
        else run<8, 8>(l, a, false, nblocks, st);
        // the sums go straight to pinned host memory
        k_max_count<<<1, 1024, 0, st>>>((const int *)l->part_count.p, nregions, item_entries(g->nn), ctx->h_pinned);
        MXN_HIP(hipGetLastError());
        MXN_HIP(hipStreamSynchronize(st));
        const long mx = ctx->h_pinned[0];
        const long size = mx + mx / 4 + 8;
        if (size * nregions > (1L << 31) - 1) return fail(NB_ERR_OOM, "nb_pairlist_build: list larger than 2^31 entries");
        const long ce = size * nregions;
        const bool grows = ce > l->cap_entries;
        if (grows) {
            int rc = ensure(l->ctx, l->entries, (size_t)ce * sizeof(nb_jentry));
            if (rc) return rc;
            l->cap_entries = ce;
        }
        // Work items of one or two passes while every one of them finds a free wavefront slot (eight a SIMD): the
        // GPU is not filled, and a shorter chain per wavefront ends sooner.  One pass against four: 900 atoms 8x8
        // 12.1 against 15.8 us a call, 3000 (4x4) 20.1 against 21.6; 12 000 (8x4) two passes as four, one 6 %
        // slower (15 k items); 24 000 and more four.  (The capacity bound keeps lists of very uneven regions, and
        // so the scratch nb_forces_noalloc needs for them, as they were.)  A list whose entries fit the storage it
        // has keeps that storage, which captured force calls read: shorter items only where they fit it too.
        const int full = item_entries(g->nn);
        const auto items_cap = [&](int per) { return ce / per + nregions + 256; };   // count/per + 1 for each region
        l->per_item = full;
        l->est_items = l->full_items = ctx->h_pinned[1];
        for (int k = 2; k > 0 && !l->batched() && l->per_item == full; --k)
            if (ctx->h_pinned[3 + k] <= kSmallItems && ce / (full >> k) + nregions <= 8 * kSmallItems &&
                (grows || items_cap(full >> k) <= l->cap_items)) {
                l->per_item = full >> k;
                l->est_items = ctx->h_pinned[3 + k];
            }
        const long cit = items_cap(l->per_item);
        if (cit > l->cap_items) {
            int rc = ensure(l->ctx, l->items, (size_t)cit * sizeof(int4));
            if (rc) return rc;
            l->cap_items = cit;
        }
        // j-cluster view and force-call buffers for this capacity; the counters start cleared
        const long njc = g->slots_cap / g->nn;
        const long nsc = (long)kRankSets * rank_stride(njc);
        int rc = ensure(l->ctx, l->jcount, (size_t)nsc * 4);
        rc = rc ? rc : ensure(l->ctx, l->joff, joff_bytes(njc, nregions));
        rc = rc ? rc : ensure(l->ctx, l->jstart, (size_t)(njc + 1) * 4);
        rc = rc ? rc : ensure(l->ctx, l->jrank, (size_t)l->cap_entries * 4);
        // j-force rows (one per entry, 12 N bytes): the synchronous build's entries plus a quarter, not the regions'
        // capacity (about three times the entries); a later asynchronous build with more entries than that
        // latches NB_ERR_OVERFLOW like an outgrown region
        const long ent = ctx->h_pinned[2];
        const long rows = std::min(l->cap_entries, ent + ent / 4 + 1024);
        if (l->resv_nn != g->nn) l->cap_rows = 0;   // rows of another width
        if (rows > l->cap_rows) {
            rc = rc ? rc : ensure(l->ctx, l->fj, (size_t)rows * g->nn * 12);
            if (rc == NB_OK) l->cap_rows = rows;
        }
        rc = rc ? rc : ensure(l->ctx, l->fi, (size_t)l->cap_items * g->m * 16);
        if (rc) return rc;
        k_reserve<<<(nregions + 256) / 256, 256, 0, st>>>(nregions, (int)size, (int *)l->part_start.p, (int)nsc,
                                                          (int *)l->jcount.p, (int *)l->totals.p);
        l->resv_parts = parts;
        l->resv_nci = nci_cap;
        l->resv_m = g->m;
        l->resv_nn = g->nn;
        l->last_entries = ce;
        l->resv_size = size;
    }
    if (by_distance) {   // the fill pass writes canonical order and keys; the sort orders each region
        int rc = ensure(l->ctx, l->entries_canon, (size_t)l->cap_entries * sizeof(nb_jentry));
        if (rc) return rc;
        rc = ensure(l->ctx, l->keys, (size_t)l->cap_entries * sizeof(float));
        if (rc) return rc;
        rc = ensure(l->ctx, l->jrank_canon, (size_t)l->cap_entries * 4);
        if (rc) return rc;
    }
    a.entries = (nb_jentry *)(by_distance ? l->entries_canon.p : l->entries.p);
    a.keys = by_distance ? (float *)l->keys.p : nullptr;
    // the j-cluster counters and ranks (allocated by a reserving build)
    a.jcount = (int *)l->jcount.p;
    a.jrank = (int *)(by_distance ? l->jrank_canon.p : l->jrank.p);
    if (!a.jcount || !a.jrank || !l->jstart.p || !l->fj.p || !l->fi.p)
        return fail(NB_ERR_STATE, "nb_pairlist_build: j-cluster view buffers missing");
    if (g->m == 4 && g->nn == 4) run<4, 4>(l, a, true, nblocks, st);
    else if (g->m == 4 && g->nn == 8) run<4, 8>(l, a, true, nblocks, st);
    else if (g->m == 8 && g->nn == 4) run<8, 4>(l, a, true, nblocks, st);
    else run<8, 8>(l, a, true, nblocks, st);
    const FinishArgs f = make_finish(l, nregions, parts);
    finish_list(f, st);
    if (by_distance)
        k_sort_entries<<<nregions, 64, 0, st>>>((const int *)l->part_start.p, (const int *)l->part_count.p,
                                                (const nb_jentry *)l->entries_canon.p, (const float *)l->keys.p,
                                                (nb_jentry *)l->entries.p, (const int *)l->jrank_canon.p,
                                                (int *)l->jrank.p);
    finish_rows(f, st);
    l->sci_valid = false;
    MXN_HIP(hipGetLastError());
    return NB_OK;
}

int launch_full_items(nb_list *l) {
    if (!short_items(l)) return NB_OK;
    l->per_item = item_entries(l->grid->nn);   // capacities hold: fewer items of the same entries
    l->est_items = l->full_items;
    const int nregions = l->resv_nci * l->resv_parts;
    k_full_items<<<1, 1024, 0, l->ctx->stream>>>(nregions, l->per_item, (const int *)l->part_count.p,
                                                 (int *)l->part_istart.p, (int *)l->totals.p);
    k_items<<<(nregions + 255) / 256, 256, 0, l->ctx->stream>>>(
        nregions, l->resv_parts, l->per_item, (const int *)l->part_count.p, (const int *)l->part_start.p,
        (const int *)l->part_istart.p, l->cap_items, (int4 *)l->items.p);
    MXN_HIP(hipGetLastError());
    return NB_OK;
}

// i-clusters per super-cluster for a list (0: no super-cluster view): the
// largest of 8 and 4 (at most want, if nonzero) whose span of regions fits
// the LDS sort
int sci_size(const nb_list *l, int want) {
    const nb_grid *g = l->grid;
    if (!g || g->m != 8 || g->nn != 8 || l->resv_parts <= 0 || l->resv_size <= 0) return 0;
    if ((long)g->slots_cap / 8 >= (1L << 24)) return 0;   // j-cluster index in 24 key bits
    for (int S = 8; S >= 4; S >>= 1)
        if ((want == 0 || S <= want) && (long)S * l->resv_parts * l->resv_size <= kSciKeys) return S;
    return 0;
}

// Build the super-cluster view of l (S i-clusters per super-cluster, per_item
// entries per work item) on the context stream: keys and entries, work
// items, the j-cluster rows of the entries.
int launch_sci_view(const nb_list *l, int S, int per_item) {
    const nb_grid *g = l->grid;
    hipStream_t st = l->ctx->stream;
    const int nregions = l->resv_nci * l->resv_parts;
    const int ngroups = (l->resv_nci + S - 1) / S;
    const long njc = g->slots_cap / g->nn;
    const long cap_items = l->cap_entries / per_item + ngroups + 256;
    const size_t old_jc = l->sci_jcount.bytes, old_tot = l->sci_totals.bytes;   // larger: new memory, wherever it lies
    int rc = ensure(l->ctx, l->sci_ent, (size_t)l->cap_entries * sizeof(int4));
    rc = rc ? rc : ensure(l->ctx, l->sci_mask, (size_t)l->cap_entries * S * sizeof(uint2));
    rc = rc ? rc : ensure(l->ctx, l->sci_count, (size_t)(ngroups + 1) * 4);
    rc = rc ? rc : ensure(l->ctx, l->sci_base, (size_t)(ngroups + 1) * 4);
    rc = rc ? rc : ensure(l->ctx, l->sci_istart, (size_t)(ngroups + 1) * 4);
    rc = rc ? rc : ensure(l->ctx, l->sci_items, (size_t)cap_items * sizeof(int4));
    rc = rc ? rc : ensure(l->ctx, l->sci_jcount, (size_t)(njc + 1) * 4);
    rc = rc ? rc : ensure(l->ctx, l->sci_jstart, (size_t)(njc + 1) * 4);
    rc = rc ? rc : ensure(l->ctx, l->sci_totals, 16);
    rc = rc ? rc : ensure(l->ctx, l->sci_fi, (size_t)cap_items * S * 8 * sizeof(float4));
    if (rc) return rc;
    if (l->sci_jcount.bytes != old_jc || l->sci_njc != njc) {   // counters start cleared; the scan clears them after use
        clear_ints(l->sci_jcount.p, njc + 1, st);
        l->sci_njc = njc;
    }
    if (l->sci_totals.bytes != old_tot) clear_ints(l->sci_totals.p, 4, st);
    SciArgs a{};
    a.nslots = (const int *)g->nslots.p;
    a.totals = (const int *)l->totals.p;
    a.part_start = (const int *)l->part_start.p;
    a.part_count = (const int *)l->part_count.p;
    a.entries = (const nb_jentry *)l->entries.p;
    a.parts = l->resv_parts;
    a.nregions = nregions;
    a.S = S;
    a.ngroups = ngroups;
    a.ent = (int4 *)l->sci_ent.p;
    a.mask = (uint2 *)l->sci_mask.p;
    a.count = (int *)l->sci_count.p;
    a.base = (int *)l->sci_base.p;
    a.jcount = (int *)l->sci_jcount.p;
    int *tot = (int *)l->sci_totals.p;
    k_sci_view<<<ngroups, 256, 0, st>>>(a);
    // rows: a super-cluster entry stands for one or more of the list's entries, which fit l's rows
    FinishArgs f{};
    f.nregions = ngroups;
    f.per_item = per_item;
    f.part_count = a.count;
    f.part_istart = (int *)l->sci_istart.p;
    f.cap_items = cap_items;
    f.cap_rows = l->cap_rows;
    f.totals = tot;
    f.flags = l->ctx->d_flags;
    f.jcount = a.jcount;
    f.jstart = (int *)l->sci_jstart.p;
    f.njc = (int)njc;
    f.nsets = 1;
    f.jstride = (int)njc;
    k_finish<<<2, 1024, 0, st>>>(f);
    k_items<<<(ngroups + 255) / 256, 256, 0, st>>>(ngroups, 1, per_item, a.count, a.base,
                                                  (const int *)l->sci_istart.p, cap_items, (int4 *)l->sci_items.p);
    const int nb = (int)std::max<long>(1, std::min<long>((cap_items + 3) / 4, kJposBlocks));
    k_sci_rows<<<nb, 256, 0, st>>>(tot, (const int4 *)l->sci_items.p, a.ent, (const int *)l->sci_jstart.p);
    MXN_HIP(hipGetLastError());
    l->sci_cap_items = cap_items;
    l->sci_S = S;
    l->sci_per_item = per_item;
    l->sci_valid = true;
    return NB_OK;
}

int launch_prune(nb_list *in, const nb_list *outer, float r) {
    const nb_grid *g = outer->grid;
    nb_ctx *ctx = in->ctx;
    hipStream_t st = ctx->stream;
    const int nregions = outer->resv_nci * outer->resv_parts;
    // the outer list's layout, with buffers of its capacity; new counters start cleared
    const long njc = g->slots_cap / g->nn;
    const size_t nreg = (size_t)outer->resv_nci * kMaxSearchParts + 1;
    const size_t old_jc = in->jcount.bytes, old_tot = in->totals.bytes;   // larger: new memory, wherever it lies
    int rc = ensure(in->ctx, in->part_count, nreg * 4);
    rc = rc ? rc : ensure(in->ctx, in->part_start, nreg * 4);
    rc = rc ? rc : ensure(in->ctx, in->part_istart, nreg * 4);
    rc = rc ? rc : ensure(in->ctx, in->totals, 16);
    rc = rc ? rc : ensure(in->ctx, in->entries, (size_t)outer->cap_entries * sizeof(nb_jentry));
    rc = rc ? rc : ensure(in->ctx, in->items, (size_t)outer->cap_items * sizeof(int4));
    const long nsc = (long)kRankSets * rank_stride(njc);
    rc = rc ? rc : ensure(in->ctx, in->jcount, (size_t)nsc * 4);
    rc = rc ? rc : ensure(in->ctx, in->joff, joff_bytes(njc, nregions));
    rc = rc ? rc : ensure(in->ctx, in->jstart, (size_t)(njc + 1) * 4);
    rc = rc ? rc : ensure(in->ctx, in->jrank, (size_t)outer->cap_entries * 4);
    rc = rc ? rc : ensure(in->ctx, in->fj, (size_t)outer->cap_rows * g->nn * 12);
    rc = rc ? rc : ensure(in->ctx, in->fi, (size_t)outer->cap_items * g->m * 16);
    if (rc) return rc;
    if (in->jcount.bytes != old_jc || in->resv_nci != outer->resv_nci)
        clear_ints(in->jcount.p, nsc, st);
    if (in->totals.bytes != old_tot) clear_ints(in->totals.p, 4, st);
    in->grid = g;
    in->grid_generation = outer->grid_generation;
    in->rlist = r;
    in->rbb = outer->rbb;
    in->cap_entries = outer->cap_entries;
    in->cap_items = outer->cap_items;
    in->resv_parts = outer->resv_parts;
    in->resv_nci = outer->resv_nci;
    in->resv_m = outer->resv_m;
    in->resv_nn = outer->resv_nn;
    in->last_entries = outer->last_entries;
    in->per_item = outer->per_item;
    in->est_items = outer->est_items;
    in->full_items = outer->full_items;
    in->cap_rows = outer->cap_rows;
    in->resv_size = outer->resv_size;
    in->sci_valid = false;
    MXN_HIP(hipMemcpyAsync(in->part_start.p, outer->part_start.p, (size_t)(nregions + 1) * 4, hipMemcpyDeviceToDevice,
                           st));
    PruneArgs a{};
    a.nslots = (const int *)g->nslots.p;
    a.xs_now = (const float4 *)g->xs_now.p;
    a.bbi_lo = (const float4 *)g->bbi_lo.p;
    a.bbj_lo = (const float4 *)(g->nn == g->m ? g->bbi_lo.p : g->bbj_lo.p);
    a.part_start = (const int *)outer->part_start.p;
    a.part_count_in = (const int *)outer->part_count.p;
    a.totals_in = (const int *)outer->totals.p;
    a.in = (const nb_jentry *)outer->entries.p;
    a.part_count = (int *)in->part_count.p;
    a.out = (nb_jentry *)in->entries.p;
    a.jcount = (int *)in->jcount.p;
    a.jrank = (int *)in->jrank.p;
    a.region_overflow = (int *)in->totals.p + 3;
    a.Lx = g->Lf[0]; a.Ly = g->Lf[1]; a.Lz = g->Lf[2];
    volatile float r2 = r * r;
    a.r2 = r2;
    a.nregions = nregions;
    a.parts = outer->resv_parts;
    a.jstride = rank_stride(njc);
    const int nb = (nregions + 3) / 4;
    if (g->m == 4 && g->nn == 4) k_prune<4, 4><<<nb, 256, 0, st>>>(a);
    else if (g->m == 4 && g->nn == 8) k_prune<4, 8><<<nb, 256, 0, st>>>(a);
    else if (g->m == 8 && g->nn == 4) k_prune<8, 4><<<nb, 256, 0, st>>>(a);
    else k_prune<8, 8><<<nb, 256, 0, st>>>(a);
    const FinishArgs f = make_finish(in, nregions, outer->resv_parts);
    finish_list(f, st);
    finish_rows(f, st);
    MXN_HIP(hipGetLastError());
    return NB_OK;
}

}  // namespace mxn
