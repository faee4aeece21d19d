// Pair distance histogram over a cluster-pair list: the pair correlation
// function, which Sec. 1 names as a limited-range pair evaluation like the
// forces.  Sec. 2.3: when the list is built for every evaluation the particle
// prune is skipped (a list built from bounding boxes, rbb = rlist), and for
// interactions this cheap the kernel needs no cut-off conditional.
//
// Work items as in the force kernel: a wavefront takes entries of one
// i-cluster, a lane one j-particle of one entry, and loops over the M
// i-particles (scalar registers).  A pair below r_max is counted in a
// per-workgroup LDS histogram (rows by ordered type pair, folded onto the
// unordered one at the end); integer sums, so the result is exact.
//
// The bin is decided in FP32 from r2 alone: e_k = (float)((k dr)^2) in FP64,
// bin k the largest with e_k <= r2.  t = sqrt(r2)/dr from the hardware square
// root is within 2.4e-7 t of the exact quotient, and an edge within 3e-8 k of k,
// so the integer part of t is that bin unless t lies within `near` of an
// integer; only then are the edges themselves read.  r2 is formed as the
// search forms its particle test (j moved back by the entry's image shift,
// separately rounded operations; this file is compiled with
// -ffp-contract=off).
//
// Bound: 26 vector instructions per listed pair (64 with an IEEE square root
// and both edges read for every pair), whose issue takes 33 to 49 of the
// 96 000-atom frame's 57 us (113 us before), beside the LDS atomics, one a
// counted pair; and the workgroups' histograms: flushed with global atomics by
// 768 workgroups they took 25 us, written to scratch and summed by a second
// launch 5 us.
#include <cmath>
#include <type_traits>
#include <vector>

#include "internal.h"

namespace {

struct RdfArgs {
    const float4 *xs_now;   // slot positions at the evaluated time (gathered)
    const int *type_s;      // -1 for dummy slots
    const int4 *items;
    const nb_jentry *entries;
    const int *totals;      // [2]: usable work items
    const float4 *shiftvec;
    const float *edge;      // nbins + 1 squared bin edges
    unsigned long long *hist;
    unsigned *parts;        // histogram of each workgroup (null: counts go to hist at once)
    int nbins, nt, skip_excl;
    float inv_dr, near;
};

constexpr int kRdfGroups = 768;   // most workgroups of a call
constexpr int kRdfWaves = 8;   // wavefronts per workgroup (three to a CU fit: scalar registers)

// The exact bin of a pair whose t lies next to an integer.
__device__ inline int edge_bin(const float *edge, int nbins, float inv_dr, float r2) {
    int bin = (int)(sqrtf(r2) * inv_dr);   // also for an r2 the hardware root flushes to zero
    bin = bin > nbins - 1 ? nbins - 1 : bin;
    bin -= bin > 0 && edge[bin] > r2 ? 1 : 0;
    bin += (bin + 1 < nbins && !(edge[bin + 1] > r2)) ? 1 : 0;
    return bin;
}

// Counts of bin t of the ordered type pair (p, q) go to the pair (min, max).
__device__ inline void add_count(const RdfArgs &a, int t, unsigned long long c) {
    const int row = t / a.nbins, p = row / a.nt, q = row % a.nt;
    if (c) atomicAdd(a.hist + (p <= q ? t : (q * a.nt + p) * a.nbins + t % a.nbins), c);
}

template <int M, int N>
__global__ __launch_bounds__(64 * kRdfWaves) void k_rdf(RdfArgs a) {
    constexpr int B = 64 / N;
    constexpr unsigned FULL = (1u << M) - 1u;
    extern __shared__ float4 smem[];
    float4 *svec = smem;                                         // 27 image shift vectors
    float *edge = reinterpret_cast<float *>(smem + 32);          // nbins + 1
    unsigned *h = reinterpret_cast<unsigned *>(edge + a.nbins + 1);
    const int nh = a.nt * a.nt * a.nbins;
    for (int t = threadIdx.x; t < 27; t += blockDim.x) svec[t] = a.shiftvec[t];
    for (int t = threadIdx.x; t <= a.nbins; t += blockDim.x) edge[t] = a.edge[t];
    for (int t = threadIdx.x; t < nh; t += blockDim.x) h[t] = 0u;
    __syncthreads();
    const float r2max = edge[a.nbins];
    const long total = a.totals[2];
    const int lane = threadIdx.x & 63, jb = lane % N, eo = lane / N;
    for (long item = (long)blockIdx.x * kRdfWaves + (threadIdx.x >> 6); item < total;
         item += (long)gridDim.x * kRdfWaves) {
        const int4 it = a.items[item];
        const int ci = __builtin_amdgcn_readfirstlane(it.x);
        const int js = __builtin_amdgcn_readfirstlane(it.y);
        const int je = __builtin_amdgcn_readfirstlane(it.z);
        float xi[M], yi[M], zi[M];
        int ti[M];   // histogram row of the i-particle's type
        unsigned ireal = 0;
#pragma unroll
        for (int k = 0; k < M; ++k) {
            const float4 p = a.xs_now[ci * M + k];
            xi[k] = p.x; yi[k] = p.y; zi[k] = p.z;
            const int t = a.type_s[ci * M + k];
            ireal |= (t >= 0 ? 1u : 0u) << k;
            ti[k] = (t < 0 ? 0 : (t >= a.nt ? a.nt - 1 : t)) * a.nt * a.nbins;
        }
        ireal = __builtin_amdgcn_readfirstlane(ireal);
        for (int e0 = js; e0 < je; e0 += B) {
            const int e = e0 + eo;
            const bool valid = e < je;
            const nb_jentry en = a.entries[valid ? e : e0];
            const int jslot = en.cj * N + jb;
            const float4 pj = a.xs_now[jslot];
            const int tjr = a.type_s[jslot];
            const int tj = (tjr < 0 ? 0 : (tjr >= a.nt ? a.nt - 1 : tjr)) * a.nbins;
            const float4 sv = svec[en.shift];
            const float xj = pj.x - sv.x, yj = pj.y - sv.y, zj = pj.z - sv.z;
            const unsigned long long m64 = ((unsigned long long)en.mhi << 32) | en.mlo;
            const unsigned mb = (unsigned)(m64 >> (jb * M)) & FULL;
            unsigned act = ireal;
            if (en.shift == 13) {   // self or overlapping cluster pair: only slot(i) < slot(j)
                const int t = jslot - ci * M;
                act &= t >= M ? FULL : (t <= 0 ? 0u : (1u << t) - 1u);
            }
            if (a.skip_excl) act &= mb;
            if (!valid || tjr < 0) act = 0u;
            const float lim = act ? r2max : -1.0f;
            auto pairs = [&](auto whole) {   // whole: every lane takes all M i-particles or none
#pragma unroll
                for (int k = 0; k < M; ++k) {
                    const float dx = xi[k] - xj, dy = yi[k] - yj, dz = zi[k] - zj;
                    const float r2 = (dx * dx + dy * dy) + dz * dz;
                    if (r2 < lim && (whole || ((act >> k) & 1u))) {
                        const float t = __builtin_amdgcn_sqrtf(r2) * a.inv_dr;
                        int bin = (int)t;
                        if (fabsf(t - rintf(t)) < a.near) bin = edge_bin(edge, a.nbins, a.inv_dr, r2);
                        atomicAdd(h + ti[k] + tj + bin, 1u);
                    }
                }
            };
            if (__ballot(act != 0u && act != FULL) == 0ull) pairs(std::true_type{});
            else pairs(std::false_type{});
        }
    }
    __syncthreads();
    if (a.parts) {
        unsigned *row = a.parts + (size_t)blockIdx.x * nh;
        for (int t = threadIdx.x; t < nh; t += blockDim.x) row[t] = h[t];
    } else {
        for (int t = threadIdx.x; t < nh; t += blockDim.x) add_count(a, t, h[t]);
    }
}

// Sum of the workgroups' histograms: a workgroup takes 64 bins (x) of an eighth of the rows (y), each of its 16
// wavefronts every 16th of those rows.
constexpr int kRdfShares = 8;
__global__ __launch_bounds__(1024) void k_rdf_sum(RdfArgs a, int nparts) {
    __shared__ unsigned long long red[16][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nh = a.nt * a.nt * a.nbins, t = blockIdx.x * 64 + lane;
    unsigned long long s = 0;
    if (t < nh) {
#pragma unroll 8
        for (int k = blockIdx.y * 16 + w; k < nparts; k += 16 * kRdfShares) s += a.parts[(size_t)k * nh + t];
    }
    red[w][lane] = s;
    __syncthreads();
    if (w > 0 || t >= nh) return;
    for (int k = 1; k < 16; ++k) s += red[k][lane];
    add_count(a, t, s);
}

}  // namespace

namespace mxn {

size_t rdf_lds_bytes(int nbins, int nt) { return 32 * 16 + (size_t)(nbins + 1) * 4 + (size_t)nt * nt * nbins * 4; }

int launch_rdf(nb_ctx *ctx, const nb_grid *g, const nb_list *l, float r_max, int nbins, int nt, int skip_excl,
               unsigned long long *hist) {
    hipStream_t st = ctx->stream;
    // squared bin edges e_k = (float)((k dr)^2), dr = r_max / nbins, in FP64 (rebuilt when they change)
    if (!ctx->rdf_edge.p || ctx->rdf_rmax != r_max || ctx->rdf_nbins != nbins) {
        std::vector<float> e((size_t)nbins + 1);
        const double dr = (double)r_max / nbins;
        for (int k = 0; k <= nbins; ++k) e[(size_t)k] = (float)((k * dr) * (k * dr));
        int rc = ensure(ctx, ctx->rdf_edge, e.size() * sizeof(float));
        if (rc) return rc;
        MXN_HIP(hipMemcpyAsync(ctx->rdf_edge.p, e.data(), e.size() * sizeof(float), hipMemcpyHostToDevice, st));
        MXN_HIP(hipStreamSynchronize(st));   // e is released on return
        ctx->rdf_rmax = r_max;
        ctx->rdf_nbins = nbins;
    }
    RdfArgs a{};
    a.xs_now = (const float4 *)g->xs_now.p;
    a.type_s = (const int *)g->type_s.p;
    a.items = (const int4 *)l->items.p;
    a.entries = (const nb_jentry *)l->entries.p;
    a.totals = (const int *)l->totals.p;
    a.shiftvec = (const float4 *)g->shiftvec.p;
    a.edge = (const float *)ctx->rdf_edge.p;
    a.hist = hist;
    a.nbins = nbins;
    a.nt = nt;
    a.skip_excl = skip_excl;
    a.inv_dr = (float)((double)nbins / (double)r_max);
    a.near = 4e-7f * (float)(nbins + 1);   // t <= nbins up to rounding; relative errors: root 1.2e-7, 1/dr and the
                                           // product 6e-8 each, an edge 3e-8
    // persistent workgroups, three to a CU; each flushes its histogram once
    const long need = (std::min(l->cap_items, l->est_items + l->est_items / 4 + 256) + kRdfWaves - 1) / kRdfWaves;
    const int nb = (int)std::max(1L, std::min(need, (long)kRdfGroups));
    const size_t lds = rdf_lds_bytes(nbins, nt);
    std::lock_guard<std::mutex> lock(ctx->rdf_parts.mu);
    // Workgroups' counts added with atomics take 26 to 45 ns a workgroup, one after the other (more the more bins
    // are counted); written and summed by a second launch, 5 us and 2.7 ps for each counter of each workgroup.
    // 900 atoms 8x8 (208 workgroups): 800 counters 12.3 us with atomics and 10.3 summed, 12 000 counters 14.0 and
    // 19.0; 3000 atoms (726) 30.2 and 12.5, 38.2 and 32.0; 96 000 atoms (768) 66.8 and 50.0, 115.4 and 86.9.
    const long counters = (long)nt * nt * nbins;
    if ((double)nb * (42e-3 - 2.7e-6 * (double)counters) > 5.0)
        a.parts = (unsigned *)ctx->rdf_parts.get(ctx, (size_t)counters * kRdfGroups * sizeof(unsigned));
    if (g->m == 4 && g->nn == 4) k_rdf<4, 4><<<nb, 64 * kRdfWaves, lds, st>>>(a);
    else if (g->m == 4 && g->nn == 8) k_rdf<4, 8><<<nb, 64 * kRdfWaves, lds, st>>>(a);
    else if (g->m == 8 && g->nn == 4) k_rdf<8, 4><<<nb, 64 * kRdfWaves, lds, st>>>(a);
    else k_rdf<8, 8><<<nb, 64 * kRdfWaves, lds, st>>>(a);
    if (a.parts) k_rdf_sum<<<dim3((nt * nt * nbins + 63) / 64, kRdfShares), 1024, 0, st>>>(a, nb);
    MXN_HIP(hipGetLastError());
    return NB_OK;
}

}  // namespace mxn
