// kernels_analysis.hip -- on-device radial distribution histogram and
// mean-square displacement.
//
// This translation unit is compiled without floating-point contraction so that
// the pair distance of the histogram is evaluated exactly as the definition
// reads: separations in binary64, minimum image by one +-L correction when
// the separation exceeds L/2 (the branch form of Sec. III.D),
// r^2 = (dx dx + dy dy) + dz dz, r = sqrt(r^2) (IEEE, correctly rounded),
// bin = int(r / dr) by a true division (Sec. VI.A.1).  The counts are then
// identical to those of any other IEEE evaluation of the same definition.
// (Most pairs are far enough from a bin's edge that a distance with a known
// error bound gives the same bin; the definition decides the others.)
#include "common_dev.hpp"

#include <algorithm>

namespace kamd {

// RDF grid: per replica nc^3 cells (a planar system: one layer of nc^2) of
// edge L/nc >= n_bins*dr, or >= n_bins*dr/2 where such cells still hold
// several particles; both particle types together.  The grid of replica r is
// rdf_grid[r] = {nc, first cell, cells}, chosen on the device (k_rdf_setup),
// so that a measurement needs no host round trip.
// Counting sort into rdf_pos (replica-relative positions, w = type + 2*cell).

// One block: the grid of every replica for the histogram range r_max, and
// how its histogram is split over blocks.  Cells as wide as r_max, or half as
// wide where such cells would still hold six particles or more on average; at
// most 2 n + 64 cells per replica (wider cells stay correct, they only add
// candidates), so that every grid fits the capacity the workspace reserves
// (2 n_total + 64 n_rep cells).
//
// A replica gets its share (by particles) of RDF_BLOCKS histogram blocks.
// Each owns a partial histogram in the workspace (9 n doubles of staging,
// 3 n / n_bins histograms) which a last kernel adds up; where fewer than the
// share fit, up to RDF_ATOMIC_BLOCKS blocks add to the result by atomics.
// The work of a replica is cut into items of RDF_THREADS particles x a range
// of stencil cells, about RDF_ITEMS per block, which the blocks take from a
// ticket counter: with one block per 256 particles the 32,000-particle system
// to half its box had 125 blocks of very uneven work for 256 compute units.
constexpr int RDF_THREADS = 512;
constexpr int RDF_BLOCKS = 1024;        // four per CU, 8 wavefronts each
constexpr int RDF_ATOMIC_BLOCKS = 256;
constexpr int RDF_ITEMS = 8;
constexpr int RDF_SETUP_THREADS = 256;
constexpr int RDF_ATOMICS = 1, RDF_NONFINITE = 2;  // bits of rdf_grid[r].w
constexpr int64_t RDF_ITEM_CANDIDATES = (int64_t)1 << 21;  // per thread and item: keeps 32-bit block counts exact

__device__ inline int rdf_reach(double rmax, int nc, double L) { return rmax * nc > L * (1.0 + 1e-12) ? 2 : 1; }

__device__ inline int rdf_units(int nc, int reach, int dim)  // stencil cells per particle
{
    const int noff = min(nc, 2 * reach + 1);
    return dim == 2 ? noff * noff : noff * noff * noff;
}

__global__ __launch_bounds__(RDF_SETUP_THREADS) void k_rdf_setup(Dev d, double rmax, int nbins)
{
    __shared__ int2 part[RDF_SETUP_THREADS];
    const bool planar = d.dim == 2;
    const int cap = planar ? 4096 : 256;
    auto cells = [&](int64_t k) { return planar ? k * k : k * k * k; };
    int2 carry = make_int2(0, 0);  // cells and blocks of the replicas before this chunk
    for (int r0 = 0; r0 < d.nrep; r0 += RDF_SETUP_THREADS) {
        const int r = r0 + threadIdx.x;
        int nc = 0, ncell = 0, nblk = 0, nsplit = 0, atomics = 0;
        if (r < d.nrep) {
            const RepInfo &R = d.rep[r];
            const double L = R.L;
            const double hr = 0.5 * rmax;
            const double per_cell = planar ? R.n / (L * L) * (hr * hr) : R.n / (L * L * L) * (hr * hr * hr);
            const double per_range = per_cell >= 6.0 ? 2.0 : 1.0;
            nc = (int)fmax(1.0, fmin(floor(per_range * L / rmax), (double)cap));
            const int64_t lim = 2 * (int64_t)R.n + 64;
            int nmax = (int)floor(planar ? sqrt((double)lim) : cbrt((double)lim));
            while (cells(nmax + 1) <= lim) ++nmax;
            while (nmax > 1 && cells(nmax) > lim) --nmax;
            nc = max(1, min(nc, nmax));
            ncell = (int)cells(nc);
            const int iblk = (R.n + RDF_THREADS - 1) / RDF_THREADS;
            const int units = rdf_units(nc, rdf_reach(rmax, nc, L), d.dim);
            const int share = (int)(((int64_t)RDF_BLOCKS * R.n + d.n_total - 1) / d.n_total);
            const int fit = (int)min((int64_t)share, 3 * (int64_t)R.n / nbins);
            atomics = fit < min(share, RDF_ATOMIC_BLOCKS) ? RDF_ATOMICS : 0;
            nblk = atomics ? min(share, RDF_ATOMIC_BLOCKS) : fit;
            const int64_t want = ((int64_t)RDF_ITEMS * nblk + iblk - 1) / iblk;
            const int64_t must = (R.n + RDF_ITEM_CANDIDATES - 1) / RDF_ITEM_CANDIDATES;
            nsplit = (int)min((int64_t)units, max(want, must));
            nblk = (int)min((int64_t)nblk, (int64_t)iblk * nsplit);
        }
        part[threadIdx.x] = make_int2(ncell, nblk);
        __syncthreads();
        for (int o = 1; o < RDF_SETUP_THREADS; o <<= 1) {
            int2 v = make_int2(0, 0);
            if ((int)threadIdx.x >= o) v = part[threadIdx.x - o];
            __syncthreads();
            part[threadIdx.x].x += v.x;
            part[threadIdx.x].y += v.y;
            __syncthreads();
        }
        if (r < d.nrep) {
            const int2 inc = part[threadIdx.x];
            d.rdf_grid[r] = make_int4(nc, carry.x + inc.x - ncell, ncell, atomics);
            d.rdf_plan[r] = make_int4(carry.y + inc.y - nblk, nblk, nsplit, 0);
        }
        carry.x += part[RDF_SETUP_THREADS - 1].x;
        carry.y += part[RDF_SETUP_THREADS - 1].y;
        __syncthreads();
    }
}

// Cell of every particle and its rank there.  The slots are sorted by list
// cell, so consecutive lanes mostly share an RDF cell: one atomic per run of
// such lanes (one per particle took 125 us for 32,000 particles in 64 cells).
__global__ __launch_bounds__(BLOCK) void k_rdf_assign(Dev d)
{
    const int w = blockIdx.x * WAVES_PER_BLOCK + (threadIdx.x >> 6);
    if (w >= d.nwaves) return;
    const SegInfo &S = d.seg[d.wave_seg[w]];
    const int lane = lane_id();
    const int s = w * WAVE + lane;
    const bool real = s - S.slot0 < S.n;
    int c = -1 - lane;  // distinct dummy for padding lanes
    if (real) {
        const int4 g = d.rdf_grid[S.rep];
        const int nc = g.x;
        const uint4 m = d.mirror[s];
        const int cz = d.dim == 2 ? 0 : fix_cell(m.z, nc);
        c = g.y + (cz * nc + fix_cell(m.y, nc)) * nc + fix_cell(m.x, nc);
        d.rdf_cell_of[s] = c;
    }
    int first;
    const int base = run_reserve(d.rdf_count, c, real, first);
    if (real) d.rdf_rank[s] = base + (lane - first);
}

// Exclusive scan per replica; rdf_start holds indices into rdf_pos (the
// replica's range begins at its caller offset).  A block scans RDF_SCAN_CHUNK
// cells, 8 consecutive ones per thread, after adding up the counts of all
// cells before them (cheap next to a serial pass per chunk: 54,872 cells took
// one block 51 us).
constexpr int RDF_SCAN_CHUNK = 8192;
__global__ __launch_bounds__(1024) void k_rdf_scan(Dev d)
{
    constexpr int PER = RDF_SCAN_CHUNK / 1024;
    __shared__ int wtot[1024 / WAVE], wbef[1024 / WAVE];
    const int rep = blockIdx.x;
    const int4 g = d.rdf_grid[rep];
    const int n = g.z, lane = lane_id(), wv = threadIdx.x >> 6;
    const int32_t *cnt = d.rdf_count + g.y;
    int32_t *out = d.rdf_start + g.y;
    for (int c0 = blockIdx.y * RDF_SCAN_CHUNK; c0 < n; c0 += gridDim.y * RDF_SCAN_CHUNK) {
        const int b = c0 + (int)threadIdx.x * PER;
        int v[PER], sum = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            v[k] = b + k < n ? cnt[b + k] : 0;
            sum += v[k];
        }
        int before = 0;
#pragma unroll 8
        for (int c = threadIdx.x; c < c0; c += 1024) before += cnt[c];
        before = wave_sum_i(before);
        int inc = sum;
#pragma unroll
        for (int o = 1; o < WAVE; o <<= 1) {
            const int u = __shfl_up(inc, o, WAVE);
            if (lane >= o) inc += u;
        }
        if (lane == WAVE - 1) wtot[wv] = inc;
        if (lane == 0) wbef[wv] = before;
        __syncthreads();
        int run = (int)d.rep[rep].caller_off + inc - sum;
        for (int k = 0; k < 1024 / WAVE; ++k) run += wbef[k] + (k < wv ? wtot[k] : 0);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (b + k < n) out[b + k] = run;
            run += v[k];
        }
        __syncthreads();
    }
}

// Particles in cell order: FP64 positions, and their fixed-point positions
// with type * nbins in the last word, so that the words of a pair add up to
// its histogram row (in the list builder's sorted mirror, which holds nothing
// between two rebuilds).
__global__ __launch_bounds__(BLOCK) void k_rdf_scatter(Dev d, int nbins)
{
    const int w = blockIdx.x * WAVES_PER_BLOCK + (threadIdx.x >> 6);
    if (w >= d.nwaves) return;
    const SegInfo &S = d.seg[d.wave_seg[w]];
    const int s = w * WAVE + lane_id();
    if (s - S.slot0 >= S.n) return;
    const int c = d.rdf_cell_of[s];
    const int t = d.rdf_start[c] + d.rdf_rank[s];
    const double x = d.x[s], y = d.y[s], z = d.z[s];
    d.rdf_pos[t] = make_double4(x, y, z, (double)(S.type + 2 * (c - d.rdf_grid[S.rep].y)));
    if (!(isfinite(x) && isfinite(y) && isfinite(z))) atomicOr(&d.rdf_grid[S.rep].w, RDF_NONFINITE);
    const uint4 m = d.mirror[s];
    d.smirror[t] = make_uint4(m.x, m.y, m.z, (uint32_t)(S.type * nbins));
}

__device__ inline double min_image_branch(double dd, double L, double half)
{
    if (dd > half) dd -= L;
    else if (dd < -half) dd += L;
    return dd;
}

__device__ inline double cell_gap(int o, int c, double cw, double u)
{
    // distance along one axis from coordinate u (in cell c) to cell c + o
    return o > 0 ? (c + o) * cw - u : (o < 0 ? u - (c + o + 1) * cw : 0.0);
}

// The bin by the definition, for a pair whose bin the fast distance leaves open.
__device__ inline int rdf_bin_exact(const double4 &pi, const double4 &pj, double L, double half, double dr)
{
    const double dx = min_image_branch(pi.x - pj.x, L, half);
    const double dy = min_image_branch(pi.y - pj.y, L, half);
    const double dz = min_image_branch(pi.z - pj.z, L, half);
    const double r = sqrt(dx * dx + dy * dy + dz * dz);
    return (int)(r / dr);
}

// Histogram blocks.  Each particle of an item visits the cells of its
// stencil (3 per axis with cells as wide as the histogram range r_max, 5 with
// cells half as wide) that come within r_max of it, row by row (the cells of a
// row are consecutive in the sorted order: one or two runs), and counts the
// partners with a larger index there, so every unordered pair is counted once:
// a partner within range lies in a cell within range of both particles, and
// the one with the smaller index counts it.  With the finer cells, leaving out
// the far ones takes the candidates per particle from 27 cells of edge r_max
// to about 10 of them.
//
// The pair's bin comes from an FP32 distance of the fixed-point positions
// (minimum image for free).  Its error in units of a bin is below eps: each
// component is exact to one fixed-point step h and rounded once (2^-24), the
// sum of squares adds at most 3 roundings, the square root, its scale and the
// product 4 more, in all under 6e-7 of r / dr <= n_bins, plus 2.5 h / dr.  A
// pair closer than eps to a bin's edge (a few in 10^4 at 200 bins) is binned
// by the FP64 definition instead, so every count is the definition's.  That
// takes the work per candidate from about 70 instructions (FP64 square root
// and division) to about 20.  (Histogram copies per wavefront measured the
// same: the LDS atomics do not bound it.)
//
// Bound by the vector ALU.  Measured (MI355X): 32,000 particles to half the
// box, 200 bins 10.7 -> 0.50 ms; 2^20 particles to 5.0, 200 bins 3.0 -> 1.03 ms
// (steps of 2 or 8 candidates: 0.56 / 0.49 and 1.15 / 1.19 ms).
__global__ __launch_bounds__(RDF_THREADS) void k_rdf_hist(Dev d, double dr, int nbins, uint64_t *hist, double *scratch)
{
    extern __shared__ uint32_t lh[];  // [3][nbins]
    __shared__ int item_s;
    const int row = 3 * nbins;
    int rep = 0;
    for (int hi = d.nrep - 1; rep < hi;) {  // the last replica whose first block is <= this one
        const int mid = (rep + hi + 1) >> 1;
        if (d.rdf_plan[mid].x <= (int)blockIdx.x) rep = mid;
        else hi = mid - 1;
    }
    const int4 plan = d.rdf_plan[rep];
    if ((int)blockIdx.x >= plan.x + plan.y) return;  // past the last replica's blocks
    for (int b = threadIdx.x; b < row; b += RDF_THREADS) lh[b] = 0u;
    const RepInfo &R = d.rep[rep];
    const int4 g = d.rdf_grid[rep];
    const int nc = g.x;
    const double L = R.L, half = 0.5 * R.L;
    const double rmax = nbins * dr;
    const int reach = rdf_reach(rmax, nc, L);
    const int noff = min(nc, 2 * reach + 1);
    const bool whole = nc < 2 * reach + 1;  // every cell along an axis is in the stencil
    const int nz = d.dim == 2 ? 1 : noff, oz0 = d.dim == 2 ? 0 : -reach;  // planar: one layer
    const int units = nz * noff * noff;
    const int i00 = (int)R.caller_off, iend = i00 + R.n;
    const int iblk = (R.n + RDF_THREADS - 1) / RDF_THREADS;
    const int nitem = iblk * plan.z;
    const double cw = L / nc;
    // pruning radius: the histogram range with a margin far above rounding
    const double rp = rmax * (1.0 + 1e-9) + 1e-12 * L;
    const double rp2 = rp * rp;
    const double h = R.fx_to_len;
    // every pair by the definition: a replica with a position that is not
    // finite, and bins about as narrow as the fixed-point step
    const double eps_d = 6e-7 * nbins + 2.5 * h / dr + 1e-6;
    const bool odd = (g.w & RDF_NONFINITE) != 0 || !(eps_d < 0.5);
    const float eps = (float)eps_d, scale = odd ? 0.0f : (float)(h / dr);
    const float sure = odd ? -1.0f : 0.5f - eps;  // |fraction - 1/2| up to which the bin is certain
    const float lim = odd ? INFINITY : (float)nbins + eps;
    uint64_t *part = reinterpret_cast<uint64_t *>(scratch) + 9 * (int64_t)R.caller_off +
                     (int64_t)((int)blockIdx.x - plan.x) * row;
    const bool atomics = (g.w & RDF_ATOMICS) != 0;
    bool fresh = true;  // nothing in the partial histogram yet
    // LDS counts into the block's partial histogram (or the result); AA and BB
    // pairs count twice
    auto flush = [&](bool last) {
        __syncthreads();
        for (int b = threadIdx.x; b < row; b += RDF_THREADS) {
            uint64_t v = lh[b];
            if (!last) lh[b] = 0u;
            if (b < nbins || b >= 2 * nbins) v *= 2;
            if (atomics) {
                if (v) atomicAdd((unsigned long long *)&hist[(size_t)rep * row + b], (unsigned long long)v);
            } else {
                part[b] = fresh ? v : part[b] + v;
            }
        }
        fresh = false;
        __syncthreads();
    };
    uint32_t tested = 0;  // candidates of this thread since the last flush
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) item_s = atomicAdd(&d.rdf_plan[rep].w, 1);
        const bool full = __syncthreads_or(tested > (uint32_t)RDF_ITEM_CANDIDATES) != 0;
        if (full) {
            flush(false);
            tested = 0;
        }
        const int item = item_s;
        if (item >= nitem) break;
        const int i = i00 + (item / plan.z) * RDF_THREADS + (int)threadIdx.x;
        const int part_i = item % plan.z;
        const int u0 = (int)((int64_t)units * part_i / plan.z), u1 = (int)((int64_t)units * (part_i + 1) / plan.z);
        if (i >= iend) continue;
        const double4 pi = d.rdf_pos[i];
        const uint4 mi = d.smirror[i];
        const int cl = (int)pi.w >> 1;
        const int cx = cl % nc, cy = (cl / nc) % nc, cz = cl / (nc * nc);
        uint32_t *hi = lh + mi.w;
        auto scan = [&](int st, int en) __attribute__((always_inline)) {
            for (int j = st; j < en; j += 4) {  // the mirror has spare entries past its end
                uint4 m[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) m[u] = d.smirror[j + u];
#pragma unroll
                for (int u = 0; u < 4; ++u) asm volatile("" : "+v"(m[u].w));  // or its load sinks into the branch below
                const int left = en - j;
                bool open[4], any = false;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float dx = (float)(int)(mi.x - m[u].x), dy = (float)(int)(mi.y - m[u].y),
                                dz = (float)(int)(mi.z - m[u].z);
                    const float t = __builtin_amdgcn_sqrtf(fmaf(dx, dx, fmaf(dy, dy, dz * dz))) * scale;
                    const bool in = t < lim && u < left;
                    open[u] = in && fabsf(__builtin_amdgcn_fractf(t) - 0.5f) > sure;
                    any |= open[u];
                    if (in && !open[u]) atomicAdd(&hi[m[u].w + (uint32_t)(int)t], 1u);
                }
                if (any) {
#pragma unroll 1
                    for (int u = 0; u < 4; ++u) {
                        if (!(u == 0 ? open[0] : u == 1 ? open[1] : u == 2 ? open[2] : open[3])) continue;
                        const double4 pj = d.rdf_pos[j + u];
                        const int bin = rdf_bin_exact(pi, pj, L, half, dr);
                        if (bin < nbins) atomicAdd(&hi[((int)pj.w & 1) * nbins + bin], 1u);
                    }
                }
            }
        };
        for (int ur = u0 / noff; ur * noff < u1; ++ur) {  // stencil rows of the item
            const int oz = oz0 + ur / noff, oy = -reach + ur % noff;
            const double gz = whole ? 0.0 : cell_gap(oz, cz, cw, pi.z), gy = whole ? 0.0 : cell_gap(oy, cy, cw, pi.y);
            const double g2 = gy * gy + gz * gz;
            if (g2 > rp2) continue;
            const int qz = (cz + oz + 2 * nc) % nc, qy = (cy + oy + 2 * nc) % nc;
            int xl = -reach + max(0, u0 - ur * noff), xr = -reach + min(noff, u1 - ur * noff) - 1;
            if (!whole) {
                while (xl <= xr) {
                    const double gx = cell_gap(xl, cx, cw, pi.x);
                    if (!(gx * gx + g2 > rp2)) break;
                    ++xl;
                }
                while (xr >= xl) {
                    const double gx = cell_gap(xr, cx, cw, pi.x);
                    if (!(gx * gx + g2 > rp2)) break;
                    --xr;
                }
            }
            if (xl > xr) continue;
            const int rowc = g.y + (qz * nc + qy) * nc;
            // the row's cells [a, b], unwrapped (fewer than nc of them): one
            // run, or two where they wrap around the box
            const int a = cx + xl, b = cx + xr;
            const int sh = b < 0 ? nc : (a >= nc ? -nc : 0);
            const int a0 = a + sh, b0 = b + sh;
            const bool wl = a0 < 0, wr = b0 >= nc;
            const int r0 = wl ? a0 + nc : a0, r1 = wl || wr ? nc - 1 : b0;
            int st = max(d.rdf_start[rowc + r0], i + 1), en = d.rdf_start[rowc + r1] + d.rdf_count[rowc + r1];
            int st2 = 0, en2 = 0;
            if (wl || wr) {
                const int e = wl ? b0 : b0 - nc;
                st2 = max(d.rdf_start[rowc], i + 1);
                en2 = d.rdf_start[rowc + e] + d.rdf_count[rowc + e];
            }
#pragma unroll 1
            for (int p = 0; p < 2; ++p) {
                scan(st, en);
                tested += (uint32_t)max(0, en - st);
                st = st2;
                en = en2;
            }
        }
    }
    flush(true);
}

// The partial histograms of every replica, added to the result: one block
// per replica and 64 bins, 16 partial histograms at a time.  The additions are
// atomic: another context may be adding to the same result on its own stream.
__global__ __launch_bounds__(1024) void k_rdf_reduce(Dev d, int nbins, uint64_t *hist, const double *scratch)
{
    __shared__ uint64_t red[16][WAVE];
    const int rep = blockIdx.x, row = 3 * nbins;
    const int b = blockIdx.y * WAVE + lane_id(), q = threadIdx.x >> 6;
    if (d.rdf_grid[rep].w & RDF_ATOMICS) return;
    const int nblk = d.rdf_plan[rep].y;
    const uint64_t *part = reinterpret_cast<const uint64_t *>(scratch) + 9 * (int64_t)d.rep[rep].caller_off;
    uint64_t v = 0;
    if (b < row) {
#pragma unroll 8
        for (int k = q; k < nblk; k += 16) v += part[(int64_t)k * row + b];
    }
    red[q][lane_id()] = v;
    __syncthreads();
    if (q == 0 && b < row) {
        for (int k = 1; k < 16; ++k) v += red[k][lane_id()];
        if (v) atomicAdd((unsigned long long *)&hist[(size_t)rep * row + b], (unsigned long long)v);
    }
}

// MSD: origin[slot][k][id] = unwrapped coordinate k (x + img L, Sec. VI.B.1).
__global__ __launch_bounds__(BLOCK) void k_msd_set(Dev d, int slot)
{
    const int w = blockIdx.x * WAVES_PER_BLOCK + (threadIdx.x >> 6);
    if (w >= d.nwaves) return;
    const SegInfo &S = d.seg[d.wave_seg[w]];
    const int s = w * WAVE + lane_id();
    if (s - S.slot0 >= S.n) return;
    const double L = d.rep[S.rep].L;
    const int np = d.npad_total;
    const int g = d.id[s];
    double *o = d.origin + (size_t)slot * 3 * d.n_total;
    o[g] = d.x[s] + (double)d.img[s] * L;
    o[d.n_total + g] = d.y[s] + (double)d.img[np + s] * L;
    o[2 * d.n_total + g] = d.z[s] + (double)d.img[2 * np + s] * L;
}

// Per-wave sum of |r_u - r_u(origin)|^2, stored in component `type` of the
// wave partials (a wave holds one type).
__global__ __launch_bounds__(BLOCK) void k_msd_measure(Dev d, int slot)
{
    const int w = blockIdx.x * WAVES_PER_BLOCK + (threadIdx.x >> 6);
    if (w >= d.nwaves) return;
    const SegInfo &S = d.seg[d.wave_seg[w]];
    const int s = w * WAVE + lane_id();
    double d2 = 0.0;
    if (s - S.slot0 < S.n) {
        const double L = d.rep[S.rep].L;
        const int np = d.npad_total;
        const int g = d.id[s];
        const double *o = d.origin + (size_t)slot * 3 * d.n_total;
        const double ux = d.x[s] + (double)d.img[s] * L - o[g];
        const double uy = d.y[s] + (double)d.img[np + s] * L - o[d.n_total + g];
        const double uz = d.z[s] + (double)d.img[2 * np + s] * L - o[2 * d.n_total + g];
        d2 = ux * ux + uy * uy + uz * uz;
    }
    d2 = wave_sum(d2);
    if (lane_id() == 0) {
        d.wred[4 * w + 0] = S.type == 0 ? d2 : 0.0;
        d.wred[4 * w + 1] = S.type == 1 ? d2 : 0.0;
    }
}

// Self part of the van Hove function: per replica and species, the histogram
// of |r_u - r_u(origin)| over particles, bin = int(r / dr) kept when < n_bins.
// Particle of slot s (replica and type of S) into the histogram h.
__device__ inline void vh_count(const Dev &d, const SegInfo &S, int s, int slot, double dr, int nbins, uint32_t *h)
{
    if (s - S.slot0 >= S.n) return;
    const double L = d.rep[S.rep].L;
    const int np = d.npad_total;
    const int g = d.id[s];
    const double *o = d.origin + (size_t)slot * 3 * d.n_total;
    const double dx = d.x[s] + (double)d.img[s] * L - o[g];
    const double dy = d.y[s] + (double)d.img[np + s] * L - o[d.n_total + g];
    const double dz = d.z[s] + (double)d.img[2 * np + s] * L - o[2 * d.n_total + g];
    const double r = sqrt(dx * dx + dy * dy + dz * dz);
    const int bin = (int)(r / dr);
    if (bin < nbins) atomicAdd(&h[bin], 1u);
}

// A block takes a run of consecutive waves (a wave holds one replica and one
// type) and counts into one u32 histogram in LDS, which it adds to the uint64
// result [n_rep][2][n_bins] whenever the replica or type changes and at the
// end.  Bound by those 64-bit atomics, which all go to the same few lines: one
// flush per 16 or more waves instead of one per wave took 262,147 particles
// with 200 bins from 76 to 13.5 us.
constexpr int VH_THREADS = 1024;
constexpr int VH_BLOCKS = 256;
__global__ __launch_bounds__(VH_THREADS) void k_van_hove(Dev d, int slot, double dr, int nbins, int per, uint64_t *hist)
{
    __shared__ uint32_t h[VH_MAX_BINS];
    constexpr int NW = VH_THREADS / WAVE;
    const int wv = threadIdx.x / WAVE, lane = lane_id();
    const int w0 = blockIdx.x * per, w1 = min(w0 + per, d.nwaves);
    for (int b = threadIdx.x; b < nbins; b += VH_THREADS) h[b] = 0u;
    __syncthreads();
    for (int w = w0; w < w1;) {  // block-uniform
        const SegInfo &S = d.seg[d.wave_seg[w]];
        const int e = min(w1, (S.slot0 + S.npad) / WAVE);  // this segment's waves of the block
        for (int q = w + wv; q < e; q += NW) vh_count(d, S, q * WAVE + lane, slot, dr, nbins, h);
        __syncthreads();
        uint64_t *out = hist + ((size_t)S.rep * 2 + S.type) * nbins;
        for (int b = threadIdx.x; b < nbins; b += VH_THREADS)
            if (h[b]) {
                atomicAdd((unsigned long long *)&out[b], (unsigned long long)h[b]);
                h[b] = 0u;
            }
        __syncthreads();
        w = e;
    }
}

// The same for small replicas, whose segments of a wave or a few the kernel
// above would take one after the other: all waves of a block at once, with a
// histogram in LDS for each segment that the block has waves of, at the place of
// its first one.
constexpr int VH_SMALL_WAVES = 8;
__global__ __launch_bounds__(VH_SMALL_WAVES * WAVE) void k_van_hove_small(Dev d, int slot, double dr, int nbins,
                                                                          uint64_t *hist)
{
    extern __shared__ uint32_t lh[];  // [VH_SMALL_WAVES][nbins]
    const int wv = threadIdx.x / WAVE, lane = lane_id();
    const int w0 = blockIdx.x * VH_SMALL_WAVES, w = w0 + wv;
    for (int b = lane; b < nbins; b += WAVE) lh[wv * nbins + b] = 0u;
    __syncthreads();
    const SegInfo &S = d.seg[d.wave_seg[min(w, d.nwaves - 1)]];
    const int first = max(S.slot0 / WAVE - w0, 0);  // of the segment's waves, in the block
    if (w < d.nwaves) vh_count(d, S, w * WAVE + lane, slot, dr, nbins, lh + first * nbins);
    __syncthreads();
    if (w >= d.nwaves || first != wv) return;
    uint64_t *out = hist + ((size_t)S.rep * 2 + S.type) * nbins;
    for (int b = lane; b < nbins; b += WAVE) {
        const uint32_t n = lh[wv * nbins + b];
        if (n) atomicAdd((unsigned long long *)&out[b], (unsigned long long)n);
    }
}

__global__ void k_msd_finish(Dev d, double *out)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= d.nrep) return;
    const RepInfo &R = d.rep[r];
    out[2 * r + 0] = R.na > 0 ? d.rsum[4 * r + 0] / (double)R.na : 0.0;
    out[2 * r + 1] = R.n - R.na > 0 ? d.rsum[4 * r + 1] / (double)(R.n - R.na) : 0.0;
}

static inline int nblk(const Dev &d) { return (d.nwaves + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK; }

hipError_t launch_rdf_prepare(const Dev &d, double rmax, int nbins, int max_n, hipStream_t s)
{
    hipLaunchKernelGGL(k_rdf_setup, dim3(1), dim3(RDF_SETUP_THREADS), 0, s, d, rmax, nbins);
    hipError_t e = launch_zero_i32(d.rdf_count, d.rdf_cells_cap, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_rdf_assign, dim3(nblk(d)), dim3(BLOCK), 0, s, d);
    const int chunks = (int)((2 * (int64_t)max_n + 64 + RDF_SCAN_CHUNK - 1) / RDF_SCAN_CHUNK);  // of the largest grid allowed
    hipLaunchKernelGGL(k_rdf_scan, dim3(d.nrep, std::min(chunks, 1024)), dim3(1024), 0, s, d);
    hipLaunchKernelGGL(k_rdf_scatter, dim3(nblk(d)), dim3(BLOCK), 0, s, d, nbins);
    return hipGetLastError();
}

hipError_t launch_rdf(const Dev &d, double dr, int nbins, uint64_t *hist, double *scratch, hipStream_t s)
{
    hipLaunchKernelGGL(k_rdf_hist, dim3(RDF_BLOCKS + d.nrep), dim3(RDF_THREADS), sizeof(uint32_t) * 3 * nbins, s, d, dr,
                       nbins, hist, scratch);
    hipLaunchKernelGGL(k_rdf_reduce, dim3(d.nrep, (3 * nbins + WAVE - 1) / WAVE), dim3(1024), 0, s, d, nbins, hist,
                       scratch);
    return hipGetLastError();
}

hipError_t launch_msd_set(const Dev &d, int slot, hipStream_t s)
{
    hipLaunchKernelGGL(k_msd_set, dim3(nblk(d)), dim3(BLOCK), 0, s, d, slot);
    return hipGetLastError();
}

hipError_t launch_msd_measure(const Dev &d, int slot, hipStream_t s)
{
    hipLaunchKernelGGL(k_msd_measure, dim3(nblk(d)), dim3(BLOCK), 0, s, d, slot);
    return hipGetLastError();
}

// By the mean number of waves per segment.  Measured (us per call, calls in a row,
// 200 bins, k_van_hove / small): 4096 replicas of 70 (1 wave) 36 / 7, 126 of 75 18 /
// 5, 64 of 1000 (8.5) 6 / 5, 512 of 1000 10 / 11, 2000 of 1000 35 / 30, 64 of 2000 (16)
// 5 / 5, 256 of 2000 9 / 12, 64 of 4000 (31) 8 / 9; one of 64,000 6 / 6.
constexpr int VH_SMALL_SEG = 12;
hipError_t launch_van_hove(const Dev &d, int slot, double dr, int nbins, uint64_t *hist, hipStream_t s)
{
    if (d.nwaves <= 2 * VH_SMALL_SEG * (int64_t)d.nrep) {
        hipLaunchKernelGGL(k_van_hove_small, dim3((d.nwaves + VH_SMALL_WAVES - 1) / VH_SMALL_WAVES),
                           dim3(VH_SMALL_WAVES * WAVE), sizeof(uint32_t) * VH_SMALL_WAVES * nbins, s, d, slot, dr, nbins,
                           hist);
    } else {
        constexpr int nw = VH_THREADS / WAVE;  // at least one pass of the block's wavefronts per block
        const int per = std::max(nw, (d.nwaves + VH_BLOCKS - 1) / VH_BLOCKS);
        hipLaunchKernelGGL(k_van_hove, dim3((d.nwaves + per - 1) / per), dim3(VH_THREADS), 0, s, d, slot, dr, nbins, per,
                           hist);
    }
    return hipGetLastError();
}

hipError_t launch_msd_finish(const Dev &d, double *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_msd_finish, dim3((d.nrep + 63) / 64), dim3(64), 0, s, d, out);
    return hipGetLastError();
}

}  // namespace kamd
