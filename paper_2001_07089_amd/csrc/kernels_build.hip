// kernels_build.hip -- cell binning, stable counting sort of the internal
// particle order and the neighbour lists.
//
// The paper evaluates forces by a double loop over all pairs and names the
// neighbour list as the optimisation it leaves out (end of Sec. III.E); its
// LAMMPS runs use a binned list with a skin and a rebuild check every step
// (Sec. IV, "neighbor 0.3 bin" with "check yes").  Here each replica has a
// cubic grid of nc^3 cells of edge L/nc >= (largest cutoff + skin)/cell_div
// (a planar system, whose particles all sit at z = 0, a single layer of nc^2),
// and each particle keeps the list of all partners within r_c(ab) + skin,
// rebuilt when some particle of the replica has moved more than skin/2 since
// the last build (so no pair can enter the cutoff unseen).
//
// A rebuild runs as a few kernels, all launched on every step, so that the
// decision stays on the device and the step loop can be captured in a HIP
// graph:
//   rb_gate       one block: rebuild flag of every replica (rebuild_flag),
//                 worklist of the waves of the replicas that rebuild (several
//                 replicas only: a single one's flag is decided in rb_assign)
//   rb_assign     per listed wave: sub-cell index of its particles; runs of
//                 lanes that share a sub-cell are counted and linked
//   rb_scan_sum   per chunk of a segment's cells (segments of many chunks
//                 only): the particles of the chunk
//   rb_scan       per chunk of a segment's cells: exclusive scan of the
//                 counters -> cell ranges
//   rb_sortgather per listed particle: its rank by previous slot inside its
//                 sub-cell (a stable sort: the result does not depend on
//                 atomic timing), its state gathered into the scratch
//                 arrays, the counter cleared
//   rb_list       per listed wave: copy its state back, record the build
//                 position, write its neighbour list
// Every kernel returns at once when the worklist is empty; the scan also
// skips replicas whose flag is clear.  Plans of small replicas only run
// everything before rb_list as one kernel (k_rb_sort_small; in batches of many
// replicas after the gate).
#include <climits>

#include "common_dev.hpp"

namespace kamd {

// The gate: one block evaluates the rebuild flag of every replica and writes
// the worklist of the waves of the replicas that rebuild (rb_wlist), replica
// by replica in slot order, with their count in rb_any[0].  On the (most
// frequent) steps without a rebuild every later kernel of the chain exits
// after one load; on a step where a few replicas of a batch rebuild, the
// per-wave kernels spread just their work over the whole device.
constexpr int GATE_THREADS = 1024;
// Replicas come along with those that must rebuild (rebuild_flag) while the
// latter have fewer wavefronts than this: four per SIMD of 256 CUs.
constexpr int LIST_ALONG_WAVES = 4096;

// Rebuild decision of replica r for the running step.  A replica must
// rebuild when forced or when a particle has moved more than half its skin
// since the last build.  On a step where the replicas that must rebuild are
// too few to fill the device (the gate decides, rb_any[1]), the others whose
// largest move has passed REBUILD_ALONG of that come along (`along`): the
// rebuilds of a batch's replicas then fall on fewer steps, whose list builds
// would otherwise each run at the latency of a lone wavefront (an early
// rebuild is always valid).  Every kernel of the rebuild chain evaluates it
// identically: nothing it reads changes before the force kernel of the same
// step closes the check.
constexpr double REBUILD_ALONG = 0.8;
__device__ inline bool rebuild_flag(const Dev &d, int r, bool along)
{
    const double m2 = (double)__uint_as_float(d.maxdisp[DISP_STRIDE * r]), t2 = d.rep[r].disp_thr2;
    return d.rb_force[r] != 0 || m2 > t2 || (along && m2 > REBUILD_ALONG * REBUILD_ALONG * t2);
}

// Append, for the replicas of one chunk (one per thread, n of them per
// thread, numbered from first), the numbers first .. first + n - 1 to out,
// in thread order.  Returns the number appended.  Every thread of the block
// calls it.  The threads with n > 0 are compacted first; then the whole block
// writes their ranges with plain stores.
struct GateShared {
    int wtot[GATE_THREADS / WAVE];  // per wavefront: sum of n, then its exclusive prefix
    int wcnt[GATE_THREADS / WAVE];  // per wavefront: threads with n > 0, then their prefix
    int tot, cnt;
    int at[GATE_THREADS], first[GATE_THREADS], n[GATE_THREADS];  // compacted ranges
};

__device__ inline int gate_append(int32_t *out, int n, int first, GateShared &g)
{
    const int t = threadIdx.x, lane = t & (WAVE - 1), wv = t / WAVE;
    int inc = n;  // inclusive scan over the wavefront
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
        const int u = __shfl_up(inc, o, WAVE);
        if (lane >= o) inc += u;
    }
    const uint64_t has = __ballot(n > 0);
    const int rank = __popcll(has & ((1ull << lane) - 1ull));
    if (lane == WAVE - 1) {
        g.wtot[wv] = inc;
        g.wcnt[wv] = __popcll(has);
    }
    __syncthreads();
    if (t == 0) {
        int run = 0, cnt = 0;
        for (int k = 0; k < GATE_THREADS / WAVE; ++k) {
            const int x = g.wtot[k], c = g.wcnt[k];
            g.wtot[k] = run;
            g.wcnt[k] = cnt;
            run += x;
            cnt += c;
        }
        g.tot = run;
        g.cnt = cnt;
    }
    __syncthreads();
    if (n > 0) {
        const int k = g.wcnt[wv] + rank;
        g.at[k] = g.wtot[wv] + inc - n;
        g.first[k] = first;
        g.n[k] = n;
    }
    __syncthreads();
    // The block spreads the output positions, not the ranges: position o
    // belongs to the last range whose start is <= o (the starts ascend, and
    // the first is 0), found by a binary search.
    const int cnt = g.cnt, tot = g.tot;
    for (int o = t; o < tot; o += GATE_THREADS) {
        int lo = 0, hi = cnt - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (g.at[mid] <= o) lo = mid;
            else hi = mid - 1;
        }
        out[o] = g.first[lo] + (o - g.at[lo]);
    }
    __syncthreads();  // the shared arrays are reused
    return tot;
}

__global__ __launch_bounds__(GATE_THREADS) void k_rb_gate(Dev d)
{
    __shared__ GateShared g;
    __shared__ int wmust;
    // the wavefronts of the replicas that must rebuild; the others come
    // along only while those leave most of the device idle
    if (threadIdx.x == 0) wmust = 0;
    __syncthreads();
    for (int r = threadIdx.x; r < d.nrep; r += GATE_THREADS)
        if (rebuild_flag(d, r, false)) atomicAdd(&wmust, d.rep[r].wave1 - d.rep[r].wave0);
    __syncthreads();
    const int wm = wmust;
    const bool along = wm > 0 && wm < LIST_ALONG_WAVES;
    int nwl = 0;
    for (int r0 = 0; wm > 0 && r0 < d.nrep; r0 += GATE_THREADS) {
        const int r = r0 + threadIdx.x;
        int nw = 0, w0 = 0;
        if (r < d.nrep) {
            const RepInfo &R = d.rep[r];
            w0 = R.wave0;
            if (rebuild_flag(d, r, along)) nw = R.wave1 - R.wave0;
        }
        // most steps rebuild nothing: skip the compaction (block-uniform)
        if (!__syncthreads_or(nw > 0)) continue;
        nwl += gate_append(d.rb_wlist + nwl, nw, w0, g);
    }
    if (threadIdx.x == 0) {
        d.rb_any[0] = nwl;
        d.rb_any[1] = along ? 1 : 0;
    }
}

// Worklist entry of this wavefront for the per-wave kernels that run one
// wave per worklist entry: the first ceil(count / WAVES_PER_BLOCK) blocks
// take part, each XCD a contiguous part of the list; -1 for the rest.
__device__ inline int rb_work_wave(const Dev &d)
{
    const int nact = d.rb_any[0];
    const int nab = (nact + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK;
    if ((int)blockIdx.x >= nab) return -1;
    const int i = xcd_block(blockIdx.x, nab) * WAVES_PER_BLOCK + (threadIdx.x >> 6);
    return i < nact ? d.rb_wlist[i] : -1;
}

// The per-particle kernels of the chain walk the worklist with a grid
// stride over a capped grid (their work per unit is small).
//
// Lanes of one sub-cell are mostly consecutive (the slots are still in the
// order of the previous build).  The first lane of such a run counts the whole
// run and links it into the sub-cell's chain of runs: order[first slot] is the
// run before it, rank[first slot] its length, cell_head the last one linked.
// The chain needs no end mark and cell_head no clearing: the sub-cell's count
// says when all of its runs are found.
__device__ inline void assign_wave(const Dev &d, int w)
{
    const SegInfo &S = d.seg[d.wave_seg[w]];
    const int lane = lane_id();
    const int s = w * WAVE + lane;
    const bool real = (s - S.slot0) < S.n;
    const int nc = d.rep[S.rep].nc;
    int c = -1 - lane;  // distinct dummy for padding lanes
    if (real) {
        const uint4 m = d.mirror[s];
        const int cz = d.dim == 2 ? 0 : fix_cell(m.z, nc);  // planar: one layer of cells
        // sub-cell: the cell, then the quarter of its edge along x
        c = CELL_SUBX * (S.cell0 + (cz * nc + fix_cell(m.y, nc)) * nc) + fix_cell(m.x, CELL_SUBX * nc);
        d.cell_of[s] = c;
    }
    bool head;
    const int len = run_length(c, head);
    if (head && real) {
        atomicAdd(&d.cell_count[c], len);
        d.order[s] = atomicExch(&d.cell_head[c], s);
        d.rank[s] = len;
    }
}

// Chains without the gate (a single replica) decide here: each block by
// itself, the first one for the kernels after it.
__global__ __launch_bounds__(BLOCK) void k_rb_assign(Dev d)
{
    const bool gate = d.nrep == 1;
    int nact;
    if (gate) {
        nact = rebuild_flag(d, 0, false) ? d.nwaves : 0;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            d.rb_any[0] = nact;
            d.rb_any[1] = 0;
        }
    } else {
        nact = d.rb_any[0];
    }
    const int stride = gridDim.x * WAVES_PER_BLOCK;
    for (int i = blockIdx.x * WAVES_PER_BLOCK + (threadIdx.x >> 6); i < nact; i += stride) {
        if (gate && lane_id() == 0) d.rb_wlist[i] = i;
        assign_wave(d, gate ? i : d.rb_wlist[i]);
    }
}

// Exclusive scan of each segment's sub-cell counters into absolute slot
// numbers; a sub-cell ends where the next one starts (the last one at an entry of
// the segment's spare cell).  A segment's cells come in chunks of
// SCAN_CHUNK (8 consecutive cells per thread of a SCAN_THREADS block; block
// (segment, chunk) of a two-dimensional grid).  Each chunk starts at the
// segment's first slot plus the totals of the chunks before it, so that the
// chunks of a large system are scanned in parallel instead of one after
// another.  Segments of up to SCAN_DIRECT chunks have them summed by each
// chunk itself, larger ones by k_rb_scan_sum: a launch on every step (2 us)
// against some microseconds on the steps that rebuild.  (Totals counted by
// atomics in k_rb_assign: 15 -> 190 us at 2^20, whose wavefronts queue for
// 150 addresses.)  A cell's CELL_SUBX = 4 sub-cell counters are read as one
// int4 and its ranges written as int4s, so a pass moves no more loads and
// stores than a scan of the cells alone would.
constexpr int SCAN_DIRECT = 8;
static_assert(CELL_SUBX == 4, "the scan reads the sub-cells of a cell as one int4");

__device__ inline int chunk_cells(const SegInfo &S, int c)
{
    return min(S.ncell - c * SCAN_CHUNK, SCAN_CHUNK);
}

constexpr int SCAN_THREADS = SCAN_CHUNK / 8;
constexpr int SCAN_WAVES = SCAN_THREADS / WAVE;

// Particles of the cells cnt[8 t .. 8 t + 7] (of n).
__device__ inline int scan_sum8(const int4 *cnt, int n, int4 v[8])
{
    int sum = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int i = 8 * threadIdx.x + k;
        v[k] = i < n ? cnt[i] : make_int4(0, 0, 0, 0);
        sum += v[k].x + v[k].y + v[k].z + v[k].w;
    }
    return sum;
}

__global__ __launch_bounds__(SCAN_THREADS) void k_rb_scan_sum(Dev d)
{
    __shared__ int wtot[SCAN_WAVES];
    if (d.rb_any[0] == 0) return;
    const SegInfo &S = d.seg[blockIdx.x];
    const int c = blockIdx.y;
    const int n = chunk_cells(S, c);
    if (n <= 0 || !rebuild_flag(d, S.rep, d.rb_any[1] != 0)) return;
    int4 v[8];
    const int4 *cnt = reinterpret_cast<const int4 *>(d.cell_count + CELL_SUBX * (S.cell0 + c * SCAN_CHUNK));
    const int sum = wave_sum_i(scan_sum8(cnt, n, v));
    if (lane_id() == 0) wtot[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        int tot = 0;
        for (int k = 0; k < SCAN_WAVES; ++k) tot += wtot[k];
        d.chunk_sum[blockIdx.x * d.scan_cps + c] = tot;
    }
}

__global__ __launch_bounds__(SCAN_THREADS) void k_rb_scan(Dev d)
{
    __shared__ int wtot[SCAN_WAVES], wcarry[SCAN_WAVES];
    if (d.rb_any[0] == 0) return;
    const SegInfo &S = d.seg[blockIdx.x];
    const int c = blockIdx.y;
    const int n = chunk_cells(S, c);
    if (n <= 0 || !rebuild_flag(d, S.rep, d.rb_any[1] != 0)) return;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    int carry = 0;  // the particles of the segment's chunks before this one
    int4 v[8];
    if (d.scan_cps <= SCAN_DIRECT) {
        for (int k = 0; k < c; ++k)
            carry += scan_sum8(reinterpret_cast<const int4 *>(d.cell_count + CELL_SUBX * (S.cell0 + k * SCAN_CHUNK)),
                               SCAN_CHUNK, v);
    } else {
        for (int k = t; k < c; k += SCAN_THREADS) carry += d.chunk_sum[blockIdx.x * d.scan_cps + k];
    }
    carry = wave_sum_i(carry);
    if (lane == 0) wcarry[wv] = carry;
    if (t == 0 && S.type == 0 && c == 0) atomicAdd(&d.counters[0], 1);
    const int4 *cnt = reinterpret_cast<const int4 *>(d.cell_count + CELL_SUBX * (S.cell0 + c * SCAN_CHUNK));
    int4 *cst = reinterpret_cast<int4 *>(d.cell_start + CELL_SUBX * (S.cell0 + c * SCAN_CHUNK));
    const int i0 = 8 * t, sum = scan_sum8(cnt, n, v);
    int inc = sum;  // inclusive scan over the wavefront
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(inc, o, 64);
        if (lane >= o) inc += u;
    }
    if (lane == 63) wtot[wv] = inc;
    __syncthreads();
    if (t == 0) {
        int run = 0;
        for (int k = 0; k < SCAN_WAVES; ++k) run += wcarry[k];
        for (int k = 0; k < SCAN_WAVES; ++k) { const int x = wtot[k]; wtot[k] = run; run += x; }
    }
    __syncthreads();
    int run = S.slot0 + wtot[wv] + inc - sum;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        if (i0 + k < n) {
            int4 a;
            a.x = run; run += v[k].x;
            a.y = run; run += v[k].y;
            a.z = run; run += v[k].z;
            a.w = run; run += v[k].w;
            cst[i0 + k] = a;
            if (c * SCAN_CHUNK + i0 + k + 1 == S.ncell) d.cell_start[CELL_SUBX * (S.cell0 + S.ncell)] = run;
        }
    }
}

// A position reduced to its high 16 bits per axis: x and y packed (x low), z.
__device__ inline uint2 coarse_of(const uint4 &m) { return make_uint2((m.x >> 16) | (m.y & 0xffff0000u), m.z >> 16); }

// One particle's state from slot v to sorted slot t.  The old copy is dead
// once read (non-temporal loads); the sorted copy is read back soon by the
// list builder, and the sorted mirror is its candidates (plain stores).
__device__ inline void gather_one(const Dev &d, int v, int t)
{
    const int np = d.npad_total;
    d.sx[t] = ld_stream(&d.x[v]);
    d.sy[t] = ld_stream(&d.y[v]);
    d.sz[t] = ld_stream(&d.z[v]);
    d.svx[t] = ld_stream(&d.vx[v]);
    d.svy[t] = ld_stream(&d.vy[v]);
    d.svz[t] = ld_stream(&d.vz[v]);
    d.sax[t] = ld_stream(&d.ax[v]);
    d.say[t] = ld_stream(&d.ay[v]);
    d.saz[t] = ld_stream(&d.az[v]);
    d.simg[t] = ld_stream(&d.img[v]);
    d.simg[np + t] = ld_stream(&d.img[np + v]);
    d.simg[2 * np + t] = ld_stream(&d.img[2 * np + v]);
    d.sid[t] = ld_stream(&d.id[v]);
    const uint4 m = d.mirror[v];
    d.smirror[t] = m;  // the list builder's candidates: cached
    d.scoarse[t] = coarse_of(m);
}

// One thread per particle of the replicas that rebuild.  A particle's
// destination is its sub-cell's start plus its rank by previous slot among the
// sub-cell's members, which makes the counting sort stable: the walk over the
// sub-cell's chain of runs (a few runs of a few particles, in the order of the
// atomics that linked them) adds what each run holds below the particle's slot.
// Each member also clears its sub-cell's counter for the next rebuild (a
// sub-cell without members was never counted).
//
// The chain ran two kernels more, one that scattered slot numbers into their
// sub-cells for this one to rank and, for a single replica, the gate: between
// rebuilds each is an empty launch of 2 us.  Measured (us per step, with the
// direct scan offsets): 32,000 particles MIXED NVE 29.1 -> 26.1, 64,000 41.6 ->
// 36.8, 32,000 FP64 Nose-Hoover 53.0 -> 49.6, 2^20 MIXED 297 -> 293.
__global__ __launch_bounds__(BLOCK) void k_rb_sortgather(Dev d)
{
    const int nact = d.rb_any[0];
    if (nact == 0) return;
    const int stride = gridDim.x * WAVES_PER_BLOCK;
    for (int i = blockIdx.x * WAVES_PER_BLOCK + (threadIdx.x >> 6); i < nact; i += stride) {
        const int w = d.rb_wlist[i];
        const SegInfo &S = d.seg[d.wave_seg[w]];
        const int s = w * WAVE + lane_id();
        if (s - S.slot0 < S.n) {
            const int sc = d.cell_of[s];
            int f = d.cell_head[sc];
            const int st = d.cell_start[sc];
            int left = d.cell_start[sc + 1] - st, rank = 0;
            while (left > 0) {
                const int len = d.rank[f], before = d.order[f];
                rank += min(max(s - f, 0), len);
                left -= len;
                f = before;
            }
            gather_one(d, s, st + rank);
            d.cell_count[sc] = 0;
        }
    }
}

// Small replicas (every one of the plan within SORT_SLOTS slots and SORT_CELLS
// sub-cells): the gate and the whole counting sort in one kernel, one block per
// replica, with the counters, their scan and the order in LDS.  A step without
// a rebuild then launches two chain kernels instead of six, and a rebuild's sort
// is one pass over its replica instead of five kernels.  Up to SORT_ALONE_REPS
// replicas every block decides the flags of all of them by itself (the rule of
// k_rb_gate), from which follow the worklist's length and the place of its own
// replica in it; beyond, where that would be quadratic work, the gate runs
// first (GATED).  The result is that of the other chain: a stable sort by
// sub-cell.
//
// Bound by latency: on a step that rebuilds, the passes over the counters and
// particles of one replica by one block (12 us at 1000 particles); otherwise by
// its launch.  Measured (us per MIXED step, the chain of kernels, then this):
// 1000 particles NVE 23.7 -> 17.4, 64 replicas of 1000 under the bath 68 -> 60,
// 256 replicas 415 -> 402.
constexpr int SORT_THREADS = 1024;
constexpr int SORT_PER = SORT_SLOTS / SORT_THREADS;

__device__ inline int block_sum(int v, int *part)  // all threads of a SORT_THREADS block
{
    v = wave_sum_i(v);
    if (lane_id() == 0) part[threadIdx.x / WAVE] = v;
    __syncthreads();
    int t = 0;
#pragma unroll
    for (int k = 0; k < SORT_THREADS / WAVE; ++k) t += part[k];
    __syncthreads();
    return t;
}

template <bool GATHER, bool GATED>
__global__ __launch_bounds__(SORT_THREADS) void k_rb_sort_small(Dev d)
{
    __shared__ int start[SORT_CELLS];         // counters, then the sub-cells' first slots
    __shared__ uint16_t order[SORT_SLOTS];
    __shared__ int part[SORT_THREADS / WAVE];
    const int me = blockIdx.x, t = threadIdx.x, lane = lane_id();
    // the gate
    int before = 0;
    if (GATED) {
        if (d.rb_any[0] == 0 || !rebuild_flag(d, me, d.rb_any[1] != 0)) return;
    } else if (d.nrep == 1) {
        const bool mine = rebuild_flag(d, 0, false);
        if (t == 0) {
            d.rb_any[0] = mine ? d.nwaves : 0;
            d.rb_any[1] = 0;
        }
        if (!mine) return;
    } else {
        int must = 0;
        for (int r = t; r < d.nrep; r += SORT_THREADS)
            if (rebuild_flag(d, r, false)) must += d.rep[r].wave1 - d.rep[r].wave0;
        must = block_sum(must, part);
        const bool along = must > 0 && must < LIST_ALONG_WAVES;
        int total = 0;
        if (must > 0) {
            for (int r = t; r < d.nrep; r += SORT_THREADS)
                if (rebuild_flag(d, r, along)) {
                    const int nw = d.rep[r].wave1 - d.rep[r].wave0;
                    total += nw;
                    before += r < me ? nw : 0;
                }
            if (me == 0) total = block_sum(total, part);
            before = block_sum(before, part);
        }
        if (me == 0 && t == 0) {
            d.rb_any[0] = total;
            d.rb_any[1] = along ? 1 : 0;
        }
        if (must == 0 || !rebuild_flag(d, me, along)) return;
    }
    const RepInfo &R = d.rep[me];
    const SegInfo &A = d.seg[R.seg[0]], &B = d.seg[R.seg[1]];
    const int base = R.wave0 * WAVE, nc = R.nc, nslot = (R.wave1 - R.wave0) * WAVE;
    const int b0 = B.slot0 - base;                            // the replica's first B slot
    const int sub0 = CELL_SUBX * A.cell0, nsub = CELL_SUBX * (A.ncell + 1 + B.ncell);  // A's spare cell between
    if (!GATED)
        for (int i = t; i < R.wave1 - R.wave0; i += SORT_THREADS) d.rb_wlist[before + i] = R.wave0 + i;
    if (t == 0) atomicAdd(&d.counters[0], 1);
    for (int i = t; i < nsub; i += SORT_THREADS) start[i] = 0;
    __syncthreads();
    // count; each thread keeps the sub-cell and the arrival rank of its particles
    int cell[SORT_PER], rank[SORT_PER];
#pragma unroll
    for (int k = 0; k < SORT_PER; ++k) {
        const int l = k * SORT_THREADS + t;
        cell[k] = -1;
        if (l < nslot && (l < b0 ? l < A.n : l - b0 < B.n)) {
            const uint4 m = d.mirror[base + l];
            const int cz = d.dim == 2 ? 0 : fix_cell(m.z, nc);
            const SegInfo &S = l < b0 ? A : B;
            cell[k] = CELL_SUBX * (S.cell0 + (cz * nc + fix_cell(m.y, nc)) * nc) + fix_cell(m.x, CELL_SUBX * nc) - sub0;
            rank[k] = atomicAdd(&start[cell[k]], 1);
        }
    }
    __syncthreads();
    // exclusive scan: nsub / 1024 consecutive sub-cells per thread
    constexpr int CPT = SORT_CELLS / SORT_THREADS;
    const int per = (nsub + SORT_THREADS - 1) / SORT_THREADS;
    int cnt[CPT], sum = 0;
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
        const int c = t * per + k;
        cnt[k] = k < per && c < nsub ? start[c] : 0;
        sum += cnt[k];
    }
    int inc = sum;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
        const int u = __shfl_up(inc, o, WAVE);
        if (lane >= o) inc += u;
    }
    if (lane == WAVE - 1) part[t / WAVE] = inc;
    __syncthreads();
    int run = inc - sum;
    for (int k = 0; k < t / WAVE; ++k) run += part[k];
    const int nsubA = CELL_SUBX * A.ncell, shift = b0 - A.n;  // B's slots start at the next wavefront
    if (t == 0) d.cell_start[sub0 + nsub] = base + b0 + B.n;
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
        const int c = t * per + k;
        if (k < per && c < nsub) {
            const int at = run + (c < nsubA + CELL_SUBX ? 0 : shift);
            start[c] = at;
            d.cell_start[sub0 + c] = base + at;
        }
        run += cnt[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < SORT_PER; ++k)
        if (cell[k] >= 0) order[start[cell[k]] + rank[k]] = (uint16_t)(k * SORT_THREADS + t);
    __syncthreads();
    // rank by previous slot among the sub-cell's members, then the state moves
#pragma unroll
    for (int k = 0; k < SORT_PER; ++k)
        if (cell[k] >= 0) {
            const int l = k * SORT_THREADS + t, c = cell[k], st = start[c];
            const int en = c + 1 == nsub ? b0 + B.n : start[c + 1];
            int at = st;
            for (int e = st; e < en; ++e) at += order[e] < l ? 1 : 0;
            if (GATHER) gather_one(d, base + l, base + at);
            else d.rank[base + l] = base + at;
        }
}

// The state of the listed waves into the sorted places in d.rank.
__global__ __launch_bounds__(BLOCK) void k_rb_gather(Dev d)
{
    const int nact = d.rb_any[0];
    if (nact == 0) return;
    const int stride = gridDim.x * WAVES_PER_BLOCK;
    for (int i = blockIdx.x * WAVES_PER_BLOCK + (threadIdx.x >> 6); i < nact; i += stride) {
        const int w = d.rb_wlist[i];
        const SegInfo &S = d.seg[d.wave_seg[w]];
        const int s = w * WAVE + lane_id();
        if (s - S.slot0 < S.n) gather_one(d, s, d.rank[s]);
    }
}

// Maximum of v over the 64 lanes of a wavefront whose lanes are all active:
// a running maximum along each row of 16 lanes by DPP row shifts (a lane
// with no source lane in its row keeps the identity), then the last lane of
// each row read into a scalar.  A few cycles, where a butterfly of lane
// permutes waits on the LDS crossbar six times.
__device__ inline int wave_max_all(int v)
{
    v = max(v, __builtin_amdgcn_update_dpp(INT_MIN, v, 0x111, 0xf, 0xf, false));  // row_shr:1
    v = max(v, __builtin_amdgcn_update_dpp(INT_MIN, v, 0x112, 0xf, 0xf, false));  // row_shr:2
    v = max(v, __builtin_amdgcn_update_dpp(INT_MIN, v, 0x114, 0xf, 0xf, false));  // row_shr:4
    v = max(v, __builtin_amdgcn_update_dpp(INT_MIN, v, 0x118, 0xf, 0xf, false));  // row_shr:8
    const int r0 = __builtin_amdgcn_readlane(v, 15), r1 = __builtin_amdgcn_readlane(v, 31);
    const int r2 = __builtin_amdgcn_readlane(v, 47), r3 = __builtin_amdgcn_readlane(v, 63);
    return max(max(r0, r1), max(r2, r3));
}

// Two signed 16-bit lanes of one 32-bit register.
typedef short short2_t __attribute__((ext_vector_type(2)));

// Squared separation minus `bound` (bound >= 1), in units of 2^16 fixed-point
// steps, from coordinates reduced to their high 16 bits: x and y packed in
// one word (x low), z in the low half of another.  Differences wrap modulo
// 2^16, which is the minimum image, as for the full 32-bit coordinates.  The
// x-y sum minus the bound lies in [-bound, 2^31 - bound], so only the final
// sum can saturate, and it does so upwards: the result is negative exactly
// when the squared separation is below the bound.
__device__ inline int r2_coarse_below(uint32_t ixy, uint32_t iz, uint32_t jxy, uint32_t jz, int bound)
{
    const short2_t dxy = __builtin_bit_cast(short2_t, ixy) - __builtin_bit_cast(short2_t, jxy);
    const short2_t dz = __builtin_bit_cast(short2_t, iz) - __builtin_bit_cast(short2_t, jz);
    return __builtin_amdgcn_sdot2(dz, dz, __builtin_amdgcn_sdot2(dxy, dxy, -bound, true), true);
}

__device__ inline double gap(int o, int c, double cw, double u)
{
    return o > 0 ? (c + o) * cw - u : (o < 0 ? u - (c + o + 1) * cw : 0.0);
}

// Base slot of a wavefront's 16-bit entries in the part of its own type (cells
// from cell0 on): the lowest slot that its lanes' stencils and its own slots s
// reach, if all of them lie within 2^16 of it; else -1.  All lanes take part.
__device__ inline int own_base(const Dev &d, int cell0, int s, bool real, int cy, int cz, int reach, int noff, int oz0,
                               int nz, int nc)
{
    int lo = s, hi = s + 1;
    if (real) {
        // lowest and highest stencil row (qz * nc + qy) in slot order; a range
        // that wraps around the box covers both ends
        int z0 = cz + oz0, z1 = cz + oz0 + nz - 1;
        if (z0 < 0 || z1 >= nc) z0 = 0, z1 = nc - 1;
        int y0 = cy - reach, y1 = cy - reach + noff - 1;
        if (y0 < 0 || y1 >= nc) y0 = 0, y1 = nc - 1;
        lo = min(lo, d.cell_start[CELL_SUBX * (cell0 + (z0 * nc + y0) * nc)]);
        hi = max(hi, d.cell_start[CELL_SUBX * (cell0 + (z1 * nc + y1) * nc + nc)]);
    }
    lo = -wave_max_all(-lo);
    hi = wave_max_all(hi);
    return hi - lo <= 65536 ? lo : -1;
}

// Entries of the parts of a list (16-bit ones where `base` is not -1) cut to
// the rows there are, so that the force kernels stay inside it.
__device__ inline int2 cut_to_rows(int2 k, int2 base, int rows)
{
    const bool h0 = base.x != -1, h1 = base.y != -1;
    const int w0 = min(h0 ? k.x / 2 : k.x, rows);
    const int w1 = min(h1 ? k.y / 2 : k.y, rows - w0);
    return make_int2(h0 ? 2 * w0 : w0, h1 ? 2 * w1 : w1);
}

// Neighbour lists.  One thread per particle.  Entries [0, kA) of a list hold
// the particle's A partners, entries [kA, kA + kB) its B partners, where kA,
// kB are the wavefront maxima rounded up to LIST_ROW_ALIGN.  The part of the
// particle's own type also holds its own slot once (it passes the distance
// test), and unused entries hold it too; the force kernels skip it (zero
// separation).  Storage follows list_index: a particle appends 16 contiguous
// bytes at a time, so cache lines fill completely before they leave the L2.
//
// The stencil is walked row by row: the cells of one stencil row differ only
// in x and are consecutive in the cell-sorted slot order, so a row is one
// contiguous slot range (two when it wraps around the box), scanned eight
// candidates at a time.  With cells as wide as the list radius (reach 1) all
// particles of a cell walk the same 27 cells in the same order, so the lanes
// of a wavefront that share a cell load the same addresses and one cache-line
// access serves all of them; no per-particle pruning is done there, since it
// would break that sharing for little gain.  With finer cells (reach 2) rows,
// and the end cells of a row, that lie farther than the list radius from the
// particle are skipped (in FP64, with a margin), which removes most of the
// 125-cell stencil.  Grids with fewer than 2*reach+1 cells per edge scan
// whole rows.
//
// Candidate test in u32 fixed-point units: the integer difference of two
// coordinates is the minimum-image separation (the box maps onto the full
// 2^32 range), converted to float; rl2_fx is enlarged by a few parts in 10^6
// so that the list is a superset of the exact one.  The sorted mirror has
// LIST_UNROLL spare entries past its end, so the unrolled loads need no clamp.
//
// Accepted entries are staged in LDS, LIST_STAGE per lane, and written out
// four at a time (one 16-byte store per lane) when some lane's stage fills.
// Staging keeps stores out of the scan loop: on this architecture a wait for
// loaded data also waits for every store issued before those loads, so a
// store per candidate batch would expose the store latency on every batch.
//
// Candidate positions are staged too.  With one cell per list radius every
// particle scans, per stencil row, at most two pieces: the main run of cells
// and, where the row wraps around the box, its wrapped end cell.  For each
// piece the wavefront loads the union of its lanes' slot ranges into LDS
// once, with coalesced loads, and the lanes then scan their own ranges out
// of LDS; lanes of one cell read the same LDS words (a broadcast).  A union
// longer than LIST_WIN (lanes in different rows of the grid) is scanned
// straight from global memory instead.
constexpr int LIST_STAGE = 16;
// Boxes up to this edge (in the model's length unit) use the coarse staged
// candidate test; a 2^16-step unit is then at most 0.0034, and the list grows
// by under 0.6%.
constexpr double COARSE_MAX_BOX = 220.0;
constexpr int LIST_WIN = 384;
constexpr int LIST_QUEUE = 10;  // k_rb_list_masks: entries of 64 candidates per lane

// The sorted state of slot s back into place, with the mirror (mi) and the
// build position.
__device__ inline void copy_back(const Dev &d, int s, bool real, const uint4 &mi)
{
    const int np = d.npad_total;
    double px, py, pz;  // the position, for the FP64 packed copy
    if (real) {
        px = ld_stream(&d.sx[s]);
        py = ld_stream(&d.sy[s]);
        pz = ld_stream(&d.sz[s]);
        st_stream(px, &d.x[s]);
        st_stream(py, &d.y[s]);
        st_stream(pz, &d.z[s]);
        st_stream(ld_stream(&d.svx[s]), &d.vx[s]);
        st_stream(ld_stream(&d.svy[s]), &d.vy[s]);
        st_stream(ld_stream(&d.svz[s]), &d.vz[s]);
        st_stream(ld_stream(&d.sax[s]), &d.ax[s]);
        st_stream(ld_stream(&d.say[s]), &d.ay[s]);
        st_stream(ld_stream(&d.saz[s]), &d.az[s]);
        st_stream(ld_stream(&d.simg[s]), &d.img[s]);
        st_stream(ld_stream(&d.simg[np + s]), &d.img[np + s]);
        st_stream(ld_stream(&d.simg[2 * np + s]), &d.img[2 * np + s]);
        st_stream(ld_stream(&d.sid[s]), &d.id[s]);
        d.mirror[s] = mi;  // gathered by the next step: cached
        st_stream(mi, &d.mbuild[s]);
    } else {
        px = d.x[s];
        py = d.y[s];
        pz = d.z[s];
    }
    if (d.pos4) d.pos4[s] = make_double4(px, py, pz, 0.0);  // FP64: gathers see the new order
}

// STAGE: the window variant of the force kernels is on (d.stage_ok), so
// parts whose windows fit are written in the window format; without it the
// window code is compiled out.
template <bool STAGE>
__global__ __launch_bounds__(BLOCK) void k_rb_list(Dev d, int reach)
{
    __shared__ int32_t stage[WAVES_PER_BLOCK][LIST_STAGE][WAVE];
    __shared__ __attribute__((aligned(16))) uint32_t win_s[WAVES_PER_BLOCK][3][LIST_WIN + LIST_UNROLL];
    const int w = rb_work_wave(d);  // each XCD walks a contiguous part of the worklist
    if (w < 0) return;
    const SegInfo &S = d.seg[d.wave_seg[w]];
    const int rep = S.rep;
    const RepInfo &R = d.rep[rep];
    const int lane = lane_id();
    const int s = w * WAVE + lane;
    const bool real = (s - S.slot0) < S.n;
    uint4 mi = make_uint4(0, 0, 0, 0);
    if (real) mi = d.smirror[s];
    copy_back(d, s, real, mi);
    const int nc = R.nc;
    const int noff = min(nc, 2 * reach + 1);
    const bool whole = nc < 2 * reach + 1;  // every cell of a row is in the stencil
    const bool prune = !whole && reach > 1;
    const int fx = fix_cell(mi.x, CELL_SUBX * nc);  // x in quarter cells
    const int cx = fx / CELL_SUBX, qx = fx % CELL_SUBX;
    const int cy = fix_cell(mi.y, nc), cz = d.dim == 2 ? 0 : fix_cell(mi.z, nc);
    // slot range [cs(c), ce(c)) of cell c (its sub-cells together)
    auto cs = [&](int c) __attribute__((always_inline)) { return d.cell_start[CELL_SUBX * c]; };
    auto ce = [&](int c) __attribute__((always_inline)) { return d.cell_start[CELL_SUBX * (c + 1)]; };
    // a planar system has every particle in its single (z = 0) layer of cells
    const int oz0 = d.dim == 2 ? 0 : -reach, nz = d.dim == 2 ? 1 : noff;
    const double cw = 4294967296.0 / (double)nc;  // cell edge in fixed units
    const double ux = (double)mi.x, uy = (double)mi.y, uz = (double)mi.z;
    // The staged candidate test compares coordinates reduced to their high
    // 16 bits (x and y packed, z alone) when the box is small enough that the
    // coarse units cost the list almost nothing (below); otherwise full ones.
    const uint32_t ixy = (mi.x >> 16) | (mi.y & 0xffff0000u), iz = mi.z >> 16;
    const bool coarse = R.L <= COARSE_MAX_BOX;
    int32_t *col = d.nbr + list_index(w, d.rows, 0, lane);
    int32_t(*buf)[WAVE] = stage[threadIdx.x / WAVE];
    uint32_t *wx = win_s[threadIdx.x / WAVE][0];
    uint32_t *wy = win_s[threadIdx.x / WAVE][1];
    uint32_t *wz = win_s[threadIdx.x / WAVE][2];
    uint2 *wc = reinterpret_cast<uint2 *>(wx);  // the coarse window: spans wx and wy
    const int rows = d.rows;
    int row = 0;  // 32-bit words of the list used so far
    int total = 0;
    int2 kpart = make_int2(0, 0), bpart = make_int2(-1, -1);  // per part: entries, base
    int2 pcnt = make_int2(0, 0);                              // per part: window pieces (staged)
    int n16 = 0;
    for (int tj = 0; tj < 2; ++tj) {
        const SegInfo &SJ = d.seg[R.seg[tj]];
        const float rl2 = R.rl2_fx[S.type + tj];
        const double rp = sqrt((double)rl2) + 4096.0;  // pruning radius with margin
        // Coarse test.  Truncating both coordinates to 2^16-step units changes
        // their difference by less than one unit per axis, so a pair within
        // the list radius r (in those units) has a coarse separation below
        // r + sqrt(3).  Accepting every coarse r2 below that bound squared
        // keeps the list a superset of the exact one; the extra entries lie
        // in a shell sqrt(3) units thick (0.3% more entries at L = 100).
        // r2c = ceil((r + sqrt(3))^2) + 1, from the host.
        const int r2c = R.r2c[S.type + tj];
        const double rp2 = rp * rp;
        // lowest start and highest end of the lanes' non-empty ranges
        // (x = INT_MAX when no lane has one); all lanes take part
        auto span = [&](int st, int en) __attribute__((always_inline)) {
            const bool has = st < en;
            return make_int2(-wave_max_all(has ? -st : INT_MIN + 1), wave_max_all(has ? en : -1));
        };
        // Slot ranges of one stencil row: the main run of cells, and the end
        // cell that wraps around the box where the row does.
        const int32_t *cstart = d.cell_start, *cend = d.cell_start + 1;
        const int cell0 = SJ.cell0;  // kept in a register across the list stores
        auto bounds = [&](int oz, int oy) __attribute__((always_inline)) {
            int4 b = make_int4(0, 0, 0, 0);
            if (real) {
                const int qz = (cz + oz + nc) % nc;
                const int qy = (cy + oy + nc) % nc;
                const int rowc = cell0 + (qz * nc + qy) * nc;  // cell (0, qy, qz)
                if (whole) {
                    b.x = cs(rowc);
                    b.y = ce(rowc + nc - 1);
                } else {
                    // One cell per list radius (reach 1): a particle in
                    // quarter qx of its cell is more than a cell edge, and
                    // so more than the list radius, away along x from the
                    // quarters of the left cell below qx and of the right
                    // cell above qx; both are left out.
                    const int a = cx - reach, e = cx + reach;
                    b.x = cstart[a < 0 ? CELL_SUBX * rowc : CELL_SUBX * (rowc + a) + qx];
                    b.y = cend[e >= nc ? CELL_SUBX * (rowc + nc) - 1 : CELL_SUBX * (rowc + e) + qx];
                    // the left cell wraps to the high end of the row, or
                    // the right cell to its low end
                    const bool lw = a < 0;
                    if (lw || e >= nc) {
                        b.z = cstart[lw ? CELL_SUBX * (rowc + a + nc) + qx : CELL_SUBX * rowc];
                        b.w = cend[lw ? CELL_SUBX * (rowc + nc) - 1 : CELL_SUBX * (rowc + e - nc) + qx];
                    }
                }
            }
            return b;
        };
        // The force kernels' windows (mixed precisions, one cell per list
        // radius).  The part's stencil rows are split into groups, in row
        // order, each as many rows as fit one window: the wavefront's union
        // span of every row piece of the group, one after the other, plus
        // one slot per lane holding that lane's own position.  The force
        // kernel stages and reads one group's window at a time.  Entries of
        // a staged part are 16-bit offsets into their group's window; every
        // lane's entries of a group end at a common count (padding), and
        // the padding points at the lane's own copy (zero separation,
        // skipped like the own slot).  The groups are found in a first pass
        // over the rows, since they decide the format of every entry.
        const int nrow = nz * noff;
        int2 *ptab = d.pieces + ((size_t)w * 2 + tj) * STAGE_PIECES;
        int4 *gtab = d.sgroups + ((size_t)w * 2 + tj) * STAGE_GROUPS;
        int npiece = 0, ngroup = 0, gw = 0, gmax = 0;
        int gw0 = 0, gw1 = 0, gw2 = 0, gw3 = 0;  // window slots of each group (selects, not an array)
        uint32_t gbound = 0;                      // bit r: a new group starts at stencil row r
        const bool try_stage = STAGE && SJ.n > 0 && !prune && nrow <= 32;
        auto close_group = [&]() __attribute__((always_inline)) {
            if (lane == 0 && ngroup < STAGE_GROUPS) gtab[ngroup] = make_int4(npiece, gw, 0, 0);
            gw0 = ngroup == 0 ? gw : gw0;
            gw1 = ngroup == 1 ? gw : gw1;
            gw2 = ngroup == 2 ? gw : gw2;
            gw3 = ngroup == 3 ? gw : gw3;
            gmax = max(gmax, gw);
            ++ngroup;
            gw = 0;
        };
        if (try_stage) {
            int oz = oz0, oy = -reach;
            for (int r = 0; r < nrow; ++r) {
                const int4 b = bounds(oz, oy);
                const int2 p1 = span(b.x, b.y), p2 = span(b.z, b.w);
                const int l1 = p1.x != INT_MAX ? p1.y - p1.x : 0, l2 = p2.x != INT_MAX ? p2.y - p2.x : 0;
                if (gw > 0 && gw + l1 + l2 + WAVE > STAGE_SLOTS) {
                    close_group();
                    gbound |= 1u << r;
                }
                if (l1 > 0) {
                    if (lane == 0 && npiece < STAGE_PIECES) ptab[npiece] = make_int2(p1.x, l1);
                    ++npiece;
                    gw += l1;
                }
                if (l2 > 0) {
                    if (lane == 0 && npiece < STAGE_PIECES) ptab[npiece] = make_int2(p2.x, l2);
                    ++npiece;
                    gw += l2;
                }
                if (++oy == -reach + noff) {
                    oy = -reach;
                    ++oz;
                }
            }
            close_group();
        }
        const bool staged = try_stage && npiece <= STAGE_PIECES && ngroup <= STAGE_GROUPS && gmax + WAVE <= STAGE_SLOTS;
        // Otherwise entries of the part of the particle's own type are stored
        // as 16-bit offsets from a base slot, two to a 32-bit word, when every
        // slot the wavefront can accept (the cell rows of its stencils) and
        // its own slots lie within 2^16 of the lowest of them; else, and for
        // the other part, as 32-bit slot indices.  base = -1 marks 32-bit
        // entries; staged windows use base 0.
        int base = staged ? 0 : -1;
        if (!staged && tj == S.type && SJ.n > 0) base = own_base(d, SJ.cell0, s, real, cy, cz, reach, noff, oz0, nz, nc);
        const bool half = base >= 0;
        const int group = half ? 8 : 4;  // entries per 16-byte store
        auto pack = [&](int a, int b) __attribute__((always_inline)) { return (a - base) | ((b - base) << 16); };
        int cnt = 0;   // entries accepted (and padding between window groups)
        int npad = 0;  // of them padding
        int done = 0;  // entries written to the list (a multiple of group)
        auto flush = [&]() __attribute__((always_inline)) {  // write every complete group of staged entries
            while (done + group <= cnt) {
                const int k = row + (half ? done / 2 : done);  // 32-bit word of the list
                int e[8];
#pragma unroll
                for (int t = 0; t < 4; ++t) e[t] = buf[(done + t) & (LIST_STAGE - 1)][lane];
                if (half) {
#pragma unroll
                    for (int t = 4; t < 8; ++t) e[t] = buf[(done + t) & (LIST_STAGE - 1)][lane];
                }
                const int4 q = half ? make_int4(pack(e[0], e[1]), pack(e[2], e[3]), pack(e[4], e[5]), pack(e[6], e[7]))
                                    : make_int4(e[0], e[1], e[2], e[3]);
                if (k < rows) *reinterpret_cast<int4 *>(col + (k >> 2) * 256) = q;
                done += group;
            }
        };
        // Each candidate is written to the next free stage slot whether or
        // not it is accepted; only an accepted one advances the count.  At
        // the start of a batch at most LIST_STAGE - LIST_UNROLL entries are
        // pending, so the slot written is never one still to be flushed.
        // The particle's own slot passes the test (zero separation) and stays
        // in its list, where the force kernels skip it like the padding.
        // `in` is false only past the end of a range, in the last batch.
        // The entry of slot j is j + dl: dl = 0 for slot indices, the
        // piece's offset in the window minus its first slot when staged.
        int dl = 0;
        auto test = [&](int j, bool in, uint32_t jx, uint32_t jy, uint32_t jz) __attribute__((always_inline)) {
            const float dx = (float)(int)(mi.x - jx);
            const float dy = (float)(int)(mi.y - jy);
            const float dz = (float)(int)(mi.z - jz);
            const float r2 = dx * dx + dy * dy + dz * dz;
            const int acc = (int)in & (int)(r2 < rl2);
            buf[cnt & (LIST_STAGE - 1)][lane] = j + dl;
            cnt += acc;
        };
        auto test_coarse = [&](int j, bool in, uint32_t jxy, uint32_t jz) __attribute__((always_inline)) {
            // the sign bit of r2 - r2c
            const int acc = (int)in & (int)((uint32_t)r2_coarse_below(ixy, iz, jxy, jz, r2c) >> 31);
            buf[cnt & (LIST_STAGE - 1)][lane] = j + dl;
            cnt += acc;
        };
        auto scan = [&](int st, int en) __attribute__((always_inline)) {  // straight from global memory
            int j = st;
            for (; j + LIST_UNROLL <= en; j += LIST_UNROLL) {  // whole batches
                const uint4 *src = d.smirror + j;
                uint4 mj[LIST_UNROLL];
#pragma unroll
                for (int u = 0; u < LIST_UNROLL; ++u) mj[u] = src[u];
#pragma unroll
                for (int u = 0; u < LIST_UNROLL; ++u) test(j + u, true, mj[u].x, mj[u].y, mj[u].z);
                if (__any(cnt - done > LIST_STAGE - LIST_UNROLL)) flush();
            }
            if (j < en) {  // the last, partial batch
                const uint4 *src = d.smirror + j;
                uint4 mj[LIST_UNROLL];
#pragma unroll
                for (int u = 0; u < LIST_UNROLL; ++u) mj[u] = src[u];
#pragma unroll
                for (int u = 0; u < LIST_UNROLL; ++u) test(j + u, j + u < en, mj[u].x, mj[u].y, mj[u].z);
            }
            if (__any(cnt - done > LIST_STAGE - LIST_UNROLL)) flush();
        };
        auto scan_staged = [&](int st, int en, int2 sp) __attribute__((always_inline)) {
            const int lo = sp.x, hi = sp.y;
            if (lo == INT_MAX) return;
            if (hi - lo > LIST_WIN) {
                if (st < en) scan(st, en);
                return;
            }
            // up to three loads per lane in flight at once, so that most
            // unions take one memory round trip
            const int n = hi - lo;
            for (int e0 = 0; e0 < n; e0 += 3 * WAVE) {
                uint4 m[3];
#pragma unroll
                for (int t = 0; t < 3; ++t)
                    if (t == 0 || e0 + t * WAVE < n) m[t] = d.smirror[lo + min(e0 + t * WAVE + lane, n - 1)];
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    const int e = e0 + t * WAVE + lane;
                    if (e < n) {
                        if (coarse) {  // (x-y word, z word) pairs: one 8-byte read per candidate
                            wc[e] = make_uint2((m[t].x >> 16) | (m[t].y & 0xffff0000u), m[t].z >> 16);
                        } else {
                            wx[e] = m[t].x;
                            wy[e] = m[t].y;
                            wz[e] = m[t].z;
                        }
                    }
                }
                // No load of this pass is left in flight.  Stated, so that the
                // compiler need not wait for every load (the next row's bounds
                // among them) before it reuses these registers.
                __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
            int j = st;
            if (coarse) {
                for (; j + LIST_UNROLL <= en; j += LIST_UNROLL) {  // whole batches
                    const int o = j - lo;
#pragma unroll
                    for (int u = 0; u < LIST_UNROLL; ++u) test_coarse(j + u, true, wc[o + u].x, wc[o + u].y);
                    if (__any(cnt - done > LIST_STAGE - LIST_UNROLL)) flush();
                }
                if (j < en) {  // the last, partial batch
                    const int o = j - lo;
#pragma unroll
                    for (int u = 0; u < LIST_UNROLL; ++u) test_coarse(j + u, j + u < en, wc[o + u].x, wc[o + u].y);
                }
            } else {
                for (; j + LIST_UNROLL <= en; j += LIST_UNROLL) {  // whole batches
                    const int o = j - lo;
#pragma unroll
                    for (int u = 0; u < LIST_UNROLL; ++u) test(j + u, true, wx[o + u], wy[o + u], wz[o + u]);
                    if (__any(cnt - done > LIST_STAGE - LIST_UNROLL)) flush();
                }
                if (j < en) {  // the last, partial batch
                    const int o = j - lo;
#pragma unroll
                    for (int u = 0; u < LIST_UNROLL; ++u) test(j + u, j + u < en, wx[o + u], wy[o + u], wz[o + u]);
                }
            }
            if (__any(cnt - done > LIST_STAGE - LIST_UNROLL)) flush();
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
        };
        if (SJ.n > 0 && prune) {  // finer cells: per-particle pruning, direct scans
            if (real) {
                for (int oz = oz0; oz < oz0 + nz; ++oz) {
                    const double gz = fmax(gap(oz, cz, cw, uz), 0.0);
                    const int qz = (cz + oz + nc) % nc;
                    for (int oy = -reach; oy < -reach + noff; ++oy) {
                        const double gy = fmax(gap(oy, cy, cw, uy), 0.0);
                        const double g2 = gy * gy + gz * gz;
                        if (g2 > rp2) continue;
                        const int qy = (cy + oy + nc) % nc;
                        const int rowc = SJ.cell0 + (qz * nc + qy) * nc;  // cell (0, qy, qz)
                        int xl = -reach, xr = reach;
                        while (xl < 0) {
                            const double gx = gap(xl, cx, cw, ux);
                            if (gx * gx + g2 <= rp2) break;
                            ++xl;
                        }
                        while (xr > 0) {
                            const double gx = gap(xr, cx, cw, ux);
                            if (gx * gx + g2 <= rp2) break;
                            --xr;
                        }
                        const int a = cx + xl, b = cx + xr;  // unwrapped cell range [a, b]
                        if (a < 0) {
                            scan(cs(rowc + a + nc), ce(rowc + nc - 1));
                            scan(cs(rowc), ce(rowc + b));
                        } else if (b >= nc) {
                            scan(cs(rowc + a), ce(rowc + nc - 1));
                            scan(cs(rowc), ce(rowc + b - nc));
                        } else {
                            scan(cs(rowc + a), ce(rowc + b));
                        }
                    }
                }
            }
        } else if (SJ.n > 0) {  // every lane walks the same rows: staged scans
            // Slot ranges of one stencil row: the main run of cells, and the
            // end cell that wraps around the box where the row does.  Rows
            // are read one step ahead of their scan, so that the loads of a
            // row's bounds overlap the staging loads of the row before.
            int oz = oz0, oy = -reach;
            int4 next = bounds(oz, oy);
            int woff = 0;  // window offset of the next piece (staged)
            int g = 0;     // window group of the row (staged)
            for (int r = 0; r < nrow; ++r) {
                const int4 cur = next;
                const int2 sp1 = span(cur.x, cur.y), sp2 = span(cur.z, cur.w);
                // This row's bounds are used above, before the next row's
                // loads are issued: a wait for them placed after those loads
                // would wait for those loads too.
                __builtin_amdgcn_sched_barrier(0);
                // the next row; after the last one, row 0 again (read, not used)
                if (++oy == -reach + noff) {
                    oy = -reach;
                    if (++oz == oz0 + nz) oz = oz0;
                }
                next = bounds(oz, oy);
                if (staged && ((gbound >> r) & 1u)) {
                    // close group g: every lane's entries up to a common
                    // count (a multiple of the force kernels' 4 entries per
                    // step), padded with its own copy of group g's window
                    const int wg = g == 0 ? gw0 : (g == 1 ? gw1 : (g == 2 ? gw2 : gw3));
                    const int pv = wg + lane;
                    const int kend = (wave_max_all(cnt) + 3) & ~3;
                    while (__any(cnt < kend)) {
                        if (cnt < kend) {
                            buf[cnt & (LIST_STAGE - 1)][lane] = pv;
                            ++cnt;
                            ++npad;
                        }
                        if (__any(cnt - done > LIST_STAGE - LIST_UNROLL)) flush();
                    }
                    if (lane == 0 && g < STAGE_GROUPS) gtab[g].z = kend;
                    ++g;
                    woff = 0;
                }
                if (staged && sp1.x != INT_MAX) {
                    dl = woff - sp1.x;
                    woff += sp1.y - sp1.x;
                }
                scan_staged(cur.x, cur.y, sp1);
                if (staged && sp2.x != INT_MAX) {
                    dl = woff - sp2.x;
                    woff += sp2.y - sp2.x;
                }
                scan_staged(cur.z, cur.w, sp2);
            }
            dl = 0;
        }
        flush();
        total += cnt - npad;
        // padding: the own slot, or in a window the lane's own position copy
        // (of the last group's window)
        const int wlast = ngroup == 1 ? gw0 : (ngroup == 2 ? gw1 : (ngroup == 3 ? gw2 : gw3));
        const int padv = staged ? wlast + lane : s;
        int kmax = wave_max_all(cnt);
        const int align = half ? 2 * LIST_ROW_ALIGN : LIST_ROW_ALIGN;  // whole 16-byte words
        kmax = (kmax + align - 1) / align * align;
        if (done < cnt) {  // the last partial group, padded with the particle's own slot
            const int k = row + (half ? done / 2 : done);
            int e[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) e[t] = done + t < cnt ? buf[(done + t) & (LIST_STAGE - 1)][lane] : padv;
            const int4 q = half ? make_int4(pack(e[0], e[1]), pack(e[2], e[3]), pack(e[4], e[5]), pack(e[6], e[7]))
                                : make_int4(e[0], e[1], e[2], e[3]);
            if (k < rows) *reinterpret_cast<int4 *>(col + (k >> 2) * 256) = q;
            done += group;
        }
        const int words = half ? kmax / 2 : kmax;  // 32-bit words the part occupies
        const int pad = half ? pack(padv, padv) : padv;
        for (int k = row + (half ? done / 2 : done); k < row + words && k < rows; k += 4)
            *reinterpret_cast<int4 *>(col + (k >> 2) * 256) = make_int4(pad, pad, pad, pad);
        if (row + words > rows && lane == 0) set_err(d.err, KAMD_DEV_LIST_OVERFLOW);
        // selects rather than an array indexed by the part, which would
        // live in scratch memory when this loop is not unrolled
        kpart.x = tj == 0 ? kmax : kpart.x;
        kpart.y = tj == 1 ? kmax : kpart.y;
        const int code = staged ? -2 : base;  // -2: entries are offsets into window groups
        bpart.x = tj == 0 ? code : bpart.x;
        bpart.y = tj == 1 ? code : bpart.y;
        pcnt.x = tj == 0 ? (staged ? ngroup : 0) : pcnt.x;
        pcnt.y = tj == 1 ? (staged ? ngroup : 0) : pcnt.y;
        if (half) n16 += cnt - npad - (tj == S.type ? 1 : 0);  // 16-bit partner entries (not the own slot)
        row += words;
    }
    if (row > rows) {  // keep the force kernels inside the list
        if (lane == 0) atomicMax(&d.counters[3], row);  // the rows a healing rebuild must provide
        kpart = cut_to_rows(kpart, bpart, rows);
    }
    if (lane == 0) {
        d.kmax[w] = kpart;
        d.lbase[w] = bpart;
        d.pcount[w] = pcnt;
    }
    // partners (without the own slot) in the low 16 bits, those of them
    // stored as 16-bit entries in the high 16 bits
    d.nlen[s] = real ? (total - 1) | (n16 << 16) : 0;
}

// {m, d} shifted left by one: m with the sign bit of d appended.
__device__ inline uint32_t push_sign(uint32_t m, int d) { return __builtin_amdgcn_alignbit(m, (uint32_t)d, 31); }

// x + o on a ring of nc cells, -1 <= o <= 1, 0 <= x < nc.
__device__ inline int ring_cell(int x, int o, int nc)
{
    x += o;
    x += x < 0 ? nc : 0;
    return x >= nc ? x - nc : x;
}

// The list builder of k_rb_list for one cell per list radius, boxes of the
// coarse test and no windows: the same rows and entries, but a row's candidates
// are tested 32 at a time into a bit mask per lane (five vector operations each:
// two subtractions, two dot products, one shift that appends the sign; k_rb_list
// spends ten, with a stage write per candidate).  Only the accepted ones, about a
// sixth, are then taken out of the masks, and not as they come: the masks of 64
// candidates go into a queue in LDS per lane, and at the end of the part (or when
// the queue is full) every lane takes its next entries from its own queue, all
// lanes in step.  A 16-byte piece of every list is thus complete in registers
// at the same time, and the steps are those of the longest list, 110, where
// emptying each mask before the next tests took 350 at a quarter of the lanes.
//
// Candidates are read from an 8-byte copy of the sorted mirror that the sort
// writes (scoarse), two per load.  Staging the rows' unions in LDS first costs
// more (the unions, the copies, and the LDS that limits the occupancy) than it
// takes off the vector cache: 511 us per build against 469.  Cells of a row are
// found without divisions, and the wrapped piece is looked at only where a lane
// has one.  Queues of 8 / 10 / 12 entries: 490 / 482 / 487 us.  Five wavefronts
// per SIMD (96 registers; the particle's own position is read again at the end
// for that): 482 -> 469.
//
// Bound by the vector ALU (9,200 instructions per wavefront; 14,800 in k_rb_list)
// and the candidate loads (430 per wavefront).  Measured, a build (sort and
// lists, k_rb_list / masks emptied at once / this): 2^20 particles - / 537 / 469
// us, 100,000 - / 143 / 121, 256 replicas of 4096 - / 600 / 503; the 2^20 MIXED
// step 310 / 287 / 276.
__global__ __launch_bounds__(BLOCK, 5) void k_rb_list_masks(Dev d, int min_waves)
{
    __shared__ uint32_t queue[WAVES_PER_BLOCK][LIST_QUEUE][3][WAVE];  // two masks, the entry of the first bit
    if (d.rb_any[0] < min_waves) return;  // nothing to do, or k_rb_list_wide's
    const int w = rb_work_wave(d);        // each XCD walks a contiguous part of the worklist
    if (w < 0) return;
    const int lane = lane_id();
    const int s = w * WAVE + lane;
    uint4 mi = d.smirror[s];
    const SegInfo &S = d.seg[d.wave_seg[w]];
    const RepInfo &R = d.rep[S.rep];
    const bool real = (s - S.slot0) < S.n;
    if (!real) mi = make_uint4(0, 0, 0, 0);
    const int nc = R.nc;
    const int noff = min(nc, 3);
    const bool whole = nc < 3;  // every cell of a row is in the stencil
    const int oz0 = d.dim == 2 ? 0 : -1, nz = d.dim == 2 ? 1 : noff;
    const int nrow = nz * noff;
    const int fx = fix_cell(mi.x, CELL_SUBX * nc);  // x in quarter cells
    const int cx = fx / CELL_SUBX, qx = fx % CELL_SUBX;
    const int cy = fix_cell(mi.y, nc), cz = d.dim == 2 ? 0 : fix_cell(mi.z, nc);
    const uint32_t ixy = coarse_of(mi).x, iz = coarse_of(mi).y;
    // sub-cells of the lane's main run within a row, and of the end cell that
    // wraps around (see k_rb_list): first and last of each
    const bool lw = !whole && cx == 0, rw = !whole && cx == nc - 1;
    const int m0 = whole || lw ? 0 : CELL_SUBX * (cx - 1) + qx;
    const int m1 = whole || rw ? CELL_SUBX * nc - 1 : CELL_SUBX * (cx + 1) + qx;
    const int e0 = lw ? CELL_SUBX * (nc - 1) + qx : 0, e1 = lw ? CELL_SUBX * nc - 1 : qx;
    const bool wraps = lw || rw;
    const bool any_wrap = __any(real && wraps);
    int32_t *col = d.nbr + list_index(w, d.rows, 0, lane);
    uint32_t(*q)[3][WAVE] = queue[threadIdx.x / WAVE];
    const int rows = d.rows;
    const int32_t *cstart = d.cell_start, *cend = d.cell_start + 1;
    int row = 0;  // 32-bit words of the list used so far
    int total = 0;
    int2 kpart = make_int2(0, 0), bpart = make_int2(-1, -1);  // per part: entries, base
    int n16 = 0;
#pragma unroll 1
    for (int tj = 0; tj < 2; ++tj) {
        const SegInfo &SJ = d.seg[R.seg[tj]];
        const int r2c = R.r2c[S.type + tj];
        const int cell0 = SJ.cell0;
        // base slot of 16-bit entries (the part of the own type), or -1
        int base = -1;
        if (tj == S.type && SJ.n > 0) base = own_base(d, cell0, s, real, cy, cz, 1, noff, oz0, nz, nc);
        const bool half = base >= 0;
        const int group = half ? 8 : 4;    // entries per 16-byte store
        const int sub = half ? base : 0;   // entries are held as the list stores them
        const int padv = s - sub;          // padding: the own slot
        int cnt = 0;                       // entries accepted
        int emitted = 0;                   // of those, written (a multiple of group)
        int qh = 0, qn = 0;                // queue: first entry, entries
        uint32_t ma = 0, mb = 0;           // the queue entry being taken apart
        int ent = 0;
        auto take = [&]() __attribute__((always_inline)) {
            if (ma == 0) {
                if (mb) {
                    ma = mb;
                    ent += 32;
                    mb = 0;
                } else if (qn) {
                    ma = q[qh][0][lane];
                    mb = q[qh][1][lane];
                    ent = (int)q[qh][2][lane];
                    qh = qh == LIST_QUEUE - 1 ? 0 : qh + 1;
                    --qn;
                }
            }
            const int e = ma ? ent + __builtin_ctz(ma) : padv;
            ma &= ma - 1;
            return e;
        };
        auto write = [&](int4 v) __attribute__((always_inline)) {
            const int k = row + (half ? emitted / 2 : emitted);  // 32-bit word of the list
            if (k < rows) *reinterpret_cast<int4 *>(col + (k >> 2) * 256) = v;
            emitted += group;
        };
        auto emit = [&]() __attribute__((always_inline)) {  // the lane's next group of entries
            int e[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                e[t] = take();
                if (half) e[t] |= take() << 16;
            }
            write(make_int4(e[0], e[1], e[2], e[3]));
        };
        // The queue of some lane is full: as many groups as every lane has
        // entries for or, where one has too few, one group of those that have
        // (the full one among them: each entry of its queue holds a partner).
        auto make_room = [&]() __attribute__((always_inline)) {
            const int have = -wave_max_all(real ? emitted - cnt : -INT_MAX);
            if (have >= group) {
#pragma unroll 1
                for (int k = group; k <= have; k += group) emit();
            } else if (cnt - emitted >= group) {
                emit();
            }
        };
        // slot ranges of one stencil row: main run and wrapped end cell
        auto bounds = [&](int oz, int oy) __attribute__((always_inline)) {
            int4 b = make_int4(0, 0, 0, 0);
            if (real) {
                const int rowc = CELL_SUBX * (cell0 + (ring_cell(cz, oz, nc) * nc + ring_cell(cy, oy, nc)) * nc);
                b.x = cstart[rowc + m0];
                b.y = cend[rowc + m1];
                if (wraps) {
                    b.z = cstart[rowc + e0];
                    b.w = cend[rowc + e1];
                }
            }
            return b;
        };
        // two candidates with one load (their address is a multiple of 8 only)
        typedef uint32_t pair8 __attribute__((ext_vector_type(4), aligned(8)));
        // 32 candidates from slot j, candidate i's bit in bit i; left: how many are the lane's
        auto test32 = [&](int j, int left) __attribute__((always_inline)) {
            const int ng = 1 + (__any(left > 8) ? 1 : 0) + (__any(left > 16) ? 1 : 0) + (__any(left > 24) ? 1 : 0);
            const uint2 *v = d.scoarse + (left > 0 ? j : s);  // with spare entries past its end
            uint32_t m = 0;
#pragma unroll 1
            for (int g = 0; g < ng; ++g, v += 8) {
                pair8 c[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) c[i] = *reinterpret_cast<const pair8 *>(v + 2 * i);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    m = push_sign(m, r2_coarse_below(ixy, iz, c[i].x, c[i].y, r2c));
                    m = push_sign(m, r2_coarse_below(ixy, iz, c[i].z, c[i].w, r2c));
                }
            }
            m = __brev(m << (32 - 8 * ng));
            return left >= 32 ? m : left > 0 ? m & ~(0xffffffffu << left) : 0u;
        };
        auto piece = [&](int st, int en) __attribute__((always_inline)) {
#pragma unroll 1
            for (int j = st; __any(j < en); j += 64) {
                uint32_t a = test32(j, en - j), b = 0;
                if (__any(j + 32 < en)) b = test32(j + 32, en - j - 32);
                while (__any(qn == LIST_QUEUE)) make_room();
                if (a | b) {
                    int at = qh + qn;
                    at -= at >= LIST_QUEUE ? LIST_QUEUE : 0;
                    q[at][0][lane] = a ? a : b;
                    q[at][1][lane] = a ? b : 0u;
                    q[at][2][lane] = (uint32_t)(j - sub + (a ? 0 : 32));
                    ++qn;
                    cnt += __popc(a) + __popc(b);
                }
            }
        };
        if (SJ.n > 0) {
            // rows are read one step ahead of their scan, so that the loads of
            // a row's bounds overlap the staging loads of the row before
            int oz = oz0, oy = -1;
            int4 next = bounds(oz, oy);
#pragma unroll 1
            for (int r = 0; r < nrow; ++r) {
                const int4 cur = next;
                // the next row; after the last one, row 0 again (read, not used)
                if (++oy == -1 + noff) {
                    oy = -1;
                    if (++oz == oz0 + nz) oz = oz0;
                }
                next = bounds(oz, oy);
                piece(cur.x, cur.y);
                if (any_wrap) piece(cur.z, cur.w);
            }
        }
        while (__any(emitted < cnt))
            if (emitted < cnt) emit();
        total += cnt;
        const int kmax = (wave_max_all(cnt) + group - 1) & -group;  // whole 16-byte words
        const int words = half ? kmax / 2 : kmax;  // 32-bit words the part occupies
        const int pad = half ? padv | (padv << 16) : padv;
        while (__any(emitted < kmax))
            if (emitted < kmax) write(make_int4(pad, pad, pad, pad));
        if (row + words > rows && lane == 0) set_err(d.err, KAMD_DEV_LIST_OVERFLOW);
        kpart.x = tj == 0 ? kmax : kpart.x;
        kpart.y = tj == 1 ? kmax : kpart.y;
        bpart.x = tj == 0 ? base : bpart.x;
        bpart.y = tj == 1 ? base : bpart.y;
        if (half) n16 += cnt - 1;  // 16-bit partner entries (not the own slot)
        row += words;
    }
    if (row > rows) {  // keep the force kernels inside the list
        if (lane == 0) atomicMax(&d.counters[3], row);  // the rows a healing rebuild must provide
        kpart = cut_to_rows(kpart, bpart, rows);
    }
    if (lane == 0) {
        d.kmax[w] = kpart;
        d.lbase[w] = bpart;
        d.pcount[w] = make_int2(0, 0);
    }
    // partners (without the own slot) in the low 16 bits, those of them
    // stored as 16-bit entries in the high 16 bits
    d.nlen[s] = real ? (total - 1) | (n16 << 16) : 0;
    mi = d.smirror[s];  // again: its registers are worth more in between
    if (!real) mi = make_uint4(0, 0, 0, 0);
    copy_back(d, s, real, mi);
}

// Neighbour lists, a block of LIST_ROWS wavefronts per listed wave: wavefront r
// takes stencil row r of both partner types.  The lists are those of k_rb_list
// (one cell per list radius, no windows, coarse test), entry for entry.
//
// Why: a wave's lists are a chain of 18 row pieces (bounds, union, staging,
// scan), and a lone wavefront takes 100 us for it however small the system;
// on the steps of a batch where a few replicas rebuild it is as long.  Here
// the rows run side by side.  A wavefront stages the unions of its row's pieces
// that fit its LDS window (the others it reads from global memory) and tests
// the candidates 32 at a time into bit masks (five vector operations each);
// the rows' counts then give every lane the place of its entries, and the
// accepted ones, about a sixth, go from the masks into an LDS image of the
// wave's lists (slots relative to the replica's first, 16 bits), which the
// block writes out 16 bytes a lane.  A wave with rows of more chunks than there
// are masks, or lists longer than the image, is scanned a second time and
// stored entry by entry.
//
// Bound by latency and, inside its compute unit, by the vector ALU: of 19 us a
// block, 2.4 are the chain of dependent loads up to the cell ranges, 2.8 the
// staging, 4.7 the tests and 4.8 the expansion of the middle row.  A rebuild of
// one to 256 waves takes 27 us, of k_rb_list 100 us.
constexpr int LIST_ROWS = 9;
constexpr int WIDE_WIN = 432;     // candidates staged per wavefront
constexpr int WIDE_CHUNKS = 8;    // masks per wavefront
constexpr int WIDE_LIST = 192;    // entries of the list image
constexpr int WIDE_BLOCKS = 512;  // two blocks of nine wavefronts per compute unit

__global__ __launch_bounds__(WAVE * LIST_ROWS) void k_rb_list_wide(Dev d, int max_waves)
{
    // the windows (a chunk reads up to 31 past a range), then the list image
    __shared__ union {
        uint2 win[LIST_ROWS][WIDE_WIN + 32];
        uint16_t fin[WIDE_LIST + 1][WAVE];  // and a row that takes the rejected
    } u;
    __shared__ uint32_t mask_s[LIST_ROWS][WIDE_CHUNKS][WAVE];
    __shared__ uint16_t rowcnt[2][LIST_ROWS][WAVE];
    const int nact = d.rb_any[0];
    if (nact == 0 || nact > max_waves) return;
    const int nrw = blockDim.x / WAVE;  // rows at most: 9, or 3 of a planar system
    const int r = threadIdx.x / WAVE, lane = lane_id();
    const int np = d.npad_total, rows = d.rows;
    uint2 *wc = u.win[r];
    uint16_t(*fin)[WAVE] = u.fin;
    uint32_t(*mk)[WAVE] = mask_s[r];
    for (int i0 = 0; i0 < nact; i0 += gridDim.x) {
        const int nb = min((int)gridDim.x, nact - i0);
        if ((int)blockIdx.x >= nb) return;  // block-uniform
        const int w = d.rb_wlist[i0 + xcd_block(blockIdx.x, nb)];
        const int s = w * WAVE + lane;
        uint4 mi = d.smirror[s];
        // the sorted state, for its way back at the end: wavefront r takes the
        // FP64 arrays r, r + nrw, ... and a share of the others
        double sv[3];
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (k == 0 || nrw == 3) sv[k] = ld_stream(&d.sx[(size_t)(r + 3 * k) * np + s]);
        const int vi = r < 3 ? ld_stream(&d.simg[r * np + s]) : 0;
        const SegInfo &S = d.seg[d.wave_seg[w]];
        const RepInfo &R = d.rep[S.rep];
        const bool real = (s - S.slot0) < S.n;
        if (!real) mi = make_uint4(0, 0, 0, 0);
        const int nc = R.nc, slot0 = R.wave0 * WAVE;
        const int noff = min(nc, 3);
        const bool whole = nc < 3;  // every cell of a row is in the stencil
        const int oz0 = d.dim == 2 ? 0 : -1, nz = d.dim == 2 ? 1 : noff;
        const bool active = r < nz * noff;
        const int oz = oz0 + r / noff, oy = -1 + r % noff;
        const int fx = fix_cell(mi.x, CELL_SUBX * nc);  // x in quarter cells
        const int cx = fx / CELL_SUBX, qx = fx % CELL_SUBX;
        const int cy = fix_cell(mi.y, nc), cz = d.dim == 2 ? 0 : fix_cell(mi.z, nc);
        const uint32_t ixy = coarse_of(mi).x, iz = coarse_of(mi).y;
        const int32_t *cstart = d.cell_start, *cend = d.cell_start + 1;
        // pieces of the lane's row: per partner type the main run of cells and
        // the end cell that wraps around (see k_rb_list); [st, en) in slots
        int st_[4], en_[4];
#pragma unroll
        for (int tj = 0; tj < 2; ++tj) {
            const SegInfo &SJ = d.seg[R.seg[tj]];
            st_[2 * tj] = en_[2 * tj] = st_[2 * tj + 1] = en_[2 * tj + 1] = 0;
            if (real && active && SJ.n > 0) {
                const int qz = (cz + oz + nc) % nc, qy = (cy + oy + nc) % nc;
                const int rowc = SJ.cell0 + (qz * nc + qy) * nc;
                if (whole) {
                    st_[2 * tj] = cstart[CELL_SUBX * rowc];
                    en_[2 * tj] = cend[CELL_SUBX * (rowc + nc) - 1];
                } else {
                    const int a = cx - 1, e = cx + 1;
                    st_[2 * tj] = cstart[a < 0 ? CELL_SUBX * rowc : CELL_SUBX * (rowc + a) + qx];
                    en_[2 * tj] = cend[e >= nc ? CELL_SUBX * (rowc + nc) - 1 : CELL_SUBX * (rowc + e) + qx];
                    const bool lw = a < 0;
                    if (lw || e >= nc) {
                        st_[2 * tj + 1] = cstart[lw ? CELL_SUBX * (rowc + a + nc) + qx : CELL_SUBX * rowc];
                        en_[2 * tj + 1] = cend[lw ? CELL_SUBX * (rowc + nc) - 1 : CELL_SUBX * (rowc + e - nc) + qx];
                    }
                }
            }
        }
        // base slot of 16-bit entries (the part of the own type), or -1
        const int base = own_base(d, d.seg[R.seg[S.type]].cell0, s, real, cy, cz, 1, noff, oz0, nz, nc);
        // Unions over the lanes, staged one after the other while they fit;
        // longest range and chunks of each piece.  (The loops over the pieces
        // stay rolled: the kernel runs for some 20 us, and four copies of its
        // loops cost more in instruction fetches than the selects do.)
        auto sel = [](int4 v, int p) __attribute__((always_inline)) {
            int x = v.x;
            x = p == 1 ? v.y : x;
            x = p == 2 ? v.z : x;
            return p == 3 ? v.w : x;
        };
        auto vec = [](const int (&v)[4]) __attribute__((always_inline)) { return make_int4(v[0], v[1], v[2], v[3]); };
        int lo_[4], off_[4], long_[4], used = 0, chunks = 0;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const bool has = st_[p] < en_[p];
            long_[p] = wave_max_all(en_[p] - st_[p]);
            lo_[p] = has ? st_[p] : INT_MAX;
            lo_[p] = -wave_max_all(-lo_[p]);
            const int len = wave_max_all(has ? en_[p] : -1) - lo_[p];
            const bool fits = long_[p] > 0 && used + len <= WIDE_WIN;
            chunks += (long_[p] + 31) / 32;
            off_[p] = fits ? used : -1;
            used += fits ? len : 0;
        }
        const int4 st = vec(st_), en = vec(en_), lo = vec(lo_), off = vec(off_), longest = vec(long_);
#pragma unroll 1
        for (int p = 0; p < 4; ++p) {
            const int o = sel(off, p);
            if (o < 0) continue;
            int next = used;  // where the next staged piece starts
            for (int q = 3; q > p; --q) next = sel(off, q) >= 0 ? sel(off, q) : next;
            const int len = next - o;
            const uint2 *src = d.scoarse + sel(lo, p);
            for (int e = lane; e < len; e += 2 * WAVE) {
                const uint2 a = src[e], b = src[min(e + WAVE, len - 1)];
                wc[o + e] = a;
                if (e + WAVE < len) wc[o + e + WAVE] = b;
            }
        }
        const bool masked = chunks <= WIDE_CHUNKS;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // the general path: every candidate of the lane's ranges in slot
        // order, from global memory: take(part, j) for the accepted ones
        auto walk = [&](auto take) __attribute__((always_inline)) {
#pragma unroll 1
            for (int p = 0; p < 4; ++p) {
                const int r2c = R.r2c[S.type + (p >> 1)], e = sel(en, p);
#pragma unroll 1
                for (int j = sel(st, p); j < e; ++j) {
                    const uint2 v = d.scoarse[j];
                    if (r2_coarse_below(ixy, iz, v.x, v.y, r2c) < 0) take(p >> 1, j);
                }
            }
        };
        int cnt0 = 0, cnt1 = 0;
        if (masked) {
            int c = 0;
#pragma unroll 1
            for (int p = 0; p < 4; ++p) {
                const int r2c = R.r2c[S.type + (p >> 1)], top = sel(longest, p), o = sel(off, p), l = sel(lo, p);
                const int a = sel(st, p), len = sel(en, p) - a;
#pragma unroll 1
                for (int k = 0; k < top; k += 32, ++c) {
                    const int n = min(max(len - k, 0), 32);  // candidates of the lane's chunk
                    const int j = n > 0 ? a + k : l;
                    const int ng = (min(top - k, 32) + 7) / 8;
                    uint32_t m = 0;
                    if (o >= 0) {
                        const uint2 *v = wc + (o + j - l);
#pragma unroll 1
                        for (int g = 0; g < ng; ++g, v += 8)
#pragma unroll
                            for (int i = 0; i < 8; ++i) m = push_sign(m, r2_coarse_below(ixy, iz, v[i].x, v[i].y, r2c));
                    } else {
                        const uint2 *v = d.scoarse + j;  // with spare entries past its end
#pragma unroll 1
                        for (int g = 0; g < ng; ++g, v += 8) {
                            uint2 q[8];
#pragma unroll
                            for (int i = 0; i < 8; ++i) q[i] = v[i];
#pragma unroll
                            for (int i = 0; i < 8; ++i) m = push_sign(m, r2_coarse_below(ixy, iz, q[i].x, q[i].y, r2c));
                        }
                    }
                    m <<= 32 - 8 * ng;  // candidate i of the chunk in bit 31 - i
                    m = n > 0 ? m & (0xffffffffu << (32 - n)) : 0u;
                    mk[c][lane] = m;
                    cnt0 += p < 2 ? __popc(m) : 0;
                    cnt1 += p < 2 ? 0 : __popc(m);
                }
            }
        } else {
            walk([&](int tj, int) __attribute__((always_inline)) {
                cnt0 += 1 - tj;
                cnt1 += tj;
            });
        }
        rowcnt[0][r][lane] = (uint16_t)cnt0;
        rowcnt[1][r][lane] = (uint16_t)cnt1;
        const bool all_masked = __syncthreads_and(masked) != 0;
        int at0 = 0, at1 = 0, tot0 = 0, tot1 = 0;
#pragma unroll 1
        for (int q = 0; q < nrw; ++q) {
            const int a = rowcnt[0][q][lane], b = rowcnt[1][q][lane];
            at0 += q < r ? a : 0;
            at1 += q < r ? b : 0;
            tot0 += a;
            tot1 += b;
        }
        int2 kpart, bpart = make_int2(S.type == 0 ? base : -1, S.type == 1 ? base : -1);
        const bool h0 = bpart.x >= 0, h1 = bpart.y >= 0;
        const int al0 = h0 ? 2 * LIST_ROW_ALIGN : LIST_ROW_ALIGN, al1 = h1 ? 2 * LIST_ROW_ALIGN : LIST_ROW_ALIGN;
        kpart.x = (wave_max_all(tot0) + al0 - 1) & -al0;
        kpart.y = (wave_max_all(tot1) + al1 - 1) & -al1;
        const int row1 = h0 ? kpart.x / 2 : kpart.x;  // 32-bit words of the A part
        const int used_rows = row1 + (h1 ? kpart.y / 2 : kpart.y);
        int32_t *col = d.nbr + list_index(w, rows, 0, lane);
        if (all_masked && kpart.x + kpart.y <= WIDE_LIST) {  // block-uniform: through the image
            uint16_t *out = &fin[at0][lane], *dump = &fin[WIDE_LIST][lane];
            int c = 0;
#pragma unroll 1
            for (int p = 0; p < 4; ++p) {
                const int top = sel(longest, p);
                if (p == 2) out = &fin[kpart.x + at1][lane];
                int j = sel(st, p) - slot0;
#pragma unroll 1
                for (int k = 0; k < top; k += 32, ++c) {
                    int m = (int)mk[c][lane];
                    const int ng = (min(top - k, 32) + 7) / 8;
#pragma unroll 1
                    for (int g = 0; g < ng; ++g) {
                        // a rejected candidate goes to the dump row and leaves the place free
#pragma unroll
                        for (int i = 0; i < 8; ++i, ++j, m <<= 1) {
                            *(m < 0 ? out : dump) = (uint16_t)j;
                            out += m < 0 ? WAVE : 0;
                        }
                    }
                }
            }
            // padding up to the wavefront's longest part: the own slot
#pragma unroll 1
            for (int k = tot0 + r; k < kpart.x; k += nrw) fin[k][lane] = (uint16_t)(s - slot0);
#pragma unroll 1
            for (int k = tot1 + r; k < kpart.y; k += nrw) fin[kpart.x + k][lane] = (uint16_t)(s - slot0);
            __syncthreads();
#pragma unroll 1
            for (int q = r; q < (min(used_rows, rows) >> 2); q += nrw) {  // 16-byte words of the lists
                const bool second = 4 * q >= row1;
                const int kw = second ? 4 * q - row1 : 4 * q;  // word of the part
                const bool half = second ? h1 : h0;
                const uint16_t(*f)[WAVE] = fin + (second ? kpart.x : 0) + (half ? 2 * kw : kw);
                int4 v;
                if (half) {
                    int e[8];
#pragma unroll
                    for (int t = 0; t < 8; ++t) e[t] = f[t][lane] + slot0 - base;
                    v = make_int4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
                } else {
                    v = make_int4(f[0][lane] + slot0, f[1][lane] + slot0, f[2][lane] + slot0, f[3][lane] + slot0);
                }
                *reinterpret_cast<int4 *>(col + q * 256) = v;
            }
        } else {
            auto put = [&](int tj, int k, int j) __attribute__((always_inline)) {
                const bool half = tj ? h1 : h0;
                const int kw = (tj ? row1 : 0) + (half ? k >> 1 : k);
                if (kw >= rows) return;
                int32_t *q = col + (kw >> 2) * 256 + (kw & 3);
                if (half) reinterpret_cast<uint16_t *>(q)[k & 1] = (uint16_t)(j - base);
                else *q = j;
            };
            walk([&](int tj, int j) __attribute__((always_inline)) {
                put(tj, tj ? at1 : at0, j);
                at0 += 1 - tj;
                at1 += tj;
            });
            for (int tj = 0; tj < 2; ++tj)
                for (int k = (tj ? tot1 : tot0) + r; k < (tj ? kpart.y : kpart.x); k += nrw) put(tj, k, s);
        }
        // the sorted state back into place (last: a wait for loaded data would
        // wait for these stores too)
        if (real) {
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (k == 0 || nrw == 3) st_stream(sv[k], &d.x[(size_t)(r + 3 * k) * np + s]);
            if (r < 3) st_stream(vi, &d.img[r * np + s]);
            if (r == nrw - 1) st_stream(ld_stream(&d.sid[s]), &d.id[s]);
            if (r == nrw - 2) {
                d.mirror[s] = mi;  // gathered by the next step: cached
                st_stream(mi, &d.mbuild[s]);
            }
        }
        if (d.pos4 && r == nrw - 1)  // FP64: gathers see the new order
            d.pos4[s] = real ? make_double4(d.sx[s], d.sy[s], d.sz[s], 0.0) : make_double4(d.x[s], d.y[s], d.z[s], 0.0);
        if (r == 0) {
            int2 kp = kpart;
            if (used_rows > rows) {  // keep the force kernels inside the list
                if (lane == 0) {
                    set_err(d.err, KAMD_DEV_LIST_OVERFLOW);
                    atomicMax(&d.counters[3], used_rows);  // the rows a healing rebuild must provide
                }
                kp = cut_to_rows(kpart, bpart, rows);
            }
            if (lane == 0) {
                d.kmax[w] = kp;
                d.lbase[w] = bpart;
                d.pcount[w] = make_int2(0, 0);
            }
            const int n16 = base >= 0 ? (S.type == 0 ? tot0 : tot1) - 1 : 0;
            d.nlen[s] = real ? (tot0 + tot1 - 1) | (n16 << 16) : 0;
        }
        __syncthreads();  // the image is read before the next windows come
    }
}

static inline int nblk_slots(const Dev &d) { return (d.nwaves + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK; }
constexpr int CHAIN_MAX_BLOCKS = 1024;  // grid cap of the grid-stride chain kernels
static inline int nblk_capped(int waves) { return std::min((waves + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK, CHAIN_MAX_BLOCKS); }

constexpr int SORT_GATHER_WAVES = 48;  // N = 3000: equal either way
// Measured (us per MIXED step, each block for itself / the gate first / the other
// chain): 256 replicas of 100 19.6 / 20.5 / 24.2, 512 32.9 / 32.0 / 35.7, 1024
// 50.5 / 44.3 / 47.4, 4096 215 / 104 / 104, 16,384 2352 / 388 / 379; 256 of 1000
// 86.5 / 88.0 / 91.5, 700 184.4 / 183.3 / 186.1.
constexpr int SORT_ALONE_REPS = 384;
template <bool GATHER>
static void launch_sort_small(const Dev &d, hipStream_t s)
{
    if (d.nrep <= SORT_ALONE_REPS) {
        hipLaunchKernelGGL((k_rb_sort_small<GATHER, false>), dim3(d.nrep), dim3(SORT_THREADS), 0, s, d);
    } else {
        hipLaunchKernelGGL(k_rb_gate, dim3(1), dim3(GATE_THREADS), 0, s, d);
        hipLaunchKernelGGL((k_rb_sort_small<GATHER, true>), dim3(d.nrep), dim3(SORT_THREADS), 0, s, d);
    }
}
hipError_t launch_rb_sort_small(const Dev &d, hipStream_t s)
{
    if (d.rep_waves_max <= SORT_GATHER_WAVES) {
        launch_sort_small<true>(d, s);
    } else {
        launch_sort_small<false>(d, s);
        hipLaunchKernelGGL(k_rb_gather, dim3(nblk_capped(d.nwaves)), dim3(BLOCK), 0, s, d);
    }
    return hipGetLastError();
}
hipError_t launch_rb_gate(const Dev &d, hipStream_t s)  // a single replica: k_rb_assign decides
{
    if (d.nrep > 1) hipLaunchKernelGGL(k_rb_gate, dim3(1), dim3(GATE_THREADS), 0, s, d);
    return hipGetLastError();
}
hipError_t launch_rb_assign(const Dev &d, hipStream_t s)
{
    hipLaunchKernelGGL(k_rb_assign, dim3(nblk_capped(d.nwaves)), dim3(BLOCK), 0, s, d);
    return hipGetLastError();
}
hipError_t launch_rb_scan(const Dev &d, int nseg, hipStream_t s)
{
    const dim3 grid(nseg, d.scan_cps);
    if (d.scan_cps > SCAN_DIRECT) hipLaunchKernelGGL(k_rb_scan_sum, grid, dim3(SCAN_THREADS), 0, s, d);
    hipLaunchKernelGGL(k_rb_scan, grid, dim3(SCAN_THREADS), 0, s, d);
    return hipGetLastError();
}
hipError_t launch_rb_sortgather(const Dev &d, hipStream_t s)
{
    hipLaunchKernelGGL(k_rb_sortgather, dim3(nblk_capped(d.nwaves)), dim3(BLOCK), 0, s, d);
    return hipGetLastError();
}
// Which list builder: the wide one for short worklists where it can build them
// (one cell per list radius, boxes of the coarse test, replicas of up to 2^16
// slots, no windows), k_rb_list_masks otherwise, k_rb_list for finer cells,
// windows and larger boxes.
//
// A single system rebuilds all its waves or none, so only one of the two is
// launched.  Measured (us per NVE step, masks / wide, MIXED and MIXED_FIXED):
// 32,000 particles (501 waves) 28.6 / 25.1 and 27.0 / 23.5; 40,000 (626) 30.2 /
// 29.0 and 30.0 / 28.7; 45,000 (704) 30.6 / 29.7 and 30.1 / 29.1; 50,000 (782)
// 33.0 / 33.1 and 33.6 / 33.5; 55,000 (860) 33.1 / 33.6 and 33.2 / 33.7; 62,000
// (970) 33.2 / 33.8 and 33.0 / 33.6.
//
// A batch launches both and the worklist decides, except where its worklists are
// hardly ever that short (the extra launch would cost 256 replicas of 250 to 8000
// particles 0.5%).  Limits of 800 / 1100 / 1280 / 1600: baths of 64 replicas of 1000
// (worklists of up to 1088) 40.5 / 39.2 / 39.2 / 39.2, 75 (1275) 43.7 / 43.7 / 42.5 /
// 42.5, 96 (1632) 53.4 / 53.9 / 54.0 / 54.2, 128 62.9 / 63.0 / 63.4 / 64.0; NVE of 10 x
// 8000 (1260) 51.0 / 50.9 / 49.6 / 49.6, 16 x 8000 63.1 / 62.9 / 63.5 / 64.3, 256 x
// 1000 104.0 / 104.8 / 107.3 / 110.4, 64 of 250 to 8000 114.0 / 114.3 / 115.0 / 119.6.
constexpr int WIDE_WAVES = 768, WIDE_BATCH_LIST = 1280, WIDE_BATCH_WAVES = 8192;
hipError_t launch_rb_list(const Dev &d, int cell_div, hipStream_t s)
{
    const bool can = cell_div == 1 && !d.stage_ok && d.box_max <= COARSE_MAX_BOX && d.rep_waves_max <= 65536 / WAVE;
    const int limit = d.nrep > 1 ? WIDE_BATCH_LIST : WIDE_WAVES;  // of a worklist
    const bool wide = can && d.nwaves <= (d.nrep > 1 ? WIDE_BATCH_WAVES : limit);
    const int rows = d.dim == 2 ? 3 : LIST_ROWS;
    if (wide)
        hipLaunchKernelGGL(k_rb_list_wide, dim3(std::min(d.nwaves, WIDE_BLOCKS * (LIST_ROWS / rows))), dim3(WAVE * rows),
                           0, s, d, limit);
    if (!wide || d.nwaves > limit) {
        if (cell_div == 1 && !d.stage_ok && d.box_max <= COARSE_MAX_BOX)
            hipLaunchKernelGGL(k_rb_list_masks, dim3(nblk_slots(d)), dim3(BLOCK), 0, s, d, wide ? limit + 1 : 1);
        else if (d.stage_ok)
            hipLaunchKernelGGL(k_rb_list<true>, dim3(nblk_slots(d)), dim3(BLOCK), 0, s, d, cell_div);
        else
            hipLaunchKernelGGL(k_rb_list<false>, dim3(nblk_slots(d)), dim3(BLOCK), 0, s, d, cell_div);
    }
    return hipGetLastError();
}

}  // namespace kamd
