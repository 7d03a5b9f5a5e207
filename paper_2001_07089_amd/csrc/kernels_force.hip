// kernels_force.hip -- Kob-Andersen pair forces over the neighbour lists.
//
// Force on particle i, Eq. (KAFix): F_i = 48 sum_j eps_ab (sig_ab^12/r^14 -
// 0.5 sig_ab^6/r^8)(r_i - r_j) over partners with r < 2.5 sig_ab (strict),
// computed as 48 eps * s6 (s6 - 1/2) / r^2 with s6 = (sig^2/r^2)^3 so that no
// square root is needed and the factor 48 eps is applied once per partner
// type (the paper's own two savings, Sec. III.D).  With the energy flag the
// shifted potential of Eq. (VshiftedKALJ), 4 eps s6 (s6 - 1) - V(r_c), and the
// virial r.F = 48 eps s6 (s6 - 1/2) are accumulated too (each pair appears in
// both partners' lists, so the per-particle sums are halved), together with
// the number of (ordered) pairs inside the cutoff.
//
// One thread per particle (or one of P threads that share its list, see
// force_split); a wavefront holds 64 particles of one replica and one type, so
// the parameters of each list part (A partners, then B partners, the paper's
// type-split loops) are wavefront-uniform and live in scalar
// registers.  Work is plain vector ALU arithmetic: a pair force is not a dense
// contraction, so there is nothing for the matrix cores here.
//
// Precision variants (template PREC):
//   0  FP64: binary64 separations with the minimum image taken as
//      d - L rint(d/L), binary64 LJ terms and sums.
//   1  MIXED: the separation is the exact integer difference of u32
//      fixed-point coordinates (minimum image for free), converted to FP32;
//      FP32 r^2, 1/r^2, LJ terms and per-part partial sums; the part sums are
//      scaled to force units and added in FP64.
//   2  MIXED_FIXED: as MIXED, but every pair force component is rounded to an
//      integer number of 2^-26 force units (one FP64 fma against 1.5*2^52)
//      and summed in 64-bit integers, so the sum is exact and independent of
//      the order of the list; F_ij = -F_ji holds bit for bit.  The rounding
//      is exact only while |F| < 2^25 per pair: each list part tracks its
//      largest in-cutoff 1/r^2 and the kernel sets KAMD_DEV_FORCE_RANGE when
//      a pair came closer than the separation where that bound is reached.
#include "common_dev.hpp"

namespace kamd {

// Close the rebuild check of the running step (every kernel of the rebuild
// chain has finished reading it) and optionally advance the device step
// counter.  Done by the first block of every force launch.
__device__ inline void close_step(const Dev &d, int flags)
{
    if (blockIdx.x != 0) return;
    for (int r = threadIdx.x; r < d.nrep; r += blockDim.x) {
        d.maxdisp[DISP_STRIDE * r] = 0u;
        d.rb_force[r] = 0;
    }
    if ((flags & FORCE_STEP) && threadIdx.x == 0) d.counters[1] += 1;
}

// The same without a force launch (after an explicit list build).
__global__ void k_close_check(Dev d) { close_step(d, 0); }

// Closing half kick of slot s: v = v_h + c a, with c = dt/2 or the replica's
// Nose-Hoover factor.  Returns v^2.
__device__ inline double close_kick(const Dev &d, int s, int rep, int flags, double dt, const double v[3], double ax,
                                    double ay, double az)
{
    const double c = flags & FORCE_KICK_NH ? d.dyn[rep].c_kick : 0.5 * dt;
    const double vx = fma(c, ax, v[0]), vy = fma(c, ay, v[1]), vz = fma(c, az, v[2]);
    d.vx[s] = vx;
    d.vy[s] = vy;
    d.vz[s] = vz;
    return vx * vx + vy * vy + vz * vz;
}

__device__ inline double rcp_f64(double a)
{
    double y = __builtin_amdgcn_rcp(a);
    double e = fma(-a, y, 1.0);
    y = fma(y, e, y);
    e = fma(-a, y, 1.0);
    return fma(y, e, y);
}

// Entries k .. k+3 of a list part (k a multiple of 4).  32-bit entries fill
// a 16-byte word.  16-bit entries (offsets from base) fill half of one, and
// the next four are the other half of the same word (a cache hit), so that
// both formats gather four neighbours per pass.
__device__ inline void list_quad32(const int4 *nb, int k, int jj[4])
{
    const int4 q = ld_stream(nb + (k >> 2) * WAVE);  // read once per step
    jj[0] = q.x;
    jj[1] = q.y;
    jj[2] = q.z;
    jj[3] = q.w;
}
__device__ inline void list_quad16(const int4 *nb, int k, int base, int jj[4])
{
    const int4 q = nb[(k >> 3) * WAVE];
    const bool hi = (k & 4) != 0;
    const uint32_t a = (uint32_t)(hi ? q.z : q.x), b = (uint32_t)(hi ? q.w : q.y);
    jj[0] = base + (int)(a & 0xffffu);
    jj[1] = base + (int)(a >> 16);
    jj[2] = base + (int)(b & 0xffffu);
    jj[3] = base + (int)(b >> 16);
}

// FP64 positions of every slot packed as (x, y, z, 0), so that the FP64 force
// kernel gathers a neighbour with two 16-byte loads instead of three 8-byte
// ones: the gathers bound that kernel, and their cost is per instruction.
// (Steps have them from the drift, or from the step before.)
__global__ __launch_bounds__(BLOCK) void k_pack_pos(Dev d)
{
    const int s = blockIdx.x * BLOCK + threadIdx.x;
    if (s < d.npad_total) d.pos4[s] = make_double4(d.x[s], d.y[s], d.z[s], 0.0);
}

// LDS visible to the whole wavefront (the lanes wrote it, others read it).
__device__ inline void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// KD (NVE steps only): after the force of slot s, close the step with the
// half kick v += a dt/2 and open the next one (v += a dt/2, r += v dt, wrap,
// new mirror into mirror_out, displacement into md_out) in the same pass.
// Neighbours read their positions from d.mirror while mirror_out receives the
// new ones, so the two must be different buffers; the forces are not stored.
//
// STAGE: a list part whose windows fit (lbase = -2, written by the list
// builder) is gathered from LDS.  Its stencil rows come in up to STAGE_GROUPS
// groups; for each group the wavefront copies the slot ranges of the group's
// row pieces (its lanes' union span of each stencil row, coalesced loads of
// d.mirror) one after the other into its window, and each lane its own
// position after them, then reads the group's entries, 16-bit offsets into
// that window.  A gather from global memory costs the kernel one cache-line
// access per lane and waits on the vector L1; a window read does neither.
// Parts whose windows do not fit keep the slot-index entries.
// Wavefronts per SIMD the register allocation of the staged step variant
// must allow: its LDS allows 5 (four wavefronts per block), and unbounded it
// takes a few registers too many for that (two 8-byte values then live in
// scratch, stored once per wavefront).
constexpr int WPE_STAGED = 5;

template <bool FIXED, bool ENERGY, bool KD, bool STAGE, int WPB>
__global__ __launch_bounds__(WAVE * WPB) __attribute__((amdgpu_waves_per_eu(STAGE && !ENERGY ? WPE_STAGED : 1))) void k_force_mixed(Dev d, Model m, int flags, double dt,
                                                             uint4 *mirror_out, uint32_t *md_out)
{
    __shared__ uint32_t swin[STAGE ? WPB : 1][STAGE ? 3 * STAGE_SLOTS : 1];
    close_step(d, flags);
    const int w = wave_id_remapped<WPB>();
    const bool valid = w < d.nwaves;
    float d2 = 0.0f;
    int rep = -1;
    if (valid) {
    const SegInfo &S = d.seg[d.wave_seg[w]];
    rep = S.rep;
    const RepInfo &R = d.rep[S.rep];
    const int s = w * WAVE + lane_id();
    const uint4 mi = d.mirror[s];
    const int2 km = d.kmax[w];
    const int2 lb = d.lbase[w];
    const int2 pc = STAGE ? d.pcount[w] : make_int2(0, 0);
    uint32_t *win = swin[STAGE ? threadIdx.x >> 6 : 0];
    double fx = 0.0, fy = 0.0, fz = 0.0, pe = 0.0, vir = 0.0, npair = 0.0, ke2 = 0.0;
    uint64_t qx = 0, qy = 0, qz = 0;
    bool range_bad = false;
    int row = 0;  // 32-bit words of the list
#pragma unroll 1
    for (int tj = 0; tj < 2; ++tj) {
        const int p = S.type + tj;
        const float rc2 = R.rc2_fx[p], sig2 = R.sig2_fx[p];
        const double fk = R.fix_k[p];
        const int nrows = tj ? km.y : km.x;
        const int base = tj ? lb.y : lb.x;
        float sx = 0.0f, sy = 0.0f, sz = 0.0f, se = 0.0f, sv = 0.0f;
        float irmax = 0.0f;  // largest 1/r^2 of an in-cutoff pair (fixed-point range check)
        int cnt = 0;
        const int4 *nb = reinterpret_cast<const int4 *>(d.nbr + list_index(w, d.rows, row, lane_id()));
        auto pair = [&](const uint4 mj) {
                const int ix = (int)(mi.x - mj.x);
                const int iy = (int)(mi.y - mj.y);
                const int iz = (int)(mi.z - mj.z);
                const float dx = (float)ix, dy = (float)iy, dz = (float)iz;
                const float r2 = dx * dx + dy * dy + dz * dz;
                const bool in = (r2 < rc2) && (r2 > 0.0f);
                const float ir2 = in ? __builtin_amdgcn_rcpf(r2) : 0.0f;
                const float s2 = sig2 * ir2;
                const float s6 = s2 * s2 * s2;
                const float t = s6 * (s6 - 0.5f);
                const float f = t * ir2;
                if (FIXED) {
                    irmax = fmaxf(irmax, ir2);
                    const double wd = (double)f * fk;
                    qx += (uint64_t)__double_as_longlong(fma(wd, (double)ix, FIX_MAGIC));
                    qy += (uint64_t)__double_as_longlong(fma(wd, (double)iy, FIX_MAGIC));
                    qz += (uint64_t)__double_as_longlong(fma(wd, (double)iz, FIX_MAGIC));
                } else {
                    sx = fmaf(f, dx, sx);
                    sy = fmaf(f, dy, sy);
                    sz = fmaf(f, dz, sz);
                }
                if (ENERGY) {
                    se += fmaf(-0.5f, s6, t);
                    sv += t;
                    cnt += in ? 1 : 0;
                }
        };
        auto quad = [&](const int jj[4]) {
            uint4 mj[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) mj[u] = d.mirror[jj[u]];
#pragma unroll
            for (int u = 0; u < 4; ++u) pair(mj[u]);
        };
        if (!STAGE && base <= -2) {  // a window list for the direct variant: never read it as slots
            if (lane_id() == 0) set_err(d.err, KAMD_DEV_LIST_FORMAT);
        } else if (STAGE && base <= -2) {
            const int ng = tj ? pc.y : pc.x;
            const int2 *pt = d.pieces + ((size_t)w * 2 + tj) * STAGE_PIECES;
            const int4 *gt = d.sgroups + ((size_t)w * 2 + tj) * STAGE_GROUPS;
            int q = 0, k = 0;
            for (int g = 0; g < ng; ++g) {
                const int4 gi = gt[g];  // (end of its pieces, window slots, end of its entries, -)
                const int kend = min(g + 1 < ng ? gi.z : nrows, nrows);
                int off = 0;
                for (; q < gi.x; ++q) {
                    const int2 pq = pt[q];
                    // two loads in flight per lane before the first store
                    for (int e = lane_id(); e < pq.y; e += 2 * WAVE) {
                        const bool two = e + WAVE < pq.y;
                        const uint4 ma = d.mirror[pq.x + e];
                        const uint4 mb = d.mirror[pq.x + (two ? e + WAVE : e)];
                        uint32_t *o = win + 3 * (off + e);
                        o[0] = ma.x;
                        o[1] = ma.y;
                        o[2] = ma.z;
                        if (two) {
                            o[3 * WAVE + 0] = mb.x;
                            o[3 * WAVE + 1] = mb.y;
                            o[3 * WAVE + 2] = mb.z;
                        }
                    }
                    off += pq.y;
                }
                uint32_t *o = win + 3 * (gi.y + lane_id());
                o[0] = mi.x;
                o[1] = mi.y;
                o[2] = mi.z;
                wave_lds_sync();
                for (; k < kend; k += 4) {
                    int jj[4];
                    list_quad16(nb, k, 0, jj);
                    uint4 mj[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const uint32_t *src = win + 3 * jj[u];
                        mj[u] = make_uint4(src[0], src[1], src[2], 0u);
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) pair(mj[u]);
                }
                wave_lds_sync();  // the next group (or part) stages over this window
            }
        } else if (base >= 0) {
            for (int k = 0; k < nrows; k += 4) {
                int jj[4];
                list_quad16(nb, k, base, jj);
                quad(jj);
            }
        } else {
            for (int k = 0; k < nrows; k += 4) {
                int jj[4];
                list_quad32(nb, k, jj);
                quad(jj);
            }
        }
        if (FIXED) {
            range_bad = range_bad || irmax > R.ir2_lim_fx[p];
            const uint64_t mb = (uint64_t)__double_as_longlong(FIX_MAGIC) * (uint64_t)nrows;
            qx -= mb;
            qy -= mb;
            qz -= mb;
        } else {
            const double c = R.c48_h[p];
            fx = fma(c, (double)sx, fx);
            fy = fma(c, (double)sy, fy);
            fz = fma(c, (double)sz, fz);
        }
        if (ENERGY) {
            pe += 0.5 * (4.0 * m.eps[p] * (double)se - (double)cnt * m.vshift[p]);
            vir += 0.5 * 48.0 * m.eps[p] * (double)sv;
            npair += (double)cnt;
        }
        row += base != -1 ? nrows / 2 : nrows;  // 16-bit entries: base >= 0, or a staged window
    }
    if (FIXED) {
        const double inv = 1.0 / FIX_SCALE;
        fx = (double)(int64_t)qx * inv;
        fy = (double)(int64_t)qy * inv;
        fz = (double)(int64_t)qz * inv;
        // the per-pair bound, and a net force beyond which the int64 -> FP64
        // conversion of the sum is no longer exact (2^53 units)
        const double lim = 1.0e8;
        if (range_bad || fabs(fx) > lim || fabs(fy) > lim || fabs(fz) > lim) set_err(d.err, KAMD_DEV_FORCE_RANGE);
    }
    if (!(isfinite(fx) && isfinite(fy) && isfinite(fz))) set_err(d.err, KAMD_DEV_NONFINITE);
    if (!KD) {
        d.ax[s] = fx;
        d.ay[s] = fy;
        d.az[s] = fz;
        if ((flags & FORCE_KICK) && (s - S.slot0) < S.n) {
            const double v[3] = {ld_stream(&d.vx[s]), ld_stream(&d.vy[s]), ld_stream(&d.vz[s])};
            ke2 = close_kick(d, s, S.rep, flags, dt, v, fx, fy, fz);
        }
    } else if ((s - S.slot0) < S.n) {
        const double h = 0.5 * dt;
        const double a[3] = {fx, fy, fz};
        const double v[3] = {fma(h, fx, ld_stream(&d.vx[s])), fma(h, fy, ld_stream(&d.vy[s])), fma(h, fz, ld_stream(&d.vz[s]))};
        if (ENERGY) ke2 = v[0] * v[0] + v[1] * v[1] + v[2] * v[2];
        DriftIn in = drift_load(d, s);
        drift_core(d, s, R, dt, 0.0, 0.0, h, v, a, in, mirror_out, d2);
    }
    if (KD ? ENERGY : (flags & FORCE_KE) != 0) {
        ke2 = wave_sum(ke2);
        if (lane_id() == 0) d.wred[4 * w + 0] = ke2;
    }
    if (ENERGY) {
        pe = wave_sum(pe);
        vir = wave_sum(vir);
        npair = wave_sum(npair);
        if (lane_id() == 0) {
            d.wred[4 * w + 1] = pe;
            d.wred[4 * w + 2] = vir;
            d.wred[4 * w + 3] = npair;
        }
    }
    }
    if (KD) block_disp_max<WPB>(md_out, valid, rep, d2);
}

// Shared lists: the P wavefronts of a block walk the list of one particle
// wavefront together; unit u of the list (SPLIT_UNIT entries) goes to
// wavefront u % P, and the sums are combined in LDS.
//
// What it is for: with fewer wavefronts than the device has SIMDs nothing
// hides the round trips list word -> neighbour positions -> sums, which a lone
// wavefront takes one after the other (28 us in FP64 for 1000 particles, 22 us
// in MIXED for 32,000).  Large systems gain too: eight gathers are in flight
// per pass instead of four, the particles' state, which the closing
// integration needs, is requested before the walk, and the wavefronts of a
// block gather from the same rows at the same time.
//
// The sums:
//   FP64 and MIXED_FIXED: each wavefront sums what it takes, and wavefront 0
//   adds the P sums up (FP64 in a fixed order, the fixed-point sums exactly).
//   MIXED's FP32 force sums, and the FP32 energy and virial sums of both mixed
//   modes, keep the order of the list (ORD): the wavefronts put their pair
//   terms in LDS, P units at a time, and every sum is run over them in list
//   order by one wavefront with the operations of the unsplit kernel, so that
//   it has the unsplit kernel's bits.  (P = 1, MIXED forces: one wavefront
//   keeps the order by itself.)
// Wavefront 0 closes the step.  KD (NVE steps): as in the mixed kernel above;
// in FP64 neighbours gather from d.pos4, so the new positions go to d.x, d.y,
// d.z in place and, packed, to pos4_out (a different buffer), where the next
// step's neighbours find them; padding slots copy their unchanged position,
// which keeps their own list entry at zero separation.
constexpr int SPLIT_UNIT = 8;

template <int PREC, bool ENERGY, bool KD, int P>
__device__ __forceinline__ void force_split(const Dev &d, const Model &m, int flags, double dt, uint4 *mirror_out,
                                            uint32_t *md_out, double4 *pos4_out)
{
    constexpr bool FP64 = PREC == 0, FIXED = PREC == 2;
    constexpr bool SEQ = PREC == 1 && P == 1;  // one wavefront: the list order by itself
    constexpr bool ORD_F = PREC == 1 && !SEQ, ORD_E = !FP64 && ENERGY && !SEQ, ORD = ORD_F || ORD_E;
    static_assert(!ORD || P == 4, "the ordered sums are spread over four wavefronts");
    static_assert(!(SEQ && ENERGY), "energies take the ordered sums");
    constexpr int NF = ORD_F ? 4 : 0, NT = NF + (ORD_E ? 2 : 0);  // terms per pair: f, dx, dy, dz; energy term, s2
    constexpr int ND = ORD_F ? 1 : FP64 && ENERGY ? 5 : 3;        // sums per wavefront: force, or its fixed-point bits; FP64 PE, W
    __shared__ float term[ORD ? P * SPLIT_UNIT : 1][ORD ? NT : 1][ORD ? WAVE : 1];
    __shared__ float osum[ORD ? 2 : 1][ORD ? 5 : 1][ORD ? WAVE : 1];  // ordered sums per part: x, y, z, e, v
    __shared__ double psum[ORD_F ? 1 : P][ND][ORD_F ? 1 : WAVE];
    __shared__ int ncut[ENERGY ? P : 1][ENERGY ? 2 : 1][ENERGY ? WAVE : 1];
    close_step(d, flags);
    const int w = xcd_block(blockIdx.x, gridDim.x);
    const int q = threadIdx.x >> 6, lane = lane_id();
    const SegInfo &S = d.seg[d.wave_seg[w]];
    const RepInfo &R = d.rep[S.rep];
    const int s = w * WAVE + lane;
    const double L = R.L, invL = R.invL;
    double v0[3] = {0.0, 0.0, 0.0};
    DriftIn in;
    if (q == 0 && (KD || (flags & FORCE_KICK))) {  // in flight during the walk
        if (KD) in = drift_load(d, s);
        v0[0] = ld_stream(&d.vx[s]);
        v0[1] = ld_stream(&d.vy[s]);
        v0[2] = ld_stream(&d.vz[s]);
    }
    double xi = 0.0, yi = 0.0, zi = 0.0;
    uint4 mi = make_uint4(0, 0, 0, 0);
    if (FP64) {
        xi = d.x[s];
        yi = d.y[s];
        zi = d.z[s];
    } else {
        mi = d.mirror[s];
    }
    const int2 km = d.kmax[w];
    const int2 lb = d.lbase[w];
    double fx = 0.0, fy = 0.0, fz = 0.0, pe = 0.0, vir = 0.0;
    uint64_t qx = 0, qy = 0, qz = 0;
    bool range_bad = false;
    int row = 0;    // 32-bit words of the list
    int first = q;  // this wavefront's first unit of the next part
#pragma unroll 1
    for (int tj = 0; tj < 2; ++tj) {
        const int p = S.type + tj;
        const int base = tj ? lb.y : lb.x;
        const int nrows = base <= -2 ? 0 : tj ? km.y : km.x;  // a window list: the unsplit kernel's only
        if (base <= -2 && threadIdx.x == 0) set_err(d.err, KAMD_DEV_LIST_FORMAT);
        const int nunit = (nrows + SPLIT_UNIT - 1) / SPLIT_UNIT;
        const int4 *nb = reinterpret_cast<const int4 *>(d.nbr + list_index(w, d.rows, row, lane));
        const double rc2d = m.rc2[p], sig2d = m.sig2[p];
        const float rc2 = R.rc2_fx[p], sig2 = R.sig2_fx[p];
        const double fk = R.fix_k[p];
        double sx = 0.0, sy = 0.0, sz = 0.0, se = 0.0, sv = 0.0;
        float tx = 0.0f, ty = 0.0f, tz = 0.0f;
        float irmax = 0.0f;
        int cnt = 0, taken = 0;
        auto pair64 = [&](double xj, double yj, double zj) {
            double dx = xi - xj;
            double dy = yi - yj;
            double dz = zi - zj;
            dx = fma(-L, rint(dx * invL), dx);
            dy = fma(-L, rint(dy * invL), dy);
            dz = fma(-L, rint(dz * invL), dz);
            const double r2 = dx * dx + dy * dy + dz * dz;
            const bool on = (r2 < rc2d) && (r2 > 0.0);
            const double ir2 = on ? rcp_f64(r2) : 0.0;
            const double s2 = sig2d * ir2;
            const double s6 = s2 * s2 * s2;
            const double t = s6 * (s6 - 0.5);
            const double f = t * ir2;
            sx = fma(f, dx, sx);
            sy = fma(f, dy, sy);
            sz = fma(f, dz, sz);
            if (ENERGY) {
                se += fma(-0.5, s6, t);
                sv += t;
                cnt += on ? 1 : 0;
            }
        };
        auto pair32 = [&](const uint4 mj, int e) {
            const int ix = (int)(mi.x - mj.x);
            const int iy = (int)(mi.y - mj.y);
            const int iz = (int)(mi.z - mj.z);
            const float dx = (float)ix, dy = (float)iy, dz = (float)iz;
            const float r2 = dx * dx + dy * dy + dz * dz;
            const bool on = (r2 < rc2) && (r2 > 0.0f);
            const float ir2 = on ? __builtin_amdgcn_rcpf(r2) : 0.0f;
            const float s2 = sig2 * ir2;
            const float s6 = s2 * s2 * s2;
            const float t = s6 * (s6 - 0.5f);
            const float f = t * ir2;
            if (FIXED) {
                irmax = fmaxf(irmax, ir2);
                const double wd = (double)f * fk;
                qx += (uint64_t)__double_as_longlong(fma(wd, (double)ix, FIX_MAGIC));
                qy += (uint64_t)__double_as_longlong(fma(wd, (double)iy, FIX_MAGIC));
                qz += (uint64_t)__double_as_longlong(fma(wd, (double)iz, FIX_MAGIC));
            }
            if (SEQ) {
                tx = fmaf(f, dx, tx);
                ty = fmaf(f, dy, ty);
                tz = fmaf(f, dz, tz);
            }
            if constexpr (ORD_F) {
                term[e][0][lane] = f;
                term[e][1][lane] = dx;
                term[e][2][lane] = dy;
                term[e][3][lane] = dz;
            }
            if constexpr (ORD_E) {
                term[e][NF][lane] = fmaf(-0.5f, s6, t);
                term[e][NF + 1][lane] = s2;
            }
            if (ENERGY) cnt += on ? 1 : 0;
        };
        // Unit u: entries 8 u .. 8 u + 7.  A 32-bit part may end in half
        // a unit; the own slot stands in for the rest (zero separation:
        // adds nothing, like the padding).
        auto unit = [&](int u) {
            int jj[SPLIT_UNIT];
            const int k = u * SPLIT_UNIT;
            if (base >= 0) {
                list_quad16(nb, k, base, jj);
                if constexpr (SPLIT_UNIT == 8) list_quad16(nb, k + 4, base, jj + 4);
            } else {
                list_quad32(nb, k, jj);
                if constexpr (SPLIT_UNIT == 8) {
                    jj[4] = jj[5] = jj[6] = jj[7] = s;
                    if (k + 4 < nrows) list_quad32(nb, k + 4, jj + 4);
                }
            }
            if (FP64) {
                double4 pj[SPLIT_UNIT];
#pragma unroll
                for (int e = 0; e < SPLIT_UNIT; ++e) pj[e] = d.pos4[jj[e]];
#pragma unroll
                for (int e = 0; e < SPLIT_UNIT; ++e) pair64(pj[e].x, pj[e].y, pj[e].z);
            } else {
                uint4 mj[SPLIT_UNIT];
#pragma unroll
                for (int e = 0; e < SPLIT_UNIT; ++e) mj[e] = d.mirror[jj[e]];
#pragma unroll
                for (int e = 0; e < SPLIT_UNIT; ++e) pair32(mj[e], q * SPLIT_UNIT + e);
            }
            ++taken;
        };
        if constexpr (ORD) {
            float sum = 0.0f, sum2 = 0.0f;  // wavefronts 0..2: x, y, z (MIXED); 3: energy and virial
            for (int u0 = 0; u0 < nunit; u0 += P) {
                if (u0 + q < nunit) unit(u0 + q);
                __syncthreads();
                const int ne = min(P, nunit - u0) * SPLIT_UNIT;
                if (ORD_F && q < 3) {
#pragma unroll 8
                    for (int e = 0; e < ne; ++e) sum = fmaf(term[e][0][lane], term[e][ORD_F ? 1 + q : 0][lane], sum);
                }
                if (ORD_E && q == 3) {
#pragma unroll 8
                    for (int e = 0; e < ne; ++e) {
                        sum += term[e][NF][lane];
                        // the virial term s6 (s6 - 1/2), fused as the compiler fuses it in the unsplit kernel
                        const float s2 = term[e][ORD_E ? NF + 1 : 0][lane], s4 = s2 * s2;
                        sum2 = fmaf(s2 * s4, fmaf(s2, s4, -0.5f), sum2);
                    }
                }
                __syncthreads();
            }
            osum[tj][q][lane] = sum;
            if (q == 3) osum[tj][4][lane] = sum2;
        } else {
            for (int u = first; u < nunit; u += P) unit(u);
            first = (first + P - nunit % P) % P;  // the units of all parts go round together
        }
        if (FP64) {
            const double e48 = 48.0 * m.eps[p];
            fx = fma(e48, sx, fx);
            fy = fma(e48, sy, fy);
            fz = fma(e48, sz, fz);
            if (ENERGY) {
                pe += 0.5 * (4.0 * m.eps[p] * se - (double)cnt * m.vshift[p]);
                vir += 0.5 * e48 * sv;
            }
        }
        if (SEQ) {
            const double c = R.c48_h[p];
            fx = fma(c, (double)tx, fx);
            fy = fma(c, (double)ty, fy);
            fz = fma(c, (double)tz, fz);
        }
        if (FIXED) {
            range_bad = range_bad || irmax > R.ir2_lim_fx[p];
            const uint64_t mb = (uint64_t)__double_as_longlong(FIX_MAGIC) * (uint64_t)(taken * SPLIT_UNIT);
            qx -= mb;
            qy -= mb;
            qz -= mb;
        }
        if constexpr (ENERGY) ncut[q][tj][lane] = cnt;
        row += base != -1 ? nrows / 2 : nrows;
    }
    if constexpr (FP64 || SEQ) {
        psum[q][0][lane] = fx;
        psum[q][1][lane] = fy;
        psum[q][2][lane] = fz;
        if constexpr (FP64 && ENERGY) {
            psum[q][3][lane] = pe;
            psum[q][4][lane] = vir;
        }
    }
    if constexpr (FIXED) {
        psum[q][0][lane] = __longlong_as_double((long long)qx);
        psum[q][1][lane] = __longlong_as_double((long long)qy);
        psum[q][2][lane] = __longlong_as_double((long long)qz);
        if (range_bad) set_err(d.err, KAMD_DEV_FORCE_RANGE);
    }
    __syncthreads();
    if (q != 0) return;
    double npair = 0.0, ke2 = 0.0;
    if constexpr (FP64 || SEQ) {
        double t[ND];
#pragma unroll
        for (int c = 0; c < ND; ++c) {
            t[c] = psum[0][c][lane];
#pragma unroll
            for (int k = 1; k < P; ++k) t[c] += psum[k][c][lane];
        }
        fx = t[0];
        fy = t[1];
        fz = t[2];
        if constexpr (FP64 && ENERGY) {
            pe = t[3];
            vir = t[4];
        }
    }
    if constexpr (ENERGY || ORD_F) {
        for (int tj = 0; tj < 2; ++tj) {
            const int p = S.type + tj;
            int cnt = 0;
            if constexpr (ENERGY)
                for (int k = 0; k < P; ++k) cnt += ncut[k][tj][lane];
            if constexpr (ORD_F) {
                const double c = R.c48_h[p];
                fx = fma(c, (double)osum[tj][0][lane], fx);
                fy = fma(c, (double)osum[tj][1][lane], fy);
                fz = fma(c, (double)osum[tj][2][lane], fz);
            }
            if constexpr (ORD_E) {
                pe += 0.5 * (4.0 * m.eps[p] * (double)osum[tj][3][lane] - (double)cnt * m.vshift[p]);
                vir += 0.5 * 48.0 * m.eps[p] * (double)osum[tj][4][lane];
            }
            npair += (double)cnt;
        }
    }
    if constexpr (FIXED) {
        uint64_t t[3] = {0, 0, 0};
#pragma unroll
        for (int k = 0; k < P; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c) t[c] += (uint64_t)__double_as_longlong(psum[k][c][lane]);
        const double inv = 1.0 / FIX_SCALE;
        fx = (double)(int64_t)t[0] * inv;
        fy = (double)(int64_t)t[1] * inv;
        fz = (double)(int64_t)t[2] * inv;
        // a net force beyond which the int64 -> FP64 conversion is not exact
        const double lim = 1.0e8;
        if (fabs(fx) > lim || fabs(fy) > lim || fabs(fz) > lim) set_err(d.err, KAMD_DEV_FORCE_RANGE);
    }
    if (!(isfinite(fx) && isfinite(fy) && isfinite(fz))) set_err(d.err, KAMD_DEV_NONFINITE);
    float d2 = 0.0f;
    if (!KD) {
        d.ax[s] = fx;
        d.ay[s] = fy;
        d.az[s] = fz;
        if ((flags & FORCE_KICK) && (s - S.slot0) < S.n) ke2 = close_kick(d, s, S.rep, flags, dt, v0, fx, fy, fz);
    } else if ((s - S.slot0) < S.n) {
        const double h = 0.5 * dt;
        const double a[3] = {fx, fy, fz};
        const double v[3] = {fma(h, fx, v0[0]), fma(h, fy, v0[1]), fma(h, fz, v0[2])};
        if (ENERGY) ke2 = v[0] * v[0] + v[1] * v[1] + v[2] * v[2];
        drift_core(d, s, R, dt, 0.0, 0.0, h, v, a, in, mirror_out, d2);
        if (FP64) pos4_out[s] = make_double4(in.r[0], in.r[1], in.r[2], 0.0);
    } else if (FP64) {
        pos4_out[s] = make_double4(xi, yi, zi, 0.0);
    }
    if (KD ? ENERGY : (flags & FORCE_KE) != 0) {
        ke2 = wave_sum(ke2);
        if (lane == 0) d.wred[4 * w + 0] = ke2;
    }
    if (ENERGY) {
        pe = wave_sum(pe);
        vir = wave_sum(vir);
        npair = wave_sum(npair);
        if (lane == 0) {
            d.wred[4 * w + 1] = pe;
            d.wred[4 * w + 2] = vir;
            d.wred[4 * w + 3] = npair;
        }
    }
    if (KD) {
        d2 = wave_max(d2);
        if (lane == 0) disp_push(md_out, S.rep, d2);
    }
}

template <bool ENERGY, bool KD, int P>
__global__ __launch_bounds__(WAVE * P) void k_force_fp64(Dev d, Model m, int flags, double dt, uint4 *mirror_out,
                                                         uint32_t *md_out, double4 *pos4_out)
{
    force_split<0, ENERGY, KD, P>(d, m, flags, dt, mirror_out, md_out, pos4_out);
}

template <bool FIXED, bool ENERGY, bool KD, int P>
__global__ __launch_bounds__(WAVE * P) void k_force_split(Dev d, Model m, int flags, double dt, uint4 *mirror_out,
                                                          uint32_t *md_out)
{
    force_split<FIXED ? 2 : 1, ENERGY, KD, P>(d, m, flags, dt, mirror_out, md_out, nullptr);
}

// Wavefronts that share a list, by the number of particle wavefronts.
// Measured (MI355X, us per NVE step, all kernels; unsplit, then P = 1, 2, 4, 8):
//   FP64         N = 1000     54.1,    -, 37.8, 34.8, 34.0
//                32,000       60.7,    -, 44.4, 41.1, 41.1
//                100,000      81.5,    -, 75.3, 70.6, 72.4
//                2^20          450,  490,  472,  420,  493
//   MIXED_FIXED  1000         44.2,    -, 34.9, 32.0, 30.8
//                32,000       51.9,    -, 41.5, 38.1, 38.3
//                100,000      70.7,    -, 58.0, 59.2, 63.9
//                2^20          331,  328,  304,  329,  389
//                80,000          -,    -, 42.1, 40.5     (these three with the later list
//                120,000         -,    -, 50.1, 51.9     builders, chain and maxima apart)
//                64 x 1000, bath -,    -, 51.6, 49.2
//   MIXED        1000         43.3, 40.0,    -, 35.1
//                64,000       54.9, 49.3,    -, 45.7
//                100,000      67.6, 58.9,    -, 61.0
//                400,000       152,  145,    -,  148
//                2^20          314,  319,    -,  357
// Either side of 512 wavefronts, with the other kernels as they are now (P = 4,
// 8): FP64 32,000 particles (501) 26.8, 26.6, 36,000 (563) 32.6, 34.2;
// MIXED_FIXED 28,000 22.7, 22.3, 32,000 24.2, 23.6, 36,000 27.5, 31.8.
// FP64 with short lists: four wavefronts find too few units.  300,000 particles
// at densities 0.02, 0.1, 0.2, 0.4, 0.6, 0.7 (2, 9, 17, 34, 50, 59 entries expected),
// unsplit, then P = 1, 2, 4: 53.4, 45.9, 50.5, 57.6; 57.4, 46.5, 48.6, 56.7; 65.6, 56.5,
// 53.5, 58.8; 82.0, 67.9, 64.0, 69.6; 95.9, -, 77.2, 79.1; 104, -, 84.7, 83.6; 4096 x 70 (42
// entries) 108.9, 90.7, 94.6, 106.8; 60,000 at 0.02, 0.1, 0.6 25.3, 25.6, 27.1, 25.9;
// 27.9, 24.6, 23.5, 24.2; 39.9, -, 27.2, 26.7.
// A whole md_forces call with energies, 100,000 / 200,000 particles: MIXED 115
// -> 104 / 155 -> 154 us, MIXED_FIXED 114 -> 108 / 144 -> 139 us (2^20: slower).
// Two wavefronts that share the lists of two (each closing one) measured 306
// (MIXED_FIXED) and 460 us (FP64) at 2^20; units of 4 entries 326 and 434.
constexpr int SPLIT8_WAVES = 512, SPLIT4_WAVES = 1280, SPLIT_ORD_WAVES = 1024, SPLIT1_WAVES = 8192;
constexpr int SPLIT_ORD_ENERGY_WAVES = 2048, SHORT_LIST = 54, TINY_LIST = 12;

template <bool ENERGY, bool KD, int P>
static void launch_fp64(const Dev &d, const Model &m, int flags, double dt, uint4 *mirror_out, uint32_t *md_out,
                        double4 *pos4_out, hipStream_t s)
{
    hipLaunchKernelGGL((k_force_fp64<ENERGY, KD, P>), dim3(d.nwaves), dim3(WAVE * P), 0, s, d, m, flags, dt, mirror_out,
                       md_out, pos4_out);
}

template <bool ENERGY, bool KD>
static void launch_fp64(const Dev &d, const Model &m, int flags, double dt, uint4 *mirror_out, uint32_t *md_out,
                        double4 *pos4_out, hipStream_t s)
{
    if (d.nwaves <= SPLIT8_WAVES) launch_fp64<ENERGY, KD, 8>(d, m, flags, dt, mirror_out, md_out, pos4_out, s);
    else if (d.nwaves > SPLIT4_WAVES && d.list_len <= TINY_LIST)
        launch_fp64<ENERGY, KD, 1>(d, m, flags, dt, mirror_out, md_out, pos4_out, s);
    else if (d.nwaves > SPLIT4_WAVES && d.list_len <= SHORT_LIST)
        launch_fp64<ENERGY, KD, 2>(d, m, flags, dt, mirror_out, md_out, pos4_out, s);
    else launch_fp64<ENERGY, KD, 4>(d, m, flags, dt, mirror_out, md_out, pos4_out, s);
}

template <bool FIXED, bool ENERGY, bool KD, int P>
static bool launch_split(const Dev &d, const Model &m, int flags, double dt, uint4 *mirror_out, uint32_t *md_out,
                         hipStream_t s)
{
    hipLaunchKernelGGL((k_force_split<FIXED, ENERGY, KD, P>), dim3(d.nwaves), dim3(WAVE * P), 0, s, d, m, flags, dt,
                       mirror_out, md_out);
    return true;
}

// False: the rule leaves this launch to k_force_mixed.
template <bool FIXED, bool ENERGY, bool KD>
static bool launch_split(const Dev &d, const Model &m, int flags, double dt, uint4 *mirror_out, uint32_t *md_out,
                         hipStream_t s)
{
    const int nw = d.nwaves;
    if (d.stage_ok) return false;  // window lists
    if constexpr (ENERGY) {
        return nw <= SPLIT_ORD_ENERGY_WAVES && launch_split<FIXED, ENERGY, KD, 4>(d, m, flags, dt, mirror_out, md_out, s);
    } else if constexpr (FIXED) {
        if (nw <= SPLIT8_WAVES) return launch_split<FIXED, ENERGY, KD, 8>(d, m, flags, dt, mirror_out, md_out, s);
        if (nw <= SPLIT4_WAVES) return launch_split<FIXED, ENERGY, KD, 4>(d, m, flags, dt, mirror_out, md_out, s);
        return launch_split<FIXED, ENERGY, KD, 2>(d, m, flags, dt, mirror_out, md_out, s);
    } else {
        if (nw <= SPLIT_ORD_WAVES) return launch_split<FIXED, ENERGY, KD, 4>(d, m, flags, dt, mirror_out, md_out, s);
        return nw <= SPLIT1_WAVES && launch_split<FIXED, ENERGY, KD, 1>(d, m, flags, dt, mirror_out, md_out, s);
    }
}

// The unsplit mixed kernel, with windows (as the lists were built) or where
// launch_split leaves it the launch, in blocks of WPB wavefronts.
template <bool FIXED, bool ENERGY, bool KD, int WPB>
static void launch_mixed_wpb(const Dev &d, const Model &m, int flags, double dt, uint4 *mirror_out, uint32_t *md_out,
                             hipStream_t s)
{
    const int nb = (d.nwaves + WPB - 1) / WPB;
    if (d.stage_ok) {
        hipLaunchKernelGGL((k_force_mixed<FIXED, ENERGY, KD, true, WPB>), dim3(nb), dim3(WAVE * WPB), 0, s, d, m, flags,
                           dt, mirror_out, md_out);
    } else if (!launch_split<FIXED, ENERGY, KD>(d, m, flags, dt, mirror_out, md_out, s)) {
        if constexpr (!FIXED || ENERGY)
            hipLaunchKernelGGL((k_force_mixed<FIXED, ENERGY, KD, false, WPB>), dim3(nb), dim3(WAVE * WPB), 0, s, d, m,
                               flags, dt, mirror_out, md_out);
    }
}

template <bool FIXED, bool ENERGY, bool KD>
static void launch_mixed(const Dev &d, const Model &m, int flags, double dt, uint4 *mirror_out, uint32_t *md_out,
                         int wpb, hipStream_t s)
{
    if (wpb == 1) launch_mixed_wpb<FIXED, ENERGY, KD, 1>(d, m, flags, dt, mirror_out, md_out, s);
    else if (wpb == 2) launch_mixed_wpb<FIXED, ENERGY, KD, 2>(d, m, flags, dt, mirror_out, md_out, s);
    else launch_mixed_wpb<FIXED, ENERGY, KD, 4>(d, m, flags, dt, mirror_out, md_out, s);
}

// Launches that store the forces (md_forces; the last step of a call and the
// steps under a thermostat, which kick): unsplit ones in blocks of
// WAVES_PER_BLOCK wavefronts.
hipError_t launch_force(const Dev &d, const Model &m, int prec, bool energy, int flags, double dt, hipStream_t s)
{
    constexpr int W4 = WAVES_PER_BLOCK;
    if (prec == 0) {
        if (!(flags & FORCE_STEP))
            hipLaunchKernelGGL(k_pack_pos, dim3((d.npad_total + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, s, d);
        if (energy)
            launch_fp64<true, false>(d, m, flags, dt, nullptr, nullptr, nullptr, s);
        else
            launch_fp64<false, false>(d, m, flags, dt, nullptr, nullptr, nullptr, s);
    } else if (prec == 1) {
        if (energy)
            launch_mixed_wpb<false, true, false, W4>(d, m, flags, dt, nullptr, nullptr, s);
        else
            launch_mixed_wpb<false, false, false, W4>(d, m, flags, dt, nullptr, nullptr, s);
    } else {
        if (energy)
            launch_mixed_wpb<true, true, false, W4>(d, m, flags, dt, nullptr, nullptr, s);
        else
            launch_mixed_wpb<true, false, false, W4>(d, m, flags, dt, nullptr, nullptr, s);
    }
    return hipGetLastError();
}

bool step_blocks_matter(const Dev &d, int prec)
{
    return prec != 0 && (d.stage_ok || (prec == 1 && d.nwaves > SPLIT1_WAVES));
}

hipError_t launch_close_check(const Dev &d, hipStream_t s)
{
    hipLaunchKernelGGL(k_close_check, dim3(1), dim3(BLOCK), 0, s, d);
    return hipGetLastError();
}

hipError_t launch_force_kd(const Dev &d, const Model &m, int prec, double dt, uint4 *mirror_out, uint32_t *md_out,
                           double4 *pos4_out, bool energy, int wpb, hipStream_t s)
{
    if (wpb != 1 && wpb != 2 && wpb != 4) return hipErrorInvalidValue;
    if (prec == 0) {
        if (!d.pos4 || !pos4_out || pos4_out == d.pos4) return hipErrorInvalidValue;
        if (energy)
            launch_fp64<true, true>(d, m, FORCE_STEP, dt, mirror_out, md_out, pos4_out, s);
        else
            launch_fp64<false, true>(d, m, FORCE_STEP, dt, mirror_out, md_out, pos4_out, s);
    } else if (prec == 1) {
        if (energy)
            launch_mixed<false, true, true>(d, m, FORCE_STEP, dt, mirror_out, md_out, wpb, s);
        else
            launch_mixed<false, false, true>(d, m, FORCE_STEP, dt, mirror_out, md_out, wpb, s);
    } else if (prec == 2) {
        if (energy)
            launch_mixed<true, true, true>(d, m, FORCE_STEP, dt, mirror_out, md_out, wpb, s);
        else
            launch_mixed<true, false, true>(d, m, FORCE_STEP, dt, mirror_out, md_out, wpb, s);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace kamd
